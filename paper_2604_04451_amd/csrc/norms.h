// The step between a projection and attention as the block runs it.
#pragma once
#include <stdint.h>

namespace chorus {

// chorus_qk_norm_rope on the queries (scale q_scale; none where q is null) and on the keys and chorus_v_transpose on the
// values, in one launch: three column ranges of one [L, ld] projection, or of two. The same results bit for bit. The
// caller has checked the shapes (dh 64 or 128, Lpad % 64 == 0, D % 64 == 0, ld % 8 == 0) and alignments.
// The launch also clears n_clear words at `clear`.
// With `text` the same launch prepares the text keys and values too (neither queries nor rotation), the same H and dh.
struct PrepareText {
  const uint16_t *k, *v;
  long ld;
  const float* gain_k;
  uint16_t *kh, *vt;
  long L, Lpad;
};
int32_t attn_prepare(const uint16_t* q, const uint16_t* k, const uint16_t* v, long ld, const float* gain_q, const float* gain_k,
                     uint16_t* qh, uint16_t* kh, uint16_t* vt, long L, long Lpad, int H, int dh, const int32_t* token_idx, int gH,
                     int gW, int rope, float q_scale, void* stream, const PrepareText* text = nullptr, uint32_t* clear = nullptr,
                     int n_clear = 0);

// chorus_ln_modulate in a launch that also clears n_clear words at `clear`
int32_t ln_modulate(const float* x, uint16_t* out, long L, int D, const float* mul0, const float* mul1, const float* add0,
                    const float* add1, int plus_one, uint32_t* clear, int n_clear, void* stream);

}  // namespace chorus
