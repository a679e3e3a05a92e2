// Self-attention as a block runs it: chorus_attention's variant 6 over 512 keys or more, with scratch. A last round of tiles that would
// leave half of the compute units idle then runs in slices of the keys.
#pragma once
#include <stddef.h>
#include <stdint.h>

namespace chorus {

// Two pieces of scratch (16-byte aligned device memory, either may be empty), used only by the kernels of the call.
struct AttnScratch {
  void* first;
  size_t first_bytes;
  void* rest;
  size_t rest_bytes;
};

// How the launch goes with that scratch on a GPU of `cus` compute units: the first `whole` tiles of 256 rows (row tiles fastest, then
// heads) a workgroup each, the `sliced` tiles behind them in `slices` workgroups each; slices 0: as chorus_attention does it.
// Depends on the sizes given here and on nothing else.
struct AttnSlices {
  long whole;
  int sliced, slices;
};
// The first of a tile's `units` tiles of keys that slice i of `slices` takes (i == slices: their end): i units / slices, in 32 bits for all
// that chorus_attention_slices admits (65536 slices), where that product would not fit.
constexpr int first_of_slice(int i, int units, int slices) {
  return units / slices * i + (int)((uint32_t)(units % slices) * (uint32_t)i / (uint32_t)slices);
}
AttnSlices attention_slices(long L, int H, int dh, int cus, const AttnScratch& scratch);
// 32-bit words at the start of scratch.first that have to be zero when that launch starts
inline int attention_slices_words(const AttnSlices& p) { return 2 * p.sliced; }
int32_t attention_sliced(const uint16_t* Q, const uint16_t* K, const uint16_t* Vt, uint16_t* O, long L, long LPad, int H, int dh,
                         const AttnSlices& plan, const AttnScratch& scratch, void* stream);
// Whether attention over Lk keys takes its queries as the rows of their projection, and that attention: chorus_qk_norm_rope without
// rotation and with scale 1 on q [Lq, H * dh], then chorus_attention's default choice, in one launch, the same bits.
bool attention_raw_queries(long Lq, long Lk, long LkPad, int H, int dh, bool factor, int cus);
int32_t attention_raw(const uint16_t* q, const float* gain, const uint16_t* K, const uint16_t* Vt, uint16_t* O, const float* col_scale, long Lq,
                      long Lk, long LkPad, int H, void* stream);
// compute units of the current device; a negative status on failure
int device_cus();

}  // namespace chorus
