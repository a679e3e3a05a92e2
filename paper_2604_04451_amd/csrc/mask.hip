// Region-mask pipeline (Sec. 3.3.1 stages 2-3, Sec. 3.3.2 Eq. 5): key-frame propagation
// fused with the max-pool projection onto the latent / token grid, and the two box
// dilations that give M_edit and M_see. Byte masks, any non-zero byte is "set",
// outputs are 0/1. Integer work: results are exact.
#include "chorus_ops.h"
#include "common.h"

namespace chorus {

constexpr int kProjThreads = 256;
constexpr int kProjWaves = kProjThreads / 64;

// One workgroup per output row (t_o, y_o). Phase 1 ORs every input row of the window
// (kh rows of each distinct key frame the window's frames map to) into a per-column
// byte vector in LDS; phase 2 ORs kw columns per output site. The kernel is a chain of latencies: the window's
// key frames are looked up together, a wave has four rows in flight, and the columns are read in pieces of 16 bytes wherever
// a row starts (an unaligned piece is one load too; the columns behind the last whole piece are read singly).
__global__ __launch_bounds__(kProjThreads) void mask_project_kernel(const uint8_t* __restrict__ key_masks, int Kf,
                                                                    const int32_t* __restrict__ frame_key, int Tp, int Hp,
                                                                    int Wp, int kt, int kh, int kw, int t_lead, int Ho, int Wo,
                                                                    uint8_t* __restrict__ out) {
  extern __shared__ uint32_t col_any[];  // ceil(Wp / 16) * 4 words, byte c = OR over the window's rows of column c
  const int t_o = blockIdx.x / Ho, y_o = blockIdx.x % Ho;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int words = ((Wp + 15) / 16) * 4;

  int t0, t1;
  if (t_o < t_lead) {
    t0 = t_o;
    t1 = t_o + 1;
  } else {
    t0 = t_lead + (t_o - t_lead) * kt;
    t1 = min(t0 + kt, Tp);
  }
  const int y0 = y_o * kh, rows_per_frame = min(y0 + kh, Hp) - y0;
  const size_t plane = (size_t)Hp * Wp;
  const int chunks = Wp >> 4;
  constexpr int F = 8, U = 4;  // frames looked up together, rows in flight

  for (int tb = t0; tb < t1; tb += F) {
    int key[F];
#pragma unroll
    for (int f = 0; f < F; ++f) {
      const int t = min(tb + f, t1 - 1);
      key[f] = frame_key ? frame_key[t] : t;
    }
    if (tb == t0) {
      for (int i = tid; i < words; i += kProjThreads) col_any[i] = 0;
      __syncthreads();
    }
    int prev_key = -1;
#pragma unroll
    for (int f = 0; f < F; ++f) {
      if (key[f] == prev_key) continue;  // same key frame as the previous frame of this window: nothing new
      prev_key = key[f];
      if (key[f] < 0 || key[f] >= Kf) continue;  // a frame with no key frame contributes nothing
      const uint8_t* frame = key_masks + (size_t)key[f] * plane + (size_t)y0 * Wp;
      // lanes walk the 16-byte pieces of a row, the waves share the rows; past the last row that row again
      for (int c = lane; c < chunks; c += 64) {
        u32x4 acc = {0u, 0u, 0u, 0u};
        for (int r = wave; r < rows_per_frame; r += U * kProjWaves) {
          u32x4 v[U];
#pragma unroll
          for (int u = 0; u < U; ++u)
            __builtin_memcpy(&v[u], frame + (size_t)min(r + u * kProjWaves, rows_per_frame - 1) * Wp + (size_t)c * 16, 16);
#pragma unroll
          for (int u = 0; u < U; ++u) acc |= v[u];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (acc[k]) atomicOr(&col_any[c * 4 + k], acc[k]);
      }
      const int tail = Wp & 15;
      for (int i = tid; i < tail * rows_per_frame; i += kProjThreads) {
        const int c = chunks * 16 + i % tail;
        if (frame[(size_t)(i / tail) * Wp + c]) atomicOr(&col_any[c >> 2], 1u << ((c & 3) * 8));
      }
    }
  }
  __syncthreads();
  const uint8_t* cols = reinterpret_cast<const uint8_t*>(col_any);
  uint8_t* orow = out + ((size_t)t_o * Ho + y_o) * Wo;
  for (int x = tid; x < Wo; x += kProjThreads) {
    const int c0 = x * kw, c1 = min(c0 + kw, Wp);
    uint32_t any = 0;
    if ((kw & 3) == 0) {  // whole words: the bytes behind the last column are zeros
      for (int c = c0; c < c1; c += 4) any |= col_any[c >> 2];
    } else {
      for (int c = c0; c < c1; ++c) any |= cols[c];
    }
    orow[x] = any ? 1 : 0;
  }
}

// Eq. 5 with box kernels is separable, and a row of sites is a row of bits. One workgroup per (frame t, strip of rows): a wave
// takes a row of the strip or of its r_see rows of halo, 64 sites at a time, ORs them over the time window and leaves the
// ballot in LDS; a thread per 64 sites then ORs a row's bits shifted by up to the radius along x, then another the rows of
// the window along y, for both radii; the bits leave as bytes. Sites beyond the grid count as 0. (On bytes throughout, each
// step a loop over a neighbourhood in LDS, 6.4 us at 21 x 30 x 52, now 5.4.)
constexpr int kHierThreads = 256;
constexpr int kHierLdsBytes = 48 * 1024;

// 64 bits from bit position at on (any sign) of a row of n words; 0 outside
__device__ __forceinline__ uint64_t bits_at(const uint64_t* row, int n, int at) {
  const int q = at >> 6, m = at & 63;  // (towards minus infinity)
  const uint64_t lo = q >= 0 && q < n ? row[q] : 0, hi = m && q + 1 >= 0 && q + 1 < n ? row[q + 1] : 0;
  return m ? (lo >> m) | (hi << (64 - m)) : lo;
}

__global__ __launch_bounds__(kHierThreads) void mask_hierarchy_lds_kernel(const uint8_t* __restrict__ base, int T, int H, int W,
                                                                          int et, int eh, int ew, int st, int sh, int sw,
                                                                          int strip, int nstrips, uint8_t* __restrict__ edit,
                                                                          uint8_t* __restrict__ see) {
  extern __shared__ uint64_t hier_lds[];
  const int t = blockIdx.x / nstrips, y0 = (blockIdx.x % nstrips) * strip, y1 = min(H, y0 + strip);
  const int ya = max(0, y0 - sh), yb = min(H, y1 + sh);  // rows held in LDS
  const int nw = (W + 63) / 64, n_in = (yb - ya) * nw, n_out = (y1 - y0) * nw;
  uint64_t* S0 = hier_lds;       // [rows held][nw]: OR over the see time window
  uint64_t* E0 = S0 + n_in;      // OR over the edit time window
  uint64_t* S1 = E0 + n_in;      // [rows of the strip][nw]: the result's bits
  uint64_t* E1 = S1 + n_out;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int t0 = max(0, t - st), t1 = min(T - 1, t + st);
  const size_t plane = (size_t)H * W;
  constexpr int U = 4, R = 4, kW = kHierThreads / 64;  // frames and rows in flight; past the last that one again
  for (int i0 = wave; i0 < n_in; i0 += R * kW) {
    const uint8_t* p[R];
    uint32_t s[R] = {}, e[R] = {};
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int i = min(i0 + r * kW, n_in - 1), row = i / nw;
      p[r] = base + (size_t)(ya + row) * W + min((i - row * nw) * 64 + lane, W - 1);
    }
    for (int tt = t0; tt <= t1; tt += U) {
      uint32_t v[R][U];
#pragma unroll
      for (int r = 0; r < R; ++r)
#pragma unroll
        for (int u = 0; u < U; ++u) v[r][u] = p[r][min(tt + u, t1) * plane];
#pragma unroll
      for (int r = 0; r < R; ++r)
#pragma unroll
        for (int u = 0; u < U; ++u) {
          s[r] |= v[r][u];
          e[r] |= abs(min(tt + u, t1) - t) <= et ? v[r][u] : 0u;
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int i = i0 + r * kW;
      if (i >= n_in) break;
      const bool in = (i - i / nw * nw) * 64 + lane < W;
      const uint64_t sb = __ballot(in && s[r]), eb = __ballot(in && e[r]);
      if (lane == 0) {
        S0[i] = sb;
        E0[i] = eb;
      }
    }
  }
  __syncthreads();
  // along x, then along y
  for (int i = threadIdx.x; i < n_in; i += kHierThreads) {
    const int row = i / nw, at = (i - row * nw) * 64;
    uint64_t s = 0, e = 0;
    for (int k = -sw; k <= sw; ++k) s |= bits_at(S0 + row * nw, nw, at + k);
    for (int k = -ew; k <= ew; ++k) e |= bits_at(E0 + row * nw, nw, at + k);
    E1[n_out + i] = s;
    E1[n_out + n_in + i] = e;
  }
  __syncthreads();
  const uint64_t* Sx = E1 + n_out;
  const uint64_t* Ex = Sx + n_in;
  for (int i = threadIdx.x; i < n_out; i += kHierThreads) {
    const int row = i / nw, w = i - row * nw, y = y0 + row;
    uint64_t s = 0, e = 0;
    for (int yy = max(ya, y - sh); yy <= min(yb - 1, y + sh); ++yy) s |= Sx[(yy - ya) * nw + w];
    for (int yy = max(ya, y - eh); yy <= min(yb - 1, y + eh); ++yy) e |= Ex[(yy - ya) * nw + w];
    S1[i] = s;
    E1[i] = e;
  }
  __syncthreads();
  for (int i = wave; i < n_out; i += kHierThreads / 64) {
    const int row = i / nw, x = (i - row * nw) * 64 + lane;
    if (x >= W) continue;
    const size_t o = (size_t)t * plane + (size_t)(y0 + row) * W + x;
    if (edit) edit[o] = (uint8_t)((E1[i] >> lane) & 1);
    if (see) see[o] = (uint8_t)((S1[i] >> lane) & 1);
  }
}

// Fallback for planes too wide for the LDS kernel. One thread per site: scans the (2 r_see + 1)^3 box once;
// the inner (2 r_edit + 1)^3 box feeds M_edit. Sites beyond the grid count as 0 (the box is cut at the border).
__global__ __launch_bounds__(256) void mask_hierarchy_kernel(const uint8_t* __restrict__ base, int T, int H, int W, int et,
                                                             int eh, int ew, int st, int sh, int sw,
                                                             uint8_t* __restrict__ edit, uint8_t* __restrict__ see) {
  const int n = T * H * W;
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const int x = i % W, y = (i / W) % H, t = i / (W * H);
  const int x0 = max(0, x - sw), x1 = min(W - 1, x + sw);
  const int y0 = max(0, y - sh), y1 = min(H - 1, y + sh);
  const int t0 = max(0, t - st), t1 = min(T - 1, t + st);
  uint32_t any_see = 0, any_edit = 0;
  for (int tt = t0; tt <= t1; ++tt) {
    const bool in_t = abs(tt - t) <= et;
    for (int yy = y0; yy <= y1; ++yy) {
      const bool in_ty = in_t && abs(yy - y) <= eh;
      const uint8_t* row = base + ((size_t)tt * H + yy) * W;
      uint32_t row_see = 0, row_edit = 0;
      for (int xx = x0; xx <= x1; ++xx) {
        uint32_t v = row[xx];
        row_see |= v;
        row_edit |= (abs(xx - x) <= ew) ? v : 0u;
      }
      any_see |= row_see;
      any_edit |= in_ty ? row_edit : 0u;
    }
  }
  if (edit) edit[i] = any_edit ? 1 : 0;
  if (see) see[i] = any_see ? 1 : 0;
}

// The radii that the kernels are given are cut at the grid: a radius of n - 1 reaches every one of n sites, so a larger one (a
// caller's "everything") has the same result; the kernels' loops then take at most 2 n - 1 steps and their sums stay in 32 bits.
// Strips of rows: enough workgroups to spread over the chip, each strip with its r_see halo within the LDS budget (two
// sets of bits per row held, before and after the pass along x, and one per row of the strip); strip 0: the rows do not fit,
// the kernel that takes a site at a time.
chorus_hierarchy_plan plan_hierarchy(int T, int H, int W, const int32_t* r_edit, const int32_t* r_see) {
  chorus_hierarchy_plan p{};
  const int n[3] = {T, H, W};
  for (int a = 0; a < 3; ++a) {
    p.r_edit[a] = r_edit[a] < n[a] ? r_edit[a] : n[a] - 1;
    p.r_see[a] = r_see[a] < n[a] ? r_see[a] : n[a] - 1;
  }
  const long halo = 2L * p.r_see[1], word = ((long)W + 63) / 64 * 8;
  auto lds = [&](long strip) { return (4 * (strip + halo < H ? strip + halo : (long)H) + 2 * strip) * word; };
  int nstrips = (128 + T - 1) / T;
  if (nstrips > H) nstrips = H;
  long strip = (H + nstrips - 1) / nstrips;
  if (lds(strip) > kHierLdsBytes) {
    const long cut = (kHierLdsBytes / word - 4 * halo) / 6, whole = (kHierLdsBytes / word - 4L * H) / 2;
    const long fit = cut > whole ? cut : whole;  // the halo's rows beyond the strip's own, or every row of the grid
    strip = fit < strip ? fit : strip;
  }
  if (strip < 1) return p;
  p.strip = (int)strip;
  p.nstrips = (int)((H + strip - 1) / strip);
  p.lds_bytes = (int)lds(strip);
  return p;
}

}  // namespace chorus

using namespace chorus;

extern "C" {

int32_t chorus_mask_pooled_extent(int32_t n, int32_t k, int32_t lead) {
  if (k < 1 || lead < 0 || n < lead) return CHORUS_E_ARG;
  return lead + (int32_t)(((int64_t)n - lead + k - 1) / k);
}

int32_t chorus_mask_project(const uint8_t* key_masks, int32_t Kf, const int32_t* frame_key, int32_t Tp, int32_t Hp,
                            int32_t Wp, int32_t kt, int32_t kh, int32_t kw, int32_t t_lead, uint8_t* out, void* stream) {
  if (Kf < 0 || Tp < 0 || Hp < 0 || Wp < 0 || kt < 1 || kh < 1 || kw < 1 || t_lead < 0 || t_lead > Tp) return CHORUS_E_ARG;
  if (!frame_key && Kf != Tp) return CHORUS_E_ARG;
  const int64_t To = t_lead + ((int64_t)Tp - t_lead + kt - 1) / kt;
  const int64_t Ho = ((int64_t)Hp + kh - 1) / kh, Wo = ((int64_t)Wp + kw - 1) / kw;
  if (To * Ho * Wo == 0) return CHORUS_OK;
  if (!key_masks || !out || Kf == 0) return CHORUS_E_ARG;
  if (To * Ho > 0x7fffffffLL || (int64_t)Kf * Hp * Wp > 0x7fffffffffLL) return CHORUS_E_SHAPE;
  const size_t lds = (size_t)((Wp + 15) / 16) * 16;
  if (lds > 64 * 1024) return CHORUS_E_SHAPE;
  // a window longer than the axis holds all of it, and the kernel's t0 + kt and y0 + kh stay in 32 bits
  kt = kt < Tp ? kt : Tp;
  kh = kh < Hp ? kh : Hp;
  kw = kw < Wp ? kw : Wp;
  hipStream_t s = (hipStream_t)stream;
  hipLaunchKernelGGL(mask_project_kernel, dim3((unsigned)(To * Ho)), dim3(kProjThreads), lds, s, key_masks, Kf, frame_key, Tp, Hp,
                     Wp, kt, kh, kw, t_lead, (int)Ho, (int)Wo, out);
  CHORUS_LAUNCH_CHECK();
  return CHORUS_OK;
}

int32_t chorus_mask_hierarchy(const uint8_t* mask_base, int32_t T, int32_t H, int32_t W, const int32_t r_edit[3],
                              const int32_t r_see[3], uint8_t* mask_edit, uint8_t* mask_see, void* stream) {
  if (T < 0 || H < 0 || W < 0 || !r_see) return CHORUS_E_ARG;
  int32_t re[3];
  for (int a = 0; a < 3; ++a) {
    re[a] = r_edit ? r_edit[a] : 0;
    if (re[a] < 0 || r_see[a] < re[a]) return CHORUS_E_ARG;  // Eq. 5 needs r' >= r on every axis
  }
  if (mask_edit && !r_edit) return CHORUS_E_ARG;
  const int64_t n = (int64_t)T * H * W;
  if (n == 0) return CHORUS_OK;
  if (!mask_base || (!mask_edit && !mask_see)) return CHORUS_E_ARG;
  if (mask_base == mask_edit || mask_base == mask_see) return CHORUS_E_ARG;  // every site reads its neighbours
  if (n > 0x7fffffffLL - 256) return CHORUS_E_SHAPE;
  hipStream_t s = (hipStream_t)stream;
  const chorus_hierarchy_plan p = plan_hierarchy(T, H, W, re, r_see);
  if (p.strip > 0)
    hipLaunchKernelGGL(mask_hierarchy_lds_kernel, dim3((unsigned)((long)T * p.nstrips)), dim3(kHierThreads), (size_t)p.lds_bytes, s,
                       mask_base, T, H, W, p.r_edit[0], p.r_edit[1], p.r_edit[2], p.r_see[0], p.r_see[1], p.r_see[2], p.strip,
                       p.nstrips, mask_edit, mask_see);
  else
    hipLaunchKernelGGL(mask_hierarchy_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, mask_base, T, H, W, p.r_edit[0],
                       p.r_edit[1], p.r_edit[2], p.r_see[0], p.r_see[1], p.r_see[2], mask_edit, mask_see);
  CHORUS_LAUNCH_CHECK();
  return CHORUS_OK;
}

int32_t chorus_mask_hierarchy_plan(int32_t T, int32_t H, int32_t W, const int32_t r_edit[3], const int32_t r_see[3],
                                   chorus_hierarchy_plan* out) {
  if (T < 1 || H < 1 || W < 1 || !r_edit || !r_see || !out) return CHORUS_E_ARG;
  for (int a = 0; a < 3; ++a)
    if (r_edit[a] < 0 || r_see[a] < r_edit[a]) return CHORUS_E_ARG;
  if ((int64_t)T * H > 0x7fffffffLL || (int64_t)T * H * W > 0x7fffffffLL - 256) return CHORUS_E_SHAPE;
  *out = plan_hierarchy(T, H, W, r_edit, r_see);
  return CHORUS_OK;
}

}  // extern "C"
