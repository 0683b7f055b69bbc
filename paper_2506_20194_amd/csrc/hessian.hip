// Stage 1 of the DuoGPT layer solver on gfx950: per-token activation
// sparsification and accumulation of H = Xh Xh^T, G = dX Xh^T and
// a = diag(dX dX^T) (paper Sec. 4.2-4.3, Algorithm 1 first lines).
//
// Pipeline per chunk of tokens:
//   act_select  finds each token's largest dropped key (|x|, channel) by a
//               search on the magnitude bits (one wave or one workgroup per
//               token; the same kernels can write the sparsified row);
//   pack        applies the per-token threshold and writes Xh and dX (and,
//               for two input streams, the low part of dX) in an MFMA-ready
//               token-blocked layout [token block][group][channel][16 bytes];
//               also sums dX^2 per channel;
//   gram        gram_bf16_kernel or gram_f32_kernel over 256 x 256 tiles, each of H
//               (on and above the diagonal) or of G (there, or everywhere);
//   reductions  fixed-order sums of the partial tiles (deterministic), and H's
//               lower triangle from its upper one.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "common.h"
#include "internal.h"
#include "pingpong.h"

namespace duo {

// ---------------------------------------------------------------------------
// element traits
// ---------------------------------------------------------------------------
template <typename T>
struct Elem;
template <>
struct Elem<uint16_t> {  // bf16 stored as raw bits
  static constexpr int kMagBits = 15;
  static constexpr uint32_t kInfMag = 0x7f80u;  // magnitudes >= this are inf or NaN
  __device__ static inline uint32_t mag(uint16_t v) { return v & 0x7fffu; }
  __device__ static inline float to_f32(uint16_t v) { return bf16_bits_to_f32(v); }
  __device__ static inline uint16_t from_f32(float f) { return f32_to_bf16_bits(f); }
};
template <>
struct Elem<float> {
  static constexpr int kMagBits = 31;
  static constexpr uint32_t kInfMag = 0x7f800000u;
  __device__ static inline uint32_t mag(float v) { return __float_as_uint(v) & 0x7fffffffu; }
  __device__ static inline float to_f32(float v) { return v; }
  __device__ static inline float from_f32(float f) { return f; }
};

// ---------------------------------------------------------------------------
// block-wide helpers for 256 threads
// ---------------------------------------------------------------------------
__device__ inline int wave_sum(int v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// Sum over the 256 threads; `red` is LDS int[8], `slot` alternates 0/1 so a
// single barrier per call is enough.
__device__ inline int block_sum256(int v, int* red, int slot) {
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) red[slot * 4 + (threadIdx.x >> 6)] = v;
  __syncthreads();
  return red[slot * 4] + red[slot * 4 + 1] + red[slot * 4 + 2] + red[slot * 4 + 3];
}

// ---------------------------------------------------------------------------
// act_select: per-token threshold key.  Element (t, c) is kept iff
// (mag(x) << 32 | c) > thr[t] (signed compare).  thr = -1 keeps everything,
// INT64_MAX drops everything.
// ---------------------------------------------------------------------------
// Non-finite inputs (NaN or +-inf: the magnitude's exponent field all ones)
// are reported by setting *nf (when not null) to 1; they still take part in
// the selection with their magnitude bits (NaN above inf above any finite
// value), so the kept set stays a function of the bit patterns.
__device__ inline void flag_nonfinite(bool bad, uint32_t* nf) {
  if (nf && __ballot(bad) != 0 && (threadIdx.x & 63) == 0) atomicOr(nf, 1u);
}

template <typename T, int C>
__global__ __launch_bounds__(256) void act_select_kernel(const T* __restrict__ X, int64_t ldx, int m,
                                                         int k, int z, int64_t* __restrict__ thr,
                                                         uint32_t* __restrict__ nf) {
  __shared__ int red[8];
  const int t = blockIdx.x;
  if (t >= m) return;
  const T* row = X + (int64_t)t * ldx;
  uint32_t mag[C];
  bool bad = false;
#pragma unroll
  for (int e = 0; e < C; ++e) {
    const int c = threadIdx.x + 256 * e;  // coalesced: consecutive threads, consecutive channels
    mag[e] = c < k ? Elem<T>::mag(row[c]) : 0xffffffffu;
    bad |= c < k && mag[e] >= Elem<T>::kInfMag;
  }
  flag_nonfinite(bad, nf);
  if (z <= 0 || z >= k) {
    if (threadIdx.x == 0) thr[t] = z <= 0 ? (int64_t)-1 : INT64_MAX;
    return;
  }
  // smallest v with count(mag <= v) >= z
  uint32_t lo = 0, hi = (1u << Elem<T>::kMagBits) - 1u;
  int slot = 0;
  while (lo < hi) {
    const uint32_t mid = lo + ((hi - lo) >> 1);
    int cnt = 0;
#pragma unroll
    for (int e = 0; e < C; ++e) cnt += mag[e] <= mid;
    cnt = block_sum256(cnt, red, slot);
    slot ^= 1;
    if (cnt >= z)
      hi = mid;
    else
      lo = mid + 1;
  }
  const uint32_t v = lo;
  int lt = 0;
#pragma unroll
  for (int e = 0; e < C; ++e) lt += mag[e] < v;
  lt = block_sum256(lt, red, slot);
  slot ^= 1;
  int need = z - lt;  // 1 <= need <= (number of ties)
  // the need-th tie in channel order, i.e. in (e, thread) order
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
  for (int e = 0; e < C; ++e) {
    const int eq = mag[e] == v;
    int incl = eq;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int y = __shfl_up(incl, o);
      if (lane >= o) incl += y;
    }
    if (lane == 63) red[slot * 4 + wv] = incl;
    __syncthreads();
    int base = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const int q = red[slot * 4 + w];
      base += w < wv ? q : 0;
      tot += q;
    }
    slot ^= 1;
    if (need <= tot) {  // uniform
      if (eq && base + incl == need) thr[t] = ((int64_t)v << 32) | (int64_t)(threadIdx.x + 256 * e);
      return;
    }
    need -= tot;
  }
}

// One wave per token (bf16, 16-byte aligned rows, k % 8 == 0, k <= 512 V):
// lane l holds channels 512u + 8l + j (u < V, j < 8) in registers, so the
// bisection and the tie scan reduce with cross-lane operations only.  Same
// threshold key as act_select_kernel.  APPLY: the token with the dropped entries
// zeroed goes to Y instead of its key to thr (the row is read again from L2).
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

__device__ inline int wave_sum_i(int v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

__device__ inline int wave_incl_scan(int v) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(v, o);
    if (lane >= o) v += y;
  }
  return v;
}

// Entries of one 16-byte vector (channels c .. c + 7) with magnitude above v, or
// equal to it past channel tc, kept; the others zero.
__device__ __forceinline__ u32x4 apply_key(const u32x4& x, int c, int v, int tc) {
  u32x4 y;
#pragma unroll
  for (int h = 0; h < 4; ++h) {
    const int m0 = (int)(x[h] & 0x7fffu), m1 = (int)((x[h] >> 16) & 0x7fffu);
    const uint32_t k0 = m0 > v || (m0 == v && c + 2 * h > tc) ? 0xffffu : 0u;
    const uint32_t k1 = m1 > v || (m1 == v && c + 2 * h + 1 > tc) ? 0xffff0000u : 0u;
    y[h] = x[h] & (k0 | k1);
  }
  return y;
}

template <int V, bool APPLY>
__global__ __launch_bounds__(256) void act_select_wave_kernel(const uint16_t* __restrict__ X, int64_t ldx, int m,
                                                              int k, int z, int64_t* __restrict__ thr,
                                                              uint32_t* __restrict__ nf, uint16_t* __restrict__ Y,
                                                              int64_t ldy) {
  const int t = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (t >= m) return;  // uniform per wave
  const uint16_t* row = X + (int64_t)t * ldx;
  uint32_t mag[8 * V];
  bool bad = false;
#pragma unroll
  for (int u = 0; u < V; ++u) {
    const int c = 512 * u + 8 * lane;
    const bool ok = c < k;
    const u32x4 w = *(const u32x4*)(row + (ok ? c : 0));
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      mag[8 * u + j] = ok ? (w[j >> 1] >> (16 * (j & 1))) & 0x7fffu : 0xffffffffu;
      bad |= ok && mag[8 * u + j] >= 0x7f80u;
    }
  }
  flag_nonfinite(bad, nf);
  // APPLY's last step: everything above magnitude v, and at v past channel tc
  auto write = [&](int v, int tc) {
#pragma unroll
    for (int u = 0; u < V; ++u) {
      const int c = 512 * u + 8 * lane;
      if (c < k) *(u32x4*)(Y + (int64_t)t * ldy + c) = apply_key(*(const u32x4*)(row + c), c, v, tc);
    }
  };
  if (z <= 0 || z >= k) {
    if (APPLY)
      write(z <= 0 ? -1 : 0x10000, 0);
    else if (lane == 0)
      thr[t] = z <= 0 ? (int64_t)-1 : INT64_MAX;
    return;
  }
  // v = the smallest magnitude with count(mag <= v) >= z, from two LDS
  // histograms of the wave's own: the top 10 of the 15 magnitude bits (lane l
  // scans bins 16l .. 16l+15), then the low 5 bits of the entries in the bin of
  // the z-th entry (lane l < 32: bin l).  Coarse bins of exponent plus two
  // mantissa bits spread a token's entries over four times as many bins as
  // the exponent alone, so fewer lanes of an atomic collide on one address.
  // Within a wave the LDS operations run in order, so no barrier is needed.
  constexpr int kFineBits = 5, kCoarse = 1 << (15 - kFineBits), kFine = 1 << kFineBits;
  __shared__ __attribute__((aligned(16))) uint32_t hist_w[4][kCoarse + kFine];
  uint32_t* hc = hist_w[threadIdx.x >> 6];
  uint32_t* hf = hc + kCoarse;
  for (int i = lane; i < (kCoarse + kFine) / 4; i += 64) ((u32x4*)hc)[i] = u32x4{0u, 0u, 0u, 0u};
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int e = 0; e < 8 * V; ++e)
    if (mag[e] < 0x8000u) atomicAdd(&hc[mag[e] >> kFineBits], 1u);
  __builtin_amdgcn_wave_barrier();
  constexpr int PER = kCoarse / 64;
  int h[PER], loc = 0;
#pragma unroll
  for (int i = 0; i < PER / 4; ++i) {
    const u32x4 q = ((const u32x4*)hc)[(PER / 4) * lane + i];
#pragma unroll
    for (int j = 0; j < 4; ++j) h[4 * i + j] = (int)q[j];
  }
#pragma unroll
  for (int i = 0; i < PER; ++i) loc += h[i];
  int incl = wave_incl_scan(loc), run = incl - loc, cb = -1, below = 0;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    if (run < z && z <= run + h[i]) {
      cb = PER * lane + i;
      below = run;
    }
    run += h[i];
  }
  const int src = __builtin_ctzll(__ballot(cb >= 0));  // the one lane holding the z-th entry's bin
  cb = __shfl(cb, src);
  below = __shfl(below, src);
#pragma unroll
  for (int e = 0; e < 8 * V; ++e)
    if ((int)(mag[e] >> kFineBits) == cb) atomicAdd(&hf[mag[e] & (kFine - 1u)], 1u);
  __builtin_amdgcn_wave_barrier();
  const int f0 = lane < kFine ? (int)hf[lane] : 0;
  incl = wave_incl_scan(f0);
  run = below + incl - f0;
  int fb = -1, lt = 0;
  if (run < z && z <= run + f0) {
    fb = lane;
    lt = run;
  }
  const int src2 = __builtin_ctzll(__ballot(fb >= 0));
  const uint32_t v = ((uint32_t)cb << kFineBits) | (uint32_t)__shfl(fb, src2);
  int need = z - __shfl(lt, src2);  // 1 <= need <= number of ties
  // the need-th tie in channel order (u, lane, j)
  int tc = -1;  // its channel, in the lane that holds it
#pragma unroll
  for (int u = 0; u < V; ++u) {
    int eq = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) eq += mag[8 * u + j] == v;
    const int incl = wave_incl_scan(eq);
    const int tot = __shfl(incl, 63);
    if (need <= tot) {  // uniform
      int cnt = incl - eq;
      if (cnt < need && need <= incl) {
#pragma unroll
        for (int j = 0; j < 8; ++j)
          if (mag[8 * u + j] == v && ++cnt == need) tc = 512 * u + 8 * lane + j;
      }
      break;
    }
    need -= tot;
  }
  if (APPLY)
    write((int)v, __shfl(tc, __builtin_ctzll(__ballot(tc >= 0))));
  else if (tc >= 0)
    thr[t] = ((int64_t)v << 32) | (int64_t)tc;
}

// One 256-thread workgroup per token (bf16, 16-byte aligned rows, k % 8 == 0,
// 8192 < k <= 2048 V): thread i holds channels 2048u + 8i + j (u < V, j < 8)
// in registers, loaded as 16-byte vectors (coalesced); the two histograms of
// the wave kernel (top 10 magnitude bits, then the low 5 of the z-th entry's
// bin) are shared by the workgroup, and ties are resolved in channel order
// (u, thread, j) with one block scan per u until the need-th tie is reached.
// APPLY as in the wave kernel, from the registers.
template <int V, bool APPLY>
__global__ __launch_bounds__(256) void act_select_block_kernel(const uint16_t* __restrict__ X, int64_t ldx, int m,
                                                               int k, int z, int64_t* __restrict__ thr,
                                                               uint32_t* __restrict__ nf, uint16_t* __restrict__ Y,
                                                               int64_t ldy) {
  constexpr int kFineBits = 5, kCoarse = 1 << (15 - kFineBits), kFine = 1 << kFineBits;
  __shared__ __attribute__((aligned(16))) uint32_t hc[kCoarse];
  __shared__ uint32_t hf[kFine];
  __shared__ int wsum[2][4];
  __shared__ int found[2];
  __shared__ int tie_w[4][V];
  const int t = blockIdx.x;
  if (t >= m) return;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const uint16_t* row = X + (int64_t)t * ldx;
  // the raw bf16 pairs (two channels per register: 8 V values in 4 V
  // registers, so the largest form still fits without spilling); vector u is
  // valid when 2048 u + 8 tid < k (k % 8 == 0)
  uint32_t w[4 * V];
  bool bad = false;
#pragma unroll
  for (int u = 0; u < V; ++u) {
    const bool ok = 2048 * u + 8 * tid < k;
    const u32x4 x4 = *(const u32x4*)(row + (ok ? 2048 * u + 8 * tid : 0));
#pragma unroll
    for (int h = 0; h < 4; ++h) {
      w[4 * u + h] = x4[h];
      bad |= ok && (x4[h] & 0x7f80u) == 0x7f80u;
      bad |= ok && (x4[h] & 0x7f800000u) == 0x7f800000u;
    }
  }
  flag_nonfinite(bad, nf);
  auto write = [&](int v, int tc) {
#pragma unroll
    for (int u = 0; u < V; ++u) {
      const int c = 2048 * u + 8 * tid;
      const u32x4 x = {w[4 * u], w[4 * u + 1], w[4 * u + 2], w[4 * u + 3]};
      if (c < k) *(u32x4*)(Y + (int64_t)t * ldy + c) = apply_key(x, c, v, tc);
    }
  };
  if (z <= 0 || z >= k) {
    if (APPLY)
      write(z <= 0 ? -1 : 0x10000, 0);
    else if (tid == 0)
      thr[t] = z <= 0 ? (int64_t)-1 : INT64_MAX;
    return;
  }
#define DUO_MAG(u, j) ((w[4 * (u) + ((j) >> 1)] >> (16 * ((j) & 1))) & 0x7fffu)
  ((u32x4*)hc)[tid] = u32x4{0u, 0u, 0u, 0u};  // 256 x 4 = kCoarse bins
  if (tid < kFine) hf[tid] = 0u;
  __syncthreads();
#pragma unroll
  for (int u = 0; u < V; ++u)
    if (2048 * u + 8 * tid < k)
#pragma unroll
      for (int j = 0; j < 8; ++j) atomicAdd(&hc[DUO_MAG(u, j) >> kFineBits], 1u);
  __syncthreads();
  // thread i owns coarse bins 4i .. 4i + 3: block exclusive scan of their sums
  const u32x4 q = ((const u32x4*)hc)[tid];
  const int loc = (int)(q[0] + q[1] + q[2] + q[3]);
  int incl = wave_incl_scan(loc);
  if (lane == 63) wsum[0][wv] = incl;
  __syncthreads();
  int run = incl - loc;
#pragma unroll
  for (int ww = 0; ww < 4; ++ww) run += ww < wv ? wsum[0][ww] : 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (run < z && z <= run + (int)q[i]) {
      found[0] = 4 * tid + i;
      found[1] = run;
    }
    run += (int)q[i];
  }
  __syncthreads();
  const int cb = found[0], below = found[1];
#pragma unroll
  for (int u = 0; u < V; ++u)
    if (2048 * u + 8 * tid < k)
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if ((int)(DUO_MAG(u, j) >> kFineBits) == cb) atomicAdd(&hf[DUO_MAG(u, j) & (kFine - 1u)], 1u);
  __syncthreads();
  if (wv == 0) {
    const int f0 = lane < kFine ? (int)hf[lane] : 0;
    const int fi = wave_incl_scan(f0);
    const int r0 = below + fi - f0;
    if (lane < kFine && r0 < z && z <= r0 + f0) {
      wsum[1][0] = lane;
      wsum[1][1] = r0;
    }
  }
  __syncthreads();
  const uint32_t v = ((uint32_t)cb << kFineBits) | (uint32_t)wsum[1][0];
  int need = z - wsum[1][1];  // 1 <= need <= number of ties
  // ties in channel order (u, thread, j): per-u totals from one block
  // reduction, then a scan over the threads for the u that holds the need-th
  // tie (static register indices throughout: u is selected, never indexed)
  int cnt[V];
#pragma unroll
  for (int u = 0; u < V; ++u) {
    const bool ok = 2048 * u + 8 * tid < k;
    int e = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) e += ok && DUO_MAG(u, j) == v;
    cnt[u] = e;
    const int ws_ = wave_sum(e);
    if (lane == 0) tie_w[wv][u] = ws_;
  }
  __syncthreads();
  int us = V - 1, base_u = 0;
  {
    int acc = 0;
    bool hit = false;
#pragma unroll
    for (int u = 0; u < V; ++u) {
      const int tu = tie_w[0][u] + tie_w[1][u] + tie_w[2][u] + tie_w[3][u];
      if (!hit && need <= acc + tu) {
        hit = true;
        us = u;
        base_u = acc;
      }
      acc += tu;
    }
  }
  int e = 0, wbase = 0;
#pragma unroll
  for (int u = 0; u < V; ++u)
    if (u == us) {
      e = cnt[u];
#pragma unroll
      for (int ww = 0; ww < 4; ++ww) wbase += ww < wv ? tie_w[ww][u] : 0;
    }
  const int wi = wave_incl_scan(e);
  int c0 = base_u + wbase + wi - e;  // ties before this thread's in channel order
  if (e > 0 && c0 < need && need <= c0 + e) {
#pragma unroll
    for (int u = 0; u < V; ++u)
      if (u == us)
#pragma unroll
        for (int j = 0; j < 8; ++j)
          if (DUO_MAG(u, j) == v && ++c0 == need) {
            const int tc = 2048 * u + 8 * tid + j;
            if (APPLY)
              found[0] = tc;  // (its bin index was read by every thread several barriers ago)
            else
              thr[t] = ((int64_t)v << 32) | (int64_t)tc;
          }
  }
  if (APPLY) {
    __syncthreads();
    // opaque: the entries are unpacked anew here, not kept unpacked from above
#pragma unroll
    for (int i = 0; i < 4 * V; ++i) asm volatile("" : "+v"(w[i]));
    write((int)v, found[0]);
  }
}
#undef DUO_MAG

// Whether the bf16 fast paths apply: 16-byte aligned rows of whole 8-channel
// vectors.
__host__ inline bool bf16_vec_ok(const void* X, int64_t ldx, int64_t k) {
  return X && (reinterpret_cast<uintptr_t>(X) % 16) == 0 && ldx % 8 == 0 && k % 8 == 0;
}

// The wave and workgroup kernels (aligned bf16 rows): thresholds, or with APPLY
// the sparsified rows.
template <bool APPLY>
static duo_status launch_act_select16(const uint16_t* X, int64_t ldx, int m, int k, int z, int64_t* thr, uint32_t* nf,
                                      uint16_t* Y, int64_t ldy, hipStream_t s) {
  if (k <= 8192) {
    const int v = (int)cdiv(k, 512);
    dim3 g((unsigned)cdiv(m, 4)), b(256);
#define DUO_WSEL(VV) \
  hipLaunchKernelGGL((act_select_wave_kernel<VV, APPLY>), g, b, 0, s, X, ldx, m, k, z, thr, nf, Y, ldy)
    if (v <= 1)
      DUO_WSEL(1);
    else if (v <= 2)
      DUO_WSEL(2);
    else if (v <= 4)
      DUO_WSEL(4);
    else if (v <= 8)
      DUO_WSEL(8);
    else
      DUO_WSEL(16);
#undef DUO_WSEL
  } else {
    const int v = (int)cdiv(k, 2048);
    dim3 g((unsigned)m), b(256);
#define DUO_BSEL(VV) \
  hipLaunchKernelGGL((act_select_block_kernel<VV, APPLY>), g, b, 0, s, X, ldx, m, k, z, thr, nf, Y, ldy)
    if (v <= 6)
      DUO_BSEL(6);
    else if (v <= 8)
      DUO_BSEL(8);
    else if (v <= 12)
      DUO_BSEL(12);
    else
      DUO_BSEL(16);
#undef DUO_BSEL
  }
  DUO_LAUNCH_CHECK();
  return DUO_OK;
}

template <typename T>
static duo_status launch_act_select(const T* X, int64_t ldx, int m, int k, int z, int64_t* thr, uint32_t* nf,
                                    hipStream_t s) {
  if (m <= 0) return DUO_OK;
  if constexpr (sizeof(T) == 2) {
    if (bf16_vec_ok(X, ldx, k) && k <= 32768)
      return launch_act_select16<false>((const uint16_t*)X, ldx, m, k, z, thr, nf, nullptr, 0, s);
  }
  const int per = (int)cdiv(k, 256);
  dim3 g(m), b(256);
#define DUO_SEL(CC) hipLaunchKernelGGL((act_select_kernel<T, CC>), g, b, 0, s, X, ldx, m, k, z, thr, nf)
  if (per <= 1)
    DUO_SEL(1);
  else if (per <= 2)
    DUO_SEL(2);
  else if (per <= 4)
    DUO_SEL(4);
  else if (per <= 8)
    DUO_SEL(8);
  else if (per <= 16)
    DUO_SEL(16);
  else if (per <= 32)
    DUO_SEL(32);
  else if (per <= 64)
    DUO_SEL(64);
  else
    DUO_SEL(128);
#undef DUO_SEL
  DUO_LAUNCH_CHECK();
  return DUO_OK;
}

duo_status act_threshold_run(const void* X, int32_t dtype, int64_t m, int64_t k, int64_t ldx, int z, int64_t* thr,
                             hipStream_t s) {
  if (dtype == DUO_BF16)
    return launch_act_select<uint16_t>((const uint16_t*)X, ldx, (int)m, (int)k, z, thr, nullptr, s);
  return launch_act_select<float>((const float*)X, ldx, (int)m, (int)k, z, thr, nullptr, s);
}

// Y = the sparsified rows of X in one pass: each row is read from memory once.
// (Thresholds first and a second kernel over X: 245 us for 16384 x 11008, now 146 us.)
duo_status act_sparsify_run(const uint16_t* X, int64_t m, int64_t k, int64_t ldx, int z, uint16_t* Y, int64_t ldy,
                            bool* done, hipStream_t s) {
  *done = bf16_vec_ok(X, ldx, k) && bf16_vec_ok(Y, ldy, k) && k <= 32768;
  return *done ? launch_act_select16<true>(X, ldx, (int)m, (int)k, z, nullptr, nullptr, Y, ldy, s) : DUO_OK;
}

// ---------------------------------------------------------------------------
// mask export (test hook): bit c of token t = kept
// ---------------------------------------------------------------------------
template <typename T>
__global__ void act_mask_kernel(const T* __restrict__ X, int64_t ldx, int m, int k,
                                const int64_t* __restrict__ thr, uint32_t* __restrict__ mask) {
  const int words = (int)cdiv(k, 32);
  const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (id >= (int64_t)m * words) return;
  const int t = (int)(id / words), w = (int)(id % words);
  const int64_t th = thr[t];
  uint32_t bits = 0;
  for (int e = 0; e < 32; ++e) {
    const int c = w * 32 + e;
    if (c >= k) break;
    const int64_t key = ((int64_t)Elem<T>::mag(X[(int64_t)t * ldx + c]) << 32) | c;
    if (key > th) bits |= 1u << e;
  }
  mask[id] = bits;
}

// ---------------------------------------------------------------------------
// pack: 256 channels x tpb tiles of 32 tokens per workgroup.
// Packed layout (EPG = 16 / sizeof(T) elements per group, NG = 32 / EPG):
//   P[((tb * NG + g) * kp + c) * EPG + e]  = value of token tb*32 + g*EPG + e.
// A workgroup takes tpb blocks of 32 tokens (pack_blocks); apart[workgroup row][kp]
// receives per-channel partial sums of dX^2.
// ---------------------------------------------------------------------------
template <typename T, bool TWO>
__global__ __launch_bounds__(256) void pack_kernel(const T* __restrict__ Xs, const T* __restrict__ Xd,
                                                   int64_t ldx, int mc, int k, int kp,
                                                   const int64_t* __restrict__ thr, T* __restrict__ Ph,
                                                   T* __restrict__ Pz, T* __restrict__ Pl,
                                                   float* __restrict__ apart, int tpb) {
  constexpr int EPG = 16 / (int)sizeof(T);
  constexpr int NG = kTokBlk / EPG;
  constexpr bool LO = TWO && sizeof(T) == 2;  // bf16 two-stream: dX = hi + lo
  constexpr int RS = kTokBlk + EPG;           // LDS row stride (elements)
  constexpr int NSLOT = LO ? 3 : 2;
  constexpr int STAGE = NSLOT * 256 * RS * (int)sizeof(T);
  constexpr int RED = 32 * 257 * (int)sizeof(float);
  __shared__ __attribute__((aligned(16))) uint8_t raw[STAGE > RED ? STAGE : RED];
  T* sh = (T*)raw;
  T* sz = sh + 256 * RS;
  T* sl = sz + 256 * RS;
  float* sa = (float*)raw;  // reused after the token loop

  const int cb0 = blockIdx.x * 256;
  const int tsb = blockIdx.y * tpb * kTokBlk;
  const int tr = threadIdx.x >> 3;        // token row inside a 32-token tile
  const int cg = (threadIdx.x & 7) * 32;  // first of 32 channels
  const T zero = Elem<T>::from_f32(0.f);
  float acc[32];
#pragma unroll
  for (int e = 0; e < 32; ++e) acc[e] = 0.f;

  for (int tt = 0; tt < tpb; ++tt) {
    const int tok0 = tsb + tt * kTokBlk;
    if (tok0 >= (int)rup(mc, 2 * kTokBlk)) break;  // uniform; zeros fill up the last pair of token blocks
    const int t = tok0 + tr;
    const bool tok_ok = t < mc;
    const int64_t th = tok_ok ? thr[t] : INT64_MAX;
#pragma unroll 8
    for (int e = 0; e < 32; ++e) {
      const int c = cb0 + cg + e;
      float d = 0.f;
      T vh = zero, vz = zero, vl = zero;
      if (tok_ok && c < k) {
        const T x = Xs[(int64_t)t * ldx + c];
        const int64_t key = ((int64_t)Elem<T>::mag(x) << 32) | c;
        const bool keep = key > th;
        vh = keep ? x : zero;
        if (TWO) {
          d = Elem<T>::to_f32(Xd[(int64_t)t * ldx + c]) - Elem<T>::to_f32(vh);
          vz = Elem<T>::from_f32(d);
          if (LO) vl = Elem<T>::from_f32(d - Elem<T>::to_f32(vz));
        } else {
          vz = keep ? zero : x;
          d = Elem<T>::to_f32(vz);
        }
      }
      acc[e] += d * d;
      sh[(cg + e) * RS + tr] = vh;
      sz[(cg + e) * RS + tr] = vz;
      if (LO) sl[(cg + e) * RS + tr] = vl;
    }
    __syncthreads();
    const int c = cb0 + threadIdx.x;
    if (c < kp) {
      const int tb = tok0 / kTokBlk;
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        const int64_t off = (((int64_t)tb * NG + g) * kp + c) * EPG;
        *(uint4*)(Ph + off) = *(const uint4*)&sh[threadIdx.x * RS + g * EPG];
        *(uint4*)(Pz + off) = *(const uint4*)&sz[threadIdx.x * RS + g * EPG];
        if (LO) *(uint4*)(Pl + off) = *(const uint4*)&sl[threadIdx.x * RS + g * EPG];
      }
    }
    __syncthreads();
  }
  // per-channel sum of dX^2 over this block's tokens, fixed order
#pragma unroll
  for (int e = 0; e < 32; ++e) sa[tr * 257 + cg + e] = acc[e];
  __syncthreads();
  const int c = cb0 + threadIdx.x;
  if (apart && c < kp) {
    float s = 0.f;
    for (int r = 0; r < 32; ++r) s += sa[r * 257 + threadIdx.x];
    apart[(int64_t)blockIdx.y * kp + c] = s;
  }
}

// bf16 pack (16-byte aligned rows, k % 8 == 0).  Workgroup (x, y) covers
// channels [512x, 512x + 512) of token blocks [tpb y, tpb (y + 1)): wave w handles
// tokens 8w..8w+7 of every 32-token block, lane l channels 512x + 8l .. +7.
// Each lane loads its 8 x 8 tile with 16-byte reads, applies the threshold in
// registers and transposes it (tokens become the contiguous dimension): one
// 16-byte vector per channel, exactly the packed layout above.  A wave's
// vectors for one token block are 8 KB of contiguous output per operand;
// they pass through LDS so that every global store writes 1 KB contiguously
// (stored straight from registers, each store touched 64 cache lines).
__device__ inline uint32_t lo_pair(uint32_t a, uint32_t b) { return (a & 0xffffu) | (b << 16); }
__device__ inline uint32_t hi_pair(uint32_t a, uint32_t b) { return (a >> 16) | (b & 0xffff0000u); }

template <bool TWO>
__global__ __launch_bounds__(256) void pack16_kernel(const uint16_t* __restrict__ Xs, const uint16_t* __restrict__ Xd,
                                                     int64_t ldx, int mc, int k, int kp,
                                                     const int64_t* __restrict__ thr, uint16_t* __restrict__ Ph,
                                                     uint16_t* __restrict__ Pz, uint16_t* __restrict__ Pl,
                                                     float* __restrict__ apart, int tpb) {
  __shared__ float red[4][512];
  __shared__ u32x4 stg[4][576];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int c0 = blockIdx.x * 512 + 8 * lane;
  const bool cv = c0 < k;   // all 8 channels valid (k % 8 == 0) or none
  float acc[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) acc[j] = 0.f;
  for (int tt = 0; tt < tpb; ++tt) {
    const int tb = blockIdx.y * tpb + tt;
    if (tb * kTokBlk >= (int)rup(mc, 2 * kTokBlk)) break;  // uniform; zeros fill up the last pair of token blocks
    const int tbase = tb * kTokBlk + 8 * wave;
    u32x4 xs[8], xd[8];
    int64_t th[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int t = tbase + e;
      const bool ok = cv && t < mc;
      const int64_t off = ok ? (int64_t)t * ldx + c0 : 0;
      xs[e] = *(const u32x4*)(Xs + off);
      if (TWO) xd[e] = *(const u32x4*)(Xd + off);
      if (!ok) xs[e] = u32x4{0u, 0u, 0u, 0u};
      if (TWO && !ok) xd[e] = u32x4{0u, 0u, 0u, 0u};
      th[e] = t < mc ? thr[t] : INT64_MAX;
    }
    u32x4 oh[8], oz[8], ol[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
#pragma unroll
      for (int w2 = 0; w2 < 4; ++w2) {
        uint32_t hv[2], zv[2], lv[2];
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) {
          const uint32_t x = (xs[e][w2] >> (16 * hf)) & 0xffffu;
          const int64_t key = ((int64_t)(x & 0x7fffu) << 32) | (int64_t)(c0 + 2 * w2 + hf);
          const bool keep = key > th[e];
          const uint32_t vh = keep ? x : 0u;
          float d;
          if (TWO) {
            d = bf16_bits_to_f32((uint16_t)((xd[e][w2] >> (16 * hf)) & 0xffffu)) - bf16_bits_to_f32((uint16_t)vh);
            const uint16_t vz = f32_to_bf16_bits(d);
            zv[hf] = vz;
            lv[hf] = f32_to_bf16_bits(d - bf16_bits_to_f32(vz));
          } else {
            zv[hf] = keep ? 0u : x;
            d = bf16_bits_to_f32((uint16_t)zv[hf]);
            lv[hf] = 0u;
          }
          hv[hf] = vh;
          acc[2 * w2 + hf] = fmaf(d, d, acc[2 * w2 + hf]);
        }
        oh[e][w2] = hv[0] | (hv[1] << 16);
        oz[e][w2] = zv[0] | (zv[1] << 16);
        ol[e][w2] = lv[0] | (lv[1] << 16);
      }
    }
    {
      // the wave's output for this token block is 512 contiguous 16-byte
      // chunks per operand (chunk 8 lane + j); staged through LDS (skewed by
      // one chunk per lane) so that each global store writes 1 KB contiguously
      u32x4* sw = stg[wave];
      const int64_t wbase = ((int64_t)(tb * (kTokBlk / 8) + wave) * kp + blockIdx.x * 512) * 8;
      auto put = [&](uint16_t* P, const u32x4 (&o)[8]) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const int w2 = j >> 1;
          u32x4 v;
#pragma unroll
          for (int p = 0; p < 4; ++p)
            v[p] = (j & 1) ? hi_pair(o[2 * p][w2], o[2 * p + 1][w2]) : lo_pair(o[2 * p][w2], o[2 * p + 1][w2]);
          sw[9 * lane + j] = v;
        }
#pragma unroll
        for (int jj = 0; jj < 8; ++jj) {
          const int q = 64 * jj + lane;
          const u32x4 v = sw[q + (q >> 3)];
          if (blockIdx.x * 512 + 8 * (q >> 3) < kp) *(u32x4*)(P + wbase + 8 * q) = v;
        }
      };
      put(Ph, oh);
      put(Pz, oz);
      if (TWO) put(Pl, ol);
    }
  }
  // per-channel sum of dX^2 over this workgroup's tokens, fixed order
#pragma unroll
  for (int j = 0; j < 8; ++j) red[wave][8 * lane + j] = acc[j];
  __syncthreads();
  if (apart)
    for (int i = threadIdx.x; i < 512; i += 256) {
      const int c = blockIdx.x * 512 + i;
      if (c < kp) apart[(int64_t)blockIdx.y * kp + c] = (red[0][i] + red[1][i]) + (red[2][i] + red[3][i]);
    }
}

// a[c] += the sum of the per-block partials of channel c, in a fixed order:
// eight strided running sums (partials g, g + 8, ...), then the eight in
// order.  A workgroup takes 32 channels, so every thread has only nblk / 8
// independent loads in flight instead of nblk sequential ones.
__global__ __launch_bounds__(256) void a_reduce_kernel(const float* __restrict__ apart, int nblk, int kp, int k,
                                                       float* __restrict__ a) {
  __shared__ float part[8][33];
  const int l = threadIdx.x & 31, g = threadIdx.x >> 5;
  const int c = blockIdx.x * 32 + l;
  float s = 0.f;
  if (c < k) {
#pragma unroll 8
    for (int b = g; b < nblk; b += 8) s += apart[(int64_t)b * kp + c];
  }
  part[g][l] = s;
  __syncthreads();
  if (g == 0 && c < k) {
    float v = 0.f;
#pragma unroll
    for (int h = 0; h < 8; ++h) v += part[h][l];
    a[c] += v;
  }
}

// ---------------------------------------------------------------------------
// gram: C = [Xh ; Z] Xh^T restricted to the tiles the method needs.
// 256 x 256 output tiles: H tiles (I, J) with I <= J (the upper triangle,
// added in place with coalesced writes; mirror_lower_kernel copies it to the
// lower triangle once per call) and G tiles (I, J) for every I, J.  H and G
// together cost 1.5 k^2 m multiply-adds (H's lower triangle is never
// computed, except inside the T diagonal tiles).
// ---------------------------------------------------------------------------
constexpr int GT = 256;  // gram tile edge (channels)

template <typename T>
struct GramArgs {
  const T* Ph;  // packed Xh
  const T* Pz;  // packed dX (single stream) or its high part (two streams)
  const T* Pl;  // packed low part of dX (two bf16 streams), else NULL
  int kp, k, nt;     // padded channels, channels, kp / 256
  int nh, ntiles;    // H tiles (0 when H is not wanted) and H + G tiles
  int g_full;        // G tiles: all nt x nt (1) or the upper triangle I <= J (0)
  int mixed;         // two bf16 streams: G tiles cost twice an H tile and come first
  int nsplit, nseg;  // the last nsplit tiles of the order are split into nseg token segments
  int seg_len, ntb;  // token blocks per segment, in all
  int piece;         // token blocks that one set of accumulators sums up
  float* run;        // [whole tiles][256 * 256]: sums of their pieces so far, or NULL
  float* H;
  int64_t ldh;
  float* G;
  int64_t ldg;
  float* part;  // [nseg][nsplit][256 * 256]
  int vec4;     // k, ldh, ldg multiples of 4 and H, G 16-byte aligned: 16-byte reduction path
};

// Tiles are numbered H first, then G.  H tiles cover the upper triangle of H
// (row block I <= column block J; the lower triangle is mirrored once per
// call), G tiles all of G.  Within each kind, bands of 4 blocks
// are walked across, so neighbouring ids share operand tiles; the
// XCD remap below gives each XCD a contiguous id range (and so its own L2 set).
__device__ inline void gram_tile(int t, int nh, int nt, int g_full, int* isg, int* I, int* J) {
  constexpr int GB = 4;
  // H tiles, and G tiles when only G's upper triangle is wanted, walk the
  // upper triangle of nt x nt (I <= J) in bands of GB columns
  const bool tri = t < nh || !g_full;
  *isg = t < nh ? 0 : 1;
  if (t >= nh && tri) t -= nh;
  if (tri) {
    // enumerated as the lower triangle (bands of GB rows), then transposed
    int* const tmp = I;
    I = J;
    J = tmp;
    for (int b0 = 0; b0 < nt; b0 += GB) {
      const int b1 = min(nt, b0 + GB), h = b1 - b0;
      const int cnt = b0 * h + h * (h + 1) / 2;
      if (t < cnt) {
        if (t < b0 * h) {
          *J = t / h;
          *I = b0 + t % h;
          return;
        }
        t -= b0 * h;
        for (int c = b0; c < b1; ++c) {
          const int nr = b1 - c;
          if (t < nr) {
            *J = c;
            *I = c + t;
            return;
          }
          t -= nr;
        }
      }
      t -= cnt;
    }
    *I = *J = 0;
    return;
  }
  t -= nh;
  const int b0 = (t / (GB * nt)) * GB;
  const int h = min(GB, nt - b0);
  const int r = t - b0 * nt;
  *J = r / h;
  *I = b0 + r % h;
}

typedef unsigned int v4u __attribute__((ext_vector_type(4)));

// fp32: two fragments per stage, four 16x16x4 fp32 MFMAs each; in fragment f, lane
// group l/16 holds the 4 tokens of group 4f + l/16 (the same tokens on both
// operands, so the sum runs over all 32 tokens of the stage)
__device__ inline f4 mma_f32(const v4u& a, const v4u& b, f4 c) {
  const float* x = (const float*)&a;
  const float* y = (const float*)&b;
  c = __builtin_amdgcn_mfma_f32_16x16x4f32(x[0], y[0], c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_16x16x4f32(x[1], y[1], c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_16x16x4f32(x[2], y[2], c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_16x16x4f32(x[3], y[3], c, 0, 0, 0);
  return c;
}

// Tile number o of the launch order: H then G, or (mixed) G then H.
template <typename T>
__device__ inline int gram_order(const GramArgs<T>& A, int o) {
  const int ng = A.ntiles - A.nh;
  return !A.mixed ? o : (o < ng ? A.nh + o : o - ng);
}

// Work of a workgroup: a whole tile (*part = -1 - its number), or token segment *seg
// of a split tile whose partial is number *part.  Each XCD takes a contiguous range of the
// whole tiles (of the whole G tiles and of the whole H tiles when mixed: an XCD
// that held only the dearer kind would finish last; neighbouring tiles share
// operand panels in that XCD's L2), then one of the segments, segment by segment.
template <typename T>
__device__ inline bool gram_unit(const GramArgs<T>& A, int* tile, int* seg, int* part) {
  const int x = blockIdx.x % 8;
  int y = blockIdx.x / 8;
  const int nfull = A.ntiles - A.nsplit;
  const int n1 = A.mixed ? min(A.ntiles - A.nh, nfull) : nfull, n2 = nfull - n1, n3 = A.nsplit * A.nseg;
  const int p1 = (n1 + 7) / 8, p2 = (n2 + 7) / 8, p3 = (n3 + 7) / 8;
  *seg = 0;
  if (y < p1) {
    *part = -1 - (x * p1 + y);
    *tile = gram_order(A, x * p1 + y);
    return x * p1 + y < n1;
  }
  y -= p1;
  if (y < p2) {
    *part = -1 - (n1 + x * p2 + y);
    *tile = gram_order(A, n1 + x * p2 + y);
    return x * p2 + y < n2;
  }
  y -= p2;
  const int v = x * p3 + y;
  if (y >= p3 || v >= n3) return false;
  *seg = v / A.nsplit;
  *part = v;
  *tile = gram_order(A, nfull + v % A.nsplit);
  return true;
}

// End of a piece in both Gram kernels: the tile's accumulators to the partial
// tile of its segment (stored first, then added to), or added to H or G; of a whole
// tile with several pieces (`run`) to its running sum, which joins H or G with the
// last piece, so that H and G are rounded once per call.  The running sum is kept
// as the lanes hold it, 1 KB per access.  The
// products run with the tile's columns (J) as the MFMA's rows, so that a lane
// holds four consecutive entries of one row: accumulator element r of block (a,
// b) is row 64 wj + 16 b + lane % 16, column 128 wi + 16 a + 4 (lane / 16) + r.
// Sixteen 16-byte reads per lane are in flight at a time, with no LDS and no
// barrier (adding a piece to H or G at k = 4096: 44 us staged through LDS, 25 so).
template <typename T>
__device__ inline void gram_store(const GramArgs<T>& A, int isg, int I, int J, int part, bool first, bool last,
                                  f4 (&acc)[8][4]) {
  // opaque, so that the addresses of a piece's stores are not kept in registers
  // through the main loop
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  if (part < 0 && A.run && !(first && last)) {  // uniform
    f4* const r = (f4*)(A.run + (int64_t)(-1 - part) * GT * GT) + tid;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      if (!first) {
        f4 c[8];
#pragma unroll
        for (int a = 0; a < 8; ++a) c[a] = r[(8 * b + a) * 512];
#pragma unroll
        for (int a = 0; a < 8; ++a) acc[a][b] = c[a] + acc[a][b];
      }
      if (!last)
#pragma unroll
        for (int a = 0; a < 8; ++a) r[(8 * b + a) * 512] = acc[a][b];
      __builtin_amdgcn_sched_barrier(0);  // 8 reads at a time, for the registers
    }
    if (!last) return;
  }
  const int lane = tid & 63, wave = tid >> 6;
  const int r0 = (wave & 3) * 64 + (lane & 15), c0 = (wave >> 2) * 128 + 4 * (lane >> 4);
  float* base;  // of the tile
  int64_t ld;
  int rows = GT, cols = GT;
  if (part >= 0) {
    base = A.part + (int64_t)part * GT * GT;
    ld = GT;
  } else {
    ld = isg ? A.ldg : A.ldh;
    base = (isg ? A.G : A.H) + (int64_t)I * GT * ld + (int64_t)J * GT;
    rows = min(GT, A.k - I * GT);
    cols = min(GT, A.k - J * GT);
    first = false;
  }
  if (part >= 0 || A.vec4) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      float4 c[2][8];
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int a = 0; a < 8; ++a) {
          const int row = r0 + 32 * h + 16 * b, col = c0 + 16 * a;
          c[b][a] = make_float4(0.f, 0.f, 0.f, 0.f);
          if (!first && row < rows && col < cols) c[b][a] = *(const float4*)(base + row * ld + col);
        }
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int a = 0; a < 8; ++a) {
          const int row = r0 + 32 * h + 16 * b, col = c0 + 16 * a;
          const f4 v = acc[a][2 * h + b];
          if (row < rows && col < cols)
            *(float4*)(base + row * ld + col) =
                make_float4(c[b][a].x + v[0], c[b][a].y + v[1], c[b][a].z + v[2], c[b][a].w + v[3]);
        }
    }
    return;
  }
#pragma unroll
  for (int b = 0; b < 4; ++b)
#pragma unroll
    for (int a = 0; a < 8; ++a)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = r0 + 16 * b, col = c0 + 16 * a + r;
        if (row < rows && col < cols) base[row * ld + col] += acc[a][b][r];
      }
}

// fp32 inputs.  512 threads = 8 waves in a 2 x 4 grid; each wave owns 128 columns x
// 64 rows of the tile (8 x 4 accumulator blocks of 16 x 16).  Operand tiles
// stream through two LDS stages (one 32-token block each, 64 KB) filled by
// direct global->LDS loads (each lane moves 16 bytes, a wave 1 KB), one stage
// ahead.  LDS layout of one operand tile: [group][256 rows][16 bytes], identical
// to the packed global layout.
constexpr int kGram32Stage = 2 * GT * kTokBlk * 4;
__global__ __launch_bounds__(512) void gram_f32_kernel(GramArgs<float> A) {
  constexpr int NG = kTokBlk / 4;
  constexpr int CHUNKS = GT * kTokBlk * 4 / 16;  // 16-byte chunks per operand tile
  constexpr int DPW = 2 * CHUNKS / 64 / 8;       // wave-wide loads per wave per stage
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
  int seg, part, tile, isg, I, J;
  if (!gram_unit(A, &tile, &seg, &part)) return;
  gram_tile(tile, A.nh, A.nt, A.g_full, &isg, &I, &J);
  const int tb0 = seg * A.seg_len;
  const int tb1 = part < 0 ? A.ntb : min(A.ntb, tb0 + A.seg_len);
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int wi = wave >> 2, wj = wave & 3;

  // this lane's share of every stage: DPW chunks, each in its operand tile
  const int64_t tbs = (int64_t)NG * A.kp * 16;  // bytes per token block in a packed operand
  const uint8_t* src[DPW];
  uint32_t ldso[DPW];  // wave-uniform LDS offset of each load within a stage
#pragma unroll
  for (int j = 0; j < DPW; ++j) {
    const int c0 = (wave * DPW + j) * 64;  // first chunk of this wave-wide load
    const int op = c0 / CHUNKS, c = c0 % CHUNKS + lane;
    const float* base = op == 0 || !isg ? A.Ph : A.Pz;
    const int blk = op == 0 ? J : I;
    src[j] = (const uint8_t*)base + ((int64_t)(c / GT) * A.kp + (int64_t)blk * GT + c % GT) * 16;
    ldso[j] = (uint32_t)(op * CHUNKS + c0 % CHUNKS) * 16;
  }
  auto issue = [&](int t) {
    uint8_t* stage = smem + ((t - tb0) & 1) * kGram32Stage;
#pragma unroll
    for (int j = 0; j < DPW; ++j)
      __builtin_amdgcn_global_load_lds((const void*)(src[j] + (int64_t)t * tbs),
                                       (__attribute__((address_space(3))) void*)(stage + ldso[j]), 16, 0, 0);
  };
  int p0 = tb0;
  do {  // pieces; an empty segment stores its zeros
    const int p1 = min(tb1, p0 + A.piece);
    f4 acc[8][4];
#pragma unroll
    for (int a = 0; a < 8; ++a)
#pragma unroll
      for (int b = 0; b < 4; ++b) acc[a][b] = f4{0.f, 0.f, 0.f, 0.f};
    if (p0 < p1) issue(p0);
    for (int t = p0; t < p1; ++t) {
      pp::wait_vm<0>();
      pp::lds_barrier();  // every wave's part of stage t has landed; stage t-1 is free
      if (t + 1 < p1) issue(t + 1);
      const v4u* l_ = (const v4u*)(smem + ((t - tb0) & 1) * kGram32Stage);
#pragma unroll
      for (int f = 0; f < 2; ++f) {
        const int fo = (f * 4 + (lane >> 4)) * GT + (lane & 15);
        v4u bf[4];
#pragma unroll
        for (int b = 0; b < 4; ++b) bf[b] = l_[CHUNKS + fo + wj * 64 + b * 16];
#pragma unroll
        for (int h2 = 0; h2 < 2; ++h2) {
          v4u af[4];
#pragma unroll
          for (int a = 0; a < 4; ++a) af[a] = l_[fo + wi * 128 + (4 * h2 + a) * 16];
#pragma unroll
          for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int b = 0; b < 4; ++b) acc[4 * h2 + a][b] = mma_f32(af[a], bf[b], acc[4 * h2 + a][b]);
        }
      }
    }
#pragma unroll
    for (int a = 0; a < 8; ++a)
#pragma unroll
      for (int b = 0; b < 4; ++b) asm volatile("s_nop 1" : "+v"(acc[a][b]));  // the last products have been written
    gram_store(A, isg, I, J, part, p0 == tb0, p1 >= tb1, acc);
    pp::lds_barrier();  // every wave is done with the stages
    p0 = p1;
  } while (p0 < tb1);
}

// bf16 inputs: the loop of pingpong.h over stages of 64 tokens (two token blocks;
// the packing fills up the last pair with zeros).  The part of a wave, 128
// columns x 64 rows, is split in halves of 64 columns and 32 rows; a unit of LDS is [token block][group]
// [128 channels][16 bytes], filled from the packed operands in 1 KB pieces, and a
// fragment read is linear in it (no bank conflicts).  Two streams: dX = hi + lo,
// and a G tile takes both in turn for every 64 tokens (twice an H tile's stages).
// Bound: MFMA issue and the clock under that load.  Measured, whole calls: 2 x 65536
// tokens at k = 4096 5.16 -> 4.16 ms; 2 x 8192, two streams, k = 11008 7.42 -> 5.18 ms;
// one launch of 131072 at k = 28672 166 -> 140 ms (the form before had all eight waves in
// step on a ring of 32-token stages, and gave four XCDs the H tiles and four the G tiles).
constexpr int kGram16Unit = 128 * 128;  // bytes: 128 channels x 64 tokens
constexpr size_t kGram16Lds = (size_t)8 * kGram16Unit;
__global__ __launch_bounds__(512) void gram_bf16_kernel(GramArgs<uint16_t> A) {
  constexpr int NG = kTokBlk / 8;
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];  // [stage parity][columns 0, 1, rows 0, 1]
  int seg, part, tile, isg, I, J;
  if (!gram_unit(A, &tile, &seg, &part)) return;
  gram_tile(tile, A.nh, A.nt, A.g_full, &isg, &I, &J);
  const int tb0 = seg * A.seg_len;  // even
  const int ntb = (A.ntb + 1) / 2 * 2, tb1 = part < 0 ? ntb : min(ntb, tb0 + A.seg_len);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wi = wave >> 2, wj = wave & 3;
  const int64_t tbs = (int64_t)NG * A.kp * 16;  // bytes per token block in a packed operand
  const int sh = isg && A.Pl ? 1 : 0;           // two streams: hi and lo stages in turn
  const int64_t lo_off = sh ? (const uint8_t*)A.Pl - (const uint8_t*)A.Pz : 0;
  // Loads: wave w fills plane w of a unit (token block w / 4, group w % 4), 64 unit
  // rows per load; unit row u is channel 128 (u / 64) + 64 h + u % 64 of the column tile
  // J for half h, 64 (u / 32) + 32 h + u % 32 of the row tile I.  Everything but the lane's own
  // 16 bytes is wave-uniform.
  const int uw = __builtin_amdgcn_readfirstlane(wave);
  const int64_t plane = (uw >> 2) * tbs + (int64_t)(uw & 3) * A.kp * 16;
  const uint8_t* const ua = (const uint8_t*)A.Ph + plane + (int64_t)J * GT * 16;
  const uint8_t* const ub = (const uint8_t*)(isg ? A.Pz : A.Ph) + plane + (int64_t)I * GT * 16;
  const uint32_t la = lane * 16, lb = (64 * (lane >> 5) + (lane & 31)) * 16;
  const uint32_t fa = (uint32_t)((lane >> 4) * 2048 + (wi * 64 + (lane & 15)) * 16);
  const uint32_t fb = (uint32_t)((lane >> 4) * 2048 + (wj * 32 + (lane & 15)) * 16);
  auto read_a = [&](int par, int h, u32x4 (&F)[2][4]) {
    const uint8_t* p = smem + (par * 4 + h) * kGram16Unit + fa;
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
      for (int a = 0; a < 4; ++a) F[s2][a] = *(const u32x4*)(p + s2 * 8192 + a * 256);
  };
  auto read_b = [&](int par, int h, u32x4 (&F)[2][2]) {
    const uint8_t* p = smem + (par * 4 + 2 + h) * kGram16Unit + fb;
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
      for (int b = 0; b < 2; ++b) F[s2][b] = *(const u32x4*)(p + s2 * 8192 + b * 256);
  };
  int p0 = tb0;
  do {  // pieces; an empty segment stores its zeros
    const int p1 = min(tb1, p0 + A.piece);
    f4 acc[8][4];
#pragma unroll
    for (int a = 0; a < 8; ++a)
#pragma unroll
      for (int b = 0; b < 4; ++b) acc[a][b] = f4{0.f, 0.f, 0.f, 0.f};
    if (p0 < p1) {  // uniform
      const int nst = (p1 - p0) / 2 << sh;
      const int64_t base = p0 * tbs;
      auto issue = [&](int op, int st, int par) {
        const int sc = min(st, nst - 1);
        const int64_t off = base + (int64_t)(sc >> sh) * 2 * tbs + (op >= 2 && (sc & sh) ? lo_off : 0);
        const uint8_t* u = op < 2 ? ua + off + op * 1024 : ub + off + (op - 2) * 512;
        uint8_t* dst = smem + (par * 4 + op) * kGram16Unit + uw * 2048;
#pragma unroll
        for (int j = 0; j < 2; ++j)
          __builtin_amdgcn_global_load_lds((const void*)(u + j * 2048 + (op < 2 ? la : lb)),
                                           (__attribute__((address_space(3))) void*)(dst + j * 1024), 16, 0, 0);
      };
      pp::pp_loop<4, 2, 2>(nst, acc, issue, read_a, read_b);
    }
    gram_store(A, isg, I, J, part, p0 == tb0, p1 >= tb1, acc);
    pp::lds_barrier();  // every wave is done with the units
    p0 = p1;
  } while (p0 < tb1);
}

// Fixed-order sum of the per-segment partial tiles into H (upper tiles) and
// G.  Block (tile, q) takes the 64 x 64 sub-block q; its rows are added with
// coalesced accesses.
template <typename T>
__global__ __launch_bounds__(256) void gram_reduce_kernel(GramArgs<T> A) {
  int isg, I, J;
  gram_tile(gram_order(A, A.ntiles - A.nsplit + (int)blockIdx.x), A.nh, A.nt, A.g_full, &isg, &I, &J);
  const int sr = (blockIdx.y >> 2) * 64, sc = (blockIdx.y & 3) * 64;
  const int64_t stride = (int64_t)A.nsplit * GT * GT;
  const float* p0 = A.part + (int64_t)blockIdx.x * GT * GT;
  float* C = isg ? A.G : A.H;
  const int64_t ldc = isg ? A.ldg : A.ldh;
  if (A.vec4) {
    // 16-byte path (k and the leading dimensions multiples of 4): thread
    // (r, c4) sums rows r, r + 16, r + 32, r + 48 at columns c4 .. c4 + 3, with
    // every segment's loads issued before the sums need them
    const int c4 = (threadIdx.x & 15) * 4, r0 = threadIdx.x >> 4;
    float4 sum[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) sum[p] = make_float4(0.f, 0.f, 0.f, 0.f);
    // (eight segments at a time; those past the last re-read it, and are not added)
    for (int s0 = 0; s0 < A.nseg; s0 += 8) {
      float4 v[8][4];
#pragma unroll
      for (int sg = 0; sg < 8; ++sg)
#pragma unroll
        for (int p = 0; p < 4; ++p)
          v[sg][p] = *(const float4*)(p0 + min(s0 + sg, A.nseg - 1) * stride + (sr + r0 + 16 * p) * GT + sc + c4);
#pragma unroll
      for (int sg = 0; sg < 8; ++sg)
        if (s0 + sg < A.nseg) {
#pragma unroll
          for (int p = 0; p < 4; ++p) {
            sum[p].x += v[sg][p].x;
            sum[p].y += v[sg][p].y;
            sum[p].z += v[sg][p].z;
            sum[p].w += v[sg][p].w;
          }
        }
    }
    const int col = J * GT + sc + c4;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      const int rr = r0 + 16 * p, row = I * GT + sr + rr;
      if (row < A.k && col < A.k) {
        float4* cp = (float4*)(C + (int64_t)row * ldc + col);
        float4 c = *cp;
        c.x += sum[p].x;
        c.y += sum[p].y;
        c.z += sum[p].z;
        c.w += sum[p].w;
        *cp = c;
      }
    }
    return;
  }
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  for (int rr = ty; rr < 64; rr += 4) {
    const int e = (sr + rr) * GT + sc + tx;
    float s = 0.f;
    for (int sg = 0; sg < A.nseg; ++sg) s += p0[sg * stride + e];
    const int row = I * GT + sr + rr, col = J * GT + sc + tx;
    if (row < A.k && col < A.k) C[(int64_t)row * ldc + col] += s;
  }
}

// H's lower triangle from its upper one: block (bi, bj), bi >= bj, of 64 x 64
// takes the transpose of block (bj, bi) through LDS (coalesced reads and
// writes); inside a diagonal block only the entries below the diagonal are
// written.
__global__ __launch_bounds__(256) void mirror_lower_kernel(float* __restrict__ H, int64_t ldh, int k) {
  __shared__ float tr[64][65];
  int bi, bj;
  tri_pair(blockIdx.x, &bi, &bj);
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  for (int rr = ty; rr < 64; rr += 4) {  // source rows bj*64 + rr, columns bi*64 + tx
    const int r = bj * 64 + rr, c = bi * 64 + tx;
    tr[rr][tx] = (r < k && c < k) ? H[(int64_t)r * ldh + c] : 0.f;
  }
  __syncthreads();
  for (int rr = ty; rr < 64; rr += 4) {  // target rows bi*64 + rr, columns bj*64 + tx
    const int r = bi * 64 + rr, c = bj * 64 + tx;
    if (r < k && c < k && r > c) H[(int64_t)r * ldh + c] = tr[tx][rr];
  }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
// Tokens per stage-1 chunk: the packed operands of a chunk take up to
// 10 bytes per token and padded channel of workspace; up to 40 GB of them
// (of the 288 GB of HBM), so that the calibration sets of the benchmark
// shapes go through one Gram launch (at k = 28672, one chunk of 131072 tokens
// measured 3.3 ms faster per layer than three of 52224 + 52224 + 26624: one
// partly filled last round of tiles and one pass over H and G instead of
// three).
int64_t hessian_chunk_tokens(int64_t m, int64_t k) {
  const int64_t kp = rup(k, GT);
  int64_t ch = (int64_t)40e9 / (kp * 8);
  ch = ch < 4096 ? 4096 : ch;
  ch = ch > 131072 ? 131072 : ch;
  ch = ch / 256 * 256;
  return m < ch ? (m < 1 ? 1 : m) : ch;
}

// Token segments (up to eight) that fill the chip's rounds of 256 tiles when every
// tile of a launch is split: a full tile at 4.5 TFLOP/s per CU, the sum of s partial
// tiles (s + 2) * 256 KB at 4 TB/s.
static int even_segments(int64_t ntiles, int64_t ch) {
  const double t_tile = 2.0 * GT * GT * (double)ch / 4.5e12, t_sum = (double)GT * GT * 4.0 / 4e12;
  int best = 1;
  double best_cost = 1e30;
  for (int s = 1; s <= 8; ++s) {
    const double cost = (double)cdiv(ntiles * s, 256) / s * t_tile + (s > 1 ? (double)ntiles * (s + 2) * t_sum : 0.0);
    if (cost < best_cost * (1.0 - 1e-9)) {
      best_cost = cost;
      best = s;
    }
  }
  return best;
}

// How a launch of nh H tiles and ng G tiles, `ch` tokens each, is divided.
// Split tiles.  Whole rounds of 256 tiles (one per CU) run unsplit; the rest of the
// tiles, or all of them when there is less than one round, are split so that their
// segments fill the chip once more, at the price of summing the partial tiles
// afterwards.  Model, per tile: 2 * 256^2 * ch flop at 5.5 TFLOP/s (bf16) or 0.5
// (fp32) per CU, 8 us of start and epilogue per round; the sum of s partials reads s
// tiles and reads and writes the output, (s + 2) * 256 KB at about 4 TB/s, and costs a
// launch (5 us).  `cost2`: two bf16 streams, where a G tile costs twice an H tile; the
// launch then ends with the H tiles, and the split ones are the last of them.  At k =
// 4096, 65536 tokens (272 tiles) 16 tiles in 16 segments each: 1.06 rounds, where
// splitting all tiles in 8 took 1.125 rounds and 310 us of sums per call.
// Up to k = 1024 every form of a launch (H, G, both, all of G) fits one round, and the
// segments are those of the largest, so that G has the same bits in all of them.
// Pieces.  One set of accumulators sums up at most `piece` token blocks; the sums of a
// longer run are added up tile by tile in pieces.  The relative error of the
// 32-bit sums grows with the square root of the accumulation steps (32 tokens each in
// bf16, 4 in fp32).  A piece is no longer than the segments of a launch split evenly
// throughout (even_segments), which decides up to k = 9216 (65536 tokens at k = 9216: 9.0e-7 of
// H).  Above, where that is one segment, 24576 tokens up to k = 20480 and no bound
// beyond: a piece costs a pass over the output, whose rows lie further apart the
// larger k is, and takes the workgroups of an XCD out of step (65536 tokens, in one
// piece, pieces of 24576 and of 16384: k = 11008 12.20, 12.33, 12.45 ms with errors of 1.4e-6,
// 1.1e-6, 8.8e-7; k = 20480 39.1, 40.2, 40.8 ms; k = 24576 55.3, 57.0, 58.1 ms).
struct GramPlan {
  int nsplit, nseg;  // the last nsplit tiles in nseg segments each
  int piece;         // token blocks
  bool run;          // whole tiles keep running sums
};
static GramPlan gram_plan(int64_t T, int64_t nh, int64_t ng, bool cost2, bool bf16, int64_t ch) {
  const int64_t ntiles = nh + ng, nb = rup(cdiv(ch, kTokBlk), 2), k = T * GT;
  const bool small = T <= 4;
  int64_t rest;     // tiles to split
  double each = 1;  // what one of them costs, in H tiles
  if (small) {
    rest = T * T + T * (T + 1) / 2;
    if (cost2) each = 2;
  } else {
    rest = cost2 && nh > 0 ? std::min((ntiles + ng) % 256, ntiles) : ntiles % 256;
    if (cost2 && rest > nh) each = (double)(rest + rest - nh) / (double)rest;
  }
  int best = 1;
  if (rest > 0) {
    const double t_tile = 2.0 * GT * GT * (double)ch / (bf16 ? 5.5e12 : 0.5e12) * each;
    const double t_sum = (double)GT * GT * 4.0 / 4e12;
    double best_cost = 1e30;
    for (int s = 1; s <= 32; ++s) {
      if (s > 1 && rest * s > 1024) break;
      const double rounds = (double)cdiv(rest * s, 256);
      const double cost = rounds / s * t_tile + rounds * 8e-6 + (s > 1 ? 5e-6 + (double)rest * (s + 2) * t_sum : 0.0);
      if (cost < best_cost * (1.0 - 1e-9)) {
        best_cost = cost;
        best = s;
      }
    }
  }
  GramPlan p;
  p.nsplit = best > 1 ? (int)(small ? ntiles : rest) : 0;
  p.nseg = best;
  const int even = even_segments(small ? T * (T + 1) / 2 : ntiles, ch);
  const int64_t t = k <= 9216 ? 16384 : k <= 20480 ? 24576 : 131072;
  const int64_t most = (bf16 ? t : k <= 9216 ? 4096 : 8192) / kTokBlk;
  p.piece = (int)std::min(most, rup(cdiv(nb, even), 2));
  p.run = even > 1 && p.piece < nb && p.nsplit < ntiles;
  return p;
}

// Diagonal of H in fp64 for act_order: hdiag[c] += sum_t Xh[t][c]^2, read
// from the packed operand.  Each square is exact in fp64; the sum runs in a
// fixed order (token slices in sequence), so the result is deterministic and
// within a few fp64 ulps of the exact value, which lets the channel order be
// decided identically on any implementation that sums in fp64.
template <typename T>
__global__ __launch_bounds__(256) void hdiag_part_kernel(const T* __restrict__ Ph, int kp, int ntb, int slice_len,
                                                         double* __restrict__ dpart) {
  constexpr int EPG = 16 / (int)sizeof(T);
  constexpr int NG = kTokBlk / EPG;
  const int c = blockIdx.x * 256 + threadIdx.x;
  const int tb0 = blockIdx.y * slice_len;
  const int tb1 = min(ntb, tb0 + slice_len);
  if (c >= kp) return;
  double s = 0.0;
  for (int tb = tb0; tb < tb1; ++tb)
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      const uint4 v = *(const uint4*)(Ph + (((int64_t)tb * NG + g) * kp + c) * EPG);
      const T* e = (const T*)&v;
#pragma unroll
      for (int i = 0; i < EPG; ++i) {
        const double x = (double)Elem<T>::to_f32(e[i]);
        s = fma(x, x, s);
      }
    }
  dpart[(int64_t)blockIdx.y * kp + c] = s;
}

__global__ void hdiag_reduce_kernel(const double* __restrict__ dpart, int nsl, int kp, int k,
                                    double* __restrict__ hdiag) {
  const int c = blockIdx.x * 256 + threadIdx.x;
  if (c >= k) return;
  double s = 0.0;
  for (int i = 0; i < nsl; ++i) s += dpart[(int64_t)i * kp + c];
  hdiag[c] += s;
}

__global__ void clear_flags_kernel(uint32_t* f) { f[threadIdx.x] = 0u; }

struct HessWs {
  uint32_t* flags;  // [0]: a non-finite input was met by the last call on this workspace
  int64_t* thr;
  uint8_t* Ph;
  uint8_t* Pz;
  uint8_t* Pl;
  float* apart;
  float* part;  // partial tiles, then the running sums of whole tiles
  double* dpart;
  size_t bytes;
};

// token slices of the fp64 diagonal (act_order): at most kDiagSlices, and at
// most 2^21 partial sums in all
constexpr int kDiagSlices = 64;
static int diag_slices(int64_t kp, int ntb) {
  int64_t n = (int64_t(1) << 21) / kp;
  if (n > kDiagSlices) n = kDiagSlices;
  if (n > ntb) n = ntb;
  return n < 1 ? 1 : (int)n;
}

// Token blocks per packing workgroup: eight, or fewer where that leaves CUs idle
// (2048 x 512 fp32 in 16 workgroups of eight 56 us; with one block each the whole layer is 60 us
// shorter).  fp32: no more than a workgroup per CU, whose 256 rows of 128 bytes
// per operand the vector cache barely holds (8192 x 2048, two streams: two blocks each
// 1577 us, eight 1467, four 1359).
static int pack_blocks(int64_t mc, int64_t kp, bool f32) {
  if (f32) return (int)std::min<int64_t>(8, cdiv(kp / 256 * cdiv(mc, kTokBlk), 256));
  const int64_t wg = kp / 256 * cdiv(mc, 256);
  return wg >= 512 ? 8 : wg >= 128 ? 2 : 1;
}
// partial sums of a: a row per workgroup row, at most 2^20 floats where those are
// more than one per 256 tokens (128 workgroups of 8 blocks at most, or 512 of 2)
constexpr int64_t kApartMin = int64_t(1) << 20;

static HessWs carve_hessian(void* ws, int64_t m, int64_t k) {
  const int64_t ch = hessian_chunk_tokens(m, k);
  const int64_t kp = rup(k, GT);
  const int64_t tokp = rup(ch, 256);
  const int64_t T = kp / GT;
  // partial tiles and running sums: enough for every form (with and without H; all
  // of G, its upper triangle or none; one stream or two; either dtype).  Each form needs
  // no less for more tokens, so a workspace for m tokens serves any smaller m
  int64_t part_tiles = 0;
  for (int f = 0; f < 24; ++f) {
    const int64_t up = T * (T + 1) / 2, nh = f & 1 ? up : 0, ng = f / 8 == 0 ? 0 : f / 8 == 1 ? up : T * T;
    const GramPlan p = gram_plan(T, nh, ng, f & 2, f & 4, ch);
    part_tiles = std::max(part_tiles, (int64_t)p.nsplit * p.nseg + (p.run ? nh + ng - p.nsplit : 0));
  }
  Carver c(ws);
  HessWs h;
  h.flags = c.take<uint32_t>(64);
  h.thr = c.take<int64_t>(2 * tokp);  // sparse stream, then the dense stream's (checked only)
  h.Ph = c.take<uint8_t>((size_t)tokp * kp * 4);  // sized for fp32; bf16 uses half
  h.Pz = c.take<uint8_t>((size_t)tokp * kp * 4);
  h.Pl = c.take<uint8_t>((size_t)tokp * kp * 2);  // low part exists for bf16 only
  h.apart = c.take<float>((size_t)std::max((tokp / 256) * kp, kApartMin));
  h.part = c.take<float>(part_tiles > 0 ? (size_t)part_tiles * GT * GT : 1);
  h.dpart = c.take<double>((size_t)diag_slices(kp, kDiagSlices) * kp);
  h.bytes = c.off;
  return h;
}

size_t hessian_ws_bytes(int64_t m, int64_t k) { return carve_hessian(nullptr, m, k).bytes; }

duo_status hessian_status_run(const void* ws, hipStream_t s) {
  // the flags are the workspace's first slot whatever m and k were
  const uint32_t* flags = carve_hessian(const_cast<void*>(ws), 1, 1).flags;
  uint32_t f = 0;
  DUO_HIP_TRY(hipMemcpyAsync(&f, flags, sizeof(f), hipMemcpyDeviceToHost, s));
  DUO_HIP_TRY(hipStreamSynchronize(s));
  return f ? DUO_ERR_NONFINITE : DUO_OK;
}

template <typename T>
static duo_status launch_gram(const GramArgs<T>& A, hipStream_t s) {
  const int64_t nfull = A.ntiles - A.nsplit;
  const int64_t n1 = A.mixed ? std::min<int64_t>(A.ntiles - A.nh, nfull) : nfull;
  const dim3 grid((unsigned)(8 * (cdiv(n1, 8) + cdiv(nfull - n1, 8) + cdiv((int64_t)A.nsplit * A.nseg, 8))));
  if constexpr (sizeof(T) == 2) {
    if (duo_status st = set_max_lds((const void*)gram_bf16_kernel, kGram16Lds); st != DUO_OK) return st;
    hipLaunchKernelGGL(gram_bf16_kernel, grid, dim3(512), kGram16Lds, s, A);
  } else {
    if (duo_status st = set_max_lds((const void*)gram_f32_kernel, 2 * kGram32Stage); st != DUO_OK) return st;
    hipLaunchKernelGGL(gram_f32_kernel, grid, dim3(512), 2 * kGram32Stage, s, A);
  }
  DUO_LAUNCH_CHECK();
  return DUO_OK;
}

template <typename T>
static duo_status hessian_typed(const T* Xs, const T* Xd, int64_t m, int64_t k, int64_t ldx, int z, float* H,
                                int64_t ldh, float* G, int64_t ldg, int g_full, float* a, double* hdiag, void* ws,
                                bool want_h, hipStream_t s) {
  const bool want_g = G != nullptr;
  const bool two = Xd != nullptr && Xd != Xs;
  const bool lo = two && sizeof(T) == 2;
  const HessWs w = carve_hessian(ws, m, k);
  const int64_t ch = hessian_chunk_tokens(m, k);
  const int64_t kp = rup(k, GT);
  const int nt = (int)(kp / GT);
  const int nh_all = nt * (nt + 1) / 2;
  const int ng = want_g ? (g_full ? nt * nt : nh_all) : 0;
  const GramPlan plan = gram_plan(nt, want_h ? nh_all : 0, ng, lo, sizeof(T) == 2, ch);  // as the workspace was sized for
  hipLaunchKernelGGL(clear_flags_kernel, dim3(1), dim3(64), 0, s, w.flags);
  DUO_LAUNCH_CHECK();
  for (int64_t t0 = 0; t0 < m; t0 += ch) {
    const int mc = (int)(m - t0 < ch ? m - t0 : ch);
    const T* xs = Xs + t0 * ldx;
    const T* xd = two ? Xd + t0 * ldx : nullptr;
    duo_status st = launch_act_select<T>(xs, ldx, mc, (int)k, z, w.thr, w.flags, s);
    if (st != DUO_OK) return st;
    if (two) {  // the dense stream is checked too (its values enter G and a)
      st = launch_act_select<T>(xd, ldx, mc, (int)k, 0, w.thr + rup(ch, 256), w.flags, s);
      if (st != DUO_OK) return st;
    }
    const int tpb = pack_blocks(mc, kp, sizeof(T) == 4), prow = (int)cdiv(rup(mc, 2 * kTokBlk) / kTokBlk, tpb);
    dim3 pg((unsigned)(kp / 256), (unsigned)prow);
    if constexpr (sizeof(T) == 2) {
      if (bf16_vec_ok(xs, ldx, k) && (!two || bf16_vec_ok(xd, ldx, k))) {
        dim3 pg16((unsigned)cdiv(kp, 512), (unsigned)prow);
        if (two)
          hipLaunchKernelGGL(pack16_kernel<true>, pg16, dim3(256), 0, s, (const uint16_t*)xs, (const uint16_t*)xd,
                             ldx, mc, (int)k, (int)kp, w.thr, (uint16_t*)w.Ph, (uint16_t*)w.Pz, (uint16_t*)w.Pl,
                             want_g ? w.apart : nullptr, tpb);
        else
          hipLaunchKernelGGL(pack16_kernel<false>, pg16, dim3(256), 0, s, (const uint16_t*)xs, (const uint16_t*)xs,
                             ldx, mc, (int)k, (int)kp, w.thr, (uint16_t*)w.Ph, (uint16_t*)w.Pz, (uint16_t*)w.Pl,
                             want_g ? w.apart : nullptr, tpb);
        goto packed;
      }
    }
    if (two)
      hipLaunchKernelGGL((pack_kernel<T, true>), pg, dim3(256), 0, s, xs, xd, ldx, mc, (int)k, (int)kp, w.thr,
                         (T*)w.Ph, (T*)w.Pz, (T*)w.Pl, want_g ? w.apart : nullptr, tpb);
    else
      hipLaunchKernelGGL((pack_kernel<T, false>), pg, dim3(256), 0, s, xs, xs, ldx, mc, (int)k, (int)kp, w.thr,
                         (T*)w.Ph, (T*)w.Pz, (T*)w.Pl, want_g ? w.apart : nullptr, tpb);
  packed:
    DUO_LAUNCH_CHECK();
    if (hdiag) {
      const int ntb = (int)cdiv(mc, kTokBlk);
      const int nsl = diag_slices(kp, ntb);
      const int slen = (int)cdiv(ntb, nsl);
      hipLaunchKernelGGL(hdiag_part_kernel<T>, dim3((unsigned)(kp / 256), (unsigned)nsl), dim3(256), 0, s,
                         (const T*)w.Ph, (int)kp, ntb, slen, w.dpart);
      DUO_LAUNCH_CHECK();
      hipLaunchKernelGGL(hdiag_reduce_kernel, dim3((unsigned)cdiv(k, 256)), dim3(256), 0, s, (const double*)w.dpart,
                         nsl, (int)kp, (int)k, hdiag);
      DUO_LAUNCH_CHECK();
    }
    if (want_g) {
      hipLaunchKernelGGL(a_reduce_kernel, dim3((unsigned)cdiv(k, 32)), dim3(256), 0, s, w.apart, prow,
                         (int)kp, (int)k, a);
      DUO_LAUNCH_CHECK();
    }
    GramArgs<T> A;
    A.Ph = (const T*)w.Ph;
    A.Pz = (const T*)w.Pz;
    A.Pl = lo ? (const T*)w.Pl : nullptr;
    A.kp = (int)kp;
    A.k = (int)k;
    A.nt = nt;
    A.nh = want_h ? nh_all : 0;
    A.ntiles = A.nh + ng;
    A.g_full = g_full;
    A.piece = plan.piece;
    A.run = plan.run ? w.part + (int64_t)plan.nsplit * plan.nseg * GT * GT : nullptr;
    A.mixed = lo;
    A.nsplit = plan.nsplit;
    A.nseg = plan.nseg;
    A.ntb = (int)cdiv(mc, kTokBlk);
    A.seg_len = (int)rup(cdiv(A.ntb, A.nseg), 2);  // whole stages of 64 tokens (bf16)
    A.H = H;
    A.ldh = ldh;
    A.G = G;
    A.ldg = ldg;
    A.part = w.part;
    {
      auto al16 = [](const void* q) { return (reinterpret_cast<uintptr_t>(q) & 15) == 0; };
      A.vec4 = k % 4 == 0 && (!want_h || (ldh % 4 == 0 && al16(H))) && (!want_g || (ldg % 4 == 0 && al16(G)));
    }
    prof_begin(DUO_PROF_GRAM, s);
    st = launch_gram<T>(A, s);
    prof_end(DUO_PROF_GRAM, s);
    if (st != DUO_OK) return st;
    if (A.nsplit > 0) {
      hipLaunchKernelGGL(gram_reduce_kernel<T>, dim3(A.nsplit, (GT / 64) * (GT / 64)), dim3(256), 0, s, A);
      DUO_LAUNCH_CHECK();
    }
  }
  if (want_h) {
    const int64_t nb = cdiv(k, 64);
    hipLaunchKernelGGL(mirror_lower_kernel, dim3((unsigned)(nb * (nb + 1) / 2)), dim3(256), 0, s, H, ldh, (int)k);
    DUO_LAUNCH_CHECK();
  }
  return DUO_OK;
}

duo_status hessian_run(const void* Xs, const void* Xd, int32_t dtype, int64_t m, int64_t k, int64_t ldx, int z,
                       float* H, int64_t ldh, float* G, int64_t ldg, int g_full, float* a, double* hdiag, void* ws,
                       bool want_h, hipStream_t s) {
  if (dtype == DUO_BF16)
    return hessian_typed<uint16_t>((const uint16_t*)Xs, (const uint16_t*)Xd, m, k, ldx, z, H, ldh, G, ldg, g_full, a,
                                   hdiag, ws, want_h, s);
  return hessian_typed<float>((const float*)Xs, (const float*)Xd, m, k, ldx, z, H, ldh, G, ldg, g_full, a, hdiag, ws,
                              want_h, s);
}

duo_status act_mask_run(const void* X, int32_t dtype, int64_t m, int64_t k, int64_t ldx, int z, uint32_t* mask,
                        void* ws, hipStream_t s) {
  const HessWs w = carve_hessian(ws, m, k);
  const int64_t ch = hessian_chunk_tokens(m, k);
  const int64_t words = cdiv(k, 32);
  hipLaunchKernelGGL(clear_flags_kernel, dim3(1), dim3(64), 0, s, w.flags);
  DUO_LAUNCH_CHECK();
  for (int64_t t0 = 0; t0 < m; t0 += ch) {
    const int mc = (int)(m - t0 < ch ? m - t0 : ch);
    const int64_t n = mc * words;
    duo_status st;
    if (dtype == DUO_BF16) {
      const uint16_t* x = (const uint16_t*)X + t0 * ldx;
      st = launch_act_select<uint16_t>(x, ldx, mc, (int)k, z, w.thr, w.flags, s);
      if (st != DUO_OK) return st;
      hipLaunchKernelGGL(act_mask_kernel<uint16_t>, dim3((unsigned)cdiv(n, 256)), dim3(256), 0, s, x, ldx, mc,
                         (int)k, (const int64_t*)w.thr, mask + t0 * words);
    } else {
      const float* x = (const float*)X + t0 * ldx;
      st = launch_act_select<float>(x, ldx, mc, (int)k, z, w.thr, w.flags, s);
      if (st != DUO_OK) return st;
      hipLaunchKernelGGL(act_mask_kernel<float>, dim3((unsigned)cdiv(n, 256)), dim3(256), 0, s, x, ldx, mc, (int)k,
                         (const int64_t*)w.thr, mask + t0 * words);
    }
    DUO_LAUNCH_CHECK();
  }
  return DUO_OK;
}


}  // namespace duo
