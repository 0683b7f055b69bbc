// Decoder-block harness: the operations that carry the two activation streams
// of a LLaMA-style decoder block between the solver's groups (the multi-layer
// case of Sec. 4.2: the dense model sees X-tilde, the pruned model sees its
// own, sparsified input).  All activations are bf16 row-major token x feature
// arrays; arithmetic is fp32.
//
//   duo_rmsnorm       y = x / sqrt(mean(x^2) + eps)          (unit gain)
//   duo_act_sparsify  y = x with the per-token (|x|, channel) rule applied
//   duo_linear        Y = X W^T (+ R)       (bf16 MFMA tiles, fp32 accumulate)
//   duo_rope          rotary position embedding, rotate-half pairs (i, i + d/2)
//   duo_attention     causal softmax(Q K^T / sqrt(d)) V per sequence and head
//                     (two passes over the key blocks with bf16 MFMA: row
//                     maxima and sums, then the probabilities, rounded to bf16
//                     after normalisation, times V)
//   duo_silu_mul      y = SiLU(g) * u
#include <hip/hip_runtime.h>

#include <cmath>
#include <mutex>

#include "internal.h"
#include "pingpong.h"

using namespace duo;
using namespace duo::pp;

namespace {

__device__ inline float ld_bf16(const uint16_t* p) { return bf16_bits_to_f32(*p); }

// ---------------------------------------------------------------------------
// kernels
// ---------------------------------------------------------------------------

// One 256-thread workgroup per token.
__global__ __launch_bounds__(256) void rmsnorm_kernel(const uint16_t* __restrict__ X, int64_t ldx, int d, float eps,
                                                      uint16_t* __restrict__ Y, int64_t ldy) {
  __shared__ float red[4];
  const uint16_t* x = X + (int64_t)blockIdx.x * ldx;
  uint16_t* y = Y + (int64_t)blockIdx.x * ldy;
  float ss = 0.f;
  for (int c = threadIdx.x; c < d; c += 256) {
    const float v = ld_bf16(x + c);
    ss = fmaf(v, v, ss);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
  __syncthreads();
  const float tot = (red[0] + red[1]) + (red[2] + red[3]);
  const float inv = 1.0f / sqrtf(tot / (float)d + eps);
  for (int c = threadIdx.x; c < d; c += 256) y[c] = f32_to_bf16_bits(ld_bf16(x + c) * inv);
}

__global__ void act_apply_kernel(const uint16_t* __restrict__ X, int64_t ldx, int m, int k,
                                 const int64_t* __restrict__ thr, uint16_t* __restrict__ Y, int64_t ldy) {
  const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (id >= (int64_t)m * k) return;
  const int t = (int)(id / k), c = (int)(id % k);
  const uint16_t x = X[(int64_t)t * ldx + c];
  const int64_t key = ((int64_t)(x & 0x7fffu) << 32) | c;
  Y[(int64_t)t * ldy + c] = key > thr[t] ? x : (uint16_t)0;
}

// One workgroup per token: the half = head_dim / 2 rotation angles
// pos * theta^(-2i/head_dim) (pos = token % seq_len) and their cosines and
// sines are computed once in fp64 and shared by every head; each thread then
// rotates pairs (i, i + half) of the token's heads in fp32.
__global__ __launch_bounds__(256) void rope_kernel(uint16_t* __restrict__ X, int64_t ldx, int heads, int hd,
                                                   int seq_len, double theta) {
  __shared__ float cs[2][256];
  const int half = hd / 2;
  const int t = blockIdx.x;
  for (int i = threadIdx.x; i < half; i += 256) {
    const double ang = (double)(t % seq_len) * pow(theta, -2.0 * (double)i / (double)hd);
    double sd, cd;
    sincos(ang, &sd, &cd);
    cs[0][i] = (float)cd;
    cs[1][i] = (float)sd;
  }
  __syncthreads();
  uint16_t* row = X + (int64_t)t * ldx;
  for (int e = threadIdx.x; e < heads * half; e += 256) {
    const int h = e / half, i = e % half;
    uint16_t* p = row + (int64_t)h * hd;
    const float c = cs[0][i], s = cs[1][i];
    const float x1 = bf16_bits_to_f32(p[i]), x2 = bf16_bits_to_f32(p[i + half]);
    p[i] = f32_to_bf16_bits(x1 * c - x2 * s);
    p[i + half] = f32_to_bf16_bits(x2 * c + x1 * s);
  }
}

// 16-byte form of silu_mul_kernel (n, ld, ldy multiples of 8, aligned rows).
__global__ __launch_bounds__(256) void silu_mul8_kernel(const uint16_t* __restrict__ G, const uint16_t* __restrict__ U,
                                                        int64_t ld, int n, uint16_t* __restrict__ Y, int64_t ldy) {
  const int cpr = (n + 2047) / 2048;  // workgroups per token
  const int t = (int)(blockIdx.x / cpr);
  const int c0 = ((int)(blockIdx.x % cpr) * 256 + threadIdx.x) * 8;
  if (c0 >= n) return;
  const u32x4 g = *(const u32x4*)(G + (int64_t)t * ld + c0);
  const u32x4 u = *(const u32x4*)(U + (int64_t)t * ld + c0);
  u32x4 y;
#pragma unroll
  for (int h = 0; h < 4; ++h) {
    uint32_t o = 0;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const float gv = bf16_bits_to_f32((uint16_t)(g[h] >> (16 * j))), uv = bf16_bits_to_f32((uint16_t)(u[h] >> (16 * j)));
      o |= (uint32_t)f32_to_bf16_bits(gv / (1.0f + expf(-gv)) * uv) << (16 * j);
    }
    y[h] = o;
  }
  *(u32x4*)(Y + (int64_t)t * ldy + c0) = y;
}

__global__ void silu_mul_kernel(const uint16_t* __restrict__ G, const uint16_t* __restrict__ U, int64_t ld, int m,
                                int n, uint16_t* __restrict__ Y, int64_t ldy) {
  const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (id >= (int64_t)m * n) return;
  const int64_t t = id / n, c = id % n;
  const float g = bf16_bits_to_f32(G[t * ld + c]), u = bf16_bits_to_f32(U[t * ld + c]);
  Y[t * ldy + c] = f32_to_bf16_bits(g / (1.0f + expf(-g)) * u);
}

typedef __bf16 bf16v2 __attribute__((ext_vector_type(2)));
typedef float f32v2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  const bf16v2 v = __builtin_convertvector(f32v2{lo, hi}, bf16v2);  // round to nearest even
  uint32_t u;
  __builtin_memcpy(&u, &v, 4);
  return u;
}

// A row of 8 16-byte chunks stored at chunk position c ^ ((r >> 1) & 7): the 16
// rows one fragment read touches (one chunk each) cover the 64 LDS banks once.
__device__ __forceinline__ int swz8(int r, int c) { return r * 8 + (c ^ ((r >> 1) & 7)); }

// ---------------------------------------------------------------------------
// Linear: Y = X W^T (+ R), K % 64 != 0, short K and widths that fill larger tiles
// badly.  One 256-thread workgroup per 128 x 128 tile of Y, 2 x 2 waves of 64 x 64
// (4 x 4 accumulator blocks); K staged 64 at a time through two LDS buffers with
// the global loads of the stage after next held in registers (zero-filled past
// K).  Needs 16-byte aligned rows and K % 8 == 0.
// ---------------------------------------------------------------------------
constexpr int kLinT = 128, kLinK = 64;

__global__ __launch_bounds__(256, 2) void lin_kernel(const uint16_t* __restrict__ X, int64_t ldx,
                                                     const uint16_t* __restrict__ W, int64_t ldw,
                                                     const uint16_t* R, int64_t ldr, uint16_t* Y, int64_t ldy,
                                                     int M, int N, int K) {
  __shared__ u32x4 sm[2][2][kLinT * 8];  // [buffer][X, W][swizzled rows of 8 chunks]: 64 KB
  const int tn = (N + kLinT - 1) / kLinT;
  const int per = (int)((gridDim.x + 7) / 8);
  const int id = (int)(blockIdx.x % 8) * per + (int)(blockIdx.x / 8);  // contiguous tile ranges per XCD
  if (id >= (int)cdiv((int64_t)M, kLinT) * tn) return;
  const int i0 = (id / tn) * kLinT, j0 = (id % tn) * kLinT;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wi = wave >> 1, wj = wave & 1;
  const u32x4 zero = {0u, 0u, 0u, 0u};
  // this thread's loads: rows (tid / 8) + 32 q, chunk tid % 8 (8 threads per 128-byte row segment)
  const int lc = tid & 7;
  const uint16_t* xa[4];
  const uint16_t* wb[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int r = (tid >> 3) + 32 * q;
    xa[q] = X + (int64_t)min(i0 + r, M - 1) * ldx + 8 * lc;
    wb[q] = W + (int64_t)min(j0 + r, N - 1) * ldw + 8 * lc;
  }
  auto load = [&](int k0, u32x4 (&ra)[4], u32x4 (&rb)[4]) {
    const bool ok = k0 + 8 * lc < K;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      ra[q] = ok ? *(const u32x4*)(xa[q] + k0) : zero;
      rb[q] = ok ? *(const u32x4*)(wb[q] + k0) : zero;
    }
  };
  auto store = [&](int buf, const u32x4 (&ra)[4], const u32x4 (&rb)[4]) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int r = (tid >> 3) + 32 * q;
      sm[buf][0][swz8(r, lc)] = ra[q];
      sm[buf][1][swz8(r, lc)] = rb[q];
    }
  };
  f4 acc[4][4];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[a][b] = f4{0.f, 0.f, 0.f, 0.f};
  auto compute = [&](int buf) {
#pragma unroll
    for (int s2 = 0; s2 < kLinK / 32; ++s2) {
      const int c = 4 * s2 + (lane >> 4);
      u32x4 fa[4], fb[4];
#pragma unroll
      for (int a = 0; a < 4; ++a) fa[a] = sm[buf][0][swz8(wi * 64 + a * 16 + (lane & 15), c)];
#pragma unroll
      for (int b = 0; b < 4; ++b) fb[b] = sm[buf][1][swz8(wj * 64 + b * 16 + (lane & 15), c)];
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[a][b] = mma_bf16(fa[a], fb[b], acc[a][b]);
    }
  };
  const int nst = (K + kLinK - 1) / kLinK;
  u32x4 ra0[4], rb0[4], ra1[4], rb1[4];
  load(0, ra0, rb0);
  if (nst > 1) load(kLinK, ra1, rb1);
  store(0, ra0, rb0);
  lds_barrier();
#pragma nounroll
  for (int s = 0; s < nst; s += 2) {
    if (s + 2 < nst) load((s + 2) * kLinK, ra0, rb0);
    compute(0);
    if (s + 1 < nst) store(1, ra1, rb1);
    lds_barrier();
    if (s + 1 >= nst) break;
    if (s + 3 < nst) load((s + 3) * kLinK, ra1, rb1);
    compute(1);
    if (s + 2 < nst) store(0, ra0, rb0);
    lds_barrier();
  }
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = i0 + wi * 64 + a * 16 + (lane >> 4) * 4 + r, j = j0 + wj * 64 + b * 16 + (lane & 15);
        if (i < M && j < N) {
          float v = acc[a][b][r];
          if (R) v += bf16_bits_to_f32(R[(int64_t)i * ldr + j]);
          Y[(int64_t)i * ldy + j] = f32_to_bf16_bits(v);
        }
      }
}

// ---------------------------------------------------------------------------
// Linear, K % 64 == 0: a tile of 256 n by TM m (256, or 128 for launches that
// would leave CUs idle) of Y per 512-thread workgroup (one per CU), eight waves of
// v_mfma_f32_16x16x32_bf16 accumulators: 2 x 4 waves of 128 (n) x 64 (m), or
// 4 x 2 of 64 x 64, in the loop of pingpong.h.  The tile is computed as (W X^T)'s,
// so that a lane holds four consecutive n of one token; a stage is 64 k (whole
// 128-byte lines of both operands).  Bound: MFMA issue and the clock under that
// load.  Measured (16384 x 4096 -> 11008): 1847 us (800 TFLOP/s) on 128 tiles with
// the operands staged through registers, 1011 us (1462 TFLOP/s) here; the same
// tile with all eight waves in step and a ring of five slots 1190 us; one stage
// per trip of the loop (with copies of the B0 fragments) 1082 us.
// ---------------------------------------------------------------------------
constexpr int kLinB = 256;

template <int TM>
struct LinGeo {
  static constexpr int NWM = TM / 64, NWN = 8 / NWM;  // waves along m and n
  static constexpr int HW = kLinB / NWN / 2;          // rows per wave and W half
  static constexpr int HA = HW / 16;                  // their 16-row blocks (X half: 32 rows, 2 blocks)
  static constexpr int UW = 128 * 128;                // bytes of a W unit (128 rows)
  static constexpr int UX = 32 * NWM * 128;           // of an X unit
  static constexpr int LW = 2, LX = UX / 8192;        // wave-wide loads per wave and unit
  static constexpr int PAR = 2 * (UW + UX);           // one stage
  static constexpr int ELS = kLinB * 4 + 16;          // epilogue: fp32 row stride in bytes, 128 rows per pass
  static constexpr size_t LDS = (size_t)128 * ELS > (size_t)2 * PAR ? (size_t)128 * ELS : (size_t)2 * PAR;
};

template <int TM>
__global__ __launch_bounds__(512) void lin256_kernel(const uint16_t* __restrict__ X, int64_t ldx,
                                                     const uint16_t* __restrict__ W, int64_t ldw, const uint16_t* R,
                                                     int64_t ldr, uint16_t* Y, int64_t ldy, int M, int N, int K,
                                                     int vec) {
  using G = LinGeo<TM>;
  extern __shared__ __attribute__((aligned(16))) uint8_t lsm[];  // [stage parity][W0, W1, X0, X1]
  constexpr int GB = 4, HA = G::HA;
  const int tm = (M + TM - 1) / TM, tn = (N + kLinB - 1) / kLinB;
  const int per = (int)((gridDim.x + 7) / 8);
  const int id = (int)(blockIdx.x % 8) * per + (int)(blockIdx.x / 8);  // contiguous tile ranges per XCD
  if (id >= tm * tn) return;
  // bands of 4 row tiles walked across the columns: the 32 workgroups of an
  // XCD hold 4 x 8 tiles, whose operand panels they share in its L2
  const int b0 = id / (GB * tn) * GB, bh = min(GB, tm - b0), br = id - b0 * tn;
  const int i0 = (b0 + br % bh) * TM, j0 = (br / bh) * kLinB;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wi = wave / G::NWM, wj = wave % G::NWM;  // place along n, m
  const int g = lane >> 4, l16 = lane & 15;

  // this lane's chunk of each of the wave's loads per unit (8 unit rows of 128
  // bytes each); unit row u of W half h is tile row 2 HW (u / HW) + HW h + u % HW,
  // of X half h 64 (u / 32) + 32 h + u % 32
  const uint16_t* src[4][2];  // [W0, W1, X0, X1]
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int uw = wave * 16 + 8 * j + (lane >> 3), ux = wave * 8 * G::LX + 8 * j + (lane >> 3);
    const int cw = (lane & 7) ^ ((uw >> 1) & 7), cx = (lane & 7) ^ ((ux >> 1) & 7);
    const int rw = 2 * G::HW * (uw / G::HW) + uw % G::HW, rx = 64 * (ux >> 5) + (ux & 31);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      src[h][j] = W + (int64_t)min(j0 + rw + G::HW * h, N - 1) * ldw + 8 * cw;
      src[2 + h][j] = X + (int64_t)min(i0 + rx + 32 * h, M - 1) * ldx + 8 * cx;
    }
  }
  const int nst = K / 64;
  // unit `op` of stage st (of parity par; past the last stage: the last one again,
  // into a slot that is read no more)
  auto issue = [&](int op, int st, int par) {
    const int nl = op < 2 ? G::LW : G::LX;
    uint8_t* dst = lsm + par * G::PAR + (op < 2 ? op * G::UW : 2 * G::UW + (op - 2) * G::UX) + wave * nl * 1024;
    const int64_t off = (int64_t)min(st, nst - 1) * 64;
#pragma unroll
    for (int j = 0; j < nl; ++j)
      __builtin_amdgcn_global_load_lds((const void*)(src[op][j] + off),
                                       (__attribute__((address_space(3))) void*)(dst + j * 1024), 16, 0, 0);
  };
  f4 acc[2 * HA][4];
#pragma unroll
  for (int a = 0; a < 2 * HA; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[a][b] = f4{0.f, 0.f, 0.f, 0.f};

  // fragment offsets within a unit; k-step 1 of a stage is chunk ^ 4
  const uint32_t fw = (uint32_t)((wi * G::HW + l16) * 128 + ((g ^ (l16 >> 1)) * 16));
  const uint32_t fx = (uint32_t)((wj * 32 + l16) * 128 + ((g ^ (l16 >> 1)) * 16));
  auto read_w = [&](int par, int h, u32x4 (&F)[2][HA]) {
    const uint8_t* p = lsm + par * G::PAR + h * G::UW;
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
      for (int a = 0; a < HA; ++a) F[s2][a] = *(const u32x4*)(p + (fw ^ (64u * s2)) + a * 2048);
  };
  auto read_x = [&](int par, int h, u32x4 (&F)[2][2]) {
    const uint8_t* p = lsm + par * G::PAR + 2 * G::UW + h * G::UX;
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
      for (int b = 0; b < 2; ++b) F[s2][b] = *(const u32x4*)(p + (fx ^ (64u * s2)) + b * 2048);
  };
  pp_loop<HA, G::LW, G::LX>(nst, acc, issue, read_w, read_x);

  // accumulator element r of block (a, b): n = 2 HW wi + 16 a + 4 g + r, m = 64 wj + 16 b + l16
  // residual added in fp32, one rounding; staged through LDS, 128 tokens per pass,
  // so that global accesses are 16 bytes per lane, or without `vec` (rows of Y or R
  // that 16-byte accesses cannot take) consecutive in a wave.  (Straight from the
  // accumulators, two bytes per row and lane: 65536 x 64 -> 300 with a residual 99 us,
  // 46 here.)
#pragma unroll
  for (int h = 0; h < TM / 128; ++h) {
    lds_barrier();
    if (wj >> 1 == h)
#pragma unroll
      for (int a = 0; a < 2 * HA; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b)
          *(f4*)(lsm + ((wj & 1) * 64 + b * 16 + l16) * G::ELS + (wi * 2 * G::HW + a * 16 + 4 * g) * 4) = acc[a][b];
    lds_barrier();
    if (!vec) {
      // a thread takes one column, every other row, sixteen rows' loads at a time
      const int c = tid % kLinB, j = j0 + c, ib = i0 + h * 128 + tid / kLinB;
      if (j >= N) continue;
      const uint8_t* l = lsm + (tid / kLinB) * G::ELS + c * 4;
      for (int q = 0; q < 64; q += 16) {
        uint16_t rv[16];
        if (R)
#pragma unroll
          for (int e = 0; e < 16; ++e) rv[e] = R[(int64_t)min(ib + 2 * (q + e), M - 1) * ldr + j];
        float v[16];
#pragma unroll
        for (int e = 0; e < 16; ++e) v[e] = *(const float*)(l + 2 * (q + e) * G::ELS);
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int i = ib + 2 * (q + e);
          if (R) v[e] += bf16_bits_to_f32(rv[e]);
          if (i < M) Y[(int64_t)i * ldy + j] = f32_to_bf16_bits(v[e]);
        }
      }
      continue;
    }
#pragma unroll 4
    for (int q = tid; q < 128 * (kLinB / 8); q += 512) {
      const int rr = q / (kLinB / 8), c8 = (q % (kLinB / 8)) * 8;
      const int i = i0 + h * 128 + rr, j = j0 + c8;
      if (i >= M || j >= N) continue;
      const f4 v0 = *(const f4*)(lsm + rr * G::ELS + c8 * 4), v1 = *(const f4*)(lsm + rr * G::ELS + c8 * 4 + 16);
      float v[8] = {v0[0], v0[1], v0[2], v0[3], v1[0], v1[1], v1[2], v1[3]};
      if (R) {
        const u32x4 rv = *(const u32x4*)(R + (int64_t)i * ldr + j);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] += bf16_bits_to_f32((uint16_t)(rv[e >> 1] >> (16 * (e & 1))));
      }
      u32x4 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = pack_bf16(v[2 * e], v[2 * e + 1]);
      *(u32x4*)(Y + (int64_t)i * ldy + j) = o;
    }
  }
}

// Linear for rows that are not 16-byte aligned or K % 8 != 0: one thread per
// output, fp32 sum in k order.
__global__ void lin_plain_kernel(const uint16_t* __restrict__ X, int64_t ldx, const uint16_t* __restrict__ W,
                                 int64_t ldw, const uint16_t* R, int64_t ldr, uint16_t* Y, int64_t ldy, int M, int N,
                                 int K) {
  const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (id >= (int64_t)M * N) return;
  const int i = (int)(id / N), j = (int)(id % N);
  float v = 0.f;
  for (int k = 0; k < K; ++k) v = fmaf(bf16_bits_to_f32(X[(int64_t)i * ldx + k]), bf16_bits_to_f32(W[(int64_t)j * ldw + k]), v);
  if (R) v += bf16_bits_to_f32(R[(int64_t)i * ldr + j]);
  Y[(int64_t)i * ldy + j] = f32_to_bf16_bits(v);
}

// ---------------------------------------------------------------------------
// Causal attention in two passes over the key blocks: pass 1 finds each row's
// maximum and sum of exponentials, pass 2 forms the normalised probabilities,
// rounds them to bf16 (the reference's rounding point) and multiplies by V.
// One workgroup per (sequence, head, block of 32 NW queries); wave w owns
// queries 32 w .. 32 w + 31.  Everything is computed transposed, with
// v_mfma_f32_32x32x16_bf16 (lane l holds row l % 32 of A and column l % 32 of B,
// the 8 consecutive k of half l / 32; accumulator element r sits at row
// 8 (r / 4) + 4 (l / 32) + r % 4, column l % 32):
//   S^T = K Q^T    a lane's 16 elements per 32-key block belong to one query, so
//                  maxima and sums are in-lane (one exchange with lane ^ 32 at
//                  the end of pass 1);
//   O^T = V^T P^T  P^T's B fragments are the lane's own S^T registers (keys
//                  16 t + 4 h + {0..3, 8..11} for half h of step t); V^T's A
//                  fragments take the same keys from the row-major V tile with
//                  transposing LDS reads.
// So P never passes through LDS.  K and V tiles of 64 keys (pass 1: two K
// tiles) stream global -> LDS directly, double buffered (64 KB at head_dim 128:
// two workgroups per CU), the next loads in flight during this block's work.
// Chunk positions are permuted (kswz, vswz) so that neither fragment read meets
// bank conflicts.  Bound: per 64-key block a wave has about 1500 cycles of MFMA
// and as many of exponentials, maxima and sums, which only overlap between the
// two waves of a SIMD.  Measured (8 x 2048 tokens, 32 heads of 128): 2656 us for
// the form before (64 queries per workgroup, 16-wide MFMA, P and V transposed
// element by element through LDS), 569 us now (483 TFLOP/s of the two products).
// The query blocks of one (sequence, head) run on one XCD and share its K and
// V in that XCD's L2, but for heads left over from groups of eight: one head (of
// 128, 16384 tokens) on one XCD 1357 us, over all of them 608; nine heads 1558 and 1050.
// ---------------------------------------------------------------------------
typedef short s16v4 __attribute__((ext_vector_type(4)));
typedef float f16x __attribute__((ext_vector_type(16)));

__device__ __forceinline__ f16x mma32_bf16(const u32x4& a, const u32x4& b, f16x c) {
  bf16x8 av, bv;
  __builtin_memcpy(&av, &a, 16);
  __builtin_memcpy(&bv, &b, 16);
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, bv, c, 0, 0, 0);
}

// (Sequence, head) pairs left over from groups of eight, one per XCD; seven run as a
// group (spread over all XCDs they read every K and V eight times: 5 % slower up to
// 8192 tokens).
__host__ __device__ inline int attn_left(int nsh) { return nsh % 8 == 7 ? 0 : nsh % 8; }

template <int HD, int NW>
__global__ __launch_bounds__(64 * NW, NW / 2) void attn_kernel(const uint16_t* __restrict__ Q,
                                                               const uint16_t* __restrict__ Kx,
                                                          const uint16_t* __restrict__ V, int64_t ld, int L, int heads,
                                                          int nsh, float cexp, uint16_t* O, int64_t ldo, int nqb,
                                                          int vec) {
  constexpr int KB = 64;           // keys per block
  constexpr int CH = HD / 8;       // 16-byte chunks per key row
  constexpr int KS = HD / 16;      // MFMA k-steps over head_dim
  constexpr int DB = HD / 32;      // 32-wide blocks of the output row
  constexpr int TILE = KB * CH;    // chunks per operand tile
  constexpr int NL = TILE / (64 * NW);  // 16-byte loads per thread, operand and block
  __shared__ u32x4 sm[2][2][TILE];  // [buffer][K, V]
  // ids go round-robin over the XCDs: all query blocks of a head on one of them,
  // the longest first; before that the heads that make no group (attn_left), spread
  // over all XCDs, the shortest first where others follow (when all are resident a
  // CU then holds long and short ones)
  const int left = attn_left(nsh), off = (int)rup((int64_t)left * nqb, 8);
  int id = (int)blockIdx.x, sh, qb;
  if (id < off) {
    if (id >= left * nqb) return;
    sh = nsh - left + id % left;
    qb = nsh < 8 ? nqb - 1 - id / left : id / left;
  } else {
    id = (id - off) / 8;
    sh = id / nqb * 8 + (int)(blockIdx.x % 8);
    if (sh >= nsh) return;
    qb = nqb - 1 - id % nqb;
  }
  const int h = sh % heads;
  const int64_t row0 = (int64_t)(sh / heads) * L;  // the sequence's first token
  const int col0 = h * HD;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l32 = lane & 31, half = lane >> 5;
  const int q0 = qb * 32 * NW, qw = q0 + 32 * wave;  // first query of the workgroup, of this wave
  // chunk c of key row r sits at position kswz(r, c) (vswz) of its row: 16
  // consecutive keys' chunks of a K fragment, and the four keys x 64 bytes that
  // half a wave's transposing read of V touches, cover the 64 banks once
  auto kswz = [](int key, int c) { return CH == 16 ? c ^ (key & 15) : c ^ ((key >> 1) & 7); };
  auto vswz = [](int key, int c) { return CH == 16 ? c ^ (4 * (key & 3)) : c ^ (4 * ((key >> 1) & 1)); };

  u32x4 qa[KS];
  {
    const int qr = min(qw + l32, L - 1);
#pragma unroll
    for (int c = 0; c < KS; ++c) qa[c] = *(const u32x4*)(Q + (row0 + qr) * ld + col0 + 8 * (2 * c + half));
  }
  const int nkb = min((q0 + 32 * NW + KB - 1) / KB, (L + KB - 1) / KB);

  // this thread's part of one operand tile: key block kb of `src` into `dst`
  auto issue = [&](const uint16_t* src, int kb, u32x4* dst, bool is_v) {
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int base = (wave * NL + i) * 64;  // wave-uniform destination
      const int key = (base + lane) / CH, p = (base + lane) % CH;
      const int64_t off = (row0 + min(kb * KB + key, L - 1)) * ld + col0;
      __builtin_amdgcn_global_load_lds((const void*)(src + off + 8 * (is_v ? vswz(key, p) : kswz(key, p))),
                                       (__attribute__((address_space(3))) void*)(dst + base), 16, 0, 0);
    }
  };
  // S^T of key block kb (raw products; keys above the query masked)
  auto scores = [&](const u32x4* sK, int kb, f16x (&sc)[2]) {
#pragma unroll
    for (int b = 0; b < 2; ++b) {
#pragma unroll
      for (int r = 0; r < 16; ++r) sc[b][r] = 0.f;
      const int key = 32 * b + l32;
#pragma unroll
      for (int c = 0; c < KS; ++c) sc[b] = mma32_bf16(sK[key * CH + kswz(key, 2 * c + half)], qa[c], sc[b]);
    }
    if (kb * KB + KB - 1 > qw) {  // uniform per wave: the block meets the diagonal
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (kb * KB + 32 * b + 8 * (r >> 2) + 4 * half + (r & 3) > qw + l32) sc[b][r] = -INFINITY;
    }
  };

  // pass 1: maximum m and sum l of exp over this half's keys of query qw + l32.
  // mc = m cexp as rounded: every exponential is relative to that number, also
  // where a sum moves to a new maximum, so its rounding drops out of p
  float m = -INFINITY, mc = -INFINITY, l = 0.f;
  issue(Kx, 0, sm[0][0], false);
  issue(Kx, 1, sm[0][1], false);
  int kb = 0;
  do {  // two key blocks per trip; nkb >= 1
    const int buf = (kb >> 1) & 1;
    wait_vm<0>();     // this wave's part of the blocks landed
    lds_barrier();  // every wave's; and every wave is done with the blocks before
    if (kb + 2 < nkb) {
      issue(Kx, kb + 2, sm[buf ^ 1][0], false);
      issue(Kx, kb + 3, sm[buf ^ 1][1], false);
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      if ((kb + u) * KB > qw + 31) continue;  // uniform per wave: every key lies above its queries
      f16x sc[2];
      scores(sm[buf][u], kb + u, sc);
      float mn = m;
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) mn = fmaxf(mn, sc[b][r]);
      const float mcn = mn * cexp;
      const float base = mn == -INFINITY ? 0.f : mcn;  // no key of this half yet: every exponential is 0
      l *= __builtin_amdgcn_exp2f(mc - base);
      m = mn;
      mc = mcn;
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) l += __builtin_amdgcn_exp2f(fmaf(sc[b][r], cexp, -base));
    }
    kb += 2;
  } while (kb < nkb);
  // both halves' keys; p = exp2(s cexp - e) is then normalised up to e's own
  // rounding (of scores of 1e5 as large as bf16's), which `fix` takes out of O
  float e, fix;
  {
    const auto rm = __builtin_amdgcn_permlane32_swap(__float_as_uint(mc), __float_as_uint(mc), false, false);
    const auto rl = __builtin_amdgcn_permlane32_swap(__float_as_uint(l), __float_as_uint(l), false, false);
    const float m0 = __uint_as_float(rm[0]), m1 = __uint_as_float(rm[1]);
    const float mm = fmaxf(m0, m1);
    const float lt = __uint_as_float(rl[0]) * __builtin_amdgcn_exp2f(m0 - mm) +
                     __uint_as_float(rl[1]) * __builtin_amdgcn_exp2f(m1 - mm);
    const float lg = __builtin_amdgcn_logf(lt);  // log2
    e = mm + lg;
    const float d = e - mm;
    fix = __builtin_amdgcn_exp2f(-((mm - (e - d)) + (lg - d)));  // e + that difference is mm + lg exactly
  }

  // pass 2: bf16 probabilities times V
  f16x o[DB];
#pragma unroll
  for (int d = 0; d < DB; ++d)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[d][r] = 0.f;
  // transposing read: lane i of each 16 addresses key i / 4, 4 values at 4 (i % 4)
  const int tj = (lane & 15) >> 2;
  int vo[DB];
#pragma unroll
  for (int d = 0; d < DB; ++d)
    vo[d] = (4 * half + tj) * HD * 2 + vswz(tj, 4 * d + 2 * ((lane >> 4) & 1)) * 16 + (lane & 3) * 8;
  lds_barrier();  // every wave is done with pass 1's tiles
  issue(Kx, 0, sm[0][0], false);
  issue(V, 0, sm[0][1], true);
  kb = 0;
  do {
    wait_vm<0>();
    lds_barrier();
    if (kb + 1 < nkb) {
      issue(Kx, kb + 1, sm[(kb + 1) & 1][0], false);
      issue(V, kb + 1, sm[(kb + 1) & 1][1], true);
    }
    if (kb * KB > qw + 31) continue;  // uniform per wave
    const uint8_t* sV = (const uint8_t*)sm[kb & 1][1];
    f16x sc[2];
    scores(sm[kb & 1][0], kb, sc);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      u32x4 pf;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int r = 8 * (t & 1) + 2 * j;
        pf[j] = pack_bf16(__builtin_amdgcn_exp2f(fmaf(sc[t >> 1][r], cexp, -e)),
                          __builtin_amdgcn_exp2f(fmaf(sc[t >> 1][r + 1], cexp, -e)));
      }
#pragma unroll
      for (int d = 0; d < DB; ++d) {
        typedef __attribute__((address_space(3))) s16v4 lds4;
        const s16v4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4*)(sV + vo[d] + (16 * t) * HD * 2));
        const s16v4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4*)(sV + vo[d] + (16 * t + 8) * HD * 2));
        u32x4 a;
        __builtin_memcpy(&a, &v0, 8);
        __builtin_memcpy((char*)&a + 8, &v1, 8);
        o[d] = mma32_bf16(a, pf, o[d]);
      }
    }
  } while (++kb < nkb);
  // The compiler (ROCm 7.2) copied an accumulator at the loop's exit before
  // its last MFMA had written it; nothing may touch them until it has.
#pragma unroll
  for (int d = 0; d < DB; ++d) asm volatile("s_nop 15" : "+v"(o[d]));
  const int q = qw + l32;
  if (q >= L) return;
  uint16_t* y0 = O + (row0 + q) * ldo + col0 + 4 * half;
#pragma unroll
  for (int d = 0; d < DB; ++d)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      uint16_t* yp = y0 + 32 * d + 8 * g;
      const uint32_t u0 = pack_bf16(o[d][4 * g] * fix, o[d][4 * g + 1] * fix);
      const uint32_t u1 = pack_bf16(o[d][4 * g + 2] * fix, o[d][4 * g + 3] * fix);
      if (vec) {
        *(uint2*)yp = make_uint2(u0, u1);
      } else {
        yp[0] = (uint16_t)u0;
        yp[1] = (uint16_t)(u0 >> 16);
        yp[2] = (uint16_t)u1;
        yp[3] = (uint16_t)(u1 >> 16);
      }
    }
}

bool aligned(const void* ws) { return (reinterpret_cast<uintptr_t>(ws) % kAlign) == 0; }
bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) % 16) == 0; }

int act_zeros(const duo_act_rule& r, int64_t k) {
  if (r.kind == DUO_ACT_NONE) return 0;
  return (int)std::floor(r.sparsity * (double)k + 0.5);
}

}  // namespace

extern "C" {

size_t duo_block_workspace_size(int32_t op, int64_t m, int64_t seq_len, int64_t heads) {
  switch (op) {
    case DUO_BOP_ACT_SPARSIFY: return m < 1 ? 0 : (size_t)rup(m * (int64_t)sizeof(int64_t), kAlign);
    case DUO_BOP_LINEAR: return 0;  // no scratch memory
    case DUO_BOP_ATTENTION: return 0;  // no scratch memory
    default: return 0;
  }
}

duo_status duo_rmsnorm(const void* X, int64_t m, int64_t d, int64_t ldx, double eps, void* Y, int64_t ldy,
                       void* stream) {
  if (m < 0 || d < 1 || ldx < d || ldy < d || !(eps >= 0.0) || !std::isfinite(eps)) return DUO_ERR_INVALID_ARG;
  if (m == 0) return DUO_OK;
  if (!X || !Y || m > INT32_MAX) return DUO_ERR_INVALID_ARG;
  if (duo_status d = device_ok(); d != DUO_OK) return d;
  hipLaunchKernelGGL(rmsnorm_kernel, dim3((unsigned)m), dim3(256), 0, (hipStream_t)stream, (const uint16_t*)X, ldx,
                     (int)d, (float)eps, (uint16_t*)Y, ldy);
  DUO_LAUNCH_CHECK();
  return DUO_OK;
}

duo_status duo_act_sparsify(const void* X, int64_t m, int64_t k, int64_t ldx, duo_act_rule rule, void* Y, int64_t ldy,
                            void* ws, size_t ws_bytes, void* stream) {
  if (m < 0 || k < 1 || k > kMaxK || ldx < k || ldy < k) return DUO_ERR_INVALID_ARG;
  if (rule.kind != DUO_ACT_NONE &&
      !(rule.kind == DUO_ACT_TOPK_MAG_PER_TOKEN && std::isfinite(rule.sparsity) && rule.sparsity >= 0.0 &&
        rule.sparsity <= 1.0))
    return DUO_ERR_INVALID_ARG;
  if (m == 0) return DUO_OK;
  if (!X || !Y || m > INT32_MAX) return DUO_ERR_INVALID_ARG;
  const size_t need = duo_block_workspace_size(DUO_BOP_ACT_SPARSIFY, m, 0, 0);
  if (!ws || ws_bytes < need || !aligned(ws)) return DUO_ERR_WORKSPACE;
  if (duo_status d = device_ok(); d != DUO_OK) return d;
  hipStream_t s = (hipStream_t)stream;
  bool done;
  duo_status st = act_sparsify_run((const uint16_t*)X, m, k, ldx, act_zeros(rule, k), (uint16_t*)Y, ldy, &done, s);
  if (st != DUO_OK || done) return st;
  int64_t* thr = (int64_t*)ws;
  st = act_threshold_run(X, DUO_BF16, m, k, ldx, act_zeros(rule, k), thr, s);
  if (st != DUO_OK) return st;
  const int64_t tot = m * k;
  hipLaunchKernelGGL(act_apply_kernel, dim3((unsigned)cdiv(tot, 256)), dim3(256), 0, s, (const uint16_t*)X, ldx,
                     (int)m, (int)k, (const int64_t*)thr, (uint16_t*)Y, ldy);
  DUO_LAUNCH_CHECK();
  return DUO_OK;
}

duo_status duo_linear(const void* X, int64_t m, int64_t k, int64_t ldx, const void* W, int64_t n, int64_t ldw,
                      const void* R, int64_t ldr, void* Y, int64_t ldy, void* ws, size_t ws_bytes, void* stream) {
  (void)ws;
  (void)ws_bytes;
  if (m < 0 || k < 1 || n < 1 || ldx < k || ldw < k || ldy < n || (R && ldr < n)) return DUO_ERR_INVALID_ARG;
  if (m > INT32_MAX || n > INT32_MAX || k > INT32_MAX || m * n > ((int64_t)1 << 40)) return DUO_ERR_UNSUPPORTED;
  if (m == 0) return DUO_OK;
  if (!X || !W || !Y) return DUO_ERR_INVALID_ARG;
  if (duo_status d = device_ok(); d != DUO_OK) return d;
  const hipStream_t s = (hipStream_t)stream;
  const bool vec = k % 8 == 0 && ldx % 8 == 0 && ldw % 8 == 0 && aligned16(X) && aligned16(W);
  if (vec) {
    const int64_t tiles = cdiv(m, kLinT) * cdiv(n, kLinT);
    // Microseconds of the three tile sizes: rounds of the chip (256 CUs with one
    // tile each; two of the 128 tiles) times a fixed part (launch, first loads,
    // epilogue) and a part per k, fitted to measured launches (m x k -> n: 4096 x
    // 4096 -> 4096 95, 57.5 x 2 and 181 us; 40000 x 512 -> 300 41, 46 and 38 us).
    // The 128 tile keeps short sums and widths that fill 256 badly.  Two-byte
    // stores cost a large tile 9 or 4.5 us, which nothing on the CU overlaps (65536 x 64
    // -> 300 27 us on 128 tiles, 39 on 256; x 256 -> 777 80 and 91); a residual
    // read two bytes at a time costs the 128 tile more (68 and 46; 167 and 105).
    const int vy = n % 8 == 0 && ldy % 8 == 0 && aligned16(Y) && (!R || (ldr % 8 == 0 && aligned16(R)));
    const double sc = vy || R ? 0.0 : 4.5;
    const int64_t t256 = cdiv(m, 256) * cdiv(n, kLinB), t128 = cdiv(m, 128) * cdiv(n, kLinB);
    const double c256 = (double)cdiv(t256, 256) * (9.5 + 2.0 * sc + 0.0213 * (double)k);
    const double c128 = (double)cdiv(t128, 256) * (7.5 + sc + 0.0122 * (double)k);
    const double cold = (double)cdiv(tiles, 512) * (7.8 + 0.0201 * (double)k);
    if (k % 64 == 0 && (c256 <= cold || c128 <= cold)) {
      auto go = [&](auto kern, int64_t nt, size_t lds) -> duo_status {
        if (nt > INT32_MAX) return DUO_ERR_UNSUPPORTED;
        if (duo_status st = set_max_lds((const void*)kern, lds); st != DUO_OK) return st;
        hipLaunchKernelGGL(kern, dim3((unsigned)rup(nt, 8)), dim3(512), lds, s, (const uint16_t*)X, ldx,
                           (const uint16_t*)W, ldw, (const uint16_t*)R, ldr, (uint16_t*)Y, ldy, (int)m, (int)n, (int)k,
                           vy);
        DUO_LAUNCH_CHECK();
        return DUO_OK;
      };
      if (c256 <= c128) return go(lin256_kernel<256>, t256, LinGeo<256>::LDS);
      return go(lin256_kernel<128>, t128, LinGeo<128>::LDS);
    }
    if (tiles > INT32_MAX) return DUO_ERR_UNSUPPORTED;
    hipLaunchKernelGGL(lin_kernel, dim3((unsigned)rup(tiles, 8)), dim3(256), 0, s, (const uint16_t*)X, ldx,
                       (const uint16_t*)W, ldw, (const uint16_t*)R, ldr, (uint16_t*)Y, ldy, (int)m, (int)n, (int)k);
  } else {
    hipLaunchKernelGGL(lin_plain_kernel, dim3((unsigned)cdiv(m * n, 256)), dim3(256), 0, s, (const uint16_t*)X, ldx,
                       (const uint16_t*)W, ldw, (const uint16_t*)R, ldr, (uint16_t*)Y, ldy, (int)m, (int)n, (int)k);
  }
  DUO_LAUNCH_CHECK();
  return DUO_OK;
}

duo_status duo_rope(void* X, int64_t m, int64_t heads, int64_t head_dim, int64_t ldx, int64_t seq_len, double theta,
                    void* stream) {
  if (m < 0 || heads < 1 || head_dim < 2 || (head_dim & 1) || ldx < heads * head_dim || seq_len < 1 ||
      !(theta > 0.0) || !std::isfinite(theta))
    return DUO_ERR_INVALID_ARG;
  if (m == 0) return DUO_OK;
  if (!X || m > INT32_MAX) return DUO_ERR_INVALID_ARG;
  if (duo_status d = device_ok(); d != DUO_OK) return d;
  hipLaunchKernelGGL(rope_kernel, dim3((unsigned)m), dim3(256), 0, (hipStream_t)stream, (uint16_t*)X, ldx, (int)heads,
                     (int)head_dim, (int)seq_len, theta);
  DUO_LAUNCH_CHECK();
  return DUO_OK;
}

duo_status duo_attention(const void* Q, const void* K, const void* V, int64_t ld, int64_t nseq, int64_t seq_len,
                         int64_t heads, int64_t head_dim, void* O, int64_t ldo, void* ws, size_t ws_bytes,
                         void* stream) {
  (void)ws;
  (void)ws_bytes;
  if (nseq < 0 || seq_len < 1 || heads < 1 || head_dim < 1 || ld < heads * head_dim || ldo < heads * head_dim)
    return DUO_ERR_INVALID_ARG;
  if (head_dim != 64 && head_dim != 128) return DUO_ERR_UNSUPPORTED;
  if (seq_len > INT32_MAX || ld > INT32_MAX || ldo > INT32_MAX || nseq * heads * cdiv(seq_len, 64) > INT32_MAX)
    return DUO_ERR_UNSUPPORTED;
  if (nseq == 0) return DUO_OK;
  if (!Q || !K || !V || !O) return DUO_ERR_INVALID_ARG;
  if (ld % 8 != 0 || !aligned16(Q) || !aligned16(K) || !aligned16(V)) return DUO_ERR_UNSUPPORTED;
  if (duo_status d = device_ok(); d != DUO_OK) return d;
  const hipStream_t s = (hipStream_t)stream;
  // exp(s / sqrt(d)) = 2^(s cexp)
  const float cexp = (float)(1.4426950408889634 / std::sqrt((double)head_dim));
  const int nsh = (int)(nseq * heads);
  // 128 queries per workgroup; 64 when that would leave CUs without their two
  // workgroups (512 in all), so that short or few sequences spread further
  const bool wide = (int64_t)nsh * cdiv(seq_len, 128) >= 512;
  const int nqb = (int)cdiv(seq_len, wide ? 128 : 64);
  const int left = attn_left(nsh);
  const dim3 grid((unsigned)(rup((int64_t)left * nqb, 8) + rup(nsh - left, 8) * nqb));
  const int vec = ldo % 4 == 0 && (reinterpret_cast<uintptr_t>(O) & 7) == 0;
  auto go = [&](auto kern, int nw) {
    hipLaunchKernelGGL(kern, grid, dim3(64 * nw), 0, s, (const uint16_t*)Q, (const uint16_t*)K, (const uint16_t*)V, ld,
                       (int)seq_len, (int)heads, nsh, cexp, (uint16_t*)O, ldo, nqb, vec);
  };
  if (head_dim == 128)
    wide ? go(attn_kernel<128, 4>, 4) : go(attn_kernel<128, 2>, 2);
  else
    wide ? go(attn_kernel<64, 4>, 4) : go(attn_kernel<64, 2>, 2);
  DUO_LAUNCH_CHECK();
  return DUO_OK;
}

duo_status duo_silu_mul(const void* G, const void* U, int64_t m, int64_t n, int64_t ld, void* Y, int64_t ldy,
                        void* stream) {
  if (m < 0 || n < 1 || ld < n || ldy < n) return DUO_ERR_INVALID_ARG;
  if (m == 0) return DUO_OK;
  if (!G || !U || !Y) return DUO_ERR_INVALID_ARG;
  if (duo_status d = device_ok(); d != DUO_OK) return d;
  const int64_t tot = m * n;
  if (n % 8 == 0 && ld % 8 == 0 && ldy % 8 == 0 && aligned16(G) && aligned16(U) && aligned16(Y) &&
      m * cdiv(n, 2048) <= INT32_MAX)
    hipLaunchKernelGGL(silu_mul8_kernel, dim3((unsigned)(m * cdiv(n, 2048))), dim3(256), 0,
                       (hipStream_t)stream, (const uint16_t*)G, (const uint16_t*)U, ld, (int)n, (uint16_t*)Y, ldy);
  else
    hipLaunchKernelGGL(silu_mul_kernel, dim3((unsigned)cdiv(tot, 256)), dim3(256), 0, (hipStream_t)stream,
                       (const uint16_t*)G, (const uint16_t*)U, ld, (int)m, (int)n, (uint16_t*)Y, ldy);
  DUO_LAUNCH_CHECK();
  return DUO_OK;
}

}  // extern "C"
