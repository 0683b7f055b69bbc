// fp32 products on the bf16 matrix cores.  Each fp32 operand is split exactly into
// three bf16 parts, x = h + m + l (8 significant bits each, round to nearest), and
//   a b = l_a h_b + h_a l_b + m_a m_b + m_a h_b + h_a m_b + h_a h_b
// is accumulated in fp32, smallest terms first; of the three terms left out m_a l_b and
// l_a m_b reach 2^-25 |a b| each.  A term is exact, and per 64 k the accumulators are
// rounded 12 times where v_mfma_f32_16x16x4_f32 rounds them 16 times.  Six bf16 products
// at about 1500 TFLOP/s are an fp32 product at 250, against 125-137 on the fp32 matrix
// instructions (157 peak).
//
// The operands are packed first (pack_kernel; 6 bytes per element) into the layout
// of stage 1, [plane][k block of 32][group][row][16 bytes], so that the product is
// the loop of pingpong.h over six stages per 64 k.  Packing reads each operand
// once and zero-fills rows to 256 and k to 64, so any size takes this path.
//
// Values: an operand that bf16 would round to infinity keeps the largest finite
// h (m and l take the rest).  An infinite operand gives NaN (inf m + inf l), where
// fp32 gives an infinity or, if a zero of the triangle meets it, NaN.  Parts below
// 2^-126 are rounded to multiples of 2^-133, an absolute error of up to 2^-134 |b|: less
// than fp32's own rounding for operands above 2^-110.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "internal.h"
#include "pingpong.h"

namespace duo {

namespace {

constexpr int ST = 256;                 // tile edge
constexpr int kUnit = 128 * 128;        // bytes of an LDS unit: 128 rows x 64 k
constexpr size_t kLds = (size_t)8 * kUnit;

struct PackArgs {
  const float* src;  // element (r, l) at src[r * ld + l] (kc) or src[l * ld + r]
  int64_t ld;
  int kc, rows, K, rp, nkb;  // rp: rows padded to 256; nkb: k blocks of 32 (even)
  int tri;  // entries l < r count as zero, whatever is stored there
  int vec;
  uint8_t* dst;
  int64_t plane;   // bytes per plane
};

__device__ __forceinline__ uint32_t bits(float f) { return __float_as_uint(f); }

// h, m, l of two values, packed in pairs
__device__ __forceinline__ void split2(float x0, float x1, uint32_t& h, uint32_t& m, uint32_t& l) {
  uint32_t o[3] = {0u, 0u, 0u};
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const float x = e ? x1 : x0;
    uint32_t hb = f32_to_bf16_bits(x);
    const bool fin = (bits(x) & 0x7f800000u) != 0x7f800000u;
    if (fin && (hb & 0x7f80u) == 0x7f80u) hb = bits(x) >> 16;  // would round to infinity: truncate
    const float r = fin ? x - __uint_as_float(hb << 16) : 0.f;
    const uint32_t mb = f32_to_bf16_bits(r);
    const uint32_t lb = f32_to_bf16_bits(r - __uint_as_float(mb << 16));
    o[0] |= hb << (16 * e);
    o[1] |= mb << (16 * e);
    o[2] |= lb << (16 * e);
  }
  h = o[0];
  m = o[1];
  l = o[2];
}

// 64 rows x KPB blocks of 32 k per 256-thread workgroup; a thread splits the 8
// consecutive k of one group of one row and stores 16 bytes per plane.  Bound: HBM
// (4 bytes read, 6 written per element).
constexpr int KPB = 4;
__global__ __launch_bounds__(256) void pack_kernel(PackArgs A) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const float* src = A.src;
  // k-contiguous: 4 lanes cover 128 bytes of a row; else lanes along the rows
  const int r = blockIdx.x * 64 + (A.kc ? wave * 16 + (lane >> 2) : lane), g = A.kc ? lane & 3 : wave;
  const int t0 = (int)(blockIdx.x * 64) / ST * ST;
  const int rc = min(r, A.rows - 1);
  // the contraction indices of row r that do not count as zero (a chain of
  // conditions per entry in the place of these bounds was miscompiled by ROCm 7.2)
  const int lo = A.tri ? r : 0;
  const int hi = r >= A.rows ? 0 : A.K;
  for (int q = 0; q < KPB; ++q) {
    const int kb = blockIdx.y * KPB + q;
    if (kb >= A.nkb) break;
    if (A.tri && kb * 32 + 32 <= t0) continue;  // read by no tile
    const int l0 = kb * 32 + g * 8;
    float x[8];
    if (A.kc && A.vec && l0 + 8 <= A.K) {
      const float4 a = *(const float4*)(src + (int64_t)rc * A.ld + l0), b = *(const float4*)(src + (int64_t)rc * A.ld + l0 + 4);
      x[0] = a.x, x[1] = a.y, x[2] = a.z, x[3] = a.w, x[4] = b.x, x[5] = b.y, x[6] = b.z, x[7] = b.w;
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int l = min(l0 + e, A.K - 1);
        x[e] = src[A.kc ? (int64_t)rc * A.ld + l : (int64_t)l * A.ld + rc];
      }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = l0 + e >= lo && l0 + e < hi ? x[e] : 0.f;
    u32x4 h, m, l;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      uint32_t hh, mm, ll;
      split2(x[2 * e], x[2 * e + 1], hh, mm, ll);
      h[e] = hh;
      m[e] = mm;
      l[e] = ll;
    }
    uint8_t* d = A.dst + ((int64_t)(kb * 4 + g) * A.rp + r) * 16;
    *(u32x4*)d = h;
    *(u32x4*)(d + A.plane) = m;
    *(u32x4*)(d + 2 * A.plane) = l;
  }
}

struct SplitArgs {
  // packed operands of up to two products (dual: blockIdx.y selects)
  const uint8_t* pr[2];  // rows operand (A), mp rows
  const uint8_t* pc[2];  // columns operand (B), np rows
  int64_t plane_r[2], plane_c[2];
  float* C[2];
  int64_t ldc;
  int M, N, mp, np;
  int K[2];       // padded to 64
  float alpha[2], beta;
  int tri, klo, dual, vec;
  int ngc, ngr;   // groups of 4 tile columns, of 8 tile rows
  int rot;        // second product of a dual one: its first group's XCD is 8 - rot
};

// Tile of a workgroup.  An XCD takes groups of 8 x 4 tiles (its 32 CUs: 12 operand
// panels for 32 tiles in its L2), by column group: with KLO_COL (K range [j0, K)) the
// first are the longest.  A dual product's second part goes on with the XCD after
// the last group of the first (2048 x 5120: five XCDs had two groups each).
__device__ inline bool split_tile(const SplitArgs& A, int* ti, int* tj) {
  const int x = (blockIdx.x + (A.dual ? blockIdx.y * A.rot : 0)) % 8, y = blockIdx.x / 8;
  int g = (y / 32) * 8 + x;
  const int in = y % 32;
  int gc, gr;
  if (A.tri == TRI_UPPER) {
    // column group c holds the row groups 0 .. (4 c + 3) / 8
    gc = 0;
    while (gc < A.ngc && g >= gc / 2 + 1) g -= gc++ / 2 + 1;
    if (gc >= A.ngc) return false;
    gr = g;
  } else {
    if (g >= A.ngc * A.ngr) return false;
    gc = g / A.ngr;
    gr = g % A.ngr;
  }
  *ti = gr * 8 + in % 8;
  *tj = gc * 4 + in / 8;
  return *ti * ST < A.M && *tj * ST < A.N && (A.tri != TRI_UPPER || *ti <= *tj);
}

// 256 x 256 tile per 512-thread workgroup, the part of a wave 128 columns x 64
// rows (the tile's columns as the MFMA's rows, so that a lane holds four
// consecutive entries of a row of C).  Bound: MFMA issue and the clock under that
// load, and C (read and written by all CUs at about the same time): 8192 x 10240, K =
// 1024, two products with their packing 1.57 ms, 218 TFLOP/s of fp32 flop, where the
// fp32 matrix instructions take 2.63 ms.  Error against 64 bits of the weights of a
// whole solve, from the same 32-bit L, G and a (fp32 instructions, here): k = 8192 1.29e-6,
// 1.10e-6; k = 11008 1.76e-6, 1.48e-6; k = 14336 2.31e-6, 1.93e-6.
__global__ __launch_bounds__(512) void split_gemm_kernel(SplitArgs A) {
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];  // [stage parity][columns 0, 1, rows 0, 1]
  int ti, tj;
  if (!split_tile(A, &ti, &tj)) return;
  const int pb = A.dual ? (int)blockIdx.y : 0;
  const int i0 = ti * ST, j0 = tj * ST;
  const int klo = A.klo == KLO_COL ? j0 : 0, khi = A.K[pb];
  int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int wi = wave >> 2, wj = wave & 3;
  f4 acc[8][4];
#pragma unroll
  for (int a = 0; a < 8; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[a][b] = f4{0.f, 0.f, 0.f, 0.f};
  if (klo < khi) {  // uniform
    // Loads: wave w fills plane w of a unit (k block w / 4 of the stage, group
    // w % 4), 64 unit rows per load; unit row u is tile column 128 (u / 64) + 64 h + u % 64
    // for half h, tile row 64 (u / 32) + 32 h + u % 32.
    const int uw = __builtin_amdgcn_readfirstlane(wave);
    const uint8_t* const uc = A.pc[pb] + ((int64_t)(klo / 8 + uw) * A.np + j0) * 16;
    const uint8_t* const ur = A.pr[pb] + ((int64_t)(klo / 8 + uw) * A.mp + i0) * 16;
    const int64_t kc = (int64_t)A.np * 128, kr = (int64_t)A.mp * 128;  // bytes per 64 k
    const int64_t plc = A.plane_c[pb], plr = A.plane_r[pb];
    const uint32_t lc = lane * 16, lr = (64 * (lane >> 5) + (lane & 31)) * 16;
    const int nst = (khi - klo) / 64 * 6;
    // the six terms of a 64-k block: plane of the columns, of the rows (0 h, 1 m, 2 l)
    constexpr uint32_t PC = 2 | 0 << 2 | 1 << 4 | 1 << 6 | 0 << 8 | 0 << 10;
    constexpr uint32_t PR = 0 | 2 << 2 | 1 << 4 | 0 << 6 | 1 << 8 | 0 << 10;
    auto issue = [&](int op, int st, int par) {
      const int sc = min(st, nst - 1), kb = sc / 6, t = 2 * (sc - 6 * kb);
      const uint8_t* u = op < 2 ? uc + kb * kc + (PC >> t & 3) * plc + op * 1024
                                : ur + kb * kr + (PR >> t & 3) * plr + (op - 2) * 512;
      uint8_t* dst = smem + (par * 4 + op) * kUnit + uw * 2048;
#pragma unroll
      for (int j = 0; j < 2; ++j)
        __builtin_amdgcn_global_load_lds((const void*)(u + j * 2048 + (op < 2 ? lc : lr)),
                                         (__attribute__((address_space(3))) void*)(dst + j * 1024), 16, 0, 0);
    };
    const uint32_t fa = (uint32_t)((lane >> 4) * 2048 + (wi * 64 + (lane & 15)) * 16);
    const uint32_t fb = (uint32_t)((lane >> 4) * 2048 + (wj * 32 + (lane & 15)) * 16);
    auto read_a = [&](int par, int h, u32x4 (&F)[2][4]) {
      const uint8_t* p = smem + (par * 4 + h) * kUnit + fa;
#pragma unroll
      for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
        for (int a = 0; a < 4; ++a) F[s2][a] = *(const u32x4*)(p + s2 * 8192 + a * 256);
    };
    auto read_b = [&](int par, int h, u32x4 (&F)[2][2]) {
      const uint8_t* p = smem + (par * 4 + 2 + h) * kUnit + fb;
#pragma unroll
      for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
        for (int b = 0; b < 2; ++b) F[s2][b] = *(const u32x4*)(p + s2 * 8192 + b * 256);
    };
    pp::pp_loop<4, 2, 2>(nst, acc, issue, read_a, read_b);
  }
  // C = beta C + alpha acc; element r of block (a, b) is row 64 wj + 16 b + lane % 16,
  // column 128 wi + 16 a + 4 (lane / 16) + r
  float* C = A.C[pb] + (int64_t)i0 * A.ldc + j0;
  const float al = A.alpha[pb], be = A.beta;
  const int rows = min(ST, A.M - i0), cols = min(ST, A.N - j0);
  const int r0 = wj * 64 + (lane & 15), c0 = wi * 128 + 4 * (lane >> 4);
  if (A.vec) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      float4 c[2][8];
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int a = 0; a < 8; ++a) {
          const int row = r0 + 32 * h + 16 * b, col = c0 + 16 * a;
          c[b][a] = make_float4(0.f, 0.f, 0.f, 0.f);
          if (be != 0.f && row < rows && col < cols) c[b][a] = *(const float4*)(C + row * A.ldc + col);
        }
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int a = 0; a < 8; ++a) {
          const int row = r0 + 32 * h + 16 * b, col = c0 + 16 * a;
          const f4 v = acc[a][2 * h + b];
          const float4 o = c[b][a];
          if (row < rows && col < cols)
            *(float4*)(C + row * A.ldc + col) = make_float4(fmaf(be, o.x, al * v[0]), fmaf(be, o.y, al * v[1]),
                                                            fmaf(be, o.z, al * v[2]), fmaf(be, o.w, al * v[3]));
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
        if (row < rows && col < cols) {
          float* p = C + row * A.ldc + col;
          *p = be != 0.f ? fmaf(be, *p, al * acc[a][b][r]) : al * acc[a][b][r];
        }
      }
}

bool al16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

size_t packed_bytes(int64_t rows, int64_t K) { return (size_t)rup(rows, ST) * rup(K, 64) * 6; }

duo_status pack(const float* src, int64_t ld, int kc, int rows, int K, int tri, uint8_t* dst, hipStream_t s) {
  PackArgs p{};
  p.src = src;
  p.ld = ld;
  p.kc = kc;
  p.rows = rows;
  p.K = K;
  p.rp = (int)rup(rows, ST);
  p.nkb = (int)rup(K, 64) / 32;
  p.tri = tri;
  p.vec = al16(src) && ld % 4 == 0;
  p.dst = dst;
  p.plane = (int64_t)p.rp * p.nkb * 64;
  hipLaunchKernelGGL(pack_kernel, dim3((unsigned)(p.rp / 64), (unsigned)cdiv(p.nkb, KPB)), dim3(256), 0, s, p);
  DUO_LAUNCH_CHECK();
  return DUO_OK;
}

}  // namespace

// Tiles that the fullest XCD takes of a whole (not triangular) product's.
static int64_t xcd_tiles(int64_t M, int64_t N, int np) {
  const int64_t tm = cdiv(M, ST), tn = cdiv(N, ST);
  int64_t x[8] = {}, g = 0;
  for (int p = 0; p < np; ++p)
    for (int64_t c = 0; c < tn; c += 4)
      for (int64_t r = 0; r < tm; r += 8) x[g++ % 8] += std::min<int64_t>(8, tm - r) * std::min<int64_t>(4, tn - c);
  return *std::max_element(x, x + 8);
}

// Whether a product takes this path: its time by measured rates against that of
// gemm_f32.  Packing moves 10 bytes per element at 4 TB/s, 6 us per launch.
// Two products in one launch (K = 1024, n x N each): a round of the 32 CUs of an XCD
// takes 8.3 us per 64 k, against 105 TFLOP/s and a launch: measured 2048 x 5120 345
// and 370 us, 2560 x 4096 295 and 372, but 1536 x 5120 289 and 283, 2304 x 3072 276 and 260;
// of 143 sizes from 512 x 1024 to 8192 x 10240 these take the slower path at three, by 2 %
// at most.  In the sweep, where C has left the caches, the path lost up to 2 % of
// whole solves at k = 6144 where it should have gained 10 % of the product: hence the 1.2.
// (Solves at n = 2048: k = 6144 3.48 -> 3.37 ms, 8192 5.80 -> 5.19, 9216 7.20 -> 6.18.)
// The score product (upper tiles, shrinking sums): 8.6 us per 64 k and 22 us per
// round of 256 tiles, the last tile to finish may be the one with the longest sum,
// against 110 TFLOP/s: k = 4096 405 and 252 us, 8192 1204 and 1444, 11008 2426 and 3408.
static bool split_pays(const GemmDesc& d) {
  if (d.inplace || d.batch > 1 || (d.nterms == 2 && !d.dual)) return false;
  const int np = d.dual ? 2 : 1;
  const int64_t K = d.t[0].K;
  for (int i = 0; i < np; ++i)
    if (!d.t[i].a_row || d.t[i].K != K || K < 256) return false;
  const double pack = 10.0 / 4e12, launch = 6e-6, step = (double)cdiv(K, 64);
  if (d.tri == TRI_ALL && d.t[0].klo == KLO_ZERO && d.t[0].khi == KHI_FULL) {
    const double split = (double)cdiv(xcd_tiles(d.M, d.N, np), 32) * step * 8.3e-6 +
                         np * ((double)(d.M + d.N) * K * pack + 2 * launch);
    return 1.2 * split < 2.0 * np * d.M * d.N * K / 105e12 + launch;
  }
  if (d.tri == TRI_UPPER && d.t[0].klo == KLO_COL && d.t[0].khi == KHI_FULL && np == 1) {
    const int64_t tm = cdiv(d.M, ST), tiles = tm * (tm + 1) / 2;
    const double sum_k = (double)tiles / 3.0 * K;
    const double split = std::max(sum_k / 256.0, (double)K) / 64.0 * 8.6e-6 + (double)cdiv(tiles, 256) * 22e-6 +
                         0.75 * (d.M + d.N) * K * pack + 2 * launch;
    return split < (double)d.M * d.N / 3.0 * K / 110e12 + launch;
  }
  return false;
}

size_t split_bytes(const GemmDesc& d) {
  if (!split_pays(d)) return 0;
  return (packed_bytes(d.M, d.t[0].K) + packed_bytes(d.N, d.t[0].K)) * (d.dual ? 2 : 1);
}

duo_status gemm_f32_split(const GemmDesc& d, void* pk, size_t pk_bytes, hipStream_t s) {
  const int np = d.dual ? 2 : 1;
  const size_t need = split_bytes(d);
  if (need == 0 || need > pk_bytes) return gemm_f32(d, s);
  SplitArgs A{};
  uint8_t* at = (uint8_t*)pk;
  const bool tri = d.tri == TRI_UPPER;
  for (int i = 0; i < np; ++i) {
    const GemmTerm& t = d.t[i];
    A.pr[i] = at;
    if (duo_status st = pack(t.A, t.lda, 1, d.M, t.K, tri, at, s); st != DUO_OK) return st;
    at += packed_bytes(d.M, t.K);
    A.pc[i] = at;
    if (duo_status st = pack(t.B, t.ldb, !t.b_row, d.N, t.K, tri, at, s); st != DUO_OK) return st;
    at += packed_bytes(d.N, t.K);
    A.K[i] = (int)rup(t.K, 64);
    A.plane_r[i] = (int64_t)rup(d.M, ST) * A.K[i] * 2;
    A.plane_c[i] = (int64_t)rup(d.N, ST) * A.K[i] * 2;
    A.alpha[i] = t.alpha;
  }
  A.C[0] = d.C;
  A.C[1] = d.C2;
  A.ldc = d.ldc;
  A.M = d.M;
  A.N = d.N;
  A.mp = (int)rup(d.M, ST);
  A.np = (int)rup(d.N, ST);
  A.beta = d.beta;
  A.tri = d.tri;
  A.klo = d.t[0].klo;
  A.dual = d.dual;
  A.vec = d.ldc % 4 == 0 && d.N % 4 == 0 && al16(d.C) && (!d.dual || al16(d.C2));
  A.ngc = (int)cdiv(cdiv(d.N, ST), 4);
  A.ngr = (int)cdiv(cdiv(d.M, ST), 8);
  int64_t groups = (int64_t)A.ngc * A.ngr;
  if (tri) {
    groups = 0;
    for (int c = 0; c < A.ngc; ++c) groups += c / 2 + 1;
  }
  A.rot = (int)(8 - groups % 8) % 8;
  if (duo_status st = set_max_lds((const void*)split_gemm_kernel, kLds); st != DUO_OK) return st;
  hipLaunchKernelGGL(split_gemm_kernel, dim3((unsigned)(rup(groups, 8) * 32), (unsigned)np), dim3(512), kLds, s, A);
  DUO_LAUNCH_CHECK();
  return DUO_OK;
}

}  // namespace duo
