// Layer outputs straight from the stored codes and the two frames: Y = X Theta^T with
// Theta^ = P_out diag(scale) (q - zero) P_in^T (appendix "Computational Complexity during
// Inference"), taken in the order of Sec. 3 "Inference Procedure" (analysis operator on
// the inputs, the quantized D^, synthesis operator):
//   U = X P_in            (tokens x K_in)
//   V = U (q - zero)^T S  (tokens x K_out; the 2-bit codes decoded on the fly)
//   Y = V P_out^T         (tokens x d_out)
// for small token counts (decode, small batches), where every step streams its operand
// from HBM once: P_in (d_in x K_in fp32), the packed codes, P_out (d_out x K_out fp32).
// With dense frames tokens go through in blocks of at most 8; all products are those of
// fp32 values, with fp32 accumulation (the split-K partials of U are summed in fp64).
#include "fq_internal.h"
#include "codes_layout.h"

#include <algorithm>

namespace fq {
namespace {

constexpr int AT = 256;        // threads per work-group in every kernel here

template <typename T>
__device__ __forceinline__ float to_f32(T v);
template <>
__device__ __forceinline__ float to_f32<float>(float v) { return v; }
template <>
__device__ __forceinline__ float to_f32<uint16_t>(uint16_t v) {   // bf16
  return __uint_as_float((uint32_t)v << 16);
}
template <>
__device__ __forceinline__ float to_f32<_Float16>(_Float16 v) { return (float)v; }

// ---- step 1: part[s][t][j] = sum over k in split s of X[t][k] P_in[k][j]
// grid (ceil(K_in / (4 AT)), ksplit); a thread owns 4 consecutive columns.
template <typename XT, int NT, bool VEC>
__global__ __launch_bounds__(AT) void k_apply_in(const XT* __restrict__ X, int64_t ldx, int nt,
                                                 int64_t d_in, const float* __restrict__ P,
                                                 int64_t K_in, int kper,
                                                 float* __restrict__ part) {
  __shared__ float xs[NT][256];
  const int s = blockIdx.y;
  const int64_t k0 = (int64_t)s * kper;
  const int kn = (int)min((int64_t)kper, d_in - k0);
  for (int e = threadIdx.x; e < NT * kper; e += AT) {
    const int t = e / kper, k = e % kper;
    xs[t][k] = (t < nt && k < kn) ? to_f32<XT>(X[t * ldx + k0 + k]) : 0.f;
  }
  __syncthreads();
  const int64_t j = ((int64_t)blockIdx.x * AT + threadIdx.x) * 4;
  if (j >= K_in) return;
  float acc[NT][4];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[t][q] = 0.f;
  const float* p = P + k0 * K_in + j;
  for (int k = 0; k < kn; ++k, p += K_in) {
    float v[4];
    if (VEC) {
      const float4 w = *reinterpret_cast<const float4*>(p);
      v[0] = w.x; v[1] = w.y; v[2] = w.z; v[3] = w.w;
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] = (j + q < K_in) ? p[q] : 0.f;
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const float x = xs[t][k];
#pragma unroll
      for (int q = 0; q < 4; ++q) acc[t][q] = fmaf(x, v[q], acc[t][q]);
    }
  }
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (j + q < K_in) part[((int64_t)s * NT + t) * K_in + j + q] = acc[t][q];
}

// U[t][j] = sum over the splits (fp64), stored for the code product (codes_layout.h); columns
// [K_in, kpad) are 0.  grid (ceil(kpad / 64), nt): a work-group owns 64 columns of one token;
// its 4 waves sum every 4th split and combine through LDS in a fixed order.
template <int BITS>
__global__ __launch_bounds__(AT) void k_apply_in_reduce(const float* __restrict__ part, int nt_blk,
                                                        int ksplit, int64_t K_in, int64_t kpad,
                                                        int64_t quads, int ncol,
                                                        uint16_t* __restrict__ Uf) {
  __shared__ double red[AT / 64][64];
  const int lane = threadIdx.x & 63, g = threadIdx.x >> 6;
  const int t = blockIdx.y;
  const int64_t j = (int64_t)blockIdx.x * 64 + lane;
  double acc = 0.0;
  if (j < K_in) {
    const float* p = part + (int64_t)t * K_in + j;
    const int64_t step = (int64_t)nt_blk * K_in;
#pragma unroll 8
    for (int s = g; s < ksplit; s += AT / 64) acc += p[s * step];
  }
  red[g][lane] = acc;
  __syncthreads();
  if (g == 0 && j < kpad)
    codes_put_f<BITS>(Uf, quads, ncol, t, j,
                      (float)(red[0][lane] + red[1][lane] + red[2][lane] + red[3][lane]));
}

// ---- step 2: V[t][i] = scale_i (sum_j U[t][j] q_ij - zero_i sum_j U[t][j])
// (the same sum as sum_j U[t][j] (q_ij - zero_i); both forms have error bounds of the
// same size, since |q|, |q - zero| <= 3 (15)) on the matrix cores.  The codes are exact in
// bf16 and every fp32 U[t][j] is the exact sum of three bf16 values, so the products are
// exact and only the fp32 sums round.
// A work-group of CW waves owns 16 RT - 1 code rows and one tile of U's columns (the token
// triples of codes_layout.h) and splits the reduction over its waves, step by step of 16
// words a row; a wave reads its codes (4 words a lane and row, one step ahead) and its
// pieces of U (a step's together) straight into the fragments of v_mfma_f32_16x16x32_bf16.
// The last of the 16 RT rows is a row of codes 1, which gives sum_j U[t][j].  The waves' sums
// meet in LDS in a fixed order, which the choice of RT does not change.
// Bound by load latency at a few tokens (8.8 us for one token, 12112 x 4512, 13.7 MB of codes)
// and by reading U's pieces from L2 beyond; 61 tokens, 4512 x 4512: 22 us, where blocks of
// 8 tokens on the vector unit took 8 x 23.  One tile a work-group: more tiles share the
// unpacked codes, but with 2 to 5 of them the registers leave too few waves to cover the
// loads (61 tokens 22-25 us, 80 tokens 28-31 against 26).
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float fx4 __attribute__((ext_vector_type(4)));
typedef int ix4 __attribute__((ext_vector_type(4)));
constexpr int CW = 8;          // waves per work-group of the code products

// 8 codes (piece h of a word) as bf16.  2 bits: a nibble 00qq read as fp4 (e2m1) is q / 2, so a
// conversion with scale 2 unpacks a byte, two codes, exactly; the nibbles of (word >> 2 b) &
// 0x33333333, b = 0, 1, hold codes b, b + 2, b + 4, ...  (0.7 instructions a code; table
// lookups with v_perm take 1.4.)  4 bits: a byte 0000qqqq read as fp8 (e4m3) is q 2^-9 (its
// subnormals and its first binade have one spacing), so a conversion with scale 512 unpacks two
// codes exactly, one instruction a code.  (By way of v_cvt_f32_ubyte and v_perm, two: one token,
// 9008 x 31536, whole call 95 us; 75 us so, 73 us on the vector unit.)
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
template <int BITS>
__device__ __forceinline__ uint4 codes_bf16(uint32_t w, int h) {
  uint4 o;
  if constexpr (BITS == 2) {
    const uint32_t y = (w >> (2 * h)) & 0x33333333u;
    o.x = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(y, 2.0f, 0));
    o.y = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(y, 2.0f, 1));
    o.z = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(y, 2.0f, 2));
    o.w = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(y, 2.0f, 3));
  } else {
    uint32_t q[4];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const uint32_t y = (w >> (4 * b)) & 0x0F0F0F0Fu;
      q[2 * b] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(y, 512.0f, 0));
      q[2 * b + 1] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(y, 512.0f, 1));
    }
    o = make_uint4(q[0], q[1], q[2], q[3]);
  }
  return o;
}

// the four words of quad qc of a code row (words beyond the row repeat its last one: U is 0
// there); whole: no quad of this wave's step is cut by the end of the row.  Rows are only
// word aligned, which a 16-byte load of this type allows for.
typedef uint32_t u32x4u __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ void load_quad(const uint32_t* __restrict__ row, int64_t qc,
                                          int64_t nwords, bool whole, uint32_t (&w)[4]) {
  if (whole) {
    const u32x4u v = *reinterpret_cast<const u32x4u*>(row + qc * 4);
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = v[i];
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = row[min(qc * 4 + i, nwords - 1)];
  }
}

// V's position of code row i: itself, or (rho > 0) the block order of the synthesis that
// reads it, complex subspace s = i / rho of block (i mod rho) / 2
__device__ __forceinline__ int64_t v_index(int64_t i, int rho, int64_t k) {
  if (rho <= 0) return i;
  const int64_t s = i / rho;
  const int w = (int)(i - s * rho);
  return ((int64_t)(w >> 1) * k + s) * 2 + (w & 1);
}

template <int BITS, int RT>
__global__ __launch_bounds__(64 * CW) void k_apply_codes(const uint16_t* __restrict__ Uf, int ncol,
                                                         int nt, int64_t quads,
                                                         const uint32_t* __restrict__ codes,
                                                         int64_t K_out, int64_t nwords,
                                                         const float* __restrict__ scale,
                                                         const float* __restrict__ zero,
                                                         float* __restrict__ V, int64_t ldv,
                                                         int vrho, int64_t vk) {
  constexpr int CPW = 32 / BITS, NP = CPW / 8, P = 4 * NP;   // pieces of 8 codes a word, a quad
  constexpr int ROWS = 16 * RT - 1;
  __shared__ float red[CW][16 * RT][17];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int c = lane & 15, g = lane >> 4;
  const int64_t row0 = (int64_t)blockIdx.x * ROWS;
  const int tile = (int)blockIdx.y;
  const uint32_t* crow[RT];
#pragma unroll
  for (int r = 0; r < RT; ++r) crow[r] = codes + min(row0 + 16 * r + c, K_out - 1) * nwords;
  const bool ones = c == 15;         // of the last row tile
  const bool live = c < ncol;        // this lane's column of the tile exists
  const uint16_t* ub = Uf + (int64_t)tile * quads * (4 * CPW) * 16 + (live ? c : 0) * 8;
  fx4 acc[RT];
#pragma unroll
  for (int r = 0; r < RT; ++r) acc[r] = fx4{0.f, 0.f, 0.f, 0.f};
  const int64_t nsteps = (quads + 3) / 4;
  uint32_t wd[RT][4], wn[RT][4];
  auto fetch = [&](int64_t st, uint32_t (&w)[RT][4]) {
    const bool whole = (st * 4 + 4) * 4 <= nwords;
    const int64_t qc = min(st * 4 + g, quads - 1);
#pragma unroll
    for (int r = 0; r < RT; ++r) load_quad(crow[r], qc, nwords, whole, w[r]);
#pragma unroll
    for (int i = 0; i < 4; ++i) w[RT - 1][i] = ones ? (BITS == 2 ? 0x55555555u : 0x11111111u) : w[RT - 1][i];
  };
  if (wave < nsteps) fetch(wave, wd);
  for (int64_t st = wave; st < nsteps; st += CW) {
    const int64_t quad = st * 4 + g;
    const bool in = live && quad < quads;             // beyond: U is 0
    const uint16_t* uq = ub + min(quad, quads - 1) * (4 * CPW) * ncol;
    uint4 bu[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
      bu[p] = make_uint4(0u, 0u, 0u, 0u);
      if (in) bu[p] = *reinterpret_cast<const uint4*>(uq + (int64_t)p * ncol * 8);
    }
    if (st + CW < nsteps) fetch(st + CW, wn);
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
      for (int r = 0; r < RT; ++r)
        acc[r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
            __builtin_bit_cast(bf16x8, codes_bf16<BITS>(wd[r][p / NP], p % NP)),
            __builtin_bit_cast(bf16x8, bu[p]), acc[r], 0, 0, 0);
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
      for (int i = 0; i < 4; ++i) wd[r][i] = wn[r][i];
  }
  // accumulator layout: value v of lane l is row 4 (l / 16) + v, column l % 16
#pragma unroll
  for (int r = 0; r < RT; ++r)
#pragma unroll
    for (int v = 0; v < 4; ++v) red[wave][16 * r + 4 * g + v][c] = acc[r][v];
  __syncthreads();
  for (int e = threadIdx.x; e < ROWS * CODES_TOK_F; e += 64 * CW) {
    const int q = e / ROWS, r = e - q * ROWS;
    const int t = tile * CODES_TOK_F + q;
    const int64_t i = row0 + r;
    if (t >= nt || i >= K_out) continue;
    float sum = 0.f, us = 0.f;
#pragma unroll
    for (int w = 0; w < CW; ++w) {
      sum += (red[w][r][3 * q + 2] + red[w][r][3 * q + 1]) + red[w][r][3 * q];
      us += (red[w][ROWS][3 * q + 2] + red[w][ROWS][3 * q + 1]) + red[w][ROWS][3 * q];
    }
    V[(int64_t)t * ldv + v_index(i, vrho, vk)] = scale[i] * fmaf(-zero[i], us, sum);
  }
}

// ---- rounded activations (appendix "FrameQuant for Activation Quantization?"): per token
// t, Delta_t = max_j |U[t][j]| / qmax and Cq[t][j] = round(U[t][j] / Delta_t) (IEEE fp32
// divisions, ties to even; Delta_t = 0 gives a zero row).  One 1024-thread work-group per
// token.
// BITS 2 or 4 stores the bytes for the code product (codes_layout.h), columns [K, kpad) 0;
// BITS = 0 stores column j of row t at byte t K + j.
// csum (optional) receives sum_j Cq[t][j].
constexpr int QT = 1024;       // threads per token in the activation rounding kernel

template <int BITS>
__global__ __launch_bounds__(QT) void k_act_quantize(const float* __restrict__ U, int64_t ldu,
                                                     int64_t K, float qmax,
                                                     int8_t* __restrict__ Cq, int64_t kpad,
                                                     int64_t quads, int ncol,
                                                     float* __restrict__ delta,
                                                     int* __restrict__ csum) {
  __shared__ float wmax[QT / 64];
  __shared__ int wsum[QT / 64];
  const int64_t t = blockIdx.x;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const float* u = U + t * ldu;
  float mx = 0.f;
#pragma unroll 4
  for (int64_t j = threadIdx.x; j < K; j += QT) mx = fmaxf(mx, fabsf(u[j]));
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
  if (lane == 0) wmax[wave] = mx;
  __syncthreads();
  mx = 0.f;
#pragma unroll
  for (int w = 0; w < QT / 64; ++w) mx = fmaxf(mx, wmax[w]);
  const float dl = mx / qmax;
  int sum = 0;
  const int tile = (int)t / CODES_TOK_I, col = (int)t - tile * CODES_TOK_I;
#pragma unroll 4
  for (int64_t j = threadIdx.x; j < kpad; j += QT) {
    int q = 0;
    if (j < K && dl > 0.f) q = (int)rintf(u[j] / dl);
    sum += q;
    int64_t dst = t * K + j;
    if constexpr (BITS > 0)
      dst = (int64_t)tile * quads * (4 * (32 / BITS)) * 16 + codes_index<BITS, 16>(j, ncol, col);
    Cq[dst] = (int8_t)q;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
  if (lane == 0) wsum[wave] = sum;
  __syncthreads();
  if (threadIdx.x == 0) {
    delta[t] = dl;
    if (csum) {
      int total = 0;
      for (int w = 0; w < QT / 64; ++w) total += wsum[w];
      csum[t] = total;
    }
  }
}

// V[t][i] = scale_i Delta_t (sum_j Cq[t][j] q_ij - zero_i sum_j Cq[t][j]) for BITS-bit codes
// (2 or 4), the dot product exact in int32 (|sum| <= (2^BITS - 1) * 127 * K_in) and
// converted to float at the end: k_apply_codes with v_mfma_i32_16x16x64_i8, one column a
// token, a word's spread bytes being the operand as they are.
template <int BITS, int RT>
__global__ __launch_bounds__(64 * CW) void k_apply_codes_i8(
    const int8_t* __restrict__ Cq, int ncol, int nt, int64_t quads,
    const float* __restrict__ delta, const int* __restrict__ csum,
    const uint32_t* __restrict__ codes, int64_t K_out, int64_t nwords,
    const float* __restrict__ scale, const float* __restrict__ zero, float* __restrict__ V,
    int64_t ldv, int vrho, int64_t vk) {
  constexpr int CPW = 32 / BITS, NB = CPW / 4;
  constexpr int NPC = 4 * CPW / 16;                 // pieces of 16 codes a quad
  constexpr uint32_t MASK = BITS == 2 ? 0x03030303u : 0x0F0F0F0Fu;
  __shared__ int red[CW][16 * RT][17];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int c = lane & 15, g = lane >> 4;
  const int64_t row0 = (int64_t)blockIdx.x * (16 * RT);
  const int tile = (int)blockIdx.y;
  const uint32_t* crow[RT];
#pragma unroll
  for (int r = 0; r < RT; ++r) crow[r] = codes + min(row0 + 16 * r + c, K_out - 1) * nwords;
  const bool live = c < ncol;
  const int8_t* ub = Cq + (int64_t)tile * quads * (4 * CPW) * 16 + (live ? c : 0) * 16;
  ix4 acc[RT];
#pragma unroll
  for (int r = 0; r < RT; ++r) acc[r] = ix4{0, 0, 0, 0};
  const int64_t nsteps = (quads + 3) / 4;
  uint32_t wd[RT][4], wn[RT][4];
  auto fetch = [&](int64_t st, uint32_t (&w)[RT][4]) {
    const bool whole = (st * 4 + 4) * 4 <= nwords;
    const int64_t qc = min(st * 4 + g, quads - 1);
#pragma unroll
    for (int r = 0; r < RT; ++r) load_quad(crow[r], qc, nwords, whole, w[r]);
  };
  if (wave < nsteps) fetch(wave, wd);
  for (int64_t st = wave; st < nsteps; st += CW) {
    const int64_t quad = st * 4 + g;
    const bool in = live && quad < quads;
    const int8_t* uq = ub + min(quad, quads - 1) * (4 * CPW) * ncol;
    ix4 bu[NPC];
#pragma unroll
    for (int pc = 0; pc < NPC; ++pc) {
      bu[pc] = ix4{0, 0, 0, 0};
      if (in) bu[pc] = *reinterpret_cast<const ix4*>(uq + (int64_t)pc * ncol * 16);
    }
    if (st + CW < nsteps) fetch(st + CW, wn);
#pragma unroll
    for (int pc = 0; pc < NPC; ++pc)
#pragma unroll
      for (int r = 0; r < RT; ++r) {
        ix4 a;
#pragma unroll
        for (int d = 0; d < 4; ++d)       // dword d: spread d % NB of word (4 pc + d) / NB
          a[d] = (int)((wd[r][(4 * pc + d) / NB] >> (BITS * (d % NB))) & MASK);
        acc[r] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, bu[pc], acc[r], 0, 0, 0);
      }
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
      for (int i = 0; i < 4; ++i) wd[r][i] = wn[r][i];
  }
#pragma unroll
  for (int r = 0; r < RT; ++r)
#pragma unroll
    for (int v = 0; v < 4; ++v) red[wave][16 * r + 4 * g + v][c] = acc[r][v];
  __syncthreads();
  for (int e = threadIdx.x; e < 16 * RT * 16; e += 64 * CW) {
    const int q = e / (16 * RT), r = e - q * (16 * RT);
    const int t = tile * CODES_TOK_I + q;
    const int64_t i = row0 + r;
    if (t >= nt || i >= K_out) continue;
    int sum = 0;
#pragma unroll
    for (int w = 0; w < CW; ++w) sum += red[w][r][q];
    V[(int64_t)t * ldv + v_index(i, vrho, vk)] =
        scale[i] * delta[t] * fmaf(-zero[i], (float)csum[t], (float)sum);
  }
}

// ---- step 3: Y[t][o] = sum_i V[t][i] P_out[o][i]
// A work-group owns R output rows; a thread owns 4 consecutive columns of every 4 AT-wide
// chunk of P_out's rows (each V element is read once per work-group).
template <int NT, int R, bool VEC>
__global__ __launch_bounds__(AT) void k_apply_out(const float* __restrict__ V, int nt,
                                                  const float* __restrict__ P, int64_t K_out,
                                                  int64_t d_out, float* __restrict__ Y,
                                                  int64_t ldy) {
  __shared__ float red[AT / 64][R][NT];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t o0 = (int64_t)blockIdx.x * R;
  float acc[R][NT];
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[r][t] = 0.f;
  const float* prow[R];
#pragma unroll
  for (int r = 0; r < R; ++r) prow[r] = P + min(o0 + r, d_out - 1) * K_out;
  for (int64_t i = (int64_t)threadIdx.x * 4; i < K_out; i += AT * 4) {
    float v[NT][4];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      if (VEC) {
        const float4 w = *reinterpret_cast<const float4*>(V + t * K_out + i);
        v[t][0] = w.x; v[t][1] = w.y; v[t][2] = w.z; v[t][3] = w.w;
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) v[t][q] = (i + q < K_out) ? V[t * K_out + i + q] : 0.f;
      }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      float p[4];
      if (VEC) {
        const float4 w = *reinterpret_cast<const float4*>(prow[r] + i);
        p[0] = w.x; p[1] = w.y; p[2] = w.z; p[3] = w.w;
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) p[q] = (i + q < K_out) ? prow[r][i + q] : 0.f;
      }
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[r][t] = fmaf(v[t][q], p[q], acc[r][t]);
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1)
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int t = 0; t < NT; ++t) acc[r][t] += __shfl_xor(acc[r][t], o);
  if (lane == 0)
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int t = 0; t < NT; ++t) red[wave][r][t] = acc[r][t];
  __syncthreads();
  if (threadIdx.x < R * NT) {
    const int r = threadIdx.x / NT, t = threadIdx.x % NT;
    const int64_t o = o0 + r;
    if (o < d_out && t < nt) {
      float sum = 0.f;
#pragma unroll
      for (int w = 0; w < AT / 64; ++w) sum += red[w][r][t];
      Y[t * ldy + o] = sum;
    }
  }
}

// splits of d_in for step 1: about 64 (enough work-groups to fill the CUs), at least 32
// rows each, at most 256 rows each (the LDS copy of the tokens' X slice)
int apply_ksplit(int64_t d_in) {
  int64_t ks = 64;
  while (ks > 1 && d_in / ks < 32) ks >>= 1;
  if ((d_in + ks - 1) / ks > 256) ks = (d_in + 255) / 256;
  return (int)ks;
}

// Row tiles (16 rows, `ones` of the last one not code rows) per work-group: 3 share U's pieces, 2
// for a single tile of U, whose pieces are few (12112 x 4512: 1 token 10.2 us with 2, 11.0 with 3,
// 12.4 with 1; 80 tokens 72 with 2, 64 with 3, 66 with 4, event timer included), unless 3 need
// one work-group a compute unit where 2 need a short second one (1 token, 4 bits, whole call:
// 9008 x 31536 75 us with 2, 66 with 3; 12112 x 4512, 258 of them with 3: 29 and 30).
int row_tiles(int ntiles, int64_t K_out, int ones) {
  constexpr int64_t UNITS = 256;
  return ntiles == 1 && (K_out <= UNITS * (32 - ones) || K_out > UNITS * (48 - ones)) ? 2 : 3;
}

template <int NT>
hipError_t apply_block(const void* X, int xt, int64_t ldx, int nt, int64_t d_in,
                       const uint32_t* codes, int bits, const float* scale, const float* zero,
                       int64_t K_out, int64_t K_in, const float* P_out, int64_t d_out,
                       const float* P_in, float* Y, const ApplyScratch& w, hipStream_t s) {
  const int ks = apply_ksplit(d_in);
  const int kper = (int)((d_in + ks - 1) / ks);
  const int ks_eff = (int)((d_in + kper - 1) / kper);
  const bool vin = (K_in % 4 == 0) && ((reinterpret_cast<uintptr_t>(P_in) & 15) == 0);
  const bool vout = (K_out % 4 == 0) && ((reinterpret_cast<uintptr_t>(P_out) & 15) == 0);
  const dim3 gin((unsigned)((K_in + 4 * AT - 1) / (4 * AT)), (unsigned)ks_eff);
  prof_begin(s, "apply_in");
#define FQ_APPLY_IN(XT)                                                                          \
  if (vin) hipLaunchKernelGGL((k_apply_in<XT, NT, true>), gin, dim3(AT), 0, s,                    \
                              (const XT*)X, ldx, nt, d_in, P_in, K_in, kper, w.part);            \
  else hipLaunchKernelGGL((k_apply_in<XT, NT, false>), gin, dim3(AT), 0, s,                       \
                          (const XT*)X, ldx, nt, d_in, P_in, K_in, kper, w.part);
  if (xt == 0) { FQ_APPLY_IN(float) }
  else if (xt == 1) { FQ_APPLY_IN(_Float16) }
  else { FQ_APPLY_IN(uint16_t) }
#undef FQ_APPLY_IN
  const int64_t quads = codes_quads(K_in, bits), kpad = quads * 4 * (32 / bits);
  const dim3 gred((unsigned)((kpad + 63) / 64), (unsigned)nt);
  if (bits == 2)
    hipLaunchKernelGGL(k_apply_in_reduce<2>, gred, dim3(AT), 0, s, w.part, NT, ks_eff, K_in, kpad, quads,
                       codes_ncol_f(nt), w.Uf);
  else
    hipLaunchKernelGGL(k_apply_in_reduce<4>, gred, dim3(AT), 0, s, w.part, NT, ks_eff, K_in, kpad, quads,
                       codes_ncol_f(nt), w.Uf);
  prof_end(s);
  if (hipError_t e = apply_codes(w.Uf, nt, bits, codes, K_out, K_in, scale, zero, w.V, K_out, 0, 0, s);
      e != hipSuccess)
    return e;
  prof_begin(s, "apply_out");
  constexpr int R = NT >= 4 ? 8 : 4;
  const dim3 gout((unsigned)((d_out + R - 1) / R));
  if (vout)
    hipLaunchKernelGGL((k_apply_out<NT, R, true>), gout, dim3(AT), 0, s, w.V, nt, P_out, K_out, d_out, Y, d_out);
  else
    hipLaunchKernelGGL((k_apply_out<NT, R, false>), gout, dim3(AT), 0, s, w.V, nt, P_out, K_out, d_out, Y, d_out);
  prof_end(s);
  return last_launch_error();
}

}  // namespace

hipError_t apply_codes(const uint16_t* Uf, int nt, int bits, const uint32_t* codes, int64_t K_out,
                       int64_t K_in, const float* scale, const float* zero, float* V, int64_t ldv,
                       int vrho, int64_t vk, hipStream_t s) {
  if (bits != 2 && bits != 4) return hipErrorInvalidValue;
  const int cpw = 32 / bits;
  const int64_t nwords = (K_in + cpw - 1) / cpw, quads = codes_quads(K_in, bits);
  const int ntiles = (nt + CODES_TOK_F - 1) / CODES_TOK_F;
  const int rt = row_tiles(ntiles, K_out, 1), rows = 16 * rt - 1;
  const dim3 g((unsigned)((K_out + rows - 1) / rows), (unsigned)ntiles);
  prof_begin(s, "apply_codes");
#define FQ_CODES(B, R)                                                                           \
  hipLaunchKernelGGL((k_apply_codes<B, R>), g, dim3(64 * CW), 0, s, Uf, codes_ncol_f(nt), nt, quads, codes, \
                     K_out, nwords, scale, zero, V, ldv, vrho, vk);
  if (bits == 2) { if (rt == 2) { FQ_CODES(2, 2) } else { FQ_CODES(2, 3) } }
  else { if (rt == 2) { FQ_CODES(4, 2) } else { FQ_CODES(4, 3) } }
#undef FQ_CODES
  prof_end(s);
  return last_launch_error();
}

hipError_t act_quantize(const float* U, int64_t ldu, int64_t n, int64_t K, int act_bits,
                        int8_t* Cq, int code_bits, float* delta, int* csum, hipStream_t s) {
  if (n == 0) return hipSuccess;
  const float qmax = (float)((1 << (act_bits - 1)) - 1);
  const dim3 g((unsigned)n);
  const int64_t quads = code_bits > 0 ? codes_quads(K, code_bits) : 0;
  const int64_t kpad = code_bits > 0 ? quads * 4 * (32 / code_bits) : K;
  const int ncol = codes_ncol_i(n);
  prof_begin(s, "act_quantize");
  if (code_bits == 2)
    hipLaunchKernelGGL(k_act_quantize<2>, g, dim3(QT), 0, s, U, ldu, K, qmax, Cq, kpad, quads, ncol, delta, csum);
  else if (code_bits == 4)
    hipLaunchKernelGGL(k_act_quantize<4>, g, dim3(QT), 0, s, U, ldu, K, qmax, Cq, kpad, quads, ncol, delta, csum);
  else
    hipLaunchKernelGGL(k_act_quantize<0>, g, dim3(QT), 0, s, U, ldu, K, qmax, Cq, kpad, quads, ncol, delta, csum);
  prof_end(s);
  return last_launch_error();
}

hipError_t apply_codes_i8(const int8_t* Cq, const float* delta, const int* csum, int nt, int bits,
                          const uint32_t* codes, int64_t K_out, int64_t K_in, const float* scale,
                          const float* zero, float* V, int64_t ldv, int vrho, int64_t vk,
                          hipStream_t s) {
  if (bits != 2 && bits != 4) return hipErrorInvalidValue;
  const int cpw = 32 / bits;
  const int64_t nwords = (K_in + cpw - 1) / cpw, quads = codes_quads(K_in, bits);
  const int ntiles = (nt + CODES_TOK_I - 1) / CODES_TOK_I;
  const int rt = row_tiles(ntiles, K_out, 0);
  const dim3 g((unsigned)((K_out + 16 * rt - 1) / (16 * rt)), (unsigned)ntiles);
  prof_begin(s, "apply_codes");
#define FQ_CODES_I8(B, R)                                                                        \
  hipLaunchKernelGGL((k_apply_codes_i8<B, R>), g, dim3(64 * CW), 0, s, Cq, codes_ncol_i(nt), nt, quads, \
                     delta, csum, codes, K_out, nwords, scale, zero, V, ldv, vrho, vk);
  if (bits == 2) { if (rt == 2) { FQ_CODES_I8(2, 2) } else { FQ_CODES_I8(2, 3) } }
  else { if (rt == 2) { FQ_CODES_I8(4, 2) } else { FQ_CODES_I8(4, 3) } }
#undef FQ_CODES_I8
  prof_end(s);
  return last_launch_error();
}

// tokens a k_apply_in / k_apply_out work-group is built for
static int apply_template_tokens(int nt) { return nt <= 2 ? nt : nt <= 4 ? 4 : 8; }

size_t apply_scratch_floats(int64_t d_in, int64_t K_out, int64_t K_in, int nt, ApplyScratch* w,
                            float* base) {
  const int ks = apply_ksplit(d_in);
  const int64_t kper = (d_in + ks - 1) / ks;
  const int64_t ks_eff = (d_in + kper - 1) / kper;
  const int64_t rows = apply_template_tokens(nt);
  size_t off = 0;
  auto take = [&](size_t n) {
    float* p = base ? base + off : nullptr;
    off += (n + 63) / 64 * 64;
    return p;
  };
  ApplyScratch l{};
  l.nt = nt;
  l.part = take((size_t)(ks_eff * rows * K_in));
  l.Uf = reinterpret_cast<uint16_t*>(take((size_t)((codes_bytes_f(K_in, 2, nt) + 3) / 4)));
  // V goes where the partials were, which are summed by then, unless it is larger
  l.V = K_out <= ks_eff * K_in ? l.part : take((size_t)(rows * K_out));
  if (w) *w = l;
  return off;
}

size_t apply_scratch_least(int64_t d_in, int64_t K_out, int64_t K_in) {
  const int ks = apply_ksplit(d_in);
  const int64_t kper = (d_in + ks - 1) / ks;
  const int64_t ks_eff = (d_in + kper - 1) / kper;
  auto r64 = [](int64_t n) { return (size_t)((n + 63) / 64 * 64); };
  return r64(ks_eff * 8 * K_in) + r64(8 * ((K_in + 15) / 16 * 16)) + r64(8 * K_out);
}

hipError_t frame_apply(const void* X, int xt, int64_t n, int64_t ldx, int64_t d_in,
                       const uint32_t* codes, int bits, const float* scale, const float* zero,
                       int64_t K_out, int64_t K_in, const float* P_out, int64_t d_out,
                       const float* P_in, float* Y, const ApplyScratch& w, hipStream_t s) {
  const int esz = xt == 0 ? 4 : 2;
  for (int64_t t0 = 0; t0 < n; t0 += w.nt) {
    const int nt = (int)std::min<int64_t>(w.nt, n - t0);
    const void* Xb = static_cast<const char*>(X) + t0 * ldx * esz;
    float* Yb = Y + t0 * d_out;
    hipError_t e;
    if (nt == 1)
      e = apply_block<1>(Xb, xt, ldx, nt, d_in, codes, bits, scale, zero, K_out, K_in, P_out, d_out, P_in, Yb, w, s);
    else if (nt == 2)
      e = apply_block<2>(Xb, xt, ldx, nt, d_in, codes, bits, scale, zero, K_out, K_in, P_out, d_out, P_in, Yb, w, s);
    else if (nt <= 4)
      e = apply_block<4>(Xb, xt, ldx, nt, d_in, codes, bits, scale, zero, K_out, K_in, P_out, d_out, P_in, Yb, w, s);
    else
      e = apply_block<8>(Xb, xt, ldx, nt, d_in, codes, bits, scale, zero, K_out, K_in, P_out, d_out, P_in, Yb, w, s);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace fq
