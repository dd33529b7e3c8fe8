// Tight fusion frames applied from their construction instead of a dense d x K matrix
// (Sec. 2.2 "Constructing TFFs" and the appendix "Synopsis of Construction of Tight Fusion
// Frames"; the appendix "Computational Complexity during Inference" counts the cost of
// this route).
//
// The frame is P = (R1 (x) R2) T / sqrt(k) (a Parseval frame), with
//  - T's column block s (rho columns, s < k) the realification of subspace s of a complex
//    (k, rho/2, d/2) frame: row c of the base frame F (c < rho/2) is 1 on the complex
//    coordinates [c m, (c + 1) m), m = d / rho (spectral tetris when d / rho is an integer),
//    modulated by w^(j s), w = exp(2 pi i / k); complex coordinate j is the real pair
//    (2j, 2j+1), complex column c the real pair (2c, 2c+1);
//  - R1 (x) R2 the rotation: a vector of length d read row-major as a d1 x d2 matrix M is
//    mapped to R1 M R2^T.
// Analysis (u = P^T x): z = complex form of R1^T M R2, then
//   u[s rho + 2c] + i u[s rho + 2c + 1] = k^(-1/2) sum_{j < m} conj(w^((c m + j) s)) z[c m + j],
// a length-k DFT of each zero-padded m-block.  Synthesis (y = P v) is its adjoint:
//   z[c m + j] = k^(-1/2) sum_{s < k} w^((c m + j) s) (v[s rho + 2c] + i v[s rho + 2c + 1]),
// then y = R1 Z R2^T.  Work per vector: d (d1 + d2) + 2 d k FMAs instead of d k rho.
#include "fq_internal.h"
#include "codes_layout.h"

#include <algorithm>
#include <cmath>

namespace fq {
namespace {

constexpr int TT = 256;
constexpr int RT = 1024;       // threads of a one-row rotation work-group
constexpr int WT = 512;        // threads of the transform kernels (8 waves)
constexpr int LB = 16;         // k steps of a rotation product in flight per wave

typedef float floatx4 __attribute__((ext_vector_type(4)));

template <typename T>
__device__ __forceinline__ float ld_f32(const T* p);
template <>
__device__ __forceinline__ float ld_f32<float>(const float* p) { return *p; }
template <>
__device__ __forceinline__ float ld_f32<uint16_t>(const uint16_t* p) {   // bf16
  return __uint_as_float((uint32_t)*p << 16);
}
template <>
__device__ __forceinline__ float ld_f32<_Float16>(const _Float16* p) { return (float)*p; }

// tws[t] = exp(2 pi i t / k) for t < k, into LDS (fp32 sincospif of 2t/k: phase error
// below 4e-7 rad)
__device__ __forceinline__ void load_twiddles(float2* tws, int k) {
  for (int t = threadIdx.x; t < k; t += WT) {
    float sn, cs;
    sincospif(2.0f * (float)t / (float)k, &sn, &cs);
    tws[t] = make_float2(cs, sn);
  }
}

// A rotation's inner products (over d1, then over d2) are summed in one order by both of its
// kernels, so that a vector's result is the same bits in any batch: the terms in blocks of four,
// block b in chain b mod 4, a chain one fmaf after the other, the four chains added in order.
// v_mfma_f32_16x16x4_f32 adds its four products to the accumulator in just that way.  View rows
// that only k_rotate takes have one chain.
constexpr int ROT_TILE_MAX = 1008;    // 16 rows of T within 64 KB of LDS
constexpr int RC = 4;
__host__ __device__ inline int rot_chains(int d2) { return d2 <= ROT_TILE_MAX ? RC : 1; }

// LDS floats of rot_tile: T, 16 rows with a pitch that spreads the rows over the banks
__host__ __device__ inline int rot_pitch(int d2) { return (d2 + 15) / 16 * 16 + 4; }
__host__ __device__ inline int64_t rot_lds_floats(int d2) { return (int64_t)16 * rot_pitch(d2); }

// Rows a0 .. a0 + 15 (those below d1) of A M R for one vector, x = M row-major d1 x d2, with
// A(a, i) = L[a][i] (L[i][a] when TL): T = A M (16 x d2, through LDS), then T R, both on
// v_mfma_f32_16x16x4_f32; a wave takes 16-column tiles wave, wave + nwaves, ...  Bound by load
// latency, not by arithmetic (the operands were written by the launch before): the loads of LB k
// steps go out together, those of R's first LB steps before T is waited for.  put(r, b, value)
// receives row a0 + r, column b < d2.  Every thread of the work-group calls it; it begins with
// the LDS free and ends with a barrier.
// 61 vectors of 64 x 64: 5.9 us (10.4 us on the vector unit with the factors broadcast from
// LDS; 8 blocks of 8 vectors, a work-group per row, 50 us).
template <typename XT, bool TL, typename Put>
__device__ __forceinline__ void rot_tile(const XT* __restrict__ x, const float* __restrict__ L,
                                         const float* __restrict__ R, int d1, int d2, int a0,
                                         float* T, Put put) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const int c = lane & 15, g = lane >> 4;
  const int nct = (d2 + 15) / 16, pitch = rot_pitch(d2);
  const int a = a0 + c;
  const bool alive = a < d1;
  const int ac = min(a, d1 - 1);
  auto total = [](const floatx4 (&acc)[RC]) {
    floatx4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < RC; ++q) sum += acc[q];
    return sum;
  };
  float rv[LB];
  const int b0 = min(wave * 16 + c, d2 - 1);
  if (wave < nct) {
#pragma unroll
    for (int u = 0; u < LB; ++u) rv[u] = R[(uint32_t)(min(4 * u + g, d2 - 1) * d2 + b0)];
  }
  for (int jt = wave; jt < nct; jt += nw) {
    const int j = jt * 16 + c, jc = min(j, d2 - 1);
    floatx4 acc[RC] = {};
    for (int i0 = 0; i0 < d1; i0 += 4 * LB) {
      float av[LB], xv[LB];
#pragma unroll
      for (int u = 0; u < LB; ++u) {
        const int i = i0 + 4 * u + g, ic = min(i, d1 - 1);
        av[u] = L[(uint32_t)(TL ? ic * d1 + ac : ac * d1 + ic)];
        xv[u] = ld_f32<XT>(x + (uint32_t)(ic * d2 + jc));
      }
#pragma unroll
      for (int u = 0; u < LB; ++u) {
        const bool in = i0 + 4 * u + g < d1;       // both operands 0 beyond the extents
        av[u] = (in && alive) ? av[u] : 0.f;
        xv[u] = (in && j < d2) ? xv[u] : 0.f;
      }
#pragma unroll
      for (int u = 0; u < LB; u += RC) {
        if (i0 + 4 * u >= d1) break;
#pragma unroll
        for (int q = 0; q < RC; ++q)
          acc[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[u + q], xv[u + q], acc[q], 0, 0, 0);
      }
    }
    const floatx4 t4 = total(acc);
#pragma unroll
    for (int v = 0; v < 4; ++v) T[(4 * g + v) * pitch + jt * 16 + c] = t4[v];
  }
  __syncthreads();
  for (int bt = wave; bt < nct; bt += nw) {
    const int b = bt * 16 + c, bc = min(b, d2 - 1);
    floatx4 acc[RC] = {};
    for (int j0 = 0; j0 < d2; j0 += 4 * LB) {
      if (j0 > 0 || bt != wave) {
#pragma unroll
        for (int u = 0; u < LB; ++u) rv[u] = R[(uint32_t)(min(j0 + 4 * u + g, d2 - 1) * d2 + bc)];
      }
      float tv[LB];
#pragma unroll
      for (int u = 0; u < LB; ++u) tv[u] = T[c * pitch + min(j0 + 4 * u + g, nct * 16 - 1)];
#pragma unroll
      for (int u = 0; u < LB; ++u) {
        const bool in = j0 + 4 * u + g < d2;
        tv[u] = in ? tv[u] : 0.f;
        rv[u] = in ? rv[u] : 0.f;
      }
#pragma unroll
      for (int u = 0; u < LB; u += RC) {
        if (j0 + 4 * u >= d2) break;
#pragma unroll
        for (int q = 0; q < RC; ++q)
          acc[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(tv[u + q], rv[u + q], acc[q], 0, 0, 0);
      }
    }
    const floatx4 o4 = total(acc);
    if (b < d2)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if (a0 + 4 * g + v < d1) put(4 * g + v, b, o4[v]);
  }
  __syncthreads();
}

// out[t] = A M[t] R on the d1 x d2 view of n vectors (rot_tile).  grid (ceil(d1 / 16), n),
// a wave per 16 columns up to 8 waves.  Dynamic LDS: rot_lds_floats(d2).
template <typename XT, bool TL>
__global__ __launch_bounds__(WT) void k_rotate_tile(const XT* __restrict__ in, int64_t ldin,
                                                    const float* __restrict__ L,
                                                    const float* __restrict__ R, int d1, int d2,
                                                    float* __restrict__ out, int64_t ldout) {
  extern __shared__ __attribute__((aligned(16))) float rsh[];
  const int64_t t = blockIdx.y;
  const int a0 = (int)blockIdx.x * 16;
  float* o = out + t * ldout + (int64_t)a0 * d2;
  rot_tile<XT, TL>(in + t * ldin, L, R, d1, d2, a0, rsh,
                   [&](int r, int b, float v) { o[(int64_t)r * d2 + b] = v; });
}

// A row's chains in k_rotate: a thread sums chain g of column j, its terms in batches of UB blocks
// whose loads go out together.  qv = q[i d2 + j] for the terms i of batch n0 (those past nk 0).
constexpr int UB = 4, RBATCH = 4 * RC * UB;       // terms of all chains in a batch
template <typename TQ>
__device__ __forceinline__ void rot_batch(const TQ* __restrict__ q, int d2, int nk, int n0, int g, int j,
                                          float (&qv)[4 * UB]) {
  const int i0 = n0 + 4 * g;
  if (n0 + RBATCH <= nk) {
    const TQ* qq = q + (int64_t)i0 * d2 + j;
#pragma unroll
    for (int u = 0; u < 4 * UB; ++u) qv[u] = ld_f32<TQ>(qq + (4 * RC * (u >> 2) + (u & 3)) * (int64_t)d2);
  } else {
#pragma unroll
    for (int u = 0; u < 4 * UB; ++u) {
      const int i = i0 + 4 * RC * (u >> 2) + (u & 3);
      qv[u] = ld_f32<TQ>(q + (int64_t)min(i, nk - 1) * d2 + j);
      qv[u] = i < nk ? qv[u] : 0.f;
    }
  }
}

// red[g d2 + j] = chain g of sum over i < nk of p[i] q[i d2 + j]; p in LDS, 0 from nk to the end of
// its last batch.  qv: the first batch of this thread's first chain.
template <typename TQ>
__device__ __forceinline__ void rot_chains_row(int d2, int nk, float* red, const float* p,
                                               const TQ* __restrict__ q, float (&qv)[4 * UB]) {
  for (int e = threadIdx.x; e < RC * d2; e += blockDim.x) {
    const int g = e / d2, j = e - g * d2;
    float acc = 0.f;
    for (int n0 = 0; n0 < nk; n0 += RBATCH) {
      if (n0 > 0 || e != (int)threadIdx.x) rot_batch(q, d2, nk, n0, g, j, qv);
#pragma unroll
      for (int u = 0; u < 4 * UB; ++u) acc = fmaf(p[n0 + 4 * g + 4 * RC * (u >> 2) + (u & 3)], qv[u], acc);
    }
    red[e] = acc;
  }
}

// out[t] = A M[t] R as above, one row a of the result per work-group: calls of few vectors, view
// rows longer than k_rotate_tile's LDS holds, and frame generation.  Row a of A sits in LDS; the
// first loads of M go out beside it, those of R before T is waited for.  grid (n * d1),
// rot_threads(d2).  Dynamic LDS: rot_lds(d1, d2).
// With the DFT, one vector of 64 x 64 takes 6.9 us, 86 x 128 9.7, 128 x 224 20.6 (8.1, 10.2 and
// 22.4 with the row of A read by every thread and 1024 / d2 chains).
__host__ __device__ inline int rot_pad(int n) { return (n + RBATCH - 1) / RBATCH * RBATCH; }
constexpr int ROT_ROW_D1 = 8192;      // longer rows of A are read from memory
template <typename XT, bool TL>
__global__ __launch_bounds__(RT, 8) void k_rotate(const XT* __restrict__ in, int64_t ldin,
                                                  const float* __restrict__ L,
                                                  const float* __restrict__ R, int d1, int d2,
                                                  float* __restrict__ out, int64_t ldout) {
  extern __shared__ float rsh[];
  const int64_t t = blockIdx.x / d1;
  const int a = (int)(blockIdx.x - t * d1);
  const int nth = blockDim.x;
  const XT* x = in + t * ldin;
  const float* la = L + (TL ? a : (int64_t)a * d1);      // A(a, i) = la[i ls]
  const int64_t ls = TL ? d1 : 1;
  float* o = out + t * ldout + (int64_t)a * d2;
  if (rot_chains(d2) == 1) {
    float* z = rsh;
    for (int j = threadIdx.x; j < d2; j += nth) {
      float acc = 0.f;
#pragma unroll 8
      for (int i = 0; i < d1; ++i) acc = fmaf(la[i * ls], ld_f32<XT>(x + (int64_t)i * d2 + j), acc);
      z[j] = acc;
    }
    __syncthreads();
    for (int b = threadIdx.x; b < d2; b += nth) {
      float acc = 0.f;
#pragma unroll 8
      for (int j = 0; j < d2; ++j) acc = fmaf(z[j], R[(int64_t)j * d2 + b], acc);
      o[b] = acc;
    }
    return;
  }
  float* z = rsh;
  float* red = z + rot_pad(d2);
  float* pl = red + RC * d2;
  auto total = [&](int j) {
    float sum = 0.f;
#pragma unroll
    for (int g = 0; g < RC; ++g) sum += red[g * d2 + j];
    return sum;
  };
  const int g0 = (int)threadIdx.x / d2, j0 = (int)threadIdx.x - g0 * d2;
  const bool first = (int)threadIdx.x < RC * d2;
  float qv[4 * UB];
  if (d1 <= ROT_ROW_D1) {
    if (first) rot_batch(x, d2, d1, 0, g0, j0, qv);
    for (int i = threadIdx.x; i < rot_pad(d1); i += nth) pl[i] = i < d1 ? la[i * ls] : 0.f;
    __syncthreads();
    rot_chains_row(d2, d1, red, pl, x, qv);
  } else {
    for (int e = threadIdx.x; e < RC * d2; e += nth) {
      const int g = e / d2, j = e - g * d2;
      float acc = 0.f;
      for (int64_t b = 4 * g; b < d1; b += 4 * RC)
        for (int64_t i = b; i < min<int64_t>(b + 4, d1); ++i) acc = fmaf(la[i * ls], ld_f32<XT>(x + i * d2 + j), acc);
      red[e] = acc;
    }
  }
  if (first) rot_batch(R, d2, d2, 0, g0, j0, qv);
  __syncthreads();
  for (int j = threadIdx.x; j < rot_pad(d2); j += nth) z[j] = j < d2 ? total(j) : 0.f;
  __syncthreads();
  rot_chains_row(d2, d2, red, z, R, qv);
  __syncthreads();
  for (int b = threadIdx.x; b < d2; b += nth) o[b] = total(b);
}

// Rt = R^T for a d2 x d2 matrix: 32 x 32 tile b of ceil(d2 / 32)^2, through LDS
__device__ __forceinline__ void transpose_tile(const float* __restrict__ R, int d2,
                                               float* __restrict__ Rt, int b,
                                               float (*tile)[33]) {
  const int nb = (d2 + 31) / 32;
  const int bi = b / nb, bj = b - bi * nb;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5, rows = blockDim.x >> 5;
  for (int r = ty; r < 32; r += rows) {
    const int i = bi * 32 + r, j = bj * 32 + tx;
    tile[r][tx] = (i < d2 && j < d2) ? R[(int64_t)i * d2 + j] : 0.f;
  }
  __syncthreads();
  for (int r = ty; r < 32; r += rows) {
    const int i = bj * 32 + r, j = bi * 32 + tx;
    if (i < d2 && j < d2) Rt[(int64_t)i * d2 + j] = tile[tx][r];
  }
}

__global__ __launch_bounds__(TT) void k_transpose(const float* __restrict__ R, int d2,
                                                  float* __restrict__ Rt) {
  __shared__ float tile[32][33];
  transpose_tile(R, d2, Rt, blockIdx.x, tile);
}

// Sums of V per-lane values (V a power of two) over the 64 lanes, masks MASK, MASK / 2, ..:
// while V > 1 a lane keeps half of the values and hands the other half across, so that all
// sums cost V - 1 + 6 - log2 V exchanges instead of 6 V.  Lane l ends with the sum of value
// l / (64 / V).  The order of a sum's additions does not depend on V.
template <int V, int MASK = 32>
__device__ __forceinline__ float lane_sums(const float (&v)[V], int lane) {
  if constexpr (V == 1) {
    float x = v[0];
#pragma unroll
    for (int m = MASK; m > 0; m >>= 1) x += __shfl_xor(x, m);
    return x;
  } else {
    constexpr int H = V / 2;
    const bool up = (lane & MASK) != 0;
    float w[H];
#pragma unroll
    for (int i = 0; i < H; ++i) {
      const float keep = up ? v[H + i] : v[i], send = up ? v[i] : v[H + i];
      w[i] = keep + __shfl_xor(send, MASK);
    }
    return lane_sums<H, MASK / 2>(w, lane);
  }
}

// The DFT sums of T vectors for outputs o0 <= o < o1 of block c, from LDS: xs holds nin
// complex values of each vector, and output o is sum_i w^(+-(base_i)(..)) xs[i] with phase
// (c m + i) o (analysis: i < m coordinates, o a subspace; conjugated) or (c m + o) i
// (synthesis: i < k subspaces, o a coordinate).  A wave takes every 8th output; its lanes
// take i = lane, lane + 64, ..., and one twiddle read serves all T vectors.
// put(t, o, e, value) receives the real (e = 0) and imaginary part of output o.
template <int T, bool SYN, typename Put>
__device__ __forceinline__ void dft_outputs(const float2* __restrict__ tws,
                                            const float2* __restrict__ xs, int nin, int k,
                                            uint32_t cm, int o0, int o1, Put put) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  constexpr int PER = 64 / (2 * T);
  for (int o = o0 + wave; o < o1; o += WT / 64) {
    // phase indices mod k < k <= 3968: every product fits 32 bits
    const uint32_t p = SYN ? (cm + (uint32_t)o) % (uint32_t)k : (uint32_t)o;
    const uint32_t first = SYN ? (uint32_t)lane : (cm + (uint32_t)lane) % (uint32_t)k;
    int idx = (int)((first * p) % (uint32_t)k);
    const int step = (int)((64u * p) % (uint32_t)k);
    float acc[2 * T];
#pragma unroll
    for (int v = 0; v < 2 * T; ++v) acc[v] = 0.f;
#pragma unroll 2
    for (int i = lane; i < nin; i += 64) {
      const float2 w = tws[idx];
      const float wy = SYN ? w.y : -w.y;
#pragma unroll
      for (int t = 0; t < T; ++t) {
        const float2 z = xs[t * nin + i];
        acc[2 * t] = fmaf(w.x, z.x, fmaf(-wy, z.y, acc[2 * t]));
        acc[2 * t + 1] = fmaf(w.x, z.y, fmaf(wy, z.x, acc[2 * t + 1]));
      }
      idx += step;
      if (idx >= k) idx -= k;
    }
    const float r = lane_sums<2 * T>(acc, lane);
    if (lane % PER == 0) {
      const int v = lane / PER;
      put(v >> 1, o, v & 1, r);
    }
  }
}

// Analysis DFT of T rotated vectors a work-group.  grid (slices of the k subspaces, rho / 2
// blocks, ceil(n / T)).  BITS 0: U (n x k rho fp32); 2 or 4: U as the product with codes of
// that width reads it (codes_layout.h), its padding columns zeroed by work-groups (0, 0, .).
// Dynamic LDS: k + T m complex.
template <int T, int BITS>
__global__ __launch_bounds__(WT) void k_tff_analysis(const float* __restrict__ y, int64_t d, int n,
                                                     int k, int rho, int m, float scale,
                                                     void* __restrict__ U, int64_t quads, int ncol) {
  extern __shared__ __attribute__((aligned(16))) float sh[];
  float2* tws = reinterpret_cast<float2*>(sh);
  float2* zs = tws + k;
  const int c = blockIdx.y;
  const int t0 = (int)blockIdx.z * T, nt = min(T, n - t0);
  load_twiddles(tws, k);
  for (int e = threadIdx.x; e < T * m; e += WT) {
    const int t = e / m, i = e - t * m;
    zs[e] = t < nt ? reinterpret_cast<const float2*>(y + (t0 + t) * d)[(int64_t)c * m + i]
                   : make_float2(0.f, 0.f);
  }
  __syncthreads();
  const int per = (k + (int)gridDim.x - 1) / (int)gridDim.x;
  const int s0 = (int)blockIdx.x * per, s1 = min(k, s0 + per);
  const int64_t K = (int64_t)k * rho;
  dft_outputs<T, false>(tws, zs, m, k, (uint32_t)(((int64_t)c * m) % k), s0, s1,
                        [&](int t, int s, int e, float v) {
                          if (t >= nt) return;
                          const int64_t col = (int64_t)s * rho + 2 * c + e;
                          if constexpr (BITS == 0)
                            reinterpret_cast<float*>(U)[(t0 + t) * K + col] = scale * v;
                          else
                            codes_put_f<BITS>(reinterpret_cast<uint16_t*>(U), quads, ncol, t0 + t, col,
                                              scale * v);
                        });
  if constexpr (BITS > 0) {
    if (c == 0 && blockIdx.x == 0)
      for (int t = 0; t < nt; ++t)
        for (int64_t j = K + threadIdx.x; j < quads * (4 * (32 / BITS)); j += WT)
          codes_put_f<BITS>(reinterpret_cast<uint16_t*>(U), quads, ncol, t0 + t, j, 0.f);
  }
}

// Synthesis DFT of T vectors a work-group.  grid: nwork = slices * (rho / 2) * ceil(n / T)
// work-groups (slices of the m coordinates of a block), then ceil(d2 / 32)^2 more that write
// Rt = R2^T for the rotation that follows.  V: complex value (subspace s, block c) of a vector
// at s ss + c cs.  Dynamic LDS: k + T k complex.  Z contiguous (d per vector).
template <int T>
__global__ __launch_bounds__(WT) void k_tff_synthesis(const float2* __restrict__ V, int64_t ldv,
                                                      int64_t ss, int64_t cs,
                                                      int n, int slices, int nwork, int k,
                                                      int rho, int m, int64_t d, float scale,
                                                      float* __restrict__ Z,
                                                      const float* __restrict__ R2, int d2,
                                                      float* __restrict__ Rt) {
  extern __shared__ __attribute__((aligned(16))) float sh[];
  if ((int)blockIdx.x >= nwork) {
    transpose_tile(R2, d2, Rt, (int)blockIdx.x - nwork, reinterpret_cast<float(*)[33]>(sh));
    return;
  }
  float2* tws = reinterpret_cast<float2*>(sh);
  float2* nus = tws + k;
  const int nb = rho / 2;
  const int sl = (int)blockIdx.x % slices;
  const int c = ((int)blockIdx.x / slices) % nb;
  const int t0 = ((int)blockIdx.x / (slices * nb)) * T, nt = min(T, n - t0);
  load_twiddles(tws, k);
  for (int e = threadIdx.x; e < T * k; e += WT) {
    const int t = e / k, i = e - t * k;
    nus[e] = t < nt ? V[(t0 + t) * ldv + i * ss + c * cs] : make_float2(0.f, 0.f);
  }
  __syncthreads();
  const int per = (m + slices - 1) / slices;
  const int j0 = sl * per, j1 = min(m, j0 + per);
  dft_outputs<T, true>(tws, nus, k, k, (uint32_t)(((int64_t)c * m) % k), j0, j1,
                       [&](int t, int j, int e, float v) {
                         if (t < nt) Z[(t0 + t) * d + 2 * ((int64_t)c * m + j) + e] = scale * v;
                       });
}

unsigned blocks_for(int64_t total) { return (unsigned)((total + TT - 1) / TT); }

// Columns c0 .. c0 + nc - 1 of T / sqrt(k) as rows of Z (nc x d, complex pairs): column
// s rho + 2c + e is zero outside the m-block c, where complex coordinate c m + j holds
// k^(-1/2) w^((c m + j) s) (e = 0) or i k^(-1/2) w^((c m + j) s) (e = 1).  One thread per
// complex coordinate; the phase index (c m + j) s mod k is exact in 64-bit integers.
__global__ __launch_bounds__(TT) void k_tff_columns(int64_t c0, int64_t nc, int64_t d, int k,
                                                    int rho, int m, float scale,
                                                    float* __restrict__ Z) {
  const int64_t dc = d / 2;
  const int64_t e = (int64_t)blockIdx.x * TT + threadIdx.x;
  if (e >= nc * dc) return;
  const int64_t r = e / dc, j = e - r * dc;
  const int64_t col = c0 + r;
  const int64_t sidx = col / rho;
  const int within = (int)(col - sidx * rho), c = within >> 1, odd = within & 1;
  float2 v = make_float2(0.f, 0.f);
  if (j / m == c) {
    const int64_t t = (j % k) * (sidx % k) % k;
    float sn, cs;
    sincospif(2.0f * (float)t / (float)k, &sn, &cs);
    v = odd ? make_float2(-sn * scale, cs * scale) : make_float2(cs * scale, sn * scale);
  }
  *reinterpret_cast<float2*>(Z + r * d + 2 * j) = v;
}

// P[i][c0 + r] = Pt[r][i] for r < nc, i < d: 32 x 32 tiles through LDS.
// grid (ceil(nc / 32) * ceil(d / 32)).
__global__ __launch_bounds__(TT) void k_scatter_columns(const float* __restrict__ Pt, int64_t nc,
                                                        int64_t d, float* __restrict__ P,
                                                        int64_t ldp, int64_t c0) {
  __shared__ float tile[32][33];
  const int64_t nbi = (d + 31) / 32;
  const int64_t br = blockIdx.x / nbi, bi = blockIdx.x - br * nbi;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  for (int q = ty; q < 32; q += 8) {
    const int64_t r = br * 32 + q, i = bi * 32 + tx;
    tile[q][tx] = (r < nc && i < d) ? Pt[r * d + i] : 0.f;
  }
  __syncthreads();
  for (int q = ty; q < 32; q += 8) {
    const int64_t i = bi * 32 + q, r = br * 32 + tx;
    if (i < d && r < nc) P[i * ldp + c0 + r] = tile[tx][q];
  }
}

// vectors per work-group of the DFT kernels: up to 8 share the twiddles (fewer where their
// inputs would not fit beside them), 4 while 8 would leave too few work-groups.  Both
// transforms of d = 11008, k = 757 with 1, 2, 4, 8 vectors: 16 vectors 36 / 29 / 26 / 26 us,
// 61 vectors 117 / 83 / 71 / 67 us.
int dft_vectors(int64_t n, int64_t nin, int64_t k) {
  int T = n >= 17 ? 8 : n >= 3 ? 4 : (int)n;
  while (T > 1 && (k + T * nin) * 8 > 96 * 1024) T /= 2;
  return T;
}

// slices of an output range: about 512 work-groups in all (two a compute unit), at least
// one output a wave.  256: 71 us for 61 vectors of d = 11008 against 67, 1024: 65 us there
// and 19 against 18 for d = 4096.
int dft_slices(int64_t nout, int64_t nb, int64_t groups) {
  const int64_t want = std::max<int64_t>(1, 512 / std::max<int64_t>(1, nb * groups));
  return (int)std::max<int64_t>(1, std::min<int64_t>(want, (nout + WT / 64 - 1) / (WT / 64)));
}

size_t rot_lds(int d1, int d2) {
  if (rot_chains(d2) == 1) return (size_t)d2 * sizeof(float);
  return (size_t)(rot_pad(d2) + RC * d2 + (d1 <= ROT_ROW_D1 ? rot_pad(d1) : 0)) * sizeof(float);
}
unsigned rot_threads(int d2) { return (unsigned)std::min(RT, (rot_chains(d2) * d2 + 63) / 64 * 64); }

// n vectors rotated.  Up to ROT_ROW_MAX vectors take a work-group per row of the view, whose many
// short work-groups hide the loads' latency best (with the DFT, d = 11008: 7 vectors 18.5 us, 8 in
// tiles 18.8; one token through 11008 x 4096, both rotations in tiles 36 us against 27); more
// take 16-row tiles on the matrix cores, which read X once per tile (61 vectors 67 us against
// 108).  View rows beyond the tile kernel's LDS take the former too.
constexpr int ROT_TILE_D1 = 32768;    // 32-bit offsets into R1
constexpr int64_t ROT_ROW_MAX = 7;
template <typename XT, bool TL>
hipError_t rotate_rows(const XT* in, int64_t ldin, int64_t n, const TffDev& F,
                       const float* R, float* out, int64_t ldout, hipStream_t s) {
  prof_begin(s, "tff_rotate");
  if (n <= ROT_ROW_MAX || F.d2 > ROT_TILE_MAX || F.d1 > ROT_TILE_D1) {
    hipLaunchKernelGGL((k_rotate<XT, TL>), dim3((unsigned)(n * F.d1)), dim3(rot_threads(F.d2)), rot_lds(F.d1, F.d2), s, in,
                       ldin, F.R1, R, F.d1, F.d2, out, ldout);
  } else {
    const int threads = 64 * std::min(WT / 64, (F.d2 + 15) / 16);
    hipLaunchKernelGGL((k_rotate_tile<XT, TL>), dim3((unsigned)((F.d1 + 15) / 16), (unsigned)n), dim3(threads),
                       (size_t)rot_lds_floats(F.d2) * sizeof(float), s, in, ldin, F.R1, R, F.d1, F.d2, out, ldout);
  }
  prof_end(s);
  return last_launch_error();
}

// ---- the dense frame.  Column (s, c, e) of T is supported on the 2 m coordinates of block c,
// which lie in na or fewer rows of the d1 x d2 view (from row r0 = floor(2 m c / d2) on), so
//   P[a d2 + b][col] = sum_r R1[a][r0 + r] G[b][r][col],
//   G[b][r][col] = sum_q R2[b][q] T[(r0 + r) d2 + q][col]:
// na d2 + 2 m multiply-adds an entry group instead of rotating whole vectors, d (d1 + d2) a
// column (a work-group per row of each of K vectors, 2.36 ms for d = 4096 and K = 4512).

// complex coordinate jj of column (s, ., e) as the real pair's entry `par`, w = w^(jj s)
__device__ __forceinline__ float t_entry(float2 w, int e, int par) {
  return e == par ? w.x : (e ? -w.y : w.y);
}

// G for columns c0 .. c0 + nc: G[(b na + r) ncp + col].  Lanes take columns; the products with
// R2 are of a scalar and a per-lane entry, summed eight at a time (one sum of d2 = 64 terms: error
// of P against 64 bits 1.8e-7 at d = 4096, 1.4e-7 when a work-group per row split it in 16).  The
// twiddles carry the rounding of their angle as a correction.  grid (ceil(nc / 64), na,
// ceil(d2 / 64)), 4 waves of 16 rows b each.  Dynamic LDS: k complex.
constexpr int MB = 16;
constexpr int GS = 8;       // terms per partial sum
__global__ __launch_bounds__(TT) void k_frame_g(const float* __restrict__ R2, int d2, int k, int rho,
                                                int m, float scale, int64_t c0, int64_t nc, int na,
                                                int64_t ncp, float* __restrict__ G) {
  extern __shared__ __attribute__((aligned(16))) float sh[];
  float2* tws = reinterpret_cast<float2*>(sh);
  for (int t = threadIdx.x; t < k; t += TT) {
    const float x = 2.0f * (float)t / (float)k;
    const float dx = fmaf(-x, (float)k, 2.0f * (float)t) / (float)k * 3.14159265f;   // radians
    float s0, c0s;
    sincospif(x, &s0, &c0s);
    const float sn = fmaf(dx, c0s, s0), cs = fmaf(-dx, s0, c0s);
    tws[t] = make_float2(cs, sn);
  }
  __syncthreads();
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int64_t x = (int64_t)blockIdx.x * 64 + lane;
  const int64_t col = c0 + min(x, nc - 1);
  const int s = (int)(col / rho), w = (int)(col - (int64_t)s * rho), c = w >> 1, e = w & 1;
  const int p0 = 2 * m * c, p1 = p0 + 2 * m;
  const int r = blockIdx.y;
  const int b0 = ((int)blockIdx.z * 4 + wave) * MB;
  if (b0 >= d2) return;
  int p = (p0 / d2 + r) * d2;                          // coordinate of q = 0 in this view row
  int idx = (int)((uint32_t)((p >> 1) % k) * (uint32_t)s % (uint32_t)k);
  float acc[MB], part[MB];
#pragma unroll
  for (int u = 0; u < MB; ++u) acc[u] = part[u] = 0.f;
  auto close = [&] {
#pragma unroll
    for (int u = 0; u < MB; ++u) {
      acc[u] += part[u];
      part[u] = 0.f;
    }
  };
  const float* rb[MB];
#pragma unroll
  for (int u = 0; u < MB; ++u) rb[u] = R2 + (int64_t)min(b0 + u, d2 - 1) * d2;
  if ((d2 & 1) == 0) {                                 // a complex pair lies in one view row
    for (int q = 0; q < d2; q += 2, p += 2) {
      const float2 t = tws[idx];
      const bool in = p >= p0 && p < p1;
      const float t0 = in ? t_entry(t, e, 0) : 0.f, t1 = in ? t_entry(t, e, 1) : 0.f;
#pragma unroll
      for (int u = 0; u < MB; ++u) part[u] = fmaf(rb[u][q + 1], t1, fmaf(rb[u][q], t0, part[u]));
      idx += s;
      if (idx >= k) idx -= k;
      if (q % GS == GS - 2) close();
    }
  } else {
    for (int q = 0; q < d2; ++q, ++p) {
      const float t0 = (p >= p0 && p < p1) ? t_entry(tws[idx], e, p & 1) : 0.f;
#pragma unroll
      for (int u = 0; u < MB; ++u) part[u] = fmaf(rb[u][q], t0, part[u]);
      if (p & 1) {
        idx += s;
        if (idx >= k) idx -= k;
      }
      if (q % GS == GS - 1) close();
    }
  }
  close();
  if (x >= nc) return;
#pragma unroll
  for (int u = 0; u < MB; ++u)
    if (b0 + u < d2) G[((int64_t)(b0 + u) * na + r) * ncp + x] = scale * acc[u];
}

// P[a d2 + b][c0 + x] = sum_r R1[a][r0 + r] G[b][r][x]: a wave takes one b and 64 columns, keeps
// their na <= NA values of G and walks the rows a.  Bound by writing P, in 256-byte runs.
// grid (ceil(nc / 64), ceil(d2 / 4)).  LR: R1 fits in (dynamic) LDS, d1^2 floats.
template <int NA, bool LR>
__global__ __launch_bounds__(TT) void k_frame_rows(const float* __restrict__ R1, int d1, int d2,
                                                   int rho, int m, const float* __restrict__ G,
                                                   int64_t c0, int64_t nc, int na, int64_t ncp,
                                                   float* __restrict__ P, int64_t ldp) {
  extern __shared__ __attribute__((aligned(16))) float sh[];
  if (LR) {
    for (int t = threadIdx.x; t < d1 * d1; t += TT) sh[t] = R1[t];
    __syncthreads();
  }
  const float* L = LR ? sh : R1;
  const int lane = threadIdx.x & 63;
  const int b = (int)blockIdx.y * 4 + (int)(threadIdx.x >> 6);
  const int64_t x = (int64_t)blockIdx.x * 64 + lane;
  if (b >= d2 || x >= nc) return;
  const int c = (int)((c0 + x) % rho) >> 1;
  const int r0 = 2 * m * c / d2;
  float g[NA];
  int off[NA];
#pragma unroll
  for (int r = 0; r < NA; ++r) {
    g[r] = r < na ? G[((int64_t)b * na + r) * ncp + x] : 0.f;   // rows past block c hold 0
    off[r] = min(r0 + r, d1 - 1);
  }
  float* out = P + (int64_t)b * ldp + c0 + x;
  const int64_t step = (int64_t)d2 * ldp;
#pragma unroll 2
  for (int a = 0; a < d1; ++a, out += step, L += d1) {
    float sum = 0.f;
#pragma unroll
    for (int r = 0; r < NA; ++r) sum = fmaf(L[off[r]], g[r], sum);
    *out = sum;
  }
}

}  // namespace

hipError_t tff_analysis(const void* X, int xt, int64_t ldx, int64_t n, const TffDev& F, float* y,
                        void* U, int code_bits, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipError_t e;
  if (xt == 0) e = rotate_rows<float, true>((const float*)X, ldx, n, F, F.R2, y, F.d, s);
  else if (xt == 1) e = rotate_rows<_Float16, true>((const _Float16*)X, ldx, n, F, F.R2, y, F.d, s);
  else e = rotate_rows<uint16_t, true>((const uint16_t*)X, ldx, n, F, F.R2, y, F.d, s);
  if (e != hipSuccess) return e;
  const int64_t nb = F.rho / 2;
  const int T = dft_vectors(n, F.m, F.k);
  const int64_t groups = (n + T - 1) / T;
  const size_t lds = (size_t)((F.k + T * F.m) * 8);
  const dim3 g((unsigned)dft_slices(F.k, nb, groups), (unsigned)nb, (unsigned)groups);
  const float scale = (float)(1.0 / std::sqrt((double)F.k));
  prof_begin(s, "tff_dft");
  const int64_t quads = code_bits > 0 ? codes_quads(F.k * F.rho, code_bits) : 0;
  const int ncol = codes_ncol_f(n);
#define FQ_ANA(T, B)                                                                            \
  e = launch_lds(k_tff_analysis<T, B>, g, dim3(WT), lds, s, y, F.d, n, F.k, F.rho, F.m, scale, U, quads, ncol);
#define FQ_ANA_T(B) \
  { if (T == 1) { FQ_ANA(1, B) } else if (T == 2) { FQ_ANA(2, B) } else if (T == 4) { FQ_ANA(4, B) } else { FQ_ANA(8, B) } }
  if (code_bits == 0) FQ_ANA_T(0) else if (code_bits == 2) FQ_ANA_T(2) else FQ_ANA_T(4)
#undef FQ_ANA_T
#undef FQ_ANA
  prof_end(s);
  return e != hipSuccess ? e : last_launch_error();
}

hipError_t tff_synthesis(const float* V, bool block_order, int64_t n, const TffDev& F, float* R2t,
                         float* z, float* Y, int64_t ldy, hipStream_t s) {
  if (n == 0) return hipSuccess;
  const int64_t nb = F.rho / 2;
  const int T = dft_vectors(n, F.k, F.k);
  const int64_t groups = (n + T - 1) / T;
  const int slices = dft_slices(F.m, nb, groups);
  const int64_t nwork = slices * nb * groups;
  const int tb = (F.d2 + 31) / 32;
  const size_t lds = (size_t)std::max<int64_t>((F.k + T * F.k) * 8, 32 * 33 * 4);
  const float scale = (float)(1.0 / std::sqrt((double)F.k));
  const int64_t ldv = F.k * nb, ss = block_order ? 1 : nb, cs = block_order ? F.k : 1;   // complex
  prof_begin(s, "tff_dft");
  hipError_t e = hipSuccess;
#define FQ_SYN(T)                                                                               \
  e = launch_lds(k_tff_synthesis<T>, dim3((unsigned)(nwork + tb * tb)), dim3(WT), lds, s,       \
                 reinterpret_cast<const float2*>(V), ldv, ss, cs, n, slices, nwork, F.k, F.rho, F.m, F.d, scale, z, \
                 F.R2, F.d2, R2t);
  if (T == 1) { FQ_SYN(1) } else if (T == 2) { FQ_SYN(2) } else if (T == 4) { FQ_SYN(4) } else { FQ_SYN(8) }
#undef FQ_SYN
  prof_end(s);
  if (e != hipSuccess) return e;
  return rotate_rows<float, false>(z, F.d, n, F, R2t, Y, ldy, s);
}

// rows of the view that hold a block's 2 m consecutive coordinates, at most
static int64_t frame_block_rows(const TffDev& F) {
  const int64_t p = 2 * F.m;
  return p % F.d2 == 0 ? p / F.d2 : std::min<int64_t>((p - 1) / F.d2 + 2, F.d1);
}

hipError_t tff_materialize(const TffDev& F, float* R2t, float* Z, float* Pt, int64_t nc_max,
                           float* P, int64_t ldp, hipStream_t s) {
  const int64_t K = F.k * F.rho;
  const float scale = (float)(1.0 / std::sqrt((double)F.k));
  const int64_t rows = frame_block_rows(F);
  // columns per pass: G takes na d2 floats of each, rounded up to 64 columns, in Z and Pt
  const int64_t fit = (Pt - Z) * 2 / (rows * F.d2) / 64 * 64;
  // (views of one or two rows are faster by whole vectors: 2080 = 2 x 1040 1017 us by blocks, 957
  // so, 3968 = 1 x 3968 14.4 and 12.3 ms; 6000 = 3 x 2000 9.7 and 13.3)
  if (rows <= 24 && F.d1 > 2 && fit >= 64) {
    const int na = (int)rows;
    const bool lr = F.d1 <= 128;
    const size_t lds = lr ? (size_t)F.d1 * F.d1 * sizeof(float) : 0;
    for (int64_t c0 = 0; c0 < K; c0 += fit) {
      const int64_t nc = std::min(fit, K - c0), ncp = (nc + 63) / 64 * 64;
      const unsigned gx = (unsigned)(ncp / 64);
      prof_begin(s, "tff_columns");
      hipLaunchKernelGGL(k_frame_g, dim3(gx, (unsigned)na, (unsigned)((F.d2 + 63) / 64)), dim3(TT),
                         (size_t)F.k * sizeof(float2), s, F.R2, F.d2, (int)F.k, (int)F.rho, (int)F.m, scale,
                         c0, nc, na, ncp, Z);
      prof_end(s);
      prof_begin(s, "tff_rotate");
#define FQ_ROWS(N, LR)                                                                          \
      hipLaunchKernelGGL((k_frame_rows<N, LR>), dim3(gx, (unsigned)((F.d2 + 3) / 4)), dim3(TT), lds, s, F.R1, \
                         F.d1, F.d2, (int)F.rho, (int)F.m, Z, c0, nc, na, ncp, P, ldp);
#define FQ_ROWS_N(LR)                                                                           \
      { if (na <= 4) { FQ_ROWS(4, LR) } else if (na <= 8) { FQ_ROWS(8, LR) }                     \
        else if (na <= 12) { FQ_ROWS(12, LR) } else if (na <= 16) { FQ_ROWS(16, LR) }            \
        else { FQ_ROWS(24, LR) } }
      if (lr) FQ_ROWS_N(true) else FQ_ROWS_N(false)
#undef FQ_ROWS_N
#undef FQ_ROWS
      prof_end(s);
    }
    return last_launch_error();
  }
  // blocks over many short view rows: whole vectors, nc_max columns at a time
  const int nb = (F.d2 + 31) / 32;
  prof_begin(s, "tff_rotate");
  hipLaunchKernelGGL(k_transpose, dim3((unsigned)(nb * nb)), dim3(TT), 0, s, F.R2, F.d2, R2t);
  prof_end(s);
  for (int64_t c0 = 0; c0 < K; c0 += nc_max) {
    const int64_t nc = std::min(nc_max, K - c0);
    prof_begin(s, "tff_columns");
    hipLaunchKernelGGL(k_tff_columns, dim3(blocks_for(nc * (F.d / 2))), dim3(TT), 0, s, c0, nc, F.d,
                       (int)F.k, (int)F.rho, (int)F.m, scale, Z);
    prof_end(s);
    prof_begin(s, "tff_rotate");
    hipLaunchKernelGGL((k_rotate<float, false>), dim3((unsigned)(nc * F.d1)), dim3(rot_threads(F.d2)), rot_lds(F.d1, F.d2), s,
                       (const float*)Z, F.d, F.R1, R2t, F.d1, F.d2, Pt, F.d);
    prof_end(s);
    prof_begin(s, "tff_columns");
    const int64_t g = ((nc + 31) / 32) * ((F.d + 31) / 32);
    hipLaunchKernelGGL(k_scatter_columns, dim3((unsigned)g), dim3(TT), 0, s, Pt, nc, F.d, P, ldp, c0);
    prof_end(s);
  }
  return last_launch_error();
}

}  // namespace fq
