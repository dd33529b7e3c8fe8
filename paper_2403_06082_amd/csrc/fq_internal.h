// Internal declarations shared by the libfq translation units (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>

namespace fq {

typedef uint16_t u16;

// ---------------------------------------------------------------- launch bookkeeping
// Every launch goes through prof_begin/prof_end so that the optional kernel timer can
// bracket it with events on the launch stream.
void prof_begin(hipStream_t s, const char* name);
void prof_end(hipStream_t s);
// whether the kernel timer is on (work that would otherwise go to an auxiliary stream
// then stays on the caller's stream, so that no two timed kernels overlap)
bool prof_enabled();
hipError_t last_launch_error();

// Launches a kernel whose dynamic LDS may go beyond 64 KB: the kernel's limit, which each device
// keeps for itself, is then raised on the current device before every launch (a host call without
// a stream), so that no state says on which devices it was.  Returns its error before launching.
template <typename... P, typename... A>
hipError_t launch_lds(void (*kernel)(P...), dim3 grid, dim3 block, size_t lds, hipStream_t s, A... args) {
  if (lds > 64 * 1024) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kernel, grid, block, (unsigned)lds, s, static_cast<P>(args)...);
  return hipSuccess;
}

// ---------------------------------------------------------------- bf16 MFMA GEMM engine
// C = sum over passes p of A[pa[p]] * B[pb[p]], fp32 accumulation, where A is M x K and
// B is K x N, both given as 16-bit planes (bf16, or f16 for the Hessian of f16 inputs).
//   a_kmajor: A(m, k) at a[m * lda + k]   else at a[k * lda + m]
//   b_kmajor: B(k, n) at b[n * ldb + k]   else at b[k * ldb + n]
enum Epilogue {
  EPI_F32 = 0,      // c[row * ldc + col] = acc
  EPI_SPLIT = 1,    // c_hi/c_lo[row * ldc + col] = bf16 pair of acc
  EPI_SYM = 2,      // upper tiles only; c[row][col] and c[col][row] for row <= col
  EPI_PARTIAL = 3,  // upper tiles only, split over K; fp32 partial tiles, tile-major
  EPI_TAIL = 4,     // internal: tiles of a short last round, split over K (fp32 partials)
  // products with a block of a frame, whose coordinates pair up as the real (e = 0) and
  // imaginary (e = 1) parts of complex ones (asynchronous path only)
  EPI_FOLD = 5,     // see GemmDesc::fold_k
  EPI_PAIR = 6      // c[(row / 2) * ldc + 2 col + row % 2] = acc
};

struct GemmDesc {
  int M = 0, N = 0, K = 0;
  const u16* a[2] = {nullptr, nullptr};
  const u16* b[2] = {nullptr, nullptr};
  int64_t lda = 0, ldb = 0;
  int npass = 1;
  int pa[3] = {0, 0, 0}, pb[3] = {0, 0, 0};
  bool a_kmajor = true, b_kmajor = true;
  bool f16 = false;              // operands are IEEE half instead of bf16
  int epi = EPI_F32;
  float* c = nullptr;
  int64_t ldc = 0;
  u16* c_hi = nullptr;
  u16* c_lo = nullptr;
  int ksplit = 1;                // EPI_PARTIAL only
  // EPI_PARTIAL of two M/N-major operands (asynchronous path): > 0 takes 128 x 128 tiles and folds
  // their fp32 sums every `chain` K steps of 32 into a second set; a split then writes two
  // partial slices, sums and remainders (2 ksplit in all)
  int chain = 0;
  const char* name = "gemm";     // kernel-timer label
  int64_t ldc_pad = 0;           // EPI_SPLIT: output columns [N, ldc_pad) are zeroed
  // batch > 1 (EPI_F32, EPI_FOLD, EPI_PAIR): products z < batch read A + z bsa, B + z bsb and write
  // C + z bsc (element strides; bsa and bsb multiples of 8)
  int batch = 1;
  int64_t bsa = 0, bsb = 0, bsc = 0;
  // EPI_FOLD: rows 2s and 2s + 1 of A are the cosine and sine of slot s <= fold_k / 2, and
  // columns 64 g + 32 e + x of B part e of vector t = 32 g + x < nvec.  With the products
  // a, b (cosine, sine with part 0) and c, d (with part 1), column t of C gets
  // (a + d, c - b) in rows q, q + 1, q = s rowmap, and (a - d, c + b) in those of the
  // mirrored slot fold_k - s (where that is another slot).
  int rowmap = 0, fold_k = 0, nvec = 0;
};

// Workspace bytes needed by EPI_PARTIAL for an N x N symmetric product split ksplit ways.
size_t gemm_partial_bytes(int N, int ksplit);
int gemm_sym_tiles(int N);
int64_t gemm_tiles(int64_t M, int64_t N);   // output tiles of an M x N product
// partial: EPI_PARTIAL's workspace, or (for EPI_F32 / EPI_SPLIT) an optional scratch of
// gemm_tail_bytes() that lets a short last round of tiles be split over K.
hipError_t gemm_run(const GemmDesc& d, float* partial, hipStream_t s);
size_t gemm_tail_bytes();
// whether gemm_run takes this product on the asynchronous path (any K-split of it)
bool gemm_async_ok(const GemmDesc& d);
// H (+)= sum of the ksplit partial slices (fp64) + T^T T for ntail (at most 31) more rows T
// (element type tt: 0 f32, 1 f16, 2 bf16; row stride ldt), mirrored to full symmetric storage.
hipError_t syrk_reduce(const float* partial, int N, int ksplit, float* H, int64_t ldh,
                       int accumulate, const void* tail, int tt, int64_t ldt, int ntail,
                       hipStream_t s);

// fp32 / f16 -> bf16 (hi, lo) planes with out[r * ld_out + c]; optional column scale
// (applied in fp32 before the split).  Element type: 0 = f32, 1 = f16.
hipError_t split_bf16(const void* in, int in_type, int64_t ld_in, int rows, int cols,
                      const float* col_scale, u16* hi, u16* lo, int64_t ld_out, hipStream_t s);
// Same with zero padding: out has rows_out >= rows rows and ld_out >= cols columns; rows
// [rows, rows_out) and columns [cols, ld_out) are 0.  Element type 2 = bf16.
hipError_t split_bf16_pad(const void* in, int in_type, int64_t ld_in, int rows, int cols,
                          const float* col_scale, u16* hi, u16* lo, int64_t ld_out,
                          int rows_out, hipStream_t s);
hipError_t fill_zero_f32(float* p, int rows, int cols, int64_t ld, hipStream_t s);

// ---------------------------------------------------------------- layer outputs from codes
// Y = X Theta^T from the packed codes and the frames, tokens in blocks of APPLY_NT (with
// dense frames) or of up to APPLY_BLOCK (structured frames; as many as the workspace holds).
constexpr int APPLY_NT = 8;
constexpr int APPLY_BLOCK = 80;
struct ApplyScratch {
  float* part;   // split-K partials of U = X P_in
  uint16_t* Uf;  // U as the code product reads it (codes_layout.h)
  float* V;      // tokens x K_out; as a rule in the place of part
  int nt;        // tokens per block
};
// floats of scratch for blocks of nt <= APPLY_NT tokens (and, with base, the carve-up); base
// 256-byte aligned
size_t apply_scratch_floats(int64_t d_in, int64_t K_out, int64_t K_in, int nt, ApplyScratch* w,
                            float* base);
// floats of the smallest scratch accepted (8 tokens' fp32 intermediates): one token's, at
// least, always fits in it
size_t apply_scratch_least(int64_t d_in, int64_t K_out, int64_t K_in);
// X: n x d_in (row stride ldx, element type xt: 0 f32, 1 f16, 2 bf16); Y: n x d_out fp32
// V (nt x K_out at stride ldv) = scale * (U (codes - zero)^T) for U stored as bf16 triples
// (codes_layout.h); bits 2 or 4.  vrho > 0: V's columns in the block order of a frame with
// subspaces of dimension vrho and vk of them.
hipError_t apply_codes(const uint16_t* Uf, int nt, int bits, const uint32_t* codes, int64_t K_out,
                       int64_t K_in, const float* scale, const float* zero, float* V, int64_t ldv,
                       int vrho, int64_t vk, hipStream_t s);
// ---------------------------------------------------------------- structured frames
// A validated tight fusion frame given by its construction (see tff_apply.hip):
// m = d / rho, R1 d1 x d1 and R2 d2 x d2 device fp32, d1 d2 = d.
struct TffDev {
  int64_t d, k, rho, m;
  const float* R1;
  int d1;
  const float* R2;
  int d2;
};
constexpr int64_t TFF_MAX_K = 3968;       // twiddles + one block of a vector within 64 KB of LDS
constexpr int64_t TFF_MAX_D2 = 4096;     // one row of the rotation's d1 x d2 view in LDS
constexpr int64_t TFF_CHUNK = 256;        // vectors per pass of the stand-alone transforms
// U = X P for n vectors; y: n x d scratch.  A vector's result does not depend on the others.
// code_bits 0: U is n x (k rho) fp32; 2 or 4: U is stored for the product with codes of that
// width (codes_layout.h).
hipError_t tff_analysis(const void* X, int xt, int64_t ldx, int64_t n, const TffDev& F, float* y, void* U, int code_bits, hipStream_t s);
// P (d x k rho, row stride ldp) of the frame; Z, Pt: nc_max x d scratch each (one after the
// other in memory), R2t: d2 x d2 scratch
hipError_t tff_materialize(const TffDev& F, float* R2t, float* Z, float* Pt, int64_t nc_max,
                           float* P, int64_t ldp, hipStream_t s);

// Structured analysis / synthesis of whole matrices (tff_pass.hip).  Block geometry of a
// frame: nb = rho / 2 blocks of m2 = 2m real coordinates (padded to pm) and k2 = 2k
// frame coordinates (padded to pk).  Folded form: m complex coordinates (padded to mf) and
// f2 = 2 (k / 2 + 1) cosine and sine columns (padded to kf).  Pads are multiples of 32.
struct TffPassGeom { int64_t nb, m2, pm, k2, pk, mf, f2, kf; };
TffPassGeom tff_pass_geom(const TffDev& F);
// pair planes of n folded rows: 64 rows of nb mf elements for every 32 vectors
inline int64_t tff_fold_elems(const TffPassGeom& g, int64_t n) {
  return (n + 31) / 32 * 64 * g.nb * g.mf;
}
// the blocks of P diag(colscale) (K entries): bf16 (hi, lo) planes of nb x pm x pk each
hipError_t tff_dft_blocks(const TffDev& F, u16* hi, u16* lo, hipStream_t s,
                          const float* colscale);
// the cosines and sines of all blocks of P: bf16 (hi, lo) planes of nb x mf x kf each
hipError_t tff_fold_blocks(const TffDev& F, u16* hi, u16* lo, hipStream_t s);
// out (K x n at stride ldout) = (X P)^T for n rows of X (element type xt, stride ldx), from
// the folded blocks.  Scratch: tmp n d fp32, Y pair planes of tff_fold_elems each.
hipError_t tff_rows_analysis_t(const void* X, int xt, int64_t ldx, int64_t n, const TffDev& F,
                               const u16* Fhi, const u16* Flo, float* tmp, u16* Yhi, u16* Ylo,
                               float* out, int64_t ldout, hipStream_t s);
// folded V planes (2 n x nb kf: row 2t + e, block order) from M (K x n, stride ldm)
hipError_t tff_fold_gather(const float* M, int64_t ldm, int64_t n, const TffDev& F, u16* hi,
                           u16* lo, hipStream_t s);
// V plane (cols x nb pk, block order of F) = (codes - zero)^T, exact bf16: the code
// matrix (F.k F.rho rows, cols columns) read down its columns; zero per code row
hipError_t tff_dequant_gather_t(const uint32_t* codes, int bits, const float* zero, int64_t cols,
                                const TffDev& F, u16* V, hipStream_t s);
// out (n x d at stride ldout) = V P^T from block-order planes: with Vlo, both folded (V of
// tff_fold_gather, F of tff_fold_blocks), else V exact in one plane and F of tff_dft_blocks;
// Z, tmp: n x d fp32 scratch each
hipError_t tff_rows_synthesis(const u16* Vhi, const u16* Vlo, int64_t n, const TffDev& F,
                              const u16* Fhi, const u16* Flo, float* Z, float* tmp, float* out,
                              int64_t ldout, hipStream_t s);
hipError_t sym_average(float* X, int64_t n, int64_t ld, hipStream_t s);
// true for a stream made by fq_side_stream_create (part of the device, shared with the
// caller's other streams)
bool is_side_stream(hipStream_t s);

// Seeded Haar factors (tff_seed.hip): out0 (n0 x n0 fp32) and out1 (n1 x n1) from seed; G, V:
// n x n fp64 scratch each, ab: 2n fp64, n = max(n0, n1)
constexpr int64_t TFF_SEED_MAX_N = 1024;
hipError_t tff_seeded_factors(uint64_t seed, int n0, int n1, double* G, double* V, double* ab,
                              float* out0, float* out1, hipStream_t s);
// Y (n x ldy) = V P^T with V n x (k rho); block_order: V's
// columns are [block c][subspace s][re, im] instead of the frame's s rho + 2c + e.  z: n x d
// scratch, R2t: d2 x d2 scratch
hipError_t tff_synthesis(const float* V, bool block_order, int64_t n, const TffDev& F, float* R2t, float* z, float* Y, int64_t ldy,
                         hipStream_t s);

// Per-token rounding of U (n x ldu, K columns) to act_bits-bit integers: Cq (code_bits 0: n x K
// bytes; 2 or 4: stored for the product with codes of that width, codes_layout.h), delta
// (n), and when csum is not NULL the row sums of Cq (n).
hipError_t act_quantize(const float* U, int64_t ldu, int64_t n, int64_t K, int act_bits,
                        int8_t* Cq, int code_bits, float* delta, int* csum, hipStream_t s);
// V as apply_codes, from rounded activations
hipError_t apply_codes_i8(const int8_t* Cq, const float* delta, const int* csum, int nt, int bits,
                          const uint32_t* codes, int64_t K_out, int64_t K_in, const float* scale,
                          const float* zero, float* V, int64_t ldv, int vrho, int64_t vk,
                          hipStream_t s);
hipError_t frame_apply(const void* X, int xt, int64_t n, int64_t ldx, int64_t d_in,
                       const uint32_t* codes, int bits, const float* scale, const float* zero,
                       int64_t K_out, int64_t K_in, const float* P_out, int64_t d_out,
                       const float* P_in, float* Y, const ApplyScratch& w, hipStream_t s);

// ---------------------------------------------------------------- fp64 path
struct QuantScratch {
  double* Y;          // K_out x K_in working matrix (pre-rounding values)
  double* A;          // K_in x K_in: reversed damped H~, factored in place (lower)
  double* R;          // K_in x K_in: R' = R diag(R)^-1, R the upper factor (H~_damped = R R^T)
  double* res;        // K_out x block residuals D - D^ of the current block
  uint8_t* codes8;    // K_out x K_in codes
  double* red;        // reduction partials
  double* scal;       // device scalars: [0] mu [1] sigma [2] lo [3] hi [4] lambda
  double* scale64;    // K_out
  double* zero64;     // K_out
  double* inv_rdiag;  // K_in
  double* lslots;     // 2 x 64 x 64: factors of the last two diagonal blocks
  uint8_t* dead;      // K_in
  int* flags;         // [0] not PD, [1] non-finite
};

hipError_t q_stats(const float* D, int64_t rows, int64_t cols, double clip_sigmas,
                   QuantScratch& w, hipStream_t s);
hipError_t q_hdiag_build(const float* Ht, int64_t K, double damp, QuantScratch& w,
                         hipStream_t s);
// Blocked lower Cholesky of A (K x K, in place); Lslots: 2 x 64 x 64 doubles of scratch.
hipError_t q_cholesky(double* A, int64_t K, double* Lslots, int* flags, hipStream_t s);
hipError_t q_reverse_upper(const double* A, int64_t K, double* R, double* inv_rdiag,
                           hipStream_t s);
hipError_t q_clip_grid(const float* D, int64_t rows, int64_t cols, int bits, QuantScratch& w,
                       float* scale, float* zero, hipStream_t s);
hipError_t q_gptq_block(const float* D, int64_t rows, int64_t cols, int i1, int i2, int o1,
                        int cw, int64_t ld_res, int bits, QuantScratch& w, hipStream_t s);
// C[M x N] = beta * C + alpha * A[M x K] * op(B)   (fp64 MFMA; beta is 0 or 1)
//   b_trans: op(B)(k, n) = B[n * ldb + k]  else B[k * ldb + n]
//   lower_only: only tiles with tile_row >= tile_col (for the Cholesky update)
//   tile: 32, 64 or 128 (register-staged kernel with that tile edge; 32 with K <= 128 and
//         not lower_only fetches every K step at launch), or 0: the 128 x 128
//         LDS-ring kernel where its layout rules hold (row-major operands, K % 16 == 0,
//         16-byte aligned A rows), else the 64 kernel.  The ring kernel is the faster one
//         from about 512 of its tiles up (two rounds of two work-groups per CU).
hipError_t dgemm(int64_t M, int64_t N, int64_t K, double alpha, double beta, const double* A,
                 int64_t lda, const double* B, int64_t ldb, bool b_trans, double* C, int64_t ldc,
                 bool lower_only, hipStream_t s, const char* name, int tile);
hipError_t q_pack2(const uint8_t* codes8, int64_t rows, int64_t cols, uint32_t* out,
                   hipStream_t s);
// out[r * ld_out + c] = code[r][c] - zero[r] (bf16) on a rows_out x ld_out plane, zero
// outside rows x cols; ld_out a multiple of 16 (and 16-byte aligned rows).
// 3- and 4-bit codes: floor(32 / bits) per uint32 word (2-bit: q_pack2 / dequant_bf16)
hipError_t q_pack_nbit(const uint8_t* codes8, int64_t rows, int64_t cols, int bits,
                       uint32_t* out, hipStream_t s);
// dequant_bf16 for any of 2, 3, 4 bits
hipError_t dequant_nbit_bf16(const uint32_t* codes, int bits, const float* zero, int64_t rows,
                             int64_t cols, u16* out, int64_t ld_out, int64_t rows_out,
                             hipStream_t s);
hipError_t dequant_bf16(const uint32_t* codes, const float* zero, int64_t rows, int64_t cols,
                        u16* out, int64_t ld_out, int64_t rows_out, hipStream_t s);

// ---------------------------------------------------------------- diagonal Wiener filter
// gain_i = (D_i . E_i) / (scale_i (Q_i . E_i)) (1 where the denominator is 0) with E = Q H~,
// Q the bf16 plane of codes - zero (row stride ldq); scale_out (may alias scale or be
// NULL) = gain * scale.
hipError_t wiener_rows(const float* D, const float* E, const u16* Q, int64_t ldq, int64_t K_out,
                       int64_t K_in, const float* scale, float* gain, float* scale_out,
                       hipStream_t s);

}  // namespace fq
