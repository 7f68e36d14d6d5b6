// Internal declarations shared by the HIP translation units of the library.
#pragma once
#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

namespace semfd {

// EPI_SPECTRAL (FP64 kernels only): another multiplier than the divide (EpiArgs::kind)
// EPI_UNFOLD (FP64 kernels only): the output rows (NN) or columns (NT) are orbit
// representatives r of the output axis (EpiArgs::rn, rper) and the product is the
// antisymmetric part o: out[r] = e + o, out[R(r)] = e - o with e = out[r] as stored
// by the symmetric block before (R(r) == r: out[r] only)
enum { EPI_STORE = 0, EPI_DIVIDE = 1, EPI_ACCUM = 2, EPI_SPECTRAL = 3, EPI_UNFOLD = 4 };

// Arguments of the fused epilogues.
//   EPI_DIVIDE: out = acc / (alpha + b1 L + b2 L^2),  L = lx[row] + ly[col / nz] + lz[col % nz]
//               (Helmholtz: b1 = 1, b2 = 0; the Cahn-Hilliard operator a + m dt eps L^2:
//               b1 = 0, b2 = m dt eps)
//   EPI_ACCUM : out += acc
struct EpiArgs {
  const double* lx = nullptr;
  const double* ly = nullptr;
  const double* lz = nullptr;
  double alpha = 0.0, b1 = 1.0, b2 = 0.0;
  long nz = 1;
  // multiplier of EPI_SPECTRAL: SPECTRAL_EXP = exp(-param (L + alpha)),
  // SPECTRAL_POWER = (L + alpha)^(-param); EPI_DIVIDE divides by
  // alpha + b1 L + b2 L^2
  int kind = 0;
  double param = 0.0;
  // reflection split (FP64 kernels): fold = 1 / 2 reads the contracted axis (of
  // extent rn, periodic rper, x unfolded) as v+_r = x_r + x_R(r) / v-_r = x_r - x_R(r)
  // with r = m + roff for m < K; EPI_UNFOLD reflects the output axis (extent rn,
  // periodic rper) with output row / column l at representative r = l + roff
  int fold = 0;
  int rn = 0, rper = 0, roff = 0;
};
constexpr int SPECTRAL_EXP = 1, SPECTRAL_POWER = 2;

// Reflection of node r on an axis of n nodes: n - 1 - r, or (n - r) mod n periodic.
__host__ __device__ inline int reflect_node(int r, int n, int per) { return per ? (n - r) % n : n - 1 - r; }

// Denominator of the spectral divide, FP64.
__host__ __device__ inline double spectral_den(double lam, double alpha, double b1, double b2) {
  return alpha + lam * (b1 + b2 * lam);
}

// v times the multiplier of the EPI_SPECTRAL epilogue at eigenvalue sum lam.
__device__ inline double spectral_mul(double v, double lam, const EpiArgs& e) {
  if (e.kind == SPECTRAL_EXP) return v * exp(-e.param * (lam + e.alpha));
  return v * pow(fmax(lam + e.alpha, 0.0), -e.param);  // SPECTRAL_POWER; L >= 0 up to rounding
}

// One FP64 mode product along `axis` of a row-major (dims[0], dims[1], dims[2])
// array: y[.., l, ..] = sum_m A[l][m] x[.., m, ..] with g[m * ldg + l] = A[l][m]
// (g zero-padded to a multiple of 128 in both dimensions).
hipError_t launch_mode_f64(const double* x, double* y, const double* g, int ldg, const int dims[3], int axis, int epi,
                           const EpiArgs& ea, hipStream_t stream);
// General block form: Y[p][l][q] = sum_{m < K} A[l][m] X[p][m][q] for l < L, the
// contracted axis of X of extent ldxa, the output axis of Y of extent ldya (batch
// strides ldxa Q, ldya Q); g rows >= pad16(K), ldg >= pad128(L).  K = 0 stores zeros.
// ea.fold reads X as the v+ / v- of its unfolded axis; EPI_UNFOLD writes e +- o.
hipError_t launch_mode_f64_part(const double* x, double* y, const double* g, int ldg, long P, int K, int L, long Q,
                                int ldxa, int ldya, int epi, const EpiArgs& ea, hipStream_t stream);
// Compact reflection fold of X[p][i][q] along i (n nodes): Y[p][r] = X[p][r] + X[p][R(r)]
// for the nrep representatives, then Y[p][nrep + j] = X[p][r] - X[p][R(r)] for the
// n - nrep representatives r = j + off that are not their own reflection
// (off = 1 periodic, 0 otherwise): Y has n rows like X.
hipError_t launch_fold_f64(const double* x, double* y, long P, int n, long Q, int nrep, int per, hipStream_t stream);

// ---- reflection-split products on strips in LDS (mode_strip.hip) ----
// One axis of n nodes: nrep orbit representatives (and symmetric modes), nodd =
// n - nrep antisymmetric modes, reflection n - 1 - r or, per, (n - r) mod n.
struct StripAxis {
  int n = 0, nrep = 0, nodd = 0, per = 0;
};
enum { STRIP_FWD = 0, STRIP_BWD = 1, STRIP_MUL = 2 };
// Factors in fragment order (strip_pack) with elements of the data's type: fs, fa
// forward symmetric / antisymmetric (modes x representatives), bs, ba backward
// (representatives x modes of the block).  Modes are in folded order.
struct StripArgs {
  const void* x = nullptr;
  void* y = nullptr;  // may be x where their types and pitches agree
  const void *fs = nullptr, *fa = nullptr, *bs = nullptr, *ba = nullptr;
  // planes: the y axis (ay) and its factors; ax and the factors above are the z axis
  const void *fs2 = nullptr, *fa2 = nullptr, *bs2 = nullptr, *ba2 = nullptr;
  StripAxis ax, ay;
  // columns: X[p][m][q], p < P, q < Q; rows: P rows of pitch ldx; planes: P planes
  // of ay.n rows of pitch ldx
  long P = 0, Q = 0;
  int ldx = 0;
  EpiArgs epi;  // STRIP_MUL (x axis, P = 1): multiplier with the folded eigenvalues
  // FP32 rows / planes backward: u += product (first: u = product), norm slots or null
  int first = 1;
  unsigned long long* norms = nullptr;
  // set by the launchers
  int tiles = 0, tiles2 = 0;  // 16-mode tiles in a factor's steps
  int stride = 0, stride2 = 0;
  long ntiles = 0;
};
// The order in which the strips read a factor: blocks of VU = 16 / sizeof(T) contraction
// steps of 4 rows, in each the tiles of 16 modes, in each 64 lanes of VU values, lane
// (k % 4, l % 16) holding rows 4 step + k % 4 of column l.  A wave's load of a block is
// 1 KB in one piece (in row order it was VU loads of four pieces).
inline int strip_tiles(int nrep) { return (nrep + 31) / 32 * 2; }
template <class T>
size_t strip_pack_elems(int nrep) {
  const int vu = 16 / (int)sizeof(T);
  return (size_t)(((nrep + 3) / 4 + 8 + vu - 1) / vu) * strip_tiles(nrep) * 64 * vu;  // 8 zero steps read ahead
}
// Factor A (L x M, row-major of pitch lda; rows l are outputs) into out, zero-filled.
template <class T>
void strip_pack(const double* a, int lda, int L, int M, int nrep, T* out) {
  const int vu = 16 / (int)sizeof(T), tiles = strip_tiles(nrep);
  for (int l = 0; l < L; ++l)
    for (int m = 0; m < M; ++m) {
      const int step = m / 4, lane = (m % 4) * 16 + l % 16;
      out[(((size_t)(step / vu) * tiles + l / 16) * 64 + lane) * vu + step % vu] = (T)a[(size_t)l * lda + m];
    }
}
// All four factors of an axis (ffold n x nrep, bfold_sym nrep x nrep, bfold_anti nrep x
// nodd) one after the other: 4 strip_pack_elems elements, zero-filled by the caller.
template <class T>
void strip_pack_axis(const double* ffold, const double* bsym, const double* banti, int nrep, int nodd, T* out) {
  const size_t block = strip_pack_elems<T>(nrep);
  strip_pack(ffold, nrep, nrep, nrep, nrep, out);
  strip_pack(ffold + (size_t)nrep * nrep, nrep, nodd, nrep, nrep, out + block);
  strip_pack(bsym, nrep, nrep, nrep, nrep, out + 2 * block);
  strip_pack(banti, nodd, nrep, nodd, nrep, out + 3 * block);
}
constexpr long STRIP_MAX_Q = 1L << 22;  // 32-bit offsets of 64 rows inside a strip's base
// Whether the strips take an axis / a pair of axes with elements of `elem` bytes.
bool strip_axis_ok(const StripAxis& a, int elem);
bool strip_plane_ok(const StripAxis& ay, const StripAxis& az, int elem);
// y and x products: op STRIP_FWD, STRIP_BWD, or STRIP_MUL (forward, multiplier,
// backward).  T = double or float.
template <class T>
hipError_t launch_strip_col(const StripArgs& g, int op, hipStream_t s);
// z products: STRIP_FWD from TI rows of pitch ldx to T rows of n; STRIP_BWD from T
// rows of n to FP64 nodes (T = float: accumulated).
template <class T, class TI>
hipError_t launch_strip_row(const StripArgs& g, int op, hipStream_t s);
// z and y products of whole planes, as launch_strip_row followed / preceded by y.
template <class T, class TI>
hipError_t launch_strip_plane(StripArgs g, int op, hipStream_t s);

// ---- low-precision rotating mode products (mode_lp.hip) ----
enum { LP_F32 = 1, LP_BF16 = 2, LP_BF16X3 = 3 };

// Update norms max|delta|, max|u| of the refinement, kept as FP64 bit patterns
// (non-negative doubles order like their unsigned bits).  Blocks spread their
// atomic maxima over NORM_SLOTS slots of one 128-byte line each: with one slot for
// all, the atomics of a launch (device scope, past the XCDs' L2s) queue up at about
// 12 ns each.  Unfold at n = 119 (3600 blocks) with one slot / these: 89 / 14.5 us; last
// dense FP32 pass at (127, 163, 143) 82 us with one slot, 21 without norms.
constexpr int NORM_SLOTS = 32, NORM_STRIDE = 16;       // stride in 8-byte words
constexpr int NORM_WORDS = NORM_SLOTS * NORM_STRIDE;  // words per solve
__device__ inline void norm_max(unsigned long long* norms, double dmax, double umax) {
  unsigned long long* s = norms + (blockIdx.x % NORM_SLOTS) * NORM_STRIDE;
  atomicMax(s, (unsigned long long)__double_as_longlong(dmax));
  atomicMax(s + 1, (unsigned long long)__double_as_longlong(umax));
}

// Epilogue arguments: divide by alpha + b1 L + b2 L^2 with L = l0[l] + l1[a] +
// l2[b] (third forward pass), or accumulate into FP64 (first = 1: u = delta)
// recording max|delta| and max|u| in the slots of norms (skipped when null).
struct EpiLP {
  const double* l0 = nullptr;
  const double* l1 = nullptr;
  const double* l2 = nullptr;
  double alpha = 0.0, b1 = 1.0, b2 = 0.0;
  int first = 0;
  unsigned long long* norms = nullptr;
};

// One pass  Y[l][a][b] = sum_k F[l][k] X[a][b][k]:
//   x: input rows (P = A*B rows of K elements, row pitch ldx), kind in_kind
//      (0 FP64, 1 FP32, 2 BF16 bits);
//   y: output (L, A, B) with row pitch ldy, kind out_kind (1 FP32, 2 BF16, 0 FP64
//      accumulate);
//   f_hi / f_lo: factor [l][k] (FP32 or BF16 bits), padded with zeros to ldf
//      columns and to a multiple of 128 rows.
// The direct-to-LDS kernels (mode_dma.hip) take BF16 operands only: split-BF16
// operands are two planes, the second xplane / yplane / fplane elements after
// the first (f_lo unused).
// Output column layouts of the BF16 passes (mode_dma.hip): plain, split mode
// layout (symmetric block, then antisymmetric from column bpad), folded pairs.
enum { COL_PLAIN = 0, COL_SPLIT = 1, COL_FOLD = 2 };

struct LpPass {
  int mode = LP_BF16;
  const void* x = nullptr;
  int ldx = 0;
  long P = 0;
  int K = 0;
  void* y = nullptr;
  int ldy = 0;
  int A = 0, B = 0, L = 0;
  const void* f_hi = nullptr;
  const void* f_lo = nullptr;
  int ldf = 0;
  int in_kind = 0, out_kind = 0, epi_kind = EPI_STORE;
  long xplane = 0, yplane = 0, fplane = 0;
  EpiLP epi;
  // BF16 passes only: a second contraction block (K2 > 0): its l-tiles read factor
  // rows from frow2 (>= L rounded up to 256) and tensor k in [koff2, koff2 + K2),
  // and write L2 output rows after the L of block 1 (K, L: block 1)
  int K2 = 0, koff2 = 0, frow2 = 0, L2 = 0;
  // output column layout (COL_*) and the b axis: COL_SPLIT: bsym symmetric modes,
  // antisymmetric from column bpad; COL_FOLD: bsym = orbit representatives of the
  // b axis (length bn, periodic bper), v+ at column r, v- at bpad + r
  int col = COL_PLAIN;
  int bsym = 0, bpad = 0, bn = 0, bper = 0;
  // tuned launch shapes: FP32 factor-tile rows (128, 96, 64, 32; 0 = by rule);
  // BF16 tile order: groups of g p-strips step through the l-tiles together
  // (g = 1: every l-tile of one p-strip in a row); tile_group = g launches one
  // block per tile, DMA_PERSIST + g as many blocks as fit the CUs looping over the tiles
  int tile_rows = 0;
  int tile_group = 1;
};
constexpr int DMA_PERSIST = 16;
// FP32 passes (mode_lp.hip): mode LP_F32, in_kind 0 or 1, out_kind 1 or 0 (accumulate).
hipError_t launch_mode_lp(const LpPass& ps, hipStream_t stream);
// Factor-tile rows of a pass of L output modes that was not tuned: 96 where they cover L
// with clearly fewer padded rows than 128 (e.g. L = 257: 288 rows instead of 384).
int lp_rule_rows(int L);

// One FP32 pass of one solve inside a batched (persistent) launch: the fields of
// LpPass plus the tile bookkeeping.  Descriptor i owns tiles [tile0, tile0 +
// tiles_l * ceil(P / 128)) of the launch's global tile numbering (ascending
// tile0); sid indexes the launch's per-solve active flags.
struct LpDesc {
  const void* x = nullptr;
  void* y = nullptr;
  const void* f = nullptr;  // FP32 factor [l][k], pitch ldf
  EpiLP epi;
  long P = 0;
  long tile0 = 0;
  int ldx = 0, K = 0, ldy = 0, A = 0, B = 0, L = 0, ldf = 0;
  int tiles_l = 0;
  int sid = 0;
};
// Persistent FP32 launch over nd descriptors (device array) with tile_rows in
// {128, 96, 64, 32} (block tile tile_rows x 128), grid blocks striding over
// total_tiles; active: device array of per-solve flags.
hipError_t launch_mode_f32_batch(int in_kind, int out_kind, int epi, int tile_rows, const LpDesc* descs, int nd,
                                 long total_tiles, const int* active, int grid, hipStream_t stream);
int lp_batch_blocks_per_cu(int tile_rows);

// ---- BF16 / split-BF16 passes with direct global -> LDS loads (mode_dma.hip) ----
// Requirements: in_kind 2, ldx, ldy and ldf multiples of 8, each contraction
// block inside the tensor pitch and the factor pitch rounded to 32; tensor pitch
// padding holds finite values; factor zero outside its blocks.  Outputs: BF16
// planes (out_kind 2, any column layout, STORE or DIVIDE) or FP32 (out_kind 1,
// COL_PLAIN, STORE).  Padding columns receive finite values.
bool dma_supported(const LpPass& ps);
// Rows of the block tile that launch_mode_dma takes for ps: 256, 128 or 64.
int dma_tile_rows(const LpPass& ps);
hipError_t launch_mode_dma(const LpPass& ps, hipStream_t stream);
// Reflection split of one axis: nrep orbit representatives (v+ at columns
// [0, pad), v- at [pad, 2 pad) of a folded row), reflection n - 1 - r or, per,
// (n - r) mod n.
struct FoldAxis {
  int nrep = 0, pad = 0, per = 0;
};
// FP64 array (rows dims[0]*dims[1], pitch dims[2]) -> BF16 hi (+ lo plane plane_o
// elements later when split) with pitch ldo, padding zeroed; fold != null: the rows
// folded along z first.
hipError_t launch_to_lowp(const double* f, void* out, long plane_o, int split, const int dims[3], int ldo,
                          const FoldAxis* fold, hipStream_t stream);
// BF16 (split) rows of pitch ldi -> the same rows folded along z, pitch ldo.
hipError_t launch_fold_lowp(const void* in, long plane_i, int ldi, void* out, long plane_o, int ldo, int split,
                            const int dims[3], const FoldAxis& fold, hipStream_t stream);
// Weighted inner products an unfold with first = 1 forms as it writes u: per-block
// partial sums of <r, u>_M and <u, q>_M (mass weight mx_i my_j mz_l of node (i, j, l))
// into partial[2 b] and partial[2 b + 1], b < blocks (the grid of such a launch).
struct UnfoldDot {
  const double* r = nullptr;
  const double* q = nullptr;
  const double *mx = nullptr, *my = nullptr, *mz = nullptr;
  double* partial = nullptr;
  int blocks = 0;
};
// u (+)= the correction d (FP32, every axis in folded node form: e rows then o
// rows, pitch ldd for z''), see unfold_accum_kernel; dot (first = 1 only): also
// the partial sums of UnfoldDot.
hipError_t launch_unfold_accum(const float* d, int ldd, double* u, const int dims[3], const FoldAxis fold[3],
                               int first, unsigned long long* norms, hipStream_t stream,
                               const UnfoldDot* dot = nullptr);

// Generalised nodal residual  r = cf f - cd d - ch (H_x + H_y + H_z) v  with banded
// H rows hb[a][g * (2k+1) + d] = H_a(g, g - k + d), FP64 arithmetic.
//   f == nullptr: the f term is absent;  d == nullptr: d is v itself.
//   Helmholtz residual f - alpha u - H u: (v = u, f, d = null, cf = 1, cd = alpha, ch = 1).
// r is written with row pitch ldr >= dims[2] as FP64 (r_kind 0), FP32 (1), BF16
// (2) or split BF16 (3: hi plane, lo plane rplane elements later); the pitch
// padding [dims[2], ldr) is written with zeros.  r must not alias v.
struct ResidualArgs {
  const double* v = nullptr;
  const double* f = nullptr;
  const double* d = nullptr;
  // optional per-node weight of the d term, cd * (wa + wt) * (d or v); FP64 output
  // (r_kind 0) of the single launch only
  const double* wt = nullptr;
  double wa = 0.0;
  void* r = nullptr;
  int r_kind = 0;
  int ldr = 0;
  long rplane = 0;
  double cf = 1.0, cd = 0.0, ch = 1.0;
  int periodic = 0;  // bit a set: axis a is periodic (its neighbours wrap around)
  // weighted march only (wt set, k <= 8, FP64 output): also the per-block partial
  // sums of <v, r>_M = sum Mx_i My_j Mz_l v r, written to dot_partial[2 b] for
  // block b of the launch (residual_march_blocks blocks); dot_mass = the 1D masses
  double* dot_partial = nullptr;
  const double* dot_mass[3] = {nullptr, nullptr, nullptr};
};
// Blocks of the single-launch march for these dimensions and k (0 for k > 8,
// which takes the generic kernel).
long residual_march_blocks(const int dims[3], int k);
hipError_t launch_residual(const ResidualArgs& ra, const double* const hb[3], int k, const int dims[3],
                           hipStream_t stream);

// Residuals of many solves with the same k (1..8) and rows in one launch.  Descriptor i
// (device array, ascending block0) owns blocks [block0, block0 + gx*gy*gz);
// active: device array of per-solve flags indexed by sid.
struct ResDesc {
  const double* v = nullptr;
  const double* f = nullptr;
  const double* d = nullptr;
  void* r = nullptr;
  const double* hx = nullptr;
  const double* hy = nullptr;
  const double* hz = nullptr;
  long rplane = 0;
  long block0 = 0;
  int ldr = 0, nx = 0, ny = 0, nz = 0, xchunk = 0, gx = 0, gy = 0, gz = 0;
  int sid = 0;
  double cf = 1.0, cd = 0.0, ch = 1.0;
  int per = 0;   // bit a set: axis a is periodic (neighbours wrap around)
  int rows = 2;  // rows of y per wave: launches take descriptors of one kind
};
// Fill the geometry and operands of one descriptor (block0 and sid are the
// caller's); false if k or the arguments are outside what the batch kernel takes.
bool residual_desc(const ResidualArgs& ra, const double* const hb[3], int k, const int dims[3], ResDesc* d);
hipError_t launch_residual_batch(int k, int rows, int r_kind, const ResDesc* descs, int nd, long total_blocks,
                                 const int* active, hipStream_t stream);

}  // namespace semfd
