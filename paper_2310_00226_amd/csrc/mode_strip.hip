// Reflection-split mode products on strips held in LDS, FP64 and FP32.
//
// A product along an axis of n nodes takes v+_r = x_r + x_R(r) of the nrep orbit
// representatives into the nrep symmetric modes and v-_r = x_r - x_R(r) of the nodd
// pairs into the antisymmetric ones (forward), or e = S_sym c_sym and o = S_anti
// c_anti into u_r = e_r + o_r, u_R(r) = e_r - o_r (backward).  The 128 x 128 tiles of
// mode_f64.hip do the two halves in two launches, with fold passes between some products
// and a read-back of e; on short axes most of their time is tile padding, launches and
// the latency of short contractions.  Here a block owns a strip of 16 TC lines of the
// array along the contracted axis, folds it on its way into LDS,
// and each wave multiplies it by TT tiles of 16 modes, both halves at once, so that
//  * both halves, the fold and the unfold are one launch that reads and writes every
//    value once, in place if wanted (a block reads its strip before it writes it);
//  * along x the forward product, the spectral multiplier and the backward product
//    are one launch (the coefficients stay in LDS);
//  * small (y, z) planes do z and y in one launch: three launches for a solve.
// The factors are not staged: a wave reads its fragments from L1 / L2 four contraction
// steps ahead, in 1 KB pieces (an FP64 fragment pair feeds 2 TC MFMAs of 64 cycles).
// What bounds them on long axes is the MFMA rate and the padding of the modes to 16; below
// about 250 nodes the loads and stores of the strips as well, which the other blocks of a
// CU hide only in part (192^3 FP64: 57 us a launch, 24 of bytes and 19 to 38 of MFMAs).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cfloat>
#include <cstdint>

#include "kernels.h"

namespace semfd {

namespace stripk {

typedef double d4_t __attribute__((ext_vector_type(4)));
typedef float f4_t __attribute__((ext_vector_type(4)));

template <class T>
struct Mfma;
// accumulator register r of a lane is row RB r + RL (lane / 16), column lane % 16
template <>
struct Mfma<double> {
  typedef d4_t acc_t;
  static __device__ __forceinline__ d4_t mac(double a, double b, d4_t c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static constexpr int RB = 4, RL = 1;
};
template <>
struct Mfma<float> {
  typedef f4_t acc_t;
  static __device__ __forceinline__ f4_t mac(float a, float b, f4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static constexpr int RB = 1, RL = 4;
};

template <class T>
__device__ __forceinline__ int acc_row(int r, int fk) {
  return Mfma<T>::RB * r + Mfma<T>::RL * fk;
}

template <class T, int TT, int TC>
struct Acc {
  typename Mfma<T>::acc_t s[TT][TC], a[TT][TC];
};

// Factor fragments of U contraction steps, symmetric and antisymmetric, from factors
// in fragment order (strip_pack): one 16-byte load per lane holds VU steps.
constexpr int U = 4;
template <class T, int TT>
struct Frag {
  static constexpr int VU = 16 / (int)sizeof(T), NV = U / VU;
  typedef T vec_t __attribute__((ext_vector_type(VU)));
  vec_t s[NV][TT], a[NV][TT];
  // steps k0 .. k0 + U - 1 (k0 a multiple of U)
  __device__ __forceinline__ void load(const vec_t* __restrict__ gs, const vec_t* __restrict__ ga, int tiles, int k0) {
    const unsigned lane = threadIdx.x & 63;
#pragma unroll
    for (int h = 0; h < NV; ++h)
#pragma unroll
      for (int i = 0; i < TT; ++i) {
        const size_t at = ((size_t)(k0 / VU + h) * tiles + i) * 64;  // uniform
        s[h][i] = (gs + at)[lane];
        a[h][i] = (ga + at)[lane];
      }
  }
};

// Both halves of one product for the mode tiles t0 .. t0 + TT - 1: s += G_s^T ds,
// a += G_a^T da over nk steps of 4 contraction rows.  ds(k, j), da(k, j): this lane's
// data element of column tile j in step k.  DATA_A: the data is the first operand, so
// that the data index runs along the accumulator's rows.
// Two sets of U steps take turns, without copies: a copy would wait for its load.
// Vector memory answers a CU in order, so a fragment also waits for the strips that
// other blocks of the CU are loading: with U = 2 FP64 511^3 took 8298 instead of 7670 us
// (U = 6 the same, U = 8 8056).
template <class T, int TT, int TC, bool DATA_A, class FS, class FA>
__device__ __forceinline__ void dual_product(Acc<T, TT, TC>& c, const void* fs, const void* fa, int tiles, int nk,
                                             int t0, FS ds, FA da) {
  typedef Frag<T, TT> F;
  const typename F::vec_t* __restrict__ gs = (const typename F::vec_t*)fs + (size_t)t0 * 64;
  const typename F::vec_t* __restrict__ ga = (const typename F::vec_t*)fa + (size_t)t0 * 64;
#pragma unroll
  for (int i = 0; i < TT; ++i)
#pragma unroll
    for (int j = 0; j < TC; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) c.s[i][j][r] = c.a[i][j][r] = T(0);
  auto mul = [&](const F& f, int u, int k) {
    T s[TC], a[TC];
#pragma unroll
    for (int j = 0; j < TC; ++j) {
      s[j] = ds(k, j);
      a[j] = da(k, j);
    }
#pragma unroll
    for (int i = 0; i < TT; ++i) {
      const T gs1 = f.s[u / F::VU][i][u % F::VU], ga1 = f.a[u / F::VU][i][u % F::VU];
#pragma unroll
      for (int j = 0; j < TC; ++j) {
        c.s[i][j] = DATA_A ? Mfma<T>::mac(s[j], gs1, c.s[i][j]) : Mfma<T>::mac(gs1, s[j], c.s[i][j]);
        c.a[i][j] = DATA_A ? Mfma<T>::mac(a[j], ga1, c.a[i][j]) : Mfma<T>::mac(ga1, a[j], c.a[i][j]);
      }
    }
  };
  F f0, f1;
  f0.load(gs, ga, tiles, 0);
  int k = 0;
  for (; k + 2 * U <= nk; k += 2 * U) {
    f1.load(gs, ga, tiles, k + U);
#pragma unroll
    for (int u = 0; u < U; ++u) mul(f0, u, k + u);
    f0.load(gs, ga, tiles, k + 2 * U);
#pragma unroll
    for (int u = 0; u < U; ++u) mul(f1, u, k + U + u);
  }
  if (k + U < nk) f1.load(gs, ga, tiles, k + U);
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (k + u < nk) mul(f0, u, k + u);
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (k + U + u < nk) mul(f1, u, k + U + u);
}

__device__ __forceinline__ int refl(int r, const StripAxis& a) { return a.per ? (r ? a.n - r : 0) : a.n - 1 - r; }

template <bool SPECTRAL>
__device__ __forceinline__ double multiply(double v, double lam, const EpiArgs& e) {
  return SPECTRAL ? spectral_mul(v, lam, e) : v / spectral_den(lam, e.alpha, e.b1, e.b2);
}
// FP32 solves: the quotient is rounded to FP32 anyway, a fast float divide suffices
template <bool SPECTRAL>
__device__ __forceinline__ float multiply(float v, double lam, const EpiArgs& e) {
  return __fdividef(v, (float)spectral_den(lam, e.alpha, e.b1, e.b2));
}

// Element (row m, column c) of a column strip of W columns.  A fragment read takes 16
// columns of four consecutive rows, FP64 two rows at a time: where a row (pair) spans
// all 64 banks, every second one swaps its 16-column halves, so that they do not meet.
template <class T, int W>
__device__ __forceinline__ int at(int m, int c) {
  static_assert(W == 16 || W == 32, "one or two column tiles");
  constexpr int SPAN = W * (int)sizeof(T) / 128;  // 1: two rows span the banks
  if constexpr (sizeof(T) == 8 && SPAN >= 2) return m * W + (c ^ ((m & 1) << 4));
  else if constexpr (sizeof(T) == 4 && SPAN == 1) return m * W + (c ^ (((m ^ (m >> 1)) & 1) << 4));
  else return m * W + c;
}

// A strip holds K = nrep rounded up to 4 symmetric elements of each line, then K
// antisymmetric ones: v+ and v- of the representatives or the coefficients, zeros
// behind them (and v- = 0 where a node is its own reflection).
__host__ __device__ inline int pad4(int n) { return (n + 3) & ~3; }

// (v+, v-) of representative m and its reflection, or two coefficients as they are.
template <class T, int OP, class TI>
__device__ __forceinline__ void pair_values(int m, TI a, TI b, const StripAxis& ax, T* s, T* v) {
  if constexpr (OP == STRIP_BWD) {
    *s = (T)a;
    *v = (T)b;
  } else {
    const bool pair = refl(m, ax) != m;
    *s = (T)(a + (pair ? b : a));
    *v = pair ? (T)(a - b) : T(0);
  }
}

// A block takes one strip, its XCD a contiguous range of them (neighbouring strips
// share cache lines).  Looping blocks that held the next strip in registers while
// they multiplied were 10-30% slower: vector memory returns in order, so every
// factor load then waits for the strip loads and stores that were issued before it.
__device__ __forceinline__ long xcd_tile() {
  return (long)(blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
}

// ---- y and x axes: X[p][m][q], a strip is W = 16 TC columns q of one p --------------
template <class T, int TT, int TC, int OP, bool SPECTRAL>
__global__ void col_kernel(StripArgs g) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  T* const V = reinterpret_cast<T*>(smem);
  constexpr int W = 16 * TC, NP = 4 * TC * TT;
  const long strips = (g.Q + W - 1) / W;
  const long tile = xcd_tile();
  if (tile >= g.ntiles) return;  // the whole block
  const long p = tile / strips, q0 = (tile - p * strips) * W;
  const StripAxis ax = g.ax;
  const T* x = reinterpret_cast<const T*>(g.x) + (size_t)p * ax.n * g.Q + q0;
  T* y = reinterpret_cast<T*>(g.y) + (size_t)p * ax.n * g.Q + q0;
  const int tid = threadIdx.x, nt = blockDim.x;
  const int lane = tid & 63, fr = lane & 15, fk = lane >> 4;
  const int t0 = __builtin_amdgcn_readfirstlane(tid >> 6) * TT;
  // pair u of a thread: row m0 + u step, column c0
  const int c0 = tid % W, m0 = tid / W, step = nt / W;
  const unsigned vlo = (unsigned)m0 * (unsigned)g.Q, vhi = (unsigned)(step - 1 - m0) * (unsigned)g.Q;

  const int K = pad4(ax.nrep), nk = K >> 2;
  auto ds = [&](int k, int j) { return V[at<T, W>(4 * k + fk, 16 * j + fr)]; };
  auto da = [&](int k, int j) { return V[at<T, W>(K + 4 * k + fk, 16 * j + fr)]; };

  {
    T pa[NP], pb[NP];
    const unsigned cq = (unsigned)min((long)c0, g.Q - 1 - q0);
#pragma unroll
    for (int u = 0; u < NP; ++u) {
      const int m = m0 + u * step;
      pa[u] = pb[u] = T(0);
      if (m >= ax.nrep) continue;
      pa[u] = (x + (long)u * step * g.Q)[vlo + cq];
      if constexpr (OP == STRIP_BWD) {
        if (m < ax.nodd) pb[u] = (x + (long)(ax.nrep + u * step) * g.Q)[vlo + cq];
      } else {
        // R(m) = n - 1 - m + per, past the axis only for the fixed node 0
        if (m >= ax.per) pb[u] = (x + (long)(ax.n + ax.per - (u + 1) * step) * g.Q)[vhi + cq];
      }
    }
#pragma unroll
    for (int u = 0; u < NP; ++u) {
      const int m = m0 + u * step;
      if (m >= K) continue;
      T s, v;
      pair_values<T, OP>(m, pa[u], pb[u], ax, &s, &v);
      V[at<T, W>(m, c0)] = s;
      V[at<T, W>(K + m, c0)] = v;
    }
  }
  __syncthreads();

  Acc<T, TT, TC> c;
  if constexpr (OP != STRIP_BWD) {
    dual_product<T, TT, TC, false>(c, g.fs, g.fa, g.tiles, nk, t0, ds, da);
  }
  // output addresses: a uniform row of the accumulator register plus the lane's
  // offset; mirrored rows run the other way
  constexpr int RB = Mfma<T>::RB, RL = Mfma<T>::RL;
  const unsigned wlo = (unsigned)(RL * fk) * (unsigned)g.Q + fr, whi = (unsigned)(3 * RL - RL * fk) * (unsigned)g.Q + fr;
  if constexpr (OP == STRIP_FWD) {
#pragma unroll
    for (int i = 0; i < TT; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int lb = 16 * (t0 + i) + RB * r, l = lb + RL * fk;
        T* ys = y + (long)lb * g.Q;
        T* ya = y + (long)(ax.nrep + lb) * g.Q;
#pragma unroll
        for (int j = 0; j < TC; ++j) {
          if (q0 + 16 * j + fr >= g.Q) continue;
          if (l < ax.nrep) ys[wlo + 16 * j] = c.s[i][j][r];
          if (l < ax.nodd) ya[wlo + 16 * j] = c.a[i][j][r];
        }
      }
    return;
  }
  if constexpr (OP == STRIP_MUL) {
    // x axis: coefficients back into the strip, then the multiplier
    __syncthreads();  // every wave is done with the node values
#pragma unroll
    for (int i = 0; i < TT; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int l = 16 * (t0 + i) + acc_row<T>(r, fk);
#pragma unroll
        for (int j = 0; j < TC; ++j) {
          if (l < ax.nrep) V[at<T, W>(l, 16 * j + fr)] = c.s[i][j][r];
          if (l < ax.nodd) V[at<T, W>(K + l, 16 * j + fr)] = c.a[i][j][r];
        }
      }
    __syncthreads();
    const int qi = (int)min(q0 + c0, g.Q - 1);
    const int jy = qi / (int)g.epi.nz;
    const double lq = g.epi.ly[jy] + g.epi.lz[qi - jy * (int)g.epi.nz];
    for (int m = m0; m < ax.nrep; m += step) {
      T* s = V + at<T, W>(m, c0);
      T* v = V + at<T, W>(K + m, c0);
      *s = multiply<SPECTRAL>(*s, g.epi.lx[m] + lq, g.epi);
      if (m < ax.nodd) *v = multiply<SPECTRAL>(*v, g.epi.lx[ax.nrep + m] + lq, g.epi);
      else *v = T(0);
    }
    __syncthreads();
  }
  dual_product<T, TT, TC, false>(c, g.bs, g.ba, g.tiles, nk, t0, ds, da);
#pragma unroll
  for (int i = 0; i < TT; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int lb = 16 * (t0 + i) + RB * r, l = lb + RL * fk;
      if (l >= ax.nrep) continue;
      const bool pair = refl(l, ax) != l;
      T* yl = y + (long)lb * g.Q;
      T* ym = y + (long)(ax.n - 1 + ax.per - lb - 3 * RL) * g.Q;
#pragma unroll
      for (int j = 0; j < TC; ++j) {
        if (q0 + 16 * j + fr >= g.Q) continue;
        const T e = c.s[i][j][r], o = c.a[i][j][r];
        yl[wlo + 16 * j] = e + o;
        if (pair) ym[whi + 16 * j] = e - o;
      }
    }
}

// Running maxima of a refinement update (norm_max).
struct Norms {
  double d = 0.0, u = 0.0;
  // a NaN / Inf turns the norm into +Inf (fmax alone would drop NaN)
  __device__ __forceinline__ void add(double dv, double un) {
    d = fabs(dv) <= DBL_MAX ? fmax(d, fabs(dv)) : INFINITY;
    u = fabs(un) <= DBL_MAX ? fmax(u, fabs(un)) : INFINITY;
  }
};

// The last product of a solve leaves its nodal values: FP64 solves store them, FP32
// solves add them to the FP64 solution (first: store) and track the norms.
__device__ __forceinline__ void put_node(double* u, unsigned i, double e, double o, bool first, Norms& n) {
  (void)first;
  (void)n;
  u[i] = e + o;
}
__device__ __forceinline__ void put_node(double* u, unsigned i, float e, float o, bool first, Norms& n) {
  const double dv = (double)e + (double)o;
  const double un = first ? dv : u[i] + dv;
  u[i] = un;
  n.add(dv, un);
}

// Block maxima of the waves' norms into the slots; red: 2 doubles per wave of LDS
// that no wave reads any more after the barrier.
__device__ __forceinline__ void flush_norms(const Norms& n, unsigned long long* norms, double* red) {
  double dmax = n.d, umax = n.u;
#pragma unroll
  for (int s = 32; s >= 1; s >>= 1) {
    dmax = fmax(dmax, __shfl_xor(dmax, s));
    umax = fmax(umax, __shfl_xor(umax, s));
  }
  __syncthreads();
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    red[2 * wave] = dmax;
    red[2 * wave + 1] = umax;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < (int)blockDim.x / 64; ++w) {
      dmax = fmax(dmax, red[2 * w]);
      umax = fmax(umax, red[2 * w + 1]);
    }
    norm_max(norms, dmax, umax);
  }
}

// ---- z axis: rows of n values, a strip is R = 16 TC rows ----------------------------
template <class T, class TI, int TT, int TC, int OP>
__global__ void row_kernel(StripArgs g) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  T* const V = reinterpret_cast<T*>(smem);
  constexpr int R = 16 * TC, NP = 4 * TC * TT;
  const long tile = xcd_tile();
  if (tile >= g.ntiles) return;  // the whole block
  const StripAxis ax = g.ax;
  const long p0 = tile * R;
  const int pmax = (int)min((long)R, g.P - p0) - 1;
  const int tid = threadIdx.x;
  const int lane = tid & 63, fr = lane & 15, fk = lane >> 4;
  const int t0 = __builtin_amdgcn_readfirstlane(tid >> 6) * TT, st = g.stride;
  // pair u of a thread: row 4 (u / TT) + lane / 16, representative m of its wave's tiles
  const int m0 = 16 * t0 + fr;

  const int K = pad4(ax.nrep), nk = K >> 2;
  auto ds = [&](int k, int j) { return V[(16 * j + fr) * st + 4 * k + fk]; };
  auto da = [&](int k, int j) { return V[(16 * j + fr) * st + K + 4 * k + fk]; };
  Norms norms;

  {
    TI pa[NP], pb[NP];
    const TI* x = reinterpret_cast<const TI*>(g.x) + (size_t)p0 * g.ldx;
#pragma unroll
    for (int u = 0; u < NP; ++u) {
      const int m = m0 + 16 * (u % TT), row = 4 * (u / TT);
      pa[u] = pb[u] = TI(0);
      if (m >= ax.nrep || row + fk > pmax) continue;
      const TI* src = x + (long)row * g.ldx;
      const unsigned v = (unsigned)(fk * g.ldx);
      pa[u] = src[v + m];
      if constexpr (OP == STRIP_BWD) {
        if (m < ax.nodd) pb[u] = src[v + ax.nrep + m];
      } else {
        pb[u] = src[v + refl(m, ax)];
      }
    }
#pragma unroll
    for (int u = 0; u < NP; ++u) {
      const int m = m0 + 16 * (u % TT);
      T* dst = V + (4 * (u / TT) + fk) * st;
      if (m >= K) continue;
      T s, v;
      pair_values<T, OP>(m, pa[u], pb[u], ax, &s, &v);
      dst[m] = s;
      dst[K + m] = v;
    }
  }
  __syncthreads();

  Acc<T, TT, TC> c;
  const unsigned w0 = (unsigned)(Mfma<T>::RL * fk * ax.n);  // the lane's part of an output row's address
  if constexpr (OP == STRIP_FWD) {
    T* y = reinterpret_cast<T*>(g.y) + (size_t)p0 * ax.n;
    dual_product<T, TT, TC, true>(c, g.fs, g.fa, g.tiles, nk, t0, ds, da);
#pragma unroll
    for (int j = 0; j < TC; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int rb = 16 * j + Mfma<T>::RB * r;
        if (rb + Mfma<T>::RL * fk > pmax) continue;
        T* yr = y + (long)rb * ax.n;
#pragma unroll
        for (int i = 0; i < TT; ++i) {
          const int l = 16 * (t0 + i) + fr;
          if (l < ax.nrep) yr[w0 + l] = c.s[i][j][r];
          if (l < ax.nodd) yr[w0 + ax.nrep + l] = c.a[i][j][r];
        }
      }
  } else {
    double* y = reinterpret_cast<double*>(g.y) + (size_t)p0 * ax.n;
    dual_product<T, TT, TC, true>(c, g.bs, g.ba, g.tiles, nk, t0, ds, da);
#pragma unroll
    for (int j = 0; j < TC; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int rb = 16 * j + Mfma<T>::RB * r;
        if (rb + Mfma<T>::RL * fk > pmax) continue;
        double* yr = y + (long)rb * ax.n;
#pragma unroll
        for (int i = 0; i < TT; ++i) {
          const int l = 16 * (t0 + i) + fr;
          if (l >= ax.nrep) continue;
          const int m = refl(l, ax);
          const T e = c.s[i][j][r], o = c.a[i][j][r];
          put_node(yr, w0 + l, e, o, g.first, norms);
          if (m != l) put_node(yr, w0 + m, e, -o, g.first, norms);
        }
      }
  }
  if constexpr (OP == STRIP_BWD && sizeof(T) == 4)
    if (g.norms) flush_norms(norms, g.norms, reinterpret_cast<double*>(smem));
}

// ---- small (y, z) planes: both axes in one block ----------------------------------------
// Two plane buffers: Z (rows of the z products, pitch stride) and Y (columns of the y
// products, pitch stride2).  Waves take (16 lines, 16 modes) tiles in turn.
template <class T, class TI, int OP>
__global__ void plane_kernel(StripArgs g) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const StripAxis az = g.ax, ay = g.ay;
  const int sz = g.stride, sy = g.stride2;
  T* const Z = reinterpret_cast<T*>(smem);
  T* const Y = Z + (size_t)((ay.n + 15) / 16 * 16) * sz;
  const int tid = threadIdx.x, nt = blockDim.x;
  const int lane = tid & 63, fr = lane & 15, fk = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), nw = nt >> 6;
  const long p = blockIdx.x;
  const int strips_z = (ay.n + 15) / 16, tiles_z = (az.nrep + 15) / 16;
  const int strips_y = (az.n + 15) / 16, tiles_y = (ay.nrep + 15) / 16;
  Norms norms;

  const TI* x = reinterpret_cast<const TI*>(g.x) + (size_t)p * ay.n * g.ldx;
  constexpr int LU = 4;
  const int Kz = pad4(az.nrep), Ky = pad4(ay.nrep);
  if constexpr (OP == STRIP_FWD) {
    const int cnt = ay.n * Kz;
    for (int i0 = tid; i0 < cnt; i0 += LU * nt) {
      TI a[LU], b[LU];
#pragma unroll
      for (int u = 0; u < LU; ++u) {
        const int i = min(i0 + u * nt, cnt - 1);
        const int row = i / Kz, m = min(i - row * Kz, az.nrep - 1);
        a[u] = x[(size_t)row * g.ldx + m];
        b[u] = x[(size_t)row * g.ldx + refl(m, az)];
      }
#pragma unroll
      for (int u = 0; u < LU; ++u) {
        const int i = i0 + u * nt;
        if (i >= cnt) break;
        const int row = i / Kz, m = i - row * Kz;
        T s = T(0), v = T(0);
        if (m < az.nrep) pair_values<T, OP>(m, a[u], b[u], az, &s, &v);
        Z[row * sz + m] = s;
        Z[row * sz + Kz + m] = v;
      }
    }
  } else {
    const int cnt = ay.n * az.n;
    for (int i0 = tid; i0 < cnt; i0 += LU * nt) {
      TI a[LU];
#pragma unroll
      for (int u = 0; u < LU; ++u) a[u] = x[min(i0 + u * nt, cnt - 1)];
#pragma unroll
      for (int u = 0; u < LU; ++u) {
        const int i = i0 + u * nt;
        if (i >= cnt) break;
        const int row = i / az.n;
        Y[row * sy + (i - row * az.n)] = (T)a[u];
      }
    }
  }
  __syncthreads();

  Acc<T, 1, 1> c;
  if constexpr (OP == STRIP_FWD) {
    // z: lines beyond ay.n of the last strip hold stale values; their outputs are
    // columns that nothing stores
    for (int w = wave; w < strips_z * tiles_z; w += nw) {
      const int s = w / tiles_z, t = w - s * tiles_z;
      const T* line = Z + (16 * s + fr) * sz;
      dual_product<T, 1, 1, true>(
          c, g.fs, g.fa, g.tiles, Kz >> 2, t, [&](int k, int) { return line[4 * k + fk]; },
          [&](int k, int) { return line[Kz + 4 * k + fk]; });
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = 16 * s + acc_row<T>(r, fk), l = 16 * t + fr;
        if (row >= ay.n) continue;
        if (l < az.nrep) Y[row * sy + l] = c.s[0][0][r];
        if (l < az.nodd) Y[row * sy + az.nrep + l] = c.a[0][0][r];
      }
    }
    __syncthreads();
    // y: folded as it is read
    T* y = reinterpret_cast<T*>(g.y) + (size_t)p * ay.n * az.n;
    for (int w = wave; w < strips_y * tiles_y; w += nw) {
      const int s = w / tiles_y, t = w - s * tiles_y;
      const T* col = Y + 16 * s + fr;
      dual_product<T, 1, 1, false>(
          c, g.fs2, g.fa2, g.tiles2, Ky >> 2, t,
          [&](int k, int) {
            const int m = min(4 * k + fk, ay.nrep - 1);
            return col[m * sy] + col[refl(m, ay) * sy];
          },
          [&](int k, int) {
            const int m = min(4 * k + fk, ay.nrep - 1);
            return col[m * sy] - col[refl(m, ay) * sy];
          });
      const int q = 16 * s + fr;
      if (q >= az.n) continue;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int l = 16 * t + acc_row<T>(r, fk);
        if (l < ay.nrep) y[(size_t)l * az.n + q] = c.s[0][0][r];
        if (l < ay.nodd) y[(size_t)(ay.nrep + l) * az.n + q] = c.a[0][0][r];
      }
    }
  } else {
    for (int w = wave; w < strips_y * tiles_y; w += nw) {
      const int s = w / tiles_y, t = w - s * tiles_y;
      const T* col = Y + 16 * s + fr;
      dual_product<T, 1, 1, false>(
          c, g.bs2, g.ba2, g.tiles2, Ky >> 2, t,
          [&](int k, int) { return col[min(4 * k + fk, ay.nrep - 1) * sy]; },
          [&](int k, int) { return col[min(ay.nrep + 4 * k + fk, ay.n - 1) * sy]; });
      const int q = 16 * s + fr;
      if (q >= az.n) continue;
      const int zq = q < az.nrep ? q : Kz + q - az.nrep;  // z modes as the z product reads them
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int l = 16 * t + acc_row<T>(r, fk);
        if (l >= ay.nrep) continue;
        const T e = c.s[0][0][r], o = c.a[0][0][r];
        Z[l * sz + zq] = e + o;
        const int m = refl(l, ay);
        if (m != l) Z[m * sz + zq] = e - o;
      }
    }
    __syncthreads();
    double* y = reinterpret_cast<double*>(g.y) + (size_t)p * ay.n * az.n;
    for (int w = wave; w < strips_z * tiles_z; w += nw) {
      const int s = w / tiles_z, t = w - s * tiles_z;
      const T* line = Z + (16 * s + fr) * sz;
      dual_product<T, 1, 1, true>(
          c, g.bs, g.ba, g.tiles, Kz >> 2, t,
          [&](int k, int) { return line[min(4 * k + fk, az.nrep - 1)]; },
          [&](int k, int) { return line[4 * k + fk < az.nodd ? Kz + 4 * k + fk : 0]; });
      const int l = 16 * t + fr, m = refl(l, az);
      if (l >= az.nrep) continue;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = 16 * s + acc_row<T>(r, fk);
        if (row >= ay.n) continue;
        const T e = c.s[0][0][r], o = c.a[0][0][r];
        put_node(y, (size_t)row * az.n + l, e, o, g.first, norms);
        if (m != l) put_node(y, (size_t)row * az.n + m, e, -o, g.first, norms);
      }
    }
    if constexpr (sizeof(T) == 4)
      if (g.norms) flush_norms(norms, g.norms, reinterpret_cast<double*>(smem));
  }
}

constexpr size_t LDS_MAX = 160 * 1024;
constexpr int MAX_WAVES = 16;
// Largest plane that one block takes: two launches fewer, but a block a plane.  Solve in
// planes / in separate launches: FP64 31^3 17.2 / 19.5 us, 47^3 21.7 / 21.2, 63^3 25.7 /
// 23.2, 95^3 59 / 44; FP32 31^3 16.3 / 19.2, 63^3 21.3 / 21.6, 95^3 45 / 34.
constexpr size_t PLANE_BYTES = 48 * 48 * 8;

// Smallest pitches >= len at which a fragment read meets no bank twice: 16 rows x 4
// consecutive values (FP64: 2 at a time), or 4 (2) rows x 16 values.
inline int pitch_rows(int len, int elem) {
  return elem == 8 ? (len - 2 + 31) / 32 * 32 + 2 : (len - 34 + 63) / 64 * 64 + 34;
}
inline int pitch_cols(int len, int elem) {
  return elem == 8 ? (len - 16 + 31) / 32 * 32 + 16 : (len - 16 + 63) / 64 * 64 + 16;
}
inline int pad16(int n) { return (n + 15) / 16 * 16; }
// elements of a line in a strip
inline int strip_len(const StripAxis& a) { return 2 * pad4(a.nrep); }

template <class K>
hipError_t launch(K kernel, const StripArgs& g, long blocks, int waves, size_t lds, hipStream_t s) {
  if (blocks <= 0) return hipSuccess;
  if (blocks > 0x7fffffffL || lds > LDS_MAX) return hipErrorInvalidValue;
  kernel<<<dim3((unsigned)blocks), dim3(64 * waves), lds, s>>>(g);
  return hipGetLastError();
}

// Lines of a strip (1 or 2 times 16) for P groups of Q lines: the fewer strips per CU,
// counting a quarter of a 16-line strip for what does not shrink with it.  Solves with
// 16 / 32 lines everywhere: FP64 255^3 646 / 624 us, 511^3 7945 / 7408, but 95^3 44 / 52,
// (449, 59, 59) 80 / 110 (too few strips); FP32 255^3 429 / 381, 95^3 36 / 42.  64 lines
// are no faster (FP32 255^3 379, 511^3 4290 against 4304).
inline int strip_cols(long P, long Q, size_t line_bytes) {
  auto cost = [&](int c) { return (double)((P * ((Q + 16 * c - 1) / (16 * c)) + 255) / 256) * (c + 0.25); };
  return 32 * line_bytes <= LDS_MAX && cost(2) <= cost(1) ? 2 : 1;
}

}  // namespace stripk

// Waves of a strip block take one tile of 16 modes each, two past nrep = 256, 16 waves
// at most: axes of up to 1024 nodes (1023 periodic), whose 16 FP64 lines fill 128 KB of
// LDS.  FP64 solves with tiles / strips: 539^3 16.2 / 13.4 ms, 639^3 25.7 / 23.1, 799^3
// 63.6 / 49.6, 999^3 119.9 / 99.6 (59.9 TFLOP/s of the halved products, 0.82 of what the
// library's FP64 product reaches); FP32 application 999^3 104 / 61 ms.
bool strip_axis_ok(const StripAxis& a, int elem) {
  using namespace stripk;
  return a.nrep <= 2 * 16 * MAX_WAVES && (size_t)pitch_rows(strip_len(a), elem) * elem * 16 <= LDS_MAX;
}

bool strip_plane_ok(const StripAxis& ay, const StripAxis& az, int elem) {
  using namespace stripk;
  return (size_t)ay.n * az.n * elem <= PLANE_BYTES && strip_axis_ok(ay, elem) && strip_axis_ok(az, elem) &&
         (size_t)pad16(ay.n) * (pitch_rows(strip_len(az), elem) + pitch_cols(pad16(az.n), elem)) * elem <= LDS_MAX;
}

template <class T, int TT, int OP, bool SPECTRAL>
static hipError_t col_launch(StripArgs g, hipStream_t s) {
  using namespace stripk;
  const int waves = (g.ax.nrep + 16 * TT - 1) / (16 * TT);
  g.tiles = strip_tiles(g.ax.nrep);
  const size_t line = (size_t)strip_len(g.ax) * sizeof(T);
  // (FP64, two tiles a wave: 32 lines would spill at 16 waves)
  constexpr bool WIDE = TT * sizeof(T) < 16;
  const int tc = WIDE ? strip_cols(g.P, g.Q, line) : 1;
  g.ntiles = (g.Q + 16 * tc - 1) / (16 * tc) * g.P;
  const long blocks = (g.ntiles + 7) / 8 * 8;
  if constexpr (WIDE)
    if (tc == 2) return launch(col_kernel<T, TT, 2, OP, SPECTRAL>, g, blocks, waves, 32 * line, s);
  return launch(col_kernel<T, TT, 1, OP, SPECTRAL>, g, blocks, waves, 16 * line, s);
}

template <class T, int OP, bool SPECTRAL = false>
static hipError_t col_tiles(const StripArgs& g, hipStream_t s) {
  if (g.ax.nrep > 16 * stripk::MAX_WAVES) return col_launch<T, 2, OP, SPECTRAL>(g, s);
  return col_launch<T, 1, OP, SPECTRAL>(g, s);
}

template <class T>
hipError_t launch_strip_col(const StripArgs& g, int op, hipStream_t s) {
  if (!strip_axis_ok(g.ax, sizeof(T)) || g.P < 1 || g.Q < 1 || g.Q > STRIP_MAX_Q) return hipErrorInvalidValue;
  if (op == STRIP_FWD) return col_tiles<T, STRIP_FWD>(g, s);
  if (op == STRIP_BWD) return col_tiles<T, STRIP_BWD>(g, s);
  if (g.P != 1) return hipErrorInvalidValue;
  if constexpr (sizeof(T) == 8)
    if (g.epi.kind) return col_tiles<T, STRIP_MUL, true>(g, s);
  return col_tiles<T, STRIP_MUL>(g, s);
}

template <class T, class TI, int TT, int OP>
static hipError_t row_launch(StripArgs g, hipStream_t s) {
  using namespace stripk;
  const int waves = (g.ax.nrep + 16 * TT - 1) / (16 * TT);
  g.tiles = strip_tiles(g.ax.nrep);
  g.stride = pitch_rows(strip_len(g.ax), sizeof(T));
  const size_t line = (size_t)g.stride * sizeof(T);
  constexpr bool WIDE = TT * sizeof(T) < 16;
  const int tc = WIDE ? strip_cols(1, g.P, line) : 1;
  g.ntiles = (g.P + 16 * tc - 1) / (16 * tc);
  const long blocks = (g.ntiles + 7) / 8 * 8;
  if constexpr (WIDE)
    if (tc == 2) return launch(row_kernel<T, TI, TT, 2, OP>, g, blocks, waves, 32 * line, s);
  return launch(row_kernel<T, TI, TT, 1, OP>, g, blocks, waves, 16 * line, s);
}

template <class T, class TI, int OP>
static hipError_t row_tiles(const StripArgs& g, hipStream_t s) {
  if (g.ax.nrep > 16 * stripk::MAX_WAVES) return row_launch<T, TI, 2, OP>(g, s);
  return row_launch<T, TI, 1, OP>(g, s);
}

template <class T, class TI>
hipError_t launch_strip_row(const StripArgs& g, int op, hipStream_t s) {
  if (!strip_axis_ok(g.ax, sizeof(T)) || g.P < 1 || g.ldx < g.ax.n) return hipErrorInvalidValue;
  if (op == STRIP_FWD) return row_tiles<T, TI, STRIP_FWD>(g, s);
  return row_tiles<T, T, STRIP_BWD>(g, s);
}

template <class T, class TI>
hipError_t launch_strip_plane(StripArgs g, int op, hipStream_t s) {
  using namespace stripk;
  if (!strip_plane_ok(g.ay, g.ax, sizeof(T)) || g.P < 1 || g.ldx < g.ax.n || (op == STRIP_BWD && g.ldx != g.ax.n))
    return hipErrorInvalidValue;
  g.tiles = strip_tiles(g.ax.nrep);
  g.tiles2 = strip_tiles(g.ay.nrep);
  g.stride = pitch_rows(strip_len(g.ax), sizeof(T));
  g.stride2 = pitch_cols(pad16(g.ax.n), sizeof(T));
  const size_t lds = (size_t)pad16(g.ay.n) * (g.stride + g.stride2) * sizeof(T);
  // waves: the larger of the two products' tiles in as few equal rounds as possible
  const int items = std::max((g.ay.n + 15) / 16 * ((g.ax.nrep + 15) / 16), (g.ax.n + 15) / 16 * ((g.ay.nrep + 15) / 16));
  const int rounds = (items + MAX_WAVES - 1) / MAX_WAVES;
  const int waves = (items + rounds - 1) / rounds;
  if (op == STRIP_FWD) return launch(plane_kernel<T, TI, STRIP_FWD>, g, g.P, waves, lds, s);
  return launch(plane_kernel<T, T, STRIP_BWD>, g, g.P, waves, lds, s);
}

template hipError_t launch_strip_col<double>(const StripArgs&, int, hipStream_t);
template hipError_t launch_strip_row<double, double>(const StripArgs&, int, hipStream_t);
template hipError_t launch_strip_plane<double, double>(StripArgs, int, hipStream_t);
template hipError_t launch_strip_col<float>(const StripArgs&, int, hipStream_t);
template hipError_t launch_strip_row<float, double>(const StripArgs&, int, hipStream_t);
template hipError_t launch_strip_row<float, float>(const StripArgs&, int, hipStream_t);
template hipError_t launch_strip_plane<float, double>(StripArgs, int, hipStream_t);
template hipError_t launch_strip_plane<float, float>(StripArgs, int, hipStream_t);

}  // namespace semfd
