// The blocks K_k = lambda_k I - c_k J (c_k = tau mu_k, Section 3.2) in hierarchical form.
//
// Structure.  J = scale (D+ G + D- G^T) with G Toeplitz (eq. (1.4)-(1.5)).  Split a range of rows
// at c: below the diagonal the block couples row c + p to column c - 1 - q by
//   scale (d+_{c+p} g_{p+q+2} + [p = q = 0] d-_c g_0),
// and above it the same with the sides exchanged and d+-, d-+.  H = [g_{p+q+2}] is a positive
// definite Hankel matrix (g_k is a Beta integral over (0, 1), a moment sequence), and its
// singular values fall fast: H = X X^T to FP64 rounding with 18 columns at order 64 and 31 at
// order 2048 (a pivoted Cholesky factor, set up by the host in extended precision).  With
// column 0 of the table holding e_0 (the g_0 entry) every off-diagonal block of every K_k is
//   -c_k  U V^T,   V = X (rows counted from c, mirrored on the left side),   U = scale diag(d) X,
// U and V real and the same for all frequencies.  Leaves are 64 rows; level l joins two ranges of
// h = 64 << l rows.  With y_i = K_ii^{-1} b_i (i = 1 left, 2 right), W_i = K_ii^{-1} U_i,
// G_i = -c V_i^T W_i, a_i = V_i^T y_i, block elimination gives
//   x_1 = y_1 - W_1' (a_2 - G_2 a_1),   W_1' = -c W_1 (I - G_2 G_1)^{-1},
//   x_2 = y_2 - W_2' (a_1 - G_1 a_2),   W_2' = -c W_2 (I - G_1 G_2)^{-1}.
// All the diagonal blocks that this inverts are principal blocks of a strictly row diagonally
// dominant matrix (Prop. 2.2 with Re(lambda_k conj mu_k) >= 0, which the host checks), the reason
// that the pivot-free dense LU is stable, and are dominant themselves.
//
// Per frequency this stores the leaf inverses (64 m numbers) and W' (about 25 m per level)
// instead of m^2 (dense LU) or m^2 / 2 (the band route's U), and needs no reduction of J.
//
// Layouts (c_t<T>; k frequency, R = hR[l], a multiple of 4, at most 32):
//   hD [nb][npan][64 columns][64 rows]       leaf inverses
//   hW per level: [nb][npan][R][64]          W', panel by panel, rows contiguous: a wavefront of the
//                                            apply streams one block of 64 R numbers
//   hG per level: [nb][node][2][R][R]        G_1, G_2, column by column
//   hx per level: [h][32] double             X, column 0 = e_0, zero beyond the level's rank
//   ha [2][nb][npan][32]                     a, one partial sum per 64-row panel
#include "batch.hpp"
#include "common.hpp"
#include "kernels.hpp"

namespace fde {

static constexpr int HP = 64;       // leaf order, panel
static constexpr int HCH = HIER_CHUNK;

template <typename T>
__device__ __forceinline__ c_t<T> hmul(c_t<T> a, c_t<T> b) {
  return mk<T>(fma(a.x, b.x, -a.y * b.y), fma(a.x, b.y, a.y * b.x));
}
// acc - a b
template <typename T>
__device__ __forceinline__ c_t<T> hfms(c_t<T> a, c_t<T> b, c_t<T> acc) {
  acc.x = fma(-a.x, b.x, acc.x);
  acc.x = fma(a.y, b.y, acc.x);
  acc.y = fma(-a.x, b.y, acc.y);
  acc.y = fma(-a.y, b.x, acc.y);
  return acc;
}
template <typename T>
__device__ __forceinline__ c_t<T> hfma(c_t<T> a, c_t<T> b, c_t<T> acc) {
  acc.x = fma(a.x, b.x, acc.x);
  acc.x = fma(-a.y, b.y, acc.x);
  acc.y = fma(a.x, b.y, acc.y);
  acc.y = fma(a.y, b.x, acc.y);
  return acc;
}
// global loads of complex values (see gld)
template <typename T> __device__ __forceinline__ c_t<T> cload(const c_t<T> *p) { return gld(p); }
// the same for data that one apply reads once (the caches are left to X, G and the vector)
template <typename T> __device__ __forceinline__ c_t<T> cload_once(const c_t<T> *p) {
  typedef T nv __attribute__((ext_vector_type(2)));
  typedef __attribute__((address_space(1))) const nv gnv;
  const nv v = __builtin_nontemporal_load((gnv *)p);
  return mk<T>(v.x, v.y);
}

// -c_k = -tau mu_k
template <typename T>
__device__ __forceinline__ c_t<T> minus_c(const InstDesc &d, int k) {
  const double2 mu = d.mu[k];
  return mk<T>((T)(-d.tau * mu.x), (T)(-d.tau * mu.y));
}

template <typename T>
__device__ __forceinline__ c_t<T> *hier_w(const InstDesc &d, int lev, int k) {
  return (c_t<T> *)d.hW[lev] + (size_t)k * d.hR[lev] * d.mp;  // panel p at p R 64
}
template <typename T>
__device__ __forceinline__ c_t<T> *hier_g(const InstDesc &d, int lev, int k, int node) {
  const int R = d.hR[lev];
  return (c_t<T> *)d.hG[lev] + ((size_t)k * hier_nodes(d.mp, lev) + node) * 2 * R * R;
}
__device__ __forceinline__ const double *hier_x(const InstDesc &d, int lev) {
  return d.hx + (size_t)((HP << lev) - HP) * 32;
}

__device__ __forceinline__ void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Data movement between lanes (li, lk) = (lane % 16, lane / 16) without LDS.
template <int CTRL> __device__ __forceinline__ int dpp_mov(int v) {
  return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, true);
}
template <int CTRL> __device__ __forceinline__ float dpp_mov(float v) { return __int_as_float(dpp_mov<CTRL>(__float_as_int(v))); }
template <int CTRL> __device__ __forceinline__ double dpp_mov(double v) {
  return __hiloint2double(dpp_mov<CTRL>(__double2hiint(v)), dpp_mov<CTRL>(__double2loint(v)));
}
// lane li = I of the same lk
template <int I, typename V> __device__ __forceinline__ V row_bcast(V v) {
  v.x = dpp_mov<0x150 + I>(v.x);
  v.y = dpp_mov<0x150 + I>(v.y);
  return v;
}
// lane `src` (through LDS's crossbar)
__device__ __forceinline__ float lane_get(float v, int src) {
  return __int_as_float(__builtin_amdgcn_ds_bpermute(4 * src, __float_as_int(v)));
}
__device__ __forceinline__ double lane_get(double v, int src) {
  return __hiloint2double(__builtin_amdgcn_ds_bpermute(4 * src, __double2hiint(v)),
                          __builtin_amdgcn_ds_bpermute(4 * src, __double2loint(v)));
}
// the same for one lane of the wavefront
__device__ __forceinline__ float lane_read(float v, int src) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), src));
}
__device__ __forceinline__ double lane_read(double v, int src) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), src), __builtin_amdgcn_readlane(__double2loint(v), src));
}
// 1 / v by the hardware's estimate and Newton steps (within an ulp; NaN for 0 and infinities, which
// the pivots' final check counts on)
__device__ __forceinline__ float recip(float v) {
  const float r = __builtin_amdgcn_rcpf(v);
  return fmaf(r, fmaf(-v, r, 1.0f), r);
}
__device__ __forceinline__ double recip(double v) {
  double r = __builtin_amdgcn_rcp(v);
  r = fma(r, fma(-v, r, 1.0), r);
  return fma(r, fma(-v, r, 1.0), r);
}
template <typename T> __device__ __forceinline__ c_t<T> inverse(c_t<T> p) {
  const T iv = recip(p.x * p.x + p.y * p.y);
  return mk<T>(p.x * iv, -p.y * iv);
}

// A barrier for data in LDS alone: stores to global memory stay in flight across it.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// ------------------------------------------------------------------------------------
// Products of 16 x 16 tiles.  A tile of results sits in the lane layout that the next product reads
// as its right operand, so a chain of products stays in registers: lane (li, lk) holds column li.
// Along a panel its rows are MFMA's own, mfma_row(lk, v): loads and stores of a tile then move 64
// (FP64) or 32 (FP32, two 16-byte accesses a lane) consecutive bytes of 16 columns at a time.  Along
// the R columns of V they are 4 v + lk (left operand rows by rowstr), of which those from R on are
// whole steps and are skipped.
template <typename T> __device__ __forceinline__ int rowstr(int i);
template <> __device__ __forceinline__ int rowstr<double>(int i) { return i; }
template <> __device__ __forceinline__ int rowstr<float>(int i) { return 4 * (i & 3) + (i >> 2); }

template <typename T> struct ctile {
  acc_t<T> re, im;
  __device__ __forceinline__ void zero() { re = im = acc_t<T>{0, 0, 0, 0}; }
};
template <typename T>
__device__ __forceinline__ void tile_fma(ctile<T> &c, c_t<T> a, T bx, T by) {
  c.re = mfma16(a.x, bx, c.re);
  c.re = mfma16(-a.y, by, c.re);
  c.im = mfma16(a.x, by, c.im);
  c.im = mfma16(a.y, bx, c.im);
}
template <typename T>
__device__ __forceinline__ void tile_fms(ctile<T> &c, c_t<T> a, T bx, T by) {
  c.re = mfma16(-a.x, bx, c.re);
  c.re = mfma16(a.y, by, c.re);
  c.im = mfma16(-a.x, by, c.im);
  c.im = mfma16(-a.y, bx, c.im);
}
template <typename T>
__device__ __forceinline__ void tile_fma(ctile<T> &c, T a, T bx, T by) {
  c.re = mfma16(a, bx, c.re);
  c.im = mfma16(a, by, c.im);
}

// Gauss-Jordan without pivoting on a 16 x 16 block that a wavefront holds as a left operand: lane
// (li, lk) row li, columns mfma_row(lk, s).  A pivot row is scaled at the end (rinv), which saves the
// selects of a row treated apart in every step.
template <typename T, int I>
__device__ __forceinline__ void gj16_step(c_t<T> *a, c_t<T> &rinv, int lane) {
  constexpr int lkp = sizeof(T) == 8 ? I & 3 : I >> 2, sp = sizeof(T) == 8 ? I >> 2 : I & 3;
  const int li = lane & 15, lk = lane >> 4;
  const c_t<T> f = mk<T>(lane_get(a[sp].x, 16 * lkp + li), lane_get(a[sp].y, 16 * lkp + li));
  const c_t<T> inv = inverse<T>(row_bcast<I>(f));
  const bool own = li == I;
  const c_t<T> t = hmul<T>(mk<T>(own ? (T)0 : f.x, own ? (T)0 : f.y), inv);
#pragma unroll
  for (int s = 0; s < 4; ++s) a[s] = hfms<T>(t, row_bcast<I>(a[s]), a[s]);
  if (lk == lkp) a[sp] = mk<T>(own ? (T)1 : -t.x, -t.y);
  if (own) rinv = inv;
}
template <typename T, int I>
__device__ __forceinline__ void gj16_from(c_t<T> *a, c_t<T> &rinv, int lane) {
  if constexpr (I < 16) {
    gj16_step<T, I>(a, rinv, lane);
    gj16_from<T, I + 1>(a, rinv, lane);
  }
}
template <typename T>
__device__ __forceinline__ void gj16(c_t<T> *a, int lane) {
  c_t<T> rinv = mk<T>((T)1, (T)0);
  gj16_from<T, 0>(a, rinv, lane);
#pragma unroll
  for (int s = 0; s < 4; ++s) a[s] = hmul<T>(a[s], rinv);
}

// In-place inverse of an R x R matrix in LDS ([column][row], stride R) by the four wavefronts w of
// a group, Gauss-Jordan with partial pivoting and no row exchanges: lane (r, half) holds row r,
// columns 8 i + 2 w + half.  Every wavefront of the workgroup calls it (one barrier a step).  col: 64
// entries of LDS, piv: 32.
template <typename T> __device__ __forceinline__ unsigned mag_key(T m2);
template <> __device__ __forceinline__ unsigned mag_key<float>(float m2) { return __float_as_uint(m2); }
template <> __device__ __forceinline__ unsigned mag_key<double>(double m2) { return (unsigned)__double2hiint(m2); }

template <typename T>
__device__ __forceinline__ void group_invert(c_t<T> *M, int R, int w, c_t<T> *col, int *piv, bool &bad) {
  const int lane = threadIdx.x & 63, r = lane & 31, hf = lane >> 5;
  c_t<T> a[4], rinv = mk<T>((T)1, (T)0);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int c = 8 * i + 2 * w + hf;
    const bool in = r < R && c < R;
    const c_t<T> v = M[in ? c * R + r : 0];
    a[i] = mk<T>(in ? v.x : (T)0, in ? v.y : (T)0);
  }
  bool used = r >= R;
  int mine = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll 1
    for (int j = 8 * i; j < min(R, 8 * i + 8); ++j) {
      const bool owner = w == ((j >> 1) & 3) && hf == (j & 1);
      if (owner) col[32 * (j & 1) + r] = a[i];
      lds_barrier();
      const c_t<T> v = col[32 * (j & 1) + r];
      // the largest entry (to 15 bits) in a row not used yet, the first of equals
      unsigned key = used ? 0u : (mag_key<T>(v.x * v.x + v.y * v.y) & ~31u) | (unsigned)(31 - r);
      key = max(key, (unsigned)dpp_mov<0x128>((int)key));
      key = max(key, (unsigned)dpp_mov<0x124>((int)key));
      key = max(key, (unsigned)dpp_mov<0x122>((int)key));
      key = max(key, (unsigned)dpp_mov<0x121>((int)key));
      const int pr = 31 - (int)(max((unsigned)__builtin_amdgcn_readlane((int)key, 0),
                                    (unsigned)__builtin_amdgcn_readlane((int)key, 16)) & 31);
      const c_t<T> inv = inverse<T>(mk<T>(lane_read(v.x, pr), lane_read(v.y, pr)));
      const bool own = r == pr;
      const c_t<T> t = hmul<T>(mk<T>(own ? (T)0 : v.x, own ? (T)0 : v.y), inv);
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (8 * q < R) a[q] = hfms<T>(t, mk<T>(lane_get(a[q].x, 32 * hf + pr), lane_get(a[q].y, 32 * hf + pr)), a[q]);
      if (owner) a[i] = mk<T>(own ? (T)1 : -t.x, -t.y);
      if (own) {
        rinv = inv;
        used = true;
        mine = j;
        piv[j] = pr;  // every wavefront of the group writes the same
      }
    }
  lds_barrier();
  // row r holds the unknown that it was the pivot of, column c the right-hand side of c's pivot row
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int c = 8 * i + 2 * w + hf;
    if (r < R && c < R) {
      const c_t<T> v = hmul<T>(a[i], rinv);
      bad = bad || !isfinite(v.x + v.y);
      M[piv[c] * R + mine] = v;
    }
  }
}

// ------------------------------------------------------------------------------------
// Leaf inverses, the W columns of all levels from them (K_leaf^{-1} U), and level 0 in full.
// Item = (instance, block, pair of panels); eight wavefronts, four to a leaf.
//
// Leaf.  Wavefront w of a leaf holds columns 16 w .. + 15 of the 64 x 64 diagonal block as four
// tiles, and block Gauss-Jordan (no pivoting: strict row dominance) runs over its four 16-column
// blocks: the owner puts the block into LDS, every wavefront inverts the 16 x 16 pivot for itself
// (16 dependent steps, no barrier), and updates its tiles on MFMA.  One barrier per block.
//
// Newton.  X <- X + X (I - K X).  Gauss-Jordan leaves an error of cond(K_leaf) eps in X (the leaf of
// a frequency near zero is close to a singular M-matrix), the largest error of the whole form; the
// step takes it to the size of X's own rounding (forward errors of S^{-1} v 5 to 20 times
// smaller).  In FP64 K is the matrix of rounded entries that the dense routes factor: an ulp of its
// diagonal moves S^{-1} v by more (3e-13 at 1000 x 128) than all rounding from there on (5e-14).  In
// FP32, K X = lambda X - c (J X) with J real, half the products, and all of it in FP64: X's own rounding
// is then what is left of the leaf's error.  In FP32 the weights g are off by the same amount in
// every row (by nothing where alpha, the diagonal's weight, is an FP32 number), and with constant
// coefficients so are the entries and the sums; such errors add up over the leaves where others cancel.
// Error of a single application at 1800 x 8, alpha = 1.3: 3.6e-4 with the residual in FP32, 8e-6 so,
// 6.2e-5 with dense FP32 factors; the kernel at 4095 x 256: 1.08 and 1.14 ms.
//
// Level 0.  W_0 and G on two wavefronts per leaf (a 16-column tile each), the R x R inverse and W_0' on
// four.  The columns of the levels above then pass through the pair, one 16-column tile of one leaf
// per wavefront, U -> K_leaf^{-1} U -> A -> z -> W - W_0' z, without leaving registers (the two
// wavefronts of a tile exchange their A): they are written once, where separate kernels for the
// leaves, the columns and level 0 wrote them twice and read them three times.
//
// In FP64 one workgroup fills a CU's LDS, so what counts is that its phases are short: MFMA is busy
// 0.49 of the time, 0.46 mixed (block Gauss-Jordan is bound by its 16-step chains, the R x R inverses by theirs
// of 20), and the code (54 KB) stays within the instruction cache, with the block loop rolled.  4095 x
// 256: 2.91 ms FP64 and 1.14 mixed (two workgroups per CU) for leaves, columns and level 0, from 4.48
// and 1.94 in four launches with three passes over the columns.
template <typename T> struct HierLds {
  static constexpr int R0 = sizeof(T) == 8 ? HIER_R0 : HIER_R0_32;  // level 0's largest rank
  // behind the two leaves: two R0 x R0 matrices and four columns of 32 for their inverses; later the
  // exchange of A, R0 x 16 real numbers per wavefront
  static constexpr size_t leaves = 2 * HP * HP * sizeof(c_t<T>);
  static constexpr size_t small = (2 * R0 * R0 + 128) * sizeof(c_t<T>), swap = 8 * R0 * 16 * sizeof(T);
  static constexpr size_t bytes = leaves + (small > swap ? small : swap);
};
// [column][row] of a leaf in LDS; rows are exchanged within 16 so that a column read (16 rows) and a
// tile write (16 columns) both meet every bank once
__device__ __forceinline__ int lx(int c, int r) { return c * HP + (r ^ (c & 15)); }

template <typename T, int N> __device__ __forceinline__ void zero_tiles(ctile<T> *t) {
#pragma unroll
  for (int i = 0; i < N; ++i) t[i].zero();
}
// K_leaf^{-1} U for one column per li: U's column `col` of level lev at panel p, X its leaf inverse
template <typename T>
__device__ __forceinline__ void leaf_tile(const InstDesc &d, const c_t<T> *X, int lane, int p, int lev, int col, bool ok,
                                          ctile<T> *W) {
  const int li = lane & 15, lk = lane >> 4, m = d.m;
  const int side = (p >> lev) & 1, c = (2 * (p >> (lev + 1)) + 1) << lev;  // first panel of the right half
  ok = ok && c < d.npan;
  // the e_0 column carries the other side's coefficient (the g_0 entry next to the diagonal)
  const double *dv = (side == 0) != (col == 0) ? d.dm : d.dp;
  const double *tab = hier_x(d, lev) + col;
  T u[16];
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int i = 16 * (e >> 2) + mfma_row<T>(lk, e & 3), row = p * HP + i;
    const int pi = side ? (p - c) * HP + i : (c - p) * HP - 1 - i;
    const bool in = ok && row < m;
    const double t = d.scale * (gld(dv + (row < m ? row : 0)) * gld(tab + (in ? pi : 0) * 32));
    u[e] = in ? (T)t : (T)0;
  }
#pragma unroll
  for (int mt = 0; mt < 4; ++mt) W[mt].zero();
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int k = 16 * (e >> 2) + mfma_row<T>(lk, e & 3);
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
      const c_t<T> a = X[lx(k, 16 * mt + li)];
      W[mt].re = mfma16(a.x, u[e], W[mt].re);
      W[mt].im = mfma16(a.y, u[e], W[mt].im);
    }
  }
}
// The products below take R <= 4 NE rows or columns: tiles of 4 NE with zeros in rows R and above.
// a += V^T B over the 64 rows of a panel: tab the level's table, row i of the panel at row off + dir i
// of it
template <typename T, int NE>
__device__ __forceinline__ void panel_gram(const double *tab, int lane, int off, int dir, int R, const ctile<T> *B, ctile<T> *a) {
  constexpr int NT = (NE + 3) / 4;
  const int li = lane & 15, lk = lane >> 4;
  T x[NT][16];
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const double *row = tab + (off + dir * (16 * (e >> 2) + mfma_row<T>(lk, e & 3))) * 32;
#pragma unroll
    for (int rt = 0; rt < NT; ++rt) {
      const int r = 16 * rt + rowstr<T>(li);
      const double v = gld(row + r);
      x[rt][e] = r < R ? (T)v : (T)0;
    }
  }
#pragma unroll
  for (int e = 0; e < 16; ++e)
#pragma unroll
    for (int rt = 0; rt < NT; ++rt) tile_fma<T>(a[rt], x[rt][e], B[e >> 2].re[e & 3], B[e >> 2].im[e & 3]);
}
// c -= (row tile rt of G) a for R x R G ([column][row]), in LDS or in global memory
template <typename T, int NE, bool LDS>
__device__ __forceinline__ void small_fms(const c_t<T> *G, int lane, int R, int rt, const ctile<T> *a, ctile<T> &c) {
  const int r = 16 * rt + rowstr<T>(lane & 15), lk = lane >> 4;
  c_t<T> g[NE];
#pragma unroll
  for (int e = 0; e < NE; ++e) {
    const int cc = 4 * e + lk;
    const c_t<T> *at = G + (r < R && cc < R ? cc * R + r : 0), v = LDS ? *at : cload<T>(at);
    g[e] = mk<T>(r < R ? v.x : (T)0, r < R ? v.y : (T)0);
  }
#pragma unroll
  for (int e = 0; e < NE; ++e) tile_fms<T>(c, g[e], a[e >> 2].re[e & 3], a[e >> 2].im[e & 3]);
}
// B -= W' z over the 64 rows of a panel (W: its R columns)
template <typename T, int NE>
__device__ __forceinline__ void panel_update(const c_t<T> *W, int lane, int R, const ctile<T> *z, ctile<T> *B) {
  const int li = lane & 15, lk = lane >> 4;
  W += li;
#pragma unroll
  for (int e = 0; e < NE; ++e) {
    const int cc = 4 * e + lk;
    c_t<T> w[4];
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) w[mt] = cload<T>(W + (cc < R ? cc : 0) * HP + 16 * mt);
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) tile_fms<T>(B[mt], w[mt], z[e >> 2].re[e & 3], z[e >> 2].im[e & 3]);
  }
}
// W <- mc W Q, R x R Q in LDS, over 16 rows of n panels
template <typename T, int NE>
__device__ __forceinline__ void scale_rows(c_t<T> *W, int n, int R, const c_t<T> *Q, c_t<T> mc, int lane) {
  constexpr int NT = (NE + 3) / 4;
  const int li = lane & 15, lk = lane >> 4;
  c_t<T> q[NT][NE];
#pragma unroll
  for (int ct = 0; ct < NT; ++ct)
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      const int c = 16 * ct + li, r = 4 * e + lk;
      const bool in = c < R && r < R;
      const c_t<T> b = hmul<T>(mc, Q[in ? c * R + r : 0]);
      q[ct][e] = mk<T>(in ? b.x : (T)0, in ? b.y : (T)0);
    }
#pragma unroll 1
  for (int pp = 0; pp < n; ++pp, W += R * HP) {
    c_t<T> a[NE];
#pragma unroll
    for (int e = 0; e < NE; ++e) a[e] = cload<T>(W + (4 * e + lk < R ? 4 * e + lk : 0) * HP + li);
    ctile<T> o[NT];
    zero_tiles<T, NT>(o);
#pragma unroll
    for (int e = 0; e < NE; ++e)
#pragma unroll
      for (int ct = 0; ct < NT; ++ct) tile_fma<T>(o[ct], a[e], q[ct][e].x, q[ct][e].y);
#pragma unroll
    for (int ct = 0; ct < NT; ++ct)
      if (16 * ct + li < R) {
#pragma unroll
        for (int v = 0; v < 4; ++v) W[(16 * ct + li) * HP + mfma_row<T>(lk, v)] = mk<T>(o[ct].re[v], o[ct].im[v]);
      }
  }
}
template <typename T>
__device__ __forceinline__ void panel_load(const c_t<T> *in, ctile<T> *B) {
#pragma unroll
  for (int mt = 0; mt < 4; ++mt)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const c_t<T> x = cload<T>(in + 16 * mt + mfma_row<T>(0, v));
      B[mt].re[v] = x.x;
      B[mt].im[v] = x.y;
    }
}
template <typename T>
__device__ __forceinline__ void panel_store(c_t<T> *o, const ctile<T> *B) {
#pragma unroll
  for (int mt = 0; mt < 4; ++mt)
#pragma unroll
    for (int v = 0; v < 4; ++v) o[16 * mt + mfma_row<T>(0, v)] = mk<T>(B[mt].re[v], B[mt].im[v]);
}

template <typename T>
__global__ __launch_bounds__(512, sizeof(T) == 8 ? 2 : 4) void k_hier_leaf(const InstDesc *__restrict__ Dd, ItemMap map, int *flag) {
  extern __shared__ double hier_lds[];
  __shared__ double gt[2 * HP];  // g_t at index t + 63, zero for t < 0
  __shared__ int piv[2][32];
  const int q = item_slot(map, blockIdx.x);
  const InstDesc &d = Dd[map.ids[q]];
  const int local = blockIdx.x - map.pre[q];
  const int npan = d.npan, m = d.m, pairs = (npan + 1) / 2, k = local / pairs, pair = local % pairs;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  const int leaf = wv >> 2, w = wv & 3, p = 2 * pair + leaf;
  const bool mine = p < npan, live = 2 * pair + 1 < npan;
  c_t<T> *LX = (c_t<T> *)hier_lds + leaf * HP * HP;
  c_t<T> *LM = (c_t<T> *)hier_lds + 2 * HP * HP, *pcol = LM + 2 * HierLds<T>::R0 * HierLds<T>::R0 + 64 * leaf;
  const c_t<T> mc = minus_c<T>(d, k);
  for (int t = threadIdx.x; t < 2 * HP; t += 512) gt[t] = t >= 63 && t - 63 <= m ? d.g[t - 63] : 0.0;
  lds_barrier();
  const int cl = 16 * w + li;  // this lane's column of the leaf
  ctile<T> X[4];
  bool bad = false;
  if (mine) {
    const double2 mu = d.mu[k], lam = d.lam[k];
    const bool incol = p * HP + cl < m;
#pragma unroll
    for (int I = 0; I < 4; ++I)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int i = 16 * I + mfma_row<T>(lk, v), row = p * HP + i, dd = i - cl;
        const bool in = row < m;
        const double dp = gld(d.dp + (in ? row : 0)), dm = gld(d.dm + (in ? row : 0));
        const double Jv = d.scale * fma(dp, gt[dd + 64], dm * gt[64 - dd]), J = in && incol ? Jv : 0.0;
        double re = -d.tau * mu.x * J, im = -d.tau * mu.y * J;
        if (dd == 0) {
          re = in ? re + lam.x : 1.0;
          im = in ? im + lam.y : 0.0;
        }
        X[I].re[v] = (T)re;
        X[I].im[v] = (T)im;
      }
  }
  double dpr[4], dmr[4];  // FP64: d+- at rows 16 mt + li, for the Newton step
  if constexpr (sizeof(T) == 8) {
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
      const int row = p * HP + 16 * mt + li;
      dpr[mt] = row < m ? gld(d.dp + (row < m ? row : 0)) : 0.0;
      dmr[mt] = row < m ? gld(d.dm + (row < m ? row : 0)) : 0.0;
    }
  }
#pragma unroll 1
  for (int J = 0; J < 4; ++J) {  // X[i] is row tile (J + i) % 4
    c_t<T> *buf = LX + (J & 1) * 16 * HP;  // the pivot block, two of them in turn
    if (mine && w == J) {
#pragma unroll
      for (int I = 0; I < 4; ++I)
#pragma unroll
        for (int v = 0; v < 4; ++v) buf[lx(li, 16 * ((J + I) & 3) + mfma_row<T>(lk, v))] = mk<T>(X[I].re[v], X[I].im[v]);
    }
    lds_barrier();
    if (mine) {
      const bool own = w == J;
      c_t<T> P[4];
#pragma unroll
      for (int s = 0; s < 4; ++s) P[s] = buf[lx(mfma_row<T>(lk, s), 16 * J + li)];
      gj16<T>(P, lane);
      // P times this wavefront's block row; the pivot block itself becomes P, the rest of its column -A P
      ctile<T> B;
      B.zero();
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const T one = mfma_row<T>(lk, s) == li ? (T)1 : (T)0;
        tile_fma<T>(B, P[s], own ? one : X[0].re[s], own ? (T)0 : X[0].im[s]);
      }
#pragma unroll
      for (int I = 1; I < 4; ++I) {
        if (own) X[I].zero();
#pragma unroll
        for (int s = 0; s < 4; ++s)
          tile_fms<T>(X[I], buf[lx(mfma_row<T>(lk, s), 16 * ((J + I) & 3) + li)], B.re[s], B.im[s]);
        X[I - 1] = X[I];
      }
      X[3] = B;
    }
  }
  lds_barrier();
  ctile<T> E[4];
  if (mine) {  // E = I - K X; X into LDS
    T chk = (T)0;
#pragma unroll
    for (int mt = 0; mt < 4; ++mt)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        LX[lx(cl, 16 * mt + mfma_row<T>(lk, v))] = mk<T>(X[mt].re[v], X[mt].im[v]);
        chk += X[mt].re[v] + X[mt].im[v];
      }
    bad = !isfinite(chk);
    // This lane's row of tile mt as a left operand: 16 mt + ri, so that a result's rows are X's.  gp and gm:
    // g_{i-j+1} and g_{j-i+1} for that row i and column j = 16 t + mfma_row(lk, s).  Rows j of X from m on
    // are zero in the columns before m, and E is only taken there.
    const int ri = rowstr<T>(li);
    const double *gp = gt + 64 + ri - mfma_row<T>(lk, 0), *gm = gt + 64 - ri + mfma_row<T>(lk, 0);
    if constexpr (sizeof(T) == 8) {
      const double2 lam = d.lam[k];
#pragma unroll
      for (int mt = 0; mt < 4; ++mt) E[mt].zero();
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int t = e >> 2, s = e & 3;
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) {
          const double J = d.scale * fma(dpr[mt], gp[16 * (mt - t) - mfma_row<T>(0, s)],
                                         dmr[mt] * gm[16 * (t - mt) + mfma_row<T>(0, s)]);
          const bool dg = mt == t && li == mfma_row<T>(lk, s);
          tile_fma<T>(E[mt], mk<T>(mc.x * J + (dg ? lam.x : 0.0), mc.y * J + (dg ? lam.y : 0.0)), X[t].re[s], X[t].im[s]);
        }
      }
    }
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
      v4d jr = {0, 0, 0, 0}, ji = {0, 0, 0, 0};  // FP32: rows of J X
      if constexpr (sizeof(T) == 4) {
        const int row = p * HP + 16 * mt + ri;
        const double sc = row < m ? d.scale : 0.0;
        const double dp = sc * gld(d.dp + (row < m ? row : 0)), dm = sc * gld(d.dm + (row < m ? row : 0));
        asm volatile("" ::: "memory");  // the weights are read again for each mt, not held
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int t = e >> 2, s = e & 3;
          const double J = fma(dp, gp[16 * (mt - t) - mfma_row<T>(0, s)], dm * gm[16 * (t - mt) + mfma_row<T>(0, s)]);
          jr = mfma16(J, (double)X[t].re[s], jr);
          ji = mfma16(J, (double)X[t].im[s], ji);
        }
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int r = 16 * mt + mfma_row<T>(lk, v);
        double2 t = make_double2(r == cl ? 1.0 : 0.0, 0.0);
        if constexpr (sizeof(T) == 8) {
          t = make_double2(t.x - E[mt].re[v], -E[mt].im[v]);
        } else {
          const double2 lam = d.lam[k], mu = d.mu[k];
          t = hfms<double>(lam, make_double2(X[mt].re[v], X[mt].im[v]), t);
          t = hfma<double>(make_double2(d.tau * mu.x, d.tau * mu.y), make_double2(jr[v], ji[v]), t);
        }
        const bool in = p * HP + r < m && p * HP + cl < m;
        E[mt].re[v] = in ? (T)t.x : (T)0;
        E[mt].im[v] = in ? (T)t.y : (T)0;
      }
    }
  }
  lds_barrier();
  if (mine) {
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
      ctile<T> c;
      c.zero();
#pragma unroll
      for (int e = 0; e < 16; ++e)
        tile_fma<T>(c, LX[lx(16 * (e >> 2) + mfma_row<T>(lk, e & 3), 16 * mt + li)], E[e >> 2].re[e & 3],
                    E[e >> 2].im[e & 3]);
      X[mt].re += c.re;
      X[mt].im += c.im;
    }
  }
  lds_barrier();
  if (mine) {
#pragma unroll
    for (int mt = 0; mt < 4; ++mt)
#pragma unroll
      for (int v = 0; v < 4; ++v) LX[lx(cl, 16 * mt + mfma_row<T>(lk, v))] = mk<T>(X[mt].re[v], X[mt].im[v]);
  }
  lds_barrier();
  if (mine) {
    c_t<T> *D = (c_t<T> *)d.hD + ((size_t)k * npan + p) * HP * HP;
#pragma unroll
    for (int i = 0; i < 16; ++i) D[(16 * w + i) * HP + lane] = LX[lx(16 * w + i, lane)];
  }
  if (d.nlev == 0) {
    if (bad) *flag = 1;
    return;
  }
  constexpr int NE = HierLds<T>::R0 / 4, NT = (NE + 3) / 4;
  const int R = d.hR[0];
  c_t<T> *W0 = hier_w<T>(d, 0, k), *G = hier_g<T>(d, 0, k, pair);
  if (live) {
    const int ct = w ^ (2 * leaf), col = 16 * ct + li;  // the two leaves' tiles on different SIMDs
    const bool tile = 16 * ct < R;
    c_t<T> *Ml = LM + leaf * R * R;
    ctile<T> g[NT], c[NT];
    if (tile) {
      ctile<T> W[4];
      leaf_tile<T>(d, LX, lane, p, 0, col < R ? col : 0, col < R, W);
      if (col < R) panel_store<T>(W0 + ((size_t)p * R + col) * HP + mfma_row<T>(lk, 0), W);
      zero_tiles<T, NT>(g);
      panel_gram<T, NE>(hier_x(d, 0), lane, leaf ? 0 : HP - 1, leaf ? 1 : -1, R, W, g);
#pragma unroll
      for (int e = 0; e < NE; ++e) {
        const int r = 4 * e + lk;
        const c_t<T> t = hmul<T>(mc, mk<T>(g[e >> 2].re[e & 3], g[e >> 2].im[e & 3]));
        g[e >> 2].re[e & 3] = t.x;
        g[e >> 2].im[e & 3] = t.y;
        if (r < R && col < R) {
          G[((size_t)leaf * R + col) * R + r] = t;
          Ml[col * R + r] = t;
        }
      }
    }
    __syncthreads();  // W_0 and G as well
    if (tile) {  // I - G_other G_own
#pragma unroll
      for (int rt = 0; rt < NT; ++rt)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          c[rt].re[v] = 16 * rt + 4 * v + lk == col ? (T)1 : (T)0;
          c[rt].im[v] = (T)0;
        }
#pragma unroll
      for (int rt = 0; rt < NT; ++rt) small_fms<T, NE, true>(LM + (1 - leaf) * R * R, lane, R, rt, g, c[rt]);
    }
    lds_barrier();
    if (tile && col < R) {
#pragma unroll
      for (int e = 0; e < NE; ++e)
        if (4 * e + lk < R) Ml[col * R + 4 * e + lk] = mk<T>(c[e >> 2].re[e & 3], c[e >> 2].im[e & 3]);
    }
    lds_barrier();
    group_invert<T>(Ml, R, w, pcol, piv[leaf], bad);
    lds_barrier();
    scale_rows<T, NE>(W0 + (size_t)p * R * HP + 16 * w, 1, R, Ml, mc, lane);
    __syncthreads();
  }
  if (bad) *flag = 1;
  int ncol = 0;
  for (int l = 1; l < d.nlev; ++l) ncol += d.hR[l];
  const int slot = w ^ (2 * leaf);  // the two wavefronts of a tile sit on different SIMDs
  T *xb = (T *)LM + (wv * NE) * 64, *xo = (T *)LM + ((wv ^ 6) * NE) * 64;  // own and partner's A
#pragma unroll 1
  for (int t0 = 0; 16 * t0 < ncol; t0 += 4) {
    int ln = lane;  // opaque, so that the operands' addresses are not held across iterations
    asm volatile("" : "+v"(ln)::"memory");
    int col = 16 * (t0 + slot) + (ln & 15), lev = 1;
    const bool act = mine && 16 * (t0 + slot) < ncol, ok = col < ncol;
    if (!ok) col = 0;
    while (col >= d.hR[lev]) col -= d.hR[lev++];
    ctile<T> B[4], a[NT], z[NT];
    if (act) leaf_tile<T>(d, LX, ln, p, lev, col, ok, B);
    if (live) {
      if (act) {
        zero_tiles<T, NT>(a);
        panel_gram<T, NE>(hier_x(d, 0), ln, leaf ? 0 : HP - 1, leaf ? 1 : -1, R, B, a);
#pragma unroll
        for (int e = 0; e < NE; ++e) xb[64 * e + ln] = a[e >> 2].re[e & 3];
      }
      lds_barrier();
      if (act) {
#pragma unroll
        for (int rt = 0; rt < NT; ++rt) z[rt].zero();
#pragma unroll
        for (int e = 0; e < NE; ++e) z[e >> 2].re[e & 3] = xo[64 * e + ln];
      }
      lds_barrier();
      if (act) {
#pragma unroll
        for (int e = 0; e < NE; ++e) xb[64 * e + ln] = a[e >> 2].im[e & 3];
      }
      lds_barrier();
      if (act) {
#pragma unroll
        for (int e = 0; e < NE; ++e) z[e >> 2].im[e & 3] = xo[64 * e + ln];
#pragma unroll
        for (int rt = 0; rt < NT; ++rt) small_fms<T, NE, false>(G + (size_t)(1 - leaf) * R * R, ln, R, rt, a, z[rt]);
        panel_update<T, NE>(W0 + (size_t)p * R * HP, ln, R, z, B);
      }
      lds_barrier();
    }
    if (act && ok) panel_store<T>(hier_w<T>(d, lev, k) + ((size_t)p * d.hR[lev] + col) * HP + mfma_row<T>(ln >> 4, 0), B);
  }
}

// ------------------------------------------------------------------------------------
// One node of a level from 1 on: G_1, G_2, the two R x R inverses, and W -> W' over the node's rows.
// Item = (instance, block, node); four wavefronts per half.  For G a wavefront takes a 16-column tile
// and every other panel, for W' 16 rows of every panel.  The columns are read twice and written once
// (115 to 150 us a level at 4095 x 256); an inverse's R steps and, at the upper levels, too few nodes to
// fill the chip make it 245 to 330 us FP64, 1.36 ms for five levels (mixed 0.68), from 1.77 (0.86)
// with half the wavefronts and a barrier-and-LDS inverse.
template <typename T, int NE>
__global__ __launch_bounds__(512) void k_hier_node(const InstDesc *__restrict__ Dd, ItemMap map, int lev, int *flag) {
  extern __shared__ double hier_lds[];
  __shared__ int piv[2][32];
  constexpr int NT = (NE + 3) / 4;
  const int q = item_slot(map, blockIdx.x);
  const InstDesc &d = Dd[map.ids[q]];
  const int local = blockIdx.x - map.pre[q];
  const int nodes = hier_nodes(d.mp, lev), k = local / nodes, node = local % nodes;
  const int R = d.hR[lev], hp = 1 << lev;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  const int side = wv >> 2, w = wv & 3, ct = w & 1, part = w >> 1, col = 16 * ct + li;
  const int p0 = (2 * node + side) * hp, np = min(hp, d.npan - p0);
  // [side][part][column][row] partial sums; G and then I - G G take a side's first one
  c_t<T> *S = (c_t<T> *)hier_lds, *M = S + side * 2 * R * R, *own = M + part * R * R, *Mo = S + (1 - side) * 2 * R * R;
  c_t<T> *pcol = S + 4 * R * R + 64 * side;
  c_t<T> *W = hier_w<T>(d, lev, k) + (size_t)p0 * R * HP;
  const c_t<T> mc = minus_c<T>(d, k);
  const double *tab = hier_x(d, lev);
  bool bad = false;
  ctile<T> g[NT], c;
  zero_tiles<T, NT>(g);
#pragma unroll 1
  for (int pp = part; pp < np; pp += 2) {
    ctile<T> B[4];
    panel_load<T>(W + ((size_t)pp * R + (col < R ? col : 0)) * HP + mfma_row<T>(lk, 0), B);
    panel_gram<T, NE>(tab, lane, side ? pp * HP : (hp - pp) * HP - 1, side ? 1 : -1, R, B, g);
  }
#pragma unroll
  for (int e = 0; e < NE; ++e)
    if (col < R && 4 * e + lk < R) own[col * R + 4 * e + lk] = mk<T>(g[e >> 2].re[e & 3], g[e >> 2].im[e & 3]);
  lds_barrier();
#pragma unroll
  for (int e = 0; e < NE; ++e) {
    const bool in = col < R && 4 * e + lk < R;
    const int at = in ? col * R + 4 * e + lk : 0;
    const c_t<T> a = M[at], b = M[R * R + at];
    const c_t<T> t = hmul<T>(mc, mk<T>(a.x + b.x, a.y + b.y));
    g[e >> 2].re[e & 3] = in ? t.x : (T)0;
    g[e >> 2].im[e & 3] = in ? t.y : (T)0;
  }
  lds_barrier();
  if (part == 0) {
    c_t<T> *G = hier_g<T>(d, lev, k, node) + (size_t)side * R * R;
#pragma unroll
    for (int e = 0; e < NE; ++e)
      if (col < R && 4 * e + lk < R)
        G[col * R + 4 * e + lk] = M[col * R + 4 * e + lk] = mk<T>(g[e >> 2].re[e & 3], g[e >> 2].im[e & 3]);
  }
  lds_barrier();
  // I - G_other G_own, row tile `part`
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    c.re[v] = 16 * part + 4 * v + lk == col ? (T)1 : (T)0;
    c.im[v] = (T)0;
  }
  small_fms<T, NE, true>(Mo, lane, R, part, g, c);
  lds_barrier();
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int r = 16 * part + 4 * v + lk;
    if (col < R && r < R) M[col * R + r] = mk<T>(c.re[v], c.im[v]);
  }
  lds_barrier();
  group_invert<T>(M, R, w, pcol, piv[side], bad);
  if (bad) *flag = 1;
  __syncthreads();
  // W_1' = W_1 (-c (I - G_2 G_1)^{-1}), W_2' = W_2 (-c (I - G_1 G_2)^{-1})
  scale_rows<T, NE>(W + 16 * w, np, R, M, mc, lane);
}

// The columns of the levels above `lev` through that level's elimination,
//   B_1 -= W_1' (A_2 - G_2 A_1),  B_2 -= W_2' (A_1 - G_1 A_2),  A_i = V_i^T B_i.
// Item = (instance, block, node, 16-column tile of those columns); SW wavefronts per half, a panel's
// 64 x 16 tile at a time.  Up to PP panels of a wavefront stay in its registers between the two
// products, so a column is read once and written once (PP = 0, the levels of more than 16 panels a
// node, reads it twice).  The tiles of a node follow each other eight items apart, on one XCD: its W'
// and G come from that L2 after the first.  The products and the passes over the columns take about as
// long as each other (317 us and 370 us at level 1 of 4095 x 256 FP64, of 658); all levels from 1 on
// 1.99 ms (mixed 0.69), from 2.50 (0.96) with 32 columns a workgroup read twice.
template <typename T, int NE, int SW, int PP>
__global__ __launch_bounds__(SW * 128) void k_hier_cols(const InstDesc *__restrict__ Dd, ItemMap map, int lev) {
  extern __shared__ double hier_lds[];
  constexpr int NT = (NE + 3) / 4;
  const int q = item_slot(map, blockIdx.x);
  const InstDesc &d = Dd[map.ids[q]];
  const int local = blockIdx.x - map.pre[q];
  int ncol = 0;
  for (int l = lev + 1; l < d.nlev; ++l) ncol += d.hR[l];
  const int chunks = (ncol + 15) / 16, nodes = hier_nodes(d.mp, lev);
  const int base = local / (8 * chunks) * 8, cnt = min(8, d.nb * nodes - base), rem = local - base * chunks;
  const int kn = base + rem % cnt, ch = rem / cnt, k = kn / nodes, node = kn % nodes;
  const int R = d.hR[lev], hp = 1 << lev;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  const int side = wv / SW, w = wv % SW;
  const int p0 = (2 * node + side) * hp, np = min(hp, d.npan - p0);
  int col = 16 * ch + li, l = lev + 1;
  const bool ok = col < ncol;
  if (!ok) col = 0;
  while (col >= d.hR[l]) col -= d.hR[l++];
  const size_t pst = (size_t)d.hR[l] * HP;
  c_t<T> *Bc = hier_w<T>(d, l, k) + (size_t)p0 * pst + col * HP + mfma_row<T>(lk, 0);
  const c_t<T> *W = hier_w<T>(d, lev, k) + (size_t)p0 * R * HP;
  const double *tab = hier_x(d, lev);
  // partial A [side][w][e][lane], later z [side][e][lane]; A [side][e][lane]
  c_t<T> *S = (c_t<T> *)hier_lds, *A = S + 2 * SW * NE * 64;
  constexpr int HELD = PP > 0 ? PP : 1;
  ctile<T> B[HELD][4], a[NT], z[NT];
  zero_tiles<T, NT>(a);
  auto gram = [&](int pp, const ctile<T> *b) {
    panel_gram<T, NE>(tab, lane, side ? pp * HP : (hp - pp) * HP - 1, side ? 1 : -1, R, b, a);
  };
  if constexpr (PP > 0) {
#pragma unroll
    for (int u = 0; u < PP; ++u)
      if (w + SW * u < np) panel_load<T>(Bc + (w + SW * u) * pst, B[u]);
#pragma unroll
    for (int u = 0; u < PP; ++u)
      if (w + SW * u < np) gram(w + SW * u, B[u]);
  } else {
#pragma unroll 1
    for (int pp = w; pp < np; pp += SW) {
      panel_load<T>(Bc + pp * pst, B[0]);
      gram(pp, B[0]);
    }
  }
#pragma unroll
  for (int e = 0; e < NE; ++e) S[(wv * NE + e) * 64 + lane] = mk<T>(a[e >> 2].re[e & 3], a[e >> 2].im[e & 3]);
  lds_barrier();
#pragma unroll
  for (int e = w; e < NE; e += SW) {
    c_t<T> t = S[(side * SW * NE + e) * 64 + lane];
#pragma unroll
    for (int i = 1; i < SW; ++i) {
      const c_t<T> v = S[((side * SW + i) * NE + e) * 64 + lane];
      t.x += v.x;
      t.y += v.y;
    }
    A[(side * NE + e) * 64 + lane] = t;
  }
  lds_barrier();
  if (w < NT) {  // row tile w of A_other - G_other A_own
    ctile<T> o[NT];
    zero_tiles<T, NT>(a);
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      const c_t<T> t = A[(side * NE + e) * 64 + lane];
      a[e >> 2].re[e & 3] = t.x;
      a[e >> 2].im[e & 3] = t.y;
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int e = min(4 * w + v, NE - 1);
      const c_t<T> t = A[((1 - side) * NE + e) * 64 + lane];
      o[0].re[v] = t.x;
      o[0].im[v] = t.y;
    }
    small_fms<T, NE, false>(hier_g<T>(d, lev, k, node) + (size_t)(1 - side) * R * R, lane, R, w, a, o[0]);
#pragma unroll
    for (int v = 0; v < 4; ++v)
      if (4 * w + v < NE) S[(side * NE + 4 * w + v) * 64 + lane] = mk<T>(o[0].re[v], o[0].im[v]);
  }
  lds_barrier();
  zero_tiles<T, NT>(z);
#pragma unroll
  for (int e = 0; e < NE; ++e) {
    const c_t<T> t = S[(side * NE + e) * 64 + lane];
    z[e >> 2].re[e & 3] = t.x;
    z[e >> 2].im[e & 3] = t.y;
  }
  if constexpr (PP > 0) {
#pragma unroll
    for (int u = 0; u < PP; ++u)
      if (w + SW * u < np) {
        panel_update<T, NE>(W + (size_t)(w + SW * u) * R * HP, lane, R, z, B[u]);
        if (ok) panel_store<T>(Bc + (w + SW * u) * pst, B[u]);
      }
  } else {
#pragma unroll 1
    for (int pp = w; pp < np; pp += SW) {
      panel_load<T>(Bc + pp * pst, B[0]);
      panel_update<T, NE>(W + (size_t)pp * R * HP, lane, R, z, B[0]);
      if (ok) panel_store<T>(Bc + pp * pst, B[0]);
    }
  }
}

// ------------------------------------------------------------------------------------
// Apply.  A wavefront owns a panel, a lane a row; every sum has an order fixed by the level alone.
template <typename T>
__device__ __forceinline__ c_t<T> to_t(double2 v) { return mk<T>((T)v.x, (T)v.y); }

// A wavefront's operands, loaded ahead of the barriers they have to wait behind: up to 32 columns
// of a 64-row panel of W' (lane = row), and its 64 rows of V (lane (r, half): column r, 32 rows).
template <typename T>
__device__ __forceinline__ void load_w(const c_t<T> *W, int R, c_t<T> *w) {
#pragma unroll
  for (int g = 0; g < 8; ++g)
    if (4 * g < R) {
#pragma unroll
      for (int c = 4 * g; c < 4 * g + 4; ++c) w[c] = cload_once<T>(W + c * HP);
    }
}
// y_row - sum_c W'[c][row] z[c], in column order
template <typename T>
__device__ __forceinline__ c_t<T> row_update(const c_t<T> *w, int R, const c_t<T> *z, c_t<T> y) {
#pragma unroll
  for (int g = 0; g < 8; ++g)
    if (4 * g < R) {
#pragma unroll
      for (int c = 4 * g; c < 4 * g + 4; ++c) y = hfms<T>(w[c], z[c], y);
    }
  return y;
}
template <typename T>
__device__ __forceinline__ void load_v(const InstDesc &d, int lev, int p, T *x) {
  const int lane = threadIdx.x & 63, r = lane & 31, hf = lane >> 5;
  const int c = (2 * (p >> (lev + 1)) + 1) << lev, side = (p >> lev) & 1;
  const double *X = hier_x(d, lev) + (size_t)(side ? (p - c) * HP + 32 * hf : (c - p) * HP - 1 - 32 * hf) * 32 + r;
  const int step = side ? 32 : -32;
#pragma unroll
  for (int i = 0; i < 32; ++i) x[i] = (T)gld(X + i * step);
}
// a of one panel: the sum over its rows of V y (y: the panel's 64 values in LDS); the two halves
// are added.  Result for column r in lanes r and r + 32.
template <typename T>
__device__ __forceinline__ c_t<T> panel_vty(const T *x, const c_t<T> *y) {
  c_t<T> acc = mk<T>((T)0, (T)0);
  y += 32 * ((threadIdx.x & 63) >> 5);
#pragma unroll
  for (int i = 0; i < 32; ++i) {
    acc.x = fma(x[i], y[i].x, acc.x);
    acc.y = fma(x[i], y[i].y, acc.y);
  }
  acc.x += __shfl_xor(acc.x, 32, 64);
  acc.y += __shfl_xor(acc.y, 32, 64);
  return acc;
}

// The same sums with the operands loaded where they are used, as one batch each: the number of
// dependent memory round trips, not their bytes, is what a workgroup of the chunk kernel spends
// its time on.
template <typename T>
__device__ __forceinline__ c_t<T> stream_update(const c_t<T> *W, int R, const c_t<T> *z, c_t<T> y) {
  c_t<T> w[32];
  load_w<T>(W, R, w);
  return row_update<T>(w, R, z, y);
}
// z of one half of a node, z = a_other - G_other a_own.  G's columns form eight groups (column mod 8),
// each summed in order, the groups by pairs; lanes r and r + 32 take four groups each.
template <typename T>
__device__ __forceinline__ c_t<T> stream_z(const c_t<T> *G, int R, const c_t<T> *own, const c_t<T> *other) {
  const int lane = threadIdx.x & 63, r = lane & 31, hf = lane >> 5;
  const c_t<T> *g = G + (r < R ? r : 0);
  c_t<T> s[4], a[16];
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int c = 8 * j + 4 * hf + i;
      a[4 * j + i] = cload<T>(g + (size_t)(c < R ? c : 0) * R);
    }
#pragma unroll
  for (int i = 0; i < 4; ++i) s[i] = mk<T>((T)0, (T)0);
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int c = 8 * j + 4 * hf + i;
      const c_t<T> o = own[c];
      s[i] = hfma<T>(a[4 * j + i], mk<T>(c < R ? o.x : (T)0, c < R ? o.y : (T)0), s[i]);
    }
  c_t<T> t = mk<T>((s[0].x + s[1].x) + (s[2].x + s[3].x), (s[0].y + s[1].y) + (s[2].y + s[3].y));
  t.x += __shfl_xor(t.x, 32, 64);
  t.y += __shfl_xor(t.y, 32, 64);
  const c_t<T> o = other[r];
  return mk<T>(o.x - t.x, o.y - t.y);
}
template <typename T>
__device__ __forceinline__ c_t<T> stream_vty(const InstDesc &d, int lev, int p, const c_t<T> *y) {
  T x[32];
  load_v<T>(d, lev, p, x);
  return panel_vty<T>(x, y);
}

// Sum of the panel partials of one half (n panels from `part`, stride 32 per panel, `avail` of them
// present): up to four runs of consecutive panels, added in order.
template <typename T>
__device__ __forceinline__ c_t<T> sum_run(const c_t<T> *part, int from, int to, int avail) {
  c_t<T> a = mk<T>((T)0, (T)0);
  to = min(to, avail);
#pragma unroll 4
  for (int i = from; i < to; ++i) {
    const c_t<T> v = part[(size_t)i * 32];
    a.x += v.x;
    a.y += v.y;
  }
  return a;
}

// The leaf solves and the levels inside a chunk of four panels.  Item = (instance, block, chunk); a
// wavefront per panel.  HBM bound: 64 + R_0 + R_1 complex numbers per row, read once in whole lines.
// Each wavefront forms the z of its own half itself, so a level costs one barrier, and its loads are
// issued in batches of 32 or 64 per lane at two wavefronts per SIMD: 4095 x 256 FP64 (0.93 GB) 172 us,
// 5.4 TB/s; batches of 8 or 16 at up to eight wavefronts per SIMD take 205 to 262 us (3.5 to 4.5
// TB/s), chunks of 8 panels 252 us and 23 us less in the levels above.
template <typename T>
__global__ __launch_bounds__(256, 2) void k_hier_sub(const InstDesc *__restrict__ Dd, ItemMap map) {
  __shared__ c_t<T> y[HCH * HP], part[2][HCH * 32], as[HCH][64], zz[HCH][32];
  const int q = item_slot(map, blockIdx.x);
  if (item_gated(map, q)) return;
  const InstDesc &d = Dd[map.ids[q]];
  const int local = blockIdx.x - map.pre[q];
  const int npan = d.npan, mp = d.mp, nlev = d.nlev, nch = (npan + HCH - 1) / HCH;
  const int k = local / nch, p0 = (local % nch) * HCH, np = min(HCH, npan - p0);
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, p = p0 + w;
  const bool mine = w < np;
  double2 *Vh = d.Vh + (size_t)k * mp + (size_t)p * HP + lane;
  c_t<T> *yp = y + w * HP;
  c_t<T> v = mk<T>((T)0, (T)0);
  if (mine) {
    yp[lane] = to_t<T>(*Vh);
    const c_t<T> *D = (const c_t<T> *)d.hD + ((size_t)k * npan + p) * HP * HP + lane;
    wave_fence();
#pragma unroll
    for (int c = 0; c < HP; ++c) v = hfma<T>(cload_once<T>(D + c * HP), yp[c], v);
    wave_fence();
    yp[lane] = v;
    wave_fence();
    if (nlev > 0) {
      const c_t<T> a = stream_vty<T>(d, 0, p, yp);
      if (lane < 32) part[0][w * 32 + lane] = a;
    }
  }
  int lev = 0;
  for (; lev < nlev && (2 << lev) <= HCH; ++lev) {
    const int R = d.hR[lev], hp = 1 << lev, node = w >> (lev + 1), side = (w >> lev) & 1;
    const bool live = mine && node < hier_nodes_p(np, lev), more = mine && lev + 1 < nlev;
    __syncthreads();
    if (live) {
      const int b0 = node << (lev + 1), r = lane & 31, hf = lane >> 5, run = hp >= 4 ? hp >> 2 : 1;
      const c_t<T> *pt = part[lev & 1] + (b0 + hf * hp) * 32 + r;
      const int avail = min(hp, np - b0 - hf * hp);
      c_t<T> a = sum_run<T>(pt, 0, run, avail);
      for (int f = run; f < hp; f += run) {
        const c_t<T> b = sum_run<T>(pt, f, f + run, avail);
        a.x += b.x;
        a.y += b.y;
      }
      as[w][lane] = a;
      wave_fence();
      const c_t<T> z = stream_z<T>(hier_g<T>(d, lev, k, p >> (lev + 1)) + (size_t)(1 - side) * R * R, R,
                                   as[w] + 32 * side, as[w] + 32 * (1 - side));
      if (lane < 32) zz[w][lane] = z;
      wave_fence();
      v = stream_update<T>(hier_w<T>(d, lev, k) + (size_t)p * R * HP + lane, R, zz[w], v);
    }
    if (more) {
      yp[lane] = v;
      wave_fence();
      const c_t<T> a = stream_vty<T>(d, lev + 1, p, yp);
      if (lane < 32) part[(lev + 1) & 1][w * 32 + lane] = a;
    }
  }
  if (mine) {
    *Vh = make_double2((double)v.x, (double)v.y);
    if (lev < nlev) {  // partial sums for the first level above the chunks
      c_t<T> *A = (c_t<T> *)d.ha + ((size_t)(lev & 1) * d.nb * npan + (size_t)k * npan + p) * 32;
      wave_fence();
      if (lane < 32) A[lane] = part[lev & 1][w * 32 + lane];
    }
  }
}

// One level above the chunks.  Item = (instance, block, group of 4 panels of one half of a node), a
// wavefront per panel.  W', G and the panel partials are loaded before the first barrier; V comes from
// L2 where it is used, because with it in registers too a launch of 129 x 16 workgroups (4095 x 256) is
// a few more than two (FP32: 126 registers) or four (FP64: 240) full loads of the chip and its last
// round is nearly empty.  With 96 and 168 registers 27.8 and 57.7 us, before 36.8 and 58.6; 80 and 128
// registers spill (43 and 105 us).
template <typename T>
__global__ __launch_bounds__(256, sizeof(T) == 8 ? 3 : 5) void k_hier_up(const InstDesc *__restrict__ Dd, ItemMap map, int lev) {
  __shared__ c_t<T> ps[8][32], sg[8][32], as[64], z[32], y[4][HP];
  const int q = item_slot(map, blockIdx.x);
  if (item_gated(map, q)) return;
  const InstDesc &d = Dd[map.ids[q]];
  const int local = blockIdx.x - map.pre[q];
  const int npan = d.npan, mp = d.mp, nch = (npan + 3) / 4;
  const int k = local / nch, p0 = (local % nch) * 4;
  const int hp = 1 << lev, R = d.hR[lev], node = p0 >> (lev + 1), side = (p0 >> lev) & 1;
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, p = p0 + w, r = threadIdx.x & 31, gr = threadIdx.x >> 5;
  const int b0 = 2 * node * hp;
  const bool mine = p < npan, live = b0 + hp < npan, more = mine && lev + 1 < d.nlev;
  const size_t plane = (size_t)d.nb * npan * 32;
  c_t<T> *A = (c_t<T> *)d.ha + (size_t)k * npan * 32;
  double2 *Vh = d.Vh + (size_t)k * mp + (size_t)p * HP + lane;
  c_t<T> wr[32], g[4], v = mk<T>((T)0, (T)0);
  if (live) {
    const int hf = gr >> 2, run = hp >> 2, f = (gr & 3) * run;
    ps[gr][r] = sum_run<T>(A + (size_t)(lev & 1) * plane + (size_t)(b0 + hf * hp) * 32 + r, f, f + run,
                           min(hp, npan - b0 - hf * hp));
    const c_t<T> *G = hier_g<T>(d, lev, k, node) + (size_t)(1 - side) * R * R;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      g[j] = mk<T>((T)0, (T)0);
      if (8 * j + gr < R && r < R) g[j] = cload<T>(G + (size_t)(8 * j + gr) * R + r);
    }
  }
  if (mine) v = to_t<T>(*Vh);
  if (mine && live) load_w<T>(hier_w<T>(d, lev, k) + (size_t)p * R * HP + lane, R, wr);
  if (live) {
    __syncthreads();
    if (threadIdx.x < 64) {
      const int hf = lane >> 5;
      c_t<T> a = ps[4 * hf][r];
#pragma unroll
      for (int i = 1; i < 4; ++i) {
        a.x += ps[4 * hf + i][r].x;
        a.y += ps[4 * hf + i][r].y;
      }
      as[lane] = a;
    }
    __syncthreads();
    {
      c_t<T> s = mk<T>((T)0, (T)0);
#pragma unroll
      for (int j = 0; j < 4; ++j) s = hfma<T>(g[j], as[32 * side + 8 * j + gr], s);
      sg[gr][r] = s;
    }
    __syncthreads();
    if (threadIdx.x < 32) {
      auto pair = [&](int i) { return mk<T>(sg[i][r].x + sg[i + 1][r].x, sg[i][r].y + sg[i + 1][r].y); };
      const c_t<T> a = pair(0), b = pair(2), c = pair(4), e = pair(6), o = as[32 * (1 - side) + r];
      z[r] = mk<T>(o.x - ((a.x + b.x) + (c.x + e.x)), o.y - ((a.y + b.y) + (c.y + e.y)));
    }
    __syncthreads();
    if (mine) {
      v = row_update<T>(wr, R, z, v);
      *Vh = make_double2((double)v.x, (double)v.y);
    }
  }
  if (more) {
    T x[32];
    y[w][lane] = v;
    load_v<T>(d, lev + 1, p, x);
    wave_fence();
    const c_t<T> a = panel_vty<T>(x, y[w]);
    if (lane < 32) A[(size_t)((lev + 1) & 1) * plane + (size_t)p * 32 + lane] = a;
  }
}

// ------------------------------------------------------------------------------------
template <typename T>
hipError_t launch_hier_leaf(const InstDesc *D, const ItemMap &map, int items, int *flag, hipStream_t st) {
  if (items <= 0) return hipSuccess;
  const size_t lds = HierLds<T>::bytes;
  const hipError_t e = hipFuncSetAttribute((const void *)k_hier_leaf<T>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_hier_leaf<T>, dim3(items), dim3(512), lds, st, D, map, flag);
  return hipGetLastError();
}
template <typename T, int NE>
static hipError_t hier_node_ne(const InstDesc *D, const ItemMap &map, int items, int lev, int R, int *flag, hipStream_t st) {
  // the limit is the kernel's for the whole process: always that of the largest rank, so that threads
  // with different ranks do not lower it for each other
  const size_t lds = (4 * R * R + 128) * sizeof(c_t<T>), most = (4 * 16 * NE * NE + 128) * sizeof(c_t<T>);
  const hipError_t e = hipFuncSetAttribute((const void *)k_hier_node<T, NE>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)most);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_hier_node<T, NE>), dim3(items), dim3(512), lds, st, D, map, lev, flag);
  return hipGetLastError();
}
template <typename T, int NE, int SW, int PP>
static hipError_t hier_cols_at(const InstDesc *D, const ItemMap &map, int items, int lev, hipStream_t st) {
  const size_t lds = (2 * SW + 2) * NE * 64 * sizeof(c_t<T>);
  const hipError_t e =
      hipFuncSetAttribute((const void *)k_hier_cols<T, NE, SW, PP>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_hier_cols<T, NE, SW, PP>), dim3(items), dim3(128 * SW), lds, st, D, map, lev);
  return hipGetLastError();
}
// Two wavefronts per half at level 1 (two panels), four above; a wavefront's one or two panels in
// registers up to level 3.
template <typename T, int NE>
static hipError_t hier_cols_ne(const InstDesc *D, const ItemMap &map, int items, int lev, hipStream_t st) {
  if (lev == 1) return hier_cols_at<T, NE, 2, 1>(D, map, items, lev, st);
  if (lev == 2) return hier_cols_at<T, NE, 4, 1>(D, map, items, lev, st);
  if (lev == 3) return hier_cols_at<T, NE, 4, 2>(D, map, items, lev, st);
  return hier_cols_at<T, NE, 4, 0>(D, map, items, lev, st);
}
// R: the level's largest rank in the launch.  Products run over 4 NE rows, so NE follows it in steps of
// 8 rows.
template <typename T>
hipError_t launch_hier_node(const InstDesc *D, const ItemMap &map, int items, int lev, int R, int *flag, hipStream_t st) {
  if (items <= 0) return hipSuccess;
  if (R <= 16) return hier_node_ne<T, 4>(D, map, items, lev, R, flag, st);
  if (R <= 24) return hier_node_ne<T, 6>(D, map, items, lev, R, flag, st);
  return hier_node_ne<T, 8>(D, map, items, lev, R, flag, st);
}
template <typename T>
hipError_t launch_hier_cols(const InstDesc *D, const ItemMap &map, int items, int lev, int R, hipStream_t st) {
  if (items <= 0) return hipSuccess;
  if (R <= 16) return hier_cols_ne<T, 4>(D, map, items, lev, st);
  if (R <= 24) return hier_cols_ne<T, 6>(D, map, items, lev, st);
  return hier_cols_ne<T, 8>(D, map, items, lev, st);
}
template <typename T>
hipError_t launch_hier_sub(const InstDesc *D, const ItemMap &map, int items, hipStream_t st) {
  if (items <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_hier_sub<T>, dim3(items), dim3(256), 0, st, D, map);
  return hipGetLastError();
}
template <typename T>
hipError_t launch_hier_up(const InstDesc *D, const ItemMap &map, int items, int lev, hipStream_t st) {
  if (items <= 0) return hipSuccess;
  hipLaunchKernelGGL((k_hier_up<T>), dim3(items), dim3(256), 0, st, D, map, lev);
  return hipGetLastError();
}

#define HIER_INST(T)                                                                                       \
  template hipError_t launch_hier_leaf<T>(const InstDesc *, const ItemMap &, int, int *, hipStream_t);     \
  template hipError_t launch_hier_node<T>(const InstDesc *, const ItemMap &, int, int, int, int *, hipStream_t); \
  template hipError_t launch_hier_cols<T>(const InstDesc *, const ItemMap &, int, int, int, hipStream_t);  \
  template hipError_t launch_hier_sub<T>(const InstDesc *, const ItemMap &, int, hipStream_t);        \
  template hipError_t launch_hier_up<T>(const InstDesc *, const ItemMap &, int, int, hipStream_t);
HIER_INST(double)
HIER_INST(float)
#undef HIER_INST

}  // namespace fde
