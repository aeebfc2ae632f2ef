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
static constexpr int HS = 33;       // LDS column stride of the small matrices (32 rows and a pad)
static constexpr int HSLOT = 32 * HS;

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

// The row of a 16-row tile that element i of an MFMA operand holds, chosen so that the four
// results of a lane (mfma_row) are four consecutive rows 4 (lane / 16) + v.
template <typename T> __device__ __forceinline__ int rowperm(int i);
template <> __device__ __forceinline__ int rowperm<float>(int i) { return i; }
template <> __device__ __forceinline__ int rowperm<double>(int i) { return 4 * (i & 3) + (i >> 2); }

__device__ __forceinline__ void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// ------------------------------------------------------------------------------------
// Leaf inverses.  Item = (instance, block, panel); one workgroup of 256 forms the 64 x 64
// diagonal block from the weights and inverts it by Gauss-Jordan without pivoting (strict row
// dominance).  Thread t holds row t % 64, columns 16 (t / 64) .. + 15 in registers; a step's pivot
// row and column go through double-buffered LDS vectors, one barrier a step.  Bound by those 64
// dependent steps, so four workgroups share a CU.
template <typename T>
__global__ __launch_bounds__(256) void k_hier_leaf(const InstDesc *__restrict__ Dd, ItemMap map, int *flag) {
  __shared__ c_t<T> colb[2][HP], rowb[2][HP];
  const int q = item_slot(map, blockIdx.x);
  const InstDesc &d = Dd[map.ids[q]];
  const int local = blockIdx.x - map.pre[q];
  const int npan = d.npan, k = local / npan, p = local % npan;
  const int r = threadIdx.x & 63, cq = threadIdx.x >> 6;
  const double2 mu = d.mu[k], lam = d.lam[k];
  const int row = p * HP + r, m = d.m;
  const bool inr = row < m;
  const double dp = inr ? d.scale * d.dp[row] : 0.0, dm = inr ? d.scale * d.dm[row] : 0.0;
  c_t<T> a[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int c = 16 * cq + i, dd = r - c;
    const bool ok = inr && p * HP + c < m;
    const double gp = ok && dd >= -1 ? d.g[dd + 1] : 0.0;
    const double gm = ok && dd <= 1 ? d.g[1 - dd] : 0.0;
    const double J = fma(dp, gp, dm * gm);
    double re = -d.tau * mu.x * J, im = -d.tau * mu.y * J;
    if (dd == 0) {
      re = inr ? re + lam.x : 1.0;
      im = inr ? im + lam.y : 0.0;
    }
    a[i] = mk<T>((T)re, (T)im);
  }
  bool bad = false;
  for (int jo = 0; jo < 4; ++jo) {
#pragma unroll
    for (int ji = 0; ji < 16; ++ji) {
      const int j = 16 * jo + ji, b = ji & 1;
      if (cq == jo) colb[b][r] = a[ji];
      if (r == j) {
#pragma unroll
        for (int i = 0; i < 16; ++i) rowb[b][16 * cq + i] = a[i];
      }
      __syncthreads();
      const c_t<T> pv = rowb[b][j];
      const T m2 = pv.x * pv.x + pv.y * pv.y;
      bad = bad || !(m2 > (T)0) || !isfinite(m2);
      const T iv = (T)1 / m2;
      const c_t<T> inv = mk<T>(pv.x * iv, -pv.y * iv);
      const c_t<T> f = colb[b][r];
      const c_t<T> fi = hmul<T>(f, inv);
      const bool own = r == j;
      const c_t<T> t = mk<T>(own ? -inv.x : fi.x, own ? -inv.y : fi.y);
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const c_t<T> pr = rowb[b][16 * cq + i];
        const c_t<T> base = mk<T>(own ? (T)0 : a[i].x, own ? (T)0 : a[i].y);
        a[i] = hfms<T>(t, pr, base);
      }
      if (cq == jo) a[ji] = mk<T>(-t.x, -t.y);
    }
  }
  if (bad) *flag = 1;
  c_t<T> *D = (c_t<T> *)d.hD + ((size_t)k * npan + p) * HP * HP;
#pragma unroll
  for (int i = 0; i < 16; ++i) D[(16 * cq + i) * HP + r] = a[i];
}

// ------------------------------------------------------------------------------------
// One Newton step on the leaf inverse, then W of every level from it: K_leaf^{-1} U.  Item =
// (instance, block, panel).
//
// X <- X + X (I - K X).  Gauss-Jordan leaves an error of cond(K_leaf) eps in X (the leaf of a
// frequency near zero is close to a singular M-matrix), the largest error of the whole form; the
// step takes it to the size of X's own rounding (forward errors of S^{-1} v 5 to 20 times
// smaller).  K X = lambda X - c (J X) with J real, so it costs one real-by-complex and one complex
// product, on MFMA.
//
// Then wave w owns rows 16 w .. + 15 of the panel, its 16 x 64 slice of the inverse in registers as
// the MFMA operand, and walks the 16-column tiles of all levels; U is formed from X and d on the
// way in.
static constexpr int HLS = HP + 1;  // LDS column stride of a leaf

template <typename T>
__global__ __launch_bounds__(256) void k_hier_init(const InstDesc *__restrict__ Dd, ItemMap map) {
  extern __shared__ double hier_lds[];
  c_t<T> *S = (c_t<T> *)hier_lds;
  __shared__ T gt[2 * HP];  // g_t at index t + 63, zero for t < 0
  const int q = item_slot(map, blockIdx.x);
  const InstDesc &d = Dd[map.ids[q]];
  const int local = blockIdx.x - map.pre[q];
  const int npan = d.npan, k = local / npan, p = local % npan, m = d.m;
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  c_t<T> *D0 = (c_t<T> *)d.hD + ((size_t)k * npan + p) * HP * HP;
  for (int t = threadIdx.x; t < 2 * HP; t += 256) gt[t] = t >= 63 && t - 63 <= m ? (T)d.g[t - 63] : (T)0;
  __syncthreads();
  c_t<T> A[16];
  {  // R = I - K X, columns 16 w .. + 15, into LDS
    const int colg = p * HP + 16 * w + li;
#pragma unroll
    for (int s = 0; s < 16; ++s) A[s] = cload<T>(D0 + (16 * w + li) * HP + 4 * s + lk);
    const c_t<T> mc = minus_c<T>(d, k);
    const c_t<T> lam = mk<T>((T)d.lam[k].x, (T)d.lam[k].y);
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
      const int i = 16 * mt + li, row = p * HP + i;
      const T dp = row < m ? (T)(d.scale * d.dp[row]) : (T)0, dm = row < m ? (T)(d.scale * d.dm[row]) : (T)0;
      acc_t<T> re = {0, 0, 0, 0}, im = {0, 0, 0, 0};
#pragma unroll
      for (int s = 0; s < 16; ++s) {
        const int kc = 4 * s + lk;
        T J = fma(dp, gt[i - kc + 64], dm * gt[kc - i + 64]);
        if (p * HP + kc >= m) J = (T)0;
        re = mfma16(J, A[s].x, re);
        im = mfma16(J, A[s].y, im);
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int r = 16 * mt + mfma_row<T>(lk, v);
        const c_t<T> x = cload<T>(D0 + (16 * w + li) * HP + r);
        c_t<T> t = mk<T>(r == 16 * w + li ? (T)1 : (T)0, (T)0);
        t = hfms<T>(lam, x, t);
        t = hfms<T>(mc, mk<T>(re[v], im[v]), t);
        if (p * HP + r >= m || colg >= m) t = mk<T>((T)0, (T)0);
        S[(16 * w + li) * HLS + r] = t;
      }
    }
  }
  __syncthreads();
  const int rw = 16 * w + rowperm<T>(li);
#pragma unroll
  for (int s = 0; s < 16; ++s) A[s] = cload<T>(D0 + (4 * s + lk) * HP + rw);
  c_t<T> nx[4][4];
#pragma unroll
  for (int n = 0; n < 4; ++n) {
    acc_t<T> re = {0, 0, 0, 0}, im = {0, 0, 0, 0};
#pragma unroll
    for (int s = 0; s < 16; ++s) {
      const c_t<T> b = S[(16 * n + li) * HLS + 4 * s + lk];
      re = mfma16(A[s].x, b.x, re);
      re = mfma16(-A[s].y, b.y, re);
      im = mfma16(A[s].x, b.y, im);
      im = mfma16(A[s].y, b.x, im);
    }
    c_t<T> *o = D0 + (16 * n + li) * HP + 16 * w + 4 * lk;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const c_t<T> x = cload<T>(o + v);
      nx[n][v] = mk<T>(x.x + re[v], x.y + im[v]);
      o[v] = nx[n][v];
    }
  }
  __syncthreads();  // R is used up: the new inverse takes its place
#pragma unroll
  for (int n = 0; n < 4; ++n)
#pragma unroll
    for (int v = 0; v < 4; ++v) S[(16 * n + li) * HLS + 16 * w + 4 * lk + v] = nx[n][v];
  __syncthreads();
#pragma unroll
  for (int s = 0; s < 16; ++s) A[s] = S[(4 * s + lk) * HLS + rw];
  for (int lev = 0; lev < d.nlev; ++lev) {
    const int R = d.hR[lev], node = p >> (lev + 1), side = (p >> lev) & 1;
    const int c = (2 * node + 1) << lev;  // first panel of the right half
    const bool live = c < npan;
    const double *X = hier_x(d, lev);
    c_t<T> *W = hier_w<T>(d, lev, k);
    for (int n = 0; n < R; n += 16) {
      const int col = n + li;
      const bool ok = live && col < R;
      // the e_0 column carries the other side's coefficient (the g_0 entry next to the diagonal)
      const double *dv = (side == 0) != (col == 0) ? d.dm : d.dp;
      acc_t<T> re = {0, 0, 0, 0}, im = {0, 0, 0, 0};
#pragma unroll
      for (int s = 0; s < 16; ++s) {
        const int i = 4 * s + lk, row = p * HP + i;
        const int pi = side ? (p - c) * HP + i : (c - p) * HP - 1 - i;
        T u = (T)0;
        if (ok && row < m) u = (T)(d.scale * (dv[row] * X[(size_t)pi * 32 + col]));
        re = mfma16(A[s].x, u, re);
        im = mfma16(A[s].y, u, im);
      }
      if (col < R) {
        c_t<T> *o = W + ((size_t)p * R + col) * HP + 16 * w + 4 * lk;
#pragma unroll
        for (int v = 0; v < 4; ++v) o[v] = mk<T>(re[v], im[v]);
      }
    }
  }
}

// ------------------------------------------------------------------------------------
// V^T B over one half of a node for two 16-column tiles: MFMA, the half's 16-row groups divided
// between two waves (part).  Lane (j, kk) takes rows 4 kk .. + 3 of a group of column j, so its four
// loads are consecutive.  Bc: the columns' first panel, pst their panel strides.  The partial products go to an LDS slot ([column][row], stride HS).
template <typename T>
__device__ __forceinline__ void hier_gram(const double *X, int h, int side, int len,
                                          const c_t<T> *const *Bc, const int *pst, const bool *ok, int part, bool two,
                                          c_t<T> *slot) {
  const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  acc_t<T> acc[2][2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) acc[a][b][0] = acc[a][b][1] = acc_t<T>{0, 0, 0, 0};
  for (int g = part; g < (len >> 4); g += 2) {
    const int r0 = 16 * g + 4 * lk;
    c_t<T> b[2][4];
    T x[2][4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int pi = side ? r0 + v : h - 1 - r0 - v;
      x[0][v] = (T)X[(size_t)pi * 32 + li];
      x[1][v] = two ? (T)X[(size_t)pi * 32 + 16 + li] : (T)0;
#pragma unroll
      for (int n = 0; n < 2; ++n) {
        b[n][v] = mk<T>((T)0, (T)0);
        if (ok[n]) b[n][v] = cload<T>(Bc[n] + (size_t)(g >> 2) * pst[n] + (r0 & 63) + v);
      }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int n = 0; n < 2; ++n) {
        acc[0][n][0] = mfma16(x[0][v], b[n][v].x, acc[0][n][0]);
        acc[0][n][1] = mfma16(x[0][v], b[n][v].y, acc[0][n][1]);
        if (two) {
          acc[1][n][0] = mfma16(x[1][v], b[n][v].x, acc[1][n][0]);
          acc[1][n][1] = mfma16(x[1][v], b[n][v].y, acc[1][n][1]);
        }
      }
  }
#pragma unroll
  for (int n = 0; n < 2; ++n)
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        slot[(16 * n + li) * HS + 16 * mt + mfma_row<T>(lk, v)] = mk<T>(acc[mt][n][0][v], acc[mt][n][1][v]);
}

// In-place inverses of two R x R matrices in LDS ([column][row], stride HS) by Gauss-Jordan with
// partial pivoting: threads 0..127 the first, 128..255 the second.
template <typename T>
__device__ __forceinline__ void hier_invert2(c_t<T> *P1, c_t<T> *P2, int R, int (*piv)[32], bool &bad) {
  const int sel = threadIdx.x >> 7, r = threadIdx.x & 31, cq = (threadIdx.x >> 5) & 3;
  c_t<T> *P = sel ? P2 : P1;
  for (int j = 0; j < R; ++j) {
    if (cq == 0) {  // half a wavefront: the largest entry of column j at or below the diagonal
      const c_t<T> v = P[j * HS + r];
      T best = r >= j && r < R ? v.x * v.x + v.y * v.y : (T)-1;
      int at = r;
#pragma unroll
      for (int o = 16; o > 0; o >>= 1) {
        const T ob = __shfl_xor(best, o, 32);
        const int oa = __shfl_xor(at, o, 32);
        if (ob > best || (ob == best && oa < at)) {
          best = ob;
          at = oa;
        }
      }
      if (r == 0) piv[sel][j] = at;
      bad = bad || !(best > (T)0) || !isfinite(best);
    }
    __syncthreads();
    const int pr = piv[sel][j];
    const int src = r == j ? pr : r == pr ? j : r;
    const c_t<T> pv = P[j * HS + pr];
    const T iv = (T)1 / (pv.x * pv.x + pv.y * pv.y);
    const c_t<T> inv = mk<T>(pv.x * iv, -pv.y * iv);
    const c_t<T> f = P[j * HS + src];
    const c_t<T> fi = hmul<T>(f, inv);
    const bool own = r == j;
    const c_t<T> t = mk<T>(own ? -inv.x : fi.x, own ? -inv.y : fi.y);
    c_t<T> e[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int c = cq + 4 * i;
      const c_t<T> a = P[c * HS + src], b = P[c * HS + pr];
      const c_t<T> base = mk<T>(own ? (T)0 : a.x, own ? (T)0 : a.y);
      e[i] = hfms<T>(t, b, base);
      if (c == j) e[i] = mk<T>(-t.x, -t.y);
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int c = cq + 4 * i;
      if (c < R && r < R) P[c * HS + r] = e[i];
    }
    __syncthreads();
  }
  for (int j = R - 1; j >= 0; --j) {  // undo the row exchanges: exchange columns, last first
    const int pr = piv[sel][j];
    if (pr != j && cq == 0 && r < R) {
      const c_t<T> a = P[j * HS + r];
      P[j * HS + r] = P[pr * HS + r];
      P[pr * HS + r] = a;
    }
  }
  __syncthreads();
}

// One node of a level: G_1, G_2, the two R x R inverses, and W -> W' over the node's rows.
// Item = (instance, block, node).  Waves 0, 1 the left half, 2, 3 the right.
template <typename T>
__global__ __launch_bounds__(256) void k_hier_node(const InstDesc *__restrict__ Dd, ItemMap map, int lev, int *flag) {
  extern __shared__ double hier_lds[];
  c_t<T> *S = (c_t<T> *)hier_lds;  // four slots
  __shared__ int piv[2][32];
  const int q = item_slot(map, blockIdx.x);
  const InstDesc &d = Dd[map.ids[q]];
  const int local = blockIdx.x - map.pre[q];
  const int nodes = hier_nodes(d.mp, lev), k = local / nodes, node = local % nodes;
  const int R = d.hR[lev], mp = d.mp, h = HP << lev;
  const bool two = R > 16;
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  const int side = w >> 1, part = w & 1;
  const int r0 = (2 * node + side) * h, len = min(h, mp - r0);
  c_t<T> *W = hier_w<T>(d, lev, k) + (size_t)r0 * R;
  const c_t<T> *Bc[2] = {W + li * HP, W + (16 + li) * HP};
  const int pst[2] = {R * HP, R * HP};
  const bool ok[2] = {li < R, 16 + li < R};
  hier_gram<T>(hier_x(d, lev), h, side, len, Bc, pst, ok, part, two, S + w * HSLOT);
  __syncthreads();
  // G_i = -c (V_i^T W_i): slots 0 (left) and 2 (right), and to memory
  const c_t<T> mc = minus_c<T>(d, k);
  {
    c_t<T> *G = hier_g<T>(d, lev, k, node);
    const int sel = threadIdx.x >> 7, r = threadIdx.x & 31, cq = (threadIdx.x >> 5) & 3;
    c_t<T> *A = S + 2 * sel * HSLOT, *B = A + HSLOT;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int c = cq + 4 * i;
      const c_t<T> a = A[c * HS + r], b = B[c * HS + r];
      const c_t<T> g = hmul<T>(mc, mk<T>(a.x + b.x, a.y + b.y));
      A[c * HS + r] = g;
      if (c < R && r < R) G[((size_t)sel * R + c) * R + r] = g;
    }
    __syncthreads();
    // slot 1: I - G_1 G_2, slot 3: I - G_2 G_1
    const c_t<T> *Ga = S + 2 * sel * HSLOT, *Gb = S + 2 * (1 - sel) * HSLOT;
    c_t<T> acc[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = mk<T>(cq + 4 * i == r ? (T)1 : (T)0, (T)0);
    for (int t = 0; t < R; ++t) {
      const c_t<T> a = Ga[t * HS + r];
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[i] = hfms<T>(a, Gb[(cq + 4 * i) * HS + t], acc[i]);
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) B[(cq + 4 * i) * HS + r] = acc[i];
    __syncthreads();
  }
  bool bad = false;
  hier_invert2<T>(S + HSLOT, S + 3 * HSLOT, R, piv, bad);
  if (bad) *flag = 1;
  // W_1' = W_1 (-c (I - G_2 G_1)^{-1}), W_2' = W_2 (-c (I - G_1 G_2)^{-1}): in place, 16 rows at a time
  const c_t<T> *Q = S + (side == 0 ? 3 : 1) * HSLOT;
  c_t<T> qb[2][8];
#pragma unroll
  for (int n = 0; n < 2; ++n)
#pragma unroll
    for (int s = 0; s < 8; ++s) qb[n][s] = hmul<T>(mc, Q[(16 * n + li) * HS + 4 * s + lk]);
  for (int g = part; g < (len >> 4); g += 2) {
    c_t<T> a[8];
    auto *Wg = W + (size_t)(g >> 2) * R * HP + 16 * (g & 3);
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      a[s] = mk<T>((T)0, (T)0);
      if (4 * s < R) a[s] = cload<T>(Wg + (4 * s + lk) * HP + rowperm<T>(li));
    }
#pragma unroll
    for (int n = 0; n < 2; ++n) {
      if (n == 1 && !two) break;
      acc_t<T> re = {0, 0, 0, 0}, im = {0, 0, 0, 0};
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        if (4 * s < R) {
          re = mfma16(a[s].x, qb[n][s].x, re);
          re = mfma16(-a[s].y, qb[n][s].y, re);
          im = mfma16(a[s].x, qb[n][s].y, im);
          im = mfma16(a[s].y, qb[n][s].x, im);
        }
      }
      if (16 * n + li < R) {
        c_t<T> *o = Wg + (16 * n + li) * HP + 4 * lk;
#pragma unroll
        for (int v = 0; v < 4; ++v) o[v] = mk<T>(re[v], im[v]);
      }
    }
  }
}

// The columns of the levels above `lev` through that level's elimination: 32 columns B of a node,
//   B_1 -= W_1' (A_2 - G_2 A_1),  B_2 -= W_2' (A_1 - G_1 A_2),  A_i = V_i^T B_i.
// Item = (instance, block, node, 32-column chunk of those levels' columns).
template <typename T>
__global__ __launch_bounds__(256) void k_hier_cols(const InstDesc *__restrict__ Dd, ItemMap map, int lev) {
  extern __shared__ double hier_lds[];
  c_t<T> *S = (c_t<T> *)hier_lds;
  const int q = item_slot(map, blockIdx.x);
  const InstDesc &d = Dd[map.ids[q]];
  const int local = blockIdx.x - map.pre[q];
  int ncol = 0;
  for (int l = lev + 1; l < d.nlev; ++l) ncol += d.hR[l];
  const int chunks = (ncol + 31) / 32, nodes = hier_nodes(d.mp, lev);
  const int ch = local % chunks, kn = local / chunks, k = kn / nodes, node = kn % nodes;
  const int R = d.hR[lev], mp = d.mp, h = HP << lev;
  const bool two = R > 16;
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  const int side = w >> 1, part = w & 1;
  const int r0 = (2 * node + side) * h, len = min(h, mp - r0);
  c_t<T> *Bc[2];
  int pst[2];
  bool ok[2];
#pragma unroll
  for (int n = 0; n < 2; ++n) {
    int col = 32 * ch + 16 * n + li, l = lev + 1;
    ok[n] = col < ncol;
    if (!ok[n]) col = 0;
    while (col >= d.hR[l]) col -= d.hR[l++];
    pst[n] = d.hR[l] * HP;
    Bc[n] = hier_w<T>(d, l, k) + (size_t)(r0 >> 6) * pst[n] + col * HP;
  }
  const c_t<T> *Br[2] = {Bc[0], Bc[1]};
  hier_gram<T>(hier_x(d, lev), h, side, len, Br, pst, ok, part, two, S + w * HSLOT);
  __syncthreads();
  {  // A_1 into slot 0, A_2 into slot 2
    const int sel = threadIdx.x >> 7, r = threadIdx.x & 31, cq = (threadIdx.x >> 5) & 3;
    c_t<T> *A = S + 2 * sel * HSLOT;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int e = (cq + 4 * i) * HS + r;
      const c_t<T> a = A[e], b = A[HSLOT + e];
      A[e] = mk<T>(a.x + b.x, a.y + b.y);
    }
  }
  __syncthreads();
  {  // slot 1: A_2 - G_2 A_1 (waves 0, 1: one column tile each), slot 3: A_1 - G_1 A_2 (waves 2, 3)
    const c_t<T> *G = hier_g<T>(d, lev, k, node) + (size_t)(1 - side) * R * R;
    const c_t<T> *Am = S + 2 * side * HSLOT, *Ao = S + 2 * (1 - side) * HSLOT;
    c_t<T> *To = S + (1 + 2 * side) * HSLOT;
    acc_t<T> acc[2][2];
#pragma unroll
    for (int a = 0; a < 2; ++a) acc[a][0] = acc[a][1] = acc_t<T>{0, 0, 0, 0};
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      if (4 * s < R) {
        const c_t<T> b = Am[(16 * part + li) * HS + 4 * s + lk];
#pragma unroll
        for (int mt = 0; mt < 2; ++mt) {
          c_t<T> a = mk<T>((T)0, (T)0);
          if (16 * mt + li < R) a = cload<T>(G + (size_t)(4 * s + lk) * R + 16 * mt + li);
          acc[mt][0] = mfma16(a.x, b.x, acc[mt][0]);
          acc[mt][0] = mfma16(-a.y, b.y, acc[mt][0]);
          acc[mt][1] = mfma16(a.x, b.y, acc[mt][1]);
          acc[mt][1] = mfma16(a.y, b.x, acc[mt][1]);
        }
      }
    }
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int e = (16 * part + li) * HS + 16 * mt + mfma_row<T>(lk, v);
        const c_t<T> a = Ao[e];
        To[e] = mk<T>(a.x - acc[mt][0][v], a.y - acc[mt][1][v]);
      }
  }
  __syncthreads();
  const c_t<T> *Tm = S + (1 + 2 * side) * HSLOT;
  c_t<T> tb[2][8];
#pragma unroll
  for (int n = 0; n < 2; ++n)
#pragma unroll
    for (int s = 0; s < 8; ++s) tb[n][s] = Tm[(16 * n + li) * HS + 4 * s + lk];
  const c_t<T> *W = hier_w<T>(d, lev, k) + (size_t)r0 * R;
  for (int g = part; g < (len >> 4); g += 2) {
    c_t<T> a[8];
    auto *Wg = W + (size_t)(g >> 2) * R * HP + 16 * (g & 3);
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      a[s] = mk<T>((T)0, (T)0);
      if (4 * s < R) a[s] = cload<T>(Wg + (4 * s + lk) * HP + rowperm<T>(li));
    }
#pragma unroll
    for (int n = 0; n < 2; ++n) {
      c_t<T> o[4];
      c_t<T> *po = Bc[n] + (size_t)(g >> 2) * pst[n] + 16 * (g & 3) + 4 * lk;
      if (ok[n])
#pragma unroll
        for (int v = 0; v < 4; ++v) o[v] = cload<T>(po + v);
      acc_t<T> re = {0, 0, 0, 0}, im = {0, 0, 0, 0};
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        if (4 * s < R) {
          re = mfma16(a[s].x, tb[n][s].x, re);
          re = mfma16(-a[s].y, tb[n][s].y, re);
          im = mfma16(a[s].x, tb[n][s].y, im);
          im = mfma16(a[s].y, tb[n][s].x, im);
        }
      }
      if (ok[n])
#pragma unroll
        for (int v = 0; v < 4; ++v) po[v] = mk<T>(o[v].x - re[v], o[v].y - im[v]);
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
// wavefront per panel; everything but the panel sums is loaded before the first barrier.
template <typename T>
__global__ __launch_bounds__(256, 2) void k_hier_up(const InstDesc *__restrict__ Dd, ItemMap map, int lev) {
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
  T x[32];
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
  if (more) load_v<T>(d, lev + 1, p, x);
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
    y[w][lane] = v;
    wave_fence();
    const c_t<T> a = panel_vty<T>(x, y[w]);
    if (lane < 32) A[(size_t)((lev + 1) & 1) * plane + (size_t)p * 32 + lane] = a;
  }
}

// ------------------------------------------------------------------------------------
template <typename T>
hipError_t launch_hier_leaf(const InstDesc *D, const ItemMap &map, int items, int *flag, hipStream_t st) {
  if (items <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_hier_leaf<T>, dim3(items), dim3(256), 0, st, D, map, flag);
  return hipGetLastError();
}
template <typename T>
hipError_t launch_hier_init(const InstDesc *D, const ItemMap &map, int items, hipStream_t st) {
  if (items <= 0) return hipSuccess;
  const size_t lds = HP * HLS * sizeof(c_t<T>);
  const hipError_t e = hipFuncSetAttribute((const void *)k_hier_init<T>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_hier_init<T>, dim3(items), dim3(256), lds, st, D, map);
  return hipGetLastError();
}
template <typename T>
hipError_t launch_hier_node(const InstDesc *D, const ItemMap &map, int items, int lev, int *flag, hipStream_t st) {
  if (items <= 0) return hipSuccess;
  const size_t lds = 4 * HSLOT * sizeof(c_t<T>);
  const hipError_t e = hipFuncSetAttribute((const void *)k_hier_node<T>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_hier_node<T>, dim3(items), dim3(256), lds, st, D, map, lev, flag);
  return hipGetLastError();
}
template <typename T>
hipError_t launch_hier_cols(const InstDesc *D, const ItemMap &map, int items, int lev, hipStream_t st) {
  if (items <= 0) return hipSuccess;
  const size_t lds = 4 * HSLOT * sizeof(c_t<T>);
  const hipError_t e = hipFuncSetAttribute((const void *)k_hier_cols<T>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_hier_cols<T>, dim3(items), dim3(256), lds, st, D, map, lev);
  return hipGetLastError();
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
  template hipError_t launch_hier_init<T>(const InstDesc *, const ItemMap &, int, hipStream_t);            \
  template hipError_t launch_hier_node<T>(const InstDesc *, const ItemMap &, int, int, int *, hipStream_t); \
  template hipError_t launch_hier_cols<T>(const InstDesc *, const ItemMap &, int, int, hipStream_t);       \
  template hipError_t launch_hier_sub<T>(const InstDesc *, const ItemMap &, int, hipStream_t);        \
  template hipError_t launch_hier_up<T>(const InstDesc *, const ItemMap &, int, int, hipStream_t);
HIER_INST(double)
HIER_INST(float)
#undef HIER_INST

}  // namespace fde
