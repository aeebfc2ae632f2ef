// Space-time kernels of the all-at-once operator (gfx950), batched over instances:
//  * Toeplitz symbol of G_a (eq. (1.5)) by an LDS FFT of its circulant embedding,
//  * the fused product M z = (A (x) I) z - tau (B (x) J) z of eq. (1.10): for every time
//    level the banded BVM rows are combined first, then J is applied once through the
//    FFT (J sum_q b_q z_q = sum_q b_q J z_q because J is time-independent),
//  * the right-hand side of the s-form system,
//  * the real DFT along time that diagonalises s(A), s(B) (Section 3.2), two spatial
//    columns packed per complex FFT.
#include "batch.hpp"
#include "common.hpp"
#include "fft_lds.hpp"
#include "kernels.hpp"

namespace fde {

static constexpr int ST_NT = 256;

// chat_br = FFT_L(c), c real [L]; result left in bit-reversed order.
__global__ __launch_bounds__(ST_NT) void k_symbol(const double *__restrict__ cG,
                                                  double2 *__restrict__ chat_br, int log2L,
                                                  const double2 *__restrict__ twL) {
  extern __shared__ double2 buf[];
  const int L = 1 << log2L;
  for (int i = threadIdx.x; i < L; i += ST_NT) buf[i] = make_double2(cG[i], 0.0);
  __syncthreads();
  fft_dif<ST_NT>(buf, log2L, 1, twL);
  for (int i = threadIdx.x; i < L; i += ST_NT) chat_br[i] = buf[i];
}

// Item = (instance, row n).
// mode 0 (M z):  v = sum_q b[n][q] Z[col_q], u = sum_q a[n][q] Z[col_q]  (col_q = c[n]+q-1 >= 0)
//                W[n] = u - tau J v
// mode 1 (J x):  W[n] = J Z[n]
// mode 2 (S z):  the Strang circulant rows: every row carries the main formula on the
//                wrapped columns (n - nu + q) mod s:  W[n] = u_S - tau J v_S
// mode 3 ((S - M) z): W[n] = (u_S - u) - tau J (v_S - v); nonzero only on the nu + (mu-nu)
//                boundary rows where the circulant and the BVM matrices differ.
// J v = scale/L * (d+ Re + d- Im) of IFFT(chat*V + i conj(chat)*V) = L (G v + i G^T v).
//
// Shape: one butterfly of eight elements per thread, L / 8 threads per row and 8 NT / L rows per
// workgroup, so that in a batch the short rows share the workgroups that the longest one needs.  The
// transforms are fft_lds.hpp's radix-2 stages in the same order (each element sees the same operations
// and the result does not depend on the grouping), arranged for few passes through LDS:
//  * thread t combines elements t + r L / 8, r < 4, which with the zeros of the embedding are its
//    operands of the first three stages, and ends with the same elements of the result;
//  * the last one to three stages forward, the product with the spectrum and the first stages back
//    need only eight neighbours, and are one visit to LDS;
//  * the twiddles of the passes between lie compactly in LDS, and rows are exchanged within 16 by the
//    next four address bits, so that both kinds of access meet every bank once.
// For L = 4096 that is 6 barriers instead of 10.  us per product of m x s, with a pass per stage triple
// and the longest row's LDS for every row / so: 63 x 64 9.0 / 8.3, 701 x 64 16.6 / 11.7, 1023 x 512
// 23.1 / 15.2, 2047 x 64 25.7 / 15.4, 4095 x 256 45.7 / 33.3, eight instances of 64 to 2047 rows
// 88 / 28.  Latency bounds it (one or two workgroups per CU), LDS bandwidth for a third of the time.
__device__ __forceinline__ int fft_sw(int i) { return i ^ ((i >> 4) & 15); }

// three stages with half-spans 4h, 2h, h (forward) on elements j + r h of a group of 8 h; t[k] the
// twiddle e^{-2 pi i k / (8 h)}
__device__ __forceinline__ void dif8(double2 (&x)[8], const double2 *t, int j, int h) {
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const double2 a = x[r], c = x[r + 4];
    x[r] = cadd(a, c);
    x[r + 4] = cmul(csub(a, c), t[j + r * h]);
  }
#pragma unroll
  for (int r = 0; r < 8; r += (r & 1) ? 3 : 1) {
    const double2 a = x[r], c = x[r + 2];
    x[r] = cadd(a, c);
    x[r + 2] = cmul(csub(a, c), t[2 * (j + (r & 1) * h)]);
  }
#pragma unroll
  for (int r = 0; r < 8; r += 2) {
    const double2 a = x[r], c = x[r + 1];
    x[r] = cadd(a, c);
    x[r + 1] = cmul(csub(a, c), t[4 * j]);
  }
}
// and back, with half-spans h, 2h, 4h; the upper half of the results is not formed if `low`
template <bool low>
__device__ __forceinline__ void dit8(double2 (&x)[8], const double2 *t, int j, int h) {
#pragma unroll
  for (int r = 0; r < 8; r += 2) {
    const double2 a = x[r], c = cmulc(x[r + 1], t[4 * j]);
    x[r] = cadd(a, c);
    x[r + 1] = csub(a, c);
  }
#pragma unroll
  for (int r = 0; r < 8; r += (r & 1) ? 3 : 1) {
    const double2 a = x[r], c = cmulc(x[r + 2], t[2 * (j + (r & 1) * h)]);
    x[r] = cadd(a, c);
    x[r + 2] = csub(a, c);
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const double2 a = x[r], c = cmulc(x[r + 4], t[j + r * h]);
    x[r] = cadd(a, c);
    if (!low) x[r + 4] = csub(a, c);
  }
}
// the stages with half-spans below 2^K, K <= 3, on eight neighbours; w1, w2, w3 = the twiddles
// e^{-2 pi i q / 8}
template <int K>
__device__ __forceinline__ void dif_tail(double2 (&x)[8], double2 w1, double2 w2, double2 w3) {
  if (K == 3) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const double2 a = x[r], c = x[r + 4], e = csub(a, c);
      x[r] = cadd(a, c);
      x[r + 4] = r == 0 ? e : cmul(e, r == 1 ? w1 : r == 2 ? w2 : w3);
    }
  }
  if (K >= 2) {
#pragma unroll
    for (int r = 0; r < 8; r += (r & 1) ? 3 : 1) {
      const double2 a = x[r], c = x[r + 2], e = csub(a, c);
      x[r] = cadd(a, c);
      x[r + 2] = (r & 1) ? cmul(e, w2) : e;
    }
  }
#pragma unroll
  for (int r = 0; r < 8; r += 2) {
    const double2 a = x[r], c = x[r + 1];
    x[r] = cadd(a, c);
    x[r + 1] = csub(a, c);
  }
}
template <int K>
__device__ __forceinline__ void dit_head(double2 (&x)[8], double2 w1, double2 w2, double2 w3) {
#pragma unroll
  for (int r = 0; r < 8; r += 2) {
    const double2 a = x[r], c = x[r + 1];
    x[r] = cadd(a, c);
    x[r + 1] = csub(a, c);
  }
  if (K >= 2) {
#pragma unroll
    for (int r = 0; r < 8; r += (r & 1) ? 3 : 1) {
      const double2 a = x[r], c = (r & 1) ? cmulc(x[r + 2], w2) : x[r + 2];
      x[r] = cadd(a, c);
      x[r + 2] = csub(a, c);
    }
  }
  if (K == 3) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const double2 a = x[r], c = r == 0 ? x[4] : cmulc(x[r + 4], r == 1 ? w1 : r == 2 ? w2 : w3);
      x[r] = cadd(a, c);
      x[r + 4] = csub(a, c);
    }
  }
}

template <int NT>
__global__ __launch_bounds__(NT) void k_bvm_matvec(const InstDesc *__restrict__ D, ItemMap map, int src_sel, int src_j,
                                                   int dst_sel, int dst_j, int mode, int nrows) {
  extern __shared__ double2 buf[];
  const int item = xcd_item(blockIdx.x, gridDim.x);
  const int q = item_slot(map, item);
  if (item_gated(map, q)) return;
  const InstDesc &d = D[map.ids[q]];
  const int m = d.m, s = d.s, mu1 = d.mu1, lg = d.log2L, L = 1 << lg, T = L >> 3, tid = threadIdx.x;
  const int tl = tid & (T - 1), row = tid >> (lg - 3), rows = nrows > 0 ? nrows : s;
  const int n = (item - map.pre[q]) * (NT >> (lg - 3)) + row, nn = min(n, rows - 1);
  const double *Z = vsel(d, src_sel, src_j);
  double *W = vsel(d, dst_sel, dst_j);
  // interior rows: S and M apply the same main formula without wrap-around, so the difference is zero
  const bool zero = mode == 3 && nn >= d.nu && nn < s - (mu1 - 1 - d.nu);
  if (T == NT && zero) {  // the whole workgroup
    for (int i = tid; i < m; i += NT) W[(size_t)n * m + i] = 0.0;
    return;
  }
  // twiddles of pass p >= 1, t_p[k] = tw[k << 3p], one behind the other
  const int K = lg % 3 == 0 ? 3 : lg % 3, n8 = (lg - K) / 3;
  double2 *tw = buf + 8 * NT;
  {
    int at = 0;
    for (int p = 1; p < n8; ++p) {
      const int cnt = L >> (3 * p + 1);
      for (int k = tid; k < cnt; k += NT) tw[at + k] = gld(d.twL + (k << (3 * p)));
      at += cnt;
    }
  }
  double u[4], v[4];
  int ix[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    u[r] = v[r] = 0.0;
    ix[r] = min(tl + r * T, m - 1);
  }
  // u += a_t Z[col_t], v += b_t Z[col_t], t in order; four coefficients' loads in flight
  auto combine = [&](const double *ra, const double *rb, int c0, bool wrap) {
    for (int t0 = 0; t0 < mu1; t0 += 4) {
      double z[4][4], ca[4], cb[4];
      bool ok[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int t = min(t0 + e, mu1 - 1);
        int col = c0 + t;
        if (wrap) col = (col % s + s) % s;
        const int cc = min(max(col, 0), s - 1);
        ok[e] = t0 + e < mu1 && cc == col;
        ca[e] = gld(ra + t);
        cb[e] = gld(rb + t);
#pragma unroll
        for (int r = 0; r < 4; ++r) z[e][r] = gld(Z + (size_t)cc * m + ix[r]);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          u[r] = ok[e] ? fma(ca[e], z[e][r], u[r]) : u[r];
          v[r] = ok[e] ? fma(cb[e], z[e][r], v[r]) : v[r];
        }
    }
  };
  if (mode == 1) {
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = gld(Z + (size_t)nn * m + ix[r]);
  } else {
    if (mode != 2) combine(d.band_a + (size_t)nn * mu1, d.band_b + (size_t)nn * mu1, d.band_c[nn] - 1, false);
    if (mode == 3) {  // BVM rows, subtracted
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        u[r] = -u[r];
        v[r] = -v[r];
      }
    }
    // circulant rows: the main formula (stored in s-form row nu - 1) wrapped mod s
    if (mode >= 2) combine(d.band_a + (size_t)(d.nu - 1) * mu1, d.band_b + (size_t)(d.nu - 1) * mu1, nn - d.nu, true);
  }
  double2 x[8];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    x[r] = make_double2(tl + r * T < m ? v[r] : 0.0, 0.0);
    x[r + 4] = make_double2(0.0, 0.0);
  }
  double2 *rb = buf + (size_t)row * L;
  dif8(x, d.twL, tl, T);
#pragma unroll
  for (int r = 0; r < 8; ++r) rb[fft_sw(tl + r * T)] = x[r];
  __syncthreads();
  int at = 0;
  for (int p = 1; p < n8; ++p) {
    const int lh = lg - 3 * (p + 1), h = 1 << lh, j = tl & (h - 1), i0 = ((tl >> lh) << (lh + 3)) + j;
#pragma unroll
    for (int r = 0; r < 8; ++r) x[r] = rb[fft_sw(i0 + r * h)];
    dif8(x, tw + at, j, h);
#pragma unroll
    for (int r = 0; r < 8; ++r) rb[fft_sw(i0 + r * h)] = x[r];
    __syncthreads();
    at += L >> (3 * p + 1);
  }
  {
    const double2 w1 = gld(d.twL + (L >> 3)), w2 = gld(d.twL + (L >> 2)), w3 = gld(d.twL + 3 * (L >> 3));
    double2 ch[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) ch[r] = gld(d.chat + 8 * tl + r);
#pragma unroll
    for (int r = 0; r < 8; ++r) x[r] = rb[fft_sw(8 * tl + r)];
    if (K == 3) dif_tail<3>(x, w1, w2, w3);
    else if (K == 2) dif_tail<2>(x, w1, w2, w3);
    else dif_tail<1>(x, w1, w2, w3);
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const double2 P = cmul(ch[r], x[r]);
      const double2 Qv = cmulc(x[r], ch[r]);
      x[r] = make_double2(P.x - Qv.y, P.y + Qv.x);
    }
    if (K == 3) dit_head<3>(x, w1, w2, w3);
    else if (K == 2) dit_head<2>(x, w1, w2, w3);
    else dit_head<1>(x, w1, w2, w3);
#pragma unroll
    for (int r = 0; r < 8; ++r) rb[fft_sw(8 * tl + r)] = x[r];
  }
  __syncthreads();
  for (int p = n8 - 1; p >= 1; --p) {
    const int lh = lg - 3 * (p + 1), h = 1 << lh, j = tl & (h - 1), i0 = ((tl >> lh) << (lh + 3)) + j;
    at -= L >> (3 * p + 1);
#pragma unroll
    for (int r = 0; r < 8; ++r) x[r] = rb[fft_sw(i0 + r * h)];
    dit8<false>(x, tw + at, j, h);
#pragma unroll
    for (int r = 0; r < 8; ++r) rb[fft_sw(i0 + r * h)] = x[r];
    __syncthreads();
  }
#pragma unroll
  for (int r = 0; r < 8; ++r) x[r] = rb[fft_sw(tl + r * T)];
  dit8<true>(x, d.twL, tl, T);
  const double coef = (mode == 1 ? 1.0 : -d.tau) * d.scale / (double)L;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int i = tl + r * T;
    if (i < m && n < rows) {
      const double y = fma(coef, fma(d.dp[i], x[r].x, d.dm[i] * x[r].y), u[r]);
      W[(size_t)n * m + i] = zero ? 0.0 : y;
    }
  }
}

// Item = (instance, row n):  b[n] = tau sum_q bhat[n][q] f[c+q] - a0[n] u0 + tau b0[n] Ju0,
// where a0[n], b0[n] are the coefficients on u_0 (nonzero only when the band starts at u_0).
__global__ __launch_bounds__(ST_NT) void k_rhs(const InstDesc *__restrict__ D, ItemMap map,
                                               int use_ju0) {
  const int q = item_slot(map, blockIdx.x);
  if (item_gated(map, q)) return;
  const InstDesc &d = D[map.ids[q]];
  const int n = blockIdx.x - map.pre[q];
  const int m = d.m, c = d.band_c[n];
  const double *ra = d.band_a + (size_t)n * d.mu1;
  const double *rb = d.band_b + (size_t)n * d.mu1;
  for (int i = threadIdx.x; i < m; i += ST_NT) {
    double acc = 0.0;
    for (int t = 0; t < d.mu1; ++t) acc = fma(rb[t], d.f[(size_t)(c + t) * m + i], acc);
    acc *= d.tau;
    if (c == 0) {
      acc = fma(-ra[0], d.u0[i], acc);
      if (use_ju0 && d.need_ju0) acc = fma(d.tau * rb[0], d.Ju0[i], acc);
    }
    d.b[(size_t)n * m + i] = acc;
  }
}

// Time-axis real DFT.  Item = (instance, group of 2*TP spatial columns); TP complex FFTs of
// length s per workgroup (TP = 2, 4 or 8, chosen per plan so that the launch has enough
// workgroups).  Items in XCD-contiguous order (xcd_item), so the column groups that share a
// cache line of a row are read through the same L2.  The twiddle table (s/2 entries) is copied
// into LDS behind the data.

// If epoch_ctr is set, the first workgroup also draws the next block-solve epoch from the
// device-wide counter into epoch_slot[0] (read by the block solve that follows on the stream),
// so a recorded launch sequence gets a fresh epoch on every replay, and clears the block
// solve's unit counter epoch_slot[1].
//
// Source VS_VN: the basis vector v_j of an instance whose Gram-Schmidt runs in two passes is w / H[j];
// this kernel, its only reader before the next Gram-Schmidt pass, scales it on the way in and stores
// it (instead of a launch of its own per step: 255 x 128 1388 to 1363 us).
template <int TP>
__global__ __launch_bounds__(ST_NT) void k_time_rfft(const InstDesc *__restrict__ D, ItemMap map,
                                                     int src_sel, int src_j, int max_log2s,
                                                     unsigned long long *epoch_ctr,
                                                     unsigned long long *epoch_slot) {
  extern __shared__ double2 buf[];
  if (epoch_ctr && blockIdx.x == 0 && threadIdx.x == 0) {
    *epoch_slot = atomicAdd(epoch_ctr, 1ull) + 1ull;
    epoch_slot[1] = 0ull;  // the block solve's unit counter
  }
  const int item = xcd_item(blockIdx.x, gridDim.x);
  const int q = item_slot(map, item);
  if (item_gated(map, q)) return;
  const InstDesc &d = D[map.ids[q]];
  const int m = d.m, mp = d.mp, log2s = d.log2s, s = 1 << log2s;
  const bool next = src_sel == VS_VN && d.nwide > 0;
  const double *V = next ? d.w : vsel(d, src_sel == VS_VN ? (int)VS_V : src_sel, src_j);
  double *Vn = d.V + (size_t)src_j * s * m;
  const double nrm = next ? d.H[src_j] : 1.0, inv = nrm > 0.0 ? 1.0 / nrm : 0.0;
  const int col0 = (item - map.pre[q]) * 2 * TP;
  double2 *twl = buf + ((size_t)TP << max_log2s);
  for (int i = threadIdx.x; i < s / 2; i += ST_NT) twl[i] = d.tws[i];
  for (int e = threadIdx.x; e < s * 2 * TP; e += ST_NT) {
    const int n = e / (2 * TP), c = e % (2 * TP);
    const int col = col0 + c;
    double v = (col < m) ? V[(size_t)n * m + col] : 0.0;
    if (next) {
      v *= inv;
      if (col < m) Vn[(size_t)n * m + col] = v;
    }
    reinterpret_cast<double *>(&buf[(c >> 1) * s + n])[c & 1] = v;
  }
  __syncthreads();
  fft_dif<ST_NT>(buf, log2s, TP, twl);
  const int nbk = s / 2 + 1;
  for (int e = threadIdx.x; e < nbk * 2 * TP; e += ST_NT) {
    const int k = e / (2 * TP), c = e % (2 * TP), f = c >> 1;
    const int col = col0 + c;
    if (col >= mp) continue;
    const int kk = (s - k) & (s - 1);
    const double2 Zk = buf[f * s + bitrev(k, log2s)];
    const double2 Zn = cconj(buf[f * s + bitrev(kk, log2s)]);
    double2 o;
    if ((c & 1) == 0) {
      o = make_double2(0.5 * (Zk.x + Zn.x), 0.5 * (Zk.y + Zn.y));
    } else {  // (Zk - Zn) * (-i/2)
      o = make_double2(0.5 * (Zk.y - Zn.y), -0.5 * (Zk.x - Zn.x));
    }
    if (col >= m) o = make_double2(0.0, 0.0);
    d.Vh[(size_t)k * mp + col] = o;
  }
}

template <int TP>
__global__ __launch_bounds__(ST_NT) void k_time_irfft(const InstDesc *__restrict__ D, ItemMap map,
                                                      int dst_sel, int dst_j, int max_log2s) {
  extern __shared__ double2 buf[];
  const int item = xcd_item(blockIdx.x, gridDim.x);
  const int q = item_slot(map, item);
  if (item_gated(map, q)) return;
  const InstDesc &d = D[map.ids[q]];
  const int m = d.m, mp = d.mp, log2s = d.log2s, s = 1 << log2s;
  double *W = vsel(d, dst_sel, dst_j);
  const double2 *Wh = d.Vh;
  const int col0 = (item - map.pre[q]) * 2 * TP;
  double2 *twl = buf + ((size_t)TP << max_log2s);
  for (int i = threadIdx.x; i < s / 2; i += ST_NT) twl[i] = d.tws[i];
  // position p of the bit-reversed input holds Z[k], k = bitrev(p); Z = What_a + i What_b
  for (int e = threadIdx.x; e < s * TP; e += ST_NT) {
    const int p = e / TP, f = e % TP;
    const int k = bitrev(p, log2s);
    const int ca = col0 + 2 * f;
    double2 a, b;
    if (k <= s / 2) {
      a = Wh[(size_t)k * mp + ca];
      b = Wh[(size_t)k * mp + ca + 1];
      if (k == 0 || k == s / 2) {
        a.y = 0.0;
        b.y = 0.0;
      }
    } else {
      a = cconj(Wh[(size_t)(s - k) * mp + ca]);
      b = cconj(Wh[(size_t)(s - k) * mp + ca + 1]);
    }
    buf[f * s + p] = make_double2(a.x - b.y, a.y + b.x);
  }
  __syncthreads();
  fft_dit_inv<ST_NT>(buf, log2s, TP, twl);
  const double inv_s = 1.0 / (double)s;
  for (int e = threadIdx.x; e < s * 2 * TP; e += ST_NT) {
    const int n = e / (2 * TP), c = e % (2 * TP);
    const int col = col0 + c;
    if (col >= m) continue;
    const double2 z = buf[(c >> 1) * s + n];
    W[(size_t)n * m + col] = ((c & 1) ? z.y : z.x) * inv_s;
  }
}

// BCCB preconditioners (the 2-D diagonalisation of Section 3.2): after the time DFT, each time
// frequency k needs Y = F_m^{-1} diag(1/(lam_k - tau mu_k lamx_j)) F_m X over the space index.
// DFT of order m (any m) by Bluestein's method: with w_n = e^{-i pi n^2/m} (nj = (n^2 + j^2 -
// (j-n)^2)/2),  X_j = w_j sum_n (x_n w_n) conj(w_{j-n}),  a linear convolution done through the
// power-of-two FFT of length L >= 2m - 1 with the stored spectrum of conj(w) (bit-reversed).
// The inverse uses F^{-1} y = conj(F conj(y)) / m.  Item = (instance, k); one LDS buffer.
__device__ __forceinline__ void chirp_filter(double2 *buf, const InstDesc &d) {
  fft_dif<ST_NT>(buf, d.log2L, 1, d.twL);
  const int L = 1 << d.log2L;
  for (int i = threadIdx.x; i < L; i += ST_NT) buf[i] = cmul(buf[i], d.bh[i]);
  __syncthreads();
  fft_dit_inv<ST_NT>(buf, d.log2L, 1, d.twL);
}

__global__ __launch_bounds__(ST_NT) void k_bccb_solve(const InstDesc *__restrict__ D, ItemMap map) {
  extern __shared__ double2 buf[];
  const int q = item_slot(map, blockIdx.x);
  if (item_gated(map, q)) return;
  const InstDesc &d = D[map.ids[q]];
  const int k = blockIdx.x - map.pre[q];
  const int m = d.m, L = 1 << d.log2L;
  double2 *v = d.Vh + (size_t)k * d.mp;
  const double invL = 1.0 / (double)L;
  double2 lk = d.lam[k];
  if (k == 0 && d.pc == 2) lk = make_double2(d.lam0s, 0.0);
  const double2 tmk = cscale(d.mu[k], -d.tau);
  for (int i = threadIdx.x; i < L; i += ST_NT) buf[i] = i < m ? cmul(v[i], d.chirp[i]) : make_double2(0.0, 0.0);
  __syncthreads();
  chirp_filter(buf, d);
  // X_j = w_j conv_j / L; Y_j = X_j / (lam_k - tau mu_k lamx_j); next input conj(Y_j) w_j
  for (int j = threadIdx.x; j < L; j += ST_NT) {
    double2 t = make_double2(0.0, 0.0);
    if (j < m) {
      const double2 X = cscale(cmul(d.chirp[j], buf[j]), invL);
      const double2 e = cadd(lk, cmul(tmk, d.lamx[j]));
      const double ee = e.x * e.x + e.y * e.y;
      const double2 Y = cscale(cmulc(X, e), 1.0 / ee);
      t = cmul(cconj(Y), d.chirp[j]);
    }
    buf[j] = t;
  }
  __syncthreads();
  chirp_filter(buf, d);
  const double sc = invL / (double)m;
  for (int n = threadIdx.x; n < m; n += ST_NT) v[n] = cscale(cconj(cmul(d.chirp[n], buf[n])), sc);
}

// ------------------------------------------------------------------------------------
static hipError_t set_lds(const void *fn, size_t bytes) {
  if (bytes <= 65536) return hipSuccess;
  return hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

hipError_t launch_symbol(const double *cG, double2 *chat_br, int log2L, const double2 *twL,
                         hipStream_t st) {
  const size_t lds = sizeof(double2) << log2L;
  hipError_t e = set_lds((const void *)k_symbol, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_symbol, dim3(1), dim3(ST_NT), lds, st, cG, chat_br, log2L, twL);
  return hipGetLastError();
}

// Threads per workgroup: an eighth of the longest row, at least a wavefront.
static int matvec_threads(int max_log2L) { return std::max(64, (1 << max_log2L) >> 3); }

int bvm_matvec_items(int rows, int log2L, int max_log2L) {
  const int per = matvec_threads(max_log2L) >> (log2L - 3);
  return (rows + per - 1) / per;
}

template <int NT>
static hipError_t bvm_matvec_nt(const InstDesc *D, const ItemMap &map, int items, int src_sel, int src_j, int dst_sel,
                                int dst_j, int mode, int rows, hipStream_t st) {
  const size_t lds = sizeof(double2) * (8 * NT + NT * 5 / 8);  // rows, and NT (1/2 + 1/16 + ..) twiddles
  hipError_t e = set_lds((const void *)k_bvm_matvec<NT>, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_bvm_matvec<NT>, dim3(items), dim3(NT), lds, st, D, map, src_sel, src_j, dst_sel, dst_j, mode, rows);
  return hipGetLastError();
}

hipError_t launch_bvm_matvec(const InstDesc *D, const ItemMap &map, int items, int max_log2L,
                             int src_sel, int src_j, int dst_sel, int dst_j, int mode, int rows,
                             hipStream_t st) {
  if (items <= 0) return hipSuccess;
  switch (matvec_threads(max_log2L)) {
    case 64: return bvm_matvec_nt<64>(D, map, items, src_sel, src_j, dst_sel, dst_j, mode, rows, st);
    case 128: return bvm_matvec_nt<128>(D, map, items, src_sel, src_j, dst_sel, dst_j, mode, rows, st);
    case 256: return bvm_matvec_nt<256>(D, map, items, src_sel, src_j, dst_sel, dst_j, mode, rows, st);
    case 512: return bvm_matvec_nt<512>(D, map, items, src_sel, src_j, dst_sel, dst_j, mode, rows, st);
    case 1024: return bvm_matvec_nt<1024>(D, map, items, src_sel, src_j, dst_sel, dst_j, mode, rows, st);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_rhs(const InstDesc *D, const ItemMap &map, int items, int use_ju0,
                      hipStream_t st) {
  if (items <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_rhs, dim3(items), dim3(ST_NT), 0, st, D, map, use_ju0);
  return hipGetLastError();
}

template <int TP>
static hipError_t rfft_tp(const InstDesc *D, const ItemMap &map, int items, int max_log2s,
                          int src_sel, int src_j, hipStream_t st, unsigned long long *epoch_ctr,
                          unsigned long long *epoch_slot) {
  const size_t lds = ((sizeof(double2) * (2 * TP + 1)) << max_log2s) / 2;
  hipError_t e = set_lds((const void *)k_time_rfft<TP>, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_time_rfft<TP>, dim3(items), dim3(ST_NT), lds, st, D, map, src_sel, src_j,
                     max_log2s, epoch_ctr, epoch_slot);
  return hipGetLastError();
}

template <int TP>
static hipError_t irfft_tp(const InstDesc *D, const ItemMap &map, int items, int max_log2s,
                           int dst_sel, int dst_j, hipStream_t st) {
  const size_t lds = ((sizeof(double2) * (2 * TP + 1)) << max_log2s) / 2;
  hipError_t e = set_lds((const void *)k_time_irfft<TP>, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_time_irfft<TP>, dim3(items), dim3(ST_NT), lds, st, D, map, dst_sel, dst_j,
                     max_log2s);
  return hipGetLastError();
}

hipError_t launch_time_rfft(const InstDesc *D, const ItemMap &map, int items, int max_log2s,
                            int cols, int src_sel, int src_j, hipStream_t st,
                            unsigned long long *epoch_ctr, unsigned long long *epoch_slot) {
  if (items <= 0) return hipSuccess;
  switch (cols) {
    case 4: return rfft_tp<2>(D, map, items, max_log2s, src_sel, src_j, st, epoch_ctr, epoch_slot);
    case 8: return rfft_tp<4>(D, map, items, max_log2s, src_sel, src_j, st, epoch_ctr, epoch_slot);
    case 16: return rfft_tp<8>(D, map, items, max_log2s, src_sel, src_j, st, epoch_ctr, epoch_slot);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_time_irfft(const InstDesc *D, const ItemMap &map, int items, int max_log2s,
                             int cols, int dst_sel, int dst_j, hipStream_t st) {
  if (items <= 0) return hipSuccess;
  switch (cols) {
    case 4: return irfft_tp<2>(D, map, items, max_log2s, dst_sel, dst_j, st);
    case 8: return irfft_tp<4>(D, map, items, max_log2s, dst_sel, dst_j, st);
    case 16: return irfft_tp<8>(D, map, items, max_log2s, dst_sel, dst_j, st);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_bccb_solve(const InstDesc *D, const ItemMap &map, int items, int max_log2L,
                             hipStream_t st) {
  if (items <= 0) return hipSuccess;
  const size_t lds = sizeof(double2) << max_log2L;
  hipError_t e = set_lds((const void *)k_bccb_solve, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_bccb_solve, dim3(items), dim3(ST_NT), lds, st, D, map);
  return hipGetLastError();
}

// Spatial columns per time-FFT workgroup: 16 (128-byte row segments) while that still gives
// the launch at least two workgroups per CU, else 8, else 4.
int time_fft_cols_per_item(long long total_mp, int cus) {
  for (int cols = 16; cols > 4; cols >>= 1)
    if (total_mp / cols >= 2LL * cus) return cols;
  return 4;
}

}  // namespace fde
