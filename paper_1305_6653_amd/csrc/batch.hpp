// Per-instance descriptors shared by every kernel.  A launch covers a set of instances: the
// host passes, per launch, the prefix sums of the number of work items each instance
// contributes (`pre[0] = 0, pre[i+1] = pre[i] + items_i`) and the instance ids; a workgroup
// finds its instance by binary search and decodes its local item from that instance's sizes.
// A single solve is a batch of one.
#pragma once
#include <hip/hip_runtime.h>

namespace fde {

// Hierarchical form of the blocks (k_hier.hip): levels of 64 << l rows a half, ranks up to 32
static constexpr int HIER_LEVELS = 6, HIER_RMAX = 32;
static constexpr int HIER_R0 = 20, HIER_R0_32 = 16;  // level 0's largest rank, FP64 and FP32 (any alpha in (1, 2))
static constexpr int HIER_CHUNK = 4;  // panels per workgroup of the apply's first kernel

struct InstDesc {
  // sizes
  int m, s, mp, nb, npan, log2L, log2s, mu1, nu;
  int W;     // workgroups per block in the cooperative block solve
  int nblk;  // Krylov reduction blocks
  int need_ju0;  // the right-hand side uses J u_0 (a u_0 coefficient in B)
  double tau, scale;
  // operator tables
  const double *dp, *dm, *g;
  const double2 *chat, *twL, *tws, *lam, *mu;
  const int *band_c;
  const double *band_a, *band_b;
  // factors (complex FP64 or FP32 per the plan), block-solve flags (epoch of the last
  // published panel, [nb][npan][2])
  void *K, *dinv;
  unsigned long long *tsflags;
  // BCCB preconditioners (pc = 1: S2, 2: S2~ with the zero time frequency moved to lam0s):
  // chirp w_n = e^{-i pi n^2/m} [m], FFT_L of the chirp filter in bit-reversed order [L], and
  // the eigenvalues of s(J) [m]
  int pc;
  double lam0s;
  const double2 *chirp, *bh, *lamx;
  // Hessenberg route to the blocks (blk = 1): H, Q and Q^T of J = Q H Q^T (real, [m][mp]);
  // per block the multipliers and row exchanges of the shifted Hessenberg LU ([nb][mp]).
  // Vts is the frequency-domain vector the block solve works on: Vh for the LU route, a
  // second [nb][mp] buffer for the Hessenberg route (Q^T is applied out of place).
  int blk;
  const double *hH, *hQ, *hQt;
  double2 *hl;
  int *hpiv;
  double2 *Vts;
  // hierarchical form of the blocks: levels in use (0: one leaf), columns per level, the basis
  // tables, leaf inverses, W', G and the panel partials of an apply (layouts in k_hier.hip)
  int nlev, hR[HIER_LEVELS];
  const double *hx;
  void *hD, *hW[HIER_LEVELS], *hG[HIER_LEVELS], *ha;
  // vectors (FP64, [s][m] unless noted)
  double *V, *Z;              // (R+1) and R vectors
  double *w, *x, *b, *tmp, *sio;
  double *u0, *f, *Ju0;       // [m], [s+1][m], [m]
  double2 *Vh;                // [nb][mp]
  double *part0, *part1;      // [nblk] reduction partials
  double *partm;              // [R+1][nblk] partials of the Gram-Schmidt projections
  double *H, *y, *nrm;        // Hessenberg column [R+2], LSQ solution [R], norms [2]
  double *h2;                 // [R+2] second Gram-Schmidt pass of the current column
  unsigned *gctr;             // [1] chunks done in the current Gram-Schmidt launch (0 between)
  // Gram-Schmidt in two launches (k_krylov.hip): chunks (0: the launch chain), their partials
  // [2 R + 3][nwide] and the strictly lower part of V^T V of the current cycle, [R + 1][R + 1]
  int nwide, ldgram;
  double *wpart, *gram;
};

// Nodes of level `lev` over npan panels: pairs of 1 << lev panels whose right half is not empty.
__host__ __device__ inline int hier_nodes_p(int npan, int lev) {
  return (npan + (1 << lev) - 1) >> (lev + 1);
}
__host__ __device__ inline int hier_nodes(int mp, int lev) { return hier_nodes_p(mp >> 6, lev); }

// vector selectors resolved on the device
// (VS_VN, the time FFT's only: V_j, formed from w where the two-pass Gram-Schmidt left it unscaled)
enum VSel : int { VS_V = 0, VS_Z, VS_W, VS_X, VS_B, VS_TMP, VS_SIO, VS_U0, VS_JU0, VS_VN };

__device__ __forceinline__ double *vsel(const InstDesc &d, int sel, int j) {
  const size_t n = (size_t)d.s * d.m;
  switch (sel) {
    case VS_V: return d.V + (size_t)j * n;
    case VS_Z: return d.Z + (size_t)j * n;
    case VS_W: return d.w;
    case VS_X: return d.x;
    case VS_B: return d.b;
    case VS_TMP: return d.tmp;
    case VS_SIO: return d.sio;
    case VS_U0: return d.u0;
    default: return d.Ju0;
  }
}

// Launch-wide item map: instance ids[count], prefix pre[count+1].  If gate is set, the
// items of instance i are skipped unless gate[i] != 0 (a device array written by earlier
// launches, so a fixed launch sequence can follow the instances' progress).
struct ItemMap {
  const int *ids;
  const int *pre;
  int count;
  const int *gate;
};

__device__ __forceinline__ bool item_gated(const ItemMap &mp, int q) {
  return mp.gate != nullptr && mp.gate[mp.ids[q]] == 0;
}

// Restarted GMRES control, one record per instance of a plan, advanced on the device between
// launches.  Restart lengths up to GM_RMAX.
static constexpr int GM_RMAX = 64;

struct GmresCtl {
  double bnorm;     // ||b||
  double tol;       // relative tolerance on ||b - M x|| / ||b||
  double truer;     // last true relative residual
  double est;       // Givens estimate of the relative residual
  int maxit, its, k, restarts;
  int conv, done, fail, active;  // active: taking part in the current cycle (mirrors the gate)
  int badrhs, pad;               // badrhs: ||b|| is not finite (set by k_gm_init)
};

struct GmresWork {
  double H[GM_RMAX + 1][GM_RMAX];  // rotated Hessenberg matrix of the current cycle
  double cs[GM_RMAX], sn[GM_RMAX], g[GM_RMAX + 1];
};

// gate arrays of a plan, [GATE_COUNT][count]
enum GateSel : int { GATE_LIVE = 0, GATE_ACTIVE, GATE_X0, GATE_COUNT };

// Returns the position q in the map with pre[q] <= item < pre[q+1].
// Workgroups are dispatched to the eight XCDs in turn (workgroup b to XCD b mod 8).  This
// bijection of [0, n) gives XCD x a contiguous range of item indices, so items that share data
// (neighbouring columns, the tiles of one block) are served by the same L2.
__device__ __forceinline__ int xcd_item(int bid, int n) {
  const int per = n >> 3, rem = n & 7, x = bid & 7;
  return x * per + (x < rem ? x : rem) + (bid >> 3);
}

__device__ __forceinline__ int item_slot(const ItemMap &mp, int item) {
  int lo = 0, hi = mp.count - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (mp.pre[mid] <= item) lo = mid; else hi = mid - 1;
  }
  return lo;
}

}  // namespace fde
