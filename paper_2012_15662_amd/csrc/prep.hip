// Preparation of the three-index factors b from the three-centre integrals
// T[k][mu][nu] = (mu nu|k) and the metric G_kl = (k|l) (Sec. II, RI): the
// metric is factorised as G = P L D L^T P^T (L unit lower triangular, D block
// diagonal with 1x1 and 2x2 blocks, Bunch-Kaufman partial pivoting), each D
// block's eigenvalues below delta are raised to delta (D~), and
//   b^T = D~^(-1/2) L^-1 P^T T,
// i.e. the solution of P L D~^(1/2) b^T = T.  Done once per molecule.
//
//   k_rowsum     ||G||_inf (max row sum of |G|), for the default delta
//   k_bk_init    working copy of G, L = I, perm, step state
//   k_bk_coop    the factorisation in one launch, up to 2048 auxiliary functions
//                (k_bk_coop_l: L in the order of the pivots); above, per column:
//   k_bk_pivot   one workgroup: the pivot decision at the current column, the
//                symmetric interchange, the D block and the L column(s)
//   k_bk_update  trailing update A -= L_k D_k L_k^T (all workgroups)
//   k_bk_correct D~^(-1/2) per block (2x2 blocks in closed form)
//   k_linv_rows  X = L^-1, one wave per column (forward substitution), one
//                launch; k_linv (one column step at a time, rank-1 updates)
//                above 2048 auxiliary functions
//   k_compose    M'^T[i][k] = sum_r D~^(-1/2)[k][r] X[r][i]  (M' = D~^(-1/2) L^-1,
//                zero right of its first superdiagonal)
//   k_prep_solve b^T = M T from T to b, on the 8 x 16 blocks of (mu, nu) with an
//                element on or above the diagonal (k_prep_solve_small: a single
//                function or pair)
//
// Pivot rule (alpha = (1 + sqrt 17)/8) at column k, with colmax/imax the
// largest |A_ik| below the diagonal (lowest index on ties) and rowmax the
// largest off-diagonal |A_{imax,j}| of the trailing row imax: 1x1 at k if
// |A_kk| >= alpha colmax or |A_kk| rowmax >= alpha colmax^2; else 1x1 at imax
// if |A_{imax,imax}| >= alpha rowmax; else 2x2 on (k, imax).  Interchanges
// also swap the rows of the L columns already computed (P L form).
#include <algorithm>
#include <cmath>
#include <string>

#include "rif_internal.hpp"
#include "strip64.hpp"
#include "wave.hpp"

namespace rif {

namespace {
constexpr double kAlpha = 0.6403882032022076;   // (1 + sqrt(17)) / 8
constexpr int kPivThreads = 1024;
struct BkState { int k, kstep, next; };
}  // namespace

__global__ __launch_bounds__(256) void k_rowsum(int n, const double* __restrict__ G, double* __restrict__ rs) {
  // row sum i of |G| per wave, the lanes reading along the row
  const int i = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (i >= n) return;
  const double* g = G + (long)i * n;
  double s = 0.0;
  for (int j = lane; j < n; j += 64) s += fabs(g[j]);
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
  if (lane == 0) rs[i] = s;
}

__global__ __launch_bounds__(256) void k_delta(int nblk, const double* __restrict__ part, double* __restrict__ del) {
  // delta = sqrt(2^-52) * max row sum = 2^-26 * ||G||_inf
  __shared__ double red[256];
  double m = 0.0;
  for (int i = threadIdx.x; i < nblk; i += 256) m = fmax(m, part[i]);
  red[threadIdx.x] = m;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if (threadIdx.x < h) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + h]);
    __syncthreads();
  }
  if (threadIdx.x == 0) del[0] = red[0] * 0x1p-26;
}

__global__ __launch_bounds__(256) void k_bk_init(int n, const double* __restrict__ G, double* __restrict__ A,
                                                 double* __restrict__ L, double* __restrict__ D,
                                                 int* __restrict__ perm, int* __restrict__ bsz, BkState* st) {
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  const long nn = (long)n * n;
  if (i < nn) {
    const int r = (int)(i / n), c = (int)(i - (long)r * n);
    A[i] = G[i];
    L[i] = r == c ? 1.0 : 0.0;
    D[i] = 0.0;
  }
  if (i < n) { perm[i] = (int)i; bsz[i] = 0; }
  if (i == 0) { st->k = 0; st->kstep = 0; st->next = 0; }
}

// Max of |v| with its index (lowest index on ties) over a workgroup.
__device__ void block_argmax(double& v, int& idx, double* sv, int* si) {
  const int t = threadIdx.x;
  sv[t] = v;
  si[t] = idx;
  __syncthreads();
  for (int h = kPivThreads / 2; h > 0; h >>= 1) {
    if (t < h) {
      const double a = sv[t], b = sv[t + h];
      const int ia = si[t], ib = si[t + h];
      if (b > a || (b == a && ib < ia)) { sv[t] = b; si[t] = ib; }
    }
    __syncthreads();
  }
  v = sv[0];
  idx = si[0];
  __syncthreads();
}

__global__ __launch_bounds__(kPivThreads) void k_bk_pivot(int n, double* __restrict__ A, double* __restrict__ L,
                                                          double* __restrict__ D, int* __restrict__ perm,
                                                          int* __restrict__ bsz, BkState* st) {
  __shared__ double sv[kPivThreads];
  __shared__ int si[kPivThreads];
  const int t = threadIdx.x;
  const int k = st->next;
  if (k >= n) {   // factorisation finished: the update launched after this does nothing
    if (t == 0) st->kstep = 0;
    return;
  }
  auto a = [&](int i, int j) -> double& { return A[(long)i * n + j]; };
  // column search below the diagonal
  double cm = 0.0;
  int im = n;
  for (int i = k + 1 + t; i < n; i += kPivThreads) {
    const double v = fabs(a(i, k));
    if (v > cm || (v == cm && i < im)) { cm = v; im = i; }
  }
  block_argmax(cm, im, sv, si);
  const double absakk = fabs(a(k, k));
  int kstep = 1, kp = k;
  if (k + 1 < n && fmax(absakk, cm) != 0.0 && absakk < kAlpha * cm) {
    // rowmax: row imax left of the diagonal (columns k..imax-1), column imax
    // below it (the trailing matrix is symmetric only to rounding)
    double rm = 0.0;
    int dummy = 0;
    for (int j = k + t; j < n; j += kPivThreads)
      if (j != im) rm = fmax(rm, fabs(j < im ? a(im, j) : a(j, im)));
    block_argmax(rm, dummy, sv, si);
    if (absakk * rm >= kAlpha * cm * cm) {
      kstep = 1; kp = k;
    } else if (fabs(a(im, im)) >= kAlpha * rm) {
      kstep = 1; kp = im;
    } else {
      kstep = 2; kp = im;
    }
  }
  const int kk = k + kstep - 1;
  if (kp != kk) {
    // symmetric interchange: rows kk <-> kp (all columns), then columns
    for (int j = t; j < n; j += kPivThreads) {
      const double x = a(kk, j);
      a(kk, j) = a(kp, j);
      a(kp, j) = x;
    }
    __syncthreads();
    for (int i = t; i < n; i += kPivThreads) {
      const double x = a(i, kk);
      a(i, kk) = a(i, kp);
      a(i, kp) = x;
    }
    for (int j = t; j < k; j += kPivThreads) {   // rows of the L columns already final
      const double x = L[(long)kk * n + j];
      L[(long)kk * n + j] = L[(long)kp * n + j];
      L[(long)kp * n + j] = x;
    }
    if (t == 0) {
      const int x = perm[kk];
      perm[kk] = perm[kp];
      perm[kp] = x;
    }
    __syncthreads();
  }
  if (kstep == 1) {
    const double d = a(k, k);
    if (t == 0) { D[(long)k * n + k] = d; bsz[k] = 1; }
    if (d != 0.0)
      for (int i = k + 1 + t; i < n; i += kPivThreads) L[(long)i * n + k] = a(i, k) / d;
  } else {
    const double e00 = a(k, k), e10 = a(k + 1, k), e11 = a(k + 1, k + 1);
    const double det = e00 * e11 - e10 * e10;
    const double i00 = e11 / det, i01 = -e10 / det, i11 = e00 / det;
    if (t == 0) {
      D[(long)k * n + k] = e00;
      D[(long)k * n + k + 1] = e10;
      D[(long)(k + 1) * n + k] = e10;
      D[(long)(k + 1) * n + k + 1] = e11;
      bsz[k] = 2;
      bsz[k + 1] = 0;
    }
    for (int i = k + 2 + t; i < n; i += kPivThreads) {
      const double x0 = a(i, k), x1 = a(i, k + 1);
      L[(long)i * n + k] = x0 * i00 + x1 * i01;
      L[(long)i * n + k + 1] = x0 * i01 + x1 * i11;
    }
  }
  if (t == 0) {
    st->k = k;
    st->kstep = kstep;
    st->next = k + kstep;
  }
}

// Trailing update of the step just decided: for i, j >= k + kstep,
//   1x1: A_ij -= L_ik A_jk;  2x2: A_ij -= L_ik A_jk + L_i,k+1 A_j,k+1.
__global__ __launch_bounds__(256) void k_bk_update(int n, double* __restrict__ A, const double* __restrict__ L,
                                                   const BkState* st) {
  const int k = st->k, s = st->kstep;
  const int k0 = k + s;
  if (s == 0 || k0 >= n) return;
  const long m = n - k0, mm = m * m;
  for (long e = (long)blockIdx.x * 256 + threadIdx.x; e < mm; e += (long)gridDim.x * 256) {
    const int i = k0 + (int)(e / m), j = k0 + (int)(e - (e / m) * m);
    double v = A[(long)i * n + j] - L[(long)i * n + k] * A[(long)j * n + k];
    if (s == 2) v -= L[(long)i * n + k + 1] * A[(long)j * n + k + 1];
    A[(long)i * n + j] = v;
  }
}

// D~^(-1/2) per block into Dih (dense, zero outside the blocks); counts the
// raised eigenvalues.
__global__ __launch_bounds__(256) void k_bk_correct(int n, const double* __restrict__ D,
                                                    const int* __restrict__ bsz, const double* __restrict__ delta_p,
                                                    double delta_in, double* __restrict__ Dih,
                                                    int* __restrict__ nraised) {
  const int k = blockIdx.x * 256 + threadIdx.x;
  if (k >= n) return;
  const double delta = delta_in > 0.0 ? delta_in : delta_p[0];
  const int s = bsz[k];
  if (s == 1) {
    const double w = D[(long)k * n + k];
    const double wt = w < delta ? delta : w;
    if (w < delta) atomicAdd(nraised, 1);
    Dih[(long)k * n + k] = 1.0 / sqrt(wt);
  } else if (s == 2) {
    const double a = D[(long)k * n + k], b = D[(long)(k + 1) * n + k], c = D[(long)(k + 1) * n + k + 1];
    // eigenvalues and the unit eigenvector (cs, sn) of the larger one
    const double h = 0.5 * (a - c), r = sqrt(h * h + b * b);
    const double w1 = 0.5 * (a + c) + r, w2 = 0.5 * (a + c) - r;
    double cs, sn;
    if (h >= 0.0) {
      const double x = h + r;
      const double nrm = sqrt(x * x + b * b);
      cs = nrm > 0.0 ? x / nrm : 1.0;
      sn = nrm > 0.0 ? b / nrm : 0.0;
    } else {
      const double y = r - h;
      const double nrm = sqrt(b * b + y * y);
      cs = nrm > 0.0 ? b / nrm : 1.0;
      sn = nrm > 0.0 ? y / nrm : 0.0;
    }
    const double t1 = w1 < delta ? delta : w1, t2 = w2 < delta ? delta : w2;
    if (w1 < delta) atomicAdd(nraised, 1);
    if (w2 < delta) atomicAdd(nraised, 1);
    const double f1 = 1.0 / sqrt(t1), f2 = 1.0 / sqrt(t2);
    // Q = [[cs, -sn], [sn, cs]], Dih = Q diag(f1, f2) Q^T
    Dih[(long)k * n + k] = cs * cs * f1 + sn * sn * f2;
    Dih[(long)k * n + k + 1] = cs * sn * (f1 - f2);
    Dih[(long)(k + 1) * n + k] = cs * sn * (f1 - f2);
    Dih[(long)(k + 1) * n + k + 1] = sn * sn * f1 + cs * cs * f2;
  }
}

__global__ __launch_bounds__(256) void k_fill_eye(long nn, int n, double* __restrict__ X, double* __restrict__ Dih) {
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i >= nn) return;
  const int r = (int)(i / n), c = (int)(i - (long)r * n);
  X[i] = r == c ? 1.0 : 0.0;
  Dih[i] = 0.0;
}

// Column step k of X = L^-1: X[i][j] -= L[i][k] X[k][j] for i > k, j <= k.
__global__ __launch_bounds__(256) void k_linv(int n, int k, const double* __restrict__ L, double* __restrict__ X) {
  const long m = n - k - 1, w = k + 1, mm = m * w;
  for (long e = (long)blockIdx.x * 256 + threadIdx.x; e < mm; e += (long)gridDim.x * 256) {
    const int i = k + 1 + (int)(e / w), j = (int)(e - (e / w) * w);
    X[(long)i * n + j] -= L[(long)i * n + k] * X[(long)k * n + j];
  }
}

// M^T[perm[i]][k] = sum_r Dih[k][r] X[r][i] (Dih block diagonal: r in k's block).
__global__ __launch_bounds__(256) void k_compose(int n, const double* __restrict__ Dih, const int* __restrict__ bsz,
                                                 const double* __restrict__ X, double* __restrict__ Mt) {
  const long e = (long)blockIdx.x * 256 + threadIdx.x;
  if (e >= (long)n * n) return;
  const int k = (int)(e / n), i = (int)(e - (long)k * n);
  double v = Dih[(long)k * n + k] * X[(long)k * n + i];
  if (k + 1 < n && bsz[k] == 2) v += Dih[(long)k * n + k + 1] * X[(long)(k + 1) * n + i];
  if (k > 0 && bsz[k] == 0) v += Dih[(long)k * n + k - 1] * X[(long)(k - 1) * n + i];
  Mt[(long)i * n + k] = v;
}

// ---- the factorisation in one cooperative launch -----------------------------
// Workgroup 0 decides every step; the others hold A, a row's n elements in the
// registers of their 512 threads (thread t has columns t, t + 512, ...), and
// keep it up to date.  Rows and columns stay where they are: an interchange only
// exchanges the positions that every thread keeps of its own columns (and every
// workgroup of its rows), and ties are broken by position.
//   - At the start of a panel of 8 to 16 positions the row holders publish the
//     panel's columns (P); workgroup 0 takes them into registers, a row per
//     thread, and takes the panel's steps alone: the maximum over the column, the
//     pivot test, the L entries, and the update of the columns left in the panel.
//     A step costs it one workgroup barrier and no exchange.
//   - Each step's pivot column goes out as W[k], the kind of step as M1[k].  The
//     row holders take the steps of a panel two at a time as they appear, form
//     their rows' L entries from W and update their rows: rank-one updates in the
//     order of the steps, as a step at a time would do them.
//   - Where the first pivot test fails, M1[k] asks for column imax (CI) and row
//     imax (RI); the row holders, which have all earlier steps applied, answer;
//     M2[k] tells them the decision.
// Data pass between workgroups through single-write slots: each is filled
// beforehand with a signalling-NaN pattern that no arithmetic result takes
// (arithmetic on NaNs yields quiet NaNs), written once with an agent-scope atomic
// store, and read by polling it with agent-scope atomic loads until it no longer
// holds that pattern.  Every wait is bounded; past the limit, or once another
// workgroup has flagged a timeout, a workgroup flags it and returns.
//
// What bounds it: the chain of n steps in workgroup 0 (barrier, two reductions, a
// division: 1.1 us at n = 1044) and one exchange to the row holders and back a
// panel (7 us).  1.8 ms at n = 1044 where no interchange is needed and 5 where
// most columns need the second test, 1.5 and 4.4 at n = 1020; with an exchange of
// each column between all workgroups at every step it was 4.2 and 6.8.  512
// threads: with 1024 the panel does not fit the registers above n = 1024, with 256
// it does not above 1280; panels of 16 where it fits.  Waves without rows left do
// no arithmetic.
constexpr unsigned long long kBkEmpty = 0x7FF4C0FFEE5E7F11ull;   // signalling NaN
constexpr int kBkThreads = 512, kBkWaves = kBkThreads / 64;
constexpr int kBkBatch = 2;    // steps the row holders take at once: 4 are 1 us later at a panel's end, 3 half
                               // of that (preparation at n = 1044: 3866, 3829, 3787 us with 4, 3, 2)
constexpr int kBkMaxN = 4 * kBkThreads;
// For rows of up to 512 U elements: the positions of a panel (U times that in
// doubles a thread) and the rows a workgroup holds, at most (n / 255 rounded up).
constexpr int bk_panel(int U) { return U > 3 ? 8 : (U > 2 ? 12 : 16); }
constexpr int bk_rows(int U) { return 2 * U + 1; }
inline int bk_u(int n) { return (n + kBkThreads - 1) / kBkThreads; }

struct BkcArgs {
  int n, G;                      // G workgroups: the deciding one and G - 1 row holders
  const double* Gm;              // [n][n] the metric
  double *Lr, *D;                // [n][n] out; row i of Lr: the L entries of row i of Gm
  int *perm, *bsz;               // [n] out (perm the identity, bsz zero-filled beforehand)
  double *P, *W, *CI, *RI;       // [n][n] slots, by position and row (P, W, CI) or column (RI) of Gm
  double *M1, *M2;               // [n] slots, by position
  int* err;
  long long spin;                // polls of one value before giving up; < 0: give up at once
};

__device__ __forceinline__ void bk_put(double* p, double v) {
  __hip_atomic_store((unsigned long long*)p, (unsigned long long)__double_as_longlong(v), __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void bk_put_word(double* p, unsigned long long v) {
  __hip_atomic_store((unsigned long long*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long bk_peek(const double* p) {
  return __hip_atomic_load((const unsigned long long*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Slot of a row of slots (uniform) and a byte offset in it.
__device__ __forceinline__ const double* bk_at(const double* row, unsigned bytes) {
  return (const double*)((const char*)row + bytes);
}
// Reads slots until none of those wanted is empty; the N of a thread (and those of
// its wave) are in flight together.  All lanes of a wave call it.
template <int N, class P, class Want>
__device__ __forceinline__ bool bk_take(unsigned long long (&x)[N], P slot, Want want, const int* err, long long spin) {
  if (spin < 0) return false;
  for (long long s = 0;; ++s) {
    bool missing = false;
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] = want(i) ? bk_peek(slot(i)) : 0;
#pragma unroll
    for (int i = 0; i < N; ++i) missing = missing || x[i] == kBkEmpty;
    if (!__any(missing)) return true;
    if (s >= spin || ((s & 15) == 15 && __hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0))
      return false;
    __builtin_amdgcn_s_sleep(1);
  }
}
__device__ __forceinline__ double bk_val(unsigned long long v) { return __longlong_as_double((long long)v); }
// a value that all lanes hold, for the scalar unit
__device__ __forceinline__ int bk_uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }
// M1: 1 = the step at k is 1x1 without an interchange, 2 + imax = column and row
// imax (a position) are wanted; M2: kstep + 4 kp
constexpr unsigned long long kBkPlain = 1;

// A barrier for data passed through the LDS: global stores in flight stay in
// flight (a slot says itself that it is written), where __syncthreads would wait
// the microsecond that they take.
__device__ __forceinline__ void bk_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
// Loads are done: on a rare path, so that the common one it joins need not wait.
__device__ __forceinline__ void bk_loads_done() { __builtin_amdgcn_s_waitcnt(0 | (7 << 4) | (15 << 8)); }

// Max of values >= 0, none a signalling NaN: over groups of 8 lanes, every lane
// getting it, and over the wave, lane 63 getting it.
__device__ __forceinline__ double bk_max2(double a, double b) {
  double r;
  asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
template <int kCtrl>
__device__ __forceinline__ double bk_dpp(double x) {
  const unsigned long long v = (unsigned long long)__double_as_longlong(x);
  const int lo = __builtin_amdgcn_mov_dpp((int)(unsigned)v, kCtrl, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(v >> 32), kCtrl, 0xF, 0xF, true);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
__device__ __forceinline__ double bk_max8(double x) {
  x = bk_max2(x, bk_dpp<0xB1>(x));          // quad_perm [1,0,3,2]
  x = bk_max2(x, bk_dpp<0x4E>(x));          // quad_perm [2,3,0,1]
  return bk_max2(x, bk_dpp<0x141>(x));      // row_half_mirror
}
__device__ __forceinline__ double bk_max64(double x) {
  x = bk_max8(x);
  x = bk_max2(x, bk_dpp<0x128>(x));        // row_ror:8
  x = bk_max2(x, bk_dpp<0x142>(x));        // row_bcast:15
  return bk_max2(x, bk_dpp<0x143>(x));     // row_bcast:31
}
// a b + c, the result in a register of its own: the columns of a panel move down
// by one at each step without copies
__device__ __forceinline__ double bk_fma(double a, double b, double c) {
  double r;
  asm("v_fma_f64 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}

template <int U>
struct BkPanelLds {
  static constexpr int NB = bk_panel(U);
  double red[2][kBkWaves], cand[2][NB];                 // by parity of the step
  double red2[kBkWaves], cand2[NB + 1], candq[NB + 1], arr;
  int redi[kBkWaves], fail;
};

// The inverse of a 2x2 block and the L entries of a row in its two columns, each
// product sum with one rounding less: the second product rounded, the first not.
struct BkBlock { double i00, i01, i11; };
__device__ __forceinline__ BkBlock bk_block(double e00, double e10, double e11) {
  const double det = fma(e00, e11, -(e10 * e10));
  return {e11 / det, -e10 / det, e00 / det};
}
__device__ __forceinline__ void bk_l2(const BkBlock& v, double x0, double x1, double& l0, double& l1) {
  l0 = fma(x0, v.i00, x1 * v.i01);
  l1 = fma(x0, v.i01, x1 * v.i11);
}

// Workgroup 0: thread t has rows t + 512 u; C[p][u] is the entry in the column at
// position k + p.
template <int U>
__device__ void bk_decide(const BkcArgs& a, BkPanelLds<U>& s) {
  constexpr int NB = bk_panel(U);
  const int n = a.n, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  int pos[U];
#pragma unroll
  for (int u = 0; u < U; ++u) pos[u] = tid + kBkThreads * u < n ? tid + kBkThreads * u : -1;
  auto at = [&](int u) { return 8u * (unsigned)(tid + kBkThreads * u); };   // byte offset of the row in a row of slots
  double C[NB][U];
  int k = 0, b = 0;
  if (tid == 0) s.fail = 0;
  bk_barrier();
  while (k < n) {
    const int kend = min(k + NB, n);
    bool ok = true;
#pragma unroll
    for (int h = 0; h < NB; h += NB / 2) {   // by halves, for the registers
      unsigned long long x[NB / 2 * U];
      ok = ok && bk_take(x, [&](int i) { return bk_at(a.P + (long)(k + h + i / U) * n, at(i % U)); },
                         [&](int i) { return k + h + i / U < kend && pos[i % U] >= k; }, a.err, a.spin);
#pragma unroll
      for (int i = 0; i < NB / 2 * U; ++i) C[h + i / U][i % U] = ok ? bk_val(x[i]) : 0.0;
    }
    if (!ok) s.fail = 1;
    bk_barrier();
    if (bk_uniform(s.fail)) {
      if (tid == 0) atomicExch(a.err, 1);
      return;
    }
    bk_loads_done();
    while (k < kend) {
      // colmax below the diagonal; NaNs are never chosen.  No wave reduces or
      // divides for rows it no longer has.
      bool act[U], any = false;
      {
        double cm = 0.0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
          act[u] = __any(pos[u] > k);
          any = any || act[u];
          if (act[u] && pos[u] > k) cm = fmax(cm, fabs(C[0][u]));
          if ((unsigned)(pos[u] - k) < NB) s.cand[b][pos[u] - k] = C[0][u];
        }
        if (any) cm = bk_max64(cm);
        if (lane == 63) s.red[b][wv] = cm;
      }
      bk_barrier();
      double cm = s.red[b][lane & (kBkWaves - 1)], d = s.cand[b][0];
      const double* cd = s.cand[b];
      double l[U];   // on its way while the maxima are compared
#pragma unroll
      for (int u = 0; u < U; ++u) l[u] = C[0][u] / d;
      cm = bk_max8(cm);
      const double absakk = fabs(d);
      int kstep = 1;
      if (bk_uniform(k + 1 < n && fmax(absakk, cm) != 0.0 && absakk < kAlpha * cm)) {
        // the first position of the maximum, its column and its row; rowmax over
        // row imax left of the diagonal and column imax below it
        int im = n;
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (pos[u] > k && fabs(C[0][u]) == cm) im = min(im, pos[u]);
        im = wave_min_int_dpp(im);
        if (lane == 0) s.redi[wv] = im;
        bk_barrier();
        im = s.redi[0];
#pragma unroll
        for (int i = 1; i < kBkWaves; ++i) im = min(im, s.redi[i]);
        im = bk_uniform(im);
        if (tid == 0) bk_put_word(a.M1 + k, 2 + (unsigned long long)im);
        unsigned long long x[2 * U];
        ok = bk_take(x, [&](int i) { return bk_at((i < U ? a.CI : a.RI) + (long)k * n, at(i % U)); },
                            [&](int i) { return pos[i % U] >= k; }, a.err, a.spin);
        if (!ok) s.fail = 1;
        bk_loads_done();
        double ci[U], rm = 0.0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
          ci[u] = bk_val(x[u]);
          const double ri = bk_val(x[U + u]);
          if (pos[u] >= k && pos[u] != im) rm = fmax(rm, fabs(pos[u] < im ? ri : ci[u]));
          if (pos[u] == im) s.arr = ri;
        }
        rm = bk_max64(rm);
        if (lane == 63) s.red2[wv] = rm;
        bk_barrier();
        if (bk_uniform(s.fail)) {
          if (tid == 0) atomicExch(a.err, 1);
          return;
        }
        rm = bk_max8(s.red2[lane & (kBkWaves - 1)]);
        int kp = im;
        if (absakk * rm >= kAlpha * cm * cm) kp = k;
        else if (!(fabs(s.arr) >= kAlpha * rm)) kstep = 2;
        kp = bk_uniform(kp);
        kstep = bk_uniform(kstep);
        if (tid == 0) bk_put_word(a.M2 + k, (unsigned long long)kstep + 4 * (unsigned long long)kp);
        // the interchange of positions kk and kp: the column that leaves kk goes
        // to kp, if kp is in the panel
        const int kk = k + kstep - 1;
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (kp != kk) {
#pragma unroll
            for (int p = 1; p < NB; ++p)
              if (p == kp - k) C[p][u] = kstep == 1 ? C[0][u] : C[1][u];
            if (kstep == 1) C[0][u] = ci[u];
            if (pos[u] == kk) pos[u] = kp;
            else if (pos[u] == kp) pos[u] = kk;
          }
          const int q = pos[u] - k;
          if (q >= 0 && q <= NB) {
            s.cand2[q] = C[0][u];
            s.candq[q] = ci[u];
          }
          act[u] = __any(q > 0);
        }
        bk_barrier();
        cd = s.cand2;
        d = cd[0];
        if (kstep == 1) {
#pragma unroll
          for (int u = 0; u < U; ++u) l[u] = C[0][u] / d;
        }
        if (kstep == 2) {
          const double e00 = d, e10 = cd[1], e11 = s.candq[1];
          const BkBlock inv = bk_block(e00, e10, e11);
          if (tid == 0) {
            a.D[(long)k * n + k] = e00;
            a.D[(long)k * n + k + 1] = e10;
            a.D[(long)(k + 1) * n + k] = e10;
            a.D[(long)(k + 1) * n + k + 1] = e11;
            a.bsz[k] = 2;
            a.bsz[k + 1] = 0;
          }
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const double x0 = C[0][u], x1 = ci[u];
            if (pos[u] >= k) {
              bk_put(a.W + (long)k * n + tid + kBkThreads * u, x0);
              bk_put(a.W + (long)(k + 1) * n + tid + kBkThreads * u, x1);
            }
            double l0, l1;
            bk_l2(inv, x0, x1, l0, l1);
#pragma unroll
            for (int p = 2; p < NB; ++p) {
              C[p - 2][u] = bk_fma(-l1, s.candq[p], bk_fma(-l0, cd[p], C[p][u]));
              asm volatile("" ::: "memory");   // or all of both columns is loaded ahead, into registers there are not
            }
          }
        }
      } else if (tid == 0) {
        bk_put_word(a.M1 + k, kBkPlain);
      }
      if (kstep == 1) {
        if (tid == 0) {
          a.D[(long)k * n + k] = d;
          a.bsz[k] = 1;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (pos[u] >= k) bk_put(a.W + (long)k * n + tid + kBkThreads * u, C[0][u]);
          l[u] = d != 0.0 ? -l[u] : -0.0;
        }
        // the pivot column's entries in the panel, four at a time for all rows
#pragma unroll
        for (int p0 = 0; p0 < NB; p0 += 4) {
          if (k + p0 >= kend) break;
          double e[4];
#pragma unroll
          for (int p = 0; p < 4; ++p) e[p] = cd[p0 + p];
#pragma unroll
          for (int u = 0; u < U; ++u)
            if (act[u]) {
#pragma unroll
              for (int p = 0; p < 4; ++p)
                if (p0 + p > 0) C[p0 + p - 1][u] = bk_fma(l[u], e[p], C[p0 + p][u]);
            }
        }
      }
      k += kstep;
      b ^= 1;
    }
  }
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (pos[u] >= 0) a.perm[pos[u]] = tid + kBkThreads * u;
}

template <int U>
struct BkRowsLds {
  static constexpr int R = bk_rows(U);
  double w[kBkBatch][R], l[kBkBatch][R], d[kBkBatch];   // pivot columns in the rows held here, L entries, pivots
  double e[3];                                          // a 2x2 block
  int rp[R], cnt, im, fail;                             // positions of the rows; the next steps
};

// A row holder: rows g + (G - 1) t in A[t][u], columns tid + 512 u.
template <int U>
__device__ void bk_rows_holder(const BkcArgs& a, BkRowsLds<U>& s) {
  constexpr int R = bk_rows(U), B = kBkBatch, NB = bk_panel(U);
  const int n = a.n, tid = threadIdx.x, Gw = a.G - 1, g = (int)blockIdx.x - 1;
  auto col = [&](int u) { return tid + kBkThreads * u; };
  int pos[U], own[U];   // position of the column; the row held here of the same index, or -1
  double A[R][U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    pos[u] = col(u) < n ? col(u) : -1;
    own[u] = col(u) < n && col(u) % Gw == g ? col(u) / Gw : -1;
#pragma unroll
    for (int t = 0; t < R; ++t) A[t][u] = g + Gw * t < n && col(u) < n ? a.Gm[(long)(g + Gw * t) * n + col(u)] : 0.0;
  }
  if (tid < R) s.rp[tid] = g + Gw * tid < n ? g + Gw * tid : -1;
  if (tid == 0) s.fail = 0;
  bk_barrier();
  auto failed = [&]() {
    const bool f = bk_uniform(s.fail) != 0;
    if (f && tid == 0) atomicExch(a.err, 1);
    return f;
  };
  // rows at or past position k, in the columns at positions k .. k + NB - 1
  auto publish = [&](int k) {
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (pos[u] >= k && pos[u] < k + NB) {
#pragma unroll
        for (int t = 0; t < R; ++t)
          if (s.rp[t] >= k) bk_put(a.P + (long)pos[u] * n + g + Gw * t, A[t][u]);
      }
  };
  publish(0);
  int k = 0, kend = min(NB, n);
  while (k < n) {
    // Wave 0 watches the words of the next steps, one a lane: cnt plain steps, and
    // imax where a step is none.  (All threads polling their own entries of W keep
    // the deciding workgroup's stores from the same few channels: 2 us a step.)
    if (tid < 64) {
      const int left = min(B, kend - k);
      unsigned long long m = 0;
      int c = 0;
      bool in = a.spin >= 0;
      for (long long i = 0; in; ++i) {
        m = tid < left ? bk_peek(a.M1 + k + tid) : kBkPlain;
        c = (int)__builtin_ctzll(~__ballot(m == kBkPlain) | (1ull << 63));
        const bool posted = c >= left || bk_uniform(__shfl(m != kBkEmpty, c));
        if (posted) break;
        if (i >= a.spin ||
            ((i & 15) == 15 && __hip_atomic_load(a.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0))
          in = false;
        __builtin_amdgcn_s_sleep(1);
      }
      c = min(c, left);
      if (tid == c) s.im = c < left ? (int)(m - 2) : -1;
      if (tid == 0) {
        s.cnt = c;
        if (!in) s.fail = 1;
      }
    }
    bk_barrier();
    if (failed()) return;
    const int cnt = bk_uniform(s.cnt), im = bk_uniform(s.im);
    unsigned long long x[B * U];
    bool ok = bk_take(x, [&](int i) { return bk_at(a.W + (long)(k + i / U) * n, 8u * (unsigned)col(i % U)); },
                            [&](int i) { return i / U < cnt && pos[i % U] >= k + i / U; }, a.err, a.spin);
    if (!ok) s.fail = 1;
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int q = 0; q < B; ++q) {
        if (q < cnt && own[u] >= 0) s.w[q][own[u]] = bk_val(x[q * U + u]);
        if (q < cnt && pos[u] == k + q) s.d[q] = bk_val(x[q * U + u]);
      }
    bk_barrier();
    if (failed()) return;
    if (cnt > 0) {
      if (tid < B * R) {
        const int q = tid / R, t = tid - q * R;
        double l = 0.0;
        if (q < cnt && s.rp[t] > k + q) {
          const double d = s.d[q];
          l = d != 0.0 ? s.w[q][t] / d : 0.0;
          a.Lr[(long)(g + Gw * t) * n + k + q] = l;
        }
        s.l[q][t] = l;
      }
      bk_barrier();
#pragma unroll
      for (int q = 0; q < B; ++q)
        if (q < cnt) {
#pragma unroll
          for (int t = 0; t < R; ++t)
#pragma unroll
            for (int u = 0; u < U; ++u) A[t][u] = fma(-s.l[q][t], bk_val(x[q * U + u]), A[t][u]);
        }
      k += cnt;
    }
    if (im >= 0) {
      // column and row imax, then the decision
#pragma unroll
      for (int t = 0; t < R; ++t)
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (pos[u] == im && s.rp[t] >= k) bk_put(a.CI + (long)k * n + g + Gw * t, A[t][u]);
          if (s.rp[t] == im && pos[u] >= k) bk_put(a.RI + (long)k * n + col(u), A[t][u]);
        }
      unsigned long long dec[1], y[2 * U];
      ok = bk_take(dec, [&](int) { return a.M2 + k; }, [](int) { return true; }, a.err, a.spin);
      const int kstep = bk_uniform((int)(dec[0] & 3)), kp = bk_uniform((int)(dec[0] >> 2)), kk = k + kstep - 1;
      ok = ok && bk_take(y, [&](int i) { return bk_at(a.W + (long)(k + i / U) * n, 8u * (unsigned)col(i % U)); },
                                [&](int i) { return i / U < kstep && pos[i % U] >= k; }, a.err, a.spin);
      if (!ok) s.fail = 1;
      bk_loads_done();
      bk_barrier();   // every thread has read the rows' positions and the last steps' L entries
      if (failed()) return;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (pos[u] == kk) pos[u] = kp;
        else if (pos[u] == kp) pos[u] = kk;
        if (own[u] >= 0) {
          s.w[0][own[u]] = bk_val(y[u]);
          s.w[1][own[u]] = bk_val(y[U + u]);
        }
        if (pos[u] == k) s.e[0] = bk_val(y[u]);
        if (pos[u] == k + 1) {
          s.e[1] = bk_val(y[u]);
          s.e[2] = bk_val(y[U + u]);
        }
      }
      if (tid < R) {
        const int r = s.rp[tid];
        s.rp[tid] = r == kk ? kp : (r == kp ? kk : r);
      }
      bk_barrier();
      if (tid < R) {
        const int t = tid;
        double l0 = 0.0, l1 = 0.0;
        double* Lt = a.Lr + (long)(g + Gw * t) * n + k;
        if (kstep == 1) {
          if (s.rp[t] > k) {
            const double d = s.e[0];
            l0 = d != 0.0 ? s.w[0][t] / d : 0.0;
            Lt[0] = l0;
          }
        } else {
          if (s.rp[t] == k + 1) Lt[0] = 0.0;   // L is I on the block
          if (s.rp[t] > k + 1) {
            bk_l2(bk_block(s.e[0], s.e[1], s.e[2]), s.w[0][t], s.w[1][t], l0, l1);
            Lt[0] = l0;
            Lt[1] = l1;
          }
        }
        s.l[0][t] = l0;
        s.l[1][t] = l1;
      }
      bk_barrier();
#pragma unroll
      for (int t = 0; t < R; ++t)
#pragma unroll
        for (int u = 0; u < U; ++u) {
          A[t][u] = fma(-s.l[0][t], bk_val(y[u]), A[t][u]);
          if (kstep == 2) A[t][u] = fma(-s.l[1][t], bk_val(y[U + u]), A[t][u]);
        }
      k += kstep;
    }
    if (k >= kend && k < n) {
      publish(k);
      kend = min(k + NB, n);
    }
  }
}

template <int U>
__global__ __launch_bounds__(kBkThreads) void k_bk_coop(BkcArgs a) {
  __shared__ BkPanelLds<U> sp;
  __shared__ BkRowsLds<U> sr;
  if (blockIdx.x == 0) bk_decide<U>(a, sp);
  else bk_rows_holder<U>(a, sr);
}

// L by positions: the rows' L entries, unit diagonal, zero above
__global__ __launch_bounds__(256) void k_bk_coop_l(int n, const double* __restrict__ Lr, const int* __restrict__ perm,
                                                   double* __restrict__ L) {
  const int i = blockIdx.x;
  const double* src = Lr + (long)perm[i] * n;
  for (int j = threadIdx.x; j < n; j += 256) L[(long)i * n + j] = j < i ? src[j] : (j == i ? 1.0 : 0.0);
}

__global__ void k_bk_coop_reset(unsigned long long* slots, long count, int* err) {
  for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < count; i += (long)gridDim.x * 256) slots[i] = kBkEmpty;
  if (blockIdx.x == 0 && threadIdx.x == 0) *err = 0;
}
// a timed-out factorisation leaves 1x1 blocks of NaN on the diagonal of D, so
// every slab of b comes out NaN, never silently wrong
__global__ void k_bk_coop_check(int n, const int* err, double* D, int* bsz) {
  if (*err == 0) return;
  for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) {
    D[(long)i * n + i] = __longlong_as_double(0x7FF8000000000000ll);
    bsz[i] = 1;
  }
}

// X = L^-1 by columns, one wave per column j: x_j = 1 and, for i > j in order,
// x_i = -sum_{j <= k < i} L[i][k] x_k (forward substitution on L x = e_j), lane t
// summing k = j + t, j + t + 64, ... and wave_sum_dpp the lanes.  x stays in
// registers: the blocks of 64 that are complete in xr, the one under way in xc.
// The W waves of a workgroup take adjacent columns and share kLinvStage rows of L
// at a time through the LDS, the loads of the next two stages in flight meanwhile.  The sums
// over the complete blocks need none of the stage's own x and go first, so a row's
// chain is one multiply-add, the wave's sum and the insertion.
// What bounds it: that chain, n rows long for the first column, and the LDS reads
// beside it: 410 us at n = 1044; a row at a time with x in the LDS and a barrier
// each it was 894.
constexpr int kLinvMaxN = 2048, kLinvStage = 4, kLinvBlocks = kLinvMaxN / 64, kLinvPad = 256;
inline size_t linv_lds(int n) { return (size_t)2 * kLinvStage * (n + kLinvPad) * sizeof(double); }
template <int W>
__global__ __launch_bounds__(64 * W) void k_linv_rows(int n, const double* __restrict__ L, double* __restrict__ X) {
  extern __shared__ double sh[];
  constexpr int S = kLinvStage, NT = 64 * W, V = W * 256 / NT;   // V: elements a thread loads of a row, n <= 256 W
  const int NP = n + kLinvPad;   // the last block's group of four reads past the row; what it reads is zero
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, j0 = blockIdx.x * W, j = j0 + w;
  for (int k = tid; k < 2 * S * NP; k += NT) sh[k] = 0.0;
  double pa[S][V], pb[S][V];   // the rows of the next two stages, on their way
  // rows ib .. up to their last chunk of NT left of the diagonal; past the diagonal
  // a row meets x = 0, left of j0 it is not read
  auto fetch = [&](double (&pre)[S][V], int ib) {
#pragma unroll
    for (int v = 0; v < V; ++v)
      if (NT * v < ib + S && NT * v < n) {
        const int k = min(tid + NT * v, n - 1);
#pragma unroll
        for (int r = 0; r < S; ++r) pre[r][v] = L[(long)min(ib + r, n - 1) * n + k];
      }
  };
  auto store = [&](const double (&pre)[S][V], int ib, double* buf) {
#pragma unroll
    for (int v = 0; v < V; ++v)
      if (NT * v < ib + S && tid + NT * v < n) {
#pragma unroll
        for (int r = 0; r < S; ++r) buf[r * NP + tid + NT * v] = pre[r][v];
      }
  };
  fetch(pa, j0 + 1);
  fetch(pb, j0 + 1 + S);
  __syncthreads();
  store(pa, j0 + 1, sh);
  __syncthreads();
  double xr[kLinvBlocks], xc = lane == 0 ? 1.0 : 0.0;
#pragma unroll
  for (int u = 0; u < kLinvBlocks; ++u) xr[u] = 0.0;
  int ub = 0;
  // rows ib .. from one buffer; the next stage's go from next to the other, and
  // the loads of the one after it start
  auto stage = [&](int ib, const double* cur, double* other, double (&next)[S][V], double (&after)[S][V]) {
    fetch(after, ib + 2 * S);
    const double* row = cur + j + lane;
    if (j < n && ib + S - 1 > j) {
      double s[S], c[S];
#pragma unroll
      for (int r = 0; r < S; ++r) {
        s[r] = 0.0;
        c[r] = row[r * NP + 64 * ub];
      }
#pragma unroll
      for (int u = 0; u < kLinvBlocks; u += 4) {
        if (u >= ub) break;
#pragma unroll
        for (int v = u; v < u + 4; ++v)
#pragma unroll
          for (int r = 0; r < S; ++r) s[r] = fma(row[r * NP + 64 * v], xr[v], s[r]);
      }
#pragma unroll
      for (int r = 0; r < S; ++r) {
        const int i = ib + r;
        if (i <= j || i >= n) continue;
        const double x = -wave_sum_dpp(fma(c[r], xc, s[r]));
        if (((i - j) & 63) == 0) {   // the block is complete: the rows left here take it before the next
#pragma unroll
          for (int u = 0; u < kLinvBlocks; ++u) xr[u] = u == ub ? xc : xr[u];
          ++ub;
#pragma unroll
          for (int q = r + 1; q < S; ++q) {
            s[q] = fma(c[q], xc, s[q]);
            c[q] = row[q * NP + 64 * ub];
          }
          xc = 0.0;
        }
        if (lane == ((i - j) & 63)) xc = x;
      }
    }
    store(next, ib + S, other);
    bk_barrier();
  };
  double* const buf1 = sh + (long)S * NP;
  for (int ib = j0 + 1; ib < n; ib += 2 * S) {
    stage(ib, sh, buf1, pb, pa);
    if (ib + S < n) stage(ib + S, buf1, sh, pa, pb);
  }
  // columns j0 .. j0 + W - 1 of X, W adjacent doubles per row
  if (j < n) {
    double* xs = sh + (long)w * n;
    for (int k = lane; k < j; k += 64) xs[k] = 0.0;
#pragma unroll
    for (int u = 0; u < kLinvBlocks; ++u) {
      const int i = j + lane + 64 * u;
      if (i < n) xs[i] = u == ub ? xc : xr[u];
    }
  }
  __syncthreads();
  for (int y = tid; y < W * n; y += NT) {
    const int i = y / W, c = y % W;
    if (j0 + c < n) X[(long)i * n + j0 + c] = sh[(long)c * n + i];
  }
}

// ---- the solve ---------------------------------------------------------------
// b[k] = sum_i M'[k][i] T[perm[i]], a product over i whose columns are the pairs
// (mu, nu): T and b are symmetric in them, so 8 x 16 blocks (mu x nu) with an
// element on or above the diagonal are computed and stored both ways.  Rows k run in
// tiles of up to 128 on the strip loop; a tile stops at the k past which its rows
// of M' are zero.  An LDS load of the loop holds one row i of the 128 columns, so
// the pivot order is a scalar base per load and T is read where it lies.
//
// What bounds it: the matrix cores (n_aux^2 x 128 flops a block).  Before, T was
// packed in pivot order (240 us at n_bf 348, n_aux 1044), multiplied (1690) and the
// packed result spread over b (430): 1570 us in one pass here, at 74% of
// the cycles in matrix instructions.
struct SolveArgs {
  int n, nb;
  const double* Mt;   // [n][n] M'^T
  const double* T;    // [n][nb][nb]
  const int* perm;
  double* b;          // [n][nb][nb]
  int rows, nrt;      // rows k a tile (multiple of 16), row tiles
  long nblk;          // column blocks
};
using SolveCfg = StripCfg<128, 8>;
constexpr int kSolveMu = 8, kSolveNu = 16;   // (the blocks of block_offset)

// Column blocks by strips of 8 mu: strip r has the nu blocks from that of 8 r on.
__host__ __device__ __forceinline__ int solve_cols(int nb) { return (pair_len(nb) + kSolveNu - 1) / kSolveNu; }
__host__ __device__ __forceinline__ long solve_blocks(int nb) {
  const int nr = (nb + kSolveMu - 1) / kSolveMu, nc = solve_cols(nb);
  long s = 0;
  for (int r = 0; r < nr; ++r) s += nc - r / 2;
  return s;
}

template <class L>
struct SolveStage {
  StripStage<L> st;   // its A loads; the B loads' bases are set here
  const double* T;
  const int* perm;
  long slab;
  int n;
  int p, next;   // perm of the 64 rows under way and the next 64, one a lane
  // rows past n: replaced by zeros in st.issue
  __device__ __forceinline__ int rows64(int k0) const { return perm[min(k0 + (int)(threadIdx.x & 63), n - 1)]; }
  __device__ __forceinline__ void issue(lds_char* dst, int kt) {   // called for kt = 0, 1, 2, ...
    if (kt % 4 == 0) {
      p = next;
      next = rows64(16 * kt + 64);
    }
#pragma unroll
    for (int i = 0; i < L::NU; ++i) {
      const int u = st.w + i * L::NW;
      if (u >= L::NIA && st.have(i))
        st.base[i] = (const char*)(T + slab * __builtin_amdgcn_readlane(p, kt % 4 * 16 + u - L::NIA));
    }
    st.issue(dst, n - 16 * kt);
  }
};

__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4))) void k_prep_solve(SolveArgs a) {
  __shared__ __attribute__((aligned(16))) char smem[strip_smem<SolveCfg>()];
  const int n = a.n, nb = a.nb;
  // the longest row tiles first: the tiles in flight share their rows of M', and
  // the short ones fill the end
  long blk = blockIdx.x % a.nblk;
  const int rt = a.nrt - 1 - (int)(blockIdx.x / a.nblk);
  int r = 0;
  const int nc = solve_cols(nb);
  {
    // strips 2 j and 2 j + 1 have nc - j blocks each
    long rem = blk;
    int j = 0;
    while (rem >= 2l * (nc - j)) rem -= 2l * (nc - j++);
    r = 2 * j;
    if (rem >= nc - j) { rem -= nc - j; ++r; }
    blk = rem + j;
  }
  const int mu0 = r * kSolveMu, nu0 = (int)blk * kSolveNu, m0 = rt * a.rows;
  const int plen = pair_len(n), ncol = pair_len(nb);
  const int tm = (min(a.rows, plen - m0) + 15) / 16;
  with_frags(tm, [&](auto frags) {
    using L = Strip<SolveCfg, decltype(frags)::value>;
    SolveStage<L> ld;
    ld.T = a.T + (long)mu0 * nb;   // (a slab may pass 2^32 bytes, a lane's offset from the block's first row not)
    ld.perm = a.perm;
    ld.slab = (long)nb * nb;
    ld.n = n;
    ld.next = ld.rows64(0);
    ld.st.init(
        a.Mt, n, [&](int x) -> long { return pair_start(min(m0 + x, plen - 2), n); }, a.T, 0,
        [&](int x) { return block_offset(x, mu0, nu0, nb); });
    StripAcc<L> acc;
    // M' is zero right of its first superdiagonal
    const int K = min(n, m0 + L::BM + 1);
    strip_mainloop<L>((K + 15) / 16, ld.st.w, acc, smem, [&](int kt, lds_char* dst) { ld.issue(dst, kt); });
    // b[k][mu][nu] from the registers, b[k][nu][mu] through the LDS, a row of
    // fragments at a time: 8 mu of a nu lie together
    const int lane = threadIdx.x & 63;
    double* sh = (double*)smem;
    constexpr int RI = 16 * L::WVM, MS = kSolveNu + 1, RS = kSolveMu * MS;
    static_assert(RI * RS * 8 <= strip_smem<SolveCfg>(), "LDS of the transposition");
#pragma unroll
    for (int i = 0; i < L::FM; ++i) {
      const int mrow = acc.wm + 16 * i, g = L::WVM == 2 && acc.wm ? 16 : 0;
#pragma unroll
      for (int j = 0; j < L::FN; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int q = (lane >> 4) + 4 * e, x = acc.wn + 16 * j + (lane & 15);
          const int k = m0 + mrow + q < plen ? pair_column(m0 + mrow + q, n) : -1;
          const int mu = mu0 + x / kSolveNu, nu = nu0 + x % kSolveNu < ncol ? pair_column(nu0 + x % kSolveNu, nb) : -1;
          if (k >= 0 && mu < nb && nu >= mu) a.b[((long)k * nb + mu) * nb + nu] = acc.v[i][j][e];
          sh[(g + q) * RS + x / kSolveNu * MS + x % kSolveNu] = acc.v[i][j][e];
        }
      __syncthreads();
      for (int y = threadIdx.x; y < RI * 128; y += SolveCfg::NT) {
        const int q = y >> 7, nup = (y >> 3) & 15, mu = mu0 + (y & 7);
        const int m = m0 + (q >= 16 ? L::FM * 16 : 0) + 16 * i + (q & 15);
        const int k = m < plen ? pair_column(m, n) : -1, nu = nu0 + nup < ncol ? pair_column(nu0 + nup, nb) : -1;
        if (k >= 0 && mu < nb && nu > mu) a.b[((long)k * nb + nu) * nb + mu] = sh[q * RS + (y & 7) * MS + nup];
      }
      __syncthreads();
    }
  });
}

// A single pair or a single function, which the loads by pairs do not take.
__global__ __launch_bounds__(256) void k_prep_solve_small(int n, long npair, const double* __restrict__ Mt,
                                                          const double* __restrict__ T, const int* __restrict__ perm,
                                                          double* __restrict__ b) {
  const long e = (long)blockIdx.x * 256 + threadIdx.x;
  if (e >= n * npair) return;
  const long k = e / npair, x = e - k * npair;
  double s = 0.0;
  for (int i = 0; i < n; ++i) s = fma(Mt[(long)i * n + k], T[perm[i] * npair + x], s);
  b[e] = s;
}

rif_status op_prepare_b(rif_ctx* c, int nb, int na, const double* T, const double* Gm, double delta,
                        double* b, int* perm_out, double* L_out, double* D_out, int* nraised_out) {
  const int n = na;
  const long nn = (long)n * n;
  Carve cv;
  const size_t oA = cv.take<double>(nn), oL = cv.take<double>(nn), oD = cv.take<double>(nn);
  const size_t oX = cv.take<double>(nn), oM = cv.take<double>(nn), oDih = cv.take<double>(nn);
  const size_t oP = cv.take<int>(n), oB = cv.take<int>(n), oS = cv.take<BkState>(1);
  const size_t oPart = cv.take<double>((size_t)n), oDel = cv.take<double>(1);
  const size_t oR = cv.take<int>(1);
  // the one-launch factorisation where a row fits four elements a thread, the rows
  // the registers of one workgroup per CU and its slots the arena, else a pivot and an
  // update launch per column
  int G = 0;
  if (n <= kBkMaxN) {
    int ncu = 0, coop = 0;
    if (hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, c->device) == hipSuccess &&
        hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, c->device) == hipSuccess && coop) {
      G = std::min({ncu, n + 1, 256});
      if (G < 2 || (n + G - 2) / (G - 1) > bk_rows(bk_u(n))) G = 0;
    }
    (void)hipGetLastError();
  }
  const long nslots = 4 * nn + 2 * n;
  const size_t columns = cv.off;
  const size_t oSlots = G ? cv.take<double>((size_t)nslots) : 0, oErr = G ? cv.take<int>(1) : 0;
  bool roomy = false;
  rif_status st = ws_reserve_either(c, cv.off, columns, &roomy);
  if (st) return st;
  if (!roomy) G = 0;
  char* w = (char*)c->ws;
  double *A = (double*)(w + oA), *L = (double*)(w + oL), *D = (double*)(w + oD), *X = (double*)(w + oX);
  double *Mt = (double*)(w + oM), *Dih = (double*)(w + oDih), *part = (double*)(w + oPart);
  double* del = (double*)(w + oDel);
  int *perm = (int*)(w + oP), *bsz = (int*)(w + oB), *nr = (int*)(w + oR);
  BkState* sp = (BkState*)(w + oS);
  const unsigned gnn = (unsigned)((nn + 255) / 256);
  {
    ProfScope ps(c, "prep_factorise");
    hipLaunchKernelGGL(k_rowsum, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, c->stream, n, Gm, part);
    // max over the row sums, times sqrt(2^-52), into del
    hipLaunchKernelGGL(k_delta, dim3(1), dim3(256), 0, c->stream, n, part, del);
    hipLaunchKernelGGL(k_bk_init, dim3(gnn), dim3(256), 0, c->stream, n, Gm, A, L, D, perm, bsz, sp);
    if ((st = check_launch(c, "prep_init"))) return st;
    if (G) {
      BkcArgs ba{};
      ba.n = n;
      ba.G = G;
      ba.Gm = Gm;
      ba.Lr = A;
      ba.D = D;
      ba.perm = perm;
      ba.bsz = bsz;
      double* sl = (double*)(w + oSlots);
      ba.P = sl;
      ba.W = sl + nn;
      ba.CI = sl + 2 * nn;
      ba.RI = sl + 3 * nn;
      ba.M1 = sl + 4 * nn;
      ba.M2 = ba.M1 + n;
      ba.err = (int*)(w + oErr);
      ba.spin = c->wait_limit;
      hipLaunchKernelGGL(k_bk_coop_reset, dim3((unsigned)std::min(4096L, (nslots + 255) / 256)), dim3(256), 0,
                         c->stream, (unsigned long long*)sl, nslots, ba.err);
      if ((st = check_launch(c, "prep_factorise_reset"))) return st;
      void* args[] = {&ba};
      const void* fns[] = {(const void*)k_bk_coop<1>, (const void*)k_bk_coop<2>, (const void*)k_bk_coop<3>,
                           (const void*)k_bk_coop<4>};
      const void* fn = fns[bk_u(n) - 1];
      const hipError_t he = hipLaunchCooperativeKernel(fn, dim3(G), dim3(kBkThreads), args, 0, c->stream);
      if (he != hipSuccess) {
        (void)hipGetLastError();
        return fail(c, RIF_EHIP, std::string("cooperative launch of the factorisation failed: ") +
                                     hipGetErrorString(he));
      }
      hipLaunchKernelGGL(k_bk_coop_check, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, c->stream, n,
                         (const int*)ba.err, D, bsz);
      hipLaunchKernelGGL(k_bk_coop_l, dim3((unsigned)n), dim3(256), 0, c->stream, n, (const double*)A,
                         (const int*)perm, L);
    } else {
      const unsigned gup = (unsigned)std::min(1024L, (nn + 255) / 256);
      for (int it = 0; it < n; ++it) {
        hipLaunchKernelGGL(k_bk_pivot, dim3(1), dim3(kPivThreads), 0, c->stream, n, A, L, D, perm, bsz, sp);
        hipLaunchKernelGGL(k_bk_update, dim3(gup), dim3(256), 0, c->stream, n, A, L, (const BkState*)sp);
      }
    }
    if ((st = check_launch(c, "prep_factorise"))) return st;
  }
  {
    ProfScope ps(c, "prep_correct_invert");
    hipLaunchKernelGGL(k_fill_eye, dim3(gnn), dim3(256), 0, c->stream, nn, n, X, Dih);
    if (hipMemsetAsync(nr, 0, sizeof(int), c->stream) != hipSuccess) return fail(c, RIF_EHIP, "hipMemsetAsync failed");
    hipLaunchKernelGGL(k_bk_correct, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, c->stream, n, D, bsz, del,
                       delta, Dih, nr);
    if (n <= kLinvMaxN) {
      // four columns a workgroup while that fills no more than the 256 CUs
      const bool four = n <= 1024;
      const void* fn = four ? (const void*)k_linv_rows<4> : (const void*)k_linv_rows<8>;
      const size_t lds = linv_lds(n);
      if (lds > 64 * 1024 &&
          hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess) {
        (void)hipGetLastError();
        return fail(c, RIF_EHIP, "L^-1: LDS attribute failed");
      }
      if (four) hipLaunchKernelGGL(k_linv_rows<4>, dim3((unsigned)((n + 3) / 4)), dim3(256), lds, c->stream, n, L, X);
      else hipLaunchKernelGGL(k_linv_rows<8>, dim3((unsigned)((n + 7) / 8)), dim3(512), lds, c->stream, n, L, X);
    } else {
      for (int k = 0; k + 1 < n; ++k) {
        const long work = (long)(n - k - 1) * (k + 1);
        const unsigned g = (unsigned)std::max(1L, std::min(1024L, (work + 255) / 256));
        hipLaunchKernelGGL(k_linv, dim3(g), dim3(256), 0, c->stream, n, k, L, X);
      }
    }
    hipLaunchKernelGGL(k_compose, dim3(gnn), dim3(256), 0, c->stream, n, Dih, bsz, X, Mt);
    if ((st = check_launch(c, "prep_correct_invert"))) return st;
  }
  {
    ProfScope ps(c, "prep_solve_gemm");
    if (n < 2 || nb < 2) {
      const long ne = (long)n * nb * nb;
      hipLaunchKernelGGL(k_prep_solve_small, dim3((unsigned)((ne + 255) / 256)), dim3(256), 0, c->stream, n,
                         (long)nb * nb, (const double*)Mt, T, (const int*)perm, b);
    } else {
      SolveArgs sa{};
      sa.n = n;
      sa.nb = nb;
      sa.Mt = Mt;
      sa.T = T;
      sa.perm = perm;
      sa.b = b;
      sa.nblk = solve_blocks(nb);
      // 128 rows a tile; 64 where that leaves CUs without their two workgroups
      sa.rows = sa.nblk * ((n + 127) / 128) >= 512 ? 128 : 64;
      sa.nrt = (pair_len(n) + sa.rows - 1) / sa.rows;
      hipLaunchKernelGGL(k_prep_solve, dim3((unsigned)(sa.nblk * sa.nrt)), dim3(SolveCfg::NT), 0, c->stream, sa);
    }
    if ((st = check_launch(c, "prep_solve"))) return st;
  }
  if (perm_out && hipMemcpyAsync(perm_out, perm, sizeof(int) * n, hipMemcpyDeviceToDevice, c->stream) != hipSuccess)
    return fail(c, RIF_EHIP, "copying perm failed");
  if (L_out && hipMemcpyAsync(L_out, L, sizeof(double) * nn, hipMemcpyDeviceToDevice, c->stream) != hipSuccess)
    return fail(c, RIF_EHIP, "copying L failed");
  if (D_out && hipMemcpyAsync(D_out, D, sizeof(double) * nn, hipMemcpyDeviceToDevice, c->stream) != hipSuccess)
    return fail(c, RIF_EHIP, "copying D failed");
  if (nraised_out && hipMemcpyAsync(nraised_out, nr, sizeof(int), hipMemcpyDeviceToDevice, c->stream) != hipSuccess)
    return fail(c, RIF_EHIP, "copying the correction count failed");
  return RIF_OK;
}

}  // namespace rif
