// Occupation-number optimisation at fixed orbitals and the learned warm start.
//
// The paper's occupancy optimisation (Sec. II) minimises Eq. (2) over the ONs
// with J, K fixed, through auxiliary variables gamma that keep the bounds and
// the pair normalisation.  Parametrisation used here, per pair g with ncwo weak
// orbitals (ascending index):
//   n_g = (1 + cos^2 gamma_g)/2,   n_{w_k} = (1 - n_g) w_k,
//   w_1 = cos^2 b_1, w_k = prod_{j<k} sin^2 b_j cos^2 b_k, w_last = prod sin^2 b_j,
//   variables [gamma_g, b_1 .. b_{ncwo-1}] at g*ncwo + j.
//
//   k_on_opt      one workgroup per problem runs L-BFGS (history 8, backtracking
//                 with Armijo or, within rounding noise, approximate Wolfe) to max|dE/dgamma| <= tol, all in FP64 with
//                 fixed-order reductions.
//   k_on_feat     per-pair features (39) and ON targets/masks for the MLP.
//   k_on_warm     MLP ON predictions -> starting gamma.
//   MLP           39 -> 128 -> 128 -> 128 -> 7 (tanh, masked softmax), FP32 on
//                 the FP32 MFMA engine: forward, backward, softmax/loss, Adam.
#include <math.h>

#include <algorithm>

#include "mfma_engine.hpp"
#include "rif_internal.hpp"
#include "wave.hpp"

namespace rif {

__host__ __device__ static inline int cdiv_i(long a, long b) { return (int)((a + b - 1) / b); }

constexpr int kHist = 8;        // L-BFGS history
constexpr int kOnThreads = 256;
constexpr int kKmax = 6;         // weak slots in the features
constexpr int kNin = 3 + 5 * kKmax + kKmax;   // 39
constexpr int kNhid = 128;
constexpr int kNout = 1 + kKmax;               // 7

__device__ __forceinline__ int on_pair(const int* pair_of, int p, int npairs, int ncwo) {
  if (pair_of) return pair_of[p];
  return p < npairs ? p : npairs - 1 - (p - npairs) / ncwo;
}

// Fixed-order sum over the 256 threads of a block; every thread gets the result.
__device__ double block_sum(double v, double* red) {
  const int t = threadIdx.x;
  __syncthreads();
  red[t] = v;
  __syncthreads();
  for (int s = kOnThreads / 2; s > 0; s >>= 1) {
    if (t < s) red[t] += red[t + s];
    __syncthreads();
  }
  const double r = red[0];
  __syncthreads();
  return r;
}
__device__ double block_max(double v, double* red) {
  const int t = threadIdx.x;
  __syncthreads();
  red[t] = v;
  __syncthreads();
  for (int s = kOnThreads / 2; s > 0; s >>= 1) {
    if (t < s) red[t] = fmax(red[t], red[t + s]);
    __syncthreads();
  }
  const double r = red[0];
  __syncthreads();
  return r;
}

// Hyperspherical weights w[0..m-1] and their derivatives dw[k][j] = dw_k/db_j.
__device__ void weights(const double* beta, int m, double* w, double* dw /* [m][m-1] or null */) {
  double s = 1.0;
  for (int k = 0; k < m - 1; ++k) {
    const double c = cos(beta[k]);
    w[k] = s * c * c;
    const double sn = sin(beta[k]);
    s *= sn * sn;
  }
  w[m - 1] = s;
  if (!dw) return;
  for (int k = 0; k < m; ++k)
    for (int j = 0; j < m - 1; ++j) {
      double v = 0.0;
      if (k == m - 1 || j <= k) {
        v = 1.0;
        for (int i = 0; i < (k < m - 1 ? k : m - 1); ++i) {
          const double si = sin(beta[i]), ci = cos(beta[i]);
          v *= (i == j) ? 2.0 * si * ci : si * si;
        }
        if (k < m - 1) {
          const double sk = sin(beta[k]), ck = cos(beta[k]);
          v *= (j == k) ? -2.0 * ck * sk : ck * ck;
        }
      }
      dw[k * (m - 1) + j] = v;
    }
}

// Workspace of one problem, in doubles (the weak-orbital table follows as ints).
__host__ __device__ inline long on_ws_doubles(int nw, int npairs, int ncwo) {
  const long nv = (long)npairs * ncwo;
  return (2L * kHist + 5) * nv + 2L * nw + (npairs * (long)ncwo + 1) / 2 + 4;
}

struct OnView {
  int nw, npairs, ncwo, nv, functional;
  const double *Hpp, *J, *K;
  const int* pair_of;
  double *S, *Y, *x, *g, *d, *xn, *gn, *n, *dn;
  int* weak;
};

// Problems that k_on_opt_small takes
constexpr int kOnSmall = 128;
__host__ __device__ inline bool on_small(const OnProblem& P) { return P.n_omega <= kOnSmall; }

// E(x) and dE/dx for the problem; writes n, dn and gout.  Returns E.
__device__ double on_eval(const OnView& v, const double* x, double* gout, double* red) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // ONs from the variables
  for (int g = tid; g < v.npairs; g += kOnThreads) {
    const double* xg = x + (long)g * v.ncwo;
    const double c = cos(xg[0]);
    const double ng = 0.5 * (1.0 + c * c);
    v.n[g] = ng;
    double w[kKmax + 8];
    weights(xg + 1, v.ncwo, w, nullptr);
    for (int k = 0; k < v.ncwo; ++k) v.n[v.weak[g * v.ncwo + k]] = (1.0 - ng) * w[k];
  }
  __syncthreads();
  // dE/dn and the energy, one wave per row p, lanes over q
  double erow = 0.0;
  for (int p = wave; p < v.nw; p += kOnThreads / 64) {
    const double np = v.n[p];
    const int gp = on_pair(v.pair_of, p, v.npairs, v.ncwo);
    const double php = sqrt(np * (1.0 - np));
    const double dphp = (1.0 - 2.0 * np) / (2.0 * fmax(php, 1e-300));
    double e = 0.0, dsum = 0.0;
    for (int q = lane; q < v.nw; q += 64) {
      const double nq = v.n[q];
      const double Jpq = v.J[(long)p * v.nw + q], Kpq = v.K[(long)p * v.nw + q];
      const int gq = on_pair(v.pair_of, q, v.npairs, v.ncwo);
      if (gp == gq) {
        if (p == q) {
          e += np * Kpq;
        } else {
          const double sg = (p >= v.npairs && q >= v.npairs) ? 1.0 : -1.0;
          e += sg * sqrt(np * nq) * Kpq;
          dsum += 2.0 * sg * 0.5 * sqrt(nq / fmax(np, 1e-300)) * Kpq;
        }
      } else {
        const double phq = sqrt(nq * (1.0 - nq));
        double bb = -np * nq, db = -nq;
        if (v.functional == RIF_PNOF7) {
          bb -= php * phq;
          db -= dphp * phq;
        }
        e += 2.0 * np * nq * Jpq + bb * Kpq;
        dsum += 2.0 * (2.0 * nq * Jpq + db * Kpq);
      }
    }
    for (int off = 32; off > 0; off >>= 1) {
      e += __shfl_xor(e, off, 64);
      dsum += __shfl_xor(dsum, off, 64);
    }
    if (lane == 0) {
      v.dn[p] = 2.0 * v.Hpp[p] + v.K[(long)p * v.nw + p] + dsum;
      erow += 2.0 * np * v.Hpp[p] + e;
    }
  }
  const double E = block_sum(erow, red);  // includes the __syncthreads that publishes dn
  // chain rule to the variables, one thread per pair
  for (int g = tid; g < v.npairs; g += kOnThreads) {
    const double* xg = x + (long)g * v.ncwo;
    double* gg = gout + (long)g * v.ncwo;
    const double c = cos(xg[0]), s = sin(xg[0]);
    const double h = 0.5 * s * s, dh = c * s;
    double w[kKmax + 8], dw[(kKmax + 8) * (kKmax + 8)];
    weights(xg + 1, v.ncwo, w, dw);
    double t = -c * s * v.dn[g];
    for (int k = 0; k < v.ncwo; ++k) t += dh * w[k] * v.dn[v.weak[g * v.ncwo + k]];
    gg[0] = t;
    for (int j = 0; j < v.ncwo - 1; ++j) {
      double u = 0.0;
      for (int k = 0; k < v.ncwo; ++k) u += h * dw[k * (v.ncwo - 1) + j] * v.dn[v.weak[g * v.ncwo + k]];
      gg[1 + j] = u;
    }
  }
  __syncthreads();
  return E;
}

__device__ double dot(const double* a, const double* b, int n, double* red) {
  double s = 0.0;
  for (int i = threadIdx.x; i < n; i += kOnThreads) s += a[i] * b[i];
  return block_sum(s, red);
}

__global__ __launch_bounds__(kOnThreads) void k_on_opt(const OnProblem* __restrict__ probs) {
  __shared__ double red[kOnThreads];
  const OnProblem& P = probs[blockIdx.x];
  if (on_small(P)) return;
  const int tid = threadIdx.x;
  OnView v;
  v.nw = P.n_omega; v.npairs = P.n_pairs; v.ncwo = P.n_cwo; v.nv = P.n_pairs * P.n_cwo;
  v.functional = P.functional;
  v.Hpp = P.Hpp; v.J = P.J; v.K = P.K; v.pair_of = P.pair_of;
  double* w = P.work;
  const int nv = v.nv;
  v.S = w; w += (long)kHist * nv;
  v.Y = w; w += (long)kHist * nv;
  double rho[kHist], alpha[kHist];  // identical in every thread (block-reduced)
  v.x = w; w += nv;
  v.g = w; w += nv;
  v.d = w; w += nv;
  v.xn = w; w += nv;
  v.gn = w; w += nv;
  v.n = w; w += v.nw;
  v.dn = w; w += v.nw;
  v.weak = (int*)w;
  // weak-orbital table (ascending index); a bad map stops the problem
  __shared__ int bad;
  if (tid == 0) bad = 0;
  __syncthreads();
  for (int g = tid; g < v.npairs; g += kOnThreads) {
    int k = 0;
    for (int p = v.npairs; p < v.nw; ++p)
      if (on_pair(v.pair_of, p, v.npairs, v.ncwo) == g) {
        if (k < v.ncwo) v.weak[g * v.ncwo + k] = p;
        ++k;
      }
    if (k != v.ncwo || v.ncwo > kKmax + 8) atomicOr(&bad, 1);
  }
  for (int i = tid; i < nv; i += kOnThreads) v.x[i] = P.gamma[i];
  __syncthreads();
  if (bad) {
    if (tid == 0) { *P.status = 3; *P.iters = 0; }
    return;
  }
  double E = on_eval(v, v.x, v.g, red);
  int it = 0, hist = 0, head = 0, status = 1;
  while (true) {
    double gm = 0.0;
    for (int i = tid; i < nv; i += kOnThreads) gm = fmax(gm, fabs(v.g[i]));
    gm = block_max(gm, red);
    if (gm <= P.tol) { status = 0; break; }
    if (it >= P.max_it) { status = 1; break; }
    // two-loop recursion: d = -H g
    for (int i = tid; i < nv; i += kOnThreads) v.d[i] = v.g[i];
    __syncthreads();
    for (int j = 0; j < hist; ++j) {
      const int h = (head - 1 - j + kHist) % kHist;
      const double a = rho[h] * dot(v.S + (long)h * nv, v.d, nv, red);
      alpha[h] = a;
      for (int i = tid; i < nv; i += kOnThreads) v.d[i] -= a * v.Y[(long)h * nv + i];
      __syncthreads();
    }
    double scale;
    if (hist > 0) {
      const int h = (head - 1 + kHist) % kHist;
      scale = 1.0 / (rho[h] * dot(v.Y + (long)h * nv, v.Y + (long)h * nv, nv, red));
    } else {
      scale = fmin(1.0, 1.0 / gm);
    }
    for (int i = tid; i < nv; i += kOnThreads) v.d[i] *= scale;
    __syncthreads();
    for (int j = hist - 1; j >= 0; --j) {
      const int h = (head - 1 - j + kHist) % kHist;
      const double b = rho[h] * dot(v.Y + (long)h * nv, v.d, nv, red);
      const double a = alpha[h];
      for (int i = tid; i < nv; i += kOnThreads) v.d[i] += (a - b) * v.S[(long)h * nv + i];
      __syncthreads();
    }
    for (int i = tid; i < nv; i += kOnThreads) v.d[i] = -v.d[i];
    __syncthreads();
    double gd = dot(v.g, v.d, nv, red);
    if (!(gd < 0.0)) {  // not a descent direction: restart from steepest descent
      for (int i = tid; i < nv; i += kOnThreads) v.d[i] = -v.g[i] * fmin(1.0, 1.0 / gm);
      __syncthreads();
      hist = 0;
      gd = dot(v.g, v.d, nv, red);
    }
    // Backtracking with the Armijo test, or, once the energy change is below
    // its rounding noise, the approximate Wolfe conditions on the directional
    // derivative (Hager and Zhang, 2005): 0.9 phi'(0) <= phi'(a) <= -0.8 phi'(0).
    const double epsE = 1e-12 * fabs(E);
    double step = 1.0, En = 0.0;
    bool ok = false;
    for (int ls = 0; ls < 50; ++ls) {
      for (int i = tid; i < nv; i += kOnThreads) v.xn[i] = v.x[i] + step * v.d[i];
      __syncthreads();
      En = on_eval(v, v.xn, v.gn, red);
      if (En <= E + 1e-4 * step * gd) { ok = true; break; }
      if (En <= E + epsE) {
        const double gnd = dot(v.gn, v.d, nv, red);
        if (gnd >= 0.9 * gd && gnd <= -0.8 * gd) { ok = true; break; }
      }
      step *= 0.5;
    }
    if (!ok) { status = 2; break; }
    // history update (skipped without positive curvature)
    double sy = 0.0;
    for (int i = tid; i < nv; i += kOnThreads) {
      const double si = v.xn[i] - v.x[i], yi = v.gn[i] - v.g[i];
      v.S[(long)head * nv + i] = si;
      v.Y[(long)head * nv + i] = yi;
      sy += si * yi;
    }
    sy = block_sum(sy, red);
    if (sy > 1e-300) {
      rho[head] = 1.0 / sy;
      head = (head + 1) % kHist;
      hist = hist < kHist ? hist + 1 : kHist;
    }
    for (int i = tid; i < nv; i += kOnThreads) {
      v.x[i] = v.xn[i];
      v.g[i] = v.gn[i];
    }
    __syncthreads();
    E = En;
    ++it;
  }
  // outputs: the ONs of the final point (re-evaluated so n matches x)
  E = on_eval(v, v.x, v.g, red);
  for (int i = tid; i < nv; i += kOnThreads) P.gamma[i] = v.x[i];
  for (int p = tid; p < v.nw; p += kOnThreads) P.occ[p] = v.n[p];
  if (tid == 0) {
    *P.energy = E;
    *P.iters = it;
    *P.status = status;
  }
}

// ---- up to 128 orbitals in Omega ----------------------------------------------
// The same optimisation, every sum in the order of k_on_opt, with one problem in
// the registers and the LDS of eight waves:
//   - J and K stay in registers for the whole run (rows p = wave + 8 r, columns
//     lane and lane + 64);
//   - sines and cosines of the variables are taken once an evaluation, a variable
//     per thread, and so are the square roots and the quotient of a row and the
//     intra-pair terms, a pair of orbitals per thread;
//   - the row sums of eight rows are taken together (lane swaps halve the values
//     with each of the first two steps);
//   - L-BFGS runs in wave 0 with its vectors in registers, so that a scalar product
//     is six additions across the lanes and no barrier.
// What bounds it: the chain of an evaluation (six barriers) and of the recursion.
// k_on_opt takes a workgroup barrier for every step of every sum, and the sines and
// cosines of the derivatives again for each product: 2430 -> 600 us for 200
// problems of up to 112 orbitals.
constexpr int kOnSmallThreads = 512, kOnSmallWaves = kOnSmallThreads / 64;
constexpr int kOnRows = kOnSmall / kOnSmallWaves;

struct OnLds {
  double x[kOnSmall], cs[kOnSmall], sn[kOnSmall], w[kOnSmall], g[kOnSmall];
  double n[kOnSmall], ph[kOnSmall], dphp[kOnSmall], dn[kOnSmall], row[kOnSmall];
  double S[kHist][kOnSmall], Y[kHist][kOnSmall], rho[kHist];
  double te[kOnSmall * (kKmax + 9)], td[kOnSmall * (kKmax + 9)];   // intra-pair terms [p][member of p's pair]
  int weak[kOnSmall], pair[kOnSmall], slot[kOnSmall];
  int bad, odd, done;
};

// lane ^ 4: rows of 16 lanes moved up by 4 and down by 4, each where it applies
__device__ __forceinline__ int lane_xor4(int x) {
  const int up = __builtin_amdgcn_update_dpp(x, x, 0x104, 0xF, 0x5, false);      // row_shl:4 into banks 0, 2
  return __builtin_amdgcn_update_dpp(up, x, 0x114, 0xF, 0xA, false);             // row_shr:4 into banks 1, 3
}
// v + (v of lane ^ 8), then ^ 4, ^ 2, ^ 1
__device__ __forceinline__ double sum_in_row(double v) {
  v += dpp_move<0x128>(v);   // row_ror:8
  const long long u = __double_as_longlong(v);
  v += __longlong_as_double(((long long)lane_xor4((int)(u >> 32)) << 32) | (unsigned)lane_xor4((int)u));
  v += dpp_move<0x4E>(v);    // quad_perm [2,3,0,1]
  return v + dpp_move<0xB1>(v);
}
// a + (a of lane ^ kDist) in the lanes without the bit, b + ... in those with it
template <bool kHalves>
__device__ __forceinline__ double sum_two(double a, double b) {
  const long long u = __double_as_longlong(a), w = __double_as_longlong(b);
  const auto l = kHalves ? __builtin_amdgcn_permlane32_swap((unsigned)u, (unsigned)w, false, false)
                         : __builtin_amdgcn_permlane16_swap((unsigned)u, (unsigned)w, false, false);
  const auto h = kHalves ? __builtin_amdgcn_permlane32_swap((unsigned)(u >> 32), (unsigned)(w >> 32), false, false)
                         : __builtin_amdgcn_permlane16_swap((unsigned)(u >> 32), (unsigned)(w >> 32), false, false);
  return __longlong_as_double(((long long)h[0] << 32) | (unsigned)l[0]) +
         __longlong_as_double(((long long)h[1] << 32) | (unsigned)l[1]);
}
// The sum over the lanes in the order of block_sum's tree below 64: ^ 32, 16, 8, 4, 2, 1.
__device__ __forceinline__ double tree_sum(double v) {
  v = sum_two<true>(v, v);
  v = sum_two<false>(v, v);
  return sum_in_row(v);
}

// The factors of K_pq in e and dsum for q in p's pair
__device__ __forceinline__ void pair_term(int p, int q, int npairs, double np, double nq, double& te, double& td) {
  const double sg = (p >= npairs && q >= npairs) ? 1.0 : -1.0;
  te = p == q ? np : sg * sqrt(np * nq);
  td = p == q ? 0.0 : 2.0 * sg * 0.5 * sqrt(nq / fmax(np, 1e-300));
}

// A product that is rounded before it is added, as k_on_opt's compiled sums have it.
__device__ __forceinline__ double rounded_product(double a, double b) {
#pragma clang fp contract(off)
  return a * b;
}
// q's terms in p's row: those of another pair, and of p's own
__device__ __forceinline__ void other_terms(int functional, double np, double php, double dphp, double nq, double phq,
                                            double J, double K, double& e, double& ds) {
  double bb = -np * nq, db = -nq;
  if (functional == RIF_PNOF7) {
    bb = fma(-php, phq, bb);
    db = fma(-dphp, phq, db);
  }
  e += fma(2.0 * np * nq, J, rounded_product(bb, K));
  ds = fma(2.0, fma(2.0 * nq, J, rounded_product(db, K)), ds);
}
__device__ __forceinline__ void own_terms(double te, double td, double K, double& e, double& ds) {
  e += rounded_product(te, K);
  ds = fma(td, K, ds);
}

struct OnRegs {
  double J[kOnRows][2], K[kOnRows][2];
};

// dn and the energy rows at s.x, then the gradient in s.g; every thread gets E.
__device__ __forceinline__ double on_eval_small(const OnProblem& P, OnLds& s, const OnRegs& r) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int nw = P.n_omega, npairs = P.n_pairs, m = P.n_cwo, nv = npairs * m;
  if (tid < nv) s.cs[tid] = cos(s.x[tid]);
  else if (tid >= 256 && tid - 256 < nv) s.sn[tid - 256] = sin(s.x[tid - 256]);
  __syncthreads();
  if (tid < npairs) {
    const double* cs = s.cs + tid * m;
    const double* sn = s.sn + tid * m;
    const double ng = 0.5 * (1.0 + cs[0] * cs[0]);
    s.n[tid] = ng;
    double q = 1.0;
    for (int k = 0; k < m; ++k) {
      const double w = k < m - 1 ? q * cs[1 + k] * cs[1 + k] : q;
      s.w[tid * m + k] = w;
      s.n[s.weak[tid * m + k]] = (1.0 - ng) * w;
      if (k < m - 1) q *= sn[1 + k] * sn[1 + k];
    }
  }
  __syncthreads();
  if (tid < nw) {
    const double np = s.n[tid], ph = sqrt(np * (1.0 - np));
    s.ph[tid] = ph;
    s.dphp[tid] = (1.0 - 2.0 * np) / (2.0 * fmax(ph, 1e-300));
  }
  const bool odd = s.odd;   // a strong orbital outside its pair: the members are not the table's
  for (int t = tid; t < nw * (m + 1) && !odd; t += kOnSmallThreads) {
    const int p = t / (m + 1), j = t - p * (m + 1), gp = s.pair[p];
    const int q = j == 0 ? gp : s.weak[gp * m + j - 1];
    const double np = s.n[p], nq = s.n[q];
    pair_term(p, q, npairs, np, nq, s.te[t], s.td[t]);
  }
  __syncthreads();
  double nq[2], phq[2];
  int gq[2], sq[2];
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const int q = lane + 64 * c;
    nq[c] = q < nw ? s.n[q] : 0.0;
    phq[c] = q < nw ? s.ph[q] : 0.0;
    gq[c] = q < nw ? s.pair[q] : -1;
    sq[c] = q < nw ? s.slot[q] : 0;
  }
  if (odd) {
    for (int p = wave; p < nw; p += kOnSmallWaves) {
      const double np = s.n[p], php = s.ph[p], dphp = s.dphp[p];
      double e = 0.0, ds = 0.0;
      for (int c = 0; c < 2; ++c) {
        const int q = lane + 64 * c;
        if (q >= nw) continue;
        const double Jpq = P.J[(long)p * nw + q], Kpq = P.K[(long)p * nw + q];
        if (s.pair[p] == gq[c]) {
          double te, td;
          pair_term(p, q, npairs, np, nq[c], te, td);
          own_terms(te, td, Kpq, e, ds);
        } else {
          other_terms(P.functional, np, php, dphp, nq[c], phq[c], Jpq, Kpq, e, ds);
        }
      }
      e = tree_sum(e);
      ds = tree_sum(ds);
      if (lane == 0) {
        s.dn[p] = 2.0 * P.Hpp[p] + P.K[(long)p * nw + p] + ds;
        s.row[p] = 2.0 * np * P.Hpp[p] + e;
      }
    }
  }
#pragma unroll
  for (int r0 = 0; r0 < kOnRows; r0 += 8) {
    if (odd || wave + kOnSmallWaves * r0 >= nw) break;
    double e[8], ds[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int p = min(wave + kOnSmallWaves * (r0 + i), nw - 1), gp = s.pair[p];
      const double np = s.n[p], php = s.ph[p], dphp = s.dphp[p];
      e[i] = ds[i] = 0.0;
      asm volatile("" ::: "memory");   // no row's reads ahead of the last row's: the registers hold J and K
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const double Jpq = r.J[r0 + i][c], Kpq = r.K[r0 + i][c];
        const bool same = gp == gq[c];
        const int t = p * (m + 1) + (same ? sq[c] : 0);
        const double te = s.te[t], td = s.td[t];
        double eo = e[i], dso = ds[i], ei = e[i], di = ds[i];
        other_terms(P.functional, np, php, dphp, nq[c], phq[c], Jpq, Kpq, eo, dso);
        own_terms(te, td, Kpq, ei, di);
        if (gq[c] >= 0) {
          e[i] = same ? ei : eo;
          ds[i] = same ? di : dso;
        }
      }
    }
    // values 4 j + {0, 2, 1, 3} in the rows of 16 lanes of v[j]: e of rows 0 - 7, then ds
    double v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const double* src = j < 2 ? e + 4 * j : ds + 4 * (j - 2);
      v[j] = sum_in_row(sum_two<false>(sum_two<true>(src[0], src[1]), sum_two<true>(src[2], src[3])));
    }
    if ((lane & 15) == 0) {
      const int i = ((lane >> 4 & 1) << 1) | (lane >> 5);
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int p = wave + kOnSmallWaves * (r0 + 4 * j + i);
        if (p < nw) {
          const double Hp = P.Hpp[p];
          s.dn[p] = 2.0 * Hp + P.K[(long)p * nw + p] + v[2 + j];
          s.row[p] = 2.0 * s.n[p] * Hp + v[j];
        }
      }
    }
  }
  __syncthreads();
  // rows p = j, j + 4, ... in order for j = 0 .. 3, then (0 + 2) + (1 + 3)
  double E = 0.0;
  for (int p = lane & 3; p < nw; p += 4) E += s.row[p];
  E += dpp_move<0x4E>(E);
  E += dpp_move<0xB1>(E);
  if (tid < nv) {
    const int g = tid / m, j = tid - g * m;
    const double* cs = s.cs + g * m;
    const double* sn = s.sn + g * m;
    const double c = cs[0], si = sn[0];
    if (j == 0) {
      const double dh = c * si;
      double t = -c * si * s.dn[g];
      for (int k = 0; k < m; ++k) t += dh * s.w[g * m + k] * s.dn[s.weak[g * m + k]];
      s.g[tid] = t;
    } else {
      const double h = 0.5 * si * si;
      double u = 0.0;
      for (int k = 0; k < m; ++k) {
        double v = 0.0;
        if (k == m - 1 || j - 1 <= k) {
          v = 1.0;
          for (int i = 0; i < (k < m - 1 ? k : m - 1); ++i)
            v *= (i == j - 1) ? 2.0 * sn[1 + i] * cs[1 + i] : sn[1 + i] * sn[1 + i];
          if (k < m - 1) v *= (j - 1 == k) ? -2.0 * cs[1 + k] * sn[1 + k] : cs[1 + k] * cs[1 + k];
        }
        u += h * v * s.dn[s.weak[g * m + k]];
      }
      s.g[tid] = u;
    }
  }
  __syncthreads();
  return E;
}

__global__ __launch_bounds__(kOnSmallThreads) void k_on_opt_small(const OnProblem* __restrict__ probs) {
  __shared__ OnLds s;
  const OnProblem& P = probs[blockIdx.x];
  if (!on_small(P)) return;   // k_on_opt's
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int nw = P.n_omega, npairs = P.n_pairs, m = P.n_cwo, nv = npairs * m;
  if (tid == 0) s.bad = s.odd = s.done = 0;
  for (int i = tid; i < nv; i += kOnSmallThreads) s.weak[i] = 0;
  __syncthreads();
  for (int p = tid; p < nw; p += kOnSmallThreads) {
    const int g = on_pair(P.pair_of, p, npairs, m);
    s.pair[p] = g;
    s.slot[p] = 0;
    if (p < npairs && g != p) s.odd = 1;
  }
  __syncthreads();
  if (tid < npairs) {
    int k = 0;
    for (int p = npairs; p < nw; ++p)
      if (s.pair[p] == tid) {
        if (k < m) {
          s.weak[tid * m + k] = p;
          s.slot[p] = 1 + k;
        }
        ++k;
      }
    if (k != m) s.bad = 1;
  }
  if (tid < nv) s.x[tid] = P.gamma[tid];
  __syncthreads();
  if (s.bad) {
    if (tid == 0) { *P.status = 3; *P.iters = 0; }
    return;
  }
  OnRegs r;
#pragma unroll
  for (int i = 0; i < kOnRows; ++i)
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const int p = min(wave + kOnSmallWaves * i, nw - 1), q = min(lane + 64 * c, nw - 1);
      r.J[i][c] = P.J[(long)p * nw + q];
      r.K[i][c] = P.K[(long)p * nw + q];
    }
  // Wave 0 keeps the vectors, elements lane and lane + 64; the others only evaluate.
  double x[2], g[2], d[2], alpha[kHist];
  double E = 0.0, step = 1.0, gd = 0.0;
  int it = 0, hist = 0, head = 0, status = 1, ls = 0, stage = 0;   // stage: first point, line search, final point
#pragma unroll
  for (int c = 0; c < 2; ++c) x[c] = wave == 0 && lane + 64 * c < nv ? s.x[lane + 64 * c] : 0.0;
  auto dot = [&](const double (&a)[2], const double (&b)[2]) {
    double t[2];
#pragma unroll
    for (int c = 0; c < 2; ++c) t[c] = fma(a[c], b[c], 0.0);
    return tree_sum(t[0] + t[1]);
  };
  auto load = [&](const double* v, double (&out)[2]) {
#pragma unroll
    for (int c = 0; c < 2; ++c) out[c] = lane + 64 * c < nv ? v[lane + 64 * c] : 0.0;
  };
  while (true) {
    const double En = on_eval_small(P, s, r);
    if (wave == 0) {
      double xn[2], gn[2];
      load(s.x, xn);
      load(s.g, gn);
      bool top = stage == 0, stop = false;
      if (stage == 1) {
        const double epsE = 1e-12 * fabs(E);
        bool ok = En <= E + 1e-4 * step * gd;
        if (!ok && En <= E + epsE) {
          const double gnd = dot(gn, d);
          ok = gnd >= 0.9 * gd && gnd <= -0.8 * gd;
        }
        if (ok) {
          double sy[2], t[2];
#pragma unroll
          for (int c = 0; c < 2; ++c) {
            sy[c] = xn[c] - x[c];
            t[c] = gn[c] - g[c];
            if (lane + 64 * c < nv) {
              s.S[head][lane + 64 * c] = sy[c];
              s.Y[head][lane + 64 * c] = t[c];
            }
          }
          const double q = dot(sy, t);
          if (q > 1e-300) {
            s.rho[head] = 1.0 / q;   // every lane the same: what a lane reads it has written
            head = (head + 1) % kHist;
            hist = hist < kHist ? hist + 1 : kHist;
          }
          ++it;
          top = true;
        } else {
          step *= 0.5;
          if (++ls == 50) { status = 2; stop = true; }
        }
      }
      if (top) {
        E = En;
        double gm = 0.0;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          x[c] = xn[c];
          g[c] = gn[c];
          gm = fmax(gm, fabs(g[c]));
        }
        gm = wave_max_dpp(gm);
        if (gm <= P.tol) { status = 0; stop = true; }
        else if (it >= P.max_it) { status = 1; stop = true; }
        else {
          // two-loop recursion: d = -H g
#pragma unroll
          for (int c = 0; c < 2; ++c) d[c] = g[c];
#pragma unroll
          for (int j = 0; j < kHist; ++j)
            if (j < hist) {
              const int h = (head - 1 - j + kHist) % kHist;
              double S[2], Y[2];
              load(s.S[h], S);
              load(s.Y[h], Y);
              const double a = s.rho[h] * dot(S, d);
              alpha[j] = a;
#pragma unroll
              for (int c = 0; c < 2; ++c) d[c] -= a * Y[c];
            }
          double scale;
          if (hist > 0) {
            const int h = (head - 1 + kHist) % kHist;
            double Y[2];
            load(s.Y[h], Y);
            scale = 1.0 / (s.rho[h] * dot(Y, Y));
          } else {
            scale = fmin(1.0, 1.0 / gm);
          }
#pragma unroll
          for (int c = 0; c < 2; ++c) d[c] *= scale;
#pragma unroll
          for (int j = kHist - 1; j >= 0; --j)
            if (j < hist) {
              const int h = (head - 1 - j + kHist) % kHist;
              double S[2], Y[2];
              load(s.S[h], S);
              load(s.Y[h], Y);
              const double b = s.rho[h] * dot(Y, d), a = alpha[j];
#pragma unroll
              for (int c = 0; c < 2; ++c) d[c] += (a - b) * S[c];
            }
#pragma unroll
          for (int c = 0; c < 2; ++c) d[c] = -d[c];
          gd = dot(g, d);
          if (!(gd < 0.0)) {   // not a descent direction: restart from steepest descent
#pragma unroll
            for (int c = 0; c < 2; ++c) d[c] = -g[c] * fmin(1.0, 1.0 / gm);
            hist = 0;
            gd = dot(g, d);
          }
          step = 1.0;
          ls = 0;
          stage = 1;
        }
      }
      // the next point: along d, or the final one once more so that n matches x
#pragma unroll
      for (int c = 0; c < 2; ++c)
        if (lane + 64 * c < nv) s.x[lane + 64 * c] = stop ? x[c] : x[c] + step * d[c];
      if (stage == 2) {
        E = En;
        if (lane == 0) {
          s.done = 1;
          *P.energy = E;
          *P.iters = it;
          *P.status = status;
        }
#pragma unroll
        for (int c = 0; c < 2; ++c)
          if (lane + 64 * c < nv) P.gamma[lane + 64 * c] = x[c];
      }
      if (stop) stage = 2;
    }
    __syncthreads();
    if (s.done) break;
  }
  for (int p = tid; p < nw; p += kOnSmallThreads) P.occ[p] = s.n[p];
}

// ---- features, targets and warm start ------------------------------------

// Row block of problem i starts at P.row0; one row per pair.  One wave per
// (pair g, problem): the pair's weak orbitals (ascending index, the first
// kKmax) found by a ballot over the orbitals, and each mean field
// m_x = sum_{u strong, u != g} (2 J_xu - K_xu) as a lane-parallel FP64 sum with
// a fixed-order wave reduction.
__global__ __launch_bounds__(64) void k_on_feat(const OnProblem* __restrict__ probs, float* __restrict__ X,
                                                float* __restrict__ T, float* __restrict__ M,
                                                const float* __restrict__ mu, const float* __restrict__ sigma) {
  const OnProblem& P = probs[blockIdx.y];
  const int g = blockIdx.x;
  const int nw = P.n_omega, np_ = P.n_pairs, nc = P.n_cwo;
  if (g >= np_) return;   // the whole wave
  const int lane = threadIdx.x;
  int weak[kKmax];
  int k = 0;
  for (int p0 = np_; p0 < nw && k < kKmax; p0 += 64) {
    const int p = p0 + lane;
    unsigned long long m = __ballot(p < nw && on_pair(P.pair_of, p, np_, nc) == g);
    while (m && k < kKmax) {
      weak[k++] = p0 + __ffsll((long long)m) - 1;
      m &= m - 1;
    }
  }
  auto mf = [&](int x) {
    double s = 0.0;
    for (int u = lane; u < np_; u += 64)
      if (u != g) s += 2.0 * P.J[(long)x * nw + u] - P.K[(long)x * nw + u];
    return wave_sum_dpp(s);
  };
  float f[kNin];
  for (int i = 0; i < kNin; ++i) f[i] = 0.f;
  float t[kNout], m[kNout];
  for (int i = 0; i < kNout; ++i) { t[i] = 0.f; m[i] = 0.f; }
  const int s0 = g;
  f[0] = (float)P.Hpp[s0];
  f[1] = (float)P.J[(long)s0 * nw + s0];
  f[2] = (float)mf(s0);
  t[0] = P.occ ? (float)P.occ[s0] : 0.f;
  m[0] = 1.f;
  for (int q = 0; q < k; ++q) {
    const int p = weak[q];
    f[3 + 5 * q + 0] = (float)(P.Hpp[p] - P.Hpp[s0]);
    f[3 + 5 * q + 1] = (float)P.J[(long)p * nw + p];
    f[3 + 5 * q + 2] = (float)P.K[(long)s0 * nw + p];
    f[3 + 5 * q + 3] = (float)P.J[(long)s0 * nw + p];
    f[3 + 5 * q + 4] = (float)mf(p);
    f[3 + 5 * kKmax + q] = 1.f;
    t[1 + q] = P.occ ? (float)P.occ[p] : 0.f;
    m[1 + q] = 1.f;
  }
  const long row = P.row0 + g;
  for (int i = lane; i < kNin; i += 64) {
    float z = f[i];
    if (mu && sigma && sigma[i] > 0.f) z = (z - mu[i]) / sigma[i];
    X[row * kNin + i] = z;
  }
  for (int i = lane; i < kNout; i += 64) {
    if (T) T[row * kNout + i] = t[i];
    if (M) M[row * kNout + i] = m[i];
  }
}

// Predicted pair ONs p (rows as in k_on_feat) -> starting variables gamma.
__global__ __launch_bounds__(64) void k_on_warm(const OnProblem* __restrict__ probs, const float* __restrict__ Pn) {
  const OnProblem& P = probs[blockIdx.x];
  const int nc = P.n_cwo;
  for (int g = threadIdx.x; g < P.n_pairs; g += 64) {
    const float* p = Pn + (P.row0 + g) * (long)kNout;
    const double ng = fmin(fmax((double)p[0], 0.5), 1.0);
    double* x = P.gamma + (long)g * nc;
    x[0] = acos(sqrt(fmin(fmax(2.0 * ng - 1.0, 0.0), 1.0)));
    double tot = 0.0;
    for (int k = 0; k < nc && k < kKmax; ++k) tot += fmax((double)p[1 + k], 0.0);
    double s = 1.0;
    for (int k = 0; k < nc - 1; ++k) {
      const double wk = (tot > 0.0 && k < kKmax) ? fmax((double)p[1 + k], 0.0) / tot : 1.0 / nc;
      const double c2 = s > 1e-300 ? fmin(fmax(wk / s, 0.0), 1.0) : 1.0;
      x[1 + k] = acos(sqrt(c2));
      s *= 1.0 - c2;
    }
  }
}

// ---- MLP ---------------------------------------------------------------------
// FP32 MFMA (v_mfma_f32_16x16x4: A row / B column lane % 16, k = lane / 16; D
// row 4 (lane / 16) + r, column lane % 16).  Each weight block is stored
// augmented: W_aug = [W (I x O); b (O)].  FP32 partial sums over at most 128 k
// are folded into FP64, where the bias, tanh, the softmax and the loss are.
//
// The network is tiny (39 k weights, 157 KB) and its rows are many, so what
// counts is passes and launches: one workgroup carries 16 RT rows through every
// layer with the activations in LDS and the weights read from L2 (each
// fragment once per workgroup), forward and backward alike, and the weight
// gradients are one split contraction over the rows for all four layers.  Every
// FP32 sum runs over its k in ascending order, 128 at a time: a training run's
// FP64 losses keep the digits of weights updated that way.
// At 19,553 rows (an epoch of the 2000-molecule training set) forward, backward
// and Adam took 3665 us with a launch per layer and the weight gradients as 6
// workgroups of 64 x 64 tiles walking all the rows (864 us a layer); now 131 us
// (forward 51, backward 76, Adam 4).
constexpr int kActLd = kNhid + 4;   // LDS row of an activation: 16-byte aligned, rows 4 banks apart
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));   // 16 bytes at any float address

constexpr int kMlpThreads = 512;    // eight waves, one 16-column strip of a hidden layer each
__host__ __device__ constexpr long mlp_in(int l) { return l == 0 ? kNin : kNhid; }
__host__ __device__ constexpr long mlp_out(int l) { return l == 3 ? kNout : kNhid; }
__host__ __device__ constexpr long layer_off(int l) {
  long o = 0;
  for (int i = 0; i < l; ++i) o += (mlp_in(i) + 1) * mlp_out(i);
  return o;
}

// acc[i] += x rows (16 i ..) . B over K, x in LDS ([row][k], zero from K up to
// a multiple of 16); bval(k, b) gives this lane's column of B at the four steps
// k + 4 m + lane / 16 of the slice at k.
template <int RT, int K, class BV>
__device__ __forceinline__ void mlp_strip(const float* x, f4 (&acc)[RT], BV&& bval) {
  const int lane = threadIdx.x & 63, kr = lane >> 4, xc = lane & 15;
#pragma unroll
  for (int c = 0; c < (K + 15) / 16; ++c) {
    float a[RT][4], b[4];
    bval(16 * c, b);
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int m = 0; m < 4; ++m) a[i][m] = x[(16 * i + xc) * kActLd + 16 * c + 4 * m + kr];
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
      for (int i = 0; i < RT; ++i) acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][m], b[m], acc[i], 0, 0, 0);
  }
}
// b[m] of lane group g holds element 4 g + m on entry, 4 m + g on return.
__device__ __forceinline__ void transpose_groups(float (&b)[4]) {
  auto swap32 = [](float& x, float& y) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    x = __uint_as_float(r[0]);
    y = __uint_as_float(r[1]);
  };
  auto swap16 = [](float& x, float& y) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    x = __uint_as_float(r[0]);
    y = __uint_as_float(r[1]);
  };
  swap32(b[0], b[2]);
  swap32(b[1], b[3]);
  swap16(b[0], b[1]);
  swap16(b[2], b[3]);
}

// tanh |x| = E / (E + 2), E = exp(2|x|) - 1 = 2^n expm1(r) + (2^n - 1) with 2|x| =
// n ln 2 + r, |r| <= ln 2 / 2, expm1 from its Taylor series to r^14 (the next
// term is below 2^-54 of it) and the quotient from the reciprocal with two Newton
// steps: a few FP64 roundings from the true value down to x = 0, so its FP32
// rounding is the library tanh's, at about a third of the FP64 instructions.  1
// from |x| = 20 on.
__device__ __forceinline__ double tanh_for_f32(double x) {
  double y = 2.0 * fabs(x);
  y = y > 40.0 ? 40.0 : y;   // (a NaN stays)
  const double n = rint(y * 1.4426950408889634);
  const double r = fma(n, -1.9082149292705877e-10, fma(n, -0.69314718036912381, y));   // ln 2 in two parts
  double q = 1.0 / 87178291200.0;   // 1/14!, down to 1/1!
  q = fma(q, r, 1.0 / 6227020800.0);
  q = fma(q, r, 1.0 / 479001600.0);
  q = fma(q, r, 1.0 / 39916800.0);
  q = fma(q, r, 1.0 / 3628800.0);
  q = fma(q, r, 1.0 / 362880.0);
  q = fma(q, r, 1.0 / 40320.0);
  q = fma(q, r, 1.0 / 5040.0);
  q = fma(q, r, 1.0 / 720.0);
  q = fma(q, r, 1.0 / 120.0);
  q = fma(q, r, 1.0 / 24.0);
  q = fma(q, r, 1.0 / 6.0);
  q = fma(q, r, 0.5);
  q = fma(q, r, 1.0);
  const double two_n = ldexp(1.0, (int)n);
  const double E = fma(two_n * q, r, two_n - 1.0), d = E + 2.0;
  double c = __builtin_amdgcn_rcp(d);
  c = fma(fma(-d, c, 1.0), c, c);
  c = fma(fma(-d, c, 1.0), c, c);
  const double t = E * c;
  return copysign(fma(fma(-d, t, E), c, t), x);
}

// masked softmax of one row of logits
__device__ __forceinline__ void masked_softmax(const float* z, const float* m, double (&p)[kNout]) {
  double zmax = -1e300, e = 0.0;
#pragma unroll
  for (int k = 0; k < kNout; ++k)
    if (m[k] > 0.f) zmax = fmax(zmax, (double)z[k]);
#pragma unroll
  for (int k = 0; k < kNout; ++k) {
    p[k] = m[k] > 0.f ? exp((double)z[k] - zmax) : 0.0;
    e += p[k];
  }
#pragma unroll
  for (int k = 0; k < kNout; ++k) p[k] /= e;
}

// Forward, all layers: hidden y = tanh(x_aug W_aug), logits, masked softmax.
template <int RT>
__global__ __launch_bounds__(kMlpThreads) void k_mlp_fwd(int nrows, const float* __restrict__ X,
                                                         const float* __restrict__ M,
                                                         const float* __restrict__ theta, float* __restrict__ H,
                                                         float* __restrict__ Z, float* __restrict__ Pout) {
  constexpr int ROWS = 16 * RT;
  __shared__ __attribute__((aligned(16))) float act[2][ROWS * kActLd];
  __shared__ float zs[ROWS][kNout];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, kr = lane >> 4, xc = lane & 15;
  const long r0 = (long)blockIdx.x * ROWS;
  for (int i = tid; i < ROWS * 48; i += kMlpThreads) {
    const int r = i / 48, k = i - r * 48;
    // column kNin: the 1 that meets the bias row
    act[0][r * kActLd + k] = r0 + r >= nrows || k > kNin ? 0.f : k == kNin ? 1.f : X[(r0 + r) * kNin + k];
  }
  __syncthreads();
  auto hidden = [&](auto layer) {
    constexpr int l = decltype(layer)::value, I = (int)mlp_in(l);
    const float* W = theta + layer_off(l) + 16 * wave + xc;   // this lane's column
    f4 acc[RT] = {};
    // layer 0's 40 rows of W_aug are one sum; with 128 inputs the bias joins in FP64
    constexpr int K = I % 16 == 0 ? I : I + 1;
    mlp_strip<RT, K>(act[l & 1], acc, [&](int k0, float (&b)[4]) {
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const int k = k0 + 4 * m + kr;
        b[m] = K % 16 == 0 || k < K ? W[(long)(K % 16 == 0 || k < K ? k : 0) * kNhid] : 0.f;
      }
    });
    const double bias = K == I ? (double)W[(long)I * kNhid] : 0.0;
    float* y = act[(l + 1) & 1];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = 16 * i + 4 * kr + r;
        const float v = (float)tanh_for_f32((double)acc[i][r] + bias);
        y[row * kActLd + 16 * wave + xc] = v;
        if (r0 + row < nrows) H[((long)l * nrows + r0 + row) * kNhid + 16 * wave + xc] = v;
      }
    __syncthreads();
  };
  hidden(std::integral_constant<int, 0>());
  hidden(std::integral_constant<int, 1>());
  hidden(std::integral_constant<int, 2>());
  if (wave < RT) {   // logits: one wave per 16 rows, columns past the last unused
    const float* W = theta + layer_off(3) + (xc < kNout ? xc : 0);
    f4 acc[1] = {};
    mlp_strip<1, kNhid>(act[1] + 16 * wave * kActLd, acc, [&](int k0, float (&b)[4]) {
#pragma unroll
      for (int m = 0; m < 4; ++m) b[m] = W[(long)(k0 + 4 * m + kr) * kNout];
    });
    const double bias = W[(long)kNhid * kNout];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = 16 * wave + 4 * kr + r;
      const float v = (float)((double)acc[0][r] + bias);
      if (xc < kNout) {
        zs[row][xc] = v;
        if (r0 + row < nrows) Z[(r0 + row) * kNout + xc] = v;
      }
    }
  }
  __syncthreads();
  if (tid < ROWS && r0 + tid < nrows) {
    double p[kNout];
    masked_softmax(zs[tid], M + (r0 + tid) * kNout, p);
#pragma unroll
    for (int k = 0; k < kNout; ++k) Pout[(r0 + tid) * kNout + k] = (float)p[k];
  }
}

// Backward through the activations: loss partials (one per workgroup), dZ of
// the loss, then dA_l[row][i] = (sum_o dY[row][o] W[i][o]) (1 - h[row][i]^2) for
// l = 2, 1, 0 (the gradients at the pre-activations, which the weight
// gradients read); a null output is not stored.
template <int RT>
__global__ __launch_bounds__(kMlpThreads) void k_mlp_bwd(int nrows, const float* __restrict__ T,
                                                         const float* __restrict__ M,
                                                         const float* __restrict__ theta,
                                                         const float* __restrict__ H, const float* __restrict__ Z,
                                                         float* __restrict__ dZ, float* __restrict__ dA2,
                                                         float* __restrict__ dA1, float* __restrict__ dA0,
                                                         double* __restrict__ lpart) {
  constexpr int ROWS = 16 * RT;
  __shared__ __attribute__((aligned(16))) float act[2][ROWS * kActLd];
  __shared__ double red[ROWS];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, kr = lane >> 4, xc = lane & 15;
  const long r0 = (long)blockIdx.x * ROWS;
  if (tid < ROWS) {
    const long row = r0 + tid;
    double l = 0.0;
    float g[16] = {};
    if (row < nrows) {
      const float* m = M + row * kNout;
      double p[kNout], dp[kNout], sdp = 0.0;
      masked_softmax(Z + row * kNout, m, p);
#pragma unroll
      for (int k = 0; k < kNout; ++k) {
        const double t = T[row * kNout + k];
        l += m[k] * (p[k] - t) * (p[k] - t);
        dp[k] = 2.0 * m[k] * (p[k] - t) / nrows;
        sdp += dp[k] * p[k];
      }
#pragma unroll
      for (int k = 0; k < kNout; ++k) {
        g[k] = (float)(p[k] * (dp[k] - sdp));
        if (dZ) dZ[row * kNout + k] = g[k];
      }
    }
#pragma unroll
    for (int k = 0; k < 16; ++k) act[0][tid * kActLd + k] = g[k];
    red[tid] = l;
  }
  __syncthreads();
  if (tid == 0 && lpart) {
    double s = 0.0;
    for (int i = 0; i < ROWS; ++i) s += red[i];
    lpart[blockIdx.x] = s;
  }
  auto back = [&](auto layer, float* __restrict__ out) {   // through layer l to the activations below it
    constexpr int l = decltype(layer)::value, O = (int)mlp_out(l);
    const int col = 16 * wave + xc;   // i
    const float* W = theta + layer_off(l) + (long)col * O;
    f4 acc[RT] = {};
    mlp_strip<RT, O>(act[(3 - l) & 1], acc, [&](int k0, float (&b)[4]) {
      if constexpr (O % 16 == 0) {
        const f4u w = *(const f4u*)(W + k0 + 4 * kr);
#pragma unroll
        for (int m = 0; m < 4; ++m) b[m] = w[m];
        transpose_groups(b);
      } else {
#pragma unroll
        for (int m = 0; m < 4; ++m) b[m] = k0 + 4 * m + kr < O ? W[k0 + 4 * m + kr] : 0.f;
      }
    });
    float* y = act[(4 - l) & 1];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const long row = r0 + 16 * i + 4 * kr + r;
        float v = 0.f;
        if (row < nrows) {
          const double h = H[((long)(l - 1) * nrows + row) * kNhid + col];
          v = (float)((double)acc[i][r] * (1.0 - h * h));
          if (out) out[row * kNhid + col] = v;
        }
        if (l > 1) y[(16 * i + 4 * kr + r) * kActLd + col] = v;
      }
    if (l > 1) __syncthreads();
  };
  back(std::integral_constant<int, 3>(), dA2);
  back(std::integral_constant<int, 2>(), dA1);
  back(std::integral_constant<int, 1>(), dA0);
}

// Weight gradients of every layer, dW_aug[i][o] = sum_row x_aug[row][i]
// dY[row][o], split over the rows: workgroup (s, l) sums the rows
// [s chunk, (s+1) chunk) of layer l into part[s], eight waves of TM x TN
// fragments (WN waves along o) whose operands come straight from memory: a
// fragment is 16 consecutive floats of four rows, and the fragments of a wave
// feed TM TN MFMAs per four rows, so nothing is staged.  The bias row is a row
// of ones among x's: row 39 of layer 0's last fragment, else a fragment of its
// own, one column fragment of it to each strip of i.
struct WgradArgs {
  int nrows, chunk;
  const float *X, *H, *dZ, *dA[3];
  double* part;   // [splits][n_params], or null: one split, straight into grad
  float* grad;
  int first;      // blockIdx.y + first: 0, 1, 2, 3 for layers 1, 2, 3, 0
};
template <int L, int TM, int TN, int WN>
__device__ __forceinline__ void wgrad_layer(const WgradArgs& a) {
  constexpr int I = (int)mlp_in(L), O = (int)mlp_out(L);
  const float* x = L == 0 ? a.X : a.H + (long)(L - 1) * a.nrows * kNhid;
  const float* dy = L == 3 ? a.dZ : a.dA[L];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, kr = lane >> 4, xc = lane & 15;
  const int i0 = (wave / WN) * TM * 16, o0 = (wave % WN) * TN * 16;
  const int k0 = blockIdx.x * a.chunk, k1 = min(a.nrows, k0 + a.chunk);
  f4 s[TM][TN] = {};
  d4 v[TM][TN] = {};
  f4 sb = {};   // bias, column fragment (strip of i) of this wave
  d4 vb = {};
  constexpr bool kOwnBias = I % 16 == 0;
  const int jb = wave / WN;
  int ic[TM], oc[TN];   // fragment columns, clamped: those past the end are never stored
#pragma unroll
  for (int i = 0; i < TM; ++i) ic[i] = min(i0 + 16 * i + xc, I - 1);
#pragma unroll
  for (int j = 0; j < TN; ++j) oc[j] = min(o0 + 16 * j + xc, O - 1);
  // sixteen rows a step, the next step's loads in flight during this one's
  // MFMAs; rows past the end read the last one and count as zero
  float av[4][TM], bv[4][TN], an[4][TM], bn[4][TN];
  auto fetch = [&](int k, float (&x4)[4][TM], float (&y4)[4][TN]) {
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const long rc = min(k + 4 * m + kr, k1 - 1);
#pragma unroll
      for (int i = 0; i < TM; ++i) x4[m][i] = x[rc * I + ic[i]];
#pragma unroll
      for (int j = 0; j < TN; ++j) y4[m][j] = dy[rc * O + oc[j]];
    }
  };
  auto step = [&](int k, float (&x4)[4][TM], float (&y4)[4][TN]) {
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const bool ok = k + 4 * m + kr < k1;
#pragma unroll
      for (int i = 0; i < TM; ++i)
        x4[m][i] = !ok ? 0.f : !kOwnBias && i0 + 16 * i + xc == I ? 1.f : x4[m][i];
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        y4[m][j] = ok ? y4[m][j] : 0.f;
        if (kOwnBias && j == jb) sb = __builtin_amdgcn_mfma_f32_16x16x4f32(1.f, y4[m][j], sb, 0, 0, 0);
      }
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          s[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(x4[m][i], y4[m][j], s[i][j], 0, 0, 0);
    }
    if (((k - k0) & 127) == 112 || k + 16 >= k1) {   // 128 rows, or the last of them
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
#pragma unroll
          for (int r = 0; r < 4; ++r) v[i][j][r] += (double)s[i][j][r];
          s[i][j] = f4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
      for (int r = 0; r < 4; ++r) vb[r] += (double)sb[r];
      sb = f4{0.f, 0.f, 0.f, 0.f};
    }
  };
  fetch(k0, av, bv);
  for (int k = k0; k < k1; k += 32) {
    fetch(min(k + 16, k1 - 1), an, bn);
    step(k, av, bv);
    if (k + 16 >= k1) break;
    fetch(min(k + 32, k1 - 1), av, bv);
    step(k + 16, an, bn);
  }
  double* out = a.part ? a.part + (long)blockIdx.x * layer_off(4) + layer_off(L) : nullptr;
  auto put = [&](int i, int o, double g) {
    if (out) out[(long)i * O + o] = g;
    else a.grad[layer_off(L) + (long)i * O + o] = (float)g;
  };
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int ii = i0 + 16 * i + 4 * kr + r, oo = o0 + 16 * j + xc;
        if (ii < I + (kOwnBias ? 0 : 1) && oo < O) put(ii, oo, v[i][j][r]);
      }
  if (kOwnBias && jb < TN && kr == 0 && o0 + 16 * jb + xc < O) put(I, o0 + 16 * jb + xc, vb[0]);   // every row alike
}
__global__ __launch_bounds__(kMlpThreads) void k_mlp_wgrad(WgradArgs a) {
  switch (a.first + (int)blockIdx.y) {   // layer 0 last, on its own where the arena is capped
    case 0: wgrad_layer<1, 2, 4, 2>(a); break;
    case 1: wgrad_layer<2, 2, 4, 2>(a); break;
    case 2: wgrad_layer<3, 1, 1, 1>(a); break;
    default: wgrad_layer<0, 3, 1, 8>(a); break;
  }
}

// grad[i] = sum over the splits, in a fixed order (four strided quarters, then
// their sum); the last workgroup adds up the loss partials.
__global__ __launch_bounds__(256) void k_mlp_reduce(int n, int splits, const double* __restrict__ part,
                                                    float* __restrict__ grad, int nl,
                                                    const double* __restrict__ lpart, double scale,
                                                    double* __restrict__ loss) {
  __shared__ double red[256];
  const int tid = threadIdx.x;
  if (blockIdx.x + 1 < gridDim.x) {
    const int i = blockIdx.x * 64 + (tid & 63);
    double s = 0.0;
    if (i < n) {
#pragma unroll 8
      for (int k = tid >> 6; k < splits; k += 4) s += part[(long)k * n + i];
    }
    red[tid] = s;
    __syncthreads();
    if (tid < 64 && i < n) grad[i] = (float)((red[tid] + red[tid + 64]) + (red[tid + 128] + red[tid + 192]));
    return;
  }
  double s = 0.0;
  for (int i = tid; i < nl; i += 256) s += lpart[i];
  red[tid] = s;
  __syncthreads();
  for (int k = 128; k > 0; k >>= 1) {
    if (tid < k) red[tid] += red[tid + k];
    __syncthreads();
  }
  if (tid == 0) *loss = red[0] * scale;
}

// Adam with bias correction (step counts from 1)
__global__ __launch_bounds__(256) void k_adam(int n, float* __restrict__ th, const float* __restrict__ g,
                                              float* __restrict__ m, float* __restrict__ v, int step, float lr,
                                              float b1, float b2, float eps) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.f - b1) * gi;
  const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  const float mh = mi / (1.f - powf(b1, (float)step));
  const float vh = vi / (1.f - powf(b2, (float)step));
  th[i] -= lr * mh / (sqrtf(vh) + eps);
}

// H_pp = c_p^T H c_p: one workgroup per orbital; threads over mu read H[nu][mu]
// (H symmetric) coalesced, then a fixed-order block sum.
__global__ __launch_bounds__(256) void k_hpp(int nb, int nmo, const double* __restrict__ H,
                                             const double* __restrict__ C, double* __restrict__ Hpp) {
  __shared__ double red[256];
  const int p = blockIdx.x;
  double acc = 0.0;
  for (int mu = threadIdx.x; mu < nb; mu += 256) {
    double t = 0.0;
    for (int nu = 0; nu < nb; ++nu) t = fma(H[(long)nu * nb + mu], C[(long)nu * nmo + p], t);
    acc = fma(C[(long)mu * nmo + p], t, acc);
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) Hpp[p] = red[0];
}

// ---- host entry points --------------------------------------------------------

rif_status op_hpp(rif_ctx* c, int nb, int nmo, int nw, const double* H, const double* C, double* Hpp) {
  ProfScope ps(c, "hpp");
  hipLaunchKernelGGL(k_hpp, dim3(nw), dim3(256), 0, c->stream, nb, nmo, H, C, Hpp);
  return check_launch(c, "hpp");
}

static rif_status upload_problems(rif_ctx* c, int n, const OnProblem* probs, OnProblem** dptr) {
  const size_t bytes = sizeof(OnProblem) * (size_t)n;
  Carve cv;
  const size_t o = cv.take<OnProblem>((size_t)n);
  rif_status st = ws_reserve(c, cv.off);
  if (st) return st;
  *dptr = (OnProblem*)((char*)c->ws + o);
  if (hipMemcpyAsync(*dptr, probs, bytes, hipMemcpyHostToDevice, c->stream) != hipSuccess)
    return fail(c, RIF_EHIP, "uploading the problem table failed");
  // the host array may be reused by the caller right after return
  if (hipStreamSynchronize(c->stream) != hipSuccess) return fail(c, RIF_EHIP, "hipStreamSynchronize failed");
  return RIF_OK;
}

long on_work_doubles(int nw, int npairs, int ncwo) { return on_ws_doubles(nw, npairs, ncwo); }

rif_status op_on_optimize(rif_ctx* c, int n, const OnProblem* probs) {
  OnProblem* d = nullptr;
  rif_status st = upload_problems(c, n, probs, &d);
  if (st) return st;
  ProfScope ps(c, "on_opt");
  bool small = false, large = false;
  for (int i = 0; i < n; ++i) (on_small(probs[i]) ? small : large) = true;
  if (small) hipLaunchKernelGGL(k_on_opt_small, dim3(n), dim3(kOnSmallThreads), 0, c->stream, d);
  if (large) hipLaunchKernelGGL(k_on_opt, dim3(n), dim3(kOnThreads), 0, c->stream, d);
  return check_launch(c, "on_opt");
}

rif_status op_on_features(rif_ctx* c, int n, const OnProblem* probs, float* X, float* T, float* M, const float* mu,
                          const float* sigma) {
  OnProblem* d = nullptr;
  rif_status st = upload_problems(c, n, probs, &d);
  if (st) return st;
  int maxp = 1;
  for (int i = 0; i < n; ++i) maxp = std::max(maxp, probs[i].n_pairs);
  ProfScope ps(c, "on_features");
  hipLaunchKernelGGL(k_on_feat, dim3((unsigned)maxp, (unsigned)n), dim3(64), 0, c->stream, d, X, T, M, mu, sigma);
  return check_launch(c, "on_features");
}

rif_status op_on_warmstart(rif_ctx* c, int n, const OnProblem* probs, const float* Pn) {
  OnProblem* d = nullptr;
  rif_status st = upload_problems(c, n, probs, &d);
  if (st) return st;
  ProfScope ps(c, "on_warm");
  hipLaunchKernelGGL(k_on_warm, dim3(n), dim3(64), 0, c->stream, d, Pn);
  return check_launch(c, "on_warm");
}

long mlp_n_params() { return layer_off(4); }

// Rows per workgroup of the fused passes: 32 halve the weight reads, 16 fill the
// chip sooner and halve a workgroup's chain.  Forward + backward, 16 against 32
// rows: 50.8 / 60.8 us at 4,096 rows, 83.4 / 89.1 at 12,000, 105 / 93.6 at 14,336,
// 130 / 127 at 19,553; the line lies at three 16-row workgroups per CU.
static bool mlp_wide(int nrows) { return nrows > 256 * 48; }

rif_status op_mlp_forward(rif_ctx* c, int nrows, const float* X, const float* M, const float* theta, float* H,
                          float* Z, float* Pn) {
  ProfScope ps(c, "mlp_fwd");
  if (mlp_wide(nrows))
    hipLaunchKernelGGL(k_mlp_fwd<2>, dim3(cdiv_i(nrows, 32)), dim3(kMlpThreads), 0, c->stream, nrows, X, M, theta, H,
                       Z, Pn);
  else
    hipLaunchKernelGGL(k_mlp_fwd<1>, dim3(cdiv_i(nrows, 16)), dim3(kMlpThreads), 0, c->stream, nrows, X, M, theta, H,
                       Z, Pn);
  return check_launch(c, "mlp_fwd");
}

rif_status op_mlp_backward(rif_ctx* c, int nrows, const float* X, const float* M, const float* T,
                           const float* theta, const float* H, const float* Z, float* dA, float* grad,
                           double* loss) {
  const bool wide = mlp_wide(nrows);
  const int nl = cdiv_i(nrows, wide ? 32 : 16), n = (int)mlp_n_params();
  // splits of the weight gradients: whole 128-row FP32 sums, at most about 160
  // workgroups for each wide layer (two of them fill the chip)
  int chunk = 128 * cdiv_i(nrows, 128 * 160), splits = cdiv_i(nrows, chunk);
  Carve cv;
  const size_t o_dz = cv.take<float>((size_t)nrows * kNout);
  // the rest only if the arena may hold it (rif_set_workspace_limit): without
  // it each gradient is one split, stored straight into grad, and the third
  // dA shares dA's first buffer in a second backward pass.  The loss partials (half
  // a byte a row) come from that pass and take dZ's place (28 bytes a row), which
  // layer 0's gradients have no use for
  Carve full = cv;
  const size_t o_lp = full.take<double>((size_t)nl);
  const size_t o_part = full.take<double>((size_t)splits * n);
  const size_t o_da = full.take<float>((size_t)nrows * kNhid);
  bool roomy = false;
  rif_status st = ws_reserve_either(c, full.off, cv.off, &roomy);
  if (st) return st;
  const bool lean = !roomy;
  char* ws = (char*)c->ws;
  float* dZ = (float*)(ws + o_dz);
  double* lp = lean ? (double*)dZ : (double*)(ws + o_lp);
  float *d2 = dA, *d1 = dA + (long)nrows * kNhid, *d0 = lean ? dA : (float*)(ws + o_da);
  auto back = [&](float* pz, float* p2, float* p1, float* p0, double* pl) {
    ProfScope ps(c, "mlp_dgrad");
    if (wide)
      hipLaunchKernelGGL(k_mlp_bwd<2>, dim3(nl), dim3(kMlpThreads), 0, c->stream, nrows, T, M, theta, H, Z, pz, p2, p1,
                         p0, pl);
    else
      hipLaunchKernelGGL(k_mlp_bwd<1>, dim3(nl), dim3(kMlpThreads), 0, c->stream, nrows, T, M, theta, H, Z, pz, p2, p1,
                         p0, pl);
    return check_launch(c, "mlp_dgrad");
  };
  if (lean) { chunk = nrows; splits = 1; }
  WgradArgs a{nrows, chunk, X, H, dZ, {d0, d1, d2}, splits > 1 ? (double*)(ws + o_part) : nullptr, grad, 0};
  auto weights_of = [&](int first, int count) {
    a.first = first;
    ProfScope ps(c, "mlp_wgrad");
    hipLaunchKernelGGL(k_mlp_wgrad, dim3((unsigned)splits, (unsigned)count), dim3(kMlpThreads), 0, c->stream, a);
    return check_launch(c, "mlp_wgrad");
  };
  if (lean) {
    if ((st = back(dZ, d2, d1, nullptr, nullptr)) || (st = weights_of(0, 3)) ||
        (st = back(nullptr, nullptr, nullptr, d0, lp)) || (st = weights_of(3, 1)))
      return st;
  } else if ((st = back(dZ, d2, d1, d0, lp)) || (st = weights_of(0, 4))) {
    return st;
  }
  ProfScope ps(c, "mlp_reduce");
  hipLaunchKernelGGL(k_mlp_reduce, dim3((unsigned)((splits > 1 ? cdiv_i(n, 64) : 0) + 1)), dim3(256), 0, c->stream, n,
                     splits, a.part, grad, nl, lp, 1.0 / nrows, loss);
  return check_launch(c, "mlp_reduce");
}

rif_status op_adam(rif_ctx* c, int n, float* theta, const float* grad, float* m, float* v, int step, float lr,
                   float b1, float b2, float eps) {
  ProfScope ps(c, "adam");
  hipLaunchKernelGGL(k_adam, dim3(cdiv_i(n, 256)), dim3(256), 0, c->stream, n, theta, grad, m, v, step, lr, b1, b2,
                     eps);
  return check_launch(c, "adam");
}

}  // namespace rif
