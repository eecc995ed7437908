// FP64 MFMA main loop for products of two x-contiguous operands (element (x, k)
// at base[k ld + x]): the half transform, J^q, K^q, the Fock step and the solve of
// the preparation.
//
// What bounds these kernels is how much of a slice's time the matrix cores are
// busy.  A 16-deep slice of a 128 x 128 tile holds 32 v_mfma_f64_16x16x4 (64
// cycles each) per wave of 64 x 32, and two workgroups of eight waves share a
// CU, so loads, fragment reads and barriers hide, but every other instruction
// of the loop takes issue slots.  Measured with every load in L2 on a J^q-shaped
// product: 64-65 TFLOP/s with per-lane 64-bit load addresses, bounds tests and
// padded LDS rows, 71-72 here (73 is what a large vendor product reaches): the
// loads' bases are scalars that advance by a scalar, the lanes keep 32-bit
// offsets, a slice with rows past K is told apart by one uniform branch, and the
// loop is unrolled over the LDS stages.
//
// Rows of a tile.  The row count is a multiple of 16 chosen at run time for the
// operand (strip_rows: n_omega = 200 runs as two tiles of 112 rows, not two of
// 128), so one kernel serves every n_omega with little padding.  An even count of
// 16-row fragments splits over two waves, an odd one goes down a single wave:
// columns are dealt to the waves either way.
//
// Staging.  A stage holds 16 k rows of the A columns, then of the B columns,
// unpadded and contiguous; a wave moves 1 KB of it per global_load_lds_dwordx4.
// With an even number of 16-column groups odd rows swap the two groups of each
// pair, so the two k rows of a half-wave's fragment read use different banks (an
// odd number shifts them by itself).  Nothing needs alignment beyond the 8 bytes
// of a double.  A row of odd length n is staged as n + 1 columns whose last pair
// is loaded one element early: column n-2 again, then n-1 (pair_start,
// pair_column), so no load leaves its row.
#pragma once
#include "mfma_engine.hpp"

namespace rif {

// Zeros, read for k rows past the end.
static __device__ __attribute__((aligned(16))) double kDmaZeros[128];

// First column of the pair staged at (even) position p of an n-long row, and the
// column that position p holds (-1: none).  n >= 2.
__host__ __device__ __forceinline__ int pair_start(int p, int n) { return (n & 1) && p == n - 1 ? n - 2 : p; }
__host__ __device__ __forceinline__ int pair_column(int p, int n) {
  if (!(n & 1)) return p < n ? p : -1;
  return p < n - 1 ? p : p == n ? n - 1 : -1;
}
__host__ __device__ __forceinline__ int pair_len(int n) { return n + (n & 1); }

// 16-row fragments of a tile for n rows: equal tiles of at most 128 rows.
__host__ __device__ __forceinline__ int strip_tiles(int n) { return (n + 127) / 128; }
__host__ __device__ __forceinline__ int strip_frags(int n) {
  const int t = strip_tiles(n);
  return ((n + t - 1) / t + 15) / 16;
}

// Tile configuration: BN columns, NW waves.  (BM is the largest row count.)
template <int BN_, int NW_>
struct StripCfg {
  static constexpr bool kStrip = true;
  static constexpr int BM = 128, BN = BN_, NWAVES = NW_, NT = 64 * NW_, BK = 16;
};
template <class Cfg, class = void>
struct is_strip : std::false_type {};
template <class Cfg>
struct is_strip<Cfg, std::void_t<decltype(Cfg::kStrip)>> : std::true_type {};

// Layout of a tile of TM fragments: waves WVM x WVN, each FM x FN fragments;
// stages of LDS (small tiles hold less work per slice, so three).
template <class Cfg, int TM_>
struct Strip {
  static constexpr int TM = TM_, BM = 16 * TM, BN = Cfg::BN, NW = Cfg::NWAVES;
  static constexpr int WVM = TM % 2 == 0 ? 2 : 1, WVN = NW / WVM, FM = TM / WVM, FN = BN / 16 / WVN;
  static constexpr int S = TM <= 4 ? 3 : 2;
  static constexpr int NIA = BM / 8, NIB = BN / 8, NI = NIA + NIB, NU = (NI + NW - 1) / NW;   // 1 KB loads
  static constexpr int ST = NI * 1024;
  static_assert(FN >= 1 && FN * 16 * WVN == BN && (BN / 16) % 2 == 0, "columns per wave");
};
template <class Cfg, int TM = 8>
constexpr int strip_smem() {
  constexpr int here = Strip<Cfg, TM>::S * Strip<Cfg, TM>::ST;
  if constexpr (TM == 1) return here;
  else return here > strip_smem<Cfg, TM - 1>() ? here : strip_smem<Cfg, TM - 1>();
}
// f(std::integral_constant<int, tm>) for tm in 1..8
template <int TM = 8, class F>
__device__ __forceinline__ void with_frags(int tm, F&& f) {
  if (tm >= TM) f(std::integral_constant<int, TM>());
  else if constexpr (TM > 1) with_frags<TM - 1>(tm, f);
}

// Byte offset of lane's part of 1 KB load u of a stage from its operand's base (A of
// row stride lda for u < NIA, else B); fa(x) / fb(x) as in StripStage.
template <class L, class FA, class FB>
__host__ __device__ __forceinline__ long strip_offset(int u, int lane, long lda, FA fa, long ldb, FB fb) {
  const bool isA = u < L::NIA;
  const int v = (isA ? u : u - L::NIA) * 64 + lane;
  const int k = isA ? v / (L::BM / 2) : v / (L::BN / 2);
  int x = 2 * (isA ? v % (L::BM / 2) : v % (L::BN / 2));
  if ((!isA || L::TM % 2 == 0) && (k & 1)) x ^= 16;
  return 8 * ((isA ? fa(x) : fb(x)) + k * (isA ? lda : ldb));
}

// Whether the FP64 build steps' operands are staged by strips: column pairs (two
// columns at least) at lane offsets of 32 bits.  The farthest are those of a slab
// per k row (J^q, Fock): 15 slabs and a block's rows, 8 (15 n_bf^2 + 8 n_bf) bytes,
// below 2^32 up to n_bf = 5982.
inline bool strip_fits(int nb, int nmo, int nw) { return nb >= 2 && nw >= 2 && nb < 5900 && nmo < 5900; }

// The pair at (even) column x of the block of (mu, nu) that starts at row mu0 and
// position nu0 (16 nu a row): its offset from element (mu0, 0) of the slab, in
// doubles (odd n_bf: the last pair one early).  Pairs that are not there read
// that row's first.
__host__ __device__ __forceinline__ long block_offset(int x, int mu0, int nu0, int nb) {
  const int m = x / 16, p = nu0 + x % 16;
  return mu0 + m < nb && p < nb ? (long)m * nb + pair_start(p, nb) : 0;
}

// Direct-load staging of both operands.  fa(x) / fb(x): offset of the (even)
// tile column x from A / B in doubles; offsets plus 15 rows must fit 32 bits of
// bytes, so whatever a tile's lanes share goes into A / B.
template <class L>
struct StripStage {
  unsigned off[L::NU];
  const char* base[L::NU];
  long inc[L::NU];
  int w;
  template <class FA, class FB>
  __device__ __forceinline__ void init(const double* A, long lda, FA fa, const double* B, long ldb, FB fb) {
    w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int i = 0; i < L::NU; ++i) {
      const int u = w + i * L::NW;
      off[i] = (unsigned)strip_offset<L>(u, lane, lda, fa, ldb, fb);
      inc[i] = 128 * (u < L::NIA ? lda : ldb);
    }
    rebase(A, B);
  }
  // the k rows from here on start at A and B
  __device__ __forceinline__ void rebase(const double* A, const double* B) {
#pragma unroll
    for (int i = 0; i < L::NU; ++i) base[i] = (const char*)(w + i * L::NW < L::NIA ? A : B);
  }
  __device__ __forceinline__ bool have(int i) const {
    return L::NI % L::NW == 0 || i + 1 < L::NU || w + i * L::NW < L::NI;
  }
  // The next 16 k rows into stage st; left: rows there are (the rest read zeros).
  __device__ __forceinline__ void issue(lds_char* st, int left) {
    if (left >= 16) {
#pragma unroll
      for (int i = 0; i < L::NU; ++i)
        if (have(i)) {
          __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(base[i] + off[i]),
                                           (__attribute__((address_space(3))) void*)(st + (w + i * L::NW) * 1024), 16,
                                           0, 0);
          base[i] += inc[i];
        }
    } else {
      const int lane = threadIdx.x & 63;
#pragma unroll
      for (int i = 0; i < L::NU; ++i)
        if (have(i)) {
          const int u = w + i * L::NW;
          const int k = u < L::NIA ? (u * 64 + lane) / (L::BM / 2) : ((u - L::NIA) * 64 + lane) / (L::BN / 2);
          const char* p = k < left ? base[i] + off[i] : (const char*)(kDmaZeros + 2 * lane);
          __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)p,
                                           (__attribute__((address_space(3))) void*)(st + u * 1024), 16, 0, 0);
        }
    }
  }
};

// A barrier past which any wave may fill or write the LDS that this one has read: its
// LDS operations are done, its global loads in flight stay in flight (no fence).  The
// wait is not left to the MFMAs that use the values: some are moved past the barrier.
__device__ __forceinline__ void strip_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (0 << 8) | (3 << 14));   // lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

template <class L>
struct StripAcc {
  d4 v[L::FM][L::FN];
  int wm, wn;   // this wave's first row and column; element e of a lane: row lane / 16 + 4 e, column lane % 16
};

// nk slices; issue(kt, stage) stages slice kt (called once per slice, in order).
// Ends with every wave past its last LDS read and no load in flight.
template <class L, class Issue>
__device__ __forceinline__ void strip_mainloop(int nk, int w, StripAcc<L>& acc, char* smem_generic, Issue&& issue) {
  lds_char* sm = (lds_char*)smem_generic;
  const int lane = threadIdx.x & 63, kr = lane >> 4, xc = lane & 15;
  acc.wm = (w / L::WVN) * L::FM * 16;
  acc.wn = (w % L::WVN) * L::FN * 16;
#pragma unroll
  for (int i = 0; i < L::FM; ++i)
#pragma unroll
    for (int j = 0; j < L::FN; ++j) acc.v[i][j] = d4{0.0, 0.0, 0.0, 0.0};
  // this lane's reads: a fragment of an even 16-column group sits 16 up in odd
  // rows, one of an odd group 16 down
  const int sa = L::TM % 2 == 0 && (kr & 1) ? 16 : 0, sb = (kr & 1) ? 16 : 0;
  const int pa = acc.wm / 16 & 1, pb = acc.wn / 16 & 1;   // parity of the first fragment's group
  const int a0 = kr * L::BM + acc.wm + xc, b0 = kr * L::BN + acc.wn + xc;
  const int ae = a0 + (pa ? -sa : sa), ao = a0 + (pa ? sa : -sa);
  const int be = b0 + (pb ? -sb : sb), bo = b0 + (pb ? sb : -sb);
#pragma unroll
  for (int j = 0; j < L::S - 1; ++j)
    if (j < nk) issue(j, sm + j * L::ST);
  auto slice = [&](int kt, int s) {
    if (L::S == 3 && kt + 1 < nk) {   // the loads of slice kt+1 may stay in flight
      if (L::NI % L::NW == 0 || w + (L::NU - 1) * L::NW < L::NI) __builtin_amdgcn_s_waitcnt(L::NU | (7 << 4) | (15 << 8));
      else __builtin_amdgcn_s_waitcnt((L::NU - 1) | (7 << 4) | (15 << 8));
    } else {
      __builtin_amdgcn_s_waitcnt(0 | (7 << 4) | (15 << 8));
    }
    strip_barrier();
    if (kt + L::S - 1 < nk) issue(kt + L::S - 1, sm + ((s + L::S - 1) % L::S) * L::ST);
    const lds_f64* As = (const lds_f64*)(sm + s * L::ST);
    const lds_f64* Bs = As + 16 * L::BM;
#pragma unroll
    for (int kk = 0; kk < 16; kk += 4) {
      double a[L::FM], b[L::FN];
#pragma unroll
      for (int j = 0; j < L::FN; ++j) b[j] = Bs[kk * L::BN + ((j & 1) ? bo : be) + 16 * j];
#pragma unroll
      for (int i = 0; i < L::FM; ++i) a[i] = As[kk * L::BM + ((i & 1) ? ao : ae) + 16 * i];
#pragma unroll
      for (int i = 0; i < L::FM; ++i)
#pragma unroll
        for (int j = 0; j < L::FN; ++j)
          acc.v[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc.v[i][j], 0, 0, 0);
    }
  };
  static_assert(L::NU <= 15, "wait count");
  int kt = 0;
  for (; kt + L::S <= nk; kt += L::S) {
#pragma unroll
    for (int s = 0; s < L::S; ++s) slice(kt + s, s);
  }
#pragma unroll
  for (int s = 0; s < L::S - 1; ++s)
    if (kt + s < nk) slice(kt + s, s);
  strip_barrier();
}

}  // namespace rif
