// HIP kernels for gfx950 (MI355X): FP64 contractions of the packed Cholesky tensor.
//
// Every dense contraction runs on the FP64 matrix cores (v_mfma_f64_16x16x4_f64,
// 64 cycles per issue per SIMD; one wave per SIMD can keep the unit busy).  Operand
// tiles go global -> registers -> LDS in a [row][k] layout with a row stride of 17
// doubles.  The LDS serves 32 lanes of 8-byte accesses per cycle over 64 banks.  With this
// stride the "row fastest" stores are conflict-free; the "k fastest" stores and the MFMA
// operand reads have one colliding pair per 32 lanes.  An 18-double stride makes the reads
// conflict-free and the stores worse; the kernels run equally fast with either, because
// the conflicts hide behind the MFMAs.
//
// Main loop: two LDS stages; the global loads of slab s+1 are issued before the MFMAs
// of slab s and written to the other stage after them, one barrier per slab.  Loads
// are branch-free (out-of-range elements read a valid address and are replaced by 0
// with a select), so no wait on outstanding loads sits between the prefetch and the
// MFMA block.
//
// Operand layout of v_mfma_f64_16x16x4_f64 (measured on gfx950):
//   A[i][k] in lane i + 16k, B[k][j] in lane j + 16k,
//   D[i][j] in lane j + 16*(i%4), accumulator register i/4.
#include "kernels.h"

#include <math.h>

#include <algorithm>
#include <type_traits>
#include <utility>

namespace dfk {

typedef double d4 __attribute__((ext_vector_type(4)));

// WM x WN waves, each TM x TN MFMA tiles of 16 x 16; WPE: waves per SIMD the half transform's kernels
// are compiled for (at least).
template <int WM_, int WN_, int TM_, int TN_, int WPE_ = 2>
struct Cfg {
  static constexpr int WM = WM_, WN = WN_, TM = TM_, TN = TN_, WPE = WPE_;
  static constexpr int NT = 64 * WM * WN;
  static constexpr int BM = 16 * TM * WM, BN = 16 * TN * WN, BK = 16;
  static constexpr int LD = BK + 1;
  static constexpr int LDS_A = BM * LD, LDS_B = BN * LD, STAGE = LDS_A + LDS_B;
  static_assert((BM * BK) % NT == 0 && (BN * BK) % NT == 0, "tile must split evenly over threads");
};

// Every MFMA kernel is compiled for at least two waves per SIMD (256 registers per lane, two workgroups' LDS per
// CU), so one wave's barrier and LDS latency hide behind the other's MFMAs; smaller tiles for three or four.
// generic products and the K SYRK: 128 x 128 tiles, 2 x 2 waves of 64 x 64
typedef Cfg<2, 2, 4, 4> CfgSq;
// tall products (M >= 256): 256 x 128 tiles, 4 x 2 waves of 64 x 64, one workgroup per CU; the
// same per-wave work with a quarter fewer loads per MFMA
typedef Cfg<4, 2, 4, 4> CfgTall;
typedef Cfg<2, 2, 4, 4> CfgSyrk;
// small products: 64 x 64 tiles, four workgroups per CU
typedef Cfg<2, 2, 2, 2> CfgSmall;
// small matrices (fragment sizes): 64 x 64 SYRK tiles pad the triangle less (grouped launches)
typedef Cfg<2, 2, 2, 2> CfgSyrk64;
// K SYRK of one call: 64-row bands on 64 x 128 tiles, 64 x 64 where a band's columns end half way, the last rows
// (at most 32) on 32 x 128 (SyrkTiles); all three workgroups per CU
typedef Cfg<2, 2, 2, 4, 3> CfgKA;
typedef Cfg<2, 2, 2, 2, 3> CfgKD;
typedef Cfg<1, 4, 2, 2, 3> CfgKT;
// half transform: 64-row bands on tiles of 128 columns (three workgroups per CU), the columns past the
// last whole one on one tile of 96, 64, 48, 32 or 16.  At N_ao = 512 (2048 rows of P, columns that fill
// the tile) 128 columns run at 57.9 TF/s, as fast as 128 x 128 tiles (58.5) and with half the rows
// to pad; 96: 54.6, 64: 49.6, 48: 45.6, 32: 39.5, 16: 24.3 (there bound by the latency of the loads of b^P,
// so these take four waves per SIMD and more).  Where the rows past the last whole band fit 32, they take
// 32 x 128 tiles, if the columns fill a tile of 128 at all.  176 columns on one row of waves: 48.6;
// grouped launches may ask for it.
typedef Cfg<2, 2, 2, 4, 3> CfgH128;
typedef Cfg<2, 2, 2, 3, 3> CfgH96;
typedef Cfg<2, 2, 2, 2, 4> CfgH64;
typedef Cfg<4, 1, 1, 3, 4> CfgH48;
typedef Cfg<4, 1, 1, 2, 4> CfgH32;
typedef Cfg<4, 1, 1, 1, 4> CfgH16;
typedef Cfg<1, 4, 2, 2, 3> CfgHTail;
// The same with 128-row bands, for b^P larger than an XCD's L2 (see half_cols).  128 columns there: 61.6 TF/s.
typedef Cfg<2, 2, 4, 4> CfgQ128;
typedef Cfg<2, 2, 4, 3> CfgQ96;
typedef Cfg<2, 2, 4, 2> CfgQ64;
typedef Cfg<4, 1, 2, 3> CfgQ48;
typedef Cfg<2, 2, 2, 4> CfgQTail;
typedef Cfg<4, 1, 1, 11> CfgH176;

// ---------------------------------------------------------------------------------------
// Block index -> work item, keeping runs of consecutive work items on one XCD.  The
// dispatcher hands consecutive workgroups to the 8 XCDs in turn; this remap makes XCD x
// process the x-th eighth of the index range in order, so tiles that share operands
// (the same P slab, the same B tile) share that XCD's L2.
__device__ __forceinline__ int64_t xcd_remap(int64_t id, int64_t n) {
  const int64_t full = (n / 8) * 8;
  if (id >= full) return id;
  return (id % 8) * (full / 8) + id / 8;
}

// One k-step (4 deep) worth of MFMA operands of one wave.
template <class C>
struct Frag {
  double a[C::TM];
  double b[C::TN];
};

template <class C>
__device__ __forceinline__ void read_frag(const double* __restrict__ As, const double* __restrict__ Bs, int kk,
                                          Frag<C>& f, int wm, int wn, int lane) {
  const int lr = lane & 15, lk = lane >> 4;
#pragma unroll
  for (int i = 0; i < C::TM; ++i) f.a[i] = As[((wm * C::TM + i) * 16 + lr) * C::LD + kk + lk];
#pragma unroll
  for (int j = 0; j < C::TN; ++j) f.b[j] = Bs[((wn * C::TN + j) * 16 + lr) * C::LD + kk + lk];
}

template <class C>
__device__ __forceinline__ void zero_acc(d4 (&acc)[C::TM][C::TN]) {
#pragma unroll
  for (int i = 0; i < C::TM; ++i)
#pragma unroll
    for (int j = 0; j < C::TN; ++j) acc[i][j] = d4{0.0, 0.0, 0.0, 0.0};
}

// Compile-time loops.
template <int... I, class F>
__device__ __forceinline__ void static_for_impl(std::integer_sequence<int, I...>, F&& f) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(std::make_integer_sequence<int, N>{}, f);
}

// Sources.  A source feeds both operand tiles of a product slab by slab:
//   begin()          set up the next slab (uniform values only)
//   load<q>()        issue global load q (of NL) of the slab
//   finish()         advance to the following slab (clamped at the last one)
//   store<q>(A, B)   write loaded element q to the LDS tiles A, B
// Rows and columns past the end of a matrix are read at clamped (valid) addresses and never
// zeroed: they only reach output rows and columns that are not stored.  Only contraction
// indices past the end (a partial last slab) must contribute zero.

// One slab of the software pipeline.  LDS stage `cur` holds the slab being
// multiplied and F[0] already holds its first k-step of operands.  While its TM*TN*BK/4 MFMAs
// issue one by one, the wave reads the operands of the next k-step, issues the global loads of
// the next slab in the first half and writes those registers to the other LDS stage in the
// second half.  Then one barrier and the first operands of the next slab.  Every slot is
// generated at compile time, so the body is one basic block; scheduling fences keep the
// interleave.  (One body per kernel: alternative slab bodies in one loop overflow the 256
// registers a lane has at two waves per SIMD.)
template <class C, class Src>
__device__ __forceinline__ void slab_step(Src& src, double* smem, int cur, d4 (&acc)[C::TM][C::TN], Frag<C> (&F)[2],
                                          int wm, int wn, int lane) {
  const double* As = smem + cur * C::STAGE;
  const double* Bs = As + C::LDS_A;
  double* An = smem + (cur ^ 1) * C::STAGE;
  double* Bn = An + C::LDS_A;
  constexpr int KS = C::BK / 4;            // k-steps per slab
  constexpr int PK = C::TM * C::TN;        // MFMAs per k-step
  constexpr int NM = PK * KS;              // MFMAs per slab
  constexpr int HALF = NM / 2;
  constexpr int NL = Src::NL;
  static_assert(HALF > 0, "at least two MFMAs per slab");
  src.begin();
  static_for<NM>([&](auto IDXc) {
    constexpr int IDX = decltype(IDXc)::value;
    constexpr int ks = IDX / PK, ij = IDX % PK, i = ij / C::TN, j = ij % C::TN;
    if constexpr (ij == 0) {
      if constexpr (ks + 1 < KS) read_frag<C>(As, Bs, (ks + 1) * 4, F[(ks + 1) & 1], wm, wn, lane);
      __builtin_amdgcn_sched_barrier(0);
    }
    acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(F[ks & 1].a[i], F[ks & 1].b[j], acc[i][j], 0, 0, 0);
    if constexpr (IDX < HALF) {
      constexpr int Q0 = IDX * NL / HALF, Q1 = (IDX + 1) * NL / HALF;
      static_for<Q1 - Q0>([&](auto R) { src.template load<Q0 + decltype(R)::value>(); });
    } else {
      constexpr int Q0 = (IDX - HALF) * NL / HALF, Q1 = (IDX - HALF + 1) * NL / HALF;
      static_for<Q1 - Q0>([&](auto R) { src.template store<Q0 + decltype(R)::value>(An, Bn); });
    }
    __builtin_amdgcn_sched_barrier(0);
  });
  src.finish();
  __syncthreads();
  read_frag<C>(An, Bn, 0, F[0], wm, wn, lane);
}

// Runs nslab slabs through the pipeline (nslab >= 1).  The loads issued during the last slab
// re-read it (the sources clamp) and land in the stage nobody reads any more.
template <class C, class Src>
__device__ __forceinline__ void mainloop(Src& src, double* smem, int64_t nslab, d4 (&acc)[C::TM][C::TN], int wm,
                                         int wn, int lane) {
  src.begin();
  static_for<Src::NL>([&](auto Q) { src.template load<decltype(Q)::value>(); });
  src.finish();
  static_for<Src::NL>([&](auto Q) { src.template store<decltype(Q)::value>(smem, smem + C::LDS_A); });
  __syncthreads();
  Frag<C> F[2];
  read_frag<C>(smem, smem + C::LDS_A, 0, F[0], wm, wn, lane);
  for (int64_t s = 0; s < nslab; ++s) slab_step<C>(src, smem, (int)(s & 1), acc, F, wm, wn, lane);
}

// Epilogue.  GEN = false stores the accumulators as they are (o.alpha must be 1 and
// o.accumulate 0); GEN = true applies alpha and accumulate.  Arithmetic on the accumulators
// here moves them out of the matrix-core registers for the whole main loop (a copy per MFMA
// operand per slab), so only launches that need it instantiate GEN.
template <class C, bool GEN>
__device__ __forceinline__ void store_tile(const OutMap& o, int64_t z, int64_t m0, int64_t n0,
                                           const d4 (&acc)[C::TM][C::TN], int wm, int wn, int lane) {
  const int lr = lane & 15, lg = lane >> 4;
  const int64_t zo1 = z * o.s_z, zo2 = z * o.s2_z;
#pragma unroll
  for (int j = 0; j < C::TN; ++j) {
    const int64_t n = n0 + (wn * C::TN + j) * 16 + lr;
    const bool nok = n < o.N, first = n < o.nsplit;
    const uint32_t nh = o.s_nh ? (uint32_t)n / (uint32_t)o.nl : 0u;
    const int64_t noff1 = (int64_t)nh * o.s_nh + (n - (int64_t)nh * o.nl) * o.s_nl;
    // integer select: p2 is null when every column goes to p
    const uintptr_t col = first ? (uintptr_t)o.p + 8u * (uint64_t)(zo1 + noff1)
                                : (uintptr_t)o.p2 + 8u * (uint64_t)(zo2 + n - o.nsplit);
#pragma unroll
    for (int i = 0; i < C::TM; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t m = m0 + (wm * C::TM + i) * 16 + 4 * r + lg;
        const uint32_t mh = o.s_mh ? (uint32_t)m / (uint32_t)o.ml : 0u;
        const int64_t moff = first ? (int64_t)mh * o.s_mh + (m - (int64_t)mh * o.ml) * o.s_ml : m * o.s2_m;
        double* const dst = (double*)col + moff;
        if constexpr (GEN) {
          const double val = o.alpha * acc[i][j][r];
          if (nok && m < o.M) *dst = o.accumulate ? *dst + val : val;
        } else {
          if (nok && m < o.M) *dst = acc[i][j][r];
        }
      }
  }
}

// Operand described by an OpMap, staged through registers.  Slabs are walked in order (kb outer,
// kc in chunks of 16 inner) from slab `s_begin` to `s_end - 1`; the cursor stops at the last one.
//   KC = true : lanes run along k (16 consecutive k of one row per 16 lanes)
//   KC = false: lanes run along the row index
//   SCALE     : element (r, kc) times ks[z*s_ksz + kc]
//   CLAMP     : kc_n need not be a multiple of 16: in a partial slab k is clamped to the last
//               entry and entries past kc_n are zeroed.  Without CLAMP, every slab is read whole,
//               so kc_n must be a multiple of 16 or the rows padded with zeros up to one.
//   FLAT      : (KC only; no SCALE) the contraction index is flat, k = kb * kc_n + kc, and slab s
//               holds k in [16 s, 16 s + 16), running across kb blocks (kc_n >= 16: at most one
//               block boundary per slab), so kc_n need not be a multiple of 16 and no slab is
//               padded but the last of the whole contraction; slab numbers s_begin, s_end count
//               these flat slabs.
// Element q of a thread sits at base + eoff[q] with base uniform per slab, so without CLAMP a
// slab costs no per-element arithmetic.
template <class C, int R, bool KC, bool SCALE = false, bool CLAMP = true, bool FLAT = false>
struct Operand {
  static_assert(!FLAT || (KC && !SCALE), "flat contraction: lanes along k, no weights");
  static constexpr int E = R * C::BK / C::NT;
  uint32_t eoff[E];     // offset of element q from the slab base (row clamped to the last one)
  double v[E];
  double sc[SCALE ? E : 1];
  int kval;             // valid k entries of the slab set up by begin() (FLAT: entries before the block boundary)
  const double* base;
  const double* cur;    // start of the next slab to load (kept up to date by finish: no multiplies per slab)
  const double* ksb;
  int64_t zoff, kso;
  int64_t kb, kb_last;  // cursor: next slab to load is (kb, kc0)
  int kc0, kc_last;
  int64_t krem;         // FLAT: entries of the contraction from the next slab's start to its end
  int rem;              // FLAT: valid entries of the slab set up by begin()
  uint32_t dwrap;       // FLAT: s_kb - kc_n s_kc, from entry (kb, kc_n + j) to (kb + 1, j)

  __device__ __forceinline__ static int rr(int t, int q) {
    const int e = t + C::NT * q;
    return KC ? e / C::BK : e % R;
  }
  __device__ __forceinline__ static int kk(int t, int q) {
    const int e = t + C::NT * q;
    return KC ? e % C::BK : e / R;
  }
  // rows [r0, r0 + R) of batch z
  __device__ __forceinline__ void init(const OpMap& o, int64_t r0, int64_t z, int64_t s_begin, int64_t s_end,
                                       int t) {
    zoff = z * o.s_z;
    kso = z * o.s_ksz;
    if constexpr (FLAT) {
      const int64_t k0 = s_begin * C::BK, kl = (s_end - 1) * C::BK;
      kb = k0 / o.kc_n;
      kc0 = (int)(k0 - kb * o.kc_n);
      kb_last = kl / o.kc_n;
      kc_last = (int)(kl - kb_last * o.kc_n);
      krem = o.kb_n * o.kc_n - k0;
      dwrap = (uint32_t)(o.s_kb - o.kc_n * o.s_kc);
    } else {
      const int64_t nkc = (o.kc_n + C::BK - 1) / C::BK;
      kb = s_begin / nkc;
      kc0 = (int)(s_begin % nkc) * C::BK;
      kb_last = (s_end - 1) / nkc;
      kc_last = (int)((s_end - 1) % nkc) * C::BK;
    }
    cur = o.p + zoff + kb * o.s_kb + (int64_t)kc0 * o.s_kc;
#pragma unroll
    for (int q = 0; q < E; ++q) {
      const int64_t r = r0 + rr(t, q);
      const uint32_t rc = (uint32_t)(r < o.rows ? r : o.rows - 1);
      uint32_t rh = 0, rlo = rc;
      if (o.s_rh != 0) {
        rh = rc / (uint32_t)o.rl;
        rlo = rc - rh * (uint32_t)o.rl;
      }
      eoff[q] = rh * (uint32_t)o.s_rh + rlo * (uint32_t)o.s_rlo + (uint32_t)kk(t, q) * (uint32_t)o.s_kc;
    }
  }
  __device__ __forceinline__ void begin(const OpMap& o) {
    base = cur;
    kval = (int)o.kc_n - kc0;
    if constexpr (FLAT) rem = krem < C::BK ? (int)krem : C::BK;
    if constexpr (SCALE) ksb = o.ks + kso + kc0;
  }
  template <int q>
  __device__ __forceinline__ void load(const OpMap& o, int t) {
    if constexpr (FLAT) {
      // entries past the block boundary continue in the next kb block; entries past the end of
      // the contraction read the slab's first entry (row 0, in bounds; zeroed in store)
      const int kq = kk(t, q);
      const uint32_t off = eoff[q] + (kq >= kval ? dwrap : 0u);
      v[q] = base[kq < rem ? off : 0u];
    } else if constexpr (!CLAMP) {
      v[q] = base[eoff[q]];
      if constexpr (SCALE) sc[q] = ksb[kk(t, q)];
    } else {
      // entries past kc_n read the last valid k of the row instead (zeroed in store)
      const int over = kk(t, q) - (kval - 1);
      const uint32_t back = over > 0 ? (uint32_t)over * (uint32_t)o.s_kc : 0u;
      v[q] = base[eoff[q] - back];
      if constexpr (SCALE) sc[q] = ksb[min(kk(t, q), kval - 1)];
    }
  }
  __device__ __forceinline__ void finish(const OpMap& o) {
    // advance the cursor, but never past the last slab
    const bool at_end = kb == kb_last && kc0 == kc_last;
    if constexpr (FLAT) {
      int nkc = kc0 + C::BK;
      int64_t nkb = kb, step = (int64_t)C::BK * o.s_kc;
      if (nkc >= o.kc_n) {
        nkc -= (int)o.kc_n;
        ++nkb;
        step += o.s_kb - o.kc_n * o.s_kc;
      }
      kc0 = at_end ? kc0 : nkc;
      kb = at_end ? kb : nkb;
      cur = at_end ? cur : cur + step;
      krem = at_end ? krem : krem - C::BK;
      return;
    }
    int nkc = kc0 + C::BK;
    int64_t nkb = kb;
    // the next slab starts BK columns on, or at column 0 of the next kb block
    int64_t step = (int64_t)C::BK * o.s_kc;
    if (nkc >= o.kc_n) {
      nkc = 0;
      ++nkb;
      step = o.s_kb - (int64_t)kc0 * o.s_kc;
    }
    kc0 = at_end ? kc0 : nkc;
    kb = at_end ? kb : nkb;
    cur = at_end ? cur : cur + step;
  }
  template <int q>
  __device__ __forceinline__ void store(double* Sm, int t) const {
    const double x = SCALE ? v[q] * sc[q] : v[q];
    const int slot = rr(t, q) * C::LD + kk(t, q);
    if constexpr (FLAT) Sm[slot] = kk(t, q) < rem ? x : 0.0;
    else if constexpr (!CLAMP) Sm[slot] = x;
    else Sm[slot] = kk(t, q) < kval ? x : 0.0;
  }
};

// Source of a product with both operands from OpMaps over the same slab sequence.
template <class C, bool AK, bool BK, bool SCALE, bool CLAMP, bool FLAT = false>
struct PairSrc {
  static constexpr int EA = Operand<C, C::BM, AK, false, CLAMP, FLAT>::E;
  static constexpr int NL = EA + Operand<C, C::BN, BK, SCALE, CLAMP, FLAT>::E;
  Operand<C, C::BM, AK, false, CLAMP, FLAT> a;
  Operand<C, C::BN, BK, SCALE, CLAMP, FLAT> b;
  const OpMap* A;
  const OpMap* B;
  int t;
  __device__ __forceinline__ void begin() {
    a.begin(*A);
    b.begin(*B);
  }
  template <int q>
  __device__ __forceinline__ void load() {
    if constexpr (q < EA) a.template load<q>(*A, t);
    else b.template load<q - EA>(*B, t);
  }
  __device__ __forceinline__ void finish() {
    a.finish(*A);
    b.finish(*B);
  }
  template <int q>
  __device__ __forceinline__ void store(double* As, double* Bs) const {
    if constexpr (q < EA) a.template store<q>(As, t);
    else b.template store<q - EA>(Bs, t);
  }
};

// ---------------------------------------------------------------------------------------
// Generic tiled product  C(m, n) = sum_k A(m, k) B(n, k)  over a batch (grid z).  With grid
// y = nsplit > 1 each workgroup set covers a contiguous range of k slabs and writes its partial
// sums to part[split][M][N] (nz must be 1 then).
// Output tile (m0, n0) of batch z, split `split` of nsplit (partials to part when given).
template <class C, bool AK, bool BK, bool GEN, bool CLAMP>
__device__ __forceinline__ void gemm_tile(const OpMap& A, const OpMap& B, const OutMap& O, int64_t m0, int64_t n0,
                                          int64_t z, int nsplit, int split, double* part, double* smem) {
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int wm = wave % C::WM, wn = wave / C::WM;
  const int64_t nslab_all = A.kb_n * ((A.kc_n + C::BK - 1) / C::BK);
  const int64_t s0 = nslab_all * split / nsplit, s1 = nslab_all * (split + 1) / nsplit;

  d4 acc[C::TM][C::TN];
  zero_acc<C>(acc);
  if (s1 > s0) {
    PairSrc<C, AK, BK, false, CLAMP> src;
    src.A = &A;
    src.B = &B;
    src.t = t;
    src.a.init(A, m0, z, s0, s1, t);
    src.b.init(B, n0, z, s0, s1, t);
    mainloop<C>(src, smem, s1 - s0, acc, wm, wn, lane);
  }
  if (part) {
    const OutMap po = out_plain(part + (int64_t)split * O.M * O.N, O.M, O.N, O.N);
    store_tile<C, false>(po, 0, m0, n0, acc, wm, wn, lane);
  } else {
    store_tile<C, GEN>(O, z, m0, n0, acc, wm, wn, lane);
  }
}

template <class C, bool AK, bool BK, bool GEN, bool CLAMP>
__global__ void __launch_bounds__(C::NT) __attribute__((amdgpu_waves_per_eu(2))) gemm_kernel(OpMap A, OpMap B, OutMap O, int64_t tilesM, int64_t tilesN,
                                                     double* part) {
  __shared__ double smem[2 * C::STAGE];
  const int64_t tile = xcd_remap(blockIdx.x, tilesM * tilesN);
  const int64_t m0 = (tile % tilesM) * C::BM, n0 = (tile / tilesM) * C::BN;
  gemm_tile<C, AK, BK, GEN, CLAMP>(A, B, O, m0, n0, blockIdx.z, gridDim.y, blockIdx.y, part, smem);
}

// Rows in whole 64-row bands on 64 x 128 tiles and the rest (at most 32 rows) on 32 x 128 tiles, in one launch: per
// column block the band tiles, then the tail tile, the column block turning their order so that the short
// tiles do not all fall on the same shader engines (see half_tile).  Where the larger tiles would pad the
// rows by much more (see gemm_launch): 800 rows 896 -> 800 (the adjoint's S X at 800 x 3200 x 200 15.9 -> 14.5 ms).
typedef Cfg<2, 2, 2, 4, 3> CfgBand;
typedef Cfg<1, 4, 2, 2, 3> CfgBandTail;
template <bool AK, bool BK, bool CLAMP>
__global__ void __launch_bounds__(CfgBand::NT) __attribute__((amdgpu_waves_per_eu(CfgBand::WPE))) gemm_band_kernel(OpMap A, OpMap B, OutMap O, int64_t nband, int64_t per,
                                                          int64_t tilesN, double* part) {
  static_assert(CfgBandTail::NT == CfgBand::NT && CfgBandTail::BN == CfgBand::BN && CfgBandTail::STAGE <= CfgBand::STAGE,
                "one workgroup shape and column block");
  __shared__ double smem[2 * CfgBand::STAGE];
  const int64_t tile = xcd_remap(blockIdx.x, per * tilesN);
  const int64_t c = tile / per, i = (tile + c) % per, n0 = c * CfgBand::BN;
  if (i < nband)
    gemm_tile<CfgBand, AK, BK, false, CLAMP>(A, B, O, i * CfgBand::BM, n0, blockIdx.z, gridDim.y, blockIdx.y, part, smem);
  else
    gemm_tile<CfgBandTail, AK, BK, false, CLAMP>(A, B, O, nband * CfgBand::BM, n0, blockIdx.z, gridDim.y, blockIdx.y, part, smem);
}

// Row i and column j <= i of packed pair p = i(i+1)/2 + j.
__device__ __forceinline__ void pair_ij(int64_t p, int64_t* i, int64_t* j) {
  int64_t r = (int64_t)((sqrt(8.0 * (double)p + 1.0) - 1.0) * 0.5);
  while (r * (r + 1) / 2 > p) --r;
  while ((r + 1) * (r + 2) / 2 <= p) ++r;
  *i = r;
  *j = p - r * (r + 1) / 2;
}

// Gram matrix  G(m, n) = sum_k A(m, k) A(n, k): the tiles on and below the diagonal only (tile pair I >= J
// of the triangle), lanes along the rows of A.  Without a split a tile is stored to G and, mirrored,
// to the transposed place (accumulate adds to both); with one the partial sums go to part [split][M][M],
// lower tiles only, for syrk_reduce.  Half the MFMAs of the full product; bound by the matrix cores and its last round
// (6000 rows over 2000: 1128 workgroups, 2.2 rounds, busy 0.67).
template <class C, bool CLAMP>
__global__ void __launch_bounds__(C::NT) __attribute__((amdgpu_waves_per_eu(2))) gram_kernel(OpMap A, double* G, int64_t npairs, int accumulate, double* part) {
  static_assert(C::BM == C::BN, "square tiles");
  __shared__ double smem[2 * C::STAGE];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int wm = wave % C::WM, wn = wave / C::WM;
  int64_t I, J;
  pair_ij(xcd_remap(blockIdx.x, npairs), &I, &J);
  const int64_t m0 = I * C::BM, n0 = J * C::BN, M = A.rows;
  const int nsplit = gridDim.y, split = blockIdx.y;
  const int64_t S = A.kb_n * ((A.kc_n + C::BK - 1) / C::BK), s0 = S * split / nsplit, s1 = S * (split + 1) / nsplit;
  d4 acc[C::TM][C::TN];
  zero_acc<C>(acc);
  if (s1 > s0) {
    PairSrc<C, false, false, false, CLAMP> src;
    src.A = &A;
    src.B = &A;
    src.t = t;
    src.a.init(A, m0, 0, s0, s1, t);
    src.b.init(A, n0, 0, s0, s1, t);
    mainloop<C>(src, smem, s1 - s0, acc, wm, wn, lane);
  }
  if (part) {
    store_tile<C, false>(out_plain(part + (int64_t)split * M * M, M, M, M), 0, m0, n0, acc, wm, wn, lane);
    return;
  }
  // A lane's column index is lane % 16 and its rows come four apart, so the mirrored stores write runs
  // of four doubles; the four of a block fill its 128-byte lines in L2.
  const int lr = lane & 15, lg = lane >> 4;
#pragma unroll
  for (int i = 0; i < C::TM; ++i)
#pragma unroll
    for (int j = 0; j < C::TN; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t m = m0 + (wm * C::TM + i) * 16 + 4 * r + lg, n = n0 + (wn * C::TN + j) * 16 + lr;
        if (m >= M || n > m) continue;   // each pair from its lower element
        double *a = G + m * M + n, *b = G + n * M + m;
        const double x = acc[i][j][r];
        const double xa = accumulate ? *a + x : x, xb = accumulate ? *b + x : x;
        *a = xa;
        *b = xb;
      }
}

// Rows in whole 128-row bands on 128 x 128 tiles and the rest (at most 64 rows) on 64 x 128 tiles
// (4 waves of 64 x 32), in one launch: per column block the band tiles, then the tail tile.
// Where the 256 x 128 or 128 x 128 tiles would pad the rows by more than 64 (1200 rows: 1280).
typedef Cfg<1, 4, 4, 2> CfgRowTail;
template <bool AK, bool BK>
__global__ void __launch_bounds__(CfgSq::NT) __attribute__((amdgpu_waves_per_eu(2))) gemm_tail_kernel(OpMap A, OpMap B, OutMap O, int64_t nband, int64_t tilesN) {
  static_assert(CfgRowTail::NT == CfgSq::NT && CfgRowTail::BN == CfgSq::BN && CfgRowTail::STAGE <= CfgSq::STAGE,
                "one workgroup shape and column block");
  __shared__ double smem[2 * CfgSq::STAGE];
  const int64_t per = nband + 1;
  const int64_t tile = xcd_remap(blockIdx.x, per * tilesN);
  const int64_t i = tile % per, n0 = (tile / per) * CfgSq::BN;
  if (i < nband)
    gemm_tile<CfgSq, AK, BK, false, false>(A, B, O, i * CfgSq::BM, n0, 0, 1, 0, nullptr, smem);
  else
    gemm_tile<CfgRowTail, AK, BK, false, false>(A, B, O, nband * CfgSq::BM, n0, 0, 1, 0, nullptr, smem);
}

// Sum over s < nsplit of q[s * stride] by the G threads of a column (thread y takes s = y, y + G,
// ...; then the G partial sums in order): the same order for every launch.  256 threads, 256 / G
// columns; every thread calls it, and the threads with y == 0 hold the sum.  Bound by latency when
// the splits are many and the columns few (a thread per column took 123 us for 77 x 77 over 310
// splits), so G = 8 from 8 splits on; below that the extra threads would find nothing to add.
constexpr int kRedThreads = 256;
template <int G>
__device__ __forceinline__ double split_sum(const double* q, int nsplit, int64_t stride, bool live) {
  constexpr int W = kRedThreads / G;
  const int x = threadIdx.x % W, y = threadIdx.x / W;
  double s = 0.0;
  if (live) {
#pragma unroll 4
    for (int sp = y; sp < nsplit; sp += G) s += q[(int64_t)sp * stride];
  }
  if constexpr (G == 1) return s;
  __shared__ double red[G][W];
  red[y][x] = s;
  __syncthreads();
  double r = 0.0;
  if (y == 0)
#pragma unroll
    for (int g = 0; g < G; ++g) r += red[g][x];
  return r;
}
static inline int red_group(int nsplit) { return nsplit >= 8 ? 8 : 1; }

// C(m, n) = alpha * sum_s part[s][m][n] (+ C), fixed order over s.
template <int G>
__global__ void __launch_bounds__(kRedThreads) split_reduce_kernel(const double* __restrict__ part, int nsplit, OutMap O) {
  constexpr int W = kRedThreads / G;
  const int64_t idx = (int64_t)blockIdx.x * W + threadIdx.x % W;
  const int64_t MN = O.M * O.N;
  const double s = split_sum<G>(part + idx, nsplit, MN, idx < MN);
  if (threadIdx.x >= W || idx >= MN) return;
  const int64_t m = idx / O.N, n = idx % O.N;
  double* dst;
  if (n < O.nsplit) {
    dst = O.p + (m / O.ml) * O.s_mh + (m % O.ml) * O.s_ml + (n / O.nl) * O.s_nh + (n % O.nl) * O.s_nl;
  } else {
    dst = O.p2 + m * O.s2_m + (n - O.nsplit);
  }
  *dst = O.accumulate ? *dst + O.alpha * s : O.alpha * s;
}

// Rows m of sums over packed pairs (u >= v of nac orbitals), spread over the full square:
//   q(m, (u, v)) = q(m, (v, u)) = sum_s part[s][m][pair(max, min)],
// rows m < M1 to out1[m][nac][nac], the rest to out2[m - M1][nac][nac] (either may be null); fixed
// order over s.  A workgroup takes `rpb` rows; the reads of a row repeat within it and stay in L1.
__global__ void __launch_bounds__(256) expand_pairs_kernel(const double* __restrict__ part, int nsplit, int64_t M,
                                                           int nac, int rpb, double* __restrict__ out1, int64_t M1,
                                                           double* __restrict__ out2, int accumulate) {
  const int n2 = nac * nac, nuv = nac * (nac + 1) / 2;
  const int64_t m0 = (int64_t)blockIdx.x * rpb, stride = M * nuv;
  const int rows = (int)(M - m0 < rpb ? M - m0 : rpb);
  for (int idx = threadIdx.x; idx < rows * n2; idx += 256) {
    const int r = idx / n2, e = idx - r * n2, u = e / nac, v = e - u * nac;
    const int64_t m = m0 + r;
    double* dst = m < M1 ? out1 : out2;
    if (!dst) continue;
    dst += (m < M1 ? m : m - M1) * n2 + e;
    const int i = u > v ? u : v, j = u > v ? v : u;
    const double* q = part + m * nuv + i * (i + 1) / 2 + j;
    double s = 0.0;
#pragma unroll 4
    for (int sp = 0; sp < nsplit; ++sp) s += q[sp * stride];
    *dst = accumulate ? *dst + s : s;
  }
}

// ---------------------------------------------------------------------------------------
// Lower-triangle tile SYRK with the contraction split over workgroups: one (tile, split) item of density z,
//   Kpart[split][z] tile (m0, n0) = sum_{kb in split} sum_kc A(i, kb, kc) Bw(j, kb, kc),
// where Bw is A times an optional per-kc weight.  FLAT: the contraction (kb, kc) runs as one flat
// index in slabs of 16 (see Operand) and the flat slabs are split evenly, so no kb block is padded
// to whole slabs; otherwise the kb range is split and each block padded.
template <class C, bool SCALE, bool CLAMP, bool FLAT>
__device__ __forceinline__ void syrk_run(const OpMap& A, const OpMap& Bw, int64_t n, int64_t nz, int nsplit,
                                         int split, int64_t m0, int64_t n0, double* Kpart, int64_t z, double* smem) {
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int wm = wave % C::WM, wn = wave / C::WM;
  int64_t s_lo, s_hi;   // slabs of this split
  if constexpr (FLAT) {
    const int64_t S = (A.kb_n * A.kc_n + C::BK - 1) / C::BK;
    s_lo = S * split / nsplit;
    s_hi = S * (split + 1) / nsplit;
  } else {
    const int64_t nkc = (A.kc_n + C::BK - 1) / C::BK;
    s_lo = A.kb_n * split / nsplit * nkc;
    s_hi = A.kb_n * (split + 1) / nsplit * nkc;
  }

  d4 acc[C::TM][C::TN];
  zero_acc<C>(acc);
  const int64_t nslab = s_hi - s_lo;
  if (nslab > 0) {
    PairSrc<C, true, true, SCALE, CLAMP, FLAT> src;
    src.A = &A;
    src.B = &Bw;
    src.t = t;
    src.a.init(A, m0, z, s_lo, s_hi, t);
    src.b.init(Bw, n0, z, s_lo, s_hi, t);
    mainloop<C>(src, smem, nslab, acc, wm, wn, lane);
  }
  OutMap o = out_plain(Kpart + ((int64_t)split * nz + z) * n * n, n, n, n);
  store_tile<C, false>(o, 0, m0, n0, acc, wm, wn, lane);
}

// Tiles of the lower triangle of an n x n SYRK, and their splits of the contraction.  Band i of `bands` 64-row
// bands needs columns 0 ... 64 (i + 1): (i + 1) / 2 tiles of 64 x 128 (A) and, in even bands, one of
// 64 x 64 on the diagonal (D); the rows past the bands take tiles of 32 x 128 (T).  Each kind has its own split
// count, in proportion to the time of its tiles, so that all work items take about as long, or twice that for D and
// T where the items are long: the chain of sums of a D item would be 1.7 times an A item's, and the diagonal is
// the largest part of K.  (Relative error of K at 1200 x 4800 x 300 1.6e-15 so, 8.3e-16 with 37 equal chains,
// 7.7e-16 now; at 800 6.9e-16, 4.0e-16, 3.1e-16.)  Bound by the
// matrix cores (busy 0.78 at 1200 x 4800 x 300, 0.69 at 600 x 2400 x 150) and the padding of the triangle.  Against square tiles of 64 (128 past n = 640): K at
// 341 x 1365 x 85 0.41 -> 0.38 ms, 600 x 2400 x 150 3.30 -> 3.03, 700 x 1400 x 128 1.91 -> 1.52, 1200 x 1200 x 300
// 10.5 -> 9.8.  128 x 128 tiles with 64-row tails: 2.98 at 600, 1.69 at 700.
struct SyrkTiles {
  int bands;              // 0: every element has na partials (launch_syrk_reduce)
  int a, d, t;            // tiles of each kind
  int na, nd, nt;         // splits of each kind
  __host__ __device__ int64_t items() const { return (int64_t)a * na + (int64_t)d * nd + (int64_t)t * nt; }
};

// Items: the A tiles of split 0, of split 1, ..., then the D tiles so, then the T tiles; the items of each kind are dealt
// to the XCDs by themselves (all in one row, the last XCDs got the D and T items alone).
template <bool SCALE, bool CLAMP, bool FLAT>
__global__ void __launch_bounds__(CfgKA::NT) __attribute__((amdgpu_waves_per_eu(CfgKA::WPE))) syrk_kernel(OpMap A, OpMap Bw, int64_t n, int64_t nz, SyrkTiles T,
                                                     double* Kpart) {
  static_assert(CfgKD::STAGE <= CfgKA::STAGE && CfgKT::STAGE <= CfgKA::STAGE, "the A tile's LDS holds the others");
  __shared__ double smem[2 * CfgKA::STAGE];
  const int64_t id = blockIdx.x, z = blockIdx.z;
  const int64_t na = (int64_t)T.a * T.na, nd = (int64_t)T.d * T.nd, nad = na + nd;
  if (id < na) {
    const int64_t item = xcd_remap(id, na);
    const int q = (int)(item % T.a);
    int i = (int)(2.0f * sqrtf((float)q));   // i^2 / 4 A tiles lie in the bands before band i
    while (i * i / 4 > q) --i;
    while ((i + 1) * (i + 1) / 4 <= q) ++i;
    syrk_run<CfgKA, SCALE, CLAMP, FLAT>(A, Bw, n, nz, T.na, (int)(item / T.a), (int64_t)i * CfgKA::BM,
                                        (int64_t)(q - i * i / 4) * CfgKA::BN, Kpart, z, smem);
  } else if (id < nad) {
    const int64_t item = xcd_remap(id - na, nd), m0 = item % T.d * 2 * CfgKD::BM;
    syrk_run<CfgKD, SCALE, CLAMP, FLAT>(A, Bw, n, nz, T.nd, (int)(item / T.d), m0, m0, Kpart, z, smem);
  } else {
    const int64_t item = xcd_remap(id - nad, (int64_t)T.t * T.nt);
    syrk_run<CfgKT, SCALE, CLAMP, FLAT>(A, Bw, n, nz, T.nt, (int)(item / T.t), (int64_t)T.bands * CfgKA::BM,
                                        item % T.t * CfgKT::BN, Kpart, z, smem);
  }
}

// Grouped K SYRK on square tiles (64 x 64 at fragment sizes: four workgroups per CU and a batch's X, much
// larger than the caches, read once; 92.5 ms for the 64-density fragments against 97 on SyrkTiles):
// problem p owns items [start[p], start[p + 1]) = (density z, split, tile pair), z outermost; unit weights.
struct SyrkDesc {
  OpMap A;
  int64_t n, nz, npairs;
  double* Kpart;
  int nsplit;
};
struct SyrkGroup {
  int n;
  int64_t start[kMaxGroup + 1];
  int64_t xs[9];   // items of XCD x: [xs[x], xs[x + 1])
  SyrkDesc d[kMaxGroup];
};

// With the per-XCD chunks of half_group_kernel.
template <class C, bool CLAMP, bool FLAT = false>
__global__ void __launch_bounds__(C::NT) syrk_group_kernel(SyrkGroup g) {
  __shared__ double smem[2 * C::STAGE];
  const int x = blockIdx.x % 8;
  const int64_t it = g.xs[x] + blockIdx.x / 8;
  if (it >= g.xs[x + 1]) return;
  int p = 0;
  while (p + 1 < g.n && it >= g.start[p + 1]) ++p;
  const SyrkDesc& d = g.d[p];
  const int64_t item = it - g.start[p], per_z = d.npairs * d.nsplit;
  const int64_t in_z = item % per_z;
  int64_t I, J;
  pair_ij(in_z % d.npairs, &I, &J);
  syrk_run<C, false, CLAMP, FLAT>(d.A, d.A, d.n, d.nz, d.nsplit, (int)(in_z / d.npairs), I * C::BM, J * C::BN, d.Kpart,
                                  item / per_z, smem);
}

// K[z][i][j] and K[z][j][i] (+)= sum_s Kpart[s][z][i][j] for the lower pairs i >= j, G threads each, over
// the splits of the pair's tile (SyrkTiles).
template <int G>
__global__ void __launch_bounds__(kRedThreads) syrk_reduce_kernel(const double* __restrict__ Kpart, SyrkTiles T,
                                                                  int64_t n, int64_t npair, double* __restrict__ K,
                                                                  int accumulate) {
  constexpr int W = kRedThreads / G;
  const int64_t p = (int64_t)blockIdx.x * W + threadIdx.x % W, z = blockIdx.y, nz = gridDim.y, nn = n * n;
  int64_t i = 0, j = 0;
  if (p < npair) pair_ij(p, &i, &j);
  int nsplit = T.na;
  if (T.bands > 0) {
    const int band = (int)(i / CfgKA::BM);
    if (band >= T.bands) nsplit = T.nt;
    else if (band % 2 == 0 && j >= (int64_t)band * CfgKA::BM) nsplit = T.nd;
  }
  const double s = split_sum<G>(Kpart + z * nn + i * n + j, nsplit, nz * nn, p < npair);
  if (threadIdx.x >= W || p >= npair) return;
  double* a = K + z * nn + i * n + j;
  double* b = K + z * nn + j * n + i;
  const double x = accumulate ? *a + s : s, y = accumulate ? *b + s : s;
  *a = x;
  *b = y;
}

// ---------------------------------------------------------------------------------------
// Half transform of one packed, symmetric b^P against a dense C.
// A operand element (m, k) = b^P_{mk}, packed at T(max(m, k)) + min(m, k), T(i) = i(i+1)/2.
// A slab wholly below the diagonal of its row band (k0 + 15 <= m0: every k <= every m) is read
// along k, as 16-element runs of packed rows m: T(m) + k0 + (t % 16), a uniform base plus a
// per-thread constant.  Any other slab is read along m through (max, min); there k is uniform
// per wave and element, so T(k) is scalar work.  Both addresses are formed and a uniform select
// picks one.  The dense operand (C, or Y in the P-summed form) is read without clamping: its k
// extent must be padded with zero rows to a multiple of 16, which also cancels the clamped
// duplicates of b^P read for k past the end.  Packed offsets stay in 32 bits (nao <= 46340).
template <class C>
struct HalfSrc {
  static constexpr int EA = C::BM * C::BK / C::NT;
  static constexpr int NL = EA + Operand<C, C::BN, false, false, false>::E;
  static_assert(C::NT % C::BK == 0 && C::NT % C::BM == 0, "per-thread row / column of the A loads");
  static constexpr bool UK = C::BM % 64 == 0;   // t / BM is the same for all lanes of a wave
  Operand<C, C::BN, false, false, false> c;
  const OpMap* Cm;
  const double* Bbase;  // packed b^P of the current P: Bbase + P*npair
  const double* Bp;
  int64_t npair, P, P_last;
  unsigned last;        // nao - 1
  int m0, t, nks, ks;   // k slabs per P, current k slab
  unsigned k0, kw;      // slab start; k offset t / BM of the along-m mapping (wave-uniform with UK)
  bool below;
  uint32_t offB[EA];    // along-k mapping: T(m) + t % 16 for row m = m0 + e / 16 (clamped)
  uint32_t mAc, mAoff;  // along-m mapping: row m0 + t % BM (clamped) and T of it
  double va[EA];

  // slabs run over P in [P0, P1) (outer) and the k chunks of nao (inner)
  __device__ __forceinline__ void init(const double* B, int64_t npair_, int64_t P0, int64_t P1, int nao, int m0_,
                                       int t_) {
    Bbase = B;
    npair = npair_;
    P = P0;
    P_last = P1 - 1;
    last = (unsigned)nao - 1u;
    m0 = m0_;
    t = t_;
    nks = (nao + C::BK - 1) / C::BK;
    ks = 0;
    Bp = Bbase + P * npair;
#pragma unroll
    for (int q = 0; q < EA; ++q) {
      const unsigned m = (unsigned)(m0 + (t + C::NT * q) / C::BK);
      const unsigned mc = m <= last ? m : last;
      offB[q] = mc * (mc + 1u) / 2u + (unsigned)(t % C::BK);
    }
    const unsigned mA = (unsigned)(m0 + t % C::BM);
    mAc = mA <= last ? mA : last;
    mAoff = mAc * (mAc + 1u) / 2u;
    kw = UK ? (unsigned)__builtin_amdgcn_readfirstlane(t / C::BM) : (unsigned)(t / C::BM);
  }
  __device__ __forceinline__ void begin() {
    k0 = (unsigned)ks * C::BK;
    below = (int)k0 + C::BK - 1 <= m0;
    c.begin(*Cm);
  }
  template <int q>
  __device__ __forceinline__ void load() {
    if constexpr (q < EA) {
      const unsigned kr = k0 + kw + (unsigned)(q * (C::NT / C::BM));
      const unsigned kc = kr <= last ? kr : last;
      const unsigned Tk = kc * (kc + 1u) / 2u;
      // bit-mask blends: conditionals here compile to a divergent branch (per lane) or to uniform
      // branches (on `below`) per load
      const unsigned sel = 0u - (unsigned)(mAc >= kc);
      const unsigned other = ((mAoff + kc) & sel) | ((Tk + mAc) & ~sel);
      const unsigned bsel = 0u - (unsigned)below;
      va[q] = Bp[((offB[q] + k0) & bsel) | (other & ~bsel)];
    } else {
      c.template load<q - EA>(*Cm, t);
    }
  }
  __device__ __forceinline__ void finish() {
    const bool at_end = P == P_last && ks == nks - 1;
    int nk = ks + 1;
    int64_t nP = P;
    if (nk == nks) {
      nk = 0;
      ++nP;
    }
    ks = at_end ? ks : nk;
    Bp = at_end || nP == P ? Bp : Bp + npair;
    P = at_end ? P : nP;
    c.finish(*Cm);
  }
  template <int q>
  __device__ __forceinline__ void store(double* As, double* Bs) const {
    if constexpr (q < EA) {
      const int e = t + C::NT * q;
      As[below ? (e / C::BK) * C::LD + e % C::BK : (e % C::BM) * C::LD + e / C::BM] = va[q];
    } else {
      c.template store<q - EA>(Bs, t);
    }
  }
};

// The J-vector of Eq. (J_1) formed in the half transform's epilogue: with X_P = b^P C the tile
// just computed, v_P = sum_{m < nao, c < nv} X_P[m][c] C[m][c] w[c] (w NULL: all ones), since
// sum_c X_P[m][c] C[m][c] w[c] summed over m is <b^P, C diag(w) C^T>.  Each tile leaves its
// partial sum in part[P * tiles + tile]; jv_reduce_kernel adds them up in a fixed order.
struct JvEpi {
  const double* C;   // C[m * ldc + c], the operand of the half transform (L2-resident: the main loop read it)
  int64_t ldc;
  const double* w;
  int nv;
  double* part;      // partial of tile `tile` of P at part[P * T + tile]
  int64_t T;
};

// The output tile of b^P at (m0, n0); with JV its J-vector partial goes to slot `tile` of P.
template <class C, bool GEN = false, bool JV = false>
__device__ __forceinline__ void half_tile_at(const double* __restrict__ B, int nao, int64_t npair, const OpMap& Cm,
                                             const OutMap& out, int64_t P, int m0, int n0, int64_t tile,
                                             double* smem, const JvEpi* jv) {
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int wm = wave % C::WM, wn = wave / C::WM;
  const int nslab = (nao + C::BK - 1) / C::BK;

  HalfSrc<C> src;
  src.Cm = &Cm;
  src.c.init(Cm, n0, 0, 0, nslab, t);
  src.init(B, npair, P, P + 1, nao, m0, t);
  d4 acc[C::TM][C::TN];
  zero_acc<C>(acc);
  mainloop<C>(src, smem, nslab, acc, wm, wn, lane);
  store_tile<C, GEN>(out, P, m0, n0, acc, wm, wn, lane);
  if constexpr (JV) {
    const int lr = lane & 15, lg = lane >> 4;
    double s = 0.0;
    // rows past the end read the last one and columns past nv column 0, both dropped by a select: the loads are
    // branch-free, so eight of a column block are in flight together.  (All sixteen of a 128-row tile, and the next
    // block's moved up, spilled 38 registers: 84.5 ms at 1200 x 4800 x 340 instead of 83.8.)
    constexpr int NQ = C::TM * 4, JB = NQ < 8 ? NQ : 8;
#pragma unroll
    for (int j = 0; j < C::TN; ++j) {
      const int n = n0 + (wn * C::TN + j) * 16 + lr;
      const bool nok = n < jv->nv;
      const int nc = nok ? n : 0;
      const double wc = nok ? (jv->w ? jv->w[nc] : 1.0) : 0.0;
      double sj = 0.0;
#pragma unroll
      for (int h = 0; h < NQ; h += JB) {
        double cm[JB];
#pragma unroll
        for (int e = 0; e < JB; ++e) {
          const int q = h + e, m = m0 + (wm * C::TM + q / 4) * 16 + 4 * (q % 4) + lg;
          cm[e] = jv->C[(int64_t)(m < nao ? m : nao - 1) * jv->ldc + nc];
        }
#pragma unroll
        for (int e = 0; e < JB; ++e) {
          const int q = h + e, m = m0 + (wm * C::TM + q / 4) * 16 + 4 * (q % 4) + lg;
          sj = m < nao ? fma(acc[q / 4][j][q % 4], cm[e], sj) : sj;
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      s = fma(sj, wc, s);
    }
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
    __syncthreads();   // the main loop's last LDS reads are done before smem is reused
    if (lane == 0) smem[wave] = s;
    __syncthreads();
    if (t == 0) {
      double r = 0.0;
      for (int q = 0; q < C::WM * C::WN; ++q) r += smem[q];
      jv->part[P * jv->T + tile] = r;
    }
  }
}

// Tiles of the half transform of one P: nA tiles of CA per 64-row band from column 0, one of CB
// (nB = 1) on the columns from nA CA::BN on, and nT tiles of CT, along the columns, on the rows past the
// `bands` bands.
struct HalfTiles {
  int bands, nA, nB, nT;
  __host__ __device__ int64_t count() const { return (int64_t)bands * (nA + nB) + nT; }
};

// Tile of work item `item`.  Band by band, so that the column tiles of a band run side by side and share
// its reads in L2, then the tiles of CT.  Consecutive workgroups go to the four shader engines of an XCD in turn:
// with an even number of column tiles, the last one short, some engines would get all the short ones
// (600 x 170 columns ran 7.8 ms so, 500 x 140 4.4).  The bands therefore turn their tiles so that the short ones fall on
// every engine alike (5.9 and 3.0 ms); without CB tiles P turns the whole order, for the CT tiles (455 x 226
// columns 3.73 -> 3.60 ms).
template <class CA, class CB, class CT, bool GEN, bool JV>
__device__ __forceinline__ void half_tile(const double* __restrict__ B, int nao, int64_t npair, const OpMap& Cm,
                                          const OutMap& out, const HalfTiles& T, int64_t item, double* smem,
                                          const JvEpi* jv = nullptr) {
  static_assert(CA::NT == CB::NT && CA::NT == CT::NT && CA::BM == CB::BM, "one workgroup shape, one band");
  constexpr bool kB = !std::is_same<CA, CB>::value, kT = !std::is_same<CA, CT>::value;
  const int64_t ntile = T.count(), P = item / ntile;
  const int per = T.nA + T.nB;
  int tile = (int)(item % ntile);
  if (kT && T.nB == 0) tile = (int)((tile + P) % ntile);
  const int band = tile / per;
  if (kT && band >= T.bands) {
    half_tile_at<CT, GEN, JV>(B, nao, npair, Cm, out, P, T.bands * CA::BM, (tile - T.bands * per) * CT::BN, tile, smem, jv);
    return;
  }
  int j = tile % per;
  if (kB && per % 2 == 0) j = (int)((unsigned)(j + (per % 4 == 0 ? band : band >> 1) + (int)(P & 0xffff)) % (unsigned)per);
  if (!kB || j < T.nA)
    half_tile_at<CA, GEN, JV>(B, nao, npair, Cm, out, P, band * CA::BM, j * CA::BN, tile, smem, jv);
  else if constexpr (kB)
    half_tile_at<CB, GEN, JV>(B, nao, npair, Cm, out, P, band * CA::BM, T.nA * CA::BN, tile, smem, jv);
}

template <class CA, class CB, class CT>
struct HalfLds {
  static constexpr int A = CA::STAGE > CB::STAGE ? CA::STAGE : CB::STAGE;
  static constexpr int N = 2 * (A > CT::STAGE ? A : CT::STAGE);
};

// GEN: the epilogue applies out.alpha and out.accumulate (a separate instantiation, see store_tile);
// JV: the J-vector partials are formed in it (JvEpi).
template <class CA, class CB, class CT, bool GEN, bool JV>
__global__ void __launch_bounds__(CA::NT) __attribute__((amdgpu_waves_per_eu(CA::WPE))) half_kernel(const double* __restrict__ B, int64_t naux, int nao,
                                                     int64_t npair, OpMap Cm, OutMap out, HalfTiles T, JvEpi jv) {
  __shared__ double smem[HalfLds<CA, CB, CT>::N];
  half_tile<CA, CB, CT, GEN, JV>(B, nao, npair, Cm, out, T, xcd_remap(blockIdx.x, T.count() * naux), smem, &jv);
}

// v[P] (+)= sum_{t < tiles} part[P * tiles + t], four sums over every fourth tile, then those in order: one chain over the
// tiles of 64-row bands is twice as long as over 128-row ones (relative error of v at 1000 x 4000 x 250 4.38e-16 so,
// 4.23e-16 then, 4.12e-16 now).
__global__ void __launch_bounds__(256) jv_reduce_kernel(const double* __restrict__ part, int64_t tiles, int64_t naux,
                                                        double* __restrict__ v, int accumulate) {
  const int64_t P = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (P >= naux) return;
  const double* q = part + P * tiles;
  double r[4] = {0.0, 0.0, 0.0, 0.0};
  int64_t t = 0;
  for (; t + 4 <= tiles; t += 4)
#pragma unroll
    for (int j = 0; j < 4; ++j) r[j] += q[t + j];
#pragma unroll
  for (int j = 0; j < 3; ++j)
    if (t + j < tiles) r[j] += q[t + j];
  const double s = (r[0] + r[1]) + (r[2] + r[3]);
  v[P] = accumulate ? v[P] + s : s;
}

// Grouped half transform over several problems in one launch.  Work items of problem p are
// [start[p], start[p + 1]); problems are listed largest first, so the big ones start first and
// the small ones fill in behind them.
struct HalfDesc {
  const double* B;
  int64_t npair;
  OpMap Cm;
  OutMap out;
  int nao;
  HalfTiles T;
};
struct HalfGroup {
  int n;
  int64_t start[kMaxGroup + 1];
  int64_t xs[9];   // items of XCD x: [xs[x], xs[x + 1])
  HalfDesc d[kMaxGroup];
};

// Grouped launches: the item list is cut into 8 contiguous chunks of about equal cost, one per
// XCD.  The dispatcher deals workgroups to the 8 XCDs in turn, so workgroup b runs on XCD b % 8
// and takes item b / 8 of that XCD's chunk (workgroups past the end of their chunk exit):
// consecutive items run side by side on one XCD and share its L2, and every XCD gets the same
// work although the items of different problems differ in cost.  (A persistent grid striding
// through the chunks balanced uneven items worse than the dispatcher does.)
template <class CA, class CB, class CT>
__global__ void __launch_bounds__(CA::NT) __attribute__((amdgpu_waves_per_eu(CA::WPE))) half_group_kernel(HalfGroup g) {
  __shared__ double smem[HalfLds<CA, CB, CT>::N];
  const int x = blockIdx.x % 8;
  const int64_t item = g.xs[x] + blockIdx.x / 8;
  if (item >= g.xs[x + 1]) return;
  int p = 0;
  while (p + 1 < g.n && item >= g.start[p + 1]) ++p;
  const HalfDesc& d = g.d[p];
  half_tile<CA, CB, CT, false, false>(d.B, d.nao, d.npair, d.Cm, d.out, d.T, item - g.start[p], smem);
}

// part[split] (m, n) = sum_{P in split} sum_k b^P_{mk} Y(n, (P, k)): the packed half-transform
// product with the right operand changing with P and the P sum split over workgroups.  The tiles are
// those of half_kernel in up to three regions of the output (CA, CB and CT tiles), each with its own
// split count, so that the items of all take about the same time, and its own partials
// [ns][r1 - r0][c1 - c0].  (With one count for all, 1200 x 300 took 98 ms in four rounds of uneven
// items, 75 in three launches.)
struct ReduceRegion {
  int64_t item0;                    // first work item
  int r0, r1, c0, c1, tilesM, tilesN, ns;
  double* part;
};
struct ReduceRegions {
  ReduceRegion a, b, t;
  int64_t items;
};

template <class C>
__device__ __forceinline__ void half_reduce_tile(const double* __restrict__ B, int64_t naux, int nao, int64_t npair,
                                                 const OpMap& Y, const ReduceRegion& g, int64_t item, double* smem) {
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int wm = wave % C::WM, wn = wave / C::WM;
  const int nks = (nao + C::BK - 1) / C::BK;
  // split major, then row band: the tiles of one P range sit on one XCD, and the column tiles
  // of a band side by side
  const int64_t ntile = (int64_t)g.tilesM * g.tilesN;
  const int split = (int)(item / ntile), tile = (int)(item % ntile);
  const int m0 = g.r0 + tile / g.tilesN * C::BM, n0 = g.c0 + tile % g.tilesN * C::BN;
  const int64_t P0 = naux * split / g.ns, P1 = naux * (split + 1) / g.ns;
  d4 acc[C::TM][C::TN];
  zero_acc<C>(acc);
  if (P1 > P0) {
    HalfSrc<C> src;
    src.Cm = &Y;
    src.c.init(Y, n0, 0, P0 * nks, P1 * nks, t);
    src.init(B, npair, P0, P1, nao, m0, t);
    mainloop<C>(src, smem, (P1 - P0) * nks, acc, wm, wn, lane);
  }
  const int rows = g.r1 - g.r0, cols = g.c1 - g.c0;
  store_tile<C, false>(out_plain(g.part + (int64_t)split * rows * cols, rows, cols, cols), 0, m0 - g.r0, n0 - g.c0, acc,
                       wm, wn, lane);
}

template <class CA, class CB, class CT>
__global__ void __launch_bounds__(CA::NT) __attribute__((amdgpu_waves_per_eu(CA::WPE))) half_reduce_kernel(const double* __restrict__ B, int64_t naux, int nao,
                                                            int64_t npair, OpMap Y, ReduceRegions R) {
  __shared__ double smem[HalfLds<CA, CB, CT>::N];
  constexpr bool kB = !std::is_same<CA, CB>::value, kT = !std::is_same<CA, CT>::value;
  // each region dealt to the XCDs by itself: in one row, the last XCDs would get the short items alone
  const int64_t id = blockIdx.x;
  if (!(kB || kT) || id < R.b.item0)
    half_reduce_tile<CA>(B, naux, nao, npair, Y, R.a, xcd_remap(id, kB || kT ? R.b.item0 : R.items), smem);
  else if (kB && (!kT || id < R.t.item0))
    half_reduce_tile<CB>(B, naux, nao, npair, Y, R.b, xcd_remap(id - R.b.item0, R.t.item0 - R.b.item0), smem);
  else if constexpr (kT)
    half_reduce_tile<CT>(B, naux, nao, npair, Y, R.t, xcd_remap(id - R.t.item0, R.items - R.t.item0), smem);
}

// ---------------------------------------------------------------------------------------
// v[z][P] = sum_{m, c} C[z][m][c] w[z][c] X[P][m][z*nocc + c], one workgroup per (P, z),
// fixed-order reduction (deterministic).
__global__ void __launch_bounds__(256) jvec_kernel(const double* __restrict__ X, int64_t nao, int64_t ldx,
                                                   const double* __restrict__ Cm, const double* __restrict__ w,
                                                   int64_t nocc, double* __restrict__ v, int64_t ldv,
                                                   int accumulate) {
  __shared__ double red[4];
  const int64_t P = blockIdx.x, z = blockIdx.y;
  const double* Xp = X + P * nao * ldx + z * nocc;
  const double* Cz = Cm + z * nao * nocc;
  const double* wz = w ? w + z * nocc : nullptr;
  double s = 0.0;
  if (ldx == nocc && !wz) {
    // X_P and the factor are both contiguous [nao * nocc]: a dot product with four loads in flight
    const int64_t n = nao * nocc;
    double s1 = 0.0, s2 = 0.0, s3 = 0.0;
    int64_t e = threadIdx.x;
    for (; e + 768 < n; e += 1024) {
      s = fma(Cz[e], Xp[e], s);
      s1 = fma(Cz[e + 256], Xp[e + 256], s1);
      s2 = fma(Cz[e + 512], Xp[e + 512], s2);
      s3 = fma(Cz[e + 768], Xp[e + 768], s3);
    }
    for (; e < n; e += 256) s = fma(Cz[e], Xp[e], s);
    s = (s + s1) + (s2 + s3);
  } else {
  int64_t m = threadIdx.x / nocc, c = threadIdx.x % nocc;
  while (m < nao) {
    const double cw = wz ? Cz[m * nocc + c] * wz[c] : Cz[m * nocc + c];
    s = fma(cw, Xp[m * ldx + c], s);
    c += 256;
    while (c >= nocc) {
      c -= nocc;
      ++m;
    }
  }
  }
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    const double r = (red[0] + red[1]) + (red[2] + red[3]);
    v[z * ldv + P] = accumulate ? v[z * ldv + P] + r : r;
  }
}

// J[z][i][j] = sum_P v[z][P] b^P_{ij} for NZ densities, streaming B once.  Bound by HBM.  A workgroup
// owns kCoulombPairs * 256 consecutive packed pairs (thread t the pairs t + 256 r), so each P row is
// read as runs of 8 KB; v is staged through LDS in blocks of 256 P.  The pairs alone give 704
// workgroups at N_ao = 1200 but 8 at 120, so the P range is split over grid y too (launch_coulomb):
// partial sums go to part [split][z][npair] and coulomb_reduce_kernel adds them in split order.
// Where the pairs alone fill the card (!DEEP) a thread reads one row at a time, four loads in flight: with sixteen, or with
// the compiler's own choice, 1200 x 4800 took 4.67 ms instead of 4.38 (6.3 TB/s), 1400 x 2000 2.76 instead of 2.55.  Below that
// sixteen are as good or better (1000 x 4000 2.92 -> 2.71 ms).
constexpr int kCoulombZ = 4;
constexpr int kCoulombPairs = 4;
template <int NZ, bool DEEP>
__global__ void __launch_bounds__(256) coulomb_kernel(const double* __restrict__ B, int64_t naux, int64_t nao,
                                                      int64_t npair, const double* __restrict__ v, int64_t vstride,
                                                      double* __restrict__ J, int64_t jstride, int accumulate,
                                                      double* __restrict__ part) {
  __shared__ double vs[NZ][256];
  const int64_t p0 = (int64_t)blockIdx.x * (256 * kCoulombPairs) + threadIdx.x;
  const int64_t Pb = naux * blockIdx.y / gridDim.y, Pe = naux * (blockIdx.y + 1) / gridDim.y;
  int64_t pc[kCoulombPairs];   // the pairs, clamped to the last one (read, never stored)
#pragma unroll
  for (int r = 0; r < kCoulombPairs; ++r) pc[r] = p0 + 256 * r < npair ? p0 + 256 * r : npair - 1;
  double acc[kCoulombPairs][NZ];
#pragma unroll
  for (int r = 0; r < kCoulombPairs; ++r)
#pragma unroll
    for (int z = 0; z < NZ; ++z) acc[r][z] = 0.0;
  for (int64_t P0 = Pb; P0 < Pe; P0 += 256) {
    const int cnt = (int)(Pe - P0 < 256 ? Pe - P0 : 256);
    __syncthreads();
#pragma unroll
    for (int z = 0; z < NZ; ++z)
      vs[z][threadIdx.x] = (int)threadIdx.x < cnt ? v[z * vstride + P0 + threadIdx.x] : 0.0;
    __syncthreads();
    const double* Bp = B + P0 * npair;
    int q = 0;
    if constexpr (DEEP) {
      for (; q + 4 <= cnt; q += 4) {   // 16 loads in flight per thread
        double b[4][kCoulombPairs];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int r = 0; r < kCoulombPairs; ++r) b[u][r] = Bp[(int64_t)(q + u) * npair + pc[r]];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int z = 0; z < NZ; ++z) {
            const double w = vs[z][q + u];
#pragma unroll
            for (int r = 0; r < kCoulombPairs; ++r) acc[r][z] = fma(w, b[u][r], acc[r][z]);
          }
      }
    } else {
#pragma unroll 2
      for (; q < cnt; ++q) {   // the fences keep the loads of later rows where they are
        double b[kCoulombPairs];
#pragma unroll
        for (int r = 0; r < kCoulombPairs; ++r) b[r] = Bp[(int64_t)q * npair + pc[r]];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int z = 0; z < NZ; ++z) {
          const double w = vs[z][q];
#pragma unroll
          for (int r = 0; r < kCoulombPairs; ++r) acc[r][z] = fma(w, b[r], acc[r][z]);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    for (; q < cnt; ++q) {
#pragma unroll
      for (int r = 0; r < kCoulombPairs; ++r) {
        const double b = Bp[(int64_t)q * npair + pc[r]];
#pragma unroll
        for (int z = 0; z < NZ; ++z) acc[r][z] = fma(vs[z][q], b, acc[r][z]);
      }
    }
  }
#pragma unroll
  for (int r = 0; r < kCoulombPairs; ++r) {
    const int64_t p = p0 + 256 * r;
    if (p >= npair) break;
    if (part) {
#pragma unroll
      for (int z = 0; z < NZ; ++z) part[((int64_t)blockIdx.y * NZ + z) * npair + p] = acc[r][z];
      continue;
    }
    int64_t i, j;
    pair_ij(p, &i, &j);
#pragma unroll
    for (int z = 0; z < NZ; ++z) {
      const double x = accumulate ? J[z * jstride + i * nao + j] + acc[r][z] : acc[r][z];   // J is symmetric
      J[z * jstride + i * nao + j] = x;
      J[z * jstride + j * nao + i] = x;
    }
  }
}

// J[z][i][j] = J[z][j][i] = sum_s part[s][z][pair(i, j)] (+ J), G threads per pair.
template <int G>
__global__ void __launch_bounds__(kRedThreads) coulomb_reduce_kernel(const double* __restrict__ part, int nsplit,
                                                                     int64_t nao, int64_t npair,
                                                                     double* __restrict__ J, int accumulate) {
  constexpr int W = kRedThreads / G;
  const int64_t p = (int64_t)blockIdx.x * W + threadIdx.x % W, z = blockIdx.y, nz = gridDim.y;
  const double s = split_sum<G>(part + z * npair + p, nsplit, nz * npair, p < npair);
  if (threadIdx.x >= W || p >= npair) return;
  int64_t i, j;
  pair_ij(p, &i, &j);
  double* Jz = J + z * nao * nao;
  const double x = accumulate ? Jz[i * nao + j] + s : s;
  Jz[i * nao + j] = x;
  Jz[j * nao + i] = x;
}

// Column blocks side by side (ColBlocks): dst[m][c], rows past nao zero.  One launch instead of a 2-D copy per
// block and a fill: a copy's launch alone takes 10 to 20 us of a small call, and 64 densities
// of eight fragments were 520 copies.
__global__ void __launch_bounds__(256) gather_cols_kernel(ColBlocks k, int64_t nao, int64_t total,
                                                          double* __restrict__ dst) {
  const int64_t n = k.nz * k.n1, ncol = k.n0 + n + k.n2;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (int64_t)gridDim.x * 256) {
    const int64_t m = i / ncol, c = i - m * ncol - k.n0;
    double x = 0.0;
    if (m < nao) {
      if (c < 0) {
        x = k.s0[m * k.n0 + c + k.n0];
      } else if (c < n) {
        const int64_t z = c / k.n1;
        x = k.s1[(z * nao + m) * k.n1 + c - z * k.n1];
      } else {
        x = k.s2[m * k.n2 + c - n];
      }
    }
    dst[i] = x;
  }
}

__global__ void __launch_bounds__(256) add_kernel(const double* __restrict__ x, int64_t n, double* __restrict__ y) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) y[i] += x[i];
}

// y[r][c] (+)= x[r][c] for a contiguous x [rows][cols] and y of row stride ldy
__global__ void __launch_bounds__(256) copy_rows_kernel(const double* __restrict__ x, int64_t rows, int64_t cols,
                                                        double* __restrict__ y, int64_t ldy, int accumulate) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= rows * cols) return;
  double* d = y + (i / cols) * ldy + i % cols;
  *d = accumulate ? *d + x[i] : x[i];
}

__global__ void __launch_bounds__(256) scale_cols_kernel(const double* __restrict__ X, int64_t n, int64_t ncol,
                                                         const double* __restrict__ w, double* __restrict__ Xw) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) Xw[i] = X[i] * w[i % ncol];
}

// g[pair(i,j)] = G[i][j] + G[j][i] for i > j, G[i][i] on the diagonal
__global__ void __launch_bounds__(256) pair_weights_kernel(const double* __restrict__ G, int64_t nao,
                                                           double* __restrict__ g) {
  const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t npair = nao * (nao + 1) / 2;
  if (p >= npair) return;
  G += (int64_t)blockIdx.y * nao * nao;   // matrix blockIdx.y of a batch
  g += (int64_t)blockIdx.y * npair;
  int64_t i = (int64_t)((sqrt(8.0 * (double)p + 1.0) - 1.0) * 0.5);
  while (i * (i + 1) / 2 > p) --i;
  while ((i + 1) * (i + 2) / 2 <= p) ++i;
  const int64_t j = p - i * (i + 1) / 2;
  g[p] = i == j ? G[i * nao + i] : G[i * nao + j] + G[j * nao + i];
}

// u[P] = sum_pair B[P][pair] g[pair]: four rows of B per workgroup share each read of g; a
// fixed-order reduction keeps it deterministic.
constexpr int kJvRows = 4;
// Partial sums part[c][P] = sum_{pair in chunk c} B[P][pair] g[pair] for kJvRows rows per
// workgroup (grid x) and kJvChunks chunks of the pairs (grid y).  Each step a thread takes the
// pairs p + 256 u (u < 4) of every row: each row is read as runs of 8 KB per workgroup.
constexpr int kJvChunks = 8;
__global__ void __launch_bounds__(256) jvec_packed_kernel(const double* __restrict__ B, int64_t naux, int64_t npair,
                                                          const double* __restrict__ g, double* __restrict__ part) {
  __shared__ double red[kJvRows][4];
  const int64_t P0 = (int64_t)blockIdx.x * kJvRows;
  const int64_t c = blockIdx.y, chunk = (npair + kJvChunks - 1) / kJvChunks;
  const int64_t p0 = c * chunk, p1 = p0 + chunk < npair ? p0 + chunk : npair;
  const double* rows[kJvRows];   // rows past the end read the last one (never stored)
#pragma unroll
  for (int r = 0; r < kJvRows; ++r) rows[r] = B + (P0 + r < naux ? P0 + r : naux - 1) * npair;
  double s[kJvRows];
#pragma unroll
  for (int r = 0; r < kJvRows; ++r) s[r] = 0.0;
  for (int64_t p = p0 + threadIdx.x; p < p1; p += 1024) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t q = p + 256 * u;
      const bool ok = q < p1;
      const int64_t qc = ok ? q : p1 - 1;
      const double gq = ok ? g[qc] : 0.0;
#pragma unroll
      for (int r = 0; r < kJvRows; ++r) s[r] = fma(rows[r][qc], gq, s[r]);
    }
  }
#pragma unroll
  for (int r = 0; r < kJvRows; ++r) {
    double x = s[r];
    for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off);
    if ((threadIdx.x & 63) == 0) red[r][threadIdx.x >> 6] = x;
  }
  __syncthreads();
  if (threadIdx.x < kJvRows && P0 + threadIdx.x < naux) {
    const int r = threadIdx.x;
    part[c * naux + P0 + r] = (red[r][0] + red[r][1]) + (red[r][2] + red[r][3]);
  }
}

__global__ void __launch_bounds__(256) jvec_chunks_kernel(const double* __restrict__ part, int64_t naux,
                                                          double* __restrict__ u) {
  const int64_t P = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (P >= naux) return;
  double s = 0.0;
  for (int c = 0; c < kJvChunks; ++c) s += part[c * naux + P];
  u[P] = s;
}

// out[z] = in[z] + in[z]^T (in place allowed: each pair (i, j), i <= j, is handled by one thread)
__global__ void __launch_bounds__(256) symmetrize_kernel(const double* in, int64_t n, int64_t nz, double* out) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t nn = n * n;
  if (idx >= nn * nz) return;
  const int64_t z = idx / nn, rem = idx % nn, i = rem / n, j = rem % n;
  if (i > j) return;
  const double* a = in + z * nn;
  const double s = a[i * n + j] + a[j * n + i];
  out[z * nn + i * n + j] = s;
  out[z * nn + j * n + i] = s;
}

__global__ void __launch_bounds__(256) unpack_sym_kernel(const double* __restrict__ Jp, int64_t nz, int64_t nao,
                                                         int64_t npair, double* __restrict__ J) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= nz * npair) return;
  const int64_t z = idx / npair, p = idx % npair;
  int64_t i = (int64_t)((sqrt(8.0 * (double)p + 1.0) - 1.0) * 0.5);
  while (i * (i + 1) / 2 > p) --i;
  while ((i + 1) * (i + 2) / 2 <= p) ++i;
  const int64_t j = p - i * (i + 1) / 2;
  const double x = Jp[idx];
  J[z * nao * nao + i * nao + j] = x;
  J[z * nao * nao + j * nao + i] = x;
}

__global__ void __launch_bounds__(256) pack_lower_kernel(const double* __restrict__ A, int64_t s_z, int64_t nz,
                                                         int64_t n, int64_t npair, double* __restrict__ Ap) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= nz * npair) return;
  const int64_t z = idx / npair, p = idx % npair;
  int64_t i = (int64_t)((sqrt(8.0 * (double)p + 1.0) - 1.0) * 0.5);
  while (i * (i + 1) / 2 > p) --i;
  while ((i + 1) * (i + 2) / 2 <= p) ++i;
  const int64_t j = p - i * (i + 1) / 2;
  Ap[idx] = A[z * s_z + i * n + j];
}

// Cholesky factor of one kb x kb diagonal block (kb <= kCholNB) of the metric, in LDS, and the
// inverse of that factor.  A (row stride lda) holds the block with the earlier blocks' updates
// already subtracted; its lower triangle is read (rows past kb are those of the identity).
// Right-looking over 16-wide blocks: one wave factors the diagonal block and inverts it, a row
// (a column of the inverse) per lane, the other lanes' values by readlane; the blocks below take its
// inverse and the trailing blocks their update on the matrix cores.  The inverse follows by block columns, two
// per wave, no barrier between: X_ij = -Linv_ii sum_{k=j}^{i-1} L_ik X_kj, kept in the upper blocks of S; the sum
// leaves the matrix cores in the very layout in which the product with Linv_ii reads its right
// operand.  One workgroup, so bound by latency: a column at a time (128 columns, three barriers each, and a
// serial substitution for the inverse) took 331 us, so 83.  Only the blocks that hold rows of A are worked on: all
// eight of them for the 5 rows of an N_ao 20 build took the whole call from 24 to 80 us, 20 now.  Outputs: the factor back to
// A (lower, the block's strictly upper part zeroed) and L^-1 to Linv [kCholNB][kCholNB] (lower,
// upper zeroed).  info: the first block (first != 0) writes 0; a block that meets a pivot that
// is not positive writes k0 + j + 1 unless info already holds an earlier one.  After such a
// pivot the block goes on with pivot 1 so that every wave finishes.
__device__ __forceinline__ double lane_value(double x, int lane) {   // lane: uniform
  const long long b = __double_as_longlong(x);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)b, lane);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(b >> 32), lane);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__global__ void __launch_bounds__(256) chol_block_kernel(double* __restrict__ A, int64_t lda, int kb,
                                                         double* __restrict__ Linv, int* info, int64_t k0,
                                                         int first) {
  constexpr int N = kCholNB, NB = N / 16, LS = N + 1;
  __shared__ double S[N][LS];
  __shared__ double D[NB][16][17];   // inverses of the diagonal blocks
  __shared__ int bad;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6, lr = lane & 15, lk = lane >> 4;
  const int nb = (kb + 15) / 16;   // blocks with rows of A
  for (int idx = t; idx < nb * 16 * N; idx += 256) {
    const int i = idx / N, j = idx % N;
    S[i][j] = i < kb ? (j <= i ? A[i * lda + j] : 0.0) : (i == j ? 1.0 : 0.0);
  }
  if (t == 0) bad = -1;
  __syncthreads();
  for (int p = 0; p < nb; ++p) {
    const int o = p * 16;
    if (wave == 0) {
      // lane l < 16 holds row l of the block (the other lanes copies, never stored)
      double a[16], x[16], rd[16];
#pragma unroll
      for (int c = 0; c < 16; ++c) a[c] = S[o + lr][o + c];
      int b = -1;
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const double d = lane_value(a[j], j);
        const bool ok = d > 0.0;
        if (!ok && b < 0) b = o + j;
        const double sd = ok ? sqrt(d) : 1.0;
        rd[j] = 1.0 / sd;
        a[j] = lr == j ? sd : a[j] * rd[j];
#pragma unroll
        for (int c = j + 1; c < 16; ++c) a[c] -= a[j] * lane_value(a[j], c);
      }
      // column lr of the inverse: L x = e_lr
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        double v = i == lr ? 1.0 : 0.0;
#pragma unroll
        for (int j = 0; j < i; ++j) v -= lane_value(a[j], i) * x[j];
        x[i] = v * rd[i];
      }
      if (lane < 16) {
#pragma unroll
        for (int c = 0; c < 16; ++c) {
          S[o + lr][o + c] = c <= lr ? a[c] : 0.0;
          D[p][c][lr] = c >= lr ? x[c] : 0.0;
        }
        if (lane == 0 && b >= 0 && bad < 0) bad = b;
      }
    }
    __syncthreads();
    // the blocks below: L_rp = A_rp Linv_pp^T, and once more with the residual A_rp - L_rp L_pp^T (a block is read and
    // written by one wave, whose LDS accesses stay in order).  With the inverse alone the error of L was 2.7 times that of an
    // elimination by columns at 40 rows and condition 1e10, 1.6 at 1e6; so 1.1 and 1.06.
    for (int r = p + 1 + wave; r < nb; r += 4) {
      d4 acc = {0.0, 0.0, 0.0, 0.0}, res;
#pragma unroll
      for (int q = 0; q < 4; ++q) res[q] = S[r * 16 + 4 * q + lk][o + lr];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int kk = 0; kk < 16; kk += 4)
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64(S[r * 16 + lr][o + kk + lk], D[p][lr][kk + lk], acc, 0, 0, 0);
#pragma unroll
        for (int q = 0; q < 4; ++q) S[r * 16 + 4 * q + lk][o + lr] = acc[q];
        if (h > 0) break;
#pragma unroll
        for (int kk = 0; kk < 16; kk += 4)
          res = __builtin_amdgcn_mfma_f64_16x16x4f64(-S[r * 16 + lr][o + kk + lk], S[o + lr][o + kk + lk], res, 0, 0, 0);
#pragma unroll
        for (int q = 0; q < 4; ++q) S[r * 16 + 4 * q + lk][o + lr] = res[q];
      }
    }
    __syncthreads();
    // trailing blocks (r >= c > p): A_rc -= L_rp L_cp^T
    const int m = nb - 1 - p;
    for (int w = wave; w < m * (m + 1) / 2; w += 4) {
      int r = 0;
      while ((r + 1) * (r + 2) / 2 <= w) ++r;
      const int rb = (p + 1 + r) * 16, cb = (p + 1 + w - r * (r + 1) / 2) * 16;
      d4 acc;
#pragma unroll
      for (int q = 0; q < 4; ++q) acc[q] = S[rb + 4 * q + lk][cb + lr];
#pragma unroll
      for (int kk = 0; kk < 16; kk += 4)
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(-S[rb + lr][o + kk + lk], S[cb + lr][o + kk + lk], acc, 0, 0, 0);
#pragma unroll
      for (int q = 0; q < 4; ++q) S[rb + 4 * q + lk][cb + lr] = acc[q];
    }
    __syncthreads();
  }
  // block columns wave and NB - 1 - wave of the inverse; X_ij (i > j) at rows 16 j, columns 16 i of S, which the
  // factor does not use and no other wave reads
  for (int h = 0; h < 2; ++h) {
    const int j = h == 0 ? wave : NB - 1 - wave;
    for (int i = j + 1; i < nb; ++i) {
      d4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int kk = 0; kk < 16; kk += 4)
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(S[i * 16 + lr][j * 16 + kk + lk], D[j][kk + lk][lr], acc, 0, 0, 0);
      for (int k = j + 1; k < i; ++k)
#pragma unroll
        for (int kk = 0; kk < 16; kk += 4)
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64(S[i * 16 + lr][k * 16 + kk + lk], S[j * 16 + kk + lk][k * 16 + lr],
                                                     acc, 0, 0, 0);
      d4 x = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int q = 0; q < 4; ++q)
        x = __builtin_amdgcn_mfma_f64_16x16x4f64(-D[i][lr][4 * q + lk], acc[q], x, 0, 0, 0);
#pragma unroll
      for (int q = 0; q < 4; ++q) S[j * 16 + 4 * q + lk][i * 16 + lr] = x[q];
    }
  }
  __syncthreads();
  for (int idx = t; idx < kb * kb; idx += 256) {
    const int i = idx / kb, j = idx % kb, bi = i / 16, bj = j / 16;
    A[i * lda + j] = j <= i ? S[i][j] : 0.0;
    Linv[i * N + j] = j > i ? 0.0 : bi == bj ? D[bi][i % 16][j % 16] : S[bj * 16 + i % 16][bi * 16 + j % 16];
  }
  if (t == 0) {
    int cur = first ? 0 : *info;
    if (cur == 0 && bad >= 0) cur = (int)(k0 + bad + 1);
    *info = cur;
  }
}

// One block row of the forward substitution:  B_k = Linv_k (E_k - sum_{j < k} L_kj B_j)  for 128 columns per
// workgroup.  Waves side by side (1 x 4), so that a wave holds all kb <= 128 rows of its 32 columns of
// T = E_k - sum: the accumulators then have the layout in which the product with Linv_k reads
// its right operand, and T never leaves the registers.  Linv_k goes through LDS in two halves
// of 64 rows; its zero upper part is skipped.  49 TF/s at 2400 x 180300, matrix cores busy 0.62: the waves wait a third
// of their cycles, and 1409 workgroups a block row fill 2.75 rounds.  As a copy of E_k, a product that subtracts from it and a product with
// Linv_k the substitution took 25.7 ms there, so 22.0.
typedef Cfg<1, 4, 8, 2> CfgSub;
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) subst_row_kernel(OpMap A, OpMap B, int64_t nslab, const double* E,
                                                          const double* __restrict__ Linv, int kb, int64_t npair,
                                                          double* out) {
  typedef CfgSub C;
  static_assert(C::BM == kCholNB && C::TM == 8, "a wave holds every row");
  constexpr int LS = kCholNB + 1;
  static_assert(64 * LS <= 2 * C::STAGE, "half of Linv in the LDS of the main loop");
  __shared__ double smem[2 * C::STAGE];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6, lr = lane & 15, lk = lane >> 4;
  const int64_t n0 = (int64_t)xcd_remap(blockIdx.x, gridDim.x) * C::BN;
  d4 acc[C::TM][C::TN];
  zero_acc<C>(acc);
  const int nb = (kb + 15) / 16;   // 16-row blocks to form
  if (nslab > 0) {
    PairSrc<C, true, false, false, false> src;
    src.A = &A;
    src.B = &B;
    src.t = t;
    src.a.init(A, 0, 0, 0, nslab, t);
    src.b.init(B, n0, 0, 0, nslab, t);
    mainloop<C>(src, smem, nslab, acc, 0, wave, lane);
  }
  int64_t col[C::TN], colc[C::TN];
#pragma unroll
  for (int j = 0; j < C::TN; ++j) {
    col[j] = n0 + (wave * C::TN + j) * 16 + lr;
    colc[j] = col[j] < npair ? col[j] : npair - 1;
  }
#pragma unroll
  for (int i = 0; i < C::TM; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int m = i * 16 + 4 * q + lk;
#pragma unroll
      for (int j = 0; j < C::TN; ++j) {
        const double e = E[(int64_t)(m < kb ? m : kb - 1) * npair + colc[j]];
        acc[i][j][q] = m < kb ? e - acc[i][j][q] : 0.0;
      }
    }
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    if (4 * h >= nb) break;
    __syncthreads();   // the last reads of what is overwritten are done
    for (int idx = t; idx < min(64, 16 * nb - 64 * h) * kCholNB; idx += 256) {
      const int r = 64 * h + idx / kCholNB, k = idx % kCholNB;
      smem[(idx / kCholNB) * LS + k] = r < kb && k < kb ? Linv[r * kCholNB + k] : 0.0;
    }
    __syncthreads();
#pragma unroll
    for (int i4 = 0; i4 < 4; ++i4) {
      const int i = 4 * h + i4;
      if (i >= nb) break;
      d4 x[C::TN];
#pragma unroll
      for (int j = 0; j < C::TN; ++j) x[j] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int k = 0; k <= i; ++k)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const double a = smem[(i4 * 16 + lr) * LS + k * 16 + 4 * q + lk];
#pragma unroll
          for (int j = 0; j < C::TN; ++j) x[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, acc[k][j][q], x[j], 0, 0, 0);
        }
#pragma unroll
      for (int j = 0; j < C::TN; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int m = i * 16 + 4 * q + lk;
          if (m < kb && col[j] < npair) out[(int64_t)m * npair + col[j]] = x[j][q];
        }
    }
  }
}

// A[i][j] = 0 for j > i, n x n
__global__ void __launch_bounds__(256) zero_upper_kernel(double* A, int64_t n) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= n * n) return;
  if (idx % n > idx / n) A[idx] = 0.0;
}

__global__ void __launch_bounds__(256) fill_zero_kernel(double* p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = 0.0;
}

__global__ void __launch_bounds__(256) fill_zero_strided_kernel(double* p, int64_t nz, int64_t s_z, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n * nz) p[(i / n) * s_z + i % n] = 0.0;
}

// ---------------------------------------------------------------------------------------
// Launchers

static inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

// A flat contraction pays where padding each kb block to whole slabs wastes more than 4% of the
// slabs (at 300 per block, 1.3%, the padded loads measured faster than the flat ones).
static bool flat_pays(const OpMap& o) { return o.kc_n >= 16 && cdiv(o.kc_n, 16) * 16 * 100 > o.kc_n * 104; }

// A flat contraction adds the step from one kb block to the next to the within-slab offsets.
static bool flat_fits(const OpMap& o) {
  if (o.rows <= 0 || o.kc_n <= 0) return true;
  const int64_t last = o.rows - 1;
  const int64_t rh = o.s_rh ? last / o.rl : 0, rlo = o.s_rh ? o.rl - 1 : last;
  const int64_t top = rh * o.s_rh + rlo * o.s_rlo + 15 * o.s_kc + (o.s_kb - o.kc_n * o.s_kc);
  return o.s_kb >= o.kc_n * o.s_kc && top < (1LL << 32);
}

bool offsets_fit(const OpMap& o) {
  if (o.rows <= 0 || o.kc_n <= 0) return true;
  const int64_t last = o.rows - 1;
  const int64_t rh = o.s_rh ? last / o.rl : 0, rlo = o.s_rh ? o.rl - 1 : last;
  const int64_t kmax = o.kc_n - 1 + 15;   // a slab may address up to 15 entries past the end before clamping
  const int64_t top = rh * o.s_rh + rlo * o.s_rlo + kmax * o.s_kc;
  return o.rows < (1LL << 31) && o.rl < (1LL << 31) && top < (1LL << 32);
}

// Tiling of the half transform: nA tiles of 128 columns and one narrower (or, past 96, one more of 128)
// for the rest, `rest` its width (0: none); `tail` rows past the last whole band (at most half a band) on
// tiles of their own, which need at least one whole 128-wide tile beside them (a narrow output is
// bound by latency, not by its padding).  Bands have 64 rows, 128 (`big`) where the packed b^P does not
// fit the 4 MB L2 of an XCD: every band reads all of b^P's columns, from the last-level cache then
// (P-summed product at 1200 x 4800 x 300: 79 ms with 64-row bands, 75 with 128; at N_ao = 1000 the
// 64-row bands still win, 17.9 ms against 18.1), but not beside a rest of at most 32 columns, which 128 rows
// have no tile for: on one of 48 the half transform ran 4.45 ms at 1030 x 600 x 140 instead of 3.77, 5.79 instead of 5.29
// at 1200 x 600 x 150.  64 or 96 columns alone take 128 rows too from N_ao = 449 on, where that pads no more rows
// (64 x 64 and 128 x 64 tiles: 677 and 651 us at 512 x 1024, 1361 and 1323 at 720 x 1000, 575 and 576 at 384 x 1500).
struct HalfCols {
  int64_t nA;
  int rest, tail;
  bool big;
  int bm() const { return big ? CfgQ128::BM : CfgH128::BM; }
};
static HalfCols half_cols(int64_t nao, int64_t ncol) {
  HalfCols h{ncol / 128, 0, 0, false};
  const int64_t rem = ncol % 128;
  if (rem > 96) ++h.nA;
  else if (rem > 0) h.rest = rem <= 16 ? 16 : rem <= 32 ? 32 : rem <= 48 ? 48 : rem <= 64 ? 64 : 96;
  if (h.nA > 0) h.big = nao * (nao + 1) / 2 > (int64_t(4) << 20) / 8 && (h.rest == 0 || h.rest >= 48);
  else h.big = h.rest >= 64 && nao > 448 && cdiv(nao, CfgH128::BM) % 2 == 0;
  const int64_t rows = nao % h.bm();
  if (h.nA > 0 && rows > 0 && rows <= h.bm() / 2) h.tail = (int)rows;
  return h;
}
static HalfTiles half_counts(int64_t nao, int64_t ncol) {
  const HalfCols h = half_cols(nao, ncol);
  HalfTiles T{(int)cdiv(nao - h.tail, h.bm()), (int)h.nA, h.rest ? 1 : 0, h.tail ? (int)cdiv(ncol, 128) : 0};
  if (T.nA == 0) {   // one narrow tile per band: it takes CA's place
    T.nA = T.nB;
    T.nB = 0;
  }
  return T;
}

int64_t half_tiles(int64_t nao, int64_t ncol) { return half_counts(nao, ncol).count(); }

// f(CA, CB, CT) with the tile types: CB = CA or CT = CA where there are no such tiles (the kernel then
// holds fewer bodies, and narrow tiles alone run as many waves as fit them).
template <class F>
static auto half_dispatch(const HalfCols& h, F&& f) {
  typedef CfgH128 A;
  typedef CfgHTail T;
  if (h.big && h.nA == 0) {
    if (h.rest == 64) return f(CfgQ64{}, CfgQ64{}, CfgQ64{});
    return f(CfgQ96{}, CfgQ96{}, CfgQ96{});
  }
  if (h.big) switch (h.rest) {
      case 0: return f(CfgQ128{}, CfgQ128{}, CfgQTail{});
      case 48: return f(CfgQ128{}, CfgQ48{}, CfgQTail{});
      case 64: return f(CfgQ128{}, CfgQ64{}, CfgQTail{});
      default: return f(CfgQ128{}, CfgQ96{}, CfgQTail{});
    }
  if (h.nA == 0) switch (h.rest) {
      case 16: return f(CfgH16{}, CfgH16{}, CfgH16{});
      case 32: return f(CfgH32{}, CfgH32{}, CfgH32{});
      case 48: return f(CfgH48{}, CfgH48{}, CfgH48{});
      case 64: return f(CfgH64{}, CfgH64{}, CfgH64{});
      default: return f(CfgH96{}, CfgH96{}, CfgH96{});
    }
  switch (h.rest) {
    case 0: return h.tail ? f(A{}, A{}, T{}) : f(A{}, A{}, A{});
    case 16: return f(A{}, CfgH16{}, T{});
    case 32: return f(A{}, CfgH32{}, T{});
    case 48: return f(A{}, CfgH48{}, T{});
    case 64: return f(A{}, CfgH64{}, T{});
    default: return f(A{}, CfgH96{}, T{});
  }
}

static hipError_t half_run(const double* B, int64_t naux, int64_t nao, const double* C, int64_t ldc, int64_t ncol,
                           const OutMap& out, const JvEpi* jv, hipStream_t s) {
  const OpMap cm = op_map(C, ncol, 1, nao, ldc);
  const HalfTiles T = half_counts(nao, ncol);
  const int64_t nblk = T.count() * naux, npair = nao * (nao + 1) / 2;
  if (nblk == 0) return hipSuccess;
  if (nblk > 0x7fffffffLL || !offsets_fit(cm)) return hipErrorInvalidValue;
  const bool gen = out.alpha != 1.0 || out.accumulate;
  if (jv && gen) return hipErrorInvalidValue;
  const dim3 g((unsigned)nblk);
  const JvEpi j = jv ? *jv : JvEpi{};
  return half_dispatch(half_cols(nao, ncol), [&](auto ca, auto cb, auto ct) {
    typedef decltype(ca) CA;
    typedef decltype(cb) CB;
    typedef decltype(ct) CT;
    if (jv) half_kernel<CA, CB, CT, false, true><<<g, CA::NT, 0, s>>>(B, naux, (int)nao, npair, cm, out, T, j);
    else if (gen) half_kernel<CA, CB, CT, true, false><<<g, CA::NT, 0, s>>>(B, naux, (int)nao, npair, cm, out, T, j);
    else half_kernel<CA, CB, CT, false, false><<<g, CA::NT, 0, s>>>(B, naux, (int)nao, npair, cm, out, T, j);
    return hipGetLastError();
  });
}

hipError_t launch_half_transform(const double* B, int64_t naux, int64_t nao, const double* C, int64_t ldc,
                                 int64_t ncol, const OutMap& out, hipStream_t s) {
  return half_run(B, naux, nao, C, ldc, ncol, out, nullptr, s);
}

hipError_t launch_half_transform_jvec(const double* B, int64_t naux, int64_t nao, const double* C, int64_t ldc,
                                      int64_t ncol, const OutMap& out, const double* w, int64_t nv, double* part,
                                      double* v, int accumulate, hipStream_t s) {
  if (nv < 0 || nv > ncol || nv > 0x7fffffffLL || out.s_nh != 0) return hipErrorInvalidValue;
  if (naux == 0) return hipSuccess;
  const JvEpi jv{C, ldc, w, (int)nv, part, half_tiles(nao, ncol)};
  if (jv.T == 0) return hipErrorInvalidValue;
  hipError_t e = half_run(B, naux, nao, C, ldc, ncol, out, &jv, s);
  if (e != hipSuccess) return e;
  jv_reduce_kernel<<<(unsigned)cdiv(naux, 256), 256, 0, s>>>(part, jv.T, naux, v, accumulate);
  return hipGetLastError();
}

// The 256-row tile when it pads the rows no more than the 128-row one.
static bool gemm_tall(int64_t M) {
  return M >= 256 && cdiv(M, CfgTall::BM) * CfgTall::BM <= cdiv(M, CfgSq::BM) * CfgSq::BM;
}

template <class Cg, bool GEN, bool CLAMP>
static void gemm_go(const OpMap& A, const OpMap& Bm, const OutMap& O, dim3 grid, int64_t tm, int64_t tn, double* part,
                    hipStream_t s) {
  const bool ak = A.s_kc == 1, bk = Bm.s_kc == 1;
  if (ak && bk) gemm_kernel<Cg, true, true, GEN, CLAMP><<<grid, Cg::NT, 0, s>>>(A, Bm, O, tm, tn, part);
  else if (ak) gemm_kernel<Cg, true, false, GEN, CLAMP><<<grid, Cg::NT, 0, s>>>(A, Bm, O, tm, tn, part);
  else if (bk) gemm_kernel<Cg, false, true, GEN, CLAMP><<<grid, Cg::NT, 0, s>>>(A, Bm, O, tm, tn, part);
  else gemm_kernel<Cg, false, false, GEN, CLAMP><<<grid, Cg::NT, 0, s>>>(A, Bm, O, tm, tn, part);
}

template <class Cg>
static hipError_t gemm_launch_cfg(const OpMap& A, const OpMap& Bm, const OutMap& O, int64_t nz, int nsplit,
                                  double* part, hipStream_t s) {
  const int64_t tm = cdiv(O.M, Cg::BM), tn = cdiv(O.N, Cg::BN);
  if (tm * tn == 0 || nz == 0) return hipSuccess;
  if (tm * tn > 0x7fffffffLL || nz > 65535 || nsplit < 1 || nsplit > 65535 || !offsets_fit(A) || !offsets_fit(Bm) ||
      A.kc_n != Bm.kc_n || A.kb_n != Bm.kb_n)
    return hipErrorInvalidValue;
  const dim3 grid((unsigned)(tm * tn), (unsigned)nsplit, (unsigned)nz);
  // whole slabs (no clamping) when the contraction chunks are multiples of 16
  const bool clamp = A.kc_n % 16 != 0;
  if (!part && (O.alpha != 1.0 || O.accumulate)) gemm_go<Cg, true, true>(A, Bm, O, grid, tm, tn, part, s);
  else if (clamp) gemm_go<Cg, false, true>(A, Bm, O, grid, tm, tn, part, s);
  else gemm_go<Cg, false, false>(A, Bm, O, grid, tm, tn, part, s);
  return hipGetLastError();
}

int64_t gemm_slabs(const OpMap& A) { return A.kb_n * cdiv(A.kc_n, 16); }

// Estimated time (us) of W equal workgroups of `slabs` slabs each on 128 x 128 or (small) 64 x 64
// tiles.  A slab takes 4.6 us with two 128-wide workgroups on a CU and 2.6 with one, where the
// latency of its loads shows (one workgroup over 30 slabs: 79 us); 64-wide tiles issue a quarter
// of the MFMAs, fit four to a CU and take 1.3 us alone, 2.7 with four.
static double gemm_us(int64_t W, double slabs, bool small) {
  const int64_t per = small ? 1024 : 512;
  const int64_t rem = W % per;
  const double full = small ? 2.7 : 4.6;
  double last = 0.0;
  if (rem > 0) last = small ? (rem <= 256 ? 1.3 : rem <= 512 ? 1.6 : rem <= 768 ? 2.1 : 2.7) : rem <= 256 ? 2.6 : 4.6;
  return ((double)(W / per) * full + last) * (slabs + 4.0);
}
// 64 x 64 tiles where they are estimated faster: products of few 128-wide tiles, or that fill them badly
// (b_uv and b_pu at 120 x 480 36 + 35 -> 18 us in one product, b_uv at 600 x 2400 185 -> 90 us).
static bool gemm_small(int64_t M, int64_t N, int64_t nw, double slabs) {
  return gemm_us(cdiv(M, CfgSmall::BM) * cdiv(N, CfgSmall::BN) * nw, slabs, true) <
         gemm_us(cdiv(M, CfgSq::BM) * cdiv(N, CfgSq::BN) * nw, slabs, false);
}

static hipError_t gemm_launch(const OpMap& A, const OpMap& Bm, const OutMap& O, int64_t nz, int nsplit,
                              double* part, hipStream_t s) {
  if (gemm_small(O.M, O.N, nz * nsplit, (double)gemm_slabs(A) / nsplit))
    return gemm_launch_cfg<CfgSmall>(A, Bm, O, nz, nsplit, part, s);
  const int64_t rem = O.M % CfgSq::BM, tn = cdiv(O.N, CfgSq::BN);
  // At least 512 rows that the larger tiles pad by over 8% more than 64-row bands with a 32-row tail.  Time of the
  // product on bands against the larger tiles, second transform at 600 x 2400 (N 38400) / 480 x 1300 (N 16900), and of the whole adjoint
  // with S X on that many rows: 513-576 rows (10 to 15% less padding) 0.92-0.98 / 0.99-1.00, 0.95-0.98; 769-800 (11%) 0.93 / 0.98-0.99,
  // 0.95-0.98; 1025-1056 (8%) 0.97-0.99 / 0.79, 0.98-1.00.  The other side: 801-830 (7%) 0.93-0.97 / 0.93, 0.97-0.98; 577-608 (5%)
  // 1.08-1.09 / 0.78, 1.01-1.03; 864 (4%) 1.00 / 1.07, 0.99; 1100 (3%) 1.04 / 0.92, 1.03; none, 1200 rows, 1.04 / 1.01, 1.00: a band
  // reads more per MFMA, and its gain past the padding comes and goes with the last round.  Below 512 rows: 416 rows 0.77 / 1.00, 0.91;
  // 341 1.00 / 1.01, 1.00; but with 210, W of (pq|uv) at 600 x 2400, 3.65 ms instead of 3.85, the whole call took 9.25 ms
  // instead of 8.89, for a reason not found.
  const int64_t large = rem > 0 && rem <= CfgRowTail::BM && gemm_tall(O.M) ? O.M - rem + CfgRowTail::BM
                        : gemm_tall(O.M) ? cdiv(O.M, CfgTall::BM) * CfgTall::BM : cdiv(O.M, CfgSq::BM) * CfgSq::BM;
  const int64_t brem = O.M % CfgBand::BM, tail = brem > 0 && brem <= CfgBandTail::BM ? 1 : 0;
  const int64_t nband = tail ? O.M / CfgBand::BM : cdiv(O.M, CfgBand::BM);
  const bool ak = A.s_kc == 1, bk = Bm.s_kc == 1;
  if (O.M >= 512 && (nband * CfgBand::BM + tail * CfgBandTail::BM) * 108 < large * 100 && (ak || !bk) && (part || (O.alpha == 1.0 && !O.accumulate)) &&
      (nband + tail) * tn <= 0x7fffffffLL && tn > 0 && nz > 0 && nz <= 65535 && nsplit >= 1 && nsplit <= 65535 &&
      offsets_fit(A) && offsets_fit(Bm) && A.kc_n == Bm.kc_n && A.kb_n == Bm.kb_n) {
    const dim3 grid((unsigned)((nband + tail) * tn), (unsigned)nsplit, (unsigned)nz);
    auto go = [&](auto k, auto l, auto cl) {
      gemm_band_kernel<decltype(k)::value, decltype(l)::value, decltype(cl)::value>
          <<<grid, CfgBand::NT, 0, s>>>(A, Bm, O, nband, nband + tail, tn, part);
    };
    auto pick = [&](auto cl) {
      if (ak && bk) go(std::true_type{}, std::true_type{}, cl);
      else if (ak) go(std::true_type{}, std::false_type{}, cl);
      else go(std::false_type{}, std::false_type{}, cl);   // no caller has k contiguous in B alone
    };
    if (A.kc_n % 16 != 0) pick(std::true_type{});
    else pick(std::false_type{});
    return hipGetLastError();
  }
  if (gemm_tall(O.M) && rem > 0 && rem <= CfgRowTail::BM && nz == 1 && nsplit == 1 && !part && O.alpha == 1.0 &&
      !O.accumulate && A.kc_n % 16 == 0 && (O.M / CfgSq::BM + 1) * tn <= 0x7fffffffLL && offsets_fit(A) &&
      offsets_fit(Bm) && A.kc_n == Bm.kc_n && A.kb_n == Bm.kb_n) {
    const int64_t nb = O.M / CfgSq::BM;
    const dim3 grid((unsigned)((nb + 1) * tn));
    if (ak && bk) gemm_tail_kernel<true, true><<<grid, CfgSq::NT, 0, s>>>(A, Bm, O, nb, tn);
    else if (ak) gemm_tail_kernel<true, false><<<grid, CfgSq::NT, 0, s>>>(A, Bm, O, nb, tn);
    else if (bk) gemm_tail_kernel<false, true><<<grid, CfgSq::NT, 0, s>>>(A, Bm, O, nb, tn);
    else gemm_tail_kernel<false, false><<<grid, CfgSq::NT, 0, s>>>(A, Bm, O, nb, tn);
    return hipGetLastError();
  }
  return gemm_tall(O.M) ? gemm_launch_cfg<CfgTall>(A, Bm, O, nz, nsplit, part, s)
                        : gemm_launch_cfg<CfgSq>(A, Bm, O, nz, nsplit, part, s);
}

hipError_t launch_gemm(const OpMap& A, const OpMap& Bm, const OutMap& O, int64_t nz, hipStream_t s) {
  return gemm_launch(A, Bm, O, nz, 1, nullptr, s);
}

// Workgroups resident at once for the MFMA kernels on MI355X: 256 CUs x 2 (each kernel is sized
// for two workgroups per CU).  A launch of W equal workgroups takes ceil(W / kResident) rounds.
static constexpr int64_t kResident = 512;

// Split count s in [1, max_split] for a launch of tiles * s equal workgroups over a contraction of
// `slabs` 16-deep slabs: the one of least estimated time.  A workgroup takes its share of the slabs
// plus about 4 for its prologue and epilogue, a slab `slab_us` with two workgroups on its CU (3.6 us
// for a 128 x 128 tile: 64 MFMAs a wave); a last round that fills at most one workgroup per CU
// takes 0.6 of a full one, and workgroups that start together do not end together: 0.2 of an item
// more (K at 341 x 1365 took 492 us in one round of long items, 427 in four).  A split costs the write and the read of its partial sums (`out` doubles,
// 4 TB/s) and, as soon as there is one, the reduction's launch (5 us).  Candidates fill whole rounds
// of 256.  (Filling the rounds alone cut K at 77 x 310 into 310 splits of one P: 126 us of K against
// 21 with this rule.)
static int balanced_splits(int64_t tiles, int64_t max_split, int64_t slabs, int64_t out, double slab_us) {
  if (tiles <= 0) return 1;
  if (max_split > 4096) max_split = 4096;
  max_split = std::min(max_split, 4 * cdiv(kResident, tiles));
  if (max_split <= 1 || slabs <= 1) return 1;
  int best = 1;
  double best_us = 0.0;
  for (int64_t m = 0; m <= 32; ++m) {
    int64_t sp = m == 0 ? 1 : 256 * m / tiles;
    if (sp < 1) continue;
    if (sp > max_split) sp = max_split;
    const int64_t w = tiles * sp, full = w / kResident, rem = w % kResident;
    const double rounds = (double)full + (rem == 0 ? 0.0 : rem <= kResident / 2 ? 0.6 : 1.0);
    const double us = (rounds + 0.2) * (double)(cdiv(slabs, sp) + 4) * slab_us +
                      (sp > 1 ? 5.0 + (double)sp * (double)out * 16.0 / 4.0e6 : 0.0);
    if (m == 0 || us < best_us * (1.0 - 1e-9)) {
      best_us = us;
      best = (int)sp;
    }
    if (sp == max_split && m > 0) break;
  }
  return best;
}
static double slab_us(int64_t bm, int64_t bn) { return 3.6 * (double)(bm * bn) / 16384.0; }

// balanced_splits(tiles, m, ...) for any m <= max_split is at most this.
static int balanced_splits_bound(int64_t tiles, int64_t max_split) {
  if (tiles <= 0 || max_split < 1) return 1;
  const int64_t b = 4 * cdiv(kResident, tiles);
  return (int)(max_split < b ? max_split : b);
}

int gemm_splits_bound(int64_t M, int64_t N, int64_t nslab) {
  if (gemm_tall(M)) return balanced_splits_bound(2 * cdiv(M, CfgTall::BM) * cdiv(N, CfgTall::BN), nslab / 4);
  return balanced_splits_bound(cdiv(M, CfgSq::BM) * cdiv(N, CfgSq::BN), nslab / 4);
}

int gemm_splits(int64_t M, int64_t N, int64_t nslab) {
  // at least four slabs per split; a tall tile takes the room of two resident workgroups
  if (gemm_tall(M))
    return balanced_splits(2 * cdiv(M, CfgTall::BM) * cdiv(N, CfgTall::BN), nslab / 4, nslab, M * N,
                           slab_us(CfgSq::BM, CfgSq::BN));
  return balanced_splits(cdiv(M, CfgSq::BM) * cdiv(N, CfgSq::BN), nslab / 4, nslab, M * N,
                         slab_us(CfgSq::BM, CfgSq::BN));
}

// Split count of a product whose partial sums are read by a kernel of their own in any case
// (expand_pairs): the least estimated time over both tiles, at least two slabs per split, and at
// most 64 MB of partials beyond the first.
int part_splits(int64_t M, int64_t N, int64_t nslab) {
  int best = 1;
  double best_us = 0.0;
  const int64_t most = std::max<int64_t>(1, std::min<int64_t>({nslab / 2, 64, 1 + (int64_t(8) << 20) / std::max<int64_t>(M * N, 1)}));
  for (int ns = 1; ns <= most; ++ns) {
    const double slabs = (double)cdiv(nslab, ns);
    const double us = std::min(gemm_us(cdiv(M, CfgSmall::BM) * cdiv(N, CfgSmall::BN) * ns, slabs, true),
                               gemm_us(cdiv(M, CfgSq::BM) * cdiv(N, CfgSq::BN) * ns, slabs, false)) +
                      (double)ns * (double)(M * N) * 16.0 / 4.0e6;
    if (ns == 1 || us < best_us) {
      best_us = us;
      best = ns;
    }
  }
  return best;
}

hipError_t launch_gemm_part(const OpMap& A, const OpMap& Bm, int64_t M, int64_t N, int nsplit, double* part,
                            hipStream_t s) {
  return gemm_launch(A, Bm, out_plain(part, M, N, N), 1, nsplit, part, s);
}

hipError_t launch_expand_pairs(const double* part, int nsplit, int64_t M, int64_t nac, double* out1, int64_t M1,
                               double* out2, int accumulate, hipStream_t s) {
  if (M <= 0 || nac <= 0) return hipSuccess;
  if (nac > 32768) return hipErrorInvalidValue;
  const int rpb = (int)std::max<int64_t>(1, 256 / (nac * nac));
  const int64_t nb = cdiv(M, rpb);
  if (nb > 0x7fffffffLL) return hipErrorInvalidValue;
  expand_pairs_kernel<<<(unsigned)nb, 256, 0, s>>>(part, nsplit, M, (int)nac, rpb, out1, M1, out2, accumulate);
  return hipGetLastError();
}

hipError_t launch_split_reduce(const double* part, int nsplit, const OutMap& O, hipStream_t s) {
  const int64_t MN = O.M * O.N;
  if (MN == 0) return hipSuccess;
  const int g = red_group(nsplit);
  const unsigned nb = (unsigned)cdiv(MN, kRedThreads / g);
  if (g == 8) split_reduce_kernel<8><<<nb, kRedThreads, 0, s>>>(part, nsplit, O);
  else split_reduce_kernel<1><<<nb, kRedThreads, 0, s>>>(part, nsplit, O);
  return hipGetLastError();
}

hipError_t launch_gemm_split(const OpMap& A, const OpMap& Bm, const OutMap& O, int nsplit, double* part,
                             hipStream_t s) {
  if (nsplit <= 1) return gemm_launch(A, Bm, O, 1, 1, nullptr, s);
  hipError_t e = gemm_launch(A, Bm, O, 1, nsplit, part, s);
  if (e != hipSuccess) return e;
  return launch_split_reduce(part, nsplit, O, s);
}

// The regions of the P-summed packed product (ReduceRegions): `unit` splits of the 128-wide tiles, and as many
// of the others or, where those take less than 0.7 of the time, up to twice as many as their time is worth, so
// that their items last half as long and no chain of sums is longer than the 128-wide tiles'.  (In proportion to
// the time, the chains of a 48-wide rest were 2.1 times as long; the rounding error of dCocc at 1200 x 4800 x 300
// 1.45e-15 so, 9.8e-16 with chains of 68000 products at most, 6.8e-16 now.)
static double half_tile_time(int rest) {   // of a tile, against 128 columns (rates at CfgH128)
  return rest == 96 ? 0.80 : rest == 64 ? 0.58 : rest == 48 ? 0.48 : rest == 32 ? 0.37 : 0.30;
}
constexpr double kHTailTime = 0.55;
static int64_t region_splits(int64_t unit, double w, int64_t naux) {
  const double f = w < 0.7 ? std::max(1.0, 2.0 * w) : 1.0;
  return std::min<int64_t>(naux, (int64_t)((double)unit * f));
}
static ReduceRegions reduce_regions(int64_t naux, int64_t nao, int64_t N, int64_t unit) {
  const HalfCols h = half_cols(nao, N);
  const HalfTiles T = half_counts(nao, N);
  const bool one = h.nA == 0;   // one narrow tile per band: region a alone
  const int rows = (int)nao - h.tail, ca = one ? (int)N : (int)std::min<int64_t>(N, h.nA * 128);
  ReduceRegions R{};
  R.a = ReduceRegion{0, 0, rows, 0, ca, T.bands, T.nA, (int)std::min(unit, naux), nullptr};
  R.b = ReduceRegion{0, 0, rows, ca, (int)N, T.bands, T.nB, T.nB ? (int)region_splits(unit, half_tile_time(h.rest), naux) : 0, nullptr};
  R.t = ReduceRegion{0, rows, (int)nao, 0, (int)N, T.nT ? 1 : 0, T.nT, T.nT ? (int)region_splits(unit, kHTailTime, naux) : 0, nullptr};
  R.b.item0 = (int64_t)R.a.tilesM * R.a.tilesN * R.a.ns;
  R.t.item0 = R.b.item0 + (int64_t)R.b.tilesM * R.b.tilesN * R.b.ns;
  R.items = R.t.item0 + (int64_t)R.t.tilesM * R.t.tilesN * R.t.ns;
  return R;
}
static int64_t region_part(const ReduceRegion& g) { return (int64_t)g.ns * (g.r1 - g.r0) * (g.c1 - g.c0); }
// workgroups resident at once: three per CU, two with 128-row bands
static int64_t half_resident(const HalfCols& h) { return h.big ? 512 : 768; }
// A chain of sums of the 128-wide tiles has at most this many 16-deep slabs (as far as naux goes): the rounding error
// grows with its length.  At 1200 x 4800 x 300, with 64 such chains, the product was 0.7 per cent faster.
constexpr int64_t kReduceChain = 2048;
static int64_t half_reduce_least(int64_t nao, int64_t naux) {
  return std::max<int64_t>(1, std::min(naux, cdiv(naux * cdiv(nao, 16), kReduceChain)));
}
static int64_t half_reduce_bound(int64_t nao, int64_t N, int64_t naux) {
  // a quarter past the least, to choose one that fills its last round
  return std::min<int64_t>(naux, std::max(half_reduce_least(nao, naux) * 5 / 4,
                                          4 * cdiv(half_resident(half_cols(nao, N)), half_tiles(nao, N))));
}
static int64_t half_reduce_unit(int64_t naux, int64_t nao, int64_t N) {
  const HalfCols h = half_cols(nao, N);
  const int64_t res = half_resident(h);
  const double slab = (h.big ? 4.4 : 3.5) * (h.nA == 0 ? half_tile_time(h.rest) : 1.0);   // us, all resident
  const int64_t most = half_reduce_bound(nao, N, naux);
  int64_t best = 0;
  double best_us = 0.0;
  for (int64_t u = half_reduce_least(nao, naux); u <= most; u += 1 + u / 64) {
    const ReduceRegions R = reduce_regions(naux, nao, N, u);
    // in items of region a: the others' last 0.8 of its, or half and then fill the last round
    const int64_t ia = (int64_t)R.a.tilesM * R.a.tilesN * R.a.ns, ib = R.t.item0 - R.b.item0, it = R.items - R.t.item0;
    const double items = (double)ia + (h.rest == 96 ? 0.8 : 0.5) * (double)ib + 0.5 * (double)it;
    const int64_t w = (int64_t)ceil(items), full = w / res, rem = w % res;
    const double last = h.big ? (rem * 2 <= res ? 0.6 : 1.0) : (rem * 3 <= res ? 0.5 : rem * 3 <= 2 * res ? 0.7 : 1.0);
    const double rounds = it > 0 || (ib > 0 && h.rest != 96) ? items / (double)res + 0.25
                                                             : (double)full + (rem == 0 ? 0.0 : last);
    const double us = (rounds + 0.2) * (double)(cdiv(naux, u) * cdiv(nao, 16) + 4) * slab +
                      (double)u * (double)(nao * N) * 16.0 / 4.0e6;
    if (best == 0 || us < best_us) {
      best_us = us;
      best = u;
    }
  }
  return best;
}

// the partial sums grow with the unit and with naux
int64_t half_reduce_part_bound(int64_t nao, int64_t N, int64_t naux) {
  const ReduceRegions R = reduce_regions(naux, nao, N, half_reduce_bound(nao, N, naux));
  return region_part(R.a) + region_part(R.b) + region_part(R.t);
}

hipError_t launch_half_reduce(const double* B, int64_t naux, int64_t nao, const OpMap& Y, const OutMap& O,
                              double* part, hipStream_t s) {
  if (nao <= 0 || O.N <= 0) return hipSuccess;
  if (naux < 1 || !offsets_fit(Y) || O.s_nh != 0 || O.s_mh != 0 || Y.rows != O.N || O.M != nao)
    return hipErrorInvalidValue;
  ReduceRegions R = reduce_regions(naux, nao, O.N, half_reduce_unit(naux, nao, O.N));
  if (R.items > 0x7fffffffLL) return hipErrorInvalidValue;
  R.a.part = part;
  R.b.part = R.a.part + region_part(R.a);
  R.t.part = R.b.part + region_part(R.b);
  const hipError_t e = half_dispatch(half_cols(nao, O.N), [&](auto ca, auto cb, auto ct) {
    typedef decltype(ca) CA;
    half_reduce_kernel<CA, decltype(cb), decltype(ct)><<<dim3((unsigned)R.items), CA::NT, 0, s>>>(
        B, naux, (int)nao, nao * (nao + 1) / 2, Y, R);
    return hipGetLastError();
  });
  if (e != hipSuccess) return e;
  for (const ReduceRegion* g : {&R.a, &R.b, &R.t}) {
    if (g->ns == 0) continue;
    OutMap Og = O;   // the region's rows and columns of O
    if (g->c0 < O.nsplit) {
      Og.p += g->c0 * Og.s_nl;
      Og.nsplit -= g->c0;
    } else {
      Og.p2 += g->c0 - O.nsplit;
      Og.nsplit = 0;
    }
    Og.M = g->r1 - g->r0;
    Og.N = g->c1 - g->c0;
    if (Og.nsplit > 0) Og.p += g->r0 * Og.s_ml;
    if (Og.p2) Og.p2 += g->r0 * Og.s2_m;
    if (hipError_t er = launch_split_reduce(g->part, g->ns, Og, s)) return er;
  }
  return hipSuccess;
}

hipError_t launch_pair_weights(const double* G, int64_t nao, double* g, hipStream_t s) {
  const int64_t npair = nao * (nao + 1) / 2;
  if (npair == 0) return hipSuccess;
  pair_weights_kernel<<<(unsigned)cdiv(npair, 256), 256, 0, s>>>(G, nao, g);
  return hipGetLastError();
}

hipError_t launch_dens_pairs(const double* C, int64_t nao, int64_t nocc, int64_t ndm, double* D, double* Dw,
                             hipStream_t s) {
  const int64_t npair = nao * (nao + 1) / 2;
  if (npair == 0 || ndm == 0) return hipSuccess;
  if (ndm > 65535) return hipErrorInvalidValue;
  // D_z = C_z C_z^T on the matrix cores, then packed with the pair weights
  OpMap Cz = op_map(C, nao, nocc, nocc, 1);
  Cz.s_z = nao * nocc;
  OutMap O = out_plain(D, nao, nao, nao);
  O.s_z = nao * nao;
  hipError_t e = launch_gemm(Cz, Cz, O, ndm, s);
  if (e != hipSuccess) return e;
  pair_weights_kernel<<<dim3((unsigned)cdiv(npair, 256), (unsigned)ndm), 256, 0, s>>>(D, nao, Dw);
  return hipGetLastError();
}

int jvec_packed_chunks() { return kJvChunks; }

hipError_t launch_jvec_packed(const double* B, int64_t naux, int64_t nao, const double* g, double* part, double* u,
                              hipStream_t s) {
  if (naux == 0) return hipSuccess;
  jvec_packed_kernel<<<dim3((unsigned)cdiv(naux, kJvRows), kJvChunks), 256, 0, s>>>(B, naux, nao * (nao + 1) / 2, g,
                                                                                    part);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  jvec_chunks_kernel<<<(unsigned)cdiv(naux, 256), 256, 0, s>>>(part, naux, u);
  return hipGetLastError();
}

hipError_t launch_symmetrize(const double* in, int64_t n, int64_t nz, double* out, hipStream_t s) {
  const int64_t tot = n * n * nz;
  if (tot == 0) return hipSuccess;
  symmetrize_kernel<<<(unsigned)cdiv(tot, 256), 256, 0, s>>>(in, n, nz, out);
  return hipGetLastError();
}



// Gram products: tile and split count of least estimated time over the tiles of the triangle, the
// partial sums (written, read, and the reduction's launch) included; at most 64 MB of partials
// beyond the first.
static int64_t gram_tiles(int64_t M, bool small) {
  const int64_t T = cdiv(M, small ? CfgSmall::BM : CfgSq::BM);
  return T * (T + 1) / 2;
}
static int gram_plan(int64_t M, int64_t nslab, int max_split, bool* small) {
  int best = 1;
  double best_us = 0.0;
  const int64_t most = std::max<int64_t>(1, std::min<int64_t>({nslab / 4, max_split, 1 + (int64_t(8) << 20) / std::max<int64_t>(M * M, 1)}));
  *small = false;
  for (int ns = 1; ns <= most; ++ns)
    for (int sm = 0; sm < 2; ++sm) {
      const double us = gemm_us(gram_tiles(M, sm) * ns, (double)cdiv(nslab, ns), sm) +
                        (ns > 1 ? 5.0 + (double)ns * (double)(M * M) * 8.0 / 4.0e6 : 0.0);
      if ((ns == 1 && sm == 0) || us < best_us) {
        best_us = us;
        best = ns;
        *small = sm;
      }
    }
  return best;
}
int64_t gram_part(int64_t M, int64_t nslab) {
  bool small;
  const int ns = gram_plan(M, nslab, 64, &small);
  return ns > 1 ? ns * M * M : 0;
}

template <class Cg>
static void gram_go(const OpMap& A, double* G, int64_t npairs, int ns, int accumulate, double* part, hipStream_t s) {
  const dim3 grid((unsigned)npairs, (unsigned)ns);
  if (A.kc_n % 16 != 0) gram_kernel<Cg, true><<<grid, Cg::NT, 0, s>>>(A, G, npairs, accumulate, part);
  else gram_kernel<Cg, false><<<grid, Cg::NT, 0, s>>>(A, G, npairs, accumulate, part);
}

hipError_t launch_gram(const OpMap& A, double* G, double* part, int64_t part_n, int accumulate, hipStream_t s) {
  const int64_t M = A.rows;
  if (M <= 0) return hipSuccess;
  if (!offsets_fit(A)) return hipErrorInvalidValue;
  bool small;
  const int64_t room = part ? part_n / (M * M) : 0;
  const int ns = gram_plan(M, gemm_slabs(A), (int)std::max<int64_t>(1, std::min<int64_t>(room, 64)), &small);
  const int64_t npairs = gram_tiles(M, small);
  if (npairs > 0x7fffffffLL) return hipErrorInvalidValue;
  double* pt = ns > 1 ? part : nullptr;
  if (small) gram_go<CfgSmall>(A, G, npairs, ns, accumulate, pt, s);
  else gram_go<CfgSq>(A, G, npairs, ns, accumulate, pt, s);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || !pt) return e;
  return launch_syrk_reduce(pt, ns, M, 1, G, s, accumulate);
}

int syrk_tile_for(int64_t n) { return n <= 640 ? CfgSyrk64::BM : CfgSyrk::BM; }

static int scaled_splits(int unit, double w, int64_t kb_n) {
  return (int)std::max<int64_t>(1, std::min<int64_t>(kb_n, (int64_t)((double)unit * w + 0.5)));
}
// Tiles of an n x n SYRK with `unit` splits of the 64 x 128 tiles over `slabs` slabs in kb_n blocks; a 64 x 64 tile
// takes 0.58 and a 32 x 128 one 0.55 of their time (rates at CfgH128).
static SyrkTiles syrk_tiles(int64_t n, int64_t kb_n, int64_t slabs, int unit) {
  SyrkTiles T{};
  const int64_t rows = n % CfgKA::BM, tail = n > CfgKA::BM && rows > 0 && rows <= CfgKT::BM ? rows : 0;
  T.bands = (int)cdiv(n - tail, CfgKA::BM);
  T.a = T.bands * T.bands / 4;
  T.d = (T.bands + 1) / 2;
  T.t = tail ? (int)cdiv(n, CfgKT::BN) : 0;
  T.na = unit;
  T.nd = scaled_splits(unit, 0.58, kb_n);
  T.nt = T.t ? scaled_splits(unit, 0.55, kb_n) : 0;
  // halves of 64 slabs at least: an item's prologue and epilogue take about four
  if (T.nd < unit && slabs >= (int64_t)128 * T.nd) {
    T.nd = (int)std::min<int64_t>(2 * T.nd, kb_n);
    T.nt = (int)std::min<int64_t>(2 * T.nt, kb_n);
  }
  return T;
}
static SyrkTiles syrk_tiles(const OpMap& A, int64_t n, int unit) {
  return syrk_tiles(n, A.kb_n, cdiv(A.kb_n * A.kc_n, 16), unit);
}

// The most units: four rounds of resident workgroups, or five where that leaves fewer than 64.  With four, N_ao = 1200
// had 32, chains of 45000 products.
static int64_t syrk_most(int64_t n, int64_t kb_n, int64_t nz) {
  const SyrkTiles T = syrk_tiles(n, 1, 0, 1);
  const int64_t per = cdiv(768, (T.a + T.d + T.t) * std::max<int64_t>(nz, 1));
  return std::max<int64_t>(1, std::min<int64_t>({kb_n, 4096, std::max(4 * per, std::min<int64_t>(5 * per, 64))}));
}
int syrk_splits_bound(int64_t n, int64_t kb_n, int64_t nz) { return (int)syrk_most(n, kb_n, nz); }

// Units of least estimated time, as in half_reduce_unit (halved D and T items count as whole ones): three workgroups per
// CU, 3.5 us a slab of a 64 x 128 tile (two 2.4, one 1.6); partial sums of the triangle written and read.
// At least one unit per 640 slabs, as far as there may be so many: the rounding error grows with the length of a chain.
int syrk_splits(int64_t n, int64_t kb_n, int64_t kc_n, int64_t nz) {
  if (nz < 1) nz = 1;
  const int64_t most = syrk_most(n, kb_n, nz), slabs = cdiv(kb_n * kc_n, 16);
  const int least = (int)std::max<int64_t>(1, std::min(most, cdiv(slabs, 640)));
  int best = least;
  double best_us = 0.0;
  for (int u = least; u <= most; u += 1 + u / 32) {   // (every count: 25 us of host time at N_ao 64)
    const int64_t w = syrk_tiles(n, kb_n, 0, u).items() * nz, full = w / 768, rem = w % 768;
    const double last = rem == 0 ? 0.0 : rem <= 256 ? 1.6 : rem <= 512 ? 2.4 : 3.5;
    const double us = ((double)full * 3.5 + last + 0.7) * (double)(cdiv(slabs, u) + 4) +
                      (double)u * (double)(n * (n + 1) / 2 * nz) * 16.0 / 4.0e6;
    if (u == least || us < best_us * (1.0 - 1e-9)) {
      best_us = us;
      best = u;
    }
  }
  return best;
}
int64_t syrk_parts(int64_t kb_n, int unit) {
  return std::max<int64_t>(unit, std::min<int64_t>(kb_n, 2 * scaled_splits(unit, 0.58, kb_n)));
}

hipError_t launch_syrk_partial(const OpMap& A, const OpMap& Bw, int64_t n, int64_t nz, int nsplit, double* Kpart,
                               hipStream_t s) {
  if (n == 0 || nz == 0) return hipSuccess;
  const SyrkTiles T = syrk_tiles(A, n, nsplit);
  if (nz > 65535 || !offsets_fit(A) || T.items() > 0x7fffffffLL) return hipErrorInvalidValue;
  const dim3 grid((unsigned)T.items(), 1, (unsigned)nz);
  const bool clamp = A.kc_n % 16 != 0;
  // contraction chunks that are not whole slabs: one flat contraction (no padded slabs) unless
  // weighted or shorter than a slab
  const bool flat = clamp && !Bw.ks && flat_pays(A) && flat_fits(A);
  if (Bw.ks) syrk_kernel<true, true, false><<<grid, CfgKA::NT, 0, s>>>(A, Bw, n, nz, T, Kpart);
  else if (flat) syrk_kernel<false, false, true><<<grid, CfgKA::NT, 0, s>>>(A, Bw, n, nz, T, Kpart);
  else if (clamp) syrk_kernel<false, true, false><<<grid, CfgKA::NT, 0, s>>>(A, Bw, n, nz, T, Kpart);
  else syrk_kernel<false, false, false><<<grid, CfgKA::NT, 0, s>>>(A, Bw, n, nz, T, Kpart);
  return hipGetLastError();
}

// ---- grouped launches ----
// Cuts items [0, start[n]) into 8 contiguous chunks of about equal cost (each item of problem p
// costs cost[p]) and returns the length of the longest (the grid is 8 times that).
static int64_t xcd_chunks(const int64_t* start, const double* cost, int n, int64_t* xs) {
  double total = 0.0;
  for (int p = 0; p < n; ++p) total += (double)(start[p + 1] - start[p]) * cost[p];
  xs[0] = 0;
  int p = 0;
  double before = 0.0;   // cost of the items of problems before p
  for (int x = 1; x < 8; ++x) {
    const double target = total * x / 8.0;
    while (p < n && before + (double)(start[p + 1] - start[p]) * cost[p] <= target) {
      before += (double)(start[p + 1] - start[p]) * cost[p];
      ++p;
    }
    int64_t i = start[n];
    if (p < n) {
      i = start[p] + (int64_t)((target - before) / cost[p] + 0.5);
      if (i > start[p + 1]) i = start[p + 1];
    }
    xs[x] = i < xs[x - 1] ? xs[x - 1] : i;
  }
  xs[8] = start[n];
  int64_t longest = 1;
  for (int x = 0; x < 8; ++x) longest = xs[x + 1] - xs[x] > longest ? xs[x + 1] - xs[x] : longest;
  return longest;
}

template <class CA, class CB, class CT>
static hipError_t half_group_go(const GroupHalf* probs, int n, hipStream_t s) {
  constexpr bool kB = !std::is_same<CA, CB>::value, kT = !std::is_same<CA, CT>::value;
  HalfGroup g{};
  g.n = n;
  g.start[0] = 0;
  double cost[kMaxGroup];   // slabs per item, plus about two for the prologue and the epilogue
  for (int p = 0; p < n; ++p) {
    const GroupHalf& q = probs[p];
    HalfDesc& d = g.d[p];
    d.B = q.B;
    d.nao = (int)q.nao;
    d.npair = q.nao * (q.nao + 1) / 2;
    d.Cm = op_map(q.C, q.ncol, 1, q.nao, q.ldc);
    d.out = q.out;
    // the rest of the columns and of the rows on CB and CT where those hold them
    const int64_t rem = q.ncol % CA::BN, rows = q.nao % CA::BM;
    const bool tail = kT && rows > 0 && rows <= CT::BM && q.ncol >= CT::BN;
    d.T.nB = kB && rem > 0 && rem <= CB::BN && q.ncol >= CA::BN ? 1 : 0;
    d.T.nA = (int)(d.T.nB ? q.ncol / CA::BN : cdiv(q.ncol, CA::BN));
    d.T.bands = (int)(tail ? q.nao / CA::BM : cdiv(q.nao, CA::BM));
    d.T.nT = tail ? (int)cdiv(q.ncol, CT::BN) : 0;
    if (!offsets_fit(d.Cm) || q.out.alpha != 1.0 || q.out.accumulate) return hipErrorInvalidValue;
    g.start[p + 1] = g.start[p] + d.T.count() * q.naux;
    const double w = d.T.bands * (d.T.nA + 0.6 * d.T.nB) + kHTailTime * d.T.nT;
    cost[p] = ((double)cdiv(q.nao, CA::BK) + 2.0) * w / (double)std::max<int64_t>(1, d.T.count());
  }
  if (g.start[g.n] == 0) return hipSuccess;
  if (g.start[g.n] > 0x7fffffffLL) return hipErrorInvalidValue;
  const int64_t per = xcd_chunks(g.start, cost, g.n, g.xs);
  if (8 * per > 0x7fffffffLL) return hipErrorInvalidValue;
  half_group_kernel<CA, CB, CT><<<(unsigned)(8 * per), CA::NT, 0, s>>>(g);
  return hipGetLastError();
}

hipError_t launch_half_group(const GroupHalf* probs, int n, int tile_n, hipStream_t s) {
  if (n < 1 || n > kMaxGroup) return hipErrorInvalidValue;
  switch (tile_n) {
    case 176: return half_group_go<CfgH176, CfgH176, CfgH176>(probs, n, s);
    case 96: return half_group_go<CfgH96, CfgH96, CfgH96>(probs, n, s);
    case 48: return half_group_go<CfgH48, CfgH48, CfgH48>(probs, n, s);
    case 0:
    case 128: return half_group_go<CfgH128, CfgH64, CfgHTail>(probs, n, s);
    default: return hipErrorInvalidValue;
  }
}

template <class Cg>
static hipError_t syrk_group_go(const GroupSyrk* probs, int n, hipStream_t s) {
  SyrkGroup g{};
  g.n = n;
  g.start[0] = 0;
  bool clamp = false, flat_ok = true, flat_any = false;
  for (int p = 0; p < n; ++p) {
    const GroupSyrk& q = probs[p];
    SyrkDesc& d = g.d[p];
    d.A = q.A;
    d.n = q.n;
    d.nz = q.nz;
    const int64_t T = cdiv(q.n, Cg::BM);
    d.npairs = T * (T + 1) / 2;
    d.nsplit = q.nsplit;
    d.Kpart = q.Kpart;
    if (!offsets_fit(q.A) || q.nsplit < 1) return hipErrorInvalidValue;
    clamp = clamp || q.A.kc_n % 16 != 0;
    flat_ok = flat_ok && q.A.kc_n >= 16 && flat_fits(q.A);
    flat_any = flat_any || flat_pays(q.A);
    g.start[p + 1] = g.start[p] + d.npairs * d.nsplit * q.nz;
  }
  if (g.start[n] == 0) return hipSuccess;
  if (g.start[n] > 0x7fffffffLL) return hipErrorInvalidValue;
  // contraction chunks that are not whole slabs: one flat contraction per density (no padded
  // slabs) when every chunk is at least a slab long and the padding would cost
  const bool flat = clamp && flat_ok && flat_any;
  double cost[kMaxGroup];   // slabs of one split, plus about two for the prologue and the epilogue
  for (int p = 0; p < n; ++p) {
    const OpMap& A = g.d[p].A;
    cost[p] = (flat ? (double)cdiv(A.kb_n * A.kc_n, Cg::BK) / g.d[p].nsplit
                    : (double)cdiv(A.kb_n, g.d[p].nsplit) * (double)cdiv(A.kc_n, Cg::BK)) + 2.0;
  }
  const int64_t per = xcd_chunks(g.start, cost, n, g.xs);
  if (8 * per > 0x7fffffffLL) return hipErrorInvalidValue;
  if (flat) syrk_group_kernel<Cg, false, true><<<(unsigned)(8 * per), Cg::NT, 0, s>>>(g);
  else if (clamp) syrk_group_kernel<Cg, true><<<(unsigned)(8 * per), Cg::NT, 0, s>>>(g);
  else syrk_group_kernel<Cg, false><<<(unsigned)(8 * per), Cg::NT, 0, s>>>(g);
  return hipGetLastError();
}

int syrk_group_tile(const GroupSyrk* probs, int n) {
  int64_t nmax = 0;
  for (int p = 0; p < n; ++p) nmax = probs[p].n > nmax ? probs[p].n : nmax;
  return syrk_tile_for(nmax);
}

hipError_t launch_syrk_group(const GroupSyrk* probs, int n, int tile, hipStream_t s) {
  if (n < 1 || n > kMaxGroup) return hipErrorInvalidValue;
  if (tile == 0) tile = syrk_group_tile(probs, n);
  if (tile == CfgSyrk64::BM) return syrk_group_go<CfgSyrk64>(probs, n, s);
  if (tile == CfgSyrk::BM) return syrk_group_go<CfgSyrk>(probs, n, s);
  return hipErrorInvalidValue;
}

static hipError_t syrk_reduce_go(const double* Kpart, const SyrkTiles& T, int64_t n, int64_t nz, double* K,
                                 hipStream_t s, int accumulate) {
  const int64_t npair = n * (n + 1) / 2;
  if (npair == 0 || nz == 0) return hipSuccess;
  if (nz > 65535) return hipErrorInvalidValue;
  const int g = red_group(T.na);
  const dim3 grid((unsigned)cdiv(npair, kRedThreads / g), (unsigned)nz);
  if (g == 8) syrk_reduce_kernel<8><<<grid, kRedThreads, 0, s>>>(Kpart, T, n, npair, K, accumulate);
  else syrk_reduce_kernel<1><<<grid, kRedThreads, 0, s>>>(Kpart, T, n, npair, K, accumulate);
  return hipGetLastError();
}

hipError_t launch_syrk_reduce(const double* Kpart, int nsplit, int64_t n, int64_t nz, double* K, hipStream_t s,
                              int accumulate) {
  SyrkTiles T{};
  T.na = nsplit;
  return syrk_reduce_go(Kpart, T, n, nz, K, s, accumulate);
}

hipError_t launch_syrk_partial_reduce(const double* Kpart, const OpMap& A, int nsplit, int64_t n, int64_t nz, double* K,
                                      hipStream_t s, int accumulate) {
  return syrk_reduce_go(Kpart, syrk_tiles(A, n, nsplit), n, nz, K, s, accumulate);
}

hipError_t launch_jvec(const double* X, int64_t naux, int64_t nao, int64_t ldx, const double* C, const double* w,
                       int64_t nocc, int64_t nz, double* v, hipStream_t s, int accumulate, int64_t ldv) {
  if (naux == 0 || nz == 0) return hipSuccess;
  if (nz > 65535 || naux > 0x7fffffffLL || (ldv != 0 && ldv < naux)) return hipErrorInvalidValue;
  jvec_kernel<<<dim3((unsigned)naux, (unsigned)nz), 256, 0, s>>>(X, nao, ldx, C, w, nocc, v, ldv ? ldv : naux,
                                                                  accumulate);
  return hipGetLastError();
}

// P splits of a Coulomb build: enough workgroups to keep HBM busy (1024 with at least 4 rows of B
// each; with one split N_ao = 120 had 8 workgroups).  None where the pairs alone give 512 (at 704,
// N_ao = 1200, two splits read B no faster).  Unsplit against split: step at 120 x 480 583 -> 415 us,
// J and K at 77 x 310 260 -> 157 us, two densities at 455 x 1822 8.21 -> 7.31 ms.
constexpr int64_t kCoulombFull = 512;
static int coulomb_want(int64_t naux, int64_t nao) {
  const int64_t bx = cdiv(nao * (nao + 1) / 2, 256 * kCoulombPairs);
  if (bx >= kCoulombFull) return 1;
  return (int)std::max<int64_t>(1, std::min<int64_t>({cdiv(1024, bx), naux / 4, 128}));
}

int64_t coulomb_part(int64_t naux, int64_t nao, int64_t nz) {
  const int64_t s = coulomb_want(naux, nao);
  return s > 1 ? s * std::min<int64_t>(nz, kCoulombZ) * (nao * (nao + 1) / 2) : 0;
}

hipError_t launch_coulomb(const double* B, int64_t naux, int64_t nao, const double* v, int64_t nz, double* J,
                          double* part, int64_t part_n, hipStream_t s, int accumulate, int64_t ldv) {
  const int64_t npair = nao * (nao + 1) / 2;
  if (ldv == 0) ldv = naux;
  if (ldv < naux) return hipErrorInvalidValue;
  const bool deep = cdiv(npair, 256 * kCoulombPairs) < kCoulombFull;
  for (int64_t z0 = 0; z0 < nz; z0 += kCoulombZ) {
    const int nzc = (int)(nz - z0 < kCoulombZ ? nz - z0 : kCoulombZ);
    const int64_t room = part ? part_n / (nzc * npair) : 0;
    const int ns = (int)std::max<int64_t>(1, std::min<int64_t>(coulomb_want(naux, nao), room));
    double* pt = ns > 1 ? part : nullptr;
    const dim3 grid((unsigned)cdiv(npair, 256 * kCoulombPairs), (unsigned)ns);
    const double* vz = v + z0 * ldv;
    double* Jz = J + z0 * nao * nao;
    auto go = [&](auto k) {
      constexpr int NZ = decltype(k)::value;
      if (deep) coulomb_kernel<NZ, true><<<grid, 256, 0, s>>>(B, naux, nao, npair, vz, ldv, Jz, nao * nao, accumulate, pt);
      else coulomb_kernel<NZ, false><<<grid, 256, 0, s>>>(B, naux, nao, npair, vz, ldv, Jz, nao * nao, accumulate, pt);
    };
    switch (nzc) {
      case 1: go(std::integral_constant<int, 1>{}); break;
      case 2: go(std::integral_constant<int, 2>{}); break;
      case 3: go(std::integral_constant<int, 3>{}); break;
      default: go(std::integral_constant<int, 4>{});
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (pt) {
      const int g = red_group(ns);
      const dim3 rg((unsigned)cdiv(npair, kRedThreads / g), (unsigned)nzc);
      if (g == 8) coulomb_reduce_kernel<8><<<rg, kRedThreads, 0, s>>>(pt, ns, nao, npair, Jz, accumulate);
      else coulomb_reduce_kernel<1><<<rg, kRedThreads, 0, s>>>(pt, ns, nao, npair, Jz, accumulate);
      e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
  }
  return hipSuccess;
}

hipError_t launch_gather_cols(const ColBlocks& k, int64_t nao, int64_t rows, double* dst, hipStream_t s) {
  const int64_t total = rows * (k.n0 + k.nz * k.n1 + k.n2);
  if (total <= 0) return hipSuccess;
  if ((k.n0 > 0 && !k.s0) || (k.nz * k.n1 > 0 && !k.s1) || (k.n2 > 0 && !k.s2)) return hipErrorInvalidValue;
  gather_cols_kernel<<<(unsigned)std::min<int64_t>(cdiv(total, 256), 16384), 256, 0, s>>>(k, nao, total, dst);
  return hipGetLastError();
}

hipError_t launch_add(const double* x, int64_t n, double* y, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  add_kernel<<<(unsigned)cdiv(n, 256), 256, 0, s>>>(x, n, y);
  return hipGetLastError();
}

hipError_t launch_copy_rows(const double* x, int64_t rows, int64_t cols, double* y, int64_t ldy, int accumulate,
                            hipStream_t s) {
  if (rows <= 0 || cols <= 0) return hipSuccess;
  if (ldy < cols) return hipErrorInvalidValue;
  copy_rows_kernel<<<(unsigned)cdiv(rows * cols, 256), 256, 0, s>>>(x, rows, cols, y, ldy, accumulate);
  return hipGetLastError();
}

hipError_t launch_scale_cols(const double* X, int64_t n, int64_t ncol, const double* w, double* Xw, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  if (ncol <= 0) return hipErrorInvalidValue;
  scale_cols_kernel<<<(unsigned)cdiv(n, 256), 256, 0, s>>>(X, n, ncol, w, Xw);
  return hipGetLastError();
}

hipError_t launch_fill_zero(double* p, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  fill_zero_kernel<<<(unsigned)cdiv(n, 256), 256, 0, s>>>(p, n);
  return hipGetLastError();
}

hipError_t launch_unpack_sym(const double* Jp, int64_t nz, int64_t nao, double* J, hipStream_t s) {
  const int64_t npair = nao * (nao + 1) / 2, tot = nz * npair;
  if (tot <= 0) return hipSuccess;
  unpack_sym_kernel<<<(unsigned)cdiv(tot, 256), 256, 0, s>>>(Jp, nz, nao, npair, J);
  return hipGetLastError();
}

hipError_t launch_chol_block(double* A, int64_t lda, int kb, double* Linv, int* info, int64_t k0, bool first,
                             hipStream_t s) {
  if (kb < 1 || kb > kCholNB) return hipErrorInvalidValue;
  chol_block_kernel<<<1, 256, 0, s>>>(A, lda, kb, Linv, info, k0, first ? 1 : 0);
  return hipGetLastError();
}

hipError_t launch_subst_row(const double* L, int64_t ldl, int64_t k, const double* E, const double* Linv, int kb,
                            int64_t npair, double* B, hipStream_t s) {
  if (kb < 1 || kb > kCholNB || npair < 1) return hipErrorInvalidValue;
  // the contraction over the k earlier (full) blocks, one 64-bit-strided block of B each
  OpMap A = op_map(L, kb, ldl, kCholNB, 1);
  A.kb_n = k;
  A.s_kb = kCholNB;
  OpMap Bm = op_map(B, npair, 1, kCholNB, npair);
  Bm.kb_n = k;
  Bm.s_kb = kCholNB * npair;
  const int64_t nblk = cdiv(npair, CfgSub::BN);
  // without earlier blocks nothing is read through A and Bm; E and B take 64-bit offsets
  if (nblk > 0x7fffffffLL || (k > 0 && (!offsets_fit(A) || !offsets_fit(Bm)))) return hipErrorInvalidValue;
  subst_row_kernel<<<(unsigned)nblk, CfgSub::NT, 0, s>>>(A, Bm, k * (kCholNB / CfgSub::BK), E, Linv, kb, npair,
                                                         B + k * kCholNB * npair);
  return hipGetLastError();
}

hipError_t launch_zero_upper(double* A, int64_t n, hipStream_t s) {
  if (n <= 1) return hipSuccess;
  zero_upper_kernel<<<(unsigned)cdiv(n * n, 256), 256, 0, s>>>(A, n);
  return hipGetLastError();
}

hipError_t launch_pack_lower(const double* A, int64_t s_z, int64_t nz, int64_t n, double* Ap, hipStream_t s) {
  const int64_t npair = n * (n + 1) / 2, tot = nz * npair;
  if (tot <= 0) return hipSuccess;
  pack_lower_kernel<<<(unsigned)cdiv(tot, 256), 256, 0, s>>>(A, s_z, nz, n, npair, Ap);
  return hipGetLastError();
}

hipError_t launch_fill_zero_strided(double* p, int64_t nz, int64_t s_z, int64_t n, hipStream_t s) {
  const int64_t tot = n * nz;
  if (tot <= 0) return hipSuccess;
  fill_zero_strided_kernel<<<(unsigned)cdiv(tot, 256), 256, 0, s>>>(p, nz, s_z, n);
  return hipGetLastError();
}

}  // namespace dfk
