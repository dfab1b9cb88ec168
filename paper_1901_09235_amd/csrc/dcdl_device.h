// dcdl_device.h -- gfx950 device code of the DiCoDiLe CSC library.
//
// Internal layout (all on the device):
//   beta, z : position-major (H, W, KS), the atom index innermost and padded
//             to KS = K rounded up to a 16-byte vector (4 floats or 2 doubles;
//             padding entries stay 0).  The beta patch of one update (Sec. 3,
//             eq. beta_update) is (2L1-1) contiguous, 16-byte aligned runs of
//             (2L2-1)*KS values, read and written as vectors.
//   score   : per position, the best move score over its K atoms (Alg. 1's
//             selection key); read by neighbouring workers, so it is accessed
//             with coherent atomics.
//   meta    : per position, the number of non-zero atoms (high 16 bits);
//             private to the owner.  The atom of a best move is not kept: the
//             worker that selects a position finds it from beta and z.
//   A       : apply table A[k0][d1][d2][k] = DtD[k][k0][d1][d2] (k padded to KS):
//             the row of eq. beta_update for an update of atom k0, indexed by
//             the offset d = w - w0 + L - 1 of the patched position w.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dcdl {

template <class R> struct Vec;
template <> struct Vec<float> {
  typedef float4 T;
  static constexpr int N = 4;
  static __device__ __forceinline__ float get(const float4 &v, int e) {
    return e == 0 ? v.x : e == 1 ? v.y : e == 2 ? v.z : v.w;
  }
  static __device__ __forceinline__ float4 zero() { return make_float4(0.f, 0.f, 0.f, 0.f); }
};
template <> struct Vec<double> {
  typedef double2 T;
  static constexpr int N = 2;
  static __device__ __forceinline__ double get(const double2 &v, int e) { return e == 0 ? v.x : v.y; }
  static __device__ __forceinline__ double2 zero() { return make_double2(0.0, 0.0); }
};

// Padded atom stride: K rounded up to a whole vector.
__host__ __device__ inline int atom_stride(int K, int elem_bytes) {
  const int ve = 16 / elem_bytes;
  return (K + ve - 1) / ve * ve;
}

// Per-instance control block, followed in memory by a ring of kRing 64-bit
// per-round counters (completions in the low word, quiet workers in the high
// word).
struct Ctl {
  int32_t converged;
  int32_t stop;
  int32_t status;  // 0 ok, 1 round cap, 2 diverged, 3 neighbour wait timed out
  int32_t max_round;
  int32_t sweeps_done;
  int32_t pad[3];
  unsigned long long n_updates, n_candidates, n_softlocked;
  unsigned long long n_visits;        // rounds in which a worker scanned a sub-domain
  unsigned long long n_checked;       // positions read by soft-lock tests
  unsigned long long n_patched;       // positions of beta patched (summed over workers)
  unsigned long long tk_wait, tk_select, tk_collect, tk_apply;  // clock ticks summed over workers
};
constexpr int kRing = 4096;

// Everything one instance of eq. csc needs inside the round kernel.
template <class R> struct Inst {
  int K, KS, L1, L2, U1, U2;
  int H, W;
  int W1, W2, tile1, tile2, mmax, wg_base;
  // workgroups ("teams") of this instance: TW1 x TW2, each running a block of
  // G1 x G2 workers (fewer at the far edges)
  int G1, G2, TW1, TW2;
  int lane_sh;  // lane_map(KS / vector).sh
  int box_share;   // area per update of a box that a round's updates are patched in together (0: never)
  int inner;  // sub-domain visits per round (at most Mw); 0 -> 1
  int positive, certify, soft_lock;
  int strategy;  // dcdl_select: 0 LGCD, 1 greedy, 2 cyclic (both through tile1/tile2), 3 random
  R lambda, tol, div_guard;
  long long max_rounds;
  long long budget_ticks;  // wall-clock cap of one launch, 100 MHz clock ticks
  unsigned long long seed;  // generator seed of the random rule
  R *beta, *z;
  R *score;        // shared: coherent accesses only
  uint32_t *meta;  // private to the owning worker
  const R *A, *inv_n;
  unsigned long long *cand;  // kCandWords words per worker
  int *prog;                 // one word per team
  Ctl *ctl;
  int *ring;  // kRing 64-bit slots: completions (low word) and quiet workers (high word) of a round
  // optional, 2 per worker: visits so far and the quiet count, loaded at the
  // start of a launch and stored at its end, so that a solve split over
  // several launches (each capped by max_rounds) keeps its stopping state
  long long *wstate;
  // optional round log: for rounds r < audit_rounds, audit[r * W1 W2 + w]
  // records worker w's published candidate (audit_record)
  unsigned long long *audit;
  int audit_rounds;
};

// A worker's published candidate of one round: 0 when it had none; otherwise
// bit 63 set, bit 62 set if it passed the soft-lock test (and was applied),
// the atom in bits 32..47 and the position (row-major in the valid domain)
// in bits 0..31.
__device__ __forceinline__ unsigned long long audit_record(bool has, bool accepted, int k0, int pos) {
  if (!has) return 0ull;
  return (1ull << 63) | ((accepted ? 1ull : 0ull) << 62) | ((unsigned long long)(k0 & 0xffff) << 32) |
         (unsigned long long)(unsigned)pos;
}

// ----------------------------------------------------------------- arithmetic

// Closed-form coordinate target of eq. pb_coord: ST(b, lambda) / ||D_k||^2,
// one-sided when positive.  The product is rounded on its own (no
// contraction into a later subtraction): the move score |zn - z| must be that
// of the value z takes, or a coordinate at its target keeps a score of the
// size of zn's rounding error and a tolerance below it is never certified.
template <class R>
__device__ __forceinline__ R st_target(R b, R lam, R inv_n, int positive) {
#pragma clang fp contract(off)
  R u;
  if (positive)
    u = b > lam ? b - lam : R(0);
  else
    u = b > lam ? b - lam : (b < -lam ? b + lam : R(0));
  return u * inv_n;
}

// Selection score of the move z -> zn: |zn - z|, raised to at least tol for a
// move that changes the support or the sign when certify is set.
template <class R>
__device__ __forceinline__ R move_score(R z, R zn, R tol, int certify) {
  R dz = zn > z ? zn - z : z - zn;
  if (certify && z != R(0) && (zn == R(0) || ((zn > R(0)) != (z > R(0)))))
    dz = dz > tol ? dz : tol;
  return dz;
}

// Counter-based draw of the random selection rule: SplitMix64 (Steele, Lea
// and Flood, OOPSLA 2014).  Its n-th output from seed s mixes
// s + (n + 1) * 0x9e3779b97f4a7c15 with two xor-shift-multiply steps and a
// final xor-shift; worker w draws at counter n + w * 2^40.
__device__ __forceinline__ unsigned long long sm64_draw(unsigned long long seed, unsigned long long w,
                                                        unsigned long long n) {
  unsigned long long x = seed + ((w << 40) + n + 1ull) * 0x9e3779b97f4a7c15ull;
  x = (x ^ (x >> 30)) * 0xbf58476d1ce4e5b9ull;
  x = (x ^ (x >> 27)) * 0x94d049bb133111ebull;
  return x ^ (x >> 31);
}

__device__ __forceinline__ int part_start(int j, int N, int Wn) {
  return (int)(((long long)j * N) / Wn);
}
// part_start in 32 bits where its products fit.
__device__ __forceinline__ int part_start_fast(int j, int N, int Wn) {
  if (((unsigned long long)(unsigned)N * (unsigned)Wn) >> 32) return part_start(j, N, Wn);
  return (int)((unsigned)j * (unsigned)N / (unsigned)Wn);
}
__device__ __forceinline__ int part_owner(int x, int N, int Wn) {
  return (int)((((long long)x + 1) * Wn - 1) / N);
}

// n / d for 0 <= n < 2^22 and d >= 1, in a few instructions.
__device__ __forceinline__ int div_small(int n, int d) {
  int q = (int)((float)n * __builtin_amdgcn_rcpf((float)d));
  const int rest = n - q * d;
  if (rest < 0) --q;
  if (rest >= d) ++q;
  return q;
}

// ------------------------------------------------------------ synchronisation
//
// Workers exchange three kinds of data: the cached best move of positions on
// their borders (read by the soft-lock test of a neighbour), the candidate of
// each round and a progress counter.  These are read and written only with
// relaxed agent-scope atomics, which are coherent across the chip's L2
// caches; a writer waits for its atomic stores to complete (vmcnt 0) before it
// publishes the progress counter or the tag of a candidate, and a reader
// issues its reads after it observed that counter or tag.  beta, z and the
// DtD table are only ever touched by one workgroup during a launch and stay
// in ordinary cached memory, so no cache write-back or invalidation is
// needed between rounds.

__device__ __forceinline__ unsigned long long ld_shared_u64(const unsigned long long *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_shared_u64(unsigned long long *p, unsigned long long v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int ld_shared_i32(const int *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_shared_i32(int *p, int v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Wait until every vector memory operation this wave issued has completed.
__device__ __forceinline__ void wait_vm() {
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0), expcnt/lgkmcnt untouched
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

// Shared best-move scores, accessed atomically.
__device__ __forceinline__ float score_ld(const float *p) {
  return __uint_as_float(__hip_atomic_load(reinterpret_cast<const unsigned *>(p), __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT));
}
__device__ __forceinline__ double score_ld(const double *p) {
  return __longlong_as_double((long long)ld_shared_u64(reinterpret_cast<const unsigned long long *>(p)));
}
__device__ __forceinline__ void score_st(float *p, float v) {
  __hip_atomic_store(reinterpret_cast<unsigned *>(p), __float_as_uint(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void score_st(double *p, double v) {
  st_shared_u64(reinterpret_cast<unsigned long long *>(p), (unsigned long long)__double_as_longlong(v));
}
__device__ __forceinline__ uint32_t meta_pack(int nzc) { return (uint32_t)nzc << 16; }
__device__ __forceinline__ int meta_nzc(uint32_t m) { return (int)(m >> 16); }

// A candidate is a tag word (word 0) holding the round (22 bits), the atom (10
// bits) and the position (32 bits; all ones for "no accepted candidate"), and
// the bits of its delta, 32 per word (word 1, in FP64 also word 2) beside the
// round in the high half.  A reader polls the words together until each
// carries its round, so no store waits for another.
constexpr int kCandWords = 4;  // words per worker (the last one is padding)
constexpr unsigned kNoPos = 0xffffffffu;
constexpr int kRoundBits = 22;
__device__ __forceinline__ unsigned long long cand_tag(int r, int k0, unsigned pos) {
  return ((unsigned long long)(r & ((1 << kRoundBits) - 1)) << 42) | ((unsigned long long)(k0 & 0x3ff) << 32) |
         (unsigned long long)pos;
}
__device__ __forceinline__ int tag_round(unsigned long long t) { return (int)(t >> 42); }
__device__ __forceinline__ int tag_k0(unsigned long long t) { return (int)((t >> 32) & 0x3ff); }
__device__ __forceinline__ unsigned tag_pos(unsigned long long t) { return (unsigned)(t & 0xffffffffull); }

template <class R> __device__ __forceinline__ unsigned long long delta_bits(R d);
template <> __device__ __forceinline__ unsigned long long delta_bits<float>(float d) { return __float_as_uint(d); }
template <> __device__ __forceinline__ unsigned long long delta_bits<double>(double d) {
  return (unsigned long long)__double_as_longlong(d);
}
template <class R> __device__ __forceinline__ R bits_delta(unsigned long long v);
template <> __device__ __forceinline__ float bits_delta<float>(unsigned long long v) { return __uint_as_float((unsigned)v); }
template <> __device__ __forceinline__ double bits_delta<double>(unsigned long long v) {
  return __longlong_as_double((long long)v);
}

// ------------------------------------------------------------- the round kernel

// Words of the LDS bitmask that marks the positions of a team's region holding
// a non-zero coordinate (regions of up to 32 * kNzWords positions keep one).
constexpr int kNzWords = 2048;

// Workers one team runs at most, and updates that can touch its region (its
// own workers' and those of the ring of workers around them).
constexpr int kTeamMax = 16, kUpdMax = 32;

// Rows and columns of one patch block whose cover masks (the updates whose
// patch covers that row or column) are tabulated in LDS.
constexpr int kMaskRows = 128, kMaskCols = 512;

// How the lanes of a wave share a position's atoms: 2^sh neighbouring lanes
// per position, each with up to ng of its 16-byte atom groups (group
// lane + i 2^sh), so that the lanes of a position read 16 2^sh contiguous
// bytes per load.  ng = 0: more groups than 3 per lane of a whole wave.
struct LaneMap {
  int sh, ng;
};
__host__ __device__ inline LaneMap lane_map(int G) {
  LaneMap best{6, 0};
  int slots = 1 << 30;
  for (int ng = 1; ng <= 3; ++ng) {
    int sh = 0;
    while ((ng << sh) < G) ++sh;
    if (sh <= 6 && (ng << sh) <= slots) {  // fewest idle slots; on a tie the more groups per lane
      slots = ng << sh;
      best = LaneMap{sh, ng};
    }
  }
  return best;
}

// 16-byte vectors and pointers known to be global (pointers read from a
// struct are generic to the compiler, whose flat accesses wait on LDS too).
template <class R> struct NVec;
template <> struct NVec<float> {
  typedef float T __attribute__((ext_vector_type(4)));
};
template <> struct NVec<double> {
  typedef double T __attribute__((ext_vector_type(2)));
};
template <class T> using GPtr = __attribute__((address_space(1))) T *;
template <class T> __device__ __forceinline__ GPtr<T> as_global(T *p) { return (GPtr<T>)p; }

template <class R> struct PatchCtx {
  GPtr<R> beta;
  GPtr<const R> z, A;
  GPtr<R> score;
  R *ls;                  // LDS copy of the region's scores, or null
  uint32_t *rowm, *colm;  // cover masks of a block's rows and columns
  const R *inv_n;
  uint32_t *nzb;     // bit (h - a1) * ext2 + (w - a2) set when position (h, w) of the region has a
                     // non-zero; null for larger regions, whose patches read z everywhere
  R lam, nlam, tolc;  // lambda; -lambda (-infinity when positive); tol (0 without certify)
  int W, U2, KS, G;  // G: 16-byte atom groups per position
  int sh;            // lane_map(G).sh
  int a1, a2, ext2;  // origin and width of the region
};

// An accepted update as the apply phase uses it: atom k0 at (ch, cw0), change
// delta, and the rows [r1, r2) x columns [c1, c2) of this team's region it
// patches.
template <class R> struct UCand {
  int k0, ch, cw0, r1, r2, c1, c2;
  int aoff;  // element offset in A of (row 0, column 0) for this update: ((k0 U1 - ch + L1 - 1) U2 - cw0 + L2 - 1) KS
  R delta;
  unsigned ov;  // earlier updates of the list whose patches overlap this one's
};

// The lane's value moved by a DPP control within rows of 16 lanes.
template <int CTRL> __device__ __forceinline__ float dpp_mov(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), CTRL, 0xf, 0xf, false));
}
template <int CTRL> __device__ __forceinline__ double dpp_mov(double v) {
  const int lo = __double2loint(v), hi = __double2hiint(v);
  return __hiloint2double(__builtin_amdgcn_update_dpp(hi, hi, CTRL, 0xf, 0xf, false),
                          __builtin_amdgcn_update_dpp(lo, lo, CTRL, 0xf, 0xf, false));
}

// Maximum over the aligned groups of 2^sh lanes, in every lane of a group.
template <class R> __device__ __forceinline__ R lanes_max(R v, int sh) {
  if (sh > 0) v = fmax(v, dpp_mov<0xB1>(v));   // quad_perm 1 0 3 2
  if (sh > 1) v = fmax(v, dpp_mov<0x4E>(v));   // quad_perm 2 3 0 1
  if (sh > 2) v = fmax(v, dpp_mov<0x141>(v));  // row_half_mirror: the other quad of 8 lanes
  if (sh > 3) v = fmax(v, dpp_mov<0x140>(v));  // row_mirror: the other 8 of 16 lanes
  if (sh > 4) v = fmax(v, __shfl_xor(v, 16, 64));
  if (sh > 5) v = fmax(v, __shfl_xor(v, 32, 64));
  return v;
}

// b minus b clipped to [nlam, lam]: ST(b, lambda) for nlam = -lambda and its
// one-sided form for nlam = -infinity, with st_target's values (b - lam,
// b + lam or an exact 0).
__device__ __forceinline__ float shrink(float b, float nlam, float lam) {
  return b - __builtin_amdgcn_fmed3f(b, nlam, lam);
}
__device__ __forceinline__ double shrink(double b, double nlam, double lam) { return b - fmin(fmax(b, nlam), lam); }

__device__ __forceinline__ float fma_neg(float b, float a, float d) { return __builtin_fmaf(-a, d, b); }
__device__ __forceinline__ double fma_neg(double b, double a, double d) { return __builtin_fma(-a, d, b); }

// v, negated where s is negative.
__device__ __forceinline__ float with_sign(float v, float s) {
  return __uint_as_float(__float_as_uint(v) ^ (__float_as_uint(s) & 0x80000000u));
}
__device__ __forceinline__ double with_sign(double v, double s) {
  return __hiloint2double(__double2hiint(v) ^ (__double2hiint(s) & (int)0x80000000), __double2loint(v));
}

// Best move score over a lane's NG groups (the scores of st_target and
// move_score; a NaN beta scores nothing).  Where no position of the wave
// holds a non-zero, the short form |ST(b)| / n.
template <class R, int NG>
__device__ __forceinline__ R lane_best(const typename NVec<R>::T *b, const typename NVec<R>::T *z,
                                       const typename NVec<R>::T *inv, bool nz, R nlam, R lam, R tolc) {
#pragma clang fp contract(off)
  constexpr int VE = Vec<R>::N;
  R best = R(0);
  if (!__any(nz)) {
#pragma unroll
    for (int i = 0; i < NG; ++i)
#pragma unroll
      for (int e = 0; e < VE; ++e) best = fmax(best, fabs(shrink(b[i][e], nlam, lam) * inv[i][e]));
    return best;
  }
#pragma unroll
  for (int i = 0; i < NG; ++i)
#pragma unroll
    for (int e = 0; e < VE; ++e) {
      const R zv = z[i][e];
      const R zn = shrink(b[i][e], nlam, lam) * inv[i][e];
      const R dz = fabs(zn - zv);
      // a move that changes the support or the sign scores at least tolc
      const R floor = zv != R(0) ? tolc : R(0);
      best = fmax(best, with_sign(zn, zv) > R(0) ? dz : fmax(dz, floor));
    }
  return best;
}

template <class R>
__device__ __forceinline__ void put_score(const PatchCtx<R> &P, GPtr<R> at, int lt, R v) {
  if (P.ls) P.ls[lt] = v;
  score_st((R *)at, v);
}

// One lane's part of a position: up to NG groups of beta, of the first
// covering update's DtD row and, where the position holds non-zeros, of z.
template <class R, int NG> struct PStage {
  typename NVec<R>::T b[NG], a[NG], z[NG];
  unsigned m;  // updates covering the position
  bool nz;
};

// Applies updates to the rows [R1, R2) x columns [C1, C2) of this team's
// region: beta -= delta * DtD row (eq. beta_update; the updated coordinate of
// an update keeps its value), and the position's cached best score.  With
// MULTI false every position is covered by the one update uc[0].  With MULTI
// the updates covering a position are those of both its row's and its
// column's mask, summed in increasing worker order as applying them one after
// another would; positions none covers are left untouched.  Every thread of
// the workgroup takes part, as number vt.
//
// An item of eight atoms costs about as many issue cycles as its memory round
// trip, so the work per item is kept short: the lanes of a position are
// neighbours whose shares of a row are contiguous (coalesced reads), (row,
// column) and every byte offset step by constants (no division), the inverse
// norms stay in registers, only the best score is formed (the atom of a
// candidate is found when it is selected), and it is combined between the
// lanes of a position by DPP.  The next item's reads are issued before the
// current one is used.
template <class R, int NT, int NG, bool MULTI>
__device__ __forceinline__ void patch_lanes(const PatchCtx<R> &P, const UCand<R> *uc, int vt, int R1, int R2, int C1,
                                            int C2) {
  typedef typename NVec<R>::T V;
  constexpr int VE = Vec<R>::N;
  const int sh = P.sh, LP = 1 << sh, j = vt & (LP - 1), pstep = NT >> sh;
  const int ncol = C2 - C1, npos = (R2 - R1) * ncol;
  const unsigned KSB = (unsigned)P.KS * sizeof(R);
  int p = vt >> sh;
  if (p >= npos) return;
  int row = div_small(p, ncol), col = p - row * ncol;
  const int drow = div_small(pstep, ncol), dcol = pstep - drow * ncol;
  // offsets of the position from (R1, C1): in positions, in the bitmask, in bytes of beta and of A
  unsigned oe = (unsigned)row * P.W + col;
  int lt = (R1 - P.a1 + row) * P.ext2 + (C1 - P.a2) + col;
  unsigned ob = oe * KSB + 16u * j;
  unsigned oa = ((unsigned)row * P.U2 + col) * KSB + 16u * j;
  const unsigned doe = (unsigned)drow * P.W + dcol, woe = (unsigned)(P.W - ncol);
  const unsigned dob = doe * KSB, wob = woe * KSB;
  const unsigned doa = ((unsigned)drow * P.U2 + dcol) * KSB, woa = (unsigned)(P.U2 - ncol) * KSB;
  const int dlt = drow * P.ext2 + dcol, wlt = P.ext2 - ncol;
  const long long pos0 = (long long)R1 * P.W + C1;
  const GPtr<char> bb = (GPtr<char>)(P.beta + pos0 * P.KS);
  const GPtr<const char> zb = (GPtr<const char>)(P.z + pos0 * P.KS);
  const int ar0 = (R1 * P.U2 + C1) * P.KS;  // element of A at (R1, C1) relative to an update's aoff
  const GPtr<const char> ab = (GPtr<const char>)(P.A + (MULTI ? 0 : uc[0].aoff + ar0));
  const bool vl = j + (NG - 1) * LP < P.G;  // the lane's last group exists
  const R d0 = uc[0].delta;
  // FP64 items and those of three groups hold too many registers to have two
  // in flight: there an item is loaded when it is used.  So it is for the
  // large patches of a single update, which are bound by the traffic past the
  // L2 (4096^2 RGB image: 69.5 ms of rounds, 72.8 ms with the next item ahead).
  constexpr bool kAhead = sizeof(R) == 4 && NG <= 2 && MULTI;
  V inv[NG];
  auto norms = [&]() {
#pragma unroll
    for (int i = 0; i < NG; ++i)
      inv[i] = i < NG - 1 || vl ? *reinterpret_cast<const V *>(P.inv_n + (j + i * LP) * VE) : V(R(0));
  };
  if (kAhead) norms();
  // single update: its own position in the patch
  const int ps = MULTI ? -1
                       : (uc[0].ch >= R1 && uc[0].ch < R2 && uc[0].cw0 >= C1 && uc[0].cw0 < C2
                              ? (uc[0].ch - R1) * ncol + uc[0].cw0 - C1
                              : -1);
  auto load = [&](PStage<R, NG> &x, int rw, int cl, unsigned xb, unsigned xa, int xl) {
    unsigned ua = xa;
    x.m = 1u;
    if (MULTI) {
      x.m = P.rowm[rw] & P.colm[cl];
      if (!x.m) return;
      ua += (unsigned)(uc[__ffs(x.m) - 1].aoff + ar0) * (unsigned)sizeof(R);
    }
#pragma unroll
    for (int i = 0; i < NG; ++i) {
      const bool on = i < NG - 1 || vl;
      x.b[i] = on ? *(GPtr<const V>)(bb + xb + 16u * (i * LP)) : V(R(0));
      x.a[i] = on ? *(GPtr<const V>)(ab + ua + 16u * (i * LP)) : V(R(0));
    }
    x.nz = P.nzb ? (P.nzb[xl >> 5] >> (xl & 31)) & 1u : true;
    if (__any(x.nz)) {  // z is used only where a lane of the wave has non-zeros
#pragma unroll
      for (int i = 0; i < NG; ++i)
        x.z[i] = x.nz && (i < NG - 1 || vl) ? *(GPtr<const V>)(zb + xb + 16u * (i * LP)) : V(R(0));
    }
  };
  auto hold = [&](V *a, int k0) {  // the updated coordinate keeps its beta: no contribution there
    const int kq = k0 / VE, ke = k0 - kq * VE;
#pragma unroll
    for (int i = 0; i < NG; ++i)
#pragma unroll
      for (int e = 0; e < VE; ++e) a[i][e] = kq == j + i * LP && e == ke ? R(0) : a[i][e];
  };
  const GPtr<R> sb = P.score + pos0;
  // One item, loaded in x (or loaded here); the next one's loads go to y.
  auto step = [&](PStage<R, NG> &x, PStage<R, NG> &y) {
    if (!kAhead) load(x, row, col, ob, oa, lt);
    const int pn = p + pstep;
    int coln = col + dcol, rown = row + drow, ltn = lt + dlt;
    unsigned oen = oe + doe, oan = oa + doa, obn = ob + dob;
    if (coln >= ncol) {
      coln -= ncol;
      ++rown;
      oen += woe;
      obn += wob;
      oan += woa;
      ltn += wlt;
    }
    y.m = 0u;
    if (kAhead && pn < npos) load(y, rown, coln, obn, oan, ltn);
    if (x.m) {
      V *const b = x.b;
      if (!MULTI) {
        if (p == ps) hold(x.a, uc[0].k0);
#pragma unroll
        for (int i = 0; i < NG; ++i)
#pragma unroll
          for (int e = 0; e < VE; ++e) b[i][e] = fma_neg(b[i][e], x.a[i][e], d0);
      } else {
        unsigned m = x.m;
        for (;;) {
          const UCand<R> &u = uc[__ffs(m) - 1];
          m &= m - 1;
          if (R1 + row == u.ch && C1 + col == u.cw0) hold(x.a, u.k0);
          const R d = u.delta;
#pragma unroll
          for (int i = 0; i < NG; ++i)
#pragma unroll
            for (int e = 0; e < VE; ++e) b[i][e] = fma_neg(b[i][e], x.a[i][e], d);
          if (!m) break;
          const unsigned ua = oa + (unsigned)(uc[__ffs(m) - 1].aoff + ar0) * (unsigned)sizeof(R);
#pragma unroll
          for (int i = 0; i < NG; ++i)
            x.a[i] = i < NG - 1 || vl ? *(GPtr<const V>)(ab + ua + 16u * (i * LP)) : V(R(0));
        }
      }
#pragma unroll
      for (int i = 0; i < NG; ++i)
        if (i < NG - 1 || vl) *(GPtr<V>)(bb + ob + 16u * (i * LP)) = b[i];
      if (!kAhead) norms();
      const R best = lanes_max(lane_best<R, NG>(b, x.z, inv, x.nz, P.nlam, P.lam, P.tolc), sh);
      if (j == 0) put_score(P, sb + oe, lt, best);
    }
    p = pn;
    row = rown;
    col = coln;
    lt = ltn;
    oe = oen;
    ob = obn;
    oa = oan;
  };
  PStage<R, NG> x, y;
  if (kAhead) load(x, row, col, ob, oa, lt);
  for (;;) {
    step(x, y);
    if (p >= npos) break;
    if constexpr (kAhead) {
      step(y, x);
      if (p >= npos) break;
    }
  }
}

// patch_lanes for positions of more atom groups than a wave's lanes hold at
// three each: the lanes of a wave loop over a position's groups.
template <class R, int NT, bool MULTI>
__device__ __forceinline__ void patch_wide(const PatchCtx<R> &P, const UCand<R> *uc, int vt, int R1, int R2, int C1,
                                           int C2) {
  typedef typename NVec<R>::T V;
  constexpr int VE = Vec<R>::N;
  const int lane = threadIdx.x & 63, ncol = C2 - C1, npos = (R2 - R1) * ncol;
  for (int p = vt >> 6; p < npos; p += NT / 64) {
    const int row = p / ncol, h = R1 + row, w = C1 + p - row * ncol;
    const unsigned m0 = MULTI ? P.rowm[row] & P.colm[w - C1] : 1u;
    if (!m0) continue;
    const long long pos = (long long)h * P.W + w;
    R best = R(0);
    for (int q = lane; q < P.G; q += 64) {
      const long long e = pos * P.KS + q * VE;
      V b = *(GPtr<const V>)(P.beta + e);
      const V z = *(GPtr<const V>)(P.z + e), inv = *reinterpret_cast<const V *>(P.inv_n + q * VE);
      for (unsigned m = m0; m; m &= m - 1) {
        const UCand<R> &u = uc[__ffs(m) - 1];
        const V a = *(GPtr<const V>)(P.A + (u.aoff + (h * P.U2 + w) * P.KS + q * VE));
        const V old = b;
#pragma unroll
        for (int i = 0; i < VE; ++i) {
          b[i] = fma_neg(b[i], a[i], u.delta);
          if (h == u.ch && w == u.cw0 && u.k0 == q * VE + i) b[i] = old[i];
        }
      }
      *(GPtr<V>)(P.beta + e) = b;
      best = fmax(best, lane_best<R, 1>(&b, &z, &inv, true, P.nlam, P.lam, P.tolc));
    }
    best = lanes_max(best, 6);
    if (lane == 0) put_score(P, P.score + pos, (h - P.a1) * P.ext2 + w - P.a2, best);
  }
}

template <class R, int NT, int NG, bool MULTI>
__device__ __forceinline__ void patch_rect(const PatchCtx<R> &P, const UCand<R> *uc, int vt, int R1, int R2, int C1,
                                           int C2) {
  if constexpr (NG == 0) {
    patch_wide<R, NT, MULTI>(P, uc, vt, R1, R2, C1, C2);
  } else {
    // bands of rows whose byte offsets stay below 2^31 (one band unless rows are huge)
    const long long pitch = (long long)max(P.W, P.U2) * P.KS * (long long)sizeof(R);
    const int rows = (int)max(1ll, min(1ll << 20, ((1ll << 31) - 1) / pitch - 1));
    for (int r = R1; r < R2; r += rows) patch_lanes<R, NT, NG, MULTI>(P, uc, vt, r, min(r + rows, R2), C1, C2);
  }
}

// Every update of `uc` in one pass over the bounding box of their patches, in
// blocks whose row and column masks fit the LDS tables.
template <class R, int NT, int NG>
__device__ __forceinline__ void patch_union(const PatchCtx<R> &P, const UCand<R> *uc, int nc, int R1, int R2, int C1,
                                            int C2) {
  const int tid = threadIdx.x;
  const long long pitch = (long long)max(P.W, P.U2) * P.KS * (long long)sizeof(R);
  const int rc = (int)max(1ll, min((long long)kMaskRows, ((1ll << 31) - 1) / pitch - 1));
  for (int rr0 = R1; rr0 < R2; rr0 += rc) {
    const int rr1 = min(rr0 + rc, R2), nrow = rr1 - rr0;
    for (int cc0 = C1; cc0 < C2; cc0 += kMaskCols) {
      const int cc1 = min(cc0 + kMaskCols, C2);
      if (rr0 != R1 || cc0 != C1) __syncthreads();
      for (int j = tid; j < nrow + cc1 - cc0; j += NT) {
        unsigned mk = 0;
        if (j < nrow) {
          for (int c = 0; c < nc; ++c)
            if (rr0 + j >= uc[c].r1 && rr0 + j < uc[c].r2) mk |= 1u << c;
          P.rowm[j] = mk;
        } else {
          for (int c = 0; c < nc; ++c)
            if (cc0 + j - nrow >= uc[c].c1 && cc0 + j - nrow < uc[c].c2) mk |= 1u << c;
          P.colm[j - nrow] = mk;
        }
      }
      __syncthreads();
      patch_rect<R, NT, NG, true>(P, uc, tid, rr0, rr1, cc0, cc1);
    }
  }
}

// Sets or clears a position's bit (other workers of the team may change
// other bits of the word).
__device__ __forceinline__ void nzb_put(uint32_t *nzb, int t, bool on) {
  if (!nzb) return;
  if (on)
    atomicOr(&nzb[t >> 5], 1u << (t & 31));
  else
    atomicAnd(&nzb[t >> 5], ~(1u << (t & 31)));
}

// The instance read through the constant address space (scalar loads), from a
// pointer the compiler cannot see through: what a phase derives from it is
// loaded and derived again in each phase of each round.  Without this the
// compiler keeps every loop-invariant of every phase in registers and spills
// those the patch loop needs.
template <class R> using CInst = const __attribute__((address_space(4))) Inst<R>;
template <class R> __device__ __forceinline__ CInst<R> *fresh(CInst<R> *p) {
  asm volatile("" : "+s"(p));
  return p;
}
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }

// Largest value over a wave; smallest int over a wave: rows of 16 lanes by
// DPP, the four rows by lane reads.
template <class R> __device__ __forceinline__ R read_lane(R v, int l);
template <> __device__ __forceinline__ float read_lane<float>(float v, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}
template <> __device__ __forceinline__ double read_lane<double>(double v, int l) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l),
                          __builtin_amdgcn_readlane(__double2loint(v), l));
}
template <int CTRL> __device__ __forceinline__ int dpp_mov_i(int v) {
  return __builtin_amdgcn_update_dpp(v, v, CTRL, 0xf, 0xf, false);
}
// Largest score of a wave.  Scores are not negative but for the marker -1, so
// FP32 ones order like their bits.
__device__ __forceinline__ float wave_max(float f) {
  int v = __float_as_int(f);
  v = max(v, dpp_mov_i<0xB1>(v));
  v = max(v, dpp_mov_i<0x4E>(v));
  v = max(v, dpp_mov_i<0x141>(v));
  v = max(v, dpp_mov_i<0x140>(v));
  return __int_as_float(max(max(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)),
                            max(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48))));
}
__device__ __forceinline__ double wave_max(double v) {
  v = lanes_max(v, 4);
  return fmax(fmax(read_lane<double>(v, 0), read_lane<double>(v, 16)),
              fmax(read_lane<double>(v, 32), read_lane<double>(v, 48)));
}
__device__ __forceinline__ int wave_min(int v) {
  v = min(v, dpp_mov_i<0xB1>(v));
  v = min(v, dpp_mov_i<0x4E>(v));
  v = min(v, dpp_mov_i<0x141>(v));
  v = min(v, dpp_mov_i<0x140>(v));
  return min(min(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)),
             min(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
}
// Largest (score, lowest position) over a wave, in every lane.  Called by
// whole waves.
template <class R> __device__ __forceinline__ void wave_argmax(R &s, int &pos) {
  const R m = wave_max(s);
  pos = wave_min(s == m ? pos : 0x7fffffff);
  s = m;
}

// The best move at position `pos` (the lowest atom among equal scores, as the
// caches have it), found by one whole wave from beta and z: its atom, the
// coordinate's value and its target.
template <class R>
__device__ __forceinline__ void best_move(CInst<R> *I, const R *inv_n, long long pos, int *k0, R *zc, R *zn) {
  const int lane = threadIdx.x & 63, K = I->K;
  const GPtr<const R> zp = as_global((const R *)I->z) + pos * I->KS, bp = as_global((const R *)I->beta) + pos * I->KS;
  R bs = R(-1), bz = R(0), bt = R(0);
  int bk = 0x7fffffff;
  for (int k = lane; k < K; k += 64) {
    const R zv = zp[k];
    const R t = st_target((R)bp[k], (R)I->lambda, inv_n[k], I->positive);
    const R sc = move_score(zv, t, (R)I->tol, I->certify);
    if (sc > bs) {
      bs = sc;
      bk = k;
      bz = zv;
      bt = t;
    }
  }
  R ms = bs;
  int mk = bk;
  wave_argmax(ms, mk);
  *k0 = mk;
  *zc = read_lane<R>(bz, mk & 63);
  *zn = read_lane<R>(bt, mk & 63);
}

// One workgroup is a team: it runs a block of G1 x G2 neighbouring workers of
// Alg. 3 (DiCoDiLe-Z).  Worker w of an instance owns S_w, a block of a W1 x W2
// balanced split of the valid domain, cut into Mw balanced sub-domains of
// about tile1 x tile2 positions that it visits cyclically.  The team owns the
// region of its workers' blocks.
//
// A round runs:
//   A  every worker visits `inner` sub-domains (Alg. 1's local greedy choice),
//      a group of waves per worker.  With several visits, candidates whose
//      patch stays clear of the border band (which other workers read) are
//      applied at once and the first band-reaching one is held.  The held
//      candidate is tested against the other workers' scores in V(w0) when
//      V(w0) leaves S_w (eq. soft_lock, lower worker index wins a tie) and
//      published, tagged with the round;
//   B  the team applies, to the part of beta, z and the cache it owns, the
//      accepted candidates of its workers and of the ring of workers around
//      them whose neighbourhood meets its region (eq. beta_update), in
//      increasing worker order, all its waves on each patch, then publishes
//      progress r + 1.
// Phase A of round r reads scores of the neighbouring teams' border bands,
// which only they write, in their phase B: it does so once each neighbour's
// progress is >= r.  A neighbour starts its phase B of round r only after
// reading this team's round-r candidates, published after this team's phase A
// reads.  Worker sizes of at least L_i keep every interaction between grid
// neighbours.
//
// Why teams: the patches of a round fall unevenly on the workers, and a round
// lasts as long as the slowest worker of a neighbourhood.  A worker per
// workgroup left a quarter of a CU's waves on each patch while the CU's other
// workers waited; a team of the CU's workers puts all of them on every patch,
// and its workers read each other's scores and candidates without a wait
// between workgroups.  The order of the updates at every position, and so
// every result, is that of one worker per workgroup.
//
// Stopping: a worker is quiet once its last Mw visits found no move scoring
// >= tol and no patch touched S_w since (random rule: once the scan at the
// end of its last epoch found none and no patch touched S_w since).  When
// every worker reports quiet at the end of the same round, every
// coordinate's move is below tol and no further update can happen: all
// teams exit.
//
// Under the random rule a candidate's score is that of its drawn coordinate,
// at most the cached best of its position, so of two interacting candidates
// the soft-lock test still rejects at least one: each sees the other's
// position holding a score >= its own (ties go to the lower worker index).
// What a team keeps of one of its workers between phases.
struct TeamWorker {
  int w, a1, b1, a2, b2;  // worker index and block
  int nb1, nb2;           // sub-domains per axis: about extent / tile, balanced (sizes differ by <= 1)
  int mcur, quiet;        // the next sub-domain; consecutive visits with no move >= tol and no patch of S_w
  int s1, e1, s2, e2;     // rows [s1, e1) x columns [s2, e2) of the next sub-domain
  long long cursor;       // visits so far
  unsigned upd, cand, lock, visit;
  unsigned long long chk, patch;
};

template <class R, int NT> struct TeamSmem {
  // positions of a region whose scores are also kept in LDS
  static constexpr int kScores = (NT == 1024 ? 65536 : 16384) / (int)sizeof(R);
  R score[kScores];
  R inv_n[1024];
  uint32_t nzb[kNzWords];
  uint32_t rowm[kMaskRows], colm[kMaskCols];
  UCand<R> uc[kUpdMax];
  UCand<R> ui[kTeamMax];  // interior candidates applied within phase A
  TeamWorker wk[kTeamMax];
  R ps[NT / 64];          // per-wave partial selections
  int pp[NT / 64];
  R cs[kTeamMax];         // candidates under test: score, position, soft-lock outcome
  int cp[kTeamMax], clk[kTeamMax];
  int done[kTeamMax];     // 1: the worker is quiet
  int ion[kTeamMax];      // interior candidate of the current visit
  int A1, B1, A2, B2;     // the region
  int nbt[9];             // the neighbouring teams (-1: none, or this one)
  int ncn, cnw[kUpdMax], cnt[kUpdMax];  // the workers whose updates can touch the region, in order; their teams
  int nuc, ub[4], ub_union;
  unsigned long long patched;  // positions of beta patched in phase B
  int bad, exit_f;
  unsigned long long tk[4], mark;  // phase times: wait, select, collect, apply
};

// Bounds of a worker's next sub-domain (its divisions are kept off the path
// between a round's end and the next selection).
__device__ __forceinline__ void next_visit(TeamWorker &k) {
  const int bi = k.mcur / k.nb2, bj = k.mcur - bi * k.nb2, e1w = k.b1 - k.a1, e2w = k.b2 - k.a2;
  k.s1 = k.a1 + part_start_fast(bi, e1w, k.nb1);
  k.e1 = k.a1 + part_start_fast(bi + 1, e1w, k.nb1);
  k.s2 = k.a2 + part_start_fast(bj, e2w, k.nb2);
  k.e2 = k.a2 + part_start_fast(bj + 1, e2w, k.nb2);
}

// Adds the time since the last mark to one phase's, by one thread: one round
// in kTimed is timed (reading the clock takes a good part of a short phase).
constexpr int kTimed = 16;
template <class R, int NT> __device__ __forceinline__ void team_mark(TeamSmem<R, NT> &sm, int r, int phase) {
  if (r & (kTimed - 1)) return;
  const unsigned long long t = __builtin_amdgcn_s_memrealtime();
  if (phase >= 0) sm.tk[phase] += t - sm.mark;
  sm.mark = t;
}

// The soft-lock test of a candidate of score `bs` at (ch, cw) of the worker
// [a1, b1) x [a2, b2): whether a position of V(w0) outside its block holds a
// larger score, or an equal one owned by a lower worker (eq. soft_lock), over
// the positions of the waves gw, gw + nw, ... of V(w0).  Scores of the team's
// own region come from LDS where it keeps them.  Whole waves call it.
template <class R, int NT>
__device__ __forceinline__ bool soft_test(CInst<R> *I, const TeamSmem<R, NT> &sm, bool ls, int w, int a1, int b1,
                                          int a2, int b2, R bs, int ch, int cw, int gw, int nw) {
  const int H = I->H, W = I->W, lane = threadIdx.x & 63;
  const int A1 = uni(sm.A1), B1 = uni(sm.B1), A2 = uni(sm.A2), B2 = uni(sm.B2);
  const int v1 = max(ch - I->L1 + 1, 0), u1 = min(ch + I->L1, H);
  const int v2 = max(cw - I->L2 + 1, 0), u2 = min(cw + I->L2, W);
  const int vw = u2 - v2, nv = (u1 - v1) * vw, gs = 64 * nw;
  R *const sg = I->score;
  constexpr int U = 8;  // positions per pass, their loads in flight together
  const int dh = div_small(gs, vw), dw = gs - dh * vw;
  int th = v1 + div_small(gw * 64 + lane, vw), tw = v2 + gw * 64 + lane - (th - v1) * vw;
  for (int t = gw * 64; t < nv; t += U * gs) {
    R sc[U];
    const int th0 = th, tw0 = tw;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      sc[u] = R(-1);
      if (t + u * gs < nv) {  // the same for the whole wave
        const bool mine = th >= a1 && th < b1 && tw >= a2 && tw < b2;
        if (t + u * gs + lane < nv && !mine) {
          if (ls && th >= A1 && th < B1 && tw >= A2 && tw < B2)
            sc[u] = sm.score[(th - A1) * (B2 - A2) + tw - A2];
          else
            sc[u] = score_ld(sg + (long long)th * W + tw);
        }
        tw += dw;
        th += dh;
        if (tw >= u2) {
          tw -= vw;
          ++th;
        }
      }
    }
    R mx = sc[0];
#pragma unroll
    for (int u = 1; u < U; ++u) mx = sc[u] > mx ? sc[u] : mx;
    if (__any(mx > bs)) return true;
    if (__any(mx == bs)) {  // ties: the owners decide
      th = th0;
      tw = tw0;
      bool lk = false;
#pragma unroll 1
      for (int u = 0; u < U; ++u) {
        R sv = sc[0];
#pragma unroll
        for (int v = 1; v < U; ++v) sv = u == v ? sc[v] : sv;
        if (sv == bs && part_owner(th, H, I->W1) * I->W2 + part_owner(tw, W, I->W2) < w) lk = true;
        tw += dw;
        th += dh;
        if (tw >= u2) {
          tw -= vw;
          ++th;
        }
      }
      if (__any(lk)) return true;
    }
  }
  return false;
}

// The candidate a worker's lead wave holds.
template <class R> struct Held {
  bool has = false;
  R bs = R(-1), zc = R(0), zn = R(0);
  int bp = 0, k0 = 0;
};

// One visit's selection: the best score of worker q's next sub-domain, over the
// positions of the group's wave `gw` of `wpl` (Alg. 1's local greedy choice).
template <class R, int NT>
__device__ __forceinline__ void scan_visit(CInst<R> *I, const TeamSmem<R, NT> &sm, bool ls, int q, int gw, int wpl,
                                           R &vs, int &vp) {
  const TeamWorker &k = sm.wk[q];
  const int W = I->W, A1 = uni(sm.A1), A2 = uni(sm.A2), ext2 = uni(sm.B2) - A2;
  const int s1 = uni(k.s1), e1 = uni(k.e1), s2 = uni(k.s2), e2 = uni(k.e2);
  const int bw = e2 - s2, np = (e1 - s1) * bw, gs = 64 * wpl;
  const GPtr<const R> sg = as_global((const R *)I->score);
  // eight positions per pass with their loads in flight together; the (row,
  // column) of position t steps by the group's lanes each time
  constexpr int U = 8;
  const int lane = threadIdx.x & 63;
  const int dh = div_small(gs, bw), dw = gs - dh * bw;
  int th = div_small(gw * 64 + lane, bw), tw = gw * 64 + lane - th * bw;
  for (int t = gw * 64; t < np; t += U * gs) {
    R sc[U];
    int ps[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      sc[u] = R(-1);
      if (t + u * gs < np) {  // the same for the whole wave
        ps[u] = (s1 + th) * W + s2 + tw;
        if (t + u * gs + lane < np) sc[u] = ls ? sm.score[(s1 - A1 + th) * ext2 + s2 - A2 + tw] : sg[ps[u]];
        tw += dw;
        th += dh;
        if (tw >= bw) {
          tw -= bw;
          ++th;
        }
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (t + u * gs < np && sc[u] > vs) {  // a lane's positions ascend: the first of equal scores stays
        vs = sc[u];
        vp = ps[u];
      }
  }
  wave_argmax(vs, vp);
}

// z and the non-zero count of a coordinate that moves, and the divergence guard.
template <class R, int NT>
__device__ __forceinline__ void move_z(CInst<R> *I, TeamSmem<R, NT> &sm, bool nzb, int pos, int h, int w, int k0,
                                       R zc, R zn) {
  as_global(I->z)[(long long)pos * I->KS + k0] = zn;
  const GPtr<uint32_t> mg = as_global(I->meta) + pos;
  const int nzc = meta_nzc(*mg) + (zn != R(0)) - (zc != R(0));
  *mg = meta_pack(nzc);
  if (nzb) nzb_put(sm.nzb, (h - sm.A1) * (sm.B2 - sm.A2) + (w - sm.A2), nzc != 0);
  const R guard = I->div_guard;
  if (guard > R(0) && (zn > guard || -zn > guard)) {
    st_shared_i32(&I->ctl->stop, 1);
    atomicCAS(&I->ctl->status, 0, 2);
  }
}

// A further visit of a round with several (`inner` > 1): interior candidates are
// handed to the whole team, the first band-reaching one is held.
template <class R, int NT>
__device__ __forceinline__ void visit_multi(CInst<R> *I, TeamSmem<R, NT> &sm, bool nzb, int q, R vs, int vp,
                                            Held<R> &c, long long visit, long long &restart) {
  TeamWorker &k = sm.wk[q];
  const int L1 = I->L1, L2 = I->L2, W = I->W;
  const int a1 = uni(k.a1), b1 = uni(k.b1), a2 = uni(k.a2), b2 = uni(k.b2);
  const int wi = uni(k.w) / I->W2, wj = uni(k.w) - wi * I->W2;
  const int h0 = vp / W, w0 = vp - h0 * W;
  // candidates in [in_lo, in_hi[ patch nothing of the band neighbours read
  const int in_lo1 = wi > 0 ? a1 + 2 * (L1 - 1) : a1, in_hi1 = wi < I->W1 - 1 ? b1 - 2 * (L1 - 1) : b1;
  const int in_lo2 = wj > 0 ? a2 + 2 * (L2 - 1) : a2, in_hi2 = wj < I->W2 - 1 ? b2 - 2 * (L2 - 1) : b2;
  if (!(h0 >= in_lo1 && h0 < in_hi1 && w0 >= in_lo2 && w0 < in_hi2)) {
    if (!c.has) {
      c.has = true;
      c.bs = vs;
      c.bp = vp;
    } else if (restart < 0) {
      restart = visit;  // a second band-reaching candidate waits for the next round
    }
    return;
  }
  if (c.has && abs(h0 - c.bp / W) < L1 && abs(w0 - c.bp % W) < L2) {  // would interact with the held one
    if (restart < 0) restart = visit;
    return;
  }
  int k0 = 0;
  R zc = R(0), zn = R(0);
  best_move<R>(I, sm.inv_n, vp, &k0, &zc, &zn);
  if ((threadIdx.x & 63) == 0) {
    move_z<R, NT>(I, sm, nzb, vp, h0, w0, k0, zc, zn);
    UCand<R> &u = sm.ui[q];
    u.k0 = k0;
    u.ch = h0;
    u.cw0 = w0;
    u.r1 = max(h0 - L1 + 1, a1);
    u.r2 = min(h0 + L1, b1);
    u.c1 = max(w0 - L2 + 1, a2);
    u.c2 = min(w0 + L2, b2);
    u.aoff = ((k0 * I->U1 - h0 + L1 - 1) * I->U2 - w0 + L2 - 1) * I->KS;
    u.delta = zn - zc;
    k.patch += (unsigned long long)(u.r2 - u.r1) * (u.c2 - u.c1);
    k.upd += 1;
    sm.ion[q] = 1;
  }
}

// Collects this round's candidates of the workers whose updates can touch the
// region (the team's own and the ring around it), clipped to the region, in
// increasing worker order: the work list of phase B.  Run by one wave.
template <class R, int NT>
__device__ __forceinline__ void collect(CInst<R> *I, TeamSmem<R, NT> &sm, int r, long long timeout_ticks) {
  const int lane = threadIdx.x & 63;
  const int W = I->W, L1 = I->L1, L2 = I->L2;
  const int A1 = uni(sm.A1), B1 = uni(sm.B1), A2 = uni(sm.A2), B2 = uni(sm.B2);
  bool uval = false;
  int uk0 = 0, uch = 0, ucw = 0, ur1 = 0, ur2 = 0, uc1 = 0, uc2 = 0;
  R udl = R(0);
  if (lane < sm.ncn) {
    const unsigned long long *const c = I->cand + (long long)kCandWords * sm.cnw[lane];
    const int *const pr = I->prog + sm.cnt[lane];
    unsigned long long t = 0, d1 = 0, d2 = 0;
    const unsigned long long t0 = __builtin_amdgcn_s_memrealtime();
    const int rtag = r & ((1 << kRoundBits) - 1);
    for (;;) {
      // all words and the team's progress are read together, one round trip per poll
      t = ld_shared_u64(c);
      d1 = ld_shared_u64(c + 1);
      d2 = sizeof(R) == 8 ? ld_shared_u64(c + 2) : d1;
      const int pg = ld_shared_i32(pr);
      if (tag_round(t) == rtag && (int)(d1 >> 32) == r && (int)(d2 >> 32) == r) break;
      if (pg == 0x7fffffff) {
        // the worker's team has left; it stored its last words before its
        // progress word, so words of this round are seen by a reread
        t = ld_shared_u64(c);
        d1 = ld_shared_u64(c + 1);
        d2 = sizeof(R) == 8 ? ld_shared_u64(c + 2) : d1;
        if (tag_round(t) != rtag || (int)(d1 >> 32) != r || (int)(d2 >> 32) != r) t = cand_tag(r, 0, kNoPos);
        break;
      }
      __builtin_amdgcn_s_sleep(1);
      if ((long long)(__builtin_amdgcn_s_memrealtime() - t0) > timeout_ticks) {
        sm.bad = 1;
        t = cand_tag(r, 0, kNoPos);
        break;
      }
    }
    const unsigned cpos = tag_pos(t);
    if (cpos != kNoPos) {
      udl = bits_delta<R>(sizeof(R) == 8 ? (d1 & 0xffffffffull) | (d2 << 32) : d1);
      uk0 = tag_k0(t);
      uch = (int)(cpos / (unsigned)W);
      ucw = (int)(cpos - (unsigned)uch * (unsigned)W);
      ur1 = max(uch - L1 + 1, A1);
      ur2 = min(uch + L1, B1);
      uc1 = max(ucw - L2 + 1, A2);
      uc2 = min(ucw + L2, B2);
      uval = ur1 < ur2 && uc1 < uc2;
    }
  }
  const unsigned long long bal = __ballot(uval);
  const int nu = __popcll(bal);
  if (uval) {
    UCand<R> &u = sm.uc[__popcll(bal & ((1ull << lane) - 1ull))];
    u.k0 = uk0;
    u.ch = uch;
    u.cw0 = ucw;
    u.r1 = ur1;
    u.r2 = ur2;
    u.c1 = uc1;
    u.c2 = uc2;
    u.aoff = ((uk0 * I->U1 - uch + L1 - 1) * I->U2 - ucw + L2 - 1) * I->KS;
    u.delta = udl;
  }
  __builtin_amdgcn_wave_barrier();
  // bounding box and area of the patches
  if (uval) atomicAdd(&sm.patched, (unsigned long long)((ur2 - ur1) * (uc2 - uc1)));
  const int x1 = wave_min(uval ? ur1 : B1), x2 = -wave_min(uval ? -ur2 : -A1);
  const int y1 = wave_min(uval ? uc1 : B2), y2 = -wave_min(uval ? -uc2 : -A2);
  // One pass over the bounding box pays for small patches, whose cost is
  // mostly per-update latency (positions no update covers cost no loads), as
  // long as it is little larger than the patches: at up to twice their area.
  // Workers of large sub-domains have updates far apart, whose box is mostly
  // empty (signal of 60,000 samples, 32 atoms of 64 taps, sub-domains of 4000:
  // 9.2 us per round in one pass over any box, 7.9 so; 800^2 image, 16 atoms of
  // 10x10, sub-domains of 100^2: 15.3 and 12.2; at four times the area 13.3).
  // Large patches (over 1024 positions) are bandwidth-bound and go one by one.
  const bool un = nu > 1 && (float)(x2 - x1) * (float)(y2 - y1) <= (float)(nu * I->box_share);
  if (lane < nu && !un) {
    unsigned ov = 0;
    const UCand<R> &u = sm.uc[lane];
    for (int c = 0; c < lane; ++c) {
      const UCand<R> &o = sm.uc[c];
      if (o.r1 < u.r2 && u.r1 < o.r2 && o.c1 < u.c2 && u.c1 < o.c2) ov |= 1u << c;
    }
    sm.uc[lane].ov = ov;
  }
  if (lane == 0) {
    sm.nuc = nu;
    sm.ub[0] = x1;
    sm.ub[1] = x2;
    sm.ub[2] = y1;
    sm.ub[3] = y2;
    sm.ub_union = un;
  }
}

// What the patch loops need, derived where they run.
template <class R, int NT>
__device__ __forceinline__ PatchCtx<R> patch_ctx(CInst<R> *I, TeamSmem<R, NT> &sm, bool ls, bool nzb) {
  PatchCtx<R> P;
  P.beta = as_global(I->beta);
  P.z = as_global((const R *)I->z);
  P.A = as_global(I->A);
  P.score = as_global(I->score);
  P.ls = ls ? sm.score : nullptr;
  P.rowm = sm.rowm;
  P.colm = sm.colm;
  P.inv_n = sm.inv_n;
  P.nzb = nzb ? sm.nzb : nullptr;
  P.lam = I->lambda;
  P.nlam = I->positive ? -R(__builtin_inf()) : -I->lambda;
  P.tolc = I->certify ? I->tol : R(0);
  P.W = I->W;
  P.U2 = I->U2;
  P.KS = I->KS;
  P.G = I->KS / Vec<R>::N;
  P.sh = I->lane_sh;
  P.a1 = uni(sm.A1);
  P.a2 = uni(sm.A2);
  P.ext2 = uni(sm.B2) - P.a2;
  return P;
}

// EXT: the random rule and several visits per round (kept out of the usual
// kernel, whose rounds are paced by the instructions of one wave).
template <class R, int NT, int NG, bool EXT>
__device__ __forceinline__ void run_team(CInst<R> *const I0, const int team, const long long timeout_ticks,
                                         TeamSmem<R, NT> &sm) {
  constexpr int NW = NT / 64;
  // the last wave collects the candidates and the one before keeps the
  // stopping consensus: with few workers per team neither leads one, so both
  // wait on memory beside the leads
  constexpr int kCollect = NW - 1, kConsensus = NT - 128;
  const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
  int gn, wpl = 1;
  bool ls, nzb;
  {
    CInst<R> *const I = fresh<R>(I0);
    const int H = I->H, W = I->W;
    const int ti = team / I->TW2, tj = team - ti * I->TW2;
    const int w1a = ti * I->G1, g1 = min(I->G1, I->W1 - w1a), w2a = tj * I->G2, g2 = min(I->G2, I->W2 - w2a);
    const int A1 = part_start(w1a, H, I->W1), B1 = part_start(w1a + g1, H, I->W1);
    const int A2 = part_start(w2a, W, I->W2), B2 = part_start(w2a + g2, W, I->W2), ext2 = B2 - A2;
    const long long nreg = (long long)(B1 - A1) * ext2;
    gn = g1 * g2;
    ls = nreg <= TeamSmem<R, NT>::kScores;
    nzb = nreg <= 32 * kNzWords;
    // Each worker has a group of wpl waves, the first of which leads (selects,
    // tests, publishes).  One wave reads up to 512 positions of a sub-domain or
    // of a V(w0); larger ones share half of the workgroup's waves, or all of
    // them where a wave would still read over 1024 (the others collect and keep
    // the consensus meanwhile: 1024^2 image, 1024 positions, 195 ms of rounds
    // with all of them and 191 with half; 4096^2 RGB image, 4096 positions,
    // 11.4 us per selection and 16.1).
    const long long tp = max((long long)min(I->tile1, H) * min(I->tile2, W), (long long)I->U1 * I->U2);
    int gp = 1;
    while (gp < gn) gp <<= 1;
    if (tp > 512)
      while (wpl * 4 * gp <= NW || (wpl * 2 * gp <= NW && (long long)wpl * 1024 < tp)) wpl <<= 1;
    if (tid < gn) {
      TeamWorker &k = sm.wk[tid];
      const int wi = w1a + tid / g2, wj = w2a + tid % g2;
      k.w = wi * I->W2 + wj;
      k.a1 = part_start(wi, H, I->W1);
      k.b1 = part_start(wi + 1, H, I->W1);
      k.a2 = part_start(wj, W, I->W2);
      k.b2 = part_start(wj + 1, W, I->W2);
      k.nb1 = max(1, (k.b1 - k.a1 + I->tile1 / 2) / I->tile1);
      k.nb2 = max(1, (k.b2 - k.a2 + I->tile2 / 2) / I->tile2);
      k.cursor = I->wstate ? I->wstate[2 * k.w] : 0;
      k.quiet = I->wstate ? (int)I->wstate[2 * k.w + 1] : 0;
      k.mcur = (int)(k.cursor % (k.nb1 * k.nb2));
      k.upd = k.cand = k.lock = k.visit = 0;
      k.chk = k.patch = 0;
      next_visit(k);
    }
    const GPtr<uint32_t> mg = as_global(I->meta);
    const GPtr<const R> sg = as_global((const R *)I->score);
    if (nzb)
      for (int wd = tid; wd < (int)(nreg + 31) / 32; wd += NT) {
        uint32_t m = 0;
        for (int b = 0; b < 32; ++b) {
          const int t = wd * 32 + b;
          if (t < nreg && meta_nzc(mg[(A1 + t / ext2) * W + A2 + t % ext2])) m |= 1u << b;
        }
        sm.nzb[wd] = m;
      }
    if (ls)
      for (int t = tid; t < (int)nreg; t += NT) sm.score[t] = sg[(A1 + t / ext2) * W + A2 + t % ext2];
    for (int k = tid; k < I->KS; k += NT) sm.inv_n[k] = k < I->K ? I->inv_n[k] : R(0);
    if (tid == 0) {
      sm.A1 = A1;
      sm.B1 = B1;
      sm.A2 = A2;
      sm.B2 = B2;
      sm.bad = 0;
      sm.patched = 0;
      sm.exit_f = ld_shared_i32(&I->ctl->converged) | ld_shared_i32(&I->ctl->stop);
      for (int i = 0; i < 4; ++i) sm.tk[i] = 0;
    }
    if (tid < 9) {
      const int ni = ti + tid / 3 - 1, nj = tj + tid % 3 - 1;
      sm.nbt[tid] =
          tid != 4 && ni >= 0 && ni < I->TW1 && nj >= 0 && nj < I->TW2 ? ni * I->TW2 + nj : -1;
    }
    const int c1a = max(w1a - 1, 0), c1b = min(w1a + I->G1 + 1, I->W1);
    const int c2a = max(w2a - 1, 0), c2b = min(w2a + I->G2 + 1, I->W2), cn2 = c2b - c2a;
    if (tid == 0) sm.ncn = (c1b - c1a) * cn2;
    if (tid < (c1b - c1a) * cn2) {
      const int ci = c1a + tid / cn2, cj = c2a + tid % cn2;
      sm.cnw[tid] = ci * I->W2 + cj;
      sm.cnt[tid] = (ci / I->G1) * I->TW2 + cj / I->G2;
    }
  }
  __syncthreads();
  const int l = wave / wpl;  // this wave's worker within the team
  const bool mine = l < gn, lead = mine && wave == l * wpl;
  const unsigned long long t_launch = __builtin_amdgcn_s_memrealtime();
  int r = 0, exit_status = 0;
  bool leave = sm.exit_f != 0, capped = false;
  __syncthreads();  // before exit_f is rewritten
  for (; !leave; ++r) {
    // ---- phase A
    {
      CInst<R> *const I = fresh<R>(I0);
      // every team runs exactly max_rounds rounds: all moves of the last round
      // are then applied everywhere and the launch can be resumed
      if (I->max_rounds > 0 && r >= I->max_rounds) {
        if (tid == 0) atomicCAS(&I->ctl->status, 0, 1);
        capped = true;
        break;
      }
      if (tid == 0) team_mark(sm, r, -1);
      // Stopping consensus of the round before: one 64-bit counter per ring
      // slot, completions in the low word and quiet workers in the high word.
      // One thread adds its team's and reads the exit flags while the
      // others select; the team acts on them in this round (a flag raised
      // later only costs empty rounds).
      unsigned long long ring_old = 0, ring_q = 0;
      int flags = 0;
      if (tid == kConsensus) {
        if (r > 0) {
          for (int q = 0; q < gn; ++q) ring_q += (unsigned)sm.done[q];
          ring_old = __hip_atomic_fetch_add(reinterpret_cast<unsigned long long *>(I->ring) + (r - 1) % kRing,
                                            (unsigned long long)gn + (ring_q << 32), __ATOMIC_RELAXED,
                                            __HIP_MEMORY_SCOPE_AGENT);
        }
        flags = ld_shared_i32(&I->ctl->converged) | ld_shared_i32(&I->ctl->stop);
      }
      const bool rnd = EXT && I->strategy == 3;
      const int inner = !EXT || rnd ? 1 : (I->inner > 0 ? I->inner : 1);  // a worker makes at most Mw visits per round
      const R tol = I->tol;
      // the neighbouring teams' progress, read while the selection runs
      const int *npr = nullptr;
      int npg = 0x7fffffff;
      if (lead && lane < 9) {
        const int n = sm.nbt[lane];
        if (n >= 0) {
          npr = I->prog + n;
          npg = ld_shared_i32(npr);
        }
      }
      // V(w0) of more than 512 positions is read by the worker's whole group
      const bool bigv = wpl > 1 && (long long)I->U1 * I->U2 > 512;
      int locked = 0;
      Held<R> c;
      long long restart = -1;  // first visit whose candidate had to wait: the next round starts there
      TeamWorker &k = sm.wk[mine ? l : 0];
      for (int v = 0; v < inner; ++v) {
        R vs = R(-1);
        int vp = 0x7fffffff;
        const int Mw = uni(k.nb1) * uni(k.nb2);
        const bool on = mine && !rnd && (inner == 1 || v < Mw);
        if (on) {
          scan_visit<R, NT>(I, sm, ls, l, wave - l * wpl, wpl, vs, vp);
          if (wpl > 1 && lane == 0) {
            sm.ps[wave] = vs;
            sm.pp[wave] = vp;
          }
        }
        if (inner > 1 && lead && lane == 0) sm.ion[l] = 0;
        if (wpl > 1 || inner > 1) __syncthreads();
        if (lead && on) {
          if (wpl > 1) {
            vs = lane < wpl ? sm.ps[wave + lane] : R(-1);
            vp = lane < wpl ? sm.pp[wave + lane] : 0x7fffffff;
            wave_argmax(vs, vp);
          }
          vp = uni(vp);
          const bool hit = __any(vs >= tol && vs > R(0));
          const long long visit = k.cursor;
          if (hit) {
            if (inner == 1 || Mw == 1) {  // (a worker of one sub-domain makes one visit)
              c.has = true;
              c.bs = vs;
              c.bp = vp;
            } else {
              visit_multi<R, NT>(I, sm, nzb, l, vs, vp, c, visit, restart);
            }
          }
          if (lane == 0) {
            k.cursor = visit + 1;
            const int m = k.mcur + 1;
            k.mcur = m == Mw ? 0 : m;
            if (inner > 1) next_visit(k);
            k.visit += 1;
            k.cand += hit;
            k.quiet = hit ? 0 : k.quiet + 1;
          }
        }
        if (inner > 1) {
          // the interior candidates of this visit lie in different workers'
          // blocks: their patches are disjoint
          __syncthreads();
          const PatchCtx<R> P = patch_ctx<R, NT>(I, sm, ls, nzb);
          for (int q = 0; q < gn; ++q)
            if (sm.ion[q])
              patch_rect<R, NT, NG, false>(P, sm.ui + q, tid, sm.ui[q].r1, sm.ui[q].r2, sm.ui[q].c1, sm.ui[q].c2);
          __syncthreads();
        }
      }
      if (lead) {
        const int w = uni(k.w), a1 = uni(k.a1), b1 = uni(k.b1), a2 = uni(k.a2), b2 = uni(k.b2);
        if (rnd) {
          const unsigned npw = (unsigned)((b1 - a1) * (b2 - a2)), K = (unsigned)I->K;
          const unsigned long long u = sm64_draw(I->seed, (unsigned long long)w, (unsigned long long)k.cursor);
          const unsigned long long jd = u % ((unsigned long long)npw * K), jp = jd / K;
          c.k0 = uni((int)(jd - jp * K));
          c.bp = uni((a1 + (int)jp / (b2 - a2)) * I->W + a2 + (int)jp % (b2 - a2));
          const long long i0 = (long long)c.bp * I->KS + c.k0;
          c.zc = as_global((const R *)I->z)[i0];
          c.zn = st_target((R)as_global((const R *)I->beta)[i0], (R)I->lambda, sm.inv_n[c.k0], I->positive);
          c.bs = move_score(c.zc, c.zn, tol, I->certify);
          c.has = __any(c.bs >= tol && c.bs > R(0));
          if (lane == 0) {
            k.cursor += 1;
            k.visit += 1;
            k.cand += c.has;
            if (c.has) k.quiet = 0;
          }
        }
        if (restart >= 0 && lane == 0) {
          k.cursor = restart;
          k.mcur = (int)(restart % (k.nb1 * k.nb2));
          next_visit(k);
        }
        // The visits read only S_w, which this team alone writes and finished
        // patching in its last phase B; so do the candidate's reads (its best
        // atom, value and target).  Only the soft-lock test (the neighbours'
        // scores of round r - 1) and the reuse of the candidate slot (read by
        // the neighbours in round r - 1) need the neighbours' progress.
        if (c.has && !rnd) best_move<R>(I, sm.inv_n, c.bp, &c.k0, &c.zc, &c.zn);
        if (tid == 0) team_mark(sm, r, 1);
        if (npg < r) {
          const unsigned long long t0 = __builtin_amdgcn_s_memrealtime();
          while (ld_shared_i32(npr) < r) {
            __builtin_amdgcn_s_sleep(1);
            if ((long long)(__builtin_amdgcn_s_memrealtime() - t0) > timeout_ticks) {
              sm.bad = 1;
              break;
            }
          }
        }
        __builtin_amdgcn_wave_barrier();
        if (tid == 0) team_mark(sm, r, 0);
        const int L1 = I->L1, L2 = I->L2, W = I->W;
        const int h0 = c.has ? c.bp / W : 0, w0 = c.has ? c.bp - h0 * W : 0;
        const bool test =
            c.has && I->soft_lock && (h0 - L1 + 1 < a1 || h0 + L1 > b1 || w0 - L2 + 1 < a2 || w0 + L2 > b2);
        if (test && lane == 0)
          k.chk += (unsigned long long)(min(h0 + L1, I->H) - max(h0 - L1 + 1, 0)) *
                   (unsigned long long)(min(w0 + L2, W) - max(w0 - L2 + 1, 0));
        if (bigv) {
          if (lane == 0) {
            sm.cp[l] = test ? c.bp : -1;
            sm.cs[l] = c.bs;
            sm.clk[l] = 0;
          }
        } else if (test) {
          locked = soft_test<R, NT>(I, sm, ls, w, a1, b1, a2, b2, c.bs, h0, w0, 0, 1);
        }
      }
      if (bigv) {
        __syncthreads();
        const int cp = mine ? uni(sm.cp[l]) : -1;
        if (cp >= 0) {
          const int ch = cp / I->W;
          const bool lk = soft_test<R, NT>(I, sm, ls, uni(k.w), uni(k.a1), uni(k.b1), uni(k.a2), uni(k.b2), sm.cs[l],
                                           ch, cp - ch * I->W, wave - l * wpl, wpl);
          if (lk && lane == 0) sm.clk[l] = 1;
        }
        __syncthreads();
        if (lead) locked = sm.clk[l];
      }
      if (lead && lane == 0) {
        // the band reads above are complete before the candidate becomes visible
        wait_vm();
        const bool acc = c.has && !locked;
        const unsigned long long dbits = acc ? delta_bits<R>(c.zn - c.zc) : 0ull;
        const unsigned long long rt = (unsigned long long)(unsigned)r << 32;
        const int w = k.w;
        unsigned long long *const cw = I->cand + (long long)kCandWords * w;
        st_shared_u64(cw + 1, rt | (dbits & 0xffffffffull));
        if (sizeof(R) == 8) st_shared_u64(cw + 2, rt | (dbits >> 32));
        st_shared_u64(cw, acc ? cand_tag(r, c.k0, (unsigned)c.bp) : cand_tag(r, 0, kNoPos));
        if (acc) {
          // z and its non-zero count change now; beta and the cache in phase B
          const int h0 = c.bp / I->W;
          move_z<R, NT>(I, sm, nzb, c.bp, h0, c.bp - h0 * I->W, c.k0, c.zc, c.zn);
          k.upd += 1;
        } else if (c.has) {
          k.lock += 1;
        }
        if (I->audit && r < I->audit_rounds)
          I->audit[(long long)r * (I->W1 * I->W2) + w] = audit_record(c.has, acc, c.k0, c.bp);
        next_visit(k);
      }
      if (tid == 0) team_mark(sm, r, 1);
      if (tid == kConsensus) {
        // the outcome of the stopping consensus
        const unsigned long long nW = (unsigned long long)(I->W1 * I->W2);
        if (r > 0 && (ring_old & 0xffffffffull) + (unsigned long long)gn == nW) {
          st_shared_u64(reinterpret_cast<unsigned long long *>(I->ring) + (r - 1) % kRing, 0ull);
          if ((ring_old >> 32) + ring_q == nW) {
            st_shared_i32(&I->ctl->converged, 1);
            flags = 1;
          }
        }
        if (!flags && (long long)(__builtin_amdgcn_s_memrealtime() - t_launch) > I->budget_ticks) {
          st_shared_i32(&I->ctl->stop, 1);
          atomicCAS(&I->ctl->status, 0, 4);
          flags = 1;
        }
        sm.exit_f = flags;
      }
    }
    if (wave == kCollect) collect<R, NT>(fresh<R>(I0), sm, r, timeout_ticks);
    __syncthreads();
    if (tid == 0) team_mark(sm, r, 2);
    if (sm.bad) {
      exit_status = 3;
      break;
    }
    leave = sm.exit_f != 0;

    // ---- phase B: apply the accepted candidates that touch the region (eq. beta_update)
    const int nuc = uni(sm.nuc);
    if (nuc > 0) {
      CInst<R> *const I = fresh<R>(I0);
      const PatchCtx<R> P = patch_ctx<R, NT>(I, sm, ls, nzb);
      if (uni(sm.ub_union)) {
        patch_union<R, NT, NG>(P, sm.uc, nuc, uni(sm.ub[0]), uni(sm.ub[1]), uni(sm.ub[2]), uni(sm.ub[3]));
      } else {
        // one after another; a barrier only before a patch that overlaps one
        // since the last barrier, and each patch continues where the last
        // left off in the order of the threads
        int base = 0, rot = 0;
        for (int c = 0; c < nuc; ++c) {
          const UCand<R> &u = sm.uc[c];
          if ((unsigned)uni((int)u.ov) >> base) {
            __syncthreads();
            base = c;
          }
          const int r1 = uni(u.r1), r2 = uni(u.r2), c1 = uni(u.c1), c2 = uni(u.c2);
          patch_rect<R, NT, NG, false>(P, &u, (tid - rot) & (NT - 1), r1, r2, c1, c2);
          rot = (rot + (((r2 - r1) * (c2 - c1)) << P.sh)) & (NT - 64);
        }
      }
    }
    const bool rnd = EXT && I0->strategy == 3;
    if (lead) {
      TeamWorker &k = sm.wk[l];
      bool tch = false;
      if (lane < nuc) {
        const UCand<R> &u = sm.uc[lane];
        tch = u.r1 < k.b1 && u.r2 > k.a1 && u.c1 < k.b2 && u.c2 > k.a2;
      }
      const int quiet = __any(tch) ? 0 : uni(k.quiet);
      const int qthr = rnd ? 1 : uni(k.nb1) * uni(k.nb2);  // quiet count of a worker with no pending move
      if (lane == 0) {
        k.quiet = quiet;
        sm.done[l] = quiet >= qthr ? 1 : 0;
      }
    }
    // cache stores complete before the progress counter moves
    wait_vm();
    __syncthreads();
    if (tid == 0) {
      st_shared_i32(I0->prog + team, r + 1);
      team_mark(sm, r, 3);
    }
    if (rnd) {
      if (lead) {
        CInst<R> *const I = fresh<R>(I0);
        TeamWorker &k = sm.wk[l];
        const int e2w = k.b2 - k.a2, npw = (k.b1 - k.a1) * e2w;
        if (k.cursor % npw == 0) {
          // end of an epoch: the worker is quiet if no position of S_w holds a
          // move scoring >= tol (every later patch of S_w clears it again)
          const GPtr<const R> sg = as_global((const R *)I->score);
          R mx = R(-1);
          for (int t = lane; t < npw; t += 64) {
            const int h = k.a1 + t / e2w, w = k.a2 + t % e2w;
            mx = fmax(mx, ls ? sm.score[(h - sm.A1) * (sm.B2 - sm.A2) + w - sm.A2] : sg[(long long)h * I->W + w]);
          }
          mx = wave_max(mx);
          if (lane == 0) sm.done[l] = k.quiet = mx >= I->tol && mx > R(0) ? 0 : 1;
        }
      }
      __syncthreads();
    }
  }
  // ---- leave: neighbours must never wait on a finished team
  wait_vm();
  __syncthreads();
  CInst<R> *const I = fresh<R>(I0);
  Ctl *const ctl = I->ctl;
  if (capped && r > 0 && tid == kConsensus) {  // the last round's consensus
    const unsigned long long nW = (unsigned long long)(I->W1 * I->W2);
    unsigned long long q = 0;
    for (int i = 0; i < gn; ++i) q += (unsigned)sm.done[i];
    const unsigned long long old =
        __hip_atomic_fetch_add(reinterpret_cast<unsigned long long *>(I->ring) + (r - 1) % kRing,
                               (unsigned long long)gn + (q << 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if ((old & 0xffffffffull) + (unsigned long long)gn == nW && (old >> 32) + q == nW)
      st_shared_i32(&ctl->converged, 1);
  }
  if (tid < gn) {
    const TeamWorker &k = sm.wk[tid];
    atomicAdd(&ctl->n_updates, (unsigned long long)k.upd);
    atomicAdd(&ctl->n_candidates, (unsigned long long)k.cand);
    atomicAdd(&ctl->n_softlocked, (unsigned long long)k.lock);
    atomicAdd(&ctl->n_visits, (unsigned long long)k.visit);
    atomicAdd(&ctl->n_checked, k.chk);
    atomicAdd(&ctl->n_patched, k.patch);
    const int sweep = I->strategy == 3 ? (k.b1 - k.a1) * (k.b2 - k.a2) : k.nb1 * k.nb2;
    atomicMax(&ctl->sweeps_done, (int)(k.cursor / sweep));
    if (I->wstate) {
      I->wstate[2 * k.w] = k.cursor;
      I->wstate[2 * k.w + 1] = k.quiet;
    }
  }
  if (tid == 0) {
    if (exit_status) {
      st_shared_i32(&ctl->stop, 1);
      atomicCAS(&ctl->status, 0, exit_status);
    }
    atomicAdd(&ctl->n_patched, sm.patched);
    // the timed rounds stand for all, the team's phase times for those of each of its workers
    const unsigned long long timed = (r + kTimed - 1) / kTimed;
    for (int i = 0; i < 4; ++i) sm.tk[i] = timed ? sm.tk[i] * (unsigned long long)r / timed : 0;
    atomicAdd(&ctl->tk_wait, sm.tk[0] * gn);
    atomicAdd(&ctl->tk_select, sm.tk[1] * gn);
    atomicAdd(&ctl->tk_collect, sm.tk[2] * gn);
    atomicAdd(&ctl->tk_apply, sm.tk[3] * gn);
    atomicMax(&ctl->max_round, r);
    st_shared_i32(I->prog + team, 0x7fffffff);
  }
}

// One 1024-thread team per CU, or four of 256 threads (at most 128 VGPRs).
template <class R, int NT, int NG, bool EXT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4))) void lgcd_rounds(
    const Inst<R> *__restrict__ insts, const int *__restrict__ wg_inst, long long timeout_ticks) {
  __shared__ TeamSmem<R, NT> sm;
  CInst<R> *I = (CInst<R> *)(insts + wg_inst[blockIdx.x]);
  run_team<R, NT, NG, EXT>(I, blockIdx.x - I->wg_base, timeout_ticks, sm);
}

// The kernel for positions of `ng` groups per lane (LaneMap::ng), with the
// random rule and several visits per round if `ext`.  Defined per type and
// workgroup size by rounds.hip.
template <class R, int NT> const void *rounds_kernel(int ng, bool ext);

}  // namespace dcdl
