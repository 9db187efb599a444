// vp_plan: online channel-guided demand decomposition (Sec. 4.2, Alg. 2) as
// one persistent workgroup of 512 threads that runs the whole iteration
// loop on the device (vp_plan_batch: one such workgroup per matrix).
//
// An iteration is a serial chain of short steps, so what bounds the planner
// is latency: LDS round trips, workgroup barriers and the instructions of
// single wavefronts, not bytes or operations.  The loop is therefore laid out
// for the fewest round trips: three barriers per iteration, every wavefront
// with its own share of the work in registers.
//   1. shape scores, Eq. (5)-(6), from node-block aggregates kept in LDS:
//      A = sum over nodes of the diagonal node block of D-hat and B_k = sum of
//      the blocks (n, n+k), in units of the pack granule as int32 (every
//      demand entry is a whole number of units, so scores keep their order).
//      A shape (k, L, R) scores sum A.L + sum B_k.R = sum D-hat.M, and its B
//      part depends on the pattern only through its set of NIC lanes.  Each
//      wavefront owns some of the sets and every pattern of them: its lanes
//      keep the sums of their set over up to eight shifts in registers and
//      re-read only the one shift that the last activation changed, reduce
//      to the set's best shift and add it to their patterns' A parts.
//   -- barrier --
//   2. the argmax (ties to the lowest canonical shape) is one LDS word that
//      the wavefronts' best candidates have met in by an atomic maximum.
//      MultiStartAA (Eq. (8)): one wavefront
//      per (family, start).  A lane owns up to a few rank groups: it reads
//      the family's record of their slots and the residuals of their in- and
//      out-lanes into registers, turns them into the binding credits
//      h' = min(D^rem_ij, cap) (Eq. (7) scaled by tau), draws its shuffles,
//      and exchanges the AA halves' assignments with the other lanes by
//      cross-lane permutes.  Meanwhile the other wavefronts write the
//      previous activation to the schedule arrays.
//   -- barrier --
//   3. Evaluate (Eq. (9)-(10)): the exact utility argmax in 128 bits over
//      families, redundantly in every wavefront (a one-family shape needs only
//      its best start).  The wavefront that ran the winner still holds its
//      binding: it subtracts the volumes from D^rem and the aggregates and
//      leaves the lanes in LDS for the schedule writers.
//   -- barrier --
// D^rem is kept in units, 32 bits each, blocked by group pair so that the
// g x g credits of a lane are one 16-byte load (g = 2): in LDS where the
// matrix fits beside the tables (up to 160 ranks or so), in the caller's
// workspace otherwise.  No host round trip happens between iterations.
//
// Measured, per activation: 2.1-2.2 us at 8 to 128 ranks and 3.4 us at 256 (16
// wavefronts, five barriers, the family's lists and credits staged in LDS for
// the runs, schedule stores by the winner's wavefronts: 4.6-4.9 and 6.3 us).
// A wavefront alone on its SIMD issues a dependent vector or scalar
// instruction every eight cycles, an independent one every four; an LDS read
// takes 64 cycles, a cross-lane permute 71, a taken branch about 30 and a
// barrier of eight wavefronts under 20, so instructions on the longest
// wavefront are what counts.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>
#include <string>

#include "divide.h"
#include "internal.h"

namespace vp {
namespace {

constexpr int kMaxQG = kMaxSlotsPerNode * kMaxGpusPerSwitch;   // lanes per node
constexpr int kMaxLTerms = 3 * kMaxSlotsPerNode;   // PIX, PXB and NIC entries of one diagonal block
constexpr int kHeldShifts = 8;                     // shifts of a set that one lane holds
constexpr int kFamChunk = 64;                      // families evaluated together

// Phase timing, compiled only with -DVP_PHASE_STAMPS (phase_stamps.py builds
// such a copy): one lane of the first start's wavefront stores the cycle
// counter at each phase boundary of every iteration, row = iteration (4096
// rows of 16); column k opens the phase that phase_stamps.py names.
#ifdef VP_PHASE_STAMPS
__device__ unsigned long long g_phase_stamps[4096 * 16];
#define VP_STAMP(k)                                                                              \
  do {                                                                                           \
    if (threadIdx.x == 0 && blockIdx.x == 0)                                                     \
      g_phase_stamps[(K < 4095 ? K : 4095) * 16 + (k)] = __builtin_readcyclecounter();           \
  } while (0)
#else
#define VP_STAMP(k) ((void)0)
#endif

struct Shared {
  int64_t total, total_units;
  int64_t Lmax;                // largest row or column sum in bytes, of a refused demand only
  // Aligned only for the code that the compiler then makes: with this and all
  // that follows 8 bytes lower an activation takes 2.24 us for 2.20 at 8 ranks
  // and 3.79 for 3.59 at 16 with cross-socket paths (other scalars spilled).
  alignas(16) uint32_t Lmax_units;   // largest row or column sum
  int32_t err, huge;           // huge: some demand entry reaches 2^42 bytes
  // Argmaxes of even and odd iterations: of the shapes, score << 33 |
  // (2^20 - 1 - shape code) << 13 | payload, with code = shift << 12 |
  // pattern and the payload the pattern's only family, or 2^12 where that has
  // to be looked up; and of the starts of a one-family shape, F << 4 |
  // (15 - start).
  uint64_t key[2];
  uint64_t step_key[2];        // shuffle keys of even and odd iterations: seed and iteration absorbed
  uint32_t top[2];
  uint64_t triple[4];          // two wavefronts per run: the canonical start's highest-credit triple of each slot
  int32_t changed[4];          // and whether a half-step changed any run
  const int64_t* D;
  const int32_t* inst_id;
  int32_t *family, *dst, *inst;
  int64_t *bytes, *send_off, *stream_off;
  int32_t* recv_src;
  int64_t unit, lambda, bw_p, bw_n;
};

struct PlanArgs {
  const int32_t* cat;
  DevCatalogLayout L;
  const int64_t* D;
  int64_t* Drem;
  int64_t k_target, lambda, unit;
  uint64_t seed;
  uint64_t odd_inv, odd_lim;
  int32_t unit_shift;
  int32_t n_start, i_aa, k_max, FC;
  int32_t LPS_log2, SPT;      // shift scoring: lanes per NIC-lane set (a power of two) and shifts per lane
  int32_t held;               // the lanes hold their shifts' sums (one round of sets, SPT <= kHeldShifts)
  int32_t MRT;                // largest NIC-lane set
  int32_t rec_lds;            // the family records are in LDS
  int32_t *K, *family, *dst, *inst;
  int64_t *bytes, *tau;
  int64_t *send_off, *stream_off;   // optional [k_max][N] buffer layout per rank
  int32_t* recv_src;                // optional [k_max][N]: the rank whose lane lands at each rank
  int32_t* status;
  int32_t batch;                    // matrices, one workgroup each; every buffer above holds `batch` of them
  // LDS layout (byte offsets)
  int32_t o_agg, o_rb, o_pr, o_xw, o_out, o_sacc, o_tab, o_res;
};

// ------------------------------------------------------------------ helpers

__device__ inline void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

extern "C" __device__ __attribute__((const)) long long __ockl_wfred_add_i64(long long);
__device__ inline int64_t wave_sum64(int64_t v) { return __ockl_wfred_add_i64(v); }

// lane 0's value in every lane (the whole wavefront active)
__device__ inline int32_t lane0(int32_t v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ inline int64_t lane0(int64_t v) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)v);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)(v >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}
__device__ inline uint32_t read_lane(uint32_t v, int l) { return (uint32_t)__builtin_amdgcn_readlane((int)v, l); }

// v of the lane n further on in its row of 16 lanes (cyclic)
template <int n>
__device__ inline uint32_t row_ror(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x120 + n, 0xF, 0xF, true);
}
// v of the lane whose index differs in bit n (1 or 2)
template <int n>
__device__ inline uint32_t quad_xor(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, n == 1 ? 0xB1 : 0x4E, 0xF, 0xF, true);
}
struct OpMax {
  __device__ static uint32_t f(uint32_t a, uint32_t b) { return a > b ? a : b; }
};
struct OpMin {
  __device__ static uint32_t f(uint32_t a, uint32_t b) { return a < b ? a : b; }
};
struct OpAdd {
  __device__ static uint32_t f(uint32_t a, uint32_t b) { return a + b; }
};
// Reduction over the wavefront (every lane active), wavefront-uniform.
template <class Op>
__device__ inline uint32_t wave_reduce(uint32_t v) {
  v = Op::f(v, row_ror<8>(v));
  v = Op::f(v, row_ror<4>(v));
  v = Op::f(v, row_ror<2>(v));
  v = Op::f(v, row_ror<1>(v));
  return Op::f(Op::f(read_lane(v, 0), read_lane(v, 16)), Op::f(read_lane(v, 32), read_lane(v, 48)));
}

// Binding credits are held in pack units as int32 (every credit is a whole
// number of units, so dividing by the unit keeps every comparison).  A self
// pair holds kForbiddenU = -2^29: valid credits are below 2^27, so a sum of at
// most four credits that includes a self pair is negative (it loses to every
// assignment without one), and four self pairs still fit in 32 bits.
constexpr int32_t kForbiddenU = -(1 << 29);

// SplitMix64 (Steele, Lea, Flood 2014): key absorbs the fields one at a time.
constexpr uint64_t kGolden = 0x9E3779B97F4A7C15ull;
__device__ inline uint64_t sm_mix(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}
// z mod (m + 1) for m + 1 in 2..4
template <int m1>
__device__ inline int small_mod(uint64_t z) {
  if constexpr (m1 == 3) return (int)(((uint32_t)(z >> 32) % 3u + (uint32_t)z % 3u) % 3u);   // 2^32 = 1 mod 3
  else return (int)((uint32_t)z & (uint32_t)(m1 - 1));
}

// Utility order of Eq. (10): (S1, x1/b1) beats (S2, x2/b2) exactly.
__device__ inline bool utility_greater(int64_t S1, int64_t x1, int64_t b1, int64_t S2, int64_t x2,
                                       int64_t b2, int64_t lam) {
  if (S1 == 0) return false;
  if (S2 == 0) return true;
  typedef unsigned __int128 u128;
  u128 lhs = (u128)S1 * (u128)b1 * ((u128)lam * (u128)b2 + (u128)x2);
  u128 rhs = (u128)S2 * (u128)b2 * ((u128)lam * (u128)b1 + (u128)x1);
  return lhs > rhs;
}

// Lexicographic permutations of g > 2 elements.
template <int g>
struct Perms;
template <>
struct Perms<3> {
  static constexpr int n = 6;
  __device__ static int at(int p, int m) {
    constexpr unsigned char t[6][3] = {{0, 1, 2}, {0, 2, 1}, {1, 0, 2}, {1, 2, 0}, {2, 0, 1}, {2, 1, 0}};
    return t[p][m];
  }
};
template <>
struct Perms<4> {
  static constexpr int n = 24;
  __device__ static int at(int p, int m) {
    constexpr unsigned char t[24][4] = {
        {0, 1, 2, 3}, {0, 1, 3, 2}, {0, 2, 1, 3}, {0, 2, 3, 1}, {0, 3, 1, 2}, {0, 3, 2, 1},
        {1, 0, 2, 3}, {1, 0, 3, 2}, {1, 2, 0, 3}, {1, 2, 3, 0}, {1, 3, 0, 2}, {1, 3, 2, 0},
        {2, 0, 1, 3}, {2, 0, 3, 1}, {2, 1, 0, 3}, {2, 1, 3, 0}, {2, 3, 0, 1}, {2, 3, 1, 0},
        {3, 0, 1, 2}, {3, 0, 2, 1}, {3, 1, 0, 2}, {3, 1, 2, 0}, {3, 2, 0, 1}, {3, 2, 1, 0}};
    return t[p][m];
  }
};

// Words of D^rem per group pair (a, d): the residual units of its g x g rank
// pairs, row by source, padded to whole 16-byte vectors.
template <int g>
constexpr int kResWords = g == 2 ? 4 : g == 3 ? 12 : 16;

template <int g>
__device__ inline void load_block(const uint32_t* p, uint32_t (&v)[g * g]) {
  const uint4* q = (const uint4*)p;
#pragma unroll
  for (int b = 0; b < kResWords<g> / 4; ++b) {
    const uint4 x = q[b];
    const uint32_t w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (b * 4 + e < g * g) v[b * 4 + e] = w[e];
  }
}

// Element idx of a global array whose byte offsets stay below 2^32 (checked
// on the host): a 32-bit offset from a wavefront-uniform base, which the
// compiler addresses as scalar base + vector offset.
template <typename T>
__device__ inline T& at32(T* base, uint32_t idx) {
  return *(T*)((char*)base + (uint32_t)(idx * (uint32_t)sizeof(T)));
}

// Workgroup barrier that orders LDS only: outstanding global stores of the
// waves are not waited for.
__device__ inline void lds_barrier() {
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0), other counters untouched
  __builtin_amdgcn_s_barrier();
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

// mask ? a : b, bit by bit
__device__ inline int32_t bit_select(int32_t mask, int32_t a, int32_t b) { return (mask & a) | (~mask & b); }

// Order of a group's g members over its g out-lanes (or in-lanes): at(m) is
// the member of lane m.  Two members need one bit; more are held one by one
// and are never indexed at run time.
template <int g>
struct Order {
  static constexpr int bits = 2 * g;
  int a[g];
  __device__ void identity() {
#pragma unroll
    for (int m = 0; m < g; ++m) a[m] = m;
  }
  __device__ int at(int m) const {
    int v = a[0];
#pragma unroll
    for (int x = 1; x < g; ++x) v = bit_select(m == x ? -1 : 0, a[x], v);   // values, so that no one indexes a[]
    return v;
  }
  __device__ void swap_if(bool c, int i, int j) {
    const int x = at(i), y = at(j);
#pragma unroll
    for (int m = 0; m < g; ++m) {
      a[m] = bit_select(c && m == j ? -1 : 0, x, a[m]);
      a[m] = bit_select(c && m == i ? -1 : 0, y, a[m]);
    }
  }
  __device__ uint32_t word() const {
    uint32_t w = 0;
#pragma unroll
    for (int m = 0; m < g; ++m) w |= (uint32_t)a[m] << (2 * m);
    return w;
  }
  // member of lane `pos` in a word shifted to this group
  __device__ static int member(uint32_t w, int pos) { return (int)((w >> (2 * pos)) & 3); }
  // Fisher-Yates on a SplitMix64 stream
  __device__ void shuffle(uint64_t state) {
    identity();
#pragma unroll
    for (int m = g - 1; m >= 1; --m) {
      state += kGolden;
      const uint64_t z = sm_mix(state);
      swap_if(true, m, m == 1 ? small_mod<2>(z) : m == 2 ? small_mod<3>(z) : small_mod<4>(z));
    }
  }
  // The best order where lane m earns h[m][x] with member x, the first one in
  // lexicographic order, if it beats the present one (whose self pairs earn
  // nothing).
  __device__ bool improve(const int32_t (&h)[g][g]) {
    int32_t cur = 0;
#pragma unroll
    for (int m = 0; m < g; ++m) {
      int32_t v = h[m][0];
#pragma unroll
      for (int x = 1; x < g; ++x) v = bit_select(a[m] == x ? -1 : 0, h[m][x], v);
      cur += v > 0 ? v : 0;
    }
    int32_t bestv = -1;
    uint32_t bw = 0;   // the best order's word, chosen as a constant: no table is indexed
#pragma unroll
    for (int p = 0; p < Perms<g>::n; ++p) {
      int32_t v = 0;
      uint32_t w = 0;
#pragma unroll
      for (int m = 0; m < g; ++m) {
        v += h[m][Perms<g>::at(p, m)];
        w |= (uint32_t)Perms<g>::at(p, m) << (2 * m);
      }
      bw = v > bestv ? w : bw;
      bestv = max(bestv, v);
    }
    const bool up = bestv > cur;
#pragma unroll
    for (int m = 0; m < g; ++m) a[m] = up ? (int)((bw >> (2 * m)) & 3) : a[m];
    return up;
  }
};
// Two members: the order is a mask, 0 or all ones (swapped), and everything
// follows by bit operations; a compare that feeds a select costs two more
// wait states here.
template <>
struct Order<2> {
  static constexpr int bits = 1;
  int32_t p;
  __device__ void identity() { p = 0; }
  __device__ int at(int m) const { return (p & 1) ^ m; }
  __device__ int32_t at_mask(int m) const { return m ? ~p : p; }   // all ones: member 1
  __device__ void swap_if(bool c, int i, int j) { p = c && i != j ? ~p : p; }
  __device__ uint32_t word() const { return (uint32_t)p & 1u; }
  __device__ void shuffle(uint64_t state) { p = (int32_t)((uint32_t)sm_mix(state + kGolden) & 1u) - 1; }
  // the present order's sum counts only if it beats itself clamped, which it
  // never does: the other order is the one to compare
  __device__ bool improve(const int32_t (&h)[2][2]) {
    const int32_t c0 = max(h[0][0], 0) + max(h[1][1], 0), c1 = max(h[0][1], 0) + max(h[1][0], 0);
    const int32_t s0 = h[0][0] + h[1][1], s1 = h[0][1] + h[1][0];
    const int32_t up = (bit_select(p, c1, c0) - bit_select(p, s0, s1)) >> 31;   // sums stay far inside 32 bits
    p ^= up;
    return up != 0;
  }
};

// g: ranks per group; MG: groups per lane; RL: D^rem in LDS; S: wavefronts
// per (family, start) run.  One wavefront runs a start of up to 128 groups of
// two ranks (64 larger groups), exchanging assignments by cross-lane
// permutes.  Beyond that two wavefronts share it (128 MG groups) and exchange
// through LDS with a workgroup barrier per half-step: halving a lane's groups
// then saves more than the barriers cost (512 ranks of two per group: 9.5 us
// per activation against 15.1 with four groups per lane, whose registers
// spill; 320 ranks of four: 16.5 against 28), while at 256 ranks of two it
// costs more (4.1 against 3.5 us).
// MS: more starts than run side by side, which then take turns on a slot: it
// reads the family's lanes and credits once and keeps its best binding.  As
// single runs on the path of many families, with a second run of the winner,
// sixteen starts took 7.2 us per activation at 64 ranks, 11.6 at 256 and 28 at
// 512; this way 3.9, 6.6 and 17.4.  (1,024 threads give every start its own
// wavefront but 128 registers: 4.0, 9.6 and 31.)
template <int g, int MG, bool RL, int S, bool MS>
__global__ void __launch_bounds__(kPlanThreads) plan_kernel(PlanArgs P) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  constexpr int g2 = g * g, RW = kResWords<g>;
  static_assert(Order<g>::bits * MG <= 32, "the orders of a lane's groups are exchanged in one word");
  constexpr int kSlots = kPlanWaves / S;   // runs side by side
  // The credit rows of a lane's groups are held in registers for a whole run
  // where they fit; else each half-step reads the entries it needs again.
  constexpr bool kHold = 2 * MG * g * g2 <= 64;
  constexpr int HM = kHold ? MG : 1;
  const int tid = threadIdx.x, lane = tid & 63, wave = lane0(tid >> 6);
  const int slot = wave & (kSlots - 1), part = wave / kSlots;
  const DevCatalogLayout& L = P.L;
  const int N = L.N, G = L.G, Q = L.Q, nn = L.nn, QG = Q * g, NS = P.n_start, kS = L.kS;
  // workgroup b plans matrix b of the batch: every global buffer is offset by b
  const size_t b = blockIdx.x, NN = (size_t)N * N, KN = (size_t)P.k_max * N;
  const int32_t* cat = P.cat;

  Shared* sh = (Shared*)smem;
  int32_t* agg = (int32_t*)(smem + P.o_agg);        // [q * Q + q2][kS] units: column 0 is A, column k is B_k; a zero row
  uint2* rb = (uint2*)(smem + P.o_rb);              // [nS + 1] best {units, shift} of each set; the last is zero
  const int npr = P.FC * NS * S;
  int32_t* prF = (int32_t*)(smem + P.o_pr);         // [FC * NS][S] score of each (family, start) run of the chunk (S parts),
  int32_t* prxp = prF + npr;                        // its largest lane volume on a PCIe-rate path
  int32_t* prxn = prxp + npr;                       // and on a NIC path (units)
  uint32_t* xw = (uint32_t*)(smem + P.o_xw) + slot * 256;   // S = 2: [2][128] orders of the out- and in-lanes
  uint2* out = (uint2*)(smem + P.o_out);            // [N] last activation: {destination | lane << 16, units} of each rank
  uint32_t* colsum = (uint32_t*)(smem + P.o_out);   // [N], prologue only
  int64_t* sacc = (int64_t*)(smem + P.o_sacc);      // [N] bytes each rank has sent so far
  const unsigned char* tab = smem + P.o_tab;
  const uint4* rows = (const uint4*)tab;
  const uint2* info = (const uint2*)(tab + L.pl_info);
  const int32_t* wtab = (const int32_t*)(tab + L.pl_wave);
  const uint4* set_rows = (const uint4*)(tab + L.pl_sets);
  // D^rem, [G][G][RW] units; a workspace slice is aligned up to 16 bytes (it holds 8 N^2 bytes, of which
  // the blocks take at most 16/3 N^2)
  uint32_t* res = RL ? (uint32_t*)(smem + P.o_res)
                     : (uint32_t*)(((uintptr_t)(P.Drem + b * NN) + 15) & ~(uintptr_t)15);
  auto div_q = [&](int x) { return Q == 1 ? x : (int)__umulhi((unsigned)x, L.q_magic); };

  // ---------------------------------------------------------------- prologue
  if (tid == 0) {
    sh->total = 0;
    sh->total_units = 0;
    sh->Lmax = 0;
    sh->Lmax_units = 0;
    sh->err = 0;
    sh->huge = 0;
    sh->key[0] = sh->key[1] = 0;
    sh->top[0] = sh->top[1] = 0;
    for (int x = 0; x < 4; ++x) {
      sh->triple[x] = 0;
      sh->changed[x] = 0;
    }
    sh->step_key[0] = sm_mix(sm_mix(P.seed + kGolden) + kGolden);
    // what only the writers and the comparison of families use is read from
    // LDS there: held in scalar registers through the loop it would push out
    // what every wavefront needs
    sh->D = P.D + b * NN;
    sh->inst_id = cat + L.off_fam_info;
    sh->family = P.family + b * P.k_max;
    sh->dst = P.dst + b * KN;
    sh->inst = P.inst + b * KN;
    sh->bytes = P.bytes + b * KN;
    sh->send_off = P.send_off ? P.send_off + b * KN : nullptr;
    sh->stream_off = P.stream_off ? P.stream_off + b * KN : nullptr;
    sh->recv_src = P.recv_src ? P.recv_src + b * KN : nullptr;
    sh->unit = P.unit;
    sh->lambda = P.lambda;
    sh->bw_p = L.bw_cls[VP_PATH_PIX];
    sh->bw_n = L.bw_cls[VP_PATH_NIC];
  }
  {
    const uint4* src = (const uint4*)(cat + L.off_plan);
    uint4* dst = (uint4*)(smem + P.o_tab);
    const int n = (P.rec_lds ? L.pl_end : L.pl_recs) / 16;
    for (int x = tid; x < n; x += 4 * kPlanThreads) {
      uint4 v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = src[min(x + u * kPlanThreads, n - 1)];
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (x + u * kPlanThreads < n) dst[x + u * kPlanThreads] = v[u];
    }
  }
  for (int x = tid; x < kS * (Q * Q + 1); x += kPlanThreads) agg[x] = 0;
  for (int x = tid; x <= L.nS; x += kPlanThreads) rb[x] = make_uint2(0, 0);
  for (int x = tid; x < N; x += kPlanThreads) {
    colsum[x] = 0;
    sacc[x] = 0;
  }
  __syncthreads();

  // One pass over D, eight rows per wavefront at a time: validate, store the
  // units blocked by group pair, sum rows, columns and aggregates.  An entry
  // of 2^42 bytes or more is refused before anything uses the sums: at most
  // 2^20 entries below 2^42 keep the total below 2^62, and the 32-bit unit
  // sums are exact whenever the total passes its check.
  {
    constexpr int RU = 8;
    bool bad = false, huge = false;
    int64_t tot = 0, totu = 0;
    uint32_t lmax = 0;
    const uint64_t mask = (uint64_t(1) << P.unit_shift) - 1;
    const int64_t* gD = P.D + b * NN;
    for (int i0 = wave * RU; i0 < N; i0 += kPlanWaves * RU) {
      uint32_t rs[RU];
#pragma unroll
      for (int u = 0; u < RU; ++u) rs[u] = 0;
      for (int j0 = 0; j0 < N; j0 += 64) {
        const int j = j0 + lane, jc = min(j, N - 1);
        int64_t v[RU];
#pragma unroll
        for (int u = 0; u < RU; ++u) v[u] = gD[(size_t)min(i0 + u, N - 1) * N + jc];
        const int gj = jc / g, nj = div_q(gj), qj = gj - nj * Q;
        uint32_t cs = 0;
#pragma unroll
        for (int u = 0; u < RU; ++u) {
          const int i = i0 + u;
          if (i >= N) break;   // uniform
          const int gi = i / g, ni = div_q(gi), qi = gi - ni * Q;
          if (j < N) {
            const uint64_t w = (uint64_t)v[u] >> P.unit_shift, units = w * P.odd_inv;   // exact quotient by the unit
            if (v[u] < 0 || (i == j && v[u] != 0) || ((uint64_t)v[u] & mask) != 0 || units > P.odd_lim) bad = true;
            if (v[u] >= (int64_t(1) << 42)) huge = true;
            tot += v[u];
            totu += (int64_t)units;
            const uint32_t vu = (uint32_t)units;
            res[((size_t)gi * G + gj) * RW + (i - gi * g) * g + (j - gj * g)] = vu;
            rs[u] += vu;
            cs += vu;
            int kk = nj - ni;
            if (kk < 0) kk += nn;
            if (vu) atomicAdd(&agg[(qi * Q + qj) * kS + kk], (int32_t)vu);
          }
        }
        if (j < N && cs) atomicAdd(&colsum[j], cs);
      }
#pragma unroll
      for (int u = 0; u < RU; ++u) {
        const uint32_t s = wave_reduce<OpAdd>(rs[u]);
        lmax = s > lmax ? s : lmax;
      }
    }
    if (bad) atomicCAS(&sh->err, 0, VP_ERR_INVALID_DEMAND);
    if (huge) sh->huge = 1;
    tot = wave_sum64(tot);
    totu = wave_sum64(totu);
    if (lane == 0) {
      atomicAdd((unsigned long long*)&sh->total, (unsigned long long)tot);
      atomicAdd((unsigned long long*)&sh->total_units, (unsigned long long)totu);
      atomicMax(&sh->Lmax_units, lmax);
    }
  }
  __syncthreads();
  {
    uint32_t lmax = 0;
    for (int j = tid; j < N; j += kPlanThreads) lmax = colsum[j] > lmax ? colsum[j] : lmax;
    lmax = wave_reduce<OpMax>(lmax);
    if (lane == 0) atomicMax(&sh->Lmax_units, lmax);
  }
  __syncthreads();
  // the quantum and the lane caps, in every wavefront
  int err = lane0(sh->err);
  const int64_t total_units = lane0(sh->total_units);
  auto quantum = [&](int64_t Lmax) {
    const int64_t den = L.bw_max * P.k_target, t = exact_div(Lmax + den - 1, den);
    return t < 1 ? (int64_t)1 : t;
  };
  int64_t tau = quantum(lane0((int64_t)sh->Lmax_units) * P.unit);
  uint32_t cap_p = 1, cap_n = 1;   // units
  {
    bool over = false;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      int64_t cu = exact_div(tau * L.bw_cls[c ? VP_PATH_NIC : VP_PATH_PIX], P.unit);
      if (cu < 1) cu = 1;
      // credits are int32 units below 2^27; a lane's bytes stay below 2^31
      over |= cu >= (int64_t(1) << 27) || cu * P.unit >= (int64_t(1) << 31);
      (c ? cap_n : cap_p) = (uint32_t)cu;
    }
    over |= sh->huge != 0 || sh->total >= (int64_t(1) << 42) || total_units >= (int64_t(1) << 28);
    if (err == 0 && over) {
      // the quantum goes out with the refusal too: the 32-bit sums may have
      // wrapped, so row and column sums again in 64 bits
      err = VP_ERR_UNSUPPORTED;
      const int64_t* gD = P.D + b * NN;
      for (int x = tid; x < 2 * N; x += kPlanThreads) {
        int64_t sum = 0;
        for (int y = 0; y < N; ++y) sum += x < N ? gD[(size_t)x * N + y] : gD[(size_t)y * N + (x - N)];
        if (sum > 0) atomicMax((unsigned long long*)&sh->Lmax, (unsigned long long)sum);
      }
      __syncthreads();
      tau = quantum(sh->Lmax);
    }
  }
  err = lane0(err);
  cap_p = (uint32_t)lane0((int32_t)cap_p);
  cap_n = (uint32_t)lane0((int32_t)cap_n);

  // this lane's groups; a lane past the last group computes on group 0 and
  // changes nothing
  int ga[MG], gn[MG], gq[MG];
  bool own[MG];
  uint32_t my_cap_p[MG], my_cap_n[MG];
#pragma unroll
  for (int r = 0; r < MG; ++r) {
    ga[r] = lane + 64 * (r * S + part);
    own[r] = ga[r] < G;
    ga[r] = own[r] ? ga[r] : 0;
    gn[r] = div_q(ga[r]);
    gq[r] = ga[r] - gn[r] * Q;
    my_cap_p[r] = own[r] ? cap_p : 0;
    my_cap_n[r] = own[r] ? cap_n : 0;
  }
  // this lane's share of the shape scores
  const int ib = lane0(wtab[wave]), ie = lane0(wtab[wave + 1]);
  const int sb = lane0(wtab[kPlanWaves + 1 + wave]), ns = lane0(wtab[kPlanWaves + 2 + wave]) - sb;
  const int nitem = (ie - ib + 63) >> 6, RW8 = L.RW / 8, LPS = 1 << P.LPS_log2;
  const bool has_set = P.held && lane < (ns << P.LPS_log2);
  const int my_set = has_set ? sb + (lane >> P.LPS_log2) : 0;
  const int SPT = P.SPT, k0 = 1 + (lane & (LPS - 1)) * SPT;
  // rows of this lane's set and first item (two to a register), absent ones
  // the zero row
  const uint32_t zero2 = (uint32_t)(Q * Q * kS) * 0x10001u;
  uint4 srow = make_uint4(zero2, zero2, zero2, zero2), irow = srow;
  uint2 info0 = make_uint2(0, 0);
  if (has_set) srow = set_rows[my_set];
  if (ib + lane < ie) {
    irow = rows[(ib + lane) * RW8];
    info0 = info[ib + lane];
  }
  auto row_of = [&](const uint4& o, int m) -> const int32_t* {
    const uint32_t w = m < 2 ? o.x : m < 4 ? o.y : m < 6 ? o.z : o.w;
    return agg + ((w >> (16 * (m & 1))) & 0xFFFF);
  };
  // sum of B_k over a set's lanes
  auto shift_sum = [&](int k) {
    int32_t s = row_of(srow, 0)[k] + row_of(srow, 1)[k] + row_of(srow, 2)[k] + row_of(srow, 3)[k];
    if (P.MRT > 4) s += row_of(srow, 4)[k] + row_of(srow, 5)[k] + row_of(srow, 6)[k] + row_of(srow, 7)[k];
    return s;
  };
  int32_t held[kHeldShifts];
#pragma unroll
  for (int u = 0; u < kHeldShifts; ++u) {
    const int k = k0 + u;
    held[u] = has_set && u < SPT && k < nn ? shift_sum(k) : -1;
  }

  // ---------------------------------------------------------------- loop
  // Every wavefront keeps these itself (they follow from LDS values that all
  // of them read): activations so far, units left, the last activation's
  // shift and family.
  int K = 0, kprev = -1, lf_prev = 0, f_prev = 0, written = 0;
  uint32_t rem = (uint32_t)total_units;

  // The last activation (step k, local family lf) to the schedule arrays,
  // the first ranks by the last wavefront.  What the stores wait for in
  // global memory is asked for ahead of them.
  struct Lane {
    uint2 w;       // {destination | lane << 16, units}
    int id;        // instance
    int64_t d;     // demand of the pair
    uint32_t left;   // and its residual, this activation subtracted
  };
  auto read_lane_out = [&](int i, int lf) {
    Lane x{};
    x.w = out[i];
    const int j = (int)(x.w.x & 0xFFFF);
    x.id = sh->inst_id[lf * QG + (int)(x.w.x >> 16)];
    if (sh->send_off) {
      x.d = sh->D[(size_t)i * N + j];
      const int a = i / g, c = j / g;
      const uint32_t* dp = res + ((size_t)a * G + c) * RW + (i - a * g) * g + (j - c * g);
      x.left = *dp;
    }
    return x;
  };
  auto write_lane = [&](int i, int k, int f, const Lane& l) {
    const int j = (int)(l.w.x & 0xFFFF);
    const uint32_t unit = (uint32_t)sh->unit;   // below 2^31
    const int64_t x = (int64_t)((uint64_t)l.w.y * unit);
    const uint32_t o = (uint32_t)(k * N + i);
    if (sh->send_off) {
      // Sec. 5 buffer layout: where this lane's slice sits in rank i's send
      // buffer and in its stream to j (the bytes sent there before)
      const int64_t so = sacc[i];
      sacc[i] = so + x;
      at32(sh->send_off, o) = so;
      at32(sh->stream_off, o) = l.d - x - (int64_t)((uint64_t)l.left * unit);
    }
    at32(sh->dst, o) = j;
    at32(sh->inst, o) = l.id >> 12;
    at32(sh->bytes, o) = x;
    if (sh->recv_src) at32(sh->recv_src, (uint32_t)(k * N + j)) = i;   // pi_k is a permutation
    if (i == 0) sh->family[k] = f;
  };
  const int i_first = (kPlanWaves - 1 - wave) * 64 + lane;

  // The half-steps of S = 2 so far (see publish).
  int half_step = 0;
  // The records of local family lf for this lane's groups: g out-lanes, then
  // g in-lanes, 16 bits each.
  auto read_records = [&](uint32_t (&rec)[MG][g], int lf) {
#pragma unroll
    for (int r = 0; r < MG; ++r) {
      const int at = (lf * Q + gq[r]) * g;
      if (__builtin_expect(P.rec_lds, 1)) {
#pragma unroll
        for (int m = 0; m < g; ++m) {
          rec[r][m] = ((const uint32_t*)(tab + L.pl_recs))[at + m];
          asm("" : "+v"(rec[r][m]));   // keeps the two loads apart: merged they would be one flat load
        }
      } else {
#pragma unroll
        for (int m = 0; m < g; ++m) rec[r][m] = ((const uint32_t*)((const char*)(cat + L.off_plan) + L.pl_recs))[at + m];
      }
    }
  };
  // all ones if bit `bit` of e is set
  auto bit_mask = [](uint32_t e, int bit) { return (int32_t)(e << (31 - bit)) >> 31; };
  // Positions in an in- or out-list are masks for two ranks per group (all
  // ones is 1), as the orders are.
  auto pos_index = [](int p) { return g == 2 ? p & 1 : p; };
  // Out-lanes under shift kstar: descriptor, destination group, position in
  // that group's in-list.
  struct OutLanes {
    uint32_t e[MG][g], d[MG][g];
    int pos[MG][g];
    __device__ int32_t nic(int r, int m) const { return (int32_t)(e[r][m] << 16) >> 31; }   // mask
  };
  auto decode_out = [&](OutLanes& o, const uint32_t (&rec)[MG][g], int kstar) {
#pragma unroll
    for (int r = 0; r < MG; ++r) {
      int dn = gn[r] + kstar;
      dn = (int)min((uint32_t)dn, (uint32_t)(dn - nn));
      const int dq = dn * Q, nq = ga[r] - gq[r];
      // cross-node lanes come first in an in-list exactly where their source
      // node is lower: the lanes of the other kind before this one
      const int32_t far_after = dn >= kstar ? 0 : -1, near_after = gn[r] >= kstar ? -1 : 0;
#pragma unroll
      for (int m = 0; m < g; ++m) {
        const uint32_t e = m & 1 ? rec[r][m >> 1] >> 16 : rec[r][m >> 1];   // bits above 15 are not read
        const int32_t nic = bit_mask(e, 15), after = bit_select(nic, far_after, near_after);
        o.e[r][m] = e;
        o.d[r][m] = (uint32_t)bit_select(nic, dq, nq) + (e & 7);
        o.pos[r][m] = g == 2 ? bit_mask(e, 3) | (bit_mask(e, 5) & after)
                             : (int)((e >> 3) & 3) + ((int)((e >> 5) & 7) & after);
      }
    }
  };
  // credit: min(D^rem, cap) (none on a lane past the last group), kForbiddenU
  // for a self pair
  auto credit = [&](uint32_t w, uint32_t cap, bool self) {
    return self ? kForbiddenU : (int32_t)(w < cap ? w : cap);
  };
  auto lane_cap = [&](int r, int32_t nic) { return (uint32_t)bit_select(nic, (int32_t)my_cap_n[r], (int32_t)my_cap_p[r]); };
  // The highest-credit triple, ties to the smallest (lane, i, j): `top` is the
  // wavefront's largest credit (0: none); on the one lane that holds the
  // triple, `mine`, its key (lane, i, j), and its fields packed for bind_top.
  // entry(x) is the lane's x-th credit in (group, out-lane, i, j) order, which
  // is the order of the lanes: a group's out-lanes are in lane order, groups
  // in node order.
  struct Triple {
    uint32_t top, key, pack;
    bool mine;
  };
  auto find_top = [&](const OutLanes& o, auto entry) {
    constexpr int kEnt = MG * g * g2, kIdx = kEnt <= 8 ? 3 : kEnt <= 16 ? 4 : 5;
    uint32_t tv = 0, tw = 0;   // the largest credit and the first entry that has it
    if constexpr (kEnt <= 32) {
      // credits stay below 2^27: value and (inverted) index in one word
      uint32_t key = 0;
#pragma unroll
      for (int x = 0; x < kEnt; ++x)
        key = max(key, (uint32_t)max(entry(x), 0) << kIdx | (uint32_t)((1 << kIdx) - 1 - x));
      tv = key >> kIdx;
      tw = (uint32_t)((1 << kIdx) - 1) - (key & ((1 << kIdx) - 1));
    } else {
#pragma unroll
      for (int x = 0; x < kEnt; ++x) {
        const int32_t v = entry(x);
        tw = v > (int32_t)tv ? (uint32_t)x : tw;
        tv = (uint32_t)max((int32_t)tv, v);
      }
    }
    // this lane's fields, while the reduction is under way
    const uint32_t om = tw / g2, e = tw % g2;
    uint32_t t = 0, d = 0, a = 0;
    int mi = 0;
#pragma unroll
    for (int r = 0; r < MG; ++r)
#pragma unroll
      for (int m = 0; m < g; ++m) {
        const bool it = om == (uint32_t)(r * g + m);
        t = it ? (uint32_t)(gn[r] * QG) + ((o.e[r][m] >> 8) & 31) : t;
        d = it ? o.d[r][m] : d;
        mi = it ? pos_index(o.pos[r][m]) : mi;
        a = it ? (uint32_t)ga[r] : a;
      }
    Triple T;
    T.key = t * (uint32_t)g2 + e;
    T.pack = a | d << 9 | (om % g) << 18 | (e / g) << 20 | (e % g) << 22 | (uint32_t)mi << 24;
    T.top = wave_reduce<OpMax>(tv);
    T.mine = tv == T.top;
    const uint64_t eq = __ballot(T.mine);
    if ((eq & (eq - 1)) != 0) {   // the whole wavefront reduces
      const uint32_t key = T.mine ? T.key : ~0u, lo = wave_reduce<OpMin>(key);
      T.mine = key == lo;
    }
    return T;
  };
  // Both sides' shuffled orders of a start: independent Fisher-Yates shuffles
  // of every group's sources and destinations on SplitMix64 streams keyed by
  // seed, iteration, family, start, group and side; the key prefix is uniform
  // over the wavefront.
  auto draw = [&](Order<g> (&sig)[MG], Order<g> (&del)[MG], uint64_t step_key, int family, int start) {
    uint64_t k3 = step_key ^ (uint64_t)family;
    k3 = sm_mix(k3 + kGolden) ^ (uint64_t)start;
    const uint64_t k4 = sm_mix(k3 + kGolden);
#pragma unroll
    for (int r = 0; r < MG; ++r) {
      const uint64_t k5 = sm_mix((k4 ^ (uint64_t)ga[r]) + kGolden);
      sig[r].shuffle(k5);
      del[r].shuffle(k5 ^ 1);
    }
  };
  auto order_word = [&](const Order<g> (&a)[MG]) -> uint32_t {
    uint32_t w = a[0].word();
#pragma unroll
    for (int r = 1; r < MG; ++r) w |= a[r].word() << (r * Order<g>::bits);
    return w;
  };

  // One MultiStartAA run: local family lf, one start, on this wavefront.
  // Leaves the binding in `sig` (source of each out-lane), `jf` (member of
  // its destination), `ent` (out-lane descriptor), `dg` (destination group)
  // and `xv` (units); returns the binding score F (Eq. (8)) and, if need_x,
  // the largest lane volume on PCIe-rate and NIC paths.
  struct Bound {
    Order<g> sig[MG];
    int jf[MG][g];   // for g = 2 a mask, all ones for member 1
    __device__ int member(int r, int m) const { return g == 2 ? jf[r][m] & 1 : jf[r][m]; }
    uint32_t xv[MG][g];
    uint32_t left[RL || MS ? 1 : MG][g];   // D^rem in global memory: the residual of each lane's pair
  };
  struct Binding : Bound {
    OutLanes o;
  };
  // MS, all_starts: the slot's starts one after another on the same lanes and
  // credits; `start` becomes the one kept, its first best.
  auto run = [&](Binding& B, int lf, int kstar, int fbase, int& start, uint64_t step_key, bool all_starts, bool need_x,
                 uint32_t& xp, uint32_t& xn) __attribute__((always_inline)) -> uint32_t {
    uint32_t rec[MG][g];
    read_records(rec, lf);
    OutLanes& o = B.o;
    decode_out(o, rec, kstar);
    uint32_t raw[HM][g][g2], rin[HM][g][g2];
    // where group d's order is: its word (byte offset: lane, and with two
    // wavefronts its part) and the bit its order starts at
    auto word_of = [&](uint32_t d) {
      constexpr uint32_t n = 64 * S;
      return MG == 1 ? d << 2 : (d & (n - 1)) << 2 | (d / n * Order<g>::bits) << 16;
    };
    uint32_t oword[MG][g], iword[MG][g];   // word | bit << 16
    int ipos[MG][g];
    bool oself[MG][g], iself[MG][g];
    uint32_t ocap[MG][g], icap[MG][g], sg[MG][g];
#pragma unroll
    for (int r = 0; r < MG; ++r) {
#pragma unroll
      for (int m = 0; m < g; ++m)
        if constexpr (kHold) load_block<g>(res + ((uint32_t)(ga[r] * G) + o.d[r][m]) * RW, raw[r][m]);
      // in-lanes, stored cross-node lanes first: same-node lanes lead where
      // the source node of the others is the higher one
      int sn = gn[r] - kstar;
      sn = (int)min((uint32_t)sn, (uint32_t)(sn + nn));
      const int sq = sn * Q, nq = ga[r] - gq[r];
      uint32_t ein[g];
      if constexpr (g == 2) {
        const uint32_t w = rec[r][1];
        const int32_t turn = bit_mask(w, 14) & (gn[r] >= kstar ? 0 : 16);   // one lane of each kind
        const uint32_t v = __builtin_amdgcn_alignbit(w, w, (uint32_t)turn);
        ein[0] = v;
        ein[1] = v >> 16;
      } else {
        auto in_at = [&](int x) { return (x & 1 ? rec[r][x >> 1] >> 16 : rec[r][x >> 1]) & 0xFFFFu; };
        int nr = 0;
#pragma unroll
        for (int m = 0; m < g; ++m) nr += (int)(in_at(g + m) >> 15);
        const int rot = gn[r] >= kstar ? 0 : nr;
#pragma unroll
        for (int m = 0; m < g; ++m) {
          ein[m] = in_at(g + m);
#pragma unroll
          for (int t = 1; t < g; ++t) ein[m] = (uint32_t)bit_select(rot == t ? -1 : 0, (int)in_at(g + (m + t) % g), (int)ein[m]);
        }
      }
#pragma unroll
      for (int m = 0; m < g; ++m) {
        const uint32_t e = ein[m];
        const int32_t nic = bit_mask(e, 15);
        const uint32_t s = (uint32_t)bit_select(nic, sq, nq) + (e & 7);
        sg[r][m] = s;
        if constexpr (kHold) load_block<g>(res + (s * (uint32_t)G + (uint32_t)ga[r]) * RW, rin[r][m]);
        iself[r][m] = own[r] && s == (uint32_t)ga[r];
        icap[r][m] = lane_cap(r, nic);
        ipos[r][m] = g == 2 ? bit_mask(e, 3) : (int)((e >> 3) & 3);
        iword[r][m] = word_of(s);
      }
#pragma unroll
      for (int m = 0; m < g; ++m) {
        oself[r][m] = own[r] && o.d[r][m] == (uint32_t)ga[r];
        ocap[r][m] = lane_cap(r, o.nic(r, m));
        oword[r][m] = word_of(o.d[r][m]);
      }
    }
    int32_t hs[HM][g][g2], hd[HM][g][g2];
    auto hold = [&]() __attribute__((always_inline)) {
      if constexpr (kHold) {
#pragma unroll
        for (int r = 0; r < MG; ++r)
#pragma unroll
          for (int m = 0; m < g; ++m)
#pragma unroll
            for (int e = 0; e < g2; ++e) {
              hs[r][m][e] = credit(raw[r][m][e], ocap[r][m], e / g == e % g && oself[r][m]);
              hd[r][m][e] = credit(rin[r][m][e], icap[r][m], e / g == e % g && iself[r][m]);
            }
      }
    };
    if constexpr (MS) hold();
    // credit of out-lane (r, m) from source il to member jl, and of in-lane
    // (r, m) from member il to destination jl
    auto out_credit = [&](int r, int m, int il, int jl) {
      return credit(res[((uint32_t)(ga[r] * G) + o.d[r][m]) * RW + il * g + jl], ocap[r][m], il == jl && oself[r][m]);
    };
    auto in_credit = [&](int r, int m, int il, int jl) {
      return credit(res[(sg[r][m] * (uint32_t)G + (uint32_t)ga[r]) * RW + il * g + jl], icap[r][m], il == jl && iself[r][m]);
    };
    auto bind = [&](Bound& B, int start) __attribute__((always_inline)) -> uint32_t {
      Order<g> del[MG];
      if (start == 0) {
#pragma unroll
        for (int r = 0; r < MG; ++r) {
          B.sig[r].identity();
          del[r].identity();
        }
      } else {
        draw(B.sig, del, step_key, fbase + lf, start);
      }
      if constexpr (!MS) hold();   // the loads are under way while the orders are drawn
      // Start 0: the canonical binding with the highest-credit triple put in;
      // its lane's out- and in-list positions are protected (-1: none here).
      int prot_o[MG], prot_i[MG];
#pragma unroll
      for (int r = 0; r < MG; ++r) prot_o[r] = prot_i[r] = -1;
      auto bind_top = [&](int a, int m0, int il, int jl, int d, int mi) {
#pragma unroll
        for (int r = 0; r < MG; ++r) {
          // members are still in order: the one to move is at its own position
          const bool so = ga[r] == a && own[r], di = ga[r] == d && own[r];
          prot_o[r] = so ? m0 : -1;
          B.sig[r].swap_if(so, m0, il);
          prot_i[r] = di ? mi : -1;
          del[r].swap_if(di, mi, jl);
        }
      };
      auto bind_pack = [&](uint32_t w) {
        bind_top((int)(w & 511), (int)((w >> 18) & 3), (int)((w >> 20) & 3), (int)((w >> 22) & 3), (int)((w >> 9) & 511),
                 (int)((w >> 24) & 3));
      };
      auto top_here = [&]() {
        return find_top(o, [&](int x) -> int32_t {
          const int r = x / (g * g2), m = x / g2 % g, e = x % g2;
          if constexpr (kHold) return hs[r][m][e];
          else return out_credit(r, m, e / g, e % g);
        });
      };
      if constexpr (S == 1) {
        if (start == 0) {
          const Triple T = top_here();
          if (T.top != 0) bind_pack(read_lane(T.pack, __builtin_ctzll(__ballot(T.mine))));
        }
      } else {
        if (start == 0) {
          // the two wavefronts' triples meet in one word: credit, (lane, i, j)
          // inverted (below 2^14), destination group, position there
          const Triple T = top_here();
          if (T.mine && T.top != 0)
            atomicMax((unsigned long long*)&sh->triple[slot],
                      (unsigned long long)T.top << 32 | (unsigned long long)(0x3FFF - T.key) << 16 |
                          (unsigned long long)(((T.pack >> 9) & 511) << 2 | ((T.pack >> 24) & 3)));
        }
        lds_barrier();   // every wavefront comes here: runs are in step
        if (start == 0) {
          const uint64_t w = (uint64_t)lane0((int64_t)sh->triple[slot]);
          if (w != 0) {
            const uint32_t key = 0x3FFF - ((uint32_t)(w >> 16) & 0x3FFF), t = key / (uint32_t)g2, e = key % (uint32_t)g2;
            int a = -1, m0 = 0;   // on the lane that owns it
#pragma unroll
            for (int r = 0; r < MG; ++r)
#pragma unroll
              for (int m = 0; m < g; ++m)
                if (own[r] && (uint32_t)(gn[r] * QG) + ((o.e[r][m] >> 8) & 31) == t) {
                  a = ga[r];
                  m0 = m;
                }
            bind_top(a, m0, (int)(e / g), (int)(e % g), (int)((w >> 2) & 0x3FFF), (int)(w & 3));
          }
        }
      }
      // Self-binding repair, per group in out-list order: trade destinations
      // with the first other unprotected in-lane, else sources with the first
      // other unprotected out-lane.
#pragma unroll
      for (int r = 0; r < MG; ++r)
#pragma unroll
        for (int m = 0; m < g; ++m) {
          const int mi = pos_index(o.pos[r][m]);
          if (oself[r][m] && B.sig[r].at(m) == del[r].at(mi)) {
            int pi = -1, po = -1;
#pragma unroll
            for (int x = g - 1; x >= 0; --x) {
              pi = x != mi && x != prot_i[r] ? x : pi;
              po = x != m && x != prot_o[r] ? x : po;
            }
            del[r].swap_if(pi >= 0, mi, pi);
            B.sig[r].swap_if(pi < 0 && po >= 0, m, po);
          }
        }
      // Alternating Algorithm: source half, then destination half.  A half that
      // changes nothing, other than the very first, leaves a fixed point: the
      // half before it made its own side optimal against this side, which has
      // not moved.  Stopping there gives the same binding as stopping after a
      // whole unchanged sweep.
      auto pack = [&](const Order<g> (&a)[MG]) -> uint32_t {
        if constexpr (g == 2 && MG == 1) return (uint32_t)a[0].p;
        else return order_word(a);
      };
      // entry `i` of a row (or column) of credits, i a member or, for g = 2, its mask
      auto pick = [&](const int32_t (&c)[g], int i) {
        if constexpr (g == 2) {
          return bit_select(i, c[1], c[0]);
        } else {
          int32_t v = c[0];
#pragma unroll
          for (int x = 1; x < g; ++x) v = bit_select(i == x ? -1 : 0, c[x], v);
          return v;
        }
      };
      // Member at the other side of a lane, from this lane's view of that side's
      // orders `w`: a permute, or (S = 2) the words that publish() left in LDS.
      auto fetch = [&](uint32_t from, int pos, uint32_t w, int side) {
        const uint32_t at = MG == 1 ? from : from & 0xFFFF, shift = MG == 1 ? 0 : from >> 16;
        uint32_t v;
        if constexpr (S == 1) v = (uint32_t)__builtin_amdgcn_ds_bpermute((int)at, (int)w);
        else v = *(const uint32_t*)((const char*)(xw + side * S * 64) + at);
        if constexpr (g == 2) {   // a mask: all ones is member 1 (`pos` is one as well)
          if constexpr (MG == 1) return (int)v ^ pos;
          else return ((int)(v << (31 - shift)) >> 31) ^ pos;
        } else {
          if constexpr (MG > 1) v >>= shift;
          return Order<g>::member(v, pos);
        }
      };
      VP_STAMP(5);
      // S = 2: leave the orders in LDS and learn whether any run has changed in
      // this half-step (a run at its fixed point stays there).  The flags of
      // four half-steps rotate: one is cleared two half-steps before it is used.
      auto publish = [&](int side, uint32_t w, bool changed) {
        xw[side * S * 64 + part * 64 + lane] = w;
        if (changed && lane == 0) sh->changed[half_step & 3] = 1;
        if (tid == 0) sh->changed[(half_step + 2) & 3] = 0;
        lds_barrier();
      };
      auto any_changed = [&]() -> bool { return lane0(sh->changed[half_step++ & 3]) != 0; };
      int il[MG][g];
      auto fetch_out = [&](uint32_t w) {
#pragma unroll
        for (int r = 0; r < MG; ++r)
#pragma unroll
          for (int m = 0; m < g; ++m) B.jf[r][m] = fetch(oword[r][m], o.pos[r][m], w, 1);
      };
      auto fetch_in = [&](uint32_t w) {
#pragma unroll
        for (int r = 0; r < MG; ++r)
#pragma unroll
          for (int m = 0; m < g; ++m) il[r][m] = fetch(iword[r][m], ipos[r][m], w, 0);
      };
      uint32_t dw = pack(del);
      if constexpr (S == 2) {
        publish(1, dw, false);
        ++half_step;
        fetch_out(dw);
        if (part == 0 && lane == 0) sh->triple[slot] = 0;   // both wavefronts have read it
        // The next run's maximum must find the word cleared: a half-step's
        // barrier lies between, or this one where there is none.
        if (P.i_aa == 0) lds_barrier();
      }
      bool stale = S == 1;   // jf is older than del
      for (int sweep = 0; sweep < P.i_aa; ++sweep) {
        bool changed = false;
        if constexpr (S == 1) {
          fetch_out(dw);
          stale = false;
        }
#pragma unroll
        for (int r = 0; r < MG; ++r) {
          int32_t h[g][g];
#pragma unroll
          for (int m = 0; m < g; ++m)
#pragma unroll
            for (int il = 0; il < g; ++il) {
              if constexpr (kHold) {
                int32_t row[g];
#pragma unroll
                for (int jj = 0; jj < g; ++jj) row[jj] = hs[r][m][il * g + jj];
                h[m][il] = pick(row, B.jf[r][m]);
              } else {
                h[m][il] = out_credit(r, m, il, B.member(r, m));
              }
            }
          changed |= B.sig[r].improve(h);
        }
        changed = __any(changed);
        if constexpr (S == 1) {
          if (sweep > 0 && !changed) break;
          fetch_in(pack(B.sig));
        } else {
          const uint32_t sw = pack(B.sig);
          publish(0, sw, changed);
          fetch_in(sw);
          if (!any_changed() && sweep > 0) break;
        }
        changed = false;
#pragma unroll
        for (int r = 0; r < MG; ++r) {
          int32_t h[g][g];
#pragma unroll
          for (int m = 0; m < g; ++m)
#pragma unroll
            for (int jl = 0; jl < g; ++jl) {
              if constexpr (kHold) {
                int32_t col[g];
#pragma unroll
                for (int ii = 0; ii < g; ++ii) col[ii] = hd[r][m][ii * g + jl];
                h[m][jl] = pick(col, il[r][m]);
              } else {
                h[m][jl] = in_credit(r, m, g == 2 ? il[r][m] & 1 : il[r][m], jl);
              }
            }
          changed |= del[r].improve(h);
        }
        changed = __any(changed);
        if constexpr (S == 1) {
          if (!changed) break;
          dw = pack(del);
          stale = true;
        } else {
          dw = pack(del);
          publish(1, dw, changed);
          fetch_out(dw);
          if (!any_changed()) break;
        }
      }
      VP_STAMP(6);
      if (stale) fetch_out(dw);
      // in global memory the residuals that the winner lowers are asked for
      // ahead of the comparison of the starts
      if constexpr (!RL && !MS) {
#pragma unroll
        for (int r = 0; r < MG; ++r)
#pragma unroll
          for (int m = 0; m < g; ++m)
            B.left[r][m] = res[((uint32_t)(ga[r] * G) + o.d[r][m]) * RW + (uint32_t)(B.sig[r].at(m) * g + B.member(r, m))];
      }
      uint32_t F = 0;
      xp = xn = 0;
#pragma unroll
      for (int r = 0; r < MG; ++r)
#pragma unroll
        for (int m = 0; m < g; ++m) {
          int32_t x;
          if constexpr (kHold) {
            int32_t row[g], col[g];
#pragma unroll
            for (int j2 = 0; j2 < g; ++j2) {
#pragma unroll
              for (int i2 = 0; i2 < g; ++i2) col[i2] = hs[r][m][i2 * g + j2];
              if constexpr (g == 2) row[j2] = pick(col, B.sig[r].at_mask(m));
              else row[j2] = pick(col, B.sig[r].at(m));
            }
            x = pick(row, B.jf[r][m]);
          } else {
            x = out_credit(r, m, B.sig[r].at(m), B.member(r, m));
          }
          const uint32_t xu = (uint32_t)max(x, 0);   // a self pair serves nothing
          B.xv[r][m] = xu;
          F += xu;
          xn = max(xn, xu & (uint32_t)o.nic(r, m));
          xp = max(xp, xu & ~(uint32_t)o.nic(r, m));
        }
      F = wave_reduce<OpAdd>(F);
      if (need_x) {   // the lane maxima only serve comparisons between families
        xp = wave_reduce<OpMax>(xp);
        xn = wave_reduce<OpMax>(xn);
      }
      return F;
    };
    if constexpr (!MS) {
      return bind(B, start);
    } else {
      uint32_t top = 0;
      const int first = start;
      for (int s0 = first - slot;; s0 += kSlots) {
        const int s = all_starts ? min(s0 + slot, NS - 1) : first;
        Bound C;
        uint32_t F = bind(C, s);
        if (S == 2 && all_starts) {   // the score of both wavefronts
          if (lane == 0) prF[s * S + part] = (int32_t)F;
          lds_barrier();
          const int2 f2 = ((const int2*)prF)[s];
          F = (uint32_t)lane0(f2.x + f2.y);
        }
        if (s0 == first - slot || F > top) {
          (Bound&)B = C;
          top = F;
          start = s;
        }
        if (!all_starts || (S == 1 ? s0 + kSlots + slot : s0 + kSlots) >= NS) return top;
      }
    }
  };
  // Subtract X(E*) from D^rem and the aggregates and leave the lanes for the
  // writers.
  auto apply = [&](const Binding& B, int kstar) __attribute__((always_inline)) {
#pragma unroll
    for (int r = 0; r < MG; ++r) {
      if (!own[r]) continue;
#pragma unroll
      for (int m = 0; m < g; ++m) {
        const uint32_t e = B.o.e[r][m], x = B.xv[r][m], d = B.o.d[r][m];
        const int il = B.sig[r].at(m), jl = B.member(r, m);
        out[ga[r] * g + il] = make_uint2((d * g + (uint32_t)jl) | (e & 0x1F00) << 8, x);
        uint32_t* dp = res + ((uint32_t)(ga[r] * G) + d) * RW + (uint32_t)(il * g + jl);
        if constexpr (RL) atomicSub(dp, x);
        else if (x != 0) *dp = (MS ? *dp : B.left[r][m]) - x;
        // the lane's node block: its own node's, or the shifted one
        atomicSub(&agg[gq[r] * Q * kS + (int)(e & 7) * kS + (B.o.nic(r, m) & kstar)], (int32_t)x);
      }
    }
  };

  while (err == 0 && rem != 0) {
    if (__builtin_expect(K >= P.k_max, 0)) {
      err = VP_ERR_CAPACITY;
      break;
    }
    VP_STAMP(0);
    // Step 1: this wavefront's sets, then its patterns.  The A part of the
    // first pattern does not wait for the sets.
    int32_t a0[8];
#pragma unroll
    for (int m = 0; m < 8; ++m) a0[m] = *row_of(irow, m);
    if (kprev != 0 && ns > 0) {
      // a set's best shift changes only with the column of the last
      // activation's shift
      if (__builtin_expect(P.held, 1)) {
        if (kprev > 0) {
          // SPT is as many as the loop goes through, so that a lane takes its
          // own shifts only: a copy of the next lane's would win a tie against
          // a lower one there (an idle lane's sums are not used)
          const int u0 = kprev - k0;
          const int32_t s = shift_sum(kprev);
#pragma unroll
          for (int u = 0; u < kHeldShifts; ++u) {
            if ((u == 2 || u == 4) && u >= SPT) break;   // uniform
            held[u] = u0 == u ? s : held[u];
          }
        }
        // sums are never negative; a strict gain keeps the lowest of equal shifts
        int32_t bv = held[0];
        int bk = k0;
#pragma unroll
        for (int u = 1; u < kHeldShifts; ++u) {
          if ((u == 2 || u == 4) && u >= SPT) break;
          bk = held[u] > bv ? k0 + u : bk;
          bv = max(bv, held[u]);
        }
        // the lanes of a set are neighbours
        // and in shift order: of equals the lower lane's stays
        auto take = [&](int32_t v2, int k2, int o) {
          bk = v2 + ((lane & o) != 0 ? 1 : 0) > bv ? k2 : bk;
          bv = max(bv, v2);
        };
        if (LPS >= 2) take((int32_t)quad_xor<1>((uint32_t)bv), (int)quad_xor<1>((uint32_t)bk), 1);
        if (LPS >= 4) take((int32_t)quad_xor<2>((uint32_t)bv), (int)quad_xor<2>((uint32_t)bk), 2);
        for (int o = 4; o < LPS; o <<= 1) take(__shfl_xor(bv, o), __shfl_xor(bk, o), o);
        if (has_set && (lane & (LPS - 1)) == 0) rb[my_set] = make_uint2((uint32_t)bv, (uint32_t)bk);
      } else {
        // more sets or shifts than the registers hold: every sum again
        for (int x0 = 0; x0 < ns << P.LPS_log2; x0 += 64) {
          const int x = x0 + lane;
          const bool in = x < ns << P.LPS_log2;
          const int si = sb + (in ? x >> P.LPS_log2 : 0), c0 = 1 + (x & (LPS - 1)) * P.SPT;
          const int c1 = min(nn, c0 + P.SPT);
          const uint4 o4 = set_rows[si];
          int32_t bv = -1;
          int bk = 0;
          for (int k = c0; k < c1; ++k) {
            int32_t s = 0;
#pragma unroll
            for (int m = 0; m < 8; ++m) s += row_of(o4, m)[k];
            if (s > bv) {
              bv = s;
              bk = k;
            }
          }
          for (int o = 1; o < LPS; o <<= 1) {
            const int32_t v2 = __shfl_xor(bv, o);
            const int k2 = __shfl_xor(bk, o);
            if (v2 > bv || (v2 == bv && k2 < bk)) {
              bv = v2;
              bk = k2;
            }
          }
          if (in && (x & (LPS - 1)) == 0) rb[si] = make_uint2((uint32_t)bv, (uint32_t)bk);
        }
      }
      wave_sync();
    }
    VP_STAMP(1);
    {
      // candidate of a pattern: {score, shape code, payload}, compared by
      // score, then by the lower code
      const uint2 r = rb[info0.x >> 16];
      uint32_t sc = (uint32_t)(a0[0] + a0[1] + a0[2] + a0[3] + a0[4] + a0[5] + a0[6] + a0[7]);
      if (__builtin_expect(RW8 > 1, 0))
        for (int m = 1; m < RW8; ++m) {
          const uint4 t = rows[min(ib + lane, L.J0 + L.J1 - 1) * RW8 + m];
#pragma unroll
          for (int x = 0; x < 8; ++x) sc += (uint32_t)row_of(t, x)[0];
        }
      uint32_t code = (r.y << 12) | (info0.x & 0xFFFF), pay = info0.y;
      sc = ib + lane < ie ? sc + r.x : 0;
      if (__builtin_expect(nitem > 1, 0)) {
        // a round's rows and sets are asked for one round ahead (cross-socket
        // nodes have five: 4.07 us per activation without, 3.5 with)
        uint4 t_next;
        uint2 inf_next;
        auto fetch_item = [&](int it) {
          const int ic = min(it, ie - 1);
          t_next = rows[ic * RW8];
          inf_next = info[ic];
        };
        fetch_item(ib + lane + 64);
        for (int it = ib + lane + 64; it - lane < ie; it += 64) {
          const uint4 t = t_next;
          const uint2 inf = inf_next, rs = rb[inf.x >> 16];
          int32_t v[8];
#pragma unroll
          for (int x = 0; x < 8; ++x) v[x] = *row_of(t, x);
          fetch_item(it + 64);
          uint32_t s = rs.x + (uint32_t)(v[0] + v[1] + v[2] + v[3] + v[4] + v[5] + v[6] + v[7]);
          for (int m = 1; m < RW8; ++m) {
            const uint4 tm = rows[min(it, ie - 1) * RW8 + m];
#pragma unroll
            for (int x = 0; x < 8; ++x) s += (uint32_t)row_of(tm, x)[0];
          }
          s = it < ie ? s : 0;
          const uint32_t c = (rs.y << 12) | (inf.x & 0xFFFF);
          const bool take = s > sc || (s == sc && c < code);
          sc = take ? s : sc;
          code = take ? c : code;
          pay = take ? inf.y : pay;
        }
      }
      // the wavefront's best, or its equals, to the workgroup's argmax
      if (sc == wave_reduce<OpMax>(sc) && sc != 0)
        atomicMax((unsigned long long*)&sh->key[K & 1],
                  (unsigned long long)sc << 33 | (unsigned long long)(0xFFFFF - code) << 13 | pay);
    }
    VP_STAMP(2);
    // in global memory D^rem has to be complete before it is read again
    if (RL) lds_barrier();
    else __syncthreads();
    VP_STAMP(3);
    const uint64_t key = (uint64_t)lane0((int64_t)sh->key[K & 1]), step_key = (uint64_t)lane0((int64_t)sh->step_key[K & 1]);
    if (__builtin_expect(key == 0, 0)) {
      err = VP_ERR_NO_PROGRESS;
      break;
    }
    // the last activation to the schedule, and the next iteration's argmaxes
    // and shuffle key, on wavefronts that have no run or have ended it
    Lane ahead;
    const bool pending = K > written;
    if (S == 2 && pending && i_first < N) ahead = read_lane_out(i_first, lf_prev);   // its wavefront has a run to do first
    auto between = [&]() {
      if (pending && i_first < N) {
        if (S == 1) ahead = read_lane_out(i_first, lf_prev);
        write_lane(i_first, K - 1, f_prev, ahead);
        for (int i = i_first + kPlanThreads; i < N; i += kPlanThreads) write_lane(i, K - 1, f_prev, read_lane_out(i, lf_prev));
      }
      written = K;
      if (wave == kPlanWaves - 1) {
        const uint64_t k1 = sm_mix((sm_mix(P.seed + kGolden) ^ (uint64_t)(K + 1)) + kGolden);
        if (lane == 0) {
          sh->key[(K + 1) & 1] = 0;
          sh->top[(K + 1) & 1] = 0;
          sh->step_key[(K + 1) & 1] = k1;
        }
      }
    };
    const uint32_t code = 0xFFFFF - ((uint32_t)(key >> 13) & 0xFFFFF);
    const int kstar = (int)(code >> 12), fbase = kstar == 0 ? 0 : (kstar - 1) * L.F1;
    VP_STAMP(4);

    // Steps 2-4 over the shape's families
    uint32_t best_F;
    // (The probability only places the code.  As all but certain it took a
    // further 5 % off 256 ranks, but put 10 % on shapes of many families.)
    const bool one_family = (key & 0x1000) == 0 && (MS || NS <= kSlots);
    if (MG > 1 ? __builtin_expect(one_family, 1) : __builtin_expect_with_probability(one_family, 1, 0.6)) {
      // one family: the first start with the highest score wins, no utility
      // to compare
      const int lf = (int)(key & 0xFFF);
      Binding B;
      uint32_t xp, xn;
      // a slot without a start: with two wavefronts per start it repeats the
      // last one, so that the wavefronts stay in step
      int start = S == 1 ? slot : min(slot, NS - 1);
      if (MS || S == 2 || slot < NS) {
        const uint32_t F = run(B, lf, kstar, fbase, start, step_key, MS, false, xp, xn);
        if constexpr (S == 1) {
          if (lane == 0) atomicMax(&sh->top[K & 1], F << 4 | (uint32_t)(15 - start));   // F < 2^28
        } else if constexpr (!MS) {
          if (lane == 0 && slot < NS) prF[slot * S + part] = (int32_t)F;
        }
      }
      between();
      VP_STAMP(7);
      lds_barrier();
      VP_STAMP(8);
      int best;
      if constexpr (S == 1) {
        const uint32_t top = (uint32_t)lane0((int32_t)sh->top[K & 1]);
        best_F = top >> 4;
        best = 15 - (int)(top & 15);
      } else {
        constexpr int kRow = MS ? kMaxStarts : kSlots;
        const int2 f2 = ((const int2*)prF)[min(lane & (kRow - 1), NS - 1)];
        const uint32_t f = (uint32_t)(f2.x + f2.y);
        // the starts repeat along the rows of sixteen lanes
        uint32_t m = MS ? OpMax::f(f, row_ror<8>(f)) : f;
        if constexpr (MS) m = OpMax::f(m, row_ror<4>(m));
        m = OpMax::f(m, row_ror<2>(m));
        m = OpMax::f(m, row_ror<1>(m));
        best_F = (uint32_t)lane0((int32_t)m);
        best = __builtin_ctzll(__ballot(f == best_F));
      }
      if constexpr (MS) best &= kSlots - 1;   // its slot
      VP_STAMP(9);
      if (best_F != 0 && slot == best) apply(B, kstar);
      lf_prev = lf;
    } else {
      // FC families at a time, one (family, start) run per slot per round.
      // A slot that has run another job since the winner's runs
      // the winner's once more (the same inputs, the same binding).
      const int ip = kstar ? L.J0 + (int)(code & 0xFFF) : (int)code;
      const int lb = lane0(cat[L.off_fb + ip]), nf = lane0(cat[L.off_fe + ip]) - lb;
      bool have = false, redo = false;
      int64_t best_S = 0, best_xm = 0, best_bm = 1;
      int best_c = 0, best_s = 0, best_chunk = 0, win_slot = 0;
      int c0 = 0, nc = min(nf, P.FC), j0 = 0;
      best_F = 0;
      between();
      while (true) {
        int job = redo ? (best_c - best_chunk) * NS + best_s : j0 + slot;
        const bool runs = redo ? slot == win_slot : job < nc * NS;
        // past the chunk's last job a slot repeats it, so that the wavefronts stay in step; the winner's job counts
        // in its own chunk, which may be longer than the last one
        if (S == 2 && !redo) job = min(job, nc * NS - 1);
        const int cj = job / NS;
        int start = job - cj * NS;
        Binding B;
        if (S == 2 || runs) {
          uint32_t xp, xn;
          const uint32_t F = run(B, lb + (redo ? best_chunk : c0) + cj, kstar, fbase, start, step_key, false, true, xp, xn);
          if (lane == 0 && !redo && runs) {
            prF[job * S + part] = (int32_t)F;
            prxp[job * S + part] = (int32_t)xp;
            prxn[job * S + part] = (int32_t)xn;
          }
        }
        bool held_here = redo;
        if (!redo) {
          j0 += kSlots;
          if (j0 < nc * NS) continue;
          lds_barrier();
          // Evaluate (Eq. (9)-(10)): the first start with the highest score
          // of every family, then the best family
          const int64_t unit = sh->unit, lambda = sh->lambda;
          auto score_of = [&](int job) { return S == 1 ? prF[job] : prF[job * S] + prF[job * S + S - 1]; };
          int64_t V = 0, xm = 0, bm = 1;
          int c = -1, bs = 0;
          for (int cc = lane; cc < nc; cc += 64) {
            int32_t F0 = -1;
            int s0 = 0;
            for (int s = 0; s < NS; ++s) {
              const int32_t f = score_of(cc * NS + s);
              if (f > F0) {
                F0 = f;
                s0 = s;
              }
            }
            int64_t xm2 = 0, bm2 = 1;
            for (int cl = 0; cl < 2; ++cl) {
              const int64_t bw = cl ? sh->bw_n : sh->bw_p;
              const int32_t* px = (cl ? prxn : prxp) + (cc * NS + s0) * S;
              const int64_t xc = max(px[0], px[S - 1]);
              if (xc * bm2 > xm2 * bw) {
                xm2 = xc;
                bm2 = bw;
              }
            }
            // Eq. (10) in bytes: served volume and slowest lane
            const int64_t Sb = (int64_t)F0 * unit;
            xm2 *= unit;
            if (c < 0 || utility_greater(Sb, xm2, bm2, V, xm, bm, lambda)) {
              V = Sb;
              xm = xm2;
              bm = bm2;
              c = cc;
              bs = s0;
            }
          }
          // wave argmax under the exact order, ties to the lower family
          // index; lanes past the last family hold none
          for (int off = 1; off < nc; off <<= 1) {
            const int64_t V2 = __shfl_xor(V, off), xm2 = __shfl_xor(xm, off), bm2 = __shfl_xor(bm, off);
            const int c2 = __shfl_xor(c, off), bs2 = __shfl_xor(bs, off);
            bool take = false;
            if (c2 >= 0) {
              if (c < 0) take = true;
              else if (utility_greater(V2, xm2, bm2, V, xm, bm, lambda)) take = true;
              else if (!utility_greater(V, xm, bm, V2, xm2, bm2, lambda) && c2 < c) take = true;
            }
            if (take) {
              V = V2;
              xm = xm2;
              bm = bm2;
              c = c2;
              bs = bs2;
            }
          }
          V = lane0(V);
          xm = lane0(xm);
          bm = lane0(bm);
          c = lane0(c);
          bs = lane0(bs);
          if (!have || utility_greater(V, xm, bm, best_S, best_xm, best_bm, lambda)) {
            have = true;
            best_S = V;
            best_xm = xm;
            best_bm = bm;
            best_c = c0 + c;
            best_s = bs;
            best_chunk = c0;
            best_F = (uint32_t)lane0(score_of(c * NS + bs));
          }
          if (c0 + nc < nf) {
            c0 += nc;
            nc = min(nf - c0, P.FC);
            j0 = 0;
            lds_barrier();   // the next chunk's scores replace these
            continue;
          }
          const int wj = (best_c - best_chunk) * NS + best_s;
          win_slot = wj & (kSlots - 1);
          held_here = best_chunk == c0 && wj >= j0 - kSlots;
        }
        if (held_here) {
          if (best_F != 0 && slot == win_slot) apply(B, kstar);
          break;
        }
        redo = true;
      }
      lf_prev = lb + best_c;
    }
    if (__builtin_expect(best_F == 0, 0)) {
      err = VP_ERR_NO_PROGRESS;
      break;
    }
    rem -= best_F;
    kprev = kstar;
    f_prev = fbase + lf_prev;
    VP_STAMP(10);
    lds_barrier();
    VP_STAMP(11);
    ++K;
  }
  // the last activation; every one before it has been written
  if (K > written) {
    if (!RL) __syncthreads();   // D^rem is complete
    for (int i = i_first; i < N; i += kPlanThreads) write_lane(i, K - 1, f_prev, read_lane_out(i, lf_prev));
  }

  if (tid == 0) {
    P.K[b] = K;
    if (P.tau) P.tau[b] = err == VP_ERR_INVALID_DEMAND ? 0 : tau;
    if (err) atomicCAS(P.status + b, 0, err);
  }
}

size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

template <int g, int MG, bool RL, int S, bool MS>
vp_status launch_s(const PlanArgs& P, size_t lds, hipStream_t st) {
  auto kern = plan_kernel<g, MG, RL, S, MS>;
  if (hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) !=
      hipSuccess)
    return set_error(VP_ERR_HIP, "cannot raise the planner's LDS limit");
  hipLaunchKernelGGL(kern, dim3((unsigned)P.batch), dim3(kPlanThreads), lds, st, P);
  if (hipGetLastError() != hipSuccess) return set_error(VP_ERR_HIP, "planner launch failed");
  return VP_OK;
}

template <int g, int MG, bool RL, int S>
vp_status launch_t(const PlanArgs& P, size_t lds, hipStream_t st) {
  if (P.n_start > kPlanWaves / S) return launch_s<g, MG, RL, S, true>(P, lds, st);
  return launch_s<g, MG, RL, S, false>(P, lds, st);
}

// Wavefronts per (family, start) run (see plan_kernel).  Quads of 65 to 128
// groups with more starts than fit two wavefronts each go back to one: 320
// ranks, 8 and 16 starts 26.7 and 47 us per activation against 30.3 and 56.
// Triples do not (384 ranks 21 against 13 us at 8 starts), nor more groups.
int run_waves(int g, int G, int n_start) {
  if (G <= (g == 2 ? 128 : 64)) return 1;
  return g == 4 && G <= 128 && n_start > kPlanWaves / 2 ? 1 : 2;
}

template <int g>
vp_status launch_g(const PlanArgs& P, size_t lds, hipStream_t st, bool res_lds) {
  const int G = P.L.G;
  if (G <= 64) return res_lds ? launch_t<g, 1, true, 1>(P, lds, st) : launch_t<g, 1, false, 1>(P, lds, st);
  if (G <= 128 && run_waves(g, G, P.n_start) == 1) {
    if constexpr (g != 3) return res_lds ? launch_t<g, 2, true, 1>(P, lds, st) : launch_t<g, 2, false, 1>(P, lds, st);
  }
  if constexpr (g != 2) {
    if (G <= 128) return res_lds ? launch_t<g, 1, true, 2>(P, lds, st) : launch_t<g, 1, false, 2>(P, lds, st);
  }
  if (G <= 256) return launch_t<g, 2, false, 2>(P, lds, st);
  if constexpr (g < 4) return launch_t<g, 4, false, 2>(P, lds, st);
  return set_error(VP_ERR_UNSUPPORTED, "too many rank groups");
}

}  // namespace

// ------------------------------------------------- library-owned residual

// vp_plan_noalloc keeps the residual D^rem in this array instead of a
// caller's workspace: one copy per device, held until the process ends,
// room for kStaticRanks ranks.  Host code never passes the array's name to
// a kernel: it passes the device address looked up below.
static __device__ __align__(256) int64_t scratch[(size_t)kStaticRanks * kStaticRanks];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_addr[kMaxDevices] = {};
}  // namespace

vp_status static_residual(int32_t n_ranks, void** out) {
  if (n_ranks < 1 || n_ranks > kStaticRanks)
    return set_error(VP_ERR_UNSUPPORTED, "vp_plan_noalloc plans at most " + std::to_string(kStaticRanks) +
                                             " ranks (its residual is a fixed device array)");
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return set_error(VP_ERR_HIP, "hipGetDevice failed");
  if (dev < 0 || dev >= kMaxDevices) return set_error(VP_ERR_UNSUPPORTED, "device index too large");
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_addr[dev]) {
    // once per device, with that device current: its copy's address
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || p == nullptr)
      return set_error(VP_ERR_HIP, std::string("hipGetSymbolAddress of the static residual failed: ") +
                                       hipGetErrorString(e));
    g_scratch_addr[dev] = p;
  }
  *out = g_scratch_addr[dev];
  return VP_OK;
}

namespace {

// The library's limit on catalogs, in bytes to be held against one workgroup's
// LDS: a measure of patterns, families, NIC-lane sets, ranks and starts, fixed
// so that the catalogs taken do not change with the kernel's layout.  What the
// kernel lays out (launch_plan) stays below it: of one pattern 2 Q g + 22 bytes
// at most against 2 Q g + 28 here, its only family included.
size_t catalog_measure(const DevCatalogLayout& L, int n_start) {
  const size_t pairs = (size_t)((L.TS + 7) & ~7);   // slot pairs of a pattern
  const size_t patterns = (size_t)(L.J0 + L.J1), families = (size_t)(L.F0 + L.F1);
  const size_t N = (size_t)L.N, starts = (size_t)n_start;
  const size_t lane_groups = L.G <= 64 ? 64 : L.G <= 128 ? 128 : L.G <= 256 ? 256 : 512;
  size_t sum = 0;
  for (size_t x : {112 + 35 * lane_groups * (size_t)L.g, (size_t)((L.nn + 3) | 1) * (size_t)(L.Q * L.Q + 1) * 4,
                   patterns * pairs * 2, patterns * 8, patterns * 4, families * (size_t)(L.Q * L.g) * 2,
                   (size_t)L.nS * kMaxRTerms * 2, (size_t)L.nS * 8, (size_t)L.J1 * 2, starts * 24,
                   2 * align_up(N * 2, 16), 3 * align_up(N, 16), 2 * N * (size_t)((L.g * L.g) | 1) * 4,
                   2 * align_up(starts * N, 16), (size_t)16, starts * (size_t)L.G * 2})
    sum += align_up(x, 16);
  return sum;
}

}  // namespace

vp_status launch_plan(const PlanLaunch& a, void* stream) {
  const vp_catalog& c = *a.cat;
  const DevCatalogLayout& L = c.lay;
  const int N = L.N, g = L.g, NS = a.p.n_start;
  const int QG = L.Q * g;
  if (L.J0 > 4095 || L.J1 > 4095 || L.nn > 255) return set_error(VP_ERR_UNSUPPORTED, "catalog too large");
  if (QG > kMaxQG || L.Q > 8 || g > 4) return set_error(VP_ERR_UNSUPPORTED, "too many lanes per node");
  if (N > 65535 || L.G > 64 * 8) return set_error(VP_ERR_UNSUPPORTED, "too many ranks for the planner");
  if (L.n_inst > 256) return set_error(VP_ERR_UNSUPPORTED, "too many node-local instances");
  // the kernel addresses one matrix's schedule with 32-bit byte offsets
  if ((uint64_t)a.p.k_max * (uint64_t)N * 8 >= (uint64_t(1) << 32))
    return set_error(VP_ERR_UNSUPPORTED, "k_max * N too large for the planner");
  if (L.MLT > kMaxLTerms) return set_error(VP_ERR_UNSUPPORTED, "too many intra-node lane classes");
  if (L.MRT > kMaxRTerms) return set_error(VP_ERR_UNSUPPORTED, "too many NIC lanes in one pattern");

  PlanArgs P{};
  P.cat = (const int32_t*)c.dev;
  P.L = L;
  P.D = a.demand;
  P.Drem = a.drem;
  P.k_target = a.p.k_target;
  P.lambda = a.p.lambda_ns;
  P.unit = a.p.unit_bytes;
  P.seed = a.p.seed;
  // divisibility by unit = 2^s * odd: low s bits clear and (v >> s) * odd^-1 <= (2^64-1)/odd
  uint64_t u = (uint64_t)a.p.unit_bytes;
  int s = 0;
  while (!(u & 1)) {
    u >>= 1;
    ++s;
  }
  uint64_t inv = u;
  for (int it = 0; it < 6; ++it) inv *= 2 - u * inv;
  P.unit_shift = s;
  P.odd_inv = inv;
  P.odd_lim = ~uint64_t(0) / u;
  P.n_start = NS;
  P.MRT = L.MRT;
  P.i_aa = a.p.i_aa;
  P.k_max = a.p.k_max;
  P.K = a.K;
  P.family = a.family;
  P.dst = a.dst;
  P.inst = a.inst;
  P.bytes = a.bytes;
  P.tau = a.tau;
  P.send_off = a.send_off;
  P.stream_off = a.stream_off;
  P.recv_src = a.recv_src;
  P.status = a.status;
  P.batch = a.batch;
  // Lanes per NIC-lane set (a power of two) and shifts per lane: up to four
  // lanes, a quad, combine by two cheap steps, so the shifts of a set go to a
  // quad where the wavefront has room, to more lanes only beyond eight shifts
  // each.  Held shifts per lane are two, four or eight, as many as the kernel's
  // loops over them run; the last lanes may hold none.  Sets that then do not
  // fit a wavefront's 64 lanes are summed again in every iteration.
  {
    const int shifts = std::max(1, L.nn - 1), sets = std::max(1, L.max_sets);
    int lg = 0;
    while (lg < 6 && (kHeldShifts << lg) < shifts) ++lg;
    while (lg < 2 && (2 << lg) * sets <= 64 && (2 << lg) <= shifts) ++lg;
    P.LPS_log2 = lg;
    int spt = (shifts + (1 << lg) - 1) >> lg;
    P.held = (sets << lg) <= 64 && spt <= kHeldShifts;
    P.SPT = !P.held ? spt : spt <= 2 ? 2 : spt <= 4 ? 4 : kHeldShifts;
  }

  int dev = 0;
  size_t budget = 0;
  const vp_status ds = device_lds(&dev, &budget);
  if (ds != VP_OK) return ds;
  if (catalog_measure(L, NS) > budget)
    return set_error(VP_ERR_UNSUPPORTED, "catalog beyond the planner's limit (its size measure exceeds one workgroup's LDS)");
  P.FC = std::min(L.hmax, kFamChunk);
  size_t o = align_up(sizeof(Shared), 16);
  auto take = [&](int32_t* field, size_t bytes) {
    *field = (int32_t)o;
    o = align_up(o + bytes, 16);
  };
  take(&P.o_agg, (size_t)L.kS * (L.Q * L.Q + 1) * 4);
  take(&P.o_rb, (size_t)(L.nS + 1) * 8);
  const int parts = run_waves(g, L.G, NS);
  take(&P.o_pr, (size_t)P.FC * NS * parts * 12);
  take(&P.o_xw, parts == 1 ? 0 : (size_t)kPlanWaves / 2 * 256 * 4);
  take(&P.o_out, (size_t)N * 8);
  take(&P.o_sacc, (size_t)N * 8);
  // The residual goes to LDS before the family records: a run reads four or
  // more blocks of the one per lane and a single record of the other, and a
  // global residual also has to be waited for after every update.
  const size_t rw = g == 2 ? 4 : g == 3 ? 12 : 16;
  const size_t res = (size_t)L.G * L.G * rw * 4;
  const bool res_lds = L.G <= 128 && align_up(o + L.pl_recs, 16) + res <= budget;
  P.rec_lds = align_up(o + L.pl_end, 16) + (res_lds ? res : 0) <= budget;
  take(&P.o_tab, P.rec_lds ? L.pl_end : L.pl_recs);
  take(&P.o_res, res_lds ? res : 0);
  if (o > budget) return set_error(VP_ERR_UNSUPPORTED, "plan state does not fit in LDS");

  hipStream_t st = (hipStream_t)stream;
  switch (g) {
    case 2: return launch_g<2>(P, o, st, res_lds);
    case 3: return launch_g<3>(P, o, st, res_lds);
    case 4: return launch_g<4>(P, o, st, res_lds);
  }
  return set_error(VP_ERR_UNSUPPORTED, "gpus_per_switch must be 2, 3 or 4");
}

}  // namespace vp

#ifdef VP_PHASE_STAMPS
// Reader of the phase stamps of the last plan (stamped builds only).
extern "C" int vp_phase_stamps_read(unsigned long long* out) {
  return (int)hipMemcpyFromSymbol(out, HIP_SYMBOL(vp::g_phase_stamps), sizeof(unsigned long long) * 4096 * 16);
}
#endif
