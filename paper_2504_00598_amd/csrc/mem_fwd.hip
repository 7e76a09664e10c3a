// Search under a memory budget (Sec. 4.4: least Eq. T cost with Eq. M within
// the memory limit, memory quantised into buckets):
//     D[0][s][m] = c[0][s]                                   if mem[0][s] <= m
//     D[i][s][m] = c[i][s] + min_t D[i-1][t][m - mem[i][s]] + R_{e(i)}[t][s]
// with D = +inf where m < mem[i][s]; the answer is min_s D[N-1][s][budget].
// D[i][s][m] is the least cost of a prefix whose memory total is at most m,
// so it does not increase with m.
//
// Product then shift.  A state s with memory shift d = mem[i][s] takes its
// candidates from column m - d, so
//     D[i][s][m] = c[i][s] + P[s][m - d],   P[s][m'] = min_t D[i-1][t][m'] + R[t][s]:
// a step is one min-plus product of the previous rows (buckets x states) with
// the K x K table, followed by a per-state shift of the product along m.
//
// Layout.  The buckets of a search are cut into chunks of 64; one workgroup
// computes one chunk for all states with four compute waves, a loading wave
// and a storing wave (the compute waves issue no global stores, so none of
// their waits for a load ever covers a store).  Compute wave w owns buckets
// 16w .. 16w+15 of its chunk, lane (g, m) = (lane / 16, lane % 16) the bucket
// 16w + m and the K/4 states g K/4 .. g K/4 + K/4 - 1.  The previous row of a
// bucket sits in registers (32 predecessors at a time), and the table entry
// R[t][s] of predecessor t = 16q + j reaches every lane of a row of 16 through
// a DPP row broadcast of lane j of a register that holds R[16q .. 16q+15][s]
// in that row: a candidate is one add with a DPP operand, two candidates one
// three-input minimum.  The tables stream from the L2 cache, each lane loading
// the 16 entries of its row's state, a few items ahead.
// Step i of bucket m reads products at m - d >= m - 16, i.e. of the wave below
// (through a product buffer in LDS) or, for wave 0, of the top 16 buckets of
// the chunk below, which that chunk's storing wave passes through a ring of
// eight slots in device memory together with its offsets.  The loading wave
// fetches the slots and stages the next step's per-state records (and, for
// K <= 64, the step's table) in LDS; the storing wave writes the ring slots,
// the publication counter and the argmin bytes of earlier steps.  Every ring word carries
// the number of its step in its upper half, so no store is ever waited for:
// the chunk above loads a slot ahead of the step that needs it and reloads it
// until every word has the step's number; a chunk waits before
// reusing a slot until the chunk above has consumed it (all waits bounded).
// The chunks of one launch are resident together (the host launches the
// searches in rounds that fit), so the ring stays in the L2 cache.
//
// Arithmetic.  Bucket m carries an exact int64 offset o[m] = min_s D[s][m];
// the row is kept as Q[s][m] = min(D[s][m] - o[m], QCAP) << b with
// QCAP = 2^(31-b) and b index bits, and the packed table words as
// (R << b) | t with R < 2^(31-b), so a candidate Q + R never leaves 32 bits
// and one unsigned minimum yields the value and the lowest argmin.  The best
// candidate of a column with a finite offset is at most R_max < QCAP (through
// the column's minimum state), so capped states never win.
// The new value of state s at bucket m is, relative to the offset
// o[m - dmin] of the least shift dmin over the block's available states,
//     y[s] = c[s] + P[s][m - d] + (o[m - d] - o[m - dmin]),
// where the bracket is >= 0 because o does not increase with m.  A state with
// shift dmin has y < 2^31 + R_max, so y is computed in saturating 32-bit
// arithmetic: the column minimum cm = min_s y[s] is exact, the new offset is
// o[m - dmin] + cm, and a saturated y exceeds cm by more than QCAP.
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "cfp_internal.h"
#include "common.h"

namespace cfp {

constexpr int kMemChunk = 64;        // buckets per workgroup
constexpr int kMemShift = 16;        // largest supported mem entry = halo width = buckets per wave
constexpr int kMemBlocks = 4;        // bucket blocks of 16 per chunk
constexpr int kMemSlots = 8;         // ring slots per chunk
constexpr int kMemFlagStride = 16;   // ints per chunk flag (one 64-byte line each)
constexpr int kMemMaxK = 256;
constexpr int kMemPD = 4;            // table items loaded ahead
// Ring slot of KP states: the top 16 buckets' products of all states, then
// their offsets as two halves, every word tagged with its step.
constexpr int mem_slot_words(int kp) { return 16 * kp + 32; }
constexpr int64_t kOffInf = (int64_t)1 << 62;
constexpr int kSpinLimit = 1 << 20;

enum { MEMF_TIMEOUT = 2 };

template <int KP>
struct MemShape {
  static constexpr int BITS = KP <= 32 ? 5 : KP <= 64 ? 6 : KP <= 128 ? 7 : 8;
  static constexpr bool ALIAS = KP > 128;   // rows kept in the product buffer, single-buffered
  static constexpr int CW = kMemBlocks;     // compute waves, one per bucket block
  static constexpr int THREADS = 64 * (CW + 2);    // and a loading and a storing wave
  static constexpr int SPL = KP / 4;        // states per lane
  static constexpr int TB = KP / 32;        // blocks of 32 predecessors
  static constexpr bool HALF = KP % 32 != 0;       // and one of 16 at the end
  static constexpr int NB = SPL % 8 ? 4 : 8;       // states per turn of phase B
  static constexpr bool RLDS = KP <= 64;    // tables staged in LDS by the loading wave
  static constexpr int SP = kMemShift + kMemChunk + 1;  // product buffer row stride (words)
  static constexpr int QS = KP + 4;         // row stride of a wave's rows (words)
  static constexpr uint32_t QCAP = 1u << (31 - BITS);
  static constexpr uint32_t MASK = (1u << BITS) - 1u;
  static_assert(SPL % kMemPD == 0 && SPL % 4 == 0 && SPL % 2 == 0, "items and record words per lane");
};

// Padded states: multiples of 16 up to 128, where the products' K^2 cost of the
// padding is the larger part of a step (45 states as 48 instead of 64: 57%).
static int mem_kp(int k) { return k <= 128 ? (k + 15) / 16 * 16 : k <= 192 ? 192 : 256; }
static int mem_bits(int k) { return k <= 32 ? 5 : k <= 64 ? 6 : k <= 128 ? 7 : 8; }

struct MemWs {
  uint32_t *cst;       // [B][N][KP]
  uint8_t *dsh;        // [B][N][KP]
  int32_t *dmin;       // [B][N]
  uint32_t *rT;        // [E][KP][KP]
  int32_t *mflags;     // [B]: MEMF_TIMEOUT
  uint8_t *rowbad;     // [B][N]: a value of this row is out of range (row 0: or the budget)
  int32_t *rbad;       // range flags of R, one per workgroup of the first launch
  int32_t *cons;       // [B][nchunk] (stride kMemFlagStride): last step whose slot a chunk has consumed
  uint64_t *ring;      // [B][nchunk][kMemSlots][mem_slot_words(KP)]: word | step << 32
  int nchunk;
};

struct MemPrepArgs {
  const int32_t *cost, *rtab;
  const uint8_t *mem;
  int32_t *budget;      // [B]; written (M - 1) where fill is set, else checked
  bool fill;
  int N, K, KP, M, B, E, bits;
  int32_t rlimit;
  MemWs w;
  size_t nring;
  int nflag;
  uint8_t *mem_copy;
  EdgeMap em;
  int32_t *redge;
};
constexpr int kMemPrepBlocks = 1024;  // most workgroups of the first launch

// The first launch of a call (three of their own, a budget fill and an upload of
// the header took 20 us more):
//   * stamps every ring word with an impossible step number, so that nothing a
//     previous call left in the workspace is taken for a fresh slot, marks every
//     slot as consumed before step 0 and clears the flags;
//   * writes out a periodic edge map, and the budgets of a frontier call;
//   * packs the tables, state-major: rT[e][s][t] = (R[e][t][s] << b) | t.  A
//     padding predecessor or state gets ((QCAP - 1) << b) | t: with the capped row
//     value QCAP its candidate is the largest value that fits, above every
//     candidate through a column's minimum state.  Every R entry is read here, so
//     the range check (entries in [0, 2^(31-b))) is made on the way;
//   * per-(search, block) records, one wave per row: cost cst[s] (kSat for an
//     unavailable or padding state), shift dsh[s], the least shift dmin over the
//     available states; a copy of mem for the traceback; validation of mem, the
//     costs and the budget.
__global__ __launch_bounds__(256) void mem_prep_kernel(MemPrepArgs a) {
  const int lane = threadIdx.x & 63, N = a.N, K = a.K, KP = a.KP;
  const size_t stride = (size_t)gridDim.x * blockDim.x, first = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  for (size_t x = first; x < a.nring; x += stride) a.w.ring[x] = ~0ull;
  for (size_t x = first; x < (size_t)a.nflag; x += stride) a.w.cons[x] = -1;
  for (size_t x = first; x < (size_t)a.B; x += stride) {
    a.w.mflags[x] = 0;
    if (a.fill) a.budget[x] = a.M - 1;
  }
  a.em.write(a.redge, N);
  const size_t total = (size_t)a.E * KP * KP;
  const uint32_t pad = (((1u << (31 - a.bits)) - 1u) << a.bits);
  bool off = false;
  for (size_t x = first; x < total; x += stride) {
    const int t = (int)(x % KP), s = (int)((x / KP) % KP), e = (int)(x / ((size_t)KP * KP));
    uint32_t v = pad | (uint32_t)t;
    if (s < K && t < K) {
      const int32_t r = a.rtab[((size_t)e * K + t) * K + s];
      off |= r < 0 || r >= a.rlimit;
      v = ((uint32_t)r << a.bits) | (uint32_t)t;
    }
    a.w.rT[x] = v;
  }
  const int any = __syncthreads_or(off);
  if (threadIdx.x == 0) a.w.rbad[blockIdx.x] = any ? 1 : 0;
  for (size_t row = (size_t)blockIdx.x * 4 + (threadIdx.x >> 6); row < (size_t)a.B * N; row += (size_t)gridDim.x * 4) {
    const size_t base = row * K;
    bool bad = false;
    int dm = kMemShift + 1;
    for (int s = lane; s < KP; s += 64) {
      uint32_t c = kSat;
      int d = 0;
      if (s < K) {
        d = a.mem[base + s];
        const int32_t cv = a.cost[base + s];
        a.mem_copy[base + s] = (uint8_t)d;
        bad |= d >= a.M || d > kMemShift || cv < 0;
        if (d > kMemShift) d = kMemShift;
        if (cv >= 0 && cv != CFP_COST_INF) {
          c = (uint32_t)cv;
          dm = min(dm, d);
        }
      }
      a.w.cst[row * KP + s] = c;
      a.w.dsh[row * KP + s] = (uint8_t)d;
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) dm = min(dm, __shfl_xor(dm, o, 64));
    if (!a.fill && row % N == 0) {
      const int32_t bud = a.budget[row / N];
      bad |= bud < 0 || bud >= a.M;
    }
    const bool rb = __any(bad);
    if (lane == 0) {
      a.w.dmin[row] = dm > kMemShift ? 0 : dm;  // a block with no available state: every y saturates
      a.w.rowbad[row] = rb;
    }
  }
}

struct MemArgs {
  const int32_t *budget;
  MemWs w;
  int N, K, M, B;
  int b0, nb, B8;        // searches b0 .. b0+nb-1 of this launch; grid = nchunk * B8
  uint8_t *table;        // [B][N][K][MS]
  int MS;                // bucket stride of the table
  SearchResult *res;
  int nbad;              // words of w.rbad
  int64_t *opt;
  int32_t *status;
  int64_t *frontier;     // [B][M] or null
};

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// a = min(a, ra[j] + q_j) and b = min(b, rb[j] + q_j) for predecessors
// j = J0 .. J0+3 of a row of 16, where r[j] is lane j of r's row (a DPP row
// broadcast): two states at once, so that no instruction needs the result of
// the one before it (a wave alone on its SIMD would otherwise wait for it).
// NOP: the first block reading ra and rb, which waits the two states a DPP
// read of a fresh VALU result needs.
#define CFP_M_ADD(T, R, Q, J) "v_add_u32_dpp " T ", " R ", " Q " row_newbcast:" J " row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
template <int J0, bool NOP>
__device__ __forceinline__ void mcand4x2(uint32_t &a, uint32_t &b, uint32_t ra, uint32_t rb, uint32_t q0, uint32_t q1,
                                         uint32_t q2, uint32_t q3) {
  uint32_t t0, t1, t2, t3;
  asm(".if %[nop]\n s_nop 1\n .endif\n"
      CFP_M_ADD("%[t0]", "%[ra]", "%[q0]", "%[j0]")
      CFP_M_ADD("%[t1]", "%[ra]", "%[q1]", "%[j1]")
      CFP_M_ADD("%[t2]", "%[rb]", "%[q0]", "%[j0]")
      CFP_M_ADD("%[t3]", "%[rb]", "%[q1]", "%[j1]")
      "v_min3_u32 %[a], %[a], %[t0], %[t1]\n"
      "v_min3_u32 %[b], %[b], %[t2], %[t3]\n"
      CFP_M_ADD("%[t0]", "%[ra]", "%[q2]", "%[j2]")
      CFP_M_ADD("%[t1]", "%[ra]", "%[q3]", "%[j3]")
      CFP_M_ADD("%[t2]", "%[rb]", "%[q2]", "%[j2]")
      CFP_M_ADD("%[t3]", "%[rb]", "%[q3]", "%[j3]")
      "v_min3_u32 %[a], %[a], %[t0], %[t1]\n"
      "v_min3_u32 %[b], %[b], %[t2], %[t3]\n"
      : [a] "+v"(a), [b] "+v"(b), [t0] "=&v"(t0), [t1] "=&v"(t1), [t2] "=&v"(t2), [t3] "=&v"(t3)
      : [ra] "v"(ra), [rb] "v"(rb), [q0] "v"(q0), [q1] "v"(q1), [q2] "v"(q2), [q3] "v"(q3), [j0] "i"(J0),
        [j1] "i"(J0 + 1), [j2] "i"(J0 + 2), [j3] "i"(J0 + 3), [nop] "i"(NOP ? 1 : 0));
}
#undef CFP_M_ADD

// Minimum over the four rows of a wave (lanes m, m+16, m+32, m+48); every
// lane gets its bucket's minimum.
__device__ __forceinline__ uint32_t rows_min(uint32_t x) {
  const auto h = __builtin_amdgcn_permlane32_swap(x, x, false, false);
  const uint32_t z = umin(h[0], h[1]);
  const auto q = __builtin_amdgcn_permlane16_swap(z, z, false, false);
  return umin(q[0], q[1]);
}

__device__ __forceinline__ bool spin_until(const int32_t *flag, int target, int &seen) {
  int spins = 0;
  while (seen < target) {
    if (++spins > kSpinLimit) return false;
    __builtin_amdgcn_s_sleep(1);
    seen = __hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  return true;
}

// Work split.  Compute wave w owns bucket block w of the chunk (buckets
// 16w .. 16w+15); its lane (g, m) has bucket 16w + m and the K/4 states of row
// g.  (Two waves per block, each with half of the states, were measured
// slower: the products already keep a SIMD's vector unit busy, and the pair
// costs two more barriers per step.)  Of the two I/O waves one does
// every global load of a step (the chunk below's top products into the halo
// columns, the next steps' tables and records into LDS) and one every global
// store (the chunk's top products to the ring for the chunk above, the argmin
// bytes to the table).  Loads and stores of one wave complete in order, so a
// wave that both stored and loaded would wait for its stores whenever it
// needed a load; the compute waves issue no global stores at all and, when
// the tables fit in LDS (K <= 64), no global loads either.
//
// Barriers of step i (P_i: products of step i, o_i: offsets after step i):
//   compute: products from Q_{i-1} and the table of step i -> P_i      | B
//            shifted products, offset gaps, bucket minima -> Q_i, o_i,
//            argmin bytes of step i (K > 128: the rows overwrite the
//            products, after a second barrier B2)
//   I/O, between the previous step's last barrier and B: halo of step i
//            (slot i of the chunk below: P_i and o_{i-1} of its top
//            buckets), table and records of step i+1, slot i-1 of this
//            chunk (P_{i-1}, o_{i-2}), argmin bytes of step i-2 (K > 128:
//            of step i-1, and slot i between B and B2, before the rows
//            overwrite P_i).
// The edge map and the least shifts are read through restrict-qualified
// arguments, so that their uniform per-step loads are scalar loads.
template <int KP>
__global__ __launch_bounds__(MemShape<KP>::THREADS) void mem_fwd_kernel(MemArgs a, const int32_t *__restrict__ redge,
                                                                        const int32_t *__restrict__ dmin) {
  using S = MemShape<KP>;
  constexpr int BITS = S::BITS, SPL = S::SPL, TB = S::TB, H = kMemShift, C = kMemChunk, SP = S::SP;
  constexpr uint32_t QCAP = S::QCAP;
  constexpr bool ALIAS = S::ALIAS, RLDS = S::RLDS;
  constexpr int CW = S::CW;
  constexpr int FL = ALIAS ? 1 : 2;  // the argmin bytes of step t are written back during step t + FL
  constexpr int NPB = ALIAS ? 1 : 2;
  constexpr int PD = kMemPD;
  constexpr int NBK = kMemBlocks;

  __shared__ uint32_t Pb[NPB][KP][SP];                                         // products (and, ALIAS, rows)
  __shared__ __align__(16) uint32_t Qw[ALIAS ? 1 : NBK][ALIAS ? 1 : 16][ALIAS ? 4 : S::QS];  // rows
  __shared__ int64_t offs[2][H + C];                                           // offsets by step parity
  __shared__ __align__(16) uint8_t argb[2][NBK][KP][16];                       // argmin bytes by step parity
  __shared__ __align__(16) uint32_t rbuf[RLDS ? 2 : 1][RLDS ? KP : 1][RLDS ? KP : 4];  // tables by step parity
  __shared__ __align__(16) uint32_t rcost[2][KP];                             // records by step parity
  __shared__ __align__(16) uint8_t rshift[2][KP];
  __shared__ int rdmin[2];
  __shared__ int s_timeout;
  __shared__ int s_done;    // last step whose halo slot was taken (loading wave -> storing wave)
  __shared__ int s_upcons;  // progress of the chunk above, as last read by the loading wave

  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool io = w >= CW;
  const int blk = w;  // compute waves: bucket block
  const int g = lane >> 4, m = lane & 15;
  const int col = H + 16 * blk + m;  // compute waves: this lane's column

  const int bl = blockIdx.x % a.B8, j = blockIdx.x / a.B8;
  if (bl >= a.nb) return;
  const int b = a.b0 + bl;
  const int N = a.N, K = a.K, M = a.M;
  const int m0 = j * C;
  const int bucket = m0 + 16 * blk + m;
  const MemWs &W = a.w;

  bool rowbad = false;  // flags of the first launch
  for (int x = tid; x < N; x += S::THREADS) rowbad |= W.rowbad[(size_t)b * N + x] != 0;
  if (__syncthreads_or(rowbad)) {
    if (a.frontier && !io && g == 0 && bucket < M) a.frontier[(size_t)b * M + bucket] = INT64_MAX;
    if (j == 0 && tid == 0) {
      a.status[b] = CFP_ST_BADINPUT;
      a.opt[b] = INT64_MAX;
      a.res[b].final_state = -1;
      a.res[b].status = CFP_ST_BADINPUT;
      a.res[b].final_m = -1;
    }
    return;
  }
  const int Bb = a.budget[b];
  const int top = min(Bb, M - 1);
  if (m0 > top) return;  // no bucket of this chunk is within the budget
  const bool has_consumer = m0 + C <= top;
  const bool consumer = j > 0;
  const size_t chunk_id = (size_t)b * W.nchunk + j;
  const size_t rowbase = (size_t)b * N;
  if (tid == 0) s_timeout = 0;


  if (io) {
    // ------------------------------------------------------------ I/O waves --
    const bool loader = w == CW;
    const size_t lo_id = consumer ? chunk_id - 1 : chunk_id;
    const size_t up_id = has_consumer ? chunk_id + 1 : chunk_id;
    int32_t *my_cons = W.cons + chunk_id * kMemFlagStride;
    const int32_t *up_cons = W.cons + up_id * kMemFlagStride;
    constexpr int SW = mem_slot_words(KP);
    uint64_t *my_ring = W.ring + chunk_id * kMemSlots * SW;
    const uint64_t *lo_ring = W.ring + lo_id * kMemSlots * SW;
    constexpr int HW = KP * 16 / 64;       // product words of a slot per lane
    constexpr int HB = HW <= 24 ? HW : HW % 16 ? HW / 2 : 16;  // words per lane in flight at once
    static_assert(HW % HB == 0, "slot words per lane in whole blocks");
    constexpr int RW = RLDS ? KP * KP / 256 : 1;  // 16-byte table pieces per lane
    bool timeout = false;

    if (loader) {
      u32x4 rv[RW];
      auto load_table = [&](int e) __attribute__((always_inline)) {
        if constexpr (RLDS) {
          const u32x4 *src = (const u32x4 *)(W.rT + (size_t)e * KP * KP);
#pragma unroll
          for (int u = 0; u < RW; ++u) rv[u] = src[lane + 64 * u];
        }
      };
      auto store_table = [&](int par) __attribute__((always_inline)) {
        if constexpr (RLDS) {
#pragma unroll
          for (int u = 0; u < RW; ++u) ((u32x4 *)&rbuf[par][0][0])[lane + 64 * u] = rv[u];
        }
      };
      // records of step t into parity buffer t & 1: KP costs and KP shift bytes,
      // four per lane, and the least shift
      auto stage_records = [&](int t, const u32x4 &c4, uint32_t s4, int dmt) __attribute__((always_inline)) {
        if (lane < KP / 4) {
          *(u32x4 *)&rcost[t & 1][4 * lane] = c4;
          *(uint32_t *)&rshift[t & 1][4 * lane] = s4;
        }
        if (lane == 0) rdmin[t & 1] = dmt;
      };
      auto load_records = [&](int t, u32x4 &c4, uint32_t &s4) __attribute__((always_inline)) {
        if (lane < KP / 4) {
          c4 = *(const u32x4 *)(W.cst + (rowbase + t) * KP + 4 * lane);
          s4 = *(const uint32_t *)(W.dsh + (rowbase + t) * KP + 4 * lane);
        }
      };
      if (N > 1) {  // the table and the records of step 1
        if (RLDS) load_table(redge[1]);
        u32x4 c4 = {};
        uint32_t s4 = 0;
        load_records(1, c4, s4);
        if (RLDS) store_table(1);
        stage_records(1, c4, s4, dmin[rowbase + 1]);
      }
      if (lane == 0) {
        s_done = -1;
        s_upcons = -1;
      }
      // Everything a step takes from memory is loaded during the step before it,
      // so that no load's latency is part of a step: the halo slot (in its first
      // HB words per lane; reloaded if it was not there yet), the table and the
      // records of the next step, the progress of the chunk above.  (Loaded and
      // used within the step they bound it where the products are short: 288
      // blocks, K = 16, 1024 buckets, 16 searches 442 us per call, now 301; from K = 32
      // on the products cover it.)
      uint64_t hv[HB], ho = 0;
      u32x4 cpc = {};  // records of the next step
      uint32_t spc = 0;
      int dmi = 0, upc = -1;
      auto load_block = [&](const uint64_t *src, int u0) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < HB; ++u)
          hv[u] = __hip_atomic_load(src + lane + 64 * (u0 + u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (u0 == 0 && lane < 32)
          ho = __hip_atomic_load(src + 16 * KP + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      };
      auto prefetch = [&](int i) __attribute__((always_inline)) {  // for step i: its halo, what it stages for step i + 1
        if (consumer) load_block(lo_ring + (size_t)(i % kMemSlots) * SW, 0);
        if (i + 1 < N) {
          if (RLDS) load_table(redge[i + 1]);
          load_records(i + 1, cpc, spc);
          dmi = dmin[rowbase + i + 1];
        }
        if (has_consumer) upc = __hip_atomic_load(up_cons, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      };
      if (N > 1) prefetch(1);
      __syncthreads();  // step 0 of the compute waves
      for (int i = 1; i < N; ++i) {
        const int par = i & 1, pprev = par ^ 1;
        const int pb = ALIAS ? 0 : par;
        const uint64_t *src = lo_ring + (size_t)(i % kMemSlots) * SW;
        if (lane >= 32) ho = (uint64_t)i << 32;
        auto block_fresh = [&]() __attribute__((always_inline)) {
          bool ok = true;
#pragma unroll
          for (int u = 0; u < HB; ++u) ok &= (uint32_t)(hv[u] >> 32) == (uint32_t)i;
          return ok;
        };
        if (consumer) {  // every word of slot i must carry the step's number (bounded reloads)
          for (int u0 = 0; u0 < HW; u0 += HB) {
            if (u0 > 0) load_block(src, u0);
            bool ok = block_fresh() && (u0 > 0 || (uint32_t)(ho >> 32) == (uint32_t)i);
            if (!__all(ok) && !timeout) {
              int spins = 0;
              do {
                if (++spins > kSpinLimit) {
                  timeout = true;
                  break;
                }
                __builtin_amdgcn_s_sleep(1);
                load_block(src, u0);
                ok = block_fresh() && (u0 > 0 || (uint32_t)(ho >> 32) == (uint32_t)i);
              } while (!__all(ok));
            }
#pragma unroll
            for (int u = 0; u < HB; ++u) {
              const int x = lane + 64 * (u0 + u);
              Pb[pb][x >> 4][x & 15] = (uint32_t)hv[u];
            }
          }
          // offset of halo bucket h from its two halves (lanes 2h and 2h+1)
          const uint32_t other = (uint32_t)__shfl_xor((int)(uint32_t)ho, 1, 64);
          if (lane < 32 && (lane & 1) == 0)
            offs[pprev][lane >> 1] = (int64_t)(((uint64_t)other << 32) | (ho & 0xFFFFFFFFull));
          if (lane == 0) s_done = i;  // published by the storing wave
        }
        if (RLDS && i + 1 < N) store_table(par ^ 1);
        if (i + 1 < N) stage_records(i + 1, cpc, spc, dmi);
        if (lane == 0) s_upcons = upc;
        if (i + 1 < N) prefetch(i + 1);
        __syncthreads();  // B
        if constexpr (ALIAS) __syncthreads();  // B2
      }
      __syncthreads();  // the last step's rows, offsets and argmin bytes
    } else {
      // Slot of step t: word x < 16 KP is the product of state x / 16 at bucket
      // 48 + x % 16, words 16 KP + 2h and +1 the offset of bucket 48 + h.
      auto store_slot = [&](int t, int pbuf, int opar) __attribute__((always_inline)) {
        uint64_t *dst = my_ring + (size_t)(t % kMemSlots) * SW;
        const uint64_t tag = (uint64_t)t << 32;
#pragma unroll
        for (int u = 0; u < HW; ++u) {
          const int x = lane + 64 * u;
          __hip_atomic_store(dst + x, (uint64_t)Pb[pbuf][x >> 4][H + 48 + (x & 15)] | tag, __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
        }
        if (lane < 32) {
          const uint64_t o = (uint64_t)offs[opar][H + 48 + (lane >> 1)];
          __hip_atomic_store(dst + 16 * KP + lane, ((lane & 1) ? (o >> 32) : (o & 0xFFFFFFFFull)) | tag,
                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      };
      // Before slot t is reused, the chunk above must have consumed its previous
      // step: the loading wave's last reading of its progress, else polling.
      auto wait_consumed = [&](int t) __attribute__((always_inline)) {
        if (t < kMemSlots || timeout) return;
        int seen = s_upcons;
        if (seen < t - kMemSlots && !spin_until(up_cons, t - kMemSlots, seen)) timeout = true;
      };
      // Argmin bytes of step t (parity buffer t & 1) to the table, the pieces of
      // 16 buckets that reach into the budget only.
      auto flush = [&](int t) __attribute__((always_inline)) {
        for (int x = lane; x < NBK * K; x += 64) {
          const int bb = x / K, s = x % K;
          if (m0 + 16 * bb > top) continue;
          uint8_t *dst = a.table + ((rowbase + t) * K + s) * (size_t)a.MS + m0 + 16 * bb;
          *(u32x4 *)dst = *(const u32x4 *)&argb[t & 1][bb][s][0];
        }
      };
      int published = -1;
      auto publish = [&]() __attribute__((always_inline)) {
        const int d = s_done;
        if (consumer && d != published) {
          published = d;
          if (lane == 0) __hip_atomic_store(my_cons, d, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      };
      __syncthreads();  // step 0 of the compute waves
      for (int i = 1; i < N; ++i) {
        publish();
        if (!ALIAS && has_consumer && i >= 2) {  // slot i-1: P_{i-1}, o_{i-2}
          wait_consumed(i - 1);
          store_slot(i - 1, (i - 1) & 1, (i - 2) & 1);
        }
        if (i - FL >= 1) flush(i - FL);  // written before the previous step's last barrier
        __syncthreads();  // B
        if constexpr (ALIAS) {  // P_i is overwritten by the rows after B2
          if (has_consumer) {
            wait_consumed(i);
            store_slot(i, 0, (i - 1) & 1);
          }
          __syncthreads();  // B2
        }
      }
      __syncthreads();  // the last step's rows, offsets and argmin bytes
      // the progress, slot N-1 (P_{N-1}, o_{N-2}) and the last steps' argmin bytes
      publish();
      if (!ALIAS && has_consumer && N >= 2) {
        wait_consumed(N - 1);
        store_slot(N - 1, (N - 1) & 1, (N - 2) & 1);
      }
      for (int t = N - FL > 1 ? N - FL : 1; t < N; ++t) flush(t);
    }
    if (timeout) {
      s_timeout = 1;  // read by the reporting wave after the last barrier
      atomicOr(&W.mflags[b], MEMF_TIMEOUT);
    }
    __syncthreads();
    return;
  }

  // -------------------------------------------------------- compute waves --
  const int s0 = g * SPL;  // first state of this lane

  // Rows of the lane's states to LDS: non-ALIAS the block's row buffer
  // [bucket][state], ALIAS the wave's own columns of the product buffer.
  auto store_rows = [&](const uint32_t *q) __attribute__((always_inline)) {
    if constexpr (ALIAS) {
#pragma unroll
      for (int k = 0; k < SPL; ++k) Pb[0][s0 + k][col] = q[k];
    } else {
#pragma unroll
      for (int v = 0; v < SPL / 4; ++v)
        *(u32x4 *)&Qw[blk][m][s0 + 4 * v] = u32x4{q[4 * v], q[4 * v + 1], q[4 * v + 2], q[4 * v + 3]};
    }
  };

  // Normalisation of the lane's values y (kSat = unreachable) against the
  // bucket minimum over all states; returns the new offset relative to `base`.
  uint32_t y[SPL];
  auto normalise = [&](int64_t base) __attribute__((always_inline)) -> int64_t {
    uint32_t x = y[0];
#pragma unroll
    for (int k = 1; k < SPL; ++k) x = umin(x, y[k]);
    const uint32_t cm = rows_min(x);
    const bool feas = cm != kSat && base < kOffInf;
#pragma unroll
    for (int k = 0; k < SPL; ++k) y[k] = (feas ? umin(y[k] - cm, QCAP) : QCAP) << BITS;
    return feas ? base + (int64_t)cm : kOffInf;
  };

  // Step 0: D[0][s][m] = c[0][s] where mem[0][s] <= m (records read directly).
  {
    const u32x4 *cp = (const u32x4 *)(W.cst + rowbase * KP + s0);
    const uint32_t *dp = (const uint32_t *)(W.dsh + rowbase * KP + s0);
#pragma unroll
    for (int v = 0; v < SPL / 4; ++v) {
      const u32x4 c4 = cp[v];
      const uint32_t d4 = dp[v];
      y[4 * v] = bucket >= (int)(d4 & 0xFF) ? c4.x : kSat;
      y[4 * v + 1] = bucket >= (int)((d4 >> 8) & 0xFF) ? c4.y : kSat;
      y[4 * v + 2] = bucket >= (int)((d4 >> 16) & 0xFF) ? c4.z : kSat;
      y[4 * v + 3] = bucket >= (int)(d4 >> 24) ? c4.w : kSat;
    }
    const int64_t o0 = normalise(0);
    store_rows(y);
    if (g == 0) offs[0][col] = o0;
  }
  if (!consumer) {  // below bucket 0: infeasible
    for (int x = tid; x < 2 * H; x += 64 * CW) offs[x / H][x % H] = kOffInf;
    for (int x = tid; x < NPB * KP * H; x += 64 * CW) Pb[x / (KP * H)][(x / H) % KP][x % H] = kSat;
  }
  __syncthreads();

  // Table items: item (tb, k) of a step is the pair of registers holding
  // R[32 tb + 16 h + l][s0 + k] in lane l of row g (h = 0, 1): from the
  // staged table in LDS (K <= 64), else from the cache, PD items ahead
  // across step ends.
  const int l16 = lane & 15;
  auto item_ptr = [&](int e, int tb, int k) __attribute__((always_inline)) {
    return W.rT + ((size_t)e * KP + s0 + k) * KP + 32 * tb + l16;
  };
  constexpr bool HALF = S::HALF;
  constexpr int NT = TB + (HALF ? 1 : 0);  // predecessor blocks, the short one included
  // second word of an item of block tb (the short block has none: its first again)
  auto half2 = [&](int tb) __attribute__((always_inline)) { return HALF && tb >= TB ? 0 : 16; };
  u32x2 rr[PD];
  int e_cur = N > 1 ? redge[1] : 0;
  int e_nn = N > 2 ? redge[2] : e_cur;
  if constexpr (!RLDS) {
#pragma unroll
    for (int x = 0; x < PD; ++x) {
      const uint32_t *p = item_ptr(e_cur, x / SPL, x % SPL);  // PD <= SPL: items of block 0
      rr[x] = u32x2{p[0], p[half2(0)]};
    }
  }

  // Records of the lane's states for step t: costs, shift bytes (four per
  // word) and the least shift, from the parity buffer t & 1.
  constexpr int RB = ALIAS ? 8 : SPL;  // states whose records are held at once
  uint32_t cr[RB], dr[RB / 4];
  int dm = 0;
  auto read_records = [&](int par, int v0) __attribute__((always_inline)) {
#pragma unroll
    for (int v = 0; v < RB / 4; ++v) {
      const u32x4 c4 = *(const u32x4 *)&rcost[par][s0 + v0 + 4 * v];
      cr[4 * v] = c4.x;
      cr[4 * v + 1] = c4.y;
      cr[4 * v + 2] = c4.z;
      cr[4 * v + 3] = c4.w;
      dr[v] = *(const uint32_t *)&rshift[par][s0 + v0 + 4 * v];
    }
  };

  for (int i = 1; i < N; ++i) {
    const int par = i & 1, pprev = par ^ 1;
    const int pb = ALIAS ? 0 : par;
    const int e_next = e_nn;
    if constexpr (!ALIAS) {  // this step's records: the buffer is restaged after the step's barrier
      read_records(par, 0);
      dm = rdmin[par];
    }
    if constexpr (!RLDS) e_nn = i + 2 < N ? redge[i + 2] : e_next;
    if constexpr (RLDS) {
#pragma unroll
      for (int x = 0; x < PD; ++x) {
        const uint32_t *p = &rbuf[par][s0 + x][l16];
        rr[x] = u32x2{p[0], p[half2(0)]};
      }
    }

    // Phase A: products of the block's buckets for the wave's states.
    uint32_t acc[SPL];
#pragma unroll
    for (int k = 0; k < SPL; ++k) acc[k] = kSat;
    // One block of 32 predecessors (FULL) or the last 16.
    auto block = [&](int tb, auto Full) __attribute__((always_inline)) {
      constexpr bool FULL = decltype(Full)::value;
      constexpr int NQ = FULL ? 32 : 16;
      uint32_t qb[32];
      if constexpr (ALIAS) {
#pragma unroll
        for (int x = 0; x < NQ; ++x) qb[x] = Pb[0][32 * tb + x][col];
      } else {
#pragma unroll
        for (int v = 0; v < NQ / 4; ++v) {
          const u32x4 q = *(const u32x4 *)&Qw[blk][m][32 * tb + 4 * v];
          qb[4 * v] = q.x;
          qb[4 * v + 1] = q.y;
          qb[4 * v + 2] = q.z;
          qb[4 * v + 3] = q.w;
        }
      }
#pragma unroll
      for (int k = 0; k < SPL; k += 2) {
        const u32x2 ra = rr[k % PD], rb = rr[(k + 1) % PD];
#pragma unroll
        for (int u = 0; u < 2; ++u) {  // the items PD ahead
          const int kk = k + u + PD;
          const bool wrap = kk >= SPL;
          const int tn = wrap ? tb + 1 : tb;
          const int kn = wrap ? kk - SPL : kk;
          if constexpr (RLDS) {
            if (FULL ? tn < NT : !wrap) {  // within the step (the next step's table is staged later)
              const uint32_t *p = &rbuf[par][s0 + kn][32 * tn + l16];
              rr[(k + u) % PD] = u32x2{p[0], p[half2(tn)]};
            }
          } else {
            const bool nstep = wrap && tn >= NT;
            const uint32_t *p = item_ptr(nstep ? e_next : e_cur, nstep ? 0 : tn, kn);
            rr[(k + u) % PD] = u32x2{p[0], p[half2(nstep ? 0 : tn)]};
          }
        }
        mcand4x2<0, true>(acc[k], acc[k + 1], ra.x, rb.x, qb[0], qb[1], qb[2], qb[3]);
        mcand4x2<4, false>(acc[k], acc[k + 1], ra.x, rb.x, qb[4], qb[5], qb[6], qb[7]);
        mcand4x2<8, false>(acc[k], acc[k + 1], ra.x, rb.x, qb[8], qb[9], qb[10], qb[11]);
        mcand4x2<12, false>(acc[k], acc[k + 1], ra.x, rb.x, qb[12], qb[13], qb[14], qb[15]);
        if constexpr (FULL) {
          mcand4x2<0, true>(acc[k], acc[k + 1], ra.y, rb.y, qb[16], qb[17], qb[18], qb[19]);
          mcand4x2<4, false>(acc[k], acc[k + 1], ra.y, rb.y, qb[20], qb[21], qb[22], qb[23]);
          mcand4x2<8, false>(acc[k], acc[k + 1], ra.y, rb.y, qb[24], qb[25], qb[26], qb[27]);
          mcand4x2<12, false>(acc[k], acc[k + 1], ra.y, rb.y, qb[28], qb[29], qb[30], qb[31]);
        }
      }
    };
    for (int tb = 0; tb < TB; ++tb) block(tb, std::integral_constant<bool, true>{});
    if constexpr (HALF) block(TB, std::integral_constant<bool, false>{});
    e_cur = e_next;
#pragma unroll
    for (int k = 0; k < SPL; ++k) Pb[pb][s0 + k][col] = acc[k];
    __syncthreads();  // B

    // Phase B: the shifted products, their offset gaps, the bucket minimum and
    // the new rows.  The gap o[m - d] - o[m - dmin] of an available state is
    // >= 0, and infinite (saturated) when column m - d is infeasible; an
    // unavailable state has cost kSat, so its gap does not matter.
    const int64_t *O = offs[pprev];
    if constexpr (ALIAS) dm = rdmin[par];
    const int64_t base = O[col - dm];
#pragma unroll
    for (int v0 = 0; v0 < SPL; v0 += S::NB) {  // up to eight states at a time (registers)
      if constexpr (ALIAS) read_records(par, v0);
      constexpr int V = ALIAS ? 0 : 1;  // ALIAS: the records of states v0 .. v0+7 are in cr[0..7]
      constexpr int NK = S::NB;
      uint32_t pvs[NK];
      int64_t ods[NK];
#pragma unroll
      for (int k = 0; k < NK; ++k) {
        const int kr = V * v0 + k;
        const int d = (int)((dr[kr >> 2] >> (8 * (kr & 3))) & 0xFF);
        pvs[k] = Pb[pb][s0 + v0 + k][col - d];
        ods[k] = O[col - d];
      }
#pragma unroll
      for (int k = 0; k < NK; ++k) {
        const uint64_t gap = (uint64_t)(ods[k] - base);
        const uint32_t dk = gap > (uint64_t)kSat ? kSat : (uint32_t)gap;  // an infinite offset gives a huge gap
        argb[par][blk][s0 + v0 + k][m] = (uint8_t)(pvs[k] & S::MASK);
        y[v0 + k] = sat_add(sat_add(pvs[k] >> BITS, cr[V * v0 + k]), dk);
      }
    }
    const int64_t onew = normalise(base);
    if constexpr (ALIAS) __syncthreads();  // B2: every product read before the rows overwrite them
    store_rows(y);
    if (g == 0) offs[par][col] = onew;
  }
  __syncthreads();  // the last step's rows and offsets (matches the I/O waves')

  const int fin = (N - 1) & 1;  // offsets of the last step
  // Budget frontier: the offset of bucket m is min_s D[N-1][s][m], the least
  // cost with memory total at most m.
  if (a.frontier && g == 0 && bucket < M)
    a.frontier[(size_t)b * M + bucket] = (bucket <= top && offs[fin][col] < kOffInf) ? offs[fin][col] : INT64_MAX;
  __syncthreads();  // the I/O waves' timeout flag

  // The chunk holding the budget bucket reports the search.
  if (Bb >= m0 && Bb < m0 + C && w == 0) {
    const int cb = Bb - m0, wb = cb >> 4, mb = cb & 15;
    uint32_t f = kSat;
    for (int s = lane; s < K; s += 64) {
      uint32_t q;
      if constexpr (ALIAS) q = Pb[0][s][H + cb];
      else q = Qw[wb][mb][s];
      f = umin(f, q | (uint32_t)s);
    }
    f = wave_min(f);
    bool rbad = false;
    for (int x = lane; x < a.nbad; x += 64) rbad |= W.rbad[x] != 0;
    rbad = __any(rbad);
    if (lane == 0) {
      const int64_t o = offs[fin][H + cb];
      const int sf = __hip_atomic_load(&W.mflags[b], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT);
      int st = CFP_ST_OK;
      if (s_timeout || (sf & MEMF_TIMEOUT)) st = CFP_ST_TIMEOUT;
      else if (rbad) st = CFP_ST_BADINPUT;
      else if (o >= kOffInf) st = CFP_ST_INFEASIBLE;
      else if ((f >> BITS) != 0) st = CFP_ST_OVERFLOW;  // the least state of a feasible bucket is 0
      a.status[b] = st;
      a.opt[b] = st == CFP_ST_OK ? o : INT64_MAX;
      a.res[b].final_state = st == CFP_ST_OK ? (int32_t)(f & S::MASK) : -1;
      a.res[b].status = st;
      a.res[b].final_m = Bb;
    }
  }
}

// Plan recovery for the memory variant.  The state is (s, m): the table gives
// the predecessor strategy t = arg[i][s][m] and the budget shrinks by
// mem[i][s].  The chase runs in windows of W rows whose reachable buckets are
// loaded into LDS, then one thread follows them.  Row k of a window that starts
// at bucket m can only be read at m - dm k .. m, dm the search's largest shift,
// so it takes ns(k) 16-byte pieces of each state, counted down from the piece
// of m.  A window costs one memory latency, its bytes at the rate of one
// compute unit and the dependent LDS reads; the packed triangle holds about
// twice the rows of a rectangle (16 searches of 288 blocks, K = 32, shifts up
// to 8: 28 rows per window instead of 12).
constexpr int kMemTbThreads = 1024;
constexpr int kMemTbWaves = kMemTbThreads / 64;
constexpr int kMemTbLoads = 8;       // pieces in flight per lane
constexpr int kMemTbRows = 64;       // most rows per window
constexpr int kMemTbLds = 144 * 1024;

__device__ __forceinline__ int mem_tb_pieces(int dm, int k) { return ((dm * k + 15) >> 4) + 1; }

__global__ __launch_bounds__(kMemTbThreads) void mem_tb_kernel(int N, int K, int MS, const uint8_t *__restrict__ table,
                                                               const uint8_t *__restrict__ mem_copy,
                                                               const SearchResult *__restrict__ res,
                                                               int32_t *__restrict__ plan) {
  __shared__ __align__(16) uint8_t wbuf[kMemTbLds];  // mem rows [W][K], then the rows' pieces [K][ns(k)][16]
  __shared__ int rowoff[kMemTbRows + 1];
  __shared__ int cur_s, cur_m, s_w, s_dm;
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  int32_t *pb = plan + (size_t)b * N;
  if (res[b].status != CFP_ST_OK) {
    for (int i = tid; i < N; i += blockDim.x) pb[i] = -1;
    return;
  }
  // The search's largest shift (a few KB read once; a counter kept by the forward
  // call's row checks cost 50 us in atomics on one word per search).
  if (tid == 0) s_dm = 0;
  __syncthreads();
  {
    const uint8_t *mb = mem_copy + (size_t)b * N * K;
    const int count = N * K, head = min(count, (int)(-(uintptr_t)mb & 3)), words = (count - head) / 4;
    uint32_t x = 0;
    for (int q = tid; q < words; q += kMemTbThreads) {
      const uint32_t v = *(const uint32_t *)(mb + head + 4 * q);
      x = max(max(x, v & 0xFF), max(max((v >> 8) & 0xFF, (v >> 16) & 0xFF), v >> 24));
    }
    if (tid < head) x = max(x, (uint32_t)mb[tid]);
    if (tid < count - head - 4 * words) x = max(x, (uint32_t)mb[head + 4 * words + tid]);
    for (int o = 32; o >= 1; o >>= 1) x = max(x, (uint32_t)__shfl_xor((int)x, o, 64));
    if (lane == 0) atomicMax(&s_dm, (int)x);
  }
  __syncthreads();
  const int dm = s_dm;
  if (tid == 0) {
    cur_s = res[b].final_state;
    cur_m = res[b].final_m;
    pb[N - 1] = cur_s;
    // as many rows as fit; the first always does (K <= 256: 256 + 4096 bytes)
    int w = 0, pieces = 0;
    while (w < kMemTbRows && w < N - 1) {
      const int next = pieces + K * mem_tb_pieces(dm, w);
      if (((w + 1) * K + 15) / 16 * 16 + next * 16 > kMemTbLds) break;
      rowoff[w] = pieces;
      pieces = next;
      ++w;
    }
    s_w = w;
  }
  __syncthreads();
  const int W = s_w;
  uint8_t *mrow = wbuf;
  typedef uint32_t u32x4l __attribute__((ext_vector_type(4)));  // copies stay in registers
  u32x4l *rows = (u32x4l *)(wbuf + (W * K + 15) / 16 * 16);
  for (int i = N - 1; i >= 1;) {
    const int steps = min(i, W);
    const int mtop = cur_m;
    // One row per wave at a time, short and long rows in turn.
    for (int r = 0; r * kMemTbWaves < steps; ++r) {
      const int k = r * kMemTbWaves + ((r & 1) ? kMemTbWaves - 1 - wid : wid);
      if (k >= steps) continue;
      const int ns = mem_tb_pieces(dm, k), total = K * ns;
      const float inv = 1.0f / (float)ns;
      const uint8_t *src = table + ((size_t)b * N + (i - k)) * K * MS;
      u32x4l *dst = rows + rowoff[k];
      for (int x0 = 0; x0 < total; x0 += 64 * kMemTbLoads) {
        u32x4l v[kMemTbLoads];
#pragma unroll
        for (int u = 0; u < kMemTbLoads; ++u) {
          const int x = min(x0 + 64 * u + lane, total - 1);
          const int t = (int)(((float)x + 0.5f) * inv), c = x - t * ns;  // x < 2^14: exact
          v[u] = *(const u32x4l *)(src + (size_t)t * MS + 16 * max((mtop >> 4) - c, 0));
        }
#pragma unroll
        for (int u = 0; u < kMemTbLoads; ++u) {
          const int x = x0 + 64 * u + lane;
          if (x < total) dst[x] = v[u];
        }
      }
    }
    for (int x = tid; x < steps * K; x += kMemTbThreads) {
      const int k = x / K;
      mrow[x] = mem_copy[((size_t)b * N + (i - k)) * K + (x - k * K)];
    }
    __syncthreads();
    if (tid == 0) {
      int s = cur_s, m = mtop;
      for (int k = 0; k < steps; ++k) {
        const int ns = mem_tb_pieces(dm, k);
        const int c = min((mtop >> 4) - (m >> 4), ns - 1);  // (the bound holds on a consistent table)
        const int t = ((const uint8_t *)(rows + rowoff[k] + s * ns + c))[m & 15];
        m = max(m - (int)mrow[k * K + s], 0);
        s = min(t, K - 1);
        pb[i - k - 1] = s;
      }
      cur_s = s;
      cur_m = m;
    }
    __syncthreads();
    i -= steps;
  }
}

// Row stride of the argmin table along the buckets: whole 16-byte pieces.
int mem_stride(int n_mem) { return (n_mem + 15) / 16 * 16; }

hipError_t launch_traceback_mem(int n, int k, int batch, int n_mem, const uint8_t *table, const uint8_t *mem,
                                const SearchResult *res, int32_t *plan, hipStream_t st) {
  hipLaunchKernelGGL(mem_tb_kernel, dim3(batch), dim3(kMemTbThreads), 0, st, n, k, mem_stride(n_mem), table, mem, res,
                     plan);
  return hipGetLastError();
}

static MemWs carve(uint8_t *region, int n, int k, int batch, int n_mem, int n_tables, size_t *bytes) {
  const int KP = mem_kp(k);
  MemWs w;
  w.nchunk = (n_mem + kMemChunk - 1) / kMemChunk;
  const size_t chunks = (size_t)batch * w.nchunk;
  size_t off = 0;
  w.cst = (uint32_t *)(region + off); off = align_up(off + (size_t)batch * n * KP * 4);
  w.dsh = region + off; off = align_up(off + (size_t)batch * n * KP);
  w.dmin = (int32_t *)(region + off); off = align_up(off + (size_t)batch * n * 4);
  w.rT = (uint32_t *)(region + off); off = align_up(off + (size_t)n_tables * KP * KP * 4);
  w.mflags = (int32_t *)(region + off); off = align_up(off + (size_t)batch * 4);
  w.rowbad = region + off; off = align_up(off + (size_t)batch * n);
  w.rbad = (int32_t *)(region + off); off = align_up(off + kMemPrepBlocks * 4);
  w.cons = (int32_t *)(region + off); off = align_up(off + chunks * kMemFlagStride * 4);
  w.ring = (uint64_t *)(region + off); off = align_up(off + chunks * kMemSlots * mem_slot_words(KP) * 8);
  if (bytes) *bytes = off;
  return w;
}

size_t mem_region_bytes(int n, int k, int batch, int n_mem, int n_tables) {
  size_t bytes = 0;
  (void)carve(nullptr, n, k, batch, n_mem, n_tables, &bytes);
  return bytes;
}

// Workgroups of one launch that the device holds at once, per XCD: the
// chunks of a search run as a pipeline whose stages wait for each other, so
// every chunk of a launch must be resident together.  Workgroup x runs on XCD
// x mod 8, and the chunks of search b of a launch are workgroups j * B8 + b,
// so they share one XCD and its L2 cache.
// The hardware spreads a workgroup's waves over the four SIMDs of a compute
// unit and does not shift the start from one workgroup to the next, so every
// SIMD must have room for ceil(waves / 4) more: a workgroup of six waves counts
// as one of eight.  (The query counts waves per compute unit.  Asked for six it
// says three workgroups of 96 registers, and two fit: 64 searches of 200 or more
// blocks with 1024 buckets then waited for chunks that could not start and ended
// with CFP_ST_TIMEOUT.)
template <int KP>
static int mem_xcd_capacity() {
  static std::once_flag once;
  static int cap = 0;
  std::call_once(once, [] {
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, mem_fwd_kernel<KP>,
                                                     (MemShape<KP>::THREADS + 255) / 256 * 256, 0) != hipSuccess)
      return;
    cap = (cus / 8) * per_cu;
  });
  return cap;
}

template <int KP>
static hipError_t launch_mem(const cfp_chain_desc &d, const uint8_t *mem, int n_mem, int32_t *budget, bool fill,
                             int32_t *redge_dev, const EdgeMap &em, uint8_t *table, uint8_t *mem_copy, uint8_t *region,
                             SearchResult *res, int64_t *opt, int32_t *status, int64_t *frontier, hipStream_t st) {
  const int N = d.n_blocks, K = d.k, B = d.batch, E = d.n_tables;
  MemWs w = carve(region, N, K, B, n_mem, E, nullptr);
  MemPrepArgs p;
  p.cost = d.cost;
  p.rtab = d.rtab;
  p.mem = mem;
  p.budget = budget;
  p.fill = fill;
  p.N = N;
  p.K = K;
  p.KP = KP;
  p.M = n_mem;
  p.B = B;
  p.E = E;
  p.bits = MemShape<KP>::BITS;
  p.rlimit = cfp_r_limit(CFP_V_MEM, K);
  p.w = w;
  p.nring = (size_t)B * w.nchunk * kMemSlots * mem_slot_words(KP);
  p.nflag = B * w.nchunk * kMemFlagStride;
  p.mem_copy = mem_copy;
  p.em = em;
  p.redge = redge_dev;
  const size_t want = std::max(std::max(((size_t)B * N + 3) / 4, (p.nring + 255) / 256),
                               ((size_t)E * KP * KP + 255) / 256);
  const int blocks = (int)std::min<size_t>(want, kMemPrepBlocks);
  hipLaunchKernelGGL(mem_prep_kernel, dim3(blocks), dim3(256), 0, st, p);
  // Rounds of searches whose chunks the device holds at once: with per_xcd
  // searches on each of the 8 XCDs, a round takes 8 * per_xcd searches.
  const int cap = mem_xcd_capacity<KP>();
  const int per_xcd = cap / w.nchunk;
  if (per_xcd < 1) return hipErrorInvalidConfiguration;
  const int round = 8 * per_xcd;
  MemArgs a;
  a.budget = budget;
  a.w = w;
  a.N = N;
  a.K = K;
  a.M = n_mem;
  a.MS = mem_stride(n_mem);
  a.B = B;
  a.table = table;
  a.res = res;
  a.nbad = blocks;
  a.opt = opt;
  a.status = status;
  a.frontier = frontier;
  timer_begin(st);
  for (int b0 = 0; b0 < B; b0 += round) {
    a.b0 = b0;
    a.nb = std::min(round, B - b0);
    a.B8 = (a.nb + 7) / 8 * 8;
    timed_launch(mem_fwd_kernel<KP>, dim3(w.nchunk * a.B8), dim3(MemShape<KP>::THREADS), 0, st, a, (const int32_t *)redge_dev,
                 (const int32_t *)w.dmin);
  }
  timer_end(st);
  return hipGetLastError();
}

bool chain_mem_supported(int k, int n_tables) { return k >= 1 && k <= kMemMaxK && n_tables >= 1; }

int32_t mem_r_limit(int k) { return k >= 1 && k <= kMemMaxK ? (int32_t)(1u << (31 - mem_bits(k))) : 0; }

hipError_t launch_chain_mem_fwd(const cfp_chain_desc &d, const uint8_t *mem, int n_mem, int32_t *budget, bool fill,
                                int32_t *redge_dev, const EdgeMap &em, uint8_t *table, uint8_t *mem_copy,
                                uint8_t *region, SearchResult *res, int64_t *opt, int32_t *status, int64_t *frontier,
                                hipStream_t st) {
#define CFP_MEM_CASE(KPV) \
  case KPV:               \
    return launch_mem<KPV>(d, mem, n_mem, budget, fill, redge_dev, em, table, mem_copy, region, res, opt, status, frontier, st);
  switch (mem_kp(d.k)) {
    CFP_MEM_CASE(16)
    CFP_MEM_CASE(32)
    CFP_MEM_CASE(48)
    CFP_MEM_CASE(64)
    CFP_MEM_CASE(80)
    CFP_MEM_CASE(96)
    CFP_MEM_CASE(112)
    CFP_MEM_CASE(128)
    CFP_MEM_CASE(192)
    CFP_MEM_CASE(256)
    default:
      return hipErrorInvalidValue;
  }
#undef CFP_MEM_CASE
}

}  // namespace cfp
