// Forward pass of the chain search for K <= 32 (Sec. 4.4, Eq. T recurrence),
// chunk-parallel on long chains.
//
// A chain of N-1 dependent steps is cut into P chunks that run at once, made
// exact by rank convergence (Maleki, Musuvathi and Mytkowicz, PPoPP 2014), as
// in the K <= 64 form: a speculative pass starts every chunk from its first
// row's costs alone, a fix-up pass reruns each chunk from the row its
// predecessor ends on until the rows meet, a second fix-up reruns, all at once,
// the chunks behind one that met no checkpoint from that chunk's end row, and a
// final pass sums the chunk offsets and reruns the chunks that no run started
// from the true row of.  A chain of one chunk is finished by the speculative pass
// itself.
//
// How far two runs go before they are parallel depends on the inputs.  On costs
// and resharding times of one range nearly every chunk meets; where the costs
// repeat with the edge map every chunk starts in the same phase, and a search
// whose runs take longer than a chunk leaves all of its chunks unmet (a few
// searches in a thousand), which the second fix-up resolves for three in four;
// where resharding dominates, no chunk meets and the final pass runs the chain.
// There one chunk takes all lanes of a wave (narrow_solo).  Per call with its
// traceback, 1152 blocks, K = 27, 32 searches, through the Python binding one after
// another (40 us of 52 on the device): 52 us on costs of their own; 48 to 55
// on repeated ones, 66 where a search leaves its chunks unmet (366 when the final
// pass reran them with one of two half-wave tasks and without a second fix-up); 95
// with resharding 30 times the costs (187); 265 where no chunk ever meets (367; a
// sequential kernel took 287 on any input).  In batches of 200 and more that last
// kind of input takes up to 1.3 times as long as sequentially, any other less.

// At K <= 32 a step is 16 or 32 candidates per state: what bounds it is the
// latency of the dependent instructions of a step (a few hundred cycles) and,
// for a whole call, the launches.  So
//   * a task (one chunk of one search) takes 16 lanes (K <= 16), a whole wave (K up
//     to 32) or, in large batches of those, half of one: the row broadcasts of the
//     previous row stay within a row of 16 lanes or come from one permlane swap,
//     and no LDS exchange or barrier is in the loop;
//   * all the packed tables stay in LDS (4 KiB each at KP = 32), staged and
//     range-checked once per workgroup from the caller's tables; a row's words
//     are read one row ahead, its costs eight rows ahead;
//   * a periodic edge map (period up to 64) travels in the launch's arguments,
//     so no header is uploaded and no packing kernel runs.
//
// Normalisation and packing are those of the K <= 64 form: candidates are
// (Q[t] << b) + ((R[t][s] << b) | t), x[s] = (m >> b) + c[i][s], d = min_s x[s],
// Q[s] = min(x[s] - d, 2^(31-b) - 1).  R < 2^(30-b), so no candidate wraps, and
// a capped state is beaten through the row's minimum.
#include <algorithm>

#include "res_common.h"

namespace cfp {

namespace {

constexpr int kNSpec = 0, kNFix = 1, kNFix2 = 2;
constexpr uint32_t kNX = 0xFFFFFFFFu;    // x of an unavailable or padding state
constexpr int kNRing = 8;                // rows of costs in flight
constexpr size_t kNMaxLds = 152 * 1024;  // packed tables of a workgroup
// Least chunks for a second fix-up: on fewer the final pass reruns the chain in less
// than 60 us, and the launch costs a call of small searches 4 us (1 in 8).
constexpr int kNSecond = 16;
constexpr int kRowRor = 0x120;           // DPP row_ror:n = kRowRor + n

template <int KP>
struct NarrowShape {
  static constexpr int BITS = KP <= 16 ? 4 : 5;
  static constexpr int CH = KP / 4;            // 16-byte pieces of a table column
  static constexpr int TABLE16 = KP * KP / 4;  // 16-byte pieces of a table
  static constexpr uint32_t QCAP = (1u << (31 - BITS)) - 1u;
};

struct NarrowRec {
  int64_t dfix;   // fix-up: offset sum at the meeting checkpoint, or at the chunk end
  int64_t dfix2;  // the same of the second fix-up
  int32_t flags;  // speculative pass: bit 0 a value out of range, bit 1 a row with no available strategy
  int32_t conv;   // fix-up: quad of the meeting checkpoint, -1 if none
  int32_t conv2;  // the same of the second fix-up
  int32_t run2;   // the second fix-up ran this chunk (from the first one's end row of the chunk before)
  int32_t same2;  // and met no checkpoint, but ended on the first one's end row of this chunk
};

// The row that the last run of a chunk ends on: its speculative end row, the end
// row of its fix-up (which the next chunk's second fix-up starts from), or that
// of its second fix-up.
enum { kEndSpec, kEnd1, kEnd2 };
__device__ __forceinline__ int narrow_end(const NarrowRec &r) {
  if (r.run2) return r.conv2 >= 0 ? kEndSpec : r.same2 ? kEnd1 : kEnd2;
  return r.conv >= 0 ? kEndSpec : kEnd1;
}

// Quad a rerun of chunk p (last quad qe) must reach before it may stop: past
// every row that earlier runs from other start rows rewrote.
__device__ __forceinline__ int narrow_qmin(const NarrowRec &r, int qe) {
  int q = r.conv < 0 ? qe : r.conv;
  if (r.run2) q = max(q, r.conv2 < 0 ? qe : r.conv2);
  return q;
}

struct NarrowArgs {
  const int32_t *cost;
  const int32_t *rtab;
  const int32_t *redge;  // device copy of the edge map; used when period is 0
  int N, K, E, B, P, CL, nq;  // CL rows per chunk (a multiple of 4), nq quads of rows
  bool second;                // a second fix-up runs
  int32_t rlimit;
  uint8_t *table;    // argmin entries [B][N][K]
  NarrowRec *rec;    // [B][P]
  int64_t *dck;      // speculative offset sum (from the chunk's start row) at every quad end [B][nq]
  uint32_t *ckrow;   // speculative row at every quad end [B][nq][KP]
  uint32_t *endrow;  // fix-up end row of chunks that met no checkpoint [B][P][KP]
  uint32_t *endrow2;     // the same of the second fix-up
  SearchResult *res;
  int64_t *opt;
  int32_t *status;
  EdgeMap em;
};

// Packs the tables into LDS: word u of piece c of column s of table e is
// (R_e[t][s] << b) | t with t = 4c + u; rows and columns past K repeat the last
// one (their predecessors hold capped words, their states are padding).
// Returns true if this thread saw an entry outside [0, rlimit).
template <int KP>
__device__ __forceinline__ bool narrow_stage(const NarrowArgs &a, u32x4 *tabs, int nthreads) {
  using S = NarrowShape<KP>;
  bool bad = false;
  const int pieces = a.E * S::TABLE16;
  for (int x = threadIdx.x; x < pieces; x += nthreads) {
    const int s = x % KP, c = (x / KP) % S::CH, e = x / S::TABLE16;
    const int32_t *src = a.rtab + (size_t)e * a.K * a.K + min(s, a.K - 1);
    uint32_t w[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int t = 4 * c + u;
      const int32_t r = src[min(t, a.K - 1) * a.K];
      bad |= r < 0 || r >= a.rlimit;
      w[u] = ((uint32_t)r << S::BITS) | (uint32_t)t;
    }
    u32x4 v;
    v.x = w[0];
    v.y = w[1];
    v.z = w[2];
    v.w = w[3];
    tabs[x] = v;
  }
  return bad;
}

// A periodic edge map as a list in LDS: per place the first 16-byte piece of its
// table and the place of the next row, so that a row costs one read.
template <int KP>
__device__ __forceinline__ void narrow_edges(const EdgeMap &em, int2 *elist) {
  const int x = threadIdx.x;
  if (x < kEdgeWords) elist[x] = make_int2(em.map[x] * NarrowShape<KP>::TABLE16, x + 1 == em.head + em.period ? em.head : x + 1);
}

// Minimum over the KP lanes of a task (every lane of the task gets it).
template <int KP>
__device__ __forceinline__ uint32_t task_min(uint32_t x) {
  x = group_min<16>(x);
  if constexpr (KP == 32) {
    const auto p = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    x = umin(p[0], p[1]);
  }
  return x;
}

// A lane's view of its task's run.
struct NarrowRun {
  uint32_t q;      // word of the lane's state in the current row
  uint64_t dsum;   // offset sum since the start row
  uint32_t cor;    // OR of the lane's costs (bit 31: a negative cost)
  bool infeasible; // a row with no available strategy
  int conv;        // fix-up: quad where the row met the checkpoint, -1 if never
  uint64_t dconv;  // fix-up: offset sum at that quad
};

// Runs rows [r0, iend] of the lane's task (search b; valid: it exists).  Rows
// and the task differ from task to task; the loop counts rows from r0.
//   kNSpec: row r0 is the start row, from its costs alone; checkpoints are
//           written.
//   kNFix:  the row before r0 is run.q; at every quad end from quad qmin on the
//           row is compared with the checkpoint of the same quad, and a task
//           that has met it stops.
template <int KP, int MODE, bool PER>
__device__ __forceinline__ void narrow_run(const NarrowArgs &a, const u32x4 *tabs, const int2 *elist, int b,
                                           bool valid, int r0, int iend, int qmin, NarrowRun &run) {
  using S = NarrowShape<KP>;
  constexpr int CH = S::CH;
  const int lane = threadIdx.x & 63, s = lane & (KP - 1);
  const int K = a.K;
  const bool sin = s < K;
  // byte offsets of the lane's entries in the chain's rows (below 2^31: N < 2^24, K <= 32)
  const char *cb = (const char *)(a.cost + (size_t)b * a.N * K + min(s, K - 1));
  uint8_t *tb = a.table + (size_t)b * a.N * K + s;
  uint32_t *ckb = a.ckrow + (size_t)b * a.nq * KP + s;
  const uint32_t K4 = 4u * (uint32_t)K, clast = (uint32_t)iend * K4;
  uint32_t coff = (uint32_t)r0 * K4, toff = (uint32_t)r0 * (uint32_t)K;  // of the next cost row to load, of the current row
  auto next_cost = [&]() __attribute__((always_inline)) {
    const uint32_t c = *(const uint32_t *)(cb + umin(coff, clast));
    coff += K4;
    return c;
  };
  uint32_t cs[kNRing];
  int er[kNRing];  // table of the row (edge map in memory)
#pragma unroll
  for (int j = 0; j < kNRing; ++j) {
    cs[j] = next_cost();
    if (!PER) er[j] = a.redge[min(r0 + j, iend)] * S::TABLE16;
  }
  // Periodic edge map: the table of the next row and the place of the row after it.
  int2 e1 = {};
  int e0;
  if (PER) {
    const int2 x = elist[a.em.place(r0)];
    e0 = x.x;
    e1 = elist[x.y];
  } else {
    e0 = er[0];
  }
  uint32_t ckv[2] = {0, 0};
  if (MODE == kNFix) {
    ckv[0] = ckb[(size_t)(r0 >> 2) * KP];
    ckv[1] = ckb[(size_t)min((r0 >> 2) + 1, iend >> 2) * KP];
  }
  u32x4 w[2][CH];
#pragma unroll
  for (int c = 0; c < CH; ++c) w[0][c] = tabs[e0 + c * KP + s];
  uint32_t q = run.q;
  uint64_t dsum = 0;
  run.cor = 0;
  run.infeasible = false;
  run.conv = -1;
  run.dconv = 0;
  bool live = valid;  // fix-up: not met yet

  // Row r0 + k; J = k mod 8.
  auto step = [&](auto Jc, int k) __attribute__((always_inline)) {
    constexpr int J = decltype(Jc)::value, cur = J & 1, nxt = cur ^ 1;
    const int row = r0 + k;
    const bool act = row <= iend && (MODE == kNSpec ? valid : live);
    // the next row's table words
    int en;
    if (PER) {
      en = e1.x;
      e1 = elist[e1.y];
    } else {
      en = er[(J + 1) % kNRing];
      er[J] = a.redge[min(row + kNRing, iend)] * S::TABLE16;
    }
#pragma unroll
    for (int c = 0; c < CH; ++c) w[nxt][c] = tabs[en + c * KP + s];

    // Row-broadcast sources: each row of 16 lanes holds the words of 16 predecessors.
    uint32_t c0 = q, c1 = q;
    if constexpr (KP == 32) {
      const auto p = __builtin_amdgcn_permlane16_swap(q, q, false, false);
      c0 = p[0];
      c1 = p[1];
    }
    uint32_t acc;
    cand4_g1_first(acc, c0, w[cur][0]);
    cand4_g1<4, false>(acc, c0, w[cur][1]);
    cand4_g1<8, false>(acc, c0, w[cur][2]);
    cand4_g1<12, false>(acc, c0, w[cur][3]);
    if constexpr (KP == 32) {
      cand4_g1<0, true>(acc, c1, w[cur][4]);
      cand4_g1<4, false>(acc, c1, w[cur][5]);
      cand4_g1<8, false>(acc, c1, w[cur][6]);
      cand4_g1<12, false>(acc, c1, w[cur][7]);
    }
    if (MODE == kNSpec && J == 0 && k == 0) acc = 0;  // the start row: no predecessor

    const uint32_t cv = cs[J];
    if (MODE == kNSpec) {
      run.cor |= cv;
      asm volatile("" : "+v"(run.cor));  // kept in its row
    }
    cs[J] = next_cost();
    const uint32_t x = sin && cv != (uint32_t)CFP_COST_INF ? (acc >> S::BITS) + cv : kNX;
    const uint32_t d = task_min<KP>(x);
    const uint32_t qn = umin(x - d, S::QCAP) << S::BITS;
    if (act) {
      q = qn;
      dsum += d;
      if (MODE == kNSpec) run.infeasible |= d == kNX;
    }
    if (act && sin) tb[toff] = (uint8_t)(acc & (KP - 1));
    toff += (uint32_t)K;
  };
  // End of quad h (0 or 1) of the turn that starts at row r0 + k.
  auto quad = [&](auto Hc, int k) __attribute__((always_inline)) {
    constexpr int H = decltype(Hc)::value;
    const int first = r0 + k + 4 * H, qd = first >> 2;
    if (MODE == kNSpec) {
      if (valid && first <= iend) {
        ckb[(size_t)qd * KP] = q;
        if (s == 0) a.dck[(size_t)b * a.nq + qd] = (int64_t)dsum;
      }
    } else {
      const bool here = live && first <= iend;
      const uint64_t off = __ballot(here && q != ckv[H]);
      const uint64_t mine = (off >> (lane & ~(KP - 1))) & ((1ull << KP) - 1);
      if (here && qd >= qmin && mine == 0) {
        run.conv = qd;
        run.dconv = dsum;
        live = false;
      }
      ckv[H] = ckb[(size_t)min(qd + 2, iend >> 2) * KP];
    }
  };
  for (int k = 0;; k += kNRing) {
    step(std::integral_constant<int, 0>{}, k);
    step(std::integral_constant<int, 1>{}, k + 1);
    step(std::integral_constant<int, 2>{}, k + 2);
    step(std::integral_constant<int, 3>{}, k + 3);
    quad(std::integral_constant<int, 0>{}, k);
    step(std::integral_constant<int, 4>{}, k + 4);
    step(std::integral_constant<int, 5>{}, k + 5);
    step(std::integral_constant<int, 6>{}, k + 6);
    step(std::integral_constant<int, 7>{}, k + 7);
    quad(std::integral_constant<int, 1>{}, k);
    if (!__ballot((MODE == kNSpec ? valid : live) && r0 + k + kNRing <= iend)) break;
  }
  run.q = q;
  run.dsum = dsum;
}

// The same for one task (search b) with all lanes of the wave: group g takes the
// predecessors 4 g .. 4 g + 3 (KP = 16) or 16 g .. 16 g + 15 (KP = 32), and every
// group holds the row.  Everything but the lane's state is uniform, and no load or
// store sits behind a branch: a padding lane computes what state K-1 does, and
// writes it to the same place.  A fix-up run ends where it meets a checkpoint.
// (A row takes 0.19 us at KP = 32 and 0.15 at 16, where two and four tasks of a wave
// take 0.35 and 0.25 together.)
template <int KP, int MODE, bool PER>
__device__ __forceinline__ void narrow_solo(const NarrowArgs &a, const u32x4 *tabs, const int2 *elist, int b, int r0,
                                            int iend, int qmin, NarrowRun &run) {
  using S = NarrowShape<KP>;
  constexpr int PPG = S::CH * KP / 64;  // 16-byte pieces of a column per group
  const int lane = threadIdx.x & 63, s = lane & (KP - 1), K = a.K;
  const bool sin = s < K;
  const int sl = min(s, K - 1), qlast = iend >> 2;
  // uniform bases and the byte offsets of the lane's entries (rows from r0 on)
  const char *cb = (const char *)(a.cost + ((size_t)b * a.N + r0) * K);
  uint8_t *tb = a.table + ((size_t)b * a.N + r0) * K;
  uint32_t *ckb = a.ckrow + (size_t)b * a.nq * KP + s;
  int64_t *dck = a.dck + (size_t)b * a.nq;
  const u32x4 *tl = tabs + (lane / KP) * PPG * KP + s;
  const uint32_t K4 = 4u * (uint32_t)K, clast = (uint32_t)(iend - r0) * K4 + 4u * (uint32_t)sl;
  uint32_t coff = 4u * (uint32_t)sl, toff = (uint32_t)sl;
  auto next_cost = [&]() __attribute__((always_inline)) {
    const uint32_t c = *(const uint32_t *)(cb + umin(coff, clast));
    coff += K4;
    return c;
  };
  uint32_t cs[kNRing];
  int er[kNRing];
#pragma unroll
  for (int j = 0; j < kNRing; ++j) {
    cs[j] = next_cost();
    if (!PER) er[j] = a.redge[min(r0 + j, iend)] * S::TABLE16;
  }
  int2 e1 = {};
  int e0;
  if (PER) {
    const int2 x = elist[a.em.place(r0)];
    e0 = x.x;
    e1 = elist[x.y];
  } else {
    e0 = er[0];
  }
  uint32_t ckv[2] = {0, 0};
  if (MODE == kNFix) {
    ckv[0] = ckb[(size_t)(r0 >> 2) * KP];
    ckv[1] = ckb[(size_t)min((r0 >> 2) + 1, qlast) * KP];
  }
  u32x4 w[2][PPG];
#pragma unroll
  for (int c = 0; c < PPG; ++c) w[0][c] = tl[e0 + c * KP];
  uint32_t q = run.q, cor = 0, top = 0;
  uint64_t dsum = 0;
  int conv = -1;
  auto step = [&](auto Jc, int row) __attribute__((always_inline)) {
    constexpr int J = decltype(Jc)::value, cur = J & 1, nxt = cur ^ 1;
    int en;
    if (PER) {
      en = e1.x;
      e1 = elist[e1.y];
    } else {
      en = er[(J + 1) % kNRing];
      er[J] = a.redge[min(row + kNRing, iend)] * S::TABLE16;
    }
#pragma unroll
    for (int c = 0; c < PPG; ++c) w[nxt][c] = tl[en + c * KP];
    // every row of 16 lanes gets the words of its group's predecessors
    uint32_t src;
    if constexpr (KP == 32) {
      const auto p = __builtin_amdgcn_permlane16_swap(q, q, false, false);
      src = lane < 32 ? p[0] : p[1];
    } else {  // row g rotated by 4 g lanes
      src = (uint32_t)__builtin_amdgcn_update_dpp((int)q, (int)q, kRowRor + 8, 0xC, 0xF, false);
      src = (uint32_t)__builtin_amdgcn_update_dpp((int)src, (int)src, kRowRor + 12, 0xA, 0xF, false);
    }
    uint32_t acc;
    cand4_g1_first(acc, src, w[cur][0]);
    if constexpr (KP == 32) {
      cand4_g1<4, false>(acc, src, w[cur][1]);
      cand4_g1<8, false>(acc, src, w[cur][2]);
      cand4_g1<12, false>(acc, src, w[cur][3]);
    } else {
      const auto r = __builtin_amdgcn_permlane16_swap(acc, acc, false, false);
      acc = umin(r[0], r[1]);
    }
    const auto h = __builtin_amdgcn_permlane32_swap(acc, acc, false, false);
    acc = umin(h[0], h[1]);
    if (MODE == kNSpec && J == 0 && row == r0) acc = 0;  // the start row: no predecessor
    const uint32_t cv = cs[J];
    if (MODE == kNSpec) {
      cor |= cv;
      asm volatile("" : "+v"(cor));  // kept in its row
    }
    cs[J] = next_cost();
    const uint32_t x = sin && cv != (uint32_t)CFP_COST_INF ? (acc >> S::BITS) + cv : kNX;
    const uint32_t d = task_min<KP>(x);
    q = umin(x - d, S::QCAP) << S::BITS;
    dsum += d;
    if (MODE == kNSpec) top = max(top, d);
    tb[toff] = (uint8_t)(acc & (KP - 1));
    toff += (uint32_t)K;
  };
  // End of quad qd; true where a fix-up run ends there.
  auto quad = [&](auto Hc, int qd) __attribute__((always_inline)) {
    constexpr int H = decltype(Hc)::value;
    if (MODE == kNSpec) {
      ckb[(size_t)qd * KP] = q;
      dck[qd] = (int64_t)dsum;
      return false;
    }
    if (qd >= qmin && __ballot(q != ckv[H]) == 0) {
      conv = qd;
      return true;
    }
    ckv[H] = ckb[(size_t)min(qd + 2, qlast) * KP];
    return false;
  };
#define CFP_N_STEP(J_) step(std::integral_constant<int, J_>{}, i + J_)
#define CFP_N_QUAD(H_) quad(std::integral_constant<int, H_>{}, (i >> 2) + H_)
  [&]() __attribute__((always_inline)) {
    int i = r0;
    for (; i + 7 <= iend; i += 8) {
      CFP_N_STEP(0), CFP_N_STEP(1), CFP_N_STEP(2), CFP_N_STEP(3);
      if (CFP_N_QUAD(0)) return;
      CFP_N_STEP(4), CFP_N_STEP(5), CFP_N_STEP(6), CFP_N_STEP(7);
      if (CFP_N_QUAD(1)) return;
    }
    if (i > iend) return;
    CFP_N_STEP(0);
    if (i + 1 <= iend) CFP_N_STEP(1);
    if (i + 2 <= iend) CFP_N_STEP(2);
    if (i + 3 <= iend) CFP_N_STEP(3);
    if (CFP_N_QUAD(0) || i + 4 > iend) return;
    CFP_N_STEP(4);
    if (i + 5 <= iend) CFP_N_STEP(5);
    if (i + 6 <= iend) CFP_N_STEP(6);
    CFP_N_QUAD(1);
  }();
#undef CFP_N_QUAD
#undef CFP_N_STEP
  run.q = q;
  run.dsum = run.dconv = dsum;
  run.conv = conv;
  run.cor = cor;
  run.infeasible = top == kNX;
}

// Lowest state of the final row (its minimum is 0), optimum and status of
// search b, written by the lane with `lead` set; every lane of the task calls it.
template <int KP>
__device__ __forceinline__ void narrow_finish(const NarrowArgs &a, int b, uint32_t q, int64_t total, int flags,
                                              bool lead) {
  using S = NarrowShape<KP>;
  const int s = threadIdx.x & (KP - 1);
  const uint32_t pk = task_min<KP>(s < a.K ? (q | (uint32_t)s) : kSat);
  if (!lead) return;
  int st = CFP_ST_OK;
  if (flags & 1) st = CFP_ST_BADINPUT;
  else if (flags & 2) st = CFP_ST_INFEASIBLE;
  else if ((pk >> S::BITS) != 0) st = CFP_ST_OVERFLOW;
  a.status[b] = st;
  a.opt[b] = st == CFP_ST_OK ? total : INT64_MAX;
  a.res[b].final_state = st == CFP_ST_OK ? (int32_t)(pk & (KP - 1)) : -1;
  a.res[b].status = st;
  a.res[b].final_m = 0;
}

// Speculative (kNSpec), fix-up (kNFix) and second fix-up (kNFix2) passes; task x of
// the launch is chunk x mod P (fix-up: 1 + x mod (P-1), second: 2 + x mod (P-2)) of
// a search.  The second one runs the chunks behind a chunk that met no checkpoint,
// whose fix-up started from a row that is not the true one; a workgroup without any
// ends at once.  A wave carries 64 / KP tasks, or with SOLO one.
template <int KP, int NW, bool SOLO, int MODE, bool PER>
__global__ __launch_bounds__(64 * NW) void chain_narrow_kernel(NarrowArgs a) {
  extern __shared__ __align__(16) u32x4 tabs[];
  __shared__ int2 elist[kEdgeWords];
  constexpr int TASKS = SOLO ? 1 : 64 / KP;
  constexpr int SKIP = MODE == kNSpec ? 0 : MODE == kNFix ? 1 : 2;  // chunks that the pass does not run
  const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6), s = lane & (KP - 1);
  const int chunks = a.P - SKIP;
  const int64_t task =
      SOLO ? (int64_t)blockIdx.x * NW + wid : ((int64_t)blockIdx.x * NW + wid) * TASKS + lane / KP;
  bool valid = task < (int64_t)a.B * chunks;
  const int b = valid ? (int)(task / chunks) : 0;
  const int p = (valid ? (int)(task % chunks) : 0) + SKIP;
  const int r0 = p * a.CL, iend = min(r0 + a.CL, a.N) - 1;
  NarrowRec *rec = a.rec + (size_t)b * a.P + p;
  NarrowRun run{};
  int qmin = 0;
  bool unmet = false;  // second fix-up: the first one met no checkpoint in this chunk either
  if (MODE == kNFix) run.q = a.ckrow[((size_t)b * a.nq + (r0 / 4 - 1)) * KP + s];
  if (MODE == kNFix2) {
    valid = valid && rec[-1].conv < 0;
    if (!__syncthreads_or(valid)) return;
    unmet = rec->conv < 0;
    qmin = unmet ? iend >> 2 : rec->conv;
    if (valid) run.q = a.endrow[((size_t)b * a.P + p - 1) * KP + s];
  }
  if (PER) narrow_edges<KP>(a.em, elist);
  const bool badr = narrow_stage<KP>(a, tabs, 64 * NW);
  const bool anybad = __syncthreads_or(badr);
  constexpr int RUN = MODE == kNSpec ? kNSpec : kNFix;
  if constexpr (!SOLO) narrow_run<KP, RUN, PER>(a, tabs, elist, b, valid, r0, iend, qmin, run);
  else if (valid) narrow_solo<KP, RUN, PER>(a, tabs, elist, b, r0, iend, qmin, run);
  // of a ballot, the bits of the lane's task
  auto mine = [&](uint64_t x) __attribute__((always_inline)) {
    return (x >> (lane & ~(KP - 1))) & ((1ull << KP) - 1);
  };
  if (MODE == kNSpec) {
    const bool tneg = mine(__ballot((int32_t)run.cor < 0)) != 0;
    const int flags = (tneg || anybad ? 1 : 0) | (run.infeasible ? 2 : 0);
    const bool lead = valid && (lane & (64 / TASKS - 1)) == 0;
    if (a.P == 1) narrow_finish<KP>(a, b, run.q, (int64_t)run.dsum, flags, lead);
    else if (lead) rec->flags = flags;
  } else {
    const size_t row = ((size_t)b * a.P + p) * KP + s;
    const bool same = MODE == kNFix2 && mine(__ballot(valid && unmet && a.endrow[row] != run.q)) == 0 && unmet;
    if (!valid) return;
    if (run.conv < 0) (MODE == kNFix ? a.endrow : a.endrow2)[row] = run.q;
    if (s != 0) return;
    const int64_t d = (int64_t)(run.conv >= 0 ? run.dconv : run.dsum);
    if (MODE == kNFix) {
      rec->conv = run.conv;
      rec->dfix = d;
      rec->run2 = 0;
    } else {
      rec->conv2 = run.conv;
      rec->dfix2 = d;
      rec->run2 = 1;
      rec->same2 = same;
    }
  }
}

// Final pass, one wave per search: the chunk offsets, the reruns of chunks that no
// run started from the true row of (tables staged only then, for all searches of
// the workgroup), the final state.
template <int KP, bool PER>
__global__ __launch_bounds__(1024) void chain_narrow_final_kernel(NarrowArgs a) {
  extern __shared__ __align__(16) u32x4 tabs[];
  __shared__ int2 elist[kEdgeWords];
  const int tid = threadIdx.x, lane = tid & 63, s = lane & (KP - 1), nthreads = blockDim.x;
  const int bx = blockIdx.x * (nthreads >> 6) + __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool valid = bx < a.B;
  const int b = valid ? bx : a.B - 1, P = valid ? a.P : 0;
  const int64_t *dk = a.dck + (size_t)b * a.nq;
  const NarrowRec *rec = a.rec + (size_t)b * a.P;
  auto endq = [&](int p) __attribute__((always_inline)) { return (min((p + 1) * a.CL, a.N) - 1) >> 2; };
  int fl = 0;
  for (int p = lane; p < P; p += 64) fl |= rec[p].flags;
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) fl |= __shfl_xor(fl, off, 64);
  // Chunk 0 runs from the true first row.  The chunks below p are accounted in
  // `total`; with spec_true the speculative end row of chunk p-1 is a true row,
  // otherwise q holds the true end row of chunk p-1.  The last run of a chunk
  // counts if it started from the true end row of the chunk before: the fix-up
  // from its speculative end row, the second fix-up from the end row of its
  // fix-up.
  int64_t total = dk[endq(0)];
  bool spec_true = true;
  uint32_t q = 0;
  int p = 1;
  // Accounts the chunks whose last run counts; true if one that does not is left.
  auto settle = [&]() {
    while (p < P) {
      if (p > 1) {
        bool counts = spec_true == !rec[p].run2;
        if (counts && !spec_true) counts = __ballot(q != a.endrow[((size_t)b * P + p - 1) * KP + s]) == 0;
        if (!counts) return true;
      }
      // Up to 64 chunks at a time: the first one behind p whose last run started from
      // another row than the last run of the chunk before it ends on, and the
      // offsets of those up to there.
      const int pl = p + lane;
      const bool in = pl < P;
      NarrowRec r{};
      if (in) r = rec[pl];
      const int conv = r.run2 ? r.conv2 : r.conv, end = narrow_end(r), before = __shfl_up(end, 1, 64);
      const uint64_t bad = __ballot(in && lane > 0 && before != (r.run2 ? kEnd1 : kEndSpec));
      const int stop = bad ? p + __ffsll((long long)bad) - 1 : min(p + 64, P);
      int64_t delta = 0;
      if (in && pl < stop) {
        delta = r.run2 ? r.dfix2 : r.dfix;
        if (conv >= 0) delta += dk[endq(pl)] - dk[conv];
      }
#pragma unroll
      for (int off = 32; off >= 1; off >>= 1) delta += __shfl_xor(delta, off, 64);
      total += delta;
      const int last = __shfl(end, stop - 1 - p, 64);
      p = stop;
      spec_true = last == kEndSpec;
      if (!spec_true) q = (last == kEnd1 ? a.endrow : a.endrow2)[((size_t)b * P + p - 1) * KP + s];
    }
    return false;
  };
  bool left = settle();
  if (__syncthreads_or(left)) {
    if (PER) narrow_edges<KP>(a.em, elist);
    narrow_stage<KP>(a, tabs, nthreads);
    __syncthreads();
  }
  for (; left; left = settle()) {  // rerun chunk p from its true row, until it meets its own checkpoints
    p = __builtin_amdgcn_readfirstlane(p);  // rows are uniform
    if (spec_true) q = a.ckrow[((size_t)b * a.nq + endq(p - 1)) * KP + s];
    NarrowRun run;
    run.q = q;
    narrow_solo<KP, kNFix, PER>(a, tabs, elist, b, p * a.CL, min((p + 1) * a.CL, a.N) - 1,
                                __builtin_amdgcn_readfirstlane(narrow_qmin(rec[p], endq(p))), run);
    q = run.q;
    spec_true = run.conv >= 0;
    total += (int64_t)run.dsum;
    if (spec_true) total += dk[endq(p)] - dk[run.conv];
    ++p;
  }
  if (spec_true) q = a.ckrow[((size_t)b * a.nq + a.nq - 1) * KP + s];
  narrow_finish<KP>(a, b, q, total, fl, valid && lane == 0);
}

int narrow_kp(int k) { return k <= 16 ? 16 : 32; }

size_t narrow_lds(int k, int e) {
  const int kp = narrow_kp(k);
  return (size_t)e * kp * kp * 4;
}

// Least rows per chunk: rows on uniform costs become parallel after 6 (K = 8)
// to 9 (K = 27) rows on average and under 30 at most; shorter chunks would leave
// more of them unmet, for the second fix-up and the final pass to rerun.
int narrow_min_rows(int k) { return k <= 16 ? 24 : 32; }

struct NarrowPlan {
  int P, CL, NW, tasks;  // tasks per wave
};

// Chunks of at least narrow_min_rows rows, longer once there are more tasks
// than about four waves per SIMD.  A chain whose costs repeat with its edge
// map can settle into rows that alternate between periods; chunks of an even
// number of periods start in phase with the chain, so their rows still meet.
//
// At K > 16 a task takes a whole wave, until there are so many that their
// instructions count and not their latency (1152 blocks, K = 27: 32 searches 52 us
// per call against 60 with two tasks per wave, 512 searches 121 against 116).
//
// Workgroups of four waves while the chip holds all of them at once, as their
// tables allow (two per compute unit up to 76 KiB of tables, else one).
NarrowPlan narrow_plan(int n, int k, int e, int batch, int period) {
  const int kp = narrow_kp(k), minrows = narrow_min_rows(k);
  NarrowPlan c;
  c.tasks = kp == 16 ? 4 : (int64_t)batch * ((n + minrows - 1) / minrows) <= 16384 ? 1 : 2;
  int unit = 4;
  for (const int m : {2, 1}) {
    int u = m * period;
    while (u % 4) u += m * period;
    if (period && u <= 64) {
      unit = u;
      break;
    }
  }
  const int64_t fill = ((int64_t)batch * n + 4096 * c.tasks - 1) / (4096 * c.tasks);
  const int64_t rows = std::max<int64_t>(minrows, fill);
  c.CL = (int)((rows + unit - 1) / unit * unit);
  c.P = (n + c.CL - 1) / c.CL;
  if (n < 2 * minrows) {
    c.P = 1;
    c.CL = (n + 3) & ~3;
  }
  const int64_t waves = ((int64_t)batch * c.P + c.tasks - 1) / c.tasks;
  c.NW = waves > (narrow_lds(k, e) <= 76 * 1024 ? 2048 : 1024) ? 16 : 4;
  return c;
}

template <int KP, int NW, bool SOLO, bool PER>
hipError_t launch_narrow_passes(const NarrowArgs &a, size_t lds, hipStream_t st) {
  const int tasks = (SOLO ? 1 : 64 / KP) * NW;
  auto groups = [&](int skip) { return dim3((unsigned)(((int64_t)a.B * (a.P - skip) + tasks - 1) / tasks)); };
  timer_begin(st);
  timed_launch(chain_narrow_kernel<KP, NW, SOLO, kNSpec, PER>, groups(0), dim3(64 * NW), (uint32_t)lds, st, a);
  timer_end(st);
  if (a.P > 1) {
    hipLaunchKernelGGL((chain_narrow_kernel<KP, NW, SOLO, kNFix, PER>), groups(1), dim3(64 * NW), lds, st, a);
    if (a.second)
      hipLaunchKernelGGL((chain_narrow_kernel<KP, NW, SOLO, kNFix2, PER>), groups(2), dim3(64 * NW), lds, st, a);
    // Searches that share a workgroup's tables, so that the chip holds them all at
    // once where the tables leave room for one workgroup per compute unit.
    const int fw = a.B <= 256 ? 1 : a.B <= 1024 ? 4 : 16;
    hipLaunchKernelGGL((chain_narrow_final_kernel<KP, PER>), dim3((a.B + fw - 1) / fw), dim3(64 * fw), lds, st, a);
  }
  return hipGetLastError();
}

template <int KP, bool SOLO>
hipError_t launch_narrow_kp(const NarrowArgs &a, int nw, size_t lds, hipStream_t st) {
  const bool per = a.em.period != 0;
  if (nw == 4) return per ? launch_narrow_passes<KP, 4, SOLO, true>(a, lds, st) : launch_narrow_passes<KP, 4, SOLO, false>(a, lds, st);
  return per ? launch_narrow_passes<KP, 16, SOLO, true>(a, lds, st) : launch_narrow_passes<KP, 16, SOLO, false>(a, lds, st);
}

}  // namespace

bool chain_narrow_supported(int n, int k, int e) {
  return k <= 32 && n < (1 << 24) && narrow_lds(k, e) <= kNMaxLds;
}

size_t narrow_region_bytes(int n, int k, int e, int batch) {
  if (!chain_narrow_supported(n, k, e)) return 0;
  const size_t kp = narrow_kp(k), nq = (n + 3) / 4, pmax = n / narrow_min_rows(k) + 1;
  return align_up((size_t)batch * pmax * sizeof(NarrowRec)) + align_up((size_t)batch * nq * 8) +
         align_up((size_t)batch * nq * kp * 4) + 2 * align_up((size_t)batch * pmax * kp * 4);
}

hipError_t launch_chain_narrow(const cfp_chain_desc &d, const int32_t *redge_dev, const EdgeMap &em, uint8_t *region,
                               uint8_t *table, SearchResult *res, int64_t *opt, int32_t *status, hipStream_t st) {
  NarrowArgs a;
  a.em = em;
  const NarrowPlan c = narrow_plan(d.n_blocks, d.k, d.n_tables, d.batch, a.em.period);
  const size_t kp = narrow_kp(d.k);
  a.cost = d.cost;
  a.rtab = d.rtab;
  a.redge = redge_dev;
  a.N = d.n_blocks;
  a.K = d.k;
  a.E = d.n_tables;
  a.B = d.batch;
  a.P = c.P;
  a.CL = c.CL;
  a.second = c.P >= kNSecond;
  a.nq = (d.n_blocks + 3) / 4;
  a.rlimit = cfp_r_limit(CFP_V_CHAIN, d.k);
  a.table = table;
  size_t off = 0;
  a.rec = (NarrowRec *)(region + off);
  off += align_up((size_t)d.batch * c.P * sizeof(NarrowRec));
  a.dck = (int64_t *)(region + off);
  off += align_up((size_t)d.batch * a.nq * 8);
  a.ckrow = (uint32_t *)(region + off);
  off += align_up((size_t)d.batch * a.nq * kp * 4);
  a.endrow = (uint32_t *)(region + off);
  off += align_up((size_t)d.batch * c.P * kp * 4);
  a.endrow2 = (uint32_t *)(region + off);
  a.res = res;
  a.opt = opt;
  a.status = status;
  const size_t lds = narrow_lds(d.k, d.n_tables);
  if (kp == 16) return launch_narrow_kp<16, false>(a, c.NW, lds, st);
  return c.tasks == 1 ? launch_narrow_kp<32, true>(a, c.NW, lds, st) : launch_narrow_kp<32, false>(a, c.NW, lds, st);
}

}  // namespace cfp
