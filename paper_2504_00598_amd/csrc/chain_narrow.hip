// Forward pass of the chain search for K <= 32 (Sec. 4.4, Eq. T recurrence),
// chunk-parallel on long chains.
//
// A chain of N-1 dependent steps is cut into P chunks that run at once, made
// exact by rank convergence (Maleki, Musuvathi and Mytkowicz, PPoPP 2014), as
// in the K <= 64 form: a speculative pass starts every chunk from its first
// row's costs alone, a fix-up pass reruns each chunk from the row its
// predecessor ends on until the rows meet, a final pass sums the chunk offsets
// and reruns the chunks whose predecessor never met.  A chain of one chunk is
// finished by the speculative pass itself.
//
// At K <= 32 a step is 16 or 32 candidates per state: what bounds it is the
// latency of the dependent instructions of a step (a few hundred cycles) and,
// for a whole call, the launches.  So
//   * a task (one chunk of one search) takes KP = 16 or 32 lanes, and a wave
//     carries 64 / KP independent tasks: the row broadcasts of the previous row
//     stay within a row of 16 lanes (KP = 16) or come from one permlane swap
//     (KP = 32), and no LDS exchange or barrier is in the loop;
//   * all the packed tables stay in LDS (4 KiB each at KP = 32), staged and
//     range-checked once per workgroup from the caller's tables; a row's words
//     are read one row ahead, its costs eight rows ahead;
//   * a periodic edge map (period up to 64) travels in the launch's arguments,
//     so no header is uploaded and no packing kernel runs.
// On 1152 blocks, K = 27, 32 searches the sequential kernel that this replaces
// took 257 us.
//
// Normalisation and packing are those of the K <= 64 form: candidates are
// (Q[t] << b) + ((R[t][s] << b) | t), x[s] = (m >> b) + c[i][s], d = min_s x[s],
// Q[s] = min(x[s] - d, 2^(31-b) - 1).  R < 2^(30-b), so no candidate wraps, and
// a capped state is beaten through the row's minimum.
#include <algorithm>

#include "res_common.h"

namespace cfp {

namespace {

constexpr int kNSpec = 0, kNFix = 1;
constexpr uint32_t kNX = 0xFFFFFFFFu;    // x of an unavailable or padding state
constexpr int kNRing = 8;                // rows of costs in flight
constexpr size_t kNMaxLds = 152 * 1024;  // packed tables of a workgroup

template <int KP>
struct NarrowShape {
  static constexpr int BITS = KP <= 16 ? 4 : 5;
  static constexpr int TASKS = 64 / KP;        // tasks per wave
  static constexpr int CH = KP / 4;            // 16-byte pieces of a table column
  static constexpr int TABLE16 = KP * KP / 4;  // 16-byte pieces of a table
  static constexpr uint32_t QCAP = (1u << (31 - BITS)) - 1u;
};

struct NarrowRec {
  int64_t dfix;   // fix-up: offset sum at the meeting checkpoint, or at the chunk end
  int32_t flags;  // speculative pass: bit 0 a value out of range, bit 1 a row with no available strategy
  int32_t conv;   // fix-up: quad of the meeting checkpoint, -1 if none
};

struct NarrowArgs {
  const int32_t *cost;
  const int32_t *rtab;
  const int32_t *redge;  // device copy of the edge map; used when period is 0
  int N, K, E, B, P, CL, nq;  // CL rows per chunk (a multiple of 4), nq quads of rows
  int32_t rlimit;
  uint8_t *table;    // argmin entries [B][N][K]
  NarrowRec *rec;    // [B][P]
  int64_t *dck;      // speculative offset sum (from the chunk's start row) at every quad end [B][nq]
  uint32_t *ckrow;   // speculative row at every quad end [B][nq][KP]
  uint32_t *endrow;  // fix-up end row of chunks that met no checkpoint [B][P][KP]
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
__device__ __forceinline__ void narrow_run(const NarrowArgs &a, const u32x4 *tabs, const int *emap, int b,
                                           bool valid, int r0, int iend, int qmin, NarrowRun &run) {
  using S = NarrowShape<KP>;
  constexpr int CH = S::CH;
  const int lane = threadIdx.x & 63, s = lane & (KP - 1);
  const int K = a.K;
  const bool sin = s < K;
  const int32_t *cb = a.cost + (size_t)b * a.N * K + min(s, K - 1);
  uint8_t *tb = a.table + (size_t)b * a.N * K + s;
  uint32_t *ckb = a.ckrow + (size_t)b * a.nq * KP + s;
  auto cost_at = [&](int row) __attribute__((always_inline)) {
    return (uint32_t)cb[__umul24((uint32_t)min(row, iend), (uint32_t)K)];
  };
  uint32_t cs[kNRing];
  int er[kNRing];  // table of the row (edge map in memory)
#pragma unroll
  for (int j = 0; j < kNRing; ++j) {
    cs[j] = cost_at(r0 + j);
    if (!PER) er[j] = a.redge[min(r0 + j, iend)];
  }
  // Periodic edge map: e1 is the table of the next row, ph the phase of the row
  // after that one.
  int ph = 0, e1 = 0;
  auto next_phase = [&](int x) __attribute__((always_inline)) {
    return x + 1 == a.em.head + a.em.period ? a.em.head : x + 1;
  };
  int e0;
  if (PER) {
    ph = a.em.place(r0);
    e0 = emap[ph];
    ph = next_phase(ph);
    e1 = emap[ph];
    ph = next_phase(ph);
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
  for (int c = 0; c < CH; ++c) w[0][c] = tabs[e0 * S::TABLE16 + c * KP + s];
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
      en = e1;
      e1 = emap[ph];
      ph = next_phase(ph);
    } else {
      en = er[(J + 1) % kNRing];
      er[J] = a.redge[min(row + kNRing, iend)];
    }
#pragma unroll
    for (int c = 0; c < CH; ++c) w[nxt][c] = tabs[en * S::TABLE16 + c * KP + s];

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
    cs[J] = cost_at(row + kNRing);
    const uint32_t x = sin && cv != (uint32_t)CFP_COST_INF ? (acc >> S::BITS) + cv : kNX;
    const uint32_t d = task_min<KP>(x);
    const uint32_t qn = umin(x - d, S::QCAP) << S::BITS;
    if (act) {
      q = qn;
      dsum += d;
      if (MODE == kNSpec) run.infeasible |= d == kNX;
    }
    if (act && sin) tb[(size_t)__umul24((uint32_t)row, (uint32_t)K)] = (uint8_t)(acc & (KP - 1));
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

// Speculative (kNSpec) and fix-up (kNFix) passes; task x of the launch is
// chunk x mod P (fix-up: 1 + x mod (P-1)) of search x / P.
template <int KP, int NW, int MODE, bool PER>
__global__ __launch_bounds__(64 * NW) void chain_narrow_kernel(NarrowArgs a) {
  using S = NarrowShape<KP>;
  extern __shared__ __align__(16) u32x4 tabs[];
  __shared__ int emap[kEdgeWords];
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6, s = lane & (KP - 1);
  const int chunks = MODE == kNSpec ? a.P : a.P - 1;
  const int64_t task = ((int64_t)blockIdx.x * NW + wid) * S::TASKS + lane / KP;
  const bool valid = task < (int64_t)a.B * chunks;
  const int b = valid ? (int)(task / chunks) : 0;
  const int p = (valid ? (int)(task % chunks) : 0) + (MODE == kNSpec ? 0 : 1);
  const int r0 = p * a.CL, iend = min(r0 + a.CL, a.N) - 1;
  NarrowRun run;
  run.q = 0;
  if (MODE == kNFix) run.q = a.ckrow[((size_t)b * a.nq + (r0 / 4 - 1)) * KP + s];
  if (PER && tid < kEdgeWords) emap[tid] = a.em.map[tid];
  const bool badr = narrow_stage<KP>(a, tabs, 64 * NW);
  const bool anybad = __syncthreads_or(badr);
  narrow_run<KP, MODE, PER>(a, tabs, emap, b, valid, r0, iend, 0, run);
  if (MODE == kNSpec) {
    const uint64_t neg = __ballot((int32_t)run.cor < 0);
    const bool tneg = ((neg >> (lane & ~(KP - 1))) & ((1ull << KP) - 1)) != 0;
    const int flags = (tneg || anybad ? 1 : 0) | (run.infeasible ? 2 : 0);
    if (a.P == 1) narrow_finish<KP>(a, b, run.q, (int64_t)run.dsum, flags, valid && s == 0);
    else if (valid && s == 0) a.rec[(size_t)b * a.P + p].flags = flags;
  } else if (valid) {
    if (run.conv < 0) a.endrow[((size_t)b * a.P + p) * KP + s] = run.q;
    if (s == 0) {
      NarrowRec &r = a.rec[(size_t)b * a.P + p];
      r.conv = run.conv;
      r.dfix = (int64_t)(run.conv >= 0 ? run.dconv : run.dsum);
    }
  }
}

// Final pass, one wave per search: the chunk offsets, the reruns after chunks
// whose fix-up met no checkpoint (tables staged only then), the final state.
template <int KP, bool PER>
__global__ __launch_bounds__(64) void chain_narrow_final_kernel(NarrowArgs a) {
  extern __shared__ __align__(16) u32x4 tabs[];
  __shared__ int emap[kEdgeWords];
  const int lane = threadIdx.x, s = lane & (KP - 1);
  const int b = blockIdx.x, P = a.P;
  const int64_t *dk = a.dck + (size_t)b * a.nq;
  const NarrowRec *rec = a.rec + (size_t)b * P;
  auto endq = [&](int p) __attribute__((always_inline)) { return (min((p + 1) * a.CL, a.N) - 1) >> 2; };
  int fl = 0;
  for (int p = lane; p < P; p += 64) fl |= rec[p].flags;
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) fl |= __shfl_xor(fl, off, 64);
  // Chunk 0 runs from the true first row.  At the top of the loop the chunks
  // below p are accounted in `total`; with spec_true the speculative end row of
  // chunk p-1 is its true one (so the fix-up of chunk p is valid), otherwise q
  // holds the true end row of chunk p-1.
  int64_t total = dk[endq(0)];
  bool spec_true = true, staged = false;
  uint32_t q = 0;
  int p = 1;
  while (p < P) {
    if (spec_true) {  // up to 64 chunks at a time
      const int pl = p + lane;
      const bool in = pl < P;
      NarrowRec r{};
      if (in) r = rec[pl];
      const uint64_t nc = __ballot(in && r.conv < 0);
      const int stop = nc ? p + __ffsll((long long)nc) - 1 : min(p + 64, P);
      int64_t delta = 0;
      if (in && pl < stop) delta = r.dfix + dk[endq(pl)] - dk[r.conv];
      else if (in && nc && pl == stop) delta = r.dfix;  // ran from a true row to its end
#pragma unroll
      for (int off = 32; off >= 1; off >>= 1) delta += __shfl_xor(delta, off, 64);
      total += delta;
      p = stop;
      if (nc) {
        q = a.endrow[((size_t)b * P + stop) * KP + s];
        spec_true = false;
        ++p;
      }
    } else {
      // Rerun chunk p (the first task of the wave) from q, at least over the
      // rows its fix-up rewrote from a wrong start.
      if (!staged) {
        if (PER && lane < kEdgeWords) emap[lane] = a.em.map[lane];
        narrow_stage<KP>(a, tabs, 64);
        staged = true;
        __syncthreads();
      }
      NarrowRun run;
      run.q = q;
      const int qmin = rec[p].conv < 0 ? endq(p) : rec[p].conv;
      narrow_run<KP, kNFix, PER>(a, tabs, emap, b, lane < KP, p * a.CL, min((p + 1) * a.CL, a.N) - 1, qmin, run);
      const int conv = __builtin_amdgcn_readfirstlane(run.conv);
      const uint64_t d = conv >= 0 ? run.dconv : run.dsum;
      total += (int64_t)__shfl((long long)d, 0, 64);
      spec_true = conv >= 0;
      if (spec_true) total += dk[endq(p)] - dk[conv];
      q = (uint32_t)__shfl((int)run.q, s, 64);
      ++p;
    }
  }
  if (spec_true) q = a.ckrow[((size_t)b * a.nq + a.nq - 1) * KP + s];
  narrow_finish<KP>(a, b, q, total, fl, lane == 0);
}

int narrow_kp(int k) { return k <= 16 ? 16 : 32; }

size_t narrow_lds(int k, int e) {
  const int kp = narrow_kp(k);
  return (size_t)e * kp * kp * 4;
}

// Least rows per chunk: rows on uniform costs become parallel after 6 (K = 8)
// to 9 (K = 27) rows on average and under 30 at most, and a chunk shorter than
// that would have to be rerun in turn.
int narrow_min_rows(int k) { return k <= 16 ? 24 : 32; }

struct NarrowPlan {
  int P, CL, NW;
};

// Chunks of at least narrow_min_rows rows, longer once there are more tasks
// than about four waves per SIMD.  A chain whose costs repeat with its edge
// map can settle into rows that alternate between periods; chunks of an even
// number of periods start in phase with the chain, so their rows still meet.
NarrowPlan narrow_plan(int n, int k, int batch, int period) {
  const int tasks = 64 / narrow_kp(k);
  int unit = 4;
  for (const int m : {2, 1}) {
    int u = m * period;
    while (u % 4) u += m * period;
    if (period && u <= 64) {
      unit = u;
      break;
    }
  }
  const int64_t fill = ((int64_t)batch * n + 4096 * tasks - 1) / (4096 * tasks);
  const int64_t rows = std::max<int64_t>(narrow_min_rows(k), fill);
  NarrowPlan c;
  c.CL = (int)((rows + unit - 1) / unit * unit);
  c.P = (n + c.CL - 1) / c.CL;
  if (n < 2 * narrow_min_rows(k)) {
    c.P = 1;
    c.CL = (n + 3) & ~3;
  }
  const int64_t waves = ((int64_t)batch * c.P + tasks - 1) / tasks;
  c.NW = waves > 2048 ? 16 : 4;
  return c;
}

template <int KP, int NW, bool PER>
hipError_t launch_narrow_passes(const NarrowArgs &a, size_t lds, hipStream_t st) {
  const int tasks = NarrowShape<KP>::TASKS * NW;
  const int64_t spec = ((int64_t)a.B * a.P + tasks - 1) / tasks;
  const int64_t fix = ((int64_t)a.B * (a.P - 1) + tasks - 1) / tasks;
  timer_begin(st);
  timed_launch(chain_narrow_kernel<KP, NW, kNSpec, PER>, dim3((unsigned)spec), dim3(64 * NW), (uint32_t)lds, st, a);
  timer_end(st);
  if (a.P > 1) {
    hipLaunchKernelGGL((chain_narrow_kernel<KP, NW, kNFix, PER>), dim3((unsigned)fix), dim3(64 * NW), lds, st, a);
    hipLaunchKernelGGL((chain_narrow_final_kernel<KP, PER>), dim3(a.B), dim3(64), lds, st, a);
  }
  return hipGetLastError();
}

template <int KP>
hipError_t launch_narrow_kp(const NarrowArgs &a, int nw, size_t lds, hipStream_t st) {
  if (nw == 4)
    return a.em.period ? launch_narrow_passes<KP, 4, true>(a, lds, st) : launch_narrow_passes<KP, 4, false>(a, lds, st);
  return a.em.period ? launch_narrow_passes<KP, 16, true>(a, lds, st) : launch_narrow_passes<KP, 16, false>(a, lds, st);
}

}  // namespace

bool chain_narrow_supported(int n, int k, int e) {
  return k <= 32 && n < (1 << 24) && narrow_lds(k, e) <= kNMaxLds;
}

size_t narrow_region_bytes(int n, int k, int e, int batch) {
  if (!chain_narrow_supported(n, k, e)) return 0;
  const size_t kp = narrow_kp(k), nq = (n + 3) / 4, pmax = n / narrow_min_rows(k) + 1;
  return align_up((size_t)batch * pmax * sizeof(NarrowRec)) + align_up((size_t)batch * nq * 8) +
         align_up((size_t)batch * nq * kp * 4) + align_up((size_t)batch * pmax * kp * 4);
}

hipError_t launch_chain_narrow(const cfp_chain_desc &d, const int32_t *redge_dev, const EdgeMap &em, uint8_t *region,
                               uint8_t *table, SearchResult *res, int64_t *opt, int32_t *status, hipStream_t st) {
  NarrowArgs a;
  a.em = em;
  const NarrowPlan c = narrow_plan(d.n_blocks, d.k, d.batch, a.em.period);
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
  a.res = res;
  a.opt = opt;
  a.status = status;
  const size_t lds = narrow_lds(d.k, d.n_tables);
  return kp == 16 ? launch_narrow_kp<16>(a, c.NW, lds, st) : launch_narrow_kp<32>(a, c.NW, lds, st);
}

}  // namespace cfp
