// Chunk-parallel forward pass of the chain search for 64 < K <= 512 (Sec. 4.4,
// Eq. T recurrence), for chains of at least two chunks.
//
// Parallelism over the chain: as in the K <= 64 form, every chain is cut into
// P chunks that run at once, made exact by rank convergence (Maleki,
// Musuvathi and Mytkowicz, PPoPP 2014): a recurrence started from an
// arbitrary row becomes parallel to the true one after a few steps.
//   1. speculative pass: chunk p starts at its first row from that row's costs
//      alone, writes its argmin rows and, at every quad end, its normalised row
//      and running offset (a checkpoint).  (Starting rows early saves the fix-up
//      as many rows as it adds here at K = 256: nothing gained);
//   2. fix-up pass, chunks p >= 1: start again from the last checkpoint row of
//      chunk p-1 and recompute until the row equals chunk p's checkpoint of the
//      same quad (from there on the speculative rows are the true ones);
//   3. second fix-up: the chunks behind a chunk that met no checkpoint run
//      again, all at once, from that chunk's end row, which is one chunk more of
//      history: of a run of unmet chunks it is the true row if two chunks of
//      history are enough.  (Left to the final pass they ran one after another:
//      1152 blocks, K = 256, one search, resharding never free: 1792 us per
//      call, 316 with this pass and chunks of 32 rows instead of 20.)  With
//      nothing to do it costs one empty launch;
//   4. final pass: sum the chunk offsets.  The last run of a chunk counts if it
//      started from the true end row of the chunk before (rows compared whole);
//      a chunk that none did is rerun from it.  The result is the sequential
//      recurrence's bit for bit.
//
// One workgroup of 8 waves (4 at KP = 128) carries four chains, or two in small
// batches (searches of the same chunk: every chain of a launch is at the same
// row, so all use the same table) and all KP states, KP = 128, 256 or 512.
// Wave g works for the predecessors t = g KP/8 .. (g+1) KP/8 - 1 and lane q for
// the states q KP/64 .. (q+1) KP/64 - 1 of every chain, so every table load of a
// wave reads one row's KP words contiguously (KP = 128: two rows, one per half
// of the wave).  Per step a thread reads its share of
// the packed words (R_e[t][s] << b) | t of the edge's table (each word serves
// the four chains) in pieces of a few rows, four pieces in flight in their
// own registers (up to KP = 256 that is the whole step, loaded a step ahead),
// and the predecessors' values from the previous rows in LDS (broadcast reads).
// A candidate is a saturating add, and one unsigned minimum keeps the value
// and the lowest predecessor.  The eight group minima of a state are combined
// through LDS, after which a thread holds one state of one chain (KP = 128), of
// two (256) or of all four (512).
//
// What bounds a step: at KP = 128 the instructions of a wave alone on its SIMD
// (1.8 us per row with four chains: products 0.8, the two exchanges through LDS
// and the normalisation 0.75, memory 0.25, measured with parts switched off),
// at KP = 256 both and at KP = 512 the table stream, KP^2 words per workgroup and
// step from the cache hierarchy (16.7 us per row whatever the number of
// workgroups).  (Before this form K <= 128 went through the split kernel, 1.9 us
// per row but one row after another: 1152 blocks, K = 128: 1960 to 108 us for
// one search, 2237 to 331 us for 128; 393 blocks, K = 81, 24 searches: 762 to 105
// us.)  At KP = 512 a batch of at most eight searches would leave most compute
// units idle; there teams of four workgroups split the states of each chunk
// (state-split teams, below).  Chunks are at least 32 rows long up to KP = 256 and 48 at KP = 512:
// runs become parallel after 14 rows on average and 38 at most at K = 128, 18
// and about 40 at K = 256, 21 and 50 at K = 512 (uniform random costs).
//
// Normalisation: x[s] = (m >> b) + c[i][s]; the row is divided into the part
// d = min_s x[s] (summed exactly, per chain) and Q[s] = min(x[s] - d, cap) << b,
// cap = 2^(32-b) - 1.  The best candidate of every state is at most
// R_max << b | t through the row's minimum, so with R below cfp_r_limit a
// capped state never wins; unavailable strategies and padding states take
// x = 2^32 - 1 (capped).
#include <algorithm>
#include <type_traits>

#include "cfp_internal.h"
#include "common.h"

namespace cfp {

namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kCThreads = 512;          // threads per workgroup
constexpr int kCWaves = kCThreads / 64;
constexpr uint32_t kCX = 0xFFFFFFFFu;   // x of an unavailable or padding state
constexpr int kCMaxChunks = 64;
constexpr int kCG = 4;                  // chains per workgroup (searches of the same chunk); 2 in small batches
// Passes: speculative; fix-up (a run stops once every chain met a checkpoint);
// second fix-up, of the chunks behind one that met none in the first.
constexpr int kCSpec = 0, kCFix = 1, kCFix2 = 2;

template <int KP, int CG>
struct CwShape {
  static constexpr int BITS = KP <= 128 ? 7 : KP <= 256 ? 8 : 9;  // index bits of a packed word
  static constexpr int THREADS = KP <= 128 ? 256 : 512;
  static constexpr int WAVES = THREADS / 64;
  static constexpr int NH = KP <= 128 ? 2 : 1;      // table rows per load instruction of a wave
  static constexpr int PG = KP / (WAVES * NH);      // predecessors per wave (NH = 2: per half of it)
  static constexpr int SPL = KP * NH / 64;          // states per lane in the products
  static constexpr int VW = 4;                      // words per table load
  static constexpr int NV = SPL / VW;               // loads per table row and lane
  static constexpr int ROWS = KP <= 128 ? 4 : KP <= 256 ? 8 : 2;  // table rows per piece
  static constexpr int PIECES = PG / ROWS;          // pieces per step
  static constexpr int NB = 4;                      // pieces held in registers
  static constexpr int TPS = THREADS / KP;        // threads per state after the reduction
  static constexpr int CH = CG / TPS;              // chains per thread after the reduction
  static constexpr int WPS = KP / 64;               // waves that hold the same chains after the reduction
  static constexpr int GROUPS = WAVES * NH;         // predecessor groups
  static constexpr int QS = KP + KP / 8;            // LDS row stride: 4 words of padding after every 32
  static constexpr int QH = QS / NH;                // NH = 2: odd predecessors follow the even ones
  static constexpr int MINROWS = KP <= 256 ? 32 : 48;            // least rows per chunk
  static constexpr uint32_t CAP = (1u << (32 - BITS)) - 1u;
  using Arg = typename std::conditional<(KP <= 256), uint8_t, uint16_t>::type;
  typedef uint32_t Vec __attribute__((ext_vector_type(VW)));
  static_assert(PIECES % NB == 0 && ROWS % 2 == 0 && SPL % VW == 0 && TPS * CH == CG, "piece layout");
};

struct CwRec {
  int64_t dfix;   // fix-up pass: offset sum at the meeting checkpoint, or at the chunk end
  int64_t dfix2;  // the same of the second fix-up
  int32_t flags;  // bit 0 a negative cost, bit 1 a row with no available strategy (speculative
                  // pass); bit 2 a wait between the workgroups of a team expired
  int32_t conv;   // fix-up pass: quad of the meeting checkpoint, -1 if none
  int32_t conv2;  // the same of the second fix-up
  int32_t run2;   // the second fix-up ran this chunk (from the first one's end row of the chunk before)
  int32_t same2;  // and met no checkpoint, but ended on the first one's end row of this chunk
};

struct CwArgs {
  const int32_t *cost;
  const uint32_t *rpk;  // packed tables [E][KP][KP]
  const int32_t *redge;
  int N, K, B, P, CL, nq;  // CL rows per chunk (a multiple of 4); nq quads of rows
  uint8_t *table;          // argmin entries [B][N][K] (1 byte for KP <= 256, 2 for 512)
  CwRec *rec;              // [B][P]
  int64_t *dck;            // speculative offset sum at every checkpoint [B][nq]
  uint32_t *ckrow;         // speculative row at every checkpoint [B][nq][KP]
  uint32_t *endrow;        // fix-up end row of chunks that met no checkpoint [B][P][KP]
  uint32_t *endrow2;       // the same of the second fix-up
  const int32_t *rbad;     // range flags of R, one per packing workgroup
  int nbad;
  uint64_t *xb;            // state-split teams: exchanged rows [team][slot][chain][KP]
  int32_t *xflag;          // state-split teams: a member gave up waiting [team]
};

template <int KP, int CG>
struct CwSmem {
  uint32_t part[CG][CwShape<KP, CG>::GROUPS][KP];         // partial minima [chain][predecessor group][state]
  uint32_t q[2][CG][CwShape<KP, CG>::QS];     // rows [buffer][chain][state, padded]
  uint32_t wm[CwShape<KP, CG>::WAVES][CwShape<KP, CG>::CH];   // wave minima of the new row, per chain of the wave
  int32_t wd[CwShape<KP, CG>::WAVES][CwShape<KP, CG>::CH];    // fix-up: the wave found a state off the checkpoint
};

__device__ __forceinline__ int qpad(int t) { return t + (t >> 5) * 4; }
// LDS position of predecessor t in a row.
template <int KP, int CG>
__device__ __forceinline__ int qat(int t) {
  return CwShape<KP, CG>::NH == 1 ? qpad(t) : (t & 1) * CwShape<KP, CG>::QH + qpad(t >> 1);
}

// min(keep, the partner lane's send): quad_perm partners lane ^ 1 and lane ^ 2;
// the half mirror pairs lane i with lane 7 - i of its eight.
template <int CTRL>
__device__ __forceinline__ uint32_t min_dpp(uint32_t keep, uint32_t send) {
  return umin(keep, (uint32_t)__builtin_amdgcn_mov_dpp((int)send, CTRL, 0xF, 0xF, true));
}
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppHalfMirror = 0x141, kDppMirror = 0x140;

// Minimum over the 64 lanes of a wave (every lane gets it).
__device__ __forceinline__ uint32_t cw_wave_min(uint32_t x) {
  x = min_dpp<kDppXor1>(x, x);
  x = min_dpp<kDppXor2>(x, x);
  x = min_dpp<kDppHalfMirror>(x, x);
  x = min_dpp<kDppMirror>(x, x);
  const auto h = __builtin_amdgcn_permlane32_swap(x, x, false, false);
  x = umin(h[0], h[1]);
  const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
  return umin(r[0], r[1]);
}

// State of the workgroup's chains as seen by one thread.  After the
// reduction thread tid holds, for its state s = tid % KP, the chains
// h TPS + tid / KP, h = 0 .. CH - 1.
template <int KP, int CG>
struct CwChains {
  uint32_t x[CwShape<KP, CG>::CH];  // the thread's values of the current row, normalised and shifted
  uint64_t dsum[CG];   // offset sums since the start row (uniform)
  int conv[CG];        // fix-up: quad of the meeting checkpoint, -1 before
  uint64_t dconv[CG];  // fix-up: dsum at that checkpoint
  uint32_t flags[CG];  // speculative: bit 0 a negative cost, bit 1 a row with no available strategy
};

// Runs rows [r0, r1] of the workgroup's chains (searches bs[c], real where
// valid[c]).  Speculative: the start row is row r0 from its costs alone; argmins
// from row r0 + 1 and checkpoints are written.  Fix-up: the start row (row r0 - 1) is start[c];
// stops at the first quad end where every real chain has met its checkpoint at
// a quad not before qmin[c].
// REAL: the chains that are computed (the others' values are not meaningful).
template <int KP, int CG, int MODE, int REAL = CG>
__device__ __forceinline__ void cw_run(const CwArgs &a, const int *bs, const bool *valid, int r0, int r1,
                                       const int *qmin, const uint32_t *const *start, CwSmem<KP, CG> &sm,
                                       CwChains<KP, CG> &ch) {
  using S = CwShape<KP, CG>;
  using Arg = typename S::Arg;
  constexpr int CH = S::CH, TPS = S::TPS, BITS = S::BITS;
  constexpr bool CHECK = MODE != kCSpec;
  const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  // state group, predecessor group (one wave each; NH = 2: half a wave, rows in turn)
  const int g = wid, hw = S::NH == 1 ? 0 : lane >> 5, qd = S::NH == 1 ? lane : lane & 31;
  const int N = a.N, K = a.K;
  // the thread's state and chains after the reduction
  const int sub = TPS == 1 ? 0 : tid / KP;
  const int ms = tid & (KP - 1);
  const bool sin = ms < K;
  // element h of the thread's chains from an array indexed by chain
  auto pick = [&](const auto &arr, int h) __attribute__((always_inline)) {
    if constexpr (TPS == 1) return arr[h];
    else if constexpr (TPS == 2) return sub ? arr[2 * h + 1] : arr[2 * h];
    else return sub == 0 ? arr[0] : sub == 1 ? arr[1] : sub == 2 ? arr[2] : arr[3];
  };
  int hc[CH];  // chain of pair h
  bool hv[CH];
  // A chain's rows start at a wave-uniform address (scalar registers); the
  // thread's state adds one 32-bit byte offset, so no 64-bit address is held
  // per chain in vector registers.
  const int32_t *cbase[CH];
  Arg *tbase[CH];
  uint32_t *ckb[CH];
#pragma unroll
  for (int h = 0; h < CH; ++h) {
    hc[h] = TPS * h + sub;
    const int b = __builtin_amdgcn_readfirstlane(pick(bs, h));
    hv[h] = pick(valid, h);
    cbase[h] = a.cost + (size_t)b * N * K;
    tbase[h] = (Arg *)a.table + (size_t)b * N * K;
    ckb[h] = a.ckrow + (size_t)b * a.nq * KP;
  }
  const uint32_t coff = (uint32_t)min(ms, K - 1) * 4u, toffb = (uint32_t)ms * (uint32_t)sizeof(Arg),
                 koff = (uint32_t)ms * 4u;
  auto cost_at = [&](int h, size_t row, uint32_t off) __attribute__((always_inline)) {
    return *(const uint32_t *)((const char *)(cbase[h] + row * K) + off);
  };
  auto ck_at = [&](int h, size_t q) __attribute__((always_inline)) -> uint32_t & {
    uint32_t off = koff;
    asm volatile("" : "+v"(off));  // (no base + offset pair hoisted out of the loop, where it would spill)
    return *(uint32_t *)((char *)(ckb[h] + q * KP) + off);
  };
  // redge is read-only for the kernel's lifetime: read through the constant
  // address space, so a row's table index is one scalar load.
  const __attribute__((address_space(4))) int32_t *redge_c =
      (const __attribute__((address_space(4))) int32_t *)a.redge;
  auto edge = [&](int row) __attribute__((always_inline)) { return redge_c[row]; };
  const int i0 = MODE == kCSpec ? r0 + 1 : r0;

  // Table pieces in flight, [buffer][row in piece][vector]; word offset of the
  // thread's first word within a table.
  const uint32_t toff = (uint32_t)(S::PG * S::NH * g * KP + hw * KP + S::SPL * qd);
  typename S::Vec tb[S::NB][S::ROWS][S::NV];
  auto tload = [&](int buf, int piece, int row) __attribute__((always_inline)) {
    const uint32_t *tab = a.rpk + (size_t)edge(row) * KP * KP + toff + piece * S::ROWS * S::NH * KP;
#pragma unroll
    for (int j = 0; j < S::ROWS; ++j)
#pragma unroll
      for (int v = 0; v < S::NV; ++v) tb[buf][j][v] = *(const typename S::Vec *)(tab + j * S::NH * KP + S::VW * v);
  };
  // Row minima of every chain from the threads' values: wave minima to LDS,
  // one barrier, then the minimum over the waves (uniform).
  auto row_min = [&](const uint32_t(&x)[CH], uint32_t(&d)[CG]) __attribute__((always_inline)) {
#pragma unroll
    for (int h = 0; h < CH; ++h) {
      const uint32_t w = cw_wave_min(x[h]);
      if (lane == 0) sm.wm[wid][h] = w;
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < CG; ++c) {
      uint32_t m = kCX;
#pragma unroll
      for (int w = 0; w < S::WPS; ++w) m = umin(m, sm.wm[(c % TPS) * S::WPS + w][c / TPS]);
      d[c] = __builtin_amdgcn_readfirstlane(m);
    }
  };

  // Start row.
#pragma unroll
  for (int c = 0; c < CG; ++c) {
    ch.flags[c] = 0;
    ch.conv[c] = -1;
    ch.dconv[c] = 0;
    ch.dsum[c] = 0;
  }
  uint32_t cor[CH];
  if (MODE == kCSpec) {
    uint32_t x[CH], d[CG];
#pragma unroll
    for (int h = 0; h < CH; ++h) {
      const uint32_t cv = cost_at(h, (size_t)r0, coff);
      cor[h] = cv;
      x[h] = (sin && cv != (uint32_t)CFP_COST_INF) ? cv : kCX;
    }
    row_min(x, d);
#pragma unroll
    for (int c = 0; c < CG; ++c) {
      if (d[c] == kCX) ch.flags[c] |= 2;
      ch.dsum[c] = d[c];
    }
#pragma unroll
    for (int h = 0; h < CH; ++h) {
      ch.x[h] = umin(x[h] - pick(d, h), S::CAP) << BITS;
      sm.q[0][hc[h]][qat<KP, CG>(ms)] = ch.x[h];
    }
    if (i0 > r1) {  // a run of one row: the start row is its checkpoint
#pragma unroll
      for (int h = 0; h < CH; ++h)
        if (hv[h]) ck_at(h, (size_t)(r0 / 4)) = ch.x[h];
#pragma unroll
      for (int c = 0; c < CG; ++c)
        if (tid == c && valid[c]) a.dck[(size_t)bs[c] * a.nq + r0 / 4] = (int64_t)ch.dsum[c];
    }
  } else {
#pragma unroll
    for (int h = 0; h < CH; ++h) {
      ch.x[h] = pick(start, h)[ms];
      sm.q[0][hc[h]][qat<KP, CG>(ms)] = ch.x[h];
      cor[h] = 0;
    }
  }
  auto negative_costs = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int c = 0; c < CG; ++c)
      if (__syncthreads_or(((c % TPS) == sub) && (cor[c / TPS] >> 31))) ch.flags[c] |= 1;
  };
  if (i0 > r1) {
    if (MODE == kCSpec) negative_costs();
    return;
  }
#pragma unroll
  for (int k = 0; k < S::NB; ++k) tload(k, k, i0);
  // Costs of the next two rows, [row parity][pair]: step i uses set i - i0 mod 2
  // and reloads it with row i + 2 (the loop runs two rows per turn, so every
  // index is a constant and no register is copied from a load in flight).
  uint32_t cq[2][CH], ckv[CH];
#pragma unroll
  for (int h = 0; h < CH; ++h) {
    cq[0][h] = cost_at(h, (size_t)i0, coff);
    cq[1][h] = cost_at(h, (size_t)min(i0 + 1, r1), coff);
    ckv[h] = 0;
    if (CHECK) ckv[h] = ck_at(h, (size_t)(i0 >> 2));
  }
  __syncthreads();

  // One row i with the previous rows in LDS buffer CUR; returns true when the
  // fix-up pass is done.
  auto step = [&](int i, auto Pc) __attribute__((always_inline)) -> bool {
    constexpr int cur = decltype(Pc)::value, nxt = cur ^ 1;
    uint32_t acc[CG][S::SPL];
#pragma unroll
    for (int c = 0; c < CG; ++c)
#pragma unroll
      for (int u = 0; u < S::SPL; ++u) acc[c][u] = kSat;
    const int inext = min(i + 1, r1);
    for (int kk = 0; kk < S::PIECES; kk += S::NB) {
#pragma unroll
      for (int bb = 0; bb < S::NB; ++bb) {
        const int k = kk + bb;
        uint32_t v[CG][S::ROWS];  // the predecessors' values of this piece, per chain
#pragma unroll
        for (int c = 0; c < REAL; ++c) {
          const uint32_t *qc = &sm.q[cur][c][hw * S::QH + qpad(S::PG * g + S::ROWS * k)];
          if constexpr (S::ROWS % 4 == 0) {
#pragma unroll
            for (int r4 = 0; r4 < S::ROWS / 4; ++r4) {
              const u32x4 w = *(const u32x4 *)(qc + 4 * r4);
              v[c][4 * r4] = w.x;
              v[c][4 * r4 + 1] = w.y;
              v[c][4 * r4 + 2] = w.z;
              v[c][4 * r4 + 3] = w.w;
            }
          } else {
#pragma unroll
            for (int r2 = 0; r2 < S::ROWS / 2; ++r2) {
              const uint2 w = *(const uint2 *)(qc + 2 * r2);
              v[c][2 * r2] = w.x;
              v[c][2 * r2 + 1] = w.y;
            }
          }
        }
#pragma unroll
        for (int j = 0; j < S::ROWS; j += 2) {
#pragma unroll
          for (int vv = 0; vv < S::NV; ++vv) {
            const typename S::Vec w = tb[bb][j][vv], y = tb[bb][j + 1][vv];
#pragma unroll
            for (int c = 0; c < REAL; ++c) {
              uint32_t *ac = &acc[c][S::VW * vv];
#pragma unroll
              for (int u = 0; u < S::VW; ++u)
                ac[u] = umin(umin(ac[u], sat_add(v[c][j], w[u])), sat_add(v[c][j + 1], y[u]));
            }
          }
        }
        // the registers just consumed take the piece NB further on (of this row or the next)
        const int nk = k + S::NB;
        if (nk < S::PIECES) tload(bb, nk, i);
        else tload(bb, nk - S::PIECES, inext);
      }
    }
    // Minima over the eight predecessor groups (one wave each) through LDS.
#pragma unroll
    for (int c = 0; c < REAL; ++c)
#pragma unroll
      for (int vv = 0; vv < S::NV; ++vv) {
        typename S::Vec pv;
#pragma unroll
        for (int u = 0; u < S::VW; ++u) pv[u] = acc[c][S::VW * vv + u];
        *(typename S::Vec *)&sm.part[c][g * S::NH + hw][S::SPL * qd + S::VW * vv] = pv;
      }
    __syncthreads();
    uint32_t m[CH];
#pragma unroll
    for (int h = 0; h < CH; ++h) {
      const int c = hc[h];
      uint32_t v = sm.part[c][0][ms];
#pragma unroll
      for (int w = 1; w < S::GROUPS; ++w) v = umin(v, sm.part[c][w][ms]);
      m[h] = v;
    }

    // New row: the thread's chains.
    uint32_t x[CH];
#pragma unroll
    for (int h = 0; h < CH; ++h) {
      const uint32_t cv = cq[cur][h];
      if (MODE == kCSpec) {
        cor[h] |= cv;
        asm volatile("" : "+v"(cor[h]));  // kept in its step (not sunk behind the argmin stores)
      }
      x[h] = (sin && cv != (uint32_t)CFP_COST_INF) ? (m[h] >> BITS) + cv : kCX;
      if (sin && hv[h])
        *(Arg *)((char *)(tbase[h] + (size_t)i * K) + toffb) = (Arg)(m[h] & (KP - 1));
    }
    // The costs of row i + 2, into the registers just read.  The lane offset
    // passes through an empty asm that also takes x[h], so the load cannot be
    // issued before the last read of the old cost: the set keeps its registers
    // and no register copy at the end of the loop waits for a load.
#pragma unroll
    for (int h = 0; h < CH; ++h) {
      uint32_t off = coff;
      asm volatile("" : "+v"(off) : "v"(x[h]));
      cq[cur][h] = cost_at(h, (size_t)min(i + 2, r1), off);
    }
    uint32_t d[CG];
    row_min(x, d);
#pragma unroll
    for (int c = 0; c < CG; ++c) {
      if (MODE == kCSpec && d[c] == kCX) ch.flags[c] |= 2;
      ch.dsum[c] += d[c];
    }
#pragma unroll
    for (int h = 0; h < CH; ++h) {
      ch.x[h] = umin(x[h] - pick(d, h), S::CAP) << BITS;
      sm.q[nxt][hc[h]][qat<KP, CG>(ms)] = ch.x[h];
    }
    const bool qend = (i & 3) == 3 || i == r1;
    if (qend) {
      const int q = i >> 2;
      if (MODE == kCSpec) {
#pragma unroll
        for (int h = 0; h < CH; ++h)
          if (hv[h]) ck_at(h, (size_t)q) = ch.x[h];
#pragma unroll
        for (int c = 0; c < CG; ++c)
          if (tid == c && valid[c]) a.dck[(size_t)bs[c] * a.nq + q] = (int64_t)ch.dsum[c];
      }
      if (CHECK) {
#pragma unroll
        for (int h = 0; h < CH; ++h) {
          const uint64_t off = __ballot(ch.x[h] != ckv[h]);
          if (lane == 0) sm.wd[wid][h] = off != 0;
        }
        if (i < r1) {
#pragma unroll
          for (int h = 0; h < CH; ++h) ckv[h] = ck_at(h, (size_t)(q + 1));
        }
      }
    }
    __syncthreads();
    if (CHECK && qend) {
      const int q = i >> 2;
      bool all = true;
#pragma unroll
      for (int c = 0; c < CG; ++c) {
        bool same = true;
#pragma unroll
        for (int w = 0; w < S::WPS; ++w) same = same && !sm.wd[(c % TPS) * S::WPS + w][c / TPS];
        if (ch.conv[c] < 0 && same && q >= qmin[c]) {
          ch.conv[c] = q;
          ch.dconv[c] = ch.dsum[c];
        }
        all = all && (ch.conv[c] >= 0 || !valid[c]);
      }
      if (all) return true;
    }
    return false;
  };
  for (int i = i0; i <= r1; i += 2) {
    if (step(i, std::integral_constant<int, 0>{})) break;
    if (i + 1 > r1 || step(i + 1, std::integral_constant<int, 1>{})) break;
  }
  if (MODE == kCSpec) negative_costs();
}

// Whether the second fix-up runs chunk p of a search: the fix-up of chunk p-1
// met no checkpoint, so that of chunk p started from a row that is not the true
// one.
__device__ __forceinline__ bool cw_second(const CwRec *rec, int p) { return p >= 2 && rec[p - 1].conv < 0; }

// The row that the last run of a chunk ends on: its speculative end row, the end
// row of its fix-up (which the next chunk's second fix-up starts from), or that
// of its second fix-up.
enum { kEndSpec, kEnd1, kEnd2 };
__device__ __forceinline__ int cw_end(const CwRec &r) {
  if (r.run2) return r.conv2 >= 0 ? kEndSpec : r.same2 ? kEnd1 : kEnd2;
  return r.conv >= 0 ? kEndSpec : kEnd1;
}

// Quad a rerun of chunk p (last quad qe) must reach before it may stop: past
// every row that earlier runs from other start rows rewrote.
__device__ __forceinline__ int cw_qmin(const CwRec &r, int qe) {
  int q = r.conv < 0 ? qe : r.conv;
  if (r.run2) q = max(q, r.conv2 < 0 ? qe : r.conv2);
  return q;
}

// Speculative (MODE kCSpec, grid (ceil(B/CG), P)), fix-up (kCFix, grid
// (ceil(B/CG), P-1)) and second fix-up (kCFix2, grid (ceil(B/CG), P-2))
// passes.  A search takes part in the second one where cw_second says so.
template <int KP, int CG, int MODE>
__global__ __launch_bounds__((CwShape<KP, CG>::THREADS), 1) void chain_cw_kernel(CwArgs a) {
  using S = CwShape<KP, CG>;
  __shared__ __align__(16) CwSmem<KP, CG> sm;
  const int p = blockIdx.y + (MODE == kCSpec ? 0 : MODE == kCFix ? 1 : 2);
  const int r0 = p * a.CL, r1 = min(r0 + a.CL, a.N) - 1;
  int bs[CG], qmin[CG];
  bool valid[CG];
  const uint32_t *start[CG];
  bool any = false;
#pragma unroll
  for (int c = 0; c < CG; ++c) {
    const int b = CG * blockIdx.x + c;
    valid[c] = b < a.B;
    bs[c] = min(b, a.B - 1);
    qmin[c] = 0;
    start[c] = a.ckrow + ((size_t)bs[c] * a.nq + (r0 > 0 ? r0 / 4 - 1 : 0)) * KP;
    if (MODE == kCFix2) {
      const CwRec *rec = a.rec + (size_t)bs[c] * a.P;
      valid[c] = valid[c] && cw_second(rec, p);
      if (valid[c]) start[c] = a.endrow + ((size_t)bs[c] * a.P + p - 1) * KP;
      qmin[c] = rec[p].conv < 0 ? r1 >> 2 : rec[p].conv;
    }
    any = any || valid[c];
  }
  if (MODE == kCFix2 && !any) return;
  CwChains<KP, CG> ch;
  cw_run<KP, CG, MODE == kCSpec ? kCSpec : kCFix>(a, bs, valid, r0, r1, qmin, start, sm, ch);
  const int tid = threadIdx.x;
  const int sub = S::TPS == 1 ? 0 : tid / KP;
  const int ms = tid & (KP - 1);
  if (MODE == kCSpec) {
#pragma unroll
    for (int c = 0; c < CG; ++c)
      if (tid == 0 && valid[c]) a.rec[(size_t)bs[c] * a.P + p].flags = (int32_t)ch.flags[c];
  } else {
#pragma unroll
    for (int c = 0; c < CG; ++c)
      if (c % S::TPS == sub && valid[c] && ch.conv[c] < 0)
        (MODE == kCFix ? a.endrow : a.endrow2)[((size_t)bs[c] * a.P + p) * KP + ms] = ch.x[c / S::TPS];
    bool same[CG];  // second fix-up: the end row is the first one's (which then met no checkpoint either)
#pragma unroll
    for (int c = 0; c < CG; ++c) {
      same[c] = false;
      if (MODE == kCFix2) {
        const size_t at = (size_t)bs[c] * a.P + p;
        const bool unmet = a.rec[at].conv < 0;  // uniform
        const bool off = unmet && c % S::TPS == sub && a.endrow[at * KP + ms] != ch.x[c / S::TPS];
        same[c] = !__syncthreads_or(off) && unmet;
      }
    }
#pragma unroll
    for (int c = 0; c < CG; ++c) {
      if (tid != c || !valid[c]) continue;
      CwRec &r = a.rec[(size_t)bs[c] * a.P + p];
      const int64_t d = (int64_t)(ch.conv[c] >= 0 ? ch.dconv[c] : ch.dsum[c]);
      if (MODE == kCFix) {
        r.conv = ch.conv[c];
        r.dfix = d;
        r.run2 = 0;
      } else {
        r.conv2 = ch.conv[c];
        r.dfix2 = d;
        r.run2 = 1;
        r.same2 = same[c];
      }
    }
  }
}

// ---------------------------------------------------------------------------
// State-split teams (KP = 512 with few searches).  Four chains fill one
// workgroup, so a batch of a few searches leaves most compute units idle while
// each workgroup streams the whole 1 MiB table of every step.  Here a team of
// kXS workgroups carries the four chains of one chunk: part z computes the
// states z W .. z W + W - 1 (W = KP / kXS) of all four chains and so streams
// only those W columns of the table (a quarter).  After each row the parts
// exchange their new values x[s] (before normalisation) as 64-bit words
// (tag << 32) | x through device memory, every part gathers the whole row, and
// all parts normalise it the same way, exactly as one workgroup would.  A
// word's tag is its row (with the top bits set in the fix-up passes), and each
// team has two slots used in turn: a part publishes row i + 2 only after it
// has gathered row i + 1, which every part publishes only after gathering row
// i, so a slot is never rewritten before every part has read it.  Every
// decision that ends a run (the fix-up's meeting test) is taken by each part
// on the whole row, so the parts of a team always run the same rows.  All the
// workgroups of a launch must be resident at once (at most one per compute
// unit); a wait that expires marks the team, and the search ends with
// CFP_ST_TIMEOUT.

constexpr int kXS = 4;                      // workgroups per team
constexpr int kXW = 512 / kXS;              // states per part
constexpr int kXSpin = 1 << 20;             // poll rounds before a part gives up
constexpr uint32_t kXFixTag = 0x80000000u;  // tag bit of the fix-up passes
constexpr uint32_t kXFix2Tag = 0x40000000u; // and of the second one
constexpr int kXMaxGroups = 2;              // teams are used for at most 2 x 4 searches
constexpr int kXQW = kXW + kXW / 8;         // padded LDS words of one part's states

struct CxSmem {
  uint32_t part[kCG][kCWaves][kXW];      // partial minima [chain][predecessor group][state of the part]
  uint32_t q[2][kCG][CwShape<512, kCG>::QS];  // whole rows [buffer][chain][state, padded]
  uint32_t wm[kCWaves];                  // wave minima of the new row (waves 2c and 2c+1 hold chain c)
  int32_t wd[kCWaves];                   // fix-up: the wave found a state off the checkpoint
  int32_t abort;                         // a wait expired, or another part of the team gave up
};

// A thread's view after the products: chain c = tid / W... of the four chains
// (two waves each), state sl = tid % W of every part.
struct CxChains {
  uint32_t q[kXS];      // the chain's normalised, shifted values at states sl + z W, z = 0 .. kXS - 1
  uint64_t dsum[kCG];   // offset sums since the start row (uniform)
  int conv[kCG];        // fix-up: quad of the meeting checkpoint, -1 before
  uint64_t dconv[kCG];  // fix-up: dsum at that checkpoint
  uint32_t flags[kCG];  // speculative: bit 1 a row with no available strategy
  uint32_t neg;         // speculative: OR of the thread's costs (bit 31: a negative cost)
  bool aborted;
};

// Runs rows [r0, r1] of the team's chains in part z.  Speculative: the start
// row r0 comes from its costs alone; argmins from row r0 + 1 and checkpoints
// are written.  Fix-up passes: the start row (row r0 - 1) of chain c is at
// startr; stops at the first quad end where every chain of `act` (bit cc: chain
// cc is real and takes part) has met its checkpoint at a quad not before its
// qmin.
// Element idx (wave-uniform) of a four-element array, by selects rather than a
// dynamic index (which would move the array to scratch memory).
template <typename T>
__device__ __forceinline__ T sel4(const T (&v)[4], int idx) {
  return idx == 0 ? v[0] : idx == 1 ? v[1] : idx == 2 ? v[2] : v[3];
}

template <int MODE>
__device__ __forceinline__ void cx_run(const CwArgs &a, int z, int team, int grp, int r0, int r1, int act,
                                       const int (&qmin)[kCG], const uint32_t *startr, CxSmem &sm, CxChains &ch) {
  constexpr int KP = 512;
  using S = CwShape<KP, kCG>;
  constexpr int BITS = S::BITS;
  constexpr uint32_t CAP = S::CAP;
  constexpr int PG = S::PG;  // predecessors per wave
  constexpr bool FIX = MODE != kCSpec;
  constexpr uint32_t PASS = MODE == kCSpec ? 0u : MODE == kCFix ? kXFixTag : kXFixTag | kXFix2Tag;
  const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = wid >> 1;          // the thread's chain after the products (uniform in the wave)
  const int sl = tid & (kXW - 1);  // the thread's state within each part
  const int N = a.N, K = a.K;
  const int b = min(kCG * grp + c, a.B - 1);  // chains past the batch repeat the last search and write nothing
  const bool hv = (act >> c) & 1;
  const int s = z * kXW + sl;      // the thread's own state (computed by this part)
  const bool sin = s < K;
  const int qsl = qpad(sl);        // LDS index of state zz W + sl: zz kXQW + qsl
  const int32_t *cbase = a.cost + (size_t)b * N * K;
  uint16_t *tbase = (uint16_t *)a.table + (size_t)b * N * K;
  uint32_t *ckb = a.ckrow + (size_t)b * a.nq * KP;
  uint64_t *xbt = a.xb + (size_t)team * 2 * kCG * KP;
  const uint32_t coff = (uint32_t)min(s, K - 1) * 4u;
  auto cost_at = [&](size_t row, uint32_t off) __attribute__((always_inline)) {
    return *(const uint32_t *)((const char *)(cbase + row * K) + off);
  };
  const __attribute__((address_space(4))) int32_t *redge_c =
      (const __attribute__((address_space(4))) int32_t *)a.redge;

  // The step's table words of the wave's predecessors t = PG wid + j, states
  // z W + 2 lane and z W + 2 lane + 1: one 8-byte load per predecessor, the
  // whole step held in registers and loaded one step ahead.
  const uint32_t toff = (uint32_t)(PG * wid * KP + z * kXW + 2 * lane) * 4u;
  uint2 tb[PG];
  auto tload = [&](int j, int row, uint32_t dep) __attribute__((always_inline)) {
    const char *tab = (const char *)(a.rpk + (size_t)redge_c[row] * KP * KP);
    // The lane offset is formed by an asm add that also takes a value computed
    // from the register's last read: the load is issued after that read, and
    // no offset is hoisted out of the loop (64 of them would not fit).  One
    // 32-bit offset from the scalar base.
    uint32_t off;
    asm volatile("v_add_u32 %0, %1, %2" : "=v"(off) : "n"(j * KP * 4), "v"(toff), "v"(dep));
    tb[j] = *(const uint2 *)(tab + off);
  };

  // Publishes the part's value x of row i and gathers the other parts' values
  // of the same chain and state sl; returns the row's values in xv.
  auto exchange = [&](int i, uint32_t x, uint32_t (&xv)[kXS]) __attribute__((always_inline)) {
    const uint32_t tag = (uint32_t)i | PASS;
    char *slot = (char *)(xbt + (size_t)((i & 1) * kCG + c) * KP);  // uniform
    auto word = [&](int zz) __attribute__((always_inline)) {
      uint32_t off = (uint32_t)sl * 8u;
      asm volatile("" : "+v"(off));
      return (uint64_t *)(slot + off + (uint32_t)(zz * kXW * 8));
    };
    __hip_atomic_store(word(z), ((uint64_t)tag << 32) | x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    bool ok[kXS];
#pragma unroll
    for (int zz = 0; zz < kXS; ++zz) {
      ok[zz] = zz == z || ch.aborted;
      xv[zz] = zz == z ? x : kCX;
    }
    int spins = 0;
    // Every word is polled at once (the own word too), and twice, a few hundred
    // cycles apart: a word that lands just after the first poll left is seen
    // by the second rather than a whole round trip later.
    auto take = [&](const uint64_t (&w)[kXS]) __attribute__((always_inline)) {
      bool all = true;
#pragma unroll
      for (int zz = 0; zz < kXS; ++zz) {
        if (!ok[zz] && (uint32_t)(w[zz] >> 32) == tag) {
          xv[zz] = (uint32_t)w[zz];
          ok[zz] = true;
        }
        all = all && ok[zz];
      }
      return all;
    };
    while (true) {
      uint64_t w[kXS], w2[kXS];
#pragma unroll
      for (int zz = 0; zz < kXS; ++zz) w[zz] = __hip_atomic_load(word(zz), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __builtin_amdgcn_s_sleep(4);
#pragma unroll
      for (int zz = 0; zz < kXS; ++zz) w2[zz] = __hip_atomic_load(word(zz), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (take(w) || take(w2)) break;
      ++spins;
      // another part gave up (checked every 256 polls), or this wait expired
      if (spins > kXSpin ||
          ((spins & 255) == 0 && __hip_atomic_load(&a.xflag[team], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))) {
        sm.abort = 1;
        __hip_atomic_store(&a.xflag[team], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        break;
      }
      __builtin_amdgcn_s_sleep(1);
    }
  };

  // Row minima of the four chains from the gathered values, the offsets, and
  // the normalised row into LDS buffer NXT.  Ends with every thread past a barrier.
  auto finish_row = [&](const uint32_t (&xv)[kXS], int nxt, uint32_t (&d)[kCG]) __attribute__((always_inline)) {
    uint32_t m = umin(umin(xv[0], xv[1]), umin(xv[2], xv[3]));
    m = cw_wave_min(m);
    if (lane == 0) sm.wm[wid] = m;
    __syncthreads();
#pragma unroll
    for (int cc = 0; cc < kCG; ++cc) d[cc] = __builtin_amdgcn_readfirstlane(umin(sm.wm[2 * cc], sm.wm[2 * cc + 1]));
    ch.aborted = sm.abort != 0;
    const uint32_t dc = sel4(d, c);
#pragma unroll
    for (int zz = 0; zz < kXS; ++zz) {
      ch.q[zz] = umin(xv[zz] - dc, CAP) << BITS;
      sm.q[nxt][c][zz * kXQW + qsl] = ch.q[zz];
    }
#pragma unroll
    for (int cc = 0; cc < kCG; ++cc) ch.dsum[cc] += d[cc];
  };

#pragma unroll
  for (int cc = 0; cc < kCG; ++cc) {
    ch.flags[cc] = 0;
    ch.conv[cc] = -1;
    ch.dconv[cc] = 0;
    ch.dsum[cc] = 0;
  }
  ch.neg = 0;
  ch.aborted = false;
  if (tid == 0) sm.abort = 0;
  __syncthreads();
  int i0;
  if (MODE == kCSpec) {
    // start row r0 from its costs alone
    const uint32_t cv = cost_at((size_t)r0, coff);
    ch.neg = cv;
    uint32_t xv[kXS], d[kCG];
    exchange(r0, (sin && cv != (uint32_t)CFP_COST_INF) ? cv : kCX, xv);
    finish_row(xv, 0, d);
#pragma unroll
    for (int cc = 0; cc < kCG; ++cc)
      if (d[cc] == kCX) ch.flags[cc] |= 2;
    if (r0 == r1) {  // a run of one row: the start row is its checkpoint
      if (hv) ckb[(size_t)(r0 / 4) * KP + s] = sel4(ch.q, z);
      if (z == 0 && sl == 0 && (wid & 1) == 0 && hv) a.dck[(size_t)b * a.nq + r0 / 4] = (int64_t)sel4(ch.dsum, c);
    }
    i0 = r0 + 1;
  } else {
    // the start row: an end row of chunk p - 1 (row r0 - 1, a quad end)
#pragma unroll
    for (int zz = 0; zz < kXS; ++zz) {
      ch.q[zz] = startr[zz * kXW + sl];
      sm.q[0][c][zz * kXQW + qsl] = ch.q[zz];
    }
    i0 = r0;
  }
  __syncthreads();
  if (i0 > r1 || ch.aborted) return;

#pragma unroll
  for (int j = 0; j < PG; ++j) tload(j, i0, 0);
  // the own state's costs of the next two rows: step i uses set (i - i0) mod 2
  uint32_t cq[2], ckv[kXS];
  cq[0] = cost_at((size_t)i0, coff);
  cq[1] = cost_at((size_t)min(i0 + 1, r1), coff);
#pragma unroll
  for (int zz = 0; zz < kXS; ++zz) ckv[zz] = FIX ? ckb[(size_t)(i0 >> 2) * KP + zz * kXW + sl] : 0u;

  // One row i with the previous row in LDS buffer CUR; returns true when the
  // run is over (fix-up: every chain met; any mode: the team gave up).
  auto step = [&](int i, auto Pc) __attribute__((always_inline)) -> bool {
    constexpr int cur = decltype(Pc)::value, nxt = cur ^ 1;
    const int inext = min(i + 1, r1);
    uint32_t acc[kCG][2];
#pragma unroll
    for (int cc = 0; cc < kCG; ++cc) acc[cc][0] = acc[cc][1] = kSat;
#pragma unroll
    for (int j4 = 0; j4 < PG / 4; ++j4) {
      u32x4 v[kCG];  // predecessors PG wid + 4 j4 .. + 3 of every chain (LDS broadcast reads)
#pragma unroll
      for (int cc = 0; cc < kCG; ++cc) v[cc] = *(const u32x4 *)&sm.q[cur][cc][qpad(PG * wid + 4 * j4)];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const uint2 w0 = tb[4 * j4 + 2 * h], w1 = tb[4 * j4 + 2 * h + 1];
#pragma unroll
        for (int cc = 0; cc < kCG; ++cc) {
          const uint32_t va = h ? v[cc].z : v[cc].x, vb = h ? v[cc].w : v[cc].y;
          acc[cc][0] = umin(umin(acc[cc][0], sat_add(va, w0.x)), sat_add(vb, w1.x));
          acc[cc][1] = umin(umin(acc[cc][1], sat_add(va, w0.y)), sat_add(vb, w1.y));
        }
      }
      // the four registers just read take the next row's words
#pragma unroll
      for (int u = 0; u < 4; ++u) tload(4 * j4 + u, inext, acc[u][u & 1]);
    }
    // minima over the eight predecessor groups through LDS
#pragma unroll
    for (int cc = 0; cc < kCG; ++cc) *(uint2 *)&sm.part[cc][wid][2 * lane] = make_uint2(acc[cc][0], acc[cc][1]);
    __syncthreads();
    uint32_t mv = sm.part[c][0][sl];
#pragma unroll
    for (int g = 1; g < kCWaves; ++g) mv = umin(mv, sm.part[c][g][sl]);
    const uint32_t cv = cq[cur];
    if (MODE == kCSpec) {
      ch.neg |= cv;
      asm volatile("" : "+v"(ch.neg));
    }
    const uint32_t x = (sin && cv != (uint32_t)CFP_COST_INF) ? (mv >> BITS) + cv : kCX;
    if (sin && hv) *(uint16_t *)((char *)(tbase + (size_t)i * K) + (uint32_t)s * 2u) = (uint16_t)(mv & (KP - 1));
    {
      uint32_t off = coff;
      asm volatile("" : "+v"(off) : "v"(x));
      cq[cur] = cost_at((size_t)min(i + 2, r1), off);
    }
    uint32_t xv[kXS], d[kCG];
    exchange(i, x, xv);
    finish_row(xv, nxt, d);
    if (MODE == kCSpec) {
#pragma unroll
      for (int cc = 0; cc < kCG; ++cc)
        if (d[cc] == kCX) ch.flags[cc] |= 2;
    }
    const bool qend = (i & 3) == 3 || i == r1;
    if (qend) {
      const int q = i >> 2;
      if (MODE == kCSpec) {
        if (hv) ckb[(size_t)q * KP + s] = sel4(ch.q, z);
        if (z == 0 && sl == 0 && (wid & 1) == 0 && hv) a.dck[(size_t)b * a.nq + q] = (int64_t)sel4(ch.dsum, c);
      } else {
        bool off = false;
#pragma unroll
        for (int zz = 0; zz < kXS; ++zz) off = off || ch.q[zz] != ckv[zz];
        const uint64_t bal = __ballot(off);
        if (lane == 0) sm.wd[wid] = bal != 0;
        if (i < r1) {
#pragma unroll
          for (int zz = 0; zz < kXS; ++zz) ckv[zz] = ckb[(size_t)(q + 1) * KP + zz * kXW + sl];
        }
      }
    }
    __syncthreads();
    if (FIX && qend) {
      const int q = i >> 2;
      bool all = true;
#pragma unroll
      for (int cc = 0; cc < kCG; ++cc) {
        const bool same = !sm.wd[2 * cc] && !sm.wd[2 * cc + 1];
        if (ch.conv[cc] < 0 && same && q >= qmin[cc]) {
          ch.conv[cc] = q;
          ch.dconv[cc] = ch.dsum[cc];
        }
        all = all && (ch.conv[cc] >= 0 || !((act >> cc) & 1));
      }
      if (all) return true;
    }
    return ch.aborted;
  };
  for (int i = i0; i <= r1; i += 2) {
    if (step(i, std::integral_constant<int, 0>{})) break;
    if (i + 1 > r1 || step(i + 1, std::integral_constant<int, 1>{})) break;
  }
}

// Clears the exchange slots and abort flags of every team and the flags of
// every chunk record before a call's passes.
__global__ void chain_cx_init_kernel(uint64_t *xb, size_t nxb, int32_t *xflag, int teams, CwRec *rec, int nrec) {
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (size_t x = (size_t)blockIdx.x * blockDim.x + threadIdx.x; x < nxb; x += stride) xb[x] = ~0ull;
  for (size_t x = (size_t)blockIdx.x * blockDim.x + threadIdx.x; x < (size_t)teams; x += stride) xflag[x] = 0;
  for (size_t x = (size_t)blockIdx.x * blockDim.x + threadIdx.x; x < (size_t)nrec; x += stride) rec[x].flags = 0;
}

// Speculative (MODE kCSpec, grid (kXS, ceil(B/kCG), P)), fix-up (kCFix, grid
// (kXS, ceil(B/kCG), P-1)) and second fix-up (kCFix2, P-2) passes of the
// state-split teams; part z is blockIdx.x, so consecutive workgroups form a
// team.  Which chains take part depends on records that the pass does not
// write, so the parts of a team agree.
template <int MODE>
__global__ __launch_bounds__(kCThreads, 1) void chain_cx_kernel(CwArgs a) {
  __shared__ __align__(16) CxSmem sm;
  const int z = blockIdx.x, grp = blockIdx.y;
  const int p = blockIdx.z + (MODE == kCSpec ? 0 : MODE == kCFix ? 1 : 2);
  const int team = grp * a.P + p;
  const int r0 = p * a.CL, r1 = min(r0 + a.CL, a.N) - 1;
  const int tid = threadIdx.x, wid = __builtin_amdgcn_readfirstlane(tid >> 6), c = wid >> 1, sl = tid & (kXW - 1);
  int act = 0, qmin[kCG];
#pragma unroll
  for (int cc = 0; cc < kCG; ++cc) {
    const int b = min(kCG * grp + cc, a.B - 1);
    bool on = kCG * grp + cc < a.B;
    qmin[cc] = 0;
    if (MODE == kCFix2) {
      const CwRec *rec = a.rec + (size_t)b * a.P;
      on = on && cw_second(rec, p);
      qmin[cc] = rec[p].conv < 0 ? r1 >> 2 : rec[p].conv;
    }
    act |= on ? 1 << cc : 0;
  }
  act = __builtin_amdgcn_readfirstlane(act);
  if (MODE == kCFix2 && act == 0) return;
  const int bc = min(kCG * grp + c, a.B - 1);
  const uint32_t *startr = a.ckrow + ((size_t)bc * a.nq + (r0 > 0 ? r0 / 4 - 1 : 0)) * 512;
  if (MODE == kCFix2 && ((act >> c) & 1)) startr = a.endrow + ((size_t)bc * a.P + p - 1) * 512;
  CxChains ch;
  cx_run<MODE>(a, z, team, grp, r0, r1, act, qmin, startr, sm, ch);
  // flags of the run, one word per chain, ORed over the parts
  int32_t fl[kCG];
#pragma unroll
  for (int cc = 0; cc < kCG; ++cc) {
    fl[cc] = (MODE == kCSpec ? (int32_t)ch.flags[cc] : 0) | (ch.aborted ? 4 : 0);
    if (MODE == kCSpec && __syncthreads_or(c == cc && (ch.neg >> 31))) fl[cc] |= 1;
  }
#pragma unroll
  for (int cc = 0; cc < kCG; ++cc)
    if (tid == cc && ((act >> cc) & 1) && fl[cc])
      atomicOr(&a.rec[(size_t)(kCG * grp + cc) * a.P + p].flags, fl[cc]);
  if (MODE != kCSpec) {
    const int s = z * kXW + sl;
    if (((act >> c) & 1) && sel4(ch.conv, c) < 0)
      (MODE == kCFix ? a.endrow : a.endrow2)[((size_t)bc * a.P + p) * 512 + s] = sel4(ch.q, z);
    // second fix-up: whether the end row is the first one's (every part holds the whole row)
    bool off[kCG];
#pragma unroll
    for (int cc = 0; cc < kCG; ++cc) {
      bool o = false;
      if (MODE == kCFix2 && cc == c) {
        const size_t at = (size_t)bc * a.P + p;
        o = a.rec[at].conv >= 0;
#pragma unroll
        for (int zz = 0; zz < kXS; ++zz) o = o || a.endrow[at * 512 + zz * kXW + sl] != ch.q[zz];
      }
      off[cc] = MODE == kCFix2 && __syncthreads_or(o);
    }
#pragma unroll
    for (int cc = 0; cc < kCG; ++cc) {
      if (z != 0 || tid != cc || !((act >> cc) & 1)) continue;
      CwRec &r = a.rec[(size_t)(kCG * grp + cc) * a.P + p];
      const int64_t d = (int64_t)(ch.conv[cc] >= 0 ? ch.dconv[cc] : ch.dsum[cc]);
      if (MODE == kCFix) {
        r.conv = ch.conv[cc];
        r.dfix = d;
        r.run2 = 0;
      } else {
        r.conv2 = ch.conv[cc];
        r.dfix2 = d;
        r.run2 = 1;
        r.same2 = !off[cc];
      }
    }
  }
}

// Final pass, one workgroup per search: the chunk offsets, the reruns after
// chunks whose fix-up met no checkpoint, and the lowest optimal final state.
template <int KP, int CG>
__global__ __launch_bounds__((CwShape<KP, CG>::THREADS), 1) void chain_cw_final_kernel(CwArgs a, SearchResult *__restrict__ res,
                                                                       int64_t *__restrict__ opt,
                                                                       int32_t *__restrict__ status) {
  using S = CwShape<KP, CG>;
  __shared__ __align__(16) CwSmem<KP, CG> sm;
  __shared__ uint32_t s_row[KP];  // a true end row of the last chunk accounted
  __shared__ int s_q, s_end;
  __shared__ int64_t s_sum;
  __shared__ uint32_t s_fin[CwShape<KP, CG>::WAVES];
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int b = blockIdx.x, P = a.P;
  const int ms = tid & (KP - 1);
  const int64_t *dk = a.dck + (size_t)b * a.nq;
  const CwRec *rec = a.rec + (size_t)b * P;
  auto endq = [&](int p) __attribute__((always_inline)) { return (min((p + 1) * a.CL, a.N) - 1) >> 2; };
  // flags, combined after the loop so that their loads are in flight during it
  int fl = tid < P ? rec[tid].flags : 0;
  for (int x = tid; x < a.nbad; x += S::THREADS) fl |= a.rbad[x];
  // Chunk 0 runs from the true first row.  Invariant at the top of the loop:
  // chunks < p are accounted in `total`; if spec_true, the speculative end row
  // of chunk p-1 is a true row, otherwise s_row holds the true end row of chunk
  // p-1.  The last run of a chunk counts if it started from the true end row of
  // the chunk before: the fix-up from its speculative end row, the second
  // fix-up from the end row of its fix-up.
  int64_t total = dk[endq(0)];
  const uint32_t xlast = a.ckrow[((size_t)b * a.nq + a.nq - 1) * KP + ms];  // (in flight during the loop)
  bool spec_true = true;
  int p = 1;
  while (p < P) {
    bool counts = p == 1;  // the last run of chunk p counts (the second fix-up never runs chunk 1)
    if (p > 1) {
      counts = spec_true == !rec[p].run2;
      if (counts && !spec_true)  // it started from the true row?
        counts = !__syncthreads_or(tid < KP && s_row[ms] != a.endrow[((size_t)b * P + p - 1) * KP + ms]);
    }
    if (counts) {
      // With wave 0: the first chunk q > p whose last run started from another
      // row than chunk q-1's last run ends on, and the offsets of chunks p .. q-1.
      if (wid == 0) {
        const int pl = p + lane;
        const bool in = pl < P;
        CwRec r{};
        if (in) r = rec[pl];
        const int conv = r.run2 ? r.conv2 : r.conv;
        const int64_t dfix = r.run2 ? r.dfix2 : r.dfix;
        const int end = cw_end(r), before = __shfl_up(end, 1, 64);
        const uint64_t bad = __ballot(in && lane > 0 && before != (r.run2 ? kEnd1 : kEndSpec));
        const int q = bad ? p + __ffsll((long long)bad) - 1 : P;
        int64_t delta = 0;
        if (in && pl < q) delta = conv < 0 ? dfix : dfix + dk[endq(pl)] - dk[conv];
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) delta += __shfl_xor(delta, off, 64);
        if (lane == q - 1 - p) s_end = end;
        if (lane == 0) {
          s_q = q;
          s_sum = delta;
        }
      }
      __syncthreads();
      p = s_q;
      total += s_sum;
      const int end = s_end;
      spec_true = end == kEndSpec;
      if (!spec_true && tid < KP) s_row[tid] = (end == kEnd1 ? a.endrow : a.endrow2)[((size_t)b * P + p - 1) * KP + tid];
      __syncthreads();
      if (p >= P) break;
    }
    // Rerun chunk p from the true row, until it meets its own checkpoints.
    if (spec_true && tid < KP) s_row[tid] = a.ckrow[((size_t)b * a.nq + endq(p - 1)) * KP + tid];
    __syncthreads();
    int bs[CG], qmin[CG];
    bool valid[CG];
    const uint32_t *start[CG];
#pragma unroll
    for (int c = 0; c < CG; ++c) {
      bs[c] = b;
      valid[c] = c == 0;  // the other chain is not computed
      start[c] = s_row;
      qmin[c] = cw_qmin(rec[p], endq(p));
    }
    CwChains<KP, CG> ch;
    const int r0 = p * a.CL, r1 = min(r0 + a.CL, a.N) - 1;
    cw_run<KP, CG, kCFix, 1>(a, bs, valid, r0, r1, qmin, start, sm, ch);
    spec_true = ch.conv[0] >= 0;
    total += spec_true ? (int64_t)ch.dconv[0] + dk[endq(p)] - dk[ch.conv[0]] : (int64_t)ch.dsum[0];
    __syncthreads();  // every thread has read s_row
    if (!spec_true && tid < KP) s_row[tid] = ch.x[0];  // chain 0 of state tid is the thread's first
    __syncthreads();
    ++p;
  }
  // The final row has minimum 0: the lowest state at the minimum.
  const uint32_t xv = spec_true ? xlast : s_row[ms];
  const uint32_t pk = cw_wave_min((tid < KP && ms < a.K) ? (xv | (uint32_t)ms) : kSat);
  if (lane == 0) s_fin[wid] = pk;
  const int timeout = __syncthreads_or(fl & 4), bad = __syncthreads_or(fl & 1), infeasible = __syncthreads_or(fl & 2);
  if (tid == 0) {
    uint32_t fin = s_fin[0];
    for (int w = 1; w < S::WAVES; ++w) fin = umin(fin, s_fin[w]);
    int st = CFP_ST_OK;
    if (timeout) st = CFP_ST_TIMEOUT;
    else if (bad) st = CFP_ST_BADINPUT;
    else if (infeasible) st = CFP_ST_INFEASIBLE;
    else if ((fin >> S::BITS) != 0) st = CFP_ST_OVERFLOW;
    status[b] = st;
    opt[b] = st == CFP_ST_OK ? total : INT64_MAX;
    res[b].final_state = st == CFP_ST_OK ? (int32_t)(fin & (KP - 1)) : -1;
    res[b].status = st;
    res[b].final_m = 0;
  }
}

struct CwPlan {
  int KP, P, CL, nq;
  int G;  // chains per workgroup: 4, or 2
  int S;  // workgroups per chunk and group of four searches: 1, or kXS for state-split teams
};

// Chunks of at least minrows rows, as many as `groups` groups of searches need
// to fill `slots` workgroups.
int cw_chunk_rows(int n, int groups, int slots, int minrows) {
  const int P = std::min(kCMaxChunks, std::max(2, (slots + groups - 1) / groups));
  return std::max(minrows, ((n + P - 1) / P + 3) & ~3);
}

// period: of the edge map (0 when it has none, or for the region's size).
CwPlan cw_plan(int n, int k, int batch, int period) {
  const CwPlan none{0, 0, 0, 0, kCG, 1};
  CwPlan c = none;
  if (k <= 64 || k > 512) return none;
  const int kp = k <= 128 ? 128 : k <= 256 ? 256 : 512;
  const int minrows = kp <= 256 ? CwShape<256, kCG>::MINROWS : CwShape<512, kCG>::MINROWS;
  const int groups = (batch + kCG - 1) / kCG;
  // K > 256 with at most two groups of four searches: state-split teams, every
  // workgroup resident on its own compute unit.
  //
  // At K > 256 a chunk-parallel call takes about as long on any number of rows up to
  // 512 (two or three chunks of rows, which a workgroup takes 16.7 us each and a team
  // 6), so shorter chains go row after row: teams 390 to 560 us against 2.7 to 3.0 us
  // per row of the split kernel (even at 144 rows), others 950 to 1150 us against the
  // same (at most 32 searches: even at about 350) or, up to 1900 in larger batches,
  // 9.3 us per row of the wide kernel.
  // (Taken from 49 rows on, whatever the batch, 64 blocks, K = 400, 9 searches took
  // 789 us instead of 206.)
  const int cus = device_cus();
  int CL;
  if (kp == 512 && groups <= kXMaxGroups && cus / (kXS * groups) >= 2) {
    if (n < 144) return none;
    c.S = kXS;
    CL = cw_chunk_rows(n, groups, cus / (kXS * groups) * groups, minrows);  // (at most cus workgroups)
  } else {
    if (kp == 512 && n < (chain_fwd_split_supported(k, 1, batch) ? 352 : 128)) return none;
    // Two chains per workgroup while all chunks of the least length fit the chip
    // so: a row takes 1.1 us against 1.8 at KP = 128 (393 blocks, K = 81, 24
    // searches: 148 -> 105 us per call) and 3.0 against 4.3 at KP = 256 (1152
    // blocks, one search: 249 -> 184 us).  Several workgroups of KP = 128 share a
    // compute unit (1152 blocks, K = 81, 40 searches as 720 of them 207 us, as
    // 360 of four chains 246; 128 searches of K = 128 415 us at 256 workgroups,
    // 331 at 512, 364 at 768); at KP = 256 a second one only adds rows (1152
    // blocks, K = 256, 128 searches: 863 us at 256, 1026 at 512).
    const int slots2 = kp == 128 ? 768 : 256, slots4 = kp == 128 ? 512 : 256;
    const int half = (batch + 1) / 2, pmax = std::min(kCMaxChunks, (n + minrows - 1) / minrows);
    c.G = (long long)half * pmax <= slots2 ? 2 : 4;
    CL = c.G == 2 ? cw_chunk_rows(n, half, slots2, minrows) : cw_chunk_rows(n, groups, slots4, minrows);
  }
  // More searches than compute units go through the wide kernel in several rounds: two
  // halves of a shorter chain instead (32 blocks, K = 200, 1000 searches: 375 to 229 us).
  if (kp == 256 && n >= 16 && n <= minrows && batch > cus) CL = ((n + 1) / 2 + 3) & ~3;
  int P = (n + CL - 1) / CL;
  if (P < 2) return none;
  // Chunks of an even number of periods start in phase with a chain whose costs
  // repeat with its edge map and whose rows alternate between periods; worth a
  // sixteenth more rows per chunk, and at K > 256 up to 64 rows in place of 48 (1152
  // blocks, K = 512, 16 tables, 8 searches of repeating costs: 7.2 ms in chunks of 48
  // rows, 0.6 in 64; costs of their own 0.72 and 0.79).
  int u = period;
  while (u % 4) u += period;
  if (period % 4 == 0) u = 2 * period;
  const int al = period ? (CL + u - 1) / u * u : CL;
  if ((16 * al <= 17 * CL || (kp == 512 && al <= 64)) && al < n) {
    CL = al;
    P = (n + CL - 1) / CL;
  }
  c.KP = kp;
  c.P = P;
  c.CL = CL;
  c.nq = (n + 3) / 4;
  return c;
}

template <int KP, int CG>
void launch_cw_kp(const CwArgs &a, SearchResult *res, int64_t *opt, int32_t *status, hipStream_t st) {
  constexpr int FG = 2;  // the final pass reruns one chain
  const int groups = (a.B + CG - 1) / CG;
  const dim3 block(CwShape<KP, CG>::THREADS);
  timer_begin(st);
  timed_launch(chain_cw_kernel<KP, CG, kCSpec>, dim3(groups, a.P), block, 0, st, a);
  timer_end(st);
  hipLaunchKernelGGL((chain_cw_kernel<KP, CG, kCFix>), dim3(groups, a.P - 1), block, 0, st, a);
  if (a.P > 2) hipLaunchKernelGGL((chain_cw_kernel<KP, CG, kCFix2>), dim3(groups, a.P - 2), block, 0, st, a);
  hipLaunchKernelGGL((chain_cw_final_kernel<KP, FG>), dim3(a.B), dim3(CwShape<KP, FG>::THREADS), 0, st, a, res, opt,
                     status);
}

void launch_cx(const CwArgs &a, int groups, SearchResult *res, int64_t *opt, int32_t *status, hipStream_t st) {
  const int teams = groups * a.P;
  hipLaunchKernelGGL(chain_cx_init_kernel, dim3(64), dim3(256), 0, st, a.xb, (size_t)teams * 2 * kCG * 512, a.xflag,
                     teams, a.rec, a.B * a.P);
  timer_begin(st);
  timed_launch(chain_cx_kernel<kCSpec>, dim3(kXS, groups, a.P), dim3(kCThreads), 0, st, a);
  timer_end(st);
  hipLaunchKernelGGL(chain_cx_kernel<kCFix>, dim3(kXS, groups, a.P - 1), dim3(kCThreads), 0, st, a);
  if (a.P > 2) hipLaunchKernelGGL(chain_cx_kernel<kCFix2>, dim3(kXS, groups, a.P - 2), dim3(kCThreads), 0, st, a);
  hipLaunchKernelGGL((chain_cw_final_kernel<512, 2>), dim3(a.B), dim3(kCThreads), 0, st, a, res, opt, status);
}

}  // namespace

bool chain_cw_supported(int n, int k, int batch) { return cw_plan(n, k, batch, 0).P >= 2; }

bool chain_cw_teams(int n, int k, int batch) { return cw_plan(n, k, batch, 0).S > 1; }

size_t cw_region_bytes(int n, int k, int n_tables, int batch) {
  const CwPlan c = cw_plan(n, k, batch, 0);  // no plan of these sizes has more chunks
  if (c.P < 2) return 0;
  const size_t kp = c.KP;
  size_t off = align_up((size_t)n_tables * kp * kp * 4);
  off += align_up(kPackBlocks * sizeof(int32_t));
  off += align_up((size_t)batch * c.P * sizeof(CwRec));
  off += align_up((size_t)batch * c.nq * 8);
  off += align_up((size_t)batch * c.nq * kp * 4);
  off += 2 * align_up((size_t)batch * c.P * kp * 4);
  if (c.S > 1) {
    const size_t teams = (size_t)((batch + kCG - 1) / kCG) * c.P;
    off += align_up(teams * 2 * kCG * kp * 8);
    off += align_up(teams * 4);
  }
  return off;
}

hipError_t launch_chain_cw(const cfp_chain_desc &d, int32_t *redge_dev, const EdgeMap &em, uint8_t *region,
                           uint8_t *table, SearchResult *res, int64_t *opt, int32_t *status, hipStream_t st) {
  const CwPlan c = cw_plan(d.n_blocks, d.k, d.batch, em.period);
  const size_t kp = c.KP;
  CwArgs a;
  a.cost = d.cost;
  a.redge = redge_dev;
  a.N = d.n_blocks;
  a.K = d.k;
  a.B = d.batch;
  a.P = c.P;
  a.CL = c.CL;
  a.nq = c.nq;
  a.table = table;
  size_t off = 0;
  uint32_t *rpk = (uint32_t *)(region + off);
  a.rpk = rpk;
  off += align_up((size_t)d.n_tables * kp * kp * 4);
  int32_t *rbad = (int32_t *)(region + off);
  a.rbad = rbad;
  off += align_up(kPackBlocks * sizeof(int32_t));
  a.rec = (CwRec *)(region + off);
  off += align_up((size_t)d.batch * c.P * sizeof(CwRec));
  a.dck = (int64_t *)(region + off);
  off += align_up((size_t)d.batch * c.nq * 8);
  a.ckrow = (uint32_t *)(region + off);
  off += align_up((size_t)d.batch * c.nq * kp * 4);
  a.endrow = (uint32_t *)(region + off);
  off += align_up((size_t)d.batch * c.P * kp * 4);
  a.endrow2 = (uint32_t *)(region + off);
  off += align_up((size_t)d.batch * c.P * kp * 4);
  const int groups = (d.batch + kCG - 1) / kCG;
  a.xb = nullptr;
  a.xflag = nullptr;
  if (c.S > 1) {
    a.xb = (uint64_t *)(region + off);
    off += align_up((size_t)groups * c.P * 2 * kCG * kp * 8);
    a.xflag = (int32_t *)(region + off);
  }
  const int bits = kp == 128 ? 7 : kp == 256 ? 8 : 9;
  a.nbad = launch_pack_rtab(d.rtab, d.n_tables, d.k, (int)kp, bits, rpk, st, cfp_r_limit(CFP_V_CHAIN, d.k), rbad, &em,
                            redge_dev, d.n_blocks);
  if (c.S > 1) launch_cx(a, groups, res, opt, status, st);
  else if (kp == 128 && c.G == 2) launch_cw_kp<128, 2>(a, res, opt, status, st);
  else if (kp == 128) launch_cw_kp<128, kCG>(a, res, opt, status, st);
  else if (kp == 256 && c.G == 2) launch_cw_kp<256, 2>(a, res, opt, status, st);
  else if (kp == 256) launch_cw_kp<256, kCG>(a, res, opt, status, st);
  else if (c.G == 2) launch_cw_kp<512, 2>(a, res, opt, status, st);
  else launch_cw_kp<512, kCG>(a, res, opt, status, st);
  return hipGetLastError();
}

}  // namespace cfp
