// Chunk-parallel forward pass of the chain search for 32 < K <= 64 (Sec. 4.4,
// Eq. T recurrence), one wave per search.
//
// Parallelism over the chain.  The recurrence is a chain of N-1 dependent
// min-plus steps per search.  Each chain is cut into P chunks that run
// concurrently, using the rank convergence of min-plus products (Maleki,
// Musuvathi and Mytkowicz, "Parallelizing dynamic programming through rank
// convergence", PPoPP 2014): the recurrence started from an arbitrary row
// becomes parallel to the true run (the rows differ by one constant in every
// state) after a few steps, and from then on both choose the same argmins.
//   1. speculative pass, every chunk: chunk p starts at its first row from that
//      row's costs alone, as if the chain began there.  It writes the argmin
//      rows of its steps and, at the end of every quad of 4 rows (a
//      checkpoint), its normalised row and the running sum of its offsets.
//   2. fix-up pass, chunks 1..P-1: chunk p starts again from the last
//      checkpoint row of chunk p-1 and recomputes its steps until its
//      normalised row equals the stored checkpoint row of the same quad,
//      rewriting the argmins on the way.  Equal normalised rows mean every
//      later step of the speculative pass is exactly the true one.
//   3. final pass, per search: sums the offsets of the chunks; if a chunk's
//      fix-up reached its end without meeting a checkpoint (so its successor
//      started from a wrong row), the next chunk is rerun from that chunk's end
//      row, which is the true one, until it meets its own speculative rows; the
//      fix-up results of the chunks after it then count again.  Then the lowest
//      optimal final state and the optimum.
// The result is the sequential recurrence's bit for bit whatever the inputs;
// only the time depends on how fast the rows converge.
//
// One step of one search in one wave.  Lane s holds the word of state s,
// Q[s] = (value << 6).  Two permlane swaps give four registers C_k whose every
// row of 16 lanes holds row k of the wave (states 16k .. 16k+15), so a DPP row
// broadcast of lane j of C_k hands predecessor t = 16k + j to every lane.  The
// candidate of (t, s) is C_k[j] + RP[t][s] with RP = (R[t][s] << 6) | t packed
// once per call, so one unsigned min gives the value and the lowest argmin.
// A step is 64 adds with a DPP operand and 32 three-input mins per search, a
// minimum over the wave and the normalisation; no other wave is involved.
//
// Normalisation.  The new row is x[s] = (m[s] >> 6) + c[i][s] with m the
// packed minimum; it is normalised by its own minimum d = min_s x[s]:
//     Q_i[s] = min(x[s] - d, qcap) << 6,   qcap = 2^25 - 1,
// and d is added to the search's offset, so the optimum is the sum of the row
// minima.  Since the previous row has minimum 0, m >> 6 <= R_max < 2^24 and
// x < 2^32; a state at the cap is more than R_max above the minimum and is
// beaten through the minimum state, so capping never changes an argmin.  An
// unavailable strategy (cost CFP_COST_INF) and a padding state (s >= K) get
// x = 2^32 - 1 and stay capped.
//
// Work split of a workgroup: 16 waves (4 for small batches), each with one
// search of the same chunk, so every wave steps through the same rows and the same
// tables.  The packed tables of four consecutive rows
// (4 x 16 KiB) sit in LDS and the next four are staged while these are used
// (double buffer, one barrier per four rows); the rows are cut into blocks of
// 12, the period of the edge map the kernels are specialised for.
#include <algorithm>

#include "res_common.h"

namespace cfp {

namespace {

constexpr int kWSpec = 0, kWFix = 1;
constexpr int kWU = 12;                 // rows per block (checkpoint spacing)
constexpr int kWWaves = 16;             // waves per workgroup on large batches
constexpr int kWTable16 = 64 * 64 / 4;  // 16-byte chunks of one packed table
constexpr int kWMaxChunks = 64;         // chunks per search (the final pass reads one per lane)
constexpr int kWMinBlocks = 4;          // least blocks of 12 rows per chunk
constexpr uint32_t kWX = 0xFFFFFFFFu;   // x of an unavailable or padding state
constexpr int kWPackBlocks = 1024;      // most workgroups of the packing kernel
constexpr int kWBits = 6;
constexpr uint32_t kWQcap6 = ((1u << 25) - 1u) << kWBits;

struct WaveRec {
  int64_t dfix;   // fix-up pass: offset sum at the meeting checkpoint, or at the chunk end
  int32_t flags;  // speculative pass: bit 0 a negative cost, bit 1 a row with no available strategy
  int32_t conv;   // fix-up pass: quad of the meeting checkpoint, -1 if none
};

struct WaveArgs {
  const int32_t *cost;
  const u32x4 *rpk;     // packed tables [E][16 chunks][64 states] of 4 words
  const int32_t *redge;
  int N, K, E, B, P, CB, nblk, nq;  // nq = quads of 4 rows
  uint8_t *table;       // argmin entries [B][N][K]
  WaveRec *rec;         // [B][P]
  int64_t *dck;         // speculative offset sum (from the chunk's start row) at every checkpoint [B][nq]
  uint32_t *ckrow;      // speculative row at every checkpoint (end of a quad of rows) [B][nq][64]
  uint32_t *endrow;     // fix-up end row of chunks that met no checkpoint [B][P][64]
  const u32x4 *rbad;    // range flags of R, one byte per packing wave
  int nbad;             // in pieces of 16
};

// Packed tables: word u of chunk c of lane s of table e is (R_e[t][s] << 6) | t
// with t = 4c + u.  Rows t >= K and columns s >= K take row or column K-1: a
// predecessor t >= K holds a capped word, so its candidate exceeds every exact
// one without wrapping, and a state s >= K is padding.
// Every R entry is read here, so the range check of R (entries in [0, limit))
// is made on the way; every wave writes its own flag byte, so none needs a reset
// (and no workgroup a barrier).  With a period in `em`, the edge map is written out
// as well.
struct NoMap {
  __device__ void write(int32_t *, int) const {}
};
template <typename Map>
__global__ void wave_pack_kernel(const int32_t *__restrict__ rtab, int E, int K, uint32_t *__restrict__ rpk,
                                 int32_t limit, uint8_t *__restrict__ bad, Map em, int32_t *__restrict__ redge,
                                 int n) {
  em.write(redge, n);
  const size_t words = (size_t)E * 64 * 64;
  bool off = false;
  for (size_t w = blockIdx.x * (size_t)blockDim.x + threadIdx.x; w < words; w += (size_t)gridDim.x * blockDim.x) {
    const int u = (int)(w & 3), s = (int)((w >> 2) & 63), c = (int)((w >> 8) & 15), e = (int)(w >> 12);
    const int t = 4 * c + u;
    const int32_t r = rtab[((size_t)e * K + min(t, K - 1)) * K + min(s, K - 1)];
    off |= r < 0 || r >= limit;
    rpk[w] = ((uint32_t)r << kWBits) | (uint32_t)t;
  }
  const bool any = __any(off);
  if ((threadIdx.x & 63) == 0) bad[blockIdx.x * 4 + (threadIdx.x >> 6)] = any ? 1 : 0;
}

// Minimum over the 64 lanes of a wave as a scalar: row minima by DPP, then the
// row broadcasts of lanes 15 and 31 fold rows 0..3 into row 3, read at lane 63.
__device__ __forceinline__ uint32_t wave_min64_s(uint32_t x) {
  x = dpp_min<kQuadSwap1>(x);
  x = dpp_min<kQuadSwap2>(x);
  x = dpp_min<kHalfMirror>(x);
  x = dpp_min<kMirror>(x);
  asm("s_nop 1\n"
      "v_min_u32_dpp %0, %0, %0 row_bcast:15 row_mask:0xa bank_mask:0xf\n"
      "s_nop 1\n"
      "v_min_u32_dpp %0, %0, %0 row_bcast:31 row_mask:0xc bank_mask:0xf\n"
      "s_nop 1\n"
      : "+v"(x));
  return __builtin_amdgcn_readlane(x, 63);
}

template <int NW>
struct WaveSmem {
  static constexpr int CPT = kWTable16 / (64 * NW);  // 16-byte chunks per thread and table
  u32x4 tb[2][4][kWTable16];                          // packed tables of two quads of rows
  uint8_t argb[NW][kWU][64];                          // argmin bytes of the block's rows, per wave
  uint32_t wact[2][NW];                               // fix-up: wave still has an unmet search, by quad parity
};

// State of a wave's search.
struct WaveChain {
  uint32_t qv;         // the lane's word of the current row
  uint64_t dsum;       // offset sum since the start row
  uint32_t flags;      // bit 0 a negative cost, bit 1 a row with no available strategy
  uint32_t cor;        // speculative pass: OR of the lane's costs (bit 31 = a negative cost)
  int conv;            // fix-up: quad where the row met the checkpoint, -1 if never
  uint64_t dconv;      // fix-up: offset sum at that quad
};

// Runs rows [12*blk0 (+1 for kSpec), min(12*blk1, N)) of the wave's search bw,
// which is real if it is below B and (in the final pass) with `real`.
//   kSpec:   the start row is row 12*blk0 from its costs alone; checkpoints are
//            written.
//   kFix:    the start row (row 12*blk0 - 1) is start; at every quad end
//            from quad qmin on the row is compared with the speculative
//            checkpoint of the same quad (LATE: any other qmin than 0).  A search that has met it stops
//            computing (its later speculative rows are the true ones) and the
//            workgroup stops once all of its searches have met.
template <int NW, int MODE, int EP, bool LATE = false>
__device__ __forceinline__ void wave_run(const WaveArgs &a, int bw, bool real, int blk0, int blk1, int qmin,
                                         const uint32_t *start, WaveSmem<NW> &sm, WaveChain &ch) {
  constexpr int U = kWU, CPT = WaveSmem<NW>::CPT;
  static_assert(CPT == 1 || CPT == 2 || CPT == 4, "1, 2 or 4 chunks per thread and table");
  const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int N = a.N, K = a.K;
  const int i0 = blk0 * U + (MODE == kWSpec ? 1 : 0);  // first computed row
  const int ilast = min(blk1 * U, N) - 1;              // last row of the run
  const int sl = min(lane, K - 1);

  const bool valid = real && bw < a.B;
  const int b = min(bw, a.B - 1);
  auto edge = [&](int row) __attribute__((always_inline)) { return EP ? row % (EP ? EP : 1) : a.redge[row]; };
  // the search's rows (wave-uniform bases; a row adds row * K and the lane its
  // state, so the loads take a scalar base and a lane offset)
  const int32_t *cb = a.cost + (size_t)b * N * K;
  uint8_t *tb = a.table + (size_t)b * N * K;

  // Memory schedule.  The tables of the next quad are loaded during the first
  // three rows of a quad of four and the costs of the quad after the next in
  // its last row; everything is consumed at a quad's end, after its one wait.  (With stores in flight the wait covers
  // every outstanding load, so a load consumed earlier would stall the row.)
  // Array indices are literals only, so every array stays in registers.
  u32x4 sq[4][4];           // next quad's tables: [row in quad][chunk of this thread]
  // Costs of three consecutive quads, [quad mod 3][row in quad]: quad
  // q reads set q mod 3 while set (q+2) mod 3 is loaded.  A block of 12 rows
  // starts at a quad that is 0 mod 3, so every index is a constant.
  uint32_t cs[3][4] = {};
#define CFP_QLOAD(V)                                                               \
  {                                                                                \
    const int row = min(qbase + (V), ilast); /* past the end: any in-range row */  \
    const u32x4 *src = a.rpk + (size_t)edge(row) * kWTable16;                      \
    sq[V][0] = src[tid];                                                           \
    if constexpr (CPT >= 2) sq[V][1] = src[tid + 64 * NW];                         \
    if constexpr (CPT == 4) {                                                      \
      sq[V][2] = src[tid + 128 * NW];                                              \
      sq[V][3] = src[tid + 192 * NW];                                              \
    }                                                                              \
  }
#define CFP_CLOAD(V, DST)                                                          \
  {                                                                                \
    const int row = min(cbase + (V), ilast);                                       \
    DST[V] = (uint32_t)(cb + (size_t)row * K)[sl];                                 \
  }
#define CFP_QSTORE(V)                                                              \
  {                                                                                \
    u32x4 *dst = sm.tb[((qbase + (V)) >> 2) & 1][V] + tid;                         \
    dst[0] = sq[V][0];                                                             \
    if constexpr (CPT >= 2) dst[64 * NW] = sq[V][1];                               \
    if constexpr (CPT == 4) {                                                      \
      dst[128 * NW] = sq[V][2];                                                    \
      dst[192 * NW] = sq[V][3];                                                    \
    }                                                                              \
  }
#define CFP_Q4(M) M(0) M(1) M(2) M(3)

  // Prologue: the first quad (rows from i0) at once, the next quad's loads,
  // and the costs of the two quads after the first.
  {
    int qbase = i0 & ~3, cbase = qbase;
#define CFP_QFIRST(V) /* rows before i0 are staged too, and never read */ \
  CFP_QLOAD(V)                                                             \
  CFP_QSTORE(V)
    CFP_Q4(CFP_QFIRST)
#undef CFP_QFIRST
    qbase += 4;
    CFP_Q4(CFP_QLOAD)
    // the first quad is 0 mod 3 (blocks start at quads 3 blk)
#define CFP_C0(V) CFP_CLOAD(V, cs[0])
#define CFP_C1(V) CFP_CLOAD(V, cs[1])
#define CFP_C2(V) CFP_CLOAD(V, cs[2])
    CFP_Q4(CFP_C0)
    cbase += 4;
    CFP_Q4(CFP_C1)
    cbase += 4;
    CFP_Q4(CFP_C2)
  }

  // Start row.
  ch.flags = 0;
  if (MODE == kWSpec) {
    const uint32_t cv = (uint32_t)(cb + (size_t)blk0 * U * K)[sl];
    const bool avail = lane < K && cv != (uint32_t)CFP_COST_INF;
    ch.cor = cv;
    const uint32_t x = avail ? cv : kWX;
    const uint32_t d = wave_min64_s(x);
    if (d == kWX) ch.flags |= 2;
    ch.qv = umin(x - d, kWQcap6 >> kWBits) << kWBits;
    ch.dsum = d;
    if (i0 > ilast && valid) {  // a run of one row: the start row is its checkpoint
      a.ckrow[((size_t)b * a.nq + (i0 - 1) / 4) * 64 + lane] = ch.qv;
      if (lane == 0) a.dck[(size_t)b * a.nq + (i0 - 1) / 4] = (int64_t)ch.dsum;
    }
  } else {
    ch.qv = start[lane];
    ch.dsum = 0;
  }
  ch.conv = valid ? -1 : 0;  // a missing search counts as met
  ch.dconv = 0;
  int endr = ilast;   // last row whose argmin bytes are written back
  uint32_t ckv = 0;   // fix-up: checkpoint of the current quad
  bool stop = false;
  __syncthreads();  // the first quad's tables

  // Argmin bytes of rows [12 blk + r0, 12 blk + nr) of the wave's searches from
  // LDS to the table: a row of one search is 64 bytes, four 16-byte pieces.
  auto flush = [&](int blk, int nr) __attribute__((always_inline)) {
    const int r0 = (MODE == kWSpec && blk == blk0) ? 1 : 0;  // the start row has no argmin
    if (!valid) return;
    uint8_t *dst = tb + (size_t)blk * U * K;
    const int nrg = MODE == kWFix ? min(nr, endr - blk * U + 1) : nr;
    for (int x = lane + 4 * r0; x < 4 * nrg; x += 64) {  // piece x: row x / 4, bytes 16 (x % 4) ..
      const int r = x >> 2, c = (x & 3) * 16;
      const u32x4 v = *(const u32x4 *)&sm.argb[wid][r][c];
      if (K == 64) {
        *(u32x4 *)(dst + (size_t)r * K + c) = v;
      } else {
        const uint8_t *vb = (const uint8_t *)&v;
        for (int q = 0; q < 16 && c + q < K; ++q) dst[(size_t)r * K + c + q] = vb[q];
      }
    }
  };

  constexpr int NPRE = 4;  // table chunks of the next row read ahead
  u32x4 wpre[NPRE];
  // One row; J = row mod 12.  GUARD: the block may end before its 12th row;
  // FIRST: the run's first block, whose rows before i0 are skipped and whose
  // first quad's loads were issued before the loop.
  auto step = [&](auto Jc, auto Gd, auto Fd, int blk) __attribute__((always_inline)) {
    constexpr int J = decltype(Jc)::value, u = J & 3;
    constexpr bool GUARD = decltype(Gd)::value, FIRST = decltype(Fd)::value;
    const int i = blk * U + J;
    if (MODE == kWFix && stop) return;
    if (GUARD && i > ilast) return;
    if (FIRST && i < i0) return;
    if (!FIRST || i >= (i0 & ~3) + 4) {  // the next quad's loads (the first quad's: prologue)
      // rows 0 and 1 at step 0, row 2 at step 1, row 3 at step 2: every load
      // has at least one row of compute before the quad's wait
      const int qbase = (i & ~3) + 4;
      if constexpr (u == 0) {
        CFP_QLOAD(0)
        CFP_QLOAD(1)
      }
      if constexpr (u == 1) CFP_QLOAD(2)
      if constexpr (u == 2) CFP_QLOAD(3)
    }
    if (MODE == kWFix && u == 0 && (!LATE || (i >> 2) >= qmin)) {  // this quad's checkpoint (runs start at a quad)
      ckv = (a.ckrow + ((size_t)b * a.nq + (i >> 2)) * 64)[lane];
    }
    if (u == 3 && (!FIRST || i >= (i0 & ~3) + 4)) {  // costs two quads ahead, after this quad's table loads
      const int cbase = (i & ~3) + 8;
      constexpr int nset = (J / 4 + 2) % 3;
      if constexpr (nset == 0) { CFP_Q4(CFP_C0) }
      if constexpr (nset == 1) { CFP_Q4(CFP_C1) }
      if constexpr (nset == 2) { CFP_Q4(CFP_C2) }
    }

    // Row-broadcast sources: C_k has row k of the wave in every row.
    const auto p = __builtin_amdgcn_permlane16_swap(ch.qv, ch.qv, false, false);
    const auto lo = __builtin_amdgcn_permlane32_swap(p[0], p[0], false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap(p[1], p[1], false, false);
    const uint32_t c0 = lo[0], c1 = hi[0], c2 = lo[1], c3 = hi[1];
    uint32_t acc = kSat;
    const u32x4 *rows = sm.tb[(i >> 2) & 1][u];
    // The row's sixteen table chunks in two halves; outside the first block the
    // first NPRE of rows 1..3 of a quad are read during the previous row's
    // normalisation (PRE).
    constexpr int WH = 8;
    constexpr bool PRE = !FIRST && u != 0;
    u32x4 w[16];
    const bool live = MODE != kWFix || ch.conv < 0;
#define CFP_CH(C, cc_)                                          \
  if constexpr ((cc_) == 0) cand4_g1_first(acc, C, w[0]);       \
  else cand4_g1<4 * ((cc_) & 3), ((cc_) & 3) == 0>(acc, C, w[cc_]);
    if (live) {
      if constexpr (PRE) {
#pragma unroll
        for (int cc_ = 0; cc_ < NPRE; ++cc_) w[cc_] = wpre[cc_];
#pragma unroll
        for (int cc_ = NPRE; cc_ < WH; ++cc_) w[cc_] = rows[cc_ * 64 + lane];
      } else {
#pragma unroll
        for (int cc_ = 0; cc_ < WH; ++cc_) w[cc_] = rows[cc_ * 64 + lane];
      }
      CFP_CH(c0, 0) CFP_CH(c0, 1) CFP_CH(c0, 2) CFP_CH(c0, 3)
      CFP_CH(c1, 4) CFP_CH(c1, 5) CFP_CH(c1, 6) CFP_CH(c1, 7)
#pragma unroll
      for (int cc_ = WH; cc_ < 16; ++cc_) w[cc_] = rows[cc_ * 64 + lane];
      CFP_CH(c2, 8) CFP_CH(c2, 9) CFP_CH(c2, 10) CFP_CH(c2, 11)
      CFP_CH(c3, 12) CFP_CH(c3, 13) CFP_CH(c3, 14) CFP_CH(c3, 15)
      if constexpr (!FIRST && u != 3) {
#pragma unroll
        for (int cc_ = 0; cc_ < NPRE; ++cc_) wpre[cc_] = rows[kWTable16 + cc_ * 64 + lane];
      }
    }
#undef CFP_CH

    // New row: add the cost, normalise by the row minimum, record the argmin.
    if (live) {
      const uint32_t cv = cs[(J / 4) % 3][u];
      const bool avail = lane < K && cv != (uint32_t)CFP_COST_INF;
      if (MODE == kWSpec) {
        ch.cor |= cv;
        // kept in its row: sunk to the end of a block, the OR waits for the
        // latest cost loads behind the block's argmin stores
        asm volatile("" : "+v"(ch.cor));
      }
      const uint32_t x = avail ? (acc >> kWBits) + cv : kWX;
      const uint32_t d = wave_min64_s(x);
      if (MODE == kWSpec && d == kWX) ch.flags |= 2;
      ch.qv = umin(x - d, kWQcap6 >> kWBits) << kWBits;
      ch.dsum += d;
      sm.argb[wid][J][lane] = (uint8_t)acc;
    }

    // End of a quad: the next quad's tables in place and one barrier, then the
    // checkpoint (speculative pass) and, at the end of a block, the argmin rows
    // (each wave writes back its own searches' bytes with 16-byte stores).  The
    // stores come after the barrier's wait for the staged loads, so that wait
    // does not cover them.
    constexpr bool QEND = u == 3;
    if (QEND || (GUARD && i == ilast)) {
      {
        const int qbase = (i & ~3) + 4;
        CFP_Q4(CFP_QSTORE)
      }
      if (MODE == kWFix && (!LATE || (i >> 2) >= qmin)) {
        if (ch.conv < 0 && __ballot(ch.qv != ckv) == 0) {
          ch.conv = i >> 2;
          ch.dconv = ch.dsum;
          endr = i;
        }
        if (lane == 0) sm.wact[(i >> 2) & 1][wid] = ch.conv < 0 ? 1u : 0u;
      }
      __syncthreads();
      if (MODE == kWFix && (!LATE || (i >> 2) >= qmin)) {  // every wave reads the same flags: a uniform decision
        const uint32_t f = lane < NW ? sm.wact[(i >> 2) & 1][lane] : 0u;
        stop = __ballot(f != 0) == 0;
        if (stop) {
          flush(blk, J + 1);
          return;
        }
      }
      if (MODE == kWSpec) {
        const int q = i >> 2;
        if (valid) {
          (a.ckrow + ((size_t)b * a.nq + q) * 64)[lane] = ch.qv;
          if (lane == 0) a.dck[(size_t)b * a.nq + q] = (int64_t)ch.dsum;
        }
      }
      if (J == U - 1 || (GUARD && i == ilast)) flush(blk, J + 1);
    }
  };
#undef CFP_Q4
#undef CFP_QSTORE
#undef CFP_QLOAD
#undef CFP_CLOAD
#undef CFP_C0
#undef CFP_C1
#undef CFP_C2

  auto block = [&](auto Gd, auto Fd, int blk) __attribute__((always_inline)) {
#define CFP_S(J_) step(std::integral_constant<int, J_>{}, Gd, Fd, blk);
    CFP_S(0) CFP_S(1) CFP_S(2) CFP_S(3) CFP_S(4) CFP_S(5)
    CFP_S(6) CFP_S(7) CFP_S(8) CFP_S(9) CFP_S(10) CFP_S(11)
#undef CFP_S
  };

  const int full_end = min(blk1, N / U);  // blocks with 12 rows
  if (blk0 >= full_end) {  // a single block, not full
    block(std::true_type{}, std::true_type{}, blk0);
    return;
  }
  block(std::false_type{}, std::true_type{}, blk0);
  int blk = blk0 + 1;
  for (; blk < full_end && !(MODE == kWFix && stop); ++blk) block(std::false_type{}, std::false_type{}, blk);
  if (blk < blk1 && !(MODE == kWFix && stop)) block(std::true_type{}, std::false_type{}, blk);
}

// Speculative pass, grid (ceil(B/NW), P).
template <int EP, int NW>
__global__ __launch_bounds__(64 * NW) void chain_wave_kernel(WaveArgs a) {
  __shared__ __align__(16) WaveSmem<NW> sm;
  const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int bw = blockIdx.x * NW + wid;  // one search per wave
  const int p = blockIdx.y;
  const int blk0 = p * a.CB, blk1 = min(blk0 + a.CB, a.nblk);
  WaveChain ch;
  wave_run<NW, kWSpec, EP>(a, bw, true, blk0, blk1, 0, nullptr, sm, ch);
  if (__ballot((int32_t)ch.cor < 0)) ch.flags |= 1;  // wave-uniform
  if (bw < a.B && lane == 0) a.rec[(size_t)bw * a.P + p].flags = (int32_t)ch.flags;
}

// Fix-up pass, grid (ceil(B/NW), P-1): the searches of a workgroup rerun chunk
// p >= 1 from the last checkpoint row of chunk p-1 (their true row once chunk
// p-1 has met) until each row equals chunk p's checkpoint at a quad
// end; the tables are staged once per quad for all of them, a search that has
// met stops computing, and the workgroup stops when all have met.
template <int EP, int NW>
__global__ __launch_bounds__(64 * NW) void chain_wave_fix_kernel(WaveArgs a) {
  __shared__ __align__(16) WaveSmem<NW> sm;
  const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int bw = blockIdx.x * NW + wid;  // one search per wave
  const int p = blockIdx.y + 1;
  const int blk0 = p * a.CB, blk1 = min(blk0 + a.CB, a.nblk);
  const int i0 = blk0 * kWU;  // a multiple of 4
  const int b = min(bw, a.B - 1);
  WaveChain ch;
  wave_run<NW, kWFix, EP>(a, bw, true, blk0, blk1, 0, a.ckrow + ((size_t)b * a.nq + (i0 / 4 - 1)) * 64, sm, ch);
  if (bw >= a.B) return;
  if (ch.conv < 0) a.endrow[((size_t)bw * a.P + p) * 64 + lane] = ch.qv;
  if (lane == 0) {
    WaveRec &r = a.rec[(size_t)bw * a.P + p];
    r.conv = ch.conv;
    r.dfix = (int64_t)(ch.conv >= 0 ? ch.dconv : ch.dsum);
  }
}

// Final pass, one workgroup of 4 waves per search (see the top of the file);
// only wave 0 carries the search, the others keep the table staging shared.
constexpr int kWFinalWaves = 4;

template <int EP>
__global__ __launch_bounds__(64 * kWFinalWaves, 1) void chain_wave_final_kernel(WaveArgs a,
                                                                                SearchResult *__restrict__ res,
                                                                                int64_t *__restrict__ opt,
                                                                                int32_t *__restrict__ status) {
  __shared__ __align__(16) WaveSmem<kWFinalWaves> sm;
  __shared__ uint32_t s_row[64];  // the true end row of the last chunk accounted
  __shared__ int s_q, s_flags;
  __shared__ int64_t s_sum;
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int b = blockIdx.x, P = a.P;
  const int64_t *dk = a.dck + (size_t)b * a.nq;
  const WaveRec *rec = a.rec + (size_t)b * P;
  auto endq = [&](int p) __attribute__((always_inline)) { return (min((p + 1) * a.CB * kWU, a.N) - 1) >> 2; };
  // flags, by wave 1 during wave 0's first sum (by all waves behind it, with two more
  // barriers, the kernel took 1.1 us longer)
  if (wid == 1) {
    const int fl = lane < P ? rec[lane].flags : 0;
    u32x4 rb = {};
    for (int x = lane; x < a.nbad; x += 64) rb |= a.rbad[x];
    const bool bad = __any((fl & 1) || (rb.x | rb.y | rb.z | rb.w) != 0), infeasible = __any(fl & 2);
    if (lane == 0) s_flags = (bad ? 1 : 0) | (infeasible ? 2 : 0);
  }
  if (P == 1) __syncthreads();
  // Chunk 0 runs from the true first row.  At the top of the loop the chunks
  // below p are accounted in `total`; with spec_true the speculative end row of
  // chunk p-1 is its true one (so the fix-up of chunk p is valid), otherwise
  // s_row holds the true end row of chunk p-1.
  int64_t total = dk[endq(0)];
  const uint32_t qlast = a.ckrow[((size_t)b * a.nq + a.nq - 1) * 64 + lane];  // (in flight during the loop)
  bool spec_true = true, reruns = false;  // reruns: the run before was a rerun that met no checkpoint
  int p = 1;
  while (p < P) {
    if (spec_true) {
      // The first chunk q >= p whose fix-up met no checkpoint, and the offsets
      // of chunks p .. q (chunk q's fix-up ran from a true row to its end).
      if (wid == 0) {
        const int pl = p + lane;
        const bool in = pl < P;
        WaveRec r{};
        if (in) r = rec[pl];
        const uint64_t nc = __ballot(in && r.conv < 0);
        const int q = nc ? p + __ffsll((long long)nc) - 1 : P;
        int64_t delta = 0;
        if (in && pl < q) delta = r.dfix + dk[endq(pl)] - dk[r.conv];
        else if (in && pl == q) delta = r.dfix;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) delta += __shfl_xor(delta, off, 64);
        if (lane == 0) {
          s_q = q;
          s_sum = delta;
        }
      }
      __syncthreads();
      const int q = s_q;
      total += s_sum;
      if (q >= P) break;
      if (wid == 0) s_row[lane] = a.endrow[((size_t)b * P + q) * 64 + lane];
      spec_true = false;
      p = q + 1;
      __syncthreads();
    } else {
      // Rerun chunk p (wave 0; the others stage) at least over the rows its
      // fix-up rewrote from a wrong start; behind a rerun that met nothing
      // either, the rest of the chain in one run.
      WaveChain ch;
      const int last = reruns ? P - 1 : p;  // last chunk of the run
      const int qmin = reruns ? endq(P - 1) : rec[p].conv < 0 ? endq(p) : rec[p].conv;
      wave_run<kWFinalWaves, kWFix, EP, true>(a, b, wid == 0, p * a.CB, min((last + 1) * a.CB, a.nblk), qmin, s_row, sm,
                                              ch);
      __syncthreads();  // every wave has read s_row and the last tables
      if (wid == 0) {
        const bool met = ch.conv >= 0;
        if (lane == 0) {
          s_q = met;
          s_sum = met ? (int64_t)ch.dconv + dk[endq(last)] - dk[ch.conv] : (int64_t)ch.dsum;
        }
        s_row[lane] = ch.qv;
      }
      __syncthreads();
      total += s_sum;
      spec_true = s_q != 0;
      reruns = !spec_true;
      p = last + 1;
      __syncthreads();  // s_q is rewritten at the top of the loop
    }
  }
  const uint32_t qv = spec_true ? qlast : s_row[lane];
  if (wid != 0) return;
  // The final row has minimum 0: the lowest state at the minimum.
  const uint32_t pk = wave_min(lane < a.K ? (qv | (uint32_t)lane) : kSat);
  if (lane == 0) {
    int st = CFP_ST_OK;
    if (s_flags & 1) st = CFP_ST_BADINPUT;
    else if (s_flags & 2) st = CFP_ST_INFEASIBLE;
    else if ((pk >> kWBits) != 0) st = CFP_ST_OVERFLOW;
    status[b] = st;
    opt[b] = st == CFP_ST_OK ? total : INT64_MAX;
    res[b].final_state = st == CFP_ST_OK ? (int32_t)(pk & 63u) : -1;
    res[b].status = st;
    res[b].final_m = 0;
  }
}

struct WavePlan {
  int P, CB, nblk, nq;
  int NW;  // waves (searches) per workgroup
};

// Workgroups of four waves (one search per SIMD) while the batch's chunks fit
// the chip with them: a row then takes about 0.5 us where sixteen searches on
// four SIMDs take 1.1 us, whether they exist or repeat the last one (1152
// blocks, K = 64: one search 88 -> 70 us per call, 16 searches 109 -> 78 us).
// A chain too short for two chunks goes to the register-resident kernel when
// its tables fit there (0.32 us per row), else runs here as one chunk.
WavePlan wave_plan(int n, int k, int e, int batch) {
  WavePlan c{0, 0, 0, 0, 0};
  if (k <= 32 || k > 64) return c;
  c.nblk = (n + kWU - 1) / kWU;
  c.nq = (n + 3) / 4;
  c.NW = (batch + 3) / 4 * std::min(kWMaxChunks, c.nblk / kWMinBlocks) <= 256 ? 4 : kWWaves;
  const int rows = (batch + c.NW - 1) / c.NW;
  int P = std::max(1, 256 / rows);  // one workgroup per compute unit
  P = std::min(P, std::min(kWMaxChunks, c.nblk / kWMinBlocks));
  if (P < 2 && e <= kResTables) return WavePlan{0, 0, 0, 0, 0};
  P = std::max(P, 1);
  c.CB = (c.nblk + P - 1) / P;
  c.P = (c.nblk + c.CB - 1) / c.CB;
  return c;
}

template <int EP, int NW>
static void launch_wave_passes(const WaveArgs &a, SearchResult *res, int64_t *opt, int32_t *status,
                               hipStream_t st) {
  const int rows = (a.B + NW - 1) / NW;
  timer_begin(st);
  timed_launch(chain_wave_kernel<EP, NW>, dim3(rows, a.P), dim3(64 * NW), 0, st, a);
  timer_end(st);
  if (a.P > 1)
    hipLaunchKernelGGL((chain_wave_fix_kernel<EP, NW>), dim3(rows, a.P - 1), dim3(64 * NW), 0, st, a);
  hipLaunchKernelGGL((chain_wave_final_kernel<EP>), dim3(a.B), dim3(64 * kWFinalWaves), 0, st, a, res, opt, status);
}

}  // namespace

bool chain_wave_supported(int n, int k, int e, int batch) { return wave_plan(n, k, e, batch).P >= 1; }

size_t wave_region_bytes(int n, int k, int e, int batch) {
  const WavePlan c = wave_plan(n, k, e, batch);
  if (c.P < 1) return 0;
  size_t off = align_up((size_t)e * 64 * 64 * 4);
  off += align_up(kWPackBlocks * 4);
  off += align_up((size_t)batch * c.P * sizeof(WaveRec));
  off += align_up((size_t)batch * c.nq * 8);
  off += align_up((size_t)batch * c.nq * 64 * 4);
  off += align_up((size_t)batch * c.P * 64 * 4);
  return off;
}

hipError_t launch_chain_wave(const cfp_chain_desc &d, int32_t *redge_dev, const EdgeMap &em, uint8_t *region,
                             uint8_t *table, SearchResult *res, int64_t *opt, int32_t *status, hipStream_t st) {
  const WavePlan c = wave_plan(d.n_blocks, d.k, d.n_tables, d.batch);
  WaveArgs a;
  a.cost = d.cost;
  a.redge = redge_dev;
  a.N = d.n_blocks;
  a.K = d.k;
  a.E = d.n_tables;
  a.B = d.batch;
  a.P = c.P;
  a.CB = c.CB;
  a.nblk = c.nblk;
  a.nq = c.nq;
  a.table = table;
  size_t off = 0;
  uint32_t *rpk = (uint32_t *)(region + off);
  a.rpk = (const u32x4 *)rpk;
  off += align_up((size_t)d.n_tables * 64 * 64 * 4);
  uint8_t *rbad = region + off;
  off += align_up(kWPackBlocks * 4);
  a.rec = (WaveRec *)(region + off);
  off += align_up((size_t)d.batch * c.P * sizeof(WaveRec));
  a.dck = (int64_t *)(region + off);
  off += align_up((size_t)d.batch * c.nq * 8);
  a.ckrow = (uint32_t *)(region + off);
  off += align_up((size_t)d.batch * c.nq * 64 * 4);
  a.endrow = (uint32_t *)(region + off);
  a.rbad = (const u32x4 *)rbad;
  const int packs = std::min(kWPackBlocks, d.n_tables * 16);  // of four waves
  a.nbad = packs / 4;
  // the usual period, and table i for phase i: the table index is a constant per
  // row of a block, and the map is not needed
  bool periodic = em.period == kWU;
  for (int i = 1; periodic && i < em.head + kWU; ++i) periodic = em.map[i] == i % kWU;
  const int32_t rlimit = cfp_r_limit(CFP_V_CHAIN, d.k);
  if (periodic || em.period == 0)
    hipLaunchKernelGGL(wave_pack_kernel<NoMap>, dim3(packs), dim3(256), 0, st, d.rtab, d.n_tables, d.k, rpk, rlimit,
                       rbad, NoMap{}, redge_dev, d.n_blocks);
  else
    hipLaunchKernelGGL(wave_pack_kernel<EdgeMap>, dim3(packs), dim3(256), 0, st, d.rtab, d.n_tables, d.k, rpk, rlimit,
                       rbad, em, redge_dev, d.n_blocks);
  if (c.NW == 4) {
    if (periodic) launch_wave_passes<12, 4>(a, res, opt, status, st);
    else launch_wave_passes<0, 4>(a, res, opt, status, st);
  } else {
    if (periodic) launch_wave_passes<12, kWWaves>(a, res, opt, status, st);
    else launch_wave_passes<0, kWWaves>(a, res, opt, status, st);
  }
  return hipGetLastError();
}

}  // namespace cfp
