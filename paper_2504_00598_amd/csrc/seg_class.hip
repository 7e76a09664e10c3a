// Segment search over boundary classes (Sec. 4.2-4.4: Eq. T with resharding
// r[last(t)][first(s)]), one launch per forward call.
//
// Only the class (last, first) of a plan meets the neighbouring segments, so
// with C_i[l][f] = min over plans s of that class of c[i][s] (and a_i[l][f] its
// lowest plan) the recurrence is one over at most eight values per segment,
//     M_i[l]     = min_f G_i[f] + C_i[l][f],        G_0 = 0,
//     G_{i+1}[f] = min_l M_i[l] + r_{e(i+1)}[l][f],
// and the class minima, which hold all the K-sized work, do not depend on it.
// What is left is a chain of N-1 tiny min-plus products.  One workgroup of 16
// waves per search:
//   1. every wave: cost rows into LDS (coalesced), class minima with LM^2 lanes per
//      segment, normalised by the segment's least cost.  A lane takes a class, or,
//      where the map gives one class so many plans that its lane would set the time,
//      every lane an equal share of the plans in the order of their classes, combined
//      per class by LDS minima (96 segments, 8 x 8 boundary pairs, 441 of 512 plans in
//      one of them, 64 searches: 338 us per call with a lane per class, 50 so; even maps
//      are 10 to 50% slower so);
//   2. wave p runs chunk p of the chain from each of the LM unit vectors at
//      once (LM = 4 or 8 padded classes: lane (g, j) holds value j of the run
//      from unit vector g), i.e. it forms the chunk's transfer matrix;
//   3. wave p applies the matrices of the chunks before it to G_0 and reruns
//      its chunk from the vector that enters it, storing every G_i;
//   4. every wave: M_i, the lowest plan that attains G_{i+1}[f], and the
//      answer.  The argmin table has LM entries per segment (the lowest
//      predecessor depends on the plan's first class only).
// A row step is two half-steps of LM adds with a DPP operand (the values of a
// group of four or eight lanes reach each other by quad broadcasts and a half
// mirror) and a row minimum: about 0.1 us, with the next rows' words read
// ahead from LDS.  The matrices are exact: nothing is speculative.
// (The form this replaces ran the recurrence over all K plans of a segment in
// chunks with fix-ups, 0.28 us per row at K = 81: 96 segments, K = 81, 256
// searches 21.3 us per launch; 50 segments, K = 216, 2 searches 57 us.)
//
// Arithmetic.  R < 2^28.  G is kept relative to its minimum, so G <= R_max; a
// class without an available plan has C = kSegInf, above every C + G that is
// exact (costs relative to their row's minimum are below 2^31 - 1), and no sum
// of the two half-steps leaves 32 bits.  Offsets are 64-bit sums.
#include <algorithm>

#include "cfp_internal.h"
#include "common.h"

namespace cfp {

namespace {

constexpr int kScWaves = 16;
constexpr int kScThreads = 64 * kScWaves;
constexpr uint32_t kSegInf = 0xA0000000u;        // class without an available plan
constexpr uint32_t kSegPadR = 0x10000000u;       // boundary entry of a padding class, above every entry
constexpr int64_t kSegFar = (int64_t)1 << 50;    // offset of a start that no plan reaches
constexpr uint32_t kSegFarRel = 1u << 30;        // cap of a start's relative offset: beyond it never wins
constexpr int kScTileBytes = 48 * 1024;          // cost rows staged at once
constexpr size_t kScMaxLds = 150 * 1024;

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct ScArgs {
  const int32_t *cost, *rbound;
  const uint8_t *last, *first;
  const int32_t *redge;  // uploaded edge map, read when em.period is 0
  EdgeMap em;
  int N, K, B, E, L, F;
  int P, CL;             // chunks and steps per chunk
  int tile;              // cost rows staged at once
  int32_t rlimit;
  uint16_t *a0;          // [B][N][LM][LM] lowest plan of a class's least cost
  uint16_t *arg;         // [B][N][LM] lowest predecessor by the plan's first class
  SearchResult *res;
  int64_t *opt;
  int32_t *status;
};

// LDS of a search, in words: class minima, then (one region in turn) the staged
// cost rows and their class keys / the G, M and argument rows; the boundary tables;
// the edge map.
template <int LM>
struct ScLds {
  static __host__ __device__ size_t cls(int n) { return (size_t)n * LM * LM; }
  static __host__ __device__ size_t rows(int n) { return (size_t)n * (2 * LM + LM / 2); }
  // room for at least one row with its class keys of two words
  static __host__ __device__ size_t shared(int n, int tile, int k) {
    const size_t a = rows(n), b = (size_t)tile * k, c = (size_t)k + 1 + 2 * LM * LM;
    return a > b ? (a > c ? a : c) : (b > c ? b : c);
  }
  static __host__ __device__ size_t tables(int e) { return (size_t)e * LM * LM; }
  static __host__ __device__ size_t edges(int n) { return (size_t)(n + 1) / 2; }
};

template <int CTRL>
__device__ __forceinline__ uint32_t sc_dpp(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, CTRL, 0xF, 0xF, true);
}
constexpr int kScHalfMirror = 0x141, kScSwap1 = 0xB1, kScSwap2 = 0x4E, kScRor4 = 0x124, kScRor8 = 0x128;
template <int Q>
__device__ __forceinline__ uint32_t sc_quad(uint32_t x) { return sc_dpp<Q * 0x55>(x); }

// min over the group's values v_k + w_k: own holds w of the lane's own quad of
// four in order, oth that of the other quad (LM = 8).
template <int LM>
__device__ __forceinline__ uint32_t sc_half(uint32_t v, const u32x4 &own, const u32x4 &oth) {
  uint32_t m = umin(umin(sc_quad<0>(v) + own.x, sc_quad<1>(v) + own.y),
                    umin(sc_quad<2>(v) + own.z, sc_quad<3>(v) + own.w));
  if constexpr (LM == 8) {
    const uint32_t h = sc_dpp<kScHalfMirror>(v);  // lane j gets value 7 - j
    m = umin(m, umin(umin(sc_quad<0>(h) + oth.w, sc_quad<1>(h) + oth.z),
                     umin(sc_quad<2>(h) + oth.y, sc_quad<3>(h) + oth.x)));
  }
  return m;
}
// Minimum over the LM lanes of a group.
template <int LM>
__device__ __forceinline__ uint32_t sc_group_min(uint32_t x) {
  x = umin(x, sc_dpp<kScSwap1>(x));
  x = umin(x, sc_dpp<kScSwap2>(x));
  if constexpr (LM == 8) x = umin(x, sc_dpp<kScHalfMirror>(x));
  return x;
}
// Minimum over the LM groups at the same lane j (LM = 4: the groups of a row of 16).
template <int LM>
__device__ __forceinline__ uint32_t sc_across(uint32_t x) {
  if constexpr (LM == 4) x = umin(x, sc_dpp<kScRor4>(x));
  x = umin(x, sc_dpp<kScRor8>(x));
  if constexpr (LM == 8) {
    const auto a = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    x = umin(a[0], a[1]);
    const auto b = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    x = umin(b[0], b[1]);
  }
  return x;
}
// Minimum over the LM^2 lanes that hold the classes of one segment.
template <int LM>
__device__ __forceinline__ int32_t sc_row_min(int32_t x) {
  auto mn = [](int32_t a, int32_t b) { return b < a ? b : a; };
  x = mn(x, (int32_t)sc_dpp<kScSwap1>((uint32_t)x));
  x = mn(x, (int32_t)sc_dpp<kScSwap2>((uint32_t)x));
  x = mn(x, (int32_t)sc_dpp<kScHalfMirror>((uint32_t)x));
  x = mn(x, (int32_t)sc_dpp<0x140>((uint32_t)x));
  if constexpr (LM == 8) {
    const auto a = __builtin_amdgcn_permlane16_swap((uint32_t)x, (uint32_t)x, false, false);
    x = mn((int32_t)a[0], (int32_t)a[1]);
    const auto b = __builtin_amdgcn_permlane32_swap((uint32_t)x, (uint32_t)x, false, false);
    x = mn((int32_t)b[0], (int32_t)b[1]);
  }
  return x;
}

// The chain of one wave: steps t in [t0, t1) from the group's value v; FIRST:
// the first step starts from unit vector g.  Returns the offset sum; with G
// set, stores the vector of every row t0 .. t1-1 (and of row t1 where `tail`).
template <int LM, bool FIRST>
__device__ __forceinline__ int64_t sc_chain(const uint32_t *C, const uint32_t *rT, const uint16_t *red, int t0, int t1,
                                            uint32_t &v, uint32_t *G, bool tail) {
  const int lane = threadIdx.x & 63, j = lane & (LM - 1), g = (lane / LM) & (LM - 1);
  const int h = LM == 8 ? 4 * ((j >> 2) & 1) : 0;
  int64_t off = 0;
  if (t0 >= t1) {
    if (G && tail && lane < LM) G[t1 * LM + j] = v;
    return off;
  }
  // words of a row's class minima (the lane as l) and boundary entries (the lane as f)
  auto crow = [&](int t, u32x4 &own, u32x4 &oth) __attribute__((always_inline)) {
    const uint32_t *p = C + (size_t)t * LM * LM + j * LM;
    own = *(const u32x4 *)(p + h);
    oth = *(const u32x4 *)(p + (LM - 4 - h));
  };
  auto rrow = [&](int e, u32x4 &own, u32x4 &oth) __attribute__((always_inline)) {
    const uint32_t *p = rT + (size_t)e * LM * LM + j * LM;
    own = *(const u32x4 *)(p + h);
    oth = *(const u32x4 *)(p + (LM - 4 - h));
  };
  u32x4 c0, c1, r0, r1;
  uint32_t cf = 0;
  if (FIRST) cf = C[(size_t)t0 * LM * LM + j * LM + g];
  crow(t0, c0, c1);
  rrow(red[t0 + 1], r0, r1);
  int en = red[min(t0 + 2, t1)];
  for (int t = t0; t < t1; ++t) {
    if (G && lane < LM) G[t * LM + j] = v;
    u32x4 n0, n1, s0, s1;  // the next step's words
    const int tn = min(t + 1, t1 - 1);
    crow(tn, n0, n1);
    rrow(en, s0, s1);
    en = red[min(t + 3, t1)];
    uint32_t m = sc_half<LM>(v, c0, c1);
    if (FIRST && t == t0) m = cf;
    const uint32_t x = sc_half<LM>(m, r0, r1);
    const uint32_t d = sc_group_min<LM>(x);
    v = x - d;
    off += d;
    if (FIRST && t == t0 && d >= kSegInf) off += kSegFar;  // no plan starts with class g
    c0 = n0;
    c1 = n1;
    r0 = s0;
    r1 = s1;
  }
  if (G && tail && lane < LM) G[t1 * LM + j] = v;
  return off;
}

template <int LM>
__global__ __launch_bounds__(kScThreads) void seg_class_kernel(ScArgs a) {
  constexpr int L2 = LM * LM;
  extern __shared__ __align__(16) uint32_t sm[];
  __shared__ uint32_t X[kScWaves][LM][LM];    // chunk matrices, relative to their row offsets
  __shared__ uint32_t xr[kScWaves][LM];       // row offsets relative to the least
  __shared__ int64_t xo[kScWaves];            // least row offset
  __shared__ uint16_t order[CFP_MAX_K];       // plans by class, ascending within a class
  __shared__ uint8_t oclass[CFP_MAX_K];       // their classes
  __shared__ uint16_t wcount[CFP_MAX_K / 64][64];
  __shared__ int cstart[65];
  __shared__ int s_most;                      // plans of the largest class
  __shared__ unsigned long long csum;         // sum of the segments' least costs
  __shared__ int64_t s_off;                   // offset of the last vector
  const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int b = blockIdx.x, N = a.N, K = a.K, L = a.L, F = a.F;
  uint32_t *C = sm;
  uint32_t *stage = C + ScLds<LM>::cls(N);    // cost rows, later G, M and the arguments of M
  const size_t shared_words = ScLds<LM>::shared(N, a.tile, K);
  uint32_t *rT = stage + (shared_words + 3) / 4 * 4;
  uint16_t *red = (uint16_t *)(rT + ScLds<LM>::tables(a.E));
  const int32_t *cost = a.cost + (size_t)b * N * K;

  // The first tile of cost rows is on its way while the classes are sorted.
  constexpr int NV = 16;
  int32_t cv[NV];
  int rows = min(a.tile, N);
#pragma unroll
  for (int u = 0; u < NV; ++u) cv[u] = cost[min(u * kScThreads + tid, rows * K - 1)];

  // 1a. Boundary tables (transposed, padded), edge map, classes.
  bool bad = false;
  for (int x = tid; x < a.E * L2; x += kScThreads) {
    const int e = x / L2, f = (x / LM) % LM, l = x % LM;
    uint32_t w = kSegPadR;
    if (l < L && f < F) {
      const int32_t r = a.rbound[((size_t)e * L + l) * F + f];
      bad |= r < 0 || r >= a.rlimit;
      w = (uint32_t)r & (kSegPadR - 1);
    }
    rT[x] = w;
  }
  for (int i = tid; i < N; i += kScThreads)
    red[i] = i == 0 ? 0 : (uint16_t)(a.em.period ? a.em.at(i) : a.redge[i]);
  if (tid == 0) csum = 0;
  int cl = -1, rank = 0;
  if (wid < (K + 63) / 64) {
    if (tid < K) {
      int l = a.last[tid], f = a.first[tid];
      bad |= l >= L || f >= F;
      cl = min(l, L - 1) * LM + min(f, F - 1);
    }
    for (int p = 0; p < L2; ++p) {
      const uint64_t m = __ballot(cl == p);
      if (cl == p) rank = __popcll(m & ((1ull << lane) - 1));
      if (lane == 0) wcount[wid][p] = (uint16_t)__popcll(m);
    }
  }
  __syncthreads();
  if (wid == 0) {  // class starts: an exclusive scan over the (at most 64) classes
    int n = 0;
    if (lane < L2)
      for (int w = 0; w < (K + 63) / 64; ++w) n += wcount[w][lane];
    int s = n;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int y = __shfl_up(s, o, 64);
      if (lane >= o) s += y;
    }
    cstart[lane + 1] = s;
    if (lane == 0) cstart[0] = 0;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) n = max(n, __shfl_xor(n, o, 64));
    if (lane == 0) s_most = n;
  }
  __syncthreads();
  if (cl >= 0) {
    int pos = cstart[cl] + rank;
    for (int w = 0; w < wid; ++w) pos += wcount[w][cl];
    order[pos] = (uint16_t)tid;
    oclass[pos] = (uint8_t)cl;
  }

  // 1b. Class minima, tile by tile.
  const int per = (K + L2 - 1) / L2;     // plans per lane in equal shares
  const bool share = s_most > 3 * per + 4;
  const int tile = share ? min(a.tile, (int)((shared_words - 1) / (K + 2 * L2))) : a.tile;
  unsigned long long *key = (unsigned long long *)(stage + (tile * K + 1) / 2 * 2);  // share: cost << 16 | plan
  bool infeasible = false;
  unsigned long long sum = 0;
  for (int i0 = 0; i0 < N; i0 += tile) {
    rows = min(tile, N - i0);
    const int words = rows * K;
    for (int x0 = 0; x0 < words; x0 += NV * kScThreads) {
      if (i0 > 0 || x0 > 0) {
#pragma unroll
        for (int u = 0; u < NV; ++u)
          cv[u] = cost[(size_t)i0 * K + min(x0 + u * kScThreads + tid, words - 1)];
      }
#pragma unroll
      for (int u = 0; u < NV; ++u) {
        const int x = x0 + u * kScThreads + tid;
        bad |= cv[u] < 0;
        if (x < words) stage[x] = (uint32_t)cv[u];
      }
    }
    if (share)
      for (int x = tid; x < rows * L2; x += kScThreads) key[x] = ~0ull;
    __syncthreads();  // the rows (and, the first time, the order)
    if (share) {
      // A thread's plans are the same in every row: eight of them at a time.
      const int qbeg = (tid % L2) * per, qend = min(qbeg + per, K);
      for (int q0 = qbeg; q0 < qend; q0 += 8) {
        uint32_t o[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int q = min(q0 + u, qend - 1);
          o[u] = (uint32_t)oclass[q] << 16 | order[q];
        }
        for (int r = tid / L2; r < rows; r += kScThreads / L2) {
          uint32_t c[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) c[u] = stage[r * K + (o[u] & 0xFFFF)];
          uint32_t best = c[0], at = o[0];
#pragma unroll
          for (int u = 1; u < 8; ++u) {
            const bool next = (o[u] ^ at) >> 16 != 0;  // a new class (the last plan is repeated at the end)
            if (next) atomicMin(&key[r * L2 + (at >> 16)], (unsigned long long)best << 16 | (at & 0xFFFF));
            if (next || c[u] < best) {
              best = c[u];
              at = o[u];
            }
          }
          atomicMin(&key[r * L2 + (at >> 16)], (unsigned long long)best << 16 | (at & 0xFFFF));
        }
      }
      __syncthreads();  // the keys
    }
    // whole groups of LM^2 lanes take a segment each (padding classes have no plan)
    for (int x = tid; x < rows * L2; x += kScThreads) {
      const int r = x / L2, p = x % L2;
      int32_t best = CFP_COST_INF;
      int at = 0;
      if (share) {
        const unsigned long long k = key[x];
        if (k != ~0ull) {
          best = (int32_t)(k >> 16);
          at = (int)(k & 0xFFFF);
        }
      } else {
        const int32_t *row = (const int32_t *)stage + r * K;
        for (int q = cstart[p]; q < cstart[p + 1]; ++q) {
          const int s = order[q];
          const int32_t c = row[s];
          if (c < best) {
            best = c;
            at = s;
          }
        }
      }
      const int32_t lo = sc_row_min<LM>(best);
      const int i = i0 + r;
      C[(size_t)i * L2 + p] = best == CFP_COST_INF ? kSegInf : (uint32_t)(best - lo);
      a.a0[((size_t)b * N + i) * L2 + p] = (uint16_t)at;
      if (p == 0) {
        infeasible |= lo == CFP_COST_INF;
        sum += (unsigned long long)(long long)lo;
      }
    }
    __syncthreads();  // the staged rows and keys are done with
  }
  if (sum) atomicAdd(&csum, sum);
  int flags = __syncthreads_or(bad) ? 1 : 0;
  flags |= __syncthreads_or(infeasible) ? 2 : 0;

  // 2. Transfer matrix of chunk wid.
  const int T = N - 1, t0 = min(wid * a.CL, T), t1 = min(t0 + a.CL, T);
  const int j = lane & (LM - 1), g = (lane / LM) & (LM - 1);
  if (wid < a.P - 1) {
    uint32_t v = 0;
    const int64_t off = sc_chain<LM, true>(C, rT, red, t0, t1, v, nullptr, false);
    // the least offset over the starts, and the offsets relative to it
    int64_t lo = off;
#pragma unroll
    for (int o = LM; o < LM * LM; o <<= 1) {
      const int64_t y = __shfl_xor((long long)lo, o, 64);
      lo = y < lo ? y : lo;
    }
    if (lane < L2) {
      X[wid][g][j] = v;
      if (j == 0) xr[wid][g] = (uint32_t)min(off - lo, (int64_t)kSegFarRel);
      if (lane == 0) xo[wid] = lo;
    }
  }
  __syncthreads();

  // 3. The vector that enters the chunk, then the chunk from it.
  uint32_t *G = stage, *M = G + (size_t)N * LM;
  uint16_t *am = (uint16_t *)(M + (size_t)N * LM);
  if (wid < a.P) {
    uint32_t vj = 0, vg = 0;  // value j (the same in every group), value g
    int64_t off = 0;
    for (int c = 0; c < wid; ++c) {
      const uint32_t x = sc_across<LM>(vg + xr[c][g] + X[c][g][j]);
      const uint32_t d = sc_group_min<LM>(x);
      vj = x - d;
      off += xo[c] + (int64_t)d;
      vg = (uint32_t)__shfl((int)vj, g, 64);
    }
    off += sc_chain<LM, false>(C, rT, red, t0, t1, vj, G, wid == a.P - 1);
    if (wid == a.P - 1 && lane == 0) s_off = off;
  }
  __syncthreads();

  // 4. M with its lowest plans, then the lowest predecessor of every first class.
  for (int x = tid; x < N * LM; x += kScThreads) {
    const int i = x / LM, l = x % LM;
    const uint32_t *Gi = G + i * LM, *Cl = C + (size_t)i * L2 + l * LM;
    const uint16_t *al = a.a0 + ((size_t)b * N + i) * L2 + l * LM;
    uint32_t best = kSat, at = 0xFFFF;
#pragma unroll
    for (int f = 0; f < LM; ++f) {
      const uint32_t v = Gi[f] + Cl[f], s = al[f];
      if (v < best || (v == best && s < at)) {
        best = v;
        at = s;
      }
    }
    M[x] = best;
    am[x] = (uint16_t)at;
  }
  __syncthreads();
  for (int x = tid + LM; x < N * LM; x += kScThreads) {  // row i >= 1, first class f
    const int i = x / LM, f = x % LM;
    const uint32_t *Mi = M + (i - 1) * LM, *rf = rT + (size_t)red[i] * L2 + f * LM;
    uint32_t best = kSat, at = 0xFFFF;
#pragma unroll
    for (int l = 0; l < LM; ++l) {
      const uint32_t v = Mi[l] + rf[l], s = am[(i - 1) * LM + l];
      if (v < best || (v == best && s < at)) {
        best = v;
        at = s;
      }
    }
    a.arg[((size_t)b * N + i) * LM + f] = (uint16_t)at;
  }
  if (tid == 0) {
    uint32_t best = kSat;
    int at = 0;
    for (int l = 0; l < LM; ++l) {
      const uint32_t v = M[(N - 1) * LM + l];
      const int s = am[(N - 1) * LM + l];
      if (v < best || (v == best && s < at)) {
        best = v;
        at = s;
      }
    }
    int st = CFP_ST_OK;
    if (flags & 1) st = CFP_ST_BADINPUT;
    else if (flags & 2) st = CFP_ST_INFEASIBLE;
    a.status[b] = st;
    a.opt[b] = st == CFP_ST_OK ? (int64_t)csum + s_off + (int64_t)best : INT64_MAX;
    a.res[b].final_state = st == CFP_ST_OK ? at : -1;
    a.res[b].status = st;
    a.res[b].final_m = 0;
  }
}

// Plan recovery from the class table: the first class of segment i's plan names
// the plan of segment i-1, so a step is a map of at most eight classes, packed
// in a word of eight nibbles.  Lane k of the first wave composes the maps of a
// run of rows (from the last row down), a scan over the lanes gives the class
// that enters each run, and each lane writes its run's plans.
constexpr int kStThreads = 256;

__device__ __forceinline__ uint32_t sc_compose(uint32_t first, uint32_t then) {
  uint32_t r = 0;
#pragma unroll
  for (int f = 0; f < 8; ++f) r |= ((then >> (4 * ((first >> (4 * f)) & 7))) & 7u) << (4 * f);
  return r;
}

template <int LM>
__global__ __launch_bounds__(kStThreads) void seg_class_tb_kernel(int N, int K, const uint16_t *__restrict__ arg,
                                                                  const uint8_t *__restrict__ first,
                                                                  const SearchResult *__restrict__ res,
                                                                  int32_t *__restrict__ plan) {
  extern __shared__ __align__(16) uint16_t rows[];  // [N][LM]
  __shared__ uint8_t fc[CFP_MAX_K];
  const int b = blockIdx.x, tid = threadIdx.x;
  int32_t *pb = plan + (size_t)b * N;
  if (res[b].status != CFP_ST_OK) {
    for (int i = tid; i < N; i += kStThreads) pb[i] = -1;
    return;
  }
  const uint16_t *src = arg + (size_t)b * N * LM;
  for (int x = LM + tid; x < N * LM; x += kStThreads) rows[x] = src[x];
  for (int s = tid; s < K; s += kStThreads) fc[s] = first[s];
  __syncthreads();
  if (tid >= 64) return;
  const int fin = res[b].final_state;
  if (tid == 0) pb[N - 1] = fin;
  const int T = N - 1, Q = (T + 63) / 64;
  const int hi = N - 1 - tid * Q, lo = max(hi - Q, 0);  // rows hi .. lo+1 of this lane
  uint32_t map = 0x76543210u;
  for (int i = hi; i > lo; --i) {
    uint32_t w = 0;
#pragma unroll
    for (int f = 0; f < LM; ++f) w |= (uint32_t)(fc[min((int)rows[i * LM + f], K - 1)] & 7u) << (4 * f);
    map = sc_compose(map, w);
  }
  uint32_t inc = map;  // maps of the lanes up to this one, composed
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = (uint32_t)__shfl_up((int)inc, o, 64);
    if (tid >= o) inc = sc_compose(y, inc);
  }
  uint32_t before = (uint32_t)__shfl_up((int)inc, 1, 64);
  if (tid == 0) before = 0x76543210u;
  int f = (int)((before >> (4 * fc[fin])) & 7u);
  for (int i = hi; i > lo; --i) {
    const int t = min((int)rows[i * LM + f], K - 1);
    pb[i - 1] = t;
    f = fc[t] & (LM - 1);
  }
}

int sc_lm(int n_last, int n_first) { return n_last <= 4 && n_first <= 4 ? 4 : 8; }

int sc_tile(int n, int k) { return std::max(1, std::min(n, kScTileBytes / (4 * k))); }

template <int LM>
size_t sc_lds(int n, int k, int e) {
  const size_t shared = ScLds<LM>::shared(n, sc_tile(n, k), k);
  return 4 * (ScLds<LM>::cls(n) + (shared + 3) / 4 * 4 + ScLds<LM>::tables(e) + ScLds<LM>::edges(n));
}

template <int LM>
hipError_t launch_sc(const ScArgs &a, hipStream_t st) {
  const size_t lds = sc_lds<LM>(a.N, a.K, a.E);
  timer_begin(st);
  timed_launch(seg_class_kernel<LM>, dim3(a.B), dim3(kScThreads), (uint32_t)lds, st, a);
  timer_end(st);
  return hipGetLastError();
}

}  // namespace

// The class minima and the rows of a search have to fit in LDS (about 1400
// segments with up to four boundary strategies, 400 with more), as do the
// boundary tables; other chains take the chunked form.  So do, as measured,
//   * few classes of many plans on chains long enough, where the minima are the work
//     and not the chain (more than 24 plans per class on average, 32768 costs per
//     search: K = 512 of one class, 384 segments, one search 200 us here against 115; K
//     = 128 of four, 1000 segments 92 against 72; K = 64 of one, 200 segments 26
//     against 34);
//   * batches of more than 768 searches, whose workgroups of sixteen waves run in
//     rounds (96 segments, K = 81: 512 searches 30 us here against 41, 1000 53 against
//     47, 4096 192 against 124), but for many plans in many classes and rows, which the
//     other form holds in more registers (K = 512 with 8 x 8 pairs, 200 segments, 1000
//     searches 250 us here against 480; 12 segments 51 against 49).
bool seg_class_supported(const cfp_segment_desc &d) {
  if (d.n_segments > (1 << 16) || d.n_tables > 4096) return false;
  const int64_t costs = (int64_t)d.n_segments * d.k;
  const int lm = sc_lm(d.n_last, d.n_first);
  if (d.k > 24 * d.n_last * d.n_first && costs > 32768) return false;
  if (d.batch > 768 && !(lm == 8 && d.k >= 200 && costs >= (int64_t)12 * d.batch)) return false;
  const size_t lds = lm == 4 ? sc_lds<4>(d.n_segments, d.k, d.n_tables) : sc_lds<8>(d.n_segments, d.k, d.n_tables);
  return lds <= kScMaxLds;
}

size_t seg_class_bytes(int n, int batch) {
  return align_up((size_t)batch * n * 64 * 2) + align_up((size_t)batch * n * 8 * 2);
}

hipError_t launch_seg_class(const cfp_segment_desc &d, const int32_t *redge_dev, const EdgeMap &em, uint8_t *region,
                            SearchResult *res, int64_t *opt, int32_t *status, hipStream_t st) {
  ScArgs a;
  a.cost = d.cost;
  a.rbound = d.rbound;
  a.last = d.last;
  a.first = d.first;
  a.redge = redge_dev;
  a.em = em;
  a.N = d.n_segments;
  a.K = d.k;
  a.B = d.batch;
  a.E = d.n_tables;
  a.L = d.n_last;
  a.F = d.n_first;
  // A chunk costs two runs of its rows and every chunk before it one product:
  // about sqrt(2 T) chunks.
  const int T = a.N - 1;
  int P = 1;
  while (P < kScWaves && P * P < 2 * T) ++P;
  a.CL = std::max(1, (T + P - 1) / P);
  a.P = std::max(1, (T + a.CL - 1) / a.CL);
  a.tile = sc_tile(a.N, a.K);
  a.rlimit = cfp_r_limit(CFP_V_SEG, d.k);
  a.a0 = (uint16_t *)region;
  a.arg = (uint16_t *)(region + align_up((size_t)d.batch * d.n_segments * 64 * 2));
  a.res = res;
  a.opt = opt;
  a.status = status;
  return sc_lm(d.n_last, d.n_first) == 4 ? launch_sc<4>(a, st) : launch_sc<8>(a, st);
}

hipError_t launch_seg_class_tb(const cfp_segment_desc &d, const uint8_t *region, const SearchResult *res, int32_t *plan,
                               hipStream_t st) {
  const uint16_t *arg = (const uint16_t *)(region + align_up((size_t)d.batch * d.n_segments * 64 * 2));
  const int lm = sc_lm(d.n_last, d.n_first);
  const size_t lds = (size_t)d.n_segments * lm * 2;
  if (lm == 4)
    hipLaunchKernelGGL(seg_class_tb_kernel<4>, dim3(d.batch), dim3(kStThreads), lds, st, d.n_segments, d.k, arg,
                       d.first, res, plan);
  else
    hipLaunchKernelGGL(seg_class_tb_kernel<8>, dim3(d.batch), dim3(kStThreads), lds, st, d.n_segments, d.k, arg,
                       d.first, res, plan);
  return hipGetLastError();
}

}  // namespace cfp
