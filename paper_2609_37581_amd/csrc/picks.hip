// Context preservation by farthest point sampling (Sec. 4.1, after Eq. (7)):
// K_d tokens are added one at a time to the pivot set, each the candidate
// whose cosine distance 1 - zbar_i . zbar_j to the nearest already-selected
// token is largest (ties to the lower index).
//
// A pick needs the distance of every candidate to one more token, and each
// depends on the one before.  Re-reading Z for each pick would cost K_d passes
// over Z; the Gram matrix of all tokens holds every distance, but most of it
// is never used.  What is always needed are the distances to the pivots, of
// which only the least per token counts: one product of pivots and other
// tokens that leaves maxima, a fraction of the Gram matrix and without its
// writes.  Distances only shrink as picks are made, so the picks come from
// the top of that order: a round takes the C farthest tokens, forms their Gram
// matrix, and picks among them until a token outside this pool could be
// farther.  Distances are then brought up to date and the next round follows.
// Where the rounds do not suffice (tokens in many large clusters), and where
// the problem is so small that a round saves nothing, the picks are made over
// the Gram matrix of all tokens.
#include <algorithm>
#include <climits>

#include "../../include/trevs.h"
#include "common.hpp"
#include "kernels.hpp"
#include "select.hpp"

namespace trevs {

__device__ __forceinline__ bool picks_done(const PickArgs& a, int b) {
  return a.ctrl[b * kPickCtrl + kCtrlPicks] >= a.K_d;
}

// ---------------------------------------------------------------------------
// Initial distances over the full Gram matrix: for every token i the maximum
// over the pivots j of G_ij / ||z_j||.  One thread per token; the pivots are
// split over n_psplit workgroups per token block (grid z), each writing the
// maximum over its share; the picks kernel takes the maximum over the splits
// (exact, so the order does not matter) and forms the distance.  The pivot loop
// is unrolled so that several row reads of G are in flight (a pivot's row is
// read at consecutive columns by consecutive threads).
// ---------------------------------------------------------------------------
constexpr int kFpsInitThreads = 256;

__global__ __launch_bounds__(kFpsInitThreads) void fps_init_kernel(PickArgs a) {
  const int b = blockIdx.y, split = blockIdx.z, N = a.N, ldg = a.p.ldg;
  const int i = min((int)(blockIdx.x * kFpsInitThreads + threadIdx.x), N - 1);
  const float* gb = a.G + (size_t)b * N * ldg;
  const float* inb = a.inv_norm + (size_t)b * N;
  const int per = (a.K_r + a.p.n_psplit - 1) / a.p.n_psplit;
  const int p_begin = min(split * per, a.K_r), p_end = min(p_begin + per, a.K_r);
  const int32_t* piv = a.pivots + (size_t)b * a.K_r;
  constexpr int U = 8;
  float mx = -INFINITY;
  int p = p_begin;
  for (; p + U <= p_end; p += U) {
    int j[U];
    float g[U], izj[U];
#pragma unroll
    for (int u = 0; u < U; ++u) j[u] = piv[p + u];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      g[u] = gb[(size_t)j[u] * ldg + i];
      izj[u] = inb[j[u]];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) mx = fmaxf(mx, g[u] * izj[u]);
  }
  for (; p < p_end; ++p) {
    const int j = piv[p];
    mx = fmaxf(mx, gb[(size_t)j * ldg + i] * inb[j]);
  }
  if (blockIdx.x * kFpsInitThreads + threadIdx.x < N) a.part[((size_t)split * a.B + b) * N + i] = mx;
}

// ---------------------------------------------------------------------------
// Pool of a round: one workgroup per sample brings the distances of the
// sample's other tokens (rest) up to date with the maxima that the list
// products left (round 0: over the pivots; later: over the last round's
// picks), and keeps the C farthest, in index order.  No token outside the pool
// is farther than the C-th largest distance (the bound), and those at that
// distance follow the pool's in index order.
// ---------------------------------------------------------------------------
template <int E>
__global__ __launch_bounds__(kSelThreads) void pool_select_kernel(PickArgs a, int round, int row_tile) {
  __shared__ SelectShared sh;
  __shared__ int first_tie;
  const int b = blockIdx.x, tid = threadIdx.x, R = a.R, C = a.p.C;
  if (picks_done(a, b)) return;
  int32_t* ctrl = a.ctrl + b * kPickCtrl;
  const int n_rows = round ? ctrl[kCtrlPicks] - ctrl[kCtrlRound] : a.K_r;
  const int n_tiles = (n_rows + row_tile - 1) / row_tile;
  const int32_t* rest = a.rest + (size_t)b * R;
  float* dist = a.dist + (size_t)b * a.N;
  const float* mxp = a.mx + (size_t)b * R;
  const size_t tstride = (size_t)a.B * R;
  if (tid == 0) first_tie = INT_MAX;
  float d[E];
  int tok[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    d[e] = -INFINITY;
    tok[e] = rest[min(e * kSelThreads + tid, R - 1)];
  }
  for (int t = 0; t < n_tiles; ++t) {
    float v[E];
#pragma unroll
    for (int e = 0; e < E; ++e) v[e] = mxp[t * tstride + min(e * kSelThreads + tid, R - 1)];
#pragma unroll
    for (int e = 0; e < E; ++e) d[e] = fmaxf(d[e], v[e]);
  }
  {
    float v[E];
    const float* src = round ? dist : a.inv_norm + (size_t)b * a.N;
#pragma unroll
    for (int e = 0; e < E; ++e) v[e] = src[tok[e]];
#pragma unroll
    for (int e = 0; e < E; ++e) d[e] = round ? (-d[e] < v[e] ? -d[e] : v[e]) : 1.f - d[e] * v[e];
  }
  uint32_t key[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    if (e * kSelThreads + tid < R) dist[tok[e]] = d[e];
    key[e] = f2key(d[e]);
  }
  int32_t* cand = a.cand + (size_t)b * C;
  float* cand_dist = a.cand_dist + (size_t)b * C;
  auto put = [&](int at, int e) {
    cand[at] = tok[e];
    cand_dist[at] = d[e];
  };
  float bound = -INFINITY;
  if (C >= R) {
#pragma unroll
    for (int e = 0; e < E; ++e)
      if (e * kSelThreads + tid < R) put(e * kSelThreads + tid, e);
  } else {
    uint32_t thr;
    int tie = INT_MAX;
    block_topk_each<E>(
        key, R, C,
        [&](int e, bool ok, bool keep, int before) {
          if (keep && before < C) put(before, e);
          if (ok && !keep && key[e] == thr) tie = min(tie, tok[e]);
        },
        sh, false, 0u, 0u, &thr);
    bound = key2f(thr);
    if (tie != INT_MAX) atomicMin(&first_tie, tie);
  }
  __syncthreads();
  if (tid == 0) {
    ctrl[kCtrlTie] = first_tie;
    ctrl[kCtrlBound] = __float_as_int(bound);
  }
}

// ---------------------------------------------------------------------------
// The picks, one workgroup per sample, over the pool of a round or (FULL) over
// all tokens, with the distances in registers: element e of thread t is entry
// (e / CH) * CH * 1024 + t * CH + e % CH, so that rows of G load as vectors of
// CH values.
// A step that reduces over the workgroup and then waits for a row of G takes
// about 2 us, so the picks are made in batches.  The entries with the largest
// distances (at most kBatch: those in the first bins of a scale that starts at
// the largest) go with their mutual distances to LDS; one wave picks among
// them, without a barrier, for as long as the best of them is above every
// other distance; then all entries take the rows of the picks at once.
// Where more than kBatch entries share the first bin the scale is refined, and
// where that many tie exactly the batch takes them by index.
// A pick must also come before every token outside the pool: its distance is
// above the round's bound, or equal and earlier in index order.  The round
// ends where that fails; at K_d picks the kept list is written.
// ---------------------------------------------------------------------------
constexpr int kMaxPool = 4096;  // entries of a pool (four per thread)
constexpr int kBatch = 64;
constexpr int kBins = 512;     // of the scale; at most 64 of TREVS_MAX_FPS_N indices each
constexpr int kZooms = 6;      // refinements of the scale, by 16 each
static_assert(TREVS_MAX_FPS_N <= kBins * kBatch, "a bin of indices fits a batch");
static_assert(TREVS_MAX_FPS_N / 32 <= kSelThreads, "a word of the kept list per thread");

template <int CH>
struct Chunk;
template <>
struct Chunk<1> {
  typedef float T;
  static __device__ __forceinline__ float at(const T& v, int) { return v; }
};
template <>
struct Chunk<2> {
  typedef float2 T;
  static __device__ __forceinline__ float at(const T& v, int i) { return i ? v.y : v.x; }
};
template <>
struct Chunk<4> {
  typedef float4 T;
  static __device__ __forceinline__ float at(const T& v, int i) {
    return i == 0 ? v.x : (i == 1 ? v.y : (i == 2 ? v.z : v.w));
  }
};

template <int E, bool FULL>
__global__ __launch_bounds__(kSelThreads) void pick_kernel(PickArgs a) {
  constexpr int CH = E < 4 ? E : 4;        // entries per vector
  constexpr int NR = E / CH;               // vectors per thread and row
  constexpr int U = E <= 2 ? 16 : 32 / E;  // rows in flight
  typedef typename Chunk<CH>::T Vec;
  __shared__ float red[kSelWaves], red_out[kSelWaves];
  __shared__ int wtot[kSelWaves];
  __shared__ uint32_t hist[kBins];
  __shared__ float bdist[kBatch], biz[kBatch], piz[kBatch];
  __shared__ int bc[kBatch], pc[kBatch];
  __shared__ float sub[kBatch][kBatch + 1];
  __shared__ int n_batch, n_new;
  __shared__ uint32_t bits[kSelThreads];
  static_assert(kBins == 8 * kWave, "eight bins a lane");
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const int n = FULL ? a.N : a.p.C, ldg = FULL ? a.p.ldg : a.p.ldc, K_d = a.K_d, N = a.N, K_r = a.K_r;
  if (picks_done(a, b)) return;
  int32_t* ctrl = a.ctrl + b * kPickCtrl;
  const int t0 = ctrl[kCtrlPicks];
  int t = t0;
  const bool after_rounds = FULL && a.p.rounds > 0;
  const float bound = FULL ? -INFINITY : __int_as_float(ctrl[kCtrlBound]);
  const int tie_tok = FULL ? INT_MAX : ctrl[kCtrlTie];
  const int32_t* cand = FULL ? nullptr : a.cand + (size_t)b * n;
  const float* G = a.G + (size_t)b * n * ldg;
  int32_t* picks = a.picks + (size_t)b * K_d;
  const int words = (N + 31) / 32;
  auto entry = [&](int e) { return (e / CH) * CH * kSelThreads + tid * CH + e % CH; };
  auto token = [&](int c) { return FULL ? c : cand[c]; };
  // bit i: token i is a pivot, or one of the picks [0, np)
  auto mark = [&](int np) {
    if (tid < words) bits[tid] = 0u;
    __syncthreads();
    for (int p = tid; p < K_r; p += kSelThreads) {
      const int j = min(max(a.pivots[(size_t)b * K_r + p], 0), N - 1);
      atomicOr(&bits[j >> 5], 1u << (j & 31));
    }
    for (int p = tid; p < np; p += kSelThreads) {
      const int j = min(max(picks[p], 0), N - 1);
      atomicOr(&bits[j >> 5], 1u << (j & 31));
    }
    __syncthreads();
  };
  // selected entries and those past n hold distance -inf: they never win, and
  // the row updates (a minimum) keep them there
  float dist[E], iz[E];
  if (FULL) mark(0);
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int c = entry(e), cc = min(c, n - 1);
    iz[e] = a.inv_norm[(size_t)b * N + token(cc)];
    float d;
    if (!FULL) {
      d = a.cand_dist[(size_t)b * n + cc];
    } else if (after_rounds) {
      d = a.dist[(size_t)b * N + cc];
    } else {
      float mx = a.part[(size_t)b * N + cc];
      for (int sp = 1; sp < a.p.n_psplit; ++sp) mx = fmaxf(mx, a.part[((size_t)sp * a.B + b) * N + cc]);
      d = 1.f - mx * iz[e];
    }
    if (c >= n || (FULL && ((bits[cc >> 5] >> (cc & 31)) & 1u))) d = -INFINITY;
    dist[e] = d;
  }
  // the rows of picks p[0, np) (entries pc, inverse norms piz), U at a time;
  // every load of a group is issued before the first is used
  auto take_rows = [&](int np) {
    for (int q0 = 0; q0 < np; q0 += U) {
      Vec g[U][NR];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const float* row = G + (size_t)__builtin_amdgcn_readfirstlane(pc[min(q0 + u, np - 1)]) * ldg;
#pragma unroll
        for (int r = 0; r < NR; ++r) {
          const int c = entry(r * CH);
          g[u][r] = *reinterpret_cast<const Vec*>(row + (c < ldg ? c : 0));
        }
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const float izw = piz[min(q0 + u, np - 1)];
#pragma unroll
        for (int e = 0; e < E; ++e) {
          const float nd = 1.f - Chunk<CH>::at(g[u][e / CH], e % CH) * iz[e] * izw;
          dist[e] = nd < dist[e] ? nd : dist[e];
        }
      }
    }
  };
  if (after_rounds) {  // the last round's picks are not yet in the distances
    for (int p0 = ctrl[kCtrlRound]; p0 < t0; p0 += kBatch) {
      const int np = min(kBatch, t0 - p0);
      __syncthreads();
      if (tid < np) {
        pc[tid] = min(max(picks[p0 + tid], 0), N - 1);
        piz[tid] = a.inv_norm[(size_t)b * N + pc[tid]];
      }
      __syncthreads();
      take_rows(np);
    }
  }
  auto eligible = [&](float d, int c) { return d > bound || (d == bound && d > -INFINITY && token(c) < tie_tok); };
  // the scale starts as wide as a pick can lie below the top: down to the
  // bound (-1), or anywhere (distances lie in 0..2)
  const float range0 = bound > -INFINITY ? -1.f : 2.f;
  float range = range0;
  int ishift = 0;  // a bin of indices
  while ((n - 1) >> ishift >= kBins) ++ishift;
  while (t < K_d) {
    // ---- the largest distance
    float v = dist[0];
#pragma unroll
    for (int e = 1; e < E; ++e) v = fmaxf(v, dist[e]);
    v = wave_max(v);
    if (lane == 0) red[wave] = v;
    if (tid == 0) n_batch = 0;
    if (tid < kBins) hist[tid] = 0u;
    __syncthreads();
    const float top = wave_max(lane < kSelWaves ? red[lane] : -INFINITY);
    if (!(top > -INFINITY) || !(top >= bound)) break;  // uniform
    if (range < 0.f) range = top - bound;
    // ---- the cut: the most bins of the scale that hold at most kBatch entries
    bool ties = false;  // the scale is the index, of the entries at the top
    float scale = 0.f;
    int cut = 0;
    auto bin_of = [&](float d, int c) {
      if (ties) return d == top ? c >> ishift : kBins;
      return d >= top ? 0 : (int)fminf((top - d) * scale, (float)kBins);
    };
    for (int zoom = 0;; ++zoom) {
      ties = zoom >= kZooms || !(range > 0.f);
      scale = (float)kBins / range;
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const int bin = bin_of(dist[e], entry(e));
        if (bin < kBins && eligible(dist[e], entry(e))) atomicAdd(&hist[bin], 1u);
      }
      __syncthreads();
      int c[8], sum = 0;
#pragma unroll
      for (int j = 0; j < 8; ++j) sum += c[j] = (int)hist[8 * lane + j];
      int before = wave_incl_scan(sum, lane) - sum, mine = 0;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        before += c[j];
        mine += before <= kBatch ? 1 : 0;  // bins 0..8*lane+j hold at most kBatch entries
      }
      cut = wave_reduce_bits(mine, 0, [](int x, int y) { return x + y; });
      if (cut > 0 || ties) break;  // uniform (a bin of indices holds at most kBatch)
      range *= 1.f / 16.f;
      __syncthreads();  // hist has been read
      if (tid < kBins) hist[tid] = 0u;
      __syncthreads();
    }
    // ---- the batch, and the largest distance outside it
    float out = bound;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int c = entry(e);
      if (bin_of(dist[e], c) < cut && eligible(dist[e], c)) {
        const int at = atomicAdd(&n_batch, 1);
        if (at < kBatch) {
          bdist[at] = dist[e];
          biz[at] = iz[e];
          bc[at] = c;
        }
      } else {
        out = fmaxf(out, dist[e]);
      }
    }
    out = wave_max(out);
    if (lane == 0) red_out[wave] = out;
    __syncthreads();
    const int m = min(n_batch, kBatch);
    if (m == 0) break;  // uniform: the largest distance ties with an earlier token outside the pool
    constexpr int SUBS = kBatch * kBatch / kSelThreads;
    float sv[SUBS];
#pragma unroll
    for (int k = 0; k < SUBS; ++k) {
      const int x = min(wave + k * kSelWaves, m - 1), y = min(lane, m - 1);
      sv[k] = G[(size_t)bc[x] * ldg + bc[y]];
    }
#pragma unroll
    for (int k = 0; k < SUBS; ++k) {
      const int x = min(wave + k * kSelWaves, m - 1), y = min(lane, m - 1);
      sub[wave + k * kSelWaves][lane] = 1.f - sv[k] * biz[y] * biz[x];
    }
    __syncthreads();
    // ---- one wave picks among the batch
    if (wave == 0) {
      const float floor_ = wave_max(lane < kSelWaves ? red_out[lane] : -INFINITY);
      const int l = min(lane, m - 1);
      float d = lane < m ? bdist[lane] : -INFINITY;
      const int cl = bc[l];
      const int n_max = min(m, K_d - t);
      int won = 0, k = 0;  // lane k: the batch entry of pick k
      for (; k < n_max; ++k) {
        const float vm = wave_max(d);
        // above every other entry, or the top itself: the first pick, and ties by index
        if (!(vm > floor_) && !(vm == top && (ties || k == 0))) break;
        unsigned long long bal = __ballot(d == vm);
        if (bal & (bal - 1)) {  // uniform: a tie goes to the lower index
          const uint32_t c0 = wave_min_u32(d == vm ? (uint32_t)cl : 0xffffffffu);
          bal = __ballot(d == vm && (uint32_t)cl == c0);
        }
        const int w = __builtin_amdgcn_readfirstlane((int)__builtin_ctzll(bal));
        const float nd = sub[w][lane];
        d = nd < d ? nd : d;
        d = lane == w ? -INFINITY : d;
        won = lane == k ? w : won;
      }
      if (lane == 0) n_new = k;
      if (lane < k) {
        const int c = bc[won], tok = token(c);
        pc[lane] = c;
        piz[lane] = biz[won];
        picks[t + lane] = tok;
        if (a.div_idx) a.div_idx[(size_t)b * K_d + t + lane] = tok;
      }
    }
    __syncthreads();
    const int np = n_new;
    if (np == 0) break;  // uniform
    take_rows(np);
    for (int q = 0; q < np; ++q) {
      const int c = pc[q];
#pragma unroll
      for (int e = 0; e < E; ++e)
        if (c == entry(e)) dist[e] = -INFINITY;
    }
    t += np;
    // a batch that is far from full asks for a wider scale
    if (m < kBatch / 2) range = m < kBatch / 8 ? range0 : 2.f * range;
  }
  __syncthreads();  // the picks written above
  if (!FULL) {  // picked tokens leave the distances that the next round reads
    for (int p = t0 + tid; p < t; p += kSelThreads) a.dist[(size_t)b * N + picks[p]] = -INFINITY;
    if (tid == 0) {
      ctrl[kCtrlPicks] = t;
      ctrl[kCtrlRound] = t0;
    }
    if (t < K_d) return;  // uniform
  }
  if (t < K_d) {  // only distances that are not numbers are left: token 0 stands in
    for (int p = t + tid; p < K_d; p += kSelThreads) {
      picks[p] = 0;
      if (a.div_idx) a.div_idx[(size_t)b * K_d + p] = 0;
    }
    t = K_d;
    __syncthreads();
  }
  // ---- the kept list: pivots and picks in ascending order, one word of 32
  // tokens per thread
  mark(t);
  uint32_t word = tid < words ? bits[tid] : 0u;
  const int cnt = __popc(word), inc = wave_incl_scan(cnt, lane);
  if (lane == kWave - 1) wtot[wave] = inc;
  __syncthreads();
  const int wt = lane < kSelWaves ? wtot[lane] : 0, wi = wave_incl_scan(wt, lane);
  int at = __builtin_amdgcn_readlane(wi - wt, wave) + inc - cnt;
  int32_t* kept = a.kept_idx + (size_t)b * (K_r + K_d);
  while (word) {
    if (at < K_r + K_d) kept[at] = tid * 32 + __builtin_ctz(word);  // K_r + K_d set; the bound guards memory
    ++at;
    word &= word - 1;
  }
}

// ---------------------------------------------------------------- launchers
size_t PickPlan::gram_floats(int N) const {
  return std::max((size_t)N * ldg, (size_t)C * ldc);
}

// Time of a Gram launch in microseconds per 128-byte slab of the feature
// dimension, as measured on this GPU: 128-row tiles take 0.9 (fp32 1.8) with at
// most one workgroup on each of the 256 CUs and 1.45 (3.5) with two, 256-row
// tiles (bf16) 1.72 with one.  A workgroup's tile takes that long however few
// there are, which is what decides at small sizes.
static double gram_us128(long wgs, int dtype) {
  const double one = dtype == 1 ? 0.9 : 1.8, two = dtype == 1 ? 1.45 : 3.5;
  return wgs <= 256 ? one : (wgs <= 512 ? two : two * (wgs / 512.0 + 0.5));
}
static double gram_us256(long wgs) { return 1.72 * ((wgs + 255) / 256); }

// Pool rounds or the full Gram matrix at once, whichever is estimated to take
// less.  The pool has room for 9/4 of the picks, and grows from there while its
// Gram matrix takes no longer: to one workgroup per CU, or to two where pivots
// are few (below a fifth of the tokens): a pick then leaves many more
// candidates behind, and the neediest sample of a batch decides.  Pool tokens that the K_d picks reach down
// to, over K_d, on features of regions of 24 tokens: 1.2 with pivots 3/8 of
// the tokens, 1.5 at 1/4, 2.0 at 3/16, 2.5-3.2 at 1/6, 8-11 at 1/12.
#ifndef TREVS_PICK_ROUNDS
#define TREVS_PICK_ROUNDS -1
#endif
PickPlan pick_plan(int B, int N, int K_r, int K_d, int dtype, int row_bytes) {
  PickPlan p{};
  auto up = [](long x, long m) { return (x + m - 1) / m; };
  auto tri = [](long n) { return n * (n + 1) / 2; };
  p.ldg = (int)up(N, 4) * 4;
  p.n_psplit = std::min(std::max(K_r / 256, 1), 8);  // about 256 pivots each
  const int R = N - K_r;
  const bool big = gram256_ok(dtype, N, row_bytes);
  const double slabs = up(row_bytes, 128);
  const double full = slabs * (big ? gram_us256(B * tri(up(N, 256))) : gram_us128(B * tri(up(N, 128)), dtype)) +
                      (double)B * N * N * 4 / 4e6 + 15;  // 4 TB/s for the stores, the initial distances
  long ct = up(9L * K_d / 4, kRoundTile);
  const long room = 5L * K_r > N ? 256 : 512;
  while (B * tri(ct + 1) <= room) ++ct;
  p.C = (int)std::min({(long)R, ct * kRoundTile, (long)kMaxPool});
  p.ldc = (int)up(p.C, 4) * 4;
  const double r128 = gram_us128(B * up(K_r, 128) * up(R, 128), dtype);
  const double r256 = gram_us256(B * up(K_r, 256) * up(R, 256));
  p.row_tile = big && r256 < r128 ? 256 : 128;
  p.n_mx = (int)std::max(up(K_r, p.row_tile), up(K_d, kRoundTile));
  const double pool = slabs * ((p.row_tile == 256 ? r256 : r128) + gram_us128(B * tri(up(p.C, 128)), dtype)) + 30;
  // a round that finds nothing left to do takes about 9 us
  p.rounds = pool < full && 2 * K_d <= kMaxPool ? (full > 1500 ? 3 : 2) : 0;
  if (TREVS_PICK_ROUNDS >= 0) p.rounds = TREVS_PICK_ROUNDS;
  if (p.C >= R) p.rounds = std::min(p.rounds, 1);
  return p;
}

hipError_t launch_picks(const PickArgs& a, const void* Z, int row_bytes, int dtype, hipStream_t s) {
  const PickPlan& p = a.p;
  GramArgs g{};
  g.Z = Z;
  g.B = a.B;
  g.N = a.N;
  g.row_bytes = row_bytes;
  g.G = a.G;
  g.K_d = a.K_d;
  g.inv_norm = a.inv_norm;
  g.mx = a.mx;
  hipError_t err;
  for (int round = 0; round < p.rounds; ++round) {
    g.ctrl = a.ctrl;
    g.rows = round ? a.picks : a.pivots;
    g.n_rows = round ? a.K_d : a.K_r;
    g.by_round = round > 0;
    g.cols = a.rest;
    g.n_cols = a.R;
    const int tile = round ? kRoundTile : p.row_tile;
    if ((err = launch_gram_max(g, tile, dtype, s)) != hipSuccess) return err;
#define CALL(E_) \
  case E_: hipLaunchKernelGGL(pool_select_kernel<E_>, dim3(a.B), dim3(kSelThreads), 0, s, a, round, tile); break
    switch (select_e(a.R)) {
      CALL(1); CALL(2); CALL(4); CALL(8); CALL(16); CALL(32);
      default: return hipErrorInvalidValue;
    }
#undef CALL
    g.rows = a.cand;
    g.n_rows = p.C;
    g.by_round = false;
    g.ldg = p.ldc;
    if ((err = launch_gram_pool(g, dtype, s)) != hipSuccess) return err;
#define CALL(E_) \
  case E_: hipLaunchKernelGGL((pick_kernel<E_, false>), dim3(a.B), dim3(kSelThreads), 0, s, a); break
    switch (select_e(p.C)) {
      CALL(1); CALL(2); CALL(4);
      default: return hipErrorInvalidValue;
    }
#undef CALL
  }
  if (p.rounds > 0 && p.C >= a.R) return hipGetLastError();  // the pool held every token
  g.ldg = p.ldg;
  if ((err = launch_gram_full(g, dtype, s)) != hipSuccess) return err;
  if (p.rounds == 0)
    hipLaunchKernelGGL(fps_init_kernel, dim3((a.N + kFpsInitThreads - 1) / kFpsInitThreads, a.B, p.n_psplit),
                       dim3(kFpsInitThreads), 0, s, a);
#define CALL(E_) \
  case E_: hipLaunchKernelGGL((pick_kernel<E_, true>), dim3(a.B), dim3(kSelThreads), 0, s, a); break
  switch (select_e(a.N)) {
    CALL(1); CALL(2); CALL(4); CALL(8); CALL(16); CALL(32);
    default: return hipErrorInvalidValue;
  }
#undef CALL
  return hipGetLastError();
}

}  // namespace trevs
