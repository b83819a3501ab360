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
// Where the rounds do not suffice (tokens in many large clusters, slow changes
// over the image), the rest of the picks is made over the Gram matrix of all tokens
// but the pivots, and where the problem is so small that a round saves nothing,
// all picks are made over the Gram matrix of all tokens.
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
// Pool of a round: one workgroup per sample brings what is known of the
// sample's other tokens (rest) up to date with the maxima that the list
// products left (round 0: over the pivots; later: over the last round's
// picks, as minus the least distance), and keeps the C farthest, in index
// order.  The distances of round 0 are formed with the norms of the relevance
// pass, which every token has, later ones with those of the Gram diagonal; the
// C-th largest is the bound (see norm_gap).
// ---------------------------------------------------------------------------
template <int E>
__global__ __launch_bounds__(kSelThreads) void pool_select_kernel(PickArgs a, int round) {
  __shared__ SelectShared sh;
  const int b = blockIdx.x, tid = threadIdx.x, R = a.R, C = a.p.C;
  if (picks_done(a, b)) return;
  int32_t* ctrl = a.ctrl + b * kPickCtrl;
  const int32_t* rest = a.rest + (size_t)b * R;
  float* near_piv = a.near_piv + (size_t)b * a.N;
  float* near_pick = a.near_pick + (size_t)b * a.N;
  uint32_t* mx = a.mx + (size_t)b * R;
  uint32_t key[E];
  // groups of 16 tokens a thread (32 at once spilled 252 registers)
  constexpr int G = E < 16 ? E : 16;
#pragma unroll
  for (int e0 = 0; e0 < E; e0 += G) {
    float d[G], v[G];
    int tok[G];
    const int first = e0 * kSelThreads + tid;
#pragma unroll
    for (int e = 0; e < G; ++e) {
      const int i = min(first + e * kSelThreads, R - 1);
      d[e] = key2f(mx[i]);
      tok[e] = rest[i];
    }
#pragma unroll
    for (int e = 0; e < G; ++e)  // the next round's maxima start over
      if (first + e * kSelThreads < R) mx[first + e * kSelThreads] = 0u;
    if (round == 0) {
#pragma unroll
      for (int e = 0; e < G; ++e)
        if (first + e * kSelThreads < R) {
          near_piv[tok[e]] = d[e];
          near_pick[tok[e]] = INFINITY;
        }
#pragma unroll
      for (int e = 0; e < G; ++e) v[e] = a.inv_norm[(size_t)b * a.N + tok[e]];
#pragma unroll
      for (int e = 0; e < G; ++e) d[e] = 1.f - d[e] * v[e];
    } else {
#pragma unroll
      for (int e = 0; e < G; ++e) v[e] = near_pick[tok[e]];
#pragma unroll
      for (int e = 0; e < G; ++e) {
        d[e] = -d[e] < v[e] ? -d[e] : v[e];
        if (first + e * kSelThreads < R) near_pick[tok[e]] = d[e];
      }
#pragma unroll
      for (int e = 0; e < G; ++e) v[e] = 1.f - near_piv[tok[e]] * a.inv_norm[(size_t)b * a.N + tok[e]];
#pragma unroll
      for (int e = 0; e < G; ++e) d[e] = d[e] < v[e] ? d[e] : v[e];
    }
#pragma unroll
    for (int e = 0; e < G; ++e) key[e0 + e] = f2key(d[e]);
    if (E > G) __builtin_amdgcn_sched_barrier(0);
  }
  int32_t* cand = a.cand + (size_t)b * C;
  float* cand_cos = a.cand_cos + (size_t)b * C;
  float* cand_piv = a.cand_piv + (size_t)b * C;
  float* cand_pick = a.cand_pick + (size_t)b * C;
  auto put = [&](int at, int e) {
    const int tok = rest[e * kSelThreads + tid];
    const float piv = near_piv[tok], pick = near_pick[tok];
    cand[at] = tok;
    cand_cos[at] = fmaxf(piv * a.inv_norm[(size_t)b * a.N + tok], 1.f - pick);
    cand_piv[at] = piv;
    cand_pick[at] = pick;
  };
  float bound = -INFINITY;
  if (C >= R) {
#pragma unroll
    for (int e = 0; e < E; ++e)
      if (e * kSelThreads + tid < R) put(e * kSelThreads + tid, e);
  } else {
    uint32_t thr;
    block_topk_each<E>(
        key, R, C, [&](int e, bool, bool keep, int before) { if (keep && before < C) put(before, e); }, sh, false, 0u,
        0u, &thr);
    bound = key2f(thr);
  }
  if (tid == 0) ctrl[kCtrlBound] = __float_as_int(bound);
}

// ---------------------------------------------------------------------------
// The picks.  A step that reduces over the workgroup and then waits for a row
// of G takes about 2 us, so one workgroup per sample makes them in batches.
// The entries with the largest distances (at most kBatch: those in the first
// bins of a scale that starts at the largest) go with their mutual distances
// to LDS; one wave picks among them, without a barrier, for as long as the
// best of them is above every other entry; then all entries take the rows of
// the picks at once.  Where more than kBatch entries share the first bin the
// scale is refined, and where that many tie exactly the batch takes them by
// index.  Distances are compared as order-preserving integers (f2key), whose
// maximum takes one instruction per step of a wave reduction; 0, below every
// key, marks selected entries.
// ---------------------------------------------------------------------------
constexpr int kMaxPool = 4096;  // entries of a pool (four per thread)
constexpr int kBatch = 64;
constexpr int kBins = 512;      // of the scale; at most 64 of TREVS_MAX_FPS_N indices each
constexpr int kZooms = 6;       // refinements of the scale, by 16 each
static_assert(TREVS_MAX_FPS_N <= kBins * kBatch, "a bin of indices fits a batch");
static_assert(TREVS_MAX_FPS_N / 32 <= kSelThreads, "a word of the kept list per thread");
static_assert(kBins == 8 * kWave, "eight bins a lane");

struct PickShared {
  uint32_t red[kSelWaves], red_out[kSelWaves];
  uint32_t hist[kBins];
  uint32_t bkey[kBatch];           // the batch: keys, inverse norms, entries
  float biz[kBatch];
  int bc[kBatch];
  uint32_t sub[kBatch][kBatch + 1];  // their mutual distances, as keys
  int pc[kBatch];                  // the picks: entries, inverse norms, places in the batch
  float piz[kBatch];
  int pslot[kBatch];
  int n_batch, n_new;
  uint32_t bits[kSelThreads];      // a bit per token
  int wtot[kSelWaves];
};

// A distance as a key; not-a-number, which brings nothing nearer, as the largest.
__device__ __forceinline__ uint32_t dist_key(float d) { return d == d ? f2key(d) : 0xffffffffu; }

__device__ __forceinline__ uint32_t block_max_u32(uint32_t v, uint32_t* red) {
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  v = wave_max_u32(v);
  if (lane == 0) red[wave] = v;
  __syncthreads();
  return wave_max_u32(lane < kSelWaves ? red[lane] : 0u);
}

// Bit i of sh.bits: token i is a pivot, or one of the first np picks.
__device__ __forceinline__ void mark_selected(const PickArgs& a, int b, int np, PickShared& sh) {
  const int tid = threadIdx.x, N = a.N;
  if (tid < (N + 31) / 32) sh.bits[tid] = 0u;
  __syncthreads();
  for (int p = tid; p < a.K_r; p += kSelThreads) {
    const int j = min(max(a.pivots[(size_t)b * a.K_r + p], 0), N - 1);
    atomicOr(&sh.bits[j >> 5], 1u << (j & 31));
  }
  for (int p = tid; p < np; p += kSelThreads) {
    const int j = min(max(a.picks[(size_t)b * a.K_d + p], 0), N - 1);
    atomicOr(&sh.bits[j >> 5], 1u << (j & 31));
  }
  __syncthreads();
}

// f(rank, token) for every set bit of the workgroup's words (32 tokens a
// thread), in token order.
template <class F>
__device__ __forceinline__ void each_token(uint32_t word, PickShared& sh, F f) {
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const int cnt = __popc(word), inc = wave_incl_scan(cnt, lane);
  if (lane == kWave - 1) sh.wtot[wave] = inc;
  __syncthreads();
  const int wt = lane < kSelWaves ? sh.wtot[lane] : 0, wi = wave_incl_scan(wt, lane);
  int at = __builtin_amdgcn_readlane(wi - wt, wave) + inc - cnt;
  while (word) {
    f(at, tid * 32 + __builtin_ctz(word));
    ++at;
    word &= word - 1;
  }
}

// Picks t.. of a sample whose other tokens have no distance (a row whose
// squares overflow is infinitely long, and its products times 1/infinity are
// not numbers): the unselected tokens in index order.
__device__ __forceinline__ void fill_picks(const PickArgs& a, int b, int t, PickShared& sh) {
  const int first = threadIdx.x * 32, N = a.N;
  mark_selected(a, b, t, sh);
  const uint32_t valid = first + 32 <= N ? ~0u : (first < N ? (1u << (N - first)) - 1u : 0u);
  each_token(valid ? ~sh.bits[threadIdx.x] & valid : 0u, sh, [&](int at, int tok) {
    if (t + at < a.K_d) {
      a.picks[(size_t)b * a.K_d + t + at] = tok;
      if (a.div_idx) a.div_idx[(size_t)b * a.K_d + t + at] = tok;
    }
  });
  __syncthreads();
}

// The kept list: pivots and all picks in ascending order.
__device__ __forceinline__ void write_kept(const PickArgs& a, int b, PickShared& sh) {
  const int K = a.K_r + a.K_d;
  mark_selected(a, b, a.K_d, sh);
  int32_t* kept = a.kept_idx + (size_t)b * K;
  each_token(threadIdx.x < (a.N + 31) / 32 ? sh.bits[threadIdx.x] : 0u, sh, [&](int at, int tok) {
    if (at < K) kept[at] = tok;  // K set; the bound guards memory
  });
}

// The scale of a batch.  bin(key, entry): steps below the largest key, kBins
// past the scale; with ties, the index bin of an entry at the largest key.
struct BatchScale {
  uint32_t top;
  float ftop, scale;
  bool ties;
  int ishift, cut;
  __device__ __forceinline__ int bin(uint32_t key, int c) const {
    if (ties) return key == top ? c >> ishift : kBins;
    return key >= top ? 0 : (int)fminf((ftop - key2f(key)) * scale, (float)kBins);
  }
};

// The cut: the most bins of the scale that hold at most kBatch entries that may
// be picked, ok(key, entry).  sh.hist holds zeros.  range: width of the scale,
// refined here.  each(f) calls f(key, entry) for every entry of the thread.
template <class Ok, class Each>
__device__ __forceinline__ void batch_cut(BatchScale& s, float& range, Ok ok, Each each, PickShared& sh) {
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  for (int zoom = 0;; ++zoom) {
    s.ties = zoom >= kZooms || !(range > 0.f);
    s.scale = (float)kBins / range;
    each([&](uint32_t key, int c) {
      if (ok(key, c)) {
        const int bin = s.bin(key, c);
        if (bin < kBins) atomicAdd(&sh.hist[bin], 1u);
      }
    });
    __syncthreads();
    int c[8], sum = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) sum += c[j] = (int)sh.hist[8 * lane + j];
    int before = wave_incl_scan(sum, lane) - sum, mine = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      before += c[j];
      mine += before <= kBatch ? 1 : 0;  // bins 0..8*lane+j hold at most kBatch entries
    }
    s.cut = wave_reduce_bits(mine, 0, [](int x, int y) { return x + y; });
    if (s.cut > 0 || s.ties) return;  // uniform (a bin of indices holds at most kBatch)
    range *= 1.f / 16.f;
    __syncthreads();  // hist has been read
    if (tid < kBins) sh.hist[tid] = 0u;
    __syncthreads();
  }
}

// The picks among the m entries of a batch, by the calling wave (all lanes).
// limit: most picks; out: the largest key that is not in the batch.  The picks' places in
// the batch go to lanes 0, 1, ... of `won`; returns their number.
__device__ __forceinline__ int batch_picks(int m, int limit, uint32_t out, const BatchScale& s, const PickShared& sh,
                                           int& won) {
  const int lane = threadIdx.x & (kWave - 1);
  uint32_t d = lane < m ? sh.bkey[lane] : 0u;
  const uint32_t cl = (uint32_t)sh.bc[min(lane, m - 1)];
  const int n_max = min(m, limit);
  won = 0;
  int k = 0;
  for (; k < n_max; ++k) {
    const uint32_t vm = wave_max_u32(d);
    // above every other entry, or the top itself: the first pick, and ties by index
    if (vm <= out && !(vm == s.top && (s.ties || k == 0))) break;  // uniform
    unsigned long long bal = __ballot(d == vm);
    if (bal & (bal - 1)) {  // uniform: a tie goes to the lower index
      const uint32_t c0 = wave_min_u32(d == vm ? cl : 0xffffffffu);
      bal = __ballot(d == vm && cl == c0);
    }
    const int w = (int)__builtin_ctzll(bal);
    d = min(d, sh.sub[w][lane]);
    d = lane == w ? 0u : d;
    won = lane == k ? w : won;
  }
  return k;
}

// Vectors of CH floats.
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

// ---------------------------------------------------------------------------
// Picks of a round, over the pool.  Distances are those of the Gram matrix
// (its diagonal gives the norms).  Few pairs matter: entry i is brought nearer
// by pick j only if their distance is below that of i, which the mask of the
// pool's Gram matrix marks.  So the batch's mask rows go to LDS, mutual
// distances are read from G for marked pairs, and a pick updates only the
// marked entries (reading whole rows of G, 9 KB for each pick at 37 GB/s a
// CU, took 12 us of a batch's 32).
// A pick must also be farther than every token outside the pool: its distance
// is above the round's bound and what the norms may differ by.  Where they
// cannot differ (later rounds, or no cosine at all: zero rows, orthogonal ones),
// tokens at the bound itself can be picked too, as far as the pool holds them:
// those outside have higher indices.  The round ends where that fails; at K_d
// picks the kept list is written.
// ---------------------------------------------------------------------------
constexpr int kHits = 4096;  // marked (pick, entry) pairs taken at once
constexpr int kMaxPoolPicks = kMaxPool / 2;

__global__ __launch_bounds__(kSelThreads) void pool_pick_kernel(PickArgs a, float gap) {
  __shared__ PickShared sh;
  __shared__ uint32_t key[kMaxPool];
  __shared__ float iz[kMaxPool];
  __shared__ u32x4 mrow[kBatch][kMaxPool / 128];
  __shared__ uint32_t hits[kHits];
  __shared__ int n_hits;
  __shared__ uint16_t order[kMaxPoolPicks];  // entries picked in this round
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const int C = a.p.C, ldc = a.p.ldc, mw4 = a.p.mask_words / 4, K_d = a.K_d, N = a.N;
  if (picks_done(a, b)) return;
  int32_t* ctrl = a.ctrl + b * kPickCtrl;
  const int t0 = ctrl[kCtrlPicks];
  int t = t0;
  const float bound = __int_as_float(ctrl[kCtrlBound]);
  // what the norms may move a distance by, and its rounding with them (an ulp on
  // either side of 1)
  const float slack = gap * fabsf(1.f - bound);
  const float floor = bound > -INFINITY ? bound + (slack > 0.f ? slack + 2.4e-7f : 0.f) : -INFINITY;
  const uint32_t floor_key = f2key(floor);
  const int32_t* cand = a.cand + (size_t)b * C;
  const float* G = a.G + (size_t)b * C * ldc;
  const u32x4* mask = reinterpret_cast<const u32x4*>(a.mask) + (size_t)b * C * mw4;
  int32_t* picks = a.picks + (size_t)b * K_d;
  // a round over few candidates is short of NaN and selected entries alike:
  // keys of NaN distances (above infinity's) never win
  const uint32_t inf_key = f2key(INFINITY);
  const bool tied = bound > -INFINITY && floor == bound;
  int last = 0;  // entries below it may be picked at the floor
  for (int c = tid; c < C; c += kSelThreads) {
    const float z = 1.f / fmaxf(sqrtf(fmaxf(G[(size_t)c * ldc + c], 0.f)), 1e-12f);
    const float d = 1.f - a.cand_piv[(size_t)b * C + c] * z, dp = a.cand_pick[(size_t)b * C + c];
    const uint32_t k = dp == -INFINITY ? 0u : f2key(dp < d ? dp : d);
    iz[c] = z;
    key[c] = k > inf_key ? 0u : k;
    if (tied && k == floor_key) last = c + 1;
  }
  const float range0 = bound > -INFINITY ? -1.f : 2.f;  // down to the bound (-1), or anywhere (distances: 0..2)
  float range = range0;
  BatchScale s;
  s.ishift = 0;
  while ((C - 1) >> s.ishift >= kBins) ++s.ishift;
  auto each = [&](auto f) {
    for (int c = tid; c < C; c += kSelThreads) f(key[c], c);
  };
  __syncthreads();
  if (tied) last = (int)block_max_u32((uint32_t)last, sh.red_out);  // uniform
  auto ok = [&](uint32_t k, int c) { return k > (c < last ? floor_key - 1u : floor_key); };
  while (t < K_d) {
    uint32_t v = 0u;
    each([&](uint32_t k, int c) { v = ok(k, c) ? max(v, k) : v; });
    if (tid == 0) sh.n_batch = n_hits = 0;
    if (tid < kBins) sh.hist[tid] = 0u;
    s.top = block_max_u32(v, sh.red);
    if (s.top == 0u) break;  // uniform
    s.ftop = key2f(s.top);
    if (range < 0.f || s.top == floor_key) range = s.ftop - bound;
    batch_cut(s, range, ok, each, sh);
    // ---- the batch, and the largest key outside it
    uint32_t out = floor_key;
    each([&](uint32_t k, int c) {
      if (ok(k, c) && s.bin(k, c) < s.cut) {
        const int at = atomicAdd(&sh.n_batch, 1);
        if (at < kBatch) {
          sh.bkey[at] = k;
          sh.biz[at] = iz[c];
          sh.bc[at] = c;
        }
      } else {
        out = max(out, k);
      }
    });
    out = block_max_u32(out, sh.red_out);
    const int m = min(sh.n_batch, kBatch);  // at least the top
    // ---- its mask rows, then its mutual distances where marked
    for (int p = tid; p < m * mw4; p += kSelThreads) {
      const int x = p / mw4, wd = p - x * mw4;
      mrow[x][wd] = mask[(size_t)sh.bc[x] * mw4 + wd];
    }
    __syncthreads();
    constexpr int SUBS = kBatch * kBatch / kSelThreads;
    float g[SUBS];
    bool on[SUBS];
#pragma unroll
    for (int k = 0; k < SUBS; ++k) {
      const int x = min(wave + k * kSelWaves, m - 1), y = min(lane, m - 1), cy = sh.bc[y];
      on[k] = (reinterpret_cast<const uint32_t*>(mrow[x])[cy >> 5] >> (cy & 31)) & 1u;
      g[k] = G[on[k] ? (size_t)sh.bc[x] * ldc + cy : 0];
    }
#pragma unroll
    for (int k = 0; k < SUBS; ++k) {
      const int x = min(wave + k * kSelWaves, m - 1), y = min(lane, m - 1);
      sh.sub[wave + k * kSelWaves][lane] = on[k] ? dist_key(1.f - g[k] * sh.biz[y] * sh.biz[x]) : 0xffffffffu;
    }
    __syncthreads();
    if (wave == 0) {
      int won;
      const int k = batch_picks(m, K_d - t, out, s, sh, won);
      if (lane == 0) sh.n_new = k;
      if (lane < k) {
        const int c = sh.bc[won];
        sh.pc[lane] = c;
        sh.piz[lane] = sh.biz[won];
        sh.pslot[lane] = won;
        key[c] = 0u;
        order[t - t0 + lane] = (uint16_t)c;
      }
    }
    __syncthreads();
    const int np = sh.n_new;
    if (np == 0) break;  // uniform
    // ---- marked entries that can still be picked in this round
    // (marks cluster, so a wave takes a row's nonzero words two at a time, a
    // lane to a bit)
    for (int q = wave; q < np; q += kSelWaves) {
      if (*(volatile int*)&n_hits > kHits) break;  // too many for the list
      const uint32_t* row = reinterpret_cast<const uint32_t*>(mrow[sh.pslot[q]]);
      for (int w0 = 0; w0 < 4 * mw4; w0 += kWave) {
        unsigned long long words = __ballot(w0 + lane < 4 * mw4 && row[min(w0 + lane, 4 * mw4 - 1)] != 0u);
        while (words) {  // uniform
          const int lo = (int)__builtin_ctzll(words);
          words &= words - 1;
          int hi = -1;
          if (words) {
            hi = (int)__builtin_ctzll(words);
            words &= words - 1;
          }
          const int wl = lane < 32 ? lo : hi, c = (w0 + wl) * 32 + (lane & 31);
          const bool hit = wl >= 0 && ((row[max(w0 + wl, 0)] >> (lane & 31)) & 1u) && key[max(c, 0)] >= floor_key;
          const unsigned long long bal = __ballot(hit);
          if (bal) {
            int base = 0;
            if (lane == 0) base = atomicAdd(&n_hits, (int)__popcll(bal));
            base = __builtin_amdgcn_readfirstlane(base);
            const int at = base + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32),
                                                                 __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
            if (hit && at < kHits) hits[at] = (uint32_t)q << 16 | (uint32_t)c;
          }
        }
      }
    }
    __syncthreads();
    auto take = [&](int q, int c) {
      const float gq = G[(size_t)sh.pc[q] * ldc + c];
      atomicMin(&key[c], dist_key(1.f - gq * iz[c] * sh.piz[q]));
    };
    if (n_hits <= kHits) {
      for (int h = tid; h < n_hits; h += kSelThreads) take(hits[h] >> 16, hits[h] & 0xffffu);
    } else {  // most pairs marked: whole rows, eight vectors of four entries in flight
      constexpr int U = 8;
      const int nv = (C + 3) / 4, total = np * nv;
      for (int i0 = tid; i0 < total; i0 += U * kSelThreads) {
        float4 g[U];
        int at[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int i = min(i0 + u * kSelThreads, total - 1), q = i / nv;
          at[u] = q << 16 | (i - q * nv) * 4;
          g[u] = *reinterpret_cast<const float4*>(G + (size_t)sh.pc[q] * ldc + (at[u] & 0xffff));
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int c0 = at[u] & 0xffff;
          const float izq = sh.piz[at[u] >> 16];
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const uint32_t k = dist_key(1.f - Chunk<4>::at(g[u], j) * iz[c0 + j] * izq);
            if (c0 + j < C && k < key[c0 + j]) atomicMin(&key[c0 + j], k);  // (a key read late is too large)
          }
        }
      }
    }
    t += np;
    // a batch that is far from full asks for a wider scale
    if (m < kBatch / 2) range = m < kBatch / 8 ? range0 : 2.f * range;
    __syncthreads();  // the keys, and n_hits
  }
  __syncthreads();  // order
  for (int p = t0 + tid; p < t; p += kSelThreads) {
    const int c = order[p - t0], tok = cand[c];
    picks[p] = tok;
    if (a.div_idx) a.div_idx[(size_t)b * K_d + p] = tok;
    a.near_pick[(size_t)b * N + tok] = -INFINITY;  // for the next round
    a.inv_norm[(size_t)b * N + tok] = iz[c];
  }
  if (tid == 0) {
    ctrl[kCtrlPicks] = t;
    ctrl[kCtrlRound] = t0;
  }
  if (t < K_d && C < a.R) return;  // uniform
  __syncthreads();                 // the picks written above
  if (t < K_d) fill_picks(a, b, t, sh);  // the pool held every token: no round follows
  write_kept(a, b, sh);
}

// ---------------------------------------------------------------------------
// Picks over the Gram matrix of all tokens, from the pivots' partial maxima, or
// (REST) over that of the tokens that are no pivots (a.rest), from where the rounds
// stopped.  The keys stay in registers: element e of thread t is row
// (e / CH) * CH * 1024 + t * CH + e % CH of the matrix, so that its rows load as
// vectors of CH values, up to U rows at a time.
// ---------------------------------------------------------------------------
template <int E, bool REST>
__global__ __launch_bounds__(kSelThreads) void full_pick_kernel(PickArgs a) {
  constexpr int CH = E < 4 ? E : 4;        // entries per vector
  constexpr int NR = E / CH;               // vectors per thread and row
  constexpr int U = E <= 2 ? 16 : 32 / E;  // rows in flight
  typedef typename Chunk<CH>::T Vec;
  __shared__ PickShared sh;
  // inverse norms: in registers, or, with 32 entries a thread (where keys, norms
  // and a row spilled 70 to 110 registers), in LDS
  constexpr bool IN_LDS = E > 16;
  __shared__ __attribute__((aligned(16))) float iz_lds[IN_LDS ? E * kSelThreads : 1];
  float iz_reg[IN_LDS ? 1 : E];
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const int N = REST ? a.R : a.N, ldg = a.p.ldg, K_d = a.K_d;
  if (picks_done(a, b)) return;
  const int32_t* ctrl = a.ctrl + b * kPickCtrl;
  const int t0 = REST ? ctrl[kCtrlPicks] : 0;
  int t = t0;
  const float* G = a.G + (size_t)b * N * ldg;
  const int32_t* rest = a.rest + (size_t)b * a.R;
  auto token = [&](int c) { return REST ? rest[c] : c; };  // of row c < N
  const float* inv_norm = a.inv_norm + (size_t)b * a.N;
  int32_t* picks = a.picks + (size_t)b * K_d;
  auto entry = [&](int e) { return (e / CH) * CH * kSelThreads + tid * CH + e % CH; };
  // selected tokens and those past N hold key 0: they never win, and the row
  // updates (a minimum) keep them there; so do tokens whose distance is not a number
  auto inv = [&](int e) { return IN_LDS ? iz_lds[entry(e)] : iz_reg[IN_LDS ? 0 : e]; };
  uint32_t key[E];
  const uint32_t inf_key = f2key(INFINITY);
  if (!REST) mark_selected(a, b, 0, sh);
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int c = entry(e), cc = min(c, N - 1), tok = token(cc);
    const float iz = inv_norm[tok];
    if (IN_LDS)
      iz_lds[c] = iz;
    else
      iz_reg[IN_LDS ? 0 : e] = iz;
    float mx, least = INFINITY;
    if (REST) {
      mx = a.near_piv[(size_t)b * a.N + tok];
      least = a.near_pick[(size_t)b * a.N + tok];
    } else {
      mx = a.part[(size_t)b * N + cc];
      for (int sp = 1; sp < a.p.n_psplit; ++sp) mx = fmaxf(mx, a.part[((size_t)sp * a.B + b) * N + cc]);
    }
    const float d = 1.f - mx * iz;
    const bool sel = c >= N || (REST ? least == -INFINITY : (sh.bits[cc >> 5] >> (cc & 31)) & 1u);
    const uint32_t k = f2key(least < d ? least : d);
    key[e] = sel || k > inf_key ? 0u : k;
  }
  // the rows of picks p[0, np) (sh.pc, sh.piz); every load of a group is
  // issued before the first is used
  auto take_rows = [&](int np) {
    for (int q0 = 0; q0 < np; q0 += U) {
      Vec g[U][NR];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const float* row = G + (size_t)__builtin_amdgcn_readfirstlane(sh.pc[min(q0 + u, np - 1)]) * ldg;
#pragma unroll
        for (int r = 0; r < NR; ++r) {
          const int c = entry(r * CH);
          g[u][r] = *reinterpret_cast<const Vec*>(row + (c < ldg ? c : 0));
        }
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const float izw = sh.piz[min(q0 + u, np - 1)];
#pragma unroll
        for (int e = 0; e < E; ++e)
          key[e] = min(key[e], dist_key(1.f - Chunk<CH>::at(g[u][e / CH], e % CH) * inv(e) * izw));
      }
    }
  };
  if (REST) {  // the last round's picks are not yet in the distances
    for (int p0 = ctrl[kCtrlRound]; p0 < t0; p0 += kBatch) {
      const int np = min(kBatch, t0 - p0);
      __syncthreads();
      if (tid < np) {
        const int tok = min(max(picks[p0 + tid], 0), a.N - 1);
        int lo = 0, hi = N - 1;  // the pick's row
        while (lo < hi) {
          const int mid = (lo + hi) >> 1;
          if (rest[mid] < tok)
            lo = mid + 1;
          else
            hi = mid;
        }
        sh.pc[tid] = lo;
        sh.piz[tid] = inv_norm[tok];
      }
      __syncthreads();
      take_rows(np);
    }
  }
  float range = 2.f;
  BatchScale s;
  s.ishift = 0;
  while ((N - 1) >> s.ishift >= kBins) ++s.ishift;
  auto each = [&](auto f) {
#pragma unroll
    for (int e = 0; e < E; ++e) f(key[e], entry(e));
  };
  while (t < K_d) {
    uint32_t v = 0u;
    each([&](uint32_t k, int) { v = max(v, k); });
    if (tid == 0) sh.n_batch = 0;
    if (tid < kBins) sh.hist[tid] = 0u;
    s.top = block_max_u32(v, sh.red);
    if (s.top == 0u) break;  // uniform
    s.ftop = key2f(s.top);
    batch_cut(s, range, [](uint32_t k, int) { return k > 0u; }, each, sh);
    uint32_t out = 0u;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int c = entry(e);
      if (key[e] > 0u && s.bin(key[e], c) < s.cut) {
        const int at = atomicAdd(&sh.n_batch, 1);
        if (at < kBatch) {
          sh.bkey[at] = key[e];
          sh.biz[at] = inv(e);
          sh.bc[at] = c;
        }
      } else {
        out = max(out, key[e]);
      }
    }
    out = block_max_u32(out, sh.red_out);
    const int m = min(sh.n_batch, kBatch);  // at least the top
    constexpr int SUBS = kBatch * kBatch / kSelThreads;
    float g[SUBS];
#pragma unroll
    for (int k = 0; k < SUBS; ++k) {
      const int x = min(wave + k * kSelWaves, m - 1), y = min(lane, m - 1);
      g[k] = G[(size_t)sh.bc[x] * ldg + sh.bc[y]];
    }
#pragma unroll
    for (int k = 0; k < SUBS; ++k) {
      const int x = min(wave + k * kSelWaves, m - 1), y = min(lane, m - 1);
      sh.sub[wave + k * kSelWaves][lane] = dist_key(1.f - g[k] * sh.biz[y] * sh.biz[x]);
    }
    __syncthreads();
    if (wave == 0) {
      int won;
      const int k = batch_picks(m, K_d - t, out, s, sh, won);
      if (lane == 0) sh.n_new = k;
      if (lane < k) {
        const int c = sh.bc[won];
        sh.pc[lane] = c;
        sh.piz[lane] = sh.biz[won];
        const int tok = token(c);
        picks[t + lane] = tok;
        if (a.div_idx) a.div_idx[(size_t)b * K_d + t + lane] = tok;
      }
    }
    __syncthreads();
    const int np = sh.n_new;
    if (np == 0) break;  // uniform
    take_rows(np);
    for (int q = 0; q < np; ++q) {
      const int c = sh.pc[q];
#pragma unroll
      for (int e = 0; e < E; ++e)
        if (c == entry(e)) key[e] = 0u;
    }
    t += np;
    if (m < kBatch / 2) range = m < kBatch / 8 ? 2.f : 2.f * range;
  }
  __syncthreads();  // the picks written above
  if (t < K_d) fill_picks(a, b, t, sh);
  write_kept(a, b, sh);
}

// ---------------------------------------------------------------- launchers
size_t PickPlan::gram_floats() const {
  return std::max((size_t)n_gram * ldg, rounds > 0 ? (size_t)C * ldc : 0);
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
static double gram_us256(long wgs, int cols = 256) { return (cols == 256 ? 1.72 : 1.5) * ((wgs + 255) / 256); }

// Pool rounds or the full Gram matrix at once, whichever is estimated to take
// less.  The pool has room for 9/4 of the picks, and grows from there while its
// Gram matrix takes no longer: to one workgroup per CU, or to two where pivots
// are few (below a fifth of the tokens; not for fp32, where two take twice as
// long): a pick then leaves many more
// candidates behind, and the neediest sample of a batch decides.  Pool tokens that the K_d picks reach down
// to, over K_d, on features of regions of 24 tokens: 1.2 with pivots 3/8 of
// the tokens, 1.5 at 1/4, 2.0 at 3/16, 2.5-3.2 at 1/6, 8-11 at 1/12.
//
// How many rounds suffice depends on the tokens: one on features of small
// regions or of no structure, 2 or 3 where few directions are far from the
// pivots (large regions, clusters, copies), up to 7 where features change
// slowly over the image; a round takes a launch each of four kernels even if it
// finds nothing to do.  What the rounds leave costs the Gram matrix of the
// other tokens on top, so:
//  - No round where one saves less than a quarter and its pool holds less than
//    two thirds of the tokens (64 x 576 tokens, 48 picks of 192: 345 -> 342 us with a
//    round that suffices, 382 -> 515 with one that does not; 37 x 795, 22 of 88,
//    pool 0.7: 234 -> 180 and 257 -> 338).
//  - A second, and a third where the matrix takes more than 1.5 ms, while the estimate with all of them in vain is within
//    1.4 times the full matrix.  16 x 2880 tokens, 160 of 640 (full
//    matrix 935-1008 us): one round 490, in vain 1135; three 505 and 1465.
//    4 x 16,384, 1024 of 4096 (6420-6590): three 1672, in vain 6275.  2 x 20,000, 500
//    of 2000 (2840-3210): three 515, in vain 3510.
PickPlan pick_plan(int B, int N, int K_r, int K_d, int dtype, int row_bytes) {
  PickPlan p{};
  auto up = [](long x, long m) { return (x + m - 1) / m; };
  auto tri = [](long n) { return n * (n + 1) / 2; };
  p.n_psplit = std::min(std::max(K_r / 256, 1), 8);  // about 256 pivots each
  const int R = N - K_r;
  const bool big = gram256_ok(dtype, N, row_bytes);
  const int d = row_bytes / (dtype == 1 ? 2 : 4);
  const double slabs = up(row_bytes, 128);
  // a square Gram matrix, its stores at 4 TB/s, the initial distances; a pick reads a row at 37 GB/s
  auto square = [&](long n) {
    return slabs * (big ? gram_us256(B * tri(up(n, 256))) : gram_us128(B * tri(up(n, 128)), dtype)) +
           B * 1e-6 * n * n + 15 + K_d * (0.25 + n * 4 / 37e3);
  };
  const double full = square(N);
  long ct = up(9L * K_d / 4, kRoundTile);
  const long room = 5L * K_r > N || dtype != 1 ? 256 : 512;
  while (B * tri(ct + 1) <= room) ++ct;
  p.C = (int)std::min({(long)R, ct * kRoundTile, (long)kMaxPool});
  p.ldc = (int)up(p.C, 4) * 4;
  const double r128 = gram_us128(B * up(K_r, 128) * up(R, 128), dtype);
  const double r256w = gram_us256(B * up(K_r, 256) * up(R, 256));
  const double r256n = gram_us256(B * up(K_r, 256) * up(R, 192), 192);
  const double r256 = std::min(r256w, r256n);
  p.mask_words = (int)up(p.C, 128) * 4;
  p.row_tile = big && r256 < r128 ? 256 : 128;
  p.col_tile = p.row_tile == 128 ? 128 : (r256n < r256w ? 192 : 256);
  // the pivots' norms, the pool selection, launches that find nothing left to do
  const double gram = slabs * gram_us128(B * tri(up(p.C, 128)), dtype);
  const double pool = slabs * (p.row_tile == 256 ? r256 : r128) + gram + (dtype == 1 ? 0.3 * slabs : 0) + 10 +
                      R / 700 + (p.C < R ? 10 : 0) + K_d * 0.35;
  p.rounds = pool < full && K_d <= kMaxPoolPicks && d <= kNormGapMaxD ? 1 : 0;
  if (p.C < R) {
    if (pool > 0.75 * full && 3 * p.C < 2 * R) p.rounds = 0;
    // a round that ends early makes few picks
    const double next = slabs * 1.25 * gram_us128(B * up(R, kRoundTile), dtype) + gram + 30 + R / 700;
    const int most = full > 1500 ? 3 : 2;
    while (p.rounds > 0 && p.rounds < most && pool + p.rounds * next + square(R) <= 1.4 * full) ++p.rounds;
  }
  p.n_gram = p.rounds > 0 ? R : N;
  p.ldg = (int)up(p.n_gram, 4) * 4;
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
    g.cols = a.rest;
    g.n_cols = a.R;
    g.near_pick = a.near_pick;
    if (round == 0 && dtype == 1 && (err = launch_gram_norms(g, s)) != hipSuccess) return err;
    err = round ? launch_gram_next(g, dtype, s) : launch_gram_max(g, p.row_tile, p.col_tile, dtype, s);
    if (err != hipSuccess) return err;
    const float gap = round ? 0.f : a.gap;
#define CALL(E_) \
  case E_: hipLaunchKernelGGL(pool_select_kernel<E_>, dim3(a.B), dim3(kSelThreads), 0, s, a, round); break
    switch (select_e(a.R)) {
      CALL(1); CALL(2); CALL(4); CALL(8); CALL(16); CALL(32);
      default: return hipErrorInvalidValue;
    }
#undef CALL
    g.rows = a.cand;
    g.n_rows = p.C;
    g.ldg = p.ldc;
    g.mask = a.mask;
    g.mask_words = p.mask_words;
    g.nearest = a.cand_cos;
    g.margin = kMaskMargin * gap + kCosRounding;
    if ((err = launch_gram_pool(g, dtype, s)) != hipSuccess) return err;
    hipLaunchKernelGGL(pool_pick_kernel, dim3(a.B), dim3(kSelThreads), 0, s, a, gap);
  }
  if (p.rounds > 0 && p.C >= a.R) return hipGetLastError();  // the pool held every token
  g.ldg = p.ldg;
  err = p.rounds > 0 ? launch_gram_rest(g, dtype, s) : launch_gram_full(g, dtype, s);
  if (err != hipSuccess) return err;
#define CALL(E_, REST_) \
  case E_: hipLaunchKernelGGL((full_pick_kernel<E_, REST_>), dim3(a.B), dim3(kSelThreads), 0, s, a); break
  if (p.rounds > 0) {
    switch (select_e(a.R)) {
      CALL(1, true); CALL(2, true); CALL(4, true); CALL(8, true); CALL(16, true); CALL(32, true);
      default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
  }
  hipLaunchKernelGGL(fps_init_kernel, dim3((a.N + kFpsInitThreads - 1) / kFpsInitThreads, a.B, p.n_psplit),
                     dim3(kFpsInitThreads), 0, s, a);
  switch (select_e(a.N)) {
    CALL(1, false); CALL(2, false); CALL(4, false); CALL(8, false); CALL(16, false); CALL(32, false);
    default: return hipErrorInvalidValue;
  }
#undef CALL
  return hipGetLastError();
}

}  // namespace trevs
