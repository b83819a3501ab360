// Diagnostics of the preliminary analysis (Sec. 3): the visual attention
// profile of every head and its text sensitivity between two questions
// (Eq. (1)), and the Spearman rank correlation of visual saliency and textual
// relevance within the top-K saliency set.
#include "common.hpp"
#include "kernels.hpp"
#include "select.hpp"

namespace trevs {

// ---------------------------------------------------------------------------
// Visual profile of one head: profile[i] = (1/T_b) sum_{q<T_b} A[h,q,i] with
// A the text->vision attention of the statistics pass (its row log-sum-exps
// come in through lse2).  A workgroup owns one (sample, query head) and one
// split of the visual keys; workgroups of one (sample, KV head) are numbered
// consecutively and mapped onto one XCD, so the keys the group's query heads
// share stay in that L2.  Wave w keeps the Q rows of text block w (of the
// current pass) resident as MFMA operand A; the 32-key tiles of the split
// stream through a ring of register stages into two alternating LDS buffers
// and are read by every wave as operand B, so a lane's 16 accumulators are
// 16 text rows of one visual column.  Each wave turns them into attention,
// sums its rows in-lane and across the half-waves, and parks the column sums
// in LDS; after the tile's barrier the first 32 threads add the waves' sums
// in a fixed order into the split's running column sums (deterministic).
// ---------------------------------------------------------------------------
// Key tiles in flight: about TREVS_PROFILE_RING_VECS 16-byte vectors per
// thread in registers.  A shallow ring keeps the kernel at 111 VGPRs, four
// waves per SIMD, which hides the loads better than a deep ring at two
// waves per SIMD (30.6 us against 38.3 us at the 16,384-token workload).
#ifndef TREVS_PROFILE_RING_VECS
#define TREVS_PROFILE_RING_VECS 2
#endif
constexpr int profile_ring(int vectors_per_tile) {
  return vectors_per_tile >= TREVS_PROFILE_RING_VECS ? 1
                                                     : TREVS_PROFILE_RING_VECS / vectors_per_tile;
}

template <class In, int DH, int QW>
__global__ __launch_bounds__(64 * QW) void t2v_profile_kernel(ProfileArgs a) {
  constexpr int ROWB = DH * In::kBytes;
  constexpr int HALFB = ROWB / 2;
  constexpr int NF = HALFB / 64;
  constexpr int NT = 64 * QW;
  constexpr int LROW = ROWB + 16;
  constexpr int CPR = ROWB / 16;
  constexpr int TV = 32 * CPR;  // 16-byte vectors of one key tile
  constexpr int TVT = (TV + NT - 1) / NT;
  constexpr int RING = profile_ring(TVT);
  __shared__ __attribute__((aligned(16))) uint8_t klds[2][32 * LROW];
  __shared__ float red[2][QW][32];
  __shared__ float colsum[kProfileSplitMax];
  const bool second = blockIdx.y != 0;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int half = lane >> 5, col = lane & 31;
  const int lin = xcd_remap(blockIdx.x, gridDim.x);
  const int split = lin % a.n_split;
  const int hl = (lin / a.n_split) % a.G;
  const int bg = lin / (a.n_split * a.G);
  const int g = bg % a.H_kv, b = bg / a.H_kv;
  const int h = g * a.G + hl;
  const size_t seq0 = (size_t)b * a.S;
  const int i_begin = split * a.split_len;
  const int i_end = min(a.K_in, i_begin + a.split_len);
  const int n_tiles = (i_end - i_begin + 31) / 32;
  for (int t = tid; t < n_tiles * 32; t += NT) colsum[t] = 0.f;

  const uint8_t* kbase = reinterpret_cast<const uint8_t*>((second ? a.k[1] : a.k[0])) + (seq0 + a.P) * a.H_kv * ROWB +
                         (size_t)g * ROWB;
  const size_t kstride = (size_t)a.H_kv * ROWB;
  // one key tile (rows ib..ib+31) into registers; rows past the split re-read
  // row i_begin (valid, cached)
  auto load_tile = [&](int ib, u32x4 (&dst)[TVT]) {
#pragma unroll
    for (int k = 0; k < TVT; ++k) {
      const int v = min(tid + k * NT, TV - 1), row = v / CPR, c = v - row * CPR;
      const int i = ib + row;
      dst[k] = ldg16(kbase + (size_t)(i < i_end ? i : i_begin) * kstride + c * 16);
    }
  };
  auto store_tile = [&](int buf, const u32x4 (&src)[TVT]) {
#pragma unroll
    for (int k = 0; k < TVT; ++k) {
      const int v = tid + k * NT;
      if (v < TV) {
        const int row = v / CPR, c = v - row * CPR;
        *reinterpret_cast<u32x4*>(&klds[buf][row * LROW + c * 16]) = src[k];
      }
    }
  };

  const int Tb = text_rows((second ? a.text_len[1] : a.text_len[0]), b, a.T_max);
  const int n_qblk = (Tb + 31) / 32;
  const int n_pass = (n_qblk + QW - 1) / QW;  // uniform over the workgroup (barriers below)
  const int n_iter = (n_tiles + RING - 1) / RING;
  for (int pass = 0; pass < n_pass; ++pass) {
    // text block of this wave; a wave past the last block reads a valid block
    // and masks every row
    const int qb = pass * QW + wave;
    const int qbc = min(qb, n_qblk - 1);
    const int qrow = min(qbc * 32 + col, a.T_max - 1);
    const uint8_t* qp = reinterpret_cast<const uint8_t*>((second ? a.q[1] : a.q[0])) +
                        ((seq0 + a.P + a.K_in + qrow) * a.H_q + h) * ROWB + half * HALFB;
    u32x4 qf[NF][4];
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
      for (int j = 0; j < 4; ++j) qf[f][j] = ldg16(qp + f * 64 + j * 16);
    // rows of lse2 are padded to a multiple of 32: the block's reads stay in
    // the row; entries past T_b are masked below
    const float* lrow = (second ? a.lse2[1] : a.lse2[0]) + ((size_t)b * a.H_q + h) * a.T_pad + qbc * 32 + 4 * half;
    float nl[16];  // minus the row log-sum-exp, or -inf for a masked row
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float4 l = *reinterpret_cast<const float4*>(lrow + 8 * j);
      const float l4[4] = {l.x, l.y, l.z, l.w};
#pragma unroll
      for (int c = 0; c < 4; ++c)
        nl[4 * j + c] = (qb * 32 + mfma_row(4 * j + c, half) < Tb) ? -l4[c] : -INFINITY;
    }

    u32x4 ring[RING][TVT];
#pragma unroll
    for (int c = 0; c < RING; ++c) load_tile(i_begin + 32 * c, ring[c]);
    for (int it = 0; it < n_iter; ++it) {
#pragma unroll
      for (int c = 0; c < RING; ++c) {
        const int t = it * RING + c;
        // LDS buffer (t % 2) was last read at tile t - 2, before every wave
        // passed the barrier of tile t - 1
        store_tile(t & 1, ring[c]);
        load_tile(i_begin + 32 * (t + RING), ring[c]);
        __syncthreads();
        if (t < n_tiles) {
          const uint8_t* p = &klds[t & 1][col * LROW + half * HALFB];
          f32x16 acc;
#pragma unroll
          for (int rr = 0; rr < 16; ++rr) acc[rr] = 0.f;
#pragma unroll
          for (int f = 0; f < NF; ++f) {
            u32x4 kf[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) kf[j] = *reinterpret_cast<const u32x4*>(p + f * 64 + j * 16);
            acc = mfma_frag(qf[f], kf, acc, In{});
          }
          float sum = 0.f;
#pragma unroll
          for (int rr = 0; rr < 16; ++rr) sum += __builtin_amdgcn_exp2f(fmaf(acc[rr], a.scale_log2e, nl[rr]));
          sum += __shfl_xor(sum, 32, 64);
          if (half == 0) red[t & 1][wave][col] = sum;
        }
        // the sums parked at this tile are read after the next barrier, and
        // red[t & 1] is written again only after the one after it
        if (t >= 1 && t - 1 < n_tiles && tid < 32) {
          float v = 0.f;
#pragma unroll
          for (int w = 0; w < QW; ++w) v += red[(t - 1) & 1][w][tid];
          colsum[(t - 1) * 32 + tid] += v;
        }
      }
    }
    __syncthreads();
    // the last tile's sums (every earlier one was added inside the loop)
    const int tl = n_iter * RING - 1;
    if (tl < n_tiles && tid < 32) {
      float v = 0.f;
#pragma unroll
      for (int w = 0; w < QW; ++w) v += red[tl & 1][w][tid];
      colsum[tl * 32 + tid] += v;
    }
    __syncthreads();
  }
  const float inv_t = 1.f / (float)Tb;
  float* out = (second ? a.profile[1] : a.profile[0]) + ((size_t)b * a.H_q + h) * a.K_in;
  for (int t = tid; t < i_end - i_begin; t += NT) out[i_begin + t] = colsum[t] * inv_t;
}

// ---------------------------------------------------------------------------
// Text sensitivity, one workgroup per (head, sample): Eq. (1) between the
// two questions' profiles, with the dot product and squared norms summed in
// double (a sensitivity near 0 is a small difference of O(1) terms).
// ---------------------------------------------------------------------------
constexpr int kSensThreads = 256;

__device__ __forceinline__ double wave_sum_f64(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

__global__ __launch_bounds__(kSensThreads) void sensitivity_kernel(SensitivityArgs a) {
  __shared__ double red[3][kSensThreads / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int h = blockIdx.x, b = blockIdx.y;
  const size_t base = ((size_t)b * a.H_q + h) * a.K_in;
  double d = 0.0, n0 = 0.0, n1 = 0.0;
  for (int i0 = tid; i0 < a.K_in; i0 += 8 * kSensThreads) {  // 16 loads in flight
    float x[8], y[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int i = min(i0 + k * kSensThreads, a.K_in - 1);
      x[k] = a.profile[0][base + i];
      y[k] = a.profile[1][base + i];
    }
#pragma unroll
    for (int k = 0; k < 8; ++k)
      if (i0 + k * kSensThreads < a.K_in) {
        d = fma((double)x[k], (double)y[k], d);
        n0 = fma((double)x[k], (double)x[k], n0);
        n1 = fma((double)y[k], (double)y[k], n1);
      }
  }
  d = wave_sum_f64(d);
  n0 = wave_sum_f64(n0);
  n1 = wave_sum_f64(n1);
  if (lane == 0) {
    red[0][wave] = d;
    red[1][wave] = n0;
    red[2][wave] = n1;
  }
  __syncthreads();
  if (tid == 0) {
    double D = 0.0, N0 = 0.0, N1 = 0.0;
    for (int w = 0; w < kSensThreads / 64; ++w) {
      D += red[0][w];
      N0 += red[1][w];
      N1 += red[2][w];
    }
    a.ts[(size_t)b * a.H_q + h] = (float)(1.0 - D / sqrt(N0 * N1));
  }
}

// ---------------------------------------------------------------------------
// Spearman correlation within the top-K saliency set.  The average rank of
// token i in a K-vector x is r_i = #{x_j < x_i} + (#{x_j == x_i} + 1) / 2
// (1-based, ties sharing the mean of the ranks they span), so
// c_i = 2 r_i - (K + 1) is an integer in [1-K, K-1] that sums to zero: the
// centred rank, doubled.  The correlation of the ranks is
// sum c^v c^t / sqrt(sum (c^v)^2 sum (c^t)^2), and all three sums are exact
// in 64-bit integers.  A workgroup ranks kRankTile tokens (one per lane of
// every wave) against the whole set: the set's (s^v, s^t) pairs are staged
// through LDS in chunks, each wave counts over every 16th entry of a chunk
// (the same entry for all lanes, an LDS broadcast), and the counts of the
// waves are added through LDS.  A second kernel adds the workgroups'
// integer sums per sample and forms the ratio in double.
// ---------------------------------------------------------------------------
constexpr int kRankWaves = 16;
constexpr int kRankThreads = 64 * kRankWaves;
constexpr int kRankChunk = 4096;                  // (s^v, s^t) pairs staged in LDS per step
constexpr int kRankPer = kRankChunk / kRankThreads;  // pairs each thread stages

__global__ __launch_bounds__(kRankThreads) void spearman_rank_kernel(SpearmanArgs a) {
  __shared__ float2 vals[kRankChunk];
  __shared__ int cnt[4][kRankWaves][64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int tile = blockIdx.x, b = blockIdx.y;
  const int K = a.K;
  const int32_t* idx = a.idx + (size_t)b * K;
  const float* sv = a.sv + (size_t)b * a.N;
  const float* st = a.st + (size_t)b * a.N;
  const int i = tile * kRankTile + lane;
  const int ii = min(max(idx[min(i, K - 1)], 0), a.N - 1);
  const float vi = sv[ii], ti = st[ii];
  int lv = 0, ev = 0, lt = 0, et = 0;
  for (int c0 = 0; c0 < K; c0 += kRankChunk) {
    const int n = min(kRankChunk, K - c0);
    // every index load of the chunk first, then every value load
    int jj[kRankPer];
#pragma unroll
    for (int e = 0; e < kRankPer; ++e) {
      const int j = tid + e * kRankThreads;
      jj[e] = j < n ? min(max(idx[c0 + j], 0), a.N - 1) : 0;
    }
    float2 v[kRankPer];
#pragma unroll
    for (int e = 0; e < kRankPer; ++e) v[e] = make_float2(sv[jj[e]], st[jj[e]]);
#pragma unroll
    for (int e = 0; e < kRankPer; ++e) {
      const int j = tid + e * kRankThreads;
      if (j < n) vals[j] = v[e];
    }
    __syncthreads();
#pragma unroll 4
    for (int j = wave; j < n; j += kRankWaves) {
      const float2 p = vals[j];
      lv += p.x < vi ? 1 : 0;
      ev += p.x == vi ? 1 : 0;
      lt += p.y < ti ? 1 : 0;
      et += p.y == ti ? 1 : 0;
    }
    __syncthreads();
  }
  cnt[0][wave][lane] = lv;
  cnt[1][wave][lane] = ev;
  cnt[2][wave][lane] = lt;
  cnt[3][wave][lane] = et;
  __syncthreads();
  if (wave == 0) {
    int LV = 0, EV = 0, LT = 0, ET = 0;
#pragma unroll
    for (int w = 0; w < kRankWaves; ++w) {
      LV += cnt[0][w][lane];
      EV += cnt[1][w][lane];
      LT += cnt[2][w][lane];
      ET += cnt[3][w][lane];
    }
    long long cv = 0, ct = 0;
    if (i < K) {
      cv = 2LL * LV + EV + 1 - ((long long)K + 1);
      ct = 2LL * LT + ET + 1 - ((long long)K + 1);
    }
    long long s_vt = cv * ct, s_vv = cv * cv, s_tt = ct * ct;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      s_vt += __shfl_xor(s_vt, o, 64);
      s_vv += __shfl_xor(s_vv, o, 64);
      s_tt += __shfl_xor(s_tt, o, 64);
    }
    if (lane == 0) {
      long long* out = a.part + ((size_t)b * a.n_tiles + tile) * 4;
      out[0] = s_vt;
      out[1] = s_vv;
      out[2] = s_tt;
      out[3] = 0;
    }
  }
}

// One wave per sample: the workgroups' integer sums, then the ratio.
__global__ __launch_bounds__(64) void spearman_final_kernel(SpearmanArgs a) {
  const int b = blockIdx.x, lane = threadIdx.x;
  long long s_vt = 0, s_vv = 0, s_tt = 0;
  const long long* p = a.part + (size_t)b * a.n_tiles * 4;
  for (int t = lane; t < a.n_tiles; t += 64) {
    s_vt += p[4 * t];
    s_vv += p[4 * t + 1];
    s_tt += p[4 * t + 2];
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    s_vt += __shfl_xor(s_vt, o, 64);
    s_vv += __shfl_xor(s_vv, o, 64);
    s_tt += __shfl_xor(s_tt, o, 64);
  }
  if (lane == 0)
    a.rho[b] = (s_vv == 0 || s_tt == 0) ? __builtin_nan("")
                                        : (double)s_vt / sqrt((double)s_vv * (double)s_tt);
}

// ---------------------------------------------------------------------------
// The same for sets of kBinRanksMin to kBinRanks tokens, in one launch with the
// selection of the set: one workgroup per sample, entries 4 t .. 4 t + 3 with
// thread t.  A token's ranks follow from the number of values below it and
// equal to it, which need only be counted among its neighbours: the values are
// spread over as many bins as there are values, between the smallest and the
// largest; the bins that hold more than kBinScan are spread again over as many
// bins as they hold, and so on (three times at most); then a token compares
// itself with the values of its bin, unless they are all equal.  Counting all
// pairs instead costs 8 K^2 lane operations: the top 4096 of 16,384 tokens,
// 4 samples, took 42 us in three launches (selection 12, pairs 25, final 4.5)
// and take 34 here; a bitonic sort and binary searches in one workgroup took 70.
// Sets below kBinRanksMin keep the pairs, which are few (a call with both questions
// of the text sensitivity: top 3888 77.8 -> 72.8 us, top 2326 75.2 -> 74.1, top
// 1586 80.8 -> 82.6, top 607 46.0 -> 52.4).  So do sets above kBinRanks: four
// entries a thread and 16 bytes of LDS an entry (64 of 160 KB) are what this is
// laid out for, and more entries were not tried (4 samples of 16,384, ranks
// alone: top 4096 31 us, top 4097 54, top 8192 89).
// ---------------------------------------------------------------------------
constexpr int kBinRanks = 4096, kBinRanksMin = 2048;
constexpr int kRankPerThread = kBinRanks / kSelThreads;
constexpr int kBinScan = 16, kBinLevels = 4;
static_assert(kRankPerThread == 4, "four entries per thread");

// Value not counted by any other: past the set, and not-a-number.
constexpr uint32_t kNoRank = 0xffffffffu;

struct RankShared {
  uint32_t cnt[kBinRanks], mn[kBinRanks], mx[kBinRanks], val[kBinRanks];
  uint32_t red_mn[kSelWaves], red_mx[kSelWaves];
};

// below[e], equal[e]: how many of the workgroup's keys lie below key[e] and how
// many equal it (itself included); 0 for kNoRank, which no key counts.
__device__ void block_ranks(const uint32_t (&key)[4], int (&below)[4], int (&equal)[4], RankShared& rs,
                            SelectShared& sh) {
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  uint32_t lo = 0xffffffffu, hi = 0u;
  int n_mine = 0;
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (key[e] != kNoRank) {
      lo = min(lo, key[e]);
      hi = max(hi, key[e]);
      ++n_mine;
    }
  int n_all;
  (void)block_excl_scan(n_mine, sh, n_all);
  lo = wave_min_u32(lo);
  hi = wave_max_u32(hi);
  if (lane == 0) {
    rs.red_mn[wave] = lo;
    rs.red_mx[wave] = hi;
  }
  __syncthreads();
  lo = wave_min_u32(lane < kSelWaves ? rs.red_mn[lane] : 0xffffffffu);
  hi = wave_max_u32(lane < kSelWaves ? rs.red_mx[lane] : 0u);
  // entry e lies in the bin of n[e] values that starts at place s[e]
  int s[4], n[4];
  uint32_t mn[4], mx[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    s[e] = 0;
    n[e] = key[e] != kNoRank ? n_all : 0;
    mn[e] = lo;
    mx[e] = hi;
  }
  for (int level = 0;; ++level) {
    int at[4];
    *reinterpret_cast<u32x4*>(&rs.cnt[4 * tid]) = zero4();
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      at[e] = s[e];
      if (n[e] > kBinScan && mn[e] != mx[e])  // the same steps for every key of the bin: order is kept
        at[e] += min((int)((float)(key[e] - mn[e]) * ((float)(n[e] - 1) / (float)(mx[e] - mn[e]))), n[e] - 1);
      if (n[e]) atomicAdd(&rs.cnt[at[e]], 1u);
    }
    __syncthreads();
    const u32x4 c = *reinterpret_cast<const u32x4*>(&rs.cnt[4 * tid]);
    int tot;
    uint32_t run = (uint32_t)block_excl_scan((int)(c[0] + c[1] + c[2] + c[3]), sh, tot);
    u32x4 st;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      st[j] = run;
      run += c[j];
    }
    *reinterpret_cast<u32x4*>(&rs.val[4 * tid]) = st;  // (the starts, until the values take their place)
    *reinterpret_cast<u32x4*>(&rs.mn[4 * tid]) = u32x4{~0u, ~0u, ~0u, ~0u};
    *reinterpret_cast<u32x4*>(&rs.mx[4 * tid]) = zero4();
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (n[e]) {
        s[e] = (int)rs.val[at[e]];
        n[e] = (int)rs.cnt[at[e]];
        if (n[e] > kBinScan) {
          atomicMin(&rs.mn[s[e]], key[e]);
          atomicMax(&rs.mx[s[e]], key[e]);
        }
      }
    __syncthreads();
    bool more = false;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (n[e] > kBinScan) {
        mn[e] = rs.mn[s[e]];
        mx[e] = rs.mx[s[e]];
        more |= mn[e] != mx[e];
      }
    if (!__syncthreads_or(more) || level + 1 == kBinLevels) break;  // uniform
  }
  // the values, bin by bin (cnt counts them in again)
  *reinterpret_cast<u32x4*>(&rs.cnt[4 * tid]) = zero4();
  __syncthreads();
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (n[e]) rs.val[s[e] + (int)atomicAdd(&rs.cnt[s[e]], 1u)] = key[e];
  __syncthreads();
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    below[e] = s[e];
    equal[e] = n[e];
    if (n[e] <= kBinScan || mn[e] != mx[e]) {
      equal[e] = 0;
      for (int j = 0; j < n[e]; ++j) {
        const uint32_t v = rs.val[s[e] + j];
        below[e] += v < key[e] ? 1 : 0;
        equal[e] += v == key[e] ? 1 : 0;
      }
    }
  }
  __syncthreads();  // rs is used again
}

template <int E>
__global__ __launch_bounds__(kSelThreads) void topk_spearman_kernel(const float* sv_all, const float* st_all, int N,
                                                                    int K, int32_t* idx_all, double* rho) {
  __shared__ SelectShared sh;
  __shared__ __attribute__((aligned(16))) RankShared rs;
  __shared__ long long red[3][kSelWaves];
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const float* sv = sv_all + (size_t)b * N;
  const float* st = st_all + (size_t)b * N;
  int32_t* idx = idx_all + (size_t)b * K;
  {
    float sc[E];
#pragma unroll
    for (int e = 0; e < E; ++e) sc[e] = sv[min(e * kSelThreads + tid, N - 1)];  // unconditional loads
#pragma unroll
    for (int e = 0; e < E; ++e)
      if (e * kSelThreads + tid >= N) sc[e] = 0.f;
    block_topk_write<E>(sc, N, K, idx, sh);
  }
  __syncthreads();  // the set is written
  int ii[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) ii[e] = min(max(idx[min(tid * 4 + e, K - 1)], 0), N - 1);
  float x[2][4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    x[0][e] = sv[ii[e]];
    x[1][e] = st[ii[e]];
  }
  // twice the centred rank: 2 #below + #equal + 1 - (K + 1)
  int c[2][4];
#pragma unroll
  for (int v = 0; v < 2; ++v) {
    uint32_t key[4];
    int below[4], equal[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) key[e] = tid * 4 + e < K && x[v][e] == x[v][e] ? f2key(x[v][e]) : kNoRank;
    block_ranks(key, below, equal, rs, sh);
#pragma unroll
    for (int e = 0; e < 4; ++e) c[v][e] = 2 * below[e] + equal[e] - K;
  }
  long long s_vt = 0, s_vv = 0, s_tt = 0;
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (tid * 4 + e < K) {
      s_vt += (long long)c[0][e] * c[1][e];
      s_vv += (long long)c[0][e] * c[0][e];
      s_tt += (long long)c[1][e] * c[1][e];
    }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    s_vt += __shfl_xor(s_vt, o, 64);
    s_vv += __shfl_xor(s_vv, o, 64);
    s_tt += __shfl_xor(s_tt, o, 64);
  }
  if (lane == 0) {
    red[0][wave] = s_vt;
    red[1][wave] = s_vv;
    red[2][wave] = s_tt;
  }
  __syncthreads();
  if (tid == 0) {
    s_vt = s_vv = s_tt = 0;
    for (int w = 0; w < kSelWaves; ++w) {
      s_vt += red[0][w];
      s_vv += red[1][w];
      s_tt += red[2][w];
    }
    rho[b] = (s_vv == 0 || s_tt == 0) ? __builtin_nan("") : (double)s_vt / sqrt((double)s_vv * (double)s_tt);
  }
}

// ---------------------------------------------------------------- launchers
static int profile_waves(int T_max) {
  const int qb = (T_max + 31) / 32;
  return qb >= 4 ? 4 : (qb >= 2 ? 2 : 1);
}

template <class In, int DH>
static void launch_profile_t(const ProfileArgs& a, hipStream_t s) {
  const dim3 grid(a.B * a.H_q * a.n_split, 2);
  switch (profile_waves(a.T_max)) {
    case 4: hipLaunchKernelGGL((t2v_profile_kernel<In, DH, 4>), grid, dim3(256), 0, s, a); break;
    case 2: hipLaunchKernelGGL((t2v_profile_kernel<In, DH, 2>), grid, dim3(128), 0, s, a); break;
    default: hipLaunchKernelGGL((t2v_profile_kernel<In, DH, 1>), grid, dim3(64), 0, s, a); break;
  }
}

template <class In>
static void launch_profile_d(const ProfileArgs& a, int dh, hipStream_t s) {
  if (dh == 64)
    launch_profile_t<In, 64>(a, s);
  else if (dh == 128)
    launch_profile_t<In, 128>(a, s);
  else
    launch_profile_t<In, 256>(a, s);
}

hipError_t launch_profile(const ProfileArgs& a, int dtype, int dh, hipStream_t s) {
  if (dtype == 1)
    launch_profile_d<BF16>(a, dh, s);
  else
    launch_profile_d<F32>(a, dh, s);
  return hipGetLastError();
}

hipError_t launch_sensitivity(const SensitivityArgs& a, int B, hipStream_t s) {
  hipLaunchKernelGGL(sensitivity_kernel, dim3(a.H_q, B), dim3(kSensThreads), 0, s, a);
  return hipGetLastError();
}

static hipError_t launch_spearman(const SpearmanArgs& a, int B, hipStream_t s) {
  hipLaunchKernelGGL(spearman_rank_kernel, dim3(a.n_tiles, B), dim3(kRankThreads), 0, s, a);
  hipLaunchKernelGGL(spearman_final_kernel, dim3(B), dim3(64), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_topk_spearman(const SpearmanArgs& a, int B, int32_t* idx, hipStream_t s) {
  if (a.K > kBinRanks || a.K < kBinRanksMin) {
    const hipError_t e = launch_topk(a.sv, B, a.N, a.K, idx, s);
    return e == hipSuccess ? launch_spearman(a, B, s) : e;
  }
#define CALL(E_)                                                                                               \
  case E_:                                                                                                     \
    hipLaunchKernelGGL(topk_spearman_kernel<E_>, dim3(B), dim3(kSelThreads), 0, s, a.sv, a.st, a.N, a.K, idx, \
                       a.rho);                                                                                 \
    break
  switch (select_e(a.N)) {
    CALL(1); CALL(2); CALL(4); CALL(8); CALL(16); CALL(32); CALL(64);
    default: return hipErrorInvalidValue;
  }
#undef CALL
  return hipGetLastError();
}

}  // namespace trevs
