// Products of the visual features with each other, for the context
// preservation by farthest point sampling (Sec. 4.1, after Eq. (7)): the Gram
// matrix of all tokens of a sample or of a pool of them, and, where only the
// nearest selected token matters, maxima over the selected tokens.
#include <algorithm>

#include "common.hpp"
#include "kernels.hpp"

namespace trevs {

// ---------------------------------------------------------------------------
// Gram matrix.  G is symmetric, so only the tiles (tj, ti) with tj <= ti are
// computed: a workgroup of 4 waves computes the 128x128 tile of G[b] (rows j
// of the tile's first operand, columns i of the second), streaming the
// feature dimension in 128-byte slabs: each thread loads its share of both
// slabs with coalesced 16-byte loads (8 lanes per 128-byte row segment) into
// a ring of two register buffers, writes them to one of two LDS buffers
// (rows XOR-swizzled by 16-byte chunk), and the waves multiply on the matrix
// cores, each a 64x64 block.  Bytes past a row's end (a partial last slab)
// load as zero.  The tile is written in place and, off the diagonal, also
// transposed; both go through LDS and out as 16-byte runs of whole rows.
// Diagonal tiles also write 1/max(||z_i||, 1e-12) from G_ii.  G is written
// with nontemporal stores: the picks read it back long after it has left the
// caches, and cached stores would evict operand slabs the other resident
// workgroups still read.  Products over lists take the k-steps in the order of
// the full matrix (a.natural: that of the 256-row tiles), so that a product is
// the same, bit for bit, wherever it is formed.
// ---------------------------------------------------------------------------
constexpr int kGramTile = 128;
constexpr int kGramThreads = 256;

// Workgroup order: the tiles on and above the diagonal are walked in
// super-blocks of gs x gs tiles (gs = min(8, tiles per side)), so that the
// workgroups resident on one XCD at a time share 2*gs row blocks of Z and
// each slab they stream is reused from L2 by up to gs workgroups (in
// row-major tile order they shared one row block and streamed 64 distinct
// ones).  Super-blocks are numbered row-major over the pairs sj <= si, and
// every workgroup gets a tile: a diagonal super-block holds only its tiles
// on and above the diagonal (row-major), so the workgroups resident at one
// time cover compact runs of tiles instead of slots that exit at once.
__host__ __device__ constexpr int gram_super(int n_tiles) { return n_tiles < 8 ? n_tiles : 8; }
__host__ __device__ constexpr int gram_tiles(int n_tiles) { return n_tiles * (n_tiles + 1) / 2; }

// tile (tj, ti), tj <= ti, of dense index t in [0, gram_tiles(nT))
__device__ __forceinline__ void gram_tile_of(int t, int nT, int& tj, int& ti) {
  const int gs = gram_super(nT), nS = (nT + gs - 1) / gs;
  tj = 0;
  ti = 0;
  for (int sj = 0; sj < nS; ++sj) {
    const int h = min(gs, nT - sj * gs);
    for (int si = sj; si < nS; ++si) {
      const int w = min(gs, nT - si * gs);
      const int cnt = si == sj ? h * (h + 1) / 2 : h * w;
      if (t < cnt) {
        if (si == sj) {
          int r = 0;
          while (t >= h - r) {
            t -= h - r;
            ++r;
          }
          tj = sj * gs + r;
          ti = sj * gs + r + t;
        } else {
          tj = sj * gs + t / w;
          ti = si * gs + t % w;
        }
        return;
      }
      t -= cnt;
    }
  }
}

// Workgroup w -> (sample b, dense tile index t).  With many tiles per sample
// (kGramStripe or more) XCD x takes the x-th eighth of every sample's tiles
// (a contiguous run in super-block order, for its L2), sample after sample,
// so that at any time all XCDs stream the same sample's Z, which fits the
// last-level cache (all samples together need not); workgroups go to the 8
// XCDs round-robin, and the grid, 8 * B * ceil(tiles / 8), has a few padding
// workgroups (false).  With few tiles per sample each XCD keeps whole
// samples instead (a contiguous range of workgroups per XCD), so that a
// sample's Z is loaded into one L2 only.
constexpr int kGramStripe = 64;
__device__ __forceinline__ bool gram_work(int w, int per_b, int B, int& b, int& t) {
  if (per_b < kGramStripe) {
    const int lin = xcd_remap(w, B * per_b);
    b = lin / per_b;
    t = lin - b * per_b;
    return true;
  }
  const int x = w & 7, k = w >> 3;
  const int r0 = (x * per_b) >> 3, L = (((x + 1) * per_b) >> 3) - r0;  // L >= 8
  b = k / L;
  t = r0 + (k - b * L);
  return b < B;
}
__host__ __device__ constexpr int gram_grid(int per_b, int B) {
  return per_b < kGramStripe ? B * per_b : 8 * B * ((per_b + 7) / 8);
}

// What a Gram launch computes.  kGramFull: all pairs of a sample's tokens.
// kGramPool: all pairs of a list of tokens (a.rows).  kGramMax: for every
// token of one list (a.cols) the maximum over another (a.rows), so that the
// products themselves are never written; row tiles meet in integer atomics, one
// for each column of a tile (a partial maximum for each row tile had to be read back
// by the one workgroup that selects the pool).  kGramNext: the same over the last
// round's picks only, as distances; the columns' norms are formed on the way,
// each wave multiplying 32 columns by themselves (a quarter more multiplies,
// in place of a launch that is empty in most calls).  kGramRest: all pairs of the
// tokens that are no pivots (a.cols), where the rounds did not suffice.
enum { kGramFull = 0, kGramPool = 1, kGramMax = 2, kGramNext = 3, kGramRest = 4 };

__device__ __forceinline__ bool gram_done(const GramArgs& a, int b) {
  return a.ctrl && a.ctrl[b * kPickCtrl + kCtrlPicks] >= a.K_d;
}

// kGramMax, kGramNext: workgroup -> (sample, row tile, column tile), false for a padding
// workgroup.  Tiles are walked in groups of four column tiles, so that the
// workgroups of one XCD share about as many rows as columns in its L2; with
// 64 tiles or more a sample's are striped over the XCDs as above.
__device__ __forceinline__ bool gram_list_work(const GramArgs& a, int w, int& b, int& tp, int& tc) {
  int t;
  if (!gram_work(w, a.n_rtiles * a.n_ctiles, a.B, b, t)) return false;
  const int full = a.n_ctiles / 4 * 4 * a.n_rtiles;
  if (t < full) {
    const int g = t / (4 * a.n_rtiles);
    t -= g * 4 * a.n_rtiles;
    tp = t >> 2;
    tc = 4 * g + (t & 3);
  } else {
    const int n = a.n_ctiles & 3;
    t -= full;
    tp = t / n;
    tc = a.n_ctiles - n + t % n;
  }
  return true;
}

// The listed rows of this launch for sample b: all of a.rows, the picks of
// the last round, or the columns.
template <int MODE>
__device__ __forceinline__ const int32_t* gram_list_rows(const GramArgs& a, int b, int& count) {
  if (MODE == kGramRest) {
    count = a.n_cols;
    return a.cols + (size_t)b * a.n_cols;
  }
  const int32_t* rows = a.rows + (size_t)b * a.n_rows;
  count = a.n_rows;
  if (MODE == kGramNext) {
    const int begin = a.ctrl[b * kPickCtrl + kCtrlRound];
    count = a.ctrl[b * kPickCtrl + kCtrlPicks] - begin;
    rows += begin;
  }
  return rows;
}

// kGramMax output of a tile of T x TC products held as MB x NB blocks by 2 x 2
// waves: max G_ij / ||z_j||, from which the distance follows as 1 - max / ||z_i||.
// kGramNext: minus the least distance, formed per product as the picks form it.
// izr, izc: the rows' and columns' inverse norms (LDS; the latter for kGramNext);
// red: 2 TC floats of LDS that nothing reads any more.
template <int MODE, int T, int TC, int MB, int NB>
__device__ __forceinline__ void gram_max_store(const GramArgs& a, const f32x16 (&acc)[MB][NB], const float* izr,
                                               const float* izc, float* red, int b, int tc, int wj, int wi) {
  const int tid = threadIdx.x, half = (tid >> 5) & 1, col = tid & 31;
  float mx[NB];
#pragma unroll
  for (int n = 0; n < NB; ++n) {
    mx[n] = -INFINITY;
    const float zc = MODE == kGramNext ? izc[wi * (TC / 2) + n * 32 + col] : 0.f;
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float iz = izr[wj * (T / 2) + m * 32 + mfma_row(r, half)];
        const float g = acc[m][n][r];
        mx[n] = fmaxf(mx[n], MODE == kGramNext ? fmaf(g * zc, iz, -1.f) : g * iz);
      }
    mx[n] = fmaxf(mx[n], __shfl_xor(mx[n], 32, 64));
  }
#pragma unroll
  for (int n = 0; n < NB; ++n)
    if (half == 0) red[wj * TC + wi * (TC / 2) + n * 32 + col] = mx[n];
  __syncthreads();
  for (int c = tid; c < TC; c += blockDim.x)
    if (tc * TC + c < a.n_cols)
      atomicMax(&a.mx[(size_t)b * a.n_cols + tc * TC + c], f2key(fmaxf(red[c], red[TC + c])));
}

__device__ __forceinline__ int gram_swizzle(int r, int c) { return c ^ ((r >> 1) & 7); }

template <class In, int MODE>
__device__ __forceinline__ void gram_tile(const GramArgs& a, int w) {
  constexpr int T = kGramTile;
  constexpr int SLAB = T * 128;                  // bytes of one operand slab
  constexpr int VPT = SLAB / 16 / kGramThreads;  // vectors per thread per operand
  constexpr int LDS = 4 * SLAB;                  // two stages of both operand slabs, then the output passes
  __shared__ __attribute__((aligned(1024))) uint8_t lds[LDS];
  uint8_t* l0 = lds;
  uint8_t* l1 = lds + 2 * SLAB;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int half = lane >> 5, col = lane & 31;
  const int nT = a.n_tiles;
  constexpr bool LISTS = MODE == kGramMax || MODE == kGramNext;
  int b, t, tj, ti;
  // (every return below is the whole workgroup's: no barrier has run)
  if (LISTS) {
    if (!gram_list_work(a, w, b, tj, ti)) return;
  } else {
    if (!gram_work(w, gram_tiles(nT), a.B, b, t)) return;
  }
  if (gram_done(a, b)) return;
  if (!LISTS) gram_tile_of(t, nT, tj, ti);
  const int rb = a.row_bytes;
  int nj = a.N, ni = a.N;  // tokens along the rows and columns
  const int32_t *rows = nullptr, *cols = nullptr;
  bool none = false;
  __shared__ float izr[MODE == kGramFull || MODE == kGramRest ? 1 : T], izc[MODE == kGramPool || MODE == kGramNext ? T : 1];
  __shared__ float xr[MODE == kGramPool ? T : 1], xc[MODE == kGramPool ? T : 1];
  if (MODE != kGramFull) {
    rows = cols = gram_list_rows<MODE>(a, b, nj);
    ni = nj;
    if (MODE == kGramPool) {  // nothing is nearer to tokens past the list, nor to selected ones (infinity)
      const int i = (tid < T ? tj * T : ti * T - T) + tid, ic = min(i, nj - 1);
      const float x = a.nearest[(size_t)b * nj + ic];
      (tid < T ? izr : izc)[tid & (T - 1)] = a.inv_norm[(size_t)b * a.N + rows[ic]];
      (tid < T ? xr : xc)[tid & (T - 1)] = i < nj ? x * (x > 0.f ? 1.f - a.margin : 1.f + a.margin) : INFINITY;
    }
    if (LISTS) {
      cols = a.cols + (size_t)b * a.n_cols;
      if (MODE == kGramNext && nj == 0) {  // a round without picks: the norms alone, with a column for a row
        none = true;
        rows = cols;
        nj = 1;
      }
      if (tj * T >= nj) return;
      ni = a.n_cols;
      if (tid < T) izr[tid] = a.inv_norm[(size_t)b * a.N + rows[min(tj * T + tid, nj - 1)]];
    }
  }
  const int N = ni, ld = a.ldg;
  const int n_slabs = (rb + 127) / 128;
  const int tail = rb & 127;  // bytes of a partial last slab, 0 if none
  const uint8_t* zb = reinterpret_cast<const uint8_t*>(a.Z) + (size_t)b * a.N * rb;
  const int cr = tid >> 3, cc = tid & 7;
  const uint8_t* src[2 * VPT];  // row starts (rows past the last re-read it)
#pragma unroll
  for (int k = 0; k < VPT; ++k) {
    const int r = cr + (kGramThreads / 8) * k;
    const int j = min(tj * T + r, nj - 1), i = min(ti * T + r, ni - 1);
    src[k] = zb + (size_t)(MODE == kGramFull ? j : rows[j]) * rb;
    src[VPT + k] = zb + (size_t)(MODE == kGramFull ? i : cols[i]) * rb;
  }
  const int sdst = cr * 128 + gram_swizzle(cr, cc) * 16;  // rows 32 apart share the swizzle
  u32x4 g[2][2 * VPT];
  // chunk cc of slab s; a chunk past the row's end reads the row's first
  // chunk (in bounds), and the store overwrites its LDS copy with zeros (a
  // select on the loaded vectors made the compiler wait for every load in
  // flight at the top of each iteration); the padding steps past the last
  // slab re-read it and are never multiplied
  auto load = [&](int s, u32x4 (&dst)[2 * VPT]) {
    const int off = min(s, n_slabs - 1) * 128 + cc * 16;
    const int o = off < rb ? off : 0;
#pragma unroll
    for (int k = 0; k < 2 * VPT; ++k) dst[k] = ldg16(src[k] + o);
  };
  auto store = [&](uint8_t* st, const u32x4 (&v)[2 * VPT], int s) {
#pragma unroll
    for (int k = 0; k < VPT; ++k) {
      *reinterpret_cast<u32x4*>(st + sdst + k * (kGramThreads / 8) * 128) = v[k];
      *reinterpret_cast<u32x4*>(st + SLAB + sdst + k * (kGramThreads / 8) * 128) = v[VPT + k];
    }
    if (s == n_slabs - 1 && tail && cc * 16 >= tail) {  // chunks past the row's end hold zeros
#pragma unroll
      for (int k = 0; k < VPT; ++k) {
        *reinterpret_cast<u32x4*>(st + sdst + k * (kGramThreads / 8) * 128) = zero4();
        *reinterpret_cast<u32x4*>(st + SLAB + sdst + k * (kGramThreads / 8) * 128) = zero4();
      }
    }
  };
  const int wj = wave >> 1, wi = wave & 1;
  f32x16 acc[2][2];
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int n = 0; n < 2; ++n)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[m][n][r] = 0.f;
  f32x16 self;  // kGramNext: columns wave * 32.. by themselves
#pragma unroll
  for (int r = 0; r < 16; ++r) self[r] = 0.f;
  // k-step q: half h holds chunk 4h + q, or 2q + h in natural order.  The
  // rows a lane reads (32 apart) share the swizzle.
  const bool natural = MODE != kGramFull && a.natural;
  uint32_t fo[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) fo[q] = col * 128 + gram_swizzle(col, natural ? 2 * q + half : 4 * half + q) * 16;
  auto frag = [&](const uint8_t* base, int row0, u32x4 (&f)[4]) {
#pragma unroll
    for (int q = 0; q < 4; ++q) f[q] = *reinterpret_cast<const u32x4*>(base + row0 * 128 + fo[q]);
  };
  auto compute = [&](const uint8_t* st) {
    u32x4 fa[2][4], fb[2][4];
#pragma unroll
    for (int m = 0; m < 2; ++m) frag(st, wj * 64 + m * 32, fa[m]);
#pragma unroll
    for (int n = 0; n < 2; ++n) frag(st + SLAB, wi * 64 + n * 32, fb[n]);
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int n = 0; n < 2; ++n) acc[m][n] = mfma_frag(fa[m], fb[n], acc[m][n], In{});
    if constexpr (MODE == kGramNext) {
      frag(st + SLAB, wave * 32, fa[0]);
      self = mfma_frag(fa[0], fa[0], self, In{});
    }
  };
  // stage 0's loads go out first: loads complete in order, so the first
  // store then waits only for them, not for stage 1's as well
  load(0, g[0]);
  __builtin_amdgcn_sched_barrier(0);
  load(1, g[1]);
  const int n_iter = (n_slabs + 1) / 2;
  for (int it = 0; it < n_iter; ++it) {
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const int s = 2 * it + c;
      uint8_t* st = c ? l1 : l0;
      // buffer c was last read at step s - 2, before every wave passed the
      // barrier of step s - 1
      store(st, g[c], s);
      load(s + 2, g[c]);
      __syncthreads();
      if (s < n_slabs) compute(st);
    }
  }
  if constexpr (MODE == kGramNext) {
    const float iz = 1.f / fmaxf(sqrtf(fmaxf(mfma_diag(self, half, col), 0.f)), 1e-12f);
    if (half == 0) izc[wave * 32 + col] = iz;
    // (picked tokens have theirs, which other workgroups may be reading)
    const int c = ti * T + wave * 32 + col;
    if (half == 0 && tj == 0 && c < ni && a.near_pick[(size_t)b * a.N + cols[c]] != -INFINITY)
      a.inv_norm[(size_t)b * a.N + cols[c]] = iz;
    if (none) return;  // uniform
  }
  if constexpr (LISTS) {
    __syncthreads();  // the operand slabs are no longer read
    gram_max_store<MODE, T, T, 2, 2>(a, acc, izr, izc, reinterpret_cast<float*>(lds), b, ti, wj, wi);
    return;
  }
  // output: register r of block (m, n) is row wj*64 + m*32 + mfma_row(r),
  // column wi*64 + n*32 + col of the tile
  if ((MODE == kGramFull || MODE == kGramRest) && tj == ti) {  // the diagonal tile holds ||z_i||^2
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int n = 0; n < 2; ++n)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int jl = wj * 64 + m * 32 + mfma_row(r, half), il = wi * 64 + n * 32 + col;
          const int i = ti * T + il;
          if (jl == il && i < N)
            a.inv_norm[(size_t)b * a.N + (MODE == kGramFull ? i : rows[i])] = 1.f / fmaxf(sqrtf(fmaxf(acc[m][n][r], 0.f)), 1e-12f);
        }
  }
  if constexpr (MODE == kGramPool) {
    // mask words of the tile, 32 tokens each: of row j, bit col where j may
    // bring col nearer (one ballot per register: a word for each half-wave's
    // row); off the diagonal of column i, bit row where i may bring row nearer
    uint32_t* mask = a.mask + (size_t)b * nj * a.mask_words;
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int n = 0; n < 2; ++n) {
        const int c = wi * 64 + n * 32 + col;
        const float iz = izc[c], x = xc[c];
        uint32_t wrow = 0u, wcol = 0u;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int row = mfma_row(r, half), j = wj * 64 + m * 32 + row;
          const float cosine = acc[m][n][r] * iz * izr[j];
          const unsigned long long bal = __ballot(cosine > x);
          wrow = lane == mfma_row(r, 0) ? (uint32_t)bal : wrow;
          wrow = lane == mfma_row(r, 1) ? (uint32_t)(bal >> 32) : wrow;
          wcol |= cosine > xr[j] ? 1u << row : 0u;
        }
        wcol |= __shfl_xor(wcol, 32, 64);
        const int j = tj * T + wj * 64 + m * 32 + lane, i = ti * T + c;
        const int jw = (tj * T + wj * 64) / 32 + m, iw = (ti * T + wi * 64) / 32 + n;
        if (lane < 32 && j < nj && iw < a.mask_words) mask[(size_t)j * a.mask_words + iw] = wrow;
        if (lane < 32 && tj != ti && i < nj && jw < a.mask_words) mask[(size_t)i * a.mask_words + jw] = wcol;
      }
  }
  // The tile leaves through LDS, 32 rows j at a time, as 16-byte runs of
  // whole rows: tA (rows j, stride TA: 16-byte aligned rows, the half-waves'
  // writes on disjoint banks) for G[j, i]; off the diagonal tB (rows i, odd
  // stride TB) for the mirrored G[i, j].  Whole tiles of a matrix whose rows
  // are a multiple of 16 bytes store without bounds checks.
  constexpr int TA = T + 8, TB = 33, PR = 32;
  static_assert((PR * TA + T * TB) * 4 <= LDS, "output staging fits the LDS");
  float* tA = reinterpret_cast<float*>(lds);
  float* tB = tA + PR * TA;
  float* gb = a.G + (size_t)b * nj * ld;
  const bool mirror = tj != ti;
  const bool fast = (ti + 1) * T <= N && (ld & 3) == 0;  // tj <= ti
#pragma unroll
  for (int p = 0; p < T / PR; ++p) {  // unrolled: the accumulator block m is a constant
    __syncthreads();  // the operand slabs, or the previous pass, are no longer read
    if (wj == p / 2) {
      const int m = p % 2;
#pragma unroll
      for (int n = 0; n < 2; ++n)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int jl = mfma_row(r, half), il = wi * 64 + n * 32 + col;
          tA[jl * TA + il] = acc[m][n][r];
          if (mirror) tB[il * TB + jl] = acc[m][n][r];
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < PR * T / 4 / kGramThreads; ++k) {  // G[j, i]: PR rows of T / 4 runs
      const int e = tid + k * kGramThreads, row = e / (T / 4), q = e % (T / 4);
      const int j = tj * T + PR * p + row, i = ti * T + 4 * q;
      const u32x4 v = *reinterpret_cast<const u32x4*>(&tA[row * TA + 4 * q]);
      if (fast) {
        stg16_stream(&gb[(size_t)j * ld + i], v);
      } else {
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (j < N && i + u < N) __builtin_nontemporal_store(__uint_as_float(v[u]), &gb[(size_t)j * ld + i + u]);
      }
    }
    if (mirror) {  // G[i, j]: T rows of PR / 4 runs
#pragma unroll
      for (int k = 0; k < PR * T / 4 / kGramThreads; ++k) {
        const int e = tid + k * kGramThreads, il = e / (PR / 4), q = e % (PR / 4);
        const int i = ti * T + il, j = tj * T + PR * p + 4 * q;
        const float* src = &tB[il * TB + 4 * q];
        const u32x4 v = {__float_as_uint(src[0]), __float_as_uint(src[1]), __float_as_uint(src[2]),
                         __float_as_uint(src[3])};
        if (fast) {
          stg16_stream(&gb[(size_t)i * ld + j], v);
        } else {
#pragma unroll
          for (int u = 0; u < 4; ++u)
            if (i < N && j + u < N) __builtin_nontemporal_store(__uint_as_float(v[u]), &gb[(size_t)i * ld + j + u]);
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Gram matrix at 256x256 tiles, bf16 (N >= kGram256MinN, N + 256 rows of Z
// under 2 GB; fp32 inputs use gram_kernel; rows are a multiple of 16 bytes): a
// workgroup of 4 waves, one per SIMD, each a 128x128 block (4x4 MFMA tiles,
// 256 accumulation registers), so that each fragment byte read from LDS
// feeds 4 multiplies.  The feature dimension streams in 128-byte stages
// (four k-steps), loaded 8 lanes to a row (whole 128-byte lines: 4 lanes to
// a row, 64 bytes, cost about a tenth of the Gram's time) into a ring of two
// register stages, then into two LDS buffers.  Stage P runs in two halves:
// the first multiplies k-steps 0-1 while it stores stage P + 1 into the
// other buffer (free since the last barrier) and loads stage P + 3 into the
// register stage it frees; after a barrier, the second multiplies k-steps
// 2-3 while it reads stage P + 1's first fragments.  Every k-step's
// fragments are read during the previous k-step's multiplies, so each half
// starts on fragments already in registers.  The loads are buffer loads:
// chunks past a row's end, rows past N and stages past the last read zeros,
// which the multiplies add exactly, so the steps need no branches.  Rows are
// XOR-swizzled in 16-byte chunks (chunk ^ ((row >> 1) & 7)): the stores (2
// rows x 128 bytes per 16 lanes) and the fragment reads (16 rows at one
// chunk) hit all 64 banks.  Same super-block order and outputs as
// gram_kernel; both output tiles leave through LDS as 16-byte runs of whole
// rows.
// ---------------------------------------------------------------------------
constexpr int kGram256Threads = 256;
constexpr int kGram256MinN = 2048;

template <int MODE, int TC = 256>
__device__ __forceinline__ void gram256_tile(const GramArgs& a, int w) {
  static_assert(TC == 256 || (TC == 192 && MODE == kGramMax), "tile columns");
  constexpr int T = 256;
  constexpr int SLAB = T * 128;                     // bytes of one operand's 128-byte stage
  constexpr int VPT = SLAB / 16 / kGram256Threads;  // 8 vectors per thread per operand
  constexpr int NB = TC / 64;                       // 32-column blocks per wave
  constexpr int SLABB = TC * 128, VPB = VPT * TC / T;  // the column operand's
  constexpr int RSTEP = kGram256Threads / 8;        // rows per load pass (8 lanes a row)
  constexpr int TA = T + 8, TB = 33, PR = 32;       // output staging (see below)
  constexpr int LDS_OPS = 2 * (SLAB + SLABB);
  constexpr int LDS_OUT = (PR * TA + T * TB) * 4;
  constexpr int LDS = MODE == kGramMax || LDS_OPS > LDS_OUT ? LDS_OPS : LDS_OUT;
  __shared__ __attribute__((aligned(1024))) uint8_t lds[LDS];
  int tid = threadIdx.x;
  // (a workgroup that walks several tiles forms its addresses anew for each: kept
  // from tile to tile they spilled 75 registers)
  if (MODE == kGramRest) asm volatile("" : "+v"(tid));
  const int lane = tid & 63, wave = tid >> 6;
  const int half = lane >> 5, col = lane & 31;
  const int nT = a.n_tiles;
  int b, t, tj, ti;
  // (every return below is the whole workgroup's: no barrier has run)
  if (MODE == kGramMax) {
    if (!gram_list_work(a, w, b, tj, ti)) return;
  } else {
    if (!gram_work(w, gram_tiles(nT), a.B, b, t)) return;
  }
  if (gram_done(a, b)) return;
  if (MODE != kGramMax) gram_tile_of(t, nT, tj, ti);
  const int N = a.N, rb = a.row_bytes;
  const int n_stages = (rb + 127) / 128;
  // rows past N read zeros (their offsets pass N * rb), and so do the chunks
  // of a stage that is past the row's end (offset + 2^31): with
  // (N + 256) * rb < 2^31 no offset wraps.  Rows and columns past N are never
  // stored.
  const __amdgpu_buffer_rsrc_t zs = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint8_t*>(reinterpret_cast<const uint8_t*>(a.Z) + (size_t)b * N * rb), 0, N * rb,
      kBufferRsrcWord3);
  const int cr = tid >> 3, cc = tid & 7;
  // the thread loads chunk cc of rows cr + RSTEP * k of both operands
  const uint32_t rowA = (uint32_t)(tj * T + cr) * rb + cc * 16;
  const uint32_t rowB = (uint32_t)(ti * TC + cr) * rb + cc * 16;
  const uint32_t kstride = (uint32_t)RSTEP * rb;
  // listed tokens: an offset per row (rows past the last re-read it)
  __shared__ float izr[MODE == kGramMax ? T : 1];
  uint32_t offA[VPT], offB[VPB];
  if constexpr (MODE != kGramFull) {
    int nj;
    const int32_t* rows = gram_list_rows<MODE>(a, b, nj);
    const int32_t* cols = a.cols + (size_t)b * a.n_cols;
    if (MODE == kGramMax && tid < T) izr[tid] = a.inv_norm[(size_t)b * N + rows[min(tj * T + tid, nj - 1)]];
#pragma unroll
    for (int k = 0; k < VPT; ++k) offA[k] = (uint32_t)rows[min(tj * T + cr + RSTEP * k, nj - 1)] * rb + cc * 16;
#pragma unroll
    for (int k = 0; k < VPB; ++k) offB[k] = (uint32_t)cols[min(ti * TC + cr + RSTEP * k, a.n_cols - 1)] * rb + cc * 16;
  } else {
#pragma unroll
    for (int k = 0; k < VPT; ++k) offA[k] = rowA + k * kstride;
#pragma unroll
    for (int k = 0; k < VPB; ++k) offB[k] = rowB + k * kstride;
  }
  // LDS: operand A of buffers 0 and 1, then operand B of buffers 0 and 1
  // (every fragment address is one register per k-step and operand plus an
  // immediate offset)
  const int sdst = cr * 128 + gram_swizzle(cr, cc) * 16;  // rows RSTEP apart share the swizzle
  u32x4 g[2][VPT + VPB];
  // stage P; a chunk past the row's end (and every chunk past the last
  // stage) takes an offset outside the buffer and reads zeros
  auto load = [&](int P, u32x4 (&dst)[VPT + VPB]) {
    const uint32_t so = P * 128 + cc * 16 < rb ? (uint32_t)P * 128u : 0x80000000u;
#pragma unroll
    for (int k = 0; k < VPT; ++k) {
      dst[k] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(zs, offA[k] + so, 0, 0));
      if (k < VPB)
        dst[VPT + k] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(zs, offB[k] + so, 0, 0));
    }
  };
  auto store = [&](int c, const u32x4 (&v)[VPT + VPB]) {
#pragma unroll
    for (int k = 0; k < VPT; ++k) {
      *reinterpret_cast<u32x4*>(lds + c * SLAB + sdst + k * RSTEP * 128) = v[k];
      if (k < VPB) *reinterpret_cast<u32x4*>(lds + 2 * SLAB + c * SLABB + sdst + k * RSTEP * 128) = v[VPT + k];
    }
  };
  const int wj = wave >> 1, wi = wave & 1;  // rows wj*128.., columns wi*128.. of the tile
  f32x16 acc[4][NB];
#pragma unroll
  for (int m = 0; m < 4; ++m)
#pragma unroll
    for (int n = 0; n < NB; ++n)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[m][n][r] = 0.f;
  // fragments of k-step q of a stage: half h holds logical chunk 2q + h.
  // Every row a lane reads (wj*128 + m*32 + col) has the swizzle of col.
  const int sw = (col >> 1) & 7;
  uint32_t fqa[4], fqb[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    fqa[q] = (wj * 128 + col) * 128 + ((2 * q + half) ^ sw) * 16;
    fqb[q] = 2 * SLAB + (wi * (TC / 2) + col) * 128 + ((2 * q + half) ^ sw) * 16;
  }
  auto frag = [&](int c, int q, u32x4 (&fa)[4][1], u32x4 (&fb)[NB][1]) {
#pragma unroll
    for (int m = 0; m < 4; ++m) fa[m][0] = *reinterpret_cast<const u32x4*>(lds + fqa[q] + c * SLAB + m * 32 * 128);
#pragma unroll
    for (int n = 0; n < NB; ++n) fb[n][0] = *reinterpret_cast<const u32x4*>(lds + fqb[q] + c * SLABB + n * 32 * 128);
  };
  auto mfma16 = [&](const u32x4 (&fa)[4][1], const u32x4 (&fb)[NB][1]) {
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
      for (int n = 0; n < NB; ++n) acc[m][n] = mfma_frag(fa[m], fb[n], acc[m][n], BF16{});
  };
  // an MFMA group of `n` multiplies, each followed by `r` LDS reads, `w` LDS
  // writes and `l` global loads (the compiler's scheduler fills the groups
  // in this order)
  auto interleave = [](auto n, auto r, auto w, auto l) {
#pragma unroll
    for (int u = 0; u < decltype(n)::value; ++u) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      if (decltype(r)::value) __builtin_amdgcn_sched_group_barrier(0x100, decltype(r)::value, 0);
      if (decltype(w)::value) __builtin_amdgcn_sched_group_barrier(0x200, decltype(w)::value, 0);
      if (decltype(l)::value) __builtin_amdgcn_sched_group_barrier(0x020, decltype(l)::value, 0);
    }
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  using I3 = std::integral_constant<int, 3>;
  using I5 = std::integral_constant<int, 5>;
  using I7 = std::integral_constant<int, 7>;
  using I8 = std::integral_constant<int, 8>;
  using I9 = std::integral_constant<int, 9>;
  // stage P sits in register stage P % 2 and LDS buffer P % 2
  load(0, g[0]);
  __builtin_amdgcn_sched_barrier(0);
  load(1, g[1]);
  __builtin_amdgcn_sched_barrier(0);
  store(0, g[0]);
  load(2, g[0]);
  __syncthreads();
  u32x4 fa0[4][1], fb0[NB][1], fa1[4][1], fb1[NB][1];
  frag(0, 0, fa0, fb0);
  const int n_iter = (n_stages + 1) / 2;
  for (int it = 0; it < n_iter; ++it) {
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const int P = 2 * it + c;
      // first half: k-steps 0 and 1; stage P + 1 to LDS, stage P + 3 loaded
      __builtin_amdgcn_sched_barrier(0);
      frag(c, 1, fa1, fb1);
      mfma16(fa0, fb0);
      store(1 - c, g[1 - c]);
      load(P + 3, g[1 - c]);
      frag(c, 2, fa0, fb0);
      mfma16(fa1, fb1);
      if constexpr (NB == 4) {
        interleave(I8{}, I1{}, I0{}, I0{});
        interleave(I8{}, I0{}, I1{}, I1{});  // the stores spread over 16 multiplies (8 cost 2% more)
        interleave(I8{}, I0{}, I1{}, I1{});
        interleave(I8{}, I1{}, I0{}, I0{});
      } else {
        interleave(I7{}, I1{}, I0{}, I0{});
        interleave(I5{}, I0{}, I1{}, I1{});
        interleave(I9{}, I0{}, I1{}, I1{});
        interleave(I3{}, I3{}, I0{}, I0{});
      }
      __syncthreads();
      // second half: k-steps 2 and 3; stage P + 1's first fragments
      __builtin_amdgcn_sched_barrier(0);
      frag(c, 3, fa1, fb1);
      mfma16(fa0, fb0);
      frag(1 - c, 0, fa0, fb0);
      mfma16(fa1, fb1);
      if constexpr (NB == 4) {
        interleave(I8{}, I1{}, I0{}, I0{});
        interleave(I8{}, I0{}, I0{}, I0{});
        interleave(I8{}, I1{}, I0{}, I0{});
        interleave(I8{}, I0{}, I0{}, I0{});
      } else {
        interleave(I7{}, I1{}, I0{}, I0{});
        interleave(I5{}, I0{}, I0{}, I0{});
        interleave(I7{}, I1{}, I0{}, I0{});
        interleave(I5{}, I0{}, I0{}, I0{});
      }
      __syncthreads();
    }
  }
  if constexpr (MODE == kGramMax) {  // (the loop ended on a barrier)
    gram_max_store<MODE, T, TC, 4, NB>(a, acc, izr, nullptr, reinterpret_cast<float*>(lds), b, ti, wj, wi);
    return;
  }
  if constexpr (MODE != kGramMax) {
  // register r of block (m, n) is row wj*128 + m*32 + mfma_row(r), column
  // wi*128 + n*32 + col of the tile
  const int n_tok = MODE == kGramRest ? a.n_cols : N;  // rows and columns of G
  if (tj == ti) {  // the diagonal tile holds ||z_i||^2
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
      for (int n = 0; n < 4; ++n)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int jl = wj * 128 + m * 32 + mfma_row(r, half), il = wi * 128 + n * 32 + col;
          const int i = ti * T + il;
          if (jl == il && i < n_tok)
            a.inv_norm[(size_t)b * N + (MODE == kGramRest ? a.cols[(size_t)b * n_tok + i] : i)] = 1.f / fmaxf(sqrtf(fmaxf(acc[m][n][r], 0.f)), 1e-12f);
        }
  }
  // The tile leaves through LDS, 32 rows j at a time, and is stored as
  // 16-byte runs of whole rows (each lane storing 4 bytes, or 16-byte runs
  // of a few bytes per row, writes G at a fraction of the rate): tA holds
  // the pass as rows j (stride TA: 16-byte aligned rows, the two half-waves'
  // writes on disjoint banks) for G[j, i]; off the diagonal tB holds it as
  // rows i (odd stride TB: the column writes spread over the banks) for the
  // mirrored G[i, j].  Whole tiles of a matrix whose rows are a multiple of
  // 16 bytes store without bounds checks.
  float* tA = reinterpret_cast<float*>(lds);
  float* tB = tA + PR * TA;
  const int ld = a.ldg;
  float* gbm = a.G + (size_t)b * n_tok * ld;
  const bool mirror = tj != ti;
  const bool fast = (ti + 1) * T <= n_tok && (ld & 3) == 0;  // tj <= ti
#pragma unroll
  for (int p = 0; p < T / PR; ++p) {  // unrolled: the accumulator block m is a constant
    __syncthreads();  // the operand slabs, or the previous pass, are no longer read
    if (wj == p / 4) {
      const int m = p % 4;
#pragma unroll
      for (int n = 0; n < 4; ++n)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int jl = mfma_row(r, half), il = wi * 128 + n * 32 + col;
          tA[jl * TA + il] = acc[m][n][r];
          if (mirror) tB[il * TB + jl] = acc[m][n][r];
        }
    }
    __syncthreads();
    // G[j, i]: PR rows of T / 4 runs
#pragma unroll
    for (int k = 0; k < PR * T / 4 / kGram256Threads; ++k) {
      const int e = tid + k * kGram256Threads, row = e / (T / 4), q = e % (T / 4);
      const int j = tj * T + PR * p + row, i = ti * T + 4 * q;
      const u32x4 v = *reinterpret_cast<const u32x4*>(&tA[row * TA + 4 * q]);
      if (fast) {
        stg16_stream(&gbm[(size_t)j * ld + i], v);
      } else {
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (j < n_tok && i + u < n_tok)
            __builtin_nontemporal_store(__uint_as_float(v[u]), &gbm[(size_t)j * ld + i + u]);
      }
    }
    if (mirror) {  // G[i, j]: T rows of PR / 4 runs
#pragma unroll
      for (int k = 0; k < PR * T / 4 / kGram256Threads; ++k) {
        const int e = tid + k * kGram256Threads, il = e / (PR / 4), q = e % (PR / 4);
        const int i = ti * T + il, j = tj * T + PR * p + 4 * q;
        const float* srcp = &tB[il * TB + 4 * q];
        const u32x4 v = {__float_as_uint(srcp[0]), __float_as_uint(srcp[1]), __float_as_uint(srcp[2]),
                         __float_as_uint(srcp[3])};
        if (fast) {
          stg16_stream(&gbm[(size_t)i * ld + j], v);
        } else {
#pragma unroll
          for (int u = 0; u < 4; ++u)
            if (i < n_tok && j + u < n_tok)
              __builtin_nontemporal_store(__uint_as_float(v[u]), &gbm[(size_t)i * ld + j + u]);
        }
      }
    }
  }
  }
}

// ---------------------------------------------------------------------------
// Inverse norms of listed bf16 tokens, from the diagonal of their products with
// themselves in the k order of the Gram matrix, so that a round's distances are
// those of the Gram matrix.  One wave per 32 tokens, operands straight from
// memory; a ring of slabs keeps 48 loads in flight (with 16 issued and awaited
// together, 480 of 2,880 tokens x 16 took 30 us instead of 15).  fp32 pivots keep
// the norms of the relevance pass, which are sums in fp32 as well (near-ties can
// swap against those of the full matrix): the multiplies alone would take 55 us
// here.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(64) void gram_norms_kernel(GramArgs a) {
  const int lane = threadIdx.x, half = lane >> 5, col = lane & 31;
  const int b = blockIdx.y, rb = a.row_bytes;
  const int tok = a.rows[(size_t)b * a.n_rows + min((int)blockIdx.x * 32 + col, a.n_rows - 1)];
  const uint8_t* src = reinterpret_cast<const uint8_t*>(a.Z) + ((size_t)b * a.N + tok) * rb;
  const int c0 = a.natural ? half : 4 * half, cs = a.natural ? 2 : 1;
  const int n_slabs = (rb + 127) / 128;
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  constexpr int U = 12;
  u32x4 z[U][4];
  auto load = [&](int s, u32x4 (&dst)[4]) {  // chunks past the row's end read its first
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int off = s * 128 + (c0 + cs * q) * 16;
      dst[q] = ldg16(src + (off < rb ? off : 0));
    }
  };
#pragma unroll
  for (int u = 0; u < U; ++u) load(u, z[u]);
  for (int s0 = 0; s0 < n_slabs; s0 += U) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      u32x4 v[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] = (s0 + u) * 128 + (c0 + cs * q) * 16 < rb ? z[u][q] : zero4();
      load(s0 + u + U, z[u]);
      __builtin_amdgcn_sched_barrier(0);
      acc = mfma_frag(v, v, acc, BF16{});
    }
  }
  const float zz = mfma_diag(acc, half, col);
  if (half == 0) a.inv_norm[(size_t)b * a.N + tok] = 1.f / fmaxf(sqrtf(fmaxf(zz, 0.f)), 1e-12f);
}

// ---------------------------------------------------------------- kernels
// One tile per workgroup.
template <class In, int MODE>
__global__ __launch_bounds__(kGramThreads, MODE == kGramNext ? 2 : 1) void gram_kernel(GramArgs a) {
  gram_tile<In, MODE>(a, blockIdx.x);
}
template <int MODE, int TC = 256>
__global__ __launch_bounds__(kGram256Threads, 1) void gram256_kernel(GramArgs a) {
  gram256_tile<MODE, TC>(a, blockIdx.x);
}

// The Gram matrix of the tokens that are no pivots, in the samples that the pool
// rounds left unfinished, most often none: as many workgroups as are resident at
// once walk the tiles (8320 workgroups that only find nothing to do take 104 us,
// these 5 us).
__device__ __forceinline__ bool gram_any_left(const GramArgs& a) {
  bool left = false;
  for (int b = threadIdx.x; b < a.B; b += blockDim.x) left |= !gram_done(a, b);
  return __syncthreads_or(left);
}
template <class In>
__global__ __launch_bounds__(kGramThreads) void gram_rest_kernel(GramArgs a, int n_work) {
  if (!gram_any_left(a)) return;
  for (int w = blockIdx.x; w < n_work; w += gridDim.x) {
    gram_tile<In, kGramRest>(a, w);
    __syncthreads();
  }
}
__global__ __launch_bounds__(kGram256Threads, 1) void gram256_rest_kernel(GramArgs a, int n_work) {
  if (!gram_any_left(a)) return;
  for (int w = blockIdx.x; w < n_work; w += gridDim.x) {
    gram256_tile<kGramRest>(a, w);
    __syncthreads();
  }
}

// ---------------------------------------------------------------- launchers
bool gram256_ok(int dtype, int N, int row_bytes) {
  return dtype == 1 && N >= kGram256MinN && (size_t)(N + 256) * row_bytes < (1u << 31);
}

hipError_t launch_gram_full(const GramArgs& g0, int dtype, hipStream_t s) {
  GramArgs g = g0;
  const bool big = gram256_ok(dtype, g.N, g.row_bytes);  // rows are a multiple of 16 bytes (checked at the boundary)
  const int T = big ? 256 : kGramTile;
  g.n_tiles = (g.N + T - 1) / T;
  const int n_work = gram_grid(gram_tiles(g.n_tiles), g.B);
  if (big)
    hipLaunchKernelGGL(gram256_kernel<kGramFull>, dim3(n_work), dim3(kGram256Threads), 0, s, g);
  else if (dtype == 1)
    hipLaunchKernelGGL((gram_kernel<BF16, kGramFull>), dim3(n_work), dim3(kGramThreads), 0, s, g);
  else
    hipLaunchKernelGGL((gram_kernel<F32, kGramFull>), dim3(n_work), dim3(kGramThreads), 0, s, g);
  return hipGetLastError();
}

hipError_t launch_gram_rest(const GramArgs& g0, int dtype, hipStream_t s) {
  GramArgs g = g0;
  const bool big = gram256_ok(dtype, g.N, g.row_bytes);  // the tiles, and so the k order, of the full matrix
  const int T = big ? 256 : kGramTile;
  g.natural = false;
  g.n_tiles = (g.n_cols + T - 1) / T;
  const int n_work = gram_grid(gram_tiles(g.n_tiles), g.B);
  const dim3 grid(std::min(n_work, big ? 256 : 512));
  if (big)
    hipLaunchKernelGGL(gram256_rest_kernel, grid, dim3(kGram256Threads), 0, s, g, n_work);
  else if (dtype == 1)
    hipLaunchKernelGGL(gram_rest_kernel<BF16>, grid, dim3(kGramThreads), 0, s, g, n_work);
  else
    hipLaunchKernelGGL(gram_rest_kernel<F32>, grid, dim3(kGramThreads), 0, s, g, n_work);
  return hipGetLastError();
}

hipError_t launch_gram_norms(const GramArgs& g0, hipStream_t s) {
  GramArgs g = g0;
  g.natural = gram256_ok(1, g.N, g.row_bytes);
  hipLaunchKernelGGL(gram_norms_kernel, dim3((g.n_rows + 31) / 32, g.B), dim3(64), 0, s, g);
  return hipGetLastError();
}

hipError_t launch_gram_pool(const GramArgs& g0, int dtype, hipStream_t s) {
  GramArgs g = g0;
  g.natural = gram256_ok(dtype, g.N, g.row_bytes);
  g.n_tiles = (g.n_rows + kGramTile - 1) / kGramTile;
  const dim3 grid(gram_grid(gram_tiles(g.n_tiles), g.B));
  if (dtype == 1)
    hipLaunchKernelGGL((gram_kernel<BF16, kGramPool>), grid, dim3(kGramThreads), 0, s, g);
  else
    hipLaunchKernelGGL((gram_kernel<F32, kGramPool>), grid, dim3(kGramThreads), 0, s, g);
  return hipGetLastError();
}

hipError_t launch_gram_max(const GramArgs& g0, int tile, int ctile, int dtype, hipStream_t s) {
  GramArgs g = g0;
  g.natural = gram256_ok(dtype, g.N, g.row_bytes);
  g.n_rtiles = (g.n_rows + tile - 1) / tile;
  g.n_ctiles = (g.n_cols + ctile - 1) / ctile;
  const dim3 grid(gram_grid(g.n_rtiles * g.n_ctiles, g.B));
  if (ctile == 192)
    hipLaunchKernelGGL((gram256_kernel<kGramMax, 192>), grid, dim3(kGram256Threads), 0, s, g);
  else if (tile == 256)
    hipLaunchKernelGGL(gram256_kernel<kGramMax>, grid, dim3(kGram256Threads), 0, s, g);
  else if (dtype == 1)
    hipLaunchKernelGGL((gram_kernel<BF16, kGramMax>), grid, dim3(kGramThreads), 0, s, g);
  else
    hipLaunchKernelGGL((gram_kernel<F32, kGramMax>), grid, dim3(kGramThreads), 0, s, g);
  return hipGetLastError();
}

hipError_t launch_gram_next(const GramArgs& g0, int dtype, hipStream_t s) {
  GramArgs g = g0;
  g.natural = gram256_ok(dtype, g.N, g.row_bytes);
  g.n_rtiles = (g.n_rows + kGramTile - 1) / kGramTile;
  g.n_ctiles = (g.n_cols + kGramTile - 1) / kGramTile;
  const dim3 grid(gram_grid(g.n_rtiles * g.n_ctiles, g.B));
  if (dtype == 1)
    hipLaunchKernelGGL((gram_kernel<BF16, kGramNext>), grid, dim3(kGramThreads), 0, s, g);
  else
    hipLaunchKernelGGL((gram_kernel<F32, kGramNext>), grid, dim3(kGramThreads), 0, s, g);
  return hipGetLastError();
}

}  // namespace trevs
