// Sketch update (Alg. 1, Sec. 3.2 and 4.1) of small sketches and small
// windows: the kernels that take a window through few launches. A launch of
// a single job takes it by value, with no table to copy to the device.
//
// linear   The binned update (see update.hip) for sketches of at most
//          LIN_TILES tiles. A batch of pairs sorted by tile in LDS leaves a
//          run per tile of a hundred bytes and more, long enough to be read
//          on its own, so a batch's words are written one after another
//          where the batch has its place (no claims, no regions, so no
//          count pass to size them), with the runs' starts in a directory
//          row. The apply then walks the directory's column of its tile.
//          Tiles are cut small enough (160 KiB >> tshift) to be about one
//          per compute unit. Against the region passes, update kernels of a
//          1M-pair window on the default sketch: 76 us in 8 launches and a
//          copy -> 35 us in 2; 9M pairs at k = 15: 150 -> 113 us. Windows
//          that would leave few workgroups with long tiles stay with the
//          regions (takes_linear, in api.hip).
// fresh    A window too small to sort: one workgroup per tile of a sketch
//          that is all zero builds its tile in LDS from every pair of the
//          window, and writes it with its LEs' zero counts. It takes the
//          place of a zero fill, a scattered update and a scan of the
//          sketch for zero counts: 3000 pairs on the default sketch, 25 us
//          in 3 kernels -> 14 us in 2 (with the scan of the zero counts).
//          Each pair costs every tile a visit (0.35 us per 1000 pairs at
//          256 tiles): linear is as fast from about 32,000 pairs on.
// direct   Alg. 1 as written. Each lane loads one 8-byte pair, hashes it in
//          registers (two multiply-add-shifts, r-1 bit fields) and sets one
//          bit in one LE of each row with a non-returning atomicOr, after a
//          plain load shows the bit unset (Alg. 1 skips a bit already 1;
//          that turns the heavy hitters' updates, whose LEs fill early, into
//          cache reads). Bound by random accesses into the sketch: about
//          15 G atomicOr/s. For a few thousand pairs on a written sketch.
#include "update_dev.h"

namespace ddhf {

constexpr uint32_t LIN_THREADS = 1024;

// The launch's jobs: one by value (no table to copy to the device first), or
// a table in device memory.
template <bool ONE, typename Find>
__device__ __forceinline__ const UpdJob &job_of(const JobArg &A, Find find) {
  if constexpr (ONE) return A.one;
  else return A.tab[find(A.tab, A.nj)];
}

// The tile of workgroup gt of a tile pass. Workgroups go to the 8 XCDs in
// turn (see BIN_GROUPS) and neighbouring tiles' runs of a batch share cache
// lines, so each XCD takes a block of consecutive tiles. A job has
// tile_groups(nbins) workgroups, a multiple of 8 (tile0 is one too); a
// workgroup without a tile gets nbins or more.
__device__ __forceinline__ uint32_t tile_of(const UpdJob &J, uint32_t gt) {
  const uint32_t i = gt - J.tile0, per = (J.nbins + BIN_GROUPS - 1) / BIN_GROUPS;
  const uint32_t t = i % BIN_GROUPS * per + i / BIN_GROUPS;
  return t;
}

// The finished LDS tile to the sketch words [w0, w0 + tw), and its LEs' zero
// counts (a tile holds whole LEs when they are kept).
__device__ __forceinline__ void tile_out(const UpdJob &J, const uint32_t *tile, size_t w0,
                                         uint32_t tw) {
  const uint4 *tile4 = reinterpret_cast<const uint4 *>(tile);
  GMEM uint4 *d4 = reinterpret_cast<GMEM uint4 *>(gmem(J.sk) + w0);
  GMEM uint32_t *lez = gmem(J.lez);
  for (uint32_t q = threadIdx.x; q < tw / 4; q += LIN_THREADS) {
    const uint4 v = tile4[q];
    st4(d4 + q, v);
    if (lez) le_zeros(J.G, lez, w0 + 4 * (size_t)q, v);
  }
}

// ----------------------------------------------------------------- scatter

// Each block takes J.chunk consecutive batches of 1024 * PPT pairs. Per
// batch: the codes' ranks inside their tile's run (LDS atomics), the runs'
// starts by one wave's scan over the tiles, the codes grouped by tile in
// LDS, and the words (three codes each, runs padded to whole words as in
// update.hip) written in order. Three barriers: a tile's count is cleared
// by the scan that reads it, and the next batch's first LDS write to the
// sorted codes follows a barrier that every wave reaches after its last
// read of them.
template <int R, int PPT>
struct LinLds {
  uint32_t cnt[LIN_TILES], lofs[LIN_TILES], n_words;
  Filter<lin_filters(PPT) ? LIN_FILT_WORDS : 32> filt;
  uint32_t sorted[LIN_THREADS * PPT * R + 2 * LIN_TILES];
};

template <int R, int PPT, bool ONE>
__global__ __launch_bounds__(LIN_THREADS) void k_lin_scatter(JobArg A) {
  constexpr uint32_t BATCH = LIN_THREADS * PPT;
  constexpr bool FILT = lin_filters(PPT);
  static_assert(sizeof(LinLds<R, PPT>) <= 163840, "the LDS of a workgroup");
  __shared__ LinLds<R, PPT> L;
  uint32_t *const cnt = L.cnt, *const lofs = L.lofs, *const sorted = L.sorted;
  auto &filt = L.filt;
  uint32_t &n_words = L.n_words;
  const UpdJob &J = job_of<ONE>(
      A, [](const UpdJob *t, uint32_t n) { return job_of_block(t, n, blockIdx.x); });
  const Geom G = J.G;
  const uint32_t ts = J.tshift, lb = blockIdx.x - J.blk0;
  const GMEM uint2 *__restrict__ pairs = gmem(J.pairs);
  GMEM uint2 *__restrict__ words = gmem(reinterpret_cast<uint2 *>(J.codes));
  GMEM uint16_t *__restrict__ dir = gmem(J.dir);
  const uint32_t n = (uint32_t)J.n;                     // a round's pairs: at most 2^28
  const uint32_t wcap = J.wcap;
  if (threadIdx.x < LIN_TILES) cnt[threadIdx.x] = 0;
  if constexpr (FILT) filt.clear(G);
  __syncthreads();
  uint32_t b = lb * (uint32_t)J.chunk;
  const uint32_t b1 = b + (uint32_t)J.chunk < J.nbatch ? b + (uint32_t)J.chunk : J.nbatch;
  if (b >= b1) return;                                  // uniform over the block
  uint2 pr[PPT];
  // loads past the window's end re-read its last pair (masked later)
  auto load = [&](uint32_t bb) {
    uint32_t tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
#pragma unroll
    for (int k = 0; k < PPT; k++) {
      const uint32_t i = bb * BATCH + (uint32_t)k * LIN_THREADS + tid;
      pr[k] = ld2(pairs + min(i, n - 1));
    }
  };
  load(b);
  const uint32_t b0 = b;
  bool filtering = FILT && filt.fits(G);               // uniform over the block
  for (; b < b1; b++) {
    uint32_t tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    uint32_t x[PPT], B0[PPT], live = (1u << PPT) - 1;
#pragma unroll
    for (int k = 0; k < PPT; k++) {
      x[k] = pr[k].x;
      B0[k] = pair_code0(G, pr[k]);
    }
    load(b + 1 < b1 ? b + 1 : b);
    if ((b + 1) * BATCH > n) {                          // the window's last batch
#pragma unroll
      for (int k = 0; k < PPT; k++)
        if (b * BATCH + (uint32_t)k * LIN_THREADS + tid >= n) live &= ~(1u << k);
    } else if (FILT && filtering) {
      live &= ~filt.template repeats<PPT>(G, x, B0, b - b0);
    }
    // ranks are < BATCH * R <= 2^15: two per register (a dropped pair's codes
    // are not used, and leave its halves zero)
    uint32_t v[PPT * R], rk2[(PPT * R + 1) / 2] = {};
    rank_codes<R, PPT, true>(G, x, B0, live, ts, cnt, v, rk2);   // in tiles of 160 KiB >> ts
    __syncthreads();
    if (tid < 64) {
      constexpr uint32_t TPL = LIN_TILES / 64;          // tiles per lane
      uint32_t c[TPL], sum = 0;
#pragma unroll
      for (uint32_t u = 0; u < TPL; u++) {
        c[u] = cnt[tid * TPL + u];
        cnt[tid * TPL + u] = 0;
        sum += 3 * ((c[u] + 2) / 3);
      }
      const uint32_t incl = wave_scan_incl(sum);
      uint32_t ex = incl - sum;
      GMEM uint16_t *row = dir + (size_t)b * LIN_DIR;
#pragma unroll
      for (uint32_t u = 0; u < TPL; u++) {
        const uint32_t t = tid * TPL + u, padded = 3 * ((c[u] + 2) / 3);
        lofs[t] = ex;
        row[t] = (uint16_t)(ex / 3);
        if (padded > c[u]) sorted[ex + c[u]] = ~0u;     // at most two pad slots
        if (padded > c[u] + 1) sorted[ex + c[u] + 1] = ~0u;
        ex += padded;
      }
      if (tid == 63) {
        row[LIN_TILES] = (uint16_t)(incl / 3);
        n_words = incl / 3;
      }
    }
    __syncthreads();
    group_codes<R, PPT, true>(live, v, rk2, lofs, sorted);
    __syncthreads();
    if constexpr (FILT) {
      if (b - b0 == FILT_CLAIM) filtering = filt.useful(BATCH);
    }
    const uint32_t nw = n_words;
    GMEM uint2 *out = words + (size_t)b * wcap;
    for (uint32_t j = tid; j < nw; j += LIN_THREADS) {
      // the word's first slot always holds a code and stands in for a pad
      const uint32_t x = sorted[3 * j], y0 = sorted[3 * j + 1], z0 = sorted[3 * j + 2];
      const uint32_t y = y0 == ~0u ? x : y0, z = z0 == ~0u ? x : z0;
      st2(out + j, code_word(x, y, z));
    }
  }
}

// ------------------------------------------------------------------- apply

// One workgroup per tile: its words of every batch into the tile in LDS.
// Wave w takes batches w, w + 16, ...: it reads 64 directory entries at once
// and walks their runs in segments of up to 64 words, one 8-byte load per
// lane, with LIN_DEPTH segments' loads in flight: a segment's slot is loaded
// again as soon as its words are set. Bound by the loads' latency and, past
// that, by the busiest source's tiles. 15M pairs at k = 16 (200 MB of
// words): four runs loaded and set in turn 178 us, eight in flight 139 us
// (16: no faster), and 79 us with the scatter's repeat filter.
constexpr int LIN_DEPTH = 8;

template <bool ONE>
__global__ __launch_bounds__(LIN_THREADS) void k_lin_apply(JobArg A, uint32_t tiles) {
  extern __shared__ __attribute__((aligned(16))) uint32_t ltile[];
  constexpr uint32_t WAVES = LIN_THREADS / 64;
  for (uint32_t gt = blockIdx.x; gt < tiles; gt += gridDim.x) {
    const UpdJob &J =
        job_of<ONE>(A, [gt](const UpdJob *t, uint32_t n) { return job_of_tile(t, n, gt); });
    const uint32_t t = tile_of(J, gt), TW = BIN_TILE_WORDS >> J.tshift;
    if (t >= J.nbins) continue;                         // uniform over the block
    const size_t w0 = (size_t)t * TW;
    const uint32_t tw = (uint32_t)(J.words - w0 < TW ? J.words - w0 : TW);
    uint4 *tile4 = reinterpret_cast<uint4 *>(ltile);
    if (J.fresh) {
      for (uint32_t q = threadIdx.x; q < tw / 4; q += LIN_THREADS)
        tile4[q] = make_uint4(0, 0, 0, 0);
    } else {
      const GMEM uint4 *src = reinterpret_cast<const GMEM uint4 *>(gmem(J.sk) + w0);
      for (uint32_t q = threadIdx.x; q < tw / 4; q += LIN_THREADS) tile4[q] = ld4(src + q);
    }
    __syncthreads();
    const GMEM uint2 *__restrict__ codes = gmem(reinterpret_cast<const uint2 *>(J.codes));
    const GMEM uint16_t *__restrict__ dir = gmem(J.dir);
    // wave-uniform, so that the walk over the runs is scalar work
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t wcap = J.wcap, nb = J.nbatch, ts = J.tshift;
    const uint32_t runs = nb > wv ? (nb - wv + WAVES - 1) / WAVES : 0;   // this wave's
    for (uint32_t i0 = 0; i0 < runs; i0 += 64) {
      uint32_t start = 0, len = 0;                      // run i0 + lane of the wave
      if (i0 + lane < runs) {
        const uint32_t run = (i0 + lane) * WAVES + wv;
        const GMEM uint16_t *row = dir + (size_t)run * LIN_DIR + t;
        const uint32_t d0 = row[0];
        start = run * wcap + d0;
        len = row[1] - d0;
      }
      const uint32_t m = runs - i0 < 64 ? runs - i0 : 64;
      // the next segment: words [s, s + l) of run i; l is 0 past the last run
      uint32_t i = 0, s = wave_lane(start, 0), l = wave_lane(len, 0);
      uint32_t n[LIN_DEPTH];
      uint2 x[LIN_DEPTH];
      auto fetch = [&](int u) {
        while (l == 0 && i + 1 < m) {
          i++;
          s = wave_lane(start, (int)i);
          l = wave_lane(len, (int)i);
        }
        n[u] = l < 64 ? l : 64;
        // lanes past the segment re-read its last word (or, past the last
        // segment, the word after it, which the directory follows)
        const GMEM uint2 *p = codes + s;
        const uint32_t at = n[u] ? n[u] - 1 : 0;
        x[u] = ld2(p + (lane < at ? lane : at));
        s += n[u];
        l -= n[u];
      };
#pragma unroll
      for (int u = 0; u < LIN_DEPTH; u++) fetch(u);
      while (n[0]) {
#pragma unroll
        for (int u = 0; u < LIN_DEPTH; u++) {
          if (lane < n[u]) or_word(ltile, x[u], ts);
          fetch(u);
        }
      }
    }
    __syncthreads();
    tile_out(J, ltile, w0, tw);
    __syncthreads();
  }
}

// ------------------------------------------------------------------- fresh

// One workgroup per tile of an all-zero sketch: every pair of the window is
// hashed, and its bits that fall into the tile are set. A tile lies in one
// row or in few (rows lo..hi).
template <bool ONE>
__global__ __launch_bounds__(LIN_THREADS) void k_update_fresh(JobArg A) {
  extern __shared__ __attribute__((aligned(16))) uint32_t ftile[];
  const UpdJob &J = job_of<ONE>(
      A, [](const UpdJob *t, uint32_t n) { return job_of_tile(t, n, blockIdx.x); });
  const Geom &G = J.G;
  const uint32_t t = tile_of(J, blockIdx.x), TW = BIN_TILE_WORDS >> J.tshift;
  if (t >= J.nbins) return;                             // uniform over the block
  const size_t w0 = (size_t)t * TW;
  const uint32_t tw = (uint32_t)(J.words - w0 < TW ? J.words - w0 : TW);
  uint4 *tile4 = reinterpret_cast<uint4 *>(ftile);
  for (uint32_t q = threadIdx.x; q < tw / 4; q += LIN_THREADS) tile4[q] = make_uint4(0, 0, 0, 0);
  __syncthreads();
  const uint32_t bit0 = (uint32_t)w0 * 32, bits = tw * 32;
  const uint32_t lo = bit0 >> (G.k + G.log2g), hi = (bit0 + bits - 1) >> (G.k + G.log2g);
  // LEs the tile touches (it holds whole LEs unless an LE is larger)
  const uint32_t le0 = bit0 >> G.log2g, nle = ((bit0 + bits - 1) >> G.log2g) - le0;
  const GMEM uint2 *__restrict__ pairs = gmem(J.pairs);
  const uint32_t n = (uint32_t)J.n;
  constexpr int U = 4;
  for (uint32_t i0 = threadIdx.x; i0 < n; i0 += LIN_THREADS * U) {
    uint2 p[U];
#pragma unroll
    for (int u = 0; u < U; u++) {
      const uint32_t i = i0 + u * LIN_THREADS;
      p[u] = ld2(pairs + (i < n ? i : n - 1));          // past the end: the last pair again
    }
#pragma unroll
    for (int u = 0; u < U; u++) {
      const uint32_t c0 = hash_dh0(G, p[u].x);
      for (uint32_t row = lo; row <= hi; row++) {
        const uint32_t cell = row == 0 ? c0 : (bit_block(G, row, p[u].x) ^ c0);
        const uint32_t le = (row << G.k) | cell;
        if (le - le0 <= nle) {
          const uint32_t B = ((le << G.log2g) | hash_h1(G, p[u].y)) - bit0;
          if (B < bits) atomicOr(&ftile[B >> 5], 1u << (B & 31));
        }
      }
    }
  }
  __syncthreads();
  tile_out(J, ftile, w0, tw);
}

// ------------------------------------------------------------------- direct

template <int R, bool CHECK, bool ONE>
__global__ __launch_bounds__(256) void k_update(JobArg A) {
  const UpdJob &J = job_of<ONE>(
      A, [](const UpdJob *t, uint32_t n) { return job_of_block(t, n, blockIdx.x); });
  const Geom G = J.G;
  GMEM uint32_t *__restrict__ sk = gmem(J.sk);
  const GMEM uint2 *__restrict__ pairs = gmem(J.pairs);
  const size_t n = J.n;
  const size_t stride = (size_t)J.nblk * blockDim.x;
  for (size_t i = (size_t)(blockIdx.x - J.blk0) * blockDim.x + threadIdx.x; i < n; i += stride) {
    const uint2 p = ld2(pairs + i);
    const uint32_t bit = hash_h1(G, p.y);
    const uint32_t c0 = hash_dh0(G, p.x);
    const uint32_t mask = 1u << (bit & 31);
    const uint32_t wofs = bit >> 5;
#pragma unroll
    for (int row = 0; row < R; row++) {
      const uint32_t cell = row == 0 ? c0 : (bit_block(G, row, p.x) ^ c0);
      GMEM uint32_t *w = sk + ((size_t)(((uint32_t)row << G.k) | cell) * G.wpl + wofs);
      if (CHECK && (*w & mask)) continue;
      atomicOr((uint32_t *)w, mask);    // stays a global atomic after inlining
    }
  }
}

// ------------------------------------------------------------------- launch

namespace {

struct Launch {
  JobArg A;
  uint32_t blocks = 0, tiles = 0, tw = 0;
};

// tw: words of the launch's largest tile (its dynamic LDS)
Launch make_launch(const UpdJob *h, const UpdJob *d, uint32_t nj) {
  Launch L;
  L.A.one = h[0];
  L.A.tab = d;
  L.A.nj = nj;
  for (uint32_t j = 0; j < nj; j++) {
    L.blocks += h[j].nblk;
    L.tiles += tile_groups(h[j].nbins);
    const uint32_t w = BIN_TILE_WORDS >> h[j].tshift;
    L.tw = w > L.tw ? w : L.tw;
  }
  return L;
}

template <int R, bool ONE>
void launch_scatter(const Launch &L, uint32_t ppt, hipStream_t st) {
  constexpr int P4 = R <= 7 ? 4 : 2, P6 = R <= 5 ? 6 : P4;
  if (ppt == 1) k_lin_scatter<R, 1, ONE><<<L.blocks, LIN_THREADS, 0, st>>>(L.A);
  else if (ppt == 2) k_lin_scatter<R, 2, ONE><<<L.blocks, LIN_THREADS, 0, st>>>(L.A);
  else if (ppt == 6) k_lin_scatter<R, P6, ONE><<<L.blocks, LIN_THREADS, 0, st>>>(L.A);
  else k_lin_scatter<R, P4, ONE><<<L.blocks, LIN_THREADS, 0, st>>>(L.A);
}

template <int R, bool ONE>
void launch_direct(const Launch &L, bool check, hipStream_t st) {
  if (check) k_update<R, true, ONE><<<L.blocks, 256, 0, st>>>(L.A);
  else k_update<R, false, ONE><<<L.blocks, 256, 0, st>>>(L.A);
}

template <int R, bool ONE>
hipError_t launch_small(const Launch &L, UpdPath path, uint32_t ppt, uint32_t apply_grid,
                        bool check, hipStream_t st) {
  if (path == UPD_DIRECT) {
    launch_direct<R, ONE>(L, check, st);
  } else if (path == UPD_FRESH) {
    k_update_fresh<ONE><<<L.tiles, LIN_THREADS, L.tw * 4, st>>>(L.A);
  } else {
    launch_scatter<R, ONE>(L, ppt, st);
    k_lin_apply<ONE><<<apply_grid ? apply_grid : L.tiles, LIN_THREADS, L.tw * 4, st>>>(L.A,
                                                                                       L.tiles);
  }
  return hipGetLastError();
}

}  // namespace

template <int R>
static hipError_t launch_one_or_many(const Launch &L, UpdPath path, uint32_t ppt,
                                     uint32_t apply_grid, bool check, hipStream_t st) {
  return L.A.nj == 1 ? launch_small<R, true>(L, path, ppt, apply_grid, check, st)
                     : launch_small<R, false>(L, path, ppt, apply_grid, check, st);
}

hipError_t launch_small_update(const UpdJob *h, const UpdJob *d, uint32_t nj, UpdPath path,
                               uint32_t r, uint32_t ppt, uint32_t apply_grid, hipStream_t st) {
  const Launch L = make_launch(h, d, nj);
  const bool check = h[0].check != 0;
  switch (r) {
    case 3: return launch_one_or_many<3>(L, path, ppt, apply_grid, check, st);
    case 4: return launch_one_or_many<4>(L, path, ppt, apply_grid, check, st);
    case 5: return launch_one_or_many<5>(L, path, ppt, apply_grid, check, st);
    case 6: return launch_one_or_many<6>(L, path, ppt, apply_grid, check, st);
    case 7: return launch_one_or_many<7>(L, path, ppt, apply_grid, check, st);
    case 8: return launch_one_or_many<8>(L, path, ppt, apply_grid, check, st);
    default: return hipErrorInvalidValue;
  }
}

hipError_t prepare_update_kernels() {
  // tiles of up to 160 KiB as dynamic LDS
  const void *fs[] = {reinterpret_cast<const void *>(k_lin_apply<true>),
                      reinterpret_cast<const void *>(k_lin_apply<false>),
                      reinterpret_cast<const void *>(k_update_fresh<true>),
                      reinterpret_cast<const void *>(k_update_fresh<false>)};
  for (const void *f : fs) {
    hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)(BIN_TILE_WORDS * 4));
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace ddhf
