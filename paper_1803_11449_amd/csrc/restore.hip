// Window-end restore (Alg. 2, Sec. 3.3, laid out as in Sec. 4.2).
//
//  1 hot scan      z0 of every LE, from the zero counts the update kept or
//                  counted here in one read of the sketch; ZR(i) per row,
//                  and a bitmap of hot LEs (z0 <= zhot, i.e. z0 < Zmin =
//                  g*exp(-theta/g)).
//  2 HE compaction the hot bitmap into HE(i), ascending, by a block prefix
//                  sum.
//  3 buckets       rows >= 2: HE(i) grouped by its low k-alpha bits, so a
//                  join probe finds exactly the entries whose overlap bits
//                  match instead of testing all of HE(i) (Algs. 3-4 test
//                  every tuple; the bucketed probe enumerates the same
//                  accepted tuples and skips only failing ones).
//                  Small sketches take 1-3 in one launch, one block per row
//                  (k_scan_rows); larger ones in chunks spread over the chip
//                  (k_hot_scan_lez, k_compact, and k_buckets for the join);
//                  without zero counts k_hot_scan, then k_rows.
//  4 scalars       psi (Lemma 1 with the flow-count estimate of Sec. 3.3),
//                  D = g(1 - psi^r) (eq. (4)), T_rep = D*exp(-theta/g) and
//                  the integer report bound floor(T_rep), in float64, by one
//                  thread of the search's first block.
//  5 candidates   the addresses whose r LEs are all hot, by one of three
//                  searches, chosen on the device from the hot-list sizes
//                  by their estimated work:
//                  join     stage 1 (Alg. 3) over HE(0) x HE(1) probing row
//                           2; stages 3..r-1 (Alg. 4) over the partial
//                           addresses probing row i. Each stage appends its
//                           outputs with one atomic per wave; counts are
//                           exact even past a buffer's capacity so the host
//                           can grow it and run again. The last stage keeps
//                           a rebuilt address only if it fits 32 bits and
//                           DH0 of it is the CL_0 it was built from.
//                  lattice  every address of every hot row-0 cell, found as
//                           the points of a lattice in a box (see Lattice),
//                           tested against the hot bitmaps of rows 1..r-1:
//                           eq. (2) read forwards, no partial addresses.
//                  pairs    of those addresses only the ones of a hot row-1
//                           cell, by an index of row 0's hash (k = 14 to 18).
//  6 estimate      per candidate, AND of its r LEs (ULE), SZ = g - popcount,
//                  report iff SZ <= floor(T_rep) (<=> C >= theta),
//                  C = -g*ln(SZ/D) (eq. (4)), +inf when SZ = 0.
//  7 sort          reported records ascending by address, and the state and
//                  the records to pinned host memory: one launch for a short
//                  list.
//
// A restore is a chain of short kernels, and for a small sketch their number
// sets its time. Where the sketch's last restore at the same threshold says
// what this one needs, and the call that launches it also waits for it, only
// that is launched (RestoreBufs::expect, sort_one).
// With the walk, the one-launch scan and sort, the 1M-pair window's restore
// went from 11 launches (47 us of kernels) to 4, and the whole window from
// 125 to 103 us; a 60,000-pair window with a few hundred hot LEs per row
// from 137 to 77 us (81 and 56 with fewer ordering events, see Lane).
#include <math.h>

#include "ddhf_internal.h"

namespace ddhf {

// ------------------------------------------------------------ wave helpers

__device__ __forceinline__ uint32_t lane_id() { return threadIdx.x & 63; }

__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v) { return wave_scan_incl(v); }

// Lanes below this one whose bit is set in mask.
__device__ __forceinline__ uint32_t lanes_below(uint64_t mask) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                   __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// Exclusive prefix sum over a workgroup of NT threads (NT a multiple of 64).
template <int NT>
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t *total,
                                                    uint32_t *sh) {
  constexpr int NW = NT / 64;
  const uint32_t lane = lane_id(), wid = threadIdx.x >> 6;
  const uint32_t inc = wave_incl_scan(v);
  if (lane == 63) sh[wid] = inc;
  __syncthreads();
  if (wid == 0) {
    uint32_t s = lane < NW ? sh[lane] : 0;
    s = wave_incl_scan(s);
    if (lane < NW) sh[lane] = s;
  }
  __syncthreads();
  const uint32_t off = wid ? sh[wid - 1] : 0;
  *total = sh[NW - 1];
  __syncthreads();
  return off + inc - v;
}

// A block's candidates on their way to the global list. Every append to that
// list is an atomic on one address, and those pass at about one in 10 ns
// whatever their number of lanes: a search that made one per wave and test
// spent 1.2 of its 1.35 ms on 115,000 candidates. The first CAP of a block
// are kept in LDS and appended by one atomic when the block ends; the rest
// go out as they come.
template <uint32_t CAP_>
struct CandBufOf {
  static constexpr uint32_t CAP = CAP_;
  uint32_t a[CAP], n;
  unsigned long long base;

  // add and put_global: all lanes of a wave; ok = the lane has an address.
  __device__ __forceinline__ static void put_global(uint32_t ad, bool ok, DevState *st,
                                                    uint32_t *cand, size_t cand_cap) {
    const unsigned long long m = __ballot(ok);
    if (m == 0) return;
    const int first = (int)__builtin_ctzll(m);
    unsigned long long b = 0;
    if (lane_id() == (uint32_t)first)
      b = atomicAdd(&st->n_cand, (unsigned long long)__popcll(m));
    b = wave_lane64(b, first) + lanes_below(m);
    if (ok && b < cand_cap) cand[b] = ad;
  }
  __device__ __forceinline__ void add(uint32_t ad, bool ok, DevState *st, uint32_t *cand,
                                      size_t cand_cap) {
    const unsigned long long m = __ballot(ok);
    if (m == 0) return;
    const int first = (int)__builtin_ctzll(m);
    uint32_t b = 0;
    if (lane_id() == (uint32_t)first) b = atomicAdd(&n, (uint32_t)__popcll(m));
    b = wave_lane(b, first);
    const uint32_t i = b + lanes_below(m);
    if (ok && i < CAP) a[i] = ad;
    if (b + (uint32_t)__popcll(m) > CAP) put_global(ad, ok && i >= CAP, st, cand, cand_cap);
  }
  // The whole block, after its last add.
  __device__ __forceinline__ void flush(DevState *st, uint32_t *cand, size_t cand_cap) {
    __syncthreads();
    const uint32_t k = n < CAP ? n : CAP;
    if (threadIdx.x == 0 && k) base = atomicAdd(&st->n_cand, (unsigned long long)k);
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < k; i += blockDim.x)
      if (base + i < cand_cap) cand[base + i] = a[i];
  }
};

using CandBuf = CandBufOf<512>;

// The most rows a sketch has.
constexpr uint32_t R_MAX = 8;

// How lanes share one LE of WPL words: LPL lanes, each reading VPL uint4.
template <int WPL>
struct LeShape {
  static constexpr int V4 = WPL >= 4 ? WPL / 4 : 0;
  static constexpr int LPL = WPL >= 4 ? (V4 < 64 ? V4 : 64) : 1;
  static constexpr int VPL = WPL >= 4 ? V4 / LPL : 0;
};

// LDS arrays handed to a device function keep their address space (a plain
// pointer would make every access a flat one).
#define LDSP __attribute__((address_space(3)))
template <typename T>
__device__ __forceinline__ LDSP T *lds_ptr(T *p) {
  return (LDSP T *)p;
}

// ----------------------------------------------------------- 0: state init

// The device state and the hot bitmap back to zero, in one launch (before
// k_hot_scan, which adds to both).
__global__ __launch_bounds__(256) void k_restore_init(DevState *st, uint32_t *hotmask,
                                                      size_t n_hm) {
  const size_t i0 = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  if (blockIdx.x == 0) {
    uint32_t *p = reinterpret_cast<uint32_t *>(st);
    for (uint32_t i = threadIdx.x; i < sizeof(DevState) / 4; i += blockDim.x) p[i] = 0;
  }
  for (size_t i = i0; i < n_hm; i += stride) hotmask[i] = 0;
}

// -------------------------------------------------------------- 1: hot scan

// Each block scans a contiguous run of `chunk` LEs; a pass covers
// 256/LPL LEs and HS_UNROLL passes are loaded before any is reduced, so every
// lane keeps several 16-byte loads in flight. ZR(i) is summed in registers
// and folded into LDS only when a lane's run crosses into the next row.
constexpr int HS_UNROLL = 4;

template <int WPL>
__global__ __launch_bounds__(256) void k_hot_scan(Geom G, const uint32_t *__restrict__ sk,
                                                  uint32_t zhot,
                                                  uint32_t *__restrict__ hotmask,
                                                  DevState *__restrict__ st, uint64_t chunk) {
  using S = LeShape<WPL>;
  constexpr uint32_t GROUPS = 256 / S::LPL;
  __shared__ unsigned long long zr_sh[8];
  if (threadIdx.x < 8) zr_sh[threadIdx.x] = 0;
  __syncthreads();
  const uint64_t n_le = (uint64_t)G.r << G.k;
  const uint64_t e_begin = (uint64_t)blockIdx.x * chunk;
  const uint64_t e_end = e_begin + chunk < n_le ? e_begin + chunk : n_le;
  const uint32_t grp = threadIdx.x / S::LPL, sub = threadIdx.x % S::LPL;
  uint32_t cur_row = (uint32_t)(e_begin >> G.k);
  unsigned long long acc = 0;
  for (uint64_t e0 = e_begin; e0 < e_end; e0 += (uint64_t)GROUPS * HS_UNROLL) {
    uint32_t ones[HS_UNROLL];
#pragma unroll
    for (int u = 0; u < HS_UNROLL; u++) {
      const uint64_t e = e0 + (uint64_t)u * GROUPS + grp;
      ones[u] = 0;
      if (e < e_end) {
        if constexpr (WPL >= 4) {
          const uint4 *le = reinterpret_cast<const uint4 *>(sk + e * WPL);
#pragma unroll
          for (int v = 0; v < S::VPL; v++) {
            const uint4 q = le[v * S::LPL + sub];
            ones[u] += __popc(q.x) + __popc(q.y) + __popc(q.z) + __popc(q.w);
          }
        } else {
#pragma unroll
          for (int w = 0; w < WPL; w++) ones[u] += __popc(sk[e * WPL + w]);
        }
      }
    }
    if constexpr (S::LPL > 1) {
#pragma unroll
      for (int u = 0; u < HS_UNROLL; u++)
#pragma unroll
        for (int m = S::LPL / 2; m >= 1; m >>= 1) ones[u] += __shfl_xor(ones[u], m, 64);
    }
    if (sub == 0) {
#pragma unroll
      for (int u = 0; u < HS_UNROLL; u++) {
        const uint64_t e = e0 + (uint64_t)u * GROUPS + grp;
        if (e >= e_end) continue;
        const uint32_t z0 = G.g - ones[u];
        const uint32_t row = (uint32_t)(e >> G.k);
        if (row != cur_row) {
          if (acc) atomicAdd(&zr_sh[cur_row], acc);
          acc = 0;
          cur_row = row;
        }
        acc += z0;
        if (z0 <= zhot) atomicOr(&hotmask[e >> 5], 1u << (e & 31));
      }
    }
  }
  if (sub == 0 && acc) atomicAdd(&zr_sh[cur_row], acc);
  __syncthreads();
  if (threadIdx.x < G.r && zr_sh[threadIdx.x])
    atomicAdd(&st->zr[threadIdx.x], zr_sh[threadIdx.x]);
}

// Zero counts of every LE from the sketch, where the update left none: the
// scans below then read them (4 <= WPL <= 256; other LEs take k_hot_scan).
// One read of the sketch at the HBM's rate; no atomics.
template <int WPL>
__global__ __launch_bounds__(256) void k_zero_counts(Geom G, const uint4 *__restrict__ sk4,
                                                     uint32_t *__restrict__ lez) {
  constexpr int L = WPL / 4;                            // lanes per LE
  constexpr int U = 4;
  const uint64_t n4 = ((uint64_t)G.r << G.k) * L;       // a multiple of 32
  const uint64_t stride = (uint64_t)gridDim.x * 256;
  for (uint64_t q0 = (uint64_t)blockIdx.x * 256 + threadIdx.x; q0 < n4; q0 += stride * U) {
    uint32_t ones[U];
#pragma unroll
    for (int u = 0; u < U; u++) {
      const uint64_t q = q0 + u * stride;
      const uint4 v = sk4[q < n4 ? q : q0];
      ones[u] = __popc(v.x) + __popc(v.y) + __popc(v.z) + __popc(v.w);
    }
#pragma unroll
    for (int u = 0; u < U; u++) {
      const uint64_t q = q0 + u * stride;
#pragma unroll
      for (int m = L / 2; m >= 1; m >>= 1) ones[u] += __shfl_xor(ones[u], m, 64);
      if (q < n4 && q % L == 0) lez[q / L] = G.g - ones[u];
    }
  }
}

// The restore's state as every restore starts it, but for the ZR(i) and
// |HE(i)| of the sketch's rows, which other blocks of the same launch write.
__device__ __forceinline__ void state_begin(const Geom &G, DevState *st) {
  const uint32_t i = threadIdx.x;
  if (i < 8) {
    st->n_out[i] = 0;
    st->seg_max[i] = 0;
    if (i >= G.r) {
      st->zr[i] = 0;
      st->he_count[i] = 0;
    }
  }
  if (i == 0) {
    st->n_cand = st->n_spl = 0;
    st->psi = st->d = st->trep = 0.0;
    st->szmax = st->saturated = st->search = st->pad = 0;
  }
}

// A lane's four LEs (zero counts z) as hot bits in bits 4 (lane mod 8) of the
// word that 8 lanes share: every lane of the 8 gets the word.
__device__ __forceinline__ uint32_t hot_word(uint4 z, uint32_t zhot, uint32_t lane) {
  uint32_t nib = (z.x <= zhot ? 1u : 0u) | (z.y <= zhot ? 2u : 0u) | (z.z <= zhot ? 4u : 0u) |
                 (z.w <= zhot ? 8u : 0u);
  nib <<= 4 * (lane & 7);
  nib |= __shfl_xor(nib, 1, 64);
  nib |= __shfl_xor(nib, 2, 64);
  nib |= __shfl_xor(nib, 4, 64);
  return nib;
}

// Hot scan of larger sketches, from the zero counts (4 bytes per LE). One
// block per SCAN_CHUNK LEs of a row: its words of the hot bitmap, its hot
// LEs' count and its zeros (k_compact adds them up: no atomics, so nothing
// has to be cleared first).
constexpr uint32_t SCAN_CHUNK = 4096;

__global__ __launch_bounds__(256) void k_hot_scan_lez(Geom G, const uint4 *__restrict__ lez4,
                                              uint32_t zhot, uint32_t *__restrict__ hotmask,
                                              uint2 *__restrict__ chunks) {
  __shared__ uint32_t sh_hot[4], sh_z[4];
  constexpr int U = SCAN_CHUNK / 4 / 256;
  const uint32_t lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const size_t q0 = (size_t)blockIdx.x * (SCAN_CHUNK / 4) + threadIdx.x;
  uint4 z[U];
#pragma unroll
  for (int u = 0; u < U; u++) z[u] = lez4[q0 + u * 256];
  uint32_t hot = 0, zeros = 0;                          // zeros of a chunk: at most 2^25
#pragma unroll
  for (int u = 0; u < U; u++) {
    const uint32_t w = hot_word(z[u], zhot, lane);
    if ((lane & 7) == 0) {
      hotmask[(q0 + u * 256) >> 3] = w;
      hot += __popc(w);
    }
    zeros += z[u].x + z[u].y + z[u].z + z[u].w;
  }
  hot = wave_incl_scan(hot);
  zeros = wave_incl_scan(zeros);
  if (lane == 63) {
    sh_hot[wid] = hot;
    sh_z[wid] = zeros;
  }
  __syncthreads();
  if (threadIdx.x == 0)
    chunks[blockIdx.x] = make_uint2(sh_hot[0] + sh_hot[1] + sh_hot[2] + sh_hot[3],
                                    sh_z[0] + sh_z[1] + sh_z[2] + sh_z[3]);
}

// HE(i) of larger sketches, one block per chunk: it starts where the row's
// chunks before it end. One block per row did this in 18 us at k = 18 and 85
// at k = 19, with the rest of the chip idle. A row's first block sums ZR(i).
__global__ __launch_bounds__(256) void k_compact(Geom G, const uint32_t *__restrict__ hotmask,
                                                 const uint2 *__restrict__ chunks,
                                                 uint32_t *__restrict__ he,
                                                 DevState *__restrict__ st) {
  __shared__ unsigned long long sh_z[4];
  __shared__ uint32_t sh_before[4], sh[4];
  const uint32_t per_row = (1u << G.k) / SCAN_CHUNK;
  const uint32_t row = blockIdx.x / per_row, c = blockIdx.x % per_row;
  const uint32_t lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  if (blockIdx.x == 0) state_begin(G, st);
  uint32_t before = 0;
  unsigned long long z = 0;
  const uint32_t upto = c == 0 ? per_row : c;
  for (uint32_t i = threadIdx.x; i < upto; i += 256) {
    const uint2 v = chunks[row * per_row + i];
    if (i < c) before += v.x;
    z += v.y;
  }
  before = wave_incl_scan(before);
  if (c == 0) {
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) z += __shfl_xor(z, m, 64);
  }
  if (lane == 63) {
    sh_before[wid] = before;
    sh_z[wid] = z;
  }
  constexpr uint32_t NW = SCAN_CHUNK / 32;              // words of the chunk: 128
  const uint32_t w0 = blockIdx.x * NW;
  uint32_t m = threadIdx.x < NW ? hotmask[w0 + threadIdx.x] : 0u;
  uint32_t total;
  const uint32_t ex = block_excl_scan<256>(__popc(m), &total, sh);   // holds barriers
  const uint32_t off = sh_before[0] + sh_before[1] + sh_before[2] + sh_before[3];
  uint32_t *out = he + ((size_t)row << G.k) + off + ex;
  while (m) {
    const uint32_t b = __ffs(m) - 1;
    *out++ = ((c * NW + threadIdx.x) << 5) | b;
    m &= m - 1;
  }
  if (threadIdx.x == 0) {
    if (c + 1 == per_row) st->he_count[row] = off + total;
    if (c == 0) st->zr[row] = sh_z[0] + sh_z[1] + sh_z[2] + sh_z[3];
  }
}

// ---------------------------------------------------------- 2: HE compaction

// Per-thread values k_rows keeps in registers: hot-mask words (all of a
// row's when 2^k / 32 <= 8 * 1024, i.e. k <= 18) and HE entries (all when
// |HE(i)| <= 8192). Loaded together, they cost one memory latency instead
// of one per loop trip; larger rows take the loops.
constexpr uint32_t ROW_REG = 8;

__device__ __forceinline__ void compact_row(const Geom &G, uint32_t row,
                                            const uint32_t *__restrict__ hotmask,
                                            uint32_t *__restrict__ he,
                                            DevState *__restrict__ st, uint32_t *sh) {
  const uint32_t nw = (1u << G.k) >> 5;
  const uint32_t *hm = hotmask + (size_t)row * nw;
  const uint32_t per = (nw + blockDim.x - 1) / blockDim.x;
  const uint32_t w0 = min(threadIdx.x * per, nw), w1 = min(w0 + per, nw);
  uint32_t total;
  if (per <= ROW_REG) {                                // uniform: k <= 18
    // the thread's words, loaded together and kept for the write pass
    uint32_t m[ROW_REG], cnt = 0;
#pragma unroll
    for (uint32_t u = 0; u < ROW_REG; u++) {
      m[u] = w0 + u < w1 ? hm[w0 + u] : 0u;
      cnt += __popc(m[u]);
    }
    const uint32_t excl = block_excl_scan<1024>(cnt, &total, sh);
    uint32_t *out = he + ((size_t)row << G.k) + excl;
#pragma unroll
    for (uint32_t u = 0; u < ROW_REG; u++) {
      while (m[u]) {
        const uint32_t b = __ffs(m[u]) - 1;
        *out++ = ((w0 + u) << 5) | b;
        m[u] &= m[u] - 1;
      }
    }
  } else {
    uint32_t cnt = 0;
    for (uint32_t w = w0; w < w1; w++) cnt += __popc(hm[w]);
    const uint32_t excl = block_excl_scan<1024>(cnt, &total, sh);
    uint32_t *out = he + ((size_t)row << G.k) + excl;
    for (uint32_t w = w0; w < w1; w++) {
      uint32_t m = hm[w];
      while (m) {
        const uint32_t b = __ffs(m) - 1;
        *out++ = (w << 5) | b;
        m &= m - 1;
      }
    }
  }
  if (threadIdx.x == 0) st->he_count[row] = total;
}

// --------------------------------------------------------------- 3: buckets



// One block per row i in 2..r-1: HE(i) grouped by its low k-alpha bits
// (the bucket a probe of stage i looks up). Counts and cursors live in LDS
// when the table fits (2^(k-alpha) <= BK_LDS buckets), else in bk_cur.
constexpr uint32_t BK_LDS = 8192;

template <typename CurPtr>
__device__ __forceinline__ void bucket_rows(const Geom &G, uint32_t row, const uint32_t *h,
                                            uint32_t n, uint32_t *off, CurPtr cur,
                                            uint32_t *val, uint32_t *sh) {
  const uint32_t nb = 1u << (G.k - G.alpha), M = nb - 1;
  const uint32_t tid = threadIdx.x, bs = blockDim.x;
  // up to ROW_REG entries per thread are loaded together, before the
  // counters are cleared, and kept for the placing pass
  const bool in_regs = n <= ROW_REG * bs;              // uniform
  uint32_t hv[ROW_REG];
  if (in_regs) {
#pragma unroll
    for (uint32_t u = 0; u < ROW_REG; u++) hv[u] = tid + u * bs < n ? h[tid + u * bs] : 0u;
  }
  for (uint32_t b = tid; b < nb; b += bs) cur[b] = 0;
  __syncthreads();
  if (in_regs) {
#pragma unroll
    for (uint32_t u = 0; u < ROW_REG; u++)
      if (tid + u * bs < n) atomicAdd((uint32_t *)&cur[hv[u] & M], 1u);
  } else {
    for (uint32_t x = tid; x < n; x += bs) atomicAdd((uint32_t *)&cur[h[x] & M], 1u);
  }
  __syncthreads();
  const uint32_t per = (nb + bs - 1) / bs;
  const uint32_t b0 = min(tid * per, nb), b1 = min(b0 + per, nb);
  uint32_t s = 0;
  for (uint32_t b = b0; b < b1; b++) s += cur[b];
  uint32_t total;
  uint32_t run = block_excl_scan<1024>(s, &total, sh);
  for (uint32_t b = b0; b < b1; b++) {
    const uint32_t c = cur[b];
    off[b] = run;
    cur[b] = run;
    run += c;
  }
  if (tid == 0) off[nb] = total;
  __syncthreads();
  if (in_regs) {
#pragma unroll
    for (uint32_t u = 0; u < ROW_REG; u++) {
      if (tid + u * bs < n) {
        const uint32_t pos = atomicAdd((uint32_t *)&cur[hv[u] & M], 1u);
        val[pos] = hv[u];
      }
    }
  } else {
    for (uint32_t x = tid; x < n; x += bs) {
      const uint32_t c = h[x];
      const uint32_t pos = atomicAdd((uint32_t *)&cur[c & M], 1u);
      val[pos] = c;
    }
  }
}

// --------------------------------------------------------------- 4: scalars

// The whole first wave of a block: a lane per row takes its logarithm, and the
// sum runs over the rows in order. One lane alone took 9 us of a search's
// first block, which has its share of the search to do: the first stage of a
// staged join 18 -> 26 us.
__device__ __forceinline__ void scalars(const Geom &G, DevState *st, double e_theta) {
  const uint32_t i = lane_id();
  const double m = (double)G.g * (double)(1ull << G.k);
  const unsigned long long zr = st->zr[i < G.r ? i : 0];
  if (__ballot(zr == 0)) {
    if (i == 0) {
      st->saturated = 1;
      st->psi = 1.0;
      st->d = 0.0;
      st->trep = 0.0;
      st->szmax = 0;
    }
    return;
  }
  const double l = log((double)zr / m);
  double lsum = 0.0;
  for (uint32_t row = 0; row < G.r; row++) lsum += __shfl(l, (int)row, 64);
  if (i != 0) return;
  const double psi = 1.0 - exp(lsum / (double)G.r);
  double pr = 1.0;
  for (uint32_t row = 0; row < G.r; row++) pr *= psi;
  const double d = (double)G.g * (1.0 - pr);
  const double trep = d * e_theta;
  st->psi = psi;
  st->d = d;
  st->trep = trep;
  st->szmax = (uint32_t)floor(trep);
}

// The bucket table of one row from its hot list (step 3).
__device__ __forceinline__ void row_buckets(const Geom &G, uint32_t row, const uint32_t *he,
                                            uint32_t n, uint32_t *bk_off, uint32_t *bk_cur,
                                            uint32_t *bk_val, uint32_t *lcur, uint32_t *sh) {
  const uint32_t nb = 1u << (G.k - G.alpha);
  uint32_t *off = bk_off + (size_t)row * (nb + 1);
  const uint32_t *h = he + ((size_t)row << G.k);
  uint32_t *val = bk_val + ((size_t)row << G.k);
  if (nb <= BK_LDS) bucket_rows(G, row, h, n, off, lds_ptr(lcur), val, sh);
  else bucket_rows(G, row, h, n, off, bk_cur + (size_t)row * nb, val, sh);
}

// One block per row i: HE(i) from the hot bitmap of k_hot_scan (step 2) and
// its bucket table when i >= 2 and the join may run (step 3).
__global__ __launch_bounds__(1024) void k_rows(Geom G, const uint32_t *__restrict__ hotmask,
                                               uint32_t *__restrict__ he,
                                               uint32_t *__restrict__ bk_off,
                                               uint32_t *__restrict__ bk_cur,
                                               uint32_t *__restrict__ bk_val,
                                               DevState *__restrict__ st, uint32_t buckets) {
  __shared__ uint32_t sh[17];
  __shared__ uint32_t lcur[BK_LDS];
  const uint32_t row = blockIdx.x;
  compact_row(G, row, hotmask, he, st, sh);
  if (row < 2 || !buckets) return;                     // uniform over the block
  __syncthreads();                                     // this row's HE and count
  row_buckets(G, row, he, st->he_count[row], bk_off, bk_cur, bk_val, lcur, sh);
}

// The bucket tables of rows 2..r-1 alone (larger sketches, after k_compact).
__global__ __launch_bounds__(1024) void k_buckets(Geom G, const uint32_t *__restrict__ he,
                                                  uint32_t *__restrict__ bk_off,
                                                  uint32_t *__restrict__ bk_cur,
                                                  uint32_t *__restrict__ bk_val,
                                                  const DevState *__restrict__ st) {
  __shared__ uint32_t sh[17];
  __shared__ uint32_t lcur[BK_LDS];
  const uint32_t row = blockIdx.x + 2;
  row_buckets(G, row, he, st->he_count[row], bk_off, bk_cur, bk_val, lcur, sh);
}

// Steps 1-3 of a small sketch (k <= SCAN_ROWS_K) in one launch, one block
// per row: the row's zero counts (at most 256 KiB) to its hot bitmap, ZR(i),
// HE(i) and bucket table, and the state's start. A small sketch's restore is
// a chain of launches of a few microseconds each: clearing, scan and rows
// took 12.5 us of kernels in three launches for the default sketch.
constexpr uint32_t SCAN_ROWS_K = 16;

__global__ __launch_bounds__(1024) void k_scan_rows(
    Geom G, const uint4 *__restrict__ lez4, uint32_t zhot, uint32_t *__restrict__ hotmask,
    uint32_t *__restrict__ he, uint32_t *__restrict__ bk_off, uint32_t *__restrict__ bk_cur,
    uint32_t *__restrict__ bk_val, DevState *__restrict__ st, uint32_t buckets) {
  __shared__ uint32_t hw[(1u << SCAN_ROWS_K) / 32];
  __shared__ uint32_t lcur[BK_LDS];
  __shared__ uint32_t sh[17];
  __shared__ unsigned long long zr;
  const uint32_t row = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  const uint32_t nq = (1u << G.k) / 4, nw = (1u << G.k) / 32;   // k >= 5: whole groups of 8 lanes
  const uint4 *z4 = lez4 + (size_t)row * nq;
  if (row == 0) state_begin(G, st);
  if (tid == 0) zr = 0;
  __syncthreads();
  uint32_t zeros = 0;                                   // a lane's: at most 64 LEs of 2^13
  constexpr uint32_t U = 4;
  for (uint32_t q0 = tid; q0 < nq; q0 += 1024 * U) {
    uint4 z[U];
#pragma unroll
    for (uint32_t u = 0; u < U; u++) z[u] = z4[q0 + u * 1024 < nq ? q0 + u * 1024 : q0];
#pragma unroll
    for (uint32_t u = 0; u < U; u++) {
      const uint32_t q = q0 + u * 1024;
      const uint32_t w = hot_word(z[u], zhot, lane);
      if (q < nq) {
        if ((lane & 7) == 0) {
          hw[q >> 3] = w;
          hotmask[(size_t)row * nw + (q >> 3)] = w;
        }
        zeros += z[u].x + z[u].y + z[u].z + z[u].w;
      }
    }
  }
  // a wave's sum is below 2^26
  zeros = wave_incl_scan(zeros);
  if (lane == 63 && zeros) atomicAdd(&zr, (unsigned long long)zeros);
  __syncthreads();
  constexpr uint32_t PER = (1u << SCAN_ROWS_K) / 32 / 1024;
  const uint32_t w0 = tid * PER;
  uint32_t m[PER], cnt = 0, total;
#pragma unroll
  for (uint32_t u = 0; u < PER; u++) {
    m[u] = w0 + u < nw ? hw[w0 + u] : 0u;
    cnt += __popc(m[u]);
  }
  const uint32_t ex = block_excl_scan<1024>(cnt, &total, sh);
  uint32_t *out = he + ((size_t)row << G.k) + ex;
#pragma unroll
  for (uint32_t u = 0; u < PER; u++) {
    while (m[u]) {
      const uint32_t b = __ffs(m[u]) - 1;
      *out++ = ((w0 + u) << 5) | b;
      m[u] &= m[u] - 1;
    }
  }
  if (tid == 0) {
    st->zr[row] = zr;
    st->he_count[row] = total;
  }
  if (row < 2 || !buckets) return;                     // uniform over the block
  __syncthreads();                                     // this row's HE
  row_buckets(G, row, he, total, bk_off, bk_cur, bk_val, lcur, sh);
}

// ------------------------------------------------------ 5: search choice

// The join's work is about its probes and partial addresses, |HE(0)||HE(1)|
// then times |HE(i)| / 2^(k-alpha) per further row, 4.5 ps each on a whole
// chip (9.7M in 44 us, 10.4M in 48 us). The lattice search's is, per hot
// row-0 cell, all 2^(32-k) addresses of the cell at 0.44 ps (162M at k = 16 in
// 71 us, 210M at k = 15 in 88 us; with the larger bitmaps 0.62 at k = 18, 263M
// in 162 us, and 0.71 at k = 19, 114M in 82 us), or by the pair index a pair
// per hot row-1 cell: 6.5 ps with the four-part records (6.1M in 42 us), 8.6
// with the six-part ones (2.6M in 26 us; 8.3M in 56), and by the lists, as k =
// 14 has it, 5 addresses' worth a part more than 13. Every kernel of the
// searches evaluates this on the same counts, so exactly one of them runs.
constexpr double LATTICE_COST = 0.1;                    // an address, in join items
// a pair, in addresses
__device__ constexpr double pair_cost(uint32_t k) {
  return k >= 16 ? 15.0 : k == 15 ? 20.0 : 13.0 + 5.0 * (pair_span(k) + 1);
}

__device__ __forceinline__ double pair_work(const Geom &G, const DevState *st) {
  return (double)st->he_count[1] * pair_cost(G.k);
}
// ways: what the sketch has, LAT_OK and LAT_PAIRS (see Lattice).
constexpr uint32_t LAT_OK = 1, LAT_PAIRS = 2;
inline uint32_t lattice_ways(const Lattice &L) {
  return (L.ok ? LAT_OK : 0u) | (L.pair_z ? LAT_PAIRS : 0u);
}
__device__ __forceinline__ bool pairs_chosen(const Geom &G, const DevState *st, uint32_t ways) {
  return (ways & LAT_PAIRS) && pair_work(G, st) < (double)(1ull << (32 - G.k));
}

// A row without a zero bit left (psi = 1): nothing to search.
// (Every block of a search asks: the loads go out together.)
__device__ __forceinline__ bool no_zeros(const Geom &G, const DevState *st) {
  bool none = false;
#pragma unroll
  for (uint32_t i = 0; i < R_MAX; i++) none = none | ((i < G.r) & (st->zr[i] == 0));
  return none;
}

// Step 4 by the first block of each search launched: both searches' kernels
// follow the scan, and the estimate follows them.
__device__ __forceinline__ void search_begin(const Geom &G, DevState *st, double e_theta,
                                             bool chosen, uint32_t search) {
  if (blockIdx.x != 0 || threadIdx.x >= 64) return;
  const bool full = no_zeros(G, st);
  if (!chosen && !full) return;
  scalars(G, st, e_theta);
  if (threadIdx.x == 0 && !full) st->search = search;
}

__device__ __forceinline__ bool lattice_chosen(const Geom &G, const DevState *st,
                                               uint32_t ways, uint32_t path) {
  if (!(ways & LAT_OK) || path == 1) return false;
  if (path == 2) return true;
  const double per = 1.0 / (double)(1u << (G.k - G.alpha));   // a power of two: exact
  uint32_t h[R_MAX];
#pragma unroll
  for (uint32_t i = 0; i < R_MAX; i++) h[i] = st->he_count[i];   // all eight, 0 past r
  double p = (double)h[0] * (double)h[1], join = p;
#pragma unroll
  for (uint32_t i = 2; i < R_MAX; i++) {
    p *= (double)h[i] * per;
    join += p;
  }
  const double cell = pairs_chosen(G, st, ways) ? pair_work(G, st) : (double)(1ull << (32 - G.k));
  const double lat = (double)st->he_count[0] * cell * LATTICE_COST;
  return lat < join;
}

// --------------------------------------------------------- 5b: lattice search
//
// Cell c of row 0 holds exactly the addresses a whose lattice point
// (a, y) lies in the box 0 <= a < 2^32, Y <= y < Y + S, where S = 2^(64-k)
// and Y = c S - B0 (mod 2^64). Every lattice point is p0 + i u + j v for a
// point p0 near (0, Y) and integers (i, j); the box is a parallelogram in
// (i, j). One work item is one line j of one cell: its lane solves the
// line's range of i (in double, widened, then narrowed exactly in 64-bit
// integers to the first and last points inside) and walks it, LAT_TRIP
// points per trip, testing each point's LE in row 1 against row 1's hot
// bitmap in LDS. About |HE(1)| / 2^k of the points pass (a few percent); they go to
// a queue per wave in LDS, and each time the queue holds 64 the wave tests
// them together, one per lane: the LEs of rows 0 and 2..r-1 read from the
// hot bitmap in global memory all at once, then one atomic per wave for
// the appends. The walk runs in step across the wave (a lane whose line is
// done walks no points), so the queue's fill is the same in every lane.
// Each address lies in exactly one cell, so there are no duplicates.
//
// Bound by the vector ALU's issue: about 6 instructions and an LDS read per
// address, and 3 to 4 for the survivors. 16 addresses per trip (the survivors'
// prefix sum and loop once for them), the bit field extract's own masking, a
// compute unit filled with waves, and candidates kept in LDS took the
// 100M-pair window's search (119M addresses) from 97 to 67 us, a k = 19
// sketch's from 126 to 58, and one of 511M addresses with 115,000 candidates
// (k = 17, 12% of the LEs hot) from 1346 to 340 us. Survivors taken per
// point by the wave's compare mask instead (9 vector instructions per
// address, but a branch each) were slower: 84 us for the first.

constexpr int LAT_THREADS = 1024;
constexpr uint32_t LAT_TRIP = 16;                       // points per lane per trip
constexpr uint32_t LAT_PUSH = 512;                      // survivors appended at once, at most
constexpr uint32_t LAT_QUEUE = 63 + LAT_PUSH + 1;       // survivors per wave
constexpr uint32_t LAT_QUEUE_BYTES = (LAT_THREADS / 64) * LAT_QUEUE * 4;
constexpr uint32_t LAT_FOUND_BYTES = sizeof(CandBuf) + 8;
// row 1's bitmap for k <= 20 (128 KiB; fewer waves, whose queues fit beside
// it), and the queues
constexpr uint32_t LATTICE_LDS_MAX = 163840;

// Rows whose hot bitmaps a block of the search holds in LDS: rows 1..n, as
// many as fit half a compute unit's LDS (its scalar registers, 106, leave a
// unit one block of 16 waves, not two). Row 1 takes every
// address, row 2 those that pass it (61M of 511M addresses at k = 17 with 12%
// of the LEs hot).
inline uint32_t lattice_rows(const Geom &G) {
  const uint32_t row = 4u << (G.k - 5);
  uint32_t n = 1;
  while (n + 1 < G.r && (n + 1) * row + LAT_FOUND_BYTES + LAT_QUEUE_BYTES <= 81920) n++;
  return n;
}
inline uint32_t lattice_lds(const Geom &G, uint32_t rows, uint32_t threads) {
  return rows * (4u << (G.k - 5)) + LAT_FOUND_BYTES + threads / 64 * LAT_QUEUE * 4;
}
// Threads of a block: as many waves as have room for their queues.
inline uint32_t lattice_threads(const Geom &G, uint32_t rows) {
  uint32_t t = LAT_THREADS;
  while (lattice_lds(G, rows, t) > LATTICE_LDS_MAX) t /= 2;
  return t;
}

__device__ __forceinline__ int64_t mul_hi_s(int64_t m, uint64_t y) {
  return (int64_t)(((__int128)m * (__int128)(unsigned __int128)y) >> 64);
}

__global__ __launch_bounds__(LAT_THREADS) void k_lattice(
    Geom G, Lattice L, uint32_t ways, uint32_t path, const uint32_t *__restrict__ he,
    const uint32_t *__restrict__ hotmask, DevState *__restrict__ st,
    uint32_t *__restrict__ cand, size_t cand_cap, double e_theta, uint32_t lds_rows) {
  // lds_rows * 2^k bits, the candidates, then the queues
  extern __shared__ __attribute__((aligned(16))) uint32_t row1[];
  const bool chosen = lattice_chosen(G, st, ways, path) && !pairs_chosen(G, st, ways);
  search_begin(G, st, e_theta, chosen, 2);
  if (!chosen || no_zeros(G, st)) return;
  const uint32_t k = G.k, kw = 1u << (k - 5);
  CandBuf *found = reinterpret_cast<CandBuf *>(row1 + lds_rows * kw + (lds_rows * kw & 1));
  if (threadIdx.x == 0) found->n = 0;
  for (uint32_t w = threadIdx.x; w < lds_rows * kw; w += blockDim.x) row1[w] = hotmask[kw + w];
  __syncthreads();
  const uint32_t lane = threadIdx.x & 63;
  uint32_t *queue = reinterpret_cast<uint32_t *>(found + 1) + (threadIdx.x >> 6) * LAT_QUEUE;
  uint32_t qn = 0;                                       // queue fill, wave-uniform

  // one survivor of row 1 per lane (ok = the lane has one): its LEs in rows
  // 2..r-1 all hot -> a candidate (row 0's is: every address walked is in a
  // hot row-0 cell). Rows in LDS first, one by one; the rest together.
  auto test = [&](uint32_t ad, bool ok) {
    const uint32_t c = hash_dh0(G, ad);
    // the row's word and bit of ad; its block's shift (row-1)*alpha (0 past
    // bit 31) worked out here rather than read from G, which would hold six
    // more scalar registers through the walk
    auto cell = [&](uint32_t row) {
      const uint32_t sh = (row - 1) * G.alpha;
      return c ^ __builtin_amdgcn_ubfe(ad, sh, sh < 32 ? k : 0u);
    };
    for (uint32_t row = 2; row <= lds_rows; row++) {
      const uint32_t x = cell(row);
      ok = ok && ((row1[(row - 1) * kw + (x >> 5)] >> (x & 31)) & 1u);
      if (__ballot(ok) == 0) return;
    }
    if (ok) {
      uint32_t wv[8], x[8];
#pragma unroll
      for (uint32_t row = 2; row < 8; row++)
        if (row > lds_rows && row < G.r) {
          x[row] = cell(row);
          wv[row] = hotmask[row * kw + (x[row] >> 5)];
        }
#pragma unroll
      for (uint32_t row = 2; row < 8; row++)
        if (row > lds_rows && row < G.r) ok = ok && ((wv[row] >> (x[row] & 31)) & 1u);
    }
    found->add(ad, ok, st, cand, cand_cap);
  };
  // append the points of this trip that passed row 1 (bit q of hit: point
  // b + q step), placed by a prefix sum over the wave; test 64 at a time
  // while the queue holds them. The queue has room for half of a trip's
  // points: a trip with more survivors goes in two halves
  auto append = [&](uint32_t b, uint32_t step_, uint32_t hit, uint32_t cnt, uint32_t incl) {
    uint32_t pos = qn + incl - cnt;
    for (uint32_t h = hit; h; h &= h - 1) queue[pos++] = b + (uint32_t)__builtin_ctz(h) * step_;
    qn += wave_lane(incl, 63);
    __builtin_amdgcn_wave_barrier();
    while (qn >= 64) {
      qn -= 64;
      const uint32_t ad2 = queue[qn + lane];
      __builtin_amdgcn_wave_barrier();
      test(ad2, true);
    }
  };
  auto push = [&](uint32_t b, uint32_t step_, uint32_t hit) {
    const uint32_t cnt = __popc(hit), incl = wave_scan_incl(cnt);
    if (wave_lane(incl, 63) <= LAT_PUSH) {
      append(b, step_, hit, cnt, incl);
    } else {
#pragma unroll 1
      for (uint32_t half = 0xFFu; half <= 0xFF00u; half <<= 8) {
        const uint32_t h = hit & half, n_h = __popc(h);
        append(b, step_, h, n_h, wave_scan_incl(n_h));
      }
    }
  };

  const uint32_t s = 64 - k;
  const uint64_t S = 1ull << s;
  const uint32_t bmask = (kw - 1) << 2;                 // byte offsets of row 1's words
  const double D = L.dneg ? -0x1p64 : 0x1p64;
  const uint32_t lines = L.lines;
  const uint32_t h0 = st->he_count[0];
  const uint32_t items = h0 * lines;                    // < 2^32 for k <= 24
  const uint32_t step = (uint32_t)L.ua;
  // every lane of a block takes the same trips (uniform bounds)
  for (uint32_t t0 = blockIdx.x * blockDim.x; t0 < items; t0 += gridDim.x * blockDim.x) {
    const uint32_t t = t0 + threadIdx.x;
    uint32_t n = 0, a = 0, c = 0;                      // n points from address a in cell c
    if (t < items) {
      // line-major: the lanes of a wave take the same line of consecutive
      // hot cells; every cell's box is the same parallelogram shifted, so
      // these lines are about equally long and the lanes end their walks
      // together (cell-major, a wave's lines differ by up to 2x)
      const uint32_t line = t / h0, x = t - line * h0;
      c = he[x];
      const uint64_t Y = ((uint64_t)c << s) - G.b0;
      // p0 = i0 u + j0 v with (i0, j0) ~ M^-1 (0, Y), M = [u v]; its offsets
      // from (0, Y) are small, so wrapping 64-bit arithmetic gives them exactly
      int64_t i0 = mul_hi_s(-L.va, Y), j0 = mul_hi_s(L.ua, Y);
      if (L.dneg) {
        i0 = -i0;
        j0 = -j0;
      }
      const int64_t a0 = (int64_t)((uint64_t)i0 * (uint64_t)L.ua + (uint64_t)j0 * (uint64_t)L.va);
      const int64_t dy0 =
          (int64_t)((uint64_t)i0 * (uint64_t)L.uy + (uint64_t)j0 * (uint64_t)L.vy - Y);
      // the cell's lines: j over the box corners
      double jmin = 0, jmax = 0;
#pragma unroll
      for (int q = 0; q < 4; q++) {
        const double da = ((q & 1) ? 4294967296.0 : 0.0) - (double)a0;
        const double dy = ((q & 2) ? (double)S : 0.0) - (double)dy0;
        const double j = (-(double)L.uy * da + (double)L.ua * dy) / D;
        jmin = q ? fmin(jmin, j) : j;
        jmax = q ? fmax(jmax, j) : j;
      }
      const int64_t jlo = (int64_t)floor(jmin) - 1, jhi = (int64_t)ceil(jmax) + 1;
      const int64_t j = jlo + line;
      if (j <= jhi) {
        // this line's i: 0 <= a0 + i ua + j va < 2^32, 0 <= dy0 + i uy + j vy < S
        const double al = -(double)a0 - (double)j * (double)L.va, ah = al + 4294967296.0;
        const double yl = -(double)dy0 - (double)j * (double)L.vy, yh = yl + (double)S;
        double lo = -1e300, hi = 1e300;
        if (L.ua) {
          const double p = al / (double)L.ua, q = ah / (double)L.ua;
          lo = fmax(lo, fmin(p, q));
          hi = fmin(hi, fmax(p, q));
        }
        if (L.uy) {
          const double p = yl / (double)L.uy, q = yh / (double)L.uy;
          lo = fmax(lo, fmin(p, q));
          hi = fmin(hi, fmax(p, q));
        }
        if (lo <= hi + 2.0) {
          // the box cuts the line in one run of i: the estimate, widened,
          // then narrowed exactly to the first and last points inside
          int64_t ilo = (int64_t)floor(lo) - 1, ihi = (int64_t)ceil(hi) + 1;
          const int64_t aj = a0 + j * L.va, yj = dy0 + j * L.vy;
          auto inside = [&](int64_t i) {
            return (uint64_t)(aj + i * L.ua) < 4294967296ull &&
                   (uint64_t)(yj + i * L.uy) < S;
          };
          while (ilo <= ihi && !inside(ilo)) ilo++;
          while (ihi >= ilo && !inside(ihi)) ihi--;
          if (ilo <= ihi) {
            // every point of [ilo, ihi] is an address of cell c
            a = (uint32_t)(aj + ilo * L.ua);
            n = (uint32_t)(ihi - ilo + 1);
          }
        }
      }
    }
    // the walk: LAT_TRIP points per trip, the row-1 words of 8 read together.
    // Point b's row-1 LE is x = (c ^ b) mod 2^k: its word is bits 5..k-1 of x
    // (byte offset: bits 3..k-4) and its bit bits 0..4 (all that the bit field
    // extract takes of its offset). Points past the line's end read a valid
    // word and are masked out of hit.
    while (__ballot(n != 0)) {
      const uint32_t m = n < LAT_TRIP ? n : LAT_TRIP;
      uint32_t hit = 0, b = a;
#pragma unroll
      for (uint32_t h = 0; h < LAT_TRIP; h += 8) {
        uint32_t x[8], w[8];
#pragma unroll
        for (uint32_t q = 0; q < 8; q++) {
          x[q] = c ^ b;
          // the block's dynamic LDS, its only LDS (prepare_restore_kernels sees
          // to that), starts at address 0; taken from row1, the address costs
          // an addition, of about six instructions per address
          w[q] = *(const LDSP uint32_t *)(uintptr_t)((x[q] >> 3) & bmask);
          b += step;
        }
#pragma unroll
        for (uint32_t q = 0; q < 8; q++)
          hit |= __builtin_amdgcn_ubfe(w[q], x[q], 1u) << (h + q);
      }
      hit &= (1u << m) - 1;
      push(a, step, hit);
      a += m * step;
      n -= m;
    }
  }
  // what is left in the queue
  if (qn) test(queue[lane < qn ? lane : 0], lane < qn);
  found->flush(st, cand, cand_cap);
}

// --------------------------------------------------- 5b: the search by pairs
//
// The lattice search's other way through the hot row-0 cells, for sketches
// with a pair index: a hot row-1 cell c1 with c0 fixes an address's low k
// bits, c0 ^ c1, and of its 2^(32-k) high parts z only those are in cell c0
// for which A0 z 2^k (mod 2^64) lies in an interval of 2^(64-k): 2^(32-2k)
// parts on average, which the index gives by the bucket the interval starts
// in: in a record, or (k = 14, and where a record does not hold them) in a
// list. So the walk's addresses that fail row 1 are never made. A wave takes
// 64 PAIR_UNROLL pairs of one c0 and looks at all parts of the interval's
// buckets, which may hold some outside it: each part's LE in row 2 is tested
// in LDS, those that pass (a few percent) go to the wave's queue, and 64 of
// them together are hashed (exactly the addresses of cell c0 stay) and
// tested in the rows past 2. Each address has one (c0, c1), so there are no
// duplicates. Bound by vector issue and the cache line that each pair's
// record brings from the L2: with the records 26 us, by the lists (two to
// three lines a pair) 43, for the 2.6M pairs (210M addresses, a walk of 88
// us) of a 9M-pair window at k = 15; k = 16, 6.1M pairs (162M addresses, 71
// us) 44 us, by the lists 61, with three parts of 21 bits a record 50 (a fifth
// of the buckets of the default seed held a fourth); a 4M-pair window at k =
// 15, r = 4, which took the join, 44 -> 13 us.
constexpr uint32_t PAIR_UNROLL = 4;                     // pairs per lane at once
constexpr uint32_t PAIR_QUEUE = 128;                    // 63 + 64 addresses per wave
constexpr uint32_t PAIR_THREADS = 1024;
constexpr uint32_t PAIR_QUEUE_BYTES = PAIR_THREADS / 64 * PAIR_QUEUE * 4;

// Rows 2.. whose hot bitmaps a block holds in LDS, two blocks to a compute
// unit where their scalar registers allow it (80 and less: not k_pairs<1>, with
// 87); row 2 always: 32 KiB at k = 18.
inline uint32_t pair_rows(const Geom &G) {
  const uint32_t row = 4u << (G.k - 5);
  uint32_t n = 1;
  while (n + 2 < G.r && (n + 1) * row + LAT_FOUND_BYTES + PAIR_QUEUE_BYTES <= 81920) n++;
  return n;
}

// RW: 64-bit words of a bucket's record (pair_rec_words).
template <int RW>
__global__ __launch_bounds__(PAIR_THREADS) void k_pairs(
    Geom G, const uint32_t *__restrict__ pair_off, const uint32_t *__restrict__ pair_z,
    const uint32_t *__restrict__ pair_rec, uint32_t ways, uint32_t path, const uint32_t *__restrict__ he,
    const uint32_t *__restrict__ hotmask, DevState *__restrict__ st,
    uint32_t *__restrict__ cand, size_t cand_cap, double e_theta, uint32_t lds_rows) {
  // lds_rows * 2^k bits, the candidates, then the queues
  extern __shared__ __attribute__((aligned(16))) uint32_t row2[];
  const bool chosen = lattice_chosen(G, st, ways, path) && pairs_chosen(G, st, ways);
  search_begin(G, st, e_theta, chosen, 3);
  if (!chosen || no_zeros(G, st)) return;
  const uint32_t k = G.k, kw = 1u << (k - 5), alpha = G.alpha;
  CandBuf *found = reinterpret_cast<CandBuf *>(row2 + lds_rows * kw);
  if (threadIdx.x == 0) found->n = 0;
  for (uint32_t w = threadIdx.x; w < lds_rows * kw; w += blockDim.x) row2[w] = hotmask[2 * kw + w];
  __syncthreads();
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t wib = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  uint32_t *queue = reinterpret_cast<uint32_t *>(found + 1) + wib * PAIR_QUEUE;
  const uint32_t *HE1 = he + (1u << k);
  const uint32_t h0 = st->he_count[0], h1 = st->he_count[1];
  const uint32_t nch = (h1 + 64 * PAIR_UNROLL - 1) / (64 * PAIR_UNROLL);
  const uint32_t items = h0 * nch, parts = 1u << (32 - k);   // items < 2^32 by the rule on h1

  for (uint32_t w = blockIdx.x + gridDim.x * wib; w < items; w += gridDim.x * (PAIR_THREADS / 64)) {
    const uint32_t x0 = w / nch, x1 = (w - x0 * nch) * (64 * PAIR_UNROLL) + lane;
    const uint32_t c0 = __builtin_amdgcn_readfirstlane(he[x0]);
    uint32_t qn = 0;                                    // queue fill, wave-uniform
    // one address that passed row 2 per lane
    auto test = [&](uint32_t ad, bool ok) {
      ok = ok && hash_dh0(G, ad) == c0;
      for (uint32_t row = 3; row < G.r; row++) {
        if (__ballot(ok) == 0) return;
        const uint32_t sh = (row - 1) * alpha;
        const uint32_t x = c0 ^ __builtin_amdgcn_ubfe(ad, sh, sh < 32 ? k : 0u);
        uint32_t v;
        if (row - 2 < lds_rows) v = row2[(row - 2) * kw + (x >> 5)];
        else v = hotmask[row * kw + (x >> 5)];
        ok = ok && ((v >> (x & 31)) & 1u);
      }
      found->add(ad, ok, st, cand, cand_cap);
    };
    // one part per lane: its address queued if its LE in row 2 is hot
    auto look = [&](uint32_t low, uint32_t z, bool ok) {
      const uint32_t ad = low | (z << k), x = c0 ^ __builtin_amdgcn_ubfe(ad, alpha, k);
      ok = ok && ((row2[x >> 5] >> (x & 31)) & 1u);
      const unsigned long long m = __ballot(ok);
      if (m == 0) return;
      if (ok) queue[qn + lanes_below(m)] = ad;
      qn += (uint32_t)__popcll(m);
      __builtin_amdgcn_wave_barrier();
      if (qn >= 64) {
        qn -= 64;
        const uint32_t ad2 = queue[qn + lane];
        __builtin_amdgcn_wave_barrier();
        test(ad2, true);
      }
    };
    const uint64_t lo0 = ((uint64_t)c0 << (64 - k)) - G.b0;
    uint32_t low[PAIR_UNROLL], b[PAIR_UNROLL];
#pragma unroll
    for (uint32_t u = 0; u < PAIR_UNROLL; u++)
      low[u] = c0 ^ HE1[x1 + 64 * u < h1 ? x1 + 64 * u : h1 - 1];
#pragma unroll
    for (uint32_t u = 0; u < PAIR_UNROLL; u++)
      b[u] = (uint32_t)((lo0 - G.a0 * low[u]) >> 32) >> k;
    uint32_t listed = 0;                                // pairs that go by off and z (bit u)
#pragma unroll
    for (uint32_t u = 0; u < PAIR_UNROLL; u++)
      if (x1 + 64 * u < h1) listed |= 1u << u;
    if constexpr (RW > 0) {
      uint32_t rec[PAIR_UNROLL][2 * RW];
#pragma unroll
      for (uint32_t u = 0; u < PAIR_UNROLL; u++)
        __builtin_memcpy(rec[u], __builtin_assume_aligned(pair_rec + (size_t)b[u] * (2 * RW), 8 * RW),
                         8 * RW);
      const uint32_t live = listed;
      listed = 0;
#pragma unroll
      for (uint32_t u = 0; u < PAIR_UNROLL; u++) {
        bool on = (live >> u) & 1u;
        if constexpr (RW == 1) {
          const uint32_t z0 = rec[u][0] & 0xFFFF, z1 = rec[u][0] >> 16, z2 = rec[u][1] & 0xFFFF,
                         z3 = rec[u][1] >> 16;
          if (on && z1 == z0 && z2 != z0) {
            listed |= 1u << u;
            on = false;
          }
          look(low[u], z0, on);
          look(low[u], z1, on && z1 != z0);
          look(low[u], z2, on && z2 != z0);
          look(low[u], z3, on && z3 != z0);
        } else {
          if (on && rec[u][1] >> 31) listed |= 1u << u;   // its words hold no part
#pragma unroll
          for (int i = 0; i < RW; i++) {
            const uint32_t lo = rec[u][2 * i], hi = rec[u][2 * i + 1];
            const uint32_t z[3] = {lo & PAIR_NONE,
                                   __builtin_amdgcn_alignbit(hi, lo, 21) & PAIR_NONE,
                                   __builtin_amdgcn_ubfe(hi, 10, 21)};
#pragma unroll
            for (int j = 0; j < 3; j++) look(low[u], z[j], on && z[j] != PAIR_NONE);
          }
        }
      }
    }
    if (RW == 0 || __ballot(listed != 0)) {
      uint32_t q[PAIR_UNROLL], n[PAIR_UNROLL], most = 0;
#pragma unroll
      for (uint32_t u = 0; u < PAIR_UNROLL; u++)
        q[u] = (listed >> u) & 1u ? pair_off[b[u]] : 0u;
#pragma unroll
      for (uint32_t u = 0; u < PAIR_UNROLL; u++) {
        n[u] = q[u] >> PAIR_PLACE_BITS;
        if (n[u] == PAIR_MANY) n[u] = parts;            // more than the index says: any part
        q[u] &= (1u << PAIR_PLACE_BITS) - 1;
        most = n[u] > most ? n[u] : most;
      }
      for (uint32_t t = 0; __ballot(t < most); t += 4) {
        uint32_t z[PAIR_UNROLL][4] = {};
#pragma unroll
        for (uint32_t u = 0; u < PAIR_UNROLL; u++)
          if (t < n[u]) __builtin_memcpy(z[u], pair_z + q[u] + t, 16);
#pragma unroll
        for (uint32_t u = 0; u < PAIR_UNROLL; u++)
#pragma unroll
          for (uint32_t i = 0; i < 4; i++) look(low[u], z[u][i], t + i < n[u]);
      }
    }
    if (qn) test(queue[lane < qn ? lane : 0], lane < qn);
    __builtin_amdgcn_wave_barrier();
  }
  found->flush(st, cand, cand_cap);
}

// The pair index, built once per hash family (a0, k): the counts per bucket
// become their starts, the parts take their places, and then the second copy of
// the parts and the bucket words are made.
__device__ __forceinline__ uint32_t pair_bucket(const Geom &G, uint32_t z) {
  return (uint32_t)((G.a0 * z) << G.k >> 32) >> G.k;
}

__global__ __launch_bounds__(256) void k_pair_count(Geom G, uint32_t *__restrict__ cnt) {
  atomicAdd(&cnt[pair_bucket(G, blockIdx.x * 256 + threadIdx.x)], 1u);
}

// Block x: the starts of 4096 buckets, after the parts of all buckets before
// them, which it adds up itself (one block for all took 80 us at k = 14).
__global__ __launch_bounds__(1024) void k_pair_starts(Geom G, const uint32_t *__restrict__ cnt,
                                                      uint32_t *__restrict__ start,
                                                      uint32_t *__restrict__ cur, uint32_t n) {
  __shared__ uint32_t sh[17];
  const uint32_t tid = threadIdx.x, i = blockIdx.x * 1024 + tid;
  const uint4 *c4 = reinterpret_cast<const uint4 *>(cnt);
  uint32_t sum = 0, before, total;
#pragma unroll 4
  for (uint32_t j = tid; j < blockIdx.x * 1024; j += 1024) {
    const uint4 c = c4[j];
    sum += c.x + c.y + c.z + c.w;
  }
  block_excl_scan<1024>(sum, &before, sh);
  const uint4 c = c4[i];
  const uint32_t x = before + block_excl_scan<1024>(c.x + c.y + c.z + c.w, &total, sh);
  const uint4 st = make_uint4(x, x + c.x, x + c.x + c.y, x + c.x + c.y + c.z);
  reinterpret_cast<uint4 *>(start)[i] = st;
  reinterpret_cast<uint4 *>(cur)[i] = st;
  if (blockIdx.x == 0) {                                // the starts that go round
    const uint32_t v[4] = {st.x, st.y, st.z, st.w};
    for (uint32_t u = 0; u < 4; u++)
      if (4 * i + u <= pair_span(G.k)) start[n + 4 * i + u] = n + v[u];
  }
}

__global__ __launch_bounds__(256) void k_pair_place(Geom G, uint32_t *__restrict__ z, uint32_t n) {
  const uint32_t i = blockIdx.x * 256 + threadIdx.x;
  z[atomicAdd(&z[n + pair_bucket(G, i)], 1u)] = i;      // the cursors: z's second half
}

__global__ __launch_bounds__(256) void k_pair_finish(Geom G, uint32_t *__restrict__ off,
                                                     uint32_t *__restrict__ z,
                                                     uint32_t *__restrict__ rec, uint32_t n) {
  const uint32_t b = blockIdx.x * 256 + threadIdx.x;
  const uint32_t *start = off + n;
  z[n + b] = z[b];
  if (b < 4) z[2 * n + b] = 0;
  const uint32_t at = start[b], parts = start[b + pair_span(G.k) + 1] - at;
  off[b] = at | (parts < PAIR_MANY ? parts : PAIR_MANY) << PAIR_PLACE_BITS;
  const uint32_t rw = pair_rec_words(G.k);
  uint64_t *words = reinterpret_cast<uint64_t *>(rec) + (size_t)b * rw;
  // part i from bucket b on, of the first copy (complete before this kernel)
  auto part = [&](uint32_t i) { return (uint64_t)z[(at + i) & (n - 1)]; };
  if (rw == 1) {
    uint64_t w = 0x0001000100000000ull;
    if (parts <= 4) {
      w = 0;
      for (uint32_t j = 0; j < 4; j++) w |= part(j < parts ? j : 0) << (16 * j);
    }
    words[0] = w;
  } else {
    const bool fits = parts <= 3 * rw;
    for (uint32_t i = 0; i < rw; i++) {
      uint64_t w = fits ? 0 : 1ull << 63;
      for (uint32_t j = 3 * i; j < 3 * i + 3; j++)
        w |= (fits && j < parts ? part(j) : PAIR_NONE) << (21 * (j - 3 * i));
      words[i] = w;
    }
  }
}

hipError_t launch_pair_index(const Geom &G, uint32_t *off, uint32_t *z, uint32_t *rec,
                             hipStream_t st) {
  const uint32_t n = 1u << (32 - G.k), blocks = n / 256;
  hipError_t e = launch_fill_u32(off, n, 0u, 64, st);
  if (e != hipSuccess) return e;
  k_pair_count<<<blocks, 256, 0, st>>>(G, off);
  k_pair_starts<<<n / 4096, 1024, 0, st>>>(G, off, off + n, z + n, n);
  k_pair_place<<<blocks, 256, 0, st>>>(G, z, n);
  k_pair_finish<<<blocks, 256, 0, st>>>(G, off, z, rec, n);
  return hipGetLastError();
}

// ------------------------------------------------------------------ 5: join
//
// Stage 1 (Alg. 3) takes every (CL_0, CL_1) of HE(0) x HE(1); stage i >= 3
// (Alg. 4) takes every partial address of stage i-1. Each item probes the
// bucket of HE(i) (i = 2 for stage 1) that holds exactly the entries whose
// low k-alpha bits continue the overlap, and every entry of it that extends
// the partial address is an output.
//
//  - The probed row's bucket table is copied into LDS when it fits: offsets
//    as uint16, and per entry only its top alpha bits (the bucket index is
//    the low k-alpha bits), as uint8 or uint16. Otherwise it is read from
//    the global tables.
//  - A wave expands its 64 items together: the bucket sizes are scanned, and
//    each lane then takes one output slot and finds the item that owns it by
//    a binary search over the scan, so uneven bucket sizes do not diverge.
//  - Every block appends its outputs to its own segment of the next
//    stage's buffer through an LDS counter (no global counter); stage i+1's
//    block b reads segment b. Counts stay exact past a segment's capacity,
//    so the host can grow it and run again.
//  - The last stage keeps an address only if it is a 32-bit value and DH0
//    of it is the CL_0 it was built from; those few are appended to the
//    candidate list with a global counter.

constexpr int JOIN_THREADS = 512;
// Scalar registers that leave four blocks of eight waves on a compute unit: a
// wave takes 16 for the trap handler beside its own, and above 80 of those
// seven waves fit a SIMD, which the compiler's occupancy does not count. With
// 83 the last stage of a join of 238M partial addresses took 3.0 ms, with 80
// 2.5.
constexpr int JOIN_SGPRS = 80;

// Orders this wave's LDS writes before its later LDS reads by other lanes.
__device__ __forceinline__ void lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
}
constexpr uint32_t TAB_OFF_MAX = 8193;          // bucket offsets held in LDS
constexpr uint32_t OWN_MAX = 256;               // output slots per wave pass set
constexpr uint32_t TAB_VAL_BYTES = 16384;       // bucket entries held in LDS (4 blocks per CU)

// Bits of the address from block i >= 2: alpha new bits at k + (i-2)*alpha.
// top = the new bits; false if any lands at or above bit 32.
__device__ __forceinline__ bool extend_top(const Geom &G, uint32_t i, uint32_t sub,
                                           uint32_t top, uint32_t *out) {
  const uint32_t pos = G.k + (i - 2) * G.alpha;
  if (pos >= 32) {
    *out = sub;
    return top == 0;
  }
  const uint64_t s2 = (uint64_t)sub | ((uint64_t)top << pos);
  *out = (uint32_t)s2;
  return (s2 >> 32) == 0;
}

// The probed row's bucket table: in LDS (offsets as uint16, entries as
// their top alpha bits) or in the global tables. Which one is a template
// parameter, so a loop over an LDS table issues no global loads that a
// wait for prefetched data would have to cover.
template <bool TLDS>
struct JoinTable {
  const LDSP uint16_t *off16;
  const LDSP uint8_t *hi8;
  const LDSP uint16_t *hi16;
  const uint32_t *off;     // global
  const uint32_t *val;     // global
  uint32_t shift;          // k - alpha
  bool wide;               // alpha > 8
  __device__ __forceinline__ uint32_t start(uint32_t key) const {
    if constexpr (TLDS) return (uint32_t)off16[key];
    else return off[key];
  }
  __device__ __forceinline__ uint32_t top_bits(uint32_t j) const {
    if constexpr (TLDS) return wide ? (uint32_t)hi16[j] : (uint32_t)hi8[j];
    else return val[j] >> shift;
  }
};

// The candidates of a block of the last stage: as many as its LDS has left
// beside the tables with four blocks on a compute unit (512 of them left room
// for three).
using JoinCand = CandBufOf<496>;

template <bool LAST>
struct JoinLds {
  uint16_t off[TAB_OFF_MAX];
  alignas(16) uint8_t val[TAB_VAL_BYTES];
  uint32_t incl[JOIN_THREADS];
  uint16_t own[(JOIN_THREADS / 64) * OWN_MAX];
  uint32_t seg_fill;
  alignas(8) uint8_t found[LAST ? sizeof(JoinCand) : 8];
};
static_assert(sizeof(JoinLds<true>) <= 163840 / 4, "four blocks on a compute unit");

// The wave items of one join block (see k_join).
template <bool FIRST, bool LAST, bool TLDS>
__device__ __forceinline__ void join_items(
    const Geom &G, uint32_t row, const uint32_t *__restrict__ he,
    const uint2 *__restrict__ in, const uint32_t *__restrict__ in_cnt,
    const JoinTable<TLDS> &T, DevState *__restrict__ st, uint2 *__restrict__ out,
    size_t seg_cap, uint32_t *__restrict__ cand, size_t cand_cap, uint32_t M,
    LDSP uint32_t *w_incl, LDSP uint16_t *w_own, LDSP uint32_t *seg_fill_p, JoinCand *found) {
  LDSP uint32_t &seg_fill = *seg_fill_p;
  const uint32_t lane = lane_id();
  const uint32_t wib = threadIdx.x >> 6;                    // wave in block
  const uint32_t wpb = blockDim.x >> 6;                     // waves per block
  LDSP uint32_t *W_incl = w_incl + wib * 64;
  LDSP uint16_t *W_own = w_own + wib * OWN_MAX;
  const uint32_t sh = G.shift[row];
  uint2 *seg = LAST ? nullptr : out + (size_t)blockIdx.x * seg_cap;

  // this block's wave items
  uint64_t w_lo, w_hi, nch = 1;
  const uint32_t *HE0 = he, *HE1 = he + (1u << G.k);
  uint32_t h1 = 0;
  const uint2 *my_in = nullptr;
  uint32_t n_in = 0;
  if (FIRST) {
    const uint32_t h0 = st->he_count[0];
    h1 = st->he_count[1];
    nch = (h1 + 63) >> 6;
    const uint64_t W = (uint64_t)h0 * nch;
    w_lo = W * blockIdx.x / gridDim.x;
    w_hi = W * (blockIdx.x + 1) / gridDim.x;
  } else {
    const uint32_t c = in_cnt[blockIdx.x];
    n_in = (uint32_t)(c < seg_cap ? c : seg_cap);
    my_in = in + (size_t)blockIdx.x * seg_cap;
    w_lo = 0;
    w_hi = (n_in + 63) >> 6;
  }

  // A wave's items are w_lo + wib, + wpb, ...; stage 1's item w is
  // (x0, xc) = (w / nch, w % nch), stepped without dividing. The next
  // item's inputs are loaded before the current one is expanded (indices
  // past the end are clamped: the loads need no branch and stay in bounds).
  uint64_t w = w_lo + wib;
  uint32_t x0 = 0, xc = 0;
  if (FIRST && w < w_hi) {
    x0 = (uint32_t)(w / nch);
    xc = (uint32_t)(w - (uint64_t)x0 * nch);
  }
  auto load_item = [&](uint64_t wi, uint32_t a0, uint32_t ac, uint32_t &sub_o, uint32_t &c0_o,
                       bool &valid_o) {
    if (FIRST) {
      const uint32_t x1 = ac * 64 + lane;
      valid_o = wi < w_hi && x1 < h1;
      const uint32_t c0v = HE0[a0];
      c0_o = c0v;
      sub_o = c0v ^ HE1[x1 < h1 ? x1 : h1 - 1];     // BL(1)
    } else {
      const uint32_t t = (uint32_t)wi * 64 + lane;
      valid_o = wi < w_hi && t < n_in;
      const uint2 p = my_in[t < n_in ? t : n_in - 1];
      sub_o = p.x;
      c0_o = p.y;
    }
  };
  uint32_t n_sub = 0, n_c0 = 0;
  bool n_valid = false;
  if (w < w_hi) load_item(w, x0, xc, n_sub, n_c0, n_valid);

  for (; w < w_hi; w += wpb) {
    // ---- this lane's item; the next one's loads go out now
    uint32_t sub = n_sub, c0 = n_c0, b0 = 0, cnt = 0;
    const bool valid = n_valid;
    {
      const uint64_t wn = w + wpb;
      const uint32_t cx0 = x0, cxc = xc;                   // this item's (x0, xc)
      if (FIRST) {
        xc += wpb;
        while (xc >= nch) {
          xc -= (uint32_t)nch;
          x0++;
        }
      }
      // past the last item: this item's inputs again (in bounds), unused
      const bool more = wn < w_hi;
      if (FIRST) load_item(more ? wn : w, more ? x0 : cx0, more ? xc : cxc, n_sub, n_c0, n_valid);
      else load_item(more ? wn : w, 0, 0, n_sub, n_c0, n_valid);
      if (!more) n_valid = false;
    }
    if (valid) {
      const uint32_t key = ((uint32_t)((uint64_t)sub >> sh) ^ c0) & M;
      b0 = T.start(key);
      cnt = T.start(key + 1) - b0;
    }
    const uint32_t incl = wave_incl_scan(cnt);
    const uint32_t total = wave_lane(incl, 63);
    if (total == 0) continue;
    // each item writes its own index into its output slots when they fit,
    // so a slot finds its item with one LDS read; otherwise by a binary
    // search over the inclusive scan
    const bool own = total <= OWN_MAX;                 // uniform over the wave
    if (own) {
      for (uint32_t q = incl - cnt; q < incl; q++) W_own[q] = (uint16_t)lane;
    } else {
      W_incl[lane] = incl;
    }
    const int32_t my_base = (int32_t)b0 - (int32_t)(incl - cnt);   // entry j = base + slot
    lds_fence();
    // ---- expand: one output slot per lane per pass
    for (uint32_t base = 0; base < total; base += 64) {
      const uint32_t slot = base + lane;
      const bool live = slot < total;
      const uint32_t sl = live ? slot : total - 1;   // lanes past the end repeat the last slot
      uint32_t o = 0;
      if (own) {
        o = W_own[sl];
      } else {
#pragma unroll
        for (uint32_t s = 32; s; s >>= 1)
          if (W_incl[o + s - 1] <= sl) o += s;
      }
      // the owning item's values straight from its lane (every lane takes part)
      const int32_t ob = __builtin_amdgcn_ds_bpermute((int)(o << 2), my_base);
      const uint32_t osub = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(o << 2), (int)sub);
      const uint32_t oc0 = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(o << 2), (int)c0);
      bool ok = false;
      uint32_t a = 0;
      if (live) {
        const uint32_t j = (uint32_t)(ob + (int32_t)slot);
        const uint32_t top = (oc0 >> (G.k - G.alpha)) ^ T.top_bits(j);
        ok = extend_top(G, row, osub, top, &a);
        if (LAST) ok = ok && hash_dh0(G, a) == oc0;
      }
      const unsigned long long mask = __ballot(ok);
      if (mask == 0) continue;
      const uint32_t n_ok = __popcll(mask);
      const uint32_t rank = __popcll(mask & ((1ull << lane) - 1));
      if (LAST) {
        found->add(a, ok, st, cand, cand_cap);
      } else {
        uint32_t lb = 0;
        if (lane == 0) lb = atomicAdd((uint32_t *)&seg_fill, n_ok);   // an LDS atomic after inlining
        lb = wave_lane(lb, 0);
        if (ok && (size_t)lb + rank < seg_cap) seg[lb + rank] = make_uint2(a, oc0);
      }
    }
    lds_fence();
  }
}

template <bool FIRST, bool LAST>
__global__ __launch_bounds__(JOIN_THREADS) __attribute__((amdgpu_num_sgpr(JOIN_SGPRS))) void k_join(
    Geom G, uint32_t ways, uint32_t path, uint32_t row, const uint32_t *__restrict__ he,
    const uint2 *__restrict__ in, const uint32_t *__restrict__ in_cnt,
    const uint32_t *__restrict__ bk_off, const uint32_t *__restrict__ bk_val,
    DevState *__restrict__ st, uint2 *__restrict__ out, uint32_t *__restrict__ out_cnt,
    size_t seg_cap, uint32_t *__restrict__ cand, size_t cand_cap, double e_theta) {
  __shared__ JoinLds<LAST> L;
  uint16_t *const t_off = L.off, *const w_own = L.own;
  uint8_t *const t_val = L.val;
  uint32_t *const w_incl = L.incl;
  uint32_t &seg_fill = L.seg_fill;
  JoinCand *const found = reinterpret_cast<JoinCand *>(L.found);   // last stage only
  const bool chosen = !lattice_chosen(G, st, ways, path);
  if (FIRST) search_begin(G, st, e_theta, chosen, 1);
  if (!chosen || no_zeros(G, st)) return;

  const uint32_t nb = 1u << (G.k - G.alpha), M = nb - 1;
  const uint32_t h = st->he_count[row];
  const bool wide = G.alpha > 8;
  const bool lds = nb + 1 <= TAB_OFF_MAX && h < 65536 && G.alpha <= 16 &&
                   (size_t)h * (wide ? 2 : 1) <= TAB_VAL_BYTES;
  const uint32_t *g_off = bk_off + (size_t)row * (nb + 1);
  const uint32_t *g_val = bk_val + ((size_t)row << G.k);
  if (threadIdx.x == 0) {
    seg_fill = 0;
    if (LAST) found->n = 0;
  }
  if (lds) {
    for (uint32_t x = threadIdx.x; x <= nb; x += blockDim.x) t_off[x] = (uint16_t)g_off[x];
    for (uint32_t x = threadIdx.x; x < h; x += blockDim.x) {
      const uint32_t hi = g_val[x] >> (G.k - G.alpha);
      if (wide) reinterpret_cast<uint16_t *>(t_val)[x] = (uint16_t)hi;
      else t_val[x] = (uint8_t)hi;
    }
  }
  __syncthreads();
  const bool wide_t = wide;
  if (lds) {
    const JoinTable<true> T{lds_ptr(t_off), lds_ptr(t_val),
                            lds_ptr(reinterpret_cast<uint16_t *>(t_val)), g_off, g_val,
                            G.k - G.alpha, wide_t};
    join_items<FIRST, LAST, true>(G, row, he, in, in_cnt, T, st, out, seg_cap, cand, cand_cap,
                                  M, lds_ptr(w_incl), lds_ptr(w_own), lds_ptr(&seg_fill), found);
  } else {
    const JoinTable<false> T{lds_ptr(t_off), lds_ptr(t_val),
                             lds_ptr(reinterpret_cast<uint16_t *>(t_val)), g_off, g_val,
                             G.k - G.alpha, wide_t};
    join_items<FIRST, LAST, false>(G, row, he, in, in_cnt, T, st, out, seg_cap, cand,
                                   cand_cap, M, lds_ptr(w_incl), lds_ptr(w_own),
                                   lds_ptr(&seg_fill), found);
  }
  if (LAST) found->flush(st, cand, cand_cap);
  if (!LAST) {
    __syncthreads();
    if (threadIdx.x == 0) {
      out_cnt[blockIdx.x] = seg_fill;
      atomicAdd(&st->n_out[row], (unsigned long long)seg_fill);
      atomicMax(&st->seg_max[row], seg_fill);
    }
  }
}

// ------------------------------------------------- 5c: the join in one launch
//
// The join of Algs. 3-4 for sketches with small bucket tables (join_walks),
// depth first: a wave's stage-1 outputs go to a
// queue of its own in LDS, and whenever a queue holds 64 partial addresses
// the wave takes them through the next row, so no partial address leaves the
// compute unit and the stages need no launches of their own. What bounds it
// is the same as k_join; the three launches it replaces took 6-7 us each on
// the 1M-pair window, most of it start-up. The tables of rows 2..r-1 are
// copied to LDS when they fit, else read where they are.

constexpr uint32_t WALK_NB = 1u << JOIN_WALK_BITS;   // buckets per row, at most
constexpr uint32_t WALK_VAL_BYTES = 8192;       // bucket entries per row held in LDS
constexpr uint32_t WALK_QUEUE = 128;            // partial addresses per wave and stage

template <int R, bool TLDS>
struct JoinWalk {
  // LDS of one wave
  struct Wave {
    uint32_t incl[R - 2][64];
    uint16_t own[R - 2][OWN_MAX];
    uint32_t queue_a[R - 3][WALK_QUEUE], queue_c[R - 3][WALK_QUEUE];
  };
  const Geom &G;
  LDSP Wave *W;
  JoinTable<TLDS> T[R - 2];                     // rows 2..R-1
  uint32_t fill[R - 2];                         // queue fill of the stage into row i + 2
  uint32_t outs[R - 2];                         // outputs of the stage into row i + 2
  DevState *st;
  uint32_t *cand;
  size_t cand_cap;
  CandBuf *found;

  // 64 items (sub, c0), one per lane, into row ROW; every output goes on.
  template <int ROW>
  __device__ __forceinline__ void expand(uint32_t sub, uint32_t c0, bool valid) {
    constexpr int S = ROW - 2;
    const uint32_t lane = lane_id();
    const uint32_t M = (1u << (G.k - G.alpha)) - 1;
    uint32_t b0 = 0, cnt = 0;
    if (valid) {
      const uint32_t sh = G.shift[ROW];
      const uint32_t key = ((sh < 32 ? sub >> sh : 0u) ^ c0) & M;
      b0 = T[S].start(key);
      cnt = T[S].start(key + 1) - b0;
    }
    const uint32_t incl = wave_incl_scan(cnt);
    const uint32_t total = wave_lane(incl, 63);
    if (total == 0) return;
    const bool owned = total <= OWN_MAX;        // as in join_items
    if (owned) {
      for (uint32_t q = incl - cnt; q < incl; q++) W->own[S][q] = (uint16_t)lane;
    } else {
      W->incl[S][lane] = incl;
    }
    const int32_t my_base = (int32_t)b0 - (int32_t)(incl - cnt);
    lds_fence();
    for (uint32_t base = 0; base < total; base += 64) {
      const uint32_t slot = base + lane;
      const bool live = slot < total;
      const uint32_t sl = live ? slot : total - 1;
      uint32_t o = 0;
      if (owned) {
        o = W->own[S][sl];
      } else {
#pragma unroll
        for (uint32_t q = 32; q; q >>= 1)
          if (W->incl[S][o + q - 1] <= sl) o += q;
      }
      const int32_t ob = __builtin_amdgcn_ds_bpermute((int)(o << 2), my_base);
      const uint32_t osub = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(o << 2), (int)sub);
      const uint32_t oc0 = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(o << 2), (int)c0);
      bool ok = false;
      uint32_t a = 0;
      if (live) {
        const uint32_t j = (uint32_t)(ob + (int32_t)slot);
        const uint32_t top = (oc0 >> (G.k - G.alpha)) ^ T[S].top_bits(j);
        ok = extend_top(G, ROW, osub, top, &a);
        if (ROW == R - 1) ok = ok && hash_dh0(G, a) == oc0;
      }
      const unsigned long long mask = __ballot(ok);
      if (mask == 0) continue;
      const uint32_t n_ok = __popcll(mask), rank = lanes_below(mask);
      if constexpr (ROW == R - 1) {
        found->add(a, ok, st, cand, cand_cap);
      } else {
        outs[S] += n_ok;
        if (ok) {
          W->queue_a[S][fill[S] + rank] = a;
          W->queue_c[S][fill[S] + rank] = oc0;
        }
        fill[S] += n_ok;                        // at most 63 + 64
        lds_fence();
        if (fill[S] >= 64) {
          fill[S] -= 64;
          const uint2 p = take(S, fill[S] + lane);
          lds_fence();
          expand<ROW + 1>(p.x, p.y, true);
        }
      }
    }
    lds_fence();
  }
  __device__ __forceinline__ uint2 take(int s, uint32_t i) const {
    return make_uint2(W->queue_a[s][i], W->queue_c[s][i]);
  }
  // What is left in the queues, row by row.
  template <int ROW>
  __device__ __forceinline__ void flush() {
    if constexpr (ROW < R) {
      constexpr int S = ROW - 3;                // the queue of the stage before
      const uint32_t n = fill[S];
      if (n) {
        fill[S] = 0;
        const uint32_t lane = lane_id();
        const uint2 p = take(S, lane < n ? lane : 0);
        lds_fence();
        expand<ROW>(p.x, p.y, lane < n);
      }
      flush<ROW + 1>();
    }
  }
};

template <int R, bool TLDS>
__device__ __forceinline__ void join_walk(const Geom &G, const uint32_t *he, const uint32_t *bk_off,
                                          const uint32_t *bk_val, LDSP uint16_t *t_off,
                                          LDSP uint8_t *t_val, DevState *st, uint32_t *cand,
                                          size_t cand_cap,
                                          typename JoinWalk<R, TLDS>::Wave *waves,
                                          LDSP uint32_t *outs, CandBuf *found) {
  const uint32_t nb = 1u << (G.k - G.alpha), lane = lane_id();
  const uint32_t wib = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  JoinWalk<R, TLDS> J{G, lds_ptr(waves) + wib, {}, {}, {}, st, cand, cand_cap,
                        found};
#pragma unroll
  for (int s = 0; s < R - 2; s++)
    J.T[s] = JoinTable<TLDS>{t_off + s * (WALK_NB + 1), t_val + s * WALK_VAL_BYTES,
                             (LDSP uint16_t *)(t_val + s * WALK_VAL_BYTES),
                             bk_off + (size_t)(s + 2) * (nb + 1),
                             bk_val + ((size_t)(s + 2) << G.k), G.k - G.alpha, G.alpha > 8};
  // stage-1 items (x0, 64 entries of HE(1)) dealt to the waves of the grid
  // in turn
  const uint32_t h0 = st->he_count[0], h1 = st->he_count[1], nch = (h1 + 63) >> 6;
  const uint64_t n_items = (uint64_t)h0 * nch;
  const uint32_t n_waves = gridDim.x * (JOIN_THREADS / 64);
  const uint32_t *HE0 = he, *HE1 = he + (1u << G.k);
  for (uint64_t w = blockIdx.x + (uint64_t)gridDim.x * wib; w < n_items; w += n_waves) {
    const uint32_t x0 = (uint32_t)(w / nch), x1 = ((uint32_t)(w - (uint64_t)x0 * nch) << 6) + lane;
    const uint32_t c0 = HE0[x0];
    const uint32_t sub = c0 ^ HE1[x1 < h1 ? x1 : h1 - 1];     // BL(1)
    J.template expand<2>(sub, c0, x1 < h1);
  }
  J.template flush<3>();
  if (lane == 0)
#pragma unroll
    for (int s = 0; s < R - 3; s++)
      if (J.outs[s]) atomicAdd((uint32_t *)&outs[s], J.outs[s]);
}

template <int R>
__global__ __launch_bounds__(JOIN_THREADS) void k_join_walk(
    Geom G, uint32_t ways, uint32_t path, const uint32_t *__restrict__ he,
    const uint32_t *__restrict__ bk_off, const uint32_t *__restrict__ bk_val,
    DevState *__restrict__ st, uint32_t *__restrict__ cand, size_t cand_cap, double e_theta) {
  __shared__ uint16_t t_off[(R - 2) * (WALK_NB + 1)];
  __shared__ __attribute__((aligned(16))) uint8_t t_val[(R - 2) * WALK_VAL_BYTES];
  __shared__ typename JoinWalk<R, true>::Wave waves[JOIN_THREADS / 64];
  __shared__ uint32_t outs[R - 2];
  __shared__ CandBuf found;
  const bool chosen = !lattice_chosen(G, st, ways, path);
  search_begin(G, st, e_theta, chosen, 1);
  if (!chosen || no_zeros(G, st)) return;
  const uint32_t nb = 1u << (G.k - G.alpha);
  const bool wide = G.alpha > 8;
  uint32_t most = 0;
  for (int i = 2; i < R; i++) most = max(most, st->he_count[i]);
  const bool lds = G.alpha <= 16 && most * (wide ? 2 : 1) <= WALK_VAL_BYTES;
  if (threadIdx.x < R - 2) outs[threadIdx.x] = 0;
  if (threadIdx.x == 0) found.n = 0;
  if (lds) {
    for (int i = 2; i < R; i++) {
      const uint32_t *g_off = bk_off + (size_t)i * (nb + 1), *g_val = bk_val + ((size_t)i << G.k);
      uint16_t *off = t_off + (i - 2) * (WALK_NB + 1);
      uint8_t *val = t_val + (i - 2) * WALK_VAL_BYTES;
      const uint32_t h = st->he_count[i];
      for (uint32_t x = threadIdx.x; x <= nb; x += blockDim.x) off[x] = (uint16_t)g_off[x];
      for (uint32_t x = threadIdx.x; x < h; x += blockDim.x) {
        const uint32_t hi = g_val[x] >> (G.k - G.alpha);
        if (wide) reinterpret_cast<uint16_t *>(val)[x] = (uint16_t)hi;
        else val[x] = (uint8_t)hi;
      }
    }
  }
  __syncthreads();
  if (lds)
    join_walk<R, true>(G, he, bk_off, bk_val, lds_ptr(t_off), lds_ptr(t_val), st, cand, cand_cap,
                       waves, lds_ptr(outs), &found);
  else
    join_walk<R, false>(G, he, bk_off, bk_val, lds_ptr(t_off), lds_ptr(t_val), st, cand, cand_cap,
                        reinterpret_cast<typename JoinWalk<R, false>::Wave *>(waves),
                        lds_ptr(outs), &found);
  found.flush(st, cand, cand_cap);                      // holds barriers
  if (threadIdx.x < R - 3 && outs[threadIdx.x])
    atomicAdd(&st->n_out[threadIdx.x + 2], (unsigned long long)outs[threadIdx.x]);
}

// ------------------------------------------------------------ 6: estimate

constexpr uint32_t SMALL_SORT = 16384;                  // see the sort

template <int WPL>
__global__ __launch_bounds__(256) void k_estimate(Geom G, const uint32_t *__restrict__ sk,
                                                  const uint32_t *__restrict__ cand,
                                                  size_t cand_cap, DevState *__restrict__ st,
                                                  uint4 *__restrict__ spl, size_t spl_cap,
                                                  uint32_t *__restrict__ rank) {
  using S = LeShape<WPL>;
  if (rank)                                             // the sort's ranks, zeroed for it
    for (uint32_t i = blockIdx.x * 256 + threadIdx.x; i < SMALL_SORT; i += gridDim.x * 256)
      rank[i] = 0;
  if (st->saturated) return;
  const unsigned long long nc_all = st->n_cand;
  const uint64_t nc = nc_all < cand_cap ? nc_all : cand_cap;
  const uint32_t szmax = st->szmax;
  const double d = st->d;
  const uint32_t sub = threadIdx.x % S::LPL;
  // a block's candidates per trip: every wave takes the same trips, and the
  // block's reports of a trip take their places with one atomic (see CandBuf)
  __shared__ uint32_t reports[2];
  __shared__ unsigned long long place[2];
  if (threadIdx.x < 2) reports[threadIdx.x] = 0;
  __syncthreads();
  const uint64_t step = (uint64_t)gridDim.x * blockDim.x / S::LPL;
  uint32_t trip = 0;
  for (uint64_t block0 = (uint64_t)blockIdx.x * blockDim.x / S::LPL; block0 < nc;
       block0 += step, trip ^= 1) {
    const uint64_t base = block0 + (threadIdx.x & ~63u) / S::LPL;
    const uint64_t e = base + lane_id() / S::LPL;
    const bool valid = e < nc;
    const uint32_t a = valid ? cand[e] : 0u;
    uint32_t ones = 0;
    if (valid) {
      // the candidate's LE in each row; all rows' loads of a slice are
      // issued before any is used (rows past r read as all ones)
      const uint32_t c0 = hash_dh0(G, a);
      size_t le[R_MAX];
#pragma unroll
      for (uint32_t i = 0; i < R_MAX; i++)
        le[i] = (size_t)((i << G.k) | (i == 0 ? c0 : (bit_block(G, i, a) ^ c0))) * WPL;
      if constexpr (WPL >= 4) {
#pragma unroll 1
        for (int v = 0; v < S::VPL; v++) {
          uint4 q[R_MAX];
#pragma unroll
          for (uint32_t i = 0; i < R_MAX; i++) {
            q[i] = make_uint4(~0u, ~0u, ~0u, ~0u);
            if (i < G.r) q[i] = reinterpret_cast<const uint4 *>(sk + le[i])[v * S::LPL + sub];
          }
          uint4 acc = q[0];
#pragma unroll
          for (uint32_t i = 1; i < R_MAX; i++) {
            acc.x &= q[i].x; acc.y &= q[i].y; acc.z &= q[i].z; acc.w &= q[i].w;
          }
          ones += __popc(acc.x) + __popc(acc.y) + __popc(acc.z) + __popc(acc.w);
        }
      } else {
        for (int w = 0; w < WPL; w++) {
          uint32_t q[R_MAX];
#pragma unroll
          for (uint32_t i = 0; i < R_MAX; i++) {
            q[i] = ~0u;
            if (i < G.r) q[i] = sk[le[i] + w];
          }
          uint32_t acc = q[0];
#pragma unroll
          for (uint32_t i = 1; i < R_MAX; i++) acc &= q[i];
          ones += __popc(acc);
        }
      }
    }
    if constexpr (S::LPL > 1) {
#pragma unroll
      for (int m = S::LPL / 2; m >= 1; m >>= 1) ones += __shfl_xor(ones, m, 64);
    }
    const uint32_t sz = G.g - ones;
    const bool report = valid && sub == 0 && sz <= szmax;
    const unsigned long long rm = __ballot(report);
    uint32_t at = 0;
    if (lane_id() == 0 && rm) at = atomicAdd(&reports[trip], (uint32_t)__popcll(rm));
    at = wave_lane(at, 0) + lanes_below(rm);
    __syncthreads();
    if (threadIdx.x == 0) {
      place[trip] = reports[trip] ? atomicAdd(&st->n_spl, (unsigned long long)reports[trip]) : 0;
      reports[trip ^ 1] = 0;                            // the next trip's, not yet in use
    }
    __syncthreads();
    const unsigned long long slot = place[trip] + at;
    if (report && slot < spl_cap) {
      const double est = sz ? -(double)G.g * log((double)sz / d) : (double)INFINITY;
      const unsigned long long bits = __double_as_longlong(est);
      spl[slot] = make_uint4(a, sz, (uint32_t)bits, (uint32_t)(bits >> 32));
    }
  }
}

// ----------------------------------------------------------------- 7: sort
//
// Records with distinct 32-bit keys (the address in .x for uint4 records,
// the value itself for uint32) are sorted ascending by rank = the number
// of smaller keys; a last kernel places each record at its rank.
// Up to SMALL_SORT entries the ranks are counted by a (SMALL_SORT/256) x
// RANK_SPLIT grid, block (x, y) comparing 256 elements against the y-th
// slice of the keys and adding its counts to a zeroed rank array. 64
// slices rather than 8 spread a few thousand records over more blocks,
// each with a shorter compare loop: 11.3 -> 5.5 us for the 100M-pair
// window's 5.7k records (32 slices: 7.7 us).
// Longer lists: each tile of SORT_TILE keys is sorted in LDS (bitonic), and
// a record's rank is the sum over the tiles of the keys below its own, one
// binary search per tile: n * (n / SORT_TILE) * log2(SORT_TILE) steps
// rather than n^2 compares.
constexpr uint32_t RANK_SPLIT = 64;
constexpr uint32_t SORT_TILE = 4096;

template <typename T>
__device__ __forceinline__ uint32_t sort_key(const T &v);
template <>
__device__ __forceinline__ uint32_t sort_key<uint4>(const uint4 &v) { return v.x; }
template <>
__device__ __forceinline__ uint32_t sort_key<uint32_t>(const uint32_t &v) { return v; }

template <typename T>
__global__ __launch_bounds__(256) void k_rank_count(const T *__restrict__ in,
                                                    const unsigned long long *__restrict__ count,
                                                    size_t cap, uint32_t *__restrict__ rank) {
  __shared__ uint32_t keys[SMALL_SORT / RANK_SPLIT];
  const unsigned long long n_all = *count;
  const uint32_t n = (uint32_t)(n_all < cap ? n_all : cap);
  if (n > SMALL_SORT) return;
  const uint32_t j = blockIdx.x * 256 + threadIdx.x;
  if (blockIdx.x * 256 >= n) return;
  const uint32_t per = (n + RANK_SPLIT - 1) / RANK_SPLIT;
  const uint32_t k0 = blockIdx.y * per, k1 = k0 + per < n ? k0 + per : n;
  if (k0 >= k1) return;
  for (uint32_t t = threadIdx.x; t < k1 - k0; t += blockDim.x) keys[t] = sort_key<T>(in[k0 + t]);
  __syncthreads();
  if (j >= n) return;
  const uint32_t mine = sort_key<T>(in[j]);
  uint32_t c = 0;
  for (uint32_t t = 0; t < k1 - k0; t++) c += keys[t] < mine;
  if (c) atomicAdd(&rank[j], c);
}

// Longer lists, step 1 (block = tile): the tile's keys sorted in LDS and
// written to skeys (the last tile padded with 0xFFFFFFFF, which is below no
// key), and the tile's ranks zeroed.
template <typename T>
__global__ __launch_bounds__(1024) void k_tile_sort(const T *__restrict__ in,
                                                    const unsigned long long *__restrict__ count,
                                                    size_t cap, uint32_t *__restrict__ skeys,
                                                    uint32_t *__restrict__ rank) {
  __shared__ uint32_t key[SORT_TILE];
  const unsigned long long n_all = *count;
  const uint64_t n = n_all < cap ? n_all : cap;
  const uint64_t t0 = (uint64_t)blockIdx.x * SORT_TILE;
  if (n <= SMALL_SORT || t0 >= n) return;
  for (uint32_t i = threadIdx.x; i < SORT_TILE; i += blockDim.x) {
    const uint64_t e = t0 + i;
    key[i] = e < n ? sort_key<T>(in[e]) : 0xFFFFFFFFu;
    if (e < n) rank[e] = 0;
  }
  __syncthreads();
  // bitonic network: pair p of a stage joins i = 2p - (p mod stride) and
  // i + stride, ascending where bit `size` of i is clear
  for (uint32_t size = 2; size <= SORT_TILE; size <<= 1)
    for (uint32_t stride = size >> 1; stride; stride >>= 1) {
      for (uint32_t p = threadIdx.x; p < SORT_TILE / 2; p += blockDim.x) {
        const uint32_t i = 2 * p - (p & (stride - 1)), j = i + stride;
        const uint32_t a = key[i], b = key[j];
        if ((a > b) == ((i & size) == 0)) {
          key[i] = b;
          key[j] = a;
        }
      }
      __syncthreads();
    }
  for (uint32_t i = threadIdx.x; i < SORT_TILE; i += blockDim.x) skeys[t0 + i] = key[i];
}

// Longer lists, step 2: for every (element tile, key tile) pair, each
// element adds the keys of the key tile below its own to its rank. The
// grid strides over the pairs.
template <typename T>
__global__ __launch_bounds__(256) void k_tile_rank(const T *__restrict__ in,
                                                   const unsigned long long *__restrict__ count,
                                                   size_t cap, const uint32_t *__restrict__ skeys,
                                                   uint32_t *__restrict__ rank) {
  __shared__ uint32_t key[SORT_TILE];
  const unsigned long long n_all = *count;
  const uint64_t n = n_all < cap ? n_all : cap;
  if (n <= SMALL_SORT) return;
  const uint64_t nt = (n + SORT_TILE - 1) / SORT_TILE;
  for (uint64_t pr = blockIdx.x; pr < nt * nt; pr += gridDim.x) {
    const uint64_t xt = pr / nt, yt = pr - xt * nt;
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < SORT_TILE; i += blockDim.x)
      key[i] = skeys[yt * SORT_TILE + i];
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < SORT_TILE; i += blockDim.x) {
      const uint64_t e = xt * SORT_TILE + i;
      if (e >= n) break;
      const uint32_t x = sort_key<T>(in[e]);
      // keys below x: the largest prefix whose last key is below x
      uint32_t pos = 0;
#pragma unroll
      for (uint32_t step = SORT_TILE / 2; step; step >>= 1)
        if (key[pos + step - 1] < x) pos += step;
      pos += key[pos] < x;                                // pos <= SORT_TILE - 1 here
      if (pos) atomicAdd(&rank[e], pos);
    }
  }
}

// Each record to its counted rank.
template <typename T>
__global__ __launch_bounds__(256) void k_rank_place(const T *__restrict__ in,
                                                    const unsigned long long *__restrict__ count,
                                                    size_t cap, const uint32_t *__restrict__ rank,
                                                    T *__restrict__ out) {
  const unsigned long long n_all = *count;
  const uint64_t n = n_all < cap ? n_all : cap;
  for (uint64_t j = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; j < n;
       j += (uint64_t)gridDim.x * blockDim.x)
    out[rank[j]] = in[j];
}

// The first SMALL_SORT sort ranks to zero (a grid of SMALL_SORT threads).
__global__ __launch_bounds__(1024) void k_zero_ranks(uint32_t *rank) {
  rank[blockIdx.x * 1024 + threadIdx.x] = 0;
}

// rank must hold SMALL_SORT zeroed entries and room for cap; skeys room for
// cap rounded up to SORT_TILE. The kernels of the path a list does not take
// return at once.
template <typename T>
static void launch_sort(const T *in, const unsigned long long *count, size_t cap, T *out,
                        uint32_t *rank, uint32_t *skeys, int grid, hipStream_t st) {
  k_rank_count<T><<<dim3(SMALL_SORT / 256, RANK_SPLIT), 256, 0, st>>>(in, count, cap, rank);
  if (cap > SMALL_SORT) {
    const size_t tiles = (cap + SORT_TILE - 1) / SORT_TILE;
    k_tile_sort<T><<<(unsigned)tiles, 1024, 0, st>>>(in, count, cap, skeys, rank);
    k_tile_rank<T><<<grid * 2, 256, 0, st>>>(in, count, cap, skeys, rank);
  }
  const int pg = grid > (int)(SMALL_SORT / 256) ? grid : (int)(SMALL_SORT / 256);
  k_rank_place<T><<<pg, 256, 0, st>>>(in, count, cap, rank, out);
}

// ---------------------------------------------------------------- 8: publish

// The device state and the first min(n, cap) sorted records written straight
// into pinned host memory, so the caller waits once for the whole restore.
__global__ __launch_bounds__(256) void k_publish(const DevState *__restrict__ st,
                                                 const uint4 *__restrict__ recs, size_t recs_cap,
                                                 DevState *h_state, uint4 *h_recs,
                                                 size_t h_cap) {
  if (blockIdx.x == 0) {
    const uint32_t *src = reinterpret_cast<const uint32_t *>(st);
    uint32_t *dst = reinterpret_cast<uint32_t *>(h_state);
    for (uint32_t i = threadIdx.x; i < sizeof(DevState) / 4; i += blockDim.x) dst[i] = src[i];
  }
  if (!h_recs) return;
  uint64_t n = st->saturated ? 0 : st->n_spl;
  if (n > recs_cap) n = recs_cap;
  if (n > h_cap) n = h_cap;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (uint64_t)gridDim.x * blockDim.x)
    h_recs[i] = recs[i];
}

// Sort and publish in one launch of one block, for lists of at most
// SORT_ONE records: the keys sorted in LDS (bitonic), each record from its
// place to its rank. A longer list is left alone (only the state goes out):
// the host runs the restore again with the kernels above. Four launches took
// 11 us of kernels, and their gaps, for the 1M-pair window's 33 records.
constexpr uint32_t SORT_ONE = RESTORE_SORT_ONE;

__global__ __launch_bounds__(1024) void k_sort_publish(
    const DevState *__restrict__ st, const uint4 *__restrict__ in, size_t cap,
    uint4 *__restrict__ out, DevState *h_state, uint4 *h_recs, size_t h_cap) {
  __shared__ unsigned long long key[SORT_ONE];          // address over place
  const uint32_t tid = threadIdx.x;
  {
    const uint32_t *src = reinterpret_cast<const uint32_t *>(st);
    uint32_t *dst = reinterpret_cast<uint32_t *>(h_state);
    for (uint32_t i = tid; i < sizeof(DevState) / 4; i += 1024) dst[i] = src[i];
  }
  if (st->saturated || st->n_spl > SORT_ONE || st->n_spl > cap) return;
  const uint32_t n = (uint32_t)st->n_spl;
  uint32_t p2 = 2;
  while (p2 < n) p2 <<= 1;
  for (uint32_t i = tid; i < p2; i += 1024)
    key[i] = i < n ? ((unsigned long long)in[i].x << 32) | i : ~0ull;   // no record: above all
  __syncthreads();
  // Thread p compares pair p of a step (at most 1024). At a stride of up to
  // 64 a wave's 64 pairs are its own 128 keys, so steps between two such
  // strides need no barrier: 66 steps of a 1264-record list took 21 us with one
  // each, now 16.
  static_assert(SORT_ONE == 2048, "one pair per thread");
  for (uint32_t size = 2; size <= p2; size <<= 1)
    for (uint32_t stride = size >> 1; stride; stride >>= 1) {
      if (tid < p2 / 2) {
        const uint32_t i = 2 * tid - (tid & (stride - 1)), j = i + stride;
        const unsigned long long a = key[i], b = key[j];
        if ((a > b) == ((i & size) == 0)) {
          key[i] = b;
          key[j] = a;
        }
      }
      const uint32_t next = stride > 1 ? stride >> 1 : size;
      if (stride > 64 || next > 64) __syncthreads();
      else lds_fence();
    }
  __syncthreads();
  for (uint32_t i = tid; i < n; i += 1024) {
    const uint4 v = in[(uint32_t)key[i]];
    out[i] = v;
    if (h_recs && i < h_cap) h_recs[i] = v;
  }
}

// ------------------------------------------------------------ orchestration

// The join's launches: one walk where the bucket tables are small, else a
// stage per row.
template <int R>
static void launch_walk(const Geom &G, const RestoreBufs &B, double e_theta, hipStream_t st) {
  k_join_walk<R><<<B.jblk, JOIN_THREADS, 0, st>>>(G, lattice_ways(B.lat), B.cand_path, B.he,
                                                  B.bk_off, B.bk_val, B.st, B.cand, B.cand_cap,
                                                  e_theta);
}

template <int RW>
static void launch_pairs(const Geom &G, const RestoreBufs &B, uint32_t ways, double e_theta,
                         int grid, hipStream_t st) {
  const uint32_t rows = pair_rows(G);
  k_pairs<RW><<<grid > 3 ? grid / 4 : 1, PAIR_THREADS,
                rows * (4u << (G.k - 5)) + LAT_FOUND_BYTES + PAIR_QUEUE_BYTES, st>>>(
      G, B.lat.pair_off, B.lat.pair_z, B.lat.pair_rec, ways, B.cand_path, B.he, B.hotmask, B.st,
      B.cand, B.cand_cap, e_theta, rows);
}

static void launch_join(const Geom &G, const RestoreBufs &B, double e_theta, hipStream_t st) {
  const uint32_t r = G.r, jb = B.jblk, pth = B.cand_path;
  const uint32_t ways = lattice_ways(B.lat);
  if (B.walk) {
    switch (r) {
      case 4: launch_walk<4>(G, B, e_theta, st); break;
      case 5: launch_walk<5>(G, B, e_theta, st); break;
      case 6: launch_walk<6>(G, B, e_theta, st); break;
      case 7: launch_walk<7>(G, B, e_theta, st); break;
      default: launch_walk<8>(G, B, e_theta, st);
    }
  } else if (r == 3) {
    k_join<true, true><<<jb, JOIN_THREADS, 0, st>>>(G, ways, pth, 2, B.he, nullptr, nullptr, B.bk_off,
                                                    B.bk_val, B.st, nullptr, nullptr, 0, B.cand,
                                                    B.cand_cap, e_theta);
  } else {
    k_join<true, false><<<jb, JOIN_THREADS, 0, st>>>(G, ways, pth, 2, B.he, nullptr, nullptr,
                                                     B.bk_off, B.bk_val, B.st, B.part[0],
                                                     B.segc[0], B.seg_cap, B.cand, B.cand_cap,
                                                     e_theta);
    for (uint32_t row = 3; row < r; row++) {
      // stage 1 wrote part[0]; stage `row` reads part[(row-3)%2], writes the other
      const int ib = (row - 3) & 1, ob = ib ^ 1;
      if (row + 1 == r)
        k_join<false, true><<<jb, JOIN_THREADS, 0, st>>>(
            G, ways, pth, row, B.he, B.part[ib], B.segc[ib], B.bk_off, B.bk_val, B.st, nullptr,
            nullptr, B.seg_cap, B.cand, B.cand_cap, e_theta);
      else
        k_join<false, false><<<jb, JOIN_THREADS, 0, st>>>(
            G, ways, pth, row, B.he, B.part[ib], B.segc[ib], B.bk_off, B.bk_val, B.st, B.part[ob],
            B.segc[ob], B.seg_cap, B.cand, B.cand_cap, e_theta);
    }
  }
}

template <int WPL>
static hipError_t launch_wpl(const Geom &G, const uint32_t *sketch, const RestoreBufs &B,
                             uint32_t zhot, double e_theta, int estimate, int grid,
                             hipStream_t st, const hipEvent_t *marks) {
  const uint32_t r = G.r, k = G.k;
  const size_t n_le = (size_t)r << k;
  auto mark = [&](int i) {
    if (marks) (void)hipEventRecord(marks[i], st);
  };
  // a search is launched unless the sketch's setting or the expectation
  // rules it out (each returns at once unless it is the chosen one)
  const uint32_t ways = lattice_ways(B.lat);
  const bool lat = B.lat.ok && B.cand_path != 1;
  const bool lattice = lat && (B.expect == 0 || B.expect == 2);
  const bool pairs = lat && B.lat.pair_z && (B.expect == 0 || B.expect == 3);
  const bool join = !(B.lat.ok && B.cand_path == 2) && B.expect <= 1;
  mark(0);
  // 1-3: hot scan, HE(i), bucket tables (which serve only the join)
  const uint4 *lez4 = reinterpret_cast<const uint4 *>(B.lez);
  if (!B.lez) {
    k_restore_init<<<(int)((n_le / 32 + 255) / 256 < 256 ? (n_le / 32 + 255) / 256 : 256), 256, 0,
                     st>>>(B.st, B.hotmask, n_le / 32);
    using S = LeShape<WPL>;
    const uint64_t pass = (uint64_t)(256 / S::LPL) * HS_UNROLL;
    const uint64_t passes = (n_le + pass - 1) / pass;
    const uint64_t blocks = passes < (uint64_t)grid ? passes : (uint64_t)grid;
    const uint64_t chunk = (passes + blocks - 1) / blocks * pass;
    const int gs = (int)((n_le + chunk - 1) / chunk);
    k_hot_scan<WPL><<<gs, 256, 0, st>>>(G, sketch, zhot, B.hotmask, B.st, chunk);
    mark(1);
    k_rows<<<r, 1024, 0, st>>>(G, B.hotmask, B.he, B.bk_off, B.bk_cur, B.bk_val, B.st, join);
  } else {
    if constexpr (WPL >= 4 && WPL <= 256) {
      if (B.lez_stale) {
        const size_t n4 = n_le * (WPL / 4);
        const size_t blocks = (n4 + 1023) / 1024;
        k_zero_counts<WPL><<<(int)(blocks < (size_t)grid ? blocks : (size_t)grid), 256, 0, st>>>(
            G, reinterpret_cast<const uint4 *>(sketch), B.lez);
      }
    }
    // phase events take the larger sketches' kernels, one per phase
    if (k <= SCAN_ROWS_K && !(marks && k >= 12)) {
      k_scan_rows<<<r, 1024, 0, st>>>(G, lez4, zhot, B.hotmask, B.he, B.bk_off, B.bk_cur, B.bk_val,
                                      B.st, join);
      mark(1);
    } else {
      const int chunks = (int)(n_le / SCAN_CHUNK);
      k_hot_scan_lez<<<chunks, 256, 0, st>>>(G, lez4, zhot, B.hotmask, B.chunks);
      mark(1);
      k_compact<<<chunks, 256, 0, st>>>(G, B.hotmask, B.chunks, B.he, B.st);
      if (join) k_buckets<<<r - 2, 1024, 0, st>>>(G, B.he, B.bk_off, B.bk_cur, B.bk_val, B.st);
    }
  }
  mark(2);
  // 4-5: scalars and candidates
  if (lattice) {
    // the rows' bitmaps and the queues (above 64 KiB by the attribute that
    // prepare_restore_kernels sets); two blocks for each compute unit, each of
    // which first copies the bitmaps
    const uint32_t rows = lattice_rows(G), threads = lattice_threads(G, rows);
    k_lattice<<<grid > 3 ? grid / 4 : 1, threads, lattice_lds(G, rows, threads), st>>>(
        G, B.lat, ways, B.cand_path, B.he, B.hotmask, B.st, B.cand, B.cand_cap, e_theta, rows);
  }
  if (pairs) {
    const uint32_t rw = pair_rec_words(k);
    if (rw == 0) launch_pairs<0>(G, B, ways, e_theta, grid, st);
    else if (rw == 1) launch_pairs<1>(G, B, ways, e_theta, grid, st);
    else launch_pairs<2>(G, B, ways, e_theta, grid, st);
  }
  if (join) launch_join(G, B, e_theta, st);
  mark(3);
  if (!estimate) {
    mark(4);
    k_zero_ranks<<<SMALL_SORT / 1024, 1024, 0, st>>>(B.rank);
    launch_sort<uint32_t>(B.cand, &B.st->n_cand, B.cand_cap, B.cand_sorted, B.rank, B.skeys,
                          grid, st);
    k_publish<<<1, 256, 0, st>>>(B.st, nullptr, 0, B.h_state, nullptr, 0);
    mark(5);
    return hipGetLastError();
  }
  // 6: estimate and report (its first blocks clear the sort ranks)
  k_estimate<WPL><<<grid, 256, 0, st>>>(G, sketch, B.cand, B.cand_cap, B.st, B.spl,
                                        B.spl_cap, B.sort_one ? nullptr : B.rank);
  mark(4);
  // 7-8: sort; state and records to the host
  if (B.sort_one) {
    k_sort_publish<<<1, 1024, 0, st>>>(B.st, B.spl, B.spl_cap, B.spl_sorted, B.h_state, B.h_recs,
                                       B.h_recs_cap);
  } else {
    launch_sort<uint4>(B.spl, &B.st->n_spl, B.spl_cap, B.spl_sorted, B.rank, B.skeys, grid, st);
    k_publish<<<16, 256, 0, st>>>(B.st, B.spl_sorted, B.spl_cap, B.h_state, B.h_recs,
                                  B.h_recs_cap);
  }
  mark(5);
  return hipGetLastError();
}

hipError_t prepare_restore_kernels() {
  // the walk reads its dynamic LDS from address 0
  hipFuncAttributes lattice;
  hipError_t e = hipFuncGetAttributes(&lattice, reinterpret_cast<const void *>(k_lattice));
  if (e == hipSuccess && lattice.sharedSizeBytes != 0) e = hipErrorInvalidConfiguration;
  if (e == hipSuccess)
    e = hipFuncSetAttribute(reinterpret_cast<const void *>(k_lattice),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)LATTICE_LDS_MAX);
  for (const void *f : {reinterpret_cast<const void *>(k_pairs<0>),
                        reinterpret_cast<const void *>(k_pairs<1>),
                        reinterpret_cast<const void *>(k_pairs<2>)})
    if (e == hipSuccess)
      e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 81920);
  return e;
}

hipError_t launch_restore(const Geom &G, const uint32_t *sketch, const RestoreBufs &B,
                          uint32_t zhot, double e_theta, int estimate, int grid,
                          hipStream_t st, const hipEvent_t *marks) {
  switch (G.wpl) {
    case 1: return launch_wpl<1>(G, sketch, B, zhot, e_theta, estimate, grid, st, marks);
    case 2: return launch_wpl<2>(G, sketch, B, zhot, e_theta, estimate, grid, st, marks);
    case 4: return launch_wpl<4>(G, sketch, B, zhot, e_theta, estimate, grid, st, marks);
    case 8: return launch_wpl<8>(G, sketch, B, zhot, e_theta, estimate, grid, st, marks);
    case 16: return launch_wpl<16>(G, sketch, B, zhot, e_theta, estimate, grid, st, marks);
    case 32: return launch_wpl<32>(G, sketch, B, zhot, e_theta, estimate, grid, st, marks);
    case 64: return launch_wpl<64>(G, sketch, B, zhot, e_theta, estimate, grid, st, marks);
    case 128: return launch_wpl<128>(G, sketch, B, zhot, e_theta, estimate, grid, st, marks);
    case 256: return launch_wpl<256>(G, sketch, B, zhot, e_theta, estimate, grid, st, marks);
    case 512: return launch_wpl<512>(G, sketch, B, zhot, e_theta, estimate, grid, st, marks);
    case 1024: return launch_wpl<1024>(G, sketch, B, zhot, e_theta, estimate, grid, st, marks);
    case 2048: return launch_wpl<2048>(G, sketch, B, zhot, e_theta, estimate, grid, st, marks);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace ddhf
