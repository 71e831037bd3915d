// Device helpers shared by the update kernels (update.hip, linear.hip):
// global-memory accesses, job lookup, the codes of a pair and the pieces of
// the tile pass.
#pragma once

#include "ddhf_internal.h"

namespace ddhf {

// Pointers read from a job table are generic to the compiler, which then
// emits flat loads and stores; those count against the LDS wait counter too,
// so every wait for an LDS result would also wait for all memory traffic in
// flight. Every job buffer is device global memory: say so.
#define GMEM __attribute__((address_space(1)))
template <typename T>
__device__ __forceinline__ GMEM T *gmem(T *p) {
  return (GMEM T *)p;
}
// HIP's vector structs cannot be copied out of a qualified pointer: 8- and
// 16-byte accesses go through the compiler's own vector types.
typedef uint32_t v2u __attribute__((ext_vector_type(2)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint2 ld2(const GMEM uint2 *p) {
  const v2u v = *reinterpret_cast<const GMEM v2u *>(p);
  return make_uint2(v.x, v.y);
}
__device__ __forceinline__ uint4 ld4(const GMEM uint4 *p) {
  const v4u v = *reinterpret_cast<const GMEM v4u *>(p);
  return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void st4(GMEM uint4 *p, uint4 x) {
  v4u v;
  v.x = x.x; v.y = x.y; v.z = x.z; v.w = x.w;
  *reinterpret_cast<GMEM v4u *>(p) = v;
}

// ------------------------------------------------------------ job lookup

__device__ __forceinline__ uint32_t job_of_block(const UpdJob *jobs, uint32_t nj, uint32_t b) {
  uint32_t lo = 0, hi = nj;
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) >> 1;
    if (jobs[mid].blk0 <= b) lo = mid; else hi = mid;
  }
  return lo;
}

__device__ __forceinline__ uint32_t job_of_tile(const UpdJob *jobs, uint32_t nj, uint32_t t) {
  uint32_t lo = 0, hi = nj;
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) >> 1;
    if (jobs[mid].tile0 <= t) lo = mid; else hi = mid;
  }
  return lo;
}

__device__ __forceinline__ uint32_t job_of_item(const UpdJob *jobs, uint32_t nj, uint32_t it) {
  uint32_t lo = 0, hi = nj;
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) >> 1;
    if (jobs[mid].item0 <= it) lo = mid; else hi = mid;
  }
  return lo;
}

constexpr uint32_t CODE_BITS = 21;
constexpr uint32_t CODE_MASK = (1u << CODE_BITS) - 1;

// Row 0's bit index of a pair (its cell over its bit), and every row's from
// it: the rows share H1's bit, and eq. (2)'s XOR is one on the index.
__device__ __forceinline__ uint32_t pair_code0(const Geom &G, uint2 p) {
  return (hash_dh0(G, p.x) << G.log2g) | hash_h1(G, p.y);
}
template <int R>
__device__ __forceinline__ void codes_of(const Geom &G, uint32_t x, uint32_t B0, uint32_t *B) {
  B[0] = B0;
#pragma unroll
  for (int row = 1; row < R; row++)
    B[row] = ((uint32_t)row << (G.k + G.log2g)) | (B0 ^ (bit_block(G, row, x) << G.log2g));
}

// A pair's bit set in every row, as sketch bit indexes (< 2^32: a binned
// sketch has at most BIN_MAX tiles).
template <int R>
__device__ __forceinline__ void pair_codes(const Geom &G, uint2 p, uint32_t *B) {
  codes_of<R>(G, p.x, pair_code0(G, p), B);
}

// ------------------------------------------------------------ repeat filter

// A (source, bit) pair that a block has seen before sets only bits that the
// block's words set already, and under skewed traffic a few sources send
// most pairs. Each scatter block keeps, in LDS, a bitmap of the bits seen for
// as many sources as fit in WORDS words: a slot belongs for the whole launch
// to the first source that comes to it twice in a row (which leaves most
// slots to the sources with the most pairs), and a pair of a slot's owner
// whose bit is already set is dropped. Dropping repeats takes out most of
// the words that pile up on the busiest source's tiles, whose workgroups
// the apply pass otherwise waits for: 4M pairs at g = 512, r = 4 (Zipf 1.1),
// apply 73 -> 27 us for 4 us more in the scatter; 15M pairs at k = 16 (Zipf
// 1.0), 139 -> 79 us for 15 us. A table shared by the blocks of an XCD drops
// more (15M pairs: apply 66 us) but its busiest lines are read by every
// wave: the scatter went from 85 to 650 us and more.
//
// Slots are claimed in a block's first FILT_CLAIM batches only (in every
// batch it cost twice as much). The next batch's drops are counted, and a
// block where fewer than one pair in 32 repeats goes on without the filter.
constexpr uint32_t FILT_FREE = 0xFFFFFFFFu;             // no source: passes unfiltered
constexpr uint32_t FILT_CLAIM = 1;

template <uint32_t WORDS>
struct Filter {
  static constexpr uint32_t SLOTS = WORDS / 32;         // at most, for LEs of 32 words and less
  uint32_t bits[WORDS + 64], own[SLOTS], last[SLOTS], drops;

  __device__ __forceinline__ void clear() {
    for (uint32_t i = threadIdx.x; i < WORDS + 64; i += blockDim.x) bits[i] = 0;
    for (uint32_t i = threadIdx.x; i < SLOTS; i += blockDim.x) own[i] = last[i] = FILT_FREE;
    if (threadIdx.x == 0) drops = 0;
  }
  // Which of N pairs (sources x, row-0 bit indexes B0) repeat an earlier one:
  // bit k of the result. live: the pairs that exist. The lookups, and the
  // test-and-sets, of all N go out together: a lane without an owned slot
  // sets nothing in a word of its own.
  template <int N>
  __device__ __forceinline__ uint32_t repeats(const Geom &G, const uint32_t *x,
                                              const uint32_t *B0, uint32_t live,
                                              uint32_t batch) {
    const uint32_t mask = (G.wpl <= 32 ? SLOTS : WORDS / G.wpl) - 1;   // WORDS >= 2048, the largest LE
    uint32_t o[N], seen = 0;
#pragma unroll
    for (int k = 0; k < N; k++) o[k] = own[(B0[k] >> G.log2g) & mask];
    if (batch < FILT_CLAIM) {                           // uniform over the block
#pragma unroll
      for (int k = 0; k < N; k++) {
        const uint32_t slot = (B0[k] >> G.log2g) & mask;
        if (((live >> k) & 1u) && x[k] != FILT_FREE && o[k] == FILT_FREE) {
          if (last[slot] == x[k]) {
            const uint32_t old = atomicCAS(&own[slot], FILT_FREE, x[k]);
            o[k] = old == FILT_FREE ? x[k] : old;
          } else {
            last[slot] = x[k];
          }
        }
      }
    }
    uint32_t old[N], m[N];
#pragma unroll
    for (int k = 0; k < N; k++) {
      const uint32_t slot = (B0[k] >> G.log2g) & mask, bit = B0[k] & (G.g - 1);
      const bool mine = o[k] == x[k] && x[k] != FILT_FREE && ((live >> k) & 1u);
      m[k] = mine ? 1u << (bit & 31) : 0u;
      old[k] = atomicOr(&bits[mine ? slot * G.wpl + (bit >> 5) : WORDS + (threadIdx.x & 63)], m[k]);
    }
#pragma unroll
    for (int k = 0; k < N; k++) seen |= (old[k] & m[k]) ? 1u << k : 0u;
    if (batch == FILT_CLAIM) atomicAdd(&drops, (uint32_t)__popc(seen));
    return seen;
  }
  // After a barrier that follows batch FILT_CLAIM: whether to go on.
  __device__ __forceinline__ bool useful(uint32_t pairs) const { return drops * 32 >= pairs; }
};

// Two 16-bit ranks per register (q is a compile-time index after unrolling).
__device__ __forceinline__ void put_rank(uint32_t *rk2, int q, uint32_t r) {
  if (q & 1) rk2[q >> 1] |= r << 16;
  else rk2[q >> 1] = r;
}
__device__ __forceinline__ uint32_t get_rank(const uint32_t *rk2, int q) {
  return (q & 1) ? rk2[q >> 1] >> 16 : rk2[q >> 1] & 0xFFFFu;
}

// Zero count of the LE that holds sketch words [w, w+4) (v), when the LE's
// W = wpl words are spread over W/4 consecutive lanes, each with one 16-byte
// vector (4 <= W <= 256): the lanes' one-counts are summed across the group
// and its first lane writes g - ones. Every lane of a group must call it.
__device__ __forceinline__ void le_zeros(const Geom &G, GMEM uint32_t *lez, size_t w, uint4 v) {
  const uint32_t L = G.wpl / 4;                         // lanes per LE, 1..64
  uint32_t ones = __popc(v.x) + __popc(v.y) + __popc(v.z) + __popc(v.w);
  for (uint32_t m = L >> 1; m >= 1; m >>= 1) ones += __shfl_xor(ones, (int)m, 64);
  if ((w / 4) % L == 0) lez[w / G.wpl] = G.g - ones;
}

// The three codes of a word into the LDS tile. Per code: its word's byte
// offset (bits 5..20 of the code, times 4) and its bit (a shift takes the low
// 5 bits of its count).
__device__ __forceinline__ void or_code(uint32_t *tile, uint32_t c) {
  constexpr uint32_t BYTES = (CODE_MASK >> 5) << 2;
  uint32_t *w = reinterpret_cast<uint32_t *>(reinterpret_cast<char *>(tile) + ((c >> 3) & BYTES));
  atomicOr(w, 1u << (c & 31));
}
__device__ __forceinline__ void or_word(uint32_t *tile, uint2 w) {
  or_code(tile, w.x);
  or_code(tile, __builtin_amdgcn_alignbit(w.y, w.x, CODE_BITS));
  or_code(tile, w.y >> (2 * CODE_BITS - 32));
}

}  // namespace ddhf
