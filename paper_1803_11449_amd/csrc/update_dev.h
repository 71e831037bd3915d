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
__device__ __forceinline__ void st2(GMEM uint2 *p, uint2 x) {
  v2u v;
  v.x = x.x; v.y = x.y;
  *reinterpret_cast<GMEM v2u *>(p) = v;
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
// (ts: every index, B0 among them, times 2^ts)
template <int R>
__device__ __forceinline__ void codes_of(const Geom &G, uint32_t x, uint32_t B0, uint32_t *B,
                                         uint32_t ts = 0) {
  B[0] = B0;
#pragma unroll
  for (int row = 1; row < R; row++)
    B[row] = ((uint32_t)row << (G.k + G.log2g + ts)) |
             (B0 ^ (bit_block(G, row, x) << (G.log2g + ts)));
}

// Four times the tile of bit index S (see bin_tile): the byte offset of its
// entry in an array of words.
__device__ __forceinline__ uint32_t tile4_of(uint32_t S) {
  return (__umul24(S >> 18, 52429u) >> 16) & ~3u;
}
// A bit set as the scatters keep it, its tile over its code (up to 2048
// tiles): one multiply-add on the index, S - t * BIN_TILE_BITS + t * 2^CODE_BITS.
__device__ __forceinline__ uint32_t tile_code(uint32_t S, uint32_t t4) {
  return S + __umul24(t4, ((1u << CODE_BITS) - BIN_TILE_BITS) / 4);
}
__device__ __forceinline__ uint32_t tile4_of_code(uint32_t v) {
  return (v >> (CODE_BITS - 2)) & ~3u;
}
// The LDS word at a byte offset from base.
__device__ __forceinline__ uint32_t *at4(uint32_t *base, uint32_t bytes) {
  return reinterpret_cast<uint32_t *>(reinterpret_cast<char *>(base) + bytes);
}
// Three of them to a code word. Bits above a field that the next field or
// the word's end does not take are left as they come: the apply masks them.
__device__ __forceinline__ uint2 code_word(uint32_t a, uint32_t b, uint32_t c) {
  return make_uint2((a & CODE_MASK) | (b << CODE_BITS),
                    __builtin_amdgcn_ubfe(b, 32 - CODE_BITS, 2 * CODE_BITS - 32) |
                        (c << (2 * CODE_BITS - 32)));
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
// 1.0), 139 -> 79 us for 15 us; in the regions, 100M pairs (Zipf 1.0, 128
// slots) apply and merge 396 -> 326 us, 190M pairs (Zipf 1.1, 64 slots) 745 ->
// 515 us, for about a tenth of the scatter. A table shared by the blocks of an XCD drops
// more (15M pairs: apply 66 us) but its busiest lines are read by every
// wave: the scatter went from 85 to 650 us and more.
//
// Slots are claimed in a block's first FILT_CLAIM batches only (in every
// batch it cost twice as much). The next batch's pairs of owned sources are
// counted, and a block where they are fewer than one in FILT_WORTH goes on
// without the filter, whose lookups take about a tenth of the scatter. Not
// the repeats: a source with a tenth of a block's pairs has set few of a
// large estimator's bits by the second batch, and most of them by the tenth.
// Going by those, 50M pairs (a power law, g = 1024, k = 15) took 710 us, 30M
// (Zipf 0.9, g = 512, k = 17) 351, and by the owned ones 505 and 284. Asked
// for one in eight instead of 32, 50M pairs with a tenth of one source (g =
// 2048) took 842 us, not 500.
//
// An unowned slot holds a source that belongs to another slot, so that one
// compare tells a pair's source from every other owner and from none.
constexpr uint32_t FILT_CLAIM = 1;
constexpr uint32_t FILT_WORTH = 32;

template <uint32_t WORDS>
struct Filter {
  static constexpr uint32_t SLOTS = WORDS / 32;         // at most, for LEs of 32 words and less
  uint32_t bits[WORDS], own[SLOTS], last[SLOTS], owned;

  // slots - 1: as many as SLOTS and the words allow (WORDS >= 2048, the
  // largest LE)
  __device__ __forceinline__ static uint32_t mask(const Geom &G) {
    return (G.wpl <= 32 ? SLOTS : WORDS / G.wpl) - 1;
  }
  // The source an unowned slot holds: 0, or in 0's own slot the next one of
  // another (there is no other with one slot: 0 then passes for its owner,
  // and other sources may claim the slot, whose bits are then theirs and
  // source 0's alike, so one-slot filters are not used). All lanes of a wave,
  // each of which tries one: with few slots, or a hash whose first values lie
  // close, there may be tens to pass over (38 for the default seed at g =
  // 65,536; one after the other in every wave they took 21 us of a scatter).
  __device__ __forceinline__ static uint32_t stranger(const Geom &G) {
    const uint32_t m = mask(G), s0 = hash_dh0(G, 0) & m, lane = threadIdx.x & 63;
    uint32_t z = 1;
    for (; m && z < 4096; z += 64) {
      const unsigned long long other = __ballot((hash_dh0(G, z + lane) & m) != s0);
      if (other) return z + (uint32_t)__builtin_ctzll(other);
    }
    return z;
  }
  // Whether the sketch's LEs leave slots to tell apart.
  __device__ __forceinline__ static bool fits(const Geom &G) {
    return mask(G) != 0 && (hash_dh0(G, stranger(G)) & mask(G)) != (hash_dh0(G, 0) & mask(G));
  }
  __device__ __forceinline__ void clear(const Geom &G) {
    const uint32_t z = stranger(G), s0 = hash_dh0(G, 0) & mask(G);
    for (uint32_t i = threadIdx.x; i < WORDS; i += blockDim.x) bits[i] = 0;
    for (uint32_t i = threadIdx.x; i < SLOTS; i += blockDim.x)
      own[i] = last[i] = i == s0 ? z : 0u;
    if (threadIdx.x == 0) owned = 0;
  }
  // Which of N pairs (sources x, row-0 bit indexes B0) repeat an earlier one:
  // bit k of the result. Every lane has N pairs of its own (a pair given
  // twice drops the one that is written). The lookups, and the
  // test-and-sets, of all N go out together; a lane without an owned slot
  // sets nothing, in any word. A slot's bits are the low bits of its source's
  // row-0 bit index: slot over H1's bit.
  template <int N>
  __device__ __forceinline__ uint32_t repeats(const Geom &G, const uint32_t *x,
                                              const uint32_t *B0, uint32_t batch) {
    const uint32_t ms = mask(G), mb = (ms << G.log2g) | (G.g - 1);
    uint32_t o[N], seen = 0;
#pragma unroll
    for (int k = 0; k < N; k++) o[k] = own[(B0[k] >> G.log2g) & ms];
    if (batch < FILT_CLAIM) {                           // uniform over the block
      const uint32_t z = stranger(G), s0 = hash_dh0(G, 0) & ms;
#pragma unroll
      for (int k = 0; k < N; k++) {
        const uint32_t slot = (B0[k] >> G.log2g) & ms, unowned = slot == s0 ? z : 0u;
        if (o[k] == unowned) {
          if (last[slot] == x[k]) {
            const uint32_t old = atomicCAS(&own[slot], unowned, x[k]);
            o[k] = old == unowned ? x[k] : old;
          } else {
            last[slot] = x[k];
          }
        }
      }
    }
    uint32_t old[N], m[N];
#pragma unroll
    for (int k = 0; k < N; k++) {
      m[k] = o[k] == x[k] ? 1u << (B0[k] & 31) : 0u;
      old[k] = atomicOr(&bits[(B0[k] & mb) >> 5], m[k]);
    }
#pragma unroll
    for (int k = 0; k < N; k++) seen |= (old[k] & m[k]) ? 1u << k : 0u;
    if (batch == FILT_CLAIM) {
      uint32_t mine = 0;
#pragma unroll
      for (int k = 0; k < N; k++) mine += m[k] ? 1u : 0u;
      atomicAdd(&owned, mine);
    }
    return seen;
  }
  // After a barrier that follows batch FILT_CLAIM: whether to go on.
  __device__ __forceinline__ bool useful(uint32_t pairs) const {
    return owned * FILT_WORTH >= pairs;
  }
};

// Two 16-bit ranks per register (q is a compile-time index after unrolling).
__device__ __forceinline__ void put_rank(uint32_t *rk2, int q, uint32_t r) {
  if (q & 1) rk2[q >> 1] |= r << 16;
  else rk2[q >> 1] = r;
}
__device__ __forceinline__ uint32_t get_rank(const uint32_t *rk2, int q) {
  return (q & 1) ? rk2[q >> 1] >> 16 : rk2[q >> 1] & 0xFFFFu;
}

// The two steps of a scatter batch that touch every code. The scatters are
// bound by vector instructions and LDS cycles about alike, so both are
// written for few of the former: byte offsets instead of indexes, LDS arrays
// whose addresses fit an instruction's offset (the arrays that are looked up
// come first in LDS, the sorted codes last), one multiply-add for tile and
// code: 33 -> 23 vector instructions per code, 604 -> 575 us for the 100M-pair
// window's scatter with its filter. (With the vector ALU at about half its
// issue slots and LDS at about half its cycles, what is left is that the
// waves of a block go through the phases together.) SPLIT: values are tile_code's, else bit indexes.
//
// Codes of the live pairs (bit k of live; x: sources, B0: row-0 bit indexes),
// and each one's rank inside its tile's run: an LDS atomic that returns it
// (a plain count here and a returning placement cursor in the grouping was
// slower: 692 against 608 us for the 100M-pair window).
template <int R, int PPT, bool SPLIT>
__device__ __forceinline__ void rank_codes(const Geom &G, const uint32_t *x, const uint32_t *B0,
                                           uint32_t live, uint32_t ts, uint32_t *cnt, uint32_t *v,
                                           uint32_t *rk2) {
#pragma unroll
  for (int k = 0; k < PPT; k++) {
    if ((live >> k) & 1u) {
      uint32_t B[R];
      codes_of<R>(G, x[k], B0[k] << ts, B, ts);
#pragma unroll
      for (int row = 0; row < R; row++) {
        const int q = k * R + row;
        const uint32_t t4 = tile4_of(B[row]);
        v[q] = SPLIT ? tile_code(B[row], t4) : B[row];
        put_rank(rk2, q, atomicAdd(at4(cnt, t4), 1u));
      }
    }
  }
}
// The codes grouped by tile: each to its run's start (lofs, in codes) plus its
// rank.
template <int R, int PPT, bool SPLIT, typename L>
__device__ __forceinline__ void group_codes(uint32_t live, const uint32_t *v, const uint32_t *rk2,
                                            L *lofs, uint32_t *sorted) {
#pragma unroll
  for (int k = 0; k < PPT; k++) {
    if ((live >> k) & 1u) {
#pragma unroll
      for (int q = k * R; q < (k + 1) * R; q++) {
        const uint32_t t4 = SPLIT ? tile4_of_code(v[q]) : tile4_of(v[q]);
        const uint32_t o = *reinterpret_cast<L *>(reinterpret_cast<char *>(lofs) +
                                                  t4 / (4 / sizeof(L)));
        sorted[o + get_rank(rk2, q)] = v[q];
      }
    }
  }
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

// The three codes of a word into the LDS tile (ts: codes are stored times
// 2^ts). Per code: its word's byte offset (bits 5..20 of the code, times 4)
// and its bit (a shift takes the low 5 bits of its count).
__device__ __forceinline__ void or_code(uint32_t *tile, uint32_t c, uint32_t ts) {
  const uint32_t bytes = (CODE_MASK >> (5 + ts)) << 2;
  uint32_t *w =
      reinterpret_cast<uint32_t *>(reinterpret_cast<char *>(tile) + ((c >> (3 + ts)) & bytes));
  atomicOr(w, 1u << ((c >> ts) & 31));
}
__device__ __forceinline__ void or_word(uint32_t *tile, uint2 w, uint32_t ts = 0) {
  or_code(tile, w.x, ts);
  or_code(tile, __builtin_amdgcn_alignbit(w.y, w.x, CODE_BITS), ts);
  or_code(tile, w.y >> (2 * CODE_BITS - 32), ts);
}

}  // namespace ddhf
