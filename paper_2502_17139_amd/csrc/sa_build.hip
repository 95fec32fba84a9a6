// Suffix-array construction on gfx950 (fc_datastore_build, fc_store_prepare).
//
// The datastore is indexed for exact suffix matching with a suffix array
// (Section III-A, after Manber and Myers; datastore organisation in
// Section IV-A).  Construction is prefix doubling, which is what Manber and
// Myers' own construction does: a first sort of all suffixes by passes over
// whole lists, then sorts inside the groups that are still tied, most of them
// in LDS:
//
//   round 0  key(i) = the first 3 tokens of suffix i, each as token+1 in as
//            many bits as the largest token + 1 needs (at most 17), with 0
//            past the end, so a suffix that ends first sorts first; all n
//            suffixes are sorted.
//   round r  (h = 3 * 2^(r-1)) only suffixes still tied with another are
//            re-sorted, each inside its group of equal h-token prefixes, by
//            rank[i+h] + 1 (0 past the end), where rank[i] is the suffix-array
//            index at which i's group starts (Larsson and Sadakane's group
//            numbering).  Suffixes whose group becomes a singleton drop out.
//   a suffix whose group becomes a singleton has its final index, rank[i],
//   and sa[rank[i]] = i is written in that round (in sorted order, so at
//   nearly sequential addresses).
//
// Round 0's keys are sorted by a global digit histogram followed by one
// "onesweep" pass per 8-bit digit (Adinets and Merrill 2022): a workgroup takes
// a tile of 4,096 keys (its tile id from an atomic ticket, so tiles start in
// order), ranks them stably inside the tile with wave ballots, publishes
// per-digit tile counts and resolves its global offsets by decoupled look-back
// over the earlier tiles, stages the tile in LDS in digit order, and writes it
// out in runs.  The later rounds sort inside the groups
// (see "sorting inside groups").
//
// After each sort, head flags of the new and old groups are turned into
// group starts with a three-phase scan (tile partials, one-workgroup scan of
// the partials, per-tile apply), which also compacts the still-tied suffixes.
// Both tile passes run wave-striped (a wave takes 1,024 consecutive sorted
// positions, 64 at a time), so every load and store of a wave is coalesced
// except the rank scatter itself, which is indexed by suffix.  Where the
// rank array outgrows the MALL (64M suffixes or more), a random 4-byte write
// costs a 32-byte memory write, so the new ranks are split into windows of
// the rank array and put together there (RankParts).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fastcoder.h"
#include "fc_device.h"
#include "fc_host.h"

namespace {

constexpr int kSortThreads = 256;
constexpr int kSortItems = 16;
constexpr int kSortTile = kSortThreads * kSortItems;  // 4,096 keys per tile
constexpr int kRadix = 256;
constexpr int kMaxDigits = 8;
constexpr int kSegThreads = 256;
constexpr int kSegItems = 16;
constexpr int kSegTile = kSegThreads * kSegItems;
constexpr int kScanThreads = 1024;
constexpr int kMaxRounds = 40;
constexpr int kHistBlocks = 2048;
constexpr uint32_t kBigKeysBlocks = 2048;
constexpr uint32_t kBigPassBlocks = 1024;  // resident: four tiles per CU
constexpr uint32_t kSpinLimit = 1u << 22;
constexpr int kLookWindow = 2;  // earlier tiles examined per look-back step (with the counts
                                // published early, wider windows only add loads)

enum class Mode { kPlain, kBatched, kExtend };

constexpr uint64_t kFlagAgg = 1ull << 46;
constexpr uint64_t kFlagInc = 2ull << 46;
constexpr uint64_t kFlagMask = 3ull << 46;
constexpr uint64_t kCountMask = (1ull << 46) - 1;

__device__ __forceinline__ uint64_t pack_status(uint32_t epoch, uint64_t flag, uint64_t count) {
  return ((uint64_t)epoch << 48) | flag | count;
}

// A value that is the same in every lane, in a scalar register (what is read
// from LDS otherwise counts as different per lane, and so does all that
// follows from it).
__device__ __forceinline__ uint32_t uniform(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_readfirstlane((int)x);
}

// ---------------------------------------------------------------- keys ----

// Digit histogram of one workgroup in LDS, added to the global one at the end.
struct LdsHist {
  uint32_t (*s)[kRadix];
  __device__ void zero() const {
    for (int i = threadIdx.x; i < kMaxDigits * kRadix; i += blockDim.x) (&s[0][0])[i] = 0;
    __syncthreads();
  }
  __device__ void add(uint64_t key, int digits) const {
    for (int d = 0; d < digits; ++d) atomicAdd(&s[d][(uint32_t)(key >> (8 * d)) & 0xFF], 1u);
  }
  __device__ void flush(int digits, uint32_t* __restrict__ hist) const {
    __syncthreads();
    for (int i = threadIdx.x; i < digits * kRadix; i += blockDim.x) {
      const uint32_t v = (&s[0][0])[i];
      if (v) atomicAdd(&hist[i], v);
    }
  }
};

// Batched build: position i belongs to the segment r with off[r] <= i <
// off[r+1] (the last r with off[r] <= i, so empty segments are skipped).
__device__ __forceinline__ uint32_t segment_of(const uint64_t* __restrict__ off, uint32_t R, uint64_t i) {
  uint32_t lo = 0, hi = R - 1;
  while (lo < hi) {
    const uint32_t mid = (lo + hi + 1) >> 1;
    if (off[mid] <= i) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// The same from segment r on (off[r] <= i), in steps that double: few reads for
// a segment near r, and never more than about twice a binary search's however
// many empty segments lie between.
__device__ __forceinline__ uint32_t segment_from(const uint64_t* __restrict__ off, uint32_t R, uint32_t r, uint64_t i) {
  uint32_t step = 1;
  while (step < R - r && off[r + step] <= i) {
    r += step;
    step *= 2;
  }
  uint32_t lo = r, hi = (step < R - r ? r + step : R) - 1;
  while (lo < hi) {
    const uint32_t mid = (lo + hi + 1) >> 1;
    if (off[mid] <= i) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// One bit per position that starts a segment (bits zeroed before); an empty
// segment starts none (thousands of them at one place were as many atomics on
// one word: 548 us for a million, 4 now).
__global__ void __launch_bounds__(256) k_seg_starts(const uint64_t* __restrict__ off, uint32_t R,
                                                      uint32_t* __restrict__ bits) {
  const uint32_t r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= R) return;
  const uint64_t i = off[r];
  if (i < off[r + 1]) atomicOr(&bits[i >> 5], 1u << (i & 31));
}

// Segment-major suffix array -> positions local to each segment.
__global__ void __launch_bounds__(256) k_localize_sa(uint32_t* __restrict__ sa, uint32_t n,
                                                       const uint64_t* __restrict__ off, uint32_t R) {
  const uint32_t r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r < n) sa[r] -= (uint32_t)off[segment_of(off, R, r)];
}

// ------------------------------------------------------------ extension --
//
// fc_datastore_extend: text = X . T, X the o new tokens in front of the old
// store T (n_old tokens) whose suffix array is known.  Suffixes of T are
// suffixes of the new text, so their order is kept.  For each new suffix p
// the build finds ins(p) = the number of old suffixes smaller than it, then
// orders the new suffixes among themselves, and merges.

// inverse of the old suffix array
__global__ void __launch_bounds__(256) k_isa(const uint32_t* __restrict__ sa, uint32_t n_old,
                                               uint32_t* __restrict__ isa) {
  const uint32_t j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j < n_old) {
    const uint32_t q = sa[j];
    if (q < n_old) isa[q] = j;  // a malformed array cannot write out of bounds
  }
}

// ins by doubling over h = 64, 128, ...: [lo, hi) is the suffix-array range
// of the old suffixes whose first h tokens equal those of new suffix p.
// Inside such a range the old suffixes are ordered by what follows their
// first h tokens, i.e. by isa[q + h] (0 for an empty rest, isa + 1 else),
// so the next range is found by two binary searches against p + h's range
// (or, once p + h lies in T, against the single old suffix there).  An
// empty range is final: its start is ins(p).

// First ranges, for h = kExtFirst tokens at once: a binary search of the
// new suffix's first kExtFirst tokens over the old array, comparing token by
// token from the common prefix both bounds share (Manber and Myers' search).
// Most new suffixes of real text are placed here; only those sharing more
// than kExtFirst tokens with an old suffix go on to the doubling rounds.
constexpr uint32_t kExtFirst = 64;

// sign of (new suffix p, at most kExtFirst tokens) - (old suffix q), from
// offset d on; *lcp receives the common length, capped at kExtFirst
__device__ __forceinline__ int ext_cmp(const uint16_t* __restrict__ tok, uint32_t o, uint64_t n, uint32_t n_old,
                                       uint32_t p, uint32_t q, uint32_t d, uint32_t* lcp) {
  for (; d < kExtFirst; ++d) {
    if ((uint64_t)q + d >= n_old) { *lcp = d; return 1; }   // the old suffix ended first
    if ((uint64_t)p + d >= n) { *lcp = d; return -1; }
    const uint32_t a = tok[p + d], b = tok[(uint64_t)o + q + d];
    if (a != b) { *lcp = d; return a > b ? 1 : -1; }
  }
  *lcp = kExtFirst;
  return 0;
}

__global__ void __launch_bounds__(256) k_ext_init(const uint16_t* __restrict__ tok, uint32_t o, uint64_t n,
                                                    const uint32_t* __restrict__ sa, uint32_t n_old,
                                                    uint32_t* __restrict__ lo0, uint32_t* __restrict__ hi0,
                                                    uint32_t* __restrict__ lo1, uint32_t* __restrict__ hi1,
                                                    uint32_t* __restrict__ active, uint32_t* __restrict__ count) {
  const uint32_t p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= o) return;
  auto old_at = [&](uint32_t r) -> uint32_t {
    const uint32_t q = sa[r];
    return q < n_old ? q : n_old;  // a malformed array reads as an ended suffix
  };
  // lower end: first r whose suffix is >= the new suffix's first tokens
  uint32_t a = 0, b = n_old, la = 0, lb = 0;
  while (a < b) {
    const uint32_t mid = (a + b) >> 1;
    uint32_t l;
    const int c = ext_cmp(tok, o, n, n_old, p, old_at(mid), la < lb ? la : lb, &l);
    if (c > 0) { a = mid + 1; la = l; } else { b = mid; lb = l; }
  }
  // upper end: first r whose suffix is > them (the search resumes from a,
  // whose left neighbour shares la tokens)
  uint32_t e = a, f = n_old, le = la, lf = 0;
  while (e < f) {
    const uint32_t mid = (e + f) >> 1;
    uint32_t l;
    const int c = ext_cmp(tok, o, n, n_old, p, old_at(mid), le < lf ? le : lf, &l);
    if (c >= 0) { e = mid + 1; le = l; } else { f = mid; lf = l; }
  }
  lo0[p] = lo1[p] = a;
  hi0[p] = hi1[p] = e;
  if (a < e) active[atomicAdd(count, 1u)] = p;
}

__device__ __forceinline__ uint32_t ext_key(const uint32_t* __restrict__ sa, const uint32_t* __restrict__ isa,
                                            uint32_t n_old, uint64_t h, uint32_t r) {
  const uint64_t q = (uint64_t)sa[r] + h;
  return q < n_old ? isa[q] + 1 : 0u;
}

__global__ void __launch_bounds__(256) k_ext_round(uint32_t o, uint64_t n, uint32_t n_old,
                                                     const uint32_t* __restrict__ sa,
                                                     const uint32_t* __restrict__ isa, uint64_t h,
                                                     const uint32_t* __restrict__ clo,
                                                     const uint32_t* __restrict__ chi, uint32_t* __restrict__ nlo,
                                                     uint32_t* __restrict__ nhi, const uint32_t* __restrict__ act,
                                                     const uint32_t* __restrict__ n_act,
                                                     uint32_t* __restrict__ act_out,
                                                     uint32_t* __restrict__ done_out,
                                                     uint32_t* __restrict__ counts) {
  const uint32_t t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= *n_act) return;
  const uint32_t p = act[t];
  const uint32_t lo = clo[p], hi = chi[p];
  const uint64_t z = (uint64_t)p + h;
  uint32_t a, b;
  if (z < o) {
    a = clo[z] + 1;
    b = chi[z] + 1;
  } else if (z < n) {
    a = b = isa[z - o] + 1;
  } else {
    a = b = 0;
  }
  uint32_t x = lo, y = hi;
  while (x < y) {
    const uint32_t mid = (x + y) >> 1;
    if (ext_key(sa, isa, n_old, h, mid) < a) x = mid + 1; else y = mid;
  }
  const uint32_t nl = x;
  if (a != b) {
    y = hi;
    while (x < y) {
      const uint32_t mid = (x + y) >> 1;
      if (ext_key(sa, isa, n_old, h, mid) < b) x = mid + 1; else y = mid;
    }
  }
  nlo[p] = nl;
  nhi[p] = x;
  if (nl < x) act_out[atomicAdd(&counts[0], 1u)] = p;
  else done_out[atomicAdd(&counts[1], 1u)] = p;
}

// a range that became final this round is copied into the other buffer
// (no other work of the next round touches it)
__global__ void __launch_bounds__(256) k_ext_fix(const uint32_t* __restrict__ done,
                                                   const uint32_t* __restrict__ n_done,
                                                   const uint32_t* __restrict__ nlo, uint32_t* __restrict__ olo,
                                                   uint32_t* __restrict__ ohi) {
  const uint32_t t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= *n_done) return;
  const uint32_t p = done[t];
  olo[p] = ohi[p] = nlo[p];
}

__global__ void __launch_bounds__(256) k_ins_sorted(const uint64_t* __restrict__ keys, uint32_t o, int shift,
                                                      uint32_t* __restrict__ out) {
  const uint32_t r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r < o) out[r] = (uint32_t)(keys[r] >> shift);
}

// number of s[0..len) that are <= j (s non-decreasing)
__device__ __forceinline__ uint32_t count_le(const uint32_t* __restrict__ s, uint32_t len, uint32_t j) {
  uint32_t a = 0, b = len;
  while (a < b) {
    const uint32_t mid = (a + b) >> 1;
    if (s[mid] <= j) a = mid + 1; else b = mid;
  }
  return a;
}

// The second half of a round's key: what the label of the position h on is.
struct NextRank {
  const uint32_t* rank;
  const uint32_t* seg_bits;    // batched: a bit per position that starts a segment
  const uint32_t* ins;         // extension: per new position
  const uint32_t* isa;         // extension: inverse of the old suffix array
  const uint32_t* ins_sorted;  // extension
  uint64_t n;                  // positions (extension: of the whole text)
  uint64_t h;
  uint32_t o;                  // extension: new positions
};

// Batched build: a suffix that is still tied on its first h tokens has all of
// them inside its segment (one that ends earlier holds its end mark at a
// place no other suffix of the segment has it), so position i + h is at most
// the segment's end, and it is the end where it starts another segment.
template <Mode M>
__device__ __forceinline__ uint32_t next_rank(const NextRank& a, uint32_t i) {
  const uint64_t z = (uint64_t)i + a.h;
  if (M == Mode::kExtend) {
    if (z < a.o) return a.rank[z] + a.ins[z] + 1u;
    if (z >= a.n) return 0u;
    const uint32_t j = a.isa[z - a.o];
    return j + count_le(a.ins_sorted, a.o, j) + 1u;
  }
  if (z >= a.n) return 0u;
  if (M == Mode::kBatched && ((a.seg_bits[z >> 5] >> (z & 31)) & 1u)) return 0u;
  return a.rank[z] + 1u;
}

// merge: new suffix p goes to ins(p) + rank[p], old suffix at index j to
// j + (new suffixes with ins <= j), at position sa[j] + o
__global__ void __launch_bounds__(256) k_ext_new_out(const uint32_t* __restrict__ rank,
                                                       const uint32_t* __restrict__ ins, uint32_t o,
                                                       uint32_t* __restrict__ out) {
  const uint32_t p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p < o) out[rank[p] + ins[p]] = p;
}

constexpr int kOldItems = 8;
constexpr int kCountShift = 11;  // one coarse count per 2048 old indexes (256 threads x kOldItems)
static_assert((256 * kOldItems) == (1 << kCountShift), "a merge workgroup covers one coarse block");

// coarse[b] = number of new suffixes with ins < b * 2048, b = 0 .. n_old/2048 + 1
__global__ void __launch_bounds__(256) k_ext_coarse(const uint32_t* __restrict__ ins_sorted, uint32_t o,
                                                      uint32_t nb, uint32_t* __restrict__ coarse) {
  const uint32_t b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= nb) return;
  const uint64_t v = (uint64_t)b << kCountShift;
  uint32_t x = 0, y = o;
  while (x < y) {
    const uint32_t mid = (x + y) >> 1;
    if (ins_sorted[mid] < v) x = mid + 1; else y = mid;
  }
  coarse[b] = x;
}

// number of new suffixes with ins <= j, from the coarse table
__device__ __forceinline__ uint32_t count_new_le(const uint32_t* __restrict__ ins_sorted,
                                                 const uint32_t* __restrict__ coarse, uint32_t j) {
  const uint32_t b = j >> kCountShift;
  uint32_t x = coarse[b], y = coarse[b + 1];
  while (x < y) {
    const uint32_t mid = (x + y) >> 1;
    if (ins_sorted[mid] <= j) x = mid + 1; else y = mid;
  }
  return x;
}

__global__ void __launch_bounds__(256) k_ext_old_out(const uint32_t* __restrict__ sa, uint32_t n_old,
                                                       const uint32_t* __restrict__ ins_sorted,
                                                       const uint32_t* __restrict__ coarse, uint32_t o,
                                                       uint32_t* __restrict__ out) {
  // workgroup b covers old indexes [2048 b, 2048 (b + 1)): one coarse block,
  // whose few inserted suffixes every thread searches; j = base + t + 256 i
  // keeps each step's reads and writes coalesced
  const uint32_t base = blockIdx.x << kCountShift;
  const uint32_t c0 = o ? coarse[blockIdx.x] : 0u, c1 = o ? coarse[blockIdx.x + 1] : 0u;
  for (int i = 0; i < kOldItems; ++i) {
    const uint32_t j = base + threadIdx.x + 256 * i;
    if (j >= n_old) break;
    uint32_t x = c0, y = c1;
    while (x < y) {
      const uint32_t mid = (x + y) >> 1;
      if (ins_sorted[mid] <= j) x = mid + 1; else y = mid;
    }
    out[j + x] = sa[j] + o;
  }
}

// inverse of the result: new position p at ins(p) + rank[p]; old position q
// (now q + o) at isa[q] + (new suffixes with ins <= isa[q])
__global__ void __launch_bounds__(256) k_ext_isa_new(const uint32_t* __restrict__ rank,
                                                       const uint32_t* __restrict__ ins, uint32_t o,
                                                       uint32_t* __restrict__ isa_out) {
  const uint32_t p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p < o) isa_out[p] = rank[p] + ins[p];
}

__global__ void __launch_bounds__(256) k_ext_isa_old(const uint32_t* __restrict__ isa, uint32_t n_old,
                                                       const uint32_t* __restrict__ ins_sorted,
                                                       const uint32_t* __restrict__ coarse, uint32_t o,
                                                       uint32_t* __restrict__ isa_out) {
  const uint32_t q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= n_old) return;
  uint32_t j = isa[q];
  j = j < n_old ? j : n_old - 1;  // a malformed inverse cannot read out of bounds
  isa_out[q + o] = j + (o ? count_new_le(ins_sorted, coarse, j) : 0u);
}

// --------------------------------------------------------- round 0's keys --


// Round 0's keys, made from the text where they are needed: once for their
// digit histogram and once in the first digit pass.  (Written out once, 12
// bytes a suffix, and read back by the first pass, 1B suffixes took 3.9 ms
// before and as long in that pass; now 1.9.)
//   plain: the first three tokens, as token + 1 in tb bits, 0 past the end.
//   batched: (segment, first ntok tokens, 0 past the segment's end), so
//     suffixes of different segments never share a group and every suffix
//     ends at its own segment's end.
//   extension: the n new positions, with ins(p) as the most significant field
//     and one or two tokens in 17 bits after it.  A new suffix's group label
//     is ins(p) + rank[p] and an old suffix's is its final index isa + (new
//     suffixes with ins <= isa): both are positions in the final array's
//     order, so the rank of whatever follows the first h tokens can be either
//     kind.
template <Mode M>
struct FirstKeys {
  const uint16_t* __restrict__ tok;
  uint64_t n;     // tokens of the text
  int tb, ntok;
  const uint64_t* __restrict__ off;  // batched: R segments
  uint32_t R;
  const uint32_t* __restrict__ ins;  // extension

  // The keys of a wave's kItems * 64 positions from `first` on, below `count`
  // (the others: ~0).  Away from the text's end, and inside one segment, all
  // loads are issued together.
  template <int kItems>
  __device__ void wave_keys(uint64_t first, uint32_t count, uint32_t lane, uint64_t (&k)[kItems]) const {
    const uint64_t last = first + kItems * fc::kWave - 1;
    uint32_t r = 0;
    uint64_t end = n;
    if constexpr (M == Mode::kBatched) {
      if (first < count) {
        r = uniform(segment_of(off, R, first));
        end = off[r + 1];
      }
    }
    const bool whole = last < count && last + 4 <= n;
    fc::u32x2_a2 w[kItems];
    if (whole) {
#pragma unroll
      for (int j = 0; j < kItems; ++j) w[j] = *(const fc::u32x2_a2*)(tok + first + (uint32_t)(j * fc::kWave) + lane);
      if (last < end) {
#pragma unroll
        for (int j = 0; j < kItems; ++j) {
          const uint64_t i = first + (uint32_t)(j * fc::kWave) + lane;
          k[j] = key(i, r, (w[j][0] & 0xFFFFu) + 1, i + 1 < end ? (w[j][0] >> 16) + 1 : 0,
                     i + 2 < end ? (w[j][1] & 0xFFFFu) + 1 : 0);
        }
        return;
      }
    }
#pragma unroll 1
    for (int j = 0; j < kItems; ++j) {
      const uint64_t x0 = first + (uint32_t)(j * fc::kWave), i = x0 + lane;
      uint32_t t01 = 0, t2 = 0;  // the position's three tokens
      if (whole) {
#pragma unroll
        for (int u = 0; u < kItems; ++u) {
          t01 = u == j ? w[u][0] : t01;
          t2 = u == j ? w[u][1] : t2;
        }
      } else if (i < count) {
        t01 = (uint32_t)tok[i] | (i + 1 < n ? (uint32_t)tok[i + 1] << 16 : 0u);
        t2 = i + 2 < n ? tok[i + 2] : 0u;
      }
      bool one = i + 1 < end, two = i + 2 < end;  // the tokens after i's belong to its suffix
      uint32_t mine = r;
      if constexpr (M == Mode::kBatched)
        if (x0 < count && x0 + fc::kWave + 1 >= end) segments(x0, count, lane, r, end, mine, one, two);
      uint64_t x = ~0ull;
      if (i < count) x = key(i, mine, (t01 & 0xFFFFu) + 1, one ? (t01 >> 16) + 1 : 0, two ? (t2 & 0xFFFFu) + 1 : 0);
      set(k, j, x);
    }
  }
  // Batched: the segments of positions x0 .. x0 + 63 and whether the next two
  // tokens are inside; r and end are x0's segment and its end, and x0 + 64's
  // afterwards.  The next 64 segments' starts are read at once and searched
  // across the lanes; more starts than that (empty segments) take a search per
  // lane.  A walk from segment to segment per lane, one dependent read each,
  // took 69 us for the first digit pass of 300,000 segments of 3 tokens (41 now),
  // and 8.5 ms for a build of 50 segments of 2,000 with 20,000 empty ones before
  // each (0.70).
  __device__ void segments(uint64_t x0, uint32_t count, uint32_t lane, uint32_t& r, uint64_t& end, uint32_t& mine,
                           bool& one, bool& two) const {
    const uint64_t at = (uint64_t)r + 1 + lane;
    const uint64_t start = at <= R ? off[at] : ~0ull;
    const uint32_t rel = start - x0 < 127 ? (uint32_t)(start - x0) : 127u;  // non-decreasing over the lanes
    if ((uint32_t)__builtin_amdgcn_readlane((int)rel, fc::kWave - 1) > fc::kWave + 1) {
      uint32_t c = 0;  // starts up to this lane's position
#pragma unroll
      for (uint32_t b = fc::kWave / 2; b > 0; b /= 2)
        if ((uint32_t)__shfl((int)rel, (int)(c + b - 1), fc::kWave) <= lane) c += b;
      mine = r + c;
      const uint32_t next = (uint32_t)__shfl((int)rel, (int)c, fc::kWave);
      one = lane + 1 < next;
      two = lane + 2 < next;
      const uint32_t past = (uint32_t)__popcll(fc::ballot(rel <= fc::kWave));  // below 64
      const uint32_t to = (uint32_t)__builtin_amdgcn_readlane((int)rel, (int)past);
      r += past;
      end = to < 127 ? x0 + to : r < R ? off[r + 1] : n;
      return;
    }
    const uint64_t i = x0 + lane < count ? x0 + lane : (uint64_t)count - 1;
    mine = segment_from(off, R, r, i);
    const uint64_t e = off[mine + 1];
    one = i + 1 < e;
    two = i + 2 < e;
    r = uniform(segment_from(off, R, r, x0 + fc::kWave < count ? x0 + fc::kWave : (uint64_t)count - 1));
    end = off[r + 1];
  }
  // k[j] = x with j known at run time only: registers cannot be indexed
  template <int kItems>
  static __device__ void set(uint64_t (&k)[kItems], int j, uint64_t x) {
#pragma unroll
    for (int u = 0; u < kItems; ++u) k[u] = u == j ? x : k[u];
  }
  // position i of segment r, tokens as token + 1
  __device__ uint64_t key(uint64_t i, uint32_t r, uint32_t a, uint32_t b, uint32_t c) const {
    if constexpr (M == Mode::kPlain) return ((uint64_t)a << (2 * tb)) | ((uint64_t)b << tb) | c;
    if constexpr (M == Mode::kBatched) {
      const uint64_t two = ((((uint64_t)r << tb) | a) << tb) | b;
      return ntok == 3 ? (two << tb) | c : two;
    }
    return ntok == 2 ? ((uint64_t)ins[i] << 34) | ((uint64_t)a << 17) | b : ((uint64_t)ins[i] << 17) | a;
  }
};

// The keys' digit histogram.
template <Mode M>
__global__ void __launch_bounds__(256) k_first_hist(FirstKeys<M> fk, uint32_t count, int digits,
                                                     uint32_t* __restrict__ hist) {
  __shared__ uint32_t s_hist[kMaxDigits][kRadix];
  const LdsHist lh{s_hist};
  lh.zero();
  const uint32_t lane = (uint32_t)fc::lane_id();
  constexpr int kItems = 4;
  constexpr uint32_t kSpan = kItems * fc::kWave;
  const uint64_t waves = (uint64_t)gridDim.x * (blockDim.x / fc::kWave);
  for (uint64_t x = (uint64_t)blockIdx.x * (blockDim.x / fc::kWave) + uniform(threadIdx.x / fc::kWave); x * kSpan < count;
       x += waves) {
    uint64_t k[kItems];
    fk.template wave_keys<kItems>(x * kSpan, count, lane, k);
#pragma unroll
    for (int j = 0; j < kItems; ++j)
      if (x * kSpan + (uint32_t)(j * fc::kWave) + lane < count) lh.add(k[j], digits);
  }
  lh.flush(digits, hist);
}

// ------------------------------------------------------------ histogram ---

// One workgroup of 256 threads per digit: its offsets (exclusive scan).
__global__ void __launch_bounds__(256) k_hist_scan(const uint32_t* __restrict__ hist,
                                                     uint32_t* __restrict__ offsets) {
  __shared__ uint32_t scratch[8];
  const uint32_t i = blockIdx.x * kRadix + threadIdx.x;
  offsets[i] = fc::block_excl_sum<uint32_t>(hist[i], scratch, nullptr);
}

// ------------------------------------------------------------- onesweep ---

// Decoupled look-back of digit t over tiles p, p - 1, .. p_end: the elements
// of the digit in those tiles, kLookWindow tiles per step: their status words
// are loaded together (for the block, a contiguous run per tile), then taken
// nearest first - aggregates are added until an inclusive prefix ends the
// walk; a tile that has published nothing yet makes the walk wait and reload
// from there.  One round trip then covers as many tiles as the window
// instead of one.  The wait is bounded: giving up sets *err.
__device__ __forceinline__ uint64_t look_back(const uint64_t* status, int64_t p, int64_t p_end, uint32_t t,
                                              uint32_t epoch, uint32_t* err) {
  uint64_t excl = 0;
  uint32_t spins = 0;
  bool done = p < p_end;
  while (!done) {
    uint64_t sw[kLookWindow];
#pragma unroll
    for (int i = 0; i < kLookWindow; ++i)
      sw[i] = p - i >= p_end ? __hip_atomic_load(status + (uint64_t)(p - i) * kRadix + t, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT)
                             : pack_status(epoch, kFlagInc, 0);  // before the first tile: an empty prefix
    int taken = 0;
    bool stalled = false;
#pragma unroll
    for (int i = 0; i < kLookWindow; ++i) {
      if (done || stalled) continue;
      const uint64_t s = sw[i];
      const uint64_t fl = s & kFlagMask;
      if ((uint32_t)(s >> 48) != epoch || fl == 0) {
        stalled = true;
        continue;
      }
      excl += s & kCountMask;
      ++taken;
      if (fl == kFlagInc) done = true;
    }
    p -= taken;
    if (stalled && !done) {
      if (++spins > kSpinLimit) {
        atomicOr(err, 1u);
        break;
      }
      __builtin_amdgcn_s_sleep(1);
    }
  }
  return excl;
}

// Stable rank of each wave's elements inside their digit: the elements of the
// wave with the same digit before this lane's; wcnt counts the wave's digits
// (zeroed before).  Every lane counts.
__device__ __forceinline__ uint32_t wave_digit_rank(uint32_t d, uint16_t* wcnt) {
  uint32_t lo = ~0u, hi = ~0u;  // the lanes with this lane's digit
#pragma unroll
  for (int b = 0; b < 8; ++b) {
    const uint32_t mine = (uint32_t)__builtin_amdgcn_sbfe((int)d, b, 1);  // the bit, in all 32
    const uint64_t ones = fc::ballot(mine != 0);
    lo &= ~((uint32_t)ones ^ mine);
    hi &= ~((uint32_t)(ones >> 32) ^ mine);
  }
  const uint32_t below = __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0u));
  const uint32_t old = wcnt[d];
  if (below == 0) wcnt[d] = (uint16_t)(old + (uint32_t)(__popc(lo) + __popc(hi)));
  __builtin_amdgcn_sched_barrier(0);  // one element after another: interleaved, their masks spill
  return old + below;
}

// kFirst: the pass that makes the keys (kin and vin unused).
template <Mode M, bool kFirst>
__global__ void __launch_bounds__(kSortThreads) k_onesweep(FirstKeys<M> fk, const uint64_t* __restrict__ kin,
                                                           const uint32_t* __restrict__ vin,
                                                           uint64_t* __restrict__ kout, uint32_t* __restrict__ vout,
                                                           uint32_t U, uint32_t shift,
                                                           const uint32_t* __restrict__ digit_base,
                                                           uint64_t* status, uint32_t* ticket, uint32_t epoch,
                                                           uint32_t* err) {
  __shared__ uint32_t s_tile;
  // per-wave digit counts and then per-wave offsets (below kSortTile), 16
  // bits each: with these the LDS of a tile fits three tiles per CU, which
  // matters because a tile spends most of its time waiting
  __shared__ uint16_t s_wcnt[kSortThreads / fc::kWave][kRadix];
  __shared__ uint16_t s_dstart[kRadix];  // tile-local digit starts (below kSortTile)
  __shared__ uint32_t s_gbase[kRadix];
  __shared__ uint32_t s_scan[kSortThreads / fc::kWave + 1];
  __shared__ uint64_t s_keys[kSortTile];
  __shared__ uint32_t s_vals[kSortTile];

  const int tid = threadIdx.x;
  const int w = (int)uniform((uint32_t)tid / fc::kWave);
  const int lane = fc::lane_id();
  for (int i = tid; i < (kSortThreads / fc::kWave) * kRadix; i += kSortThreads) (&s_wcnt[0][0])[i] = 0;
  if (tid == 0) s_tile = atomicAdd(ticket, 1u);
  __syncthreads();
  const uint32_t tile = uniform(s_tile);
  const uint64_t base = (uint64_t)tile * kSortTile;
  const uint32_t nvalid = (uint32_t)((U - base) < (uint64_t)kSortTile ? (U - base) : (uint64_t)kSortTile);

  uint64_t k[kSortItems];
  uint32_t v[kSortItems];
  uint32_t rk[kSortItems];
  if constexpr (kFirst)
    fk.template wave_keys<kSortItems>(base + (uint32_t)(w * kSortItems * fc::kWave), U, (uint32_t)lane, k);
#pragma unroll
  for (int j = 0; j < kSortItems; ++j) {
    const uint32_t idx = (uint32_t)(w * kSortItems * fc::kWave + j * fc::kWave + lane);
    const bool valid = idx < nvalid;
    if constexpr (kFirst) {
      v[j] = (uint32_t)(base + idx);
    } else {
      k[j] = valid ? kin[base + idx] : ~0ull;
      v[j] = valid ? vin[base + idx] : 0u;
    }
  }
  // what lies past the last tile's end has digit 255 and comes last: it counts
  // nowhere but behind the tile's own elements
#pragma unroll
  for (int j = 0; j < kSortItems; ++j) rk[j] = wave_digit_rank((uint32_t)(k[j] >> shift) & 0xFF, s_wcnt[w]);
  __syncthreads();

  // Per digit: offsets of each wave's elements, tile count, tile-local start.
  const uint32_t t = (uint32_t)tid;  // this thread's digit
  uint32_t total = 0;
#pragma unroll
  for (int ww = 0; ww < kSortThreads / fc::kWave; ++ww) {
    uint32_t c = s_wcnt[ww][t];
    s_wcnt[ww][t] = (uint16_t)total;
    total += c;
  }
  // publish this tile's digit count at once (tile 0: its inclusive prefix),
  // before the tile-local scan and staging, so later tiles' look-backs find it
  uint64_t* mine = status + (uint64_t)tile * kRadix + t;
  __hip_atomic_store(mine, pack_status(epoch, tile > 0 ? kFlagAgg : kFlagInc, total), __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
  uint32_t tile_sum;
  s_dstart[t] = (uint16_t)fc::block_excl_sum<uint32_t>(total, s_scan, &tile_sum);
  __syncthreads();

  // Stage in LDS in digit order (before the look-back, so the keys leave
  // the registers while the look-back runs).
#pragma unroll
  for (int j = 0; j < kSortItems; ++j) {
    const uint32_t idx = (uint32_t)(w * kSortItems * fc::kWave + j * fc::kWave + lane);
    if (idx < nvalid) {
      const uint32_t d = (uint32_t)(k[j] >> shift) & 0xFF;
      const uint32_t pos = s_dstart[d] + s_wcnt[w][d] + rk[j];
      s_keys[pos] = k[j];
      s_vals[pos] = v[j];
    }
  }

  const uint64_t excl = look_back(status, (int64_t)tile - 1, 0, t, epoch, err);
  if (tile > 0)
    __hip_atomic_store(mine, pack_status(epoch, kFlagInc, excl + total), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  s_gbase[t] = digit_base[t] + (uint32_t)excl;
  __syncthreads();

  for (uint32_t i = (uint32_t)tid; i < nvalid; i += kSortThreads) {
    const uint64_t key = s_keys[i];
    const uint32_t d = (uint32_t)(key >> shift) & 0xFF;
    const uint32_t dst = s_gbase[d] + (i - s_dstart[d]);
    if (dst < U) {  // always true unless a look-back gave up (then err is set)
      kout[dst] = key;
      vout[dst] = s_vals[i];
    }
  }
}

// ------------------------------------------------- sorting inside groups ---
//
// Rounds after the first.  The still-tied suffixes lie in a list (grp, val):
// group after group, grp = the group's first suffix-array index, so only the
// order inside each group is open, by lo = the rank h positions on.  Sorting
// (grp, lo) pairs globally moved every 12-byte element through eight digit
// passes; instead
//  - k_sort_small sorts the groups of at most kWin elements, a window of
//    whole groups per workgroup, inside LDS: lo is gathered, and the list
//    read and written, once;
//  - the larger groups (few, but up to half of the elements) go through
//    digit passes over lo alone (8-byte elements), every group for itself:
//    k_big_plan sizes them and cuts them into tiles, k_big_keys gathers lo
//    and counts each group's digits, k_big_pass is a onesweep pass whose
//    look-back ends at the group's first tile.
// At 1B suffixes this replaced 48 passes over (8-byte key, suffix) elements
// and their key and histogram kernels, 159 ms of a 305 ms build, by 67 ms
// (small groups 28, keys of the large ones 22, their passes 17); 10M suffixes
// 3.60 -> 2.83 ms, 64 repositories in one call 8.43 -> 6.04 ms.  The line
// between the two lies at what one workgroup's LDS holds next to the groups
// that start before it: in the first such round of a 10M store about half of
// the elements are in larger groups, in the third a tenth.

constexpr int kWin = 2048;          // list positions whose groups a workgroup sorts
constexpr int kCap = 2 * kWin;      // a window's last group may end this far
constexpr int kSmallThreads = 256;
constexpr int kSmallItems = kCap / kSmallThreads;
// Groups up to this size are ranked by comparing all pairs.  Builds of 1B
// tokens (ms), 10M and 64 repositories (us): 24: 176.0, 2,471, 5,126; 32: 176.2,
// 2,491, 5,163; 48: 171.0, 2,441, 5,004; 64: 171.8, 2,471, 5,066; 96: 173.3, 2,538,
// 5,177.
constexpr uint32_t kCountMax = 48;
constexpr int kMaxLoDigits = 4;
constexpr uint32_t kNone = 0xFFFFFFFFu;

// Window b takes the groups that start at list positions [b kWin, (b+1) kWin).
// All but the last one end inside the window or right after it; the last one
// is small if it ends within kWin of its start, else it is registered as
// large.  first_head[b] = where the window's first group starts (kNone: one
// group covers it).  Small groups are one contiguous run of positions: those
// of up to kCountMax elements are ranked by comparing all pairs (a group's
// lanes read the same LDS words), the others by an LDS radix sort over lo and
// then the group.  `val` is reordered in place: a position is read and
// written by the one workgroup that owns its group.
template <Mode M>
__global__ void __launch_bounds__(kSmallThreads, 4) k_sort_small(const uint32_t* __restrict__ grp, uint32_t* val,
                                                              uint32_t* __restrict__ lo,
                                                              const uint32_t* __restrict__ u_dev, NextRank nr,
                                                              int lo_digits, uint32_t* __restrict__ first_head,
                                                              uint32_t* __restrict__ big_start,
                                                              uint32_t* __restrict__ big_count) {
  constexpr int kWaves = kSmallThreads / fc::kWave;
  constexpr int kPer = kSmallItems * fc::kWave;  // positions per wave
  __shared__ uint32_t s_a[kCap], s_b[kCap];
  // a tied group has two elements or more
  __shared__ uint16_t s_head[kWin / 2 + 1];  // start of each small group (and the end), relative to the window
  __shared__ uint16_t s_slot[kWin / 2];      // first radix slot of each group that goes to the radix sort
  __shared__ uint16_t s_delta[kCap / kCountMax + 1];  // per radix group: list position minus radix slot
  __shared__ uint8_t s_rg[kWin / 2];         // its number among those
  __shared__ uint16_t s_wcnt[kWaves][kRadix];
  __shared__ uint16_t s_dstart[kRadix];
  __shared__ uint32_t s_scan[kWaves + 1];
  __shared__ uint32_t s_first[kWaves], s_heads[kWaves];
  uint32_t* const s_last = s_scan;  // read before the first scan; with it the LDS fits four workgroups per CU
  static_assert(kCap / (kCountMax + 1) < 256, "radix groups are numbered in 8 bits");

  const uint32_t U = *u_dev;
  const uint32_t w0 = blockIdx.x * kWin;
  if (w0 >= U) return;
  const int tid = (int)threadIdx.x, w = (int)uniform((uint32_t)tid / fc::kWave);
  const uint32_t lane = (uint32_t)fc::lane_id();
  const uint32_t room = U - w0;  // list positions from the window on
  const uint32_t wbase = (uint32_t)(w * kPer);

  // group starts among this wave's positions
  uint64_t hm[kSmallItems];
  uint32_t first = kNone, last = kNone;
  {
    uint32_t g[kSmallItems];
#pragma unroll
    for (int j = 0; j < kSmallItems; ++j) {
      const uint32_t x = wbase + (uint32_t)(j * fc::kWave) + lane;
      g[j] = x < room ? grp[(uint64_t)w0 + x] : 0u;
    }
    uint32_t carry = (uint64_t)w0 + wbase > 0 && wbase < room ? grp[(uint64_t)w0 + wbase - 1] : 0u;
#pragma unroll
    for (int j = 0; j < kSmallItems; ++j) {
      const uint32_t x0 = wbase + (uint32_t)(j * fc::kWave);
      const uint32_t x = x0 + lane;
      const uint32_t before = fc::wave_shr1(g[j], carry);
      carry = (uint32_t)__builtin_amdgcn_readlane((int)g[j], fc::kWave - 1);
      hm[j] = fc::ballot(x < room && (w0 + x == 0 || g[j] != before));
      if (hm[j]) {
        if (first == kNone) first = x0 + (uint32_t)__builtin_ctzll(hm[j]);
        last = x0 + 63u - (uint32_t)__builtin_clzll(hm[j]);
      }
    }
  }
  if (lane == 0) {
    s_first[w] = first;
    s_last[w] = last;
  }
  __syncthreads();
  static_assert(kWaves == 4, "two waves hold the window, two what follows");
  // the same for every lane: kept in scalar registers
  const uint32_t F = uniform(s_first[0] != kNone ? s_first[0] : s_first[1]);
  const uint32_t Lh = uniform(s_last[1] != kNone ? s_last[1] : s_last[0]);
  uint32_t E = uniform(s_first[2] != kNone ? s_first[2] : s_first[3]);
  if (E == kNone && room < (uint32_t)kCap) E = room;  // the list ends with the group
  if (E != kNone && E > room) E = room;
  if (tid == 0) first_head[blockIdx.x] = F == kNone ? kNone : w0 + F;
  if (F == kNone) return;
  const bool big = E == kNone || E - Lh > (uint32_t)kWin;
  if (big && tid == 0) big_start[atomicAdd(big_count, 1u)] = w0 + Lh;
  const uint32_t end = big ? Lh : E;  // the small groups: positions [F, end) of the window
  if (F >= end) return;

  // number the groups, gather lo
  uint32_t nh = 0;
#pragma unroll
  for (int j = 0; j < kSmallItems; ++j) {
    const uint32_t x0 = wbase + (uint32_t)(j * fc::kWave);
    // heads below `end` (the head at `end`, if any, opens the next window's or the large group)
    if (x0 >= end) hm[j] = 0;
    else if (end - x0 < 64) hm[j] &= (1ull << (end - x0)) - 1;
    nh += (uint32_t)__popcll(hm[j]);
  }
  if (lane == 0) s_heads[w] = nh;
  uint32_t v[kSmallItems], key[kSmallItems];
#pragma unroll
  for (int j = 0; j < kSmallItems; ++j) {
    const uint32_t x = wbase + (uint32_t)(j * fc::kWave) + lane;
    v[j] = x >= F && x < end ? val[(uint64_t)w0 + x] : 0u;
  }
#pragma unroll
  for (int j = 0; j < kSmallItems; ++j) {
    const uint32_t x = wbase + (uint32_t)(j * fc::kWave) + lane;
    key[j] = x >= F && x < end ? next_rank<M>(nr, v[j]) : 0u;
  }
  __syncthreads();
  uint32_t gi0 = 0, groups = 0;
#pragma unroll
  for (int u = 0; u < kWaves; ++u) {
    const uint32_t x = uniform(s_heads[u]);
    if (u < w) gi0 += x;
    groups += x;
  }
  const uint64_t le = lane == 63 ? ~0ull : (2ull << lane) - 1;
  uint16_t gi[kSmallItems];
#pragma unroll
  for (int j = 0; j < kSmallItems; ++j) {
    const uint32_t x = wbase + (uint32_t)(j * fc::kWave) + lane;
    gi[j] = (uint16_t)(gi0 + (uint32_t)__popcll(hm[j] & le) - 1u);  // positions before F: no use is made of it
    if ((hm[j] >> lane) & 1) s_head[gi[j]] = (uint16_t)x;
    gi0 += (uint32_t)__popcll(hm[j]);
    if (x >= F && x < end) s_a[x] = key[j];
  }
  if (tid == 0) s_head[groups] = (uint16_t)end;
  __syncthreads();

  // groups of up to kCountMax: every element counts those before it
  uint32_t have_large = 0;
#pragma unroll
  for (int j = 0; j < kSmallItems; ++j) {
    const uint32_t x = wbase + (uint32_t)(j * fc::kWave) + lane;
    const bool valid = x >= F && x < end;
    uint32_t gs = 0, ge = 0;
    if (valid) {
      gs = s_head[gi[j]];
      ge = s_head[gi[j] + 1];
    }
    const bool large = ge - gs > kCountMax;
    have_large |= large ? 1u : 0u;
    if (valid && !large) {
      uint32_t c = gs;
#pragma clang loop unroll(disable) vectorize(disable)
      for (uint32_t y = gs; y < ge; ++y) {
        const uint32_t k2 = s_a[y];
        c += (k2 < key[j] || (k2 == key[j] && y < x)) ? 1u : 0u;
      }
      lo[(uint64_t)w0 + c] = key[j];
      val[(uint64_t)w0 + c] = v[j];
    }
  }
  if (!__syncthreads_or((int)have_large)) return;

  // the other groups: numbered, and packed into slots [0, nl)
  uint32_t nl, nrg;
  {
    const uint32_t per = (groups + kSmallThreads - 1) / kSmallThreads;
    const uint32_t a = (uint32_t)tid * per, e = a + per < groups ? a + per : groups;
    uint32_t sum = 0;
    for (uint32_t x = a; x < e; ++x) {
      const uint32_t size = (uint32_t)s_head[x + 1] - s_head[x];
      if (size > kCountMax) sum += (1u << 16) | size;
    }
    uint32_t total;
    uint32_t run = fc::block_excl_sum<uint32_t>(sum, s_scan, &total);
    for (uint32_t x = a; x < e; ++x) {
      const uint32_t size = (uint32_t)s_head[x + 1] - s_head[x];
      if (size > kCountMax) {
        s_slot[x] = (uint16_t)(run & 0xFFFF);
        s_rg[x] = (uint8_t)(run >> 16);
        s_delta[run >> 16] = (uint16_t)(s_head[x] - (run & 0xFFFF));
        run += (1u << 16) | size;
      }
    }
    nl = uniform(total & 0xFFFF);
    nrg = uniform(total >> 16);
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kSmallItems; ++j) {
    const uint32_t x = wbase + (uint32_t)(j * fc::kWave) + lane;
    if (x >= F && x < end) {
      const uint32_t gs = s_head[gi[j]];
      if ((uint32_t)s_head[gi[j] + 1] - gs > kCountMax) {
        const uint32_t slot = s_slot[gi[j]] + (x - gs);
        s_a[slot] = key[j];
        s_b[slot] = ((uint32_t)s_rg[gi[j]] << 16) | x;
      }
    }
  }
  const int items = (int)((nl + kSmallThreads - 1) / kSmallThreads);  // per lane; a wave's elements are contiguous
  const uint32_t cbase = (uint32_t)(w * items * fc::kWave);
  const int passes = lo_digits + (nrg > 1 ? 1 : 0);
  uint32_t a[kSmallItems], b[kSmallItems], rk[kSmallItems];
  for (int ps = 0; ps < passes; ++ps) {
    for (int i = tid; i < kWaves * kRadix; i += kSmallThreads) (&s_wcnt[0][0])[i] = 0;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kSmallItems; ++j) {
      const uint32_t i = cbase + (uint32_t)(j * fc::kWave) + lane;
      const bool valid = j < items && i < nl;
      a[j] = valid ? s_a[i] : 0u;
      b[j] = valid ? s_b[i] : 0u;
    }
#pragma unroll
    for (int j = 0; j < kSmallItems; ++j) {
      if (j < items) {
        const bool valid = cbase + (uint32_t)(j * fc::kWave) + lane < nl;  // the others: last, behind all (as above)
        const uint32_t d = !valid ? 255u : ps < lo_digits ? (a[j] >> (8 * ps)) & 0xFF : b[j] >> 16;
        rk[j] = wave_digit_rank(d, s_wcnt[w]) | (d << 16);
      }
    }
    __syncthreads();
    uint32_t total = 0;
#pragma unroll
    for (int u = 0; u < kWaves; ++u) {
      const uint32_t c = s_wcnt[u][tid];
      s_wcnt[u][tid] = (uint16_t)total;
      total += c;
    }
    s_dstart[tid] = (uint16_t)fc::block_excl_sum<uint32_t>(total, s_scan, nullptr);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kSmallItems; ++j) {
      const uint32_t i = cbase + (uint32_t)(j * fc::kWave) + lane;
      if (j < items && i < nl) {
        const uint32_t d = rk[j] >> 16;
        const uint32_t pos = s_dstart[d] + s_wcnt[w][d] + (rk[j] & 0xFFFF);
        s_a[pos] = a[j];
        s_b[pos] = b[j];
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int j = 0; j < kSmallItems; ++j) {
    const uint32_t i = (uint32_t)(j * kSmallThreads + tid);
    if (i < nl) v[j] = val[(uint64_t)w0 + (s_b[i] & 0xFFFF)];
  }
  __syncthreads();  // every element is read before its place is written
#pragma unroll
  for (int j = 0; j < kSmallItems; ++j) {
    const uint32_t i = (uint32_t)(j * kSmallThreads + tid);
    if (i < nl) {
      const uint64_t p = (uint64_t)w0 + i + s_delta[s_b[i] >> 16];
      lo[p] = s_a[i];
      val[p] = v[j];
    }
  }
}

// The large groups of a round.
struct BigWs {
  uint32_t* first_head;  // per window
  uint32_t* start;       // per large group: first list position
  uint32_t* size;
  uint32_t* tile0;       // its first tile
  uint32_t* stat0;       // its first status slot: one per tile but the last, which no tile looks back to
  uint32_t* tile_group;  // per tile: its group
  uint32_t* same;        // per group: the digit places at which all of its elements agree
  uint32_t* hist;        // [group][digit place][256]
  uint32_t* count;       // [0] groups, [1] tiles, [2] status slots, [3..3+kMaxLoDigits) tickets of the passes
};
constexpr int kBigCounts = 3 + kMaxLoDigits;

// One wave per large group: its end is the first group start of a later
// window (or the list's end); its tiles are numbered consecutively and its
// histogram cleared.
__global__ void __launch_bounds__(256) k_big_plan(BigWs g, uint32_t U, int lo_digits) {
  const uint32_t groups = g.count[0];
  const uint32_t windows = (U + kWin - 1) / kWin;
  const uint32_t lane = (uint32_t)fc::lane_id();
  const uint32_t waves = gridDim.x * (blockDim.x / fc::kWave);
  for (uint32_t i = blockIdx.x * (blockDim.x / fc::kWave) + threadIdx.x / fc::kWave; i < groups; i += waves) {
    const uint32_t s = g.start[i];
    uint32_t e = U;
    // most groups end within the next 64 windows; one as long as the text itself
    // (20M equal tokens) took 47 us a round with one read in flight, 18 with eight
    uint32_t w = s / kWin + 1;
    int reads = 1;
    bool found = false;
    while (!found && w < windows) {
      uint32_t x[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const uint32_t at = w + (uint32_t)(u * fc::kWave) + lane;
        x[u] = u < reads && at < windows ? g.first_head[at] : kNone;
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const uint64_t hit = fc::ballot(x[u] != kNone);
        if (!found && hit) {
          e = (uint32_t)__builtin_amdgcn_readlane((int)x[u], (int)__builtin_ctzll(hit));
          found = true;
        }
      }
      w += (uint32_t)(reads * fc::kWave);
      reads = 8;
    }
    const uint32_t tiles = (e - s + kSortTile - 1) / kSortTile;
    uint32_t t0 = 0;
    if (lane == 0) {
      t0 = atomicAdd(&g.count[1], tiles);
      g.size[i] = e - s;
      g.tile0[i] = t0;
      g.stat0[i] = atomicAdd(&g.count[2], tiles - 1);
      g.same[i] = 0;
    }
    t0 = (uint32_t)__shfl((int)t0, 0, fc::kWave);
    for (uint32_t t = lane; t < tiles; t += fc::kWave) g.tile_group[t0 + t] = i;
    for (int t = (int)lane; t < lo_digits * kRadix; t += fc::kWave) g.hist[(uint64_t)i * lo_digits * kRadix + t] = 0;
  }
}

// lo of the large groups' elements, into the buffers the first digit pass
// reads, and each group's digit histograms.  Every workgroup takes one run of
// consecutive tiles and adds its counts once per group it meets; the add that
// fills a bin with the whole group marks the digit place as one where all of
// the group agrees.  A wave whose elements all have one lo (repeated text) adds
// them as one: 20M equal tokens, whose atomics all fell on the same four words,
// 300 us a round before, 108 now.
template <Mode M>
__global__ void __launch_bounds__(256) k_big_keys(BigWs g, const uint32_t* __restrict__ val, NextRank nr,
                                                    int lo_digits, uint32_t* __restrict__ lo_out,
                                                    uint32_t* __restrict__ val_out) {
  __shared__ uint32_t s_hist[kMaxLoDigits * kRadix];
  const uint32_t tiles = g.count[1];
  const uint32_t a = (uint32_t)((uint64_t)tiles * blockIdx.x / gridDim.x);
  const uint32_t e = (uint32_t)((uint64_t)tiles * (blockIdx.x + 1) / gridDim.x);
  if (a >= e) return;
  const int bins = lo_digits * kRadix;
  for (int i = threadIdx.x; i < bins; i += 256) s_hist[i] = 0;
  __syncthreads();
  uint32_t counted = 0;  // elements of the group in this workgroup's tiles
  for (uint32_t t = a; t < e; ++t) {
    const uint32_t gr = uniform(g.tile_group[t]);
    const uint32_t off = (t - uniform(g.tile0[gr])) * kSortTile;
    const uint32_t size = uniform(g.size[gr]), left = size - off;
    const uint32_t nv = left < (uint32_t)kSortTile ? left : (uint32_t)kSortTile;
    const uint64_t base = (uint64_t)g.start[gr] + off;
    counted += nv;
    uint32_t v[kSortItems], k[kSortItems];
#pragma unroll
    for (int j = 0; j < kSortItems; ++j) {
      const uint32_t i = (uint32_t)(j * 256) + threadIdx.x;
      v[j] = i < nv ? val[base + i] : 0u;
    }
#pragma unroll
    for (int j = 0; j < kSortItems; ++j) {
      const uint32_t i = (uint32_t)(j * 256) + threadIdx.x;
      k[j] = i < nv ? next_rank<M>(nr, v[j]) : 0u;
    }
#pragma unroll
    for (int j = 0; j < kSortItems; ++j) {
      const uint32_t i = (uint32_t)(j * 256) + threadIdx.x;
      if (i < nv) {
        lo_out[base + i] = k[j];
        if (val_out) val_out[base + i] = v[j];
        const uint64_t in = fc::ballot(true);
        const bool one = fc::ballot(k[j] == uniform(k[j])) == in;
        if (!one || (in & fc::lanemask_lt()) == 0) {
          const uint32_t c = one ? (uint32_t)__popcll(in) : 1u;
          for (int d = 0; d < lo_digits; ++d) atomicAdd(&s_hist[d * kRadix + ((k[j] >> (8 * d)) & 0xFF)], c);
        }
      }
    }
    if (t + 1 == e || g.tile_group[t + 1] != gr) {
      __syncthreads();
      for (int i = threadIdx.x; i < bins; i += 256) {
        const uint32_t c = s_hist[i];
        if (c) {
          uint32_t* const bin = &g.hist[(uint64_t)gr * bins + i];
          uint32_t sum = c;  // of the bin, if this add is the last
          if (counted == size) *bin = c; else sum += atomicAdd(bin, c);
          if (sum == size) atomicOr(&g.same[gr], 1u << (i / kRadix));
        }
        s_hist[i] = 0;
      }
      counted = 0;
      __syncthreads();
    }
  }
}

// One digit pass over every large group: a onesweep pass (see k_onesweep) on
// 8-byte elements, by a resident grid that takes tiles from a ticket counter;
// a tile's look-back stops at its group's first tile, and its digits start
// from the group's own histogram.
// A group is left where it is by the pass of a digit on which it agrees (in
// repeated text many: 20M equal tokens, 92 passes, 11.7 ms before, 9.1 now); the
// passes alternate between the two buffers for each group by itself, and an odd
// number of such digits is made even by a plain copy, so that every group ends
// in the same ones.
struct BigBufs {
  uint32_t *k[2], *v[2];  // lo and suffixes; the passes end in [0]
};
__global__ void __launch_bounds__(kSortThreads, 4) k_big_pass(BigWs g, int pass, int lo_digits, BigBufs bufs,
                                                             uint64_t* status, uint32_t epoch, uint32_t* err) {
  constexpr int kWaves = kSortThreads / fc::kWave;
  __shared__ uint32_t s_tile;
  __shared__ uint16_t s_wcnt[kWaves][kRadix];
  __shared__ uint16_t s_dstart[kRadix];
  __shared__ uint32_t s_gbase[kRadix];
  __shared__ uint32_t s_scan[kWaves + 1];
  __shared__ uint32_t s_keys[kSortTile];
  __shared__ uint32_t s_vals[kSortTile];
  const int tid = threadIdx.x;
  const int w = (int)uniform((uint32_t)tid / fc::kWave);
  const int lane = fc::lane_id();
  const uint32_t tiles = g.count[1];
  const uint32_t shift = (uint32_t)(8 * pass);
  for (;;) {
    for (int i = tid; i < kWaves * kRadix; i += kSortThreads) (&s_wcnt[0][0])[i] = 0;
    if (tid == 0) s_tile = atomicAdd(&g.count[3 + pass], 1u);
    __syncthreads();
    const uint32_t tile = uniform(s_tile);
    if (tile >= tiles) return;
    const uint32_t gr = uniform(g.tile_group[tile]);
    const uint32_t same = uniform(g.same[gr]);
    const uint32_t skip = __popc(same) & 1 ? same & (same - 1) : same;  // the lowest one's pass copies
    if ((skip >> pass) & 1) {
      __syncthreads();  // s_tile is read
      continue;
    }
    const int from = (lo_digits + __popc(~skip & ((1u << pass) - 1))) & 1;
    const uint32_t* __restrict__ kin = bufs.k[from];
    const uint32_t* __restrict__ vin = bufs.v[from];
    uint32_t* __restrict__ kout = bufs.k[from ^ 1];
    uint32_t* __restrict__ vout = bufs.v[from ^ 1];
    const uint32_t t0 = uniform(g.tile0[gr]);
    const uint64_t gstart = uniform(g.start[gr]);
    const uint64_t base = gstart + (uint64_t)(tile - t0) * kSortTile;
    const uint32_t size = uniform(g.size[gr]);
    const uint32_t left = size - (tile - t0) * kSortTile;
    const uint32_t nvalid = left < (uint32_t)kSortTile ? left : (uint32_t)kSortTile;
    const uint32_t* __restrict__ kt = kin + base;
    const uint32_t* __restrict__ vt = vin + base;
    uint32_t k[kSortItems], v[kSortItems], rk[kSortItems];
#pragma unroll
    for (int j = 0; j < kSortItems; ++j) {
      const uint32_t idx = (uint32_t)(w * kSortItems * fc::kWave + j * fc::kWave + lane);
      k[j] = idx < nvalid ? kt[idx] : ~0u;
      v[j] = idx < nvalid ? vt[idx] : 0u;
    }
    if ((same >> pass) & 1) {
#pragma unroll
      for (int j = 0; j < kSortItems; ++j) {
        const uint32_t idx = (uint32_t)(w * kSortItems * fc::kWave + j * fc::kWave + lane);
        if (idx < nvalid) {
          kout[base + idx] = k[j];
          vout[base + idx] = v[j];
        }
      }
      __syncthreads();  // s_tile is read
      continue;
    }
    const uint32_t hcount = g.hist[((uint64_t)gr * lo_digits + pass) * kRadix + tid];
    // (past a group's end: digit 255, behind the tile's own elements)
#pragma unroll
    for (int j = 0; j < kSortItems; ++j) rk[j] = wave_digit_rank((k[j] >> shift) & 0xFF, s_wcnt[w]);
    __syncthreads();
    const uint32_t t = (uint32_t)tid;  // this thread's digit
    uint32_t total = 0;
#pragma unroll
    for (int ww = 0; ww < kWaves; ++ww) {
      const uint32_t c = s_wcnt[ww][t];
      s_wcnt[ww][t] = (uint16_t)total;
      total += c;
    }
    const uint32_t slot0 = uniform(g.stat0[gr]), slot = slot0 + (tile - t0);
    const bool seen = (uint64_t)(tile - t0 + 1) * kSortTile < size;  // a later tile of the group looks back here
    uint64_t* mine = status + (uint64_t)slot * kRadix + t;
    if (seen)
      __hip_atomic_store(mine, pack_status(epoch, tile > t0 ? kFlagAgg : kFlagInc, total), __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
    s_dstart[t] = (uint16_t)fc::block_excl_sum<uint32_t>(total, s_scan, nullptr);
    const uint32_t dbase = fc::block_excl_sum<uint32_t>(hcount, s_scan, nullptr);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kSortItems; ++j) {
      const uint32_t idx = (uint32_t)(w * kSortItems * fc::kWave + j * fc::kWave + lane);
      if (idx < nvalid) {
        const uint32_t d = (k[j] >> shift) & 0xFF;
        const uint32_t pos = s_dstart[d] + s_wcnt[w][d] + rk[j];
        s_keys[pos] = k[j];
        s_vals[pos] = v[j];
      }
      if (j % 4 == 3) __builtin_amdgcn_sched_barrier(0);  // or their addresses spill
    }
    const uint64_t excl = look_back(status, (int64_t)slot - 1, (int64_t)slot0, t, epoch, err);
    if (tile > t0 && seen)
      __hip_atomic_store(mine, pack_status(epoch, kFlagInc, excl + total), __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
    s_gbase[t] = dbase + (uint32_t)excl;
    __syncthreads();
    for (uint32_t i = (uint32_t)tid; i < nvalid; i += kSortThreads) {
      const uint32_t key = s_keys[i];
      const uint32_t d = (key >> shift) & 0xFF;
      const uint32_t dst = s_gbase[d] + (i - s_dstart[d]);
      if (dst < size) {  // always true unless a look-back gave up (then err is set)
        kout[gstart + dst] = key;
        vout[gstart + dst] = s_vals[i];
      }
    }
    __syncthreads();  // the next tile reuses the LDS
  }
}

// ------------------------------------------------------ group bookkeeping --

// A round's sorted list: round 0's 64-bit keys (one group), later (grp, lo).
template <bool kRound0>
struct Sorted {
  const uint64_t* keys;
  const uint32_t *grp, *lo;
};

// The heads among a wave's kSegItems * 64 consecutive positions from `base`,
// a bit per position, in scalar registers: every element is loaded once (the
// one before it comes from the lane below), and what follows from the heads -
// an element's group start, the elements kept before it - is a bit search or
// a population count instead of a scan over the lanes.  With the tile passes
// reading each element's neighbours from memory again and scanning the heads
// step by step over the lanes, all rounds of a 1B build took 46 + 8 ms
// (k_seg_apply, k_seg_partials) against 23 + 3.6; of a 10M build 653 + 116
// against 458 + 69 us.
template <bool kRound0>
struct WaveHeads {
  uint32_t U, base;
  uint64_t nu[kSegItems + 1];    // new-group heads, and every position from U on; [kSegItems]: the next position
  uint64_t old[kSegItems];       // old-group heads
  uint32_t grp[kRound0 ? 1 : kSegItems];

  // a step's positions below U
  __device__ uint64_t valid(int j) const {
    const uint64_t x0 = (uint64_t)base + (uint32_t)(j * fc::kWave);
    return x0 >= U ? 0ull : U - x0 >= 64 ? ~0ull : (1ull << (U - x0)) - 1;
  }
  __device__ void load(const Sorted<kRound0>& in, uint32_t U_, uint32_t base_, uint32_t lane) {
    U = U_;
    base = base_;
    const uint64_t end = (uint64_t)base + kSegItems * fc::kWave;
    uint32_t k0[kSegItems], k1[kSegItems];  // round 0: the key's halves; later: lo, grp
#pragma unroll
    for (int j = 0; j < kSegItems; ++j) {
      const uint64_t r = (uint64_t)base + (uint32_t)(j * fc::kWave) + lane;
      if constexpr (kRound0) {
        const uint64_t k = r < U ? in.keys[r] : 0ull;
        k0[j] = (uint32_t)k;
        k1[j] = (uint32_t)(k >> 32);
      } else {
        k0[j] = r < U ? in.lo[r] : 0u;
        k1[j] = r < U ? in.grp[r] : 0u;
        grp[j] = k1[j];
      }
    }
    uint32_t c0 = 0, c1 = 0, e0 = 0, e1 = 0;  // the elements before and after the wave's
    if (base > 0 && base <= U) at(in, base - 1, c0, c1);
    if (end < U) at(in, end, e0, e1);
#pragma unroll
    for (int j = 0; j < kSegItems; ++j) {
      const uint64_t x0 = (uint64_t)base + (uint32_t)(j * fc::kWave);
      const bool first = x0 + lane == 0;
      const uint32_t p0 = fc::wave_shr1(k0[j], c0), p1 = fc::wave_shr1(k1[j], c1);
      nu[j] = fc::ballot(first || k0[j] != p0 || k1[j] != p1) | ~valid(j);
      old[j] = (kRound0 ? fc::ballot(first) : fc::ballot(first || k1[j] != p1)) & valid(j);
      c0 = (uint32_t)__builtin_amdgcn_readlane((int)k0[j], fc::kWave - 1);
      c1 = (uint32_t)__builtin_amdgcn_readlane((int)k1[j], fc::kWave - 1);
    }
    nu[kSegItems] = end >= U || e0 != c0 || e1 != c1 ? 1ull : 0ull;
  }
  static __device__ void at(const Sorted<kRound0>& in, uint64_t r, uint32_t& a, uint32_t& b) {
    if constexpr (kRound0) {
      a = uniform((uint32_t)in.keys[r]);
      b = uniform((uint32_t)(in.keys[r] >> 32));
    } else {
      a = uniform(in.lo[r]);
      b = uniform(in.grp[r]);
    }
  }
  // still tied: not a head right before another head
  __device__ uint64_t keep(int j) const { return valid(j) & ~(nu[j] & ((nu[j] >> 1) | (nu[j + 1] << 63))); }
  // last position of a step's mask (base + 64 j ..), or `before`
  static __device__ uint32_t last(uint64_t mask, uint32_t x0, uint32_t before) {
    return mask ? x0 + 63u - (uint32_t)__builtin_clzll(mask) : before;
  }
  // the wave's last new and old heads (0: none) and its kept elements
  __device__ void totals(uint32_t& h, uint32_t& g, uint32_t& k) const {
    h = g = k = 0;
#pragma unroll
    for (int j = 0; j < kSegItems; ++j) {
      h = last(nu[j] & valid(j), base + (uint32_t)(j * fc::kWave), h);
      g = last(old[j], base + (uint32_t)(j * fc::kWave), g);
      k += (uint32_t)__popcll(keep(j));
    }
  }
};

// Per tile: last new-group head, last old-group head, number kept.
template <bool kRound0>
__global__ void __launch_bounds__(kSegThreads) k_seg_partials(Sorted<kRound0> in, uint32_t U,
                                                                uint32_t* __restrict__ part_h,
                                                                uint32_t* __restrict__ part_g,
                                                                uint32_t* __restrict__ part_k) {
  constexpr int kWaves = kSegThreads / fc::kWave;
  __shared__ uint32_t s_tot[3][kWaves];
  const int w = (int)uniform(threadIdx.x / fc::kWave);
  const uint32_t lane = (uint32_t)fc::lane_id();
  const uint32_t base = blockIdx.x * kSegTile + (uint32_t)(w * kSegItems * fc::kWave);
  WaveHeads<kRound0> hd;
  hd.load(in, U, base, lane);
  uint32_t h, g, k;
  hd.totals(h, g, k);
  if (lane == 0) {
    s_tot[0][w] = h;
    s_tot[1][w] = g;
    s_tot[2][w] = k;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    h = g = k = 0;
    for (int v = 0; v < kWaves; ++v) {
      h = s_tot[0][v] > h ? s_tot[0][v] : h;
      g = s_tot[1][v] > g ? s_tot[1][v] : g;
      k += s_tot[2][v];
    }
    part_h[blockIdx.x] = h;
    part_g[blockIdx.x] = g;
    part_k[blockIdx.x] = k;
  }
}

// One workgroup: exclusive max / max / sum scans of the tile partials, in
// place; *u_next receives the number kept.  The partials are taken in chunks
// of kScanThreads * kScanRun, each thread a run of kScanRun consecutive ones
// (so a wave's loads and stores cover contiguous memory), with the chunk
// totals carried from chunk to chunk.
constexpr int kScanRun = 8;
__global__ void __launch_bounds__(kScanThreads) k_seg_scan(uint32_t* __restrict__ part_h,
                                                             uint32_t* __restrict__ part_g,
                                                             uint32_t* __restrict__ part_k, uint32_t ntiles,
                                                             uint32_t* __restrict__ u_next) {
  __shared__ uint32_t scratch[kScanThreads / fc::kWave + 1];
  __shared__ uint32_t s_last[3];
  uint32_t ch = 0, cg = 0, ck = 0;  // carries: maxima and sum over the earlier chunks
  for (uint32_t c0 = 0; c0 < ntiles; c0 += kScanThreads * kScanRun) {
    const uint32_t b0 = c0 + threadIdx.x * kScanRun;
    uint32_t h[kScanRun], g[kScanRun], k[kScanRun];
#pragma unroll
    for (int j = 0; j < kScanRun; ++j) {
      const uint32_t i = b0 + (uint32_t)j;
      h[j] = i < ntiles ? part_h[i] : 0u;
      g[j] = i < ntiles ? part_g[i] : 0u;
      k[j] = i < ntiles ? part_k[i] : 0u;
    }
    uint32_t mh = 0, mg = 0, kc = 0;
#pragma unroll
    for (int j = 0; j < kScanRun; ++j) {
      mh = h[j] > mh ? h[j] : mh;
      mg = g[j] > mg ? g[j] : mg;
      kc += k[j];
    }
    uint32_t total;
    uint32_t eh = fc::block_excl_max<uint32_t>(mh, 0u, scratch);
    uint32_t eg = fc::block_excl_max<uint32_t>(mg, 0u, scratch);
    uint32_t ek = fc::block_excl_sum<uint32_t>(kc, scratch, &total);
    eh = eh > ch ? eh : ch;
    eg = eg > cg ? eg : cg;
    ek += ck;
#pragma unroll
    for (int j = 0; j < kScanRun; ++j) {
      const uint32_t i = b0 + (uint32_t)j;
      if (i < ntiles) {
        part_h[i] = eh;
        part_g[i] = eg;
        part_k[i] = ek;
      }
      eh = h[j] > eh ? h[j] : eh;
      eg = g[j] > eg ? g[j] : eg;
      ek += k[j];
    }
    if (threadIdx.x == kScanThreads - 1) {
      s_last[0] = eh;
      s_last[1] = eg;
      s_last[2] = ek;
    }
    __syncthreads();
    ch = s_last[0];
    cg = s_last[1];
    ck = s_last[2];
    __syncthreads();
  }
  if (threadIdx.x == 0) *u_next = ck;
}

// Where a round's new ranks go when the rank array outgrows the MALL (a
// random 4-byte write then costs a 32-byte memory write): as (suffix << 32 |
// rank) pairs into the bucket of the suffix's high bits, then split by lower
// bits into windows of kRankWin suffixes (k_rank_split), and each window is
// put together in LDS (k_rank_window).  A suffix occurs once in a round, so a
// bucket or a window has room for all of its suffixes at its own place in the
// buffer, [d << shift, (d + 1) << shift), and its elements come in any order:
// each tile reserves room for its share of a bucket with one atomic, with no
// histogram and no look-back.  Against sorting the pairs by the suffix's top
// 24 bits (a histogram and three onesweep passes, then stores that fell on a
// few lines per wave): 1B suffixes, six rounds: 66 ms (5 counting, 51 sorting, 10
// storing) -> 35 (13 more in k_seg_apply, 13 splitting, 10 windows).
struct RankParts {
  uint64_t* out;
  uint32_t* cursor;  // elements in each of up to 256 buckets
  int shift;
  uint64_t n;        // suffixes, and room in out
};
constexpr int kRankWinBits = 14;                 // a window's ranks: 64 KB of LDS, two workgroups per CU
constexpr uint32_t kRankWin = 1u << kRankWinBits;
constexpr int kRankSplitMax = 1024;              // windows of a bucket, at most
constexpr uint64_t kPairRanksMin = 1ull << 26;   // suffixes (4-byte ranks: 256 MB)

// Per element: new rank = old group start + (new head index - old head index)
// in the sorted list; tied suffixes are compacted into (grp_next, val_next)
// with their new rank as the group.  A suffix
// whose group is now a singleton has its final index, so its suffix array
// entry is written here (sa_out, unless null), in sorted order.  The ranks
// go to rank[] directly (a random 4-byte write each), or, with kParts, into
// the buckets of RankParts.  Wave w of
// the tile takes positions [w * 1024, (w + 1) * 1024) of it, 64 consecutive
// ones per step: the running head indexes and the kept count are carried from
// step to step, started from the earlier waves' totals and the tile prefix.
template <bool kRound0, bool kParts>
__global__ void __launch_bounds__(kSegThreads) k_seg_apply(Sorted<kRound0> in, const uint32_t* __restrict__ vals,
                                                             uint32_t U, const uint32_t* __restrict__ pre_h,
                                                             const uint32_t* __restrict__ pre_g,
                                                             const uint32_t* __restrict__ pre_k,
                                                             uint32_t* __restrict__ rank, RankParts parts,
                                                             uint32_t* __restrict__ val_next,
                                                             uint32_t* __restrict__ grp_next,
                                                             uint32_t* __restrict__ sa_out) {
  constexpr int kWaves = kSegThreads / fc::kWave;
  constexpr uint32_t kPerWave = kSegTile / kWaves;
  __shared__ uint32_t s_tot[3][kWaves];
  __shared__ uint32_t s_cnt[kParts ? kRadix : 1], s_start[kParts ? kRadix : 1], s_base[kParts ? kRadix : 1];
  __shared__ uint32_t s_scan[kWaves + 1];
  __shared__ uint64_t s_pair[kParts ? kSegTile : 1];
  const int w = (int)uniform(threadIdx.x / fc::kWave);
  const uint32_t lane = (uint32_t)fc::lane_id();
  const uint32_t base = blockIdx.x * kSegTile + (uint32_t)w * kPerWave;
  if (kParts) s_cnt[threadIdx.x] = 0;
  uint32_t val[kSegItems];
#pragma unroll
  for (int j = 0; j < kSegItems; ++j) {
    const uint64_t r = (uint64_t)base + (uint32_t)(j * fc::kWave) + lane;
    val[j] = r < U ? vals[r] : 0u;
  }
  WaveHeads<kRound0> hd;
  hd.load(in, U, base, lane);
  uint32_t mh, mg, kc;
  hd.totals(mh, mg, kc);
  if (lane == 0) {
    s_tot[0][w] = mh;
    s_tot[1][w] = mg;
    s_tot[2][w] = kc;
  }
  __syncthreads();
  // running over the earlier tiles, the earlier waves and the wave's steps:
  // the last new and old heads, the kept elements
  uint32_t hh = pre_h[blockIdx.x], gg = pre_g[blockIdx.x], out = pre_k[blockIdx.x];
  for (int v = 0; v < w; ++v) {
    hh = s_tot[0][v] > hh ? s_tot[0][v] : hh;
    gg = s_tot[1][v] > gg ? s_tot[1][v] : gg;
    out += s_tot[2][v];
  }
  hh = uniform(hh);
  gg = uniform(gg);
  out = uniform(out);
  const uint64_t lt = fc::lanemask_lt(), le = lt | (1ull << lane);
  uint32_t pr[kParts ? kSegItems : 1], pos[kParts ? kSegItems : 1];
#pragma unroll
  for (int j = 0; j < kSegItems; ++j) {
    const uint32_t x0 = base + (uint32_t)(j * fc::kWave);
    const uint64_t nu = hd.nu[j] & hd.valid(j), keep = hd.keep(j);
    const uint32_t hr = hd.last(nu & le, x0, hh), gr = hd.last(hd.old[j] & le, x0, gg);
    const uint32_t kr = (uint32_t)__popcll(keep & lt);
    if (kParts) pos[j] = kNone;
    if ((hd.valid(j) >> lane) & 1) {
      uint32_t start = 0u;
      if constexpr (!kRound0) start = hd.grp[j];
      const uint32_t i = val[j];
      const uint32_t rk = start + (hr - gr);
      // in the first new group of its old group a suffix keeps its rank (the
      // old group start, already in rank[i]): only round 0 and the later
      // new groups write
      if (kRound0 || hr != gr) {
        if (kParts) {
          pr[j] = rk;
          pos[j] = atomicAdd(&s_cnt[(i >> parts.shift) & (kRadix - 1)], 1u);
        } else {
          rank[i] = rk;
        }
      }
      if ((keep >> lane) & 1) {
        val_next[out + kr] = i;
        grp_next[out + kr] = rk;
      }
      else if (sa_out) sa_out[rk] = i;  // a singleton group: rk is the suffix's final index
    }
    hh = hd.last(nu, x0, hh);
    gg = hd.last(hd.old[j], x0, gg);
    out += (uint32_t)__popcll(keep);
  }
  if constexpr (kParts) {
    __syncthreads();
    const uint32_t t = threadIdx.x, mine = s_cnt[t];  // this thread's bucket
    const uint32_t got = mine ? atomicAdd(&parts.cursor[t], mine) : 0u;
    uint32_t all;
    s_start[t] = fc::block_excl_sum<uint32_t>(mine, s_scan, &all);
    s_base[t] = got;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kSegItems; ++j)
      if (pos[j] != kNone)
        s_pair[s_start[(val[j] >> parts.shift) & (kRadix - 1)] + pos[j]] = ((uint64_t)val[j] << 32) | pr[j];
    __syncthreads();
    for (uint32_t x = threadIdx.x; x < all; x += kSegThreads) {
      const uint64_t p = s_pair[x];
      const uint32_t d = ((uint32_t)(p >> 32) >> parts.shift) & (kRadix - 1);
      const uint64_t at = ((uint64_t)d << parts.shift) + s_base[d] + (x - s_start[d]);
      if (at < parts.n) parts.out[at] = p;  // always true unless a look-back gave up (then err is set)
    }
  }
}

// Bucket blockIdx.x % buckets (its elements: cursor[bucket]) into its windows,
// tile after tile.  (Workgroups are dealt to the eight XCDs in turn, so a
// bucket's are on one XCD, and share its L2, only where the number of buckets is
// a multiple of eight; at 1B suffixes there are 239.)
constexpr int kSplitThreads = 512;
constexpr int kSplitItems = 16;
constexpr uint32_t kSplitTile = kSplitThreads * kSplitItems;
__global__ void __launch_bounds__(kSplitThreads) k_rank_split(RankParts from, uint32_t buckets,
                                                               uint64_t* __restrict__ out,
                                                               uint32_t* __restrict__ win_count) {
  __shared__ uint32_t s_cnt[kRankSplitMax], s_start[kRankSplitMax], s_base[kRankSplitMax];
  __shared__ uint32_t s_scan[kSplitThreads / fc::kWave + 1];
  __shared__ uint64_t s_pair[kSplitTile];
  const uint32_t d = blockIdx.x % buckets;
  const uint64_t d0 = (uint64_t)d << from.shift;
  const uint64_t room = from.n - d0 < (1ull << from.shift) ? from.n - d0 : 1ull << from.shift;
  const uint32_t got = uniform(from.cursor[d]), count = got < room ? got : (uint32_t)room;
  const int splits = 1 << (from.shift - kRankWinBits);
  const uint64_t* __restrict__ src = from.out + d0;
  uint32_t* const wc = win_count + ((uint64_t)d << (from.shift - kRankWinBits));
  constexpr int kPer = kRankSplitMax / kSplitThreads;
  for (uint64_t t0 = (uint64_t)(blockIdx.x / buckets) * kSplitTile; t0 < count;
       t0 += (uint64_t)(gridDim.x / buckets) * kSplitTile) {
    for (int i = (int)threadIdx.x; i < kRankSplitMax; i += kSplitThreads) s_cnt[i] = 0;
    __syncthreads();
    uint64_t p[kSplitItems];
    uint32_t pos[kSplitItems];
#pragma unroll
    for (int j = 0; j < kSplitItems; ++j) {
      const uint64_t i = t0 + (uint64_t)(j * kSplitThreads) + threadIdx.x;
      p[j] = i < count ? src[i] : 0ull;
    }
#pragma unroll
    for (int j = 0; j < kSplitItems; ++j) {
      const uint64_t i = t0 + (uint64_t)(j * kSplitThreads) + threadIdx.x;
      const uint32_t sub = (uint32_t)(p[j] >> (32 + kRankWinBits)) & (uint32_t)(splits - 1);
      pos[j] = i < count ? atomicAdd(&s_cnt[sub], 1u) : kNone;
    }
    __syncthreads();
    uint32_t c[kPer], sum = 0;
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int sub = (int)threadIdx.x * kPer + u;
      c[u] = s_cnt[sub];  // 0 past the bucket's windows
      s_base[sub] = c[u] ? atomicAdd(&wc[sub], c[u]) : 0u;
      sum += c[u];
    }
    uint32_t all;
    uint32_t run = fc::block_excl_sum<uint32_t>(sum, s_scan, &all);
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      s_start[(int)threadIdx.x * kPer + u] = run;
      run += c[u];
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kSplitItems; ++j)
      if (pos[j] != kNone) s_pair[s_start[(uint32_t)(p[j] >> (32 + kRankWinBits)) & (uint32_t)(splits - 1)] + pos[j]] = p[j];
    __syncthreads();
    for (uint32_t x = threadIdx.x; x < all; x += kSplitThreads) {
      const uint64_t q = s_pair[x];
      const uint32_t win = (uint32_t)(q >> (32 + kRankWinBits)), sub = win & (uint32_t)(splits - 1);
      const uint64_t at = ((uint64_t)win << kRankWinBits) + s_base[sub] + (x - s_start[sub]);
      if (at < from.n) out[at] = q;  // always (as above)
    }
    __syncthreads();  // the next tile reuses the LDS
  }
}

// Window blockIdx.x of the rank array.  One that changes in part is read
// first; one that changes in few places takes the stores directly (they fall
// on 64 KB).
__global__ void __launch_bounds__(kSplitThreads) k_rank_window(const uint64_t* __restrict__ pairs,
                                                               const uint32_t* __restrict__ win_count, uint64_t n,
                                                               uint32_t* __restrict__ rank) {
  __shared__ uint32_t s_rank[kRankWin];
  const uint64_t w0 = (uint64_t)blockIdx.x << kRankWinBits;
  const uint32_t size = n - w0 < kRankWin ? (uint32_t)(n - w0) : kRankWin;
  const uint32_t got = uniform(win_count[blockIdx.x]), count = got < size ? got : size;
  const uint64_t* __restrict__ src = pairs + w0;
  uint32_t* const dst = rank + w0;
  if (count <= size / 8) {
    for (uint32_t i = threadIdx.x; i < count; i += kSplitThreads) {
      const uint64_t p = src[i];
      if ((p >> 32) < n) rank[p >> 32] = (uint32_t)p;
    }
    return;
  }
  if (count < size) {
#pragma unroll 8
    for (uint32_t i = threadIdx.x; i < size; i += kSplitThreads) s_rank[i] = dst[i];
    __syncthreads();
  }
#pragma unroll 8
  for (uint32_t i = threadIdx.x; i < count; i += kSplitThreads) {
    const uint64_t p = src[i];
    s_rank[(uint32_t)(p >> 32) & (kRankWin - 1)] = (uint32_t)p;
  }
  __syncthreads();
#pragma unroll 8
  for (uint32_t i = threadIdx.x; i < size; i += kSplitThreads) dst[i] = s_rank[i];
}

// ------------------------------------------------------- first-token table --

__global__ void __launch_bounds__(256) k_bucket(const uint16_t* __restrict__ tok, const uint32_t* __restrict__ sa,
                                                  uint32_t n, uint32_t* __restrict__ bucket) {
  const uint32_t t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= FC_BUCKETS) return;
  // first SA index whose suffix starts with a token >= t
  uint32_t lo = 0, hi = n;
  while (lo < hi) {
    const uint32_t mid = lo + (hi - lo) / 2;
    if ((uint32_t)tok[sa[mid]] < t) lo = mid + 1; else hi = mid;
  }
  bucket[t] = lo;
}

// Largest token of a store (out[0] starts at 0).  Sixteen bytes a lane, and
// one atomic per workgroup that could raise the result: an atomic per wave of
// a 4,096-workgroup grid on the one word took 190 us whatever the size.
__global__ void __launch_bounds__(256) k_max_token(const uint16_t* __restrict__ tok, uint32_t n,
                                                   uint32_t* __restrict__ out) {
  __shared__ uint32_t scratch[256 / fc::kWave];
  uint32_t mx = 0;
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  const uint64_t id = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  // 16-byte pieces from the first 16-byte boundary; the tokens around them one by one
  const uint32_t to16 = (uint32_t)((16 - ((uintptr_t)tok & 15)) & 15) / 2;
  const uint32_t head = to16 < n ? to16 : n;
  const uint64_t pieces = (n - head) / 8;
  const uint4* q = (const uint4*)(tok + head);
  for (uint64_t i = id; i < pieces; i += stride) {
    const uint4 x = q[i];
    const uint32_t w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      mx = (w[u] & 0xFFFFu) > mx ? (w[u] & 0xFFFFu) : mx;
      mx = (w[u] >> 16) > mx ? (w[u] >> 16) : mx;
    }
  }
  const uint64_t rest = head + pieces * 8;  // fewer than eight tokens from here on
  if (id < head) mx = tok[id] > mx ? tok[id] : mx;
  if (id < n - rest) mx = tok[rest + id] > mx ? tok[rest + id] : mx;
  mx = fc::block_max<uint32_t>(mx, scratch);
  if (threadIdx.x == 0 && mx > __hip_atomic_load(out, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(out, mx);
}
constexpr uint32_t kMaxTokenBlocks = 1024;

// Two-token table: suffix-array position r owns the table entries between
// the previous suffix's pair key (exclusive) and its own (inclusive); keys
// never decrease along the suffix array.  r = n owns the rest up to the
// final entry.
struct PairKeys {
  const uint16_t* __restrict__ tok;
  const uint32_t* __restrict__ sa;
  uint32_t n, V;
  __device__ uint64_t end() const { return (uint64_t)V * (V + 1); }
  __device__ uint32_t suffix(uint64_t r) const { return r < n ? sa[r] : 0u; }
  // suffix j's first two tokens in one load (those of the text's last two for the last suffix)
  __device__ uint32_t two(uint32_t j) const {
    return *(const fc::u32_a2*)(tok + (j < n - 2 ? j : n - 2));
  }
  // position r's key; tokens are < V (checked before the launch)
  __device__ uint64_t key(uint64_t r, uint32_t j, uint32_t t) const {
    const bool whole = j + 1 < n;
    const uint64_t t0 = whole ? t & 0xFFFFu : t >> 16;
    return r < n ? t0 * (V + 1) + (whole ? (t >> 16) + 1u : 0u) : end();
  }
};

__device__ __forceinline__ uint64_t readlane64(uint64_t x, int l) {
  return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), l) << 32) |
         (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, l);
}

// The ranges of the lanes whose key differs from the one before, one after
// another with all 64 lanes, so long ranges are written in coalesced runs.
// (A first key before ~0: entry 0 on.)
__device__ __forceinline__ void write_pair_ranges(uint64_t key, uint64_t prev, uint32_t r, bool valid, int lane,
                                                  uint32_t* __restrict__ pair) {
  uint64_t heads = fc::ballot(valid && key != prev);
  while (heads) {
    const int l = __builtin_ctzll(heads);
    heads &= heads - 1;
    const uint64_t from = readlane64(prev, l) + 1, to = readlane64(key, l);
    const uint32_t val = (uint32_t)__builtin_amdgcn_readlane((int)r, l);
    for (uint64_t k = from + (uint64_t)lane; k <= to; k += fc::kWave) pair[k] = val;
  }
}

// A one-token store: 0 up to its only key (its token, then nothing), 1 after it.
__global__ void __launch_bounds__(256) k_pairs_one(PairKeys pk, uint32_t* __restrict__ pair) {
  const uint64_t key = (uint64_t)pk.tok[0] * (pk.V + 1);
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t k = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; k <= pk.end(); k += stride)
    pair[k] = k <= key ? 0u : 1u;
}

// A small store's table (n >= 2): a wave reads 64 consecutive positions.
__global__ void __launch_bounds__(256) k_pairs(PairKeys pk, uint32_t* __restrict__ pair) {
  const uint64_t base = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) & ~(uint64_t)(fc::kWave - 1);
  const int lane = fc::lane_id();
  if (base > pk.n) return;  // whole wave
  const uint64_t r = base + (uint64_t)lane, rb = base > 0 ? base - 1 : 0;
  const uint32_t j = pk.suffix(r), jb = pk.suffix(rb);
  const uint32_t t = pk.two(j), tb = pk.two(jb);
  const uint64_t key = pk.key(r, j, t), before = base > 0 ? pk.key(rb, jb, tb) : ~0ull;
  const uint64_t prev = ((uint64_t)fc::wave_shr1((uint32_t)(key >> 32), (uint32_t)(before >> 32)) << 32) |
                        fc::wave_shr1((uint32_t)key, (uint32_t)before);
  write_pair_ranges(key, prev, (uint32_t)r, r <= pk.n, lane, pair);
}

// A large store's: most neighbours share their pair, and a random 4-byte read
// of the text moves a whole line, so a wave reads every kPairStep-th of 512
// positions, and those between two only where they differ.  The groups
// (p, p + kPairStep] of positions that need it are taken eight at a time.
// 100M suffixes, 32,256 tokens (a 4.16 GB table): 1.75 ms; 2.55 with every
// position read once, 3.64 with every position's two tokens read twice and 64
// steps over ranges, most of them empty, per wave.  Below kPairSampleMin the
// table's own size decides and 512 positions per wave are too few waves.
constexpr int kPairStep = 8;
constexpr uint32_t kPairSpan = fc::kWave * kPairStep;  // positions per wave
constexpr uint64_t kPairSampleMin = 1ull << 23;        // suffixes
__global__ void __launch_bounds__(256) k_pairs_sampled(PairKeys pk, uint32_t* __restrict__ pair) {
  const uint64_t base = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) / fc::kWave * kPairSpan;
  const int lane = fc::lane_id();
  if (base > pk.n) return;  // whole wave
  // lane l: the position before its group, base - 1 + 8 l (position -1: ~0); and the wave's last position
  const uint64_t r0 = base + (uint64_t)(lane * kPairStep), re = base + kPairSpan - 1;
  const uint32_t j0 = pk.suffix(r0 > 0 ? r0 - 1 : 0), je = pk.suffix(re);
  const uint32_t t0 = pk.two(j0), te = pk.two(je);
  const uint64_t k0 = r0 > 0 ? pk.key(r0 - 1, j0, t0) : ~0ull, ke = pk.key(re, je, te);
  uint64_t k1 = __shfl_down(k0, 1);
  if (lane == fc::kWave - 1) k1 = ke;
  uint64_t open = fc::ballot(k0 != k1);  // groups with a head
  const int x = lane % kPairStep;
  while (open) {
    uint64_t rest = open;
    int g = -1;
#pragma unroll
    for (int u = 0; u < fc::kWave / kPairStep; ++u) {
      if (rest && lane / kPairStep == u) g = __builtin_ctzll(rest);
      rest &= rest - 1;
    }
    open = rest;
    const uint64_t r = base + (uint64_t)((g < 0 ? 0 : g) * kPairStep + x);
    uint64_t first = __shfl(k0, g < 0 ? 0 : g), key = __shfl(k1, g < 0 ? 0 : g);  // every lane takes part
    if (g >= 0 && x < kPairStep - 1) {
      const uint32_t j = pk.suffix(r);
      key = pk.key(r, j, pk.two(j));
    }
    const uint64_t below = ((uint64_t)fc::wave_shr1((uint32_t)(key >> 32), 0u) << 32) | fc::wave_shr1((uint32_t)key, 0u);
    write_pair_ranges(key, x == 0 ? first : below, (uint32_t)r, g >= 0 && r <= pk.n, lane, pair);
  }
}

// Inline-prefix records {sa[i], T[sa[i]+2 .. sa[i]+32)}: the 64 bytes of text
// at the suffix with its first two tokens replaced by the suffix's index.
// Four lanes per record, one 16-byte piece each: the four loads fall on the
// record's own 64 bytes of text (at the text's 2-byte alignment) and a wave's
// store covers 1 KB of consecutive records.  Each thread takes kRecRun
// pieces, their loads issued together; pieces that leave the text are read
// token by token, 0 past the end.  Bound by random lines of the text: 100M
// records 3.52 ms (4.30 with a record per lane, where every load and store
// touched 64 places; stores marked non-temporal: no change).
constexpr int kRecRun = 4;
constexpr uint32_t kRecBlock = 64 * kRecRun;  // records per workgroup

__global__ void __launch_bounds__(256) k_records(const uint16_t* __restrict__ tok, const uint32_t* __restrict__ sa,
                                                 uint32_t n, uint4* __restrict__ rec) {
  static_assert(FC_RECORD_BYTES == 64 && FC_RECORD_TOKENS == 30, "record layout");
  const uint32_t piece = threadIdx.x & 3;
  const uint64_t i0 = (uint64_t)blockIdx.x * kRecBlock + threadIdx.x / 4;
  uint32_t j[kRecRun];
#pragma unroll
  for (int u = 0; u < kRecRun; ++u) j[u] = i0 + 64 * u < n ? sa[i0 + 64 * u] : 0u;
  fc::u32x4_a2 v[kRecRun];
  const uint32_t last = n < 8 ? 0u : n - 8;  // the last whole piece
  if (n >= 8) {
#pragma unroll
    for (int u = 0; u < kRecRun; ++u) {
      const uint64_t p = (uint64_t)j[u] + 8 * piece;
      v[u] = *(const fc::u32x4_a2*)(tok + (p < last ? p : last));
    }
  }
#pragma unroll
  for (int u = 0; u < kRecRun; ++u) {
    const uint64_t i = i0 + 64 * u;
    if (i >= n) continue;
    const uint64_t p = (uint64_t)j[u] + 8 * piece;
    uint32_t w[4] = {0u, 0u, 0u, 0u};
    if (n >= 8 && p <= last) {
#pragma unroll
      for (int x = 0; x < 4; ++x) w[x] = v[u][x];
    } else {
#pragma unroll
      for (int x = 0; x < 8; ++x)
        if (p + x < n) w[x / 2] |= (uint32_t)tok[p + x] << (16 * (x & 1));
    }
    if (piece == 0) w[0] = j[u];
    rec[4 * i + piece] = make_uint4(w[0], w[1], w[2], w[3]);
  }
}

struct BuildWs {
  uint32_t* rank;
  uint64_t* keys[2];
  uint32_t* vals[2];
  uint64_t* status;
  uint32_t *part_h, *part_g, *part_k;
  uint32_t* hist;
  uint32_t* offsets;
  uint32_t* tickets;
  uint32_t* misc;      // [0] error flag, [1] tied suffixes, [2..2+kBigCounts) the large groups' counters, [10] largest token
  uint64_t* pairs;     // plain build: a round's (suffix, rank) pairs
  uint32_t* seg_bits;  // batched build: a bit per position that starts a segment
  uint64_t* seg_off;   // batched build: segment offsets (device copy)
};
static_assert(2 + kBigCounts <= 10, "misc words");

size_t carve_build(void* p, uint64_t n, BuildWs* w, uint32_t n_seg = 0) {
  fc::Carver c(p);
  const uint64_t tiles = (n + kSortTile - 1) / kSortTile;
  const uint64_t seg_tiles = (n + kSegTile - 1) / kSegTile;
  BuildWs tmp;
  tmp.rank = c.take<uint32_t>(n);
  tmp.keys[0] = c.take<uint64_t>(n);
  tmp.keys[1] = c.take<uint64_t>(n);
  tmp.vals[0] = c.take<uint32_t>(n);
  tmp.vals[1] = c.take<uint32_t>(n);
  tmp.status = c.take<uint64_t>(tiles * kRadix);
  tmp.part_h = c.take<uint32_t>(seg_tiles);
  tmp.part_g = c.take<uint32_t>(seg_tiles);
  tmp.part_k = c.take<uint32_t>(seg_tiles);
  tmp.hist = c.take<uint32_t>(kMaxDigits * kRadix);
  tmp.offsets = c.take<uint32_t>(kMaxDigits * kRadix);
  tmp.tickets = c.take<uint32_t>(kMaxDigits);
  tmp.misc = c.take<uint32_t>(16);
  tmp.seg_bits = n_seg ? c.take<uint32_t>(n / 32 + 1) : nullptr;
  tmp.seg_off = n_seg ? c.take<uint64_t>((size_t)n_seg + 1) : nullptr;
  tmp.pairs = n_seg == 0 && n >= kPairRanksMin ? c.take<uint64_t>(n) : nullptr;
  if (w) *w = tmp;
  return c.used + 256;
}

// The large groups' arrays, in 4 n bytes at p that a round leaves free.  A
// list of n elements has at most n / (kWin + 1) large groups, n / kWin tiles
// and n / kSortTile status slots; the histograms take 2 n bytes of the 4 n.
// Lists of up to kWin elements have no large group.
size_t carve_big(void* p, uint64_t n, BigWs* g) {
  fc::Carver c(p);
  const uint64_t groups = n / (kWin + 1);
  g->first_head = c.take<uint32_t>((n + kWin - 1) / kWin);
  g->start = c.take<uint32_t>(groups);
  g->size = c.take<uint32_t>(groups);
  g->tile0 = c.take<uint32_t>(groups);
  g->stat0 = c.take<uint32_t>(groups);
  g->tile_group = c.take<uint32_t>(n / kWin);  // ceil(size / kSortTile) < size / kWin for every large group
  g->same = c.take<uint32_t>(groups);
  g->hist = c.take<uint32_t>(groups * kMaxLoDigits * kRadix);
  return c.used;
}

int bit_length(uint64_t x) {
  int b = 0;
  while (x) {
    ++b;
    x >>= 1;
  }
  return b;
}

// LSD radix sort of round 0's keys over `digits` 8-bit digits, the suffixes
// carried alongside, the passes alternating between the two buffers; w.hist
// holds the digits' counts.  *result is the index (0 or 1) of the buffers that
// hold the result.
template <Mode M>
fc_status radix_passes(BuildWs& w, const FirstKeys<M>& fk, uint32_t U, int digits, uint32_t& epoch,
                       hipStream_t stream, int* result) {
  const uint32_t hist_blocks = fc::div_up(U, 1024) < (uint32_t)kHistBlocks ? fc::div_up(U, 1024) : kHistBlocks;
  hipLaunchKernelGGL(k_first_hist<M>, dim3(hist_blocks), dim3(256), 0, stream, fk, U, digits, w.hist);
  FC_CHECK_LAUNCH();
  hipLaunchKernelGGL(k_hist_scan, dim3(digits), dim3(256), 0, stream, w.hist, w.offsets);
  FC_CHECK_LAUNCH();
  int cur = 0;
  const uint32_t tiles = fc::div_up(U, kSortTile);
  for (int d = 0; d < digits; ++d) {
    ++epoch;
    auto pass = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, dim3(tiles), dim3(kSortThreads), 0, stream, fk, w.keys[cur], w.vals[cur],
                         w.keys[cur ^ 1], w.vals[cur ^ 1], U, (uint32_t)(8 * d), w.offsets + d * kRadix, w.status,
                         w.tickets + d, epoch, w.misc);
    };
    d == 0 ? pass(k_onesweep<M, true>) : pass(k_onesweep<M, false>);
    FC_CHECK_LAUNCH();
    cur ^= 1;
  }
  *result = cur;
  return FC_OK;
}

// The new suffixes of an extension (see FirstKeys).
struct ExtendArgs {
  const uint32_t* ins;  // per new position
  const uint32_t* isa;  // inverse of the old suffix array
  uint32_t* ins_sorted; // ins in the sorted order of the new suffixes
  uint64_t n;           // whole text
  int n_old_bits;
};

// The list of still-tied suffixes between two rounds, and what a round needs.
struct ListWs {
  uint32_t* grp[2];
  uint32_t* val[2];
  uint32_t* lo;
  BigWs big;
};

// Prefix doubling over all n suffixes (n_seg = 0), over the suffixes of
// n_seg segments at once, each ending at its segment's end (n_seg >= 1,
// offsets already in w.seg_off), or over the n new suffixes of an extension
// (ext; leaves their ranks in w.rank and writes no suffix array).
template <Mode M>
fc_status build_sa(const uint16_t* tokens, uint64_t n, uint32_t n_seg, BuildWs& w, uint32_t* sa_out,
                   hipStream_t stream, const ExtendArgs* ext = nullptr, fc_build_stats* stats = nullptr) {
  const uint32_t N = (uint32_t)n;
  const uint64_t tiles = (n + kSortTile - 1) / kSortTile;
  FC_CHECK_HIP(hipMemsetAsync(w.status, 0, sizeof(uint64_t) * tiles * kRadix, stream));
  FC_CHECK_HIP(hipMemsetAsync(w.tickets, 0, sizeof(uint32_t) * kMaxDigits, stream));
  FC_CHECK_HIP(hipMemsetAsync(w.misc, 0, sizeof(uint32_t) * 16, stream));
  FC_CHECK_HIP(hipMemsetAsync(w.hist, 0, sizeof(uint32_t) * kMaxDigits * kRadix, stream));

  // every rank + 1 <= n (an extension's labels: <= the whole text) fits in lo_digits bytes
  const int lo_digits = (bit_length(ext ? ext->n : n) + 7) / 8;
  uint32_t epoch = 0;  // of the status words: one per pass
  int key0_bits;
  int ext_shift = 0;
  FirstKeys<M> fk{tokens, ext ? ext->n : n, 17, 3, w.seg_off, n_seg, ext ? ext->ins : nullptr};
  if (M == Mode::kExtend) {
    fk.ntok = ext->n_old_bits + 34 <= 64 ? 2 : 1;
    ext_shift = 17 * fk.ntok;
    key0_bits = ext_shift + ext->n_old_bits;
  } else {
    // token + 1 in tb bits: the largest token decides tb (misc[10] is zero)
    const uint32_t blocks = fc::div_up(N, 2048) < kMaxTokenBlocks ? fc::div_up(N, 2048) : kMaxTokenBlocks;
    hipLaunchKernelGGL(k_max_token, dim3(blocks), dim3(256), 0, stream, tokens, N, w.misc + 10);
    FC_CHECK_LAUNCH();
    uint32_t mx = 0;
    FC_CHECK_HIP(hipMemcpyAsync(&mx, w.misc + 10, sizeof(uint32_t), hipMemcpyDeviceToHost, stream));
    FC_CHECK_HIP(hipStreamSynchronize(stream));
    fk.tb = bit_length((uint64_t)mx + 1);
    const int seg_bits = M == Mode::kBatched ? bit_length(n_seg - 1) : 0;
    if (M == Mode::kBatched) {
      fk.ntok = seg_bits + 3 * fk.tb <= 64 ? 3 : 2;  // 17-bit tokens and up to 2^30 segments: two always fit
      FC_CHECK_HIP(hipMemsetAsync(w.seg_bits, 0, sizeof(uint32_t) * (n / 32 + 1), stream));
      hipLaunchKernelGGL(k_seg_starts, dim3(fc::div_up(n_seg, 256)), dim3(256), 0, stream, w.seg_off, n_seg,
                         w.seg_bits);
      FC_CHECK_LAUNCH();
    }
    key0_bits = seg_bits + fk.ntok * fk.tb;
  }
  uint64_t h = (uint64_t)fk.ntok;
  int res = 0;
  // a lone suffix is in order: one pass makes its key (an extension by a single
  // token: 205 us with all eight, 163 with one)
  int sort_passes = N == 1 ? 1 : (key0_bits + 7) / 8;
  const fc_status s = radix_passes<M>(w, fk, N, sort_passes, epoch, stream, &res);
  if (s != FC_OK) return s;
  if (M == Mode::kExtend) {
    hipLaunchKernelGGL(k_ins_sorted, dim3(fc::div_up(N, 256)), dim3(256), 0, stream, w.keys[res], N, ext_shift,
                       ext->ins_sorted);
    FC_CHECK_LAUNCH();
  }
  // The lists live in the sort buffers: round 0's result is in keys[res] and
  // vals[res], so its tied suffixes go to the other two, and from then on
  // keys[res] is free as well (lo, and the large groups' arrays).
  ListWs L;
  L.grp[0] = (uint32_t*)w.keys[res ^ 1];
  L.grp[1] = L.grp[0] + n;
  L.val[0] = w.vals[res ^ 1];
  L.val[1] = w.vals[res];
  L.lo = (uint32_t*)w.keys[res];
  const uint64_t lo_words = (n + 63) & ~(uint64_t)63;  // keeps what follows aligned
  if (n > (uint64_t)kWin) {
    if (lo_words * 4 + carve_big(nullptr, n, &L.big) > 8 * n) return FC_ERR_DEVICE;
    carve_big(L.lo + lo_words, n, &L.big);
  } else {
    L.big = BigWs{};
    L.big.first_head = w.hist;  // the one window of a short list
  }
  L.big.count = w.misc + 2;
  // ranks through RankParts when the rank array is at least the size of the
  // 256 MB MALL; a smaller one takes the random writes in the MALL
  const bool pair_ranks = M == Mode::kPlain && n >= kPairRanksMin;
  NextRank nr{w.rank, w.seg_bits, ext ? ext->ins : nullptr, ext ? ext->isa : nullptr,
              ext ? ext->ins_sorted : nullptr, ext ? ext->n : n, h, N};

  uint32_t U = N;
  int cur = 1;  // the list a round sorts (round 0: none); the other one takes its tied suffixes
  for (int round = 0;; ++round) {
    if (round >= kMaxRounds) return FC_ERR_DEVICE;
    const uint32_t seg_tiles = fc::div_up(U, kSegTile);
    const Sorted<true> s0{w.keys[res], nullptr, nullptr};
    const Sorted<false> s1{nullptr, L.grp[cur], L.lo};
    const uint32_t* sorted_vals = round == 0 ? w.vals[res] : L.val[cur];
    if (round == 0)
      hipLaunchKernelGGL(k_seg_partials<true>, dim3(seg_tiles), dim3(kSegThreads), 0, stream, s0, U, w.part_h,
                         w.part_g, w.part_k);
    else
      hipLaunchKernelGGL(k_seg_partials<false>, dim3(seg_tiles), dim3(kSegThreads), 0, stream, s1, U, w.part_h,
                         w.part_g, w.part_k);
    FC_CHECK_LAUNCH();
    hipLaunchKernelGGL(k_seg_scan, dim3(1), dim3(kScanThreads), 0, stream, w.part_h, w.part_g, w.part_k, seg_tiles,
                       w.misc + 1);
    FC_CHECK_LAUNCH();
    if (pair_ranks) {
      // w.hist is free after the radix passes, the tile partials after k_seg_apply, lo's buffer until k_sort_small
      const int bits = bit_length(n - 1);
      const RankParts parts{w.pairs, w.hist, bits > 8 + kRankWinBits ? bits - 8 : kRankWinBits, n};
      const uint32_t buckets = (uint32_t)(((n - 1) >> parts.shift) + 1);  // <= 256
      const uint32_t windows = (uint32_t)((n + kRankWin - 1) >> kRankWinBits);
      FC_CHECK_HIP(hipMemsetAsync(w.hist, 0, sizeof(uint32_t) * kRadix, stream));
      if (round == 0)
        hipLaunchKernelGGL((k_seg_apply<true, true>), dim3(seg_tiles), dim3(kSegThreads), 0, stream, s0, sorted_vals,
                           U, w.part_h, w.part_g, w.part_k, w.rank, parts, L.val[cur ^ 1], L.grp[cur ^ 1], sa_out);
      else
        hipLaunchKernelGGL((k_seg_apply<false, true>), dim3(seg_tiles), dim3(kSegThreads), 0, stream, s1, sorted_vals,
                           U, w.part_h, w.part_g, w.part_k, w.rank, parts, L.val[cur ^ 1], L.grp[cur ^ 1], sa_out);
      FC_CHECK_LAUNCH();
      uint32_t* const win_count = w.part_h;  // a tile of the partials is smaller than a window
      static_assert((uint32_t)kSegTile <= kRankWin, "window counters fit the tile partials");
      FC_CHECK_HIP(hipMemsetAsync(win_count, 0, sizeof(uint32_t) * windows, stream));
      // enough workgroups per bucket for its tiles when the elements are spread evenly, up to a few per CU in all
      const uint32_t want = fc::div_up(U, kSplitTile * buckets), most = fc::div_up(2048, buckets);
      hipLaunchKernelGGL(k_rank_split, dim3(buckets * (want < most ? want : most)), dim3(kSplitThreads), 0, stream,
                         parts, buckets, w.keys[res], win_count);
      FC_CHECK_LAUNCH();
      hipLaunchKernelGGL(k_rank_window, dim3(windows), dim3(kSplitThreads), 0, stream, w.keys[res], win_count, n,
                         w.rank);
      FC_CHECK_LAUNCH();
    } else {
      const RankParts none{nullptr, nullptr, 0, 0};
      if (round == 0)
        hipLaunchKernelGGL((k_seg_apply<true, false>), dim3(seg_tiles), dim3(kSegThreads), 0, stream, s0, sorted_vals,
                           U, w.part_h, w.part_g, w.part_k, w.rank, none, L.val[cur ^ 1], L.grp[cur ^ 1],
                           ext ? nullptr : sa_out);
      else
        hipLaunchKernelGGL((k_seg_apply<false, false>), dim3(seg_tiles), dim3(kSegThreads), 0, stream, s1, sorted_vals,
                           U, w.part_h, w.part_g, w.part_k, w.rank, none, L.val[cur ^ 1], L.grp[cur ^ 1],
                           ext ? nullptr : sa_out);
      FC_CHECK_LAUNCH();
    }
    // the next round's small groups, launched before its size is known on
    // the host, so that one wait per round tells both the tied suffixes and
    // the large groups
    cur ^= 1;
    nr.h = h;
    if (U > 1) {  // a lone suffix is tied with none (a one-token store: 101 us before the group sorts, 83 now)
      FC_CHECK_HIP(hipMemsetAsync(L.big.count, 0, sizeof(uint32_t) * kBigCounts, stream));
      hipLaunchKernelGGL(k_sort_small<M>, dim3(fc::div_up(U, kWin)), dim3(kSmallThreads), 0, stream, L.grp[cur],
                         L.val[cur], L.lo, w.misc + 1, nr, lo_digits, L.big.first_head, L.big.start, L.big.count);
      FC_CHECK_LAUNCH();
    }
    uint32_t host_misc[3] = {0, 0, 0};
    FC_CHECK_HIP(hipMemcpyAsync(host_misc, w.misc, sizeof(uint32_t) * 3, hipMemcpyDeviceToHost, stream));
    FC_CHECK_HIP(hipStreamSynchronize(stream));
    if (host_misc[0]) return FC_ERR_DEVICE;
    if (stats && round < FC_MAX_BUILD_ROUNDS) {
      stats->prefix_len[round] = h;
      stats->sorted[round] = U;
      stats->unresolved[round] = host_misc[1];
      stats->rounds = round + 1;
      stats->sort_passes = sort_passes;
    }
    U = host_misc[1];
    if (U == 0) break;
    h *= 2;
    if (const uint32_t groups = host_misc[2]) {
      // passes alternate between (lo, val) and the next round's buffers, which
      // are free now; an odd number starts in those
      const BigBufs bufs{{L.lo, L.grp[cur ^ 1]}, {L.val[cur], L.val[cur ^ 1]}};
      const int from = lo_digits & 1;
      const uint32_t most = U / kWin;  // tiles, at most
      const uint32_t waves = groups < 4096u ? groups : 4096u;
      hipLaunchKernelGGL(k_big_plan, dim3(fc::div_up(waves, 4)), dim3(256), 0, stream, L.big, U, lo_digits);
      FC_CHECK_LAUNCH();
      const uint32_t kblocks = most < kBigKeysBlocks ? most : kBigKeysBlocks;
      hipLaunchKernelGGL(k_big_keys<M>, dim3(kblocks), dim3(256), 0, stream, L.big, L.val[cur], nr, lo_digits,
                         bufs.k[from], from ? bufs.v[1] : nullptr);
      FC_CHECK_LAUNCH();
      const uint32_t blocks = most < kBigPassBlocks ? most : kBigPassBlocks;
      for (int d = 0; d < lo_digits; ++d) {
        ++epoch;
        hipLaunchKernelGGL(k_big_pass, dim3(blocks), dim3(kSortThreads), 0, stream, L.big, d, lo_digits, bufs,
                           w.status, epoch, w.misc);
        FC_CHECK_LAUNCH();
        ++sort_passes;
      }
    }
  }
  if (M == Mode::kExtend) return FC_OK;
  // every suffix array entry was written when its suffix's group became a
  // singleton (k_seg_apply)
  if (M == Mode::kBatched) {
    hipLaunchKernelGGL(k_localize_sa, dim3(fc::div_up(N, 256)), dim3(256), 0, stream, sa_out, N, w.seg_off, n_seg);
    FC_CHECK_LAUNCH();
  }
  return FC_OK;
}

}  // namespace

extern "C" size_t fc_datastore_build_workspace_bytes(uint64_t n) { return carve_build(nullptr, n, nullptr); }

extern "C" fc_status fc_datastore_build_stats(const uint16_t* tokens, uint64_t n, uint32_t* sa_out, void* ws,
                                              size_t ws_bytes, fc_build_stats* stats, hipStream_t stream) {
  if (n >= 0xFFFFFFFFull) return FC_ERR_INVALID;
  if (stats) *stats = fc_build_stats{};
  if (n == 0) return FC_OK;
  if (!tokens || !sa_out) return FC_ERR_INVALID;
  if (!ws || ws_bytes < fc_datastore_build_workspace_bytes(n)) return FC_ERR_WORKSPACE;
  (void)hipGetLastError();
  BuildWs w;
  carve_build(ws, n, &w);
  return build_sa<Mode::kPlain>(tokens, n, 0, w, sa_out, stream, nullptr, stats);
}

extern "C" fc_status fc_datastore_build(const uint16_t* tokens, uint64_t n, uint32_t* sa_out, void* ws,
                                        size_t ws_bytes, hipStream_t stream) {
  return fc_datastore_build_stats(tokens, n, sa_out, ws, ws_bytes, nullptr, stream);
}

extern "C" size_t fc_datastore_build_batched_workspace_bytes(uint64_t n, int32_t n_seg) {
  return n_seg >= 1 ? carve_build(nullptr, n, nullptr, (uint32_t)n_seg) : 0;
}

extern "C" fc_status fc_datastore_build_batched(const uint16_t* tokens, const uint64_t* seg_off, int32_t n_seg,
                                                uint32_t* sa_out, void* ws, size_t ws_bytes, hipStream_t stream) {
  if (n_seg < 1 || !seg_off) return FC_ERR_INVALID;
  if (seg_off[0] != 0) return FC_ERR_INVALID;
  for (int32_t r = 0; r < n_seg; ++r)
    if (seg_off[r + 1] < seg_off[r]) return FC_ERR_INVALID;
  const uint64_t n = seg_off[n_seg];
  if (n >= 0xFFFFFFFFull || 34 + bit_length((uint64_t)n_seg - 1) > 64) return FC_ERR_INVALID;
  if (n == 0) return FC_OK;
  if (!tokens || !sa_out) return FC_ERR_INVALID;
  if (!ws || ws_bytes < fc_datastore_build_batched_workspace_bytes(n, n_seg)) return FC_ERR_WORKSPACE;
  (void)hipGetLastError();
  BuildWs w;
  carve_build(ws, n, &w, (uint32_t)n_seg);
  FC_CHECK_HIP(hipMemcpyAsync(w.seg_off, seg_off, sizeof(uint64_t) * ((size_t)n_seg + 1), hipMemcpyHostToDevice,
                              stream));
  return build_sa<Mode::kBatched>(tokens, n, (uint32_t)n_seg, w, sa_out, stream);
}

namespace {

struct ExtendWs {
  uint32_t* isa;  // inverse of the old array, unless the caller passes it
  uint32_t *lo[2], *hi[2];
  uint32_t *act[2], *done;
  uint32_t* counts;  // [0] still ranged, [1] final this round, [2] active now
  uint32_t* ins_sorted;
  uint32_t* coarse;
  BuildWs b;
};

uint32_t coarse_entries(uint64_t n_old) { return (uint32_t)((n_old + (1u << kCountShift) - 1) >> kCountShift) + 1; }

size_t carve_extend(void* p, uint64_t n, uint64_t o, bool isa_given, ExtendWs* w) {
  fc::Carver c(p);
  ExtendWs t;
  t.isa = c.take<uint32_t>(isa_given ? 0 : n - o);
  for (int i = 0; i < 2; ++i) {
    t.lo[i] = c.take<uint32_t>(o);
    t.hi[i] = c.take<uint32_t>(o);
    t.act[i] = c.take<uint32_t>(o);
  }
  t.done = c.take<uint32_t>(o);
  t.counts = c.take<uint32_t>(4);
  t.ins_sorted = c.take<uint32_t>(o);
  t.coarse = c.take<uint32_t>(coarse_entries(n - o));
  char* rest = p ? (char*)p + ((c.used + 255) & ~(size_t)255) : nullptr;
  const size_t head = (c.used + 255) & ~(size_t)255;
  const size_t tail = o ? carve_build(rest, o, &t.b) : 0;
  if (w) *w = t;
  return head + tail;
}

}  // namespace

extern "C" size_t fc_datastore_extend_workspace_bytes(uint64_t n, uint64_t n_new, int32_t isa_given) {
  return n_new <= n && n < 0xFFFFFFFFull ? carve_extend(nullptr, n, n_new, isa_given != 0, nullptr) : 0;
}

extern "C" fc_status fc_datastore_extend(const uint16_t* tokens, uint64_t n, uint64_t n_new, const uint32_t* old_sa,
                                         const uint32_t* old_isa, uint32_t* sa_out, uint32_t* isa_out, void* ws,
                                         size_t ws_bytes, hipStream_t stream) {
  if (n >= 0xFFFFFFFFull || n_new > n) return FC_ERR_INVALID;
  if (n == 0) return FC_OK;
  const uint32_t o = (uint32_t)n_new, n_old = (uint32_t)(n - n_new);
  if (!tokens || !sa_out || (n_old > 0 && !old_sa)) return FC_ERR_INVALID;
  const bool isa_given = old_isa != nullptr;
  if (!ws || ws_bytes < fc_datastore_extend_workspace_bytes(n, n_new, isa_given ? 1 : 0)) return FC_ERR_WORKSPACE;
  (void)hipGetLastError();
  ExtendWs w;
  carve_extend(ws, n, n_new, isa_given, &w);
  const uint32_t* isa = isa_given ? old_isa : w.isa;
  const bool need_isa = n_old > 0 && (o > 0 || isa_out);
  if (need_isa && !isa_given) {
    hipLaunchKernelGGL(k_isa, dim3(fc::div_up(n_old, 256)), dim3(256), 0, stream, old_sa, n_old, w.isa);
    FC_CHECK_LAUNCH();
  }
  if (o > 0) {
    FC_CHECK_HIP(hipMemsetAsync(w.counts, 0, sizeof(uint32_t) * 4, stream));
    hipLaunchKernelGGL(k_ext_init, dim3(fc::div_up(o, 256)), dim3(256), 0, stream, tokens, o, (uint64_t)n, old_sa,
                       n_old, w.lo[0], w.hi[0], w.lo[1], w.hi[1], w.act[0], w.counts + 2);
    FC_CHECK_LAUNCH();
    uint32_t n_act = 0;
    FC_CHECK_HIP(hipMemcpyAsync(&n_act, w.counts + 2, sizeof(uint32_t), hipMemcpyDeviceToHost, stream));
    FC_CHECK_HIP(hipStreamSynchronize(stream));
    int cur = 0;
    uint32_t* act_in = w.act[0];
    uint32_t* act_out = w.act[1];
    for (uint64_t h = kExtFirst; n_act > 0; h *= 2) {
      if (h > 2 * n) return FC_ERR_DEVICE;  // every new suffix is final once p + h reaches the old text
      FC_CHECK_HIP(hipMemsetAsync(w.counts, 0, sizeof(uint32_t) * 2, stream));
      hipLaunchKernelGGL(k_ext_round, dim3(fc::div_up(n_act, 256)), dim3(256), 0, stream, o, (uint64_t)n, n_old,
                         old_sa, isa, h, w.lo[cur], w.hi[cur], w.lo[cur ^ 1], w.hi[cur ^ 1], act_in,
                         w.counts + 2, act_out, w.done, w.counts);
      FC_CHECK_LAUNCH();
      hipLaunchKernelGGL(k_ext_fix, dim3(fc::div_up(n_act, 256)), dim3(256), 0, stream, w.done, w.counts + 1,
                         w.lo[cur ^ 1], w.lo[cur], w.hi[cur]);
      FC_CHECK_LAUNCH();
      FC_CHECK_HIP(hipMemcpyAsync(w.counts + 2, w.counts, sizeof(uint32_t), hipMemcpyDeviceToDevice, stream));
      FC_CHECK_HIP(hipMemcpyAsync(&n_act, w.counts, sizeof(uint32_t), hipMemcpyDeviceToHost, stream));
      FC_CHECK_HIP(hipStreamSynchronize(stream));
      uint32_t* t = act_in;
      act_in = act_out;
      act_out = t;
      cur ^= 1;
    }
    // every range is final and in both buffers: w.lo[0] holds ins
    ExtendArgs ea;
    ea.ins = w.lo[0];
    ea.isa = isa;
    ea.ins_sorted = w.ins_sorted;
    ea.n = n;
    ea.n_old_bits = bit_length(n_old);
    fc_status s = build_sa<Mode::kExtend>(tokens, o, 0, w.b, nullptr, stream, &ea);
    if (s != FC_OK) return s;
    hipLaunchKernelGGL(k_ext_new_out, dim3(fc::div_up(o, 256)), dim3(256), 0, stream, w.b.rank, w.lo[0], o, sa_out);
    FC_CHECK_LAUNCH();
    if (isa_out) {
      hipLaunchKernelGGL(k_ext_isa_new, dim3(fc::div_up(o, 256)), dim3(256), 0, stream, w.b.rank, w.lo[0], o,
                         isa_out);
      FC_CHECK_LAUNCH();
    }
  }
  if (n_old > 0) {
    const uint32_t nc = coarse_entries(n_old);
    if (o > 0) {
      hipLaunchKernelGGL(k_ext_coarse, dim3(fc::div_up(nc, 256)), dim3(256), 0, stream, w.ins_sorted, o, nc,
                         w.coarse);
      FC_CHECK_LAUNCH();
    }
    hipLaunchKernelGGL(k_ext_old_out, dim3(nc - 1), dim3(256), 0, stream, old_sa, n_old, w.ins_sorted, w.coarse, o,
                       sa_out);
    FC_CHECK_LAUNCH();
    if (isa_out) {
      hipLaunchKernelGGL(k_ext_isa_old, dim3(fc::div_up(n_old, 256)), dim3(256), 0, stream, isa, n_old, w.ins_sorted,
                         w.coarse, o, isa_out);
      FC_CHECK_LAUNCH();
    }
  }
  return FC_OK;
}

extern "C" fc_status fc_store_prepare(const uint16_t* tokens, const uint32_t* sa, uint64_t n, uint32_t* bucket_out,
                                      hipStream_t stream) {
  if (n >= 0xFFFFFFFFull || !bucket_out) return FC_ERR_INVALID;
  if (n > 0 && (!tokens || !sa)) return FC_ERR_INVALID;
  (void)hipGetLastError();
  hipLaunchKernelGGL(k_bucket, dim3(fc::div_up(FC_BUCKETS, 256)), dim3(256), 0, stream, tokens, sa, (uint32_t)n,
                     bucket_out);
  FC_CHECK_LAUNCH();
  return FC_OK;
}

extern "C" uint64_t fc_pair_table_entries(uint32_t V) { return (uint64_t)V * ((uint64_t)V + 1) + 1; }

extern "C" fc_status fc_store_prepare_pairs(const uint16_t* tokens, const uint32_t* sa, uint64_t n, uint32_t V,
                                            uint32_t* pair_out, hipStream_t stream) {
  if (n >= 0xFFFFFFFFull || !pair_out || V < 1 || V > 65536) return FC_ERR_INVALID;
  if (n > 0 && (!tokens || !sa)) return FC_ERR_INVALID;
  (void)hipGetLastError();
  if (n > 0) {
    // precondition: every token < V (pair_out[0] serves as the reduction cell)
    FC_CHECK_HIP(hipMemsetAsync(pair_out, 0, sizeof(uint32_t), stream));
    const uint32_t blocks = fc::div_up(n, 2048) < kMaxTokenBlocks ? fc::div_up(n, 2048) : kMaxTokenBlocks;
    hipLaunchKernelGGL(k_max_token, dim3(blocks), dim3(256), 0, stream, tokens, (uint32_t)n, pair_out);
    FC_CHECK_LAUNCH();
    uint32_t mx = 0;
    FC_CHECK_HIP(hipMemcpyAsync(&mx, pair_out, sizeof(uint32_t), hipMemcpyDeviceToHost, stream));
    FC_CHECK_HIP(hipStreamSynchronize(stream));
    if (mx >= V) return FC_ERR_INVALID;
  }
  if (n == 0) {  // every entry is 0
    FC_CHECK_HIP(hipMemsetAsync(pair_out, 0, sizeof(uint32_t) * fc_pair_table_entries(V), stream));
    return FC_OK;
  }
  const PairKeys pk{tokens, sa, (uint32_t)n, V};
  if (n < 2)
    hipLaunchKernelGGL(k_pairs_one, dim3(1024), dim3(256), 0, stream, pk, pair_out);
  else if (n < kPairSampleMin)
    hipLaunchKernelGGL(k_pairs, dim3(fc::div_up(n + 1, 256)), dim3(256), 0, stream, pk, pair_out);
  else
    hipLaunchKernelGGL(k_pairs_sampled, dim3(fc::div_up(n + 1, 4 * kPairSpan)), dim3(256), 0, stream, pk, pair_out);
  FC_CHECK_LAUNCH();
  return FC_OK;
}

extern "C" uint64_t fc_record_bytes(uint64_t n) { return (uint64_t)FC_RECORD_BYTES * n; }

namespace {

// entry t of the top-level sample: the first two 16-byte quads of record
// t * FC_TOP_STRIDE
__global__ void __launch_bounds__(256) k_top(const uint4* __restrict__ rec, uint64_t n_top,
                                               uint4* __restrict__ top) {
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;  // one quad per thread
  if (i >= 2 * n_top) return;
  const uint64_t t = i >> 1, q = i & 1;
  top[i] = rec[(t * FC_TOP_STRIDE) * (FC_RECORD_BYTES / 16) + q];
}

}  // namespace

extern "C" uint64_t fc_store_top_bytes(uint64_t n) {
  return ((n + FC_TOP_STRIDE - 1) / FC_TOP_STRIDE) * (uint64_t)FC_TOP_BYTES;
}

extern "C" fc_status fc_store_prepare_top(const void* rec, uint64_t n, void* top_out, hipStream_t stream) {
  if (n >= 0xFFFFFFFFull) return FC_ERR_INVALID;
  if (n == 0) return FC_OK;
  if (!rec || !top_out || ((uintptr_t)rec & (FC_RECORD_BYTES - 1)) || ((uintptr_t)top_out & (FC_TOP_BYTES - 1)))
    return FC_ERR_INVALID;
  const uint64_t n_top = (n + FC_TOP_STRIDE - 1) / FC_TOP_STRIDE;
  (void)hipGetLastError();
  hipLaunchKernelGGL(k_top, dim3(fc::div_up(2 * n_top, 256)), dim3(256), 0, stream, (const uint4*)rec, n_top,
                     (uint4*)top_out);
  FC_CHECK_LAUNCH();
  return FC_OK;
}

extern "C" fc_status fc_store_prepare_records(const uint16_t* tokens, const uint32_t* sa, uint64_t n, void* rec_out,
                                              hipStream_t stream) {
  if (n >= 0xFFFFFFFFull) return FC_ERR_INVALID;
  if (n == 0) return FC_OK;
  if (!tokens || !sa || !rec_out || ((uintptr_t)rec_out & (FC_RECORD_BYTES - 1))) return FC_ERR_INVALID;
  (void)hipGetLastError();
  hipLaunchKernelGGL(k_records, dim3(fc::div_up(n, kRecBlock)), dim3(256), 0, stream, tokens, sa, (uint32_t)n,
                     (uint4*)rec_out);
  FC_CHECK_LAUNCH();
  return FC_OK;
}
