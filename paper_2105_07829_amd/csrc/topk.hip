// Top-k compressor (Section 3.2: of a gradient only its k entries of largest magnitude travel)
// with the residual update of Algorithm 4 in its fused form (Section 4.2, operator fusion: the
// residual is the vector itself with the k sent slots set to zero).
//
// Selection is exact: a three-level radix select on the 31-bit magnitude key
// bits(v) & 0x7fffffff (11 + 10 + 10 bits); elements equal to the threshold key are admitted
// lowest index first, and the record lists its entries by ascending index.
//
// Short-list form (k of a full partition at most half of kTopkListCap, partitions of up to 8 M elements):
// one pass over the data.
//   guess      : up to 8192 elements of each partition (1024 spread chunks of eight); the key G at a rank of
//                the sample chosen so that, but for rare cases, at least k and no more than a few k
//                elements of the partition have keys >= G
//   load       : v_j from the source -> dense buffer; the elements with key >= G go to the
//                partition's short list
//   select     : several workgroups per partition find the k-th largest key among the listed ones,
//                each for itself, and write a share of the record; kept slots of the buffer zeroed
// The guess is made by the first workgroups of the load kernel itself, the others have requested their
// elements before they wait for it (none of them for a workgroup that may not be running: TopkShared); on
// the server side a kernel in front sums the sampled chunks up and finds where each message's entries of a
// group of 8192 elements begin.
// The sample only decides how much work the selection is, never its result: a partition whose
// short list came out shorter than k or longer than its room (the sample misled) is taken by the long form
// below instead, run by the partition's first select workgroup alone; partitions of more than kAloneElems
// elements by one more kernel, enqueued behind, which returns at once if no partition needs it and else runs
// the long form's passes for those partitions with its resident grid meeting between the passes.
// A key that a great many elements share (zeros, magnitudes of few values) is left off the list, which starts
// above it; if the list then holds fewer than k, it is kept whole, and ties of that key make up for the rest,
// lowest index first: the load pass has counted them per group of 8192 elements, so every select workgroup knows how
// far they are kept and reads its part of the vector again as far as that.
//
// Group-list form (larger k, up to kMostListed of a full partition, or lists that would be too long, in partitions
// of up to kAloneElems elements, where the dense workspace is free): the same guess and load pass, but every
// group of 8192 elements has a list of its own in the dense workspace.
//   bins       : histogram of the listed keys' distances from the guess, 32 steps for every power of two
//   collect    : the bin of the k-th largest key from it; per group, how many entries lie above the bin;
//                the few entries inside it to one list a partition, and whether they are all of one key
//   emit       : threshold key and ties from that list (every workgroup for itself), then (idx, val) as
//                in the select pass
//
// Long form (the rest), five passes over the dense buffer:
//   load+hist1 : as above, every element counted
//   hist2      : bin of level 1 that holds the k-th largest key, histogram inside it
//   hist3      : the same one level down
//   count      : threshold key T and the number r of elements with key == T that are kept;
//                per tile, how many keys are > T and == T
//   emit       : (idx, val) in ascending index order; kept slots of the buffer zeroed
// Each pass works out the selection so far from the histograms of the passes before it (every
// workgroup for itself), so no launches sit between the passes.
//
// Server side the vector is Delta = (sum of the n decoded messages) / n + e~.  It is never
// scattered into a dense buffer (n k read-modify-writes at random places of HBM per partition):
// the messages list their entries by ascending index, so the load pass sums the stretch of each
// message that falls into its group of 8192 elements in LDS.
#include "cluster.hpp"
#include "sources.hpp"
#include "tile_rows.hpp"

// Whether the workgroups that are there for it make the guesses; a test compiles the pass without, as if they
// were kept from running (test_gpu_late_guess.py).
#ifndef BPC_TOPK_FIRST_GUESS
#define BPC_TOPK_FIRST_GUESS 1
#endif

namespace bpc {

constexpr int kBins1 = 2048, kBins23 = 1024;
constexpr int kHist1 = 0, kHist2 = kBins1, kHist3 = kHist2 + kBins23;
static_assert(kHist3 + kBins23 == kTopkHistWords, "histogram words of a partition");
constexpr int kShift1 = 20, kShift2 = 10;
constexpr int kBits1 = 11, kBits23 = 10;
// A workgroup of the histogram / count passes handles a few consecutive tiles of one partition
// (template parameter TPG): its LDS histogram is merged into the partition's with one atomic
// per non-empty bin, so more tiles a workgroup mean fewer of those (an atomic on global memory
// costs some 11 ns of one memory channel's time; they were the larger part of the level-2
// pass), while fewer, longer workgroups hide less latency (8 tiles a workgroup doubled the
// time of the passes that only read).
constexpr int kTpgLoad = 2, kTpgHist2 = 4, kTpgHist3 = 1, kTpgCount = 1;
constexpr int kSelThreads = 1024;                       // workgroup of the select pass
constexpr int kSelPer = kTopkListCap / kSelThreads;     // list entries a thread of it keeps
constexpr int kSelBins = 8192, kSelBits = 13;           // first level of the select pass: bins of 1024 keys from the guess up, an octave of magnitudes
constexpr uint32_t kShareWords = 16384;                 // words of the bitmap of a select workgroup's share of the indices, at most
constexpr uint32_t kXcds = 8, kCusOfXcd = 32;            // of an MI355X: the select pass is spread over one workgroup a compute unit when there are few partitions
constexpr uint32_t kMostShares = 8;                     // ... of one partition (unless its bitmaps ask for more)
constexpr uint32_t kAloneElems = 1u << 21;              // partitions up to this size are left to one workgroup if the short list fails
constexpr uint32_t kMostOfList = 1u << 23;              // elements of a partition in the short-list form, at most
constexpr uint32_t kMostListed = 65536;                 // k of a full partition up to which the group-list form is taken
constexpr uint32_t kGatedGrid = 1024;                   // grid of the long-form kernel behind the short-list form, at most
constexpr uint32_t kFewInBin = kTopkListCap / 16;       // elements of a bin that the list can take unasked
// Elements of one key stay off the list from so many on (the select pass's counts of them meet in one place: 0.3 M
// elements of 16 magnitudes 80 us a call, 30 beside the list) if they are one in so many at least (the vector
// is searched for them: 4 M elements of 256 magnitudes 74 us on the list, 130 beside it).
constexpr uint32_t kTiesOffList = kTopkListCap / 8, kTiesDensity = 64;
constexpr uint32_t kFewNear = 512;                      // entries of one key in the threshold's bin that every workgroup ranks for itself
constexpr uint32_t kNearBins = 1024;                    // group-list form: bins of the listed keys by their distance from the guess,
constexpr uint32_t kBinWords = kNearBins + 3;           // the number of entries in the threshold's bin, and their highest and lowest keys
constexpr uint32_t kNoGuess = 0xffffffffu;              // no key reaches it: nothing goes to the short list

__device__ inline uint32_t key_of(float v) { return __float_as_uint(v) & 0x7fffffffu; }

// state words per partition: words 2L, 2L + 1 hold (prefix, rank left) after level L = 1..3;
// word 1 is kLongForm if the partition is left to the long form, kTiesBeside if elements beside its list are kept
enum { kStPrefix = 0, kStKRem = 1 };
enum { kStLong = 1 };
enum : uint32_t { kLongForm = 1, kTiesBeside = 2 };

// What the load pass of the short-list form hands from workgroup to workgroup, in the workspace's
// region for it (16 KB a partition): the guesses, four words each (the guess and whether there are ties beside
// the list, its exclusive or with the launch's tag, as the slots of cluster.hpp, and the tag once a workgroup
// has taken the guess on), and the lengths of the lists, a page apart since an atomic on global memory holds
// up its memory channel for some 11 ns.
//
// The first workgroups of the launch make the guesses, and the others wait for them.  Its grid is not resident
// as a whole, and workgroups are bound to an XCD by their index: beside another kernel that waits (a second
// top-k call, a single-pass kernel, on another stream), waiting workgroups of either could fill the XCD that a
// guess's workgroup is bound to, and hold each other up.  So nobody waits long for a workgroup that may not
// have started: after kPatience looks (some 2 ms) a waiting workgroup takes the guess on itself and publishes that
// there is none, which leaves the partition to the long form.  If one that is running has taken it on before,
// it waits for that one, which waits for nobody.  The guess of a workgroup that comes too late is dropped.
// (A second copy of the guess there instead took a worker's kernel from 40 to 64 registers and its call on 0.3 M
// elements from 21.2 to 22.4 us.)
constexpr int kPatience = 1024;
struct TopkShared {
  uint64_t *pairs;
  uint32_t *lengths;
  uint64_t tag;
  uint32_t *status;
  uint32_t *state;
  bool limited;   // the lists' room is (that of the group lists is not)
  static size_t pairs_bytes(uint32_t P) { return (32ull * P + 4095) / 4096 * 4096; }
  __device__ uint32_t *length(uint32_t p) const { return lengths + 1024ull * p; }
  __device__ uint64_t *pair(uint32_t p) const { return pairs + 4ull * p; }
  // One thread takes the guess on; the tag if another one has.
  __device__ uint64_t take(uint32_t p) const {
    return __hip_atomic_exchange(pair(p) + 2, tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  // One thread publishes partition p's guess; the list length is zero before anyone can see it.
  __device__ void publish(uint32_t p, uint32_t guess, bool ties) const {
    const uint64_t word = (uint64_t)(ties ? 1 : 0) << 32 | guess;
    __hip_atomic_store(length(p), 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    state[p * 8 + kStLong] = 0;
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x0F70);   // (vector memory done)
    asm volatile("" ::: "memory");
    __hip_atomic_store(pair(p), word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(pair(p) + 1, word ^ tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __device__ u32x4 look(uint32_t p) const { return TileBuf(pair(p), 16).load16<kMemorySide>(0, 0); }
  // One wave waits for the guess, `w` being its first look at it, for `looks` more; false if it is not there.
  __device__ bool wait(uint32_t p, u32x4 w, int looks, uint32_t *guess, uint32_t *ties) const {
    while ((w.x ^ w.z) != (uint32_t)tag || (w.y ^ w.w) != (uint32_t)(tag >> 32)) {
      if (--looks < 0) return false;
      __builtin_amdgcn_s_sleep(4);
      w = look(p);
    }
    *guess = w.x;
    *ties = w.y;
    return true;
  }
};

// A partition's short list: the entries' indices and values, in any order.  In the group-list form: a list
// for every group of the load pass, with room for half of its elements in the place of the group in the
// dense workspace; that of a ragged last group, and the entries near the threshold, where the short list
// would be.
struct TopkLists {
  uint32_t *base;
  uint32_t P;
  uint32_t *dense;      // null: one list a partition
  uint32_t *counts;     // two words a group: entries of its list (group lists); ties beside the list, or (group
                        // lists that hold k entries) entries above the bin of the threshold and, in the upper half, inside it
  uint32_t groups;      // of a full partition
  static constexpr uint32_t kNearCap = kTopkListCap - 8192;
  __device__ uint32_t *idx(uint32_t p) const { return base + (uint64_t)p * kTopkListCap; }
  __device__ uint32_t *val(uint32_t p) const { return base + (uint64_t)(P + p) * kTopkListCap; }
  struct List { uint32_t *idx, *val, room; };
  __device__ List of_group(const Geo &g, uint32_t p, uint32_t q, uint32_t d) const {
    if (d - q * 8192u < 8192u) return List{idx(p) + kNearCap, val(p) + kNearCap, 8192u};
    uint32_t *at = dense + g.part_base(p) + q * 8192u;
    return List{at, at + 4096, 4096u};
  }
  __device__ uint32_t *count(uint32_t p, uint32_t q) const { return counts + 2ull * ((uint64_t)p * groups + q); }
};

// Whether partition p is left to the long form (uniform over the workgroup).
__device__ inline bool long_form(const uint32_t *state, uint32_t p) {
  return __builtin_amdgcn_readfirstlane(state[p * 8 + kStLong]) == kLongForm;
}

// Group `blk` of TPG consecutive tiles of one partition.
struct GroupOf {
  uint32_t p, tile_lo, tile_hi, d;
};
template <int TPG>
__device__ inline GroupOf group_of(const Geo &g, uint32_t blk) {
  constexpr uint32_t kTilesPerGroup = TPG;
  const uint32_t groups_per_part = (uint32_t)cdiv(g.tiles_per_part, kTilesPerGroup);
  GroupOf r;
  r.p = blk / groups_per_part;
  r.d = g.part_size(r.p);
  const uint32_t n_tiles = (uint32_t)cdiv(r.d, kTile);
  r.tile_lo = (blk % groups_per_part) * kTilesPerGroup;
  r.tile_hi = r.tile_lo + kTilesPerGroup < n_tiles ? r.tile_lo + kTilesPerGroup : n_tiles;
  return r;
}
inline uint32_t group_count(const Geo &g, int tpg) { return g.P * (uint32_t)cdiv(g.tiles_per_part, tpg); }

// All threads of a workgroup of THREADS: walk a histogram `h` of BINS bins (global or LDS)
// from the highest bin down and find the bin b with
//   count(bins above b) < k_rem <= count(bins above b) + count(b).
// sel[0] = (prefix << BITS) | b (the extended prefix), sel[1] = the rank left inside b.
// Every workgroup of the pass that follows a histogram pass does this for itself (a few
// microseconds of L2 reads) instead of a launch of its own in between.
template <int BINS, int BITS, int THREADS>
__device__ inline void pick_bin(const uint32_t *h, uint32_t k_rem, uint32_t prefix, uint32_t *scan, uint32_t *sel) {
  constexpr int kPer = BINS / THREADS > 0 ? BINS / THREADS : 1;
  // thread t owns bins BINS-1 - t*kPer - i, highest first; threads past the bins own none
  uint32_t cnt[kPer];
  uint32_t local = 0;
  if constexpr (kPer % 4 == 0) {   // (the histograms start at multiples of 16 bytes)
#pragma unroll
    for (int i = 0; i < kPer; i += 4) {
      const uint4 x = *reinterpret_cast<const uint4 *>(h + (BINS - 4 - (int)threadIdx.x * kPer - i));
      cnt[i] = x.w; cnt[i + 1] = x.z; cnt[i + 2] = x.y; cnt[i + 3] = x.x;
    }
  } else {
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const uint32_t b = threadIdx.x * kPer + i;
      cnt[i] = b < (uint32_t)BINS ? h[BINS - 1 - b] : 0u;
    }
  }
#pragma unroll
  for (int i = 0; i < kPer; ++i) local += cnt[i];
  uint32_t total;
  const uint32_t above = block_exclusive_scan<THREADS>(local, scan, &total);
  if (above < k_rem && k_rem <= above + local) {
    uint32_t run = above;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      if (run < k_rem && k_rem <= run + cnt[i]) {
        sel[0] = (prefix << BITS) | (BINS - 1 - (threadIdx.x * kPer + i));
        sel[1] = k_rem - run;
      }
      run += cnt[i];
    }
  }
  __syncthreads();
}

// Radix select, inside one workgroup of THREADS, among the keys of the values the threads hold
// in registers (the low 31 bits of bits[i], i < cnt <= rounds, `rounds` the same for all
// threads).  h: LDS, kBins1 words.
// Level 2, given level 1's (b1, k_rem1): the key's first 21 bits in sel[0], the rank left among the
// keys that share them in sel[1].
template <int PER, int THREADS>
__device__ inline void level2_in_registers(const uint32_t (&bits)[PER], uint32_t cnt, uint32_t rounds, uint32_t b1,
                                             uint32_t k_rem1, uint32_t *h, uint32_t *scan, uint32_t *sel) {
  for (int b = threadIdx.x; b < kBins23; b += THREADS) h[b] = 0;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    if ((uint32_t)i >= rounds) break;
    const uint32_t key = bits[i] & 0x7fffffffu;
    if ((uint32_t)i < cnt && (key >> kShift1) == b1) atomicAdd(&h[(key >> kShift2) & (kBins23 - 1)], 1u);
  }
  __syncthreads();
  pick_bin<kBins23, kBits23, THREADS>(h, k_rem1, b1, scan, sel);
}
// Level 3, given level 2's (prefix2, k_rem2): the key in sel[0], the rank left among the keys equal to it
// in sel[1].
template <int PER, int THREADS>
__device__ inline void level3_in_registers(const uint32_t (&bits)[PER], uint32_t cnt, uint32_t rounds, uint32_t prefix2,
                                           uint32_t k_rem2, uint32_t *h, uint32_t *scan, uint32_t *sel) {
  __syncthreads();
  for (int b = threadIdx.x; b < kBins23; b += THREADS) h[b] = 0;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    if ((uint32_t)i >= rounds) break;
    const uint32_t key = bits[i] & 0x7fffffffu;
    if ((uint32_t)i < cnt && (key >> kShift2) == prefix2) atomicAdd(&h[key & (kBins23 - 1)], 1u);
  }
  __syncthreads();
  pick_bin<kBins23, kBits23, THREADS>(h, k_rem2, prefix2, scan, sel);
}

// The sample of a partition of d elements: chunk (of eight consecutive elements) number c is one of the c-th
// stretch of 1 << shift chunks, at a place that moves from stretch to stretch (chunks at equal
// distances of a power of two would all come from the same few memory channels).  Only whole chunks.
struct SamplePlan {
  uint32_t shift, chunks;
  __device__ explicit SamplePlan(uint32_t d) : shift(sample_shift(d)), chunks(sample_chunks(d)) {}
  __device__ uint32_t chunk(uint32_t c) const { return (c << shift) + ((c * 37u) & ((1u << shift) - 1u)); }
};

// Workgroup of the load pass: 16 elements a thread (of 256 threads, 32 elements each: 91 registers
// a lane and five waves a SIMD where this has 44 and eight): steps of 3 workers on 0.3 M elements 146 ->
// 135 us, of 8 workers on 25.6 M elements 911 -> 892 us, of 16 workers on 110 M f16 elements 4275 ->
// 4202 us.  (1024 threads: 131, 908 and 4402 us.)
constexpr int kLoadThreads = 512;
constexpr uint32_t kGroupElems = kTpgLoad * kTile;   // elements a workgroup of the load pass takes: 8192
static_assert(kGroupElems == 8192, "the workspace is laid out for groups of 8192 elements");

// Server side: Delta = (sum of the n decoded top-k messages) / n + e~ straight from the
// messages.  A message lists its entries by ascending index, so the entries of a group of
// 8192 elements are one stretch of it; `topk_starts_kernel` records where each stretch begins.
struct TopkMsgs {
  WorkerMsgs msgs;
  const float *res;
  const uint32_t *starts;   // [worker][partition][group .. groups_per_part]
  uint32_t groups_per_part, k_cap;
  uint64_t stride;
  int half;
  uint32_t group_shift;     // log2 of the elements of a group (13 for the load pass)
  __device__ const uint8_t *rec(int i, uint32_t p) const { return msgs.ptr[i] + (uint64_t)p * stride; }
  __device__ uint32_t k_of(int i, uint32_t p) const {
    const uint32_t k = *reinterpret_cast<const uint32_t *>(rec(i, p));
    return k > k_cap ? k_cap : k;
  }
  __device__ const uint32_t *idx(int i, uint32_t p) const { return reinterpret_cast<const uint32_t *>(rec(i, p) + kHeaderBytes); }
  __device__ float value(int i, uint32_t p, uint32_t t) const {
    const uint8_t *v = rec(i, p) + kHeaderBytes + 4 * ru4(k_cap);
    return half ? __half2float(reinterpret_cast<const __half *>(v)[t]) : reinterpret_cast<const float *>(v)[t];
  }
  // The residual's eight elements from j0 (zeros without a residual or past the end), and
  // Delta from them and the sums of the decoded messages.
  __device__ void load_res8(const Geo &g, uint32_t p, uint32_t j0, uint32_t d, float r[8]) const {
    const uint64_t i0 = g.part_base(p) + j0;
#pragma unroll
    for (int e = 0; e < 8; ++e) r[e] = 0.0f;
    if (res) {
      if (j0 + 8 <= d) load8_aligned(res + i0, r);
      else
        for (int e = 0; e < 8; ++e) r[e] = j0 + e < d ? res[i0 + e] : 0.0f;
    }
  }
  __device__ void combine8(uint32_t j0, uint32_t d, const float *sum, const float r[8], float out[8]) const {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float mean = sum[e] * msgs.inv_n;
      out[e] = j0 + e < d ? (res ? mean + r[e] : mean) : 0.0f;
    }
  }
};

// For t = 0 .. k: entry t is the first one of every group after the group of entry t - 1 up to
// its own group (t = k: up to the end).  A message that is not in ascending order leaves
// groups unset; readers clamp what they find to [0, k].  Entries t0, t0 + step, ... below `end` of worker i's
// message.
__device__ inline void topk_starts(const Geo &g, const TopkMsgs &m, uint32_t *starts, uint32_t i, uint32_t p, uint32_t t0, uint32_t step,
                                   uint32_t end = 0xffffffffu) {
  const uint32_t k = m.k_of(i, p);
  const uint32_t *idx = m.idx(i, p);
  uint32_t *tab = starts + ((uint64_t)i * g.P + p) * (m.groups_per_part + 1);
  auto group = [&](uint32_t j) { const uint32_t q = j >> m.group_shift; return q < m.groups_per_part ? q : m.groups_per_part - 1; };
  constexpr uint32_t kAhead = 4;   // entries requested before the first is looked at
  for (uint32_t t = t0; t <= k && t < end; t += kAhead * step) {
    uint32_t before[kAhead], here[kAhead];
#pragma unroll
    for (uint32_t r = 0; r < kAhead; ++r) {
      const uint32_t e = t + r * step;
      before[r] = e > 0 && e <= k && e < end ? idx[e - 1] : 0u;
      here[r] = e < k && e < end ? idx[e] : 0u;
    }
#pragma unroll
    for (uint32_t r = 0; r < kAhead; ++r) {
      const uint32_t e = t + r * step;
      if (e > k || e >= end) break;
      const uint32_t first = e == 0 ? 0u : group(before[r]) + 1;
      const uint32_t last = e == k ? m.groups_per_part : group(here[r]);
      for (uint32_t q = first; q <= last && q <= m.groups_per_part; ++q) tab[q] = e;
    }
  }
}
__global__ __launch_bounds__(kThreads) void topk_starts_kernel(Geo g, TopkMsgs m, uint32_t *starts) {
  topk_starts(g, m, starts, blockIdx.z, blockIdx.y, blockIdx.x * kThreads + threadIdx.x, gridDim.x * kThreads);
}

// The load pass's view: the workgroup's group of 8192 elements summed in LDS, worker by worker
// (a barrier in between: the order of the sum is the workers'), a thread's first entry of the
// next worker requested before the adds of this one.
struct TopkMsgsGroupSource : TopkMsgs {
  const float *sums;   // of the sampled chunks, kTopkListCap words from partition to partition
  __device__ void sampled8(const Geo &g, uint32_t p, uint32_t c, uint32_t j0, uint32_t d, float out[8]) const {
    float sum[8], r[8];
    load_res8(g, p, j0, d, r);
    load8_aligned(sums + (uint64_t)p * kTopkListCap + 8 * c, sum);
    combine8(j0, d, sum, r, out);
  }
  static constexpr int kLdsFloats = kGroupElems + 5 * kMaxWorkers + 2;   // sums, ranges, counts before, record addresses
  __device__ void begin(const Geo &, uint32_t, float *) const {}
  __device__ void begin_group(const Geo &g, uint32_t p, uint32_t grp, float *lds) const {
    uint32_t *range = reinterpret_cast<uint32_t *>(lds + kGroupElems);
    // (the records' addresses go to LDS: a thread's entries belong to workers it finds at run
    // time, and indexing the kernel arguments by such a number is a memory access of its own)
    const uint8_t **recs = reinterpret_cast<const uint8_t **>(lds + kGroupElems + 3 * kMaxWorkers + 2);
    const uint32_t lo = grp * kGroupElems;
    if (threadIdx.x < (uint32_t)msgs.n) {
      recs[threadIdx.x] = rec(threadIdx.x, p);
      const uint32_t *tab = starts + ((uint64_t)threadIdx.x * g.P + p) * (groups_per_part + 1);
      const uint32_t k = k_of(threadIdx.x, p);
      const uint32_t s = tab[grp] < k ? tab[grp] : k, e = tab[grp + 1] < k ? tab[grp + 1] : k;
      range[2 * threadIdx.x] = s;
      range[2 * threadIdx.x + 1] = e < s ? s : e;
    }
    for (uint32_t q = threadIdx.x; q < kGroupElems / 4; q += kLoadThreads) reinterpret_cast<float4 *>(lds)[q] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    __syncthreads();
    // entries of the group before worker i's, over all workers
    uint32_t *cum = range + 2 * kMaxWorkers;
    if (threadIdx.x < 64) {
      const uint32_t c = threadIdx.x < (uint32_t)msgs.n ? range[2 * threadIdx.x + 1] - range[2 * threadIdx.x] : 0u;
      const uint32_t incl = wave_inclusive_scan_u32(c);
      cum[threadIdx.x + 1] = incl;
      if (threadIdx.x == 0) cum[0] = 0;
    }
    __syncthreads();
    const uint32_t total = cum[msgs.n];
    constexpr int kMine = 2;   // entries a thread takes
    if (total <= (uint32_t)(kMine * kLoadThreads)) {
      // all the group's entries are requested at once (worker-major, so a thread's entries come
      // in worker order), then added worker by worker with a barrier in between
      uint32_t rel[kMine], who[kMine];
      float val[kMine];
#pragma unroll
      for (int r = 0; r < kMine; ++r) {
        const uint32_t q = r * kLoadThreads + threadIdx.x;
        who[r] = 0xffffffffu;
        rel[r] = 0;
        val[r] = 0.0f;
        if (q < total) {
          uint32_t a = 0, b = msgs.n;   // cum[a] <= q < cum[b]
          while (b - a > 1) {
            const uint32_t mid = (a + b) >> 1;
            if (cum[mid] <= q) a = mid; else b = mid;
          }
          const uint32_t t = range[2 * a] + (q - cum[a]);
          const uint8_t *rc = recs[a];
          who[r] = a;
          rel[r] = reinterpret_cast<const uint32_t *>(rc + kHeaderBytes)[t] - lo;
          const uint8_t *vp = rc + kHeaderBytes + 4 * ru4(k_cap);
          val[r] = half ? __half2float(reinterpret_cast<const __half *>(vp)[t]) : reinterpret_cast<const float *>(vp)[t];
        }
      }
      for (int i = 0; i < msgs.n; ++i) {
        if (cum[i + 1] != cum[i]) {   // (uniform)
#pragma unroll
          for (int r = 0; r < kMine; ++r)
            if (who[r] == (uint32_t)i && rel[r] < kGroupElems) lds[rel[r]] = lds[rel[r]] + val[r];
          __syncthreads();
        }
      }
    } else {
      for (int i = 0; i < msgs.n; ++i) {
        const uint32_t s = range[2 * i], e = range[2 * i + 1];
        for (uint32_t q = s + threadIdx.x; q < e; q += kLoadThreads) {
          const uint32_t r = idx(i, p)[q] - lo;
          if (r < kGroupElems) lds[r] = lds[r] + value(i, p, q);
        }
        __syncthreads();
      }
    }
  }
};

// The guess for partition p, published unless another workgroup has taken it on (`taken`, what TopkShared::take
// gave thread 0): `load8(j0, v)` gives the eight elements from j0, the first of
// a sampled chunk.  All threads of a workgroup of THREADS; h: LDS, kBins1 words.  Random 64-byte reads
// cost about as much as 16 times as many sequential ones, hence chunks rather than single elements.
template <int THREADS, class LOAD8>
__device__ inline void topk_guess(const Geo &g, uint32_t p, const TopkShared &sh, uint64_t taken, uint32_t *h, uint32_t *scan,
                                  uint32_t *sel, LOAD8 load8) {
  auto publish = [&](uint32_t guess, bool ties) {
    if (threadIdx.x == 0 && taken != sh.tag) sh.publish(p, guess, ties);
  };
  constexpr uint32_t kChunksPer = (kSampleChunks + THREADS - 1) / THREADS;
  constexpr int kPer = 8 * kChunksPer;
  const uint32_t d = g.part_size(p);
  const SamplePlan plan(d);
  const uint32_t m = 8 * plan.chunks;                         // elements in the sample
  const uint32_t rank = m ? sample_rank(k_of_device(g, p), m, d, sh.limited) : 0;
  if (rank >= m) {   // (uniform) the whole partition is listed
    publish(0, false);
    return;
  }
  uint32_t key[kPer];
  uint32_t cnt = 0;
  // (every load is issued, with chunk 0 standing in past the end, so that none is waited for
  // before the last is on its way)
#pragma unroll
  for (uint32_t i = 0; i < kChunksPer; ++i) {
    const uint32_t c = i * THREADS + threadIdx.x;
    float v[8];
    load8(c < plan.chunks ? c : 0u, 8 * plan.chunk(c < plan.chunks ? c : 0u), v);
#pragma unroll
    for (int e = 0; e < 8; ++e) key[8 * i + e] = key_of(v[e]);
    cnt += c < plan.chunks ? 8 : 0;
  }
  for (int b = threadIdx.x; b < kBins1; b += THREADS) h[b] = 0;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kPer; ++i)
    if ((uint32_t)i < cnt) atomicAdd(&h[key[i] >> kShift1], 1u);
  __syncthreads();
  pick_bin<kBins1, kBits1, THREADS>(h, rank, 0, scan, sel);
  const uint32_t b1 = sel[0], k_rem1 = sel[1];
  __syncthreads();
  // The lower end of the level-2 bin (1/8192 of an octave of magnitudes) will do for a guess as long as
  // the bin holds few elements, which the list then takes too.  Magnitudes that lie that close
  // together would overrun the list and leave the partition to the long form (within 2^-14 of each
  // other, 1 M elements: 59 us for the call with the third level, 690 us without).
  level2_in_registers<kPer, THREADS>(key, cnt, kPer, b1, k_rem1, h, scan, sel);
  const uint32_t prefix2 = sel[0], k_rem2 = sel[1];
  const uint64_t in_bin = (uint64_t)h[prefix2 & (kBins23 - 1)] * d;   // times m: elements of the partition
  if (in_bin <= (uint64_t)kFewInBin * m) {   // (uniform)
    publish(prefix2 << kShift2, false);
    return;
  }
  level3_in_registers<kPer, THREADS>(key, cnt, kPer, prefix2, k_rem2, h, scan, sel);
  // One key that so many elements share that they would overrun the list (zeros, gradients of few magnitudes) stays
  // off it: the list starts above, and where it then holds fewer than k, ties of that key are kept beside it.
  // (Left to one workgroup or the resident kernel instead, calls on such data took up to thirty times as long as
  // ordinary ones: partitions of 2 M f16 elements of 16 magnitudes, 16 M in all, k = 0.1 % / 1 %, 1117 -> 58 and
  // 1205 -> 72 us; 0.3 M zeros, k = 1 % / 6 %, 140 -> 35 and 245 -> 55.)
  const uint64_t equal = h[sel[0] & (kBins23 - 1)], listed = rank - sel[1] + equal;   // of the sample
  const bool ties = d > kTopkListCap &&   // (smaller partitions fit the list whole)
                    ((equal * d > kTiesOffList * (uint64_t)m && equal * kTiesDensity > m) ||
                     (sh.limited && listed * d > 3ull * kTopkListCap / 4 * m));
  publish(sel[0] + (ties ? 1u : 0u), ties);
}

// Server side, in front of the load pass.  The first rows of workgroups of a partition find the sums of the
// decoded messages in the sampled chunks, a thread searching one message for one chunk (on
// one compute unit, by a sweep over the messages or by searches, they took 25 to 150 us); the others
// where each group's entries start.  (With workgroups of 1024 threads for 16 messages whatever their number, and
// one for every message however short, calls of many partitions spent more time here than in the passes
// behind: 4 workers, 16 M elements, partitions of 8192 / 65536, 138 to 266 and 65 to 85 us a call; 129 and 56 so.)
static_assert(kSampleChunks * 8 <= kTopkListCap, "the sums lie where the lists will");
__global__ __launch_bounds__(kPrepMostThreads) void topk_server_prep_kernel(Geo g, TopkMsgs m, PrepRows rows, uint32_t *starts, float *sums) {
  extern __shared__ float part[];   // eight words a thread
  const uint32_t p = blockIdx.x, n = (uint32_t)m.msgs.n;
  if (blockIdx.y >= rows.sums) {
    for (uint32_t role = blockIdx.y - rows.sums; role < rows.roles; role += rows.starts) {
      if (rows.pieces > 1) {
        const uint32_t t0 = role % rows.pieces * 8 * rows.threads;
        topk_starts(g, m, starts, role / rows.pieces, p, t0 + threadIdx.x, rows.threads, t0 + 8 * rows.threads);
      } else {
        const uint32_t i0 = role * rows.messages, per = m.k_cap + 1;
        const uint32_t all = (n - i0 < rows.messages ? n - i0 : rows.messages) * per;
        for (uint32_t q = threadIdx.x; q < all; q += rows.threads) {
          const uint32_t t = q % per;
          topk_starts(g, m, starts, i0 + q / per, p, t, 1, t + 1);
        }
      }
    }
    return;
  }
  const SamplePlan plan(g.part_size(p));
  const uint32_t slot = threadIdx.x >> rows.chunk_bits, c = blockIdx.y * rows.chunks + (threadIdx.x & (rows.chunks - 1));
  if (blockIdx.y * rows.chunks >= plan.chunks) return;   // (uniform)
  float *acc = part + threadIdx.x * 8;   // [slot][chunk][element]
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = 0.0f;
  const uint32_t j0 = 8 * plan.chunk(c < plan.chunks ? c : 0u);
  for (uint32_t i = slot; i < n; i += rows.slots) {
    const uint32_t *idx = m.idx(i, p);
    const uint32_t k = m.k_of(i, p);
    uint32_t lo = 0, len = k;   // the first entry at or past j0 is one of [lo, lo + len]
    while (len > 0) {
      const uint32_t half = len >> 1;
      const bool below = idx[lo + half] < j0;
      lo += below ? half + 1 : 0u;
      len = below ? len - half - 1 : half;
    }
    for (; lo < k; ++lo) {
      const uint32_t j = idx[lo] - j0;
      if (j >= 8) break;
      acc[j] += m.value(i, p, lo);
    }
  }
  __syncthreads();
  const uint32_t words = rows.chunks * 8;
  for (uint32_t w = threadIdx.x; w < words; w += rows.threads) {
    float s = 0.0f;
#pragma unroll
    for (uint32_t q = 0; q < kPrepSlots; ++q) s += q < rows.slots ? part[(q < rows.slots ? q : 0u) * words + w] : 0.0f;
    sums[(uint64_t)p * kTopkListCap + blockIdx.y * words + w] = s;
  }
}

template <class SRC, class = void>
struct has_begin_group : std::false_type {};
template <class SRC>
struct has_begin_group<SRC, std::void_t<decltype(&SRC::begin_group)>> : std::true_type {};

// Load pass.  Besides the buffer, short-list form (LISTED): the elements of the workgroup's tiles whose
// key is at least the partition's guess go to its short list, together, at the place one atomic
// add on the list length hands out.  The order inside the list does not matter: the select pass puts
// what it keeps in index order through a bitmap.  Long form: the level-1 histogram of all elements.
// In the short-list form workgroup p < P makes partition p's guess and the groups follow behind; a group has
// its elements in registers before one of its waves waits for the guess (a kernel of its own for the guesses
// cost 8 us of every call).
// The group is taken as 4 rows of 2048 elements, 4 consecutive elements a thread and row: every
// 16-byte access of a wave to the gradient, the residual and the buffer covers whole cache lines
// and is marked non-temporal; everything goes through descriptors of the elements that exist
// (the rest read as zero and are not written).  All loads of the group are requested before the
// first is used.
constexpr int kLoadRowElems = kLoadThreads * 4;
constexpr int kLoadRows = kGroupElems / kLoadRowElems;
// `buf` is null where the gradient itself will do (no error feedback, short-list form): nothing is stored
// (f32 gradients, 20 M elements, k = 1 %: 65 -> 38 us).
template <class SRC, bool LISTED>
__global__ __launch_bounds__(kLoadThreads) void topk_load_kernel(Geo g, SRC src, float *buf, uint32_t *hist, uint32_t *state, TopkShared sh,
                                                                 TopkLists lists) {
  constexpr bool kServer = has_begin_group<SRC>::value;
  __shared__ __align__(16) float lds[SRC::kLdsFloats];
  constexpr int kWaves = kLoadThreads / 64;
  __shared__ uint32_t own_h[kServer && LISTED ? 1 : kBins1];
  uint32_t *h = kServer && LISTED ? reinterpret_cast<uint32_t *>(lds) : own_h;
  __shared__ uint32_t scan[kWaves];
  __shared__ uint32_t sel[2];
  const bool first = LISTED && blockIdx.x < g.P;   // is here for the guess of a partition
  GroupOf w;
  if (first) {
    w = GroupOf{blockIdx.x, 0, 0, g.part_size(blockIdx.x)};
    if (blockIdx.x == 0) status_open(sh.status, sh.tag);
    if (lists.dense)   // (the bins of the group-list form, used by later kernels)
      for (uint32_t b = threadIdx.x; b < kBinWords; b += kLoadThreads) hist[(uint64_t)w.p * kTopkHistWords + b] = 0;
    if (BPC_TOPK_FIRST_GUESS)
      topk_guess<kLoadThreads>(g, w.p, sh, threadIdx.x == 0 ? sh.take(w.p) : 0, h, scan, sel, [&](uint32_t c, uint32_t j0, float x[8]) {
        if constexpr (kServer) src.sampled8(g, w.p, c, j0, w.d, x);
        else src.at8(g, w.p, j0, w.d, nullptr, x);
      });
    return;
  } else {
    w = group_of<kTpgLoad>(g, blockIdx.x - (LISTED ? g.P : 0u));
    if (w.tile_lo >= w.tile_hi) return;  // (uniform) past the end of a shorter last partition
  }
  if constexpr (!LISTED) {
    for (int b = threadIdx.x; b < kBins1; b += kLoadThreads) h[b] = 0;
    __syncthreads();
  }
  const uint32_t wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const uint32_t j_lo = __builtin_amdgcn_readfirstlane(w.tile_lo * kTile);
  const uint32_t left = w.d - j_lo;
  const uint32_t valid = __builtin_amdgcn_readfirstlane(left < kGroupElems ? left : kGroupElems);
  const uint64_t base = uniform_off(g.part_base(w.p) + j_lo);
  const bool ef = src.res != nullptr;
  const TileBuf eb(ef ? src.res + base : nullptr, ef ? valid * 4 : 0);
  float v[kLoadRows][4];
  auto fetch = [&] {
    if constexpr (kServer) {
      // the residual's elements are requested first, so they are on their way while the group's
      // sum is formed
      u32x4 er[kLoadRows];
#pragma unroll
      for (int u = 0; u < kLoadRows; ++u) er[u] = eb.load16<kNonTemporal>(threadIdx.x * 16, u * kLoadRowElems * 4);
      src.begin_group(g, w.p, w.tile_lo / kTpgLoad, lds);
#pragma unroll
      for (int u = 0; u < kLoadRows; ++u) {
        const float4 sum = reinterpret_cast<const float4 *>(lds)[u * kLoadThreads + threadIdx.x];
        const float sv[4] = {sum.x, sum.y, sum.z, sum.w};
        float e[4];
        widen4(er[u], e);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const float mean = sv[c] * src.msgs.inv_n;
          const float delta = ef ? mean + e[c] : mean;
          v[u][c] = (uint32_t)(u * kLoadRowElems + c) + threadIdx.x * 4 < valid ? delta : 0.0f;
        }
      }
    } else {
      using T = typename SRC::Elem;
      const TileBuf gb(src.grad + base, valid * (uint32_t)sizeof(T));
      typename Vec4Of<T>::type gr[kLoadRows];
      u32x4 er[kLoadRows];
#pragma unroll
      for (int u = 0; u < kLoadRows; ++u) {
        gr[u] = tile_load4(gb, threadIdx.x * 4 * (uint32_t)sizeof(T), u * kLoadRowElems * (uint32_t)sizeof(T), (const T *)nullptr);
        er[u] = eb.load16<kNonTemporal>(threadIdx.x * 16, u * kLoadRowElems * 4);
      }
      if constexpr (sizeof(T) == 2) patch_last_half<kLoadRows, kLoadRowElems>(gb, valid, gr);
#pragma unroll
      for (int u = 0; u < kLoadRows; ++u) {
        float x[4], e[4];
        widen4(gr[u], x);
        widen4(er[u], e);
#pragma unroll
        for (int c = 0; c < 4; ++c) v[u][c] = ef ? x[c] + e[c] : x[c];
      }
    }
  };
  uint32_t G = kNoGuess;
  bool ties = false;
  if constexpr (!LISTED) {
    fetch();
  } else {
    // (the buffer is the residual, of which the guess's sample is read: no store before the guess is there)
    // (one wave looks for all: eight times fewer reads of one address)
    auto wait = [&](u32x4 look, int looks) {
      if (wave == 0) {
        uint32_t guess = kNoGuess, beside = 0;
        const bool there = sh.wait(w.p, look, looks, &guess, &beside);
        if (lane == 0) { sel[0] = guess; sel[1] = there ? 1u + beside : 0u; }
      }
      __syncthreads();
      G = __builtin_amdgcn_readfirstlane(sel[0]);
      const uint32_t there = __builtin_amdgcn_readfirstlane(sel[1]);
      ties = there > 1u;
      return there != 0;
    };
    u32x4 look{};
    if (wave == 0) look = sh.look(w.p);
    fetch();
    if (!wait(look, kPatience)) {   // (uniform)
      if (threadIdx.x == 0 && sh.take(w.p) != sh.tag) sh.publish(w.p, kNoGuess, false);
      __syncthreads();
      if (!wait(sh.look(w.p), kSpinLimit) && threadIdx.x == 0) status_give_up(sh.status, sh.tag);
    }
  }
  if (!LISTED || buf)
#pragma unroll
  for (int u = 0; u < kLoadRows; ++u)
    row_buf(buf + base, valid, u * kLoadRowElems, kLoadRowElems).store16<kNonTemporal>(as_u32x4(v[u][0], v[u][1], v[u][2], v[u][3]), threadIdx.x * 16);
  if constexpr (!LISTED) {
#pragma unroll
    for (int u = 0; u < kLoadRows; ++u)
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if ((uint32_t)(u * kLoadRowElems + c) + threadIdx.x * 4 < valid) atomicAdd(&h[key_of(v[u][c]) >> kShift1], 1u);
    __syncthreads();
    uint32_t *gh = hist + (uint64_t)w.p * kTopkHistWords + kHist1;
    for (int b = threadIdx.x; b < kBins1; b += kLoadThreads)
      if (h[b]) atomicAdd(&gh[b], h[b]);
  } else {
    uint32_t mask = 0;   // bit 4 u + c: element c of row u goes to the list
#pragma unroll
    for (int u = 0; u < kLoadRows; ++u)
#pragma unroll
      for (int c = 0; c < 4; ++c)
        mask |= (uint32_t)((uint32_t)(u * kLoadRowElems + c) + threadIdx.x * 4 < valid && key_of(v[u][c]) >= G) << (4 * u + c);
    uint32_t cnt = (uint32_t)__popc(mask);
    if (ties) {   // (uniform) ties beside the list are counted in the upper half
#pragma unroll
      for (int u = 0; u < kLoadRows; ++u)
#pragma unroll
        for (int c = 0; c < 4; ++c)
          cnt += (uint32_t)(u * kLoadRowElems + c) + threadIdx.x * 4 < valid && key_of(v[u][c]) == G - 1u ? 0x10000u : 0u;
    }
    const uint32_t incl = wave_inclusive_scan_u32(cnt);
    if (lane == 63) scan[wave] = incl;
    __syncthreads();
    uint32_t before = 0, total = 0;
#pragma unroll
    for (int q = 0; q < kWaves; ++q) {
      before += (uint32_t)q < wave ? scan[q] : 0u;
      total += scan[q];
    }
    if (ties && threadIdx.x == 0) lists.count(w.p, w.tile_lo / kTpgLoad)[1] = total >> 16;
    total &= 0xffffu;
    TopkLists::List list{lists.idx(w.p), lists.val(w.p), kTopkListCap};
    uint32_t pos = (before + incl - cnt) & 0xffffu;
    if (lists.dense) {
      list = lists.of_group(g, w.p, w.tile_lo / kTpgLoad, w.d);
      if (threadIdx.x == 0) *lists.count(w.p, w.tile_lo / kTpgLoad) = total;   // (more than its room: the vector itself will be read)
    } else {
      if (threadIdx.x == 0) sel[0] = total ? atomicAdd(sh.length(w.p), total) : 0u;
      __syncthreads();
      pos += sel[0];
    }
#pragma unroll
    for (int u = 0; u < kLoadRows; ++u)
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if ((mask >> (4 * u + c)) & 1u) {
          if (pos < list.room) {
            list.idx[pos] = j_lo + u * kLoadRowElems + threadIdx.x * 4 + c;
            list.val[pos] = __float_as_uint(v[u][c]);
          }
          ++pos;
        }
  }
}

// The selection state of partition p after `LEVEL` levels in sel[0] (prefix / threshold key)
// and sel[1] (rank left among the keys that match it): level 1 from k, each further level
// from the state the pass before recorded.  The first workgroup of the partition records the
// new state for the next pass.
template <int LEVEL>
__device__ inline void selection_after(const Geo &g, const uint32_t *hist, uint32_t *state, uint32_t p, bool first,
                                       uint32_t *scan, uint32_t *sel) {
  const uint32_t *gh = hist + (uint64_t)p * kTopkHistWords;
  if (LEVEL == 1) pick_bin<kBins1, kBits1, kThreads>(gh + kHist1, (uint32_t)k_of_device(g, p), 0, scan, sel);
  else pick_bin<kBins23, kBits23, kThreads>(gh + (LEVEL == 2 ? kHist2 : kHist3), state[p * 8 + 2 * (LEVEL - 1) + kStKRem],
                                            state[p * 8 + 2 * (LEVEL - 1) + kStPrefix], scan, sel);
  // (state words 2L, 2L+1 hold the selection after level L; nobody reads the words this pass writes)
  if (first && threadIdx.x == 0) {
    state[p * 8 + 2 * LEVEL + kStPrefix] = sel[0];
    state[p * 8 + 2 * LEVEL + kStKRem] = sel[1];
  }
}

// Keys of 4 consecutive elements from j (a multiple of 4) of a partition of d elements;
// *n receives how many of them exist.
__device__ inline void keys4(const float *part, uint32_t j, uint32_t d, uint32_t key[4], uint32_t *n) {
  if (j + 4 <= d) {
    const float4 f = *reinterpret_cast<const float4 *>(part + j);
    key[0] = key_of(f.x); key[1] = key_of(f.y); key[2] = key_of(f.z); key[3] = key_of(f.w);
    *n = 4;
  } else {
    *n = j < d ? d - j : 0u;
#pragma unroll
    for (int c = 0; c < 4; ++c) key[c] = j + c < d ? key_of(part[j + c]) : 0u;
  }
}

// The long-form kernels take their groups of tiles in a loop, so that they can be launched with
// a small grid behind the short-list form (`gated`: only partitions left to the long form).

// LEVEL 2: keys whose top 11 bits equal the prefix, histogram of the next 10 bits.
// LEVEL 3: keys whose top 21 bits equal the prefix, histogram of the last 10 bits.
// LEVEL 1 (long form behind the short-list form only, whose load pass counts nothing): all keys.
template <int LEVEL>
__device__ inline void topk_hist_body(const Geo &g, const float *buf, uint32_t *hist, uint32_t *state, uint32_t n_groups,
                                      int gated) {
  constexpr int kBins = LEVEL == 1 ? kBins1 : kBins23;
  __shared__ uint32_t h[kBins];
  __shared__ uint32_t scan[kThreads];
  __shared__ uint32_t sel[2];
  for (uint32_t blk = blockIdx.x; blk < n_groups; blk += gridDim.x) {
    const GroupOf w = group_of<LEVEL == 2 ? kTpgHist2 : kTpgHist3>(g, blk);
    if (gated && !long_form(state, w.p)) continue;
    for (int b = threadIdx.x; b < kBins; b += kThreads) h[b] = 0;
    if constexpr (LEVEL == 1) {
      __syncthreads();
      const float *part1 = buf + g.part_base(w.p);
      for (uint32_t tile = w.tile_lo; tile < w.tile_hi; ++tile) {
#pragma unroll
        for (int c = 0; c < kTile / (kThreads * 4); ++c) {
          uint32_t key[4], n;
          keys4(part1, tile * kTile + c * (kThreads * 4) + threadIdx.x * 4, w.d, key, &n);
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if ((uint32_t)e < n) atomicAdd(&h[key[e] >> kShift1], 1u);
        }
      }
      __syncthreads();
      uint32_t *gh1 = hist + (uint64_t)w.p * kTopkHistWords + kHist1;
      for (int b = threadIdx.x; b < kBins; b += kThreads)
        if (h[b]) atomicAdd(&gh1[b], h[b]);
      __syncthreads();
      continue;
    }
    selection_after<(LEVEL > 1 ? LEVEL - 1 : 1)>(g, hist, state, w.p, w.tile_lo == 0, scan, sel);
    const uint32_t prefix = sel[0];
    constexpr int kHiShift = LEVEL == 2 ? kShift1 : kShift2;
    constexpr int kLoShift = LEVEL == 2 ? kShift2 : 0;
    const float *part = buf + g.part_base(w.p);
    for (uint32_t tile = w.tile_lo; tile < w.tile_hi; ++tile) {
#pragma unroll
      for (int c = 0; c < kTile / (kThreads * 4); ++c) {
        uint32_t key[4], n;
        keys4(part, tile * kTile + c * (kThreads * 4) + threadIdx.x * 4, w.d, key, &n);
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if ((uint32_t)e < n && (key[e] >> kHiShift) == prefix) atomicAdd(&h[(key[e] >> kLoShift) & (kBins23 - 1)], 1u);
      }
    }
    __syncthreads();
    uint32_t *gh = hist + (uint64_t)w.p * kTopkHistWords + (LEVEL == 2 ? kHist2 : kHist3);
    for (int b = threadIdx.x; b < kBins23; b += kThreads)
      if (h[b]) atomicAdd(&gh[b], h[b]);
    __syncthreads();
  }
}

template <int LEVEL>
__global__ __launch_bounds__(kThreads) void topk_hist_kernel(Geo g, const float *buf, uint32_t *hist, uint32_t *state,
                                                             uint32_t n_groups) {
  topk_hist_body<LEVEL>(g, buf, hist, state, n_groups, 0);
}

// Per tile: number of keys above the threshold and equal to it.  The first workgroup of a
// partition also records the threshold key T and the number r of keys equal to T that are
// kept, for the compaction.
__device__ inline void topk_count_body(const Geo &g, const float *buf, const uint32_t *hist, uint32_t *state,
                                       uint32_t *tilecnt, uint32_t n_groups, int gated) {
  __shared__ uint32_t red[2][kThreads / 64];
  __shared__ uint32_t scan[kThreads];
  __shared__ uint32_t sel[2];
  for (uint32_t blk = blockIdx.x; blk < n_groups; blk += gridDim.x) {
    const GroupOf w = group_of<kTpgCount>(g, blk);
    if (gated && !long_form(state, w.p)) continue;
    selection_after<3>(g, hist, state, w.p, w.tile_lo == 0, scan, sel);
    const uint32_t T = sel[0];
    const float *part = buf + g.part_base(w.p);
    for (uint32_t tile = w.tile_lo; tile < w.tile_hi; ++tile) {
      uint32_t n_gt = 0, n_eq = 0;
#pragma unroll
      for (int c = 0; c < kTile / (kThreads * 4); ++c) {
        uint32_t key[4], n;
        keys4(part, tile * kTile + c * (kThreads * 4) + threadIdx.x * 4, w.d, key, &n);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          n_gt += (uint32_t)e < n && key[e] > T;
          n_eq += (uint32_t)e < n && key[e] == T;
        }
      }
      n_gt = wave_sum_u32(n_gt);
      n_eq = wave_sum_u32(n_eq);
      __syncthreads();
      if ((threadIdx.x & 63) == 0) {
        red[0][threadIdx.x >> 6] = n_gt;
        red[1][threadIdx.x >> 6] = n_eq;
      }
      __syncthreads();
      if (threadIdx.x == 0) {
        uint32_t a = 0, b = 0;
        for (int v = 0; v < kThreads / 64; ++v) { a += red[0][v]; b += red[1][v]; }
        const uint64_t t = (uint64_t)w.p * g.tiles_per_part + tile;
        tilecnt[2 * t] = a;
        tilecnt[2 * t + 1] = b;
      }
    }
    __syncthreads();
  }
}

__global__ __launch_bounds__(kThreads) void topk_count_kernel(Geo g, const float *buf, const uint32_t *hist,
                                                              uint32_t *state, uint32_t *tilecnt, uint32_t n_groups) {
  topk_count_body(g, buf, hist, state, tilecnt, n_groups, 0);
}

// Header of partition p's record; for the half-value form also the zeros the format wants from
// value k to the end of its last group of four words.
template <bool HALF>
__device__ inline void topk_write_header(const Geo &g, uint32_t p, uint8_t *payload) {
  uint8_t *rec0 = payload + (uint64_t)p * g.stride;
  uint32_t *hdr = reinterpret_cast<uint32_t *>(rec0);
  const uint32_t k = (uint32_t)k_of_device(g, p);
  hdr[0] = k;
  hdr[1] = 0; hdr[2] = 0; hdr[3] = 0;
  if (HALF) {
    uint16_t *val16 = reinterpret_cast<uint16_t *>(rec0 + kHeaderBytes + 4 * ru4(g.k_cap));
    for (uint32_t t = k; t < 2 * (uint32_t)ru4(cdiv(k, 2)); ++t) val16[t] = 0;
  }
}

// Entry `pos` of partition p's record: element j with value v; the buffer keeps 0 there, or
// what rounding to half dropped.
template <bool HALF>
__device__ inline void topk_write_entry(const Geo &g, uint8_t *rec, uint32_t pos, uint32_t j, float v, float *buf_part,
                                        int zero_selected) {
  uint32_t *idx = reinterpret_cast<uint32_t *>(rec + kHeaderBytes);
  float *val = reinterpret_cast<float *>(rec + kHeaderBytes + 4 * ru4(g.k_cap));
  idx[pos] = j;
  if (HALF) {
    const __half h = __float2half_rn(v);
    reinterpret_cast<__half *>(val)[pos] = h;
    if (zero_selected) buf_part[j] = v - __half2float(h);
  } else {
    val[pos] = v;
    if (zero_selected) buf_part[j] = 0.0f;
  }
}

// The vector that was compressed, of one partition: the buffer, or the gradient in f32 or f16.  at(j): the f32 bits
// of four elements from j on, a multiple of four; zeros past the end.
struct PartValues {
  TileBuf b;
  uint32_t d;
  bool half;
  __device__ PartValues(const void *part, uint32_t elems, bool halves) : b(part, elems * (halves ? 2 : 4)), d(elems), half(halves) {}
  __device__ u32x4 at(uint32_t j) const {
    if (!half) return b.load16(j * 4, 0);
    u32x2 hw = b.load8(j * 2, 0);
    if ((d & 1u) && d - 1 - j < 4u) {   // the last half of an odd number: its dword reads as zero
      const uint32_t one = b.load2((d - 1) * 2, 0);
      if (d - 1 - j == 0) hw.x = one; else hw.y = one;
    }
    float f[4];
    widen4(hw, f);
    return as_u32x4(f[0], f[1], f[2], f[3]);
  }
};
__device__ inline PartValues part_values(const Geo &g, uint32_t p, const float *buf, const void *values, int values16) {
  const uint64_t base = uniform_off(g.part_base(p));
  const bool half = !buf && values16;
  return PartValues(buf ? (const void *)(buf + base) : half ? (const void *)((const __half *)values + base) : (const void *)((const float *)values + base),
                    g.part_size(p), half);
}

// The long form of one partition by one workgroup of kSelThreads: three histogram passes, a pass that
// counts per wave, a pass that writes; wave w takes the w-th stretch of the partition.  h: LDS,
// kBins1 words.  Every element is read five times by one compute unit, in the rare case that the sample misled: a worker
// call on partitions of 1 M f32 elements that all do takes 0.57 to 0.59 ms (the resident kernel below 0.68 to
// 0.80), of 2 M f16 1.05 to 1.23 (0.91, and 4.7 us more in every ordinary call), of 4 M f32 2.02 (0.68 to 1.06):
// hence kAloneElems.  (Group lists of 1 M elements, k = 3 %: 1.25 ms.)
// The vector is `buf`, whose kept slots are zeroed with error feedback, or else the gradient `values` in f32 or f16.
template <bool HALF>
__device__ inline void topk_alone(const Geo &g, uint32_t p, uint32_t k, float *buf, const void *values, int values16, uint8_t *payload,
                                  int zero_selected, uint32_t *h, uint32_t *scan, uint32_t *sel) {
  constexpr int kWaves = kSelThreads / 64;
  constexpr uint32_t kRow = 256, kAhead = 4;   // elements a wave takes at once; rows in flight
  __shared__ uint32_t wave_cnt[2][kWaves];
  const uint32_t d = g.part_size(p);
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const uint32_t seg = (uint32_t)cdiv(cdiv(d, kWaves), kRow) * kRow;
  const uint32_t lo = wave * seg < d ? wave * seg : d, hi = lo + seg < d ? lo + seg : d;
  float *buf_part = buf ? buf + uniform_off(g.part_base(p)) : nullptr;
  const PartValues x_of = part_values(g, p, buf, values, values16);
  // visit(j, bits): the wave's elements in order, four consecutive ones a lane, kAhead rows requested at once
  auto walk = [&](auto visit) {
#pragma unroll 1
    for (uint32_t r0 = lo; r0 < hi; r0 += kAhead * kRow) {
      u32x4 x[kAhead];
#pragma unroll
      for (uint32_t q = 0; q < kAhead; ++q) x[q] = x_of.at(r0 + q * kRow + lane * 4);
#pragma unroll
      for (uint32_t q = 0; q < kAhead; ++q) {
        const uint32_t v[4] = {x[q].x, x[q].y, x[q].z, x[q].w};
        visit(r0 + q * kRow + lane * 4, v);
      }
    }
  };
  uint32_t prefix = 0, rem = k;
#pragma unroll 1
  for (int level = 1; level <= 3; ++level) {
    const int hi_shift = level == 1 ? 31 : level == 2 ? kShift1 : kShift2, lo_shift = level == 1 ? kShift1 : level == 2 ? kShift2 : 0;
    const uint32_t mask = level == 1 ? kBins1 - 1 : kBins23 - 1;
    __syncthreads();
    for (int q = threadIdx.x; q < kBins1; q += kSelThreads) h[q] = 0;
    __syncthreads();
    walk([&](uint32_t j, const uint32_t v[4]) {
      // a row of one bin (zeros, equal magnitudes: the usual reasons to be here) is added at once
      const uint32_t key0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)(v[0] & 0x7fffffffu));
      uint32_t differ = j + 3 < hi ? 0u : 1u;
#pragma unroll
      for (int e = 0; e < 4; ++e) differ |= ((v[e] & 0x7fffffffu) ^ key0) >> lo_shift;
      if (__ballot(differ != 0) == 0) {
        if (lane == 0 && (key0 >> hi_shift) == prefix) atomicAdd(&h[(key0 >> lo_shift) & mask], kRow);
        return;
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t key = v[e] & 0x7fffffffu;
        if (j + e < hi && (key >> hi_shift) == prefix) atomicAdd(&h[(key >> lo_shift) & mask], 1u);
      }
    });
    __syncthreads();
    if (level == 1) pick_bin<kBins1, kBits1, kSelThreads>(h, rem, 0, scan, sel);
    else pick_bin<kBins23, kBits23, kSelThreads>(h, rem, prefix, scan, sel);
    prefix = sel[0];
    rem = sel[1];
  }
  const uint32_t T = prefix, r = rem;
  uint32_t n_gt = 0, n_eq = 0;   // (the same in every lane)
  walk([&](uint32_t j, const uint32_t v[4]) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t key = v[e] & 0x7fffffffu;
      n_gt += (uint32_t)__popcll(__ballot(j + e < hi && key > T));
      n_eq += (uint32_t)__popcll(__ballot(j + e < hi && key == T));
    }
  });
  if (lane == 0) { wave_cnt[0][wave] = n_gt; wave_cnt[1][wave] = n_eq; }
  __syncthreads();
  uint32_t gt_base = 0, eq_base = 0;
  for (uint32_t q = 0; q < wave; ++q) { gt_base += wave_cnt[0][q]; eq_base += wave_cnt[1][q]; }
  uint8_t *rec = payload + (uint64_t)p * g.stride;
  walk([&](uint32_t j, const uint32_t v[4]) {
    uint32_t both = 0;   // above T | equal to T << 16
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t key = v[e] & 0x7fffffffu;
      both += j + e < hi ? (key > T ? 1u : 0u) + (key == T ? 0x10000u : 0u) : 0u;
    }
    if (__ballot((both & 0xffffu) != 0 || (both != 0 && eq_base < r)) == 0) return;   // nothing to write (and no tie to count any more)
    const uint32_t incl = wave_inclusive_scan_u32(both), ex = incl - both;
    uint32_t gt = gt_base + (ex & 0xffffu), eq = eq_base + (ex >> 16);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t key = v[e] & 0x7fffffffu;
      const bool above = j + e < hi && key > T, tie = j + e < hi && key == T;
      if (above || (tie && eq < r)) topk_write_entry<HALF>(g, rec, gt + (eq < r ? eq : r), j + e, __uint_as_float(v[e]), buf_part, zero_selected);
      gt += above;
      eq += tie;
    }
    const uint32_t all = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
    gt_base += all & 0xffffu;
    eq_base += all >> 16;
  });
}

// The entries of a list in the registers of a workgroup of kSelThreads, PER a thread of which `rounds` (a
// multiple of 4, the same for all threads) are in use: rel[i] = magnitude key - guess + 1 and the value's
// sign bit, 0 where there is no entry.
constexpr uint32_t kRelMask = 0x7fffffffu;
// body(i) for the entries in use, four at a time.
template <int PER, class BODY>
__device__ __forceinline__ void each_entry(uint32_t rounds, BODY body) {
  if constexpr (PER > 4) each_entry<PER - 4>(rounds, body);
  if ((uint32_t)(PER - 4) < rounds) {
    body(std::integral_constant<int, PER - 4>{});
    body(std::integral_constant<int, PER - 3>{});
    body(std::integral_constant<int, PER - 2>{});
    body(std::integral_constant<int, PER - 1>{});
  }
}

// pick_bin() for a histogram of 4 bins a thread or more, with two barriers: `scan` (a word a wave) and
// sel must not be in use.
template <int BINS>
__device__ inline void pick_bin_once(const uint32_t *h, uint32_t k_rem, uint32_t *scan, uint32_t *sel) {
  constexpr int kPer = BINS / kSelThreads, kWaves = kSelThreads / 64;
  uint32_t cnt[kPer], local = 0;
  if constexpr (kPer % 4 == 0) {
#pragma unroll
    for (int i = 0; i < kPer; i += 4) {
      const uint4 x = *reinterpret_cast<const uint4 *>(h + (BINS - 4 - (int)threadIdx.x * kPer - i));
      cnt[i] = x.w; cnt[i + 1] = x.z; cnt[i + 2] = x.y; cnt[i + 3] = x.x;
    }
  } else {
#pragma unroll
    for (int i = 0; i < kPer; ++i) cnt[i] = h[BINS - 1 - (int)threadIdx.x * kPer - i];
  }
#pragma unroll
  for (int i = 0; i < kPer; ++i) local += cnt[i];
  const uint32_t incl = wave_inclusive_scan_u32(local), wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 63) scan[wave] = incl;
  __syncthreads();
  uint32_t run = incl - local;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) run += (uint32_t)w < wave ? scan[w] : 0u;
  if (run < k_rem && k_rem <= run + local) {
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      if (run < k_rem && k_rem <= run + cnt[i]) {
        sel[0] = BINS - 1 - (threadIdx.x * kPer + i);
        sel[1] = k_rem - run;
      }
      run += cnt[i];
    }
  }
  __syncthreads();
}

// LDS of a select workgroup.
struct SelectLds {
  uint32_t h[kSelBins];            // first level of the threshold; the passes for rarer cases
  uint32_t h2[1024];               // second level
  uint32_t bitmap[kShareWords];
  uint16_t before[kShareWords];    // bits set before a word of it
  uint32_t scan[3][kSelThreads / 64];
  uint32_t sel[3][2];
  uint32_t tie[64], tied;          // a few entries equal to the threshold
};
static_assert(kSelThreads == 1024, "a bin a thread in the levels of 1024 bins");

// The rel R of rank k and the number r of entries equal to it that are kept, for all threads; *ties:
// how many entries equal R.  Keys are rarely an octave above the guess: bins of 1024 keys from there
// up, then the keys of one bin; else three levels over the whole range.  h and h2 are zero, and a barrier
// has been since.
template <int PER>
__device__ inline void list_threshold(const uint32_t (&rel)[PER], uint32_t rounds, uint32_t k, SelectLds &l, uint32_t *R, uint32_t *r,
                                      uint32_t *ties) {
  each_entry<PER>(rounds, [&](auto i) {
    const uint32_t x = rel[i] & kRelMask, bin = x >> 10;
    if (x) atomicAdd(&l.h[bin < (uint32_t)kSelBins ? bin : kSelBins - 1u], 1u);
  });
  __syncthreads();
  pick_bin_once<kSelBins>(l.h, k, l.scan[0], l.sel[0]);
  uint32_t prefix = l.sel[0][0], rem = l.sel[0][1];
  if (prefix == (uint32_t)kSelBins - 1) {   // (uniform) past the octave: the top 21 bits in two steps
    rem = k;
#pragma unroll 1
    for (int shift = 20; shift >= 10; shift -= 10) {
      const uint32_t above = prefix;
      __syncthreads();
      for (int b = threadIdx.x; b < 2048; b += kSelThreads) l.h[b] = 0;
      __syncthreads();
      each_entry<PER>(rounds, [&](auto i) {
        const uint32_t x = rel[i] & kRelMask;
        if (x && (shift == 20 || (x >> 20) == above)) atomicAdd(&l.h[(x >> shift) & (shift == 20 ? 2047u : 1023u)], 1u);
      });
      __syncthreads();
      if (shift == 20) pick_bin<2048, 11, kSelThreads>(l.h, rem, 0, l.scan[1], l.sel[1]);
      else pick_bin<1024, 10, kSelThreads>(l.h, rem, prefix, l.scan[1], l.sel[1]);
      prefix = l.sel[1][0];
      rem = l.sel[1][1];
    }
  }
  each_entry<PER>(rounds, [&](auto i) {
    const uint32_t x = rel[i] & kRelMask;
    if (x && (x >> 10) == prefix) atomicAdd(&l.h2[x & 1023u], 1u);
  });
  __syncthreads();
  pick_bin_once<1024>(l.h2, rem, l.scan[2], l.sel[2]);
  *R = prefix << 10 | l.sel[2][0];
  *r = l.sel[2][1];
  *ties = l.h2[l.sel[2][0]];
}

// The index of the r-th of the `ties` entries equal to R in index order (r < ties).  A few of them, as
// the sums of halves often give, are collected in LDS and each one's rank is counted; more take a
// radix select on the indices (below 2^28: 10 + 10 + 8 bits).
template <int PER>
__device__ inline uint32_t last_tie(const uint32_t (&rel)[PER], const uint32_t (&where)[PER], uint32_t rounds, uint32_t R, uint32_t r,
                                    uint32_t ties, SelectLds &l) {
  constexpr uint32_t kFew = 64;
  if (ties <= kFew) {   // (uniform)
    each_entry<PER>(rounds, [&](auto i) {
      if ((rel[i] & kRelMask) == R) l.tie[atomicAdd(&l.tied, 1u)] = where[i];
    });
    __syncthreads();
    if (threadIdx.x < ties) {
      const uint32_t mine = l.tie[threadIdx.x];
      uint32_t rank = 1;
      for (uint32_t t = 0; t < ties; ++t) rank += l.tie[t] < mine;
      if (rank == r) l.sel[0][0] = mine;
    }
    __syncthreads();
    return l.sel[0][0];
  }
  uint32_t prefix = 0, rem = ties - r + 1;   // (pick_bin counts from the largest down)
#pragma unroll 1
  for (int level = 0; level < 3; ++level) {
    const int hi_shift = level == 0 ? 28 : level == 1 ? 18 : 8, lo_shift = level == 0 ? 18 : level == 1 ? 8 : 0;
    __syncthreads();
    l.h[threadIdx.x] = 0;
    __syncthreads();
    each_entry<PER>(rounds, [&](auto i) {
      if ((rel[i] & kRelMask) == R && (where[i] >> hi_shift) == prefix)
        atomicAdd(&l.h[(where[i] >> lo_shift) & (level == 2 ? 255u : 1023u)], 1u);
    });
    __syncthreads();
    if (level == 2) pick_bin<256, 8, kSelThreads>(l.h, rem, prefix, l.scan[0], l.sel[0]);
    else pick_bin<1024, 10, kSelThreads>(l.h, rem, prefix, l.scan[0], l.sel[0]);
    prefix = l.sel[0][0];
    rem = l.sel[0][1];
  }
  return prefix;
}

// Ties beside the list of a partition: the listed elements, all above one key, are fewer than k, and the rest of
// the k are elements of that key, lowest index first.  The load pass has counted them per group, so a workgroup
// of kSelThreads finds from the counts which group holds the last one that is kept.
struct TieCut {
  uint32_t all, before;    // of them in the partition, in groups before the workgroup's
  uint32_t group, rest;    // the group of the last kept one, and how many of that group are kept
};
// `need` of them are kept; the workgroup's first group is q0 (below `groups`).
__device__ __forceinline__ TieCut tie_cut(const TopkLists &lists, uint32_t p, uint32_t groups, uint32_t need, uint32_t q0, uint32_t *scan,
                                 uint32_t *sel, uint32_t shift = 0) {
  static_assert(kMostOfList / kGroupElems <= kSelThreads && kAloneElems <= kMostOfList, "a group a thread");
  TieCut c;
  const uint32_t mine = threadIdx.x < groups ? lists.count(p, threadIdx.x)[1] >> shift : 0u;
  const uint32_t before = block_exclusive_scan<kSelThreads>(mine, scan, &c.all);
  if (before < need && need <= before + mine) { sel[0] = threadIdx.x; sel[1] = need - before; }
  if (threadIdx.x == q0) scan[0] = before;
  __syncthreads();
  c.group = __builtin_amdgcn_readfirstlane(sel[0]);
  c.rest = __builtin_amdgcn_readfirstlane(sel[1]);
  c.before = __builtin_amdgcn_readfirstlane(scan[0]);
  __syncthreads();
  return c;
}
// Ties (elements of key T) of [lo, hi), whole groups or up to the partition's end, are kept up to the index returned.
__device__ __forceinline__ uint32_t tie_end(const PartValues &x, uint32_t T, const TieCut &c, uint32_t lo, uint32_t hi, uint32_t *scan, uint32_t *sel) {
  static_assert(kGroupElems == 8 * kSelThreads, "eight elements a thread");
  const uint32_t at = c.group * kGroupElems;
  if (at < lo) return lo;
  if (at >= hi) return hi;
  const uint32_t j0 = at + threadIdx.x * 8;
  const u32x4 a = x.at(j0), b = x.at(j0 + 4);
  const uint32_t v[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
  uint32_t mask = 0;
#pragma unroll
  for (uint32_t e = 0; e < 8; ++e) mask |= (uint32_t)(j0 + e < x.d && (v[e] & 0x7fffffffu) == T) << e;
  uint32_t all;
  const uint32_t before = block_exclusive_scan<kSelThreads>((uint32_t)__popc(mask), scan, &all);
  if (before < c.rest && c.rest <= before + (uint32_t)__popc(mask)) {
    for (uint32_t skip = c.rest - before; skip > 1; --skip) mask &= mask - 1;
    sel[0] = j0 + (uint32_t)__builtin_ctz(mask) + 1;
  }
  __syncthreads();
  const uint32_t end = __builtin_amdgcn_readfirstlane(sel[0]);
  __syncthreads();
  return end;
}
// visit(j, bits) for the elements of key T in [lo, hi), lo a multiple of four.
template <class VISIT>
__device__ __forceinline__ void each_tie(const PartValues &x, uint32_t T, uint32_t lo, uint32_t hi, VISIT visit) {
  constexpr uint32_t kAhead = 4;
  for (uint32_t j0 = lo + threadIdx.x * 4; j0 < hi; j0 += kAhead * 4 * kSelThreads) {
    u32x4 r[kAhead];
#pragma unroll
    for (uint32_t q = 0; q < kAhead; ++q) r[q] = x.at(j0 + q * 4 * kSelThreads);
#pragma unroll
    for (uint32_t q = 0; q < kAhead; ++q) {
      const uint32_t v[4] = {r[q].x, r[q].y, r[q].z, r[q].w}, j = j0 + q * 4 * kSelThreads;
#pragma unroll
      for (uint32_t e = 0; e < 4; ++e)
        if (j + e < hi && (v[e] & 0x7fffffffu) == T) visit(j + e, v[e]);
    }
  }
}

// The bits before every word of the bitmap, in l.before; the sum of the threads' `below` (at most kTopkListCap, as
// the number of bits).
__device__ __forceinline__ uint32_t bits_before_words(SelectLds &l, uint32_t words, uint32_t below) {
  // bits before each word: thread t owns words per * t .. per * t + per - 1
  const uint32_t per = 4 * (uint32_t)cdiv(words, 4 * kSelThreads);
  uint32_t set = 0;
  for (uint32_t q = 0; q < per; q += 4) {
    const uint32_t w = threadIdx.x * per + q;
    if (w < words) {
      const uint4 x = *reinterpret_cast<const uint4 *>(l.bitmap + w);   // (past the last word: zeros up to the multiple of 4)
      set += (uint32_t)(__popc(x.x) + __popc(x.y) + __popc(x.z) + __popc(x.w));
    }
  }
  // (one scan for both: each total is at most kTopkListCap)
  const uint32_t both = set | below << 16, incl = wave_inclusive_scan_u32(both), wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 63) l.scan[1][wave] = incl;
  __syncthreads();
  uint32_t all = 0, at = incl - both;
#pragma unroll
  for (uint32_t w = 0; w < kSelThreads / 64; ++w) {
    const uint32_t x = l.scan[1][w];
    at += w < wave ? x : 0u;
    all += x;
  }
  at &= 0xffffu;
  for (uint32_t q = 0; q < per; q += 4) {
    const uint32_t w = threadIdx.x * per + q;
    if (w < words) {
      const uint4 x = *reinterpret_cast<const uint4 *>(l.bitmap + w);
      const uint32_t a1 = at + (uint32_t)__popc(x.x), a2 = a1 + (uint32_t)__popc(x.y), a3 = a2 + (uint32_t)__popc(x.z);
      *reinterpret_cast<uint2 *>(l.before + w) = make_uint2(at | a1 << 16, a2 | a3 << 16);
      at = a3 + (uint32_t)__popc(x.w);
    }
  }
  __syncthreads();
  return all >> 16;
}

// A share of the select pass where ties of key T beside the list make its n entries up to k: all entries are kept, and
// ties as far as they go; the share's indices are [lo, hi).  false if there are not enough of them.
template <bool HALF>
__device__ __forceinline__ bool select_with_ties(const Geo &g, uint32_t p, uint32_t share, uint32_t lo, uint32_t hi, uint32_t n, uint32_t k, uint32_t T,
                                        float *buf, const void *values, int values16, uint32_t *state, const TopkLists &lists,
                                        uint8_t *payload, int zero_selected, SelectLds &l) {
  const TieCut cut = tie_cut(lists, p, (g.part_size(p) + kGroupElems - 1) / kGroupElems, k - n, lo / kGroupElems, l.scan[0], l.sel[0]);
  if (cut.all < k - n) return false;
  if (share == 0 && threadIdx.x == 0) state[p * 8 + kStLong] = kTiesBeside;
  const PartValues x_of = part_values(g, p, buf, values, values16);
  const uint32_t ties_to = tie_end(x_of, T, cut, lo, hi, l.scan[0], l.sel[0]);
  const uint32_t words = (hi - lo + 31) / 32;
  for (uint32_t w = threadIdx.x; w < (words + 3) / 4 * 4; w += kSelThreads) l.bitmap[w] = 0;
  __syncthreads();
  const uint32_t *idx = lists.idx(p), *val = lists.val(p);
  uint32_t below = 0;
  for (uint32_t e = threadIdx.x; e < n; e += kSelThreads) {
    const uint32_t j = idx[e];
    below += j < lo;
    if (j >= lo && j < hi) atomicOr(&l.bitmap[(j - lo) >> 5], 1u << (j & 31u));
  }
  each_tie(x_of, T, lo, ties_to, [&](uint32_t j, uint32_t) { atomicOr(&l.bitmap[(j - lo) >> 5], 1u << (j & 31u)); });
  __syncthreads();
  const uint32_t pos0 = bits_before_words(l, words, below) + (cut.before < k - n ? cut.before : k - n);
  uint8_t *rec = payload + (uint64_t)p * g.stride;
  float *buf_part = zero_selected ? buf + g.part_base(p) : nullptr;
  auto write = [&](uint32_t j, uint32_t bits) {
    const uint32_t o = j - lo, w = o >> 5;
    const uint32_t pos = pos0 + l.before[w] + (uint32_t)__popc(l.bitmap[w] & ((1u << (o & 31u)) - 1u));
    topk_write_entry<HALF>(g, rec, pos, j, __uint_as_float(bits), buf_part, zero_selected);
  };
  each_tie(x_of, T, lo, ties_to, write);
  __syncthreads();   // (a listed element's slot of the buffer, once zeroed, could pass for a tie)
  for (uint32_t e = threadIdx.x; e < n; e += kSelThreads) {
    const uint32_t j = idx[e];
    if (j >= lo && j < hi) write(j, val[e]);
  }
  return true;
}

// Select pass.  `shares` workgroups take a partition: each keeps the whole list in registers and works out
// which entries are kept, marks those of its share of the indices in a bitmap in LDS, and writes
// them at the places that the bits before them give.  A list shorter than k or longer than its room
// leaves the partition to the long form, unless ties beside it make it up to k: a share then reads its indices
// of the vector as far as ties are kept.  Bound by the vector instructions per entry (sixteen waves on
// one compute unit) and some twenty barriers.  (The form before this one took the list in index
// order, run by run of the load pass's workgroups, through a table in LDS, with three radix levels
// and the idle long form behind it: 28 against 19 us on 25 partitions of 1 M elements, k = 1 %; 23 against
// 15.5 us on 53 partitions of 2 M f16 elements, k = 0.1 %.)
struct ShareRanges { uint32_t list, ties; };   // indices a share takes: multiples of 32, and (with ties beside the list) of kGroupElems
template <bool HALF>
__global__ __launch_bounds__(kSelThreads) void topk_list_select_kernel(Geo g, float *buf, const void *values, int values16, uint32_t *state, TopkShared sh, TopkLists lists,
                                                                       uint8_t *payload, int zero_selected, uint32_t shares, ShareRanges ranges) {
  __shared__ __align__(16) SelectLds l;
  static_assert(kSelPer <= 32 && kTopkListCap < 65536, "one bit an entry, 16 bits a place");
  // (workgroups go to the 8 XCDs in turn: the shares of a partition, which read the same list, to the same one)
  const uint32_t at_xcd = blockIdx.x / kXcds;
  const uint32_t p = __builtin_amdgcn_readfirstlane(at_xcd / shares * kXcds + blockIdx.x % kXcds), share = __builtin_amdgcn_readfirstlane(at_xcd % shares);
  if (p >= g.P) return;
  const uint32_t d = g.part_size(p);
  const uint32_t n = __builtin_amdgcn_readfirstlane(*sh.length(p));
  const uint64_t pair = sh.pair(p)[0];
  // (the highest key is taken for the one below it: less a guess of 0, plus one, it would read as no entry, and a
  // threshold would be looked for among fewer than k of them)
  constexpr uint32_t kTopKey = kRelMask - 1;
  const uint32_t guess = __builtin_amdgcn_readfirstlane((uint32_t)pair), G = guess < kTopKey ? guess : kTopKey;
  const uint32_t k = (uint32_t)k_of_device(g, p);
  const bool beside = n < k && __builtin_amdgcn_readfirstlane((uint32_t)(pair >> 32)) != 0;   // ties of the key below the guess are kept
  const uint32_t range = beside ? ranges.ties : ranges.list;
  const uint32_t lo = share * range, hi = lo + range < d ? lo + range : d;
  if (lo >= d) return;
  if (share == 0 && threadIdx.x == 0) topk_write_header<HALF>(g, p, payload);
  if (n < k || n > kTopkListCap) {
    if (beside && select_with_ties<HALF>(g, p, share, lo, hi, n, k, guess - 1u, buf, values, values16, state, lists, payload, zero_selected, l)) return;
    if (share != 0) return;
    if (threadIdx.x == 0) state[p * 8 + kStLong] = kLongForm;
    if (g.part_size(0) <= kAloneElems) topk_alone<HALF>(g, p, k, buf, values, values16, payload, zero_selected, l.h, l.scan[0], l.sel[0]);
    return;
  }
  // entry 4 (i * kSelThreads + thread) + c of the list is the thread's entry 4 i + c; all loads of a kind are
  // requested before the first is used, the values first
  const uint32_t rounds = 4 * (uint32_t)cdiv(n, 4 * kSelThreads);   // at most kSelPer
  uint32_t rel[kSelPer], where[kSelPer];
  {
    const TileBuf vb(lists.val(p), n * 4), ib(lists.idx(p), n * 4);
    auto load = [&](const TileBuf &b, uint32_t (&to)[kSelPer]) {
#pragma unroll
      for (int i = 0; i < kSelPer; i += 4) {
        u32x4 x{};
        if ((uint32_t)i < rounds) x = b.load16(threadIdx.x * 16, i * kSelThreads * 4);   // (the same for all threads)
        to[i] = x.x; to[i + 1] = x.y; to[i + 2] = x.z; to[i + 3] = x.w;
      }
    };
    load(vb, rel);
    load(ib, where);
  }
  const uint32_t words = range / 32;   // (at most kShareWords)
  {
    const uint4 zero = make_uint4(0, 0, 0, 0);
    for (uint32_t b = threadIdx.x; b < kSelBins / 4; b += kSelThreads) reinterpret_cast<uint4 *>(l.h)[b] = zero;
    l.h2[threadIdx.x] = 0;
    if (threadIdx.x == 0) l.tied = 0;
    for (uint32_t b = threadIdx.x; 4 * b < words; b += kSelThreads) reinterpret_cast<uint4 *>(l.bitmap)[b] = zero;
  }
  __syncthreads();
  each_entry<kSelPer>(rounds, [&](auto i) {
    constexpr uint32_t first = (i / 4) * (4 * kSelThreads) + i % 4;
    const uint32_t key = rel[i] & kRelMask;
    rel[i] = first + threadIdx.x * 4 < n ? ((key < kTopKey ? key : kTopKey) - G + 1u) | (rel[i] & ~kRelMask) : 0u;
  });
  uint32_t R, r, ties;
  list_threshold<kSelPer>(rel, rounds, k, l, &R, &r, &ties);
  uint32_t last = 0xffffffffu;   // of the entries equal to R, those up to this index are kept
  if (ties != r) last = last_tie<kSelPer>(rel, where, rounds, R, r, ties, l);
  uint32_t below = 0;   // kept entries of the shares before this one
  uint32_t mine = 0;    // bit i: the thread's entry i is kept and in this share
  auto mark = [&](auto is_kept) {
    each_entry<kSelPer>(rounds, [&](auto i) {
      const bool kept = is_kept(rel[i] & kRelMask, where[i]);
      const uint32_t at = where[i] - lo;
      below += kept && where[i] < lo;
      if (kept && at < range) {
        mine |= 1u << i;
        atomicOr(&l.bitmap[at >> 5], 1u << (at & 31u));
      }
    });
  };
  if (ties == r) mark([&](uint32_t x, uint32_t) { return x >= R; });
  else mark([&](uint32_t x, uint32_t j) { return x > R || (x == R && j <= last); });
  __syncthreads();
  const uint32_t pos0 = bits_before_words(l, words, below);
  uint8_t *rec = payload + (uint64_t)p * g.stride;
  float *buf_part = zero_selected ? buf + g.part_base(p) : nullptr;
  each_entry<kSelPer>(rounds, [&](auto i) {
    if ((mine >> i) & 1u) {
      const uint32_t o = where[i] - lo, w = o >> 5;
      const uint32_t pos = pos0 + l.before[w] + (uint32_t)__popc(l.bitmap[w] & ((1u << (o & 31u)) - 1u));
      const uint32_t bits = ((rel[i] & kRelMask) - 1u + G) | (rel[i] & ~kRelMask);
      topk_write_entry<HALF>(g, rec, pos, where[i], __uint_as_float(bits), buf_part, zero_selected);
    }
  });
}

// Group-list form.  A workgroup takes kRangeGroups groups, two waves each.
constexpr uint32_t kRangeGroups = kSelThreads / 128;
struct GroupRange {
  uint32_t p, q0, q1, d;   // groups [q0, q1) of partition p
  __device__ GroupRange(const Geo &g, const TopkLists &lists) {
    const uint32_t ranges = (lists.groups + kRangeGroups - 1) / kRangeGroups;
    p = blockIdx.x / ranges;
    d = g.part_size(p);
    const uint32_t groups = (uint32_t)cdiv(d, kGroupElems);
    q0 = blockIdx.x % ranges * kRangeGroups;
    q1 = q0 + kRangeGroups < groups ? q0 + kRangeGroups : groups;
  }
};
// The vector that was compressed, for groups more than half of which are listed (one layer's gradient may
// dwarf the rest of its partition): the buffer, or the gradient in f32 or f16.
struct TopkVector {
  const void *at;
  int half;
  __device__ uint32_t bits(uint64_t j) const {
    return __float_as_uint(half ? __half2float(reinterpret_cast<const __half *>(at)[j]) : reinterpret_cast<const float *>(at)[j]);
  }
};
// Entries `first`, `first` + STEP, ... below n of a list: the first four are kept in registers, so that a kernel
// that goes over them more than once waits for them once; visit(rel, value, index), rel = key - guess.
// Without a list (`val` null) entry e is element `at` + e of the vector, index `j0` + e.
template <uint32_t STEP, bool IDX>
struct EntriesOf {
  const uint32_t *idx, *val;
  uint32_t first, n, G;
  TopkVector vec;
  uint64_t at;
  uint32_t j0, v[4], j[4];
  __device__ __forceinline__ void load(uint32_t e0, uint32_t (&lv)[4], uint32_t (&lj)[4]) const {
    if (val) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const uint32_t e = e0 + r * STEP;
        lv[r] = e < n ? val[e] : 0u;
        lj[r] = IDX && e < n ? idx[e] : 0u;
      }
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const uint32_t e = e0 + r * STEP;
        lv[r] = e < n ? vec.bits(at + e) : 0u;
        lj[r] = j0 + e;
      }
    }
  }
  __device__ __forceinline__ void load_first() { load(first, v, j); }
  template <class VISIT>
  __device__ __forceinline__ void each(VISIT visit) const {
    auto one = [&](uint32_t e, uint32_t x, uint32_t y) {
      const uint32_t key = x & 0x7fffffffu;
      if (e < n && key >= G) visit(key - G, x, y);
    };
#pragma unroll
    for (int r = 0; r < 4; ++r) one(first + r * STEP, v[r], j[r]);
    for (uint32_t e0 = first + 4 * STEP; e0 < n; e0 += 4 * STEP) {
      uint32_t lv[4], lj[4];
      load(e0, lv, lj);
#pragma unroll
      for (int r = 0; r < 4; ++r) one(e0 + r * STEP, lv[r], lj[r]);
    }
  }
};
// The entries of the wave's group, number q of the workgroup's range (none past its end).
template <bool IDX>
__device__ __forceinline__ EntriesOf<128, IDX> entries_of_group(const Geo &g, const TopkLists &lists, const GroupRange &w, uint32_t q, uint32_t G,
                                                       const TopkVector &vec) {
  EntriesOf<128, IDX> e{};
  e.first = threadIdx.x & 127;
  e.G = G;
  if (q < w.q1) {
    const TopkLists::List list = lists.of_group(g, w.p, q, w.d);
    e.n = __builtin_amdgcn_readfirstlane(*lists.count(w.p, q));
    if (e.n <= list.room) {
      e.idx = list.idx;
      e.val = list.val;
    } else {
      e.j0 = q * kGroupElems;
      e.n = w.d - e.j0 < kGroupElems ? w.d - e.j0 : kGroupElems;
      e.vec = vec;
      e.at = g.part_base(w.p) + e.j0;
    }
    e.load_first();
  }
  return e;
}
// 32 bins for every power of two of the distance from the guess, whatever the magnitudes' spread: a bin holds a
// few per cent of the list at most (unless keys are equal).  Bins below 864; bin b starts at near_start(b).
__device__ inline uint32_t near_bin(uint32_t rel) {
  const uint32_t e = 31u - (uint32_t)__builtin_clz(rel | 1u);
  return rel < 32u ? rel : (e - 4u) * 32u + ((rel >> (e - 5u)) & 31u);
}
__device__ inline uint32_t near_start(uint32_t b) { return b < 32u ? b : (32u + b % 32u) << (b / 32u - 1u); }

__global__ __launch_bounds__(kSelThreads) void topk_bins_kernel(Geo g, uint32_t *hist, TopkShared sh, TopkLists lists, TopkVector vec) {
  __shared__ uint32_t h[kNearBins];
  const GroupRange w(g, lists);
  if (w.q0 >= w.q1) return;
  const uint32_t q = __builtin_amdgcn_readfirstlane(w.q0 + (threadIdx.x >> 7));
  const uint32_t G = __builtin_amdgcn_readfirstlane((uint32_t)sh.pair(w.p)[0]);
  h[threadIdx.x] = 0;
  __syncthreads();
  entries_of_group<false>(g, lists, w, q, G, vec).each([&](uint32_t rel, uint32_t, uint32_t) { atomicAdd(&h[near_bin(rel)], 1u); });
  __syncthreads();
  if (h[threadIdx.x]) atomicAdd(&hist[(uint64_t)w.p * kTopkHistWords + threadIdx.x], h[threadIdx.x]);
}

// The bin of the k-th largest key of a partition in sel[0], the rank left in it in sel[1] (neither if the lists
// hold fewer than k); how many they hold.
__device__ __forceinline__ uint32_t near_bin_of_k(const uint32_t *bins, uint32_t k, uint32_t *scan, uint32_t *sel) {
  static_assert(kNearBins == kSelThreads, "a bin a thread");
  const uint32_t mine = bins[kNearBins - 1 - threadIdx.x];
  uint32_t total;
  const uint32_t above = block_exclusive_scan<kSelThreads>(mine, scan, &total);
  if (above < k && k <= above + mine) {
    sel[0] = kNearBins - 1 - threadIdx.x;
    sel[1] = k - above;
  }
  __syncthreads();
  return total;
}

__global__ __launch_bounds__(kSelThreads) void topk_collect_kernel(Geo g, uint32_t *hist, TopkShared sh, TopkLists lists, TopkVector vec) {
  __shared__ uint32_t scan[kSelThreads / 64], sel[2], sure[kRangeGroups], near, at, ends[2];
  const GroupRange w(g, lists);
  if (w.q0 >= w.q1) return;
  uint32_t *bins = hist + (uint64_t)w.p * kTopkHistWords;
  const uint32_t k = (uint32_t)k_of_device(g, w.p);
  if (threadIdx.x < kRangeGroups) sure[threadIdx.x] = 0;
  if (threadIdx.x == 0) { near = 0; ends[0] = 0; ends[1] = 0; }
  if (near_bin_of_k(bins, k, scan, sel) < k) return;   // (ties beside the lists, or the long form: the next kernel finds out by itself)
  const uint32_t bin = sel[0], slot = __builtin_amdgcn_readfirstlane(threadIdx.x >> 7), q = w.q0 + slot;
  const uint32_t G = __builtin_amdgcn_readfirstlane((uint32_t)sh.pair(w.p)[0]);
  const auto mine = entries_of_group<true>(g, lists, w, q, G, vec);
  uint32_t above = 0, inside = 0, most = 0, least = 0;   // (of the keys inside, one more than the highest; not the lowest)
  mine.each([&](uint32_t rel, uint32_t, uint32_t) {
    const uint32_t b = near_bin(rel);
    above += b > bin;
    inside += b == bin;
    if (b == bin) {
      most = most > rel + 1 ? most : rel + 1;
      least = least > ~rel ? least : ~rel;
    }
  });
  if (inside) {   // (few threads' business, unless keys are equal)
    atomicMax(&ends[0], most);
    atomicMax(&ends[1], least);
  }
  const uint32_t both = wave_sum_u32(above | inside << 16);   // (a group has 8192 elements)
  if ((threadIdx.x & 63) == 0 && both) atomicAdd(&sure[slot], both);
  uint32_t place = inside ? atomicAdd(&near, inside) : 0u;
  __syncthreads();
  if (threadIdx.x == 0) at = near ? atomicAdd(&bins[kNearBins], near) : 0u;
  if (threadIdx.x < 2 && near) atomicMax(&bins[kNearBins + 1 + threadIdx.x], ends[threadIdx.x]);
  if (q < w.q1 && (threadIdx.x & 127) == 0) lists.count(w.p, q)[1] = sure[slot];
  __syncthreads();
  place += at;
  if (inside) {
    uint32_t *ni = lists.idx(w.p), *nv = lists.val(w.p);
    mine.each([&](uint32_t rel, uint32_t v, uint32_t j) {
      if (near_bin(rel) == bin) {
        if (place < TopkLists::kNearCap) { ni[place] = j; nv[place] = v; }
        ++place;
      }
    });
  }
}

constexpr uint32_t kRangeWords = kRangeGroups * kGroupElems / 32;   // of a workgroup's bitmap
static_assert(kRangeWords == 2 * kSelThreads, "two words of the bitmap a thread");
// The bits before every word of the bitmap, in `before`; the sum of the threads' `below`.
__device__ __forceinline__ uint32_t range_bits_before(const uint32_t *bitmap, uint16_t *before, uint32_t below, uint32_t *scan) {
  const uint32_t w0 = bitmap[2 * threadIdx.x], w1 = bitmap[2 * threadIdx.x + 1], c0 = (uint32_t)__popc(w0);
  uint32_t all, all_below;
  const uint32_t at = block_exclusive_scan<kSelThreads>(c0 + (uint32_t)__popc(w1), scan, &all);
  block_exclusive_scan<kSelThreads>(below, scan, &all_below);
  before[2 * threadIdx.x] = (uint16_t)at;
  before[2 * threadIdx.x + 1] = (uint16_t)(at + c0);
  __syncthreads();
  return all_below;
}

// Emit pass of the group-list form where ties of the key below the guess, beside the lists, make their `listed` entries up
// to k: a workgroup writes all entries of its groups, and its ties as far as they go.  false if there are not enough.
template <bool HALF>
__device__ __forceinline__ bool emit_with_ties(const Geo &g, const GroupRange &w, uint32_t k, uint32_t listed, uint32_t G, float *buf, const TopkVector &vec,
                                      uint32_t *state, const TopkLists &lists, uint8_t *payload, int zero_selected, uint32_t *bitmap,
                                      uint16_t *before, uint32_t *scan, uint32_t *sel) {
  const uint32_t need = k - listed;
  const TieCut cut = tie_cut(lists, w.p, (w.d + kGroupElems - 1) / kGroupElems, need, w.q0, scan, sel);
  if (cut.all < need) return false;
  if (w.q0 == 0 && threadIdx.x == 0) state[w.p * 8 + kStLong] = kTiesBeside;
  const uint32_t lo = w.q0 * kGroupElems, hi = w.q1 * kGroupElems < w.d ? w.q1 * kGroupElems : w.d;
  const PartValues x_of = part_values(g, w.p, buf, vec.at, vec.half);
  const uint32_t ties_to = tie_end(x_of, G - 1u, cut, lo, hi, scan, sel);
  const auto mine = entries_of_group<true>(g, lists, w, __builtin_amdgcn_readfirstlane(w.q0 + (threadIdx.x >> 7)), G, vec);
  uint32_t below = threadIdx.x == 0 ? (cut.before < need ? cut.before : need) : 0u;
  for (uint32_t b = threadIdx.x; b < w.q0; b += kSelThreads) below += lists.count(w.p, b)[0];
  bitmap[2 * threadIdx.x] = 0;
  bitmap[2 * threadIdx.x + 1] = 0;
  __syncthreads();
  auto mark = [&](uint32_t j) { atomicOr(&bitmap[(j - lo) >> 5], 1u << (j & 31u)); };
  mine.each([&](uint32_t, uint32_t, uint32_t j) { mark(j); });
  each_tie(x_of, G - 1u, lo, ties_to, [&](uint32_t j, uint32_t) { mark(j); });
  __syncthreads();
  const uint32_t all_below = range_bits_before(bitmap, before, below, scan);
  uint8_t *rec = payload + (uint64_t)w.p * g.stride;
  float *buf_part = zero_selected ? buf + g.part_base(w.p) : nullptr;
  auto write = [&](uint32_t j, uint32_t v) {
    const uint32_t o = j - lo, word = o >> 5;
    const uint32_t pos = all_below + before[word] + (uint32_t)__popc(bitmap[word] & ((1u << (o & 31u)) - 1u));
    topk_write_entry<HALF>(g, rec, pos, j, __uint_as_float(v), buf_part, zero_selected);
  };
  each_tie(x_of, G - 1u, lo, ties_to, write);
  __syncthreads();   // (a listed element's slot of the buffer, once zeroed, could pass for a tie)
  mine.each([&](uint32_t, uint32_t v, uint32_t j) { write(j, v); });
  return true;
}

// Emit pass of the group-list form.  The form in all, against the long form that these k took before (worker
// calls): 20 M f16 elements, k = 1 %, 77 against 122 us (load 44, bins 5, collect 6.5, emit 20); 100 M, k =
// 3 %, 328 against 566; 0.3 M 31 against 36.  (One workgroup a partition over lists that long, as in the
// select pass, took 70 to 140 us by itself.)
template <bool HALF>
__global__ __launch_bounds__(kSelThreads) void topk_group_emit_kernel(Geo g, float *buf, TopkVector vec, uint32_t *state,
                                                                      const uint32_t *hist, TopkShared sh, TopkLists lists, uint8_t *payload,
                                                                      int zero_selected) {
  __shared__ __align__(16) uint32_t h[2048];
  __shared__ uint32_t bitmap[kRangeWords];
  __shared__ uint16_t before[kRangeWords];
  __shared__ uint32_t scan[kSelThreads / 64], sel[2];
  static_assert(kBins1 <= 2048, "h holds the bins of a level");
  const GroupRange w(g, lists);
  if (w.q0 >= w.q1) return;
  const uint32_t *bins = hist + (uint64_t)w.p * kTopkHistWords;
  const uint32_t k = (uint32_t)k_of_device(g, w.p);
  if (w.q0 == 0 && threadIdx.x == 0) topk_write_header<HALF>(g, w.p, payload);
  uint32_t near = __builtin_amdgcn_readfirstlane(bins[kNearBins]);
  const uint32_t most = __builtin_amdgcn_readfirstlane(bins[kNearBins + 1]), least = __builtin_amdgcn_readfirstlane(bins[kNearBins + 2]);
  const uint32_t listed = near_bin_of_k(bins, k, scan, sel), bin = sel[0];
  uint32_t rem = sel[1];
  const uint64_t pair = sh.pair(w.p)[0];
  const uint32_t G = __builtin_amdgcn_readfirstlane((uint32_t)pair);
  const bool beside = listed < k && __builtin_amdgcn_readfirstlane((uint32_t)(pair >> 32)) != 0;   // ties of the key below the guess are kept
  // many entries in the threshold's bin (more, maybe, than their list has room for), but all of one key: that is the
  // threshold, and its ties are dealt with as those beside a list
  const bool one_key = listed >= k && near > kFewNear && most - 1u == ~least;
  if (listed < k || (near > TopkLists::kNearCap && !one_key)) {
    if (beside && emit_with_ties<HALF>(g, w, k, listed, G, buf, vec, state, lists, payload, zero_selected, bitmap, before, scan, sel)) return;
    if (w.q0 != 0) return;
    if (threadIdx.x == 0) state[w.p * 8 + kStLong] = kLongForm;
    topk_alone<HALF>(g, w.p, k, buf, vec.at, vec.half, payload, zero_selected, h, scan, sel);
    return;
  }
  TieCut cut{};
  if (one_key) {
    cut = tie_cut(lists, w.p, (w.d + kGroupElems - 1) / kGroupElems, rem, w.q0, scan, sel, 16);
    near = 0;
  }
  EntriesOf<kSelThreads, true> near_ones{lists.idx(w.p), lists.val(w.p), threadIdx.x, near, G};
  near_ones.load_first();
  auto each_near = [&](auto visit) { near_ones.each([&](uint32_t rel, uint32_t, uint32_t j) { visit(rel, j); }); };
  const uint32_t q = __builtin_amdgcn_readfirstlane(w.q0 + (threadIdx.x >> 7));
  const auto mine = entries_of_group<true>(g, lists, w, q, G, vec);
  // the threshold inside the bin (less than 2^26 keys: 6 + 10 + 10 bits), then, among ties, the index of the last
  // one kept
  uint32_t R = 0, last = 0xffffffffu;
  if (!one_key) {
    const uint32_t start = near_start(bin), width = near_start(bin + 1) - start;
    uint32_t ties = 0;
#pragma unroll 1
    for (int shift = width > 1u << 20 ? 20 : width > 1u << 10 ? 10 : 0; shift >= 0; shift -= 10) {
      const uint32_t prefix = R;
      __syncthreads();
      h[threadIdx.x] = 0;
      __syncthreads();
      each_near([&](uint32_t rel, uint32_t) {
        if (((rel - start) >> shift >> 10) == prefix) atomicAdd(&h[((rel - start) >> shift) & 1023u], 1u);
      });
      __syncthreads();
      pick_bin<1024, 10, kSelThreads>(h, rem, prefix, scan, sel);
      R = sel[0];
      rem = sel[1];
      ties = h[sel[0] & 1023u];
    }
    R += start;
    if (ties != rem) {   // (uniform) the rem-th of the ties in index order (indices below 2^28: 10 + 10 + 8 bits)
      uint32_t prefix = 0;
      rem = ties - rem + 1;   // (pick_bin counts from the largest down)
#pragma unroll 1
      for (int level = 0; level < 3; ++level) {
        const int hi_shift = level == 0 ? 28 : level == 1 ? 18 : 8, lo_shift = level == 0 ? 18 : level == 1 ? 8 : 0;
        __syncthreads();
        h[threadIdx.x] = 0;
        __syncthreads();
        each_near([&](uint32_t rel, uint32_t j) {
          if (rel == R && (j >> hi_shift) == prefix) atomicAdd(&h[(j >> lo_shift) & (level == 2 ? 255u : 1023u)], 1u);
        });
        __syncthreads();
        if (level == 2) pick_bin<256, 8, kSelThreads>(h, rem, prefix, scan, sel);
        else pick_bin<1024, 10, kSelThreads>(h, rem, prefix, scan, sel);
        prefix = sel[0];
        rem = sel[1];
      }
      last = prefix;
    }
  }
  // kept entries of the groups before the workgroup's: those above the bin, and those inside it
  const uint32_t lo = w.q0 * kGroupElems;
  uint32_t below = 0;
  if (one_key) {
    const uint32_t hi = w.q1 * kGroupElems < w.d ? w.q1 * kGroupElems : w.d;
    R = most - 1u;
    // (the index after the last tie kept is 0 for no workgroup: the first one's group has some, or a later one)
    last = tie_end(part_values(g, w.p, buf, vec.at, vec.half), G + R, cut, lo, hi, scan, sel) - 1u;
    if (threadIdx.x == 0) below = cut.before < rem ? cut.before : rem;
  }
  for (uint32_t b = threadIdx.x; b < w.q0; b += kSelThreads) below += lists.count(w.p, b)[1] & 0xffffu;
  each_near([&](uint32_t rel, uint32_t j) { below += j < lo && (rel > R || (rel == R && j <= last)); });
  bitmap[2 * threadIdx.x] = 0;
  bitmap[2 * threadIdx.x + 1] = 0;
  __syncthreads();
  mine.each([&](uint32_t rel, uint32_t, uint32_t j) {
    if (rel > R || (rel == R && j <= last)) atomicOr(&bitmap[(j - lo) >> 5], 1u << (j & 31u));
  });
  __syncthreads();
  const uint32_t all_below = range_bits_before(bitmap, before, below, scan);
  uint8_t *rec = payload + (uint64_t)w.p * g.stride;
  float *buf_part = zero_selected ? buf + g.part_base(w.p) : nullptr;
  mine.each([&](uint32_t rel, uint32_t v, uint32_t j) {
    if (rel > R || (rel == R && j <= last)) {
      const uint32_t o = j - lo, word = o >> 5;
      const uint32_t pos = all_below + before[word] + (uint32_t)__popc(bitmap[word] & ((1u << (o & 31u)) - 1u));
      topk_write_entry<HALF>(g, rec, pos, j, __uint_as_float(v), buf_part, zero_selected);
    }
  });
}

// Ordered compaction of the long form.  Thread t of a tile owns 16 consecutive elements, so
// positions follow from an exclusive scan over threads, on top of the counts of the partition's
// earlier tiles (at most a few hundred numbers, summed by every workgroup for itself).  The
// workgroup of the first tile writes the record's header.
// HALF: values are sent as halves (round to nearest even) and a kept slot of the buffer keeps
// what the rounding dropped instead of 0.
template <bool HALF>
__device__ inline void topk_emit_body(const Geo &g, float *buf, const uint32_t *state, const uint32_t *tilecnt,
                                      uint8_t *payload, int zero_selected, uint32_t n_items, int gated) {
  __shared__ uint32_t scan[kThreads];
  __shared__ uint32_t before[2][kThreads / 64];
  constexpr int kPer = kTile / kThreads;
  for (uint32_t blk = blockIdx.x; blk < n_items; blk += gridDim.x) {
    const uint32_t p = blk / g.tiles_per_part;
    const uint32_t tile = blk % g.tiles_per_part;
    if (gated && !long_form(state, p)) continue;
    const uint32_t d = g.part_size(p);
    if (tile >= (uint32_t)cdiv(d, kTile)) continue;
    const uint32_t T = state[p * 8 + 6 + kStPrefix];   // the selection after level 3
    const uint32_t r = state[p * 8 + 6 + kStKRem];
    {
      const uint32_t *tc = tilecnt + 2ull * p * g.tiles_per_part;
      uint32_t a = 0, b = 0;
      for (uint32_t t = threadIdx.x; t < tile; t += kThreads) { a += tc[2 * t]; b += tc[2 * t + 1]; }
      a = wave_sum_u32(a);
      b = wave_sum_u32(b);
      if ((threadIdx.x & 63) == 0) { before[0][threadIdx.x >> 6] = a; before[1][threadIdx.x >> 6] = b; }
      __syncthreads();
    }
    uint32_t gt_before = 0, eq_before = 0;
#pragma unroll
    for (int w = 0; w < kThreads / 64; ++w) { gt_before += before[0][w]; eq_before += before[1][w]; }
    if (tile == 0 && threadIdx.x == 0) topk_write_header<HALF>(g, p, payload);
    const uint64_t base = g.part_base(p);
    const uint32_t j0 = tile * kTile + threadIdx.x * kPer;
    float v[kPer];
    uint32_t n_gt = 0, n_eq = 0;
    if (j0 + kPer <= d) {
      // the thread's 16 elements start at a multiple of 16: four 16-byte loads
      const float4 *src4 = reinterpret_cast<const float4 *>(buf + base + j0);
#pragma unroll
      for (int q = 0; q < kPer / 4; ++q) {
        const float4 f = src4[q];
        v[4 * q] = f.x; v[4 * q + 1] = f.y; v[4 * q + 2] = f.z; v[4 * q + 3] = f.w;
      }
    } else {
#pragma unroll
      for (int i = 0; i < kPer; ++i) v[i] = j0 + i < d ? buf[base + j0 + i] : 0.0f;
    }
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      uint32_t j = j0 + i;
      uint32_t key = key_of(v[i]);
      n_gt += (j < d) && key > T;
      n_eq += (j < d) && key == T;
    }
    // one scan for both counts: a tile has 4096 elements, so each fits 16 bits
    uint32_t tot;
    const uint32_t ex_both = block_exclusive_scan<kThreads>(n_gt | (n_eq << 16), scan, &tot);
    const uint32_t ex_gt = ex_both & 0xffffu, ex_eq = ex_both >> 16;
    // ties admitted before this tile / before this thread
    const uint32_t ties_tile = eq_before < r ? eq_before : r;
    uint32_t eq_rank = eq_before + ex_eq;                 // rank of this thread's first tie
    const uint32_t ties_thread = (eq_rank < r ? eq_rank : r) - ties_tile;
    uint32_t pos = gt_before + ties_tile + ex_gt + ties_thread;
    uint8_t *rec = payload + (uint64_t)p * g.stride;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      uint32_t j = j0 + i;
      if (j >= d) continue;
      uint32_t key = key_of(v[i]);
      bool take = key > T;
      if (key == T) {
        take = eq_rank < r;
        ++eq_rank;
      }
      if (take) {
        topk_write_entry<HALF>(g, rec, pos, j, v[i], buf + base, zero_selected);
        ++pos;
      }
    }
    __syncthreads();
  }
}

template <bool HALF>
__global__ __launch_bounds__(kThreads) void topk_emit_kernel(Geo g, float *buf, const uint32_t *state,
                                                             const uint32_t *tilecnt, uint8_t *payload,
                                                             int zero_selected, uint32_t n_items) {
  topk_emit_body<HALF>(g, buf, state, tilecnt, payload, zero_selected, n_items, 0);
}

// All workgroups of a grid that is resident as a whole meet here: what they wrote before is
// visible to all of them after (release fence, one arrival each on a counter, acquire fence).
// The wait is bounded like those of cluster.hpp: a workgroup that gives up sets the status word.
__device__ inline void topk_grid_barrier(uint32_t *counter, uint32_t round, uint32_t *status) {
  __threadfence();
  __syncthreads();
  if (threadIdx.x == 0) {
    atomicAdd(counter, 1u);
    const uint32_t target = round * gridDim.x;
    int spins = 0;
    while (__hip_atomic_load(counter, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) {
      if (++spins > kSpinLimit) {
        atomicOr(status, 1u);
        break;
      }
      __builtin_amdgcn_s_sleep(16);
    }
  }
  __syncthreads();
  __threadfence();
}

// The long form behind the short-list form for partitions that are too large for one workgroup, as one
// launch: returns at once unless some partition was left to it (the usual case: one launch and one
// read instead of five of each), else runs the five passes for those partitions, with the whole
// grid meeting in between.
// The grid is resident as a whole (the host sizes it by occupancy).  `counter`: zero at launch.
template <bool HALF>
__global__ __launch_bounds__(kThreads) void topk_long_form_kernel(Geo g, float *buf, uint32_t *hist, uint32_t *state,
                                                                  uint32_t *tilecnt, uint8_t *payload, int zero_selected,
                                                                  uint32_t n2, uint32_t n3, uint32_t nc, uint32_t ne,
                                                                  uint32_t *counter, uint32_t *status) {
  __shared__ uint32_t any;
  if (threadIdx.x == 0) any = 0;
  __syncthreads();
  for (uint32_t p = threadIdx.x; p < g.P; p += kThreads)
    if (state[p * 8 + kStLong] == kLongForm) any = 1;
  __syncthreads();
  if (!any) return;   // (the same answer in every workgroup: the flags were written by the kernel before)
  topk_hist_body<1>(g, buf, hist, state, n3, 1);   // (groups of one tile, as level 3)
  topk_grid_barrier(counter, 1, status);
  topk_hist_body<2>(g, buf, hist, state, n2, 1);
  topk_grid_barrier(counter, 2, status);
  topk_hist_body<3>(g, buf, hist, state, n3, 1);
  topk_grid_barrier(counter, 3, status);
  topk_count_body(g, buf, hist, state, tilecnt, nc, 1);
  topk_grid_barrier(counter, 4, status);
  topk_emit_body<HALF>(g, buf, state, tilecnt, payload, zero_selected, ne, 1);
}

// With tiles of 1 << tile_shift elements, T of them to a full partition:
// table[p * (T + 1) + tile] = the first entry of partition p's record that lies in tile `tile`
// or after it; entry T = the number of entries.
hipError_t topk_tile_starts(const Geo &g, const uint8_t *payload, bool half, uint32_t *table, uint32_t tile_shift,
                            hipStream_t stream) {
  TopkMsgs m{};
  m.msgs.ptr[0] = payload;
  m.msgs.n = 1;
  m.groups_per_part = (uint32_t)cdiv(g.part_elems, 1ull << tile_shift);
  m.k_cap = g.k_cap;
  m.stride = g.stride;
  m.half = half ? 1 : 0;
  m.group_shift = tile_shift;
  topk_starts_kernel<<<dim3((uint32_t)cdiv(g.k_cap + 1, kThreads), g.P, 1), kThreads, 0, stream>>>(g, m, table);
  return hipGetLastError();
}

hipError_t topk_encode(const Geo &g, const bpc_params_t &prm, const bpc_params_t *, const Source &src,
                       uint8_t *payload, const Workspace &ws, hipStream_t stream) {
  uint32_t *hist = ws.at<uint32_t>(ws.lay.hist);
  uint32_t *state = ws.at<uint32_t>(ws.lay.state);
  uint32_t *tilecnt = ws.at<uint32_t>(ws.lay.tilecnt);
  float *dense = ws.at<float>(ws.lay.dense);
  const bool half = prm.kind == BPC_TOPK16;
  const int zero_selected = src.residual != nullptr;
  TopkLists lists{ws.at<uint32_t>(ws.lay.cand), g.P, nullptr, tilecnt, (uint32_t)cdiv(g.tiles_per_part, kTpgLoad)};
  // behind the short-list form of large partitions stands the long form as one resident kernel: its grid
  // comes from the occupancy query
  const void *long_fn = half ? reinterpret_cast<const void *>(&topk_long_form_kernel<true>)
                             : reinterpret_cast<const void *>(&topk_long_form_kernel<false>);
  static PerDevice cache[2];
  const uint32_t most = g.part_size(0);   // elements of the largest partition
  const bool gated = most > kAloneElems;
  const int capacity = gated ? cache[half].get([&] { return cluster_capacity(long_fn, kThreads, 0); }) : 0;
  // the short-list form wants a list that its sample is unlikely to make too long, and partitions of up to 8 M
  // elements (beyond, its few workgroups a partition take longer than the passes of the long form: one
  // partition of 64 M elements 1590 against 440 us); the group-list form wants the dense workspace and groups that
  // are not listed to a large part
  const bool fits = g.k_cap <= kTopkListCap / 2 && topk_list_fits(k_rule(g.k_ratio, most), most);
  const bool group_lists = !fits && g.k_cap <= kMostListed && g.part_elems >= 16ull * g.k_cap && !gated && (src.residual || src.grad);
  const bool short_list = group_lists || (fits && (!gated || (most <= kMostOfList && capacity > 0)));
  if (group_lists) lists.dense = reinterpret_cast<uint32_t *>(dense);
  // the vector being compressed ends up in the residual buffer (error feedback) or the workspace, or is
  // the gradient as it is
  float *buf = src.residual ? src.residual : src.grad && short_list && !gated ? nullptr : dense;
  const uint32_t load_grid = group_count(g, kTpgLoad);
  TopkShared sh{ws.at<uint64_t>(ws.lay.samp), nullptr, 0, ws.status(), state, !group_lists};
  sh.lengths = reinterpret_cast<uint32_t *>(reinterpret_cast<uint8_t *>(sh.pairs) + TopkShared::pairs_bytes(g.P));
  hipError_t e = hipSuccess;
  if (short_list) {
    // under capture every replay would carry the same tag: the guesses are cleared in front
    const bool captured = launch_tag(stream, &sh.tag);
    if (captured) {
      e = fill_zero(sh.pairs, 32ull * g.P, stream);
      if (e == hipSuccess) e = fill_zero(sh.status, 8, stream);
    }
    if (e == hipSuccess && gated) e = fill_zero(hist, ws.lay.guess - ws.lay.hist, stream);   // (and the state words)
  } else {
    e = fill_zero(hist, ws.lay.guess - ws.lay.hist, stream);
    if (e == hipSuccess) e = fill_zero(sh.status, 4, stream);
  }
  if (e != hipSuccess) return e;
  auto load = [&](auto s) {
    using Load = decltype(s);
    if (short_list) topk_load_kernel<Load, true><<<load_grid + g.P, kLoadThreads, 0, stream>>>(g, s, buf, hist, state, sh, lists);
    else topk_load_kernel<Load, false><<<load_grid, kLoadThreads, 0, stream>>>(g, s, buf, hist, state, sh, lists);
  };
  if (src.grad) {
    if (src.dtype == BPC_F16) load(GradSource<__half>{(const __half *)src.grad, src.residual});
    else load(GradSource<float>{(const float *)src.grad, src.residual});
  } else {
    // server: Delta straight from the n messages (they are taken to have the format of `prm`)
    uint32_t *starts = ws.at<uint32_t>(ws.lay.starts);
    const TopkMsgs m{src.msgs, src.residual, starts, (uint32_t)cdiv(g.tiles_per_part, kTpgLoad), g.k_cap, g.stride, half ? 1 : 0, 13};
    const PrepRows rows = prep_rows((uint32_t)src.msgs.n, g.k_cap, g.part_size(0), short_list);
    float *sums = reinterpret_cast<float *>(lists.base);
    topk_server_prep_kernel<<<dim3(g.P, rows.sums + rows.starts), rows.threads, rows.threads * 32, stream>>>(g, m, rows, starts, sums);
    load(TopkMsgsGroupSource{m, sums});
  }
  if (group_lists) {
    const uint32_t grid = g.P * (uint32_t)cdiv(lists.groups, kRangeGroups);
    const TopkVector vec{buf ? buf : src.grad, !buf && src.dtype == BPC_F16};
    topk_bins_kernel<<<grid, kSelThreads, 0, stream>>>(g, hist, sh, lists, vec);
    topk_collect_kernel<<<grid, kSelThreads, 0, stream>>>(g, hist, sh, lists, vec);
    if (half) topk_group_emit_kernel<true><<<grid, kSelThreads, 0, stream>>>(g, buf, vec, state, hist, sh, lists, payload, zero_selected);
    else topk_group_emit_kernel<false><<<grid, kSelThreads, 0, stream>>>(g, buf, vec, state, hist, sh, lists, payload, zero_selected);
    return hipGetLastError();
  }
  if (short_list) {
    // (as many workgroups as one round of them over the compute units takes)
    const uint32_t of_xcd = (uint32_t)cdiv(g.P, kXcds);
    uint32_t shares = 1;
    while (shares < kMostShares && 2 * shares * of_xcd <= kCusOfXcd) shares *= 2;
    const uint32_t least = (uint32_t)cdiv(most, 32ull * kShareWords);
    if (shares < least) shares = least;
    const ShareRanges ranges{(uint32_t)cdiv(cdiv(most, shares), 32) * 32, (uint32_t)cdiv(cdiv(most, kGroupElems), shares) * kGroupElems};
    if (half) topk_list_select_kernel<true><<<of_xcd * shares * kXcds, kSelThreads, 0, stream>>>(g, buf, src.grad, src.dtype == BPC_F16, state, sh, lists, payload, zero_selected, shares, ranges);
    else topk_list_select_kernel<false><<<of_xcd * shares * kXcds, kSelThreads, 0, stream>>>(g, buf, src.grad, src.dtype == BPC_F16, state, sh, lists, payload, zero_selected, shares, ranges);
    if (!gated) return hipGetLastError();
  }
  const uint32_t n2 = group_count(g, kTpgHist2), n3 = group_count(g, kTpgHist3), nc = group_count(g, kTpgCount);
  const uint32_t ne = g.P * g.tiles_per_part;
  if (short_list) {
    // the long form for the partitions the short list could not take: one resident kernel
    const uint32_t grid = (uint32_t)capacity < kGatedGrid ? (uint32_t)capacity : kGatedGrid;
    uint32_t *counter = state + 8ull * g.P;
    uint32_t *status = ws.status();
    e = cluster_launch_begin(stream);
    if (e != hipSuccess) return e;
    if (half) topk_long_form_kernel<true><<<grid, kThreads, 0, stream>>>(g, buf, hist, state, tilecnt, payload, zero_selected, n2, n3, nc, ne, counter, status);
    else topk_long_form_kernel<false><<<grid, kThreads, 0, stream>>>(g, buf, hist, state, tilecnt, payload, zero_selected, n2, n3, nc, ne, counter, status);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    return cluster_launch_end(stream);
  }
  topk_hist_kernel<2><<<n2, kThreads, 0, stream>>>(g, buf, hist, state, n2);
  topk_hist_kernel<3><<<n3, kThreads, 0, stream>>>(g, buf, hist, state, n3);
  topk_count_kernel<<<nc, kThreads, 0, stream>>>(g, buf, hist, state, tilecnt, nc);
  if (half) topk_emit_kernel<true><<<ne, kThreads, 0, stream>>>(g, buf, state, tilecnt, payload, zero_selected, ne);
  else topk_emit_kernel<false><<<ne, kThreads, 0, stream>>>(g, buf, state, tilecnt, payload, zero_selected, ne);
  return hipGetLastError();
}

}  // namespace bpc
