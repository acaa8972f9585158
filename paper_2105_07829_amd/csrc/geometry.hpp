// Host+device description of how a flat gradient is cut into partitions and
// how a call's device workspace is carved up.  Record format: include/bpc.h.
#pragma once
#include <stdint.h>
#include <stddef.h>
#include <math.h>
#include "../../include/bpc.h"

#if defined(__HIPCC__)
#define BPC_HD __host__ __device__
#else
#define BPC_HD
#endif

namespace bpc {

constexpr int kMaxWorkers = 64;      // most worker messages one aggregate call accepts
constexpr int kTile = 4096;          // elements one workgroup handles in the streaming kernels
constexpr int kThreads = 256;        // workgroup size of the streaming kernels
constexpr uint32_t kPartUnit = 1024; // partitions hold a multiple of this many elements
constexpr int kSThreads = 256;       // workgroup size of the server-side kernels when the number of workers is not one they are compiled for
constexpr int kWTile = 8192;         // tile of the worker-side single-pass kernels (512 threads x 16 elements)
constexpr int kSTile = 8192;         // tile of the server-side single-pass kernels and of single-pass LANS
constexpr uint32_t kHeaderBytes = 16;
constexpr int kTicketClasses = 16;   // counters the ticketed single-pass kernels draw their tiles from (workgroup w uses counter w % 16)
constexpr int kTicketStride = 4096;  // bytes between two of them, so that they lie in different memory channels
constexpr int kMaxRuns = 64;         // most runs of partitions of one class (compressed / carried as they are) a call accepts
constexpr uint32_t kTopkListCap = 32768;  // entries of a partition's top-k short list
constexpr uint32_t kTopkHistWords = 2048 + 1024 + 1024;  // top-k radix histograms of a partition

BPC_HD inline uint64_t ru4(uint64_t x) { return (x + 3) / 4 * 4; }
BPC_HD inline uint64_t cdiv(uint64_t a, uint64_t b) { return (a + b - 1) / b; }

// Everything a kernel needs to find partition p and its record.
// k = max(1, floor(ratio*d)), never above d; exact in f64 for d < 2^31.
BPC_HD inline uint64_t k_rule(double ratio, uint64_t d) {
  if (d == 0) return 0;
  uint64_t k = (uint64_t)floor(ratio * (double)d);
  if (k < 1) k = 1;
  if (k > d) k = d;
  return k;
}

struct Geo {
  uint64_t D;            // elements of the flat gradient
  uint64_t part_elems;   // elements of a full partition
  uint32_t P;            // number of partitions
  uint32_t tiles_per_part;  // kTile-sized tiles of a full partition
  uint32_t n_tiles;      // tiles over all partitions (last partition may have fewer)
  uint32_t k_cap;        // kept elements of a full partition (TOPK/RANDK), else 0
  uint64_t stride;       // bytes between records
  double k_ratio;
  uint32_t part0;        // partition number of partition 0 of this view (non-zero when a call
                         // hands the tail of a gradient to a different set of kernels)

  BPC_HD uint64_t part_base(uint32_t p) const { return (uint64_t)p * part_elems; }
  BPC_HD uint32_t part_size(uint32_t p) const {
    uint64_t rest = D - (uint64_t)p * part_elems;
    return (uint32_t)(rest < part_elems ? rest : part_elems);
  }
};

inline bool params_valid(const bpc_params_t *p) {
  if (!p) return false;
  // (2^28 elements at most: byte offsets inside a partition's record and arrays fit 32 bits everywhere)
  if (p->part_elems == 0 || p->part_elems % kPartUnit != 0 || p->part_elems > (1ull << 28)) return false;
  switch (p->kind) {
    case BPC_IDENTITY: case BPC_SIGN: case BPC_FP16: return true;
    case BPC_TOPK: case BPC_TOPK16: case BPC_RANDK: return p->k_ratio > 0.0 && p->k_ratio <= 1.0;
    case BPC_DITHER:
      return p->levels >= 1 && p->levels <= 63 && (p->norm == BPC_NORM_L2 || p->norm == BPC_NORM_LINF);
    case BPC_NATDITHER:
      return p->levels >= 1 && p->levels <= 7 && (p->norm == BPC_NORM_L2 || p->norm == BPC_NORM_LINF);
    default: return false;
  }
}

// A record has room for part_elems elements, also that of a shorter last partition.  That is whole
// rows of kPartUnit elements but not always whole tiles: kernels that read a message a row at a
// time, 4 elements a thread, read the record's last row again in place of the rows of a tile past
// its end (what they make of those is not stored).  `row0`: the row's first element in the partition.
BPC_HD inline uint32_t row_in_record(uint32_t row0, uint64_t part_elems) {
  const uint32_t last = (uint32_t)part_elems - kPartUnit;
  return row0 < last ? row0 : last;
}

// The sample of a top-k partition of d elements: up to kSampleChunks whole chunks of eight consecutive
// elements, one of every 1 << shift (up to a quarter of them in small partitions, of which calls have many: servers
// of 4 workers on 16 M elements, partitions of 8192 / 65536, 171 -> 129 and 69 -> 56 us).
constexpr uint32_t kSampleChunks = 1024, kSmallPartition = 65536;
BPC_HD inline uint32_t sample_shift(uint32_t d) {
  uint32_t shift = 0;
  while (((d / 8) >> shift) > (d <= kSmallPartition ? kSampleChunks / 4 : kSampleChunks)) ++shift;
  return shift;
}
BPC_HD inline uint32_t sample_chunks(uint32_t d) { return (d / 8) >> sample_shift(d); }
// The rank in a sample of m elements of a partition of d from which elements go to the list: the expected rank of
// the partition's k-th largest, four standard deviations of a count of twice that size further down (neighbours
// are not independent), and a little more, but no further than half way (in square roots, on which scale counts
// spread alike) to the expected rank of the first element that a list of limited room has none for.
BPC_HD inline uint32_t sample_rank(uint64_t k, uint32_t m, uint32_t d, bool limited) {
  const double expect = (double)k * (double)m / (double)d, room = (double)kTopkListCap * (double)m / (double)d;
  const double enough = expect + 4.0 * sqrt(2.0 * expect) + 3.0, way = 0.5 * (sqrt(expect) + sqrt(room));
  return (uint32_t)(!limited || enough < way * way || room <= expect ? enough : way * way + 0.5);
}
// Whether a list can be expected to hold the k largest of a partition of d elements and have room for what it
// gets: that half way is 2.75 standard deviations of an independent count.  Where it is fewer, up to one list in
// three failed, and its partition then takes 0.8 to 1.6 ms (k = 0.1 %, one partition of 8 M / 12 M elements,
// worker: 62 or 880 / 858 us).
inline bool topk_list_fits(uint64_t k, uint32_t d) {
  const uint32_t m = 8 * sample_chunks(d);
  if (!m || sample_rank(k, m, d, true) >= m) return d <= kTopkListCap;   // the whole partition is listed
  return sqrt((double)kTopkListCap * m / d) - sqrt((double)k * m / d) >= 2.75;
}

// How bpc_decompress() lays a random-k message out: drawn again for every stretch of 4096 or of 32768 elements, or
// by a zero fill and a scatter.  The draws of a stretch are those of its partition, so a call makes (stretches *
// k) of them where the scatter makes k: what each costs beyond writing the output, in us, fitted to calls of
// 0.3 M to 256 M elements.  Small / large / scatter, whole calls, k = 1 % unless stated: 16 M elements in partitions of
// 1024 18 / 157 / 23 us, of 64 K 14 / 17 / 24, of 1 M 27 / 19 / 24, of 4 M 94 / 27 / 24, of 1 M with k = 0.1 %
// 15 / 17 / 17, with k = 10 % 202 / 46 / 96; 1 M with k = 100 % 275 / 135 / 59; 256 M, one partition, - / 11 220 / 462.
constexpr uint32_t kSmallDrawTile = 4096, kLargeDrawTile = 32768;
constexpr int kSmallDrawThreads = 256, kLargeDrawThreads = 1024;
enum DrawForm { kDrawsSmall, kDrawsLarge, kDrawsScattered };
inline DrawForm randk_decode_form(uint64_t P, uint64_t d, uint64_t k) {   // P partitions of d elements at most
  const double draws = (double)P * (double)k;
  // the device's rate of draws (of many small workgroups, beside their stores), or, with few workgroups, a workgroup's
  // rounds of four draws a thread one after the other
  const double small = fmax(0.6e-6 * draws * (double)cdiv(d, kSmallDrawTile) - 0.5e-6 * (double)P * (double)d,
                            0.26 * (double)cdiv(k, 4 * kSmallDrawThreads));
  const double large = 2.5 + fmax(0.5e-6 * draws * (double)cdiv(d, kLargeDrawTile), 0.5 * (double)cdiv(k, 4 * kLargeDrawThreads));
  const double scatter = 2.3 + 48e-6 * draws;
  if (small <= large && small <= scatter) return kDrawsSmall;
  return large <= scatter ? kDrawsLarge : kDrawsScattered;
}

// What the rows of workgroups (the second grid dimension) of the kernel in front of a top-k server's load pass
// do for a partition.  Rows of sums: `slots` messages side by side, a thread searching one message for one of
// `chunks` sampled chunks.  Rows of starts: eight entries a thread (and the end) of one message, or all of
// `messages` short ones; the launch has `starts` rows of them, of which each takes every starts-th of the
// `roles`.  (A grid has at most 65535 rows.)  Long messages take larger workgroups (16 messages of 31 K
// entries, 60 M elements: 434 us a call with 1024 threads, 444 with 256; 8 messages of 10 K, 26 M: a step 778, 770).
constexpr uint32_t kPrepThreads = 256, kPrepMostThreads = 1024, kPrepSlots = 16, kPrepMostStarts = 32768;
struct PrepRows { uint32_t threads, slots, chunks, chunk_bits, sums, messages, pieces, roles, starts; };
// n messages of partitions of `d` elements at most and k_cap entries.
BPC_HD inline PrepRows prep_rows(uint32_t n, uint32_t k_cap, uint32_t d, bool guesses) {
  PrepRows r;
  r.threads = k_cap > kTopkListCap / 2 ? kPrepMostThreads : kPrepThreads;
  r.slots = r.threads == kPrepThreads ? 1 : kPrepSlots;   // (long messages: rows of as few chunks as there can be)
  while (r.slots < n && r.slots < kPrepSlots) r.slots *= 2;
  r.chunks = r.threads / r.slots;   // (a power of two)
  r.chunk_bits = 0;
  while (1u << r.chunk_bits < r.chunks) ++r.chunk_bits;
  r.sums = guesses ? (uint32_t)cdiv(sample_chunks(d), r.chunks) : 0u;
  r.pieces = (uint32_t)cdiv((uint64_t)k_cap + 1, 8 * r.threads);
  r.messages = r.pieces == 1 ? 8 * r.threads / (k_cap + 1) : 1u;
  r.roles = r.pieces == 1 ? (uint32_t)cdiv(n, r.messages) : n * r.pieces;
  r.starts = r.roles < kPrepMostStarts ? r.roles : kPrepMostStarts;
  return r;
}

// Bit planes that follow the nibbles of a linear-dithering record: level bits 3, 4, 5.
BPC_HD inline uint32_t dither_planes(uint32_t levels) {
  uint32_t planes = 0;
  while ((levels >> (3 + planes)) != 0) ++planes;
  return planes;
}
// Byte offset of plane 0 in a record, and bytes from one plane to the next.
BPC_HD inline uint64_t dither_plane0(uint64_t part_elems) { return kHeaderBytes + 4 * ru4(cdiv(part_elems, 8)); }
BPC_HD inline uint64_t dither_plane_bytes(uint64_t part_elems) { return 4 * ru4(cdiv(part_elems, 32)); }

inline size_t stride_of(const bpc_params_t *p) {
  uint64_t d = p->part_elems, words = 0;
  switch (p->kind) {
    case BPC_IDENTITY: words = ru4(d); break;
    case BPC_SIGN:     words = ru4(cdiv(d, 32)); break;
    case BPC_DITHER:   words = ru4(cdiv(d, 8)) + dither_planes(p->levels) * ru4(cdiv(d, 32)); break;
    case BPC_NATDITHER: words = ru4(cdiv(d, 8)); break;
    case BPC_TOPK:     words = 2 * ru4(k_rule(p->k_ratio, d)); break;
    case BPC_TOPK16:   words = ru4(k_rule(p->k_ratio, d)) + ru4(cdiv(k_rule(p->k_ratio, d), 2)); break;
    case BPC_RANDK:    words = ru4(k_rule(p->k_ratio, d)); break;
    case BPC_FP16:     words = ru4(cdiv(d, 2)); break;
  }
  return (size_t)(kHeaderBytes + 4 * words);
}

inline Geo make_geo(const bpc_params_t *p, uint64_t D) {
  Geo g;
  g.D = D;
  g.part_elems = p->part_elems;
  g.P = (uint32_t)cdiv(D, p->part_elems);
  g.tiles_per_part = (uint32_t)cdiv(p->part_elems, kTile);
  uint64_t last = D - (uint64_t)(g.P ? g.P - 1 : 0) * p->part_elems;
  g.n_tiles = g.P ? (g.P - 1) * g.tiles_per_part + (uint32_t)cdiv(last, kTile) : 0;
  g.k_cap = (p->kind == BPC_TOPK || p->kind == BPC_TOPK16 || p->kind == BPC_RANDK) ? (uint32_t)k_rule(p->k_ratio, p->part_elems) : 0;
  g.stride = stride_of(p);
  g.k_ratio = p->k_ratio;
  g.part0 = 0;
  return g;
}

// Device workspace of one call.  Offsets in bytes from the workspace base, each
// a multiple of 256.  Regions a kind does not use have size 0.
struct WsLayout {
  size_t status;     // u32[4 * kMaxRuns], at offset 0 whatever the shape: one slot of four words for every run of
                     // partitions a call is split into (one run unless partitions bypass compression).  Word 0 of a
                     // slot is non-zero if a single-pass kernel of that run gave up waiting
  size_t tickets;    // u32 at every kTicketStride bytes, kTicketClasses of them: the ticket counters of the
                     // ticketed single-pass kernels
  size_t partials;   // double[n_tiles]: per-tile partial norms (LANS with caller-defined blocks: a word for
                     // every tile of kSTile, its first block)
  size_t dense;      // float[D]: q / Delta / decoded message when no caller buffer can hold it
  size_t hist;       // u32[P*kTopkHistWords]: top-k radix histograms (2048 + 1024 + 1024 bins)
  size_t state;      // u32[P*8 + 8]: top-k selection state; a barrier counter
  size_t guess;      // u32[P]: not used (the sizes stay what bpc_workspace_bytes() has always answered)
  size_t starts;     // u32[kMaxWorkers * P * (groups of 8192 elements per partition + 1)]: where each group's
                     // entries start in each worker's top-k message (server side)
  size_t samp;       // 16 KB a partition: the keys from which elements go to the top-k short lists, four u64 a partition, and,
                     // 4 KB apart, the lengths of the lists
  size_t cand;       // u32[P * kTopkListCap] indices, then as many value bits: top-k short lists of the partitions
  size_t tilecnt;    // u32[2*n_tiles]: per-tile (greater, equal) counts of the long form of top-k; the lengths of its group lists,
                     // and the ties beside its lists
  size_t slots;      // double[3 * tiles of kSTile]: partition-wide reductions of the single-pass kernels
                     // (one per tile, two words per tile in a launch with a tag; three for the LANS block norms;
                     // LANS with caller-defined blocks: its pairs, which go on into `norms` and beyond)
  size_t norms;      // double[3*P]: LANS block norms when blocks are the partitions
  size_t total;
};

inline WsLayout ws_layout(const bpc_params_t *p, uint64_t D) {
  Geo g = make_geo(p, D);
  WsLayout w;
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o = off; off += (bytes + 255) / 256 * 256; return o; };
  // kinds whose update reads a dense decode of the message from the workspace
  const bool topk = p->kind == BPC_TOPK || p->kind == BPC_TOPK16;
  bool sparse = topk || p->kind == BPC_RANDK || (p->kind == BPC_DITHER && dither_planes(p->levels) > 0);
  w.status = take(16 * kMaxRuns);
  w.tickets = take((size_t)kTicketClasses * kTicketStride);
  w.partials = take(sizeof(double) * (size_t)g.n_tiles);
  w.dense = take(sparse ? sizeof(float) * (size_t)D : 0);
  w.hist = take(topk ? sizeof(uint32_t) * kTopkHistWords * (size_t)g.P : 0);
  w.state = take(topk ? sizeof(uint32_t) * (8 * (size_t)g.P + 8) : 0);
  w.guess = take(topk ? sizeof(uint32_t) * (size_t)g.P : 0);
  w.starts = take(topk ? sizeof(uint32_t) * kMaxWorkers * (size_t)g.P * (cdiv(p->part_elems, 8192) + 1) : 0);
  w.samp = take(topk ? sizeof(float) * 4096 * (size_t)g.P : 0);
  w.cand = take(topk ? 8 * (size_t)kTopkListCap * (size_t)g.P : 0);
  w.tilecnt = take(topk ? sizeof(uint32_t) * 2 * (size_t)g.n_tiles : 0);
  w.slots = take(sizeof(double) * 3 * ((size_t)g.P * cdiv(g.part_elems, kSTile)));
  w.norms = take(sizeof(double) * 3 * (size_t)g.P);
  w.total = off;
  return w;
}

// Room that LANS with caller-defined blocks has from WsLayout::norms on, `tiles` = tiles of kSTile
// elements.  What its kernels need is three doubles for every (tile, block) pair, of which there are
// fewer than tiles + n_blocks: the slots region in front of `norms` holds those of the tiles, so
// three doubles a block are enough here.  (The other terms keep the sizes at what
// bpc_update_workspace_bytes() has always answered.)
inline size_t lans_blocks_room(uint64_t n_blocks, uint64_t tiles) {
  auto r256 = [](size_t bytes) { return (bytes + 255) / 256 * 256; };
  const size_t a = r256(24 * (size_t)n_blocks);
  const size_t b = r256(16 * (size_t)n_blocks) + r256(4 * (size_t)n_blocks) + r256(48 * (size_t)tiles) + r256(4 * (size_t)tiles) +
                   r256(4 * ((size_t)tiles + 1));
  return a > b ? a : b;
}

// LANS with caller-defined blocks.  The offsets lie in device memory, so nothing on the host can look
// at them: whatever they are, the kernels stay inside the pairs (block number < n_blocks, tile
// inside the gradient).  The tiles of block [lo, hi), which ends with the gradient at the latest:
// the first one and how many (0: none).
struct BlockTiles { uint64_t t0, n; };
BPC_HD inline BlockTiles block_tiles(uint64_t lo, uint64_t hi, uint64_t D) {
  hi = hi < D ? hi : D;
  BlockTiles t{lo / kSTile, 0};
  if (hi > lo) t.n = (hi - 1) / kSTile - t.t0 + 1;
  return t;
}
// A block ends inside a tile that ends at tile_end if it ends at or before this.
BPC_HD inline uint64_t tile_edge(uint64_t tile_end, uint64_t D) { return tile_end < D ? tile_end : ~0ull; }
// One step of the search for the block that holds an element, among the n blocks from *lo: of the
// first elements of the blocks *lo, *lo + stride, ... the first c are at or before it (none: the
// element lies before the first block, which is then the answer).
BPC_HD inline void narrow_blocks(uint32_t c, uint64_t stride, uint64_t *lo, uint64_t *n) {
  const uint64_t skip = c ? (uint64_t)(c - 1) * stride : 0;
  *lo += skip;
  *n = *n - skip < stride ? *n - skip : stride;
}

BPC_HD inline uint64_t k_of_device(const Geo &g, uint32_t p) { return k_rule(g.k_ratio, g.part_size(p)); }

}  // namespace bpc
