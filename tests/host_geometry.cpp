// Host entry points to the index arithmetic that the kernels share (csrc/geometry.hpp), for the
// tests that walk a kernel's accesses on the CPU.
#include "../paper_2105_07829_amd/csrc/geometry.hpp"

extern "C" {
uint32_t geo_tiles(uint64_t part_elems) { return (uint32_t)bpc::cdiv(part_elems, bpc::kTile); }
uint32_t geo_tile_elems() { return bpc::kTile; }
uint32_t geo_row_elems() { return bpc::kThreads * 4; }
uint32_t geo_row_in_record(uint32_t row0, uint64_t part_elems) { return bpc::row_in_record(row0, part_elems); }

uint32_t geo_lans_tile() { return bpc::kSTile; }
// The wave's block search: 64 bounds at a time, those past the last offset clamped to it.
int64_t geo_find_block(const uint64_t *offs, uint64_t n_blocks, uint64_t i) {
  uint64_t lo = 0, n = n_blocks;
  for (;;) {
    const uint64_t stride = (n + 63) / 64;
    uint32_t c = 0;
    for (uint64_t lane = 0; lane < 64; ++lane) {
      const uint64_t k = lo + lane * stride;
      c += lane * stride < n && offs[k < n_blocks ? k : n_blocks] <= i;
    }
    bpc::narrow_blocks(c, stride, &lo, &n);
    if (stride == 1) return (int64_t)lo;
  }
}
uint64_t geo_tile_edge(uint64_t tile_end, uint64_t D) { return bpc::tile_edge(tile_end, D); }
void geo_block_tiles(uint64_t lo, uint64_t hi, uint64_t D, uint64_t *t0, uint64_t *n) {
  const bpc::BlockTiles t = bpc::block_tiles(lo, hi, D);
  *t0 = t.t0;
  *n = t.n;
}
// Byte offset in a workspace of the selection state of a top-k call: eight words a partition, the second
// of them 1 where the partition was left to the long form, 2 where ties beside its list are kept.
uint64_t geo_topk_state(const bpc_params_t *p, uint64_t D) { return bpc::ws_layout(p, D).state; }
// The rows of workgroups in front of a top-k server's load pass: threads, slots, chunks, sums, messages, pieces, roles, starts.
void geo_prep_rows(uint32_t n, uint32_t k_cap, uint32_t d, int guesses, uint32_t out[8]) {
  const bpc::PrepRows r = bpc::prep_rows(n, k_cap, d, guesses != 0);
  const uint32_t v[8] = {r.threads, r.slots, r.chunks, r.sums, r.messages, r.pieces, r.roles, r.starts};
  for (int i = 0; i < 8; ++i) out[i] = v[i];
}
int geo_randk_decode_form(uint64_t P, uint64_t d, uint64_t k) { return (int)bpc::randk_decode_form(P, d, k); }
int geo_topk_list_fits(uint64_t k, uint32_t d) { return bpc::topk_list_fits(k, d); }
uint32_t geo_sample_rank(uint64_t k, uint32_t m, uint32_t d) { return bpc::sample_rank(k, m, d, true); }
uint32_t geo_topk_list_cap() { return bpc::kTopkListCap; }
uint32_t geo_sample_chunks(uint32_t d) { return bpc::sample_chunks(d); }
}
