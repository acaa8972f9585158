// Host entry points to the index arithmetic that the kernels share (csrc/geometry.hpp), for the
// tests that walk a kernel's accesses on the CPU.
#include "../paper_2105_07829_amd/csrc/geometry.hpp"

extern "C" {
uint32_t geo_tiles(uint64_t part_elems) { return (uint32_t)bpc::cdiv(part_elems, bpc::kTile); }
uint32_t geo_tile_elems() { return bpc::kTile; }
uint32_t geo_row_elems() { return bpc::kThreads * 4; }
uint32_t geo_row_in_record(uint32_t row0, uint64_t part_elems) { return bpc::row_in_record(row0, part_elems); }
}
