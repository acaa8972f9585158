// Kernel wrappers and launcher shared by the single-pass (cluster) kernels.
#pragma once
#include "cluster.hpp"
#include "kernels.hpp"
#include <type_traits>

namespace bpc {

// Waves per SIMD the kernel is compiled for: 4 (at most 128 vector registers a lane) unless
// the operator asks for more with kWavesPerSimd.
template <class Op, class = void>
struct waves_per_simd { static constexpr int value = 4; };
template <class Op>
struct waves_per_simd<Op, std::void_t<decltype(Op::kWavesPerSimd)>> { static constexpr int value = Op::kWavesPerSimd; };

// TAGGED: the launch has a tag and no preset in front of it (cluster.hpp); without it `tag` is the
// constant 0 and none of that is compiled in.
template <class Op, bool TAGGED>
__global__ __launch_bounds__(Op::kThreads, waves_per_simd<Op>::value) void cluster_kernel(const Op op, double *slots, uint32_t *status, uint32_t *tickets, uint64_t launch_tag) {
  __shared__ __attribute__((aligned(16))) float table[Op::kTableFloats];
  const uint64_t tag = TAGGED ? launch_tag : 0;
  status_open(status, tag);
  if constexpr (Op::kPersistent) cluster_run_persistent(op, table, slots, status, tag);
  else cluster_run_ticketed(op, table, slots, status, tickets, tag);
}

// Calls of up to this many tenths of a tile per workgroup of the grid go without the preset launch.
// Beyond four tiles that launch is small beside the kernel and the second word of every slot costs
// as much or more (110 M / 336 M elements, always with a tag: sign worker 195 against 188 us, dithering
// worker 705 against 632, sign server 232 against 216, dithering server 1143 against 1065); below
// it a call gains what the launch costs (f16, with a tag against without: sign worker 5.1 against 7.1 us
// at 1 M elements, 10.0 against 10.6 at 4 M, 29.4 against 30.9 at 16.8 M; dithering server of 8 workers
// on 12 M f32 elements 1.04 times as fast).  Servers of 16 workers with three workgroups a compute
// unit set their own: their tiles are the longest, and with a tag they come at a fixed stride instead of
// as workgroups become free, which loses more than the launch costs from 2.7 tiles a workgroup on
// (17 M elements: 0.93 to 0.94 times as fast, 24 M: 0.94 to 0.97; 16 M, 2.5 tiles: 1.03 to 1.05).
template <class Op, class = void>
struct tagged_tenths { static constexpr uint64_t value = 40; };
template <class Op>
struct tagged_tenths<Op, std::void_t<decltype(Op::kTaggedTenths)>> { static constexpr uint64_t value = Op::kTaggedTenths; };

template <class Op, bool TAGGED>
static int resident_workgroups() {
  static PerDevice cache;  // resident workgroups of this kernel on each device
  return cache.get([] { return cluster_capacity(reinterpret_cast<const void *>(&cluster_kernel<Op, TAGGED>), Op::kThreads); });
}

// Launches `op` over the tiles of `cg`.  *used = false (and nothing is enqueued) when the
// shape cannot take the single-pass kernel: a partition has more tiles than the device holds
// workgroups at once.
template <class Op>
static hipError_t launch_cluster(const Op &op, const ClusterGeo &cg, double *slots, uint32_t *status, uint32_t *tickets,
                                 hipStream_t stream, bool *used) {
  *used = false;
  const int capacity = resident_workgroups<Op, false>(), capacity_tagged = resident_workgroups<Op, true>();
  if (capacity <= 0) return hipSuccess;
  if (cg.tiles_per_part > (uint32_t)capacity) return hipSuccess;
  *used = true;
  const bool small = capacity_tagged > 0 && cg.tiles_per_part <= (uint32_t)capacity_tagged &&
                     10ull * cg.n_items <= tagged_tenths<Op>::value * (uint64_t)capacity_tagged;
  uint64_t tag = 0;
  hipError_t e = cluster_launch_begin(stream, small ? &tag : nullptr);
  if (e != hipSuccess) return e;
  // the whole grid is resident at once
  const uint32_t most = (uint32_t)(tag ? capacity_tagged : capacity);
  const uint32_t grid = cg.n_items > most ? most : cg.n_items;
  if (tag) {
    cluster_kernel<Op, true><<<grid, Op::kThreads, 0, stream>>>(op, slots, status, tickets, tag);
  } else {
    slots_reset_kernel<<<(uint32_t)cdiv(cg.n_items, 256), 256, 0, stream>>>(slots, cg.n_items, status, tickets);
    cluster_kernel<Op, false><<<grid, Op::kThreads, 0, stream>>>(op, slots, status, tickets, 0);
  }
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  return cluster_launch_end(stream);
}

}  // namespace bpc
