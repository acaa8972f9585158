// Launchers of the HIP kernels, one group per compressor.  Every launcher only
// enqueues work on `stream` and returns the first HIP error it saw.
#pragma once
#include <hip/hip_runtime.h>
#include "geometry.hpp"

namespace bpc {

// The n worker messages of an aggregate call, passed by value in the kernel arguments.
struct WorkerMsgs {
  const uint8_t *ptr[kMaxWorkers];
  uint64_t seed[kMaxWorkers];
  uint64_t stream_id[kMaxWorkers];
  int n;
  float inv_n;
  bool shared_scale;    // every worker's params name the same scale array (norm_override): the caller's
                        // statement that the workers compressed with one common scale per partition
};

// Where the worker-side q = g + e or the server-side Delta comes from.
struct Source {
  // worker: grad (+ residual); server: msgs (+ residual)
  const void *grad;     // NULL on the server
  int dtype;            // bpc_dtype_t of grad
  float *residual;      // e (worker) or e~ (server); NULL: no error feedback
  WorkerMsgs msgs;      // used when grad == NULL
};

struct Workspace {
  uint8_t *base;
  WsLayout lay;
  uint32_t run = 0;   // which run of partitions of the call this is: selects the status slot
  template <class T> T *at(size_t off) const { return reinterpret_cast<T *>(base + off); }
  uint32_t *status() const { return reinterpret_cast<uint32_t *>(base + lay.status) + 4 * run; }
  uint32_t *tickets() const { return reinterpret_cast<uint32_t *>(base + lay.tickets); }
};

// Where the records of a payload with bypassed partitions lie: the runs of partitions of one class.
struct RecordMap {
  uint32_t n;               // runs
  uint32_t p0[kMaxRuns];    // first partition of a run
  uint64_t off[kMaxRuns];   // where its records start
  uint64_t bypass;          // bit r: run r carries its partitions as they are
  uint64_t stride, identity_stride;
  // Offset of partition p's record (p the same in every lane); *as_is: an identity record.
  __device__ uint64_t record(uint32_t p, bool *as_is) const {
    uint32_t a = 0, b = n;   // p0[a] <= p < p0[b]
    while (b - a > 1) {
      const uint32_t m = (a + b) >> 1;
      if (p0[m] <= p) a = m; else b = m;
    }
    a = __builtin_amdgcn_readfirstlane(a);
    *as_is = (bypass >> a) & 1;
    return off[a] + (uint64_t)(p - p0[a]) * (*as_is ? identity_stride : stride);
  }
};

hipError_t fill_zero(void *ptr, size_t bytes, hipStream_t stream);
// Streaming kernels with a stage's memory traffic and no arithmetic (bpc_stream_probe).
hipError_t stream_probe(int mix, const void *a, const void *b, void *c, uint64_t n, hipStream_t stream);

// C(q) and the residual update for each kind; the same entry serves worker and server.
hipError_t sign_encode(const Geo &g, const bpc_params_t &prm, const Source &src, uint8_t *payload,
                       const Workspace &ws, hipStream_t stream);
hipError_t dither_encode(const Geo &g, const bpc_params_t &prm, const Source &src, uint8_t *payload,
                         const Workspace &ws, hipStream_t stream);
hipError_t fp16_encode(const Geo &g, const bpc_params_t &prm, const Source &src, uint8_t *payload,
                       const Workspace &ws, hipStream_t stream);
// FP16 with bypassed partitions in one launch; `ws` is that of run 0.
hipError_t fp16_encode_map(const Geo &g, const RecordMap &map, const Source &src, uint8_t *payload, const Workspace &ws,
                           hipStream_t stream);
hipError_t identity_encode(const Geo &g, const bpc_params_t &prm, const Source &src, uint8_t *payload,
                           const Workspace &ws, hipStream_t stream);
hipError_t topk_encode(const Geo &g, const bpc_params_t &prm, const bpc_params_t *in_prm, const Source &src,
                       uint8_t *payload, const Workspace &ws, hipStream_t stream);
hipError_t randk_encode(const Geo &g, const bpc_params_t &prm, const bpc_params_t *in_prm, const Source &src,
                        uint8_t *payload, const Workspace &ws, hipStream_t stream);

// out[idx] += decoded random-k entries.  `out` holds the running sum.
hipError_t scatter_add_randk_shared(const Geo &g, const bpc_params_t &prm, const WorkerMsgs &msgs, float *out,
                                    hipStream_t stream);
hipError_t scatter_add_randk(const Geo &g, const bpc_params_t &prm, const uint8_t *payload, float *out,
                             hipStream_t stream);

// Single-pass (register-resident, cluster-synchronised) variants.  *used = false means the
// shape is outside what they handle and nothing was enqueued.
hipError_t sign_worker_single_pass(const Geo &g, const bpc_params_t &prm, const Source &src, uint8_t *payload,
                                   const Workspace &ws, hipStream_t stream, bool *used);

hipError_t sign_server_single_pass(const Geo &g, const bpc_params_t &prm, const Source &src, uint8_t *payload,
                                   const Workspace &ws, hipStream_t stream, bool *used);
hipError_t dither_server_single_pass(const Geo &g, const bpc_params_t &prm, const Source &src, uint8_t *payload,
                                     const Workspace &ws, hipStream_t stream, bool *used);
hipError_t dither_worker_single_pass(const Geo &g, const bpc_params_t &prm, const Source &src, uint8_t *payload,
                                     const Workspace &ws, hipStream_t stream, bool *used);

// Random-k calls in which every workgroup (`tiles` of them, of `threads` threads) makes all draws of `messages`
// messages of its partition again, instead of a launch in front that bins them: as long as that takes a
// workgroup at most 32 rounds of four draws a thread (some 0.2 us each) and the device 2^20 blocks of four
// draws (3 us) for every launch that is saved, `launches`.  Worker calls on 0.3 M / 1 M / 2 M f32 elements, k = 1 %:
// 13.4 -> 7.0 / 7.4 / 12.0 us; server calls of 8 workers on 0.3 M 23.2 -> 13.8; Adam-style updates on 0.3 M 13.3 -> 6.7.
inline bool randk_draws_again(const Geo &g, uint32_t tiles, uint32_t messages, uint32_t threads, uint32_t launches = 1) {
  const uint64_t k = k_rule(g.k_ratio, g.D < g.part_elems ? g.D : g.part_elems);   // of the largest partition
  return messages * k <= 128ull * threads && (uint64_t)tiles * messages * k <= (uint64_t)launches << 22;
}

// out = decode(payload), dense.
// Tables for the update kernel's sparse decoder (see update.hip).
constexpr uint32_t kRandkTableStride = 1025;
hipError_t topk_tile_starts(const Geo &g, const uint8_t *payload, bool half, uint32_t *table, uint32_t tile_shift,
                            hipStream_t stream);
hipError_t randk_bin_tiles(const Geo &g, const bpc_params_t &prm, const uint8_t *payload, uint2 *lists, uint32_t *table,
                           uint32_t tile_shift, hipStream_t stream);
hipError_t decode_dense(const Geo &g, const bpc_params_t &prm, const uint8_t *payload, float *out,
                        hipStream_t stream);

// Algorithm 5 update lines fused with the decode of bit-packed messages; sparse kinds are
// decoded into the workspace first.
hipError_t adaptive_update(const Geo &g, const bpc_params_t &prm, const uint8_t *payload, float *x, float *m,
                           float *v, const bpc_opt_t &opt, const Workspace &ws, hipStream_t stream);

// Adam-style update from an FP16 payload with bypassed partitions in one launch.
hipError_t adam_update_fp16_map(const Geo &g, const RecordMap &map, const uint8_t *payload, float *x, float *m, float *v,
                                const bpc_opt_t &opt, const Workspace &ws, hipStream_t stream);

}  // namespace bpc
