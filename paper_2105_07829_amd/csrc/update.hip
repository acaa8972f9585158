// Moment and parameter update of compressed LANS (Algorithm 5, the lines after the push-pull
// call), fused with the decode of the pulled message g~ = decode(p_t).
//   ADAM : one launch, x -= lr * (r + wd*x)
//   LANS : moments + block norms (||x_b||, ||r + wd x||_b, ||c + wd x||_b, f64 sums), then
//          x -= lr * phi(||x_b||) * (beta1 (r+wd x)/||.|| + (1-beta1) (c+wd x)/||.||)
#include "cluster_launch.hpp"
#include "sources.hpp"

#include <type_traits>

namespace bpc {

struct SignDec {
  const uint8_t *payload; uint64_t stride;
  __device__ const float *dense_base() const { return nullptr; }
  static constexpr int kLdsFloats = 1;
  __device__ void begin(uint32_t, float *) const {}
  __device__ float at(const Geo &, uint32_t p, uint32_t j, const float *) const {
    const uint8_t *rec = payload + (uint64_t)p * stride;
    float s = *reinterpret_cast<const float *>(rec);
    uint32_t w = reinterpret_cast<const uint32_t *>(rec + kHeaderBytes)[j >> 5];
    return ((w >> (j & 31)) & 1u) ? -s : s;
  }
  // 4 consecutive elements from j (a multiple of 4)
  __device__ void at4(const Geo &, uint32_t p, uint32_t j, const TileBuf &, const float *, float out[4]) const {
    const uint8_t *rec = payload + (uint64_t)p * stride;
    const float s = *reinterpret_cast<const float *>(rec);
    const uint32_t nib = rec[kHeaderBytes + (j >> 3)] >> (j & 4);
#pragma unroll
    for (int c = 0; c < 4; ++c) out[c] = ((nib >> c) & 1u) ? -s : s;
  }
  // The same in two steps, for callers that request a tile ahead of its use: the record's
  // header value and the raw bits first, the values later.
  using R4 = uint32_t;
  __device__ float header(uint32_t p) const { return *reinterpret_cast<const float *>(payload + (uint64_t)p * stride); }
  __device__ void table(float, float *) const {}
  __device__ R4 load4(const Geo &, uint32_t p, uint32_t j, const TileBuf &) const {
    return (payload + (uint64_t)p * stride)[kHeaderBytes + (j >> 3)];
  }
  __device__ void decode4(R4 r, uint32_t j, float hdr, const float *, float out[4]) const {
    const uint32_t nib = r >> (j & 4);
#pragma unroll
    for (int c = 0; c < 4; ++c) out[c] = ((nib >> c) & 1u) ? -hdr : hdr;
  }
};
struct DitherDec {
  const uint8_t *payload; uint64_t stride; uint32_t levels; bool natural;
  __device__ const float *dense_base() const { return nullptr; }
  static constexpr int kLdsFloats = 16;
  __device__ void begin(uint32_t p, float *lds) const {
    if (threadIdx.x < 16) {
      float nu = *reinterpret_cast<const float *>(payload + (uint64_t)p * stride);
      float mag = dither_mag(nu, threadIdx.x & 7, levels, natural);
      lds[threadIdx.x] = (threadIdx.x & 8) ? -mag : mag;
    }
    __syncthreads();
  }
  __device__ float at(const Geo &, uint32_t p, uint32_t j, const float *lds) const {
    const uint32_t *nibs = reinterpret_cast<const uint32_t *>(payload + (uint64_t)p * stride + kHeaderBytes);
    return lds[(nibs[j >> 3] >> (4 * (j & 7))) & 15u];
  }
  __device__ void at4(const Geo &, uint32_t p, uint32_t j, const TileBuf &, const float *lds, float out[4]) const {
    const uint32_t *nibs = reinterpret_cast<const uint32_t *>(payload + (uint64_t)p * stride + kHeaderBytes);
    const uint32_t w = nibs[j >> 3] >> (4 * (j & 4));
#pragma unroll
    for (int c = 0; c < 4; ++c) out[c] = lds[(w >> (4 * c)) & 15u];
  }
  using R4 = uint32_t;
  __device__ float header(uint32_t p) const { return *reinterpret_cast<const float *>(payload + (uint64_t)p * stride); }
  // all threads; the caller synchronises before and after
  __device__ void table(float nu, float *lds) const {
    if (threadIdx.x < 16) {
      float mag = dither_mag(nu, threadIdx.x & 7, levels, natural);
      lds[threadIdx.x] = (threadIdx.x & 8) ? -mag : mag;
    }
  }
  __device__ R4 load4(const Geo &, uint32_t p, uint32_t j, const TileBuf &) const {
    return reinterpret_cast<const uint32_t *>(payload + (uint64_t)p * stride + kHeaderBytes)[j >> 3];
  }
  __device__ void decode4(R4 r, uint32_t j, float, const float *lds, float out[4]) const {
    const uint32_t w = r >> (4 * (j & 4));
#pragma unroll
    for (int c = 0; c < 4; ++c) out[c] = lds[(w >> (4 * c)) & 15u];
  }
};
// Linear dithering with bit planes (more than 7 levels).  Table index = plane bits << 4 | nibble,
// i.e. (level bits 3..5, sign, level bits 0..2); entries beyond the levels in use are never read.
struct DitherWideDec {
  const uint8_t *payload; uint64_t stride; uint32_t levels; uint64_t part_elems;
  __device__ const float *dense_base() const { return nullptr; }
  static constexpr int kLdsFloats = 128;
  __device__ float entry(float nu, uint32_t e) const {
    const uint32_t level = (e & 7u) | ((e >> 4) << 3);
    const float mag = level <= levels ? dither_mag(nu, level, levels, false) : 0.0f;
    return (e & 8u) ? -mag : mag;
  }
  __device__ void begin(uint32_t p, float *lds) const {
    if (threadIdx.x < 128) lds[threadIdx.x] = entry(*reinterpret_cast<const float *>(payload + (uint64_t)p * stride), threadIdx.x);
    __syncthreads();
  }
  // The nibbles of 4 elements and the byte of each plane that holds their bits, as loaded:
  // nothing is combined here, so a caller that requests a tile ahead of its use does not wait
  // for the loads at the request.
  struct R4 { uint32_t nib, plane[3]; };
  __device__ float header(uint32_t p) const { return *reinterpret_cast<const float *>(payload + (uint64_t)p * stride); }
  __device__ void table(float nu, float *lds) const {
    if (threadIdx.x < 128) lds[threadIdx.x] = entry(nu, threadIdx.x);
  }
  __device__ R4 load4(const Geo &, uint32_t p, uint32_t j, const TileBuf &) const {
    const uint8_t *rec = payload + (uint64_t)p * stride;
    R4 r;
    r.nib = reinterpret_cast<const uint16_t *>(rec + kHeaderBytes)[j >> 2];
    const uint32_t planes = dither_planes(levels);
    const uint8_t *plane = rec + dither_plane0(part_elems) + (j >> 3);
    r.plane[0] = plane[0];
    r.plane[1] = planes > 1 ? plane[dither_plane_bytes(part_elems)] : 0u;
    r.plane[2] = planes > 2 ? plane[2 * dither_plane_bytes(part_elems)] : 0u;
    return r;
  }
  __device__ void decode4(R4 r, uint32_t j, float, const float *lds, float out[4]) const {
    uint32_t bits[3];
#pragma unroll
    for (uint32_t t = 0; t < 3; ++t) bits[t] = (r.plane[t] >> (j & 4u)) & 15u;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const uint32_t nib = (r.nib >> (4 * c)) & 15u;
      const uint32_t hi = ((bits[0] >> c) & 1u) | (((bits[1] >> c) & 1u) << 1) | (((bits[2] >> c) & 1u) << 2);
      out[c] = lds[(hi << 4) | nib];
    }
  }
  // Load and decode in one place: the nibbles of 4 elements in bits 0..15, then 4 bits of each
  // plane in bits 16.., 20.., 24..
  __device__ void at4(const Geo &, uint32_t p, uint32_t j, const TileBuf &, const float *lds, float out[4]) const {
    const uint8_t *rec = payload + (uint64_t)p * stride;
    uint32_t r = reinterpret_cast<const uint16_t *>(rec + kHeaderBytes)[j >> 2];
    const uint32_t planes = dither_planes(levels);
    const uint8_t *plane = rec + dither_plane0(part_elems) + (j >> 3);
    for (uint32_t t = 0; t < planes; ++t)
      r |= (((uint32_t)plane[t * dither_plane_bytes(part_elems)] >> (j & 4)) & 15u) << (16 + 4 * t);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const uint32_t nib = (r >> (4 * c)) & 15u;
      const uint32_t hi = ((r >> (16 + c)) & 1u) | (((r >> (20 + c)) & 1u) << 1) | (((r >> (24 + c)) & 1u) << 2);
      out[c] = lds[(hi << 4) | nib];
    }
  }
  __device__ float at(const Geo &g, uint32_t p, uint32_t j, const float *lds) const {
    float out[4];
    at4(g, p, j & ~3u, TileBuf(nullptr, 0), lds, out);
    const uint32_t c = j & 3u;
    return c == 0 ? out[0] : c == 1 ? out[1] : c == 2 ? out[2] : out[3];
  }
};
struct IdentityDec {
  const uint8_t *payload; uint64_t stride;
  __device__ const float *dense_base() const { return nullptr; }
  static constexpr int kLdsFloats = 1;
  __device__ void begin(uint32_t, float *) const {}
  __device__ float at(const Geo &, uint32_t p, uint32_t j, const float *) const {
    return reinterpret_cast<const float *>(payload + (uint64_t)p * stride + kHeaderBytes)[j];
  }
  // (j inside a full partition, which the record is padded to)
  __device__ void at4(const Geo &, uint32_t p, uint32_t j, const TileBuf &, const float *, float out[4]) const {
    const float4 a = reinterpret_cast<const float4 *>(payload + (uint64_t)p * stride + kHeaderBytes)[j >> 2];
    out[0] = a.x; out[1] = a.y; out[2] = a.z; out[3] = a.w;
  }
  using R4 = u32x4;
  __device__ float header(uint32_t) const { return 0.0f; }
  __device__ void table(float, float *) const {}
  __device__ R4 load4(const Geo &, uint32_t p, uint32_t j, const TileBuf &) const {
    return reinterpret_cast<const u32x4 *>(payload + (uint64_t)p * stride + kHeaderBytes)[j >> 2];
  }
  __device__ void decode4(R4 r, uint32_t, float, const float *, float out[4]) const {
    out[0] = __uint_as_float(r.x); out[1] = __uint_as_float(r.y); out[2] = __uint_as_float(r.z); out[3] = __uint_as_float(r.w);
  }
};
struct Fp16Dec {
  const uint8_t *payload; uint64_t stride;
  __device__ const float *dense_base() const { return nullptr; }
  static constexpr int kLdsFloats = 1;
  __device__ void begin(uint32_t, float *) const {}
  __device__ float at(const Geo &, uint32_t p, uint32_t j, const float *) const {
    return __half2float(reinterpret_cast<const __half *>(payload + (uint64_t)p * stride + kHeaderBytes)[j]);
  }
  using R4 = u32x2;
  __device__ float header(uint32_t) const { return 0.0f; }
  __device__ void table(float, float *) const {}
  // (j inside a full partition, which the record is padded to)
  __device__ R4 load4(const Geo &, uint32_t p, uint32_t j, const TileBuf &) const {
    return reinterpret_cast<const u32x2 *>(payload + (uint64_t)p * stride + kHeaderBytes)[j >> 2];
  }
  __device__ void decode4(R4 r, uint32_t, float, const float *, float out[4]) const {
    const uint32_t lo = r.x, hi = r.y;
    const float2 a = __half22float2(*reinterpret_cast<const __half2 *>(&lo));
    const float2 b = __half22float2(*reinterpret_cast<const __half2 *>(&hi));
    out[0] = a.x; out[1] = a.y; out[2] = b.x; out[3] = b.y;
  }
  __device__ void at4(const Geo &g, uint32_t p, uint32_t j, const TileBuf &row, const float *lds, float out[4]) const {
    decode4(load4(g, p, j, row), j, 0.0f, lds, out);
  }
};
// FP16 with bypassed partitions (the Adam-style kernel only): which of the two a record is, is the
// same for a whole workgroup.
struct Fp16MapDec {
  const uint8_t *payload;
  RecordMap map;
  __device__ const float *dense_base() const { return nullptr; }
  static constexpr int kLdsFloats = 1;
  __device__ void begin(uint32_t, float *) const {}
  __device__ void at4(const Geo &g, uint32_t p, uint32_t j, const TileBuf &row, const float *lds, float out[4]) const {
    bool as_is;
    const uint8_t *rec = payload + map.record(p, &as_is);
    if (as_is) IdentityDec{rec, 0}.at4(g, 0, j, row, lds, out);
    else Fp16Dec{rec, 0}.at4(g, 0, j, row, lds, out);
  }
};
struct DenseDec {
  const float *dense;
  __device__ const float *dense_base() const { return dense; }
  static constexpr int kLdsFloats = 1;
  __device__ void begin(uint32_t, float *) const {}
  __device__ float at(const Geo &g, uint32_t p, uint32_t j, const float *) const { return dense[g.part_base(p) + j]; }
  // `row` bounds the row this thread's 4 elements belong to (the same descriptor in every
  // lane); reads past the partition's end return 0
  __device__ void at4(const Geo &, uint32_t, uint32_t, const TileBuf &row, const float *, float out[4]) const {
    const u32x4 lo = row.load16<kNonTemporal>(threadIdx.x * 16, 0);
    out[0] = __uint_as_float(lo.x); out[1] = __uint_as_float(lo.y); out[2] = __uint_as_float(lo.z); out[3] = __uint_as_float(lo.w);
  }
  using R4 = u32x4;
  __device__ float header(uint32_t) const { return 0.0f; }
  __device__ void table(float, float *) const {}
  __device__ R4 load4(const Geo &, uint32_t, uint32_t, const TileBuf &row) const { return row.load16<kNonTemporal>(threadIdx.x * 16, 0); }
  __device__ void decode4(R4 r, uint32_t, float, const float *, float out[4]) const {
    out[0] = __uint_as_float(r.x); out[1] = __uint_as_float(r.y); out[2] = __uint_as_float(r.z); out[3] = __uint_as_float(r.w);
  }
};

// Top-k and random-k messages without a dense decode: the entries of a tile of kTile elements
// are one stretch of a list (top-k: of the record itself, whose entries come by ascending
// index; random-k: of the record's draws binned per tile beforehand), found through a table of
// where each tile's stretch starts, and laid out in LDS by the workgroup that has the tile.
// OWN (small calls): no table; the workgroup searches the record (top-k) or makes all draws again (random-k).
template <int TILE, int THREADS, bool OWN = false>
struct SparseTileDec {
  const uint8_t *payload;
  uint64_t stride;
  uint32_t k_cap;
  int mode;                  // 0: top-k, f32 values; 1: top-k, half values; 2: random-k pairs
  const uint32_t *starts;    // [partition][tile .. ], `starts_stride` words a partition
  uint32_t starts_stride;
  const uint2 *pairs;        // random-k: [partition][k_cap]
  struct Draws { uint64_t seed, stream_id, D, part_elems; uint32_t part0; float value_scale; };
  Draws draws;               // random-k, OWN
  __device__ const float *dense_base() const { return nullptr; }
  static constexpr int kLdsFloats = TILE;
  __device__ void begin(uint32_t, float *) const {}
  __device__ void begin_tile(uint32_t p, uint32_t tile, float *lds) const {
    __syncthreads();   // (the tile before is done with)
    for (uint32_t q = threadIdx.x; q < TILE / 4; q += THREADS) reinterpret_cast<float4 *>(lds)[q] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    const uint8_t *rec = payload + (uint64_t)p * stride;
    uint32_t k = *reinterpret_cast<const uint32_t *>(rec);
    k = k > k_cap ? k_cap : k;
    const uint32_t lo = tile * TILE;
    uint32_t s, e;
    if constexpr (OWN) {
      __shared__ uint32_t ends[2];
      const uint32_t wave = threadIdx.x >> 6;
      if (mode != 2 && wave < 2) {
        const uint32_t at = wave_lower_bound(reinterpret_cast<const uint32_t *>(rec + kHeaderBytes), k, lo + wave * TILE);
        if ((threadIdx.x & 63) == 0) ends[wave] = at;
      }
      __syncthreads();
      if (mode == 2) {
        const uint64_t rest = draws.D - (uint64_t)p * draws.part_elems;
        const uint32_t d = (uint32_t)(rest < draws.part_elems ? rest : draws.part_elems);
        const float scale = draws.value_scale >= 0.0f ? draws.value_scale : (float)d / (float)k;
        const Philox rng(draws.seed, draws.stream_id, p + draws.part0);
        const TileBuf vb(rec + kHeaderBytes, k * 4);
        for (uint32_t t4 = threadIdx.x; 4 * t4 < k; t4 += THREADS) {
          const u32x4 v = vb.load16(t4 * 16, 0);   // (before it is known which are wanted)
          const uint32_t vs[4] = {v.x, v.y, v.z, v.w};
          uint32_t rnd[4];
          rng.block(t4, rnd);
#pragma unroll
          for (uint32_t c = 0; c < 4; ++c) {
            const uint32_t rel = (uint32_t)(((uint64_t)rnd[c] * d) >> 32) - lo;
            if (rel < (uint32_t)TILE && 4 * t4 + c < k) atomicAdd(&lds[rel], scale * __uint_as_float(vs[c]));   // an index may repeat
          }
        }
        __syncthreads();
        return;
      }
      s = ends[0];
      e = ends[1];
    } else {
      const uint32_t *tab = starts + (uint64_t)p * starts_stride;
      s = tab[tile];
      e = tab[tile + 1];
      s = s < k ? s : k;
      e = e < k ? e : k;
      __syncthreads();
    }
    if (mode == 2) {
      const uint2 *list = pairs + (uint64_t)p * k_cap;
      for (uint32_t q = s + threadIdx.x; q < e; q += THREADS) {
        const uint2 ent = list[q];
        if (ent.x - lo < (uint32_t)TILE) atomicAdd(&lds[ent.x - lo], __uint_as_float(ent.y));   // an index may repeat
      }
    } else {
      const uint32_t *idx = reinterpret_cast<const uint32_t *>(rec + kHeaderBytes);
      const uint8_t *val = rec + kHeaderBytes + 4 * ru4(k_cap);
      for (uint32_t q = s + threadIdx.x; q < e; q += THREADS) {
        const uint32_t rel = idx[q] - lo;
        const float v = mode == 1 ? __half2float(reinterpret_cast<const __half *>(val)[q]) : reinterpret_cast<const float *>(val)[q];
        if (rel < (uint32_t)TILE) lds[rel] = v;
      }
    }
    __syncthreads();
  }
  __device__ void at4(const Geo &, uint32_t, uint32_t j, const TileBuf &, const float *lds, float out[4]) const {
    const float4 f = *reinterpret_cast<const float4 *>(lds + (j & (TILE - 1)));
    out[0] = f.x; out[1] = f.y; out[2] = f.z; out[3] = f.w;
  }
  // (the forms the single-pass LANS kernel uses: nothing to request ahead, the tile is in LDS)
  using R4 = uint32_t;
  __device__ float header(uint32_t) const { return 0.0f; }
  __device__ void table(float, float *) const {}
  __device__ R4 load4(const Geo &, uint32_t, uint32_t, const TileBuf &) const { return 0u; }
  __device__ void decode4(R4, uint32_t j, float, const float *lds, float out[4]) const {
    const float4 f = *reinterpret_cast<const float4 *>(lds + (j & (TILE - 1)));
    out[0] = f.x; out[1] = f.y; out[2] = f.z; out[3] = f.w;
  }
};
template <class DEC, class = void>
struct has_begin_tile : std::false_type {};
template <class DEC>
struct has_begin_tile<DEC, std::void_t<decltype(&DEC::begin_tile)>> : std::true_type {};

constexpr uint32_t kOwnTiles = 512;   // tiles of an update call that goes without tables, at most

struct OptArgs {
  float lr, beta1, beta2, eps, wd, bc1, bc2, phi_lo, phi_hi;
  const uint64_t *block_offsets;  // device, or NULL: blocks are the partitions
  uint64_t n_blocks;
  uint32_t *status;               // the workspace's status word (cleared by kernels that have no waits)
};

// r + wd*x and c + wd*x from the updated moments.
__device__ inline void ratios(const OptArgs &o, float g, float m, float v, float x, float *u_r, float *u_c) {
  float m_hat = m / o.bc1;
  float v_hat = v / o.bc2;
  float denom = sqrtf(v_hat) + o.eps;
  float decay = o.wd * x;
  *u_r = m_hat / denom + decay;
  *u_c = g / denom + decay;
}

// The same for the single-pass LANS kernel, which is bound by its arithmetic: the bias
// corrections as factors, and the hardware's reciprocal and square root (1 ulp each) in place
// of the correctly rounded sequences.  r and c differ from the divisions above by a few ulp;
// in x that is far inside the 1e-6 the update is held to.
__device__ inline void ratios_fast(const OptArgs &o, float inv_bc1, float inv_bc2, float g, float m, float v, float x,
                                   float *u_r, float *u_c) {
  float m_hat = m * inv_bc1;
  float v_hat = v * inv_bc2;
  float inv = __builtin_amdgcn_rcpf(__builtin_amdgcn_sqrtf(v_hat) + o.eps);
  float decay = o.wd * x;
  *u_r = m_hat * inv + decay;
  *u_c = g * inv + decay;
}

__device__ inline uint32_t find_block(const uint64_t *offs, uint64_t n_blocks, uint64_t i) {
  uint64_t lo = 0, hi = n_blocks;  // offs[lo] <= i < offs[hi]
  while (hi - lo > 1) {
    uint64_t mid = (lo + hi) / 2;
    if (offs[mid] <= i) lo = mid; else hi = mid;
  }
  return (uint32_t)lo;
}

template <class DEC, bool LANS>
__global__ __launch_bounds__(kThreads) void update_moments_kernel(Geo g, DEC dec, float *x, float *m, float *v,
                                                                  OptArgs o, double *norms) {
  __shared__ float lds[DEC::kLdsFloats];
  __shared__ double red[kThreads / 64];
  if (blockIdx.x == 0 && threadIdx.x == 0) o.status[0] = 0;   // no wait in this call
  const uint32_t p = blockIdx.x / g.tiles_per_part;
  const uint32_t tile = blockIdx.x % g.tiles_per_part;
  const uint32_t d = g.part_size(p);
  dec.begin(p, lds);
  const uint64_t base = g.part_base(p);
  const float omb1 = 1.0f - o.beta1, omb2 = 1.0f - o.beta2;
  // LANS: does this whole tile lie in one block?
  uint32_t blk_first = p, blk_last = p;
  if (LANS && o.block_offsets) {
    uint32_t j_last = (tile + 1) * kTile - 1;
    j_last = j_last < d ? j_last : d - 1;
    blk_first = find_block(o.block_offsets, o.n_blocks, base + tile * kTile);
    blk_last = find_block(o.block_offsets, o.n_blocks, base + j_last);
  }
  const bool one_block = blk_first == blk_last;
  double s_x = 0.0, s_r = 0.0, s_c = 0.0;
#pragma unroll
  for (int c = 0; c < kTile / kThreads; ++c) {
    uint32_t j = tile * kTile + c * kThreads + threadIdx.x;
    if (j < d) {
      uint64_t i = base + j;
      float gj = dec.at(g, p, j, lds);
      float mj = o.beta1 * m[i] + omb1 * gj;
      float vj = o.beta2 * v[i] + omb2 * (gj * gj);
      m[i] = mj;
      v[i] = vj;
      float xj = x[i], u_r, u_c;
      ratios(o, gj, mj, vj, xj, &u_r, &u_c);
      if (!LANS) {
        x[i] = xj - o.lr * u_r;
      } else if (one_block) {
        s_x = fma((double)xj, (double)xj, s_x);
        s_r = fma((double)u_r, (double)u_r, s_r);
        s_c = fma((double)u_c, (double)u_c, s_c);
      } else {
        uint32_t b = find_block(o.block_offsets, o.n_blocks, i);
        atomicAdd(&norms[3 * (uint64_t)b + 0], (double)xj * (double)xj);
        atomicAdd(&norms[3 * (uint64_t)b + 1], (double)u_r * (double)u_r);
        atomicAdd(&norms[3 * (uint64_t)b + 2], (double)u_c * (double)u_c);
      }
    }
  }
  if (LANS && one_block) {
    double t_x = block_sum<kThreads>(s_x, red);
    double t_r = block_sum<kThreads>(s_r, red);
    double t_c = block_sum<kThreads>(s_c, red);
    if (threadIdx.x == 0) {
      atomicAdd(&norms[3 * (uint64_t)blk_first + 0], t_x);
      atomicAdd(&norms[3 * (uint64_t)blk_first + 1], t_r);
      atomicAdd(&norms[3 * (uint64_t)blk_first + 2], t_c);
    }
  }
}

// ADAM in one pass.  A thread owns 4 consecutive elements per row of 1024, so every 16-byte
// access of a wave covers whole cache lines (which is what lets the stores be non-temporal);
// all loads of a tile are requested before the first is used.  x, m and v go through buffer
// descriptors that end with the partition: reads past it return 0 and stores past it are
// dropped.  The message is read through row_in_record(): a partition need not be whole tiles.
constexpr int kURow = kThreads * 4;
static_assert(kURow == kPartUnit, "a record is whole rows");
constexpr int kURows = kTile / kURow;
template <class DEC>
__global__ __launch_bounds__(kThreads) void adam_update_kernel(Geo g, DEC dec, float *x, float *m, float *v, OptArgs o) {
  __shared__ __align__(16) float lds[DEC::kLdsFloats];
  if (blockIdx.x == 0) {   // no wait in this call
    if constexpr (std::is_same_v<DEC, Fp16MapDec>) {
      if (threadIdx.x < dec.map.n) o.status[4 * threadIdx.x] = 0;
    } else {
      if (threadIdx.x == 0) o.status[0] = 0;
    }
  }
  const uint32_t p = __builtin_amdgcn_readfirstlane(blockIdx.x / g.tiles_per_part);
  const uint32_t tile = __builtin_amdgcn_readfirstlane(blockIdx.x % g.tiles_per_part);
  const uint32_t d = g.part_size(p);
  dec.begin(p, lds);
  const uint64_t tile_base = g.part_base(p) + (uint64_t)tile * kTile;
  const uint32_t valid = d - tile * kTile < (uint32_t)kTile ? d - tile * kTile : (uint32_t)kTile;
  const float omb1 = 1.0f - o.beta1, omb2 = 1.0f - o.beta2;
  u32x4 xr[kURows], mr[kURows], vr[kURows];
  if constexpr (has_begin_tile<DEC>::value) {
    // the loads of m, v, x are requested first, so they are under way while the tile of the
    // message is laid out in LDS
#pragma unroll
    for (int u = 0; u < kURows; ++u) {
      mr[u] = row_buf(m + tile_base, valid, u * kURow, kURow).load16<kNonTemporal>(threadIdx.x * 16, 0);
      vr[u] = row_buf(v + tile_base, valid, u * kURow, kURow).load16<kNonTemporal>(threadIdx.x * 16, 0);
      xr[u] = row_buf(x + tile_base, valid, u * kURow, kURow).load16<kNonTemporal>(threadIdx.x * 16, 0);
    }
    dec.begin_tile(p, tile, lds);
  }
  float gr[kURows][4];
#pragma unroll
  for (int u = 0; u < kURows; ++u) {
    if constexpr (!has_begin_tile<DEC>::value) {
      mr[u] = row_buf(m + tile_base, valid, u * kURow, kURow).load16<kNonTemporal>(threadIdx.x * 16, 0);
      vr[u] = row_buf(v + tile_base, valid, u * kURow, kURow).load16<kNonTemporal>(threadIdx.x * 16, 0);
      xr[u] = row_buf(x + tile_base, valid, u * kURow, kURow).load16<kNonTemporal>(threadIdx.x * 16, 0);
    }
    const uint32_t j = row_in_record(tile * kTile + u * kURow, g.part_elems) + threadIdx.x * 4;
    dec.at4(g, p, j, row_buf(dec.dense_base() + tile_base, valid, u * kURow, kURow), lds, gr[u]);
  }
#pragma unroll
  for (int u = 0; u < kURows; ++u) {
    const uint32_t mi[4] = {mr[u].x, mr[u].y, mr[u].z, mr[u].w};
    const uint32_t vi[4] = {vr[u].x, vr[u].y, vr[u].z, vr[u].w};
    const uint32_t xi[4] = {xr[u].x, xr[u].y, xr[u].z, xr[u].w};
    float mo[4], vo[4], xo[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const float gj = gr[u][c];
      const float mj = o.beta1 * __uint_as_float(mi[c]) + omb1 * gj;
      const float vj = o.beta2 * __uint_as_float(vi[c]) + omb2 * (gj * gj);
      const float xj = __uint_as_float(xi[c]);
      float u_r, u_c;
      ratios(o, gj, mj, vj, xj, &u_r, &u_c);
      mo[c] = mj;
      vo[c] = vj;
      xo[c] = xj - o.lr * u_r;
    }
    row_buf(m + tile_base, valid, u * kURow, kURow).store16<kNonTemporal>(as_u32x4(mo[0], mo[1], mo[2], mo[3]), threadIdx.x * 16);
    row_buf(v + tile_base, valid, u * kURow, kURow).store16<kNonTemporal>(as_u32x4(vo[0], vo[1], vo[2], vo[3]), threadIdx.x * 16);
    row_buf(x + tile_base, valid, u * kURow, kURow).store16<kNonTemporal>(as_u32x4(xo[0], xo[1], xo[2], xo[3]), threadIdx.x * 16);
  }
}

// LANS in one pass when the blocks are the partitions.  A workgroup (1024 threads, 8 elements
// a thread, an 8192-element tile; tiles at a fixed stride, the grid resident as a whole)
// updates and stores the moments, keeps x, r + wd x and c + wd x in registers and publishes its
// three partial square sums (one f64 slot each, as in cluster.hpp).  It writes a tile's x
// only after phase 1 of its next tile: by then the other tiles of the older tile's partition
// have been published, so collecting the three totals is one read of the slots, and the loads
// of the next tile are already under way.  Sums are combined in slot order, so the result
// does not depend on timing.  Same traffic as ADAM: payload, m, v, x read once, m, v, x
// written once.
constexpr int kLThreads = 1024;
constexpr int kLPer = kSTile / kLThreads;   // 8
constexpr int kLRows = kLPer / 4;           // 2 rows of 4096 elements, 4 consecutive a thread
constexpr int kLRow = kLThreads * 4;

struct LansTile {
  uint32_t p, tile, valid, tiles_in_part;
  uint64_t base;
};
__device__ inline LansTile lans_tile(const Geo &g, const ClusterGeo &cg, uint32_t item) {
  LansTile t;
  t.p = __builtin_amdgcn_readfirstlane(item / cg.tiles_per_part);
  t.tile = __builtin_amdgcn_readfirstlane(item % cg.tiles_per_part);
  const uint32_t d = g.part_size(t.p);
  t.tiles_in_part = (uint32_t)cdiv(d, kSTile);
  t.base = uniform_off(g.part_base(t.p) + (uint64_t)t.tile * kSTile);
  const uint32_t left = d - t.tile * kSTile;
  t.valid = __builtin_amdgcn_readfirstlane(left < (uint32_t)kSTile ? left : (uint32_t)kSTile);
  return t;
}
template <class DEC>
struct LansRaw {
  u32x4 m[kLRows], v[kLRows], x[kLRows];
  typename DEC::R4 g[kLRows];
  float hdr;
};
struct LansHeld { float xs[kLPer], ur[kLPer], uc[kLPer]; };

template <class DEC>
__device__ inline void lans_issue(const Geo &g, const ClusterGeo &cg, const DEC &dec, const float *x, const float *m,
                                  const float *v, uint32_t item, LansRaw<DEC> &raw) {
  const LansTile t = lans_tile(g, cg, item);
  raw.hdr = dec.header(t.p);
#pragma unroll
  for (int u = 0; u < kLRows; ++u) {
    raw.m[u] = row_buf(m + t.base, t.valid, u * kLRow, kLRow).load16<kNonTemporal>(threadIdx.x * 16, 0);
    raw.v[u] = row_buf(v + t.base, t.valid, u * kLRow, kLRow).load16<kNonTemporal>(threadIdx.x * 16, 0);
    raw.x[u] = row_buf(x + t.base, t.valid, u * kLRow, kLRow).load16<kNonTemporal>(threadIdx.x * 16, 0);
    const uint32_t j = t.tile * kSTile + u * kLRow + threadIdx.x * 4;
    raw.g[u] = dec.load4(g, t.p, j, row_buf(dec.dense_base() + t.base, t.valid, u * kLRow, kLRow));
  }
}

// phi(||x||) and the two weights beta1 / ||r + wd x||, (1 - beta1) / ||c + wd x|| of a block from its
// three sums of squares.
__device__ __forceinline__ void lans_weights(const OptArgs &o, double s_x, double s_r, double s_c, float w[3]) {
  const float norm_x = (float)sqrt(s_x);
  const float norm_r = (float)sqrt(s_r);
  const float norm_c = (float)sqrt(s_c);
  float phi = norm_x < o.phi_lo ? o.phi_lo : norm_x;
  phi = phi > o.phi_hi ? o.phi_hi : phi;
  w[0] = phi;
  w[1] = norm_r > 0.0f ? o.beta1 / norm_r : 0.0f;
  w[2] = norm_c > 0.0f ? (1.0f - o.beta1) / norm_c : 0.0f;
}

// First wave: the three totals of a partition once all its tiles have published theirs.
__device__ inline void lans_collect(const OptArgs &o, const double *ps, uint32_t tiles_in_part, uint32_t *status,
                                    float *weights_sh) {
  const uint32_t lane = threadIdx.x;
  double a0, a1, a2;
  int spins = 0;
  for (;;) {
    bool ok = true;
    a0 = 0.0; a1 = 0.0; a2 = 0.0;
    for (uint32_t s = lane; s < tiles_in_part; s += 64) {
      const double q0 = __hip_atomic_load(ps + 3 * s + 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const double q1 = __hip_atomic_load(ps + 3 * s + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const double q2 = __hip_atomic_load(ps + 3 * s + 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      ok = ok && slot_published(q0) && slot_published(q1) && slot_published(q2);
      a0 += slot_published(q0) ? q0 : 0.0;
      a1 += slot_published(q1) ? q1 : 0.0;
      a2 += slot_published(q2) ? q2 : 0.0;
    }
    if (__all(ok)) break;
    if (++spins > kSpinLimit) {
      if (lane == 0) atomicOr(status, 1u);
      break;
    }
    __builtin_amdgcn_s_sleep(16);
  }
  a0 = wave_sum(a0);
  a1 = wave_sum(a1);
  a2 = wave_sum(a2);
  // once per tile: three square roots of doubles and two divisions are as much arithmetic as a
  // thread's eight elements take, when every thread does them
  if (lane == 0) lans_weights(o, a0, a1, a2, weights_sh);
}

// x of a tile whose partition's phi and weights are in weights_sh.
__device__ inline void lans_write_x(const Geo &g, const ClusterGeo &cg, const OptArgs &o, float *x, uint32_t item,
                                    const LansHeld &h, const float *weights_sh) {
  const LansTile t = lans_tile(g, cg, item);
  const float phi = weights_sh[0], w_r = weights_sh[1], w_c = weights_sh[2];
#pragma unroll
  for (int u = 0; u < kLRows; ++u) {
    float xo[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const float dir = phi * (w_r * h.ur[4 * u + c] + w_c * h.uc[4 * u + c]);
      xo[c] = h.xs[4 * u + c] - o.lr * dir;
    }
    row_buf(x + t.base, t.valid, u * kLRow, kLRow).store16<kNonTemporal>(as_u32x4(xo[0], xo[1], xo[2], xo[3]), threadIdx.x * 16);
  }
}

template <class DEC>
__global__ __launch_bounds__(kLThreads) void lans_single_kernel(Geo g, ClusterGeo cg, DEC dec, float *x, float *m, float *v,
                                                               OptArgs o, double *slots, uint32_t *status) {
  __shared__ __align__(16) float lds[DEC::kLdsFloats];
  __shared__ double red3[3 * (kLThreads / 64)];
  __shared__ float total_sh[3];   // phi and the two weights of the tile being written
  constexpr uint32_t kNone = 0xffffffffu;
  uint32_t item = __builtin_amdgcn_readfirstlane(blockIdx.x);
  if (item >= cg.n_items) return;
  LansRaw<DEC> raw;
  lans_issue(g, cg, dec, x, m, v, item, raw);
  __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): the loop is entered with nothing in flight
  LansHeld prev_h;
  uint32_t prev = kNone;
  const float omb1 = 1.0f - o.beta1, omb2 = 1.0f - o.beta2;
  const float inv_bc1 = 1.0f / o.bc1, inv_bc2 = 1.0f / o.bc2;
  for (;;) {
    const LansTile t = lans_tile(g, cg, item);
    if constexpr (has_begin_tile<DEC>::value) {
      dec.begin_tile(t.p, t.tile, lds);   // the tile of the message, laid out in LDS
    } else {
      __syncthreads();   // the table of the tile before
      dec.table(raw.hdr, lds);
      __syncthreads();
    }
    LansHeld h;
    // a thread's eight squares are summed in f32 (a relative error of a few 1e-7 in its share,
    // the same order as the reciprocals of `ratios_fast`), everything above that in f64
    float f_x = 0.0f, f_r = 0.0f, f_c = 0.0f;
#pragma unroll
    for (int u = 0; u < kLRows; ++u) {
      const uint32_t mi[4] = {raw.m[u].x, raw.m[u].y, raw.m[u].z, raw.m[u].w};
      const uint32_t vi[4] = {raw.v[u].x, raw.v[u].y, raw.v[u].z, raw.v[u].w};
      const uint32_t xi[4] = {raw.x[u].x, raw.x[u].y, raw.x[u].z, raw.x[u].w};
      float gr[4];
      dec.decode4(raw.g[u], t.tile * kSTile + u * kLRow + threadIdx.x * 4, raw.hdr, lds, gr);
      float mo[4], vo[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const float gj = gr[c];
        const float mj = o.beta1 * __uint_as_float(mi[c]) + omb1 * gj;
        const float vj = o.beta2 * __uint_as_float(vi[c]) + omb2 * (gj * gj);
        const float xj = __uint_as_float(xi[c]);
        float u_r, u_c;
        ratios_fast(o, inv_bc1, inv_bc2, gj, mj, vj, xj, &u_r, &u_c);
        mo[c] = mj;
        vo[c] = vj;
        // what the padded record decodes to past the partition's end takes no part in the norms
        const bool in = (uint32_t)(u * kLRow) + threadIdx.x * 4 + c < t.valid;
        h.xs[4 * u + c] = xj;
        h.ur[4 * u + c] = u_r;
        h.uc[4 * u + c] = u_c;
        f_x = in ? fmaf(xj, xj, f_x) : f_x;
        f_r = in ? fmaf(u_r, u_r, f_r) : f_r;
        f_c = in ? fmaf(u_c, u_c, f_c) : f_c;
      }
      row_buf(m + t.base, t.valid, u * kLRow, kLRow).store16<kNonTemporal>(as_u32x4(mo[0], mo[1], mo[2], mo[3]), threadIdx.x * 16);
      row_buf(v + t.base, t.valid, u * kLRow, kLRow).store16<kNonTemporal>(as_u32x4(vo[0], vo[1], vo[2], vo[3]), threadIdx.x * 16);
    }
    const uint32_t next = __builtin_amdgcn_readfirstlane(item + gridDim.x);
    const bool have_next = next < cg.n_items;
    if (have_next) lans_issue(g, cg, dec, x, m, v, next, raw);
    // the three sums over the workgroup: a tree in f32 inside each wave (six levels, the same
    // order of error as the threads' own sums; shuffling doubles cost a tenth of the kernel's
    // instructions), the 16 waves' sums in f64 in fixed order
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      f_x = f_x + __shfl_xor(f_x, off, 64);
      f_r = f_r + __shfl_xor(f_r, off, 64);
      f_c = f_c + __shfl_xor(f_c, off, 64);
    }
    __syncthreads();   // (red3 of the tile before has been read)
    if ((threadIdx.x & 63) == 0) {
      red3[3 * (threadIdx.x >> 6) + 0] = (double)f_x;
      red3[3 * (threadIdx.x >> 6) + 1] = (double)f_r;
      red3[3 * (threadIdx.x >> 6) + 2] = (double)f_c;
    }
    __syncthreads();
    double t_x = 0.0, t_r = 0.0, t_c = 0.0;
    if (threadIdx.x == 0) {
#pragma unroll
      for (int w = 0; w < kLThreads / 64; ++w) {
        t_x += red3[3 * w + 0];
        t_r += red3[3 * w + 1];
        t_c += red3[3 * w + 2];
      }
    }
    if (threadIdx.x == 0) {
      // slot 3*tile + k of the partition holds this tile's k-th partial
      double *ps = slots + 3ull * t.p * cg.tiles_per_part;
      slot_publish(ps + 3 * t.tile + 0, t_x);
      slot_publish(ps + 3 * t.tile + 1, t_r);
      slot_publish(ps + 3 * t.tile + 2, t_c);
    }
    if (prev != kNone && threadIdx.x < 64) {
      const LansTile tp = lans_tile(g, cg, prev);
      lans_collect(o, slots + 3ull * tp.p * cg.tiles_per_part, tp.tiles_in_part, status, total_sh);
    }
    __syncthreads();
    if (prev != kNone) lans_write_x(g, cg, o, x, prev, prev_h, total_sh);
    prev_h = h;
    prev = item;
    if (!have_next) break;
    item = next;
  }
  // the last tile
  __syncthreads();
  if (threadIdx.x < 64) {
    const LansTile tp = lans_tile(g, cg, prev);
    lans_collect(o, slots + 3ull * tp.p * cg.tiles_per_part, tp.tiles_in_part, status, total_sh);
  }
  __syncthreads();
  lans_write_x(g, cg, o, x, prev, prev_h, total_sh);
}

template <class DEC>
__global__ __launch_bounds__(kThreads) void lans_apply_kernel(Geo g, DEC dec, float *x, const float *m,
                                                              const float *v, OptArgs o, const double *norms) {
  __shared__ float lds[DEC::kLdsFloats];
  const uint32_t p = blockIdx.x / g.tiles_per_part;
  const uint32_t tile = blockIdx.x % g.tiles_per_part;
  const uint32_t d = g.part_size(p);
  dec.begin(p, lds);
  const uint64_t base = g.part_base(p);
  const float omb1 = 1.0f - o.beta1;
#pragma unroll
  for (int c = 0; c < kTile / kThreads; ++c) {
    uint32_t j = tile * kTile + c * kThreads + threadIdx.x;
    if (j < d) {
      uint64_t i = base + j;
      uint32_t b = o.block_offsets ? find_block(o.block_offsets, o.n_blocks, i) : p;
      float norm_x = (float)sqrt(norms[3 * (uint64_t)b + 0]);
      float norm_r = (float)sqrt(norms[3 * (uint64_t)b + 1]);
      float norm_c = (float)sqrt(norms[3 * (uint64_t)b + 2]);
      float phi = norm_x < o.phi_lo ? o.phi_lo : norm_x;
      phi = phi > o.phi_hi ? o.phi_hi : phi;
      float w_r = norm_r > 0.0f ? o.beta1 / norm_r : 0.0f;
      float w_c = norm_c > 0.0f ? omb1 / norm_c : 0.0f;
      float gj = dec.at(g, p, j, lds);
      float xj = x[i], u_r, u_c;
      ratios(o, gj, m[i], v[i], xj, &u_r, &u_c);
      float dir = phi * (w_r * u_r + w_c * u_c);
      x[i] = xj - o.lr * dir;
    }
  }
}

// ---------------------------------------------------------------------------------------------
// LANS with caller-defined blocks (Algorithm 5 normalises over layers G_b): two streaming passes.
//
//   norms  : reads m, v, x and the message, writes the new m and v, and leaves the three sums of
//            squares of every (tile, block) pair; a tile whose blocks all lie inside it has its x
//            written here, too
//   totals : adds the pairs of each block that reaches beyond a tile up and turns them into the
//            block's phi and two weights
//   step   : reads the new m and v, x and the message again and writes x (the other tiles)
//
// A tile is 8192 elements, 512 threads with four rows of four elements each, one workgroup a tile,
// so nothing waits for anything inside a kernel.  Walking the pairs in element order, every step
// raises the tile or the block or both, so pair (t, b) owns the three doubles at t + b and no
// table of places is needed; a block that lies inside a tile is finished by the norms pass, which
// puts its phi and weights (three floats) where the sums would go, and the totals pass does the
// same at the first pair of each of the others.  The first block of every tile, which the norms pass
// has searched, is kept for the step pass; that word says as well that the tile is done.
// The blocks of a tile go in batches: each wave sums those of its rows that a block reaches, and one
// barrier later the waves' sums of all blocks of the batch are added up side by side.
// What bounds it: memory, 20.5 + 16.5 bytes an element with a 4-bit message, 24.5 where the blocks
// lie inside tiles (counters: 37.04 with layers).  Layer-shaped blocks, 336 M elements: norms 1.10 ms
// at 6.3 TB/s, totals 0.01, step 0.92 ms at 6.1 TB/s, 2.06 to 2.13 ms the call (from process to
// process).  100 M elements in blocks of 8192 / 1024 / 256: 418 / 450 / 898 us; one block at a time with
// barriers of its own and x in the second pass only it was 631 / 872 / 2001.  (The form that kept a
// tile's x and directions in registers until its blocks were complete, one workgroup of 1024 threads
// a CU and block totals exchanged inside the kernel, took 2.67 ms over the layers and
// 527 / 972 / 2268 us.)
constexpr int kBThreads = 512;
constexpr int kBPer = kSTile / kBThreads;   // 16
constexpr int kBRows = kBPer / 4;
constexpr int kBRow = kBThreads * 4;
constexpr uint32_t kTileDone = 0xffffffffu;   // in place of a tile's first block: the norms pass has written its x

struct LansOut { float xs[kBPer], ur[kBPer], uc[kBPer]; };
template <class DEC>
struct LansIn {
  u32x4 m[kBRows], v[kBRows], x[kBRows];
  typename DEC::R4 g[kBRows];
};
template <class DEC>
__device__ __forceinline__ void lans_request(const Geo &g, const DEC &dec, const LansTile &t, const float *x, const float *m,
                                             const float *v, LansIn<DEC> &in) {
#pragma unroll
  for (int u = 0; u < kBRows; ++u) {
    in.m[u] = row_buf(m + t.base, t.valid, u * kBRow, kBRow).load16<kNonTemporal>(threadIdx.x * 16, 0);
    in.v[u] = row_buf(v + t.base, t.valid, u * kBRow, kBRow).load16<kNonTemporal>(threadIdx.x * 16, 0);
    in.x[u] = row_buf(x + t.base, t.valid, u * kBRow, kBRow).load16<kNonTemporal>(threadIdx.x * 16, 0);
    in.g[u] = dec.load4(g, t.p, t.tile * kSTile + u * kBRow + threadIdx.x * 4,
                        row_buf(dec.dense_base() + t.base, t.valid, u * kBRow, kBRow));
  }
}
// The tables the message's values come from (contains barriers).
template <class DEC>
__device__ __forceinline__ float lans_tables(const DEC &dec, const LansTile &t, float *lds) {
  float hdr = 0.0f;
  if constexpr (has_begin_tile<DEC>::value) {
    dec.begin_tile(t.p, t.tile, lds);
  } else {
    hdr = dec.header(t.p);
    dec.table(hdr, lds);
    __syncthreads();
  }
  return hdr;
}

// Sum over the wave of an f32 (a tree: inside the 16-lane rows, then over the rows), in lane 63.
__device__ __forceinline__ float wave_sum_f32_last(float x) {
#define BPC_DPP_ADD(CTRL, ROWS)                                                                            \
  x = x + __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(x), CTRL, ROWS, 0xf, ROWS == 0xf))
  BPC_DPP_ADD(0x111, 0xf);
  BPC_DPP_ADD(0x112, 0xf);
  BPC_DPP_ADD(0x114, 0xf);
  BPC_DPP_ADD(0x118, 0xf);
  BPC_DPP_ADD(0x142, 0xa);
  BPC_DPP_ADD(0x143, 0xc);
#undef BPC_DPP_ADD
  return x;
}

// The blocks that meet a tile, in every wave: lane l of a window holds the offset lo + l (or the last
// one), block number lo + first is the first that meets the tile, and `n` of them from there on are at
// hand, at most kBatch.
constexpr uint32_t kBatch = 32;
struct BlockBatch {
  uint64_t b;        // number of the first
  uint32_t n;
  uint32_t first, cap, rel;   // lane of the first; how many this window could hold; lane: the block's first element in the tile
  uint64_t inside;   // bit q: block b + q lies inside the tile
  __device__ uint32_t lo(uint32_t q) const { return __builtin_amdgcn_readlane(rel, first + q); }
  __device__ uint32_t hi(uint32_t q) const { return __builtin_amdgcn_readlane(rel, first + q + 1); }
};
// Lane l's bound of a step of the search among the n blocks from lo.
__device__ __forceinline__ uint64_t block_bound(const OptArgs &o, uint64_t lo, uint64_t n) {
  const uint64_t k = lo + (threadIdx.x & 63) * ((n + 63) / 64);
  return o.block_offsets[k < o.n_blocks ? k : o.n_blocks];
}
// `off`: the window's offsets (stride 1 from lo), `first` the lane of block b = lo + first.
__device__ __forceinline__ BlockBatch block_batch(const OptArgs &o, uint64_t off, uint64_t lo, uint32_t first, const LansTile &t, uint64_t D) {
  const uint32_t lane = threadIdx.x & 63;
  const uint64_t tile_first = t.base, tile_end = t.base + t.valid, edge = tile_edge(tile_end, D);
  BlockBatch r;
  r.b = lo + first;
  r.first = first;
  r.cap = 63 - first < kBatch ? 63 - first : kBatch;
  const uint64_t at = off > tile_first ? off : tile_first;
  r.rel = (uint32_t)((at < tile_end ? at : tile_end) - tile_first);
  const uint64_t meets = __ballot(lane - first < r.cap && lo + lane < o.n_blocks && off < tile_end);
  r.n = (uint32_t)__builtin_ctzll(~(meets >> first));
  r.inside = (__ballot(off >= tile_first) & (__ballot(off <= edge) >> 1)) >> first;
  return r;
}
// The first batch of a tile: the last block that starts at or before the tile's first element and those
// after it.  64 bounds at a time; `off` = block_bound(o, 0, n_blocks), requested before the tile's loads (one
// more step for more than 64 blocks, two for more than 4096).
__device__ __forceinline__ BlockBatch block_search(const OptArgs &o, uint64_t off, const LansTile &t, uint64_t D) {
  uint64_t lo = 0, n = o.n_blocks;   // the answer is in [lo, lo + n)
  for (;;) {
    const uint64_t stride = (n + 63) / 64, from = lo;
    narrow_blocks((uint32_t)__popcll(__ballot((threadIdx.x & 63) * stride < n && off <= t.base)), stride, &lo, &n);
    if (stride == 1) return block_batch(o, off, from, __builtin_amdgcn_readfirstlane((uint32_t)(lo - from)), t, D);
    off = block_bound(o, lo, n);
  }
}
// The batch after one that was full.
__device__ __forceinline__ BlockBatch block_next(const OptArgs &o, uint64_t b, const LansTile &t, uint64_t D) {
  return block_batch(o, block_bound(o, b, 1), b, 0, t, D);
}
// Rows of a wave that a block [lo, hi) of the tile reaches, one call of fn(u, whole) each, `whole` where
// all of the wave's elements of the row belong to it (the same in every lane).
template <class FN>
__device__ __forceinline__ void for_rows(uint32_t lo, uint32_t hi, FN fn) {
  const uint32_t w0 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * 256;
#pragma unroll
  for (int u = 0; u < kBRows; ++u) {
    const uint32_t r0 = u * kBRow + w0, r1 = r0 + 256;
    if (lo <= r0 && hi >= r1) fn(u, true);
    else if (lo < r1 && hi > r0) fn(u, false);
  }
}
__device__ __forceinline__ bool in_block(int u, int c, uint32_t lo, uint32_t hi) {
  const uint32_t pos = (uint32_t)(u * kBRow + c) + threadIdx.x * 4;
  return pos >= lo && pos < hi;
}

// A wave's three sums of squares over its elements of the block [lo, hi), to red[0..2]: eight elements of
// a thread and the 64 threads in f32 (512 squares; the same partial sums as the one-pass kernel above),
// everything beyond that in f64.
__device__ __forceinline__ void lans_wave_sums(const LansOut &h, uint32_t lo, uint32_t hi, double *red) {
  float f[2][3] = {{0.0f, 0.0f, 0.0f}, {0.0f, 0.0f, 0.0f}};
  bool any = false;
  for_rows(lo, hi, [&](int u, bool whole) {
    any = true;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int e = 4 * u + c;
      float *s = f[u / 2];
      const bool in = whole || in_block(u, c, lo, hi);
      s[0] = in ? fmaf(h.xs[e], h.xs[e], s[0]) : s[0];
      s[1] = in ? fmaf(h.ur[e], h.ur[e], s[1]) : s[1];
      s[2] = in ? fmaf(h.uc[e], h.uc[e], s[2]) : s[2];
    }
  });
  if (any) {   // (uniform)
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      f[0][k] = wave_sum_f32_last(f[0][k]);
      f[1][k] = wave_sum_f32_last(f[1][k]);
    }
  }
  if ((threadIdx.x & 63) == 63) {
#pragma unroll
    for (int k = 0; k < 3; ++k) red[k] = (double)f[0][k] + (double)f[1][k];
  }
}
// The step of the elements of block [lo, hi): x in place.
__device__ __forceinline__ void lans_step_rows(LansOut &h, uint32_t lo, uint32_t hi, float lr, float phi, float w_r, float w_c) {
  const uint32_t w0 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * 256;
#pragma unroll
  for (int u = 0; u < kBRows; ++u) {
    if (lo < u * kBRow + w0 + 256 && hi > u * kBRow + w0) {   // (uniform)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int e = 4 * u + c;
        const float dir = phi * (w_r * h.ur[e] + w_c * h.uc[e]);
        h.xs[e] = in_block(u, c, lo, hi) ? h.xs[e] - lr * dir : h.xs[e];
      }
    }
  }
}
__device__ __forceinline__ void lans_store_x(const LansTile &t, const LansOut &h, float *x) {
#pragma unroll
  for (int u = 0; u < kBRows; ++u)
    row_buf(x + t.base, t.valid, u * kBRow, kBRow).store16<kNonTemporal>(as_u32x4(h.xs[4 * u], h.xs[4 * u + 1], h.xs[4 * u + 2], h.xs[4 * u + 3]), threadIdx.x * 16);
}

template <class DEC>
__global__ __launch_bounds__(kBThreads, 4) void lans_norms_kernel(Geo g, ClusterGeo cg, DEC dec, float *x, float *m, float *v,
                                                              OptArgs o, double *pairs, uint32_t *first_block) {
  constexpr int kWaves = kBThreads / 64;
  __shared__ __align__(16) float lds[DEC::kLdsFloats];
  __shared__ double red[kBatch][kWaves][3], tot[kBatch][3];
  __shared__ float wts[kBatch][3];
  if (blockIdx.x == 0 && threadIdx.x == 0) o.status[0] = 0;   // no wait in this call
  const uint32_t item = __builtin_amdgcn_readfirstlane(blockIdx.x);
  const LansTile t = lans_tile(g, cg, item);
  const uint64_t bound = block_bound(o, 0, o.n_blocks);
  LansIn<DEC> in;
  lans_request(g, dec, t, x, m, v, in);
  BlockBatch blk = block_search(o, bound, t, g.D);
  const uint32_t b0 = (uint32_t)blk.b;
  const float hdr = lans_tables(dec, t, lds);
  const float omb1 = 1.0f - o.beta1, omb2 = 1.0f - o.beta2;
  const float inv_bc1 = 1.0f / o.bc1, inv_bc2 = 1.0f / o.bc2;
  LansOut h;
#pragma unroll
  for (int u = 0; u < kBRows; ++u) {
    const uint32_t mi[4] = {in.m[u].x, in.m[u].y, in.m[u].z, in.m[u].w};
    const uint32_t vi[4] = {in.v[u].x, in.v[u].y, in.v[u].z, in.v[u].w};
    const uint32_t xi[4] = {in.x[u].x, in.x[u].y, in.x[u].z, in.x[u].w};
    float gr[4], mo[4], vo[4];
    dec.decode4(in.g[u], t.tile * kSTile + u * kBRow + threadIdx.x * 4, hdr, lds, gr);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      mo[c] = o.beta1 * __uint_as_float(mi[c]) + omb1 * gr[c];
      vo[c] = o.beta2 * __uint_as_float(vi[c]) + omb2 * (gr[c] * gr[c]);
      h.xs[4 * u + c] = __uint_as_float(xi[c]);
      ratios_fast(o, inv_bc1, inv_bc2, gr[c], mo[c], vo[c], h.xs[4 * u + c], &h.ur[4 * u + c], &h.uc[4 * u + c]);
    }
    row_buf(m + t.base, t.valid, u * kBRow, kBRow).store16<kNonTemporal>(as_u32x4(mo[0], mo[1], mo[2], mo[3]), threadIdx.x * 16);
    row_buf(v + t.base, t.valid, u * kBRow, kBRow).store16<kNonTemporal>(as_u32x4(vo[0], vo[1], vo[2], vo[3]), threadIdx.x * 16);
  }
  bool done = true;   // every block so far lies inside the tile: its elements' steps are made
#pragma unroll 1
  for (;;) {
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll 1
    for (uint32_t q = 0; q < blk.n; ++q) lans_wave_sums(h, blk.lo(q), blk.hi(q), red[q][wave]);
    __syncthreads();
    double *pair = pairs + 3 * (item + blk.b);
    const uint64_t all = (1ull << blk.n) - 1, inside = blk.inside & all;
    if (threadIdx.x < 3 * blk.n) {   // thread 3 q + k: the k-th sum of block q
      const uint32_t q = threadIdx.x / 3, k = threadIdx.x - 3 * q;
      double s = 0.0;
#pragma unroll
      for (int w = 0; w < kWaves; ++w) s += red[q][w][k];
      if ((inside >> q) & 1) tot[q][k] = s;
      else pair[threadIdx.x] = s;
    }
    done = done && inside == all;
    if (inside) {
      __syncthreads();
      if (threadIdx.x < blk.n && ((inside >> threadIdx.x) & 1)) {
        const uint32_t q = threadIdx.x;
        lans_weights(o, tot[q][0], tot[q][1], tot[q][2], wts[q]);
        float *w = reinterpret_cast<float *>(pair + 3 * q);
#pragma unroll
        for (int k = 0; k < 3; ++k) w[k] = wts[q][k];
      }
      if (done) {
        __syncthreads();
#pragma unroll 1
        for (uint32_t q = 0; q < blk.n; ++q) lans_step_rows(h, blk.lo(q), blk.hi(q), o.lr, wts[q][0], wts[q][1], wts[q][2]);
      }
    }
    if (blk.n < blk.cap) break;
    blk = block_next(o, blk.b + blk.n, t, g.D);
    __syncthreads();   // (red, tot and wts have been read)
  }
  if (done) lans_store_x(t, h, x);
  if (threadIdx.x == 0) first_block[item] = done ? kTileDone : b0;
}

// phi and weights of the blocks that reach beyond a tile.  A workgroup looks at `chunk` blocks at a
// time (one up to 256 blocks, at most 64; where there are many, most lie inside a tile and need
// nothing here).  Blocks of up to kTotWave tiles are a wave's each, longer ones the workgroup's.
constexpr int kTotThreads = 1024;
constexpr uint32_t kTotGrid = 256;
constexpr uint32_t kTotWave = 256;
__global__ __launch_bounds__(kTotThreads) void lans_totals_kernel(OptArgs o, uint64_t D, double *pairs, uint32_t chunk) {
  constexpr int kWaves = kTotThreads / 64;
  __shared__ double red[kWaves][3];
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  // sums over the pairs k = from, from + step, ... of n, then over the wave
  auto sums = [](const double *first, uint32_t n, uint32_t from, uint32_t step, double a[3]) {
    a[0] = a[1] = a[2] = 0.0;
    for (uint32_t k = from; k < n; k += step) {
#pragma unroll
      for (int c = 0; c < 3; ++c) a[c] += first[3 * (uint64_t)k + c];
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) a[c] = wave_sum(a[c]);
  };
  for (uint64_t c0 = (uint64_t)blockIdx.x * chunk; c0 < o.n_blocks; c0 += (uint64_t)gridDim.x * chunk) {
    const uint64_t mine = c0 + lane;
    BlockTiles bt{0, 0};
    if (lane < chunk && mine < o.n_blocks) bt = block_tiles(o.block_offsets[mine], o.block_offsets[mine + 1], D);
    const uint32_t t0 = (uint32_t)bt.t0, n_mine = (uint32_t)bt.n;
    auto block = [&](uint32_t q) { return pairs + 3 * (c0 + q + __builtin_amdgcn_readlane(t0, q)); };
    double a[3];
    uint32_t turn = 0;
    for (uint64_t todo = __ballot(n_mine > 1 && n_mine <= kTotWave); todo; todo &= todo - 1, ++turn) {
      if (turn % kWaves != wave) continue;
      const uint32_t q = (uint32_t)__builtin_ctzll(todo);
      double *first = block(q);
      sums(first, __builtin_amdgcn_readlane(n_mine, q), lane, 64, a);
      if (lane == 0) lans_weights(o, a[0], a[1], a[2], reinterpret_cast<float *>(first));
    }
    for (uint64_t todo = __ballot(n_mine > kTotWave); todo; todo &= todo - 1) {   // (the same in every wave)
      const uint32_t q = (uint32_t)__builtin_ctzll(todo);
      double *first = block(q);
      sums(first, __builtin_amdgcn_readlane(n_mine, q), threadIdx.x, kTotThreads, a);
      if (lane == 0) {
#pragma unroll
        for (int c = 0; c < 3; ++c) red[wave][c] = a[c];
      }
      __syncthreads();   // (and every pair of the block has been read)
      if (threadIdx.x == 0) {
        double s[3] = {0.0, 0.0, 0.0};
#pragma unroll
        for (int w = 0; w < kWaves; ++w)
#pragma unroll
          for (int c = 0; c < 3; ++c) s[c] += red[w][c];
        lans_weights(o, s[0], s[1], s[2], reinterpret_cast<float *>(first));
      }
      __syncthreads();
    }
  }
}

template <class DEC>
__global__ __launch_bounds__(kBThreads, 4) void lans_step_kernel(Geo g, ClusterGeo cg, DEC dec, float *x, const float *m,
                                                             const float *v, OptArgs o, const double *pairs,
                                                             const uint32_t *first_block) {
  __shared__ __align__(16) float lds[DEC::kLdsFloats];
  const uint32_t item = __builtin_amdgcn_readfirstlane(blockIdx.x);
  const uint32_t b0 = __builtin_amdgcn_readfirstlane(first_block[item]);
  if (b0 == kTileDone) return;
  const LansTile t = lans_tile(g, cg, item);
  const uint64_t bound = block_bound(o, b0, 1);
  LansIn<DEC> in;
  lans_request(g, dec, t, x, m, v, in);
  BlockBatch blk = block_batch(o, bound, b0, 0, t, g.D);
  // lane q of a batch: phi and weights of its q-th block, which stand at the block's first pair
  float w[3];
  auto weights = [&](uint64_t off) {
    const uint32_t lane = threadIdx.x & 63;
#pragma unroll
    for (int k = 0; k < 3; ++k) w[k] = 0.0f;
    if (lane < blk.n) {
      const float *at = reinterpret_cast<const float *>(pairs + 3 * (off / kSTile + blk.b + lane));
#pragma unroll
      for (int k = 0; k < 3; ++k) w[k] = at[k];
    }
  };
  weights(bound);
  const float hdr = lans_tables(dec, t, lds);
  const float inv_bc1 = 1.0f / o.bc1, inv_bc2 = 1.0f / o.bc2;
  LansOut h;
#pragma unroll
  for (int u = 0; u < kBRows; ++u) {
    const uint32_t mi[4] = {in.m[u].x, in.m[u].y, in.m[u].z, in.m[u].w};
    const uint32_t vi[4] = {in.v[u].x, in.v[u].y, in.v[u].z, in.v[u].w};
    const uint32_t xi[4] = {in.x[u].x, in.x[u].y, in.x[u].z, in.x[u].w};
    float gr[4];
    dec.decode4(in.g[u], t.tile * kSTile + u * kBRow + threadIdx.x * 4, hdr, lds, gr);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      h.xs[4 * u + c] = __uint_as_float(xi[c]);
      ratios_fast(o, inv_bc1, inv_bc2, gr[c], __uint_as_float(mi[c]), __uint_as_float(vi[c]), h.xs[4 * u + c],
                  &h.ur[4 * u + c], &h.uc[4 * u + c]);
    }
  }
#pragma unroll 1
  for (;;) {
#pragma unroll 1
    for (uint32_t q = 0; q < blk.n; ++q) {
      auto of = [&](float a) { return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(a), q)); };
      lans_step_rows(h, blk.lo(q), blk.hi(q), o.lr, of(w[0]), of(w[1]), of(w[2]));
    }
    if (blk.n < blk.cap) break;
    const uint64_t b = blk.b + blk.n, off = block_bound(o, b, 1);
    blk = block_batch(o, off, b, 0, t, g.D);
    weights(off);
  }
  lans_store_x(t, h, x);
}

// LANS with caller-defined blocks.  *used = false: shape not supported (tiles that cross
// partitions), nothing enqueued.
template <class DEC>
static hipError_t run_lans_blocks(const Geo &g, DEC dec, float *x, float *m, float *v, const OptArgs &o,
                                  const Workspace &ws, hipStream_t stream, bool *used) {
  *used = false;
  if (g.part_elems % kSTile != 0) return hipSuccess;
  const ClusterGeo cg = make_cluster_geo(g, kSTile);
  *used = true;
  // the pairs: three doubles each, fewer of them than tiles + blocks; they start where
  // the slots of the single-pass kernels do (three doubles a tile) and reach into the room for the
  // blocks that follows (three doubles a block, see update_ws_bytes())
  double *pairs = ws.at<double>(ws.lay.slots);
  const uint64_t per = cdiv(o.n_blocks, kTotGrid);
  const uint32_t chunk = per < 64 ? (uint32_t)per : 64u;
  const uint64_t chunks = cdiv(o.n_blocks, chunk);
  uint32_t *first_block = ws.at<uint32_t>(ws.lay.partials);   // a word a tile (the region has two doubles)
  lans_norms_kernel<DEC><<<cg.n_items, kBThreads, 0, stream>>>(g, cg, dec, x, m, v, o, pairs, first_block);
  lans_totals_kernel<<<chunks < kTotGrid ? (uint32_t)chunks : kTotGrid, kTotThreads, 0, stream>>>(o, g.D, pairs, chunk);
  lans_step_kernel<DEC><<<cg.n_items, kBThreads, 0, stream>>>(g, cg, dec, x, m, v, o, pairs, first_block);
  return hipGetLastError();
}

// LANS with the partitions as blocks, one pass.  *used = false: shape not supported.
template <class DEC>
static hipError_t run_lans_single(const Geo &g, DEC dec, float *x, float *m, float *v, const OptArgs &o,
                                  const Workspace &ws, hipStream_t stream, bool *used) {
  *used = false;
  if (g.part_elems % kSTile != 0) return hipSuccess;
  const ClusterGeo cg = make_cluster_geo(g, kSTile);
  static PerDevice cache;
  const int capacity = cache.get([] { return cluster_capacity(reinterpret_cast<const void *>(&lans_single_kernel<DEC>), kLThreads, 0); });
  if (capacity <= 0 || cg.tiles_per_part > (uint32_t)capacity) return hipSuccess;
  *used = true;
  double *slots = ws.at<double>(ws.lay.slots);
  uint32_t *status = ws.status();
  hipError_t e = cluster_launch_begin(stream);
  if (e != hipSuccess) return e;
  const uint32_t n_slots = 3 * g.P * cg.tiles_per_part;
  slots_reset_kernel<<<(uint32_t)cdiv(n_slots, 256), 256, 0, stream>>>(slots, n_slots, status, nullptr);
  const uint32_t grid = cg.n_items > (uint32_t)capacity ? (uint32_t)capacity : cg.n_items;
  lans_single_kernel<DEC><<<grid, kLThreads, 0, stream>>>(g, cg, dec, x, m, v, o, slots, status);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  return cluster_launch_end(stream);
}

template <class DEC>
static hipError_t run_update(const Geo &g, DEC dec, float *x, float *m, float *v, const bpc_opt_t &opt,
                             double *norms, const Workspace &ws, hipStream_t stream) {
  OptArgs o{opt.lr, opt.beta1, opt.beta2, opt.eps, opt.weight_decay, opt.bias_corr1, opt.bias_corr2,
            opt.phi_lo, opt.phi_hi, opt.block_offsets, opt.n_blocks, ws.status()};
  if (opt.kind == BPC_OPT_ADAM) {
    adam_update_kernel<DEC><<<g.n_tiles, kThreads, 0, stream>>>(g, dec, x, m, v, o);
    return hipGetLastError();
  }
  {
    bool used = false;
    hipError_t e1 = opt.block_offsets ? run_lans_blocks(g, dec, x, m, v, o, ws, stream, &used)
                                      : run_lans_single(g, dec, x, m, v, o, ws, stream, &used);
    if (e1 != hipSuccess || used) return e1;
  }
  uint64_t nb = opt.block_offsets ? opt.n_blocks : g.P;
  hipError_t e = fill_zero(norms, sizeof(double) * 3 * nb, stream);
  if (e != hipSuccess) return e;
  update_moments_kernel<DEC, true><<<g.n_tiles, kThreads, 0, stream>>>(g, dec, x, m, v, o, norms);
  lans_apply_kernel<DEC><<<g.n_tiles, kThreads, 0, stream>>>(g, dec, x, m, v, o, norms);
  return hipGetLastError();
}

hipError_t adam_update_fp16_map(const Geo &g, const RecordMap &map, const uint8_t *payload, float *x, float *m, float *v,
                                const bpc_opt_t &opt, const Workspace &ws, hipStream_t stream) {
  const OptArgs o{opt.lr, opt.beta1, opt.beta2, opt.eps, opt.weight_decay, opt.bias_corr1, opt.bias_corr2,
                  opt.phi_lo, opt.phi_hi, opt.block_offsets, opt.n_blocks, ws.status()};
  adam_update_kernel<<<g.n_tiles, kThreads, 0, stream>>>(g, Fp16MapDec{payload, map}, x, m, v, o);
  return hipGetLastError();
}

hipError_t adaptive_update(const Geo &g, const bpc_params_t &prm, const uint8_t *payload, float *x, float *m,
                           float *v, const bpc_opt_t &opt, const Workspace &ws, hipStream_t stream) {
  double *norms = ws.at<double>(ws.lay.norms);
  switch (prm.kind) {
    case BPC_SIGN: return run_update(g, SignDec{payload, g.stride}, x, m, v, opt, norms, ws, stream);
    case BPC_DITHER: case BPC_NATDITHER:
      if (prm.kind == BPC_DITHER && dither_planes(prm.levels) > 0) {
        return run_update(g, DitherWideDec{payload, g.stride, prm.levels, g.part_elems}, x, m, v, opt, norms, ws, stream);
      }
      return run_update(g, DitherDec{payload, g.stride, prm.levels, prm.kind == BPC_NATDITHER}, x, m, v, opt, norms, ws, stream);
    case BPC_IDENTITY: return run_update(g, IdentityDec{payload, g.stride}, x, m, v, opt, norms, ws, stream);
    case BPC_FP16: return run_update(g, Fp16Dec{payload, g.stride}, x, m, v, opt, norms, ws, stream);
    default: break;
  }
  float *dense = ws.at<float>(ws.lay.dense);
  const bool lans = opt.kind == BPC_OPT_LANS && g.part_elems % kSTile == 0;
  if ((opt.kind == BPC_OPT_ADAM || lans) && (prm.kind == BPC_TOPK || prm.kind == BPC_TOPK16 || prm.kind == BPC_RANDK)) {
    // no dense decode: the update kernel lays each tile of the message out in LDS itself
    // (tiles of 4096 elements in the Adam-style kernel, of 8192 in the LANS kernels)
    OptArgs o{opt.lr, opt.beta1, opt.beta2, opt.eps, opt.weight_decay, opt.bias_corr1, opt.bias_corr2,
              opt.phi_lo, opt.phi_hi, opt.block_offsets, opt.n_blocks, ws.status()};
    const uint32_t shift = lans ? 13 : 12;
    const uint32_t tiles = (uint32_t)cdiv(g.part_elems, 1ull << shift);
    const uint32_t *table = nullptr;
    const uint2 *pairs = nullptr;
    // small calls go without the launch that makes the table (top-k, Adam-style: 0.3 M elements 13.5 -> 6.7 us, 2 M
    // 13.3 -> 9.7; LANS over the partitions, 4 M, 26.3 -> 24.2; LANS over blocks, whose two passes search or draw each for
    // itself, at the largest sizes that go without it: top-k, 4 M, 37.1 -> 32.7, random-k, 1 M, k = 3 %, 47.6 -> 28.2, and 2 M,
    // k = 1 %, 29.4 -> 24.3)
    const uint32_t tiles_all = (uint32_t)cdiv(g.D, 1ull << shift);
    if (tiles_all <= kOwnTiles && (prm.kind != BPC_RANDK || randk_draws_again(g, tiles_all, 1, lans ? kBThreads : kThreads))) {
      const int mode = prm.kind == BPC_RANDK ? 2 : prm.kind == BPC_TOPK16 ? 1 : 0;
      auto run = [&](auto dec, auto call) {
        return call(decltype(dec){payload, g.stride, g.k_cap, mode, nullptr, 0, nullptr,
                                  {prm.seed, prm.stream_id, g.D, g.part_elems, g.part0, prm.value_scale}});
      };
      if (!lans)
        return run(SparseTileDec<kTile, kThreads, true>{}, [&](auto dec) {
          adam_update_kernel<<<g.n_tiles, kThreads, 0, stream>>>(g, dec, x, m, v, o);
          return hipGetLastError();
        });
      bool used = false;
      const hipError_t e = opt.block_offsets
          ? run(SparseTileDec<kSTile, kBThreads, true>{}, [&](auto dec) { return run_lans_blocks(g, dec, x, m, v, o, ws, stream, &used); })
          : run(SparseTileDec<kSTile, kLThreads, true>{}, [&](auto dec) { return run_lans_single(g, dec, x, m, v, o, ws, stream, &used); });
      if (e != hipSuccess || used) return e;
    }
    uint32_t table_stride = 0;
    int mode = -1;
    if (prm.kind == BPC_RANDK) {
      const uint64_t list_bytes = ((uint64_t)g.P * g.k_cap * sizeof(uint2) + 255) / 256 * 256;
      const uint64_t table_bytes = (uint64_t)g.P * kRandkTableStride * sizeof(uint32_t);
      if (tiles <= 1024 && list_bytes + table_bytes <= sizeof(float) * g.D) {
        uint2 *lists = reinterpret_cast<uint2 *>(dense);   // (the dense workspace is free on this path)
        uint32_t *tab = reinterpret_cast<uint32_t *>(reinterpret_cast<uint8_t *>(dense) + list_bytes);
        hipError_t e = randk_bin_tiles(g, prm, payload, lists, tab, shift, stream);
        if (e != hipSuccess) return e;
        table = tab; pairs = lists; table_stride = kRandkTableStride; mode = 2;
      }
    } else {
      uint32_t *tab = ws.at<uint32_t>(ws.lay.starts);
      const bool half = prm.kind == BPC_TOPK16;
      hipError_t e = topk_tile_starts(g, payload, half, tab, shift, stream);
      if (e != hipSuccess) return e;
      table = tab; table_stride = tiles + 1; mode = half ? 1 : 0;
    }
    if (mode >= 0) {
      if (!lans) {
        adam_update_kernel<<<g.n_tiles, kThreads, 0, stream>>>(g, SparseTileDec<kTile, kThreads>{payload, g.stride, g.k_cap, mode, table, table_stride, pairs, {}}, x, m, v, o);
        return hipGetLastError();
      }
      bool used = false;
      hipError_t e = opt.block_offsets
          ? run_lans_blocks(g, SparseTileDec<kSTile, kBThreads>{payload, g.stride, g.k_cap, mode, table, table_stride, pairs, {}}, x, m, v, o, ws, stream, &used)
          : run_lans_single(g, SparseTileDec<kSTile, kLThreads>{payload, g.stride, g.k_cap, mode, table, table_stride, pairs, {}}, x, m, v, o, ws, stream, &used);
      if (e != hipSuccess || used) return e;
      // (the single-pass kernel declined the shape: the dense decode below overwrites the lists)
    }
  }
  hipError_t e = decode_dense(g, prm, payload, dense, stream);
  if (e != hipSuccess) return e;
  return run_update(g, DenseDec{dense}, x, m, v, opt, norms, ws, stream);
}

}  // namespace bpc
