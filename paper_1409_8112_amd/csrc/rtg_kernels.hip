// rtg_kernels.hip -- gfx950 kernels of the RTG all-pairs r-NN pipeline.
//
// Steps (Sec. III, Alg. "Randomly Shifted Grids" with random orientations):
//   stage      AoS -> SoA copy of the points, finiteness check, bounding box
//   keys       cell of every (point, grid) in FP64, packed into a 64-bit key
//   sort       stable LSD radix sort of (key, point) -- groups equal cells
//   cells      runs of equal keys with >= 2 points and their 64x64 tile pairs
//   pairs      one wave per tile pair: FP32 screen, FP64 band re-test,
//              ballot-compacted output of pairs within r
//   unique     sort of packed pairs and removal of repeats (Sec. III-B)
//   csr        symmetric neighbour lists (Sec. III-B)
//
// The whole file is compiled with FMA contraction off: the cell coordinate
// y = (R p) / c + u and the FP64 re-test must round every product and sum on
// its own, in the order written, to match the FP64 definition bit for bit.
// Where a fused multiply-add is wanted (the FP32 screen) it is written out.
#pragma clang fp contract(off)

#include "rtg_internal.h"

#include <math.h>

#include <algorithm>
#include <type_traits>
#include <utility>

namespace rtgk {
namespace {

__device__ __forceinline__ uint32_t lane_id() {
  return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
}

// Number of set bits of m below this lane.
__device__ __forceinline__ uint32_t rank_below(uint64_t m) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

__device__ __forceinline__ uint64_t ballot(bool p) { return __ballot(p); }

// Orders the LDS traffic of one wave: every lane's earlier LDS writes are
// seen by every lane's later LDS reads, and no access moves across.
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// v from another lane by a DPP pattern (row_mask / bank_mask select the
// written rows and banks; lanes whose source falls outside the row, or that
// are not written, get old).  Every lane of the wave must be active.
template <int Ctrl, int RowMask = 0xf, int BankMask = 0xf>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t old, uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)old, (int)v, Ctrl, RowMask, BankMask, false);
}

// The value of lane l (a constant or wave-uniform l), in every lane.
__device__ __forceinline__ uint32_t lane_value(uint32_t v, int l) {
  return (uint32_t)__builtin_amdgcn_readlane((int)v, l);
}
__device__ __forceinline__ unsigned long long lane_value(unsigned long long v, int l) {
  const uint32_t lo = lane_value((uint32_t)v, l), hi = lane_value((uint32_t)(v >> 32), l);
  return ((unsigned long long)hi << 32) | lo;
}

// v of the first active lane, as a scalar.
template <typename T>
__device__ __forceinline__ T uniform(T v) {
  return (T)__builtin_amdgcn_readfirstlane((int)v);
}

// DPP controls: row_shr:n = 0x110 + n, row_mirror = 0x140,
// row_half_mirror = 0x141, row_bcast:15 = 0x142, row_bcast:31 = 0x143;
// quad_perm [1,0,3,2] = 0xB1, [2,3,0,1] = 0x4E.
template <typename T>
__device__ __forceinline__ T wave_inclusive_scan(T v) {
  if constexpr (sizeof(T) == 4) {
    // within each row of 16 lanes (shifts 1, 2, 4, 8), then row 0's total
    // into rows 1 and 3, then rows 0-1's total into rows 2 and 3
    uint32_t x = (uint32_t)v;
    x += dpp_u32<0x111>(0u, x);
    x += dpp_u32<0x112>(0u, x);
    x += dpp_u32<0x114>(0u, x);
    x += dpp_u32<0x118>(0u, x);
    x += dpp_u32<0x142, 0xa>(0u, x);
    x += dpp_u32<0x143, 0xc>(0u, x);
    return (T)x;
  } else {
    const uint32_t lane = lane_id();
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      T t = __shfl_up(v, o, 64);
      if (lane >= (uint32_t)o) v += t;
    }
    return v;
  }
}

// Exclusive scan of one value per thread over a 256-thread block.  wsum
// must be a __shared__ array of kWaves elements; total receives the sum.
template <typename T>
__device__ __forceinline__ T block_exclusive_scan(T v, T* wsum, T& total) {
  const uint32_t lane = lane_id();
  const int w = threadIdx.x >> 6;
  T inc = wave_inclusive_scan(v);
  if (lane == 63) wsum[w] = inc;
  __syncthreads();
  T before = 0, all = 0;
#pragma unroll
  for (int q = 0; q < kWaves; ++q) {
    T x = wsum[q];
    if (q < w) before += x;
    all += x;
  }
  __syncthreads();
  total = all;
  return before + inc - v;
}

// Order-preserving encoding of a finite float as uint32.
__device__ __forceinline__ uint32_t float_order(float f) {
  uint32_t b = __float_as_uint(f);
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

// ---------------------------------------------------------------------------
// fill

template <typename T>
__global__ void k_fill(T* p, T v, size_t count) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  size_t stride = (size_t)gridDim.x * blockDim.x;
  for (; i < count; i += stride) p[i] = v;
}

// ---------------------------------------------------------------------------
// stage: one thread per point.

// Instance that owns point block blk: the largest q with blk_first <= blk.
__device__ __forceinline__ uint32_t block_instance(const InstDesc* __restrict__ inst, uint32_t m,
                                                   uint32_t blk) {
  uint32_t lo = 0, hi = m;
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) >> 1;
    if ((uint32_t)inst[mid].blk_first <= blk) lo = mid;
    else hi = mid;
  }
  return lo;
}

// Each block writes its own per-axis min/max (order-preserving encodings)
// to part[block][2d]; k_bbox_reduce folds them per instance.  (Atomics on
// the 2d words of one bounding box would all meet at one address per axis.)
__global__ __launch_bounds__(kBlock) void k_stage(const InstDesc* __restrict__ inst, uint32_t m,
                                                  int d, int64_t npts, float* __restrict__ soa,
                                                  float* __restrict__ aos, uint32_t* bad,
                                                  uint32_t* __restrict__ part,
                                                  float* __restrict__ rec, int rs) {
  __shared__ uint32_t smin[kWaves][kMaxDim], smax[kWaves][kMaxDim];
  const uint32_t q = block_instance(inst, m, blockIdx.x);
  const float* pts = inst[q].pts;
  const int64_t i = (int64_t)(blockIdx.x - (uint32_t)inst[q].blk_first) * kBlock + threadIdx.x;
  const bool live = i < inst[q].n;
  const int64_t g = inst[q].pt_off + i;
  const int w = threadIdx.x >> 6;
  bool nonfinite = false;
  for (int l = 0; l < d; ++l) {
    float v = live ? pts[i * d + l] : 0.0f;
    uint32_t lo = 0xFFFFFFFFu, hi = 0u;
    if (live) {
      soa[(int64_t)l * npts + g] = v;
      if (aos) aos[g * d + l] = v;
      if (rec) rec[g * rs + l] = v;
      if (!isfinite(v)) nonfinite = true;
      else lo = hi = float_order(v);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      lo = min(lo, (uint32_t)__shfl_xor((int)lo, o, 64));
      hi = max(hi, (uint32_t)__shfl_xor((int)hi, o, 64));
    }
    if (lane_id() == 0) {
      smin[w][l] = lo;
      smax[w][l] = hi;
    }
  }
  if (ballot(nonfinite) && lane_id() == 0) atomicOr(bad, 1u);
  if (rec && live)
    for (int l = d; l < rs; ++l) rec[g * rs + l] = 0.0f;  // padding, then the signature word
  __syncthreads();
  if (threadIdx.x < (unsigned)d) {
    uint32_t lo = 0xFFFFFFFFu, hi = 0u;
#pragma unroll
    for (int q2 = 0; q2 < kWaves; ++q2) {
      lo = min(lo, smin[q2][threadIdx.x]);
      hi = max(hi, smax[q2][threadIdx.x]);
    }
    part[(size_t)blockIdx.x * 2 * d + 2 * threadIdx.x] = lo;
    part[(size_t)blockIdx.x * 2 * d + 2 * threadIdx.x + 1] = hi;
  }
}

// The minimum and maximum of lo / hi over the wave (every lane active), in
// every lane: quads, half rows and rows by DPP, then the four rows' values.
__device__ __forceinline__ void wave_minmax_u32(uint32_t& lo, uint32_t& hi) {
  auto step = [&](auto ctrl) {
    constexpr int C = decltype(ctrl)::value;
    lo = min(lo, dpp_u32<C>(lo, lo));
    hi = max(hi, dpp_u32<C>(hi, hi));
  };
  step(std::integral_constant<int, 0xB1>{});
  step(std::integral_constant<int, 0x4E>{});
  step(std::integral_constant<int, 0x141>{});
  step(std::integral_constant<int, 0x140>{});
  lo = min(min(lane_value(lo, 0), lane_value(lo, 16)), min(lane_value(lo, 32), lane_value(lo, 48)));
  hi = max(max(lane_value(hi, 0), lane_value(hi, 16)), max(lane_value(hi, 32), lane_value(hi, 48)));
}

// k_stage for d = D <= 16: every coordinate of the thread's point loaded at
// once, wave minima and maxima by DPP, and the point record (when asked
// for: the coordinates, then zeros -- padding and the signature word the
// key kernel writes) stored 16 bytes at a time.
template <int D>
__global__ __launch_bounds__(kBlock) void k_stage_d(const InstDesc* __restrict__ inst, uint32_t m,
                                                    int64_t npts, float* __restrict__ soa,
                                                    float* __restrict__ aos, uint32_t* bad,
                                                    uint32_t* __restrict__ part,
                                                    float* __restrict__ rec) {
  constexpr int RS = (D + 2 + 3) & ~3;  // record floats (used for D <= 6)
  __shared__ uint32_t smin[kWaves][D], smax[kWaves][D];
  const uint32_t q = block_instance(inst, m, blockIdx.x);
  const float* pts = inst[q].pts;
  const int64_t i = (int64_t)(blockIdx.x - (uint32_t)inst[q].blk_first) * kBlock + threadIdx.x;
  const bool live = i < inst[q].n;
  const int64_t g = inst[q].pt_off + i;
  const int w = threadIdx.x >> 6;
  float v[D];
#pragma unroll
  for (int l = 0; l < D; ++l) v[l] = live ? pts[i * D + l] : 0.0f;
  bool nonfinite = false;
#pragma unroll
  for (int l = 0; l < D; ++l) {
    uint32_t lo = 0xFFFFFFFFu, hi = 0u;
    if (live) {
      soa[(int64_t)l * npts + g] = v[l];
      if (aos) aos[g * D + l] = v[l];
      if (!isfinite(v[l])) nonfinite = true;
      else lo = hi = float_order(v[l]);
    }
    wave_minmax_u32(lo, hi);
    if (lane_id() == 0) {
      smin[w][l] = lo;
      smax[w][l] = hi;
    }
  }
  if (ballot(nonfinite) && lane_id() == 0) atomicOr(bad, 1u);
  if constexpr (D <= 6) {
    if (rec && live) {
      float4* r4 = reinterpret_cast<float4*>(rec + g * RS);
#pragma unroll
      for (int c4 = 0; c4 < RS / 4; ++c4) {
        float4 x;
        x.x = 4 * c4 + 0 < D ? v[4 * c4 + 0] : 0.0f;
        x.y = 4 * c4 + 1 < D ? v[4 * c4 + 1] : 0.0f;
        x.z = 4 * c4 + 2 < D ? v[4 * c4 + 2] : 0.0f;
        x.w = 4 * c4 + 3 < D ? v[4 * c4 + 3] : 0.0f;
        r4[c4] = x;
      }
    }
  }
  __syncthreads();
  if (threadIdx.x < (unsigned)D) {
    uint32_t lo = 0xFFFFFFFFu, hi = 0u;
#pragma unroll
    for (int q2 = 0; q2 < kWaves; ++q2) {
      lo = min(lo, smin[q2][threadIdx.x]);
      hi = max(hi, smax[q2][threadIdx.x]);
    }
    part[(size_t)blockIdx.x * 2 * D + 2 * threadIdx.x] = lo;
    part[(size_t)blockIdx.x * 2 * D + 2 * threadIdx.x + 1] = hi;
  }
}

// Before the stage: bbox of every instance to the identities of min and
// max (bits of the order-preserving encoding), *bad to 0, and the caller's
// zero64[0, nzero) to 0 (counters of the pass), in one launch.
__global__ void k_stage_init(uint32_t* __restrict__ bbox, uint32_t count, uint32_t* bad,
                             uint64_t* __restrict__ zero64, uint32_t nzero) {
  const uint32_t e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e < count) bbox[e] = (e & 1u) ? 0u : 0xFFFFFFFFu;
  if (e < nzero) zero64[e] = 0ull;
  if (e == 0) *bad = 0u;
}

// Block (q, y) folds slice y of instance q's per-block boxes into bbox with
// atomic min / max (one per axis and block): one instance spreads over up
// to kBboxBlocks blocks.
constexpr uint32_t kBboxBlocks = 64;
__global__ __launch_bounds__(kBlock) void k_bbox_reduce(const InstDesc* __restrict__ inst, int d,
                                                        const uint32_t* __restrict__ part,
                                                        uint32_t* __restrict__ bbox) {
  const uint32_t q = blockIdx.x;
  const uint32_t b0 = inst[q].blk_first;
  const uint32_t nb = (uint32_t)((inst[q].n + kBlock - 1) / kBlock);
  const uint32_t per = (nb + gridDim.y - 1) / gridDim.y;
  const uint32_t lo_b = blockIdx.y * per, hi_b = min(nb, lo_b + per);
  if (lo_b >= hi_b) return;
  const int w = threadIdx.x >> 6;
  const uint32_t lane = lane_id();
  for (int l = w; l < d; l += kWaves) {
    uint32_t lo = 0xFFFFFFFFu, hi = 0u;
    for (uint32_t b = lo_b + lane; b < hi_b; b += 64) {
      lo = min(lo, part[(size_t)(b0 + b) * 2 * d + 2 * l]);
      hi = max(hi, part[(size_t)(b0 + b) * 2 * d + 2 * l + 1]);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      lo = min(lo, (uint32_t)__shfl_xor((int)lo, o, 64));
      hi = max(hi, (uint32_t)__shfl_xor((int)hi, o, 64));
    }
    if (lane == 0) {
      atomicMin(&bbox[(size_t)q * 2 * d + 2 * l], lo);
      atomicMax(&bbox[(size_t)q * 2 * d + 2 * l + 1], hi);
    }
  }
}

// ---------------------------------------------------------------------------
// keys: y_j = ((R_j0 p_0 + R_j1 p_1) + ...) * inv_c + u_j, each operation
// rounded on its own (contraction is off), kappa_j = floor(y_j).

template <int D>
__device__ __forceinline__ double cell_y(const double* __restrict__ Rj, const float* p_reg,
                                         const float* __restrict__ soa, int64_t n, int64_t i,
                                         int d, double inv_c, double uj) {
  double z;
  if (D > 0) {
    z = Rj[0] * (double)p_reg[0];
#pragma unroll
    for (int l = 1; l < D; ++l) z = z + Rj[l] * (double)p_reg[l];
  } else {
    z = Rj[0] * (double)soa[i];
    for (int l = 1; l < d; ++l) z = z + Rj[l] * (double)soa[(int64_t)l * n + i];
  }
  return z * inv_c + uj;
}

// Byte j of a KeyLayout array as a scalar (a wave-uniform j): read as words,
// which the scalar unit can load; bytes go through vector registers.
__device__ __forceinline__ uint32_t layout_byte(const uint8_t* __restrict__ bytes, int j) {
  const uint32_t v = reinterpret_cast<const uint32_t*>(bytes)[j >> 2];
  return (v >> (8 * (j & 3))) & 0xFFu;
}

// A multiplier of axis j in hash h (0 or 1): 24 bits, odd.
__device__ __forceinline__ constexpr uint32_t hash_weight(int j, int h) {
  uint32_t x = (uint32_t)(2 * j + h + 1) * 0x9E3779B1u;
  x = (x ^ (x >> 15)) * 0x9E3779B1u;
  x ^= x >> 13;
  return (x & 0xFFFFFFu) | 1u;
}

// The packed cell fields and signature group of one point under one transform
// (rows Rt, shifts ut, field origins kl); false if a cell coordinate is out of
// range.  The point is p (D > 0) or soa[l n + i], l < d.  C holds both results
// (fields are taken modulo their width, at most 32 bits, so 32-bit differences
// are exact).  HASH: instead of the fields side by side, layout->hashed bits
// of a hash of all of them: two linear hashes of the fields' low 24 bits
// (full-rate 24-bit products), one mixed before they meet so that no
// difference of cells collides throughout, except where every axis differs by
// a multiple of 2^24 cells.
template <int D, typename C, bool HASH = false>
__device__ __forceinline__ bool pack_cell(const double* __restrict__ Rt,
                                          const double* __restrict__ ut,
                                          const int64_t* __restrict__ kl,
                                          const KeyLayout* __restrict__ layout, const float* p,
                                          const float* __restrict__ soa, int64_t n, int64_t i,
                                          int d, double inv_c, int sig_b, C& cell, C& grp) {
  const uint32_t bmask = (uint32_t)((1ull << sig_b) - 1ull);
  bool all_ok = true;
  cell = grp = 0;
  uint32_t h0 = 0, h1 = 0;
  for (int j = 0; j < d; ++j) {
    const double y = cell_y<D>(Rt + (size_t)j * d, p, soa, n, i, d, inv_c, ut[j]);
    const bool ok = fabs(y) < 2147483648.0;
    all_ok = all_ok && ok;
    // |y| < 2^31: the floor fits 32 bits, and one native conversion takes it
    const uint32_t f = (uint32_t)(ok ? (int32_t)floor(y) : 0) - (uint32_t)kl[j];
    if constexpr (HASH) {
      h0 += __umul24(f, hash_weight(j, 0));
      h1 += __umul24(f, hash_weight(j, 1));
    } else {
      const uint32_t mask = (uint32_t)((1ull << layout_byte(layout->bits, j)) - 1ull);
      cell |= (C)(f & mask) << layout_byte(layout->shift, j);
    }
    grp |= (C)(f & bmask) << (j * sig_b);
  }
  if constexpr (HASH) {
    uint32_t h = (h0 ^ (h0 >> 15)) * 0x9E3779B1u + h1;
    h = (h ^ (h >> 14)) * 0x9E3779B1u;
    cell = (C)(h >> (32 - layout->hashed));
  }
  return all_ok;
}

// Writes the keys of the points' segments in [sa, sb): key = (segment - sa)
// << cell_bits | packed cell, at segs[segment].key_off + the point's index in
// its instance.  The work is one FP64 dot product per axis and the packing of
// its floor; packed in 32 bits when cell and signature group fit:
// 61 -> 51 us for 8e6 keys at d = 6, 537 -> 507 us for 32e6 at d = 12.
// SPLIT = false: one thread per batch point, all of its grids.  SPLIT = true:
// a block takes 64 points, its four waves every fourth grid of a signature
// word, whose parts meet in LDS; blockIdx.y takes words_per_slice words.
// Four waves per point fill the chip where the points alone do not (see
// launch_keys).
template <int D, bool SPLIT>
__global__ __launch_bounds__(kBlock) void k_keys(const InstDesc* __restrict__ inst, uint32_t m,
                                                 int d_rt, int64_t npts,
                                                 const float* __restrict__ soa, int sa, int sb,
                                                 const SegDesc* __restrict__ segs,
                                                 const double* __restrict__ R,
                                                 const double* __restrict__ u,
                                                 const int64_t* __restrict__ klo,
                                                 const KeyLayout* __restrict__ layout,
                                                 uint64_t* __restrict__ keys,
                                                 uint32_t* __restrict__ vals, uint32_t* err,
                                                 uint64_t* __restrict__ sig, int sig_stride,
                                                 int sig_b, int sig_gpw, int idx_bits,
                                                 int sig_fresh, int words_per_slice) {
  __shared__ uint64_t part[SPLIT ? kWaves : 1][SPLIT ? 64 : 1];
  const int d = D > 0 ? D : d_rt;
  const uint32_t blk = SPLIT ? blockIdx.x / kWaves : blockIdx.x;
  const uint32_t lane = lane_id();
  const int w = uniform((int)(threadIdx.x >> 6));
  const uint32_t q = uniform(block_instance(inst, m, blk));
  const int64_t n = inst[q].n;
  const int64_t i0 = (int64_t)(blk - (uint32_t)inst[q].blk_first) * kBlock +
                     (SPLIT ? (int64_t)(blockIdx.x % kWaves) * 64 : 0);
  const int64_t i = i0 + (SPLIT ? lane : threadIdx.x);
  if (SPLIT ? i0 >= n : i >= n) return;  // (SPLIT: the whole block)
  const bool live = i < n;
  const int64_t g = inst[q].pt_off + (live ? i : n - 1);
  const int seg_first = inst[q].seg_first;
  const int t_lo = max(0, sa - seg_first), t_hi = min(inst[q].k, sb - seg_first);
  if (t_lo >= t_hi) return;
  const double inv_c = inst[q].inv_c;
  const int tr_off = inst[q].tr_off;
  float p[D > 0 ? D : 1];
  if (D > 0) {
#pragma unroll
    for (int l = 0; l < (D > 0 ? D : 1); ++l) p[l] = soa[(int64_t)l * npts + g];
  }
  const int cell_bits = layout->cell_bits;
  const int gbits = d * sig_b;
  bool bad = false;
  // one grid's key (stored) and signature group (returned)
  auto grid = [&](int t, auto zero, auto hash) -> uint64_t {
    using C = decltype(zero);
    const int s = seg_first + t;
    const int tr = tr_off + t;
    const double* Rt = R + (size_t)tr * d * d;
    const double* ut = u + (size_t)tr * d;
    const int64_t* kl = klo + (size_t)tr * d;
    C cell = 0, grp = 0;
    bad |= !pack_cell<D, C, decltype(hash)::value>(Rt, ut, kl, layout, p, soa, npts, g, d, inv_c,
                                                   sig_b, cell, grp);
    const uint64_t key =
        (cell_bits < 64) ? (((uint64_t)(s - sa) << cell_bits) | (uint64_t)cell) : (uint64_t)cell;
    const int64_t pos = segs[s].key_off + i;
    if (live) {
      if (idx_bits) {
        keys[pos] = (key << idx_bits) | (uint64_t)g;
      } else {
        keys[pos] = key;
        vals[pos] = (uint32_t)g;
      }
    }
    return (uint64_t)grp;
  };
  auto words = [&](auto zero, auto hash) {
    const int w_lo = t_lo / sig_gpw + (SPLIT ? (int)blockIdx.y * words_per_slice : 0);
    const int w_end = (t_hi + sig_gpw - 1) / sig_gpw;
    const int w_hi = SPLIT ? min(w_end, w_lo + words_per_slice) : w_end;
    for (int x = w_lo; x < w_hi; ++x) {
      const int ta = max(t_lo, x * sig_gpw), tb = min(t_hi, (x + 1) * sig_gpw);
      uint64_t word = 0;
      for (int t = ta + (SPLIT ? w : 0); t < tb; t += SPLIT ? kWaves : 1) {
        const uint64_t grp = grid(t, zero, hash);
        if (sig) word |= grp << ((t - x * sig_gpw) * gbits);
      }
      if (sig) {
        // the point owns its row: earlier passes' bits are read back and kept
        uint64_t* dst = sig + (size_t)g * sig_stride + x;
        if constexpr (SPLIT) {
          part[w][lane] = word;
          __syncthreads();
          if (w == (x & (kWaves - 1)) && live) {
#pragma unroll
            for (int o = 0; o < kWaves; ++o) word |= part[o][lane];
            *dst = sig_fresh ? word : (*dst | word);
          }
          __syncthreads();  // part is rewritten by the next word
        } else {
          *dst = sig_fresh ? word : (*dst | word);
        }
      }
    }
  };
  const std::false_type packed{};
  const std::true_type hashed{};
  if (layout->hashed) {
    if (gbits <= 32) words(uint32_t{0}, hashed);
    else words(uint64_t{0}, hashed);
  } else if (cell_bits <= 32 && gbits <= 32) {
    words(uint32_t{0}, packed);
  } else {
    words(uint64_t{0}, packed);
  }
  if (bad) atomicOr(err, 1u);
}

template <int D>
__global__ __launch_bounds__(kBlock) void k_cell_coords(const float* __restrict__ soa, int64_t n,
                                                        int d_rt, const double* __restrict__ R,
                                                        const double* __restrict__ u, double inv_c,
                                                        int64_t* __restrict__ kappa,
                                                        uint32_t* err) {
  const int d = D > 0 ? D : d_rt;
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i >= n) return;
  float p[D > 0 ? D : 1];
  if (D > 0) {
#pragma unroll
    for (int l = 0; l < (D > 0 ? D : 1); ++l) p[l] = soa[(int64_t)l * n + i];
  }
  bool bad = false;
  for (int j = 0; j < d; ++j) {
    double y = cell_y<D>(R + (size_t)j * d, p, soa, n, i, d, inv_c, u[j]);
    bool ok = fabs(y) < 2147483648.0;
    bad |= !ok;
    kappa[i * d + j] = ok ? (int64_t)(int32_t)floor(y) : 0;
  }
  if (bad) atomicOr(err, 1u);
}

// ---------------------------------------------------------------------------
// scan: 256 threads x 8 consecutive elements per block.

constexpr int kScanItems = 8;
constexpr int kScanTile = kBlock * kScanItems;
// Up to this many tile sums, every apply block adds up its predecessors' sums
// itself (at most 8 KB read per block).
constexpr int kFusedScanSums = 2048;

// With dcount the element count is min(count, *dcount): count is then the
// grid's capacity and the elements beyond the device count read as zero.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_scan_reduce(const T* __restrict__ in, size_t count,
                                                        T* __restrict__ sums,
                                                        const uint32_t* __restrict__ dcount) {
  __shared__ T wsum[kWaves];
  if (dcount) count = min(count, (size_t)*dcount);
  const size_t base = (size_t)blockIdx.x * kScanTile + (size_t)threadIdx.x * kScanItems;
  T s = 0;
#pragma unroll
  for (int q = 0; q < kScanItems; ++q)
    if (base + q < count) s += in[base + q];
  T total;
  block_exclusive_scan<T>(s, wsum, total);
  if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

// Scans each block's tile and adds its offset: offsets[block] (already
// scanned), or with FROM_SUMS the sum of the earlier blocks' tile sums, added
// up by the block itself (no separate scan of the sums; for few blocks).
template <typename T, bool FROM_SUMS = false>
__global__ __launch_bounds__(kBlock) void k_scan_apply(const T* in, T* out, size_t count,
                                                       const T* __restrict__ offsets, T* total,
                                                       const uint32_t* __restrict__ dcount) {
  __shared__ T wsum[kWaves];
  if (dcount) count = min(count, (size_t)*dcount);
  T from_sums = 0;
  if (FROM_SUMS) {
    T part = 0;
    for (uint32_t p = threadIdx.x; p < blockIdx.x; p += kBlock) part += offsets[p];
    block_exclusive_scan<T>(part, wsum, from_sums);
  }
  const size_t base = (size_t)blockIdx.x * kScanTile + (size_t)threadIdx.x * kScanItems;
  T v[kScanItems];
  T s = 0;
#pragma unroll
  for (int q = 0; q < kScanItems; ++q) {
    v[q] = (base + q < count) ? in[base + q] : (T)0;
    s += v[q];
  }
  T tile_total;
  T run = block_exclusive_scan<T>(s, wsum, tile_total);
  const T off = FROM_SUMS ? from_sums : (offsets ? offsets[blockIdx.x] : (T)0);
  run += off;
#pragma unroll
  for (int q = 0; q < kScanItems; ++q) {
    if (base + q < count) out[base + q] = run;
    run += v[q];
  }
  if (total && blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) *total = off + tile_total;
}

// ---------------------------------------------------------------------------
// radix sort: tiles of 4096 elements; element e of a tile is held by wave
// e / 1024, round (e % 1024) / 64, lane e % 64, so every load is one
// contiguous 64-element run.  Two drivers share the tile code:
//   reduce-then-scan (the default): per pass, tile histograms, a
//     device-wide scan, then the scatter (one more read of the keys per
//     pass); it can sort within segments, leaving their bits out of the
//     passes;
//   onesweep: one histogram read for all digit passes, then per pass one
//     kernel in which each tile takes the next tile id, publishes its digit
//     counts and looks back over earlier tiles' published counts (decoupled
//     look-back) to find where its digits start; its look-back reads cross
//     the XCDs' L2s, and it measured slower.

// LDS of one tile: staged keys/values and the per-wave digit counters.
// (Values are staged in key[] too, after the keys have gone out: the tile
// needs no separate value area, so a sort with values keeps the occupancy of
// one without.)
template <bool HAS_VAL>
struct TileLds {
  uint64_t key[kTile];
  uint32_t wcnt[kWaves][256];
  uint32_t dstart[256];
  uint64_t goff[256];
  uint32_t wsum[kWaves];
};

// Loads tile `tile` and ranks every element among the elements of its wave
// with the same digit (stable: wave order, then round, then lane).  After
// the call wcnt[w][dg] holds wave w's count of digit dg.  Every key (and
// value) of the thread is loaded before the first is ranked: the ranking
// rounds are ordered by wave-level fences, which kept each round's load
// behind the round before (a pass over 32e6 keys with values 218 -> 161 us;
// over 160e3 keys, where the chain was the whole time, 12.5 -> 9.9 us).
template <bool HAS_VAL, int NB>
__device__ __forceinline__ void tile_rank_n(TileLds<HAS_VAL>& S, size_t wave_base, size_t tile_end,
                                            int shift, int nbits, const uint64_t* k_,
                                            uint32_t* r_) {
  const uint32_t lane = lane_id();
  const int w = threadIdx.x >> 6;
  const uint32_t mask = (1u << nbits) - 1u;
  const uint64_t lt = (1ull << lane) - 1ull;
#pragma unroll
  for (int q = 0; q < kKeysPerThread; ++q) {
    const bool valid = wave_base + (size_t)q * 64 + lane < tile_end;
    const uint32_t dg = (uint32_t)(k_[q] >> shift) & mask;
    uint64_t peers = ballot(valid);
    auto match = [&](int b) {
      const bool bit = (dg >> b) & 1u;
      const uint64_t m = ballot(bit);
      peers &= bit ? m : ~m;
    };
    if constexpr (NB > 0) {
#pragma unroll
      for (int b = 0; b < NB; ++b) match(b);
    } else {
      for (int b = 0; b < nbits; ++b) match(b);
    }
    uint32_t before = 0;
    if (valid) before = S.wcnt[w][dg];
    r_[q] = before + (uint32_t)__popcll(peers & lt);
    wave_lds_sync();
    if (valid && (peers & lt) == 0ull) S.wcnt[w][dg] = before + (uint32_t)__popcll(peers);
    wave_lds_sync();
  }
}

template <bool HAS_VAL>
__device__ __forceinline__ void tile_rank(TileLds<HAS_VAL>& S, const uint64_t* __restrict__ kin,
                                          const uint32_t* __restrict__ vin, size_t tile_base,
                                          size_t tile_end, int shift, int nbits, uint64_t* k_,
                                          uint32_t* v_, uint32_t* r_) {
  const uint32_t lane = lane_id();
  const int w = threadIdx.x >> 6;
  const size_t wave_base = tile_base + (size_t)w * (kTile / kWaves);
  // (a tile holds at least one key: elements past its end read its last)
#pragma unroll
  for (int q = 0; q < kKeysPerThread; ++q) {
    const size_t e = min(wave_base + (size_t)q * 64 + lane, tile_end - 1);
    k_[q] = kin[e];
    if (HAS_VAL) v_[q] = vin[e];
  }
#pragma unroll
  for (int q = 0; q < kWaves; ++q) S.wcnt[q][threadIdx.x] = 0u;
  __syncthreads();
  if (nbits == kRadixBits) tile_rank_n<HAS_VAL, kRadixBits>(S, wave_base, tile_end, shift, nbits, k_, r_);
  else tile_rank_n<HAS_VAL, 0>(S, wave_base, tile_end, shift, nbits, k_, r_);
  __syncthreads();
}

// Thread dg: the tile's count of digit dg; sets dstart[dg] (its first
// position in the tile) and turns wcnt[w][dg] into wave w's first position.
template <bool HAS_VAL>
__device__ __forceinline__ uint32_t tile_layout(TileLds<HAS_VAL>& S) {
  const uint32_t dg = threadIdx.x;
  uint32_t c[kWaves];
  uint32_t tot = 0;
#pragma unroll
  for (int q = 0; q < kWaves; ++q) {
    c[q] = S.wcnt[q][dg];
    tot += c[q];
  }
  uint32_t all;
  const uint32_t start = block_exclusive_scan<uint32_t>(tot, S.wsum, all);
  S.dstart[dg] = start;
  uint32_t run = start;
#pragma unroll
  for (int q = 0; q < kWaves; ++q) {
    S.wcnt[q][dg] = run;
    run += c[q];
  }
  return tot;
}

// Sorts the tile into LDS and writes it out at goff[dg] + rank in digit.
template <bool HAS_VAL>
__device__ __forceinline__ void tile_scatter(TileLds<HAS_VAL>& S, uint64_t* __restrict__ kout,
                                             uint32_t* __restrict__ vout, size_t count,
                                             size_t tile_base, size_t tile_end, int shift,
                                             int nbits, const uint64_t* k_, const uint32_t* v_,
                                             const uint32_t* r_) {
  const uint32_t lane = lane_id();
  const int w = threadIdx.x >> 6;
  const uint32_t mask = (1u << nbits) - 1u;
  const size_t wave_base = tile_base + (size_t)w * (kTile / kWaves);
  uint32_t pos_[HAS_VAL ? kKeysPerThread : 1];
#pragma unroll
  for (int q = 0; q < kKeysPerThread; ++q) {
    const size_t e = wave_base + (size_t)q * 64 + lane;
    if (e < tile_end) {
      const uint32_t dg = (uint32_t)(k_[q] >> shift) & mask;
      const uint32_t pos = S.wcnt[w][dg] + r_[q];
      S.key[pos] = k_[q];
      if (HAS_VAL) pos_[q] = pos;
    }
  }
  __syncthreads();
  const size_t rem = tile_end - tile_base;
  const uint32_t tile_count = rem < (size_t)kTile ? (uint32_t)rem : (uint32_t)kTile;
  // the digit of each slot this thread writes out, a byte each, for the values
  uint32_t dg4[HAS_VAL ? kKeysPerThread / 4 : 1] = {};
#pragma unroll 4
  for (int q = 0; q < kKeysPerThread; ++q) {
    const uint32_t s = (uint32_t)q * kBlock + threadIdx.x;
    if (s < tile_count) {
      const uint64_t key = S.key[s];
      const uint32_t dg = (uint32_t)(key >> shift) & mask;
      const uint64_t g = S.goff[dg] + (s - S.dstart[dg]);
      if (g < count) kout[g] = key;  // always in range when the offsets are right
      if (HAS_VAL) dg4[q / 4] |= dg << (8 * (q % 4));
    }
  }
  if (HAS_VAL) {
    // the values through the same slots, once every key has been read out
    __syncthreads();
    uint32_t* sval = reinterpret_cast<uint32_t*>(S.key);
#pragma unroll
    for (int q = 0; q < kKeysPerThread; ++q) {
      const size_t e = wave_base + (size_t)q * 64 + lane;
      if (e < tile_end) sval[pos_[q]] = v_[q];
    }
    __syncthreads();
#pragma unroll 4
    for (int q = 0; q < kKeysPerThread; ++q) {
      const uint32_t s = (uint32_t)q * kBlock + threadIdx.x;
      if (s < tile_count) {
        const uint32_t dg = (dg4[q / 4] >> (8 * (q % 4))) & 0xFFu;
        const uint64_t g = S.goff[dg] + (s - S.dstart[dg]);
        if (g < count) vout[g] = sval[s];
      }
    }
  }
}

// --- reduce-then-scan ---------------------------------------------------------

// Tile b of a sort: its keys [start, start + len) and the place of its
// digit counts in the histogram table, slot + digit * stride.  Without a
// table, tile b is keys [b kTile, ...) with slot b and stride ntiles; with
// one, tiles stay inside segments and the table is segment-major, so its
// exclusive scan orders by segment, then digit, then tile.
struct TileSpan {
  size_t start, end;
  size_t slot, stride;
};
__device__ __forceinline__ TileSpan tile_span(const SortTile* tiles, size_t count,
                                              uint32_t ntiles, uint32_t b) {
  TileSpan t;
  if (tiles) {
    const SortTile d = tiles[b];
    t.start = d.start;
    t.end = d.start + d.len;
    t.slot = d.slot;
    t.stride = d.stride;
  } else {
    t.start = (size_t)b * kTile;
    t.end = min(count, t.start + (size_t)kTile);
    t.slot = b;
    t.stride = ntiles;
  }
  return t;
}

__global__ __launch_bounds__(kBlock) void k_radix_hist(const uint64_t* __restrict__ keys,
                                                       size_t count, int shift, int nbits,
                                                       uint32_t* __restrict__ tile_hist,
                                                       uint32_t ntiles,
                                                       const SortTile* __restrict__ tiles) {
  __shared__ uint32_t h[256];
  const uint32_t mask = (1u << nbits) - 1u;
  const TileSpan t = tile_span(tiles, count, ntiles, blockIdx.x);
  uint64_t k_[kKeysPerThread];  // every load in flight before the first count
#pragma unroll
  for (int q = 0; q < kKeysPerThread; ++q)
    k_[q] = keys[min(t.start + (size_t)q * kBlock + threadIdx.x, t.end - 1)];
  h[threadIdx.x] = 0u;
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kKeysPerThread; ++q) {
    const size_t e = t.start + (size_t)q * kBlock + threadIdx.x;
    if (e < t.end) atomicAdd(&h[(uint32_t)(k_[q] >> shift) & mask], 1u);
  }
  __syncthreads();
  tile_hist[t.slot + (size_t)threadIdx.x * t.stride] = h[threadIdx.x];
}

template <bool HAS_VAL>
__global__ __launch_bounds__(kBlock) void k_radix_scatter(
    const uint64_t* __restrict__ kin, const uint32_t* __restrict__ vin, uint64_t* __restrict__ kout,
    uint32_t* __restrict__ vout, size_t count, int shift, int nbits,
    const uint32_t* __restrict__ tile_off, uint32_t ntiles, const SortTile* __restrict__ tiles) {
  __shared__ TileLds<HAS_VAL> S;
  uint64_t k_[kKeysPerThread];
  uint32_t v_[kKeysPerThread];
  uint32_t r_[kKeysPerThread];
  const TileSpan t = tile_span(tiles, count, ntiles, blockIdx.x);
  tile_rank<HAS_VAL>(S, kin, vin, t.start, t.end, shift, nbits, k_, v_, r_);
  tile_layout<HAS_VAL>(S);
  S.goff[threadIdx.x] = tile_off[t.slot + (size_t)threadIdx.x * t.stride];
  __syncthreads();
  tile_scatter<HAS_VAL>(S, kout, vout, count, t.start, t.end, shift, nbits, k_, v_, r_);
}

// --- short segments -------------------------------------------------------------

// One block sorts one segment of at most kSegSortKeys keys: every pass of the
// radix sort on keys held in registers and exchanged through LDS, in place of
// a histogram, its scan and a scatter per pass over all segments (seven or so
// launches of a few microseconds each, whose time the keys hardly show:
// 25 segments of 6400 keys, three passes: 66 us, now 18).  Two segments are
// enough for it: calls of 4200, 9000 and 16384 points gain with 2 grids (d = 6:
// 233 -> 172, 251 -> 183, 254 -> 204 us, of which this is a part) as with 25.
// Wave w holds elements [64 w items, 64 (w + 1) items), items = ceil(len /
// 1024), so ranks are stable as in tile_rank.
constexpr int kSegThreads = 1024;
constexpr int kSegWaves = kSegThreads / 64;
constexpr int kSegItems = kSegSortKeys / kSegThreads;

__global__ __launch_bounds__(kSegThreads) void k_seg_sort(uint64_t* __restrict__ keys,
                                                          const SortTile* __restrict__ segs,
                                                          int begin_bit, int end_bit) {
  __shared__ uint64_t skey[kSegSortKeys];
  __shared__ uint32_t wcnt[kSegWaves][256];
  __shared__ uint32_t wsum[kWaves];
  const SortTile seg = segs[blockIdx.x];
  uint64_t* base = keys + seg.start;
  const uint32_t len = seg.len;
  const uint32_t lane = lane_id();
  const uint32_t w = uniform(threadIdx.x >> 6);
  const uint32_t items = (len + kSegThreads - 1) / kSegThreads;
  const uint32_t e0 = w * 64u * items + lane;
  const uint64_t lt = (1ull << lane) - 1ull;
  uint64_t k_[kSegItems];
  uint32_t r_[kSegItems];
#pragma unroll
  for (int q = 0; q < kSegItems; ++q)
    if ((uint32_t)q < items) k_[q] = base[min(e0 + 64u * q, len - 1u)];
  for (int b = begin_bit; b < end_bit; b += kRadixBits) {
    const int nbits = min(kRadixBits, end_bit - b);
    const uint32_t mask = (1u << nbits) - 1u;
    for (uint32_t x = threadIdx.x; x < kSegWaves * 256u; x += kSegThreads) (&wcnt[0][0])[x] = 0u;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kSegItems; ++q) {
      if ((uint32_t)q >= items) break;
      const bool valid = e0 + 64u * q < len;
      const uint32_t dg = (uint32_t)(k_[q] >> b) & mask;
      uint64_t peers = ballot(valid);
      for (int x = 0; x < nbits; ++x) {
        const bool bit = (dg >> x) & 1u;
        const uint64_t m = ballot(bit);
        peers &= bit ? m : ~m;
      }
      uint32_t before = 0;
      if (valid) before = wcnt[w][dg];
      r_[q] = before + (uint32_t)__popcll(peers & lt);
      wave_lds_sync();
      if (valid && (peers & lt) == 0ull) wcnt[w][dg] = before + (uint32_t)__popcll(peers);
      wave_lds_sync();
    }
    __syncthreads();
    // thread dg: the digit's first place, then each wave's (the first four
    // waves scan; every thread meets the barriers)
    uint32_t c[kSegWaves], tot = 0, inc = 0;
    if (threadIdx.x < 256u) {
#pragma unroll
      for (int x = 0; x < kSegWaves; ++x) {
        c[x] = wcnt[x][threadIdx.x];
        tot += c[x];
      }
      inc = wave_inclusive_scan(tot);
      if (lane == 63) wsum[w] = inc;
    }
    __syncthreads();
    if (threadIdx.x < 256u) {
      uint32_t run = inc - tot;
#pragma unroll
      for (int x = 0; x < kWaves; ++x)
        if ((uint32_t)x < w) run += wsum[x];
#pragma unroll
      for (int x = 0; x < kSegWaves; ++x) {
        wcnt[x][threadIdx.x] = run;
        run += c[x];
      }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kSegItems; ++q)
      if ((uint32_t)q < items && e0 + 64u * q < len)
        skey[wcnt[w][(uint32_t)(k_[q] >> b) & mask] + r_[q]] = k_[q];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kSegItems; ++q)
      if ((uint32_t)q < items) k_[q] = skey[min(e0 + 64u * q, len - 1u)];
  }
#pragma unroll
  for (int q = 0; q < kSegItems; ++q)
    if ((uint32_t)q < items && e0 + 64u * q < len) base[e0 + 64u * q] = k_[q];
}

// --- onesweep -------------------------------------------------------------------

constexpr int kHistBlockTiles = 4;  // tiles per block of the all-pass histogram
constexpr int kMaxPasses = 8;

// part[block][p][dg]: this block's count of digit dg in pass p.
__global__ __launch_bounds__(kBlock) void k_hist_all(const uint64_t* __restrict__ keys,
                                                     size_t count, int begin_bit, int end_bit,
                                                     uint32_t* __restrict__ part) {
  __shared__ uint32_t h[kWaves][kMaxPasses][256];
  const int w = threadIdx.x >> 6;
  const int npass = (end_bit - begin_bit + kRadixBits - 1) / kRadixBits;
  for (int p = 0; p < npass; ++p)
#pragma unroll
    for (int q = 0; q < kWaves; ++q) h[q][p][threadIdx.x] = 0u;
  __syncthreads();
  const size_t base = (size_t)blockIdx.x * kHistBlockTiles * kTile;
  for (int q = 0; q < kHistBlockTiles * kKeysPerThread; ++q) {
    const size_t e = base + (size_t)q * kBlock + threadIdx.x;
    if (e >= count) break;
    const uint64_t key = keys[e];
    for (int p = 0; p < npass; ++p) {
      const int b = begin_bit + p * kRadixBits;
      const int nb = min(kRadixBits, end_bit - b);
      atomicAdd(&h[w][p][(uint32_t)(key >> b) & ((1u << nb) - 1u)], 1u);
    }
  }
  __syncthreads();
  for (int p = 0; p < npass; ++p) {
    uint32_t s = 0;
#pragma unroll
    for (int q = 0; q < kWaves; ++q) s += h[q][p][threadIdx.x];
    part[((size_t)blockIdx.x * npass + p) * 256 + threadIdx.x] = s;
  }
}

// One block per pass: digit_off[p][dg] = number of keys with a smaller digit.
__global__ __launch_bounds__(kBlock) void k_hist_scan(const uint32_t* __restrict__ part,
                                                      uint32_t nblocks, int npass,
                                                      uint64_t* __restrict__ digit_off) {
  __shared__ uint64_t wsum[kWaves];
  const int p = blockIdx.x;
  uint64_t s = 0;
  for (uint32_t b = 0; b < nblocks; ++b) s += part[((size_t)b * npass + p) * 256 + threadIdx.x];
  uint64_t all;
  digit_off[p * 256 + threadIdx.x] = block_exclusive_scan<uint64_t>(s, wsum, all);
}

// Status word of (tile, digit): flag in the top two bits (0 not yet
// published, 1 this tile's count, 2 count of this and all earlier tiles).
constexpr uint64_t kStAggregate = 1ull << 62;
constexpr uint64_t kStInclusive = 2ull << 62;
constexpr uint64_t kStValue = (1ull << 62) - 1ull;
constexpr uint32_t kSpinLimit = 1u << 22;

template <bool HAS_VAL>
__global__ __launch_bounds__(kBlock) void k_onesweep(
    const uint64_t* __restrict__ kin, const uint32_t* __restrict__ vin, uint64_t* __restrict__ kout,
    uint32_t* __restrict__ vout, size_t count, int shift, int nbits,
    const uint64_t* __restrict__ digit_off, unsigned long long* status, unsigned int* tile_counter,
    unsigned int* err) {
  __shared__ TileLds<HAS_VAL> S;
  __shared__ uint32_t s_tile;
  // Tile ids in the order blocks start: every earlier tile is already
  // running, so each look-back wait ends.
  if (threadIdx.x == 0) s_tile = atomicAdd(tile_counter, 1u);
  __syncthreads();
  const size_t tile = s_tile;
  uint64_t k_[kKeysPerThread];
  uint32_t v_[kKeysPerThread];
  uint32_t r_[kKeysPerThread];
  const size_t tile_base = tile * kTile;
  const size_t tile_end = min(count, tile_base + (size_t)kTile);
  tile_rank<HAS_VAL>(S, kin, vin, tile_base, tile_end, shift, nbits, k_, v_, r_);
  const uint32_t tot = tile_layout<HAS_VAL>(S);
  const uint32_t dg = threadIdx.x;
  if (dg < (1u << nbits)) {
    unsigned long long* mine = status + tile * 256 + dg;
    __hip_atomic_store(mine, kStAggregate | (uint64_t)tot, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
    uint64_t excl = 0;
    for (size_t p = tile; p-- > 0;) {
      uint64_t st;
      uint32_t spins = 0;
      do {
        st = __hip_atomic_load(status + p * 256 + dg, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      } while ((st >> 62) == 0 && ++spins < kSpinLimit);
      if ((st >> 62) == 0) {  // never published: give up, report, keep writes in bounds
        atomicOr(err, 2u);
        break;
      }
      excl += st & kStValue;
      if ((st >> 62) == 2) break;
    }
    __hip_atomic_store(mine, kStInclusive | (excl + tot), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
    S.goff[dg] = digit_off[dg] + excl;
  }
  __syncthreads();
  tile_scatter<HAS_VAL>(S, kout, vout, count, tile_base, tile_end, shift, nbits, k_, v_, r_);
}

// ---------------------------------------------------------------------------
// runs of equal keys (cells with >= 2 points), unique keys.

// Run heads and tails: whether an element begins or ends a run of at least
// two equal keys.  A wave takes 1024 consecutive elements in 16 groups of
// 64; its keys and the keys beyond its two ends are all loaded first (loads
// that waited for each group in turn made this kernel a serial chain of 16
// memory latencies: 17 -> 4.8 us at 160e3 keys, 123 -> 67 us at 32e6), and a
// group's neighbours come from the adjacent lanes and groups.
__global__ __launch_bounds__(kBlock) void k_run_count(const uint64_t* __restrict__ keys,
                                                      size_t count, int shift, uint32_t* head_cnt,
                                                      uint32_t* tail_cnt,
                                                      uint64_t* __restrict__ masks) {
  __shared__ uint32_t sh[kWaves], st[kWaves];
  const uint32_t lane = lane_id();
  const int w = threadIdx.x >> 6;
  const size_t wave_base = (size_t)blockIdx.x * kTile + (size_t)w * (kTile / kWaves);
  const size_t ngroups = (count + 63) / 64;
  uint64_t k_[kKeysPerThread];
#pragma unroll
  for (int q = 0; q < kKeysPerThread; ++q)
    k_[q] = keys[min(wave_base + (size_t)q * 64 + lane, count - 1)] >> shift;
  const uint64_t before = keys[min(wave_base ? wave_base - 1 : 0, count - 1)] >> shift;
  const uint64_t after = keys[min(wave_base + kTile / kWaves, count - 1)] >> shift;
  uint32_t hc = 0, tc = 0;
#pragma unroll
  for (int q = 0; q < kKeysPerThread; ++q) {
    const size_t e = wave_base + (size_t)q * 64 + lane;
    const uint64_t k = k_[q];
    uint64_t kp = __shfl_up(k, 1, 64);
    uint64_t kn = __shfl_down(k, 1, 64);
    const uint64_t last = q ? lane_value((unsigned long long)k_[q ? q - 1 : 0], 63) : before;
    const uint64_t first =
        q + 1 < kKeysPerThread
            ? lane_value((unsigned long long)k_[q + 1 < kKeysPerThread ? q + 1 : 0], 0)
            : after;
    if (lane == 0) kp = last;
    if (lane == 63) kn = first;
    const bool in = e < count;
    const bool prev_same = in && e > 0 && kp == k;
    const bool next_same = in && e + 1 < count && kn == k;
    const uint64_t hb = ballot(!prev_same && next_same), tb = ballot(prev_same && !next_same);
    hc += (uint32_t)__popcll(hb);
    tc += (uint32_t)__popcll(tb);
    // the writing kernel reads these bits instead of the keys again
    const size_t g = (wave_base >> 6) + (size_t)q;
    if (g < ngroups && lane < 2) masks[2 * g + lane] = lane ? tb : hb;
  }
  if (lane == 0) {
    sh[w] = hc;
    st[w] = tc;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t a = 0, b = 0;
    for (int q = 0; q < kWaves; ++q) {
      a += sh[q];
      b += st[q];
    }
    head_cnt[blockIdx.x] = a;
    tail_cnt[blockIdx.x] = b;
  }
}

// head_off / tail_off: each tile's scanned offsets, or with FROM_COUNTS the
// raw per-tile counts, which each block then adds up for the tiles before it
// itself (the last block writes the totals to tot; block 0 clears *zero).
template <bool FROM_COUNTS>
__global__ __launch_bounds__(kBlock) void k_run_write(const uint64_t* __restrict__ masks,
                                                      size_t count,
                                                      const uint32_t* __restrict__ head_off,
                                                      const uint32_t* __restrict__ tail_off,
                                                      uint32_t* __restrict__ start,
                                                      uint32_t* __restrict__ end,
                                                      uint32_t* __restrict__ tot,
                                                      unsigned long long* __restrict__ zero) {
  __shared__ uint32_t sh[kWaves], st[kWaves];
  __shared__ uint32_t wsum[kWaves];
  const uint32_t lane = lane_id();
  const int w = threadIdx.x >> 6;
  const size_t wave_base = (size_t)blockIdx.x * kTile + (size_t)w * (kTile / kWaves);
  const size_t ngroups = (count + 63) / 64;
  // lane 2 q / 2 q + 1 holds the head / tail bits of the wave's group q
  static_assert(2 * kKeysPerThread <= 64, "one mask word per lane");
  unsigned long long mword = 0;
  if (lane < 2 * kKeysPerThread && (wave_base >> 6) + lane / 2 < ngroups)
    mword = masks[2 * (wave_base >> 6) + lane];
  uint32_t hc = 0, tc = 0;
#pragma unroll
  for (int q = 0; q < kKeysPerThread; ++q) {
    hc += (uint32_t)__popcll(lane_value(mword, 2 * q));
    tc += (uint32_t)__popcll(lane_value(mword, 2 * q + 1));
  }
  if (lane == 0) {
    sh[w] = hc;
    st[w] = tc;
  }
  __syncthreads();
  uint32_t hbase, tbase;
  if (FROM_COUNTS) {
    uint32_t ph = 0, pt = 0;
    for (uint32_t b = threadIdx.x; b < blockIdx.x; b += kBlock) {
      ph += head_off[b];
      pt += tail_off[b];
    }
    block_exclusive_scan<uint32_t>(ph, wsum, hbase);
    block_exclusive_scan<uint32_t>(pt, wsum, tbase);
    if (threadIdx.x == 0 && blockIdx.x == gridDim.x - 1) {
      uint32_t a = 0, b = 0;
      for (int q = 0; q < kWaves; ++q) {
        a += sh[q];
        b += st[q];
      }
      tot[0] = hbase + a;
      tot[1] = tbase + b;
    }
    if (zero && threadIdx.x == 0 && blockIdx.x == 0) *zero = 0ull;
  } else {
    hbase = head_off[blockIdx.x];
    tbase = tail_off[blockIdx.x];
  }
  for (int q = 0; q < w; ++q) {
    hbase += sh[q];
    tbase += st[q];
  }
#pragma unroll
  for (int q = 0; q < kKeysPerThread; ++q) {
    const size_t e = wave_base + (size_t)q * 64 + lane;
    const uint64_t hb = lane_value(mword, 2 * q), tbm = lane_value(mword, 2 * q + 1);
    const bool h = (hb >> lane) & 1ull, t = (tbm >> lane) & 1ull;
    if (h) start[hbase + rank_below(hb)] = (uint32_t)e;
    if (t) end[tbase + rank_below(tbm)] = (uint32_t)(e + 1);
    hbase += (uint32_t)__popcll(hb);
    tbase += (uint32_t)__popcll(tbm);
  }
}

__global__ __launch_bounds__(kBlock) void k_cell_work(const uint32_t* __restrict__ start,
                                                      const uint32_t* __restrict__ end,
                                                      uint32_t ncells,
                                                      const uint32_t* __restrict__ dcells,
                                                      uint32_t cell_unit_tiles,
                                                      uint32_t* __restrict__ units,
                                                      uint64_t* __restrict__ tests,
                                                      unsigned long long* members) {
  // cells [0, ncells), or [0, min(ncells, *dcells)) with the device count
  if (dcells) ncells = min(ncells, *dcells);
  uint64_t L = 0;
  for (uint32_t c = blockIdx.x * blockDim.x + threadIdx.x; c < ncells;
       c += gridDim.x * blockDim.x) {
    const uint64_t Lc = end[c] - start[c];
    const uint32_t nt = (uint32_t)((Lc + kPairTile - 1) / kPairTile);
    units[c] = nt <= cell_unit_tiles ? 1u : nt;
    tests[c] = Lc * (Lc - 1) / 2;
    L += Lc;
  }
  // one atomic per block: a single counter's device-scope atomics serialise
  // across the XCDs
  __shared__ unsigned long long wm[kWaves];
  unsigned long long m = L;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) m += __shfl_xor(m, o, 64);
  if (lane_id() == 0) wm[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long all = 0;
#pragma unroll
    for (int q = 0; q < kWaves; ++q) all += wm[q];
    if (all) atomicAdd(members, all);
  }
}

// k_cell_work by scan tiles: block b takes cells [b kScanTile, (b + 1)
// kScanTile), kScanItems consecutive cells per thread as the scan kernels
// hold them, and also writes the tile's sums of units and tests, so that
// the two scans need only their apply launches (each block adds up the
// sums before its own tile).
__global__ __launch_bounds__(kBlock) void k_cell_work_tiles(
    const uint32_t* __restrict__ start, const uint32_t* __restrict__ end, uint32_t ncells,
    const uint32_t* __restrict__ dcells, uint32_t cell_unit_tiles, uint32_t* __restrict__ units,
    uint64_t* __restrict__ tests, unsigned long long* members, uint32_t* __restrict__ usums,
    uint64_t* __restrict__ tsums) {
  if (dcells) ncells = min(ncells, *dcells);
  const size_t base = (size_t)blockIdx.x * kScanTile + (size_t)threadIdx.x * kScanItems;
  uint64_t L = 0, tt = 0;
  uint32_t uu = 0;
#pragma unroll
  for (int q = 0; q < kScanItems; ++q) {
    const size_t c = base + q;
    if (c < ncells) {
      const uint64_t Lc = end[c] - start[c];
      const uint32_t nt = (uint32_t)((Lc + kPairTile - 1) / kPairTile);
      const uint32_t u = nt <= cell_unit_tiles ? 1u : nt;
      const uint64_t t = Lc * (Lc - 1) / 2;
      units[c] = u;
      tests[c] = t;
      uu += u;
      tt += t;
      L += Lc;
    }
  }
  __shared__ unsigned long long wl[kWaves], wt[kWaves];
  __shared__ uint32_t wu[kWaves];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    L += __shfl_xor(L, o, 64);
    tt += __shfl_xor(tt, o, 64);
    uu += __shfl_xor(uu, o, 64);
  }
  if (lane_id() == 0) {
    wl[threadIdx.x >> 6] = L;
    wt[threadIdx.x >> 6] = tt;
    wu[threadIdx.x >> 6] = uu;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long all = 0, tall = 0;
    uint32_t uall = 0;
#pragma unroll
    for (int q = 0; q < kWaves; ++q) {
      all += wl[q];
      tall += wt[q];
      uall += wu[q];
    }
    usums[blockIdx.x] = uall;
    tsums[blockIdx.x] = tall;
    if (all) atomicAdd(members, all);
  }
}

__global__ __launch_bounds__(kBlock) void k_unique_count(const uint64_t* __restrict__ keys,
                                                         size_t count, uint32_t* tile_cnt) {
  __shared__ uint32_t sh[kWaves];
  const uint32_t lane = lane_id();
  const int w = threadIdx.x >> 6;
  const size_t wave_base = (size_t)blockIdx.x * kTile + (size_t)w * (kTile / kWaves);
  uint32_t c = 0;
  for (int q = 0; q < kKeysPerThread; ++q) {
    const size_t e = wave_base + (size_t)q * 64 + lane;
    const bool f = e < count && (e == 0 || keys[e] != keys[e - 1]);
    c += (uint32_t)__popcll(ballot(f));
  }
  if (lane == 0) sh[w] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t a = 0;
    for (int q = 0; q < kWaves; ++q) a += sh[q];
    tile_cnt[blockIdx.x] = a;
  }
}

__global__ __launch_bounds__(kBlock) void k_unique_write(const uint64_t* __restrict__ keys,
                                                         size_t count,
                                                         const uint32_t* __restrict__ tile_off,
                                                         uint64_t* __restrict__ out) {
  __shared__ uint32_t sh[kWaves];
  const uint32_t lane = lane_id();
  const int w = threadIdx.x >> 6;
  const size_t wave_base = (size_t)blockIdx.x * kTile + (size_t)w * (kTile / kWaves);
  uint32_t fmask = 0, c = 0;
  for (int q = 0; q < kKeysPerThread; ++q) {
    const size_t e = wave_base + (size_t)q * 64 + lane;
    const bool f = e < count && (e == 0 || keys[e] != keys[e - 1]);
    fmask |= (uint32_t)f << q;
    c += (uint32_t)__popcll(ballot(f));
  }
  if (lane == 0) sh[w] = c;
  __syncthreads();
  uint32_t base = tile_off[blockIdx.x];
  for (int q = 0; q < w; ++q) base += sh[q];
  for (int q = 0; q < kKeysPerThread; ++q) {
    const size_t e = wave_base + (size_t)q * 64 + lane;
    const bool f = (fmask >> q) & 1u;
    const uint64_t m = ballot(f);
    if (f) out[base + rank_below(m)] = keys[e];
    base += (uint32_t)__popcll(m);
  }
}

// ---------------------------------------------------------------------------
// cell pairs.  A work unit is (cell, tile a) with tiles of 64 points; its wave
// tests tile a against the tiles b >= a of the same cell.  Unit points are
// read by sorted position from spts / ssig (gathered once), so every tile
// load is a direct, coalesced read; the next B tile is loaded while the
// current one is tested.  Accepted pairs go through the first-owner filter
// (a pair is kept only if no earlier grid put both points in one cell: the
// signature words of the two points are compared) and are written as
// (min << pair_bits) | max.

constexpr int kSigWords = 2;  // signature words kept per point (more: read on demand)
constexpr int kOutBuf = 256;  // staged pairs per wave

// Whether x = a ^ b (signature words of two points within r) has an all-zero
// group among the first n groups: with L the lowest and H the highest bit of
// every group, (x - L) & ~x & H is nonzero exactly when some group of x is
// zero; a borrow only runs upward, out of a zero group, so masking to the
// first n groups keeps the test exact.
__device__ __forceinline__ bool zero_group(uint64_t x, int n, const PairsArgs& P) {
  const uint64_t keep = (n * P.g >= 64) ? ~0ull : ((1ull << (n * P.g)) - 1ull);
  return (((x - P.lows) & ~x & P.highs) & keep) != 0ull;
}

// Signature word q of the point at sorted position p with index i.
__device__ __forceinline__ uint64_t sig_word(const PairsArgs& P, int q, uint32_t p, uint32_t i) {
  return P.direct ? P.sigp[(size_t)i * P.sig_stride + q] : P.ssig[(size_t)q * P.N + p];
}

// Whether a pair of points within r found under grid tcell is not to be
// reported: they shared a cell under a grid t < tcell or, where keys are
// hashes, do not under tcell itself (P.same_cell).  Word q of their
// signatures is aq / bq for q < kSigWords, and is read on demand (the points
// at sorted positions pa, pb with indices ia, ib) beyond that; nw words count.
// HASHED: whether keys may be hashes (the check, unused, cost the matrix-core
// screen 2.5% at uniform d6, so it has a variant without).
template <bool HASHED>
__device__ __forceinline__ bool not_first_owner(const uint64_t* aq, const uint64_t* bq, int tcell,
                                                int nw, uint32_t pa, uint32_t ia, uint32_t pb,
                                                uint32_t ib, const PairsArgs& P) {
  bool drop = false;
#pragma unroll
  for (int q = 0; q < kSigWords; ++q)
    if (q < nw) drop |= zero_group(aq[q] ^ bq[q], min(P.gpw, tcell - q * P.gpw), P);
  for (int q = kSigWords; q < nw && !drop; ++q)
    drop = zero_group(sig_word(P, q, pa, ia) ^ sig_word(P, q, pb, ib),
                      min(P.gpw, tcell - q * P.gpw), P);
  if (HASHED && P.same_cell) {
    // grid tcell's group is in word nw - 1 (unit_view)
    const int x = nw - 1;
    const uint64_t v = x == 0   ? aq[0] ^ bq[0]
                       : x == 1 ? aq[1] ^ bq[1]
                                : sig_word(P, x, pa, ia) ^ sig_word(P, x, pb, ib);
    drop |= (v & (P.same_cell << ((tcell - x * P.gpw) * P.g))) != 0ull;
  }
  return drop;
}

// The MR-metric's FP64 decision for the points ra and rb: the robots' squared
// displacements summed in axis order, their square roots (correctly rounded)
// added in robot order, the sum tested against r.
__device__ __forceinline__ bool mr_within(const float* __restrict__ ra, const float* __restrict__ rb,
                                          int d, const MrInst& I) {
  double s = 0.0;
  for (int o = 0; o < d; o += I.sub) {
    double t = 0.0;
    for (int l = o; l < o + I.sub; ++l) {
      const double dl = (double)ra[l] - (double)rb[l];
      t = t + dl * dl;
    }
    s = s + __builtin_sqrt(t);
  }
  return s <= I.r;
}

// That decision for the points with indices ia and ib of an instance of a
// pass, read again from the rows their tiles were loaded from (they are in
// the caches: a separate pass over the pairs fetched two random rows each,
// 164 us for 5.9e6 pairs at d = 6, beside a copy and a read-back).  In FP32
// first: D differences and products, at most D square roots (1 ulp) and as
// many sums are within a relative (2 D + 8) 2^-24 < 2^-16 of the FP64 value
// where no robot's square underflows to matter (r^2 >= 2^-60: the robots'
// lost squares, below 2^-126 each, add less than 2^-57); FP64 decides the
// rest.  (Pair kernel of 200003 points, d = 6, two robots: 313 us; 437 with
// FP64 for every pair, 280 without the decision and 190 more for the pass.)
template <int D>
__device__ __forceinline__ bool mr_pair(const PairsArgs& P, uint32_t ia, uint32_t ib,
                                        const MrInst& I) {
  const float* ra = P.rows + (size_t)ia * P.row_stride;
  const float* rb = P.rows + (size_t)ib * P.row_stride;
  if (D <= 16 && I.r >= 0x1p-30) {
    float s = 0.0f, t = 0.0f;
    int c = 0;
#pragma unroll
    for (int l = 0; l < D; ++l) {
      const float df = ra[l] - rb[l];
      t = __builtin_fmaf(df, df, t);
      if (++c == I.sub) {
        s += __builtin_amdgcn_sqrtf(t);
        t = 0.0f;
        c = 0;
      }
    }
    const float r = (float)I.r;
    if (s < r * (1.0f - 0x1p-15f)) return true;
    if (s > r * (1.0f + 0x1p-15f)) return false;
  }
  return mr_within(ra, rb, P.d, I);
}

// Point index at sorted position p: the low idx_bits of the sorted key when
// keys carry it, else the separate index array.
__device__ __forceinline__ uint32_t point_at(const PairsArgs& P, uint32_t p) {
  return P.idx_bits ? (uint32_t)(P.skeys[p] & ((1ull << P.idx_bits) - 1ull)) : P.sidx[p];
}

// One tile's data for this lane: coordinates, point index and the first
// signature words.  Lanes past the tile's end hold its last point.
template <int D>
struct TileRegs {
  float c[D];
  uint32_t idx;
  uint64_t sw[kSigWords];
};

// Every lane loads a whole point, no lane or coordinate tested on its own: a
// row's loads then merge into a few wide ones (a test per coordinate made
// each a masked 4-byte gather: at d = 12 the tiles' loads took half of the
// L1's time; clustered d12 pairs 8.70 -> 7.22 ms, uniform d6 532 -> 509 us).
// D <= 16 is the dimension itself; wider D are padded with zeros.
template <int D>
__device__ __forceinline__ void load_tile(const PairsArgs& P, uint32_t p0, uint32_t n, int nw,
                                          uint32_t lane, TileRegs<D>& R) {
  const uint32_t p = p0 + min(lane, n - 1u);  // (n >= 1)
  R.idx = point_at(P, p);
  if (P.direct) {
    const float* row = P.rows + (size_t)R.idx * P.row_stride;
    if constexpr (D <= 16) {
#pragma unroll
      for (int l = 0; l < D; ++l) R.c[l] = row[l];
    } else {
#pragma unroll
      for (int l = 0; l < D; ++l) R.c[l] = l < P.d ? row[l] : 0.0f;
    }
#pragma unroll
    for (int q = 0; q < kSigWords; ++q)
      R.sw[q] = q < nw ? P.sigp[(size_t)R.idx * P.sig_stride + q] : 0ull;
  } else {
#pragma unroll
    for (int l = 0; l < D; ++l)
      R.c[l] = (D <= 16 || l < P.d) ? P.spts[(size_t)l * P.N + p] : 0.0f;
#pragma unroll
    for (int q = 0; q < kSigWords; ++q) R.sw[q] = q < nw ? P.ssig[(size_t)q * P.N + p] : 0ull;
  }
}

// A unit's fields, uniform across the wave (ok = false past the last unit).
struct UnitView {
  uint32_t s0, L, ta_begin, ta_end, nt, inst;
  int tcell, nw;  // grid; signature words to compare (0: no filtering)
  bool ok;
};

template <bool HASHED>
__device__ __forceinline__ UnitView unit_view(const PairsArgs& P, uint32_t u, uint32_t u_end) {
  UnitView v;
  v.ok = u < u_end;
  if (!v.ok) {
    v.s0 = v.L = v.ta_begin = v.ta_end = v.nt = v.inst = 0u;
    v.tcell = v.nw = 0;
    return v;
  }
  const UnitDesc U = P.units[u];
  v.s0 = uniform(U.s0);
  v.L = uniform(U.len);
  v.ta_begin = uniform(U.ta_begin);
  v.ta_end = uniform(U.ta_end);
  v.tcell = (int)uniform(U.t);
  v.inst = uniform(U.inst);
  v.nt = (v.L + kPairTile - 1) / kPairTile;
  // (with hashed keys grid t's own group counts too)
  v.nw = HASHED && P.same_cell           ? v.tcell / P.gpw + 1
         : P.first_owner && v.tcell > 0 ? (v.tcell - 1) / P.gpw + 1
                                        : 0;
  return v;
}

__device__ __forceinline__ uint32_t tile_len(const UnitView& V, uint32_t t) {
  return min((uint32_t)kPairTile, V.L - t * kPairTile);
}

// A row's tile pairs (ta, tb): its diagonal first, then its B tiles from the
// last down to ta + 1, so that a row ends on the next row's own tile.
__device__ __forceinline__ uint32_t row_step_tile(const UnitView& V, uint32_t ta, uint32_t s) {
  return s == 0 ? ta : V.nt - s;
}

// Loads the tile after (ta, tb) in the wave's stream of tile pairs: the
// row's next B tile, else -- the row ending on tile ta + 1 -- that tile again
// (kept from R_cur, not loaded) for the next row, in this unit or in the next
// one when that is the same cell's next row, else the first tile of the next
// unit Vn (nothing when the stream ends).
template <int D>
__device__ __forceinline__ void load_next(const PairsArgs& P, const UnitView& V,
                                          const UnitView& Vn, uint32_t ta, uint32_t tb,
                                          uint32_t lane, const TileRegs<D>& R_cur,
                                          TileRegs<D>& R) {
  uint32_t t = ~0u;  // the unit's next tile to load
  if (tb == ta) {
    if (V.nt > ta + 1) t = V.nt - 1;
  } else if (tb > ta + 1) {
    t = tb - 1;
  } else if (ta + 1 < V.ta_end || (Vn.ok && Vn.s0 == V.s0 && Vn.ta_begin == ta + 1)) {
    R = R_cur;  // tb = ta + 1: the next row's tile, in registers already
    return;
  }
  uint32_t p0 = 0, n = 0;
  int nw = 0;
  if (t != ~0u) {
    p0 = V.s0 + t * kPairTile;
    n = tile_len(V, t);
    nw = V.nw;
  } else if (Vn.ok) {
    p0 = Vn.s0 + Vn.ta_begin * kPairTile;
    n = tile_len(Vn, Vn.ta_begin);
    nw = Vn.nw;
  }
  if (n) load_tile<D>(P, p0, n, nw, lane, R);
}

// Appends this lane's pairs (ai, partner(j)) for the bits j of acc to the
// wave's staging buffer, flushing it to cand as needed.
struct OutStage {
  uint64_t* buf;  // kOutBuf entries of this wave
  uint32_t n = 0;
  uint64_t* dst;               // this block's output segment
  unsigned long long* count;   // and its running total
  uint64_t cap;                // the segment's capacity
  uint32_t seg;
};

__device__ __forceinline__ OutStage out_stage(const PairsArgs& P, uint64_t* buf) {
  OutStage O;
  O.buf = buf;
  O.seg = P.nseg > 1 ? blockIdx.x % P.nseg : 0u;
  O.dst = P.cand + (size_t)O.seg * P.cap;
  O.count = P.cand_count + O.seg;
  O.cap = P.cap;
  return O;
}

// SPREAD: the wave goes on to the next segment.
template <bool SPREAD = false>
__device__ __forceinline__ void flush_out(const PairsArgs& P, OutStage& O, uint32_t lane) {
  wave_lds_sync();
  if (O.n) {
    unsigned long long base = 0;
    if (lane == 0) base = atomicAdd(O.count, (unsigned long long)O.n);
    base = lane_value(base, 0);
    for (uint32_t e = lane; e < O.n; e += 64) {
      const uint64_t g = base + e;
      if (g < O.cap) O.dst[g] = O.buf[e];
    }
    O.n = 0;
    if constexpr (SPREAD) {
      O.seg = O.seg + 1 < P.nseg ? O.seg + 1 : 0u;
      O.dst = P.cand + (size_t)O.seg * P.cap;
      O.count = P.cand_count + O.seg;
    }
  }
  wave_lds_sync();
}

// Writes the pairs of acc; pair_of(bit) gives the packed pair of a bit.
template <typename PairOf>
__device__ __forceinline__ void emit_pairs(const PairsArgs& P, OutStage& O, uint32_t lane,
                                           uint64_t acc, PairOf pair_of) {
  const uint32_t cnt = (uint32_t)__popcll(acc);
  const uint32_t incl = wave_inclusive_scan(cnt);
  const uint32_t total = lane_value(incl, 63);
  if (!total) return;
  if (O.n + total > (uint32_t)kOutBuf) flush_out(P, O, lane);
  if (total > (uint32_t)kOutBuf) {
    // more than the buffer holds: straight out
    unsigned long long base = 0;
    if (lane == 0) base = atomicAdd(O.count, (unsigned long long)total);
    base = lane_value(base, 0);
    uint64_t pos = base + incl - cnt;
    while (acc) {
      const int b = __builtin_ctzll(acc);
      acc &= acc - 1;
      if (pos < O.cap) O.dst[pos] = pair_of(b);
      ++pos;
    }
  } else {
    uint32_t pos = O.n + incl - cnt;
    while (acc) {
      const int b = __builtin_ctzll(acc);
      acc &= acc - 1;
      O.buf[pos++] = pair_of(b);
    }
    O.n += total;
  }
}

__device__ __forceinline__ uint64_t pack_pair(uint64_t x, uint64_t y, int pair_bits) {
  return (min(x, y) << pair_bits) | max(x, y);
}

// Appends pair (when keep) to the wave's staging buffer: one slot per
// keeping lane, in lane order, flushing first if they would not fit.
template <bool SPREAD = false>
__device__ __forceinline__ void append_pair(const PairsArgs& P, OutStage& O, uint32_t lane,
                                            bool keep, uint64_t pair) {
  const uint64_t kb = ballot(keep);
  const uint32_t nk = (uint32_t)__popcll(kb);
  if (!nk) return;
  if (O.n + nk > (uint32_t)kOutBuf) flush_out<SPREAD>(P, O, lane);
  if (keep) O.buf[O.n + rank_below(kb)] = pair;
  O.n += nk;
}

// Accepted pairs of a tile pair listed for the first-owner check, at most
// this many per wave (more: each lane checks its own, one by one).
constexpr uint32_t kPend = 256;

// --- vector screen --------------------------------------------------------
// Lane l holds point a_l of tile a in registers and tests it against every
// point b_j of tile b, read from LDS by broadcast: FP32 squared differences
// summed with FMA; accepted j in one bit mask, j whose FP32 value lies in the
// band around r^2 in a second mask, re-tested in FP64.
template <int D>
__global__ __launch_bounds__(kBlock) void k_cell_pairs(const PairsArgs P) {
  // LDS row stride: rows of 4 floats read with 128-bit loads
  constexpr int DP = D <= 2 ? D : ((D + 3) / 4) * 4;
  __shared__ __attribute__((aligned(16))) float sB[kWaves][kPairTile][DP];
  __shared__ uint32_t sBi[kWaves][kPairTile];
  __shared__ uint64_t sBw[kWaves][kSigWords][kPairTile];
  __shared__ uint64_t sOut[kWaves][kOutBuf];

  const uint32_t lane = lane_id();
  const int w = uniform((int)(threadIdx.x >> 6));  // (a scalar: so are the unit loops)
  unsigned long long nre = 0;
  OutStage O = out_stage(P, sOut[w]);

  const uint32_t wave_id = blockIdx.x * kWaves + w;
  const uint32_t nwaves = gridDim.x * kWaves;
  // The wave's units form one stream of tiles, each loaded while the tile
  // pair before it is tested.
  // The wave's units: a contiguous run holding about an equal share of the
  // tile pairs (wave_first), else every nwaves-th unit.
  uint32_t u = wave_id, u_end = P.total_units, step = nwaves;
  if (P.wave_first) {
    u = uniform(P.wave_first[wave_id]);
    u_end = uniform(P.wave_first[wave_id + 1]);
    step = 1;
  }
  UnitView V = unit_view<true>(P, u, u_end);
  TileRegs<D> cur, nxt;
  if (V.ok)
    load_tile<D>(P, V.s0 + V.ta_begin * kPairTile, tile_len(V, V.ta_begin), V.nw, lane, cur);
  while (V.ok) {
    const UnitView Vn = unit_view<true>(P, u + step, u_end);
    const PairTest T = P.tests[V.inst];
    const MrInst mr = P.mr ? P.mr[V.inst] : MrInst{};
    for (uint32_t ta = V.ta_begin; ta < V.ta_end; ++ta) {
      const uint32_t nA = tile_len(V, ta);
      const uint32_t pa0 = V.s0 + ta * kPairTile;
      const bool rowok = lane < nA;
      const TileRegs<D> A = cur;  // the row's tile, also its diagonal B tile
      for (uint32_t s = 0; s < V.nt - ta; ++s) {
      const uint32_t tb = row_step_tile(V, ta, s);
      const uint32_t pb0 = V.s0 + tb * kPairTile;
      const uint32_t nB = tile_len(V, tb);
      wave_lds_sync();
      if (lane < nB) {
        sBi[w][lane] = cur.idx;
#pragma unroll
        for (int l = 0; l < DP; ++l) sB[w][lane][l] = (l < D) ? cur.c[l] : 0.0f;
#pragma unroll
        for (int q = 0; q < kSigWords; ++q) sBw[w][q][lane] = cur.sw[q];
      }
      wave_lds_sync();
      load_next<D>(P, V, Vn, ta, tb, lane, cur, nxt);

      // lane l tests j only when j > lim: every pair once in a diagonal tile
      const int lim = rowok ? (ta == tb ? (int)lane : -1) : 64;
      uint32_t accw[2] = {0u, 0u}, bandw[2] = {0u, 0u};
      auto test = [&](int j, int q, uint32_t& am, uint32_t& bm) {
        float b[DP];
#pragma unroll
        for (int l = 0; l < DP; ++l) b[l] = sB[w][j][l];
        float d2 = 0.0f;
#pragma unroll
        for (int l = 0; l < D; ++l) {
          const float df = A.c[l] - b[l];
          d2 = __builtin_fmaf(df, df, d2);
        }
        // bitwise, not short-circuit: every lane computes every test, so
        // the loop stays free of branches and its LDS reads can run ahead
        const uint32_t ok = (uint32_t)(j > lim);
        const uint32_t in_lo = (uint32_t)(d2 <= T.lo);
        const uint32_t in_hi = (uint32_t)(d2 <= T.hi);
        am |= (ok & in_lo) << q;
        bm |= (ok & in_hi & (in_lo ^ 1u)) << q;
      };
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int jb = h * 32;
        const int jn = min((int)nB - jb, 32);
        if (jn <= 0) break;
        uint32_t am = 0u, bm = 0u;
        if (jn == 32) {
#pragma unroll 8
          for (int q = 0; q < 32; ++q) test(jb + q, q, am, bm);
        } else {
          for (int q = 0; q < jn; ++q) test(jb + q, q, am, bm);
        }
        accw[h] = am;
        bandw[h] = bm;
      }
      uint64_t acc = ((uint64_t)accw[1] << 32) | accw[0];
      uint64_t band = ((uint64_t)bandw[1] << 32) | bandw[0];

      // Band: decide in FP64 exactly as the definition does.  Padding
      // coordinates are zero on both sides and add nothing.
      while (band) {
        const int j = __builtin_ctzll(band);
        band &= band - 1;
        double s = 0.0;
#pragma unroll
        for (int l = 0; l < D; ++l) {
          const double dl = (double)A.c[l] - (double)sB[w][j][l];
          s = s + dl * dl;
        }
        if (s <= T.r2) acc |= 1ull << j;
        ++nre;
      }

      // First owner: drop a pair that an earlier grid put in one cell; then
      // the MR-metric.
      if ((V.nw || mr.sub) && ballot(acc != 0ull)) {
        uint64_t m = acc;
        while (m) {
          const int j = __builtin_ctzll(m);
          m &= m - 1;
          uint64_t bw[kSigWords];
#pragma unroll
          for (int q = 0; q < kSigWords; ++q) bw[q] = sBw[w][q][j];
          bool drop = V.nw && not_first_owner<true>(A.sw, bw, V.tcell, V.nw, pa0 + lane, A.idx,
                                                    pb0 + (uint32_t)j, sBi[w][j], P);
          if (!drop && mr.sub) {
            drop = !mr_pair<D>(P, A.idx, sBi[w][j], mr);
            ++nre;
          }
          if (drop) acc &= ~(1ull << j);
        }
      }

      const uint64_t ai = A.idx;
      emit_pairs(P, O, lane, acc,
                 [&](int j) { return pack_pair(ai, sBi[w][j], T.pair_bits); });
      cur = nxt;
      }
    }
    u += step;
    V = Vn;
  }
  flush_out(P, O, lane);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) nre += __shfl_xor(nre, o, 64);
  if (lane == 0 && nre) atomicAdd(P.rechecks, nre);
}

// --- matrix-core screen -----------------------------------------------------
// The squared distances of a 64 x 64 tile pair come from Gram blocks.  With
// the A tile's first point o as origin, a' = a - o and b' = b - o in FP32;
// the rows [a', |a'|^2, 1] and [-2 b', 1, |b'|^2] have dot product
// |a'|^2 + |b'|^2 - 2 a'.b' = |a' - b'|^2, and v_mfma_f32_32x32x2f32
// accumulates 32 x 32 of them over K/2 steps.
//
// The screen accepts v <= lo and rejects v > hi, lo and hi = r^2 -/+ E,
// where E bounds |v - s| for s the FP64 squared distance of the definition:
// recursive-summation bounds for the K products and sums of the expansion
// and for the norms, the rounding of a - o and of r^2 to FP32, all
// proportional to S = max |a'|^2 + max |b'|^2 over the tile pair, with a
// factor 1.5 to spare.  E is set per tile pair, so it widens by itself when
// a cell's points lie far apart (aliased keys, very large cells): the screen
// stays exact and only sends more pairs to FP64.  Pairs with v in between
// are decided in FP64 from the original coordinates.

// v_mfma_f32_32x32x2f32 lane layout: lane l supplies A[l % 32][l / 32] and
// B[l / 32][l % 32]; result register i of lane l holds D[row][l % 32] with
// row = 8 (i / 4) + 4 (l / 32) + i % 4.
__device__ __forceinline__ uint32_t mfma32_row(uint32_t i, uint32_t lane) {
  return 8u * (i >> 2) + 4u * (lane >> 5) + (i & 3u);
}

typedef float floatx16 __attribute__((ext_vector_type(16)));

// The least float above x (x not NaN; +inf stays +inf).
__device__ __forceinline__ float next_up(float x) {
  const uint32_t b = __float_as_uint(x);
  if (x == 0.0f) return __uint_as_float(1u);
  if (b & 0x80000000u) return __uint_as_float(b - 1u);
  return (x == INFINITY) ? x : __uint_as_float(b + 1u);
}

// The maximum over the wave, uniform: quads (xor 1, xor 2), half rows and
// rows by mirroring, then the four rows' maxima read out.
__device__ __forceinline__ float wave_max_f(float v) {
  auto step = [](float x, uint32_t y) { return fmaxf(x, __uint_as_float(y)); };
  v = step(v, dpp_u32<0xB1>(__float_as_uint(v), __float_as_uint(v)));
  v = step(v, dpp_u32<0x4E>(__float_as_uint(v), __float_as_uint(v)));
  v = step(v, dpp_u32<0x141>(__float_as_uint(v), __float_as_uint(v)));
  v = step(v, dpp_u32<0x140>(__float_as_uint(v), __float_as_uint(v)));
  const float r0 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 0));
  const float r1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 16));
  const float r2 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 32));
  const float r3 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 48));
  return fmaxf(fmaxf(r0, r1), fmaxf(r2, r3));
}

// Bits of a tile pair's 64-bit masks: bit 16 (2R + C) + 15 - i is register
// i of block (R, C), i.e. row 32 R + mfma32_row(i, lane), column 32 C + l32.
__device__ __forceinline__ uint32_t gram_row(int b, uint32_t lane) {
  return 32u * ((uint32_t)b >> 5) + mfma32_row(15u - ((uint32_t)b & 15u), lane);
}
__device__ __forceinline__ uint32_t gram_col(int b, uint32_t lane) {
  return 32u * (((uint32_t)b >> 4) & 1u) + (lane & 31u);
}

// The screen's band for S = max |a'|^2 + max |b'|^2 (or a bound on it).  The
// products carry lo into the sums (the B rows hold |b'|^2 - lo), so each
// output is x = v - lo: x < 0 accepts, x > W rejects, anything between is
// decided in FP64.  E bounds the rounding of x, including the lo term; a
// band that reaches 0 (cells far wider than r) is decided in FP64 throughout.
struct GramBand {
  float lo;
  uint32_t Wu;    // W as bits: x <= W for x >= 0
  bool all_fp64;
};
__device__ __forceinline__ GramBand gram_band(float S, float r2f, float gain) {
  constexpr float kU = 0x1p-24f;
  const float E = (S + r2f) * gain + r2f * (4.0f * kU) + 1e-36f;
  GramBand b;
  b.all_fp64 = !(E < r2f);
  b.lo = b.all_fp64 ? 0.0f : (r2f - E) * (1.0f - 0x1p-20f);
  const float hi = (r2f + E) * (1.0f + 0x1p-20f);
  b.Wu = __float_as_uint(next_up(hi - b.lo));
  return b;
}

// The matrix cores' operands of a tile from its rows, one row per lane:
// block X (rows 32 X .. 32 X + 31) takes, in lane l, element 2 q + (l >> 5)
// of row 32 X + (l & 31).  Lanes 0-31 of block 0 keep their own even
// elements and lanes 32-63 need the odd elements of lanes 0-31; block 1
// the reverse.  Swapping the upper half of row[2 q] with the lower half of
// row[2 q + 1] across the wave (v_permlane32_swap) leaves block 0's
// operand in the first and block 1's in the second: no trip through LDS.
template <int KS>
__device__ __forceinline__ void gram_operands(const float* row, float (&op)[2][KS]) {
#pragma unroll
  for (int q = 0; q < KS; ++q) {
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(row[2 * q]),
                                                     __float_as_uint(row[2 * q + 1]), false, false);
    op[0][q] = __uint_as_float(sw[0]);
    op[1][q] = __uint_as_float(sw[1]);
  }
}

// Four waves per SIMD up to D = 12 (at most 128 registers), three above.  The
// wave's index is read as a scalar, so the units and the tile loops live in
// scalar registers (in vector registers they took up to 40 of them, spills
// and masked branches: uniform d6 509 -> 488 us, study d9 661 -> 625).  A
// fifth wave (96 registers, no spills) changes nothing: vector and matrix
// instructions together keep the SIMDs 86-91% busy.
// CHECKS: 1 for passes with hashed keys, 2 for those with an MR-metric
// instance (hashed keys or not).
template <int D, int CHECKS>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(D <= 12 ? 4 : 3))) void
k_cell_pairs_gram(
    const PairsArgs P) {
  constexpr int KA = (D + 3) & ~1;  // augmented row length, even
  constexpr int KS = KA / 2;        // MFMA steps per block
  constexpr float kGain = 1.5f * (float)(2 * KA + D + 8) * 0x1p-24f;
  // the A and B tiles' signature words
  constexpr int kRegion = 2 * kSigWords * kPairTile;
  __shared__ __attribute__((aligned(16))) float sAreg[kWaves][kRegion];
  __shared__ __attribute__((aligned(16))) float sBreg[kWaves][kRegion];
  __shared__ uint32_t sAi[kWaves][kPairTile];
  __shared__ uint32_t sBi[kWaves][kPairTile];
  __shared__ uint64_t sOut[kWaves][kOutBuf];
  __shared__ uint16_t sPend[kWaves][kPend];  // accepted (lane << 6 | bit) codes

  const uint32_t lane = lane_id();
  const uint32_t l32 = lane & 31u, h = lane >> 5;
  const int w = uniform((int)(threadIdx.x >> 6));  // (a scalar: so are the unit loops)
  uint64_t (*sAw)[kPairTile] = reinterpret_cast<uint64_t (*)[kPairTile]>(sAreg[w]);
  uint64_t (*sBw)[kPairTile] = reinterpret_cast<uint64_t (*)[kPairTile]>(sBreg[w]);
  unsigned long long nre = 0;
  OutStage O = out_stage(P, sOut[w]);

  const uint32_t wave_id = blockIdx.x * kWaves + w;
  const uint32_t nwaves = gridDim.x * kWaves;
  // The wave's units form one stream of tiles, each loaded while the tile
  // pair before it is tested.
  // The wave's units: a contiguous run holding about an equal share of the
  // tile pairs (wave_first), else every nwaves-th unit.
  uint32_t u = wave_id, u_end = P.total_units, step = nwaves;
  if (P.wave_first) {
    u = uniform(P.wave_first[wave_id]);
    u_end = uniform(P.wave_first[wave_id + 1]);
    step = 1;
  }
  UnitView V = unit_view<(CHECKS > 0)>(P, u, u_end);
  TileRegs<D> cur, nxt;
  if (V.ok)
    load_tile<D>(P, V.s0 + V.ta_begin * kPairTile, tile_len(V, V.ta_begin), V.nw, lane, cur);
  while (V.ok) {
    const UnitView Vn = unit_view<(CHECKS > 0)>(P, u + step, u_end);
    const PairTest T = P.tests[V.inst];
    const MrInst mr = CHECKS == 2 && P.mr ? P.mr[V.inst] : MrInst{};
    const float r2f = (float)T.r2;
    // When every unit is one grid cell, S <= s_bound for all of the unit's
    // tile pairs: one band for the unit, no per-tile maxima.
    const float s_bound =
        __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(T.s_bound)));
    const bool unit_band = P.unit_band && s_bound > 0.0f;
    const GramBand ub = gram_band(s_bound, r2f, kGain);
    // origin: the first point of the unit's first tile (lane 0; wave-uniform)
    float o[D];
#pragma unroll
    for (int l = 0; l < D; ++l)
      o[l] = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(cur.c[l])));
    for (uint32_t ta = V.ta_begin; ta < V.ta_end; ++ta) {
    const uint32_t nA = tile_len(V, ta);
    const uint32_t pa0 = V.s0 + ta * kPairTile;
    // tile a: centred rows, norms; invalid rows get a huge norm (rejected)
    wave_lds_sync();
    float na = 0.0f;
    float areg[2][KS];
    {
      float row[KA];
      if (lane < nA) {
        float n2 = 0.0f;
#pragma unroll
        for (int l = 0; l < D; ++l) {
          const float v = cur.c[l] - o[l];
          row[l] = v;
          n2 = __builtin_fmaf(v, v, n2);
        }
        row[D] = n2;
        na = n2;
      } else {
#pragma unroll
        for (int l = 0; l < D; ++l) row[l] = 0.0f;
        row[D] = 1e30f;
      }
      row[D + 1] = 1.0f;
#pragma unroll
      for (int l = D + 2; l < KA; ++l) row[l] = 0.0f;
      sAi[w][lane] = cur.idx;
      gram_operands<KS>(row, areg);
    }
    const float amax = unit_band ? 0.0f : wave_max_f(na);
    if (V.nw) {
#pragma unroll
      for (int q = 0; q < kSigWords; ++q) sAw[q][lane] = cur.sw[q];
    }
    wave_lds_sync();  // the A indices and words, before lanes read each other's

    for (uint32_t s = 0; s < V.nt - ta; ++s) {
      const uint32_t tb = row_step_tile(V, ta, s);
      const uint32_t pb0 = V.s0 + tb * kPairTile;
      const uint32_t nB = min((uint32_t)kPairTile, V.L - tb * kPairTile);
      wave_lds_sync();
      float nb = 0.0f;
      uint64_t bsw[kSigWords];
      float row[KA];
      if (lane < nB) {
        float n2 = 0.0f;
#pragma unroll
        for (int l = 0; l < D; ++l) {
          const float v = cur.c[l] - o[l];
          row[l] = -2.0f * v;
          n2 = __builtin_fmaf(v, v, n2);
        }
        nb = n2;
      } else {
#pragma unroll
        for (int l = 0; l < D; ++l) row[l] = 0.0f;
      }
      row[D] = 1.0f;
#pragma unroll
      for (int l = D + 2; l < KA; ++l) row[l] = 0.0f;
#pragma unroll
      for (int q = 0; q < kSigWords; ++q) bsw[q] = cur.sw[q];
      // the tile pair's band: the unit's, else from this pair's maxima
      GramBand bd = ub;
      if (!unit_band) bd = gram_band(amax + wave_max_f(nb), r2f, kGain);
      const bool all_fp64 = bd.all_fp64;
      const float lo = bd.lo;
      const uint32_t Wu = bd.Wu;
      row[D + 1] = lane < nB ? nb - lo : 1e30f;
      sBi[w][lane] = cur.idx;
      float breg[2][KS];
      gram_operands<KS>(row, breg);
      wave_lds_sync();  // the B indices, before lanes read each other's
      load_next<D>(P, V, Vn, ta, tb, lane, cur, nxt);

      const bool diag = (ta == tb);
      uint64_t acc = 0ull, band = 0ull;
#pragma unroll
      for (int R = 0; R < 2; ++R) {
        if (R == 1 && nA <= 32u) break;
#pragma unroll
        for (int C = 0; C < 2; ++C) {
          if (C == 1 && nB <= 32u) break;
          if (diag && R > C) continue;  // rows above the columns: no pairs
          floatx16 v = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f,
                        0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
          for (int q = 0; q < KS; ++q)
            v = __builtin_amdgcn_mfma_f32_32x32x2f32(areg[R][q], breg[C][q], v, 0, 0, 0);
          // Bit 15 - i of am: x[i] < 0, its sign shifted in from the right
          // (x is finite: the host keeps coordinates small enough).  The
          // least x >= 0 as bits (negative x are larger as unsigned) tells
          // whether any x lies in the band; only then are its bits built:
          // bit 15 - i of cm is x[i] <= W.
          uint32_t am = 0u, mn = 0xFFFFFFFFu;
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            am = __builtin_amdgcn_alignbit(am, __float_as_uint(v[i]), 31);
            mn = min(mn, __float_as_uint(v[i]));
          }
          uint32_t cm = 0u;
          if (ballot(mn <= Wu) || all_fp64) {
#pragma unroll
            for (int i = 0; i < 16; ++i)
              cm = __builtin_amdgcn_alignbit(cm, __float_as_uint(v[i]) - (Wu + 1u), 31);
            if (all_fp64) {
              // every pair of real points is decided in FP64; the padding
              // rows and columns of a short tile hold no points
              // (nA through an opaque copy: its 16 compares would otherwise be
              // hoisted out of this rare branch and paid by every row)
              uint32_t rows_in = nA;
              asm volatile("" : "+s"(rows_in));
              const bool col_in = 32u * (uint32_t)C + l32 < nB;
              uint32_t in = 0u;
#pragma unroll
              for (int i = 0; i < 16; ++i)
                in = (in << 1) |
                     ((col_in && 32u * (uint32_t)R + mfma32_row((uint32_t)i, lane) < rows_in) ? 1u
                                                                                             : 0u);
              cm = in;
              am = 0u;
            }
          }
          uint32_t valid = 0xFFFFu;
          if (diag && R == C) {
            // row < col holds for registers i < cnt (rows rise with i)
            const int x = (int)l32 - 4 * (int)h;
            int cnt = 0;
#pragma unroll
            for (int g = 0; g < 4; ++g) cnt += min(max(x - 8 * g, 0), 4);
            valid = (0xFFFFu << (16 - cnt)) & 0xFFFFu;
          }
          const int sh = (R * 2 + C) * 16;
          am &= valid;
          acc |= (uint64_t)am << sh;
          band |= (uint64_t)(cm & valid & ~am) << sh;
          // one block's accumulators at a time
          __builtin_amdgcn_sched_barrier(0);
        }
      }

      // Band: decide in FP64 exactly as the definition does.
      while (band) {
        const int b = __builtin_ctzll(band);
        band &= band - 1;
        const uint32_t pa = sAi[w][gram_row(b, lane)], pb = sBi[w][gram_col(b, lane)];
        double s = 0.0;
#pragma unroll
        for (int l = 0; l < D; ++l) {
          const double dl = (double)P.pts[(size_t)pa * D + l] - (double)P.pts[(size_t)pb * D + l];
          s = s + dl * dl;
        }
        if (s <= T.r2) acc |= 1ull << b;
        ++nre;
      }

      // First owner: drop a pair that an earlier grid put in one cell.  The
      // B rows are in registers by now: their space takes the B words.  The
      // accepted bits are listed in LDS as (lane, bit) codes, each lane
      // writing its own in turn, and are then worked one per lane -- the
      // pair's row and column, the check, the packed pair -- so the per-pair
      // work takes ceil(count / 64) rounds rather than the most any one lane
      // holds.
      const uint32_t cnt = (uint32_t)__popcll(acc);
      const uint32_t incl = wave_inclusive_scan(cnt);
      const uint32_t total = lane_value(incl, 63);
      const bool check = V.nw != 0;
      if (total && check) {
        wave_lds_sync();
#pragma unroll
        for (int q = 0; q < kSigWords; ++q) sBw[q][lane] = bsw[q];
      }
      if (total && total <= kPend) {
        uint32_t pos = incl - cnt;
        uint64_t m = acc;
        while (m) {
          const int b = __builtin_ctzll(m);
          m &= m - 1;
          sPend[w][pos++] = (uint16_t)((lane << 6) | (uint32_t)b);
        }
        wave_lds_sync();
        for (uint32_t e0 = 0; e0 < total; e0 += 64) {
          const uint32_t e = e0 + lane;
          bool keep = e < total;
          uint64_t pair = 0;
          if (keep) {
            const uint32_t code = sPend[w][e];
            const int b = (int)(code & 63u);
            const uint32_t row = gram_row(b, code >> 6), col = gram_col(b, code >> 6);
            const uint32_t ia = sAi[w][row], ib = sBi[w][col];
            if (check) {
              uint64_t aq[kSigWords], bq[kSigWords];
#pragma unroll
              for (int q = 0; q < kSigWords; ++q) {
                aq[q] = sAw[q][row];
                bq[q] = sBw[q][col];
              }
              keep = !not_first_owner<(CHECKS > 0)>(aq, bq, V.tcell, V.nw, pa0 + row, ia,
                                                    pb0 + col, ib, P);
            }
            if (CHECKS == 2 && keep && mr.sub) {
              keep = mr_pair<D>(P, ia, ib, mr);
              ++nre;
            }
            pair = pack_pair(ia, ib, T.pair_bits);
          }
          append_pair(P, O, lane, keep, pair);
        }
        wave_lds_sync();  // sPend is rewritten by the next tile pair
      } else if (total) {
        // more than the list holds: each lane checks and writes its own
        if (check || (CHECKS == 2 && mr.sub)) {
          wave_lds_sync();
          uint64_t m = acc;
          while (m) {
            const int b = __builtin_ctzll(m);
            m &= m - 1;
            const uint32_t row = gram_row(b, lane), col = gram_col(b, lane);
            uint64_t aq[kSigWords], bq[kSigWords];
#pragma unroll
            for (int q = 0; q < kSigWords; ++q) {
              aq[q] = sAw[q][row];
              bq[q] = sBw[q][col];
            }
            bool drop = check && not_first_owner<(CHECKS > 0)>(aq, bq, V.tcell, V.nw, pa0 + row,
                                                         sAi[w][row], pb0 + col, sBi[w][col], P);
            if (CHECKS == 2 && !drop && mr.sub) {
              drop = !mr_pair<D>(P, sAi[w][row], sBi[w][col], mr);
              ++nre;
            }
            if (drop) acc &= ~(1ull << b);
          }
        }
        emit_pairs(P, O, lane, acc, [&](int b) {
          return pack_pair(sAi[w][gram_row(b, lane)], sBi[w][gram_col(b, lane)], T.pair_bits);
        });
      }
      cur = nxt;
    }
    }
    u += step;
    V = Vn;
  }
  flush_out(P, O, lane);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) nre += __shfl_xor(nre, o, 64);
  if (lane == 0 && nre) atomicAdd(P.rechecks, nre);
}

// ---------------------------------------------------------------------------
// query mode.  A query point takes the role of one more point of the indexed
// set: under grid t it falls in the cell floor((R_t q)/(alpha r) + u_t),
// computed in FP64 in the same order as the points' cells, and is reported
// with the indexed points of that cell within r, once (first-owner rule with
// the query's own signature).

// First position in keys[lo..hi) whose cell prefix is >= K.
__device__ __forceinline__ uint32_t prefix_lower_bound(const uint64_t* __restrict__ keys,
                                                       uint32_t lo, uint32_t hi, int shift,
                                                       uint64_t K) {
  while (lo < hi) {
    const uint32_t mid = lo + ((hi - lo) >> 1);
    if ((keys[mid] >> shift) < K) lo = mid + 1;
    else hi = mid;
  }
  return lo;
}

// The cell prefix of a grid's keys: its segment above the packed cell.
__device__ __forceinline__ uint64_t query_prefix(const QueryGrid& G, int cell_bits, uint64_t cell) {
  return cell_bits < 64 ? ((G.seg << cell_bits) | cell) : cell;
}

// tab[t][x] = the first position of grid t whose cell's top tab_bits bits are
// at least x, for x <= 2^tab_bits.
__global__ __launch_bounds__(kBlock) void k_query_table(const QueryGrid* __restrict__ grids, int k,
                                                        uint32_t n, int cell_bits, int tab_bits,
                                                        uint32_t* __restrict__ tab) {
  const uint32_t size = 1u << tab_bits;
  const uint32_t x = blockIdx.x * kBlock + threadIdx.x;
  const int t = (int)blockIdx.y;
  if (x > size) return;
  const QueryGrid G = grids[t];
  tab[(size_t)t * (size + 1) + x] =
      x == size ? n
                : prefix_lower_bound(G.keys, 0, n, G.idx_bits,
                                     query_prefix(G, cell_bits, (uint64_t)x << (cell_bits - tab_bits)));
}

// rows[t][p] = the coordinates of the point at position p of grid t.
template <int D>
__global__ __launch_bounds__(kBlock) void k_query_rows(const QueryGrid* __restrict__ grids, int64_t n,
                                                       const float* __restrict__ pts,
                                                       float* __restrict__ rows) {
  const int64_t p = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (p >= n) return;
  const QueryGrid G = grids[blockIdx.y];
  const uint32_t i = G.idx_bits ? (uint32_t)(G.keys[p] & ((1ull << G.idx_bits) - 1ull)) : G.idx[p];
  const float* src = pts + (size_t)i * D;
  float* dst = rows + ((size_t)blockIdx.y * n + p) * D;
  float v[D];
#pragma unroll
  for (int l = 0; l < D; ++l) v[l] = src[l];
#pragma unroll
  for (int l = 0; l < D; ++l) dst[l] = v[l];
}

// order[q] = the top `bits` bits of the query's cell under grid 0 above its
// index: sorted on those bits, queries of one place come together.
template <int D>
__global__ __launch_bounds__(kBlock) void k_query_order(
    const QueryArgs A, const double* __restrict__ R, const double* __restrict__ u,
    const int64_t* __restrict__ klo, const KeyLayout* __restrict__ layout, int bits,
    uint64_t* __restrict__ order) {
  const int64_t q = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (q >= A.m) return;
  const int d = D > 0 ? D : A.d;
  float p[D > 0 ? D : 1];
  if (D > 0) {
#pragma unroll
    for (int l = 0; l < (D > 0 ? D : 1); ++l) p[l] = A.queries[q * d + l];
  }
  uint64_t cell, grp;
  (void)pack_cell<D>(R, u, klo, layout, p, A.queries, 1, q * d, d, A.inv_c, A.sig_b, cell, grp);
  order[q] = ((cell >> (A.cell_bits - bits)) << 32) | (uint64_t)q;
}

// Of every query under every grid: the position in the grid where the query's
// cell begins (n where the cell is empty, and for a query that is not finite
// or out of range); and its signature words.  A block takes 64 queries, its
// four waves every fourth grid of a signature word.  The binary search is a
// chain of dependent reads: tab cuts its first steps (n = 1e6, d = 3: about
// four instead of twenty).
template <int D>
__global__ __launch_bounds__(kBlock) void k_query_find(
    const QueryArgs A, const double* __restrict__ R, const double* __restrict__ u,
    const int64_t* __restrict__ klo, const KeyLayout* __restrict__ layout,
    const QueryGrid* __restrict__ grids, const uint32_t* __restrict__ tab,
    uint32_t* __restrict__ qlo, uint64_t* __restrict__ qsig) {
  __shared__ uint64_t part[kWaves][64];
  const uint32_t lane = lane_id();
  const int w = uniform((int)(threadIdx.x >> 6));
  const int d = D > 0 ? D : A.d;
  const int64_t at_ = (int64_t)blockIdx.x * 64 + lane;  // place in the order
  const bool live = at_ < A.m;
  const int64_t at = live ? at_ : A.m - 1;
  const int64_t q = A.order ? (int64_t)(uint32_t)A.order[at] : at;
  float p[D > 0 ? D : 1];
  if (D > 0) {
#pragma unroll
    for (int l = 0; l < (D > 0 ? D : 1); ++l) p[l] = A.queries[q * d + l];
  }
  bool finite = true;
  for (int l = 0; l < d; ++l) finite = finite && isfinite(D > 0 ? p[D > 0 ? l : 0] : A.queries[q * d + l]);
  bool bad = false;
  const uint32_t n = (uint32_t)A.n;
  for (int x = 0; x < A.W; ++x) {
    uint64_t word = 0;
    const int tb = min(A.k, (x + 1) * A.gpw);
    for (int t = x * A.gpw + w; t < tb; t += kWaves) {
      uint64_t cell, grp;
      const bool ok = pack_cell<D>(R + (size_t)t * d * d, u + (size_t)t * d, klo + (size_t)t * d,
                                   layout, p, A.queries, 1, q * d, d, A.inv_c, A.sig_b, cell, grp);
      bad |= !ok;
      word |= grp << ((t - x * A.gpw) * A.g);
      const QueryGrid G = grids[t];
      const uint64_t K = query_prefix(G, A.cell_bits, cell);
      uint32_t lo = 0, hi = n;
      if (tab) {
        const uint32_t* tt = tab + (size_t)t * ((1u << A.tab_bits) + 1u);
        const uint32_t top = (uint32_t)(cell >> (A.cell_bits - A.tab_bits));
        lo = tt[top];
        hi = tt[top + 1];
      }
      lo = prefix_lower_bound(G.keys, lo, hi, G.idx_bits, K);
      const bool found = finite && ok && lo < n && (G.keys[min(lo, n - 1u)] >> G.idx_bits) == K;
      if (live) qlo[(size_t)at * A.k + t] = found ? lo : n;
    }
    part[w][lane] = word;
    __syncthreads();
    if (w == (x & (kWaves - 1)) && live) {
#pragma unroll
      for (int o = 0; o < kWaves; ++o) word |= part[o][lane];
      qsig[(size_t)at * A.W + x] = word;
    }
    __syncthreads();  // part is rewritten by the next word
  }
  if (!finite) atomicOr(A.err, 2u);
  else if (bad) atomicOr(A.err, 1u);
}

// A query that lanes of a wave are at, and its output.
template <int D>
struct QueryAt {
  int64_t at, q;  // its place in the order, its index
  float c[D > 0 ? D : 1];
  uint64_t sw[kSigWords];
};

template <int D>
__device__ __forceinline__ QueryAt<D> query_at(const QueryArgs& A, int64_t at) {
  const int d = D > 0 ? D : A.d;
  QueryAt<D> Q;
  Q.at = at;
  Q.q = A.order ? (int64_t)(uint32_t)A.order[at] : at;
  if (D > 0) {
#pragma unroll
    for (int l = 0; l < (D > 0 ? D : 1); ++l) Q.c[l] = A.queries[Q.q * d + l];
  }
#pragma unroll
  for (int x = 0; x < kSigWords; ++x) Q.sw[x] = x < A.W ? A.qsig[(size_t)at * A.W + x] : 0ull;
  return Q;
}

// G lanes (this one the sub-th of them) test the query's cell under grid t,
// which begins at position lo, from member `from` on: a member a lane and
// step, at most steps steps.  True if this lane's next member is in the cell
// too.  ROWS: the coordinates come from the index's copy in grid order, so
// that neighbouring lanes read one line; else by point index.  The screen is
// the vector pair screen's: FP32 with FP64 in the band.
template <int D, bool ROWS>
__device__ __forceinline__ bool walk_cell(const QueryArgs& A, const PairsArgs& P, OutStage& O,
                                          const QueryAt<D>& Q, int t, uint32_t lo, uint32_t from,
                                          uint32_t G, uint32_t sub, uint32_t steps,
                                          uint32_t lane) {
  const int d = D > 0 ? D : A.d;
  const uint32_t n = (uint32_t)A.n;
  const QueryGrid g = A.grids[t];
  const uint64_t K = g.keys[min(lo, n - 1u)] >> g.idx_bits;  // the cell's prefix
  uint32_t pos = lo + from + sub;                            // (n < 2^31)
  // the key and coordinates at a position, loaded one step ahead
  uint64_t key, key_next;
  float c[D > 0 ? D : 1], c_next[D > 0 ? D : 1];
  const float* rows = ROWS ? A.rows + (size_t)t * A.n * D : nullptr;
  auto load = [&](uint32_t p, uint64_t& kk, float* cc) {
    const uint32_t x = min(p, n - 1u);
    kk = g.keys[x];
    if constexpr (D > 0 && ROWS) {
      const float* row = rows + (size_t)x * D;
#pragma unroll
      for (int l = 0; l < D; ++l) cc[l] = row[l];
    }
  };
  load(pos, key, c);
  for (;; --steps) {
    const bool in = pos < n && (key >> g.idx_bits) == K;
    if (!ballot(in)) return false;
    if (steps == 0) return in;
    load(pos + G, key_next, c_next);
    uint32_t i = 0;
    if (!(D > 0 && ROWS) && in)
      i = g.idx_bits ? (uint32_t)(key & ((1ull << g.idx_bits) - 1ull)) : g.idx[pos];
    float d2 = 0.0f;
    const float* row = (D > 0 && ROWS) ? c : A.pts + (size_t)i * d;
    if (D > 0) {
#pragma unroll
      for (int l = 0; l < (D > 0 ? D : 1); ++l) {
        const float df = Q.c[l] - row[l];
        d2 = __builtin_fmaf(df, df, d2);
      }
    } else {
      // eight axes at a time, their loads before the first is used
      for (int l0 = 0; l0 < d; l0 += 8) {
        float a[8], b[8];
#pragma unroll
        for (int x = 0; x < 8; ++x) {
          const int l = min(l0 + x, d - 1);
          a[x] = A.queries[Q.q * d + l];
          b[x] = row[l];
        }
#pragma unroll
        for (int x = 0; x < 8; ++x) {
          const float df = l0 + x < d ? a[x] - b[x] : 0.0f;
          d2 = __builtin_fmaf(df, df, d2);
        }
      }
    }
    bool hit = in && d2 <= A.hi;
    if (hit) {
      if (d2 > A.lo) {
        // the band: as the definition decides
        double s2 = 0.0;
        for (int l = 0; l < d; ++l) {
          const double dl = (double)(D > 0 ? Q.c[D > 0 ? l : 0] : A.queries[Q.q * d + l]) -
                            (double)row[l];
          s2 = s2 + dl * dl;
        }
        hit = s2 <= A.r2;
      }
      if (D > 0 && ROWS)
        i = g.idx_bits ? (uint32_t)(key & ((1ull << g.idx_bits) - 1ull)) : g.idx[pos];
      if (t > 0) {
        // dropped if an earlier grid put the query and the point in one cell
        const int nw = (t - 1) / A.gpw + 1;
        for (int x = 0; x < nw && hit; ++x) {
          const uint64_t xw =
              (x == 0 ? Q.sw[0] : x == 1 ? Q.sw[1] : A.qsig[(size_t)Q.at * A.W + x]) ^
              A.sig[(size_t)i * A.W + x];
          const int ng = min(A.gpw, t - x * A.gpw);
          const uint64_t keep = (ng * A.g >= 64) ? ~0ull : ((1ull << (ng * A.g)) - 1ull);
          hit = (((xw - A.lows) & ~xw & A.highs) & keep) == 0ull;
        }
      }
    }
    append_pair<true>(P, O, lane, hit, ((uint64_t)Q.q << A.pb) | i);
    pos += G;
    key = key_next;
    if constexpr (D > 0 && ROWS) {
#pragma unroll
      for (int l = 0; l < D; ++l) c[l] = c_next[l];
    }
  }
}

// Output staging shares the pair kernels' machinery.  A wave's pairs go to
// every output segment in turn: the pairs of a few queries, which one block
// finds, then fill the segments as evenly as those of many (one query with
// 76 000 neighbours overflowed its block's segment, and the launch ran again).
__device__ __forceinline__ PairsArgs query_output(const QueryArgs& A) {
  PairsArgs P{};
  P.cand = A.cand;
  P.cap = A.cap;
  P.cand_count = A.cand_count;
  P.nseg = A.nseg;
  return P;
}

// Pairs (query, indexed point).  A.lanes lanes of a wave take a query and
// walk the members of its cell under each grid together, from the cell's
// first position while the keys' prefix is the cell's: most cells are short
// (some tens of points), so a whole wave per query idled most of its lanes
// and waited on every cell's chain of loads.  Few queries get more lanes
// each, many get four (8 above d = 6), which is what fills the chip (see
// launch_query_pairs; 1e6 queries of 1e6 points, d = 3, took 6.9 ms, now
// 0.9).  Members from A.walk on are left to k_query_long: the cell is marked
// (kQueryLong in qlo, and *A.long_cells).  Without that limit a few lanes
// walked every crowded cell to its end while the wave's other queries waited:
// 64 of 70000 queries in a cell of 1e5 points took 195 ms, one wave per query
// 18.3; 70000 queries in 1e5 points, d = 12 (cells of thousands), 8.3 against
// 3.8 ms.
template <int D, bool ROWS>
__global__ __launch_bounds__(kBlock) void k_query_pairs(const QueryArgs A) {
  __shared__ uint64_t sOut[kWaves][kOutBuf];
  const uint32_t lane = lane_id();
  const int w = uniform((int)(threadIdx.x >> 6));
  const PairsArgs P = query_output(A);
  OutStage O = out_stage(P, sOut[w]);
  const uint32_t G = A.lanes, sub = lane & (G - 1u);
  const int64_t per_wave = 64 / G;
  const int64_t nwaves = (int64_t)gridDim.x * kWaves;
  bool any = false;
  for (int64_t q0 = ((int64_t)blockIdx.x * kWaves + w) * per_wave; q0 < A.m;
       q0 += nwaves * per_wave) {
    const int64_t at_ = q0 + lane / G;
    const bool live = at_ < A.m;
    const QueryAt<D> Q = query_at<D>(A, live ? at_ : A.m - 1);
    uint32_t* qlo = A.qlo + (size_t)Q.at * A.k;
    for (int t = 0; t < A.k; ++t) {
      const uint32_t lo = live ? qlo[t] & ~kQueryLong : (uint32_t)A.n;
      const bool more = walk_cell<D, ROWS>(A, P, O, Q, t, lo, 0u, G, sub, A.walk / G, lane);
      // (the lane with the next member is the group's first)
      if (more && sub == 0) qlo[t] = lo | kQueryLong;
      any |= more;
    }
  }
  if (any) *A.long_cells = 1ull;  // (every such lane writes the same)
  flush_out(P, O, lane);
}

// The marked cells' members from A.walk on, a whole wave to a cell.  The
// cells of a wave lie a long way apart in the order, so that the cells of
// queries of one crowded place go to different waves.
template <int D, bool ROWS>
__global__ __launch_bounds__(kBlock) void k_query_long(const QueryArgs A) {
  __shared__ uint64_t sOut[kWaves][kOutBuf];
  const uint32_t lane = lane_id();
  const int w = uniform((int)(threadIdx.x >> 6));
  const PairsArgs P = query_output(A);
  OutStage O = out_stage(P, sOut[w]);
  const int64_t cells = A.m * A.k;
  const int64_t share = (cells + A.lanes - 1) / A.lanes;  // A.lanes cells of a wave
  const int64_t nwaves = (int64_t)gridDim.x * kWaves;
  for (int64_t x = (int64_t)blockIdx.x * kWaves + w; x < share; x += nwaves) {
    const int64_t mine = x + (int64_t)lane * share;
    const uint32_t word = lane < A.lanes && mine < cells ? A.qlo[mine] : 0u;
    uint64_t todo = ballot((word & kQueryLong) != 0u);
    while (todo) {
      const int j = __builtin_ctzll(todo);
      todo &= todo - 1;
      const int64_t e = x + (int64_t)j * share;
      const int64_t at = e / A.k;
      const int t = (int)(e - at * A.k);
      const QueryAt<D> Q = query_at<D>(A, at);
      const uint32_t lo = lane_value(word, j) & ~kQueryLong;
      (void)walk_cell<D, ROWS>(A, P, O, Q, t, lo, A.walk, 64u, lane, ~0u, lane);
    }
  }
  flush_out(P, O, lane);
}

// The MR decision of one packed pair of the filter.
__device__ __forceinline__ bool mr_keep(const MrFilterArgs& A, uint64_t v) {
  const uint64_t a = v >> A.pair_bits, b = v & ((1ull << A.pair_bits) - 1ull);
  int lo = 0, hi = A.m - 1;  // the last instance with pt_off <= a
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (A.inst[mid].pt_off <= (int64_t)a) lo = mid;
    else hi = mid - 1;
  }
  const MrInst I = A.inst[lo];
  if (I.sub <= 0) return true;
  return mr_within(A.rows_a + (size_t)a * A.d, A.rows_b + (size_t)b * A.d, A.d, I);
}

// Keeps the packed pairs v of in[0, count) with keep(v), appended to out in
// no particular order.  One block per tile of kBlock * kCompactPer pairs
// (coalesced reads, one lane per pair and step); a tile's kept pairs take
// one atomic on out_count.  Every lane of a block runs the same tiles.
constexpr int kCompactPer = 16;
template <class Keep>
__device__ __forceinline__ void compact_tiles(const uint64_t* __restrict__ in, uint64_t count,
                                              uint64_t* __restrict__ out,
                                              unsigned long long* out_count, Keep keep) {
  __shared__ uint32_t sWave[kWaves];
  __shared__ unsigned long long sBase;
  const uint32_t lane = lane_id();
  const int w = threadIdx.x >> 6;
  const uint64_t tile = (uint64_t)kBlock * kCompactPer;
  for (uint64_t t0 = (uint64_t)blockIdx.x * tile; t0 < count; t0 += (uint64_t)gridDim.x * tile) {
    uint64_t v[kCompactPer], km[kCompactPer];
    uint32_t tot = 0;
#pragma unroll
    for (int i = 0; i < kCompactPer; ++i) {
      const uint64_t p = t0 + (uint64_t)i * kBlock + threadIdx.x;
      v[i] = p < count ? in[p] : 0ull;
    }
#pragma unroll
    for (int i = 0; i < kCompactPer; ++i) {
      const uint64_t p = t0 + (uint64_t)i * kBlock + threadIdx.x;
      km[i] = ballot(p < count && keep(v[i]));
      tot += (uint32_t)__popcll(km[i]);
    }
    if (lane == 0) sWave[w] = tot;
    __syncthreads();
    if (threadIdx.x == 0) {
      uint32_t all = 0;
#pragma unroll
      for (int x = 0; x < kWaves; ++x) all += sWave[x];
      sBase = all ? atomicAdd(out_count, (unsigned long long)all) : 0ull;
    }
    __syncthreads();
    unsigned long long at = sBase;
    for (int x = 0; x < w; ++x) at += sWave[x];
#pragma unroll
    for (int i = 0; i < kCompactPer; ++i) {
      if ((km[i] >> lane) & 1ull) out[at + rank_below(km[i])] = v[i];
      at += (uint32_t)__popcll(km[i]);
    }
    __syncthreads();  // sWave and sBase are rewritten by the next tile
  }
}

__global__ __launch_bounds__(kBlock) void k_mr_filter(const MrFilterArgs A) {
  compact_tiles(A.in, A.count, A.out, A.out_count, [&](uint64_t v) { return mr_keep(A, v); });
}

// Repeats removed with one bit per unordered pair of an instance (the
// upper triangle, a' < b' local indices, bit b'(b'-1)/2 + a'): the
// candidate whose atomic OR sets the bit is kept, any later one is not.
// Which of equal candidates survives does not matter: they are equal.
__device__ __forceinline__ bool bitmap_first(const BitmapArgs& A, uint64_t v) {
  const uint64_t a = v >> A.pair_bits, b = v & ((1ull << A.pair_bits) - 1ull);
  int lo = 0, hi = A.m - 1;  // the last instance with pt_off <= a
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (A.inst[mid].pt_off <= (int64_t)a) lo = mid;
    else hi = mid - 1;
  }
  const BitmapInst I = A.inst[lo];
  const uint64_t la = a - (uint64_t)I.pt_off, lb = b - (uint64_t)I.pt_off;
  const uint64_t bit = (uint64_t)I.bit_off + lb * (lb - 1) / 2 + la;
  const uint32_t m = 1u << (bit & 31u);
  return (atomicOr(A.bits + (bit >> 5), m) & m) == 0u;
}

__global__ __launch_bounds__(kBlock) void k_bitmap_unique(const BitmapArgs A) {
  compact_tiles(A.in, A.count, A.out, A.out_count, [&](uint64_t v) { return bitmap_first(A, v); });
}

// Segment blockIdx.y of the pair output to its place in dst.
__global__ __launch_bounds__(kBlock) void k_seg_compact(const uint64_t* __restrict__ src,
                                                        uint64_t seg_cap,
                                                        const unsigned long long* __restrict__ cnt,
                                                        uint64_t* __restrict__ dst) {
  const uint32_t g = blockIdx.y;
  uint64_t off = 0;
  for (uint32_t h = 0; h < g; ++h) off += cnt[h];
  const uint64_t n = cnt[g];
  const uint64_t* s = src + (size_t)g * seg_cap;
  for (uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x; i < n;
       i += (uint64_t)gridDim.x * kBlock)
    dst[off + i] = s[i];
}

// Unit descriptors of cell c: the whole cell, or one unit per tile.
__global__ void k_unit_fill(const uint32_t* __restrict__ start, const uint32_t* __restrict__ end,
                            const uint32_t* __restrict__ unit_off, uint32_t ncells,
                            const uint32_t* __restrict__ dcells, uint32_t cell_unit_tiles,
                            const uint64_t* __restrict__ skeys, int seg_shift, int sa,
                            const SegDesc* __restrict__ segs, UnitDesc* __restrict__ desc,
                            uint64_t* __restrict__ work) {
  if (dcells) ncells = min(ncells, *dcells);
  for (uint32_t c = blockIdx.x * blockDim.x + threadIdx.x; c < ncells;
       c += gridDim.x * blockDim.x) {
  const uint32_t s0 = start[c], L = end[c] - s0;
  const uint32_t nt = (L + kPairTile - 1) / kPairTile;
  const int seg = sa + (seg_shift >= 64 ? 0 : (int)(skeys[s0] >> seg_shift));
  UnitDesc D;
  D.s0 = s0;
  D.len = L;
  D.t = (uint32_t)segs[seg].t;
  D.inst = (uint32_t)segs[seg].inst;
  D.pad[0] = D.pad[1] = 0u;
  const uint32_t o = unit_off[c];
  if (nt <= cell_unit_tiles) {
    D.ta_begin = 0;
    D.ta_end = nt;
    desc[o] = D;
    if (work) work[o] = (uint64_t)nt * (nt + 1) / 2;  // tile pairs of the unit
  } else {
    for (uint32_t q = 0; q < nt; ++q) {
      D.ta_begin = q;
      D.ta_end = q + 1;
      desc[o + q] = D;
      if (work) work[o + q] = nt - q;
    }
  }
  }
}

// first[w] = the first unit whose exclusive prefix of tile pairs reaches
// w total / nwaves, for w <= nwaves: wave w takes units [first[w],
// first[w + 1]), a contiguous run with about an equal share of the work.
__global__ void k_wave_ranges(const uint64_t* __restrict__ work_off, uint32_t nunits,
                              const uint64_t* __restrict__ total, uint32_t nwaves,
                              uint32_t* __restrict__ first) {
  const uint32_t w = blockIdx.x * blockDim.x + threadIdx.x;
  if (w > nwaves) return;
  // w total / nwaves without overflow: total < 2^56 (units x tile pairs)
  const uint64_t T = *total;
  const uint64_t target = (T / nwaves) * w + (T % nwaves) * w / nwaves;
  uint32_t lo = 0, hi = nunits;  // first index with work_off >= target
  while (lo < hi) {
    const uint32_t mid = (lo + hi) >> 1;
    if (work_off[mid] < target) lo = mid + 1;
    else hi = mid;
  }
  first[w] = w == nwaves ? nunits : lo;
}

// spts[l][p] and ssig[w][p] for the positions p of every unit (one wave per
// unit, one lane per position).  All loads of a lane are issued before its
// stores.
template <int D>
__global__ __launch_bounds__(kBlock) void k_gather_units(const PairsArgs P,
                                                         const uint64_t* __restrict__ sig,
                                                         float* __restrict__ spts,
                                                         uint64_t* __restrict__ ssig) {
  const uint32_t u = blockIdx.x * kWaves + (threadIdx.x >> 6);
  if (u >= P.total_units) return;
  const UnitDesc U = P.units[u];
  const uint32_t lane = lane_id();
  for (uint32_t ta = U.ta_begin; ta < U.ta_end; ++ta) {
  const uint32_t n = min((uint32_t)kPairTile, U.len - ta * kPairTile);
  if (lane >= n) break;
  const uint32_t p = U.s0 + ta * kPairTile + lane;
  const uint32_t i = point_at(P, p);
  const int d = D > 0 ? D : P.d;
  const float* __restrict__ row = P.pts + (size_t)i * d;
  if (D > 0) {
    float c[D > 0 ? D : 1];
#pragma unroll
    for (int l = 0; l < (D > 0 ? D : 1); ++l) c[l] = row[l];
    uint64_t w[kSigWords];
#pragma unroll
    for (int q = 0; q < kSigWords; ++q) w[q] = (sig && q < P.W) ? sig[(size_t)i * P.W + q] : 0ull;
#pragma unroll
    for (int l = 0; l < (D > 0 ? D : 1); ++l) spts[(size_t)l * P.N + p] = c[l];
#pragma unroll
    for (int q = 0; q < kSigWords; ++q)
      if (sig && q < P.W) ssig[(size_t)q * P.N + p] = w[q];
  } else {
    for (int l = 0; l < d; ++l) spts[(size_t)l * P.N + p] = row[l];
  }
  if (sig)
    for (int q = (D > 0 ? kSigWords : 0); q < P.W; ++q)
      ssig[(size_t)q * P.N + p] = sig[(size_t)i * P.W + q];
  }
}

// ---------------------------------------------------------------------------
// CSR

__global__ void k_swap_pairs(const uint64_t* __restrict__ pairs, size_t count, int pb,
                             uint64_t* __restrict__ out) {
  const size_t p = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= count) return;
  const uint64_t k = pairs[p];
  const uint64_t mask = (1ull << pb) - 1ull;
  out[p] = ((k & mask) << pb) | (k >> pb);
}

__global__ void k_row_runs(const uint64_t* __restrict__ keys, size_t count, int pb,
                           uint32_t* __restrict__ rstart, uint32_t* __restrict__ rend) {
  const size_t p = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= count) return;
  const uint64_t row = keys[p] >> pb;
  if (p == 0 || (keys[p - 1] >> pb) != row) rstart[row] = (uint32_t)p;
  if (p + 1 == count || (keys[p + 1] >> pb) != row) rend[row] = (uint32_t)(p + 1);
}

__global__ void k_row_degree(const uint32_t* __restrict__ lo_start, const uint32_t* __restrict__ lo_end,
                             const uint32_t* __restrict__ up_start, const uint32_t* __restrict__ up_end,
                             int64_t n, uint64_t* __restrict__ deg) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  uint64_t c = (uint64_t)(up_end[i] - up_start[i]);
  if (lo_start) c += (uint64_t)(lo_end[i] - lo_start[i]);
  deg[i] = c;
}

__global__ void k_csr_fill_upper(const uint64_t* __restrict__ up, size_t count, int pb,
                                 const int64_t* __restrict__ row_ptr,
                                 const uint32_t* __restrict__ lo_start,
                                 const uint32_t* __restrict__ lo_end,
                                 const uint32_t* __restrict__ up_start, int32_t* __restrict__ col) {
  const size_t p = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= count) return;
  const uint64_t k = up[p];
  const uint64_t i = k >> pb, j = k & ((1ull << pb) - 1ull);
  int64_t pos = row_ptr[i] + (int64_t)(p - up_start[i]);
  if (lo_start) pos += (int64_t)(lo_end[i] - lo_start[i]);
  col[pos] = (int32_t)j;
}

__global__ void k_csr_fill_lower(const uint64_t* __restrict__ lo, size_t count, int pb,
                                 const int64_t* __restrict__ row_ptr,
                                 const uint32_t* __restrict__ lo_start, int32_t* __restrict__ col) {
  const size_t q = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= count) return;
  const uint64_t k = lo[q];
  const uint64_t j = k >> pb, i = k & ((1ull << pb) - 1ull);
  col[row_ptr[j] + (int64_t)(q - lo_start[j])] = (int32_t)i;
}

// ---------------------------------------------------------------------------
// Neighbour lists by row buckets.  Directed entries (row, col) -- both
// orientations of every pair, or only (i, j) for upper-only lists -- are
// partitioned into buckets of 2^rb consecutive rows: per-block bucket counts,
// one device-wide scan in bucket-major order, and a scatter in which each
// block places its entries through LDS cursors.  An entry is stored as the
// 32-bit local key (row mod 2^rb) << pb | col.  Each bucket is then ordered in
// LDS and written as its part of col and row_ptr (k_bucket_csr).  The order of
// entries inside a bucket before that does not matter.

// The pairs a partition block reads: a chunk of one array, or -- when the
// pairs are still in the pair kernels' nseg output segments (segment s at
// pairs + s seg_cap, seg_cnt[s] entries) -- an equal share of one segment
// (block b takes segment b % nseg; nblocks is a multiple of nseg).
struct PairRange {
  const uint64_t* src;
  size_t base, end;
};
__device__ __forceinline__ PairRange pair_range(const uint64_t* pairs, size_t count,
                                                uint32_t chunk, uint32_t nblocks,
                                                const unsigned long long* seg_cnt,
                                                uint64_t seg_cap, uint32_t nseg) {
  PairRange r;
  if (nseg) {
    const uint32_t seg = blockIdx.x % nseg, bps = nblocks / nseg, part = blockIdx.x / nseg;
    const size_t cnt = (size_t)min((unsigned long long)seg_cap, seg_cnt[seg]);
    const size_t ch = (cnt + bps - 1) / bps;
    r.src = pairs + (size_t)seg * seg_cap;
    r.base = min(cnt, (size_t)part * ch);
    r.end = min(cnt, r.base + ch);
  } else {
    r.src = pairs;
    r.base = (size_t)blockIdx.x * chunk;
    r.end = min(count, r.base + chunk);
  }
  return r;
}

template <int TH>
__global__ __launch_bounds__(TH) void k_bucket_hist(const uint64_t* __restrict__ pairs,
                                                    size_t count, int pb, int rb, int both,
                                                    uint32_t nbuckets, uint32_t chunk,
                                                    uint32_t nblocks,
                                                    const unsigned long long* __restrict__ seg_cnt,
                                                    uint64_t seg_cap, uint32_t nseg,
                                                    uint32_t* __restrict__ part,
                                                    uint32_t* __restrict__ zero_word) {
  extern __shared__ uint32_t h[];
  if (zero_word && blockIdx.x == 0 && threadIdx.x == 0) *zero_word = 0u;
  for (uint32_t b = threadIdx.x; b < nbuckets; b += TH) h[b] = 0u;
  __syncthreads();
  const PairRange pr = pair_range(pairs, count, chunk, nblocks, seg_cnt, seg_cap, nseg);
  const uint64_t* __restrict__ src = pr.src;
  const size_t base = pr.base, end = pr.end;
  const uint64_t cmask = (1ull << pb) - 1ull;
  // eight loads in flight per thread, then their atomics
  for (size_t q0 = base; q0 < end; q0 += 8 * TH) {
    uint64_t k8[8];
#pragma unroll
    for (int x = 0; x < 8; ++x) {
      const size_t q = q0 + (size_t)x * TH + threadIdx.x;
      k8[x] = q < end ? src[q] : ~0ull;
    }
#pragma unroll
    for (int x = 0; x < 8; ++x) {
      if (k8[x] == ~0ull) continue;
      atomicAdd(&h[(uint32_t)((k8[x] >> pb) >> rb)], 1u);
      if (both) atomicAdd(&h[(uint32_t)((k8[x] & cmask) >> rb)], 1u);
    }
  }
  __syncthreads();
  for (uint32_t b = threadIdx.x; b < nbuckets; b += TH)
    part[(size_t)b * nblocks + blockIdx.x] = h[b];
}

template <int TH>
__global__ __launch_bounds__(TH) void k_bucket_scatter(const uint64_t* __restrict__ pairs,
                                                       size_t count, int pb, int rb, int both,
                                                       uint32_t nbuckets, uint32_t chunk,
                                                       uint32_t nblocks,
                                                       const unsigned long long* __restrict__ seg_cnt,
                                                       uint64_t seg_cap, uint32_t nseg,
                                                       const uint32_t* __restrict__ offs,
                                                       uint32_t* __restrict__ entries) {
  extern __shared__ uint32_t cur[];
  for (uint32_t b = threadIdx.x; b < nbuckets; b += TH)
    cur[b] = offs[(size_t)b * nblocks + blockIdx.x];
  __syncthreads();
  const PairRange pr = pair_range(pairs, count, chunk, nblocks, seg_cnt, seg_cap, nseg);
  const uint64_t* __restrict__ src = pr.src;
  const size_t base = pr.base, end = pr.end;
  const uint64_t cmask = (1ull << pb) - 1ull;
  const uint32_t rmask = (1u << rb) - 1u;
  for (size_t q0 = base; q0 < end; q0 += 8 * TH) {
    uint64_t k8[8];
#pragma unroll
    for (int x = 0; x < 8; ++x) {
      const size_t q = q0 + (size_t)x * TH + threadIdx.x;
      k8[x] = q < end ? src[q] : ~0ull;
    }
#pragma unroll
    for (int x = 0; x < 8; ++x) {
      if (k8[x] == ~0ull) continue;
      const uint32_t i = (uint32_t)(k8[x] >> pb), j = (uint32_t)(k8[x] & cmask);
      entries[atomicAdd(&cur[i >> rb], 1u)] = ((i & rmask) << pb) | j;
      if (both) entries[atomicAdd(&cur[j >> rb], 1u)] = ((j & rmask) << pb) | i;
    }
  }
}

__device__ __forceinline__ void bucket_range(const uint32_t* __restrict__ offs, uint32_t b,
                                             uint32_t nbuckets, uint32_t nblocks, uint32_t total,
                                             uint32_t& start, uint32_t& cnt) {
  start = offs[(size_t)b * nblocks];
  const uint32_t stop = (b + 1 < nbuckets) ? offs[(size_t)(b + 1) * nblocks] : total;
  cnt = stop - start;
}

// One block per bucket: put the bucket's entries in (row, column) order and
// write them out as the bucket's part of col and row_ptr.  The input pairs are
// unique, so every entry is kept, the bucket's start in the entry array is
// its start in col, and the columns of a row are distinct.  The block's
// 1024 threads load the whole bucket into registers at once and count rows
// (LDS histogram).  Rows of at most kShortRow entries: the entries are
// scattered by row into LDS and each takes its place in the row as the number
// of smaller columns.  Buckets with longer rows go by bins: each row has
// about a quarter as many bins as entries, each an equal share of the
// bucket's column range, the entries are scattered in bin order, and an
// entry's place is its bin's start plus the number of smaller columns in the
// bin, about four reads whatever the row's length (sorting each long row by a
// wave's bitonic network took 402 us for 20e6 entries in rows of 190 and 1510
// for 107e6 in clustered d12, bins 111-120 and 550; for rows of about 20 both
// ways measure 104 us per 19e6, bound by the LDS, and with few entries per
// bucket the extra steps cost 36 against 25 us).  A quarter bin per entry,
// 16 bits each, keeps two blocks on a CU.  A bin of more than
// kMaxBin entries (long rows whose columns lie together) is sorted in place by
// one wave: 150000 points, rows of 500 whose columns lie in 2 / 4 / 8 places
// of the index order, took a call 2334 / 2257 / 1959 us, with bins ranked up to
// 128 entries and whole rows sorted beyond that 2381 / 2688 / 2150, with every
// long row sorted 2294 / 2307 / 2314 (the worst found: rows of 1000 in two
// places, 4746 against 4376).  Buckets larger than cap, and those with a bin
// of more than kLongBin, are listed in oversized for the caller.
constexpr uint32_t kLongBin = 1024;  // (what a wave sorts)
constexpr uint32_t kShortRow = 64;
constexpr uint32_t kMaxBin = 96;

// Ascending sort of v[0..len) in LDS by one wave (len <= 1024): a bitonic
// network in its flip form, where every compare-exchange puts the smaller
// key at the lower index, so the missing tail of the power-of-two size acts
// as +infinity and the sort runs in place.
__device__ __forceinline__ void wave_sort_lds(uint32_t* v, uint32_t len, uint32_t lane) {
  uint32_t P = 1;
  while (P < len) P <<= 1;
  for (uint32_t size = 2; size <= P; size <<= 1) {
    const uint32_t half = size >> 1;
    for (uint32_t i = lane; i < (P >> 1); i += 64) {
      const uint32_t blk = i / half, off = i % half;
      const uint32_t a = blk * size + off, b = blk * size + size - 1 - off;
      if (b < len) {
        const uint32_t x = v[a], y = v[b];
        if (y < x) {
          v[a] = y;
          v[b] = x;
        }
      }
    }
    wave_lds_sync();
    for (uint32_t st = half >> 1; st >= 1; st >>= 1) {
      for (uint32_t i = lane; i < (P >> 1); i += 64) {
        const uint32_t a = 2 * st * (i / st) + (i % st), b = a + st;
        if (b < len) {
          const uint32_t x = v[a], y = v[b];
          if (y < x) {
            v[a] = y;
            v[b] = x;
          }
        }
      }
      wave_lds_sync();
    }
  }
}
constexpr int kCsrThreads = 1024;
constexpr int kCsrWaves = kCsrThreads / 64;
constexpr int kCsrItems = kBucketMaxEntries / kCsrThreads;

__device__ __forceinline__ uint32_t csr_block_exclusive_scan(uint32_t v, uint32_t* wsum,
                                                             uint32_t& total) {
  const uint32_t lane = lane_id();
  const int w = threadIdx.x >> 6;
  const uint32_t inc = wave_inclusive_scan(v);
  if (lane == 63) wsum[w] = inc;
  __syncthreads();
  uint32_t before = 0, all = 0;
#pragma unroll
  for (int q = 0; q < kCsrWaves; ++q) {
    const uint32_t x = wsum[q];
    if (q < w) before += x;
    all += x;
  }
  __syncthreads();
  total = all;
  return before + inc - v;
}

// Bins of the rows before row r whose entries start at start: every row has
// at least one.
__device__ __forceinline__ uint32_t csr_bin_base(uint32_t start, uint32_t r) {
  return (start >> 2) + r;
}
constexpr uint32_t kCsrBins = kBucketMaxEntries / 4 + kBucketMaxRows + 1;
constexpr int kCsrBinsPer = (int)((kCsrBins + 2 * kCsrThreads - 1) / (2 * kCsrThreads)) * 2;

__global__ __launch_bounds__(kCsrThreads, 8) void k_bucket_csr(
    const uint32_t* __restrict__ entries, const uint32_t* __restrict__ offs, uint32_t nbuckets,
    uint32_t nblocks, const uint32_t* __restrict__ total_p, uint32_t* __restrict__ oversized,
    uint32_t* __restrict__ n_oversized, uint32_t cap, int pb, int rb, int64_t n, int64_t nnz,
    int64_t* __restrict__ row_ptr, int32_t* __restrict__ col) {
  __shared__ uint32_t s[kBucketMaxEntries];
  __shared__ uint32_t rstart[kBucketMaxRows + 1];
  __shared__ uint32_t bins[(kCsrBins + 1) / 2];  // two 16-bit counters a word
  __shared__ uint32_t wsum[kCsrWaves];
  __shared__ uint32_t s_min, s_max, s_long, s_over, s_ncrowded;
  __shared__ uint16_t s_crowded[kBucketMaxEntries / kMaxBin];
  const uint32_t b = blockIdx.x;
  const uint32_t lane = lane_id();
  if (b == 0 && threadIdx.x == 0) row_ptr[n] = nnz;
  uint32_t start, cnt;
  bucket_range(offs, b, nbuckets, nblocks, *total_p, start, cnt);
  if (cnt > cap) {
    if (threadIdx.x == 0) oversized[atomicAdd(n_oversized, 1u)] = b;
    return;
  }
  const uint32_t nrows = 1u << rb;
  const uint32_t cmask = (1u << pb) - 1u;
  uint32_t e_[kCsrItems];
#pragma unroll
  for (int q = 0; q < kCsrItems; ++q) {
    const uint32_t i = threadIdx.x + (uint32_t)q * kCsrThreads;
    e_[q] = i < cnt ? entries[start + i] : 0u;
  }
  if (threadIdx.x < nrows) rstart[threadIdx.x] = 0u;
  if (threadIdx.x == 0) {
    s_min = 0xFFFFFFFFu;
    s_max = 0u;
    s_long = 0u;
    s_over = 0u;
    s_ncrowded = 0u;
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kCsrItems; ++q)
    if (threadIdx.x + (uint32_t)q * kCsrThreads < cnt) atomicAdd(&rstart[e_[q] >> pb], 1u);
  __syncthreads();
  // row starts (at most one row per thread)
  static_assert(kBucketMaxRows <= kCsrThreads, "one row per thread");
  const uint32_t mine = threadIdx.x < nrows ? rstart[threadIdx.x] : 0u;
  if (mine > kShortRow) s_long = 1u;
  uint32_t all;
  const uint32_t run = csr_block_exclusive_scan(mine, wsum, all);
  if (threadIdx.x < nrows) {
    rstart[threadIdx.x] = run;
    bins[threadIdx.x] = run;  // the rows' cursors, when there are no long rows
    const int64_t row = ((int64_t)b << rb) + threadIdx.x;
    if (row < n) row_ptr[row] = (int64_t)start + run;
  }
  if (threadIdx.x == 0) rstart[nrows] = cnt;
  __syncthreads();
  if (!s_long) {
#pragma unroll
    for (int q = 0; q < kCsrItems; ++q)
      if (threadIdx.x + (uint32_t)q * kCsrThreads < cnt)
        s[atomicAdd(&bins[e_[q] >> pb], 1u)] = e_[q];
    __syncthreads();
    // A row's entries, at positions t, t + 1024, ... of the row-ordered array
    // for thread t: the lanes of a wave cover a few whole rows and read the
    // same row element at each step (broadcast reads, no bank conflicts).  An
    // entry's place is the number of smaller columns in its row (the row bits
    // are equal, so whole entries compare as columns).
#pragma unroll
    for (int q = 0; q < kCsrItems; ++q) {
      const uint32_t x = threadIdx.x + (uint32_t)q * kCsrThreads;
      if (x < cnt) {
        const uint32_t e = s[x];
        const uint32_t r = e >> pb;
        const uint32_t lo = rstart[r], hi = rstart[r + 1];
        uint32_t rank = lo, y = lo;
        for (; y + 4 <= hi; y += 4)
          rank += (s[y] < e ? 1u : 0u) + (s[y + 1] < e ? 1u : 0u) + (s[y + 2] < e ? 1u : 0u) +
                  (s[y + 3] < e ? 1u : 0u);
        for (; y < hi; ++y) rank += s[y] < e ? 1u : 0u;
        col[(size_t)start + rank] = (int32_t)(e & cmask);
      }
    }
    return;
  }
  // Long rows: bins.
  const uint32_t nbins = csr_bin_base(cnt, nrows);
  for (uint32_t x = threadIdx.x; x < (nbins + 1) / 2; x += kCsrThreads) bins[x] = 0u;
  uint32_t cmin = 0xFFFFFFFFu, cmax = 0u;
#pragma unroll
  for (int q = 0; q < kCsrItems; ++q)
    if (threadIdx.x + (uint32_t)q * kCsrThreads < cnt) {
      cmin = min(cmin, e_[q] & cmask);
      cmax = max(cmax, e_[q] & cmask);
    }
  wave_minmax_u32(cmin, cmax);
  if (lane == 0 && cmin <= cmax) {
    atomicMin(&s_min, cmin);
    atomicMax(&s_max, cmax);
  }
  __syncthreads();
  // bin of an entry: its column's share of the range, over its row's bins
  const uint32_t c0 = s_min;
  const uint32_t scale = 0xFFFFFFFFu / (s_max - c0 + 1u);
  auto bin_of = [&](uint32_t e) -> uint32_t {
    const uint32_t r = e >> pb;
    const uint32_t b0 = csr_bin_base(rstart[r], r), b1 = csr_bin_base(rstart[r + 1], r + 1);
    return b0 + __umulhi(((e & cmask) - c0) * scale, b1 - b0);
  };
#pragma unroll
  for (int q = 0; q < kCsrItems; ++q)
    if (threadIdx.x + (uint32_t)q * kCsrThreads < cnt) {
      const uint32_t x = bin_of(e_[q]);
      atomicAdd(&bins[x >> 1], 1u << (16 * (x & 1u)));
    }
  __syncthreads();
  {
    // bin starts: each thread scans a contiguous run of bins
    uint32_t v[kCsrBinsPer / 2], sum = 0;
#pragma unroll
    for (int x = 0; x < kCsrBinsPer / 2; ++x) {
      const uint32_t at = threadIdx.x * (kCsrBinsPer / 2) + (uint32_t)x;
      v[x] = 2 * at < nbins ? bins[at] : 0u;
      const uint32_t a0 = v[x] & 0xFFFFu, a1 = v[x] >> 16;
      sum += a0 + a1;
      if (max(a0, a1) > kMaxBin) {
        if (a0 > kMaxBin) s_crowded[atomicAdd(&s_ncrowded, 1u)] = (uint16_t)(2 * at);
        if (a1 > kMaxBin) s_crowded[atomicAdd(&s_ncrowded, 1u)] = (uint16_t)(2 * at + 1);
        if (max(a0, a1) > kLongBin) s_over = 1u;
      }
    }
    uint32_t at0 = csr_block_exclusive_scan(sum, wsum, all);
#pragma unroll
    for (int x = 0; x < kCsrBinsPer / 2; ++x) {
      const uint32_t at = threadIdx.x * (kCsrBinsPer / 2) + (uint32_t)x;
      const uint32_t a0 = v[x] & 0xFFFFu, a1 = v[x] >> 16;
      if (2 * at < nbins) bins[at] = at0 | ((at0 + a0) << 16);
      at0 += a0 + a1;
    }
  }
  __syncthreads();
  if (s_over) {
    if (threadIdx.x == 0) oversized[atomicAdd(n_oversized, 1u)] = b;
    return;
  }
#pragma unroll
  for (int q = 0; q < kCsrItems; ++q)
    if (threadIdx.x + (uint32_t)q * kCsrThreads < cnt) {
      const uint32_t x = bin_of(e_[q]);
      const uint32_t old = atomicAdd(&bins[x >> 1], 1u << (16 * (x & 1u)));
      s[(old >> (16 * (x & 1u))) & 0xFFFFu] = e_[q];
    }
  __syncthreads();
  // A bin's cursor now stands at its end, and so at the next bin's start.
  auto bin_extent = [&](uint32_t z, uint32_t& lo, uint32_t& hi) {
    hi = (bins[z >> 1] >> (16 * (z & 1u))) & 0xFFFFu;
    lo = z ? (bins[(z - 1) >> 1] >> (16 * ((z - 1) & 1u))) & 0xFFFFu : 0u;
  };
#pragma unroll
  for (int q = 0; q < kCsrItems; ++q) {
    const uint32_t x = threadIdx.x + (uint32_t)q * kCsrThreads;
    if (x < cnt) {
      const uint32_t e = s[x];
      uint32_t lo, hi;
      bin_extent(bin_of(e), lo, hi);
      if (hi - lo <= kMaxBin) {
        uint32_t rank = lo;
        for (uint32_t y = lo; y < hi; ++y) rank += s[y] < e ? 1u : 0u;
        col[(size_t)start + rank] = (int32_t)(e & cmask);
      }
    }
  }
  const uint32_t ncrowded = s_ncrowded;
  if (!ncrowded) return;
  __syncthreads();  // (the sorts move entries that were read above)
  for (uint32_t q = threadIdx.x >> 6; q < ncrowded; q += kCsrWaves) {
    uint32_t lo, hi;
    bin_extent(s_crowded[q], lo, hi);
    wave_sort_lds(s + lo, hi - lo, lane);
    for (uint32_t x = lo + lane; x < hi; x += 64)
      col[(size_t)start + x] = (int32_t)(s[x] & cmask);
  }
}

// Buckets beyond LDS capacity, all in one global sort.  Bucket ids[q] holds
// entries [start[q], start[q] + cnt[q]) of the entry array (and of col).
__global__ void k_over_extent(const uint32_t* __restrict__ ids, uint32_t nover,
                              const uint32_t* __restrict__ part, uint32_t nblocks,
                              uint32_t nbuckets, size_t np, uint32_t* __restrict__ start,
                              uint32_t* __restrict__ cnt) {
  const uint32_t q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= nover) return;
  const uint32_t b = ids[q];
  const uint32_t st = part[(size_t)b * nblocks];
  const uint32_t nx = (b + 1 < nbuckets) ? part[(size_t)(b + 1) * nblocks] : part[np];
  start[q] = st;
  cnt[q] = nx - st;
}

// The largest q with off[q] <= i (off ascending, off[0] = 0).
__device__ __forceinline__ uint32_t over_of(const uint32_t* __restrict__ off, uint32_t nover,
                                            uint32_t i) {
  uint32_t lo = 0, hi = nover - 1;
  while (lo < hi) {
    const uint32_t mid = (lo + hi + 1) >> 1;
    if (off[mid] <= i) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// w[off[q] + e] = q << sh | entry e of oversized bucket q: one sort orders
// every oversized bucket's entries, bucket by bucket.
__global__ void k_over_gather(const uint32_t* __restrict__ entries,
                              const uint32_t* __restrict__ start, const uint32_t* __restrict__ off,
                              uint32_t nover, uint32_t tot, int sh, uint64_t* __restrict__ w) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= tot) return;
  const uint32_t q = over_of(off, nover, i);
  w[i] = ((uint64_t)q << sh) | entries[(size_t)start[q] + (i - off[q])];
}

// col and row_ptr of every oversized bucket from the sorted tagged entries.
__global__ void k_over_emit(const uint64_t* __restrict__ keys, uint32_t tot,
                            const uint32_t* __restrict__ ids, const uint32_t* __restrict__ start,
                            const uint32_t* __restrict__ cnt, const uint32_t* __restrict__ off,
                            int pb, int rb, int64_t n, int64_t* __restrict__ row_ptr,
                            int32_t* __restrict__ col) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= tot) return;
  const int sh = rb + pb;
  const uint64_t emask = (1ull << sh) - 1ull;
  const uint64_t key = keys[i];
  const uint32_t q = (uint32_t)(key >> sh);
  const uint32_t e = (uint32_t)(key & emask);
  const uint32_t rr = e >> pb;
  const uint32_t local = i - off[q];
  const int64_t base = (int64_t)ids[q] << rb;
  const int64_t at = (int64_t)start[q] + local;
  col[at] = (int32_t)(e & ((1u << pb) - 1u));
  // the first entry of each row sets row_ptr for it and the empty rows before
  const uint32_t from = local == 0 ? 0u : (uint32_t)((keys[i - 1] & emask) >> pb) + 1u;
  for (uint32_t r = from; r <= rr; ++r)
    if (base + r < n) row_ptr[base + r] = at;
  // the bucket's last entry sets the empty rows after it
  if (local + 1 == cnt[q])
    for (uint32_t r = rr + 1; r < (1u << rb); ++r)
      if (base + r < n) row_ptr[base + r] = (int64_t)start[q] + cnt[q];
}

// dst[q] = src[q], zero-extended.
__global__ void k_widen(const uint32_t* __restrict__ src, size_t count, uint64_t* __restrict__ dst) {
  const size_t q = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q < count) dst[q] = src[q];
}

// Read-backs into pinned host memory: the values (words of a device buffer,
// or the scalars of a Gather), then -- after every thread's stores are
// visible at system scope -- the sequence number the host waits for.
__global__ __launch_bounds__(kBlock) void k_mailbox(const uint32_t* __restrict__ src,
                                                    uint32_t words, Gather g,
                                                    uint32_t* __restrict__ host,
                                                    uint64_t* __restrict__ host_seq,
                                                    uint64_t seq) {
  if (src) {
    for (uint32_t i = threadIdx.x; i < words; i += blockDim.x) host[i] = src[i];
  } else if (threadIdx.x < (unsigned)g.count) {
    const int q = threadIdx.x;
    const uint64_t v = g.bytes[q] == 8 ? *static_cast<const uint64_t*>(g.src[q])
                                       : (uint64_t)*static_cast<const uint32_t*>(g.src[q]);
    reinterpret_cast<uint64_t*>(host)[q] = v;
  }
  __threadfence_system();
  __syncthreads();
  if (threadIdx.x == 0)
    __hip_atomic_store(host_seq, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Point records for tile loads: the coordinates, then zeros up to rs floats
// (the last two hold the point's signature word, written by the key kernel).
__global__ void k_records(const float* __restrict__ rows, int64_t n, int d, int rs,
                          float* __restrict__ rec) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  float* r = rec + (size_t)i * rs;
  for (int l = 0; l < d; ++l) r[l] = rows[(size_t)i * d + l];
  for (int l = d; l < rs; ++l) r[l] = 0.0f;
}

// out[q] = row_ptr[first point of instance q] for q < m, out[m] = row_ptr[npts].
__global__ void k_rowptr_at(const InstDesc* __restrict__ inst, uint32_t m,
                            const int64_t* __restrict__ row_ptr, int64_t npts,
                            int64_t* __restrict__ out) {
  const uint32_t q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q < m) out[q] = row_ptr[inst[q].pt_off];
  if (q == m) out[m] = row_ptr[npts];
}

// One thread per batch point (point blocks as in the stage): the point's
// row start in its instance's own row_ptr, relative to the instance.
__global__ __launch_bounds__(kBlock) void k_localize_rows(const InstDesc* __restrict__ inst,
                                                          uint32_t m,
                                                          const int64_t* __restrict__ row_ptr,
                                                          int64_t* const* __restrict__ out_rp) {
  const uint32_t q = block_instance(inst, m, blockIdx.x);
  const int64_t n = inst[q].n;
  const int64_t i = (int64_t)(blockIdx.x - (uint32_t)inst[q].blk_first) * kBlock + threadIdx.x;
  if (i >= n) return;
  const int64_t off = inst[q].pt_off;
  const int64_t base = row_ptr[off];
  int64_t* rp = out_rp[q];
  rp[i] = row_ptr[off + i] - base;
  if (i == n - 1) rp[n] = row_ptr[off + n] - base;
}

constexpr int kLocalizePer = 16;  // entries per thread of the column copy

// The batch's col copied into the instances' own col arrays, indices made
// local: each block a contiguous run of kLocalizePer * kBlock entries (loads
// and stores coalesced); at[q] is instance q's first entry, at[m] the total.
// Each thread finds the instance of its first entry by bisection and steps
// forward past instance ends (several instances may share a run).
__global__ __launch_bounds__(kBlock) void k_localize_cols(const InstDesc* __restrict__ inst,
                                                          uint32_t m,
                                                          const int64_t* __restrict__ at,
                                                          const int32_t* __restrict__ col,
                                                          int32_t* const* __restrict__ out_col) {
  const int64_t total = at[m];
  const int64_t e0 = (int64_t)blockIdx.x * (kLocalizePer * kBlock) + threadIdx.x;
  if (e0 >= total) return;
  uint32_t lo = 0, hi = m - 1;  // the last q with at[q] <= e0
  while (lo < hi) {
    const uint32_t mid = (lo + hi + 1) >> 1;
    if (at[mid] <= e0) lo = mid; else hi = mid - 1;
  }
  uint32_t q = lo;
  int64_t q_end = at[q + 1], q_begin = at[q];
  int32_t* dst = out_col[q];
  int32_t off = (int32_t)inst[q].pt_off;
#pragma unroll 4
  for (int j = 0; j < kLocalizePer; ++j) {
    const int64_t e = e0 + (int64_t)j * kBlock;
    if (e >= total) break;
    while (e >= q_end) {
      ++q;
      q_begin = q_end;
      q_end = at[q + 1];
      dst = out_col[q];
      off = (int32_t)inst[q].pt_off;
    }
    dst[e - q_begin] = col[e] - off;
  }
}

inline unsigned grid_for(size_t count, unsigned block = kBlock) {
  size_t g = (count + block - 1) / block;
  return (unsigned)(g < 1 ? 1 : g);
}

inline unsigned tiles_for(size_t count) { return (unsigned)((count + kTile - 1) / kTile); }

// ---------------------------------------------------------------------------
// Small instances in two launches.  For n <= kTinyPoints (and d <= 8) the
// whole pipeline fits a few workgroups per grid: block (t, part) computes
// every point's cell under grids 0..t (the FP64 formula of k_keys) as a
// 32-bit word of its fields, sorts grid t's keys -- cell and point index -- in
// LDS (counting sort over few cells, else bitonic), tests its slice of the
// pairs of the cells in FP64 in the definition's order, keeps a pair within r
// only if no earlier grid's words of the two points are equal, and appends it
// to one pair list.  A second launch turns the list into the CSR lists.
// Anything outside these limits -- cells that need more bits than a word,
// wider keys, more pairs than the list holds (kTinyPairCap), a row longer than
// kTinyMaxDeg -- is flagged and the caller runs the general pipeline instead.

constexpr int kTinyThreads = 512;
constexpr int kTinyWaves = kTinyThreads / 64;
constexpr int kTinyPer = kTinyPoints / kTinyThreads;

__device__ __forceinline__ uint32_t tiny_block_scan(uint32_t v, uint32_t* wsum, uint32_t& total) {
  const uint32_t lane = lane_id();
  const int w = threadIdx.x >> 6;
  const uint32_t inc = wave_inclusive_scan(v);
  if (lane == 63) wsum[w] = inc;
  __syncthreads();
  uint32_t before = 0, all = 0;
#pragma unroll
  for (int q = 0; q < kTinyWaves; ++q) {
    const uint32_t x = wsum[q];
    if (q < w) before += x;
    all += x;
  }
  __syncthreads();
  total = all;
  return before + inc - v;
}

// The wave's staged pairs (kTinyOut per wave) go to the list in one block
// of slots; every lane of the wave takes part.
constexpr uint32_t kTinyOut = 256;
struct TinyOut {
  uint64_t* buf;
  uint32_t n;
};
__device__ __forceinline__ void tiny_flush(const TinyArgs& A, TinyOut& O, uint32_t lane) {
  wave_lds_sync();
  if (O.n) {
    unsigned long long base = 0;
    if (lane == 0) base = atomicAdd(A.count, (unsigned long long)O.n);
    base = lane_value(base, 0);
    for (uint32_t e = lane; e < O.n; e += 64)
      if (base + e < A.cap) A.pairs[base + e] = O.buf[e];
    O.n = 0;
  }
  wave_lds_sync();
}
__device__ __forceinline__ void tiny_append(const TinyArgs& A, TinyOut& O, uint32_t lane,
                                            bool keep, uint64_t val) {
  const uint64_t m = ballot(keep);
  const uint32_t c = (uint32_t)__popcll(m);
  if (!c) return;
  if (O.n + c > kTinyOut) tiny_flush(A, O, lane);
  if (keep) O.buf[O.n + rank_below(m)] = val;
  O.n += c;
}

template <int D>
__global__ __launch_bounds__(kTinyThreads) void k_tiny_grids(const TinyArgs A) {
  __shared__ float sp[kTinyFloats];         // the points, [n][D]
  __shared__ double sT[kTinyTransform];     // R then u of every grid
  __shared__ uint32_t sC[kTinyCells];       // packed cells of grids 0..t, [g][n]
  __shared__ uint32_t skey[kTinyPoints];    // (cell << idx_bits) | point, sorted
  __shared__ union {
    uint32_t hist[kTinyBins];                // the counting sort's bins
    uint64_t out[kTinyWaves][kTinyOut];      // then each wave's staged pairs
  } sU;
  __shared__ uint32_t wlo[kTinyWaves][D], whi[kTinyWaves][D];
  __shared__ uint32_t wsum[kTinyWaves];
  __shared__ uint32_t sflag;
  __shared__ int s_bits;
  // k parts workgroups: workgroup (t, part) tests slice part of grid t's
  // pairs (every part finds the grid's cells itself)
  const int t = (int)(blockIdx.x / A.parts);
  const uint32_t part = blockIdx.x % A.parts;
  const int n = A.n;
  const uint32_t lane = lane_id();
  const int w = threadIdx.x >> 6;
  if (threadIdx.x == 0) sflag = 0u;
  uint32_t bad = 0u;
  for (int e = (int)threadIdx.x; e < n * D; e += kTinyThreads) {
    const float v = A.pts[e];
    if (!isfinite(v)) bad |= 1u;
    sp[e] = v;
  }
  const int nR = A.k * D * D;
  for (int e = (int)threadIdx.x; e < nR + A.k * D; e += kTinyThreads)
    sT[e] = e < nR ? A.R[e] : A.u[e - nR];
  if (bad) atomicOr(&sflag, bad);
  __syncthreads();
  int idx_bits = 1;
  while ((1 << idx_bits) < n) ++idx_bits;

  // The cell of every point under grids 0..t.  One 32-bit word each: the
  // fields (the key kernel's FP64 formula) less point 0's, kF bits an axis.
  // The earlier grids' words decide, by one comparison, whether a pair was
  // already some earlier grid's; grid t's key the sort, once packed more
  // tightly below.  Each wave takes every eighth grid (or a share of one, when
  // there are fewer grids) on its own: one barrier for all of them, where a
  // pass over the points for each grid's field ranges and another for its
  // words, both by the whole block, took 2.3 us a grid (n = 200, k = 20: 48
  // us for the launch, now 15; n = 2000, k = 4: 28, now 23).
  constexpr int kF = 32 / D;
  constexpr uint32_t kHalf = kF < 32 ? 1u << (kF - 1) : 0x80000000u;
  constexpr uint32_t kFMask = kF < 32 ? (1u << kF) - 1u : 0xFFFFFFFFu;
  int groups = 1;  // grids at work at a time
  while (groups < kTinyWaves && groups < t + 1) groups <<= 1;
  const int per = kTinyWaves / groups;
  const int i0 = (w % per) * 64 + (int)lane;
  {
    bad = 0u;
    for (int g = w / per; g <= t; g += groups) {
      const double* Rg = sT + (size_t)g * D * D;
      const double* ug = sT + nR + (size_t)g * D;
      uint32_t base[D];
      for (int i = -1, at = 0; at < n; i = at) {
        // first the fields' origin (point 0, alike in every wave), then points
        float p[D];
#pragma unroll
        for (int l = 0; l < D; ++l) p[l] = sp[(i < 0 ? 0 : i) * D + l];
        uint32_t cell = 0;
#pragma unroll
        for (int j = 0; j < D; ++j) {
          const double y = cell_y<D>(Rg + (size_t)j * D, p, nullptr, 0, 0, D, A.inv_c, ug[j]);
          const bool ok = fabs(y) < 2147483648.0;
          const uint32_t kj = (uint32_t)(ok ? (int32_t)floor(y) : 0);
          if (!ok) bad |= 2u;
          if (i < 0) {
            base[j] = kj - kHalf;
          } else {
            const uint32_t f = kj - base[j];
            if (f > kFMask) bad |= 4u;  // too far from point 0
            cell |= (f & kFMask) << (j * kF);
          }
        }
        if (i < 0) {
          at = i0;
        } else {
          sC[(size_t)g * n + i] = cell;
          at = i + per * 64;
        }
      }
    }
    if (bad) atomicOr(&sflag, bad);
  }
  __syncthreads();
  int cell_bits = 0;
  if (sflag == 4u) {
    // Points too far from point 0 on some axis: each grid's fields less their
    // minimum, in as few bits as they take, which hold long thin sets as well
    // (2000 points on a path of 1000 cells, d = 3, k = 4: 88 us a call, 166
    // when the general pipeline ran after the two launches).  Only these
    // instances pay for it: with ranges for all, 2000 points in a cube took 85
    // us instead of 62.
    if (threadIdx.x == 0) s_bits = 0;
    for (int g0 = 0; g0 <= t; g0 += groups) {
      const int g = g0 + w / per;
      const double* Rg = sT + (size_t)g * D * D;
      const double* ug = sT + nR + (size_t)g * D;
      const int i1 = g <= t ? n : 0;  // (waves without a grid meet the barriers)
      auto fields = [&](int i, uint32_t (&f)[D]) {
        float p[D];
#pragma unroll
        for (int l = 0; l < D; ++l) p[l] = sp[i * D + l];
#pragma unroll
        for (int j = 0; j < D; ++j) {
          const double y = cell_y<D>(Rg + (size_t)j * D, p, nullptr, 0, 0, D, A.inv_c, ug[j]);
          f[j] = (uint32_t)(int32_t)floor(y) ^ 0x80000000u;  // (in the order of the cells)
        }
      };
      uint32_t lo[D], hi[D], f[D];
#pragma unroll
      for (int j = 0; j < D; ++j) {
        lo[j] = 0xFFFFFFFFu;
        hi[j] = 0u;
      }
      for (int i = i0; i < i1; i += per * 64) {
        fields(i, f);
#pragma unroll
        for (int j = 0; j < D; ++j) {
          lo[j] = min(lo[j], f[j]);
          hi[j] = max(hi[j], f[j]);
        }
      }
      __syncthreads();  // (every thread has read sflag, and the ranges before)
#pragma unroll
      for (int j = 0; j < D; ++j) {
        wave_minmax_u32(lo[j], hi[j]);
        if (lane == 0) {
          wlo[w][j] = lo[j];
          whi[w][j] = hi[j];
        }
      }
      if (g0 == 0 && threadIdx.x == 0) sflag = 0u;
      __syncthreads();
      int shift[D], bits = 0;
#pragma unroll
      for (int j = 0; j < D; ++j) {
        lo[j] = wlo[w / per * per][j];
        hi[j] = whi[w / per * per][j];
        for (int q = 1; q < per; ++q) {
          lo[j] = min(lo[j], wlo[w / per * per + q][j]);
          hi[j] = max(hi[j], whi[w / per * per + q][j]);
        }
        shift[j] = bits;
        bits += hi[j] > lo[j] ? 32 - __clz((int)(hi[j] - lo[j])) : 0;
      }
      // grid t's key holds the point index too
      const bool fits = g == t ? bits + idx_bits <= 31 : bits <= 32;
      if (g <= t && !fits && lane == 0) atomicOr(&sflag, 4u);
      if (g == t && lane == 0) s_bits = bits;
      for (int i = i0; i < (fits ? i1 : 0); i += per * 64) {
        fields(i, f);
        uint32_t cell = 0;
#pragma unroll
        for (int j = 0; j < D; ++j) cell |= (f[j] - lo[j]) << (shift[j] & 31);
        sC[(size_t)g * n + i] = cell;
      }
    }
    __syncthreads();
    const uint32_t flag = sflag;
    if (flag) {
      if (threadIdx.x == 0) atomicOr(A.err, flag);
      return;  // uniform: every thread read the same flag
    }
    cell_bits = s_bits;
  } else {
    // grid t's fields less their minimum, in as few bits as they take
    uint32_t lo[D], hi[D];
#pragma unroll
    for (int j = 0; j < D; ++j) {
      lo[j] = 0xFFFFFFFFu;
      hi[j] = 0u;
    }
    const uint32_t* words = sC + (size_t)t * n;
    for (int i = (int)threadIdx.x; i < n; i += kTinyThreads) {
#pragma unroll
      for (int j = 0; j < D; ++j) {
        const uint32_t f = (words[i] >> (j * kF)) & kFMask;
        lo[j] = min(lo[j], f);
        hi[j] = max(hi[j], f);
      }
    }
#pragma unroll
    for (int j = 0; j < D; ++j) {
      wave_minmax_u32(lo[j], hi[j]);
      if (lane == 0) {
        wlo[w][j] = lo[j];
        whi[w][j] = hi[j];
      }
    }
    __syncthreads();
    int shift[D];
#pragma unroll
    for (int j = 0; j < D; ++j) {
      lo[j] = wlo[0][j];
      hi[j] = whi[0][j];
#pragma unroll
      for (int q = 1; q < kTinyWaves; ++q) {
        lo[j] = min(lo[j], wlo[q][j]);
        hi[j] = max(hi[j], whi[q][j]);
      }
      shift[j] = cell_bits;
      cell_bits += 32 - __clz((int)(hi[j] - lo[j]));  // (0 bits for one value)
    }
    uint32_t flag = sflag;
    // the key holds the point index too (and must not match the bitonic
    // sort's padding)
    if (cell_bits + idx_bits > 31) flag |= 4u;
    if (flag) {
      if (threadIdx.x == 0) atomicOr(A.err, flag);
      return;  // uniform: every thread read the same flag
    }
    for (int i = (int)threadIdx.x; i < n; i += kTinyThreads) {
      const uint32_t word = sC[(size_t)t * n + i];
      uint32_t cell = 0;
#pragma unroll
      for (int j = 0; j < D; ++j) cell |= (((word >> (j * kF)) & kFMask) - lo[j]) << shift[j];
      sC[(size_t)t * n + i] = cell;
    }
    __syncthreads();
  }
  const uint32_t* cur = sC + (size_t)t * n;

  // Grid t's keys in cell order: a counting sort over the cells when they
  // are few, else a bitonic sort of the whole keys.
  if (cell_bits <= kTinyBinBits) {
    const int nb = 1 << cell_bits;
    for (int c = (int)threadIdx.x; c < nb; c += kTinyThreads) sU.hist[c] = 0u;
    __syncthreads();
    for (int i = (int)threadIdx.x; i < n; i += kTinyThreads) atomicAdd(&sU.hist[cur[i]], 1u);
    __syncthreads();
    constexpr int per = kTinyBins / kTinyThreads;
    uint32_t mine = 0;
#pragma unroll
    for (int e = 0; e < per; ++e) {
      const int c = (int)threadIdx.x * per + e;
      if (c < nb) mine += sU.hist[c];
    }
    uint32_t all;
    uint32_t run = tiny_block_scan(mine, wsum, all);
#pragma unroll
    for (int e = 0; e < per; ++e) {
      const int c = (int)threadIdx.x * per + e;
      if (c < nb) {
        const uint32_t h = sU.hist[c];
        sU.hist[c] = run;
        run += h;
      }
    }
    __syncthreads();
    for (int i = (int)threadIdx.x; i < n; i += kTinyThreads) {
      const uint32_t c = cur[i];
      skey[atomicAdd(&sU.hist[c], 1u)] = (c << idx_bits) | (uint32_t)i;
    }
    __syncthreads();
  } else {
    int np2 = 1;
    while (np2 < n) np2 <<= 1;
    for (int i = (int)threadIdx.x; i < np2; i += kTinyThreads)
      skey[i] = i < n ? (cur[i] << idx_bits) | (uint32_t)i : 0xFFFFFFFFu;
    __syncthreads();
    for (int size = 2; size <= np2; size <<= 1) {
      for (int stride = size >> 1; stride > 0; stride >>= 1) {
        for (int x = (int)threadIdx.x; x < np2 / 2; x += kTinyThreads) {
          const int a = 2 * stride * (x / stride) + (x % stride), b = a + stride;
          const bool up = (a & size) == 0;
          const uint32_t ka = skey[a], kb = skey[b];
          if ((ka > kb) == up) {
            skey[a] = kb;
            skey[b] = ka;
          }
        }
        __syncthreads();
      }
    }
  }

  // Pairs per sorted position: c_p = the positions after p in p's cell
  // (the cell's end: the counting sort's cursor, else found by bisection);
  // their exclusive prefix goes where grid t's cells were (no longer read).
  const uint32_t imask = (1u << idx_bits) - 1u;
  uint32_t* pre = sC + (size_t)t * n;
  uint32_t cnt[kTinyPer];
  uint32_t mine = 0, cells = 0;
#pragma unroll
  for (int e = 0; e < kTinyPer; ++e) {
    const int p = (int)threadIdx.x * kTinyPer + e;
    cnt[e] = 0;
    if (p < n) {
      const uint32_t cp = skey[p] >> idx_bits;
      int lo = p + 1, hi = n;  // the first position past p's cell
      if (cell_bits <= kTinyBinBits) {
        lo = (int)sU.hist[cp];
      } else {
        while (lo < hi) {
          const int mid = (lo + hi) >> 1;
          if ((skey[mid] >> idx_bits) == cp) lo = mid + 1; else hi = mid;
        }
      }
      cnt[e] = (uint32_t)(lo - p - 1);
      if (cnt[e] && (p == 0 || (skey[p - 1] >> idx_bits) != cp)) ++cells;
      mine += cnt[e];
    }
  }
  uint32_t T;
  uint32_t run = tiny_block_scan(mine, wsum, T);  // barriers: every c_p is read
#pragma unroll
  for (int e = 0; e < kTinyPer; ++e) {
    const int p = (int)threadIdx.x * kTinyPer + e;
    if (p < n) {
      pre[p] = run;
      run += cnt[e];
    }
  }
  __syncthreads();

  // The workgroup's slice [s0, s1) of the grid's T pairs (p, q), p < q in
  // one cell, in position order, in one contiguous run per thread: its
  // first p by bisection of pre, then q steps to the cell's end and p on to
  // the next position with pairs.  The order of a cell's points may differ
  // between the parts (the counting sort's scatter is atomic), so slices
  // hold whole cells: a nominal bound T * part / parts moves down to the
  // first pair of the cell that holds it, a value every part finds alike.
  auto cell_bound = [&](uint32_t part_i) -> uint32_t {
    const uint32_t s = (uint32_t)((uint64_t)T * part_i / A.parts);
    if (s >= T) return T;
    int lo = 0, hi = n - 1;  // the position whose pairs hold index s
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (pre[mid] <= s) lo = mid; else hi = mid - 1;
    }
    const uint32_t c = skey[lo] >> idx_bits;
    int a0 = 0, a1 = lo;  // the first position of that cell
    while (a0 < a1) {
      const int mid = (a0 + a1) >> 1;
      if ((skey[mid] >> idx_bits) < c) a0 = mid + 1; else a1 = mid;
    }
    return pre[a0];
  };
  const uint32_t s0 = cell_bound(part);
  const uint32_t s1 = cell_bound(part + 1);
  const uint32_t chunk = (s1 - s0 + kTinyThreads - 1) / kTinyThreads;
  uint32_t e = s0 + threadIdx.x * chunk;
  const uint32_t e_end = min(s1, e + chunk);
  int p = 0, q = 0;
  uint32_t pend = 0;  // pre of the position after p
  uint32_t a = 0;
  float pa[D];
  if (e < e_end) {
    int lo = 0, hi = n - 1;  // the last position with pre <= e
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (pre[mid] <= e) lo = mid; else hi = mid - 1;
    }
    p = lo;
    q = p + 1 + (int)(e - pre[p]);
    pend = p + 1 < n ? pre[p + 1] : T;
    a = skey[p] & imask;
#pragma unroll
    for (int l = 0; l < D; ++l) pa[l] = sp[a * D + l];
  }
  TinyOut O{sU.out[w], 0u};
  // sU.hist was last read before the prefix scan's barriers
  for (uint32_t round = 0; round < chunk; ++round, ++e) {
    bool keep = false;
    uint64_t val = 0;
    if (e < e_end) {
      if (e == pend) {  // on to the next position that has pairs
        do {
          ++p;
          pend = p + 1 < n ? pre[p + 1] : T;
        } while (pend == pre[p]);
        q = p + 1;
        a = skey[p] & imask;
#pragma unroll
        for (int l = 0; l < D; ++l) pa[l] = sp[a * D + l];
      }
      const uint32_t b = skey[q] & imask;
      double s2 = 0.0;
#pragma unroll
      for (int l = 0; l < D; ++l) {
        const double dl = (double)pa[l] - (double)sp[b * D + l];
        s2 = s2 + dl * dl;
      }
      keep = s2 <= A.r2;
      // first owner: no earlier grid with both points in one cell
      for (int g = 0; keep && g < t; ++g)
        if (sC[(size_t)g * n + a] == sC[(size_t)g * n + b]) keep = false;
      val = ((uint64_t)min(a, b) << 32) | (uint64_t)max(a, b);
      ++q;
    }
    tiny_append(A, O, lane, keep, val);
  }
  tiny_flush(A, O, lane);
  // the grid's cells and tests (T), counted by its first part
  if (part == 0) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) cells += __shfl_xor(cells, o, 64);
    if (lane == 0 && cells) atomicAdd(A.count + 2, (unsigned long long)cells);
    if (threadIdx.x == 0 && T) atomicAdd(A.count + 1, (unsigned long long)T);
  }
}

// The pair list to CSR lists, the rows split over the workgroups
// (kTinyListRows rows each): every workgroup counts every row's degree and
// takes the offsets of all of them, places the entries of its own rows in LDS
// (rows have at most kTinyMaxDeg entries) and writes each at its rank within
// its row, an entry a thread.  The pairs a thread loads stay in its registers
// while they fit.  count[3] receives the entries written.  (512 rows per
// workgroup, a row per thread and the pairs read twice took 19-21 us at
// n = 200 and 2000, this 6 and 8.)
constexpr int kTinyListThreads = 1024;
constexpr int kTinyListPer = kTinyPoints / kTinyListThreads;
__global__ __launch_bounds__(kTinyListThreads) void k_tiny_lists(const TinyArgs A) {
  __shared__ uint32_t cur[kTinyPoints + 1];
  __shared__ uint32_t ent[kTinyListRows * (int)kTinyMaxDeg];  // (row - r0) << 12 | column
  __shared__ uint32_t wsum[kTinyListThreads / 64];
  __shared__ uint32_t smax;
  static_assert(kTinyPoints <= 1 << 12, "columns in 12 bits");
  constexpr int kB = 8;  // pairs in flight per thread
  const uint64_t P = A.count[0];
  if (P > A.cap || *A.err) return;  // uniform: the caller reruns or fails
  const int n = A.n;
  const uint32_t r0 = blockIdx.x * kTinyListRows, r1 = min((uint32_t)n, r0 + kTinyListRows);
  uint64_t v[kB];
  auto load = [&](uint32_t base) {
#pragma unroll
    for (int e = 0; e < kB; ++e) {
      const uint32_t x = base + e * kTinyListThreads + threadIdx.x;
      v[e] = x < P ? A.pairs[x] : ~0ull;
    }
  };
  load(0);
  for (int i = (int)threadIdx.x; i < n; i += kTinyListThreads) cur[i] = 0u;
  if (threadIdx.x == 0) smax = 0u;
  __syncthreads();
  for (uint32_t base = 0; base < (uint32_t)P; base += kB * kTinyListThreads) {
    if (base) load(base);
#pragma unroll
    for (int e = 0; e < kB; ++e) {
      if (v[e] == ~0ull) continue;
      atomicAdd(&cur[(uint32_t)(v[e] >> 32)], 1u);
      if (!A.upper) atomicAdd(&cur[(uint32_t)v[e]], 1u);
    }
  }
  __syncthreads();
  // row offsets: thread t takes the rows [t kTinyListPer, (t + 1) kTinyListPer);
  // cur becomes every row's start, cur[n] the total
  uint32_t dg[kTinyListPer];
  uint32_t mine = 0, mx = 0;
#pragma unroll
  for (int e = 0; e < kTinyListPer; ++e) {
    const int i = (int)threadIdx.x * kTinyListPer + e;
    dg[e] = i < n ? cur[i] : 0u;
    mine += dg[e];
    mx = max(mx, dg[e]);
  }
  if (mx > kTinyMaxDeg) smax = 1u;
  uint32_t all;
  uint32_t run = csr_block_exclusive_scan(mine, wsum, all);
  if (smax) {
    if (threadIdx.x == 0) atomicOr(A.err, 8u);
    return;  // uniform after the scan's barriers
  }
#pragma unroll
  for (int e = 0; e < kTinyListPer; ++e) {
    const uint32_t i = threadIdx.x * kTinyListPer + e;
    if (i < (uint32_t)n) {
      if (i >= r0 && i < r1) A.row_ptr[i] = (int64_t)run;
      cur[i] = run;
    }
    run += dg[e];
  }
  if (threadIdx.x == 0) {
    cur[n] = all;
    if (blockIdx.x == gridDim.x - 1) {
      A.row_ptr[n] = (int64_t)all;
      A.count[3] = all;
    }
  }
  __syncthreads();
  const uint32_t base = cur[r0], end = cur[r1];
  __syncthreads();  // the rows' starts become cursors
  for (uint32_t b0 = 0; b0 < (uint32_t)P; b0 += kB * kTinyListThreads) {
    if (P > (uint64_t)(kB * kTinyListThreads)) load(b0);
#pragma unroll
    for (int e = 0; e < kB; ++e) {
      if (v[e] == ~0ull) continue;
      const uint32_t a = (uint32_t)(v[e] >> 32), b = (uint32_t)v[e];
      if (a >= r0 && a < r1) ent[atomicAdd(&cur[a], 1u) - base] = ((a - r0) << 12) | b;
      if (!A.upper && b >= r0 && b < r1) ent[atomicAdd(&cur[b], 1u) - base] = ((b - r0) << 12) | a;
    }
  }
  __syncthreads();
  // A row's entries are distinct, so each one's rank within the row is its
  // place; a row's cursor stands at its end, its predecessor's at its start
  // (entries of one row compare as columns).
  for (uint32_t x = threadIdx.x; x < end - base; x += kTinyListThreads) {
    const uint32_t e = ent[x];
    const uint32_t row = r0 + (e >> 12);
    const uint32_t lo = row > r0 ? cur[row - 1] - base : 0u, hi = cur[row] - base;
    uint32_t rank = lo;
    for (uint32_t y = lo; y < hi; ++y) rank += ent[y] < e ? 1u : 0u;
    A.col[base + rank] = (int32_t)(e & 0xFFFu);
  }
}

}  // namespace


// ===========================================================================
// launchers

void launch_fill_u32(uint32_t* p, uint32_t v, size_t count, hipStream_t s) {
  if (!count) return;
  size_t g = (count + kBlock - 1) / kBlock;
  if (g > 65536) g = 65536;
  hipLaunchKernelGGL(k_fill<uint32_t>, dim3((unsigned)g), dim3(kBlock), 0, s, p, v, count);
}

void launch_fill_u64(uint64_t* p, uint64_t v, size_t count, hipStream_t s) {
  if (!count) return;
  size_t g = (count + kBlock - 1) / kBlock;
  if (g > 65536) g = 65536;
  hipLaunchKernelGGL(k_fill<uint64_t>, dim3((unsigned)g), dim3(kBlock), 0, s, p, v, count);
}

void launch_stage(const InstDesc* inst, uint32_t m, uint32_t nblocks, int d, int64_t npts,
                  float* soa, float* aos, uint32_t* bad, uint32_t* bbox, uint32_t* part,
                  float* rec, int rs, hipStream_t s, uint64_t* zero64, uint32_t nzero,
                  bool cleared) {
  const uint32_t nbox = m * 2u * (uint32_t)d;
  if (!cleared)
    hipLaunchKernelGGL(k_stage_init, dim3(grid_for(std::max(nbox, nzero))), dim3(kBlock), 0, s,
                       bbox, nbox, bad, zero64, nzero);
  if (!nblocks) return;
#define RTG_STAGE(DD)                                                                         \
  hipLaunchKernelGGL(k_stage_d<DD>, dim3(nblocks), dim3(kBlock), 0, s, inst, m, npts, soa, aos, \
                     bad, part, rec)
  // records are made for d <= 6 only, rs = (d + 5) & ~3 as k_stage_d assumes
  switch (d) {
    case 1: RTG_STAGE(1); break;
    case 2: RTG_STAGE(2); break;
    case 3: RTG_STAGE(3); break;
    case 4: RTG_STAGE(4); break;
    case 5: RTG_STAGE(5); break;
    case 6: RTG_STAGE(6); break;
    case 7: RTG_STAGE(7); break;
    case 8: RTG_STAGE(8); break;
    case 9: RTG_STAGE(9); break;
    case 10: RTG_STAGE(10); break;
    case 11: RTG_STAGE(11); break;
    case 12: RTG_STAGE(12); break;
    case 13: RTG_STAGE(13); break;
    case 14: RTG_STAGE(14); break;
    case 15: RTG_STAGE(15); break;
    case 16: RTG_STAGE(16); break;
    default:
      hipLaunchKernelGGL(k_stage, dim3(nblocks), dim3(kBlock), 0, s, inst, m, d, npts, soa, aos,
                         bad, part, rec, rs);
  }
#undef RTG_STAGE
  // blocks per instance: about 256 per-block boxes each (four per lane), at
  // most kBboxBlocks
  uint32_t gy = (uint32_t)std::min<uint64_t>(kBboxBlocks, (nblocks / m + 255) / 256);
  if (gy < 1) gy = 1;
  hipLaunchKernelGGL(k_bbox_reduce, dim3(m, gy), dim3(kBlock), 0, s, inst, d, part, bbox);
}

// Point blocks below which the key kernel splits a point's grids over waves.
// A wave that loops over the grids keeps its point, but too few of them leave
// the SIMDs idle: 46 -> 8.7 us at 25 blocks (k = 25, d = 6), 81 -> 42 us at
// 400 (k = 25, d = 9), 19 us either way at 782 (k = 8, d = 6); above, the
// split's repeated loads show: 10.7 -> 14.0 us at 1172 (k = 6, d = 2),
// 51 -> 67 us at 3907 (k = 8, d = 6).
constexpr uint32_t kKeysSplitBlocks = 768;

template <int D>
static void keys_dispatch(const KeysArgs& a, hipStream_t s) {
  // without signatures the "words" only deal grids to the blocks
  const int gpw = a.sig ? a.sig_gpw : 2 * kWaves;
  if (a.nblocks < kKeysSplitBlocks) {
    // words an instance has in this pass at most (one more where the pass
    // may begin inside a word), over as many slices as fill the chip
    const int grids = std::min(a.kmax, a.sb - a.sa);
    const int words = (grids + gpw - 1) / gpw + (a.sig_fresh ? 0 : 1);
    const int slices = std::min(words, (int)(kKeysSplitBlocks / a.nblocks) + 1);
    const int per = (words + slices - 1) / slices;
    hipLaunchKernelGGL((k_keys<D, true>), dim3(a.nblocks * kWaves, slices), dim3(kBlock), 0, s,
                       a.inst, a.m, a.d, a.npts, a.soa, a.sa, a.sb, a.segs, a.R, a.u, a.klo,
                       a.layout, a.keys, a.vals, a.err, a.sig, a.sig_stride, a.sig_b, gpw,
                       a.idx_bits, a.sig_fresh, per);
    return;
  }
  hipLaunchKernelGGL((k_keys<D, false>), dim3(a.nblocks), dim3(kBlock), 0, s, a.inst, a.m, a.d,
                     a.npts, a.soa, a.sa, a.sb, a.segs, a.R, a.u, a.klo, a.layout, a.keys, a.vals,
                     a.err, a.sig, a.sig_stride, a.sig_b, gpw, a.idx_bits, a.sig_fresh, 0);
}

void launch_keys(const KeysArgs& a, hipStream_t s) {
  if (!a.nblocks) return;
  switch (a.d) {
    case 1: keys_dispatch<1>(a, s); break;
    case 2: keys_dispatch<2>(a, s); break;
    case 3: keys_dispatch<3>(a, s); break;
    case 4: keys_dispatch<4>(a, s); break;
    case 5: keys_dispatch<5>(a, s); break;
    case 6: keys_dispatch<6>(a, s); break;
    case 7: keys_dispatch<7>(a, s); break;
    case 8: keys_dispatch<8>(a, s); break;
    case 9: keys_dispatch<9>(a, s); break;
    case 10: keys_dispatch<10>(a, s); break;
    case 11: keys_dispatch<11>(a, s); break;
    case 12: keys_dispatch<12>(a, s); break;
    case 13: keys_dispatch<13>(a, s); break;
    case 14: keys_dispatch<14>(a, s); break;
    case 15: keys_dispatch<15>(a, s); break;
    case 16: keys_dispatch<16>(a, s); break;
    default: keys_dispatch<0>(a, s);
  }
}

template <int D>
static void coords_dispatch(const float* soa, int64_t n, int d, const double* R, const double* u,
                            double inv_c, int64_t* kappa, uint32_t* err, hipStream_t s) {
  hipLaunchKernelGGL(k_cell_coords<D>, dim3(grid_for((size_t)n)), dim3(kBlock), 0, s, soa, n, d, R,
                     u, inv_c, kappa, err);
}

void launch_cell_coords(const float* soa, int64_t n, int d, const double* R, const double* u,
                        double inv_c, int64_t* kappa, uint32_t* err, hipStream_t s) {
  if (n <= 0) return;
#define RTG_COORDS_CASE(DV) \
  case DV: coords_dispatch<DV>(soa, n, d, R, u, inv_c, kappa, err, s); break;
  switch (d) {
    RTG_COORDS_CASE(1) RTG_COORDS_CASE(2) RTG_COORDS_CASE(3) RTG_COORDS_CASE(4)
    RTG_COORDS_CASE(5) RTG_COORDS_CASE(6) RTG_COORDS_CASE(7) RTG_COORDS_CASE(8)
    RTG_COORDS_CASE(9) RTG_COORDS_CASE(10) RTG_COORDS_CASE(11) RTG_COORDS_CASE(12)
    RTG_COORDS_CASE(13) RTG_COORDS_CASE(14) RTG_COORDS_CASE(15) RTG_COORDS_CASE(16)
    default: coords_dispatch<0>(soa, n, d, R, u, inv_c, kappa, err, s);
  }
#undef RTG_COORDS_CASE
}

size_t scan_scratch_elems(size_t count) {
  size_t total = 0;
  while (count > (size_t)kScanTile) {
    count = (count + kScanTile - 1) / kScanTile;
    total += count;
  }
  return total + 1;
}

template <typename T>
static void scan_rec(const T* in, T* out, size_t count, T* total, T* scratch, hipStream_t s,
                     const uint32_t* dcount = nullptr) {
  if (count == 0) {
    if (total) hipLaunchKernelGGL(k_fill<T>, dim3(1), dim3(64), 0, s, total, (T)0, (size_t)1);
    return;
  }
  if (count <= (size_t)kScanTile) {
    hipLaunchKernelGGL(k_scan_apply<T>, dim3(1), dim3(kBlock), 0, s, in, out, count,
                       (const T*)nullptr, total, dcount);
    return;
  }
  const size_t nb = (count + kScanTile - 1) / kScanTile;
  T* sums = scratch;
  hipLaunchKernelGGL(k_scan_reduce<T>, dim3((unsigned)nb), dim3(kBlock), 0, s, in, count, sums,
                     dcount);
  if (nb <= (size_t)kFusedScanSums) {
    // each block adds up the sums before it: two launches instead of three
    hipLaunchKernelGGL((k_scan_apply<T, true>), dim3((unsigned)nb), dim3(kBlock), 0, s, in, out,
                       count, (const T*)sums, total, dcount);
    return;
  }
  scan_rec<T>(sums, sums, nb, (T*)nullptr, scratch + nb, s);
  hipLaunchKernelGGL(k_scan_apply<T>, dim3((unsigned)nb), dim3(kBlock), 0, s, in, out, count,
                     (const T*)sums, total, dcount);
}

void scan_exclusive_u32(const uint32_t* in, uint32_t* out, size_t count, uint32_t* total,
                        uint32_t* scratch, hipStream_t s, const uint32_t* dcount) {
  scan_rec<uint32_t>(in, out, count, total, scratch, s, dcount);
}

void scan_exclusive_u64(const uint64_t* in, uint64_t* out, size_t count, uint64_t* total,
                        uint64_t* scratch, hipStream_t s, const uint32_t* dcount) {
  scan_rec<uint64_t>(in, out, count, total, scratch, s, dcount);
}

size_t radix_scratch_bytes(size_t count, int begin_bit, int end_bit, size_t extra_tiles) {
  auto up = [](size_t b) { return (b + 255) & ~(size_t)255; };
  const size_t ntiles = tiles_for(count) + extra_tiles;
  const int npass = std::max(1, (end_bit - begin_bit + kRadixBits - 1) / kRadixBits);
  const size_t nbh = (count + (size_t)kHistBlockTiles * kTile - 1) / ((size_t)kHistBlockTiles * kTile);
  const size_t onesweep = up(nbh * npass * 256 * 4) + up((size_t)npass * 256 * 8) +
                          up(ntiles * 256 * 8) + up((size_t)npass * 4);
  const size_t h = (size_t)256 * ntiles;
  const size_t rts = up(4 * (h + scan_scratch_elems(h)));
  return std::max(onesweep, rts) + 256;
}

int radix_sort(uint64_t* keys, uint32_t* vals, uint64_t* keys_alt, uint32_t* vals_alt,
               size_t count, int begin_bit, int end_bit, void* scratch, uint32_t* err,
               hipStream_t s, const LaunchTimer* timer, int kid_hist, int kid_scatter, int algo,
               const SortTile* tiles, uint32_t ntiles_table) {
  const LaunchTimer none;
  const LaunchTimer& tm = timer ? *timer : none;
  const double elem = vals ? 12.0 : 8.0;
  if (count <= 1 || end_bit <= begin_bit) return 0;
  auto up = [](size_t b) { return (b + 255) & ~(size_t)255; };
  const unsigned ntiles = tiles_for(count);
  char* base = static_cast<char*>(scratch);
  uint64_t *kin = keys, *kout = keys_alt;
  uint32_t *vin = vals, *vout = vals_alt;
  int where = 0;
  if (algo == kSortOnesweep) {
    const int npass = (end_bit - begin_bit + kRadixBits - 1) / kRadixBits;
    const size_t nbh =
        (count + (size_t)kHistBlockTiles * kTile - 1) / ((size_t)kHistBlockTiles * kTile);
    uint32_t* part = reinterpret_cast<uint32_t*>(base);
    base += up(nbh * npass * 256 * 4);
    uint64_t* digit_off = reinterpret_cast<uint64_t*>(base);
    base += up((size_t)npass * 256 * 8);
    unsigned long long* status = reinterpret_cast<unsigned long long*>(base);
    base += up((size_t)ntiles * 256 * 8);
    unsigned int* counters = reinterpret_cast<unsigned int*>(base);
    tm.on_begin(kid_hist);
    hipLaunchKernelGGL(k_hist_all, dim3((unsigned)nbh), dim3(kBlock), 0, s, kin, count, begin_bit,
                       end_bit, part);
    hipLaunchKernelGGL(k_hist_scan, dim3(npass), dim3(kBlock), 0, s, part, (uint32_t)nbh, npass,
                       digit_off);
    tm.on_end(kid_hist, 8.0 * (double)count);
    hipLaunchKernelGGL(k_fill<unsigned int>, dim3(1), dim3(64), 0, s, counters, 0u, (size_t)npass);
    for (int p = 0; p < npass; ++p) {
      const int b = begin_bit + p * kRadixBits;
      const int nbits = std::min(kRadixBits, end_bit - b);
      launch_fill_u64(reinterpret_cast<uint64_t*>(status), 0ull, (size_t)ntiles * 256, s);
      tm.on_begin(kid_scatter);
      if (vals)
        hipLaunchKernelGGL(k_onesweep<true>, dim3(ntiles), dim3(kBlock), 0, s, kin, vin, kout, vout,
                           count, b, nbits, digit_off + (size_t)p * 256, status, counters + p, err);
      else
        hipLaunchKernelGGL(k_onesweep<false>, dim3(ntiles), dim3(kBlock), 0, s, kin,
                           (const uint32_t*)nullptr, kout, (uint32_t*)nullptr, count, b, nbits,
                           digit_off + (size_t)p * 256, status, counters + p, err);
      tm.on_end(kid_scatter, 2.0 * elem * (double)count);
      std::swap(kin, kout);
      std::swap(vin, vout);
      where ^= 1;
    }
    return where;
  }
  const unsigned nt = tiles ? ntiles_table : ntiles;
  if (nt == 0) return 0;
  uint32_t* hist = reinterpret_cast<uint32_t*>(base);
  uint32_t* sscr = hist + (size_t)256 * nt;
  for (int b = begin_bit; b < end_bit; b += kRadixBits) {
    const int nbits = (end_bit - b) < kRadixBits ? (end_bit - b) : kRadixBits;
    tm.on_begin(kid_hist);
    hipLaunchKernelGGL(k_radix_hist, dim3(nt), dim3(kBlock), 0, s, kin, count, b, nbits, hist, nt,
                       tiles);
    tm.on_end(kid_hist, 8.0 * (double)count);
    scan_rec<uint32_t>(hist, hist, (size_t)256 * nt, (uint32_t*)nullptr, sscr, s);
    tm.on_begin(kid_scatter);
    if (vals)
      hipLaunchKernelGGL(k_radix_scatter<true>, dim3(nt), dim3(kBlock), 0, s, kin, vin, kout,
                         vout, count, b, nbits, hist, nt, tiles);
    else
      hipLaunchKernelGGL(k_radix_scatter<false>, dim3(nt), dim3(kBlock), 0, s, kin,
                         (const uint32_t*)nullptr, kout, (uint32_t*)nullptr, count, b, nbits, hist,
                         nt, tiles);
    tm.on_end(kid_scatter, 2.0 * elem * (double)count);
    std::swap(kin, kout);
    std::swap(vin, vout);
    where ^= 1;
  }
  return where;
}

void launch_seg_sort(uint64_t* keys, const SortTile* segs, uint32_t nsegs, int begin_bit,
                     int end_bit, hipStream_t s) {
  if (!nsegs || end_bit <= begin_bit) return;
  hipLaunchKernelGGL(k_seg_sort, dim3(nsegs), dim3(kSegThreads), 0, s, keys, segs, begin_bit,
                     end_bit);
}

size_t run_mask_words(size_t count) { return 2 * ((count + 63) / 64); }

void launch_run_count(const uint64_t* keys, size_t count, int shift, uint32_t* head_cnt,
                      uint32_t* tail_cnt, uint64_t* masks, hipStream_t s) {
  if (!count) return;
  hipLaunchKernelGGL(k_run_count, dim3(tiles_for(count)), dim3(kBlock), 0, s, keys, count, shift,
                     head_cnt, tail_cnt, masks);
}

void launch_run_write(const uint64_t* masks, size_t count, const uint32_t* head_off,
                      const uint32_t* tail_off, uint32_t* start, uint32_t* end, uint32_t* tot,
                      unsigned long long* zero, hipStream_t s) {
  if (!count) return;
  if (tot)
    hipLaunchKernelGGL(k_run_write<true>, dim3(tiles_for(count)), dim3(kBlock), 0, s, masks, count,
                       head_off, tail_off, start, end, tot, zero);
  else
    hipLaunchKernelGGL(k_run_write<false>, dim3(tiles_for(count)), dim3(kBlock), 0, s, masks,
                       count, head_off, tail_off, start, end, (uint32_t*)nullptr,
                       (unsigned long long*)nullptr);
}

// Grid of the cell kernels: one thread per cell up to 2048 blocks, then
// every thread takes more (with a device count the host knows only a bound).
static unsigned cell_grid(uint32_t ncells) {
  return (unsigned)std::min<size_t>(grid_for(ncells), 2048);
}

void launch_cell_work(const uint32_t* start, const uint32_t* end, uint32_t ncells,
                      const uint32_t* dcells, uint32_t cell_unit_tiles, uint32_t* units,
                      uint64_t* tests, unsigned long long* members, hipStream_t s) {
  if (!ncells) return;
  hipLaunchKernelGGL(k_cell_work, dim3(cell_grid(ncells)), dim3(kBlock), 0, s, start, end, ncells,
                     dcells, cell_unit_tiles, units, tests, members);
}

bool launch_cell_work_scanned(const uint32_t* start, const uint32_t* end, uint32_t ncells,
                              const uint32_t* dcells, uint32_t cell_unit_tiles, uint32_t* units,
                              uint64_t* tests, unsigned long long* members, uint32_t* usums,
                              uint32_t* utotal, uint64_t* tsums, uint64_t* ttotal, hipStream_t s) {
  const size_t nb = ((size_t)ncells + kScanTile - 1) / kScanTile;
  if (!ncells || nb > (size_t)kFusedScanSums) return false;
  hipLaunchKernelGGL(k_cell_work_tiles, dim3((unsigned)nb), dim3(kBlock), 0, s, start, end, ncells,
                     dcells, cell_unit_tiles, units, tests, members, usums, tsums);
  hipLaunchKernelGGL((k_scan_apply<uint32_t, true>), dim3((unsigned)nb), dim3(kBlock), 0, s, units,
                     units, (size_t)ncells, (const uint32_t*)usums, utotal, dcells);
  hipLaunchKernelGGL((k_scan_apply<uint64_t, true>), dim3((unsigned)nb), dim3(kBlock), 0, s, tests,
                     tests, (size_t)ncells, (const uint64_t*)tsums, ttotal, dcells);
  return true;
}

void launch_unit_fill(const uint32_t* start, const uint32_t* end, const uint32_t* unit_off,
                      uint32_t ncells, const uint32_t* dcells, uint32_t cell_unit_tiles,
                      const uint64_t* skeys, int seg_shift, int sa, const SegDesc* segs,
                      UnitDesc* desc, uint64_t* work, hipStream_t s) {
  if (!ncells) return;
  hipLaunchKernelGGL(k_unit_fill, dim3(cell_grid(ncells)), dim3(kBlock), 0, s, start, end,
                     unit_off, ncells, dcells, cell_unit_tiles, skeys, seg_shift, sa, segs, desc,
                     work);
}

uint32_t pair_waves(const PairsArgs& a) {
  uint64_t blocks = ((uint64_t)a.total_units + kWaves - 1) / kWaves;
  const uint64_t max_blocks = a.max_blocks ? a.max_blocks : 256ull * 8ull;
  if (blocks > max_blocks) blocks = max_blocks;
  if (blocks < 1) blocks = 1;
  return (uint32_t)blocks * kWaves;
}

void launch_wave_ranges(const uint64_t* work_off, uint32_t nunits, const uint64_t* total,
                        uint32_t nwaves, uint32_t* first, hipStream_t s) {
  hipLaunchKernelGGL(k_wave_ranges, dim3(grid_for((size_t)nwaves + 1)), dim3(kBlock), 0, s,
                     work_off, nunits, total, nwaves, first);
}

void launch_gather_units(const PairsArgs& a, const uint64_t* sig, float* spts, uint64_t* ssig,
                         hipStream_t s) {
  if (!a.total_units) return;
  const unsigned blocks = (unsigned)(((uint64_t)a.total_units + kWaves - 1) / kWaves);
#define RTG_GATHER(DD) \
  hipLaunchKernelGGL(k_gather_units<DD>, dim3(blocks), dim3(kBlock), 0, s, a, sig, spts, ssig)
  switch (a.d) {
    case 1: RTG_GATHER(1); break;
    case 2: RTG_GATHER(2); break;
    case 3: RTG_GATHER(3); break;
    case 4: RTG_GATHER(4); break;
    case 5: RTG_GATHER(5); break;
    case 6: RTG_GATHER(6); break;
    case 7: RTG_GATHER(7); break;
    case 8: RTG_GATHER(8); break;
    case 9: RTG_GATHER(9); break;
    case 10: RTG_GATHER(10); break;
    case 11: RTG_GATHER(11); break;
    case 12: RTG_GATHER(12); break;
    case 13: RTG_GATHER(13); break;
    case 14: RTG_GATHER(14); break;
    case 15: RTG_GATHER(15); break;
    case 16: RTG_GATHER(16); break;
    default: RTG_GATHER(0); break;
  }
#undef RTG_GATHER
}

// Dimensions with their own query kernels; the others read coordinates one
// by one.
#define RTG_QUERY_DIMS(X) \
  RTG_QUERY_ROW_DIMS(X) X(16)
#define RTG_QUERY_ROW_DIMS(X) \
  X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12)

// (At d = 16 a row is half a line wherever it lies: 300000 queries of 20000
// points, 1644 us from the copy, 1510 by point index.)
bool query_rows_fit(int d) { return d >= 1 && d <= 12; }

void launch_query_rows(const QueryGrid* grids, int k, int64_t n, int d, const float* pts,
                       float* rows, hipStream_t s) {
  const dim3 grid(grid_for((size_t)n), (unsigned)k);
  switch (d) {
#define RTG_QR(DD) \
  case DD: hipLaunchKernelGGL(k_query_rows<DD>, grid, dim3(kBlock), 0, s, grids, n, pts, rows); break;
    RTG_QUERY_ROW_DIMS(RTG_QR)
#undef RTG_QR
  }
}

void launch_query_table(const QueryGrid* grids, int k, int64_t n, int cell_bits, int tab_bits,
                        uint32_t* tab, hipStream_t s) {
  hipLaunchKernelGGL(k_query_table, dim3(grid_for(((size_t)1 << tab_bits) + 1), (unsigned)k),
                     dim3(kBlock), 0, s, grids, k, (uint32_t)n, cell_bits, tab_bits, tab);
}

void launch_query_order(const QueryArgs& a, int bits, uint64_t* order, hipStream_t s) {
  const unsigned blocks = grid_for((size_t)a.m);
#define RTG_QO(DD)                                                                               \
  hipLaunchKernelGGL(k_query_order<DD>, dim3(blocks), dim3(kBlock), 0, s, a, a.R, a.u, a.klo,    \
                     a.layout, bits, order)
  switch (a.d) {
#define RTG_QO_CASE(DD) \
  case DD: RTG_QO(DD); break;
    RTG_QUERY_DIMS(RTG_QO_CASE)
#undef RTG_QO_CASE
    default: RTG_QO(0);
  }
#undef RTG_QO
}

void launch_query_find(const QueryArgs& a, hipStream_t s) {
  if (a.m <= 0 || a.n <= 0) return;
  const unsigned blocks = (unsigned)((a.m + 63) / 64);
#define RTG_QF(DD)                                                                             \
  hipLaunchKernelGGL(k_query_find<DD>, dim3(blocks), dim3(kBlock), 0, s, a, a.R, a.u, a.klo,   \
                     a.layout, a.grids, a.tab, a.qlo, a.qsig)
  switch (a.d) {
#define RTG_QF_CASE(DD) \
  case DD: RTG_QF(DD); break;
    RTG_QUERY_DIMS(RTG_QF_CASE)
#undef RTG_QF_CASE
    default: RTG_QF(0);
  }
#undef RTG_QF
}

static void query_dispatch(const QueryArgs& a, unsigned blocks, bool long_cells, hipStream_t s) {
#define RTG_QP(DD, RR)                                                                          \
  do {                                                                                          \
    if (long_cells)                                                                             \
      hipLaunchKernelGGL((k_query_long<DD, RR>), dim3(blocks), dim3(kBlock), 0, s, a);          \
    else                                                                                        \
      hipLaunchKernelGGL((k_query_pairs<DD, RR>), dim3(blocks), dim3(kBlock), 0, s, a);         \
  } while (0)
  switch (a.d) {
#define RTG_QP_CASE(DD)           \
  case DD:                        \
    if (a.rows) RTG_QP(DD, true); \
    else RTG_QP(DD, false);       \
    break;
    RTG_QUERY_ROW_DIMS(RTG_QP_CASE)
    case 16: RTG_QP(16, false); break;
#undef RTG_QP_CASE
    default: RTG_QP(0, false);
  }
#undef RTG_QP
}

// Lanes per query: 1e6 queries (n = 1e6, d = 3, about 29 points a cell) took
// 1.28 / 1.06 / 1.00 / 1.12 ms with 1 / 2 / 4 / 8; above d = 6, where cells are
// longer and uneven, 8 (1e5 queries of 1e5 points, d = 9: 1252 / 1119 / 1102 us
// with 4 / 8 / 16; 1e6 of 1000 points, cells of a few, 1280 with 8 and 1495 with
// 16), above d = 12 16 (300000 of 20000, d = 13: 7325 us with 8, 6792 with 16);
// few queries get as many as give the chip 2^18 lanes.  At d = 5 and 6 (cells of about a hundred
// points) queries that are not in order get 32: each cell then comes from HBM
// in a few wide steps (50000 queries of 1e6 points, d = 6: 1212 us with 8,
// 1021 with 32; 33000: 720 and 718).
uint32_t query_lanes(int d, int64_t m) {
  uint32_t lanes = d > 12 ? 16 : d > 6 ? 8 : d > 4 && m < 65536 ? 32 : 4;
  while (lanes < 64 && (uint64_t)m * lanes < (1u << 18)) lanes *= 2;
  return lanes;
}

void launch_query_pairs(const QueryArgs& args, hipStream_t s) {
  if (args.m <= 0 || args.n <= 0) return;
  QueryArgs a = args;
  a.lanes = query_lanes(a.d, a.m);
  uint64_t blocks = ((uint64_t)a.m * a.lanes + kBlock - 1) / kBlock;
  if (blocks > 4096) blocks = 4096;
  query_dispatch(a, (unsigned)blocks, false, s);
}

void launch_query_long(const QueryArgs& args, hipStream_t s) {
  if (args.m <= 0 || args.n <= 0) return;
  // about 16384 waves, each with as many cells to look at (at most 64)
  QueryArgs a = args;
  const uint64_t cells = (uint64_t)a.m * (uint64_t)a.k;
  a.lanes = (uint32_t)std::min<uint64_t>(64, (cells + 16383) / 16384);
  const uint64_t waves = std::min<uint64_t>(16384, (cells + a.lanes - 1) / a.lanes);
  query_dispatch(a, (unsigned)((waves + kWaves - 1) / kWaves), true, s);
}

void launch_seg_compact(const uint64_t* src, uint64_t seg_cap, const unsigned long long* cnt,
                        uint32_t nseg, uint64_t max_count, uint64_t* dst, hipStream_t s) {
  if (nseg == 0 || max_count == 0) return;
  uint64_t bx = (max_count + kBlock * 4 - 1) / (kBlock * 4);
  if (bx > 512) bx = 512;
  hipLaunchKernelGGL(k_seg_compact, dim3((unsigned)bx, nseg), dim3(kBlock), 0, s, src, seg_cap,
                     cnt, dst);
}

static unsigned compact_blocks(uint64_t count) {
  const uint64_t tile = (uint64_t)kBlock * kCompactPer;
  const uint64_t blocks = (count + tile - 1) / tile;
  return (unsigned)(blocks > 4096 ? 4096 : blocks);
}

void launch_mr_filter(const MrFilterArgs& a, hipStream_t s) {
  if (a.count == 0) return;
  hipLaunchKernelGGL(k_mr_filter, dim3(compact_blocks(a.count)), dim3(kBlock), 0, s, a);
}

void launch_bitmap_unique(const BitmapArgs& a, hipStream_t s) {
  if (a.count == 0) return;
  hipLaunchKernelGGL(k_bitmap_unique, dim3(compact_blocks(a.count)), dim3(kBlock), 0, s, a);
}

template <int D>
static void pairs_dispatch(const PairsArgs& a, hipStream_t s) {
  // 256 CUs, several resident blocks each (the grid wave_first was made for)
  const uint64_t blocks = pair_waves(a) / kWaves;
  if constexpr (D <= 16) {
    if (a.gram && a.d == D) {
      if (a.mr)
        hipLaunchKernelGGL((k_cell_pairs_gram<D, 2>), dim3((unsigned)blocks), dim3(kBlock), 0, s, a);
      else if (a.same_cell)
        hipLaunchKernelGGL((k_cell_pairs_gram<D, 1>), dim3((unsigned)blocks), dim3(kBlock), 0, s, a);
      else
        hipLaunchKernelGGL((k_cell_pairs_gram<D, 0>), dim3((unsigned)blocks), dim3(kBlock), 0, s, a);
      return;
    }
  }
  hipLaunchKernelGGL((k_cell_pairs<D>), dim3((unsigned)blocks), dim3(kBlock), 0, s, a);
}

void launch_tiny(const TinyArgs& a, int d, int k, hipStream_t s) {
#define RTG_TINY(DD) \
  hipLaunchKernelGGL(k_tiny_grids<DD>, dim3(k * a.parts), dim3(kTinyThreads), 0, s, a)
  switch (d) {
    case 1: RTG_TINY(1); break;
    case 2: RTG_TINY(2); break;
    case 3: RTG_TINY(3); break;
    case 4: RTG_TINY(4); break;
    case 5: RTG_TINY(5); break;
    case 6: RTG_TINY(6); break;
    case 7: RTG_TINY(7); break;
    case 8: RTG_TINY(8); break;
    default: return;
  }
#undef RTG_TINY
  hipLaunchKernelGGL(k_tiny_lists, dim3((a.n + kTinyListRows - 1) / kTinyListRows),
                     dim3(kTinyListThreads), 0, s, a);
}

void launch_cell_pairs(const PairsArgs& a, hipStream_t s) {
  if (!a.total_units) return;
  const int d = a.d;
#define RTG_PAIRS_ARGS a, s
  // Instantiations for d <= 16 exactly; larger d run the next wider one with
  // zero padding, which adds exact zeros to both sums.
  switch (d) {
    case 1: pairs_dispatch<1>(RTG_PAIRS_ARGS); break;
    case 2: pairs_dispatch<2>(RTG_PAIRS_ARGS); break;
    case 3: pairs_dispatch<3>(RTG_PAIRS_ARGS); break;
    case 4: pairs_dispatch<4>(RTG_PAIRS_ARGS); break;
    case 5: pairs_dispatch<5>(RTG_PAIRS_ARGS); break;
    case 6: pairs_dispatch<6>(RTG_PAIRS_ARGS); break;
    case 7: pairs_dispatch<7>(RTG_PAIRS_ARGS); break;
    case 8: pairs_dispatch<8>(RTG_PAIRS_ARGS); break;
    case 9: pairs_dispatch<9>(RTG_PAIRS_ARGS); break;
    case 10: pairs_dispatch<10>(RTG_PAIRS_ARGS); break;
    case 11: pairs_dispatch<11>(RTG_PAIRS_ARGS); break;
    case 12: pairs_dispatch<12>(RTG_PAIRS_ARGS); break;
    case 13: pairs_dispatch<13>(RTG_PAIRS_ARGS); break;
    case 14: pairs_dispatch<14>(RTG_PAIRS_ARGS); break;
    case 15: pairs_dispatch<15>(RTG_PAIRS_ARGS); break;
    case 16: pairs_dispatch<16>(RTG_PAIRS_ARGS); break;
    default:
      if (d <= 24) pairs_dispatch<24>(RTG_PAIRS_ARGS);
      else if (d <= 32) pairs_dispatch<32>(RTG_PAIRS_ARGS);
      else if (d <= 48) pairs_dispatch<48>(RTG_PAIRS_ARGS);
      else pairs_dispatch<64>(RTG_PAIRS_ARGS);
  }
#undef RTG_PAIRS_ARGS
}

void launch_unique_count(const uint64_t* keys, size_t count, uint32_t* tile_cnt, hipStream_t s) {
  if (!count) return;
  hipLaunchKernelGGL(k_unique_count, dim3(tiles_for(count)), dim3(kBlock), 0, s, keys, count,
                     tile_cnt);
}

void launch_unique_write(const uint64_t* keys, size_t count, const uint32_t* tile_off,
                         uint64_t* out, hipStream_t s) {
  if (!count) return;
  hipLaunchKernelGGL(k_unique_write, dim3(tiles_for(count)), dim3(kBlock), 0, s, keys, count,
                     tile_off, out);
}

void launch_swap_pairs(const uint64_t* pairs, size_t count, int pair_bits, uint64_t* swapped,
                       hipStream_t s) {
  if (!count) return;
  hipLaunchKernelGGL(k_swap_pairs, dim3(grid_for(count)), dim3(kBlock), 0, s, pairs, count,
                     pair_bits, swapped);
}

void launch_row_runs(const uint64_t* keys, size_t count, int pair_bits, uint32_t* rstart,
                     uint32_t* rend, hipStream_t s) {
  if (!count) return;
  hipLaunchKernelGGL(k_row_runs, dim3(grid_for(count)), dim3(kBlock), 0, s, keys, count, pair_bits,
                     rstart, rend);
}

void launch_row_degree(const uint32_t* lo_start, const uint32_t* lo_end, const uint32_t* up_start,
                       const uint32_t* up_end, int64_t n, uint64_t* deg, hipStream_t s) {
  if (n <= 0) return;
  hipLaunchKernelGGL(k_row_degree, dim3(grid_for((size_t)n)), dim3(kBlock), 0, s, lo_start, lo_end,
                     up_start, up_end, n, deg);
}

void launch_csr_fill_upper(const uint64_t* up, size_t count, int pair_bits, const int64_t* row_ptr,
                           const uint32_t* lo_start, const uint32_t* lo_end,
                           const uint32_t* up_start, int32_t* col, hipStream_t s) {
  if (!count) return;
  hipLaunchKernelGGL(k_csr_fill_upper, dim3(grid_for(count)), dim3(kBlock), 0, s, up, count,
                     pair_bits, row_ptr, lo_start, lo_end, up_start, col);
}

void launch_csr_fill_lower(const uint64_t* lo, size_t count, int pair_bits, const int64_t* row_ptr,
                           const uint32_t* lo_start, int32_t* col, hipStream_t s) {
  if (!count) return;
  hipLaunchKernelGGL(k_csr_fill_lower, dim3(grid_for(count)), dim3(kBlock), 0, s, lo, count,
                     pair_bits, row_ptr, lo_start, col);
}

// --- row buckets ------------------------------------------------------------

void launch_bucket_hist(const PairSource& src, size_t count, int pb, int rb, int both,
                        uint32_t nbuckets, uint32_t chunk, uint32_t nblocks, int threads,
                        uint32_t* part, uint32_t* zero_word, hipStream_t s) {
  if (!nblocks) {
    if (zero_word) launch_fill_u32(zero_word, 0u, 1, s);
    return;
  }
  const size_t lds = nbuckets * sizeof(uint32_t);
  if (threads >= 1024)
    hipLaunchKernelGGL(k_bucket_hist<1024>, dim3(nblocks), dim3(1024), lds, s, src.pairs, count,
                       pb, rb, both, nbuckets, chunk, nblocks, src.seg_cnt, src.seg_cap,
                       src.nseg, part, zero_word);
  else
    hipLaunchKernelGGL(k_bucket_hist<kBlock>, dim3(nblocks), dim3(kBlock), lds, s, src.pairs,
                       count, pb, rb, both, nbuckets, chunk, nblocks, src.seg_cnt, src.seg_cap,
                       src.nseg, part, zero_word);
}

void launch_bucket_scatter(const PairSource& src, size_t count, int pb, int rb, int both,
                           uint32_t nbuckets, uint32_t chunk, uint32_t nblocks, int threads,
                           const uint32_t* offs, uint32_t* entries, hipStream_t s) {
  if (!nblocks) return;
  const size_t lds = nbuckets * sizeof(uint32_t);
  if (threads >= 1024)
    hipLaunchKernelGGL(k_bucket_scatter<1024>, dim3(nblocks), dim3(1024), lds, s, src.pairs,
                       count, pb, rb, both, nbuckets, chunk, nblocks, src.seg_cnt, src.seg_cap,
                       src.nseg, offs, entries);
  else
    hipLaunchKernelGGL(k_bucket_scatter<kBlock>, dim3(nblocks), dim3(kBlock), lds, s, src.pairs,
                       count, pb, rb, both, nbuckets, chunk, nblocks, src.seg_cnt, src.seg_cap,
                       src.nseg, offs, entries);
}

void launch_bucket_csr(const uint32_t* entries, const uint32_t* offs, uint32_t nbuckets,
                       uint32_t nblocks, const uint32_t* total, uint32_t* oversized,
                       uint32_t* n_oversized, uint32_t cap, int pb, int rb, int64_t n,
                       int64_t nnz, int64_t* row_ptr, int32_t* col, hipStream_t s) {
  if (!nbuckets) {
    launch_fill_u64(reinterpret_cast<uint64_t*>(row_ptr + n), (uint64_t)nnz, 1, s);
    return;
  }
  if (cap > (uint32_t)kBucketMaxEntries) cap = kBucketMaxEntries;
  hipLaunchKernelGGL(k_bucket_csr, dim3(nbuckets), dim3(kCsrThreads), 0, s, entries, offs,
                     nbuckets, nblocks, total, oversized, n_oversized, cap, pb, rb, n, nnz, row_ptr,
                     col);
}

void launch_over_extent(const uint32_t* ids, uint32_t nover, const uint32_t* part,
                        uint32_t nblocks, uint32_t nbuckets, size_t np, uint32_t* start,
                        uint32_t* cnt, hipStream_t s) {
  if (!nover) return;
  hipLaunchKernelGGL(k_over_extent, dim3(grid_for(nover)), dim3(kBlock), 0, s, ids, nover, part,
                     nblocks, nbuckets, np, start, cnt);
}

void launch_over_gather(const uint32_t* entries, const uint32_t* start, const uint32_t* off,
                        uint32_t nover, uint32_t tot, int sh, uint64_t* w, hipStream_t s) {
  if (!nover || !tot) return;
  hipLaunchKernelGGL(k_over_gather, dim3(grid_for(tot)), dim3(kBlock), 0, s, entries, start, off,
                     nover, tot, sh, w);
}

void launch_over_emit(const uint64_t* keys, uint32_t tot, const uint32_t* ids,
                      const uint32_t* start, const uint32_t* cnt, const uint32_t* off, int pb,
                      int rb, int64_t n, int64_t* row_ptr, int32_t* col, hipStream_t s) {
  if (!tot) return;
  hipLaunchKernelGGL(k_over_emit, dim3(grid_for(tot)), dim3(kBlock), 0, s, keys, tot, ids, start,
                     cnt, off, pb, rb, n, row_ptr, col);
}

void launch_u32_to_u64(const uint32_t* src, size_t count, uint64_t* dst, hipStream_t s) {
  if (count == 0) return;
  hipLaunchKernelGGL(k_widen, dim3(grid_for(count)), dim3(kBlock), 0, s, src, count, dst);
}

void launch_mailbox(const uint32_t* src, uint32_t words, const Gather* g, uint32_t* host,
                    uint64_t* host_seq, uint64_t seq, hipStream_t s) {
  hipLaunchKernelGGL(k_mailbox, dim3(1), dim3(kBlock), 0, s, src, words, g ? *g : Gather{}, host,
                     host_seq, seq);
}

void launch_records(const float* rows, int64_t n, int d, int rs, float* rec, hipStream_t s) {
  if (n <= 0) return;
  hipLaunchKernelGGL(k_records, dim3(grid_for((size_t)n)), dim3(kBlock), 0, s, rows, n, d, rs,
                     rec);
}

void launch_rowptr_at(const InstDesc* inst, uint32_t m, const int64_t* row_ptr, int64_t npts,
                      int64_t* out, hipStream_t s) {
  hipLaunchKernelGGL(k_rowptr_at, dim3(grid_for((size_t)m + 1)), dim3(kBlock), 0, s, inst, m,
                     row_ptr, npts, out);
}

void launch_localize(const InstDesc* inst, uint32_t m, uint32_t nblocks, const int64_t* row_ptr,
                     const int32_t* col, const int64_t* at, int64_t total, int64_t* const* out_rp,
                     int32_t* const* out_col, hipStream_t s) {
  if (nblocks)
    hipLaunchKernelGGL(k_localize_rows, dim3(nblocks), dim3(kBlock), 0, s, inst, m, row_ptr,
                       out_rp);
  if (total > 0 && m > 0)
    hipLaunchKernelGGL(k_localize_cols,
                       dim3((unsigned)((total + kLocalizePer * kBlock - 1) / (kLocalizePer * kBlock))),
                       dim3(kBlock), 0, s, inst, m, at, col, out_col);
}

// --- memory for callers that cannot allocate ----------------------------------
// All scratch and the result of rtg_all_pairs_noalloc live here.  In host
// code the name is only a stand-in for the array, not a device address: the
// host side uses the address that noalloc_scratch_address returns for the
// current device, and the kernels get pointers into it as arguments.
static __device__ __align__(256) unsigned char scratch[kNoallocBytes];

int noalloc_scratch_address(void** ptr) {
  *ptr = nullptr;
  const hipError_t e = hipGetSymbolAddress(ptr, HIP_SYMBOL(scratch));
  if (e != hipSuccess) {
    (void)hipGetLastError();
    *ptr = nullptr;
    return (int)e;
  }
  return 0;
}

}  // namespace rtgk
