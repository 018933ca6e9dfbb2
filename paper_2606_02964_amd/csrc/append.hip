// append.hip -- gfx950 kernel that writes the fresh K/V of the packed query
// rows into their paged cache slots.
//
// One workgroup (256 threads) takes two KV heads, or all of them, of one slice:
// the n <= 16 consecutive rows of one segment that land in one cache block (the
// planner cuts every segment at block boundaries):
//   * K blocks are token-major, so each (row, head) is one contiguous d-vector
//     in both the source and the cache: 16-byte loads and stores, 16 lanes per
//     row (256 contiguous bytes for d = 128).
//   * V blocks are channel-major (the 16 tokens of one channel are adjacent),
//     so the slice is staged in LDS and written out per channel.  A half block
//     (tokens 0-7 or 8-15) that the slice covers entirely is written as one
//     16-byte store per channel; a partly covered half (the first and last
//     block of a segment) is written token by token with consecutive lanes on
//     consecutive tokens of one channel.
// A slice whose block-table entry is outside [0, num_blocks) is not written.
// The kernel is bound by HBM: it reads and writes each fresh K/V byte once.
// A full slice's heads are spread over workgroups because one workgroup of all 8
// heads runs its reads, its LDS transpose and its stores one after the other,
// in 35 KB of LDS that leave room for four per CU (20480 rows, 8 heads, d = 128:
// 1280 workgroups for 1024 places).  168 MB in 40.1 us with 8 heads a
// workgroup, 37.8 with 4, 35.6 with 2 (4.7 TB/s; a device copy reaches 4.9),
// 34.6 with 1; 128 decode rows with their attention 299.4, 299.3, 298.9 and
// 300.0 us, hence 2.  (Issuing all of a thread's loads before its stores,
// with two lanes to a V channel, took 49 us at 2 heads.)  Where two heads of a
// slice are too little work for a workgroup it takes the whole slice, eight
// heads at a time; launch_kv_append has the rule.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "append.h"

namespace msa {
namespace {

template <int D, int kHeadsPerPass>  // KV heads a workgroup takes at a time
__global__ __launch_bounds__(256) void msa_kv_append_kernel(AppendParams p) {
  constexpr int kChunks = D / 8;  // 16-byte chunks of one head vector
  constexpr int kPitch = D + 8;   // LDS row pitch (elements), breaks bank aliasing
  __shared__ __align__(16) uint16_t s_v[kHeadsPerPass][16][kPitch];

  const uint16_t* __restrict__ k_new = p.k_new;
  const uint16_t* __restrict__ v_new = p.v_new;
  uint16_t* __restrict__ k_cache = p.k_cache;
  uint16_t* __restrict__ v_cache = p.v_cache;

  const uint32_t item = blockIdx.x / (uint32_t)p.head_groups;
  const int group = (int)(blockIdx.x - item * (uint32_t)p.head_groups);
  const AppendItem it = p.items[item];
  const int32_t blk = p.block_table[(int64_t)it.seq * p.max_blocks + it.pos0 / 16];
  if (blk < 0 || blk >= p.num_blocks) return;  // uniform over the workgroup
  const int off0 = it.pos0 % 16;                // slice = tokens off0 .. off0+n-1 of the block
  const int n = it.n;
  const int tid = threadIdx.x;
  const int64_t kbase = (int64_t)blk * p.k_sb;
  const int64_t vbase = (int64_t)blk * p.v_sb;

  for (int g0 = group * kHeadsPerPass; g0 < p.num_kv_heads; g0 += p.head_groups * kHeadsPerPass) {
    const int ng = p.num_kv_heads - g0 < kHeadsPerPass ? p.num_kv_heads - g0 : kHeadsPerPass;
    // K straight to the cache; V rows into LDS (slice row i at LDS row off0 + i).
    for (int idx = tid; idx < ng * n * kChunks; idx += 256) {
      const int ch = idx % kChunks;
      const int i = (idx / kChunks) % n;
      const int gl = idx / (kChunks * n);
      const int64_t g = g0 + gl;
      const int64_t r = (int64_t)it.row0 + i;
      const uint4 kv = *reinterpret_cast<const uint4*>(k_new + r * p.kn_st + g * p.kn_sh + ch * 8);
      const uint4 vv = *reinterpret_cast<const uint4*>(v_new + r * p.vn_st + g * p.vn_sh + ch * 8);
      *reinterpret_cast<uint4*>(k_cache + kbase + g * p.k_sh + (int64_t)(off0 + i) * p.k_st +
                                ch * 8) = kv;
      *reinterpret_cast<uint4*>(&s_v[gl][off0 + i][ch * 8]) = vv;
    }
    __syncthreads();
    // V out, one half block (8 tokens) at a time.
    for (int h = 0; h < 2; ++h) {
      const int lo = off0 > 8 * h ? off0 : 8 * h;
      const int hi = off0 + n < 8 * h + 8 ? off0 + n : 8 * h + 8;
      if (lo >= hi) continue;  // the slice misses this half
      if (lo == 8 * h && hi == 8 * h + 8) {
        for (int idx = tid; idx < ng * D; idx += 256) {
          const int c = idx % D;
          const int gl = idx / D;
          uint32_t w[4];
#pragma unroll
          for (int t = 0; t < 4; ++t)
            w[t] = (uint32_t)s_v[gl][8 * h + 2 * t][c] | ((uint32_t)s_v[gl][8 * h + 2 * t + 1][c] << 16);
          *reinterpret_cast<uint4*>(v_cache + vbase + (int64_t)(g0 + gl) * p.v_sh +
                                    (int64_t)c * p.v_sd + 8 * h) = make_uint4(w[0], w[1], w[2], w[3]);
        }
      } else {
        const int w = hi - lo;
        for (int idx = tid; idx < ng * D * w; idx += 256) {
          const int t = lo + idx % w;
          const int c = (idx / w) % D;
          const int gl = idx / (w * D);
          v_cache[vbase + (int64_t)(g0 + gl) * p.v_sh + (int64_t)c * p.v_sd + t] = s_v[gl][t][c];
        }
      }
    }
    __syncthreads();
  }
}

}  // namespace

namespace {

template <int D>
int launch_heads(AppendParams p, bool whole_slices, int num_items, hipStream_t s) {
  // a workgroup per (slice, two heads); fewer, each looping over its heads,
  // where the grid would pass 2^23 workgroups
  const int passes = p.num_kv_heads / 2 + p.num_kv_heads % 2;
  const int most = (1 << 23) / num_items;
  p.head_groups = whole_slices || most < 1 ? 1 : passes <= most ? passes : most;
  const dim3 grid((uint32_t)num_items * (uint32_t)p.head_groups);
  if (whole_slices)
    hipLaunchKernelGGL((msa_kv_append_kernel<D, 8>), grid, dim3(256), 0, s, p);
  else
    hipLaunchKernelGGL((msa_kv_append_kernel<D, 2>), grid, dim3(256), 0, s, p);
  return (int)hipGetLastError();
}

}  // namespace

int launch_kv_append(const AppendParams& p, int head_dim, int num_items, void* stream) {
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (num_items <= 0) return 0;
  // One workgroup a slice, taking its heads eight at a time,
  // - where slices are short, since a workgroup's fixed cost outweighs two heads
  //   of a few rows.  The line is at 640 channels of a head, 5 rows at d = 128,
  //   10 at d = 64 (2048 slices, 8 heads, in groups of two / whole: d = 128, 1
  //   row 34.6 / 33.5 us, 4 rows 40.7 / 40.3, 6 rows 46.4 / 47.7; d = 64, 1 row
  //   20.8 / 15.6, 8 rows 25.4 / 24.5, 16 rows 27.7 / 29.7);
  // - where all heads are up to 320 channels (16384 rows, d = 64: 4 heads 9.4 /
  //   9.2 us), or an odd number of heads up to 448, whose last workgroup would
  //   hold one (d = 128, 3 heads 14.5 / 13.8; d = 64, 3 heads 8.6 / 7.2, 5 heads
  //   11.6 / 11.5; 6 heads stay in twos: 2048 full slices 21.9 / 24.3).
  const int64_t channels = (int64_t)p.num_kv_heads * head_dim;
  const bool whole = (int64_t)p.total_q * head_dim < (int64_t)640 * num_items || channels <= 320 ||
                     (channels <= 448 && p.num_kv_heads % 2 != 0);
  if (head_dim == 128) return launch_heads<128>(p, whole, num_items, s);
  if (head_dim == 64) return launch_heads<64>(p, whole, num_items, s);
  return (int)hipErrorInvalidValue;
}

}  // namespace msa
