// Fired counts of the gated convolution from its decision bitmap, and the channel mask of the
// channel-wise gate (Sec. 3.2 of the channel-gating paper) from the same sums.
#include "cg_internal.h"

namespace cg {

namespace {

// per-(image, channel) fired counts and their total from the decision bitmap: one block per
// (image, bitmap word); a wavefront takes 64 pixels at a time and counts bit b of their words with
// a ballot, lane b keeping the running count; one atomic per block adds to the total.  With `mask`
// the block instead writes the word of the channels whose count reaches `need` (the channel-wise
// gate of Sec. 3.2) and leaves `counts` alone.
__global__ void bitmap_counts_kernel(const uint32_t* __restrict__ bitmap, int words, int hw, int c_out,
                                     uint32_t* __restrict__ counts, unsigned long long* __restrict__ total,
                                     uint32_t* __restrict__ mask, uint32_t need) {
  __shared__ uint32_t cnt[32];
  const int w = blockIdx.x % words, img = blockIdx.x / words;
  const int lane = threadIdx.x & 63;
  if (threadIdx.x < 32) cnt[threadIdx.x] = 0u;
  __syncthreads();
  uint32_t mine = 0u;
  for (int base = (int)(threadIdx.x & ~63u); base < hw; base += (int)blockDim.x) {
    const int px = base + lane;
    const uint32_t v = px < hw ? bitmap[((long long)img * hw + px) * words + w] : 0u;
#pragma unroll
    for (int b = 0; b < 32; ++b) {
      const uint32_t nb = (uint32_t)__popcll(__ballot((v >> b) & 1u));
      mine += lane == b ? nb : 0u;
    }
  }
  if (lane < 32 && mine) atomicAdd(&cnt[lane], mine);
  __syncthreads();
  if (threadIdx.x < 64) {
    const int co = w * 32 + lane;
    uint32_t v = (lane < 32 && co < c_out) ? cnt[lane] : 0u;
    if (mask) {
      const unsigned long long keep = __ballot(lane < 32 && co < c_out && v >= need);
      if (lane == 0) mask[(long long)img * words + w] = (uint32_t)keep;
      return;
    }
    if (lane < 32 && co < c_out) counts[(long long)img * c_out + co] = v;
#pragma unroll
    for (int sft = 16; sft >= 1; sft >>= 1) v += (uint32_t)__shfl_xor((int)v, sft, 64);
    if (lane == 0 && v) atomicAdd(total, (unsigned long long)v);
  }
}

// The same for feature maps of a few pixels (fully connected layers are 1x1 maps): one thread per
// (image, bitmap word) walks the map's pixels, so a batch of thousands of tiny maps is a few hundred
// blocks and one atomic per block instead of one block and one atomic per word.
__global__ void bitmap_counts_small_kernel(const uint32_t* __restrict__ bitmap, int words, int hw, int c_out,
                                           long long items, uint32_t* __restrict__ counts,
                                           unsigned long long* __restrict__ total_out, uint32_t* __restrict__ mask,
                                           uint32_t need) {
  __shared__ uint32_t part[4];
  const long long id = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  uint32_t total = 0u;
  if (id < items) {
    const int w = (int)(id % words);
    const long long img = id / words;
    uint32_t keep = 0u;
    for (int b = 0; b < 32; ++b) {
      const int co = w * 32 + b;
      if (co >= c_out) break;
      uint32_t c = 0u;
      for (int px = 0; px < hw; ++px) c += (bitmap[(img * hw + px) * words + w] >> b) & 1u;
      if (mask) {
        keep |= (c >= need ? 1u : 0u) << b;
      } else {
        counts[img * c_out + co] = c;
        total += c;
      }
    }
    if (mask) mask[img * words + w] = keep;
  }
  if (mask) return;
#pragma unroll
  for (int sft = 32; sft >= 1; sft >>= 1) total += (uint32_t)__shfl_xor((int)total, sft, 64);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = total;
  __syncthreads();
  if (threadIdx.x == 0) {
    const unsigned long long v = (unsigned long long)part[0] + part[1] + part[2] + part[3];
    if (v) atomicAdd(total_out, v);
  }
}

// the channel mask from counts: one thread per word
__global__ void counts_chan_mask_kernel(const uint32_t* __restrict__ counts, int words, int c_out, long long items, uint32_t need,
                                        uint32_t* __restrict__ mask) {
  const long long id = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (id >= items) return;
  const int w = (int)(id % words);
  const long long img = id / words;
  uint32_t keep = 0u;
  for (int b = 0; b < 32 && w * 32 + b < c_out; ++b) keep |= (counts[img * c_out + w * 32 + b] >= need ? 1u : 0u) << b;
  mask[id] = keep;
}

}  // namespace

namespace {
constexpr int kSmallMap = 16;   // pixels per feature map up to which the per-thread counting kernel is used
}

hipError_t launch_bitmap_counts(const Params& p, const uint32_t* bitmap, hipStream_t s) {
  const long long blocks = (long long)p.n * p.words;
  if (blocks <= 0) return hipSuccess;
  if (p.ho * p.wo <= kSmallMap) {
    hipLaunchKernelGGL(bitmap_counts_small_kernel, dim3((unsigned)((blocks + 255) / 256)), dim3(256), 0, s, bitmap,
                       p.words, p.ho * p.wo, p.c_out, blocks, p.counts, (unsigned long long*)p.total, (uint32_t*)nullptr, 0u);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(bitmap_counts_kernel, dim3((unsigned)blocks), dim3(256), 0, s, bitmap, p.words, p.ho * p.wo,
                     p.c_out, p.counts, (unsigned long long*)p.total, (uint32_t*)nullptr, 0u);
  return hipGetLastError();
}

hipError_t launch_bitmap_chan_mask(const Params& p, const uint32_t* bitmap, uint32_t need, uint32_t* mask,
                                   hipStream_t s) {
  const long long blocks = (long long)p.n * p.words;
  if (blocks <= 0) return hipSuccess;
  if (p.ho * p.wo <= kSmallMap) {
    hipLaunchKernelGGL(bitmap_counts_small_kernel, dim3((unsigned)((blocks + 255) / 256)), dim3(256), 0, s, bitmap,
                       p.words, p.ho * p.wo, p.c_out, blocks, (uint32_t*)nullptr, (unsigned long long*)nullptr, mask, need);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(bitmap_counts_kernel, dim3((unsigned)blocks), dim3(256), 0, s, bitmap, p.words, p.ho * p.wo,
                     p.c_out, (uint32_t*)nullptr, (unsigned long long*)nullptr, mask, need);
  return hipGetLastError();
}

hipError_t launch_counts_chan_mask(const Params& p, const uint32_t* counts, uint32_t need, uint32_t* mask, hipStream_t s) {
  const long long items = (long long)p.n * p.words;
  if (items <= 0) return hipSuccess;
  hipLaunchKernelGGL(counts_chan_mask_kernel, dim3((unsigned)((items + 255) / 256)), dim3(256), 0, s, counts, p.words, p.c_out,
                     items, need, mask);
  return hipGetLastError();
}

}  // namespace cg
