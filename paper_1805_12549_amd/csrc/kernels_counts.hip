// Fired counts of the gated convolution from its decision bitmap, and the channel mask of the
// channel-wise gate (Sec. 3.2 of the channel-gating paper) from the same sums.
#include "cg_internal.h"

namespace cg {

namespace {

// Per-(image, channel) fired counts and their total from the decision bitmap; with `mask` the word of the channels
// whose count reaches `need` instead (the channel-wise gate of Sec. 3.2), and `counts` is left alone.
//
// What bounds it: atomics on one address, of which the chip does one in 12.5 ns (a block's total each: 256 blocks 3.2 us,
// 4096 blocks 50 us), so a launch has few of them (64, 128 and 256 at most measured: 256 images of 784 pixels, 4 words
// 10.2, 7.3 and 7.1 us; 256 of 49, 16 words 6.1, 5.2 and 5.9); then the latency of a load and of the steps behind it.  A
// wavefront counts 64 pixels of an (image, word) item at a time: words of four such groups are added up as bit planes,
// and a 32x32 bit transpose over the lanes leaves a channel's bits in one lane's register (25 instructions a plane, against 130
// for a ballot per channel).  In a graph, before (one block per item, ballots, an atomic per item) and now, us: 64 images of
// 784 pixels, 4 words 7.7 -> 4.7; 256 of 196, 8 words 27.4 -> 5.8; 256 of 49, 16 words 51.8 -> 5.2; 1 of 12544, 2 words
// 33.8 -> 5.7; 1 of 1024, 1 word 4.4 -> 3.0.
constexpr int kMaxBlocks = 128;

// 32x32 bit transpose over each half of the wavefront: bit j of lane i <-> bit i of lane j
__device__ __forceinline__ uint32_t transpose32(uint32_t v, int lane) {
  uint32_t m = 0x0000ffffu;
#pragma unroll
  for (int s = 16; s >= 1; s >>= 1) {
    const uint32_t p = (uint32_t)__shfl_xor((int)v, s, 64);
    v = (lane & s) ? (v & ~m) | ((p >> s) & m) : (v & m) | ((p << s) & ~m);
    m ^= m << (s >> 1);
  }
  return v;
}

// sum over the lower 32 lanes, the same in all lanes
__device__ __forceinline__ unsigned long long sum32(uint32_t v) {
  uint32_t part[2] = {v & 0xffffu, v >> 16};
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    part[i] += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)part[i], 0x111, 0xf, 0xf, true);      // row_shr:1, 2, 4, 8: a row's
    part[i] += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)part[i], 0x112, 0xf, 0xf, true);      // last lane has its sum
    part[i] += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)part[i], 0x114, 0xf, 0xf, true);
    part[i] += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)part[i], 0x118, 0xf, 0xf, true);
    part[i] = (uint32_t)__builtin_amdgcn_readlane((int)part[i], 15) + (uint32_t)__builtin_amdgcn_readlane((int)part[i], 31);
  }
  return part[0] + ((unsigned long long)part[1] << 16);
}

// x / d with magic = ceil(2^32 / d), or 0: divide
__device__ __forceinline__ unsigned divide(unsigned x, unsigned d, unsigned magic) { return magic ? __umulhi(x, magic) : x / d; }

// `wpi` wavefronts share an item (1: no exchange needed, WIDE = false); G groups of 64 pixels at a time
template <int G, bool WIDE>
__global__ void bitmap_counts_kernel(const uint32_t* __restrict__ bitmap, int words, unsigned magic, int hw, int c_out, unsigned items,
                                     int wpi_log, uint32_t* __restrict__ counts, unsigned long long* __restrict__ total_out,
                                     uint32_t* __restrict__ mask, uint32_t need) {
  __shared__ uint32_t cnt[16][32];
  __shared__ unsigned long long sum;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = (int)blockDim.x >> 6;
  const unsigned per = WIDE ? nw >> wpi_log : nw;  // items at a time
  const int mine = WIDE ? wave >> wpi_log : wave, share = WIDE ? wave & ((1 << wpi_log) - 1) : 0, step = WIDE ? 64 << wpi_log : 64;
  if (threadIdx.x == 0) sum = 0ull;
  if (WIDE && lane < 32) cnt[wave][lane] = 0u;
  __syncthreads();
  unsigned long long total = 0ull;
  for (unsigned i0 = blockIdx.x * per; i0 < items; i0 += gridDim.x * per) {      // (items < 2^31: see launch_count)
    const unsigned item = i0 + mine, img = divide(item, words, magic), w = item - img * words;
    uint32_t n = 0u;
    if (item < items) {
      const uint32_t* const src = bitmap + (size_t)img * hw * words + w;
      for (int base = share * 64; base < hw; base += G * step) {
        uint32_t v[G];
#pragma unroll
        for (int i = 0; i < G; ++i) {
          const int px = base + i * step + lane;
          v[i] = px < hw ? src[(size_t)px * words] : 0u;
        }
        if constexpr (G == 1) {
          n += (uint32_t)__popc(transpose32(v[0], lane));
        } else {                                   // the sum of four bits in three planes
          const uint32_t x = v[0] ^ v[1] ^ v[2], c = (v[0] & v[1]) | ((v[0] ^ v[1]) & v[2]), c3 = x & v[3];
          n += (uint32_t)__popc(transpose32(x ^ v[3], lane)) + 2u * (uint32_t)__popc(transpose32(c ^ c3, lane)) +
               4u * (uint32_t)__popc(transpose32(c & c3, lane));
        }
      }
      n += (uint32_t)__shfl_xor((int)n, 32, 64);
    }
    if constexpr (WIDE) {
      if (lane < 32) atomicAdd(&cnt[mine][lane], n);
      __syncthreads();
      if (share == 0 && lane < 32) {
        n = cnt[mine][lane];
        cnt[mine][lane] = 0u;
      }
      if (i0 + gridDim.x * per < items) __syncthreads();
    }
    if (item >= items || share != 0) continue;
    const int co = w * 32 + (lane & 31);
    const bool on = lane < 32 && co < c_out;
    if (mask) {
      const unsigned long long keep = __ballot(on && n >= need);
      if (lane == 0) mask[item] = (uint32_t)keep;
    } else {
      if (on) counts[(size_t)img * c_out + co] = n;
      total += sum32(on ? n : 0u);
    }
  }
  if (mask) return;
  if (lane == 0 && total) atomicAdd(&sum, total);
  __syncthreads();
  if (threadIdx.x == 0 && sum) atomicAdd(total_out, sum);
}

// The same for feature maps of at most 16 pixels (fully connected layers are 1x1 maps): a thread takes four channels of an
// image, eight threads a word, four bits spread over the bytes of a register at a time.  In the form before a thread walked a
// word's 32 channels one after the other: 173 images of 15 pixels, 4 words 50 -> 3.2 us.
// 2048 of one pixel, 128 words take 17.9 (34 MB written).
__global__ void bitmap_counts_small_kernel(const uint32_t* __restrict__ bitmap, int words, unsigned magic, int hw, int c_out,
                                           long long items, uint32_t* __restrict__ counts,
                                           unsigned long long* __restrict__ total_out, uint32_t* __restrict__ mask,
                                           uint32_t need) {
  __shared__ unsigned long long sum;
  if (threadIdx.x == 0) sum = 0ull;
  __syncthreads();
  unsigned long long total = 0ull;                 // (the wavefront's)
  const long long all = items * 8, step = (long long)gridDim.x * blockDim.x;
  for (long long id = (long long)blockIdx.x * blockDim.x + threadIdx.x; id - (threadIdx.x & 63) < all; id += step) {
    const bool on = id < all;                      // (a wavefront stays together)
    const long long item = id >> 3, img = magic ? (long long)__umulhi((unsigned)item, magic) : item / words;
    const int w = (int)(item - img * words), sft = (int)(id & 7) * 4;
    const uint32_t* const src = bitmap + img * hw * words + w;
    uint32_t n = 0u;
    for (int px = 0; on && px < hw; px += 4) {
      uint32_t v[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = px + i < hw ? src[(long long)(px + i) * words] : 0u;
#pragma unroll
      for (int i = 0; i < 4; ++i) n += ((v[i] >> sft & 15u) * 0x00204081u) & 0x01010101u;
    }
    if (mask) {
      uint32_t keep = 0u;
#pragma unroll
      for (int e = 0; e < 4; ++e) keep |= (w * 32 + sft + e < c_out && (n >> (8 * e) & 255u) >= need ? 1u : 0u) << (sft + e);
#pragma unroll
      for (int s = 4; s >= 1; s >>= 1) keep |= (uint32_t)__shfl_xor((int)keep, s, 64);
      if (on && sft == 0) mask[item] = keep;
      continue;
    }
    uint32_t* const out = counts + img * c_out + w * 32 + sft;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (on && w * 32 + sft + e < c_out) out[e] = n >> (8 * e) & 255u;
    const uint32_t four = (n * 0x01010101u) >> 24;   // (bits past c_out are zero)
    total += sum32(four + (uint32_t)__shfl_xor((int)four, 32, 64));
  }
  if (mask) return;
  if ((threadIdx.x & 63) == 0 && total) atomicAdd(&sum, total);
  __syncthreads();
  if (threadIdx.x == 0 && sum) atomicAdd(total_out, sum);
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

constexpr int kSmallMap = 16;   // pixels per feature map up to which a thread counts by itself

// counts and total, or mask
hipError_t launch_count(const Params& p, const uint32_t* bitmap, uint32_t* counts, uint32_t* total, uint32_t* mask, uint32_t need,
                        hipStream_t s) {
  const long long items = (long long)p.n * p.words;
  if (items <= 0) return hipSuccess;
  const int hw = p.ho * p.wo;
  // exact for items below 2^32 / words
  const unsigned magic = p.words > 1 && items * p.words < (1ll << 32) ? (unsigned)(((1ull << 32) + (unsigned)p.words - 1) / (unsigned)p.words) : 0u;
  if (hw <= kSmallMap) {
    // a block to 256 threads until there are kMaxBlocks of them, then larger ones; twice as many where each still goes round
    const long long threads = items * 8;
    const int bs = threads <= 256ll * kMaxBlocks ? 256 : 1024;
    const long long blocks = (threads + bs - 1) / bs;
    hipLaunchKernelGGL(bitmap_counts_small_kernel, dim3((unsigned)(blocks < 2 * kMaxBlocks ? blocks : 2 * kMaxBlocks)), dim3(bs), 0, s,
                       bitmap, p.words, magic, hw, p.c_out, items, counts, (unsigned long long*)total, mask, need);
    return hipGetLastError();
  }
  // wavefronts per item: one for 256 pixels, at most sixteen; wavefronts per block: four, more where there would be more than
  // kMaxBlocks blocks (a block of four starts 0.3 us sooner than one of sixteen)
  if (items >= (1ll << 31)) return hipErrorInvalidValue;      // (more than 2^40 outputs, which create turns away)
  int wl = 0;
  while (wl < 4 && (256 << wl) < hw) ++wl;
  int nw = wl < 2 ? 4 : 1 << wl;
  while (nw < 16 && (items << wl) > (long long)nw * (kMaxBlocks / 2)) nw *= 2;
  const long long blocks = ((items << wl) + nw - 1) / nw;
  const int most = blocks > 4 * kMaxBlocks ? 2 * kMaxBlocks : kMaxBlocks;
  const dim3 grid((unsigned)(blocks < most ? blocks : most)), block(64 * nw);
  auto* kernel = hw <= 64 ? &bitmap_counts_kernel<1, false> : wl == 0 ? &bitmap_counts_kernel<4, false> : &bitmap_counts_kernel<4, true>;
  hipLaunchKernelGGL(kernel, grid, block, 0, s, bitmap, p.words, magic, hw, p.c_out, (unsigned)items, wl, counts, (unsigned long long*)total,
                     mask, need);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_bitmap_counts(const Params& p, const uint32_t* bitmap, hipStream_t s) {
  return launch_count(p, bitmap, p.counts, p.total, nullptr, 0u, s);
}

hipError_t launch_bitmap_chan_mask(const Params& p, const uint32_t* bitmap, uint32_t need, uint32_t* mask, hipStream_t s) {
  return launch_count(p, bitmap, nullptr, nullptr, mask, need, s);
}

hipError_t launch_counts_chan_mask(const Params& p, const uint32_t* counts, uint32_t need, uint32_t* mask, hipStream_t s) {
  const long long items = (long long)p.n * p.words;
  if (items <= 0) return hipSuccess;
  hipLaunchKernelGGL(counts_chan_mask_kernel, dim3((unsigned)((items + 255) / 256)), dim3(256), 0, s, counts, p.words, p.c_out,
                     items, need, mask);
  return hipGetLastError();
}

}  // namespace cg
