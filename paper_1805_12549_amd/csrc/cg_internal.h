// Internal declarations shared by the host API and the kernels of the
// channel-gated convolution library.  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <atomic>

#include "cg_conv.h"

namespace cg {

// Everything a kernel needs to know about one forward call; passed by value.
struct Params {
  int n, h, w, c_in, c_out, c_base, c_cond;
  int kh, kw, stride, pad, ho, wo;
  long long x_pixel_stride;
  long long m_total;       // n*ho*wo
  unsigned epilogue;
  int in_dtype, out_dtype;
  int two_sided;           // an upper gate threshold was given
  int gated;               // 0: dense layer, no gate, second affine pair applies
  int one_pair;            // float layers: the two scale/shift pairs are equal in every channel
  int fit32;               // int8 -> int8 layers: the requantisation fits 32 bits (tables 1, 5 and 6 are laid out for that)
  int rq_shift, rq_res_mult;
  int words;               // bitmap words per pixel = ceil(c_out/32)
  int groups;              // >= 1; > 1: channel grouping (Sec. 3.3), output group i has input group i as base
  int cpg;                 // output channels per group = c_out / groups
  int shuffle;             // y (and the residual) in shuffled channel order: channel j of group i at j*groups + i
  int gate_only;           // first pass of the channel-wise gate: base path and gate only; writes the bitmap,
                           // nothing else
  const uint32_t* chan_mask;  // second pass: [n][words] bits of the channels that keep their conditional
                              // path (Sec. 3.2 channel-wise gate), ANDed into the decisions; or NULL

  // per-output-channel tables, device, in `packed`
  const float* thr_f;      // lower threshold on the fp32 base sum (Sec. 3.2 merged gate)
  const float* thr_hi_f;   // upper threshold (+inf when one-sided)
  const int32_t* thr_i;    // integer threshold (int8 path)
  const float *sc0, *sh0, *sc1, *sh1;
  const int32_t *mult0, *mult1, *bias;

  // weights in caller layout [c_out][kh][kw][c], copied into `packed`
  const void* w_base;
  const void* w_cond;
  size_t table_stride;     // bytes between the per-channel tables of `packed`; thr_f is table 0
  uint32_t* gave_up;       // a word of host memory that a kernel sets when it gives up a wait (its results are then wrong)
  const void* zeros;       // at least 256 bytes of zeros (source of the padding in the LDS-direct loads)

  // call arguments
  const void* x;
  const void* residual;
  void* y;
  uint32_t* bitmap;
  uint32_t* counts;        // [n][c_out] fired counts, or NULL; counted from the bitmap after the layer kernel
  uint32_t* total;         // their 64-bit sum (two words), or NULL; counting adds to it
  int clear_total;         // the layer kernel zeroes the total
  int count_here;          // plain kernel: adds to counts and total itself (both cleared before), no bitmap needed
};

// Geometry of the large-tile matrix-core kernel (kernels_tile.hip): four wavefronts per workgroup,
// one workgroup per compute unit, a wavefront multiplies `fp` 32-pixel fragments by 64 channels.
// K is walked in stages of `cps` 16-byte channel chunks per pixel times all taps.
struct TilePlan {
  int ok;
  int elem_bytes, ch;      // bytes per element; channels per 16-byte chunk
  int taps;                // 9 (3x3) or 1 (1x1)
  int cps;                 // chunks per pixel per stage
  int fp;                  // 32-pixel fragments per wavefront: 4, 2 or 1
  int wn;                  // wavefronts across the channels: 1 (64-channel block) or 2 (128)
  int bn, n_cb;            // channels per block, number of blocks
  int flat, vw;            // flat: a 1x1 stride-1 layer walked as one image of rows of vw pixels
  int tr;                  // output rows per tile
  int hp;                  // h + 2*pad of the geometry walked (for n_max)
  int logp;                // log2 of the patch row pitch in pixel slots
  int pr;                  // patch rows, maximum over tiles
  int n16;                 // 16-byte positions of a stage's patch = pr * pitch * cps
  int xcd_cb;              // 1: blocks of one channel block share an XCD; 0: blocks of one tile do
  int grp_mode, gsp;       // channel grouping, as in RowsPlan
  int stages[2];           // stages of the base / conditional phase
  int wgs;                 // workgroups of a launch
  int nb;                  // stage buffers in LDS (the loads run nb - 1 stages ahead)
  size_t lds_bytes;        // LDS of the kernel instantiation
  size_t wpk_stage_bytes;  // bytes of one (channel block, stage) slab of prepacked weights
  size_t wpk_base_bytes, wpk_cond_bytes;
};

// the image geometry the kernel walks for one call (the layer's own, or the flat renumbering)
struct TileGeo {
  int n, h, w, ho, wo, stride, pad, hp;
  unsigned magic_hp, magic_ho, magic_wo;
  long long m_valid;       // output pixels
  long long in_valid;      // input pixels
  int xps;                 // bytes between input pixels
};

TilePlan tile_plan(const cg_conv_desc& d, int n_cu);
hipError_t launch_tile_pack(const TilePlan& plan, const Params& p, void* wpk_base, void* wpk_cond, hipStream_t s);
hipError_t launch_tile(const TilePlan& plan, const Params& p, const void* wpk_base, const void* wpk_cond,
                       hipStream_t s);
// one translation unit per (dtype, kernel size): the instantiations of the tile kernel
hipError_t launch_tile_bf16_k3(const TilePlan& g, const TileGeo& q, const Params& p, const void* w0, const void* w1,
                               hipStream_t s);
hipError_t launch_tile_bf16_k1(const TilePlan& g, const TileGeo& q, const Params& p, const void* w0, const void* w1,
                               hipStream_t s);
hipError_t launch_tile_i8_k3(const TilePlan& g, const TileGeo& q, const Params& p, const void* w0, const void* w1,
                             hipStream_t s);
hipError_t launch_tile_i8_k1(const TilePlan& g, const TileGeo& q, const Params& p, const void* w0, const void* w1,
                             hipStream_t s);

// Geometry of the small-tile matrix-core kernel (kernels_direct.hip): 16*pf output pixels x 16*nh
// channels per tile, operands straight from global memory.
struct DirectPlan {
  int ok;
  int elem_bytes, ch;      // bytes per element; channels per 16-byte chunk
  int taps;                // 9 or 1
  int pf, nh;              // 16-pixel fragments and 16-channel halves of the packed groups per tile
  int split;               // wavefronts of a workgroup that share a tile's K; 1: a wavefront walks all of it
  int nwb;                 // of which walk the base path
  int n_cblk;              // tiles across the channels
  int px_wgs;              // workgroups across the pixels
  unsigned x_bytes;        // size of x
  // Channel chunks per tap and phase.  The base phase starts at the first chunk of the 64-channel block's
  // first group and walks chunks[0] of them; the conditional phase walks all chunks but the gap_len ones
  // from there on.
  int chunks[2], total_chunks, gap_len;
  int mixed;               // channel grouping: zero weights keep channels apart that a block walks together
  int straddle;            // no grouping: so do they in the chunk in which the base group ends
  int uniform;             // every K step lies inside one tap and on one side of the base group
  int ksteps[2];           // K steps (four chunks) per phase
  int n_grp;               // 32-channel groups of the packed weights
  size_t wpk_bytes[2];
  double cost, est;        // estimated time, in clocks: what plans were compared by; what the kernel is chosen by
};

DirectPlan direct_plan(const cg_conv_desc& d, int n, int n_cu);
hipError_t launch_direct_pack(const DirectPlan& plan, const Params& p, void* wpk_base, void* wpk_cond, hipStream_t s);
// beside: a 1x1 convolution that the launch does too (takes_beside), or NULL
struct PointArgs;
bool takes_beside(const DirectPlan& plan, const Params& p);
hipError_t launch_direct(const DirectPlan& plan, const Params& p, const void* wpk_base, const void* wpk_cond, hipStream_t s, const PointArgs* beside = nullptr);

// Geometry of the row-tiled matrix-core kernel (kernels_rows.hip): persistent workgroups of 64 output channels
// that walk runs of output rows in tiles of at most 256 pixels; K in stages of `cps` 16-byte channel chunks
// per pixel times nine taps; the LDS patch of a stage holds 16*cps bytes per pixel slot,
// slot = patch_row * 2^logp + (wi + pad).
struct RowsPlan {
  int ok;
  int elem_bytes, ch;      // bytes per element; channels per 16-byte chunk
  int taps;                // 9, or 1 for 1x1 layers: a row is then a pixel, and a patch the tile's pixels
  int cps;                 // chunks per pixel per stage: 4 or 2 (1x1: 8)
  int stages[2];           // stages of the base / conditional phase
  // Channel grouping.  0: none.  1: a 64-channel block lies inside one output group; its base
  // channels start at group*c_base and the conditional phase skips them.  2: a block covers
  // `gsp` whole groups; its base phase walks the gsp*c_base base channels of all of them and its
  // conditional phase all c_in channels, the packed weights holding zeros where a channel is not on
  // that path for that output channel.
  int grp_mode, gsp;
  int n_cb;                // c_out / 64
  int n_slots;             // workgroups per channel block: the batch's rows are split evenly over them
  int xcd_cb;              // 1: workgroups of one channel block share an XCD (needs n_cb % 8 == 0)
  int hp;                  // h + 2*pad
  int tr;                  // output rows per tile
  int logp, pr, n_pl;      // log2 of the patch row pitch; patch rows, maximum over tiles; 1 KB loads per patch
  int resident, nb;        // 1: all weights stay in LDS; stage buffers
  int psz, pstr;           // bytes per patch; bytes between stage buffers
  int pf;                  // fragments per wavefront: 1 or 2
  int fwl, nfc;            // fragment of a wavefront: 2^fwl columns (-1: 32 pixels in a row), fragments per row group
  int wres, shuf, shuf_bytes, tabs, lds_bytes;   // LDS offsets of resident weights (-1: none), shuffled rows, tables
  size_t wpk_base_bytes, wpk_cond_bytes;
  double cost, est;        // estimated time, in clocks: what plans were compared by; what the kernel is chosen by
};

// cps: 0 = pick, 4 or 2 = that (for a handle whose weights are packed); max_pf: the most fragments per wavefront
RowsPlan rows_plan(const cg_conv_desc& d, int n_cu, int cps, int max_pf);
// the same kernel on 1x1 layers of stride 1
RowsPlan point_plan(const cg_conv_desc& d, int n_cu);
hipError_t launch_rows_pack(const RowsPlan& plan, const Params& p, void* wpk_base, void* wpk_cond, hipStream_t s);
hipError_t launch_rows(const RowsPlan& plan, const Params& p, const void* wpk_base, const void* wpk_cond,
                         hipStream_t s);
// per-(image, channel) fired counts and their total (into p.counts / p.total) from a decision bitmap
hipError_t launch_bitmap_counts(const Params& p, const uint32_t* bitmap, hipStream_t s);
// channel-wise gate: mask[img][w] bit b = (fired count of channel 32*w + b in image img, from the bitmap) >= need
hipError_t launch_bitmap_chan_mask(const Params& p, const uint32_t* bitmap, uint32_t need, uint32_t* mask,
                                   hipStream_t s);
// the same from [n][c_out] fired counts
hipError_t launch_counts_chan_mask(const Params& p, const uint32_t* counts, uint32_t need, uint32_t* mask, hipStream_t s);

// compute units of the current device (256 where no device answers: the plan is then the MI355X one)
int cu_count();
// Lets `kernel` use up to `bytes` of LDS on the current device, which has to be asked for beyond the default of a launch,
// once per kernel and device; `done` is the kernel's own record of the devices that were asked.
hipError_t allow_lds(const void* kernel, int bytes, std::atomic<uint64_t>& done);

// launchers (return hipError_t from the last launch)
hipError_t launch_naive(const Params& p, hipStream_t s);
hipError_t launch_zero_u32(uint32_t* ptr, size_t words, hipStream_t s);

}  // namespace cg
