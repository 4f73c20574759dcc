// Row-tiled matrix-core kernel of the gated convolution (bf16 and int8 MFMA, 32x32 blocks): persistent
// workgroups whose wavefronts run free of each other, loads issued by wavefronts of their own.
//
// A workgroup of twelve wavefronts is alone on its compute unit and owns one block of 64 output
// channels and a run of consecutive output rows of the batch (rows numbered R = img*Ho + ho), which it
// walks in tiles of up to 256 pixels (whole rows, possibly straddling images).  K is walked in stages
// of CPS 16-byte channel chunks x nine taps; a stage's input patch and its weights sit in one of NB
// LDS buffers.  The sequence of stages runs through all tiles of the workgroup without a break.
//
//   loaders     wavefronts 8..11 issue every LDS-direct load and publish what has landed in LDS counters; the
//               eight multiplying wavefronts publish what they are done with.  There is no barrier: a wavefront
//               that has nothing to multiply in a stage (no gate of its pixels fired, no pixels in the tile's
//               ragged end) passes it by, and one that writes its output does not hold up the others, so
//               one wavefront's gate and output instructions run under another's matrix instructions.
//               Where all stages' weights fit into LDS together (64 channels) they stay there and only the
//               patches stream.
//   base path   implicit GEMM over taps x base channels; a wavefront multiplies a fragment of 32 pixels of the
//               tile (FH rows x 32/FH columns, or 32 in a row) by the 64 channels.  The product is taken
//               transposed (weights are the row operand, their rows permuted), which leaves a lane with 16
//               consecutive channels of one pixel per accumulator: gate and output work on registers.
//   gate        accumulators against the per-channel thresholds (merged gate, Sec. 3.2 of the
//               channel-gating paper); decision words leave straight from registers.
//   cond. path  a wavefront with a fired gate adds the conditional channels on top of a copy of its base sums and
//               picks per channel (Eq. 1).  The granule of skipping is the wavefront's fragment; a compact shape
//               of it (4x8 pixels) is what keeps it close to the fired area: with clustered maps at a firing rate
//               of 0.3, 0.64 of the 4x8 fragments of 56x56 maps hold a fired pixel, 0.90 of runs of 32.
//               (Listing the fired pixels of a tile and dealing them out 32 at a time issues 0.42, but
//               needs every wavefront at the gate at once, an exchange of sums and a second output pass; it measured
//               1.3 to 2 times slower than this form at 64 channels and no faster at 256 and 512.)
//   output      scale/shift by decision, residual, ReLU, convert (Eq. 1), stored from registers.
//
// PF = 2 (bf16 layers with many channels and pixels): a wavefront takes two fragments and reads a stage's weights from LDS once for
// both, which is what bounds the loop there (one fragment: 3 KB of LDS reads for two products, i.e. 192 of 128 clocks).
// Its registers do not hold two sets of sums per fragment; the outputs for an unfired gate are written first and
// corrected where a gate fired.
//
// TAPS = 1 (1x1 layers of stride 1): a row is a pixel, a patch the tile's pixels (no halo), a stage up to eight chunks of one
// tap.  1024 channels at 14x14, 64 images: bf16 40 us, int8 28; 99 and 105 on the large-tile kernel.
//
// What bounds the kernel: at 64 and 128 channels the instructions of gate and output (a third of a wavefront's time each
// side of the products), at 256 and 512 the LDS reads and, for few images, the start: the first stage of all workgroups
// (some 40 KB each, 10 MB for the chip) lands 2.7 us after the first instruction.  Arguments asked for at once and a column
// that is formed once per wavefront have the loads out after 1.1 us instead of 1.9: 64 channels at 56x56, 64 images 22.9 -> 22.3
// us, 128 to 256 at 28x28 stride 2 16.1 -> 15.6, int8 128 at 28x28, 32 images 10.4 -> 10.1.  The matrix cores are busy for 15 to 26 % of a layer at 64 images.
// Outputs: addresses of 32 bits in buffer accesses (the range check drops lanes without a pixel), one bit-field instruction to a decision, scale and shift
// read ahead, one question instead of four for whether there are any: 64 channels at 56x56, 256 images 94.4 -> 86.5 us, 128 at 28x28 74.1 -> 68.9,
// 256 at 14x14 61.5 -> 58.7, int8 128 at 28x28, 32 images 9.8 -> 9.4, 1x1 of 192 to 128 channels 12.3 -> 11.6.
// Layers with a residual have kernels of their own (kAdded): it is on its way while the tile's stages are multiplied, and the others have no branch
// for it at every piece of an output.  With: int8 384 to 512 at 40x40 stride 2, 42 images 54.8 -> 53.0, 1x1 of 192 to 128 channels 11.7 -> 11.1; without:
// 64 at 56x56, 64 images 22.3 -> 21.5, int8 128 at 28x28, 32 images 9.9 -> 9.4, 64 at 16x16, 216 images 8.9 -> 8.4.  Measured in a graph with
// rotated buffers, clustered maps at a firing rate of 0.3, this form against an earlier one (barrier-coupled workgroups with the pixels listed anew for
// the conditional path), before and after, us:
//   bf16, scale/shift, residual and ReLU
//         64 channels at 56x56, 64 images 36.4 -> 28.9, 256: 116 -> 95;  128 at 28x28, 64: 25.1 -> 25.2, 128: 45.4 -> 41.3,
//         256: 74.4 -> 70.6;  256 at 14x14, 64: 24.2 -> 20.5, 128: 33.5 -> 34.8, 256: 56.4 -> 60.5;  512 at 7x7, 64: 29.6 ->
//         23.6, 256: 74.0 -> 61.3;  128>256 at 28x28 stride 2, 64: 22.8 -> 19.0, 256: 83 -> 56
//   int8  128 at 28x28, 32 images 17.6 -> 11.2, 256: 71 -> 48;  512 at 7x7, 256: 53 -> 35
// Where it is not faster, skipping whole fragments is what it loses against single pixels: 256 at 14x14, 256 images, by firing
// rate 0.05: 47.6 -> 49.9, 0.1: 49.6 -> 50.4, 0.3: 55.7 -> 56.6, 0.6: 62.4 -> 60.9.
//
// kPaired (tiles of at most four fragments, which would leave four of the multiplying wavefronts idle): two wavefronts, on the same
// SIMD, take a fragment, each with 32 of the block's channels, and one's LDS reads, gate and output run under the other's
// products.  Alone on its SIMD a wavefront took half as long again as its products.  us before and after: 256 channels at 8x8, 128 images 15.7 ->
// 15.1, 64 at 56x56, 8 images 8.1 -> 7.6, 128 at 16x16, 32 images 9.1 -> 8.6, int8 256 at 14x14, 32 images 10.5 -> 9.8, 512 at
// 7x7, 64 images 15.3 -> 14.6; 256 at 14x14 by the images, 16 12.0 -> 11.4, 24 12.4 -> 12.2, slower 28 to 40 (32 13.1 -> 13.3, 40 13.7 -> 14.1).  A stage still takes 1100 clocks at 256 channels where its
// products take 576, its loads 710 (a 1 KB load is 20 clocks of the memory path, 32 where it is made of pieces of 32 bytes)
// and its LDS accesses 800.  (The other way to share a fragment, every second K step for all 64 channels, a quarter fewer LDS reads, and sums that
// meet in LDS: 1.1 to 1.6 us slower throughout.  The loads stay, and both meetings and two more stage loops are met cold.)
//
// A patch is stored [pixel slot][CPS chunk positions]; chunk q of slot s sits at position q ^ f(s),
// f(s) = (s >> 2) & 3 (CPS = 4) or (s >> 3) & 1 (CPS = 2), which spreads the operand reads over the LDS
// banks.  (A 16-byte read is served in four groups of lanes, {0-3, 12-15, 20-27}, the rest of the first 32, and the same
// again 32 lanes on.)  Where a group covers several patch rows, i.e. on narrow maps, the lowest bit of the row takes the place of f's highest
// bit: 8x8 maps 1 pass to a group instead of 2, 7x7 2 instead of 3, fragments of 8 columns 1 to 1.5 instead of 2.  That costs an
// instruction in every third read and pays only where two wavefronts share a fragment (256 channels at 8x8 3 %; with one each
// 128 channels at 28x28 lost 1 %).  Slot = patch_row * P + c with P a power of two >= max(16, W + pad) and c = wi + pad;
// positions outside the image are out-of-range buffer loads, which write zeros.
//
// The vector-memory path serves a cache line every two clocks, whatever part of it is asked for (measured: 17, 35
// and 65 bytes a clock in pieces of 32, 64 and 128+), which is why outputs are transposed between lanes before
// they are stored and why stages of four chunks are preferred where the channel counts allow.
#include <algorithm>
#include <type_traits>
#include <utility>

#include "cg_mfma_common.h"

namespace cg {

namespace {

constexpr int kBn = 64;                      // output channels per workgroup
constexpr int kCw = 8;                       // wavefronts that multiply
constexpr int kLw = 4;                       // wavefronts that load
constexpr int kNt = 64 * (kCw + kLw);
constexpr int kTabs = 8;                     // per-channel tables of `packed`
constexpr int kTabBytes = kTabs * 256 + 64;  // ... of the block's 64 channels; progress counters (12) and gave_up
constexpr int kShufRow = 144;                // bytes of a pixel's row in the shuffled store's LDS tile (128 + skew)
constexpr int kLds = 160 * 1024;
constexpr int kMaxPatchLoads = 12;           // 1 KB load instructions per loading wavefront and patch

typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(16))) int i32x16;

// d = 2*d + (v >= t) for v3, v2, v1, v0 in turn: int8 as one statement (between two the compiler puts a wait), bf16 as four
// (1x1 layers of 192 channels 11.5 us against 11.8: the table's next entries arrive in between).
#define CG_SHIFT_IN1(cmp, v, t) cmp " vcc, " v ", " t "\n\tv_addc_co_u32 %0, vcc, %0, %0, vcc\n\t"
#define CG_SHIFT_IN4_APART(cmp)                                                             \
  asm(CG_SHIFT_IN1(cmp, "%1", "%2") : "+v"(d) : "v"(v3), "v"(t[3]) : "vcc"); \
  asm(CG_SHIFT_IN1(cmp, "%1", "%2") : "+v"(d) : "v"(v2), "v"(t[2]) : "vcc"); \
  asm(CG_SHIFT_IN1(cmp, "%1", "%2") : "+v"(d) : "v"(v1), "v"(t[1]) : "vcc"); \
  asm(CG_SHIFT_IN1(cmp, "%1", "%2") : "+v"(d) : "v"(v0), "v"(t[0]) : "vcc")
#define CG_SHIFT_IN4(cmp)                                                                                                  \
  asm(CG_SHIFT_IN1(cmp, "%4", "%8") CG_SHIFT_IN1(cmp, "%3", "%7") CG_SHIFT_IN1(cmp, "%2", "%6") CG_SHIFT_IN1(cmp, "%1", "%5") \
      : "+v"(d) : "v"(v0), "v"(v1), "v"(v2), "v"(v3), "v"(t[0]), "v"(t[1]), "v"(t[2]), "v"(t[3]) : "vcc")

// 32x32 output block; lane l supplies row / column l%32 and the 16-byte K chunk l/32 of either
// operand; it receives column l%32, rows 8*(i/4) + 4*(l/32) + i%4 in register i.
struct Bf16Rows {
  using Base = Bf16Traits;
  using acc16 = f32x16;
  using acc_t = float;
  static __device__ __forceinline__ acc16 mfma(i32x4 rows, i32x4 cols, acc16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, rows), __builtin_bit_cast(bf16x8, cols),
                                                   c, 0, 0, 0);
  }
  static __device__ __forceinline__ void shift_in4(unsigned& d, float v0, float v1, float v2, float v3, i32x4 t) {
    CG_SHIFT_IN4_APART("v_cmp_ge_f32");
  }
  // (v <= t)
  static __device__ __forceinline__ void shift_in4_le(unsigned& d, float v0, float v1, float v2, float v3, i32x4 t) {
    CG_SHIFT_IN4_APART("v_cmp_le_f32");
  }
};

struct I8Rows {
  using Base = I8Traits;
  using acc16 = i32x16;
  using acc_t = int32_t;
  static __device__ __forceinline__ acc16 mfma(i32x4 rows, i32x4 cols, acc16 c) {
    return __builtin_amdgcn_mfma_i32_32x32x32_i8(rows, cols, c, 0, 0, 0);
  }
  static __device__ __forceinline__ void shift_in4(unsigned& d, int v0, int v1, int v2, int v3, i32x4 t) { CG_SHIFT_IN4("v_cmp_ge_i32"); }
};
#undef CG_SHIFT_IN4
#undef CG_SHIFT_IN4_APART
#undef CG_SHIFT_IN1

__device__ __forceinline__ int as_bits(float f) { return __float_as_int(f); }
__device__ __forceinline__ int as_bits(int v) { return v; }
__device__ __forceinline__ void from_bits(int b, float& f) { f = __int_as_float(b); }
__device__ __forceinline__ void from_bits(int b, int& v) { v = b; }

// exact x / d for x, d < 65536 with magic = ceil(2^32 / d); magic 0 stands for d = 1 (2^32 does not fit)
__device__ __forceinline__ int div16(int x, unsigned magic) { return magic ? (int)__umulhi((unsigned)x, magic) : x; }

// 16-byte LDS read with a compile-time byte offset; the caller waits (lgkmcnt) before using the value
template <int OFS>
__device__ __forceinline__ i32x4 lds_read16(unsigned addr) {
  static_assert(OFS >= 0 && OFS < 65536, "16-bit offset field");
  i32x4 v;
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFS) : "memory");
  return v;
}

// s_waitcnt vmcnt(n) for any LO <= n: the largest multiple of two below HI that is not above it (fewer in flight is safe)
#define CG_VMCNT(n) (0x0F70 | ((n) & 15) | (((n) >> 4) << 14))
template <int LO, int HI>
__device__ __forceinline__ void wait_vm(int n) {
  if constexpr (HI - LO <= 2) {
    __builtin_amdgcn_s_waitcnt(CG_VMCNT(LO));
  } else {
    constexpr int MID = LO + (HI - LO) / 4 * 2;
    if (n >= MID)
      wait_vm<MID, HI>(n);
    else
      wait_vm<LO, MID>(n);
  }
}

// the larger one (fmaxf of values that are no signalling NaNs, without the instruction that would quiet those)
__device__ __forceinline__ float max_of(float a, float b) {
  float r;
  asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
// two floats as bf16 (round to nearest even), a in the low half
__device__ __forceinline__ int bf16_pair(float a, float b) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(int, __builtin_convertvector(f32x2{a, b}, bf16x2));
}

// all ones where bit I + e of d is set, e = 0 .. 3 (as expressions they become a comparison for every use: three instructions and a wait
// instead of one; one to an asm statement, each is waited for)
template <int I>
__device__ __forceinline__ void ones_if4(unsigned d, int (&m)[4]) {
  asm("v_bfe_i32 %0, %4, %5, 1\n\tv_bfe_i32 %1, %4, %6, 1\n\tv_bfe_i32 %2, %4, %7, 1\n\tv_bfe_i32 %3, %4, %8, 1"
      : "=&v"(m[0]), "=&v"(m[1]), "=&v"(m[2]), "=v"(m[3])
      : "v"(d), "n"(I), "n"(I + 1), "n"(I + 2), "n"(I + 3));
}
__device__ __forceinline__ int select_bits(int m, int a, int b) { return (a & m) | (b & ~m); }

__device__ __forceinline__ int med3(int v, int lo, int hi) {
  int r;
  asm("v_med3_i32 %0, %1, %2, %3" : "=v"(r) : "v"(v), "v"(lo), "v"(hi));
  return r;
}

// f(slot), and the byte offset of chunk position (h ^ f(slot)) of pixel slot `slot`; `bit`: the slot's bit that is f's highest
template <int CPS>
__device__ __forceinline__ int slot_perm(int slot, int bit) {
  if constexpr (CPS == 8) return slot & 7;
  if constexpr (CPS == 4) return ((slot >> 2) & 1) | (((slot >> bit) & 1) << 1);
  return (slot >> bit) & 1;
}
template <int CPS>
__device__ __forceinline__ int slot_addr(int slot, int h, int bit) {
  return slot * (16 * CPS) + (h ^ slot_perm<CPS>(slot, bit)) * 16;
}

template <int... I, typename F>
__device__ __forceinline__ void static_for_impl(std::integer_sequence<int, I...>, F&& f) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(std::make_integer_sequence<int, N>{}, static_cast<F&&>(f));
}

__device__ __forceinline__ void wait_lds() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xC07F);        // lgkmcnt(0)
  asm volatile("" ::: "memory");
}

// barrier without the drain of every memory operation that __syncthreads() implies
__device__ __forceinline__ void bare_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Waits until each of the N progress counters at LDS address `addr` is at least `need`; `have` caches their
// minimum.  Every counter is advanced by a wavefront that never waits for this one's next step; the bound on the
// polls (near a second) only turns a mistake into a wrong result instead of a hang.  `have` is then kGaveUp, the wavefront
// waits no more, and at its end it sets a word of host memory after which every call of the library fails.
constexpr int kPolls = 1 << 22, kGaveUp = 0x7fffffff;
template <int N>
__device__ __forceinline__ void wait_counters(unsigned addr, int lane, int need, int& have) {
  if (have >= need) return;
  for (int spin = 0; spin < kPolls; ++spin) {
    int v;
    asm volatile("ds_read_b32 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(v) : "v"(addr + (lane < N ? lane : 0) * 4) : "memory");
    have = __builtin_amdgcn_readlane(v, 0);
#pragma unroll
    for (int i = 1; i < N; ++i) {
      const int w = __builtin_amdgcn_readlane(v, i);
      have = w < have ? w : have;
    }
    have = __builtin_amdgcn_readfirstlane(have);
    if (have >= need) return;
    __builtin_amdgcn_s_sleep(1);
  }
  have = kGaveUp;
}
// what is the same for the whole grid; the kernel reads each group with a few scalar loads, issued together
struct RowsArgs {
  // every wavefront
  unsigned flags;                            // kGated ...
  unsigned magic_ncb, magic_ho;
  int n_cb, n_slots, xcd_cb, per_xcd;
  int full, rows_per, rows_more;             // whole rounds of tiles; rows per workgroup after them (the first rows_more: one more)
  int tr, logp, bit;                         // rows per tile, patch pitch, chunk permutation
  int s0, s, nb, pstr, psz, wres, tabs;      // stages; buffers and LDS offsets (wres < 0: weights are in the ring)
  int ho, hp, stride, tab_stride;
  uint32_t* clear;                           // two words that the grid clears, or NULL
  // loading wavefronts
  const char* x;
  const char *w0, *w1;
  const char* tab;
  unsigned magic_hp, x_bytes;
  int n, h, w, pad, xps, n_pl;               // 1 KB patch loads
  int base_chn, gap_chn, grp_mode, grp_step; // channel walk
  // multiplying wavefronts
  int fwl, nfc;                              // log2 columns of a fragment and fragments per row group; fwl < 0: 32 in a row
  unsigned magic_wo, magic_nfc;
  char* y;
  const char* residual;
  uint32_t* bitmap;
  const uint32_t* chan_mask;
  int wo, words, c_out, rq_shift, rq_res_mult, shuf, cpg, groups;
  int spg;                                   // stages per channel group where a block covers several, else 0
  uint32_t* gave_up;                         // host memory: set where a wait came to its bound
};
enum : unsigned {
  kGated = 1u, kGateOnly = 2u, kTwoSided = 4u, kAffine = 8u, kRelu = 16u, kResidual = 32u,
  kFast = 64u,                               // 2-byte (int8 layers: 1-byte) outputs in natural channel order (or kShuf2), within 32-bit offsets (near_outputs)
  kShuf2 = 128u,                             // 2-byte outputs in shuffled channel order
  kOnePair = 256u,                           // the two scale/shift pairs are the same
  kFit32 = 512u,                             // int8: the requantisation fits 32 bits
  kPairs = 1024u,                            // two wavefronts to a fragment
  kTurns = 4096u,                            // 1x1: loading wavefronts take whole stages in turn (kInTurn)
  kFourBytes = 2048u,                        // float (int8 layers: 32-bit) outputs in natural channel order, within 32-bit offsets
};

constexpr int kParamsAt = (sizeof(RowsArgs) + alignof(Params) - 1) / alignof(Params) * alignof(Params);   // of the kernel's arguments

// What a launch can do beside the common part; what it cannot is not in its code, whose registers and spilled scalars every
// wavefront pays for (all in one, the natural order cost 160 registers instead of 128 and 1 to 5 % of the time).
enum RowsOut {
  kNatural,                                  // fast outputs (kFast) in natural channel order
  kPaired,                                   // the same, tiles of at most four fragments: two wavefronts to one, 32 channels each
  kHalves,                                   // the same, blocks that cover several channel groups
  kShuffled,                                 // fast outputs in shuffled order
  kAnyOut,                                   // the rest, one lane's pixel at a time: shuffled orders without LDS for them, int8 outputs of shifts below two,
                                             // more channels than 32-bit offsets reach over (near_outputs)
  kWide,                                     // float and 32-bit outputs in natural order
  kAdded, kPairedAdded,                      // kNatural and kPaired of layers with a residual, which is read before a tile's stages
  kInTurn = 8,                               // beside one of these, 1x1 layers: a loading wavefront takes whole stages
};

template <typename Tr, int CPS, int PF, int TAPS, int FORM>
__global__ __launch_bounds__(kNt) void gated_conv_rows_kernel(RowsArgs a, Params) {
  constexpr int OUT = FORM & ~kInTurn;
  using acc16 = typename Tr::acc16;
  using acc_t = typename Tr::acc_t;
  using Base = typename Tr::Base;
  constexpr int KS = TAPS * CPS / 2;             // K steps per stage
  constexpr int PAIRS = CPS / 2;
  constexpr int WB = KS * 2048;                // bytes of a stage's weights
  constexpr int NWL = WB / 1024 / kLw;         // weight load instructions per loading wavefront (CPS = 2: one more for some)
  constexpr int SB = 16 * CPS;                 // bytes per pixel slot
  extern __shared__ __align__(1024) char lds[];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lj = lane & 31, lh = lane >> 5;
  // fragments of 32 channels that a wavefront multiplies, and the first channel of them in the block
  constexpr bool PAIR = OUT == kPaired || OUT == kPairedAdded;
  constexpr int kF = PAIR ? 1 : 2;
  // a residual: asked for (kHalves, kAnyOut, kWide), none, or one that is read before the tile's stages (PF = 2: no registers for it)
  constexpr bool kAsk = OUT == kHalves || OUT == kAnyOut || OUT == kWide, kAhead = PF == 1 && (OUT == kAdded || OUT == kPairedAdded);
  const bool added = kAsk ? (a.flags & kResidual) != 0 : OUT == kAdded || OUT == kPairedAdded;
  const int ch0 = PAIR && wave < kCw ? (wave >> 2) * 32 : 0;
  // All arguments in one go: each further wait for some of them is 500 clocks of a start that nothing overlaps.
  asm volatile("" ::"s"(a.flags), "s"(a.magic_ncb), "s"(a.magic_ho), "s"(a.n_cb), "s"(a.n_slots), "s"(a.xcd_cb), "s"(a.per_xcd),
               "s"(a.full), "s"(a.rows_per), "s"(a.rows_more), "s"(a.tr), "s"(a.logp), "s"(a.bit), "s"(a.s0), "s"(a.s), "s"(a.nb), "s"(a.pstr),
               "s"(a.psz), "s"(a.wres), "s"(a.tabs), "s"(a.ho), "s"(a.hp), "s"(a.stride), "s"(a.tab_stride), "s"(a.clear), "s"(a.x),
               "s"(a.w0), "s"(a.w1), "s"(a.tab), "s"(a.magic_hp), "s"(a.x_bytes), "s"(a.n), "s"(a.h), "s"(a.w), "s"(a.pad), "s"(a.xps),
               "s"(a.n_pl), "s"(a.base_chn), "s"(a.gap_chn), "s"(a.grp_mode), "s"(a.grp_step), "s"(a.fwl), "s"(a.nfc), "s"(a.magic_wo),
               "s"(a.magic_nfc), "s"(a.y), "s"(a.residual), "s"(a.bitmap), "s"(a.wo), "s"(a.gave_up));

  // Block id mod 8 is the XCD.  Normally an XCD takes a contiguous run of rows with all channel blocks, so that a
  // row is fetched into one L2 once; xcd_cb: the workgroups of a channel block sit on one XCD instead, so that each
  // L2 holds an eighth of the weights (layers whose weights outweigh their input).
  int slot, cbk;
  {
    const int xcd = blockIdx.x & 7, j = blockIdx.x >> 3;
    if (a.xcd_cb) {
      const int ncb8 = a.n_cb >> 3;
      slot = j / ncb8;
      cbk = (j - slot * ncb8) * 8 + xcd;
    } else {
      const int rank = xcd * a.per_xcd + j;
      slot = div16(rank, a.magic_ncb);
      cbk = rank - slot * a.n_cb;
    }
  }
  if (slot >= a.n_slots) return;
  if (a.clear && blockIdx.x == 0 && tid < 2) a.clear[tid] = 0u;
  // The workgroup's tiles: number slot, slot + n_slots, ... of the batch's tiles of tr rows (neighbours in time on an
  // XCD are neighbours in the batch; one workgroup's tiles come from different images, whose shares of fired
  // pixels differ), then an even share of the rows that do not make a whole round.
  const int tail_a = a.full * a.n_slots * a.tr + slot * a.rows_per + (slot < a.rows_more ? slot : a.rows_more);
  const int tail_rows = a.rows_per + (slot < a.rows_more ? 1 : 0);
  const int tiles = a.full + (tail_rows > 0 ? 1 : 0);
  auto tile_row = [&](int t) __attribute__((always_inline)) { return t < a.full ? (t * a.n_slots + slot) * a.tr : tail_a; };
  const bool gated = (a.flags & kGated) != 0, gate_only = (a.flags & kGateOnly) != 0;
  const unsigned lds0 = (unsigned)(uintptr_t)lds;
  // progress counters: stages landed per loading wavefront, stages done with per multiplying wavefront
  const unsigned landed = lds0 + a.tabs + kTabs * 256, done = landed + 4 * kLw;
  auto publish = [&](unsigned addr, int value) __attribute__((always_inline)) {
    if (lane == 0) asm volatile("ds_write_b32 %0, %1" ::"v"(addr), "v"(value) : "memory");
  };
  if (tid < kLw + kCw) *(int*)(lds + a.tabs + kTabs * 256 + tid * 4) = 0;

  auto mark_if_gave_up = [&](int have) __attribute__((always_inline)) {
    if (have != kGaveUp) return;
    uint32_t* const word = *(uint32_t* const*)(lds + a.tabs + kTabs * 256 + 48);
    if (lane == 0) __hip_atomic_store(word, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  };

  if (wave >= kCw) {
    // ================================ loading wavefronts ============================================
    // They share their SIMDs with the multiplying wavefronts and every instruction between two loads counts: buffer
    // loads with a scalar offset (no address arithmetic, padding by the range check), positions formed once per tile.
    __builtin_amdgcn_s_setprio(3);
    const int lw = wave - kCw;
    const int V = tiles * a.s;
    auto rsrc = [](const void* ptr, unsigned bytes) __attribute__((always_inline)) {
      const unsigned long long q = (unsigned long long)ptr;
      return i32x4{(int)q, (int)(q >> 32) & 0xffff, (int)bytes, 0x00027000};
    };
    const i32x4 xr = rsrc(a.x, a.x_bytes);
    const i32x4 wr0 = rsrc(a.w0 + (size_t)cbk * a.s0 * WB, a.s0 * WB);
    const i32x4 wr1 = rsrc(a.w1 + (size_t)cbk * (a.s - a.s0) * WB, (a.s - a.s0) * WB);
    auto dma = [&](i32x4 r, int voff, int soff, unsigned dst) __attribute__((always_inline)) {
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(dst), "v"(voff), "s"(r), "s"(soff) : "memory");
    };
    // the block's tables, four to a load; they land before its first stage does
    if (lw == 0) {
#pragma unroll
      for (int k = 0; k < kTabs / 4; ++k)
        dma(rsrc(a.tab, kTabs * a.tab_stride), (4 * k + (lane >> 4)) * a.tab_stride + (lane & 15) * 16, cbk * kBn * 4,
            lds0 + a.tabs + k * 1024);
    }
    // byte offset of the channel of x at which stage s starts: the base phase starts at this block's first base channel;
    // the conditional phase walks the channels in order and jumps over the base channels (without grouping these are
    // the first c_base; with grouping, Sec. 3.3, those of the block's own group, or none when the block covers
    // several groups and the packed weights carry zeros instead).
    const int b0 = a.grp_mode ? (cbk * kBn / a.grp_step) * a.base_chn : 0;
    // A position of the patch (16 bytes of a pixel) is load lw + 4k, lane `lane`.  From one load to the next of a wavefront it
    // is kStep slots on, whole periods of the chunks' permutation, and whole rows where the pitch is not above that: the chunk
    // and the column are then the same in all loads.  (Positions behind the patch's last row read some row of x or zeros.)  kOut: past the end of any x (the plan keeps x below 2 GiB).
    constexpr int kOut = (int)0x80000000, kStep = kLw * 64 / CPS;
    const int sl0 = lw * (64 / CPS) + lane / CPS;
    const int chunk = ((lane % CPS) ^ slot_perm<CPS>(sl0, a.bit)) * 16;
    const int np = (a.n_pl - lw + kLw - 1) / kLw;            // patch loads of this wavefront
    const int rowx = a.w * a.xps;            // bytes per image row
    auto column = [&](int sl) __attribute__((always_inline)) {
      const int wi = (sl & ((1 << a.logp) - 1)) - a.pad;
      return (unsigned)wi < (unsigned)a.w ? wi * a.xps + chunk : kOut;
    };
    const bool one_col = TAPS == 9 && (kStep >> a.logp) != 0;
    const int col0 = TAPS == 9 ? column(sl0) : sl0 * a.xps + chunk;
    int voff[kMaxPatchLoads];
    int R0 = 0, here = 0, rho0 = 0;          // of the tile: first row, rows, stacked padded input row of patch row 0
    auto tile_setup = [&](int t) __attribute__((always_inline)) {
      R0 = tile_row(t);
      here = t < a.full ? a.tr : tail_rows;
      if constexpr (TAPS == 9) {
        const int img0 = div16(R0, a.magic_ho);
        rho0 = img0 * a.hp + (R0 - img0 * a.ho) * a.stride;
      }
    };
    // position of this wavefront's patch load k for the tile
    auto position = [&](int k) __attribute__((always_inline)) {
      const int sl = sl0 + kStep * k;
      if constexpr (TAPS == 1) return sl < here ? R0 * a.xps + kStep * k * a.xps + col0 : kOut;
      const int rho = rho0 + (sl >> a.logp), img = div16(rho, a.magic_hp), hi = rho - (int)__umul24(img, a.hp) - a.pad;
      const int col = one_col ? col0 : column(sl);
      return img < a.n && (unsigned)hi < (unsigned)a.h && col != kOut ? ((int)__umul24(img, a.h) + hi) * rowx + col : kOut;
    };
    const int nwl = NWL + (lw < (WB / 1024) % kLw ? 1 : 0);       // weight loads of this wavefront per stage
    const int lane16 = lane * 16 + lw * 1024;
    int is = 0, ib = 0, iv = 0, itile = 0;   // the next stage to issue: stage of its tile, buffer, number
    // (weights first: their addresses need nothing of the tile)
    auto issue = [&]() __attribute__((always_inline)) {
      const unsigned buf = lds0 + ib * a.pstr + lw * 1024;
      int c = is < a.s0 ? b0 + is * SB : (is - a.s0) * SB;
      if (is >= a.s0 && c >= b0) c += a.gap_chn;
      if (a.wres < 0 || iv < a.s) {
        const unsigned wd = a.wres < 0 ? buf + a.psz : lds0 + a.wres + is * WB + lw * 1024;
        const i32x4 r = is < a.s0 ? wr0 : wr1;
        const int so = (is < a.s0 ? is : is - a.s0) * WB;
#pragma unroll
        for (int k = 0; k < NWL; ++k) dma(r, lane16, so + k * (kLw * 1024), wd + k * (kLw * 1024));
        if (nwl > NWL) dma(r, lane16, so + NWL * (kLw * 1024), wd + NWL * (kLw * 1024));
      }
      if (is == 0) {                         // (each load goes out as soon as its position is known)
        tile_setup(itile);
#pragma unroll
        for (int k = 0; k < kMaxPatchLoads; ++k) {
          if (k >= np) break;
          voff[k] = position(k);
          dma(xr, voff[k], c, buf + k * (kLw * 1024));
        }
      } else {
#pragma unroll
        for (int k = 0; k < kMaxPatchLoads; ++k) {
          if (k >= np) break;
          dma(xr, voff[k], c, buf + k * (kLw * 1024));
        }
      }
      ++iv;
      if (++is == a.s) {
        is = 0;
        ++itile;
      }
      if (++ib == a.nb) ib = 0;
    };
    auto n_loads = [&](int v) { return np + (a.wres < 0 || v < a.s ? nwl : 0); };
    int out = 0;                             // stages published as landed
    auto land = [&]() __attribute__((always_inline)) {
      // stage `out` has landed once only the loads of the stages issued after it are in flight
      int fly = 0;
      for (int v = out + 1; v < iv; ++v) fly += n_loads(v);
      wait_vm<0, 62>(fly);
      ++out;
      publish(landed + 4 * lw, out);
    };
    issue();
    bare_barrier();                          // the counters are set up
    int free_to = 0;
    if constexpr ((FORM & kInTurn) != 0) {
      // Once all have filled the buffers together a loading wavefront takes whole stages, nb + lw, nb + 4 + lw ...: its waits, for a buffer and for its
      // loads, are under the others' loads.  With a quarter of every stage each, as below, all four issue at the same time, with the memory path full, and
      // then wait, look and publish at the same time, with the path idle: of 1400 clocks of a stage of 33 KB 800, of one of 8 KB nearly all.  What is
      // published is the first stage of a wavefront's own that has not landed, so the smallest of the four is again the number of stages that have.
      //   bf16 320 to 640 channels at 14x14, 100 images 43.7 -> 30.2 us, int8 35.8 -> 26.9; 192 to 128, 200 images 16.3 -> 13.1; int8 768 to 384 at
      // 20x20, 50 images 19.7 -> 18.1; bf16 1024 at 14x14, 64 images 46.1 -> 43.1.  (A kernel of its own: in one with the other loop that was 3 to 4 % slower.)
      constexpr int kPx = 64 / CPS, kOwn = 4 * CPS;          // pixels of a load; loads of the largest patch
      const int lane_at = lane / CPS * a.xps + ((lane % CPS) ^ slot_perm<CPS>(lane / CPS, a.bit)) * 16;
      int own[kOwn], t = -1, landed_to = 0;
      auto whole = [&]() __attribute__((always_inline)) {
        const unsigned buf = lds0 + ib * a.pstr;
        int c = is < a.s0 ? b0 + is * SB : (is - a.s0) * SB;
        if (is >= a.s0 && c >= b0) c += a.gap_chn;
        if (a.wres < 0 || iv < a.s) {
          const unsigned wd = a.wres < 0 ? buf + a.psz : lds0 + a.wres + is * WB;
          const i32x4 r = is < a.s0 ? wr0 : wr1;
          const int so = (is < a.s0 ? is : is - a.s0) * WB;
#pragma unroll
          for (int k = 0; k < WB / 1024; ++k) dma(r, lane * 16, so + k * 1024, wd + k * 1024);
        }
        if (t != itile) {
          t = itile;
          tile_setup(t);
#pragma unroll
          for (int k = 0; k < kOwn; ++k) own[k] = lane / CPS + kPx * k < here ? (R0 + kPx * k) * a.xps + lane_at : kOut;
        }
#pragma unroll
        for (int k = 0; k < kOwn; ++k) {
          if (k >= a.n_pl) break;
          dma(xr, own[k], c, buf + k * 1024);
        }
      };
      auto go_on = [&](int by) __attribute__((always_inline)) {       // from the stage behind the last one issued
        iv += by;
        is += by;
        ib += by;
        while (is >= a.s) {
          is -= a.s;
          ++itile;
        }
        while (ib >= a.nb) ib -= a.nb;
      };
      const int fill = V < a.nb ? V : a.nb;
      while (iv < fill) {
        issue();
        if (iv - out > 2) land();
      }
      while (out < fill - 1) land();
      wait_vm<0, 2>(0);
      go_on(lw);
      publish(landed + 4 * lw, iv);                          // (its parts of those)
      while (iv < V) {
        // its buffer is free: every multiplying wavefront is done with the stage before in it, or has passed that by, and it has landed
        wait_counters<kCw>(done, lane, iv - a.nb + 1, free_to);
        wait_counters<kLw>(landed, lane, iv - a.nb + 1, landed_to);
        whole();
        wait_vm<0, 2>(0);
        publish(landed + 4 * lw, iv + kLw);
        go_on(kLw);
      }
      mark_if_gave_up(free_to);
      mark_if_gave_up(landed_to);
      return;
    }
    while (iv < V) {
      // the buffer of stage iv is free when every multiplying wavefront is done with stage iv - nb
      while (free_to < iv - a.nb + 1 && out < iv) {
        land();
        if (out < iv) {
          int v;
          asm volatile("ds_read_b32 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(v) : "v"(done + (lane < kCw ? lane : 0) * 4) : "memory");
          if (__ballot(v < iv - a.nb + 1) == 0ull) free_to = iv - a.nb + 1;
        }
      }
      wait_counters<kCw>(done, lane, iv - a.nb + 1, free_to);
      issue();
      if (iv - out > 2) land();
    }
    while (out < V) land();
    mark_if_gave_up(free_to);
    return;
  }

  // ================================ multiplying wavefronts ==========================================
  // (the address waits in LDS: read from the arguments at the end of each wavefront it cost a launch 1.5 us)
  if (tid == 0) *(uint32_t**)(lds + a.tabs + kTabs * 256 + 48) = a.gave_up;
  acc_t* const tlo = (acc_t*)(lds + a.tabs) + ch0;   // [64] thresholds, lower and upper
  acc_t* const thi = tlo + 64;
  float* const aff = (float*)(thi + 64);             // [4][64] scale0, shift0, scale1, shift1; int8: mult0, mult1
  long long* const addends = (long long*)(aff + 192 - ch0) + ch0;      // int8: what is added before the shift
  bare_barrier();                                    // the counters are set up
  const int rowb = SB << a.logp;                     // bytes per patch row
  const int flip = !PAIR || a.bit < a.logp ? 0 : CPS * 8;     // what a patch row more changes in the chunk permutation
  const unsigned wlane = lh * 1024 + (lj + ch0) * 16;// lane's offset of its weight rows in a K step
  acc16 accP[PF][2], accS[PF][2];                    // base sums; base and conditional sums (PF = 2: accP holds these too)

  // One stage: the operand reads of K steps k+1 and k+2 are in flight while step k is multiplied.  HALVES: bit c, the block's
  // channels 32c .. 32c + 31 take part.
  auto mma_stage = [&](auto f0c, auto nfc_, auto halves_c, unsigned pat, unsigned wgt, const int (&pa)[PF][3], acc16 (&acc)[PF][2])
      __attribute__((always_inline)) {
    constexpr int F0 = decltype(f0c)::value, NF = decltype(nfc_)::value;       // fragments F0 .. F0 + NF - 1
    constexpr int PD = NF == 1 && KS > 1 ? 2 : 1, NR = PD + 1;
    constexpr int HALVES = decltype(halves_c)::value, NC = HALVES == 3 ? 2 : 1;
    i32x4 wa[NR][2], xb[NR][NF];
    const unsigned wad = wgt + wlane;
    auto read_step = [&](auto kc) __attribute__((always_inline)) {
      constexpr int k = decltype(kc)::value, n = k % NR, tap = k / PAIRS, r = tap / 3, c = tap % 3;
      if constexpr (HALVES & 1) wa[n][0] = lds_read16<k * 2048>(wad);
      if constexpr (HALVES & 2) wa[n][1] = lds_read16<k * 2048 + 512>(wad);
#pragma unroll
      for (int f = 0; f < NF; ++f)
        xb[n][f] = lds_read16<0>((unsigned)((pa[F0 + f][c] + (int)(pat + r * rowb)) ^ (r == 1 ? (k % PAIRS) * 32 ^ flip : (k % PAIRS) * 32)));
    };
    static_for<PD>([&](auto kc) __attribute__((always_inline)) { read_step(kc); });
    static_for<KS>([&](auto kc) __attribute__((always_inline)) {
      constexpr int k = decltype(kc)::value, n = k % NR;
      constexpr int later = KS - 1 - k < PD - 1 ? KS - 1 - k : PD - 1;
      __builtin_amdgcn_s_waitcnt(0xC07F | ((later * (NC + NF)) << 8));
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (k + PD < KS) read_step(std::integral_constant<int, k + PD>{});
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int f = 0; f < NF; ++f) {
        if constexpr (HALVES & 1) acc[F0 + f][0] = Tr::mfma(wa[n][0], xb[n][f], acc[F0 + f][0]);
        if constexpr (HALVES & 2) acc[F0 + f][1] = Tr::mfma(wa[n][1], xb[n][f], acc[F0 + f][1]);
      }
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  // MFMA results may be read by ordinary instructions some wait states after the last one
  auto settle = [&]() __attribute__((always_inline)) {
    asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };

  // The pixel's sums: with a fired gate the ones that hold the conditional channels.
  auto pick = [&](unsigned dl) __attribute__((always_inline)) {
    static_for<4 * kF>([&](auto ic) __attribute__((always_inline)) {
      constexpr int f = decltype(ic)::value >> 2, i = (decltype(ic)::value & 3) * 4;
      int m[4];
      ones_if4<16 * f + i>(dl, m);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const acc_t pv = accP[0][f][i + e], sv = accS[0][f][i + e];
        acc_t r;
        from_bits(select_bits(m[e], as_bits(sv), as_bits(pv)), r);
        accP[0][f][i + e] = r;
      }
    });
  };
  // bf16 accesses to y and the residual go in the transposed order of transpose4: access j is 16 pixels of one lane
  // half, four lanes per pixel, i.e. half as many cache lines as a lane's own pieces would touch; int8 ones likewise, two pieces.
  //   They are buffer accesses, at 32-bit offsets from the tile's first pixel that are formed once; the range check drops lanes without a pixel (addresses
  // of 64 bits, a branch and zeros for each of them were a quarter of an output's instructions).
  constexpr unsigned kNoPixel = 0x80000000u;
  const int rowy = Base::kDtype == CG_I8 ? a.c_out : a.c_out * 2;
  auto px_of = [&](int px, int h) __attribute__((always_inline)) {   // pixel 16*h + lane % 16 of the fragment
    return __builtin_amdgcn_ds_bpermute((lane & 15) * 4 + h * 64, px);
  };
  struct Places {
    unsigned at[2];                                  // of the lane's pixels in accesses 0 and 1 (2 and 3: 32 bytes on)
  };
  auto places = [&](int px) __attribute__((always_inline)) {
    Places w;
    if constexpr (Base::kDtype == CG_I8 && kF == 1) {
      w.at[0] = w.at[1] = px >= 0 ? __umul24((unsigned)px, (unsigned)rowy) + cbk * kBn + ch0 + 16 * lh : kNoPixel;
    } else {
      const int lane_bytes = Base::kDtype == CG_I8 ? cbk * kBn + (lane & 16) * 2 + (lane & 32) / 2
                                                   : (cbk * kBn + ch0) * 2 + (kF == 1 ? lane & 48 : (lane & 32) * 2 + (lane & 16));
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int q = px_of(px, h);
        w.at[h] = q >= 0 ? __umul24((unsigned)q, (unsigned)rowy) + lane_bytes : kNoPixel;
      }
    }
    return w;
  };
  auto tile_buffer = [&](const void* base, long long m0) __attribute__((always_inline)) {
    return __builtin_amdgcn_make_buffer_rsrc((char*)base + m0 * rowy, (short)0, 0x7fffffff, 0x00027000);
  };
  auto load_at = [&](__amdgpu_buffer_rsrc_t r, const Places& w, int j) __attribute__((always_inline)) {
    return __builtin_bit_cast(i32x4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)(w.at[j & 1] + (j >> 1) * 32), 0, 0));
  };
  typedef __attribute__((ext_vector_type(2))) unsigned u32x2;
  typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
  auto store_at = [&](__amdgpu_buffer_rsrc_t r, const Places& w, int j, i32x4 v) __attribute__((always_inline)) {
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), r, (int)(w.at[j & 1] + (j >> 1) * 32), 0, 0);
  };
  // pieces of a lane's own pixel <-> pieces in that order; two pieces: access j is 16 pixels, again four lanes per pixel
  auto swap_halves = [&](auto& u) __attribute__((always_inline)) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const auto r = __builtin_amdgcn_permlane16_swap((unsigned)u[0][e], (unsigned)u[1][e], false, false);
      u[0][e] = (int)r[0];
      u[1][e] = (int)r[1];
    }
  };
  auto transpose = [&](i32x4 (&u)[2 * kF]) __attribute__((always_inline)) {
    if constexpr (kF == 1)
      swap_halves(u);
    else
      transpose4(u);
  };
  // The residual of the lanes' pixels at w (of the tile that starts at pixel m0 of the batch), 2 x 16 channels each, as it is read: the lane's
  // 16-byte pieces in the transposed order, four of bf16, two of int8; zeros where there is no pixel.
  auto load_residual = [&](long long m0, const Places& w, auto& rs) __attribute__((always_inline)) {
    constexpr int kPieces = Base::kDtype == CG_I8 ? kF : 2 * kF;
    const auto r = tile_buffer(a.residual, m0);
#pragma unroll
    for (int j = 0; j < kPieces; ++j) rs[j] = load_at(r, w, j);
  };
  // Output of those pixels in three steps that whole wavefronts execute.  First the values, from sums, the residual and the
  // decisions in dl (bit 16*f + i; UNI: all the same).  Whether there is a scale/shift is asked once, and its table entries for the next eight channels are
  // on their way while eight are formed:
  auto finish = [&](auto uni, const acc16 (&sum)[2], unsigned dl, long long m0, const Places& w, i32x4 (&early)[2 * kF], i32x4 (&v)[2 * kF]) __attribute__((always_inline)) {
    constexpr bool UNI = decltype(uni)::value;
    // (the larger of a number and a NaN is the number: without ReLU every value stays what it is, a NaN included)
    const float relu_lo = (a.flags & kRelu) ? 0.0f : __builtin_nanf("");
    const float* const taken = aff + 16 * lh + (dl ? 128 : 0);
    i32x4 rs[2 * kF];
    if (added) {
      if constexpr (kAhead) {
#pragma unroll
        for (int j = 0; j < 2 * kF; ++j) rs[j] = early[j];
      } else {
        load_residual(m0, w, rs);
      }
      transpose(rs);
    }
    // eight channels at a time, those from 32*f + 16*lh + 8*h on
    auto rest = [&](auto kc, float (&r)[8]) __attribute__((always_inline)) {
      constexpr int k = decltype(kc)::value;
      if (added) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const unsigned q = (unsigned)rs[k][i >> 1];
          r[i] += __uint_as_float(i & 1 ? q & 0xffff0000u : q << 16);
        }
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) v[k][e] = bf16_pair(max_of(r[2 * e], relu_lo), max_of(r[2 * e + 1], relu_lo));
      if constexpr (PF == 2) __builtin_amdgcn_sched_barrier(0);      // (one piece at a time: no registers for more)
    };
    // each channel with the pair of its own decision
    auto chosen = [&](auto kc, float (&r)[8]) __attribute__((always_inline)) {
      constexpr int f = decltype(kc)::value >> 1, h = decltype(kc)::value & 1;
      const float* const at = aff + 32 * f + 16 * lh + 8 * h;
      static_for<2>([&](auto qc) __attribute__((always_inline)) {
        constexpr int q = decltype(qc)::value;
        const i32x4 a0 = *(const i32x4*)(at + 4 * q), b0 = *(const i32x4*)(at + 64 + 4 * q);
        const i32x4 a1 = *(const i32x4*)(at + 128 + 4 * q), b1 = *(const i32x4*)(at + 192 + 4 * q);
        int m[4];
        ones_if4<16 * f + 8 * h + 4 * q>(dl, m);
#pragma unroll
        for (int e = 0; e < 4; ++e)
          r[4 * q + e] = fmaf(__int_as_float(select_bits(m[e], a1[e], a0[e])), sum[f][8 * h + 4 * q + e],
                              __int_as_float(select_bits(m[e], b1[e], b0[e])));
      });
    };
    if constexpr (PAIR) {
      // (a block has few tiles here, often one, and its end comes from a cold instruction cache: in the shortest form, without the reads ahead.
      // 8x8 pixels of 256 channels, 128 images 13.9 us against 14.1)
      static_for<2 * kF>([&](auto kc) __attribute__((always_inline)) {
        constexpr int k = decltype(kc)::value, f = k >> 1, h = k & 1;
        float r[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) r[i] = sum[f][8 * h + i];
        if (a.flags & kAffine) {
          if constexpr (UNI) {
#pragma unroll
            for (int q = 0; q < 2; ++q) {
              const f32x4 at = *(const f32x4*)(taken + 32 * f + 8 * h + 4 * q), bt = *(const f32x4*)(taken + 64 + 32 * f + 8 * h + 4 * q);
#pragma unroll
              for (int e = 0; e < 4; ++e) r[4 * q + e] = fmaf(at[e], r[4 * q + e], bt[e]);
            }
          } else {
            chosen(kc, r);
          }
        }
        rest(kc, r);
      });
      return;
    }
    if (!UNI || (a.flags & kAffine)) {               // (a layer without scale/shift has one pair throughout)
      if constexpr (UNI) {
        f32x4 t[2][4];                               // scales, then shifts
        auto fetch = [&](auto kc) __attribute__((always_inline)) {
          constexpr int k = decltype(kc)::value, cl = 32 * (k >> 1) + 8 * (k & 1), n = PF == 2 ? 0 : k & 1;
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            t[n][q] = *(const f32x4*)(taken + cl + 4 * q);
            t[n][2 + q] = *(const f32x4*)(taken + 64 + cl + 4 * q);
          }
        };
        if constexpr (PF == 1) fetch(std::integral_constant<int, 0>{});
        static_for<2 * kF>([&](auto kc) __attribute__((always_inline)) {
          constexpr int k = decltype(kc)::value, n = PF == 2 ? 0 : k & 1;
          if constexpr (PF == 2)
            fetch(kc);
          else if constexpr (k + 1 < 2 * kF)
            fetch(std::integral_constant<int, k + 1>{});
          float r[8];
#pragma unroll
          for (int i = 0; i < 8; ++i) r[i] = fmaf(t[n][i >> 2][i & 3], sum[k >> 1][8 * (k & 1) + i], t[n][2 + (i >> 2)][i & 3]);
          rest(kc, r);
        });
      } else {
        static_for<2 * kF>([&](auto kc) __attribute__((always_inline)) {
          float r[8];
          chosen(kc, r);
          rest(kc, r);
        });
      }
    } else {
      static_for<2 * kF>([&](auto kc) __attribute__((always_inline)) {
        constexpr int k = decltype(kc)::value;
        float r[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) r[i] = sum[k >> 1][8 * (k & 1) + i];
        rest(kc, r);
      });
    }
  };
  // then, where y holds the values for an unfired gate already, each channel's own
  auto choose = [&](unsigned dl, long long m0, const Places& w, i32x4 (&v)[4]) __attribute__((always_inline)) {
    i32x4 base[4];
    const auto r = tile_buffer(a.y, m0);
#pragma unroll
    for (int j = 0; j < 4; ++j) base[j] = load_at(r, w, j);
    transpose4(base);
    static_for<4>([&](auto jc) __attribute__((always_inline)) {
      constexpr int j = decltype(jc)::value;
      int m[8];
      ones_if4<8 * j>(dl, *(int(*)[4])&m[0]);
      ones_if4<8 * j + 4>(dl, *(int(*)[4])&m[4]);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[j][e] = select_bits(select_bits(0xffff, m[2 * e], m[2 * e + 1]), v[j][e], base[j][e]);
    });
  };
  // and the stores
  auto store = [&](i32x4 (&v)[2 * kF], long long m0, const Places& w) __attribute__((always_inline)) {
    transpose(v);
    const auto r = tile_buffer(a.y, m0);
#pragma unroll
    for (int j = 0; j < 2 * kF; ++j) store_at(r, w, j, v[j]);
  };
  // Shuffled channel order (Sec. 3.3): channel j of group i goes to position j*groups + i of its pixel.  The block's 64 channels
  // are `ng` groups x `nj` channels: an LDS row holds a pixel's in the order [j][group], so that a run of ng elements is
  // contiguous in both, and consecutive lanes store consecutive j.  A lane's sixteen words of a row are formed in registers
  // for one, two and four groups (four: from the exchanged halves of two lanes) and the runs of several pixels are under way
  // together.  (One element and one run after the other, as it was and as other numbers of groups still are, a fragment's output
  // took 11000 clocks.)  With the products with zeros left out, in four groups, 64 images, us: 128 channels at 28x28, counts too
  // 42.0 -> 31.4, 64 at 56x56 51.7 -> 36.6; eight groups of 128 at 28x28, natural order 27.7 -> 26.0.
  // Stores through buffer accesses, at an addition each, instead of 64-bit addresses and a branch: 128 at 28x28 29.5 -> 28.4, in eight groups 25.5 -> 24.6,
  // 64 at 56x56 34.4 -> 32.8, 256 at 14x14 20.8 -> 19.6.
  auto shuffled_store = [&](i32x4 (&v)[4], long long m0, int px) __attribute__((always_inline)) {
    const int cpg = a.cpg, groups = a.groups;
    const int njl = cpg >= kBn ? 6 : 31 - __clz(cpg), ngl = 6 - njl;    // (a group narrower than a block divides it)
    const int ng = 1 << ngl, nj = 1 << njl;
    const int g0 = cbk * kBn / cpg, j0 = cbk * kBn - g0 * cpg;          // first group; first channel in it (ng = 1)
    char* const rows = lds + a.shuf + wave * (32 * kShufRow);
    int at = lane;                                   // (opaque: addresses formed from it are not kept across the K loops)
    asm volatile("" : "+v"(at));
    auto runs = [&](auto nglc) __attribute__((always_inline)) {
      constexpr int NGL = decltype(nglc)::value, NG = 1 << NGL, NJ = 64 >> NGL, PX = 64 / NJ;      // PX pixels per store
      using run_t = std::conditional_t<NG == 1, uint16_t, std::conditional_t<NG == 2, uint32_t, uint2>>;
      i32x4* const mine = (i32x4*)(rows + (at & 31) * kShufRow + (at >> 5) * (NG == 1 ? 32 : 64));
      if constexpr (NG == 1) {                       // channels 16*lh + i and 32 + 16*lh + i
        mine[0] = v[0];
        mine[1] = v[1];
        mine[4] = v[2];
        mine[5] = v[3];
      } else {
        i32x4 w[4];
        if constexpr (NG == 2) {                     // j = 16*lh + i: the pairs (v[0..1], v[2..3]) of elements
#pragma unroll
          for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const unsigned lo = (unsigned)v[q >> 1][2 * (q & 1) + (e >> 1)], hi = (unsigned)v[2 + (q >> 1)][2 * (q & 1) + (e >> 1)];
              w[q][e] = (int)__builtin_amdgcn_perm(hi, lo, e & 1 ? 0x07060302u : 0x05040100u);
            }
        } else {                                     // j = 8*lh + i: groups 2f + lh; lane halves exchange eight of their sixteen j
#pragma unroll
          for (int f = 0; f < kF; ++f)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const auto r = __builtin_amdgcn_permlane32_swap((unsigned)v[2 * f][e], (unsigned)v[2 * f + 1][e], false, false);
              v[2 * f][e] = (int)r[0];               // group 2f, then group 2f + 1, of j = 8*lh + 2e, 2e + 1
              v[2 * f + 1][e] = (int)r[1];
            }
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
              for (int f = 0; f < kF; ++f)
                w[e][2 * h + f] = (int)__builtin_amdgcn_perm((unsigned)v[2 * f + 1][e], (unsigned)v[2 * f][e], h ? 0x07060302u : 0x05040100u);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) mine[q] = w[q];
      }
      wait_lds();
      const int j = at & (NJ - 1), sub = at / NJ;    // run of the pixel, pixel of the store
      // (buffer accesses at 32-bit offsets, of which a pixel's part is formed by its own lane; the range check drops those of no pixel)
      const auto to = tile_buffer(a.y, m0);
      const int of_px = (int)(px >= 0 ? __umul24((unsigned)px, (unsigned)rowy) : kNoPixel), of_run = ((j0 + j) * groups + g0) * 2;
#pragma unroll
      for (int p0 = 0; p0 < 32; p0 += 8 * PX) {
        run_t r[8];
        int of[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const int q = p0 + k * PX + sub;
          of[k] = __builtin_amdgcn_ds_bpermute(q * 4, of_px) + of_run;
          r[k] = *(const run_t*)(rows + q * kShufRow + j * (int)sizeof(run_t));
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          if constexpr (NG == 1)
            __builtin_amdgcn_raw_buffer_store_b16(r[k], to, of[k], 0, 0);
          else if constexpr (NG == 2)
            __builtin_amdgcn_raw_buffer_store_b32(r[k], to, of[k], 0, 0);
          else
            __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, r[k]), to, of[k], 0, 0);
        }
      }
      wait_lds();
    };
    if (ng == 1) {
      runs(std::integral_constant<int, 0>{});
    } else if (ng == 2 && (groups & 1) == 0) {       // (g0 is a multiple of ng: runs lie on their own size)
      runs(std::integral_constant<int, 1>{});
    } else if (ng == 4 && (groups & 3) == 0) {
      runs(std::integral_constant<int, 2>{});
    } else {
      uint16_t* const row = (uint16_t*)(rows + (at & 31) * kShufRow);
      const int lane_ch = 16 * (at >> 5);
#pragma unroll
      for (int f = 0; f < kF; ++f)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int c = 32 * f + lane_ch + i;
          row[((c & (nj - 1)) << ngl) + (c >> njl)] = (uint16_t)((unsigned)v[2 * f + (i >> 3)][(i & 7) >> 1] >> (16 * (i & 1)));
        }
      wait_lds();
      for (int id = lane; id < 32 * nj; id += 64) {
        const int q = id >> njl, j = id & (nj - 1);                     // pixel of the fragment, channel of its group
        const int pq = __shfl(px, q, 64);
        const uint16_t* const from = (const uint16_t*)(rows + q * kShufRow) + (j << ngl);
        uint16_t* const to = (uint16_t*)a.y + (m0 + pq) * a.c_out + (j0 + j) * groups + g0;
        if (pq >= 0)
          for (int e = 0; e < ng; ++e) to[e] = from[e];
      }
      wait_lds();
    }
  };
  // one_pair: the whole fragment takes the same scale/shift pair (nothing fired, a dense layer, or the pairs are equal, as in
  // a network that was trained with one normalisation): half the table reads and a quarter of the instructions of a choice
  // per value.  ResNet-18 with equal pairs, 64 images 426 -> 413 us, 256 images 1120 -> 1091.
  auto emit_fast = [&](unsigned dl, bool one_pair, long long m0, int px, const Places& w, i32x4 (&rs)[2 * kF]) __attribute__((always_inline)) {
    if constexpr (Base::kDtype != CG_I8) {
      i32x4 v[2 * kF];
      if (one_pair)
        finish(std::true_type{}, accP[0], dl, m0, w, rs, v);
      else
        finish(std::false_type{}, accP[0], dl, m0, w, rs, v);
      if constexpr (OUT == kShuffled) {
        shuffled_store(v, m0, px);
        return;
      }
      store(v, m0, w);
    } else {
      // requantised int8: t = (S * mult_d + bias + half + residual * res_mult) >> shift, clamped (exact in 64 bits;
      // shifts of two and more: with the high word clamped to +-2^(shift-1) the shifted value fits 32 bits, and what was
      // clamped still lies beyond the bytes' range).  Access h covers 16 pixels, four 16-lane groups per pixel.
      const int lo = (a.flags & kRelu) ? 0 : -128;
      const int h_hi = (1 << (a.rq_shift - 1)) - 1, h_lo = -1 - h_hi;
      i32x4 v[2];
      if (added) {
        if constexpr (!kAhead) load_residual(m0, w, rs);
        if constexpr (kF == 2) swap_halves(rs);
      }
      // four values, clamped to the bytes' range, as bytes
      auto pack4 = [&](const unsigned (&c)[4]) __attribute__((always_inline)) {
        const unsigned p01 = __builtin_amdgcn_perm(c[1], c[0], 0x0c0c0400u), p23 = __builtin_amdgcn_perm(c[3], c[2], 0x04000c0cu);
        return (int)(p01 | p23);
      };
      // Where the layer allows (fits_32_bits), the sum is clamped to where the output still changes, and factors of 24 bits and
      // sums of 32 are exact.  64-bit products cost an output 5000 clocks a fragment: int8 128 channels at 28x28, 32 images 10.7 -> 10.1
      // us, 256 at 14x14, 64 images 13.7 -> 13.3.
      auto narrow = [&](auto uni) __attribute__((always_inline)) {
        constexpr bool UNI = decltype(uni)::value;           // nothing fired, or a dense layer: one mult
        const int* const mult = (const int*)aff + (UNI && dl ? 64 : 0);
        const int *const s_lo = (const int*)thi, *const add = (const int*)aff + 192, *const s_hi = (const int*)aff + 256;
        static_for<4 * kF>([&](auto kc) __attribute__((always_inline)) {
          constexpr int f = decltype(kc)::value >> 2, q = decltype(kc)::value & 3;
          const int cl = 32 * f + 16 * lh;
          {
            const i32x4 ma = *(const i32x4*)(mult + cl + 4 * q), lo4 = *(const i32x4*)(s_lo + cl + 4 * q);
            const i32x4 ad = *(const i32x4*)(add + cl + 4 * q), hi4 = *(const i32x4*)(s_hi + cl + 4 * q);
            i32x4 mb = ma;
            if constexpr (!UNI) mb = *(const i32x4*)(mult + 64 + cl + 4 * q);
            unsigned c[4];
            int m[4];
            if constexpr (!UNI) ones_if4<16 * f + 4 * q>(dl, m);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const int sv = accP[0][f][4 * q + e];
              int t = __mul24(med3(sv, lo4[e], hi4[e]), UNI ? ma[e] : select_bits(m[e], mb[e], ma[e])) + ad[e];
              if (added) t += __mul24((int)(int8_t)((unsigned)rs[f][q] >> (8 * e)), a.rq_res_mult);
              c[e] = (unsigned)med3(t >> a.rq_shift, lo, 127);
            }
            v[f][q] = pack4(c);
          }
        });
      };
      if (a.flags & kFit32) {
        if (one_pair)
          narrow(std::true_type{});
        else
          narrow(std::false_type{});
      } else {
#pragma unroll
      for (int f = 0; f < kF; ++f) {
        const int cl = 32 * f + 16 * lh;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const i32x4 m0_ = *(const i32x4*)(aff + cl + 4 * q), m1_ = *(const i32x4*)(aff + 64 + cl + 4 * q);
          unsigned c[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int m = (int)(dl << (31 - 16 * f - 4 * q - e)) >> 31;
            const int sv = accP[0][f][4 * q + e];
            long long t = (long long)sv * ((m1_[e] & m) | (m0_[e] & ~m)) + addends[cl + 4 * q + e];
            if (added) t += (long long)(int8_t)((unsigned)rs[f][q] >> (8 * e)) * a.rq_res_mult;
            const int th = med3((int)(t >> 32), h_lo, h_hi);
            c[e] = (unsigned)med3((int)__builtin_amdgcn_alignbit((unsigned)th, (unsigned)t, (unsigned)a.rq_shift), lo, 127);
          }
          v[f][q] = pack4(c);
        }
      }
      }
      if constexpr (kF == 2) swap_halves(v);
      const auto r = tile_buffer(a.y, m0);
#pragma unroll
      for (int h = 0; h < kF; ++h) store_at(r, w, h, v[h]);
    }
  };
  // Outputs of four bytes, 16 channels of a pixel (64 bytes) at a time: in the transposed order four lanes write them, i.e. an access touches 16
  // lines of memory instead of 64.  Scale and shift come from LDS.  bf16 layers, 64 channels at 50x50, 156 images 70.8 -> 52.1 us, 1x1 of 256
  // to 512 at 36x13, 99 images 62.5 -> 45.4, 448 to 256 at 15x96, 11 images 65.4 -> 58.1; int8 layers, 64 to 128 at 82x82, 60 images 99.1 -> 79.4,
  // 384 at 47x47, 7 images 31.7 -> 27.1.
  auto emit_wide = [&](unsigned dl, bool one_pair, long long m0, int px) __attribute__((always_inline)) {
    const int row4 = a.c_out * 4;
    unsigned at[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int q = px_of(px, h);
      at[h] = q >= 0 ? __umul24((unsigned)q, (unsigned)row4) + cbk * (kBn * 4) + (lane >> 4) * 16 : kNoPixel;
    }
    const auto yb = __builtin_amdgcn_make_buffer_rsrc(a.y + m0 * row4, (short)0, 0x7fffffff, 0x00027000);
    [[maybe_unused]] i32x4 r8[2];
    if constexpr (Base::kDtype == CG_I8)
      if (added) {
        load_residual(m0, places(px), r8);
        swap_halves(r8);
      }
    static_for<2>([&](auto fc) __attribute__((always_inline)) {
      constexpr int f = decltype(fc)::value;
      i32x4 v[4];
      if constexpr (Base::kDtype == CG_I8) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            int t = accP[0][f][4 * q + e];
            if (added) {
              long long w = (long long)t + (long long)(int8_t)((unsigned)r8[f][q] >> (8 * e)) * a.rq_res_mult;
              w = w > 2147483647ll ? 2147483647ll : w;
              w = w < -2147483648ll ? -2147483648ll : w;
              t = (int)w;
            }
            v[q][e] = (a.flags & kRelu) && t < 0 ? 0 : t;
          }
      } else {
        i32x4 rs[4];
        if (added) {
          const auto rb = __builtin_amdgcn_make_buffer_rsrc((char*)a.residual + m0 * row4, (short)0, 0x7fffffff, 0x00027000);
#pragma unroll
          for (int j = 0; j < 4; ++j)
            rs[j] = __builtin_bit_cast(i32x4, __builtin_amdgcn_raw_buffer_load_b128(rb, (int)(at[j & 1] + f * 128 + (j >> 1) * 64), 0, 0));
          transpose4(rs);
        }
        // (the larger of a number and a NaN is the number: without ReLU every value stays what it is, a NaN included)
        const float relu_lo = (a.flags & kRelu) ? 0.0f : __builtin_nanf("");
        const float* const first = aff + 32 * f + 16 * lh;
        const float* const taken = first + (dl ? 128 : 0);
        static_for<4>([&](auto qc) __attribute__((always_inline)) {
          constexpr int q = decltype(qc)::value;
          f32x4 r;
#pragma unroll
          for (int e = 0; e < 4; ++e) r[e] = accP[0][f][4 * q + e];
          if (a.flags & kAffine) {
            if (one_pair) {
              const f32x4 st = *(const f32x4*)(taken + 4 * q), bt = *(const f32x4*)(taken + 64 + 4 * q);
#pragma unroll
              for (int e = 0; e < 4; ++e) r[e] = fmaf(st[e], r[e], bt[e]);
            } else {
              const i32x4 a0 = *(const i32x4*)(first + 4 * q), b0 = *(const i32x4*)(first + 64 + 4 * q);
              const i32x4 a1 = *(const i32x4*)(first + 128 + 4 * q), b1 = *(const i32x4*)(first + 192 + 4 * q);
              int m[4];
              ones_if4<16 * f + 4 * q>(dl, m);
#pragma unroll
              for (int e = 0; e < 4; ++e)
                r[e] = fmaf(__int_as_float(select_bits(m[e], a1[e], a0[e])), r[e], __int_as_float(select_bits(m[e], b1[e], b0[e])));
            }
          }
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            if (added) r[e] += __int_as_float(rs[q][e]);
            v[q][e] = __float_as_int(max_of(r[e], relu_lo));
          }
        });
      }
      transpose4(v);
#pragma unroll
      for (int j = 0; j < 4; ++j)
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v[j]), yb, (int)(at[j & 1] + f * 128 + (j >> 1) * 64), 0, 0);
    });
  };
  // every other output type and order, one lane's pixel at a time
  auto emit_any = [&](unsigned dl, long long m) __attribute__((always_inline)) {
    // The arguments it needs are read here, and its channel numbers formed here: kept in registers across the K loops
    // (what the compiler does by itself) they would spill.
    const auto* kernarg = (const __attribute__((address_space(4))) char*)__builtin_amdgcn_kernarg_segment_ptr() + kParamsAt;
    asm volatile("" : "+s"(kernarg));
    const Params q = *(const Params*)kernarg;
    int lane_ch = 16 * lh;
    asm volatile("" : "+v"(lane_ch));
#pragma unroll
    for (int f = 0; f < kF; ++f) {
      const int co0 = cbk * kBn + 32 * f + lane_ch;
      const unsigned d16 = (dl >> (16 * f)) & 0xffffu;
      if (q.shuffle) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int co = co0 + i, grp = co / q.cpg;
          const long long o = m * q.c_out + (co - grp * q.cpg) * q.groups + grp;
          const bool fired = ((d16 >> i) & 1u) != 0u;
          const acc_t sv = accP[0][f][i];
          if constexpr (Base::kDtype == CG_I8)
            store_int(q, o, finish_int(q, sv, fired, co, o));
          else
            store_float(q, o, finish_float(q, sv, fired, co, o));
        }
        continue;
      }
      const long long o = m * q.c_out + co0;
      i32x4 v[4];
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const acc_t sv = accP[0][f][4 * q4 + e];
          v[q4][e] = as_bits(sv);
        }
      finish_store8<Base>(q, v[0], v[1], d16 & 0xffu, co0, o);
      finish_store8<Base>(q, v[2], v[3], d16 >> 8, co0 + 8, o + 8);
    }
  };

  int v = 0, b = 0, have = 0;                        // the next stage: its number and buffer; stages known to have landed
#pragma nounroll
  for (int t = 0; t < tiles; ++t) {
    const int R0 = tile_row(t), rows_here = t < a.full ? a.tr : tail_rows;
    const long long m0 = (long long)R0 * a.wo;       // the tile's first output pixel
    // this lane's pixels, one in each of the wavefront's fragments `wave` and (PF = 2) wave + kCw: row and column in the tile
    const int next = v + a.s;                        // first stage of the next tile
    int px[PF], pimg[PF], pa[PF][3];
    bool inside[PF], any[PF];                        // the pixel exists; any of the fragment does
    int lp = lj;
    if constexpr (PF == 2) asm volatile("" : "+v"(lp));       // (formed for each tile: no registers to keep them)
#pragma unroll
    for (int g = 0; g < PF; ++g) {
      const int fr = (PAIR ? wave & 3 : wave) + kCw * g;
      int lr, wo_;
      if constexpr (TAPS == 1) {                     // a row is a pixel
        const int i = fr * 32 + lp;
        px[g] = i < rows_here ? i : -1;
        inside[g] = i < rows_here;
        any[g] = __ballot(inside[g]) != 0ull;
        pa[g][0] = slot_addr<CPS>(inside[g] ? i : 0, lh, a.bit);
        pimg[g] = a.chan_mask ? (R0 + (inside[g] ? i : 0)) / a.hp : 0;
        continue;
      }
      if (a.fwl < 0) {
        const int i = fr * 32 + lp;
        lr = div16(i, a.magic_wo);
        wo_ = i - lr * a.wo;
      } else {
        const int fq = div16(fr, a.magic_nfc);
        lr = (fq << (5 - a.fwl)) + (lp >> a.fwl);
        wo_ = ((fr - fq * a.nfc) << a.fwl) + (lp & ((1 << a.fwl) - 1));
      }
      inside[g] = lr < rows_here && wo_ < a.wo;
      any[g] = __ballot(inside[g]) != 0ull;
      if (!inside[g]) lr = wo_ = 0;                  // lanes past the tile's end read pixel 0 and are dropped
      const int img0 = div16(R0, a.magic_ho);
      const int rho0 = img0 * a.hp + (R0 - img0 * a.ho) * a.stride;
      const int R = R0 + lr;
      pimg[g] = div16(R, a.magic_ho);
      const int slot0 = ((pimg[g] * a.hp + (R - pimg[g] * a.ho) * a.stride - rho0) << a.logp) + wo_ * a.stride;
#pragma unroll
      for (int c = 0; c < 3; ++c) pa[g][c] = slot_addr<CPS>(slot0 + c, lh, a.bit);
      px[g] = inside[g] ? lr * a.wo + wo_ : -1;
    }
    auto pass_by = [&]() __attribute__((always_inline)) {
      publish(done + 4 * wave, next);
      b += next - v;
      v = next;
      while (b >= a.nb) b -= a.nb;
    };
    if (!any[0]) {                                   // no pixel of this tile is this wavefront's
      pass_by();
      continue;
    }
    // The residual is on its way while the stages are multiplied.
    [[maybe_unused]] Places at_early;
    [[maybe_unused]] i32x4 rs_early[2 * kF];
    if constexpr (kAhead) {
      at_early = places(px[0]);
      if (!gate_only) {
        load_residual(m0, at_early, rs_early);
      } else {                               // (defined: else copies of the last tile's are waited for)
#pragma unroll
        for (int j = 0; j < 2 * kF; ++j) rs_early[j] = i32x4{0, 0, 0, 0};
      }
    }
#pragma unroll
    for (int g = 0; g < PF; ++g)
#pragma unroll
      for (int f = 0; f < kF; ++f)
#pragma unroll
        for (int i = 0; i < 16; ++i) accP[g][f][i] = 0;
    // stages first .. last - 1 for fragments f0 .. f0 + nf - 1 and the halves of the block's channels
    auto stages = [&](auto f0, auto nf, auto hv, int first, int last, acc16 (&acc)[PF][2]) __attribute__((always_inline)) {
#pragma nounroll
      for (int s = first; s < last; ++s) {
        wait_counters<kLw>(landed, lane, v + 1, have);
        const unsigned pat = lds0 + b * a.pstr;
        const unsigned wgt = a.wres < 0 ? pat + a.psz : lds0 + a.wres + s * WB;
        mma_stage(f0, nf, hv, pat, wgt, pa, acc);
        ++v;
        publish(done + 4 * wave, v);
        if (++b == a.nb) b = 0;
      }
      settle();
    };
    constexpr std::integral_constant<int, 0> zero{};
    constexpr std::integral_constant<int, 1> one{};
    constexpr std::integral_constant<int, 2> two{};
    constexpr std::integral_constant<int, 3> both{};
    constexpr std::integral_constant<int, (1 << kF) - 1> mine{};
    if constexpr (PF == 2) {
      if (any[1])
        stages(zero, two, both, 0, a.s0, accP);
      else
        stages(zero, one, both, 0, a.s0, accP);
    } else if constexpr (OUT == kHalves || OUT == kShuffled) {
      // Where a block covers several channel groups and a stage lies inside one (spg), its products with a half of the block's
      // channels may be products with zeros throughout; they are left out, a run of such stages by a loop of its own (chosen stage
      // by stage inside one loop the sums moved between registers: 160 of them, and a third of the gain).  A base stage belongs to one group, i.e. to one half: the first half of
      // the stages to the first.
      if (a.spg) {
        stages(zero, one, one, 0, a.s0 >> 1, accP);
        stages(zero, one, two, a.s0 >> 1, a.s0, accP);
      } else {
        stages(zero, one, both, 0, a.s0, accP);
      }
    } else {
      stages(zero, one, mine, 0, a.s0, accP);
    }

    unsigned dl[PF];                                 // a dense layer takes the second pair everywhere
    bool fired[PF];
#pragma unroll
    for (int g = 0; g < PF; ++g) {
      dl[g] = ~0u;
      fired[g] = false;
      if (!gated || !any[g]) continue;
      // ---- gate --------------------------------------------------------------------------------------
      dl[g] = 0u;
#pragma unroll
      for (int f = kF - 1; f >= 0; --f)
#pragma unroll
        for (int q4 = 3; q4 >= 0; --q4) {
          const i32x4 lo4 = *(const i32x4*)(tlo + 32 * f + 16 * lh + 4 * q4);
          Tr::shift_in4(dl[g], accP[g][f][4 * q4], accP[g][f][4 * q4 + 1], accP[g][f][4 * q4 + 2], accP[g][f][4 * q4 + 3], lo4);
        }
      if constexpr (Base::kDtype != CG_I8) {
        if (a.flags & kTwoSided) {
          unsigned below = 0u;                       // bit by bit as above, upper thresholds
#pragma unroll
          for (int f = kF - 1; f >= 0; --f)
#pragma unroll
            for (int q4 = 3; q4 >= 0; --q4) {
              const i32x4 hi4 = *(const i32x4*)(thi + 32 * f + 16 * lh + 4 * q4);
              Tr::shift_in4_le(below, accP[g][f][4 * q4], accP[g][f][4 * q4 + 1], accP[g][f][4 * q4 + 2], accP[g][f][4 * q4 + 3], hi4);
            }
          dl[g] &= below;
        }
      }
      if (!inside[g]) dl[g] = 0u;
      if (a.chan_mask) {
        // channel-wise gate (Sec. 3.2): only the channels that keep their conditional path in this image
        const uint32_t* mw = a.chan_mask + (long long)pimg[g] * a.words + cbk * 2;
        if constexpr (kF == 1)
          dl[g] &= mw[ch0 >> 5] >> (16 * lh);
        else
          dl[g] &= ((mw[0] >> (16 * lh)) & 0xffffu) | (((mw[1] >> (16 * lh)) & 0xffffu) << 16);
      }
      if (a.bitmap) {
        const unsigned other = (unsigned)__shfl_xor((int)dl[g], 32, 64);   // the pixel's other channels
        if constexpr (kF == 1) {
          if (lh == 0 && inside[g]) a.bitmap[(m0 + px[g]) * a.words + cbk * 2 + (ch0 >> 5)] = dl[g] | (other << 16);
        } else if (lh == 0 && inside[g])
          *(uint2*)(a.bitmap + (m0 + px[g]) * a.words + cbk * 2) =
              uint2{(dl[g] & 0xffffu) | (other << 16), (dl[g] >> 16) | (other & 0xffff0000u)};
      }
      fired[g] = __ballot(dl[g] != 0u) != 0ull;
    }
    if (gate_only) continue;     // first pass of the channel-wise gate: the decisions are all it produces
    // ---- conditional path, output ---------------------------------------------------------------------
    if constexpr (PF == 1) {
      if (fired[0]) {
#pragma unroll
        for (int f = 0; f < kF; ++f) accS[0][f] = accP[0][f];
        if constexpr (OUT == kHalves || OUT == kShuffled) {
          // ... and a conditional one to all groups but its own, a half where groups have 32 channels.
          int at = a.s0, to = a.spg && a.cpg == 32 ? a.s0 + 2 * cbk * a.spg : a.s;
#pragma nounroll
          for (;;) {
            stages(zero, one, both, at, to, accS);
            if (to == a.s) break;
            stages(zero, one, two, to, to + a.spg, accS);
            stages(zero, one, one, to + a.spg, to + 2 * a.spg, accS);
            at = to + 2 * a.spg;
            to = a.s;
          }
        } else {
          stages(zero, one, mine, a.s0, a.s, accS);
        }
        pick(dl[0]);
      } else if (gated) {
        pass_by();
      }
      if constexpr (kAhead) {
        emit_fast(dl[0], !fired[0] || (a.flags & kOnePair) != 0u, m0, px[0], at_early, rs_early);
      } else if constexpr (OUT == kWide) {
        emit_wide(dl[0], !fired[0] || (a.flags & kOnePair) != 0u, m0, px[0]);
      } else if constexpr (OUT != kAnyOut) {
        const Places at = places(px[0]);
        i32x4 rs[2 * kF];
        emit_fast(dl[0], !fired[0] || (a.flags & kOnePair) != 0u, m0, px[0], at, rs);
      } else if (inside[0]) {
        emit_any(dl[0], m0 + px[0]);
      }
    } else if constexpr (Base::kDtype != CG_I8) {
      // No registers for two sets of sums: every fragment's outputs for an unfired gate are written first, and where it goes
      // on the fired channels' replace them at the end.
      i32x4 w[4];
      if (gated) {
#pragma unroll
        for (int g = 0; g < PF; ++g) {
          if (!any[g]) continue;
          const Places at = places(px[g]);
          i32x4 rs[4];
          finish(std::true_type{}, accP[g], 0u, m0, at, rs, w);
          store(w, m0, at);
        }
      }
      if (fired[0] && fired[1])
        stages(zero, two, both, a.s0, a.s, accP);
      else if (fired[0])
        stages(zero, one, both, a.s0, a.s, accP);
      else if (fired[1])
        stages(one, one, both, a.s0, a.s, accP);
      else if (gated)
        pass_by();
#pragma unroll
      for (int g = 0; g < PF; ++g) {
        if (gated ? !fired[g] : !any[g]) continue;
        const Places at = places(px[g]);
        i32x4 rs[4];
        finish(std::true_type{}, accP[g], 1u, m0, at, rs, w);
        if (gated) choose(dl[g], m0, at, w);
        store(w, m0, at);
      }
    }
  }
  mark_if_gave_up(have);
}

// [c_out][9][c_phase] -> [column block][stage][kernel row r][K step k][chunk h][row][16 bytes]
// with tap = 3r + k / (CPS/2) and chunk = CPS*sigma + 2*(k % (CPS/2)) + h; row rho of a 32-row
// fragment holds channel 16*((rho/4)%2) + 4*(rho/8) + rho%4, which puts 16 consecutive channels in
// one lane of the transposed product
//
// Channel grouping with blocks that cover several groups (multi != 0): the base phase (phase 0)
// walks the base channels of all the block's groups, the conditional phase all c_in channels; a
// chunk that is not on that path for the row's output channel is packed as zeros (a chunk never
// straddles a group: c_base is a multiple of the chunk's channel count).
__global__ void pack_rows_kernel(const char* __restrict__ w, char* __restrict__ out, int c_phase, int eb, int ch,
                                 int cps, int stages, long long total, int multi, int phase, int c_base, int cpg, int taps) {
  const long long id = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (id >= total) return;
  const int gk = taps == 9 ? 3 * cps / 2 : cps / 2, pairs = cps / 2, rows = taps == 9 ? 3 : 1;
  const int rho = (int)(id & 63);
  long long r_ = id >> 6;
  const int h = (int)(r_ & 1);
  r_ >>= 1;
  const int k = (int)(r_ % gk);
  r_ /= gk;
  const int kr = (int)(r_ % rows);
  r_ /= rows;
  const int ss = (int)(r_ % stages);
  const int cb = (int)(r_ / stages);
  const int tap = 3 * kr + k / pairs;
  const int chunk = cps * ss + 2 * (k % pairs) + h;
  const int fc = rho >> 5, rr = rho & 31;
  const int co = cb * kBn + 32 * fc + 16 * ((rr >> 2) & 1) + 4 * (rr >> 3) + (rr & 3);
  int c_src = chunk * ch;          // first channel of the chunk in the row's w_base / w_cond
  bool zero = false;
  if (multi) {
    const int grp = co / cpg;      // the row's output group = its base input group
    if (phase == 0) {
      const int blk_grp0 = (cb * kBn) / cpg;                 // first group of this column block
      zero = blk_grp0 + c_src / c_base != grp;
      c_src = c_src % c_base;
    } else {
      zero = c_src / c_base == grp;
      if (c_src >= (grp + 1) * c_base) c_src -= c_base;
    }
  }
  i32x4 v = {0, 0, 0, 0};
  if (!zero) v = *(const i32x4*)(w + (((long long)co * taps + tap) * c_phase + c_src) * eb);
  *(i32x4*)(out + id * 16) = v;
}


template <typename Tr, int CPS, int PF, int TAPS, int FORM>
hipError_t launch_rows_one(const RowsPlan& g, const Params& p, const RowsArgs& a, hipStream_t s) {
  const unsigned blocks = a.xcd_cb ? (unsigned)(g.n_slots * g.n_cb) : (unsigned)a.per_xcd * 8u;
  static std::atomic<uint64_t> asked{0};
  const hipError_t attr = allow_lds((const void*)gated_conv_rows_kernel<Tr, CPS, PF, TAPS, FORM>, kLds, asked);
  if (attr != hipSuccess) return attr;
  hipLaunchKernelGGL((gated_conv_rows_kernel<Tr, CPS, PF, TAPS, FORM>), dim3(blocks), dim3(kNt), (size_t)g.lds_bytes, s, a, p);
  return hipGetLastError();
}

template <typename Tr, int OUT>
hipError_t launch_rows_out(const RowsPlan& g, const Params& p, const RowsArgs& a, hipStream_t s) {
  if constexpr (OUT != kHalves && OUT != kPaired && OUT != kPairedAdded) if (g.taps == 1) {
    if (a.flags & kTurns) {
      if (g.cps == 8) return launch_rows_one<Tr, 8, 1, 1, OUT | kInTurn>(g, p, a, s);
      return g.cps == 4 ? launch_rows_one<Tr, 4, 1, 1, OUT | kInTurn>(g, p, a, s) : launch_rows_one<Tr, 2, 1, 1, OUT | kInTurn>(g, p, a, s);
    }
    if (g.cps == 8) return launch_rows_one<Tr, 8, 1, 1, OUT>(g, p, a, s);
    return g.cps == 4 ? launch_rows_one<Tr, 4, 1, 1, OUT>(g, p, a, s) : launch_rows_one<Tr, 2, 1, 1, OUT>(g, p, a, s);
  }
  if constexpr (Tr::Base::kDtype == CG_BF16 && (OUT == kNatural || OUT == kAdded))
    if (g.pf == 2) return launch_rows_one<Tr, 4, 2, 9, OUT>(g, p, a, s);      // (planned for stages of four chunks only)
  return g.cps == 4 ? launch_rows_one<Tr, 4, 1, 9, OUT>(g, p, a, s) : launch_rows_one<Tr, 2, 1, 9, OUT>(g, p, a, s);
}

// fragments of a tile of r rows of wo pixels
int tile_fragments(int r, int fwl, int nfc, int wo) {
  const int fh = 32 >> (fwl < 0 ? 0 : fwl);
  return fwl < 0 ? (r * wo + 31) / 32 : (r + fh - 1) / fh * nfc;
}

template <typename Tr>
hipError_t launch_rows_type(const RowsPlan& g, const Params& p, const RowsArgs& a, hipStream_t s) {
  if (a.flags & kFourBytes) return launch_rows_out<Tr, kWide>(g, p, a, s);
  if (!(a.flags & kFast)) return launch_rows_out<Tr, kAnyOut>(g, p, a, s);
  if constexpr (Tr::Base::kDtype == CG_BF16)
    if (a.flags & kShuf2) return launch_rows_out<Tr, kShuffled>(g, p, a, s);
  if (g.pf == 1 && g.taps == 9 && a.spg) return launch_rows_out<Tr, kHalves>(g, p, a, s);
  const bool added = (a.flags & kResidual) != 0u;
  if (a.flags & kPairs) return added ? launch_rows_out<Tr, kPairedAdded>(g, p, a, s) : launch_rows_out<Tr, kPaired>(g, p, a, s);
  return added ? launch_rows_out<Tr, kAdded>(g, p, a, s) : launch_rows_out<Tr, kNatural>(g, p, a, s);
}

unsigned magic16(int d) { return d == 1 ? 0u : (unsigned)(((1ull << 32) + (unsigned)d - 1) / (unsigned)d); }

// Whether the outputs and the residual of a tile of pf fragments to a wavefront are within 31-bit offsets of its first pixel (a pixel's bytes are then
// within the 24 bits of the products that form them): up to 2^21 channels of four bytes, 2^22 of two (2^21 with two fragments), 2^23 of one.
// The others' outputs take 64-bit addresses (kAnyOut).
bool near_outputs(int c_out, int out_dtype, int pf) {
  const int bytes = out_dtype == CG_BF16 ? 2 : out_dtype == CG_I8 ? 1 : 4;
  return 32ll * kCw * pf * bytes * c_out < (1ll << 31);
}
// LDS for the shuffled order's rows: bf16 outputs without a residual
int shuffle_bytes(const cg_conv_desc& d) {
  return d.shuffle && d.in_dtype == CG_BF16 && d.out_dtype == CG_BF16 && !(d.epilogue & CG_EPI_RESIDUAL) && near_outputs(d.c_out, CG_BF16, 1)
             ? kCw * 32 * kShufRow : 0;
}

// The channel walk of both phases in stages of `cps` chunks; false where the shape does not allow them.
bool plan_walk(const cg_conv_desc& d, int cps, RowsPlan& g, int& base_k, int& c_cond) {
  g.elem_bytes = d.in_dtype == CG_BF16 ? 2 : 1;
  g.ch = 16 / g.elem_bytes;
  const long long xps = d.x_pixel_stride ? d.x_pixel_stride : d.c_in;
  if (xps % g.ch) return false;
  // channels the two phases walk
  base_k = d.c_base, c_cond = d.c_in - d.c_base;
  g.gsp = 1;
  if (d.groups > 1) {
    const int cpg = d.c_out / d.groups;
    if (cpg % kBn == 0) {
      g.grp_mode = 1;                       // a 64-channel block lies inside one group
    } else if (kBn % cpg == 0 && d.c_base % g.ch == 0) {
      g.grp_mode = 2;                       // a block covers kBn/cpg whole groups
      g.gsp = kBn / cpg;
      base_k = g.gsp * d.c_base;
      c_cond = d.c_in;
    } else {
      return false;
    }
  }
  if (d.groups <= 1 && base_k % (2 * g.ch) != 0 && base_k % g.ch == 0 && base_k < d.c_in && d.c_in % (2 * g.ch) == 0) {
    // A base group of one 16-byte chunk (16 int8 channels) is below the two-chunk K step: the base
    // phase then walks two chunks with zero weights on the second, and the conditional phase all
    // input channels with zero weights on the base ones - the packing of a block that covers
    // several groups, with one group.
    g.grp_mode = 2;
    g.gsp = 2;
    base_k = 2 * d.c_base;
    c_cond = d.c_in;
  }
  if (base_k % (cps * g.ch) || c_cond % (cps * g.ch)) return false;
  if (d.c_out % kBn) return false;
  g.n_cb = d.c_out / kBn;
  g.cps = cps;
  g.stages[0] = base_k / (cps * g.ch);
  g.stages[1] = c_cond / (cps * g.ch);
  // 32-bit byte offsets inside the kernel
  return (long long)d.n_max * d.h * d.w * xps * g.elem_bytes < (1ll << 31);
}

// Plan with stages of `cps` chunks; ok = 0 where the shape does not allow them.  *cost: estimated clocks.
RowsPlan plan_cps(const cg_conv_desc& d, int n_cu, int cps, int max_pf, double* cost) {
  RowsPlan g{};
  int base_k, c_cond;
  if (!plan_walk(d, cps, g, base_k, c_cond)) return g;
  const int ho = (d.h + 2 * d.pad - 3) / d.stride + 1, wo = (d.w + 2 * d.pad - 3) / d.stride + 1;
  // 16-bit row numbers inside the kernel
  if ((long long)d.n_max * ho * wo >= (1ll << 30)) return g;
  if ((long long)d.n_max * (d.h + 2 * d.pad) >= 65536 || (long long)d.n_max * ho >= 65536) return g;
  g.taps = 9;
  g.hp = d.h + 2 * d.pad;
  g.logp = 4;
  while ((1 << g.logp) < d.w + d.pad) ++g.logp;
  if ((1 << g.logp) == d.w + d.pad && d.pad) ++g.logp;   // keep a zero slot after the last column
  if (g.logp > 8) return g;
  const int S = g.stages[0] + g.stages[1], ks = 9 * cps / 2, wb = ks * 2048;
  const long long rows = (long long)d.n_max * ho;
  // which operand an XCD's L2 should see whole: the heavier one
  g.xcd_cb = (g.n_cb % 8 == 0 && 9ll * d.c_in * d.c_out > (long long)d.n_max * d.h * d.w * d.c_in) ? 1 : 0;
  if (g.n_cb > 65536 && !g.xcd_cb) return g;             // (div16)
  long long slots = n_cu / g.n_cb;
  if (slots < 1) slots = 1;
  if (slots > rows) slots = rows;
  g.n_slots = (int)slots;
  const int slot_rows = (int)((rows + slots - 1) / slots);
  // patch rows of a tile of t output rows, maximum over the rows a tile may start at
  auto patch_rows = [&](int t) {
    int pr = 0;
    for (int r0 = 0; r0 < ho; ++r0) {
      const int r1 = r0 + t - 1;
      const int here = (r1 / ho) * g.hp + (r1 % ho) * d.stride - r0 * d.stride + 3;
      if (here > pr) pr = here;
    }
    return pr;
  };
  // Fragments per wavefront and their shape, rows per tile and buffers: the choice with the least estimated time, in clocks.
  // The estimate follows what was measured for 4000 plans of 257 layers (bf16 and int8, 64 to 512 channels, firing rates of
  // 0.1 to 0.6, clustered and not): the plan it picks takes 0.5 % longer than the best one in the mean and 6 % at most.
  // (Constants fitted to half of the layers: 0.7 % and 10 % on the other half.  The ones before, which counted too little
  // for an output: 3.0 % and 32 %.)
  //   A K step costs 64 clocks of the matrix cores per fragment on one SIMD, half as much again where a lone wavefront has to
  //   wait for its LDS reads, and an eighth less where a wavefront reads the weights for two fragments; as wavefronts run
  //   free, a SIMD with fewer fragments than the fullest one helps by a third;
  //   a conditional stage costs the share of the fragments that hold a fired pixel, by the fragment's height, and some;
  //   the vector-memory path serves a line every two clocks; with two or three buffers a stage's latency shows;
  //   gate and output cost 2800 clocks a fragment, 5800 where it is written twice (two fragments to a wavefront), fragments
  //   of four columns a little more (more lines), and a tile 3500.
  // Two fragments pay with many channels and tiles that fill them: 512 at 28x28, 12 images 43 us against 50; 256 at 14x14, 256
  // images 61 and 61; 128 at 28x28, 128 images 47 and 41.
  const int shuf_bytes = shuffle_bytes(d);
  // stages that are walked with one half of the block's channels of several groups
  const int cpg = d.groups > 1 ? d.c_out / d.groups : 0;
  const bool halved = g.grp_mode == 2 && cpg > 0 && cpg <= 32 && d.c_base % (cps * g.ch) == 0;
  const double h0 = halved ? 0.55 : 1.0, h1 = halved && cpg == 32 ? 1.0 - 0.9 / d.groups : 1.0;
  const bool pairs = !halved && !d.shuffle && near_outputs(d.c_out, d.out_dtype, 1) && (d.out_dtype == CG_BF16 || (d.out_dtype == CG_I8 && d.rq_shift >= 2));
  double best = 1e30;
  const bool wide = d.in_dtype == CG_BF16 && d.out_dtype == CG_BF16 && !d.shuffle && cps == 4 && near_outputs(d.c_out, CG_BF16, 2);
  for (int pf = 1; pf <= (wide ? max_pf : 1); ++pf)
  for (int fwl = -1; fwl <= 5; ++fwl) {
    if (fwl == 0 || fwl == 1) continue;                    // (16 and 32 rows of one or two columns: no better than a run)
    const int fh = fwl < 0 ? 1 : 32 >> fwl, nfc = fwl < 0 ? 1 : (wo + (1 << fwl) - 1) >> fwl;
    const int frags_max = kCw * pf;
    if (nfc > frags_max) continue;
    const int tmax = fwl < 0 ? 32 * frags_max / wo : frags_max / nfc * fh;
    if (tmax < 1) continue;
    const double beta = fwl < 0 ? (wo >= 32 ? 0.85 : wo >= 16 ? 0.72 : 0.53) : fh == 1 ? 0.67 : fh == 8 ? 0.64 : 0.59;
    const int step = fwl < 0 ? 1 : fh;
    for (int t = tmax; t >= step && 4 * t >= tmax; t -= step) {
      const int pr = patch_rows(t);
      const bool paired = pairs && pf == 1 && t >= slot_rows && tile_fragments(t, fwl, nfc, wo) <= kCw / 2;
      const long long psz = (((long long)pr << g.logp) * 16 * cps + 1023) / 1024 * 1024;
      if (psz / 1024 > kMaxPatchLoads * kLw) continue;
      for (int resident = 1; resident >= 0; --resident) {
        const long long fixed = kTabBytes + shuf_bytes + (resident ? (long long)S * wb : 0);
        const long long per = psz + (resident ? 0 : wb);
        int nb = (int)((kLds - fixed) / per);
        if (fixed > kLds || nb < 2) continue;
        if (nb > 8) nb = 8;
        const double lines = (double)(pr * (d.w < (1 << g.logp) ? d.w : (1 << g.logp))) + (resident ? 0 : wb / 128.0);
        const double stream = 2.0 * lines + (nb == 2 ? 910.0 : nb == 3 ? 150.0 : 0.0);
        // (two wavefronts to a fragment hide some of each other's waits; counted for one tile, since of several the next ones hide them)
        auto tile = [&](int r) {
          const int frags = tile_fragments(r, fwl, nfc, wo);
          const double per_simd = 0.67 * ((frags + 3) / 4) + 0.33 * frags / 4.0;
          const double mm = ks * 64.0 * per_simd * (frags > 4 ? 1.10 : paired ? 1.30 : 1.55) * (frags > kCw ? 0.87 : 1.0), mc = mm * (beta + 0.15);
          return g.stages[0] * (mm * h0 > stream ? mm * h0 : stream) + g.stages[1] * (mc * h1 > stream ? mc * h1 : stream) + 3500.0 +
                 per_simd * (pf == 2 ? 5800.0 : paired ? 1700.0 : 2800.0) * (fwl == 2 ? 1.07 : 1.0);
        };
        const double c = (slot_rows / t) * tile(t) + (slot_rows % t ? tile(slot_rows % t) : 0.0) + 1500.0 +
                         (resident ? S * wb / 60.0 : 0.0);
        if (c < best) {
          best = c;
          g.pf = pf;
          g.fwl = fwl;
          g.nfc = nfc;
          g.tr = t;
          g.pr = pr;
          g.n_pl = (int)(psz / 1024);
          g.nb = nb;
          g.resident = resident;
          g.psz = (int)psz;
          g.pstr = (int)per;
          g.ok = 1;
        }
      }
    }
  }
  if (!g.ok) return g;
  int off = g.nb * g.pstr;
  g.wres = g.resident ? off : -1;
  if (g.resident) off += S * wb;
  g.shuf = off;
  g.shuf_bytes = shuf_bytes;
  off += shuf_bytes;
  g.tabs = off;
  g.lds_bytes = off + kTabBytes;
  g.wpk_base_bytes = (size_t)g.n_cb * g.stages[0] * wb;
  g.wpk_cond_bytes = (size_t)g.n_cb * g.stages[1] * wb;
  g.cost = best;
  *cost = best;
  return g;
}

}  // namespace

RowsPlan rows_plan(const cg_conv_desc& d, int n_cu, int cps, int max_pf) {
  RowsPlan none{};
  if (d.in_dtype != CG_BF16 && d.in_dtype != CG_I8) return none;
  if (d.kh != 3 || d.kw != 3 || d.stride < 1 || d.stride > 2 || d.pad > 1) return none;
  double c4 = 1e30, c2 = 1e30;
  const RowsPlan a = cps == 2 ? none : plan_cps(d, n_cu, 4, max_pf, &c4);
  const RowsPlan b = cps == 4 ? none : plan_cps(d, n_cu, 2, max_pf, &c2);
  return a.ok && (!b.ok || c4 <= c2) ? a : b;
}

RowsPlan point_plan(const cg_conv_desc& d, int n_cu) {
  RowsPlan g{};
  int base_k, c_cond;
  if ((d.in_dtype != CG_BF16 && d.in_dtype != CG_I8) || d.kh != 1 || d.kw != 1 || d.stride != 1 || d.pad != 0) return g;
  if (!plan_walk(d, 8, g, base_k, c_cond)) {
    g = RowsPlan{};
    if (!plan_walk(d, 4, g, base_k, c_cond)) {
      g = RowsPlan{};
      if (!plan_walk(d, 2, g, base_k, c_cond)) return g;
    }
  }
  const int wb = g.cps / 2 * 2048;
  g.taps = 1;
  g.pf = g.nfc = g.hp = 1;
  g.fwl = -1;
  const long long px = (long long)d.n_max * d.h * d.w;
  if (px >= (1ll << 30)) return g;
  g.xcd_cb = g.n_cb % 8 == 0 && d.c_out > px ? 1 : 0;
  if (g.n_cb > 65536 && !g.xcd_cb) return g;
  long long slots = n_cu / g.n_cb;
  if (slots < 1) slots = 1;
  if (slots > (px + 31) / 32) slots = (px + 31) / 32;
  g.n_slots = (int)slots;
  // A workgroup's pixels in as few tiles of at most 256 as they take, all of the same size.
  const long long each = (px + slots - 1) / slots, tiles = (each + 32 * kCw - 1) / (32 * kCw);
  g.tr = (int)((each + tiles - 1) / tiles);
  const int S = g.stages[0] + g.stages[1];
  g.psz = (g.tr * 16 * g.cps + 1023) / 1024 * 1024;
  g.n_pl = g.psz / 1024;
  g.shuf_bytes = shuffle_bytes(d);
  const int room = kLds - kTabBytes - g.shuf_bytes;
  // weights that leave room for four patches stay in LDS
  g.resident = S * wb + 4 * g.psz <= room ? 1 : 0;
  g.pstr = g.psz + (g.resident ? 0 : wb);
  g.nb = (room - (g.resident ? S * wb : 0)) / g.pstr;
  if (g.nb < 2) return g;
  if (g.nb > 8) g.nb = 8;
  int off = g.nb * g.pstr;
  g.wres = g.resident ? off : -1;
  if (g.resident) off += S * wb;
  g.shuf = off;
  off += g.shuf_bytes;
  g.tabs = off;
  g.lds_bytes = off + kTabBytes;
  g.wpk_base_bytes = (size_t)g.n_cb * g.stages[0] * wb;
  g.wpk_cond_bytes = (size_t)g.n_cb * g.stages[1] * wb;
  // The estimated time, with the call's host part, in clocks of 2.25 GHz, fitted to 40 layers of 100 to 100000 pixels (4 % off, 10 % at most): a stage
  // takes its products, its lines of memory or, where it is short, 980 clocks of latency; a conditional one half of that.  (Fitted before layers of many stages
  // had them loaded in turn, whose time is up to 40 % shorter than this.)
  g.cost = 8450.0 + (g.resident ? S * wb / 60.0 : 0.0);
  for (long long left = each; left > 0; left -= g.tr) {
    const long long here = left < g.tr ? left : g.tr, frags = (here + 31) / 32;
    const double per_simd = 0.67 * ((frags + 3) / 4) + 0.33 * frags / 4.0;
    const double mm = g.cps / 2 * 102.0 * per_simd * (frags <= 4 ? 1.55 : 1.10);
    const double stream = 7.86 * (here * 16 * g.cps + (g.resident ? 0 : wb)) / 128.0;
    g.cost += (g.stages[0] + 0.51 * g.stages[1]) * std::max(984.0, std::max(mm, stream)) + 2180.0 + 2075.0 * per_simd;
  }
  g.ok = 1;
  return g;
}

hipError_t launch_rows_pack(const RowsPlan& g, const Params& p, void* wpk_base, void* wpk_cond, hipStream_t s) {
  for (int ph = 0; ph < 2; ++ph) {
    if (g.stages[ph] == 0) continue;
    const long long total = (long long)g.n_cb * g.stages[ph] * (g.taps * g.cps / 2) * 2 * 64;
    const unsigned blocks = (unsigned)((total + 255) / 256);
    hipLaunchKernelGGL(pack_rows_kernel, dim3(blocks), dim3(256), 0, s, (const char*)(ph ? p.w_cond : p.w_base),
                       (char*)(ph ? wpk_cond : wpk_base), ph ? p.c_cond : p.c_base, g.elem_bytes, g.ch, g.cps,
                       g.stages[ph], total, g.grp_mode == 2 ? 1 : 0, ph, p.c_base, p.cpg, g.taps);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_rows(const RowsPlan& g, const Params& p, const void* w0, const void* w1, hipStream_t s) {
  RowsArgs a{};
  a.x = (const char*)p.x;
  a.w0 = (const char*)w0;
  a.w1 = (const char*)w1;
  a.tab = (const char*)p.thr_f;
  a.y = (char*)p.y;
  a.residual = (const char*)p.residual;
  a.bitmap = p.bitmap;
  a.chan_mask = p.chan_mask;
  a.clear = p.clear_total ? p.total : nullptr;
  a.gave_up = p.gave_up;
  a.magic_hp = magic16(g.hp);
  a.magic_ho = magic16(p.ho);
  a.magic_wo = magic16(p.wo);
  a.magic_ncb = magic16(g.n_cb);
  a.n = p.n;
  a.h = p.h;
  a.w = p.w;
  a.ho = p.ho;
  a.wo = g.taps == 1 ? 1 : p.wo;
  a.hp = g.taps == 1 ? p.ho * p.wo : g.hp;
  a.stride = p.stride;
  a.pad = p.pad;
  a.xps = (int)p.x_pixel_stride * g.elem_bytes;
  a.x_bytes = (unsigned)((((long long)p.n * p.h * p.w - 1) * p.x_pixel_stride + p.c_in) * g.elem_bytes);
  const int rows = g.taps == 1 ? p.n * p.ho * p.wo : p.n * p.ho;
  a.full = rows / (g.n_slots * g.tr);
  const int tail = rows - a.full * g.n_slots * g.tr;
  a.rows_per = tail / g.n_slots;
  a.rows_more = tail % g.n_slots;
  a.tr = g.tr;
  a.logp = g.logp;
  a.n_pl = g.n_pl;
  a.s0 = g.stages[0];
  a.s = g.stages[0] + (p.gated && !p.gate_only ? g.stages[1] : 0);
  a.nb = g.nb;
  a.pstr = g.pstr;
  a.psz = g.psz;
  a.wres = g.wres;
  a.tabs = g.tabs;
  a.shuf = g.shuf;
  a.fwl = g.fwl;
  a.nfc = g.nfc;
  a.magic_nfc = magic16(g.nfc);
  a.n_cb = g.n_cb;
  a.n_slots = g.n_slots;
  a.xcd_cb = g.xcd_cb;
  a.per_xcd = (g.n_slots * g.n_cb + 7) / 8;
  a.grp_mode = p.groups > 1 ? 1 : 0;
  a.grp_step = p.cpg;
  a.base_chn = p.c_base * g.elem_bytes;
  a.gap_chn = g.grp_mode == 2 ? 0 : p.c_base * g.elem_bytes;
  a.words = p.words;
  a.tab_stride = (int)p.table_stride;
  a.c_out = p.c_out;
  a.cpg = p.cpg;
  a.groups = p.groups;
  // (without grouping a padded base group is the only case of zero weights, and both halves of the channels share it)
  a.spg = g.grp_mode == 2 && p.groups > 1 && p.cpg <= 32 && p.c_base % (g.cps * g.ch) == 0 ? p.c_base / (g.cps * g.ch) : 0;
  a.rq_shift = p.rq_shift;
  a.rq_res_mult = p.rq_res_mult;
  const bool shuf2 = p.shuffle && g.shuf_bytes > 0, near = near_outputs(p.c_out, p.out_dtype, g.pf);
  a.flags = (p.gated ? kGated : 0u) | (p.gate_only ? kGateOnly : 0u) | (p.two_sided ? kTwoSided : 0u) |
            ((p.epilogue & CG_EPI_AFFINE) && p.in_dtype != CG_I8 ? kAffine : 0u) | ((p.epilogue & CG_EPI_RELU) ? kRelu : 0u) |
            ((p.epilogue & CG_EPI_RESIDUAL) ? kResidual : 0u) | (p.in_dtype != CG_I8 && (p.one_pair || !(p.epilogue & CG_EPI_AFFINE)) ? kOnePair : 0u) | (p.fit32 ? kFit32 : 0u) |
            (near && (p.out_dtype == CG_BF16 || (p.out_dtype == CG_I8 && p.rq_shift >= 2)) && (!p.shuffle || shuf2) ? kFast : 0u) | (shuf2 ? kShuf2 : 0u) |
            (near && !p.shuffle && (p.out_dtype == CG_F32 || p.out_dtype == CG_I32) ? kFourBytes : 0u);
  const bool pairs = (a.flags & kFast) && !p.shuffle && !a.spg && g.pf == 1 && g.taps == 9 && tile_fragments(g.tr, g.fwl, g.nfc, p.wo) <= kCw / 2;
  if (pairs) a.flags |= kPairs;
  // Loading wavefronts of 1x1 layers take whole stages in turn where a workgroup has enough of them behind its first ones to make up for a stage that one
  // wavefront brings more slowly than four, and where a tile's time is not mostly its outputs'.  With the stages shared and in turn, us:
  //   More than four buffers, from eight stages to a tile and three rounds of the buffers on: nine stages (int8 192 to 512 channels at 14x14, 128 images)
  // 22.8 and 20.6; twelve, bf16 192 to 1024 at 7x7, 128 images (three rounds) 16.8 and 13.6; 28, 448 to 256 at 28x28, 64 images 57.4 and 35.0; but four, 256 to
  // 512 at 28x28, 64 images 31.3 and 32.1, 64 to 256 at 52x52, 193 images 98.6 and 105.2.
  //   Four buffers, all that fit of stages of 30 KB and more, from twelve rounds on, x and y in the Infinity Cache / beyond it: bf16 from sixteen stages on, 1024 to
  // 1024 at 14x14, 64 images 46.1 and 43.1 / 49.0 and 48.8; int8 from eight on, 1024 to 1024, 128 images 48.7 and 47.7 / 48.1 and 47.9.  bf16 of fewer lose where x
  // and y come from beyond it, and, with a residual, which is read at a tile's start as its first stages are, everywhere: twelve stages, 768 to 512 at 28x28,
  // 32 images 37.7 and 36.4 / 40.4 and 42.0; eight, 512 to 1024 at 14x14, 106 images 44.8 and 44.8 / 44.5 and 45.8, with a residual 45.3 and 47.8 / 50.7 and
  // 52.8.  (Sixteen stages and more gain with fewer rounds too: 1024 to 256 at 28x28, 32 images, four rounds 26.0 and 24.8.)
  //   Not with fewer buffers (4096 to 4096, 1024 pixels 48 and 51).
  const int stages = (a.full + (tail > 0 ? 1 : 0)) * a.s;
  const int least = a.nb > kLw || p.in_dtype == CG_I8 ? 8 : 16;
  if (g.taps == 1 && a.nb >= kLw && a.s >= least && stages >= (a.nb > kLw ? 3 : 12) * a.nb) a.flags |= kTurns;
  // rows of the patch lie in the banks of others: runs of 32 pixels over several of them, fragments of up to 8 columns (counted for widths of 2
  // to 56: never more passes than with the fixed bit; from 32 columns on and at stride 2 there are)
  const bool narrow = p.stride == 1 && (g.fwl < 0 ? p.wo < 32 : g.fwl <= 3);
  a.bit = pairs && narrow && (2 << g.logp) <= kLw * 64 / g.cps ? g.logp : 3;
  return p.in_dtype == CG_I8 ? launch_rows_type<I8Rows>(g, p, a, s) : launch_rows_type<Bf16Rows>(g, p, a, s);
}

}  // namespace cg
