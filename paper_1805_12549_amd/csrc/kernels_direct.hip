// Small-tile matrix-core kernel of the gated convolution (bf16, int8 and fp32 MFMA, 16x16 blocks):
// no LDS staging, the operands go from global memory straight into registers.
//
// It takes what the two tiled kernels are no good at: layers with few output pixels (one image, deep
// layers), channel counts and groups that are not multiples of 64 channels / of whole K stages, strided 1x1 layers and
// fp32.  A tile is PF fragments of 16 output pixels by NH sixteens of output channels; the product is taken transposed
// (weights are the row operand), so a lane ends up with 4 consecutive channels of one pixel per sixteen (Eq. 1 and the
// gate work on registers).
//
// What bounds it is the vector-memory path of a compute unit, which serves the 64-byte pieces of the
// pixel operand in 50 clocks a KB and the linear weights in 12 to 30 (32-byte pieces,
// what 32x32 blocks would fetch, in 80), and where there is little to fetch the chain of latencies: 1.5 us from
// one kernel's end to the next one's first instruction, 0.2 for the arguments, 0.9 for the operands, 5 clocks for every
// instruction that waits for the one before.  Two forms:
//
//   whole   a wavefront owns a tile and walks all of K; the conditional path is walked only if one of
//           the tile's gates fired.  No barrier; LDS for its own tables only.
//   SPLIT   a workgroup of 2..8 wavefronts owns one tile and splits K: some wavefronts walk the base
//           path, the others the conditional path, all at once; the partial sums meet in LDS.  No phase waits for the
//           gate.  The weights are asked for first, then the pixels' addresses are formed; tables and residual are on their way
//           while the products are taken.
//
// Small tiles (down to 16 x 16) are what fills the chip when there are few pixels.  In the form before the tile was 32 x 64,
// K was split over up to 16 workgroups as well and a second kernel added their sums up: 4.4 us inside the first kernel, of which
// 0.7 went into divisions, 1.6 between them and 2.8 inside the second.  In a graph, scale/shift and residual, us, before and now:
// bf16 64 channels at 56x56, one image 6.7 -> 5.8; 128 at 28x28 10.0 -> 6.0; 256 at 14x14 10.3 -> 7.1; 512 at 7x7 10.8 -> 8.8;
// int8 256 at 14x14 9.2 -> 5.8; bf16 96 to 80 at 45x33, five images 11.8 -> 7.9.  Sixteen wavefronts to a tile measured
// 4 to 40 % slower than eight (128 registers to a wavefront are not enough for the larger tiles), K split over two or four
// workgroups as well 20 to 50 % slower at one to four images.
//
// (Those are with an end of branches on lanes' values and a K loop whose waits were for every load in flight.  Scalar offsets where a K step lies inside
// one tap, waits for one batch at a time, sums that meet in straight code and an end shared by up to four wavefronts a unit take 60 layers of
// 3.4 to 28 us to 0.81 of that time: int8 256 at 14x14 through the binding 5.4 -> 4.1, 96 to 80 at 45x33 7.8 -> 6.6.)
//
// K is walked in steps of four units, unit u = tap * chunks + chunk, a unit being one 16-byte channel
// chunk of one tap; lane group l/16 supplies unit 4k + l/16.  Padding (taps outside the image, units past
// the last) is an out-of-range buffer load, which returns zeros.  In the chunk in which a base group ends the
// packed weights are zero for the other path's channels; where a float sum is a NaN there, it is formed again from the path's own channels,
// in the same order (0 * inf would otherwise reach it).
#include <algorithm>
#include <type_traits>

#include "cg_mfma_common.h"
#include "point_piece.h"

namespace cg {

namespace {

struct Bf16Direct {
  using Base = Bf16Traits;
  using acc4 = f32x4;
  using acc_t = float;
  static constexpr int kCh = 8, kParts = 1;
  static __device__ __forceinline__ acc4 mma(int, i32x4 rows, i32x4 cols, acc4 c) { return Bf16Traits::mfma(rows, cols, c); }
  static __device__ __forceinline__ float element(i32x4 v, int e) { return __uint_as_float(e & 1 ? (unsigned)v[e >> 1] & 0xffff0000u : (unsigned)v[e >> 1] << 16); }
};

struct I8Direct {
  using Base = I8Traits;
  using acc4 = i32x4;
  using acc_t = int32_t;
  static constexpr int kCh = 16, kParts = 1;
  static __device__ __forceinline__ acc4 mma(int, i32x4 rows, i32x4 cols, acc4 c) { return I8Traits::mfma(rows, cols, c); }
};

// fp32: a 16-byte chunk is four channels; the e-th elements of the four lane groups' chunks make one
// 16x16x4 product (the order of the channels inside a K step is free as long as both operands share it)
struct F32Traits {
  using acc_t = float;
  static constexpr int kDtype = CG_F32;
  static __device__ __forceinline__ bool fires(float v, float lo, float hi) { return v >= lo && v <= hi; }
};
struct F32Direct {
  using Base = F32Traits;
  using acc4 = f32x4;
  using acc_t = float;
  static constexpr int kCh = 4, kParts = 4;
  static __device__ __forceinline__ float element(i32x4 v, int e) { return __int_as_float(v[e]); }
  static __device__ __forceinline__ acc4 mma(int e, i32x4 rows, i32x4 cols, acc4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(__int_as_float(rows[e]), __int_as_float(cols[e]), c, 0, 0, 0);
  }
};

__device__ __forceinline__ int bits_of(float f) { return __float_as_int(f); }
__device__ __forceinline__ int bits_of(int v) { return v; }
__device__ __forceinline__ void set_bits(int b, float& f) { f = __int_as_float(b); }
__device__ __forceinline__ void set_bits(int b, int& v) { v = b; }

// What the kernels read, in one piece: a wavefront's first instructions load all of it and wait once (argument by argument, in the
// order of use, the waits alone took over a microsecond of a six-microsecond kernel).
struct DirectArgs {
  const void* x;             // less x_bias: the offset of tap (0,0) of a pixel on the image's edge is not negative
  const char *w0, *w1;
  int x_bytes, x_bias;       // of the buffer from there on
  int m_total, h, w, xps, rowb;
  Div wo, ho, cblk, nq0, nq1, cpg;
  int n_wo, n_ho, n_cblk, n_cpg;
  int stride, pad, taps, chunks0, chunks1, total_chunks, gap_len, groups, c_base, ch_log;
  int ks0, ks1, waves, nwb, per_xcd, n_wgs;
  int kq0, kr0, kq1, kr1;    // K steps of a part of either phase: kq, the first kr parts one more
  unsigned flags;
  // the end of the layer
  const char* tab;           // per-channel tables, tab_stride bytes apart (see cg_internal.h)
  void* y;
  const void* residual;
  uint32_t* bitmap;
  const uint32_t* chan_mask;
  uint32_t* total;
  Div hw;
  int tab_stride, c_out, words, rq_shift, rq_res_mult;
};
enum : unsigned {
  kRelu = 1u, kAffine = 2u, kResidual = 4u,       // as CG_EPI_*
  kGated = 8u, kGateOnly = 16u, kClear = 32u, kShuffle = 64u,
  kOut4 = 128u,                                   // 4-byte outputs (CG_F32 / CG_I32)
  kStraddle = 256u,                               // the base group ends inside a chunk
  kFit32 = 1024u,                                 // int8 -> int8: the requantisation fits 32 bits
};

__device__ __forceinline__ void load_args(const DirectArgs& a) {
  asm volatile("" ::"s"(a.x), "s"(a.w0), "s"(a.w1), "s"(a.x_bytes), "s"(a.x_bias), "s"(a.m_total), "s"(a.h), "s"(a.w), "s"(a.xps),
               "s"(a.rowb), "s"(a.wo.m), "s"(a.wo.s), "s"(a.ho.m), "s"(a.ho.s), "s"(a.cblk.m), "s"(a.cblk.s),
               "s"(a.n_wo), "s"(a.n_ho), "s"(a.n_cblk), "s"(a.stride), "s"(a.pad), "s"(a.taps));
  asm volatile("" ::"s"(a.nq0.m), "s"(a.nq0.s), "s"(a.nq1.m), "s"(a.nq1.s), "s"(a.chunks0), "s"(a.chunks1), "s"(a.total_chunks),
               "s"(a.gap_len), "s"(a.ks0), "s"(a.ks1), "s"(a.waves), "s"(a.nwb), "s"(a.per_xcd), "s"(a.n_wgs), "s"(a.kq0), "s"(a.kr0),
               "s"(a.kq1), "s"(a.kr1), "s"(a.flags));
}
__device__ __forceinline__ void load_rest(const DirectArgs& a) {
  asm volatile("" ::"s"(a.tab), "s"(a.y), "s"(a.residual), "s"(a.bitmap), "s"(a.chan_mask), "s"(a.tab_stride), "s"(a.c_out),
               "s"(a.words), "s"(a.rq_shift), "s"(a.rq_res_mult));
}

// The end of the layer is a few wavefronts' instructions with nothing beside them, each of them some 6 clocks, and the first time through also the
// instruction cache's misses (700 of 2100 clocks).  So it is short code without a branch on a lane's value: a lane has Q = 1, 2 or 4 consecutive
// channels of a pixel, as few as there are wavefronts for; choices by decision are selections of bits; a flag of the layer is a branch that all lanes
// take.  (As conditional expressions and stores the sums of eight wavefronts alone took 2400 clocks, a store to a channel 1500.)

typedef __attribute__((ext_vector_type(2))) int i32x2;
template <int Q>
using ints = std::conditional_t<Q == 1, int, std::conditional_t<Q == 2, i32x2, i32x4>>;
template <int Q>
__device__ __forceinline__ void take(const void* from, int (&v)[Q]) {
  const ints<Q> t = *(const ints<Q>*)from;
  if constexpr (Q == 1) {
    v[0] = t;
  } else {
#pragma unroll
    for (int e = 0; e < Q; ++e) v[e] = t[e];
  }
}

constexpr int kTabs = 7;                         // tables that a layer's end reads

// The per-channel tables of a lane's channels.  (int8 layers whose requantisation fits 32 bits: hi and h1 = bounds of the sum, s1 = what is added.)
template <typename Base, int Q>
struct Tab {
  int lo[Q], hi[Q], s0[Q], h0[Q], s1[Q], h1[Q];  // int8 layers: s0 = mult0, h0 = mult1, s1 = bias
  // from a copy of the tables' sixteen channels, 64 bytes a table; what a flag leaves out is not used
  __device__ __forceinline__ void take_all(const DirectArgs& a, const char* q) {
    const bool fit = Base::kDtype == CG_I8 && (a.flags & kFit32);
    take(q, lo);
    take(q + 64, hi);
    take(q + 128, s0);
    take(q + 192, h0);
    take(q + (fit ? 320 : 256), s1);
    take(q + (fit ? 384 : 320), h1);
  }
};

// the bits of a where m has ones, of b elsewhere
__device__ __forceinline__ int select_bits(int m, int a, int b) { return (a & m) | (b & ~m); }
// all ones where bit e of d is set
__device__ __forceinline__ int ones_if(unsigned d, int e) { return (int)(d << (31 - e)) >> 31; }

// the larger one; NaN as the second: the first
__device__ __forceinline__ float max_of(float a, float b) {
  float r;
  asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ int med3(int v, int lo, int hi) {
  int r;
  asm("v_med3_i32 %0, %1, %2, %3" : "=v"(r) : "v"(v), "v"(lo), "v"(hi));
  return r;
}

// decisions of a lane's channels from their base sums
template <typename Base, int Q, typename acc_t>
__device__ __forceinline__ unsigned gate_of(const acc_t (&s)[Q], const int (&lo)[Q], const int (&hi)[Q]) {
  unsigned d = 0u;
#pragma unroll
  for (int e = 0; e < Q; ++e) {
    bool f;
    if constexpr (Base::kDtype == CG_I8)
      f = Base::fires(s[e], lo[e], 0);
    else
      f = Base::fires(s[e], __int_as_float(lo[e]), __int_as_float(hi[e]));
    d |= f ? 1u << e : 0u;
  }
  return d;
}
// the decisions that there are: of channels before the last one, of pixels before the last one
template <int Q>
__device__ __forceinline__ unsigned there_are(const DirectArgs& a, int co0, bool pixel) {
  return pixel ? (1u << med3(a.c_out - co0, 0, Q)) - 1u : 0u;
}

// Consecutive channels co0.. of an output pixel are read and stored in one piece where c_out allows, else one by one.
template <int Q>
__device__ __forceinline__ bool one_piece(const DirectArgs& a) { return !((a.c_out & (Q - 1)) || (a.flags & kShuffle)); }
__device__ __forceinline__ long long element_at(const DirectArgs& a, long long m, int co) {
  if (!(a.flags & kShuffle)) return m * a.c_out + co;
  const int grp = (int)quot(co, a.cpg);
  return m * a.c_out + (co - grp * a.n_cpg) * a.groups + grp;
}

// the residual of those channels, as it lies in memory (fetched ahead of the sums: its latency is 0.5 us of a finish)
template <typename Base, int Q>
__device__ __forceinline__ i32x4 load_residual(const DirectArgs& a, int co0, long long m, bool valid) {
  i32x4 r = {0, 0, 0, 0};
  if (!(a.flags & kResidual) || !valid || co0 >= a.c_out) return r;
  constexpr bool I8 = Base::kDtype == CG_I8;
  if (Q > 1 && one_piece<Q>(a)) {
    const long long o = m * a.c_out + co0;
    if constexpr (I8) {
      if constexpr (Q == 4)
        r[0] = *(const int*)((const int8_t*)a.residual + o);
      else
        r[0] = *(const uint16_t*)((const int8_t*)a.residual + o);
    } else if (a.flags & kOut4) {
      int v[Q];
      take((const float*)a.residual + o, v);
#pragma unroll
      for (int e = 0; e < Q; ++e) r[e] = v[e];
    } else {
      r[0] = *(const int*)((const uint16_t*)a.residual + o);
      if constexpr (Q == 4) r[1] = *(const int*)((const uint16_t*)a.residual + o + 2);
    }
    return r;
  }
#pragma unroll
  for (int e = 0; e < Q; ++e)
    if (co0 + e < a.c_out) {
      const long long o = element_at(a, m, co0 + e);
      if constexpr (I8)
        r[0] |= (int)((uint32_t) * ((const uint8_t*)a.residual + o) << (8 * e));
      else if (a.flags & kOut4)
        r[e] = ((const int*)a.residual)[o];
      else
        r[e >> 1] |= (int)((uint32_t)((const uint16_t*)a.residual)[o] << (16 * (e & 1)));
    }
  return r;
}

// where those channels are stored in one piece
template <typename Base>
__device__ __forceinline__ char* y_at(const DirectArgs& a, int co0, long long m) {
  return (char*)a.y + ((m * a.c_out + co0) << ((a.flags & kOut4) ? 2 : Base::kDtype == CG_I8 ? 0 : 1));
}

// Output function (f of Eq. 1) for consecutive channels co0.. of output pixel m: base and conditional sums, decisions in d; to `at` (y_at)
// where they are stored in one piece; nothing is stored where the pixel or the channels are past the end (live).
template <typename Base, int Q, typename acc_t>
__device__ __forceinline__ void finish(const DirectArgs& a, const acc_t (&base)[Q], const acc_t (&cond)[Q], const Tab<Base, Q>& t, i32x4 res, unsigned d,
                                       int co0, long long m, char* at, bool live) {
  acc_t s[Q];
  int on[Q];
#pragma unroll
  for (int e = 0; e < Q; ++e) {
    on[e] = ones_if(d, e);
    acc_t c;
    set_bits(bits_of(cond[e]) & on[e], c);
    s[e] = base[e] + c;
  }
  if (!(a.flags & kGated)) {                     // (a dense layer takes the second pair)
#pragma unroll
    for (int e = 0; e < Q; ++e) on[e] = -1;
  }
  int v[Q];                                      // what is stored, 4-byte outputs
  int packed[2] = {0, 0};                        // narrow ones
  if constexpr (Base::kDtype == CG_I8) {
    const int low = (a.flags & kRelu) ? 0 : -128;
    if (a.flags & kFit32) {                      // (as in the row-tiled kernel)
#pragma unroll
      for (int e = 0; e < Q; ++e) {
        const int q = __mul24(med3(s[e], t.hi[e], t.h1[e]), select_bits(on[e], t.h0[e], t.s0[e])) + t.s1[e] +
                      __mul24((int)(int8_t)((uint32_t)res[0] >> (8 * e)), a.rq_res_mult);
        v[e] = med3(q >> a.rq_shift, low, 127);
      }
    } else if ((a.flags & (kOut4 | kResidual)) == kOut4) {
      const int floor = (a.flags & kRelu) ? 0 : -2147483647 - 1;
#pragma unroll
      for (int e = 0; e < Q; ++e) v[e] = s[e] < floor ? floor : s[e];
    } else {
#pragma unroll
      for (int e = 0; e < Q; ++e) {
        const long long r = (long long)(int8_t)((uint32_t)res[0] >> (8 * e)) * a.rq_res_mult;
        long long q;
        if (a.flags & kOut4) {
          q = (long long)s[e] + r;
          if ((a.flags & kRelu) && q < 0) q = 0;
          q = q > 2147483647ll ? 2147483647ll : q;
          q = q < -2147483648ll ? -2147483648ll : q;
        } else {
          q = (long long)s[e] * select_bits(on[e], t.h0[e], t.s0[e]);
          q += (long long)t.s1[e] * (1ll << a.rq_shift) + r;
          if (a.rq_shift > 0) q = (q + (1ll << (a.rq_shift - 1))) >> a.rq_shift;
          q = q < low ? low : q > 127 ? 127 : q;
        }
        v[e] = (int32_t)q;
      }
    }
#pragma unroll
    for (int e = 0; e < Q; ++e) packed[0] |= (v[e] & 0xff) << (8 * e);
  } else {
    const float relu_lo = (a.flags & kRelu) ? 0.0f : __builtin_nanf("");
    if (a.flags & kAffine) {
#pragma unroll
      for (int e = 0; e < Q; ++e)
        s[e] = fmaf(__int_as_float(select_bits(on[e], t.s1[e], t.s0[e])), s[e], __int_as_float(select_bits(on[e], t.h1[e], t.h0[e])));
    }
    if (a.flags & kResidual) {
      if (a.flags & kOut4) {
#pragma unroll
        for (int e = 0; e < Q; ++e) s[e] += __int_as_float(res[e]);
      } else {
#pragma unroll
        for (int e = 0; e < Q; ++e) s[e] += __uint_as_float(e & 1 ? (unsigned)res[e >> 1] & 0xffff0000u : (unsigned)res[e >> 1] << 16);
      }
    }
#pragma unroll
    for (int e = 0; e < Q; ++e) v[e] = __float_as_int(max_of(s[e], relu_lo));
#pragma unroll
    for (int e = 0; e < Q; ++e) packed[e >> 1] |= (int)((uint32_t)float_to_bf16(__int_as_float(v[e])) << (16 * (e & 1)));
  }
  if (one_piece<Q>(a)) {
    if (a.flags & kOut4) {
      if constexpr (Q == 1) {
        if (live) *(int*)at = v[0];
      } else if constexpr (Q == 2) {
        if (live) *(i32x2*)at = i32x2{v[0], v[1]};
      } else {
        if (live) *(i32x4*)at = i32x4{v[0], v[1], v[2], v[3]};
      }
    } else {
      constexpr int kBytes = Q * (Base::kDtype == CG_I8 ? 1 : 2);
      if constexpr (kBytes == 1) {
        if (live) *(uint8_t*)at = (uint8_t)packed[0];
      } else if constexpr (kBytes == 2) {
        if (live) *(uint16_t*)at = (uint16_t)packed[0];
      } else if constexpr (kBytes == 4) {
        if (live) *(int*)at = packed[0];
      } else {
        if (live) *(i32x2*)at = i32x2{packed[0], packed[1]};
      }
    }
    return;
  }
#pragma unroll
  for (int e = 0; e < Q; ++e)
    if (live && co0 + e < a.c_out) {
      const long long oe = element_at(a, m, co0 + e);
      if (a.flags & kOut4)
        ((int32_t*)a.y)[oe] = v[e];
      else if constexpr (Base::kDtype == CG_I8)
        ((int8_t*)a.y)[oe] = (int8_t)v[e];
      else
        ((uint16_t*)a.y)[oe] = (uint16_t)((unsigned)packed[e >> 1] >> (16 * (e & 1)));
    }
}

// or of a value over the four lane groups, in all of them
__device__ __forceinline__ unsigned or_groups(unsigned v) {
  const auto q = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  v = (unsigned)q[0] | (unsigned)q[1];
  const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return (unsigned)r[0] | (unsigned)r[1];
}

// The sixteen decisions of a pixel from its lanes' (16/Q of them, side by side, the first channels first): in all of them.
template <int Q>
__device__ __forceinline__ unsigned sixteen(unsigned d, int lane) {
  if constexpr (Q == 1) return (unsigned)(__ballot(d != 0u) >> (lane & 48)) & 0xffffu;
  unsigned v = d << ((lane & (16 / Q - 1)) * Q);
  v |= (unsigned)__builtin_amdgcn_mov_dpp((int)v, 0xb1, 0xf, 0xf, true);       // quad_perm [1,0,3,2]
  v |= (unsigned)__builtin_amdgcn_mov_dpp((int)v, 0x4e, 0xf, 0xf, true);       // quad_perm [2,3,0,1]
  if constexpr (Q == 2) v |= (unsigned)__builtin_amdgcn_mov_dpp((int)v, 0x141, 0xf, 0xf, true);      // row_half_mirror
  return v;
}

// The decisions of a lane's channels of pixel m as the channel-wise gate (Sec. 3.2) leaves them
__device__ __forceinline__ unsigned masked(const DirectArgs& a, unsigned d, int co0, long long m) {
  if (a.chan_mask && d) d &= a.chan_mask[(long long)quot((unsigned)m, a.hw) * a.words + (co0 >> 5)] >> (co0 & 31);
  return d;
}

// 8 wavefronts per workgroup at most
constexpr int kMaxSplit = 8;

// UNIFORM: every K step lies inside one tap and on one side of the base group, so that its place in x is the same for all lanes but for the
// chunk (a scalar offset, changed by an addition; the general walk forms each lane group's own with some twenty vector instructions a step).
//
// MIXED: float layers whose blocks cover several channel groups (Sec. 3.3) or whose groups share a chunk; kStraddle: those whose base group ends
// inside a chunk.  The packed
// weights are zero where a channel is not on a row's path, which keeps its finite values out of the row's sum but turns
// an infinity or a NaN into a NaN; a wavefront that ends up with one forms the sum again, from the path's channels
// alone.  No other sum changes by it: pixels beside it, of other images among them, keep their bits.  (The look at the sums costs 1 to 2 %, one at every operand, as it is read, 5 to 7 %.)
template <typename Tr, int PF, int NH, bool SPLIT, bool MIXED, bool UNIFORM>
__device__ __forceinline__ void direct_layer(const DirectArgs& p) {
  using Base = typename Tr::Base;
  using acc4 = typename Tr::acc4;
  using acc_t = typename Tr::acc_t;
  constexpr int NU = PF * NH;                       // units of a tile: (pixel fragment, 16 channels)
  // K steps whose operands are fetched together; two such batches are in flight.  (Two steps instead of one for tiles of four
  // units and more: 133 to 181 registers, one workgroup on a compute unit instead of two, 1 to 7 % slower.)
  constexpr int kU = NU == 1 ? 4 : NU == 2 ? 2 : 1;
  constexpr bool kBlocks = SPLIT ? Base::kDtype != CG_I8 && NU < 8 : Base::kDtype == CG_F32;      // (see `carry`)
  constexpr bool kPair = !SPLIT && Base::kDtype == CG_BF16;                                        // (the same)
  __shared__ __align__(16) i32x4 ex[SPLIT ? kMaxSplit * NU * 64 : 1];     // [wavefront][unit][pixel][four channels, rotated against bank conflicts]
  __shared__ __align__(16) i32x4 tab_at[SPLIT ? (NU < 8 ? (NU == 1 ? 4 : kMaxSplit) * 4 * kTabs : 1) : 4 * NH * 4 * kTabs];    // [wavefront][(whole: sixteen channels)][table][four channels]

  load_args(p);
  load_rest(p);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), nw = p.waves;
  const int lj = lane & 15, lg = lane >> 4;

  // block -> (pixel tile, channel tile): an XCD (block id mod 8) takes a contiguous run of them, so the
  // input of neighbouring tiles is fetched into one L2
  const int id = (int)(blockIdx.x & 7) * p.per_xcd + (int)(blockIdx.x >> 3);
  if (id >= p.n_wgs) return;
  const int pt = (int)quot(id, p.cblk), cbk = id - pt * p.n_cblk;
  const int half0 = cbk * NH;                       // first 16 channels of the tile

  const int m0 = (pt * (SPLIT ? 1 : nw) + (SPLIT ? 0 : wave)) * (16 * PF);
  if (!SPLIT && m0 >= p.m_total) return;
  const bool gated = (p.flags & kGated) != 0, gate_only = (p.flags & kGateOnly) != 0;

  // channel chunks of the two phases for this channel block (see DirectPlan)
  const int bfirst = p.groups > 1 ? ((int)quot((half0 >> 2) * 64, p.cpg) * p.c_base) >> p.ch_log : 0;
  const int gap_s = p.gap_len ? bfirst : 0;

  unsigned xbase[PF];                               // offset of tap (0,0) of this lane's pixels
  unsigned vmask[PF];                               // bit t: tap t of this lane's pixel is inside the image
  auto pixels = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int f = 0; f < PF; ++f) {
      const bool valid = m0 + 16 * f + lj < p.m_total;
      const unsigned mm = valid ? (unsigned)(m0 + 16 * f + lj) : 0u;
      const unsigned q = quot(mm, p.wo);
      const unsigned img = quot(q, p.ho);
      const int hi0 = (int)(q - img * (unsigned)p.n_ho) * p.stride - p.pad, wi0 = (int)(mm - q * (unsigned)p.n_wo) * p.stride - p.pad;
      xbase[f] = (unsigned)(((int)img * p.h + hi0) * p.rowb + wi0 * p.xps + p.x_bias);
      if (p.taps == 9) {
        // rows and columns of the window inside the image, then their products
        unsigned cols = 0u;
#pragma unroll
        for (int t = 0; t < 3; ++t) cols |= (unsigned)(wi0 + t) < (unsigned)p.w ? 1u << t : 0u;
        unsigned v = 0u;
#pragma unroll
        for (int t = 0; t < 3; ++t) v |= (unsigned)(hi0 + t) < (unsigned)p.h ? cols << (3 * t) : 0u;
        vmask[f] = valid ? v : 0u;
      } else {
        vmask[f] = valid ? 1u : 0u;
      }
    }
  };
  const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc((void*)p.x, (short)0, p.x_bytes, 0x00027000);
  constexpr unsigned kOut = 0x80000000u;            // an offset beyond any x (the plan keeps x below 1 GiB)

  // How float sums are added up: a sum is rounded the more, the more sums it passes through, and a layer's error against 64 bits is to be no
  // larger than it was when tiles were 32 x 64, of few of which K was split over up to sixteen workgroups as well.
  //   A split, and fp32 sums of the whole form: blocks of two K steps to an accumulator, which are added up in this wavefront's part of
  // `ex`.  Error against 64 bits, rms, relative, as one chain and in blocks: fp32 1x1, 192 to 64 channels at 42x45 stride 2, 67 images (whole) 1.43e-7 and
  // 0.88e-7; 256 to 1664, 1011 pixels (whole) 1.82e-7 and 0.94e-7; 192 to 192 at 3x3, 6x62, 3 images (split) 1.20e-7 in blocks of four, 1.05e-7 of two.
  // It costs the whole form 2 % in the mean of 46 layers (16.9 -> 17.4 us, 18.9 -> 19.6; two of them, tiles of eight units, 24.4 -> 26.9), a
  // split 1 to 3 %.  A split's tiles of eight units have no registers for it (96 to 80 at 45x33 8.6 -> 11.2 us); a wavefront has a chain over its share.
  //   bf16 sums of the whole form, whose K steps are one product each: the base path's even and odd steps by themselves, the odd ones in the
  // registers of the conditional sums, which costs one addition (1 %).  Dense 1x1, 640 to 144 channels, 16306 pixels 1.08e-7 -> 0.78e-7, as much as with K
  // split over two wavefronts.  (In blocks of four or eight steps as above 2 to 3 % slower in the mean of 80 layers, 19 % at most.)
  // (Layers whose K was split over four, see the plan.)
  //   Sums of four wavefronts meet in pairs (4 % of a split's error, and 2 % of the time of dense layers of 4 to 6 us).
  // Over 1300 layers of 10 to 10^5 pixels the error is 0.75 (fp32) and 0.94 (bf16) times the former one in the mean, 1.01 and 1.02 at most; over 400 bf16
  // layers whose K was split and is not now, or less, 0.98, 1.09 at most (1.5 and 1.8 as one chain).
  constexpr bool kTwo = kBlocks && SPLIT && kU > 1;     // two sums at a time, of the even and of the odd steps
  auto join = [&](auto two, acc4 (&a)[PF][NH], acc4 (&odd)[PF][NH]) __attribute__((always_inline)) {
    if constexpr (decltype(two)::value) {
#pragma unroll
      for (int f = 0; f < PF; ++f)
#pragma unroll
        for (int i = 0; i < NH; ++i) {
          a[f][i] += odd[f][i];
          odd[f][i] = acc4{0, 0, 0, 0};
        }
    }
  };
  // K steps k0 .. k0 + n - 1 of phase ph into a, two: the odd ones into `odd` first (both zero before; `odd` again afterwards).
  // `meanwhile` runs once the first operands are on their way.
  //   Two batches of kU steps are in flight.  Every way through the loop has the same loads in flight at the same line, and what is left
  // at the end of K leaves it: the compiler's waits are then for the operands that are used and no others.  (With a
  // branch around the fetches the wait before each product was for every load in flight, and where a step's offset was chosen between
  // a scalar and the lanes' own each pixel load stood in a loop over the lanes.)  Steps past the end are loads out of range.
  auto walk = [&](auto two, int ph, int k0, int n, acc4 (&a)[PF][NH], acc4 (&odd)[PF][NH], auto meanwhile) __attribute__((always_inline)) {
    const int nq = ph ? p.chunks1 : p.chunks0;
    const Div dnq{ph ? p.nq1.m : p.nq0.m, ph ? p.nq1.s : p.nq0.s};
    const int cfirst = ph ? 0 : bfirst;
    const int gap_at = ph ? gap_s : 0x7fffffff;     // the chunk from which on the gap is jumped
    const unsigned wgrp = (unsigned)(ph ? p.ks1 : p.ks0) * 2048u;
    const char* const wp = (ph ? p.w1 : p.w0) + (size_t)(half0 >> 1) * wgrp + (NH == 1 ? (half0 & 1) * 1024 : 0);
    const int k1 = k0 + n;
    // (to the end of this wavefront's last step, so that a batch's steps past it are zeros; tiles of 64 channels have no such steps)
    const __amdgpu_buffer_rsrc_t wr =
        __builtin_amdgcn_make_buffer_rsrc((void*)wp, (short)0, (int)(NH == 4 ? 2 * wgrp : (unsigned)k1 * 2048u - (NH == 1 ? 1024u : 0u)), 0x00027000);
    i32x4 x[2][kU][PF], w[2][kU][NH];
    unsigned vw = (unsigned)lane * 16u + (unsigned)k0 * 2048u;      // offset of the next step's weights
    int kx = k0;                                    // the next step whose pixels are fetched
    auto fetch_w = [&](auto bt) __attribute__((always_inline)) {
      constexpr int b = decltype(bt)::value;
#pragma unroll
      for (int u = 0; u < kU; ++u)
#pragma unroll
        for (int i = 0; i < NH; ++i)
          w[b][u][i] = __builtin_bit_cast(i32x4, __builtin_amdgcn_raw_buffer_load_b128(wr, (int)(vw + u * 2048 + (i & 1) * 1024), (i >> 1) * (int)wgrp, 0));
      vw += kU * 2048;
    };
    // the walk's place: UNIFORM: the step's tap and first chunk, else the unit of this lane group
    int tap = 0, ci = 0, so = 0;                    // so (UNIFORM): offset of the step from its pixel's first tap
    unsigned vo[PF];                                // (UNIFORM) the lanes' offsets at this tap
    const int row16 = p.rowb >> 4, px16 = p.xps >> 4;                               // (otherwise) in chunks: 24 bits hold them and their differences
    const int gap16 = p.gap_len * 16, first16 = (cfirst * 16) + (gap_at <= 0 ? gap16 : 0);
    const int dt = nq > 4 ? 0 : nq >= 3 ? 1 : nq == 2 ? 2 : 4, di = 4 - dt * nq;    // (otherwise) a step on: so many taps and chunks on
    auto enter_tap = [&]() __attribute__((always_inline)) {
      const int r = (tap * 11) >> 5, s = tap - 3 * r;
      so = r * p.rowb + s * p.xps + first16;
#pragma unroll
      for (int f = 0; f < PF; ++f) vo[f] = (vmask[f] >> tap) & 1u ? xbase[f] + (unsigned)lg * 16u : kOut;
    };
    auto start = [&]() __attribute__((always_inline)) {
      const unsigned u = 4u * (unsigned)k0 + (UNIFORM ? 0u : (unsigned)lg);
      tap = (int)quot(u, dnq);
      ci = (int)u - tap * nq;
      if constexpr (UNIFORM) {
        enter_tap();
        so += ci * 16 + (gap_at > 0 && ci >= gap_at ? gap16 : 0);
      }
    };
    auto fetch_x = [&](auto bt) __attribute__((always_inline)) {
      constexpr int b = decltype(bt)::value;
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        const bool on = u == 0 || kx + u < k1;
        if constexpr (UNIFORM) {
#pragma unroll
          for (int f = 0; f < PF; ++f) x[b][u][f] = __builtin_bit_cast(i32x4, __builtin_amdgcn_raw_buffer_load_b128(xr, on ? (int)vo[f] : (int)kOut, so, 0));
          so += 64;
          ci += 4;
          so += ci == gap_at ? gap16 : 0;
          if (ci == nq) {
            ci = 0;
            ++tap;
            enter_tap();
          }
        } else {
          const int c = cfirst + ci + (ci >= gap_at ? p.gap_len : 0);
          const int t = on && c < p.total_chunks ? tap : 31;              // (bit 9 and up of the validity mask are zero)
          const int r = (int)__umul24(tap, 11) >> 5;
          const int off16 = __mul24(r, row16 - 3 * px16) + __mul24(tap, px16) + c;
#pragma unroll
          for (int f = 0; f < PF; ++f) {
            const unsigned vof = (vmask[f] >> t) & 1u ? xbase[f] + ((unsigned)off16 << 4) : kOut;
            x[b][u][f] = __builtin_bit_cast(i32x4, __builtin_amdgcn_raw_buffer_load_b128(xr, (int)vof, 0, 0));
          }
          const int next = ci + di;
          tap += dt + (next >= nq ? 1 : 0);
          ci = next - (next >= nq ? nq : 0);
        }
      }
      kx += kU;
    };
    auto mul = [&](auto bt) __attribute__((always_inline)) {
      constexpr int b = decltype(bt)::value;
#pragma unroll
      for (int u = 0; u < kU; ++u)
#pragma unroll
        for (int part = 0; part < Tr::kParts; ++part)      // (fp32: the four products of a step, each over all accumulators)
#pragma unroll
          for (int f = 0; f < PF; ++f)
#pragma unroll
            for (int i = 0; i < NH; ++i) {
              acc4& to = decltype(two)::value && ((kU == 1 ? b : u) & 1) ? odd[f][i] : a[f][i];
              to = Tr::mma(part, w[b][u][i], x[b][u][f], to);
            }
      __builtin_amdgcn_sched_barrier(0);
    };
    // the place in x of unit u of K for this lane's pixel of fragment f: its offset or kOut
    auto unit_at = [&](int f, int t, int chunk) __attribute__((always_inline)) {
      const int r = (t * 11) >> 5;
      const bool on = t < p.taps && chunk < p.total_chunks && ((vmask[f] >> (t & 31)) & 1u);
      return on ? xbase[f] + (unsigned)(r * p.rowb + (t - 3 * r) * p.xps + chunk * 16) : kOut;
    };
    // A layer whose base group ends inside a chunk: the same products in the same order once more, the other path's channels of that chunk
    // left out of x, so that a pixel has the sum that it would have if they were finite (zero weights add nothing to it), to the bit.
    [[maybe_unused]] auto products_again = [&](int f, int h, acc4& all) __attribute__((always_inline)) {
      const int own = p.c_base & (Tr::kCh - 1), at = ph ? 0 : nq - 1;      // base channels of that chunk, and where it is
      const int ln = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));      // (the lane, in no register until here)
      acc4 sum[2] = {acc4{0, 0, 0, 0}, acc4{0, 0, 0, 0}};
      auto step = [&](auto to, int k) __attribute__((always_inline)) {
        const unsigned u = 4u * (unsigned)k + (unsigned)(ln >> 4);
        const int t = (int)quot(u, dnq), i = (int)u - t * nq, chunk = cfirst + i + (i >= gap_at ? p.gap_len : 0);
        i32x4 xv = __builtin_bit_cast(i32x4, __builtin_amdgcn_raw_buffer_load_b128(xr, (int)unit_at(f, t, chunk), 0, 0));
        const i32x4 wv = __builtin_bit_cast(i32x4, __builtin_amdgcn_raw_buffer_load_b128(wr, (int)((unsigned)ln * 16u + (unsigned)k * 2048u + (h & 1) * 1024), (h >> 1) * (int)wgrp, 0));
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int bytes = own * (16 / Tr::kCh) - 4 * e;                  // of the word, base channels
          const int base = bytes >= 4 ? -1 : bytes <= 0 ? 0 : (1 << (8 * bytes)) - 1;
          xv[e] &= i == at ? (ph ? ~base : base) : -1;
        }
#pragma unroll
        for (int part = 0; part < Tr::kParts; ++part) sum[decltype(to)::value] = Tr::mma(part, wv, xv, sum[decltype(to)::value]);
      };
      constexpr int kBlock = kU == 1 ? 2 : 4;       // (two batches of one or two steps, or one of four)
#pragma nounroll
      for (int k = 0; k < n; ++k) {
        step(std::integral_constant<int, 0>{}, k0 + k);
        if constexpr (decltype(two)::value)
          if (++k < n) step(std::integral_constant<int, 1>{}, k0 + k);
        if (k + 1 >= n || (kBlocks && k % kBlock == kBlock - 1)) {
          all += decltype(two)::value ? sum[0] + sum[1] : sum[0];
          sum[0] = sum[1] = acc4{0, 0, 0, 0};
        }
      }
    };
    // Blocks of several groups: each row's products one by one.  (A lane's rows are 4*lg .. 4*lg + 3 of the 16 channels; the unit, and with it the channel, is
    // the same for all lanes.)
    [[maybe_unused]] auto rows_again = [&](int f, int h, acc4& sum) __attribute__((always_inline)) {
      if constexpr (MIXED) {
        int row_grp[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) row_grp[e] = (int)quot((half0 + h) * 16 + 4 * lg + e, p.cpg);
#pragma nounroll
        for (int u = 4 * k0; u < 4 * (k0 + n); ++u) {
          const int t = u / nq, i = u - t * nq, chunk = cfirst + i + (i >= gap_at ? p.gap_len : 0);
          if (t >= p.taps || chunk >= p.total_chunks) continue;
          const i32x4 xv = __builtin_bit_cast(i32x4, __builtin_amdgcn_raw_buffer_load_b128(xr, (int)unit_at(f, t, chunk), 0, 0));
          const char* const wu = wp + (size_t)(h >> 1) * wgrp + (size_t)(u >> 2) * 2048 + (h & 1) * 1024 + (u & 3) * 256 + lg * 64;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const i32x4 wv = *(const i32x4*)(wu + e * 16);
#pragma unroll
            for (int c = 0; c < Tr::kCh; ++c) {
              const bool on = ((chunk * Tr::kCh + c) / p.c_base == row_grp[e]) == (ph == 0);
              sum[e] = on ? fmaf(Tr::element(xv, c), Tr::element(wv, c), sum[e]) : sum[e];
            }
          }
        }
      }
    };
    acc4 tot[PF][NH];                               // the blocks so far
    if constexpr (kBlocks) {
#pragma unroll
      for (int f = 0; f < PF; ++f)
#pragma unroll
        for (int i = 0; i < NH; ++i) tot[f][i] = acc4{0, 0, 0, 0};
    }
    auto carry = [&]() __attribute__((always_inline)) {
      if constexpr (kBlocks) {
        join(two, a, odd);
#pragma unroll
        for (int f = 0; f < PF; ++f)
#pragma unroll
          for (int i = 0; i < NH; ++i) {
            tot[f][i] += a[f][i];
            a[f][i] = acc4{0, 0, 0, 0};
          }
      }
    };
    constexpr std::integral_constant<int, 0> B0{};
    constexpr std::integral_constant<int, 1> B1{};
    const int nb = (n + kU - 1) / kU;
    if (nb > 0) {
      fetch_w(B0);                                  // (their addresses need nothing of the pixels)
      pixels();
      start();
      fetch_x(B0);
    }
    meanwhile();
    if (nb > 1) {
      fetch_w(B1);
      fetch_x(B1);
#pragma nounroll
      for (int i = 2;; i += 2) {
        mul(B0);
        if (kU == 4) carry();
        if (i >= nb) {
          mul(B1);
          break;
        }
        fetch_w(B0);
        fetch_x(B0);
        mul(B1);
        carry();
        if (i + 1 >= nb) {
          mul(B0);
          break;
        }
        fetch_w(B1);
        fetch_x(B1);
      }
    } else if (nb > 0) {
      mul(B0);
    }
    carry();
    join(two, a, odd);
    if constexpr (kBlocks) {
#pragma unroll
      for (int f = 0; f < PF; ++f)
#pragma unroll
        for (int i = 0; i < NH; ++i) a[f][i] = tot[f][i];
    }
    // Sums that are a NaN are formed again without the other path's channels, 16 pixels by 16 channels at a time (there are no registers for more
    // beside those that the first pass left); no other sum changes.
    if constexpr (Base::kDtype != CG_I8 && !UNIFORM) {
      if (!MIXED && !(p.flags & kStraddle)) return;
      auto any_nan = [](const acc4& v) __attribute__((always_inline)) {
        bool nan = false;
#pragma unroll
        for (int e = 0; e < 4; ++e) nan |= v[e] != v[e];
        return nan;
      };
      bool nan = false;
#pragma unroll
      for (int f = 0; f < PF; ++f)
#pragma unroll
        for (int i = 0; i < NH; ++i) nan |= any_nan(a[f][i]);
      if (__ballot(nan) == 0ull) return;
#pragma unroll
      for (int f = 0; f < PF; ++f)
#pragma unroll
        for (int h = 0; h < NH; ++h) {
          if (__ballot(any_nan(a[f][h])) == 0ull) continue;
          acc4 again{0, 0, 0, 0};
          if constexpr (MIXED)
            rows_again(f, h, again);
          else
            products_again(f, h, again);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            float v = again[e];
            asm volatile("" : "+v"(v));             // (one by one into the first pass's registers: tiles of eight units are spilled otherwise)
            const float old = a[f][h][e];
            a[f][h][e] = old != old ? v : old;
          }
        }
    }
  };
  auto zero = [&](acc4 (&a)[PF][NH]) __attribute__((always_inline)) {
#pragma unroll
    for (int f = 0; f < PF; ++f)
#pragma unroll
      for (int i = 0; i < NH; ++i) a[f][i] = acc4{0, 0, 0, 0};
  };

  if constexpr (!SPLIT) {
    acc4 accP[PF][NH], accR[PF][NH];
    zero(accP);
    zero(accR);
    i32x4 tabs[NH];                                 // as of a split, of each sixteen channels
    walk(std::bool_constant<kPair>{}, 0, 0, p.ks0, accP, accR, [&]() __attribute__((always_inline)) {
      if ((p.flags & kClear) && blockIdx.x == 0 && tid < 2) p.total[tid] = 0u;
      if (lane < 4 * kTabs) {
#pragma unroll
        for (int i = 0; i < NH; ++i) tabs[i] = *(const i32x4*)(p.tab + (lane >> 2) * p.tab_stride + (half0 + i) * 64 + (lane & 3) * 16);
      }
    });
    i32x4* const mine = tab_at + wave * (NH * 4 * kTabs);
    if (lane < 4 * kTabs) {
#pragma unroll
      for (int i = 0; i < NH; ++i) mine[i * (4 * kTabs) + lane] = tabs[i];
    }
    __builtin_amdgcn_wave_barrier();                // (other lanes of this wavefront read them)
    unsigned d[PF][NH];                             // bit e: channel 16*(half0 + i) + 4*lg + e
#pragma unroll
    for (int f = 0; f < PF; ++f)
#pragma unroll
      for (int i = 0; i < NH; ++i) d[f][i] = 0u;
    if (gated) {
      bool any = false;
      int lo[NH][4], hi[NH][4];
#pragma unroll
      for (int i = 0; i < NH; ++i) {
        take(&mine[i * (4 * kTabs) + lg], lo[i]);
        take(&mine[i * (4 * kTabs) + 4 + lg], hi[i]);
      }
#pragma unroll
      for (int f = 0; f < PF; ++f) {
        const long long m = m0 + 16 * f + lj;
#pragma unroll
        for (int i = 0; i < NH; ++i) {
          const int co0 = (half0 + i) * 16 + 4 * lg;
          acc_t s[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) s[e] = accP[f][i][e];
          const unsigned dd = masked(p, gate_of<Base>(s, lo[i], hi[i]) & there_are<4>(p, co0, m < p.m_total), co0, m);
          d[f][i] = dd;
          any |= dd != 0u;
        }
        if (p.bitmap) {
#pragma unroll
          for (int i = 0; i < NH; i += 2) {
            const unsigned word = or_groups(d[f][i] << (4 * lg) | d[f][i + 1] << (16 + 4 * lg));
            if (lg == 0 && m < p.m_total && ((half0 + i) >> 1) < p.words) p.bitmap[m * p.words + ((half0 + i) >> 1)] = word;
          }
        }
      }
      if (gate_only) return;
      if (__ballot(any) != 0ull) walk(std::false_type{}, 1, 0, p.ks1, accR, accR, []() {});
    }
    i32x4 res[PF][NH];
#pragma unroll
    for (int f = 0; f < PF; ++f)
#pragma unroll
      for (int i = 0; i < NH; ++i) res[f][i] = load_residual<Base, 4>(p, (half0 + i) * 16 + 4 * lg, m0 + 16 * f + lj, m0 + 16 * f + lj < p.m_total);
#pragma unroll
    for (int i = 0; i < NH; ++i) {
      Tab<Base, 4> t;
      t.take_all(p, (const char*)(mine + i * (4 * kTabs) + lg));
#pragma unroll
      for (int f = 0; f < PF; ++f) {
        const long long m = m0 + 16 * f + lj;
        const int co0 = (half0 + i) * 16 + 4 * lg;
        acc_t s[4], r[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          s[e] = accP[f][i][e];
          r[e] = accR[f][i][e];
        }
        finish<Base>(p, s, r, t, res[f][i], d[f][i], co0, m, y_at<Base>(p, co0, m), m < p.m_total && co0 < p.c_out);
      }
    }
  } else {
    // wavefronts [0, nwb) walk the base path, the others the conditional path; each its part
    const int nwb = p.nwb;
    const int ph = wave >= nwb ? 1 : 0;
    const int part = ph ? wave - nwb : wave;
    const int kq = ph ? p.kq1 : p.kq0, kr = ph ? p.kr1 : p.kr0;
    const int k0 = part * kq + (part < kr ? part : kr), n = ph && gate_only ? 0 : kq + (part < kr ? 1 : 0);
    acc4 acc[PF][NH], odd[PF][NH];
    zero(acc);
    zero(odd);
    // The tile's end: wavefront `wave` has the unit un of it, in shares of 4*Q pixels where there are several wavefronts to a unit (the plan has at least
    // one); its tables, residual and places arrive behind the first operands.
    auto with_q = [&](auto f) __attribute__((always_inline)) {
      constexpr auto q_of = [](int waves) { return waves >= 4 * NU ? 1 : waves >= 2 * NU ? 2 : 4; };
      if (NU == 8 || nw == 8)
        f(std::integral_constant<int, q_of(8)>{}, std::integral_constant<int, 8>{});
      else if (NU == 4 || nw == 4)
        f(std::integral_constant<int, q_of(4)>{}, std::integral_constant<int, 4>{});
      else
        f(std::integral_constant<int, q_of(2)>{}, std::integral_constant<int, 2>{});
    };
    const int un = wave % NU, sub = wave / NU, uf = un / NH, half = half0 + un % NH;
    const bool ends = NU == 1 ? wave < 4 : true;    // (a unit has four shares at most)
    i32x4 tabs = {0, 0, 0, 0}, res = {0, 0, 0, 0};  // (a lane's share of the tables: each lane's own four channels of all of them are 20 registers more)
    char* y_here = nullptr;
    uint16_t* bits_here = nullptr;                  // the half word of the lane's pixel (of lanes that store one)
    unsigned there = 0u;
    int m = 0, co0 = 0, ex_here = 0, tab_here = 0;
    auto prepare_end = [&]() __attribute__((always_inline)) {
      if (!ends) return;
      with_q([&](auto qc, auto) __attribute__((always_inline)) {
        constexpr int Q = decltype(qc)::value, L = 16 / Q;      // lanes to a pixel
        const int ch = (lane & (L - 1)) * Q, px = sub * 4 * Q + lane / L;
        if (lane < 4 * kTabs) tabs = *(const i32x4*)(p.tab + (lane >> 2) * p.tab_stride + half * 64 + (lane & 3) * 16);
        m = m0 + 16 * uf + px;
        co0 = half * 16 + ch;
        const bool valid = m < p.m_total;
        res = load_residual<Base, Q>(p, co0, m, valid && !gate_only);
        there = there_are<Q>(p, co0, valid);
        y_here = y_at<Base>(p, co0, m);
        if (p.bitmap && ch == 0 && valid && half < 2 * p.words) bits_here = (uint16_t*)p.bitmap + ((long long)m * (2 * p.words) + half);
        ex_here = un * 1024 + px * 64 + ((ch >> 2) ^ (px >> 2)) * 16 + (ch & 3) * 4;
        tab_here = ch * 4;
        asm volatile("" : "+v"(there), "+v"(y_here), "+v"(bits_here), "+v"(ex_here), "+v"(tab_here));
      });
    };
    walk(std::bool_constant<kTwo>{}, ph, k0, n, acc, odd, [&]() __attribute__((always_inline)) {
      if ((p.flags & kClear) && blockIdx.x == 0 && tid < 2) p.total[tid] = 0u;
      if constexpr (NU < 8) prepare_end();
    });
    if constexpr (NU == 8) prepare_end();           // (its 13 registers would be spilled)
#pragma unroll
    for (int f = 0; f < PF; ++f)
#pragma unroll
      for (int i = 0; i < NH; ++i) {
        i32x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const acc_t sv = acc[f][i][e];
          v[e] = bits_of(sv);
        }
        ex[(wave * NU + f * NH + i) * 64 + lj * 4 + (lg ^ (lj >> 2))] = v;
      }
    if (NU < 8 && ends && lane < 4 * kTabs) tab_at[wave * (4 * kTabs) + lane] = tabs;
    __syncthreads();
    if (!ends) return;
    with_q([&](auto qc, auto wavesc) __attribute__((always_inline)) {
      constexpr int Q = decltype(qc)::value, N = decltype(wavesc)::value;
      // The sums of the base and of the conditional wavefronts, each added up in pairs; a way of its own for every split.
      acc_t s[Q], r[Q];
      auto add_up = [&](auto first, auto count, acc_t (&sum)[Q]) __attribute__((always_inline)) {
        constexpr int F = decltype(first)::value, C = decltype(count)::value;
#pragma unroll
        for (int e = 0; e < Q; ++e) sum[e] = 0;
        if constexpr (C > 0) {
          acc_t t[C][Q];
#pragma unroll
          for (int j = 0; j < C; ++j) {
            int v[Q];
            take((const char*)ex + ex_here + (F + j) * (NU * 1024), v);
#pragma unroll
            for (int e = 0; e < Q; ++e) set_bits(v[e], t[j][e]);
          }
#pragma unroll
          for (int step = 1; step < C; step *= 2)
#pragma unroll
            for (int j = 0; j + step < C; j += 2 * step)
#pragma unroll
              for (int e = 0; e < Q; ++e) t[j][e] += t[j + step][e];
#pragma unroll
          for (int e = 0; e < Q; ++e) sum[e] = t[0][e];
        }
      };
      auto meet = [&](auto self, auto base) __attribute__((always_inline)) -> void {
        constexpr int B = decltype(base)::value;
        if constexpr (B < N) {
          if (nwb > B) return self(self, std::integral_constant<int, B + 1>{});
        }
        add_up(std::integral_constant<int, 0>{}, base, s);
        add_up(base, std::integral_constant<int, N - B>{}, r);
      };
      meet(meet, std::integral_constant<int, 1>{});
      // (tiles of eight units leave no LDS: their tables lie where this wavefront has read the first one's sums of its unit)
      i32x4* const mine = NU < 8 ? tab_at + wave * (4 * kTabs) : ex + un * 64;
      if (NU == 8 && lane < 4 * kTabs) mine[lane] = tabs;
      __builtin_amdgcn_wave_barrier();
      Tab<Base, Q> tab;
      tab.take_all(p, (const char*)mine + tab_here);
      unsigned d = 0u;
      if (gated) {
        d = gate_of<Base>(s, tab.lo, tab.hi) & there;
        if (p.chan_mask) d = masked(p, d, co0, m);
        if (p.bitmap) {
          const unsigned word = sixteen<Q>(d, lane);
          if (bits_here) *bits_here = (uint16_t)word;
        }
      }
      if (!gate_only) finish<Base>(p, s, r, tab, res, d, co0, m, y_here, there != 0u);
    });
  }
}

template <typename Tr, int PF, int NH, bool SPLIT, bool MIXED>
__global__ __launch_bounds__(SPLIT ? 64 * kMaxSplit : 256, SPLIT ? 4 : 2) void gated_conv_direct_kernel(DirectArgs p) {
  direct_layer<Tr, PF, NH, SPLIT, MIXED, false>(p);
}
struct UniformArgs : DirectArgs {};
template <typename Tr, int PF, int NH, bool SPLIT, bool MIXED>
__global__ __launch_bounds__(SPLIT ? 64 * kMaxSplit : 256, SPLIT ? 4 : 2) void gated_conv_direct_kernel(UniformArgs p) {
  direct_layer<Tr, PF, NH, SPLIT, MIXED, true>(p);
}

// A layer and, in further workgroups of its launch, a 1x1 convolution of the same input beside it (a ResNet block's shortcut): the two need nothing of each
// other, a layer of few pixels leaves room beside it, and a launch of few workgroups is 1.5 us between two kernels and its own chain of latencies.
// K steps in batches of four here: the layer's wavefronts have 128 registers.  A few wavefronts of a further workgroup do a piece each (pieces_to_workgroup).
// ResNet-18, one image of 224x224 (three such layers) 113 -> 102 us, four 145 -> 136, eight 181 -> 174, twelve 224 -> 218.
template <typename Tr, int PF, int NH, typename Args>
__global__ __launch_bounds__(64 * kMaxSplit, 4) void gated_conv_beside_kernel(Args p, PointArgs q) {
  const unsigned layer = (unsigned)p.per_xcd * 8u;
  if (blockIdx.x >= layer) {
    const unsigned wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (wave >= (unsigned)q.waves) return;
    const unsigned piece = (blockIdx.x - layer) * (unsigned)q.waves + wave;
    const unsigned blocks = (unsigned)q.c_out >> 5, px = piece / blocks;
    if (px * 16u < (unsigned)q.m_total) point_piece<4>(q, px, (int)(piece - px * blocks));
    return;
  }
  direct_layer<Tr, PF, NH, true, false, std::is_same_v<Args, UniformArgs>>(p);
}

// [c_out][taps][c] in the caller's two weight arrays -> [32-channel group][K step][half][lane][16 bytes] of
// one phase.  Lane l holds row l%16 of its half h (channel 16*h + row of the group) and unit 4k + l/16.  Elements that are
// not on this phase's path for the row's output channel, rows past c_out and units past the last are zeros.
template <typename T>
__global__ void pack_direct_kernel(const T* __restrict__ wb, const T* __restrict__ wc, T* __restrict__ out, DirectPlan g,
                                   int phase, int c_in, int c_out, int c_base, int groups, int cpg, long long total) {
  const long long id = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (id >= total) return;
  constexpr int CH = 16 / (int)sizeof(T);
  const int lane = (int)(id & 63), h = (int)((id >> 6) & 1);
  const long long q = id >> 7;
  const int k = (int)(q % g.ksteps[phase]), grp = (int)(q / g.ksteps[phase]);
  const int u = 4 * k + (lane >> 4), tap = u / g.chunks[phase], i = u - tap * g.chunks[phase];
  const int row = lane & 15, co = grp * 32 + 16 * h + row;
  const int bfirst = groups > 1 ? (((grp >> 1) * 64) / cpg) * c_base / CH : 0;
  int chunk = phase ? i : bfirst + i;
  if (phase && g.gap_len && chunk >= bfirst) chunk += g.gap_len;
  T v[CH];
#pragma unroll
  for (int e = 0; e < CH; ++e) {
    const int c = chunk * CH + e;
    T t = 0;
    if (co < c_out && tap < g.taps && c < c_in) {
      const int b0 = groups > 1 ? (co / cpg) * c_base : 0;
      const bool base = c >= b0 && c < b0 + c_base;
      if (phase == 0 && base) t = wb[((long long)co * g.taps + tap) * c_base + c - b0];
      if (phase == 1 && !base) t = wc[((long long)co * g.taps + tap) * (c_in - c_base) + (c < b0 ? c : c - c_base)];
    }
    v[e] = t;
  }
#pragma unroll
  for (int e = 0; e < CH; ++e) out[id * CH + e] = v[e];
}

template <typename Tr, int PF, int NH, bool MIXED, typename Args>
hipError_t launch_direct_form(const DirectPlan& g, const Args& a, hipStream_t s) {
  using Kernel = void (*)(Args);
  const dim3 grid((unsigned)a.per_xcd * 8u);
  if (g.split > 1) {
    const Kernel k = gated_conv_direct_kernel<Tr, PF, NH, true, MIXED>;
    hipLaunchKernelGGL(k, grid, dim3(64 * g.split), 0, s, a);
  } else {
    if constexpr (NH == 1) {
      return hipErrorInvalidValue;
    } else {
      const Kernel k = gated_conv_direct_kernel<Tr, PF, NH, false, MIXED>;
      hipLaunchKernelGGL(k, grid, dim3(256), 0, s, a);
    }
  }
  return hipGetLastError();
}

template <typename Tr, int PF, int NH, typename Args>
hipError_t launch_beside(const DirectPlan& g, const Args& a, PointArgs q, hipStream_t s) {
  const long long pieces = ((long long)q.m_total + 15) / 16 * (q.c_out / 32);
  q.waves = pieces_to_workgroup((long long)a.per_xcd * 8, pieces, q.c_in, a.waves, g.est, cu_count());
  const unsigned more = (unsigned)((pieces + q.waves - 1) / q.waves);
  const auto k = gated_conv_beside_kernel<Tr, PF, NH, Args>;
  hipLaunchKernelGGL(k, dim3((unsigned)a.per_xcd * 8u + more), dim3(64 * g.split), 0, s, a, q);
  return hipGetLastError();
}

template <typename Tr, int PF, int NH>
hipError_t launch_direct_tile(const DirectPlan& g, const DirectArgs& a, const PointArgs* beside, hipStream_t s) {
  if constexpr (Tr::Base::kDtype == CG_BF16)
    if (beside) return g.uniform ? launch_beside<Tr, PF, NH>(g, UniformArgs{a}, *beside, s) : launch_beside<Tr, PF, NH>(g, a, *beside, s);
  if (g.uniform) return launch_direct_form<Tr, PF, NH, false>(g, UniformArgs{a}, s);
  if constexpr (Tr::Base::kDtype != CG_I8)
    if (g.mixed) return launch_direct_form<Tr, PF, NH, true>(g, a, s);
  return launch_direct_form<Tr, PF, NH, false>(g, a, s);
}

template <typename Tr>
hipError_t launch_direct_dtype(const DirectPlan& g, const DirectArgs& a, const PointArgs* beside, hipStream_t s) {
  switch (g.pf * 8 + g.nh) {
    case 2 * 8 + 4: return launch_direct_tile<Tr, 2, 4>(g, a, beside, s);
    case 2 * 8 + 2: return launch_direct_tile<Tr, 2, 2>(g, a, beside, s);
    case 1 * 8 + 4: return launch_direct_tile<Tr, 1, 4>(g, a, beside, s);
    case 1 * 8 + 2: return launch_direct_tile<Tr, 1, 2>(g, a, beside, s);
    case 1 * 8 + 1: return launch_direct_tile<Tr, 1, 1>(g, a, beside, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

DirectPlan direct_plan(const cg_conv_desc& d, int n, int n_cu) {
  DirectPlan g{};
  g.elem_bytes = d.in_dtype == CG_BF16 ? 2 : d.in_dtype == CG_I8 ? 1 : 4;
  g.ch = 16 / g.elem_bytes;
  g.taps = d.kh * d.kw;
  const long long xps = d.x_pixel_stride ? d.x_pixel_stride : d.c_in;
  if (xps % g.ch || d.c_in % g.ch) return g;                    // a pixel's channels are whole aligned chunks
  const int ho = (d.h + 2 * d.pad - d.kh) / d.stride + 1, wo = (d.w + 2 * d.pad - d.kw) / d.stride + 1;
  const long long xb = (((long long)n * d.h * d.w - 1) * xps + d.c_in) * g.elem_bytes, m = (long long)n * ho * wo;
  if (xb >= (1ll << 30) || m >= (1ll << 30)) return g;          // 32-bit offsets with room for the padding
  if ((long long)d.w * xps * g.elem_bytes >= (1 << 23)) return g;   // (24-bit products)
  g.x_bytes = (unsigned)xb;
  const bool gated = d.c_base < d.c_in;
  const int groups = d.groups > 1 ? d.groups : 1, cpg = d.c_out / groups;
  const int ngrp = (d.c_out + 31) / 32;
  g.n_grp = (ngrp + 1) / 2 * 2;
  g.total_chunks = d.c_in / g.ch;
  int last_end = 0;                                              // of the last block's base phase
  if (groups == 1) {
    g.chunks[0] = (d.c_base + g.ch - 1) / g.ch;
    g.gap_len = d.c_base / g.ch;
    g.straddle = d.c_base % g.ch ? 1 : 0;
  } else {
    // a 64-channel block walks the base channels of every group it touches; the other groups' weights are zeros
    bool single = d.c_base % g.ch == 0;
    for (int b = 0; b * 64 < d.c_out; ++b) {
      const int last = b * 64 + 63 < d.c_out ? b * 64 + 63 : d.c_out - 1;
      const int ga = b * 64 / cpg, gb = last / cpg;
      const int first = ga * d.c_base / g.ch, end = ((gb + 1) * d.c_base + g.ch - 1) / g.ch;
      if (end - first > g.chunks[0]) g.chunks[0] = end - first;
      if (ga != gb) single = false;
    }
    g.gap_len = single ? d.c_base / g.ch : 0;
    g.mixed = single ? 0 : 1;
    last_end = ((d.c_out - 1) / 64 * 64 / cpg) * d.c_base / g.ch + g.chunks[0];
  }
  g.chunks[1] = gated ? g.total_chunks - g.gap_len : 0;
  for (int ph = 0; ph < 2; ++ph) {
    g.ksteps[ph] = (g.chunks[ph] * g.taps + 3) / 4;
    g.wpk_bytes[ph] = (size_t)g.n_grp * g.ksteps[ph] * 2048;
  }
  const int ks = g.ksteps[0] + g.ksteps[1];

  // Tile and split with the least estimated time, in clocks, fitted to 4500 measured plans of 277 layers (bf16 and int8, fp32
  // by itself; one to 31000 output pixels, 16 to 4000 channels), of a form of this kernel whose K loop and end were slower.  There what it picked took 2.6 %
  // longer than the best plan in the mean, 13 % at the 95th percentile; with the present loop and end, the same constants and 60 layers of 32 to 32000
  // pixels 4.0 and 22 %, 42 % at most (bf16 1x1, 80 to 224 channels at 19x19, 16 images 7.2 us, not split 5.1).  (That is what plans are compared by.
  // `est`, by which the kernel is chosen, counts the output of many tiles more: over 123 layers it was 9 % off in that form.)
  //   A K step costs the vector-memory path 50 clocks for 16 pixels (64-byte pieces) and 12 (fp32: 32) for 16 channels of
  //   weights; the matrix cores take 16 (175) for a product, and a wavefront 450 (80) for the latency of a batch of
  //   steps.  Workgroups on a compute unit at the same time overlap in their latencies only.
  const int words = (d.c_out + 31) / 32;
  auto tiles_c = [&](int nh) { return (2 * words + nh - 1) / nh; };
  const bool f32 = d.in_dtype == CG_F32;
  auto nwb_of = [&](int split) {
    if (!gated) return split;
    const int b = (split * g.ksteps[0] + ks / 2) / ks;
    return b < 1 ? 1 : b > split - 1 ? split - 1 : b;
  };
  // K steps of one tap, on one side of the base group, that end with the input's channels in every block
  const bool uni = g.total_chunks % 4 == 0 && g.gap_len % 4 == 0 && g.chunks[0] % 4 == 0;
  g.uniform = uni && g.straddle == 0 && (groups == 1 || d.c_base % (4 * g.ch) == 0) && last_end <= g.total_chunks && (g.mixed == 0 || d.in_dtype == CG_I8);
  const double start = f32 ? 5250.0 : 5350.0, each0 = f32 ? 90.0 : 233.0, each1 = f32 ? 211.0 : 124.0, wave0 = f32 ? 3880.0 : 3790.0;
  const double cx = (f32 ? 52.0 : 50.0) * (uni ? 1.0 : f32 ? 1.25 : 0.91), cw = f32 ? 32.0 : 12.5, cm = f32 ? 175.0 : 16.0, cl = f32 ? 82.0 : 450.0;
  // bf16 layers of at least two K steps to each of four wavefronts, and fewer than four times as many tiles of 32 x 64 as compute units, are
  // split: their K always was, over four wavefronts or more, and as one chain of each path (two of a dense layer's) their error against 64 bits
  // was up to 1.8 times as large.  14 such layers: 0.98 of the whole form's time in the mean, 0.88 to 1.11.
  const bool chained = d.in_dtype == CG_BF16 && ks >= 8 && (m + 31) / 32 * (g.n_grp / 2) < 4ll * n_cu;
  const bool two_in_4g = std::max(g.ksteps[0], g.ksteps[1]) < (1 << 20);        // (tiles of 64 channels: two groups' weights, 2048 bytes a step, at 32-bit offsets)
  g.cost = 1e30;
  for (int pf = 1; pf <= (m > 16 ? 2 : 1); ++pf)
    for (int nh = pf; nh <= (ngrp >= 2 ? 4 : 2); nh *= 2)           // (32 x 16 pixels and channels were never the least)
      for (int split = 1; split <= kMaxSplit; split *= 2) {
        const int nu = pf * nh;
        if (nh == 4 && !two_in_4g) continue;
        if (split == 1 ? nh == 1 || chained : split < nu || (gated && split < 2)) continue;
        const bool whole = split == 1;
        const long long px = (m + 16 * pf - 1) / (16 * pf), wgs = (whole ? (px + 3) / 4 : px) * tiles_c(nh);
        const int waves = whole ? 4 : split, nwb = nwb_of(split);
        const double steps = whole ? g.ksteps[0] + 1.08 * g.ksteps[1]
                                   : std::max((g.ksteps[0] + nwb - 1) / nwb, gated ? (g.ksteps[1] + split - nwb - 1) / (split - nwb) : 0);
        const double rounds = (double)((wgs + n_cu - 1) / n_cu), room = whole ? (nu == 8 ? 2 : nh == 4 ? 3 : 4) : nu == 8 ? 2 : 16 / split;
        const double turns = rounds > room ? rounds / room : 1.0;
        const double vm = rounds * (whole ? 4.0 * steps : ks) * (cx * pf + cw * nh);
        const double mm = rounds * steps * waves * nu * cm / std::min(4.0, waves * std::min(rounds, 4.0));
        const double chain = turns * steps * (cl / (nu == 1 ? 4 : nu == 2 ? 2 : 1) + cm * nu), busy = std::max(vm, mm);
        const double c = start + rounds * (each0 + each1 * nu) + wave0 * turns + std::max(busy, chain) + 0.35 * std::min(busy, chain) + (whole ? 2500.0 : 0.0);
        if (c >= g.cost) continue;
        g.cost = c;
        g.est = 500.0 + 1.03 * c + nu * (100.0 * (rounds - 1.0) * (whole ? 4.0 : 1.0) + (whole ? 480.0 : 0.0));
        g.pf = pf;
        g.nh = nh;
        g.split = split;
        g.nwb = nwb;
      }
  g.n_cblk = tiles_c(g.nh);
  const long long px = (m + 16 * g.pf - 1) / (16 * g.pf), wgs = g.split > 1 ? px : (px + 3) / 4;
  if (wgs * g.n_cblk > 0x7ffffff0ll) return g;
  g.px_wgs = (int)wgs;
  g.ok = 1;
  return g;
}

hipError_t launch_direct_pack(const DirectPlan& g, const Params& p, void* wpk0, void* wpk1, hipStream_t s) {
  for (int ph = 0; ph < 2; ++ph) {
    if (g.ksteps[ph] == 0) continue;
    const long long total = (long long)g.n_grp * g.ksteps[ph] * 128;
    const dim3 grid((unsigned)((total + 255) / 256)), block(256);
    void* out = ph ? wpk1 : wpk0;
    if (g.elem_bytes == 4)
      hipLaunchKernelGGL(pack_direct_kernel<uint32_t>, grid, block, 0, s, (const uint32_t*)p.w_base, (const uint32_t*)p.w_cond,
                         (uint32_t*)out, g, ph, p.c_in, p.c_out, p.c_base, p.groups, p.cpg, total);
    else if (g.elem_bytes == 2)
      hipLaunchKernelGGL(pack_direct_kernel<uint16_t>, grid, block, 0, s, (const uint16_t*)p.w_base, (const uint16_t*)p.w_cond,
                         (uint16_t*)out, g, ph, p.c_in, p.c_out, p.c_base, p.groups, p.cpg, total);
    else
      hipLaunchKernelGGL(pack_direct_kernel<uint8_t>, grid, block, 0, s, (const uint8_t*)p.w_base, (const uint8_t*)p.w_cond,
                         (uint8_t*)out, g, ph, p.c_in, p.c_out, p.c_base, p.groups, p.cpg, total);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

bool takes_beside(const DirectPlan& g, const Params& p) { return p.in_dtype == CG_BF16 && g.split > 1 && (g.uniform || !g.mixed); }

hipError_t launch_direct(const DirectPlan& g, const Params& p, const void* w0, const void* w1, hipStream_t s, const PointArgs* beside) {
  DirectArgs a{};
  a.rowb = p.w * (int)p.x_pixel_stride * g.elem_bytes;
  a.xps = (int)p.x_pixel_stride * g.elem_bytes;
  a.x_bias = p.pad * (a.rowb + a.xps);
  a.x = (const char*)p.x - a.x_bias;
  a.x_bytes = (int)g.x_bytes + a.x_bias;
  a.w0 = (const char*)w0;
  a.w1 = (const char*)w1;
  a.tab = (const char*)p.thr_f;
  a.y = p.y;
  a.residual = p.residual;
  a.bitmap = p.bitmap;
  a.chan_mask = p.chan_mask;
  a.total = p.total;
  a.tab_stride = (int)p.table_stride;
  a.m_total = (int)p.m_total;
  a.n_wo = p.wo;
  a.n_ho = p.ho;
  a.h = p.h;
  a.w = p.w;
  a.n_wgs = g.px_wgs * g.n_cblk;
  a.per_xcd = (a.n_wgs + 7) / 8;
  a.stride = p.stride;
  a.pad = p.pad;
  a.taps = g.taps;
  a.chunks0 = g.chunks[0];
  a.chunks1 = g.chunks[1];
  a.total_chunks = g.total_chunks;
  a.gap_len = g.gap_len;
  a.ks0 = g.ksteps[0];
  a.ks1 = g.ksteps[1];
  a.n_cblk = g.n_cblk;
  a.waves = g.split > 1 ? g.split : 4;
  a.nwb = g.nwb;
  a.c_out = p.c_out;
  a.words = p.words;
  a.n_cpg = p.cpg;
  a.groups = p.groups;
  a.c_base = p.c_base;
  a.ch_log = g.ch == 16 ? 4 : g.ch == 8 ? 3 : 2;
  a.wo = div_of(p.wo);
  a.ho = div_of(p.ho);
  a.hw = div_of(p.ho * p.wo);
  a.cblk = div_of(g.n_cblk);
  a.cpg = div_of(p.cpg);
  a.nq0 = div_of(g.chunks[0]);
  a.nq1 = div_of(g.chunks[1] > 0 ? g.chunks[1] : 1);
  if (g.split > 1) {
    const int parts0 = g.nwb, parts1 = g.split - g.nwb;
    a.kq0 = g.ksteps[0] / parts0;
    a.kr0 = g.ksteps[0] % parts0;
    a.kq1 = parts1 ? g.ksteps[1] / parts1 : 0;
    a.kr1 = parts1 ? g.ksteps[1] % parts1 : 0;
  }
  a.rq_shift = p.rq_shift;
  a.rq_res_mult = p.rq_res_mult;
  static_assert(kRelu == CG_EPI_RELU && kAffine == CG_EPI_AFFINE && kResidual == CG_EPI_RESIDUAL, "the epilogue flags pass through");
  a.flags = p.epilogue | (p.gated ? kGated : 0u) | (p.gate_only ? kGateOnly : 0u) | (p.clear_total ? kClear : 0u) |
            (p.shuffle ? kShuffle : 0u) | (p.out_dtype == CG_F32 || p.out_dtype == CG_I32 ? kOut4 : 0u) | (p.fit32 ? kFit32 : 0u) | (g.straddle ? kStraddle : 0u);
  switch (p.in_dtype) {
    case CG_BF16: return launch_direct_dtype<Bf16Direct>(g, a, beside, s);
    case CG_I8: return launch_direct_dtype<I8Direct>(g, a, beside, s);
    default: return launch_direct_dtype<F32Direct>(g, a, beside, s);
  }
}

}  // namespace cg
