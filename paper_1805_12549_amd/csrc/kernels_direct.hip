// Small-tile matrix-core kernel of the gated convolution (bf16, int8 and fp32 MFMA, 16x16 blocks):
// no LDS staging, the operands go from global memory straight into registers.
//
// It takes what the two tiled kernels are no good at: layers with few output pixels (one image, deep
// layers), channel counts and groups that are not multiples of 64 channels / of whole K stages, and
// fp32.  A wavefront multiplies PF fragments of 16 output pixels by CG groups of 32 output channels; the
// product is taken transposed (weights are the row operand, their rows permuted), so a lane ends up
// with 8 consecutive channels of one pixel per group (Eq. 1 and the gate work on registers).
//
// What bounds it is the vector-memory path of a compute unit, which serves the 64-byte pieces of the
// pixel operand at some 23 bytes per clock and the linear weights at some 37 (measured; 32-byte pieces,
// what 32x32 blocks would fetch, at 13): a K step of 2 fragments x 2 groups costs 200 clocks of that path
// for 64 clocks of the matrix cores.  So the forms below exist to get every compute unit to pull:
//
//   whole   a wavefront owns a tile and walks all of K; the conditional path is walked only if one of
//           the tile's gates fired.  No barrier, no LDS.
//   SPLIT   a workgroup of 2..8 wavefronts owns one tile and splits K: some wavefronts walk the base
//           path, the others the conditional path, all at once; the partial sums meet in LDS.  Where
//           that still leaves compute units idle, `slices` workgroups share the tile's K, write
//           their sums to the workspace and a second kernel adds them up, takes the gate and finishes.
//           No phase waits for the gate, so the length of the chain is K / (wavefronts * slices).
//
// K is walked in steps of four units, unit u = tap * chunks + chunk, a unit being one 16-byte channel
// chunk of one tap; lane group l/16 supplies unit 4k + l/16.  Padding (taps outside the image, units past
// the last) is an out-of-range buffer load, which returns zeros.  A base group that ends inside a chunk is
// masked in registers on both paths, so that a channel never meets a weight of the other path (0 * inf
// would otherwise reach the sum).
#include <type_traits>

#include "cg_mfma_common.h"

namespace cg {

namespace {

struct Bf16Direct {
  using Base = Bf16Traits;
  using acc4 = f32x4;
  using acc_t = float;
  static constexpr int kCh = 8;
  static __device__ __forceinline__ acc4 mma(i32x4 rows, i32x4 cols, acc4 c) { return Bf16Traits::mfma(rows, cols, c); }
  static __device__ __forceinline__ float element(i32x4 v, int e) { return __uint_as_float(e & 1 ? (unsigned)v[e >> 1] & 0xffff0000u : (unsigned)v[e >> 1] << 16); }
};

struct I8Direct {
  using Base = I8Traits;
  using acc4 = i32x4;
  using acc_t = int32_t;
  static __device__ __forceinline__ acc4 mma(i32x4 rows, i32x4 cols, acc4 c) { return I8Traits::mfma(rows, cols, c); }
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
  static constexpr int kCh = 4;
  static __device__ __forceinline__ float element(i32x4 v, int e) { return __int_as_float(v[e]); }
  static __device__ __forceinline__ acc4 mma(i32x4 rows, i32x4 cols, acc4 c) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      c = __builtin_amdgcn_mfma_f32_16x16x4f32(__int_as_float(rows[e]), __int_as_float(cols[e]), c, 0, 0, 0);
    return c;
  }
};

__device__ __forceinline__ int bits_of(float f) { return __float_as_int(f); }
__device__ __forceinline__ int bits_of(int v) { return v; }
__device__ __forceinline__ void set_bits(int b, float& f) { f = __int_as_float(b); }
__device__ __forceinline__ void set_bits(int b, int& v) { v = b; }

// What the kernels read, in one piece: a wavefront's first instructions load it whole and wait once (argument
// by argument, in the order of use, the waits alone took over a microsecond of a six-microsecond kernel).
struct DirectArgs {
  const void* x;
  const char *w0, *w1;
  const char* tab;           // per-channel tables, tab_stride bytes apart (see cg_internal.h)
  void* y;
  const void* residual;
  uint32_t* bitmap;
  const uint32_t* chan_mask;
  i32x4* partial;
  uint32_t* total;
  int tab_stride, x_bytes, m_total, wo, ho, h, w, xps;
  unsigned magic_wo, magic_ho, magic_cblk, magic_slices;       // ceil(2^32 / d), or 0: divide
  int stride, pad, taps, chunks0, chunks1, total_chunks, gap_len, strad;
  int ks0, ks1, n_cblk, slices, nwb, px_wgs, per_xcd, n_wgs, c_out;
  int words, cpg, groups, c_base, ch, rq_shift, rq_res_mult;
  unsigned flags;
};
enum : unsigned {
  kRelu = 1u, kAffine = 2u, kResidual = 4u,       // as CG_EPI_*
  kGated = 8u, kGateOnly = 16u, kClear = 32u, kShuffle = 64u,
  kOut4 = 128u,                                   // 4-byte outputs (CG_F32 / CG_I32)
};

__device__ __forceinline__ void load_args(const DirectArgs& a) {
  asm volatile("" ::"s"(a.x), "s"(a.w0), "s"(a.w1), "s"(a.tab), "s"(a.y), "s"(a.residual), "s"(a.bitmap), "s"(a.chan_mask),
               "s"(a.partial), "s"(a.total), "s"(a.tab_stride), "s"(a.x_bytes), "s"(a.m_total), "s"(a.wo), "s"(a.ho), "s"(a.h),
               "s"(a.w), "s"(a.xps), "s"(a.magic_wo), "s"(a.magic_ho), "s"(a.magic_cblk), "s"(a.stride), "s"(a.pad), "s"(a.taps),
               "s"(a.chunks0), "s"(a.chunks1), "s"(a.gap_len), "s"(a.flags));
  asm volatile("" ::"s"(a.magic_slices), "s"(a.total_chunks), "s"(a.strad), "s"(a.ks0), "s"(a.ks1), "s"(a.n_cblk), "s"(a.slices),
               "s"(a.nwb), "s"(a.px_wgs), "s"(a.per_xcd), "s"(a.n_wgs), "s"(a.c_out), "s"(a.words), "s"(a.cpg), "s"(a.groups), "s"(a.c_base),
               "s"(a.ch), "s"(a.rq_shift), "s"(a.rq_res_mult));
}

// x / d with magic = ceil(2^32 / d) where the launcher found that exact for every x of the grid (0: divide)
__device__ __forceinline__ unsigned quot(unsigned x, unsigned d, unsigned magic) {
  return magic ? __umulhi(x, magic) : d == 1u ? x : x / d;
}

// The per-channel tables of four channels, fetched ahead of the sums they are needed for.
template <typename Base>
struct Tab4 {
  i32x4 lo, hi, s0, h0, s1, h1;                  // int8 layers: s0 = mult0, h0 = mult1, s1 = bias
  __device__ __forceinline__ void load(const DirectArgs& a, int co0) {
    lo = hi = s0 = h0 = s1 = h1 = i32x4{0, 0, 0, 0};
    if (co0 >= a.c_out) return;                  // (a table is padded to a multiple of 64 entries)
    const char* t = a.tab + co0 * 4;
    if (a.flags & kGated) {
      lo = *(const i32x4*)t;
      if constexpr (Base::kDtype != CG_I8) hi = *(const i32x4*)(t + a.tab_stride);
    }
    if (Base::kDtype == CG_I8 ? !(a.flags & kOut4) : (a.flags & kAffine) != 0) {
      s0 = *(const i32x4*)(t + 2 * a.tab_stride);
      h0 = *(const i32x4*)(t + 3 * a.tab_stride);
      s1 = *(const i32x4*)(t + 4 * a.tab_stride);
      if constexpr (Base::kDtype != CG_I8) h1 = *(const i32x4*)(t + 5 * a.tab_stride);
    }
  }
};

// decisions of four consecutive channels from their base sums
template <typename Base, typename acc_t>
__device__ __forceinline__ unsigned gate4(const DirectArgs& a, const acc_t (&s)[4], const Tab4<Base>& t, int co0) {
  unsigned d = 0u;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    bool f;
    if constexpr (Base::kDtype == CG_I8)
      f = Base::fires(s[e], t.lo[e], 0);
    else
      f = Base::fires(s[e], __int_as_float(t.lo[e]), __int_as_float(t.hi[e]));
    d |= (f ? 1u : 0u) << e;
  }
  const int left = a.c_out - co0;                // channels past the last one never fire
  return left >= 4 ? d : left > 0 ? d & ((1u << left) - 1u) : 0u;
}

// Output function (f of Eq. 1) for four consecutive channels co0.. of output pixel m, decisions in d; read and
// stored in one piece where c_out allows, else one by one.
template <typename Base, typename acc_t>
__device__ __forceinline__ void finish4(const DirectArgs& a, const acc_t (&s)[4], const Tab4<Base>& t, unsigned d, int co0, long long m) {
  if (co0 >= a.c_out) return;
  const bool whole = !((a.c_out & 3) || (a.flags & kShuffle));
  const long long o = m * a.c_out + co0;
  long long oe[4];
  if (!whole) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int co = co0 + e, grp = (a.flags & kShuffle) ? co / a.cpg : 0;
      oe[e] = m * a.c_out + ((a.flags & kShuffle) ? (co - grp * a.cpg) * a.groups + grp : co);
    }
  }
  if (!(a.flags & kGated)) d = 0xfu;             // (a dense layer takes the second pair)
  if constexpr (Base::kDtype == CG_I8) {
    int32_t v[4];
    uint32_t rb = 0u;
    if (a.flags & kResidual) {
      if (whole) {
        rb = *(const uint32_t*)((const int8_t*)a.residual + o);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (co0 + e < a.c_out) rb |= (uint32_t) * ((const uint8_t*)a.residual + oe[e]) << (8 * e);
      }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const long long r = (long long)(int8_t)(rb >> (8 * e)) * a.rq_res_mult;
      long long q;
      if (a.flags & kOut4) {
        q = (long long)s[e] + r;
        if ((a.flags & kRelu) && q < 0) q = 0;
        q = q > 2147483647ll ? 2147483647ll : q;
        q = q < -2147483648ll ? -2147483648ll : q;
      } else {
        q = (long long)s[e] * (((d >> e) & 1u) ? t.h0[e] : t.s0[e]);
        q += (long long)t.s1[e] * (1ll << a.rq_shift) + r;
        if (a.rq_shift > 0) q = (q + (1ll << (a.rq_shift - 1))) >> a.rq_shift;
        const long long lo = (a.flags & kRelu) ? 0 : -128;
        q = q < lo ? lo : q > 127 ? 127 : q;
      }
      v[e] = (int32_t)q;
    }
    if (!whole) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (co0 + e < a.c_out) {
          if (a.flags & kOut4)
            ((int32_t*)a.y)[oe[e]] = v[e];
          else
            ((int8_t*)a.y)[oe[e]] = (int8_t)v[e];
        }
    } else if (a.flags & kOut4) {
      *(i32x4*)((int32_t*)a.y + o) = i32x4{v[0], v[1], v[2], v[3]};
    } else {
      *(int32_t*)((int8_t*)a.y + o) = (v[0] & 0xff) | ((v[1] & 0xff) << 8) | ((v[2] & 0xff) << 16) | ((v[3] & 0xff) << 24);
    }
  } else {
    float r[4] = {0, 0, 0, 0}, v[4];
    if (a.flags & kResidual) {
      if (!whole) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (co0 + e < a.c_out)
            r[e] = (a.flags & kOut4) ? ((const float*)a.residual)[oe[e]] : bf16_to_float(((const uint16_t*)a.residual)[oe[e]]);
      } else if (a.flags & kOut4) {
        const f32x4 q = *(const f32x4*)((const float*)a.residual + o);
#pragma unroll
        for (int e = 0; e < 4; ++e) r[e] = q[e];
      } else {
        const uint2 q = *(const uint2*)((const uint16_t*)a.residual + o);
        r[0] = __uint_as_float(q.x << 16), r[1] = __uint_as_float(q.x & 0xffff0000u);
        r[2] = __uint_as_float(q.y << 16), r[3] = __uint_as_float(q.y & 0xffff0000u);
      }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float q = s[e];
      if (a.flags & kAffine)
        q = ((d >> e) & 1u) ? fmaf(__int_as_float(t.s1[e]), q, __int_as_float(t.h1[e]))
                            : fmaf(__int_as_float(t.s0[e]), q, __int_as_float(t.h0[e]));
      if (a.flags & kResidual) q += r[e];
      if (a.flags & kRelu) q = fmaxf(q, 0.0f);
      v[e] = q;
    }
    if (!whole) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (co0 + e < a.c_out) {
          if (a.flags & kOut4)
            ((float*)a.y)[oe[e]] = v[e];
          else
            ((uint16_t*)a.y)[oe[e]] = float_to_bf16(v[e]);
        }
    } else if (a.flags & kOut4) {
      *(f32x4*)((float*)a.y + o) = f32x4{v[0], v[1], v[2], v[3]};
    } else {
      *(uint2*)((uint16_t*)a.y + o) = uint2{(uint32_t)float_to_bf16(v[0]) | ((uint32_t)float_to_bf16(v[1]) << 16),
                                            (uint32_t)float_to_bf16(v[2]) | ((uint32_t)float_to_bf16(v[3]) << 16)};
    }
  }
}

// The end of the layer for one unit of a tile (16 pixels x 4 channels a lane): decisions, output.  The
// decision bits of the tile's words meet in LDS.
template <typename Base, typename acc_t>
__device__ __forceinline__ void finish_unit(const DirectArgs& a, acc_t (&s)[4], const acc_t (&r)[4], const Tab4<Base>& t, int co0,
                                            long long m, bool valid, uint32_t* word) {
  unsigned d = 0u;
  if (a.flags & kGated) {
    d = gate4<Base>(a, s, t, co0);
    if (!valid || co0 >= a.c_out) d = 0u;
    if (a.chan_mask && d) {
      const unsigned img = (unsigned)m / (unsigned)(a.ho * a.wo);
      d &= a.chan_mask[(long long)img * a.words + (co0 >> 5)] >> (co0 & 31);
    }
    if (d) atomicOr(word, d << (co0 & 31));
  }
  if (valid && !(a.flags & kGateOnly)) {
#pragma unroll
    for (int e = 0; e < 4; ++e) s[e] += ((d >> e) & 1u) ? r[e] : (acc_t)0;
    finish4<Base>(a, s, t, d, co0, m);
  }
}

// 8 wavefronts per workgroup at most
constexpr int kMaxSplit = 8;

// MIXED: float layers whose blocks cover several channel groups (Sec. 3.3) or whose groups share a chunk.  The packed
// weights are zero where a channel is not on a row's path, which keeps its finite values out of the row's sum but turns
// an infinity or a NaN into a NaN; a wavefront that ends up with a NaN forms its sums again, from the path's channels
// alone.  (The look at the sums costs 1 to 2 %: 96 channels at 56x56 in four groups, 16 images 52.4 -> 52.9 us, 128 at 28x28,
// two images 11.2 -> 11.4; one at every operand, as it is read, 5 to 7 %.)
template <typename Tr, int PF, int CG, bool SPLIT, bool MIXED>
__global__ __launch_bounds__(SPLIT ? 64 * kMaxSplit : 256, 2) void gated_conv_direct_kernel(DirectArgs p) {
  using Base = typename Tr::Base;
  using acc4 = typename Tr::acc4;
  using acc_t = typename Tr::acc_t;
  constexpr int NU = PF * CG * 2;                   // units of a tile: (pixel fragment, group, half of its channels)
  constexpr int kU = PF * CG >= 4 || (!SPLIT && CG == 2) ? 2 : 4;          // K steps whose operands are fetched together; two such batches are in flight
  __shared__ __align__(16) i32x4 ex[SPLIT ? kMaxSplit * NU * 64 : 1];     // [wavefront][unit][lane]
  __shared__ uint32_t words[SPLIT ? PF * 16 * CG : 1];                    // [pixel][group]

  load_args(p);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), nw = (int)blockDim.x >> 6;
  const int lj = lane & 15, lg = lane >> 4;

  // block -> (pixel tile, channel tile, K slice): an XCD (block id mod 8) takes a contiguous run of them, so the
  // input of neighbouring tiles is fetched into one L2
  const int id = (int)(blockIdx.x & 7) * p.per_xcd + (int)(blockIdx.x >> 3);
  if (id >= p.n_wgs) return;
  int rest = (int)quot(id, p.n_cblk, p.magic_cblk);
  const int cbk = id - rest * p.n_cblk;
  int slice = 0;
  if (SPLIT) {
    const int t = (int)quot(rest, p.slices, p.magic_slices);
    slice = rest - t * p.slices;
    rest = t;
  }
  const int pt = rest;
  if ((p.flags & kClear) && blockIdx.x == 0 && tid < 2) p.total[tid] = 0u;
  const int grp0 = cbk * CG;                        // first 32-channel group of the tile

  const int m0 = (pt * (SPLIT ? 1 : nw) + (SPLIT ? 0 : wave)) * (16 * PF);
  if (!SPLIT && m0 >= p.m_total) return;
  int xbase[PF];
  unsigned vmask[PF];                               // bit t: tap t of this lane's pixel is inside the image
#pragma unroll
  for (int f = 0; f < PF; ++f) {
    const bool valid = m0 + 16 * f + lj < p.m_total;
    const unsigned mm = valid ? (unsigned)(m0 + 16 * f + lj) : 0u;
    const unsigned q = quot(mm, p.wo, p.magic_wo);
    const unsigned img = quot(q, p.ho, p.magic_ho);
    const int hi0 = (int)(q - img * (unsigned)p.ho) * p.stride - p.pad, wi0 = (int)(mm - q * (unsigned)p.wo) * p.stride - p.pad;
    xbase[f] = (((int)img * p.h + hi0) * p.w + wi0) * p.xps;     // may be negative where tap (0,0) is padding
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
  const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc((void*)p.x, (short)0, p.x_bytes, 0x00027000);

  // channel chunks of the two phases for this channel block (see DirectPlan)
  const int bfirst = p.groups > 1 ? (((grp0 >> 1) * 64) / p.cpg) * p.c_base / p.ch : 0;
  const int gap_s = p.gap_len ? bfirst : 0;
  i32x4 bmask;                                      // bytes of the chunk that straddles the end of the base group that belong to it
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int n = p.strad - 4 * e;
    bmask[e] = n >= 4 ? -1 : n <= 0 ? 0 : (int)((1u << (8 * n)) - 1u);
  }
  const bool gated = (p.flags & kGated) != 0, gate_only = (p.flags & kGateOnly) != 0;

  // K steps [k0, k1) of phase ph into a
  auto walk = [&](int ph, int k0, int k1, acc4 (&a)[PF][CG][2]) __attribute__((always_inline)) {
    if (k0 >= k1) return;
    const int nq = ph ? p.chunks1 : p.chunks0;
    const int cfirst = ph ? 0 : bfirst;
    const size_t wgrp = (size_t)(ph ? p.ks1 : p.ks0) * 2048;
    const char* wp = (ph ? p.w1 : p.w0) + (size_t)grp0 * wgrp + lane * 16;
    const int dt = 4 / nq, di = 4 - dt * nq;        // a K step on: so many taps and chunks on
    int tap, ci;                                    // this lane group's unit of the next step
    {
      const unsigned u = 4u * (unsigned)k0 + (unsigned)lg;
      tap = (int)(u / (unsigned)nq);
      ci = (int)u - tap * nq;
    }
    const int rowb = p.w * p.xps, q0 = ph ? 0 : nq - 1;
    int k = k0;
    i32x4 x[2][kU][PF], w[2][kU][CG][2];
    bool cut[2][kU];                                // the step's unit is the straddling chunk (the mask is applied where the
                                                    // operand is used: at the load it would wait for it)
    auto fetch = [&](auto bt) __attribute__((always_inline)) {
      constexpr int b = decltype(bt)::value;
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        const char* wk = wp + (size_t)(k < k1 ? k : k1 - 1) * 2048;
#pragma unroll
        for (int c = 0; c < CG; ++c)
#pragma unroll
          for (int h = 0; h < 2; ++h) w[b][u][c][h] = *(const i32x4*)(wk + c * wgrp + h * 1024);
        int c = cfirst + ci;
        if (ph) c += c >= gap_s ? p.gap_len : 0;
        const int t = tap < 9 ? tap : 9;            // (bit 9 and up of the validity mask are zero)
        const int r = (t * 11) >> 5, s = t - 3 * r;
        // a chunk that does not exist: an offset beyond any x (the plan keeps x below 1 GiB)
        const unsigned off = k < k1 && c < p.total_chunks ? (unsigned)(__mul24(r, rowb) + __mul24(s, p.xps) + c * 16) : 0x80000000u;
#pragma unroll
        for (int f = 0; f < PF; ++f) {
          const unsigned o = ((vmask[f] >> t) & 1u) ? (unsigned)xbase[f] + off : 0xffffffffu;
          x[b][u][f] = __builtin_bit_cast(i32x4, __builtin_amdgcn_raw_buffer_load_b128(xr, (int)o, 0, 0));
        }
        cut[b][u] = ci == q0;
        ++k;
        tap += dt;
        ci += di;
        if (ci >= nq) {
          ci -= nq;
          ++tap;
        }
      }
    };
    auto mul = [&](auto bt) __attribute__((always_inline)) {
      constexpr int b = decltype(bt)::value;
      if (p.strad) {
#pragma unroll
        for (int u = 0; u < kU; ++u)
#pragma unroll
          for (int f = 0; f < PF; ++f)
#pragma unroll
            for (int e = 0; e < 4; ++e) x[b][u][f][e] &= cut[b][u] ? (ph ? ~bmask[e] : bmask[e]) : -1;
      }
#pragma unroll
      for (int u = 0; u < kU; ++u)
#pragma unroll
        for (int f = 0; f < PF; ++f)
#pragma unroll
          for (int c = 0; c < CG; ++c)
#pragma unroll
            for (int h = 0; h < 2; ++h) a[f][c][h] = Tr::mma(w[b][u][c][h], x[b][u][f], a[f][c][h]);
    };
    using B0 = std::integral_constant<int, 0>;
    using B1 = std::integral_constant<int, 1>;
    const int nb = (k1 - k0 + kU - 1) / kU;
    fetch(B0{});
#pragma nounroll
    for (int i = 0; i < nb; i += 2) {
      if (i + 1 < nb) fetch(B1{});
      mul(B0{});
      if (i + 1 < nb) {
        if (i + 2 < nb) fetch(B0{});
        mul(B1{});
      }
    }
    if constexpr (MIXED) {
      bool nan = false;
#pragma unroll
      for (int f = 0; f < PF; ++f)
#pragma unroll
        for (int c = 0; c < CG; ++c)
#pragma unroll
          for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int e = 0; e < 4; ++e) nan |= a[f][c][h][e] != a[f][c][h][e];
      if (__ballot(nan) == 0ull) return;
      // (a lane's rows are 8*lg .. 8*lg + 7 of each group; the unit, and with it the channel, is the same for all lanes)
      int row_grp[CG][2][4];
#pragma unroll
      for (int c = 0; c < CG; ++c)
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            row_grp[c][h][e] = ((grp0 + c) * 32 + 8 * lg + 4 * h + e) / p.cpg;
#pragma unroll
            for (int f = 0; f < PF; ++f) a[f][c][h][e] = 0.0f;
          }
#pragma nounroll
      for (int u = 4 * k0; u < 4 * k1; ++u) {
        const int t = u / nq, chunk = cfirst + u - t * nq, r = (t * 11) >> 5;
        if (t >= p.taps || chunk >= p.total_chunks) continue;
        i32x4 xv[PF];
#pragma unroll
        for (int f = 0; f < PF; ++f) {
          const int off = xbase[f] + r * rowb + (t - 3 * r) * p.xps + chunk * 16;
          xv[f] = __builtin_bit_cast(i32x4, __builtin_amdgcn_raw_buffer_load_b128(xr, ((vmask[f] >> t) & 1u) ? off : -1, 0, 0));
        }
        int ch_grp[Tr::kCh];
#pragma unroll
        for (int i = 0; i < Tr::kCh; ++i) ch_grp[i] = (chunk * Tr::kCh + i) / p.c_base;
        const char* wu = wp - lane * 16 + (size_t)(u >> 2) * 2048 + (u & 3) * 256 + lg * 64;
#pragma unroll
        for (int c = 0; c < CG; ++c)
#pragma unroll
          for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const i32x4 wv = *(const i32x4*)(wu + c * wgrp + h * 1024 + e * 16);
#pragma unroll
              for (int i = 0; i < Tr::kCh; ++i) {
                const bool on = (ch_grp[i] == row_grp[c][h][e]) == (ph == 0);
#pragma unroll
                for (int f = 0; f < PF; ++f) {
                  const float old = a[f][c][h][e];
                  a[f][c][h][e] = on ? fmaf(Tr::element(xv[f], i), Tr::element(wv, i), old) : old;
                }
              }
            }
      }
    }
  };
  auto zero = [&](acc4 (&a)[PF][CG][2]) __attribute__((always_inline)) {
#pragma unroll
    for (int f = 0; f < PF; ++f)
#pragma unroll
      for (int c = 0; c < CG; ++c)
#pragma unroll
        for (int h = 0; h < 2; ++h) a[f][c][h] = acc4{0, 0, 0, 0};
  };

  if constexpr (!SPLIT) {
    acc4 accP[PF][CG][2], accR[PF][CG][2];
    zero(accP);
    zero(accR);
    walk(0, 0, p.ks0, accP);
    unsigned d[PF][CG];                             // bit i: channel 8*lg + i of the group
#pragma unroll
    for (int f = 0; f < PF; ++f)
#pragma unroll
      for (int c = 0; c < CG; ++c) d[f][c] = 0u;
    Tab4<Base> t[CG][2];
#pragma unroll
    for (int c = 0; c < CG; ++c)
#pragma unroll
      for (int h = 0; h < 2; ++h) t[c][h].load(p, (grp0 + c) * 32 + 8 * lg + 4 * h);
    if (gated) {
      bool any = false;
#pragma unroll
      for (int f = 0; f < PF; ++f) {
        const long long m = m0 + 16 * f + lj;
#pragma unroll
        for (int c = 0; c < CG; ++c) {
          const int co0 = (grp0 + c) * 32 + 8 * lg;
          unsigned dd = 0u;
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            acc_t s[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) s[e] = accP[f][c][h][e];
            dd |= gate4<Base>(p, s, t[c][h], co0 + 4 * h) << (4 * h);
          }
          if (m >= p.m_total) dd = 0u;
          if (p.chan_mask && dd)
            dd &= (p.chan_mask[(long long)((unsigned)m / (unsigned)(p.ho * p.wo)) * p.words + grp0 + c] >> (8 * lg)) & 0xffu;
          d[f][c] = dd;
          any |= dd != 0u;
          if (p.bitmap && grp0 + c < p.words) {
            unsigned word = dd << (8 * lg);
            word |= (unsigned)__shfl_xor((int)word, 16, 64);
            word |= (unsigned)__shfl_xor((int)word, 32, 64);
            if (lg == 0 && m < p.m_total) p.bitmap[m * p.words + grp0 + c] = word;
          }
        }
      }
      if (gate_only) return;
      if (__ballot(any) != 0ull) walk(1, 0, p.ks1, accR);
    }
#pragma unroll
    for (int f = 0; f < PF; ++f) {
      const long long m = m0 + 16 * f + lj;
      if (m >= p.m_total) continue;
#pragma unroll
      for (int c = 0; c < CG; ++c)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          acc_t s[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const acc_t pv = accP[f][c][h][e], rv = accR[f][c][h][e];
            s[e] = pv + (((d[f][c] >> (4 * h + e)) & 1u) ? rv : (acc_t)0);
          }
          finish4<Base>(p, s, t[c][h], d[f][c] >> (4 * h), (grp0 + c) * 32 + 8 * lg + 4 * h, m);
        }
    }
  } else {
    // wavefronts [0, nwb) walk the base path, the others the conditional path; each its part of the slice
    const int nwb = p.nwb;
    const int ph = wave >= nwb ? 1 : 0;
    const int part = slice * (ph ? nw - nwb : nwb) + (ph ? wave - nwb : wave);
    const int parts = p.slices * (ph ? nw - nwb : nwb);
    const int ks = ph ? (gate_only ? 0 : p.ks1) : p.ks0;
    acc4 acc[PF][CG][2];
    zero(acc);
    // this wavefront's first unit of the tile's end: its tables arrive behind the sums
    const int un0 = wave < NU ? wave : 0;
    Tab4<Base> tab;
    tab.load(p, (grp0 + ((un0 >> 1) % CG)) * 32 + 8 * lg + 4 * (un0 & 1));
    walk(ph, part * ks / parts, (part + 1) * ks / parts, acc);
#pragma unroll
    for (int f = 0; f < PF; ++f)
#pragma unroll
      for (int c = 0; c < CG; ++c)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          i32x4 v;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const acc_t sv = acc[f][c][h][e];
            v[e] = bits_of(sv);
          }
          ex[(wave * NU + (f * CG + c) * 2 + h) * 64 + lane] = v;
        }
    if (tid < PF * 16 * CG) words[tid] = 0u;
    __syncthreads();
    for (int un = wave; un < NU; un += nw) {
      const int h = un & 1, c = (un >> 1) % CG, f = (un >> 1) / CG;
      acc_t s[4] = {0, 0, 0, 0}, r[4] = {0, 0, 0, 0};
      auto add_up = [&](int wa, int wb, acc_t (&to)[4]) __attribute__((always_inline)) {
#pragma nounroll
        for (int w = wa; w < wb; w += 2) {          // two wavefronts' sums at a time
          const i32x4 v0 = ex[(w * NU + un) * 64 + lane], v1 = ex[((w + 1 < wb ? w + 1 : w) * NU + un) * 64 + lane];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            acc_t t0, t1;
            set_bits(v0[e], t0);
            set_bits(v1[e], t1);
            to[e] += t0;
            to[e] += w + 1 < wb ? t1 : (acc_t)0;
          }
        }
      };
      add_up(0, nwb, s);
      add_up(nwb, nw, r);
      if (p.slices > 1) {
        // [slice][tile][unit][base, conditional][lane]
        i32x4* out = p.partial + ((((size_t)slice * p.px_wgs + pt) * p.n_cblk + cbk) * NU + un) * 128 + lane;
        out[0] = i32x4{bits_of(s[0]), bits_of(s[1]), bits_of(s[2]), bits_of(s[3])};
        if (gated) out[64] = i32x4{bits_of(r[0]), bits_of(r[1]), bits_of(r[2]), bits_of(r[3])};
      } else {
        const int co0 = (grp0 + c) * 32 + 8 * lg + 4 * h;
        if (un != un0) tab.load(p, co0);
        const int m = m0 + 16 * f + lj;
        finish_unit<Base>(p, s, r, tab, co0, m, m < p.m_total, &words[(f * 16 + lj) * CG + c]);
      }
    }
    if (p.slices == 1 && gated && p.bitmap) {
      __syncthreads();
      if (tid < PF * 16 * CG) {
        const long long m = m0 + tid / CG;
        const int gq = grp0 + tid % CG;
        if (gq < p.words && m < p.m_total) p.bitmap[m * p.words + gq] = words[tid];
      }
    }
  }
}

// The end of the layer for tiles whose K was split over several workgroups: one workgroup per tile, a
// wavefront per unit.
template <typename Tr, int PF, int CG>
__global__ __launch_bounds__(PF * CG * 128) void direct_finish_kernel(DirectArgs p) {
  using Base = typename Tr::Base;
  using acc_t = typename Tr::acc_t;
  constexpr int NU = PF * CG * 2;
  __shared__ uint32_t words[PF * 16 * CG];
  load_args(p);
  const int tid = threadIdx.x, lane = tid & 63, lj = lane & 15, lg = lane >> 4;
  const int un = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int pt = (int)quot(blockIdx.x, p.n_cblk, p.magic_cblk), cbk = blockIdx.x - pt * p.n_cblk;
  const int h = un & 1, c = (un >> 1) % CG, f = (un >> 1) / CG;
  const int co0 = (cbk * CG + c) * 32 + 8 * lg + 4 * h;
  const bool gated = (p.flags & kGated) != 0;
  if (tid < PF * 16 * CG) words[tid] = 0u;
  Tab4<Base> tab;
  tab.load(p, co0);
  acc_t s[4] = {0, 0, 0, 0}, r[4] = {0, 0, 0, 0};
  const size_t step = (size_t)p.px_wgs * p.n_cblk * NU * 128;
  const i32x4* in = p.partial + ((size_t)blockIdx.x * NU + un) * 128 + lane;
  for (int z0 = 0; z0 < p.slices; z0 += 4) {        // (slices is a power of two)
    i32x4 a[4], b[4];
#pragma unroll
    for (int z = 0; z < 4; ++z) {
      a[z] = b[z] = i32x4{0, 0, 0, 0};
      if (z0 + z < p.slices) {
        a[z] = in[(z0 + z) * step];
        if (gated) b[z] = in[(z0 + z) * step + 64];
      }
    }
#pragma unroll
    for (int z = 0; z < 4; ++z)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        acc_t t;
        set_bits(a[z][e], t);
        s[e] += t;
        set_bits(b[z][e], t);
        r[e] += t;
      }
  }
  __syncthreads();
  const int m = pt * (16 * PF) + 16 * f + lj;
  finish_unit<Base>(p, s, r, tab, co0, m, m < p.m_total, &words[(f * 16 + lj) * CG + c]);
  if (gated && p.bitmap) {
    __syncthreads();
    if (tid < PF * 16 * CG) {
      const long long mp = (long long)pt * (16 * PF) + tid / CG;
      const int gq = cbk * CG + tid % CG;
      if (gq < p.words && mp < p.m_total) p.bitmap[mp * p.words + gq] = words[tid];
    }
  }
}

// [c_out][taps][c] in the caller's two weight arrays -> [32-channel group][K step][half][lane][16 bytes] of
// one phase.  Lane l holds row l%16 of its half h (channel 8*(row/4) + 4*h + row%4 of the group, which puts 8
// consecutive channels in one lane of the transposed product) and unit 4k + l/16.  Elements that are
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
  const int row = lane & 15, co = grp * 32 + 8 * (row >> 2) + 4 * h + (row & 3);
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

template <typename Tr, int PF, int CG, bool MIXED>
hipError_t launch_direct_form(const DirectPlan& g, const DirectArgs& a, hipStream_t s) {
  const dim3 grid((unsigned)a.per_xcd * 8u);
  if (g.split == 1)
    hipLaunchKernelGGL((gated_conv_direct_kernel<Tr, PF, CG, false, MIXED>), grid, dim3(256), 0, s, a);
  else
    hipLaunchKernelGGL((gated_conv_direct_kernel<Tr, PF, CG, true, MIXED>), grid, dim3(64 * g.split), 0, s, a);
  return hipGetLastError();
}

template <typename Tr, int PF, int CG>
hipError_t launch_direct_tile(const DirectPlan& g, const DirectArgs& a, hipStream_t s) {
  hipError_t e;
  if constexpr (Tr::Base::kDtype == CG_I8)
    e = launch_direct_form<Tr, PF, CG, false>(g, a, s);
  else
    e = g.mixed ? launch_direct_form<Tr, PF, CG, true>(g, a, s) : launch_direct_form<Tr, PF, CG, false>(g, a, s);
  if (e != hipSuccess || g.slices == 1) return e;
  hipLaunchKernelGGL((direct_finish_kernel<Tr, PF, CG>), dim3((unsigned)(g.px_wgs * g.n_cblk)), dim3(PF * CG * 128), 0, s, a);
  return hipGetLastError();
}

template <typename Tr>
hipError_t launch_direct_dtype(const DirectPlan& g, const DirectArgs& a, hipStream_t s) {
  if (g.pf == 2 && g.cg == 2) return launch_direct_tile<Tr, 2, 2>(g, a, s);
  if (g.pf == 2 && g.cg == 1) return launch_direct_tile<Tr, 2, 1>(g, a, s);
  if (g.pf == 1 && g.cg == 2) return launch_direct_tile<Tr, 1, 2>(g, a, s);
  if (g.pf == 1 && g.cg == 1) return launch_direct_tile<Tr, 1, 1>(g, a, s);
  return hipErrorInvalidValue;
}

// ceil(2^32 / d) if that gives the exact quotient of every x <= most, else 0
unsigned magic_upto(long long most, int d) {
  if (d <= 1 || most * d >= (1ll << 32)) return 0u;
  return (unsigned)(((1ull << 32) + (unsigned)d - 1) / (unsigned)d);
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
  if (groups == 1) {
    g.chunks[0] = (d.c_base + g.ch - 1) / g.ch;
    g.gap_len = d.c_base / g.ch;
    g.strad = (d.c_base % g.ch) * g.elem_bytes;
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
  }
  g.chunks[1] = gated ? g.total_chunks - g.gap_len : 0;
  for (int ph = 0; ph < 2; ++ph) {
    g.ksteps[ph] = (g.chunks[ph] * g.taps + 3) / 4;
    g.wpk_bytes[ph] = (size_t)g.n_grp * g.ksteps[ph] * 2048;
  }
  const int ks = g.ksteps[0] + g.ksteps[1];

  // Tile shape and K split: the largest tile (it costs the vector-memory path least per product) that
  // gives every compute unit a workgroup's worth of K steps, K split as far as needed.
  g.pf = m > 16 ? 2 : 1;
  g.cg = ngrp >= 2 ? 2 : 1;
  long long px = (m + 16 * g.pf - 1) / (16 * g.pf);
  g.n_cblk = (ngrp + g.cg - 1) / g.cg;
  const long long tiles = px * g.n_cblk;
  g.tiles = tiles < 0x7fffffffll ? (int)tiles : 0x7fffffff;
  g.split = 1;
  g.slices = 1;
  if (tiles < 8ll * n_cu) {
    while (g.split < kMaxSplit && tiles * g.split < 8ll * n_cu && ks / (2 * g.split) >= 2) g.split *= 2;
    if (g.split > 1) {
      while (2 * tiles * g.slices <= n_cu && ks / (2 * g.slices * g.split) >= 2 && g.slices < 16) g.slices *= 2;
      g.nwb = g.split;
      if (gated) {
        g.nwb = (g.split * g.ksteps[0] + ks / 2) / ks;
        if (g.nwb < 1) g.nwb = 1;
        if (g.nwb > g.split - 1) g.nwb = g.split - 1;
      }
    }
  }
  const long long wgs = g.split > 1 ? px : (px + 3) / 4;
  if (wgs * g.n_cblk * g.slices > 0x7ffffff0ll) return g;
  g.px_wgs = (int)wgs;
  if (g.slices > 1) g.partial_bytes = (size_t)g.slices * tiles * g.pf * g.cg * 2 * 2048;
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

hipError_t launch_direct(const DirectPlan& g, const Params& p, const void* w0, const void* w1, void* partial, hipStream_t s) {
  if (g.slices > 1 && !partial) return hipErrorInvalidValue;
  DirectArgs a{};
  a.x = p.x;
  a.w0 = (const char*)w0;
  a.w1 = (const char*)w1;
  a.tab = (const char*)p.thr_f;
  a.y = p.y;
  a.residual = p.residual;
  a.bitmap = p.bitmap;
  a.chan_mask = p.chan_mask;
  a.partial = (i32x4*)partial;
  a.total = p.total;
  a.tab_stride = (int)p.table_stride;
  a.x_bytes = (int)g.x_bytes;
  a.m_total = (int)p.m_total;
  a.wo = p.wo;
  a.ho = p.ho;
  a.h = p.h;
  a.w = p.w;
  a.xps = (int)p.x_pixel_stride * g.elem_bytes;
  a.magic_wo = magic_upto(p.m_total, p.wo);
  a.magic_ho = magic_upto(p.m_total, p.ho);
  a.n_wgs = g.px_wgs * g.n_cblk * g.slices;
  a.per_xcd = (a.n_wgs + 7) / 8;
  a.magic_cblk = magic_upto(a.n_wgs, g.n_cblk);
  a.magic_slices = magic_upto(a.n_wgs, g.slices);
  a.stride = p.stride;
  a.pad = p.pad;
  a.taps = g.taps;
  a.chunks0 = g.chunks[0];
  a.chunks1 = g.chunks[1];
  a.total_chunks = g.total_chunks;
  a.gap_len = g.gap_len;
  a.strad = g.strad;
  a.ks0 = g.ksteps[0];
  a.ks1 = g.ksteps[1];
  a.n_cblk = g.n_cblk;
  a.slices = g.slices;
  a.nwb = g.nwb;
  a.px_wgs = g.px_wgs;
  a.c_out = p.c_out;
  a.words = p.words;
  a.cpg = p.cpg;
  a.groups = p.groups;
  a.c_base = p.c_base;
  a.ch = g.ch;
  a.rq_shift = p.rq_shift;
  a.rq_res_mult = p.rq_res_mult;
  static_assert(kRelu == CG_EPI_RELU && kAffine == CG_EPI_AFFINE && kResidual == CG_EPI_RESIDUAL, "the epilogue flags pass through");
  a.flags = p.epilogue | (p.gated ? kGated : 0u) | (p.gate_only ? kGateOnly : 0u) | (p.clear_total ? kClear : 0u) |
            (p.shuffle ? kShuffle : 0u) | (p.out_dtype == CG_F32 || p.out_dtype == CG_I32 ? kOut4 : 0u);
  switch (p.in_dtype) {
    case CG_BF16: return launch_direct_dtype<Bf16Direct>(g, a, s);
    case CG_I8: return launch_direct_dtype<I8Direct>(g, a, s);
    default: return launch_direct_dtype<F32Direct>(g, a, s);
  }
}

}  // namespace cg
