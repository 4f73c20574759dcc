// The dense pieces of a ResNet around the gated layers (the paper evaluates ResNet-18, Sec. 5):
// the input convolution on few channels (7x7 stride 2 on RGB), 3x3 stride-2 max pooling and global
// average pooling followed by the fully connected layer.  None of them is gated.  bf16 activations
// and weights, fp32 accumulation.  Also the 1x1 stride-2 shortcut convolutions (cg_pointwise_conv), which are dense too.
#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>

#include "cg_mfma_common.h"
#include "point_piece.h"

namespace cg {
int set_error(int code, const char* fmt, ...);   // defined with the host API
}

namespace {

using cg::bf16_to_float;
using cg::float_to_bf16;

constexpr int kTile = 8;      // output pixels per block edge
constexpr int kCb = 64;       // output channels per block

// Direct convolution for c_in <= 4.  Block = 8x8 output pixels x 64 output channels, 256 threads:
// thread (px, g) accumulates channels [16g, 16g+16) of pixel px.  A wavefront holds one g and 64
// pixels, so its weight reads are LDS broadcasts and its input reads are one word per lane.
__global__ __launch_bounds__(256) void small_cin_conv_kernel(const uint16_t* __restrict__ x,
                                                             const uint16_t* __restrict__ w,
                                                             const float* __restrict__ scale,
                                                             const float* __restrict__ shift, uint16_t* __restrict__ y,
                                                             int n, int h, int wd, int c_in, int c_out, int k, int stride,
                                                             int pad, int ho, int wo, int relu) {
  extern __shared__ float lds[];
  const int taps = k * k * c_in;
  float* wl = lds;                          // [taps][64]
  const int pe = (kTile - 1) * stride + k;  // patch edge
  float* xl = lds + taps * kCb;             // [pe][pe][c_in]
  const int tid = threadIdx.x;
  const int tiles_w = (wo + kTile - 1) / kTile, tiles_h = (ho + kTile - 1) / kTile;
  int b = blockIdx.x;
  const int tw = b % tiles_w;
  b /= tiles_w;
  const int th = b % tiles_h;
  const int img = b / tiles_h;
  const int cb = blockIdx.y;

  // weights of this channel block: caller layout [c_out][k][k][c_in] -> [tap][channel]
  for (int i = tid; i < taps * kCb; i += 256) {
    const int co = i / taps, t = i - co * taps;
    wl[t * kCb + co] = bf16_to_float(w[(long long)(cb * kCb + co) * taps + t]);
  }
  // input patch, zero outside the image
  const int h0 = th * kTile * stride - pad, w0 = tw * kTile * stride - pad;
  for (int i = tid; i < pe * pe * c_in; i += 256) {
    const int c = i % c_in, q = i / c_in;
    const int pw = q % pe, ph = q / pe;
    const int hi = h0 + ph, wi = w0 + pw;
    float v = 0.0f;
    if (hi >= 0 && hi < h && wi >= 0 && wi < wd) v = bf16_to_float(x[(((long long)img * h + hi) * wd + wi) * c_in + c]);
    xl[i] = v;
  }
  __syncthreads();

  const int px = tid & 63, g = tid >> 6;
  const int oh = px / kTile, ow = px % kTile;
  float acc[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = 0.0f;
  const float* xp = xl + ((oh * stride) * pe + ow * stride) * c_in;
  const int row_taps = k * c_in;            // contiguous taps of one kernel row
  for (int r = 0; r < k; ++r) {
    const float* xr = xp + r * pe * c_in;
    const float* wr = wl + (r * row_taps) * kCb + g * 16;
    for (int t = 0; t < row_taps; ++t) {
      const float xv = xr[t];
      const float4 w0v = *(const float4*)(wr + t * kCb);
      const float4 w1v = *(const float4*)(wr + t * kCb + 4);
      const float4 w2v = *(const float4*)(wr + t * kCb + 8);
      const float4 w3v = *(const float4*)(wr + t * kCb + 12);
      acc[0] = fmaf(xv, w0v.x, acc[0]);
      acc[1] = fmaf(xv, w0v.y, acc[1]);
      acc[2] = fmaf(xv, w0v.z, acc[2]);
      acc[3] = fmaf(xv, w0v.w, acc[3]);
      acc[4] = fmaf(xv, w1v.x, acc[4]);
      acc[5] = fmaf(xv, w1v.y, acc[5]);
      acc[6] = fmaf(xv, w1v.z, acc[6]);
      acc[7] = fmaf(xv, w1v.w, acc[7]);
      acc[8] = fmaf(xv, w2v.x, acc[8]);
      acc[9] = fmaf(xv, w2v.y, acc[9]);
      acc[10] = fmaf(xv, w2v.z, acc[10]);
      acc[11] = fmaf(xv, w2v.w, acc[11]);
      acc[12] = fmaf(xv, w3v.x, acc[12]);
      acc[13] = fmaf(xv, w3v.y, acc[13]);
      acc[14] = fmaf(xv, w3v.z, acc[14]);
      acc[15] = fmaf(xv, w3v.w, acc[15]);
    }
  }
  const int oy = th * kTile + oh, ox = tw * kTile + ow;
  if (oy < ho && ox < wo) {
    const int co0 = cb * kCb + g * 16;
    uint16_t out[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      float a = acc[i];
      if (scale) a *= scale[co0 + i];
      if (shift) a += shift[co0 + i];
      if (relu) a = fmaxf(a, 0.0f);
      out[i] = float_to_bf16(a);
    }
    uint4* dst = (uint4*)(y + (((long long)img * ho + oy) * wo + ox) * c_out + co0);
    dst[0] = *(const uint4*)(out);
    dst[1] = *(const uint4*)(out + 8);
  }
}

typedef __attribute__((ext_vector_type(8))) __bf16 stem_bf16x8;
typedef __attribute__((ext_vector_type(16))) float stem_f32x16;
typedef __attribute__((ext_vector_type(4))) int stem_i32x4;

// two floats as bf16 (round to nearest even), a in the low half
__device__ __forceinline__ uint32_t bf16_pair(float a, float b) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
}

// The ImageNet input layer's shape (7x7, stride 2, three input channels) on the matrix cores, with (POOL) the 3x3
// stride-2 max pooling (padding 1) that follows it in a ResNet.
//
// A workgroup of two wavefronts walks down a band of output rows.  A wavefront holds the weights of 64 (NFC = 2) or 32
// channels in registers (K = 7 kernel rows x 24 elements, 88 or 44 registers) and multiplies, per row of the layer's output, two
// fragments of 32 columns: the even columns 2*pc and the odd ones 2*pc + 1 of the pooled columns pc = first - 1 + lane.
// A pooled value is then the maximum of a lane's even column, its odd column and its left neighbour's odd column
// (lane 0 is there for that only), over three rows of which the last is kept for the next pooled row: the layer is
// computed once, but for one row per band and two columns per fragment.  The product is taken with the weights as the
// row operand and their rows permuted (row rho holds channel 16*((rho/4)%2) + 4*(rho/8) + rho%4), which leaves every
// lane with 16 consecutive channels of one pixel per accumulator.
//
// Rows of the input lie in a ring of LDS rows; the next step's four are loaded while this step's are multiplied.  Within a
// kernel row a pixel's 21 values (column, channel) are contiguous; with an odd padding one element before them is
// taken as well (zero weight), so that every read starts on a word; 24 elements = three 16-byte chunks, 22 chunks
// (the last one zero) = 11 K steps of 16.
//
// Maxima of sums instead of outputs: the output function is monotone in the sum, rising where the scale is not negative;
// channels with a negative scale take negated weights and the scale's magnitude (both exact).
//
// What bounds it: two wavefronts to a SIMD are not enough to keep anything busy: the matrix cores (44 instructions of 32 clocks per output row
// and 28 pooled columns) are for 41 % of the time, LDS for 43 % (a quarter of that conflicts), and a wavefront waits for operands or the other
// one's products for the rest; its 250 registers, half of them weights and sums, allow no third.  Images of 224x224 with pooling: 256 in
// 84 us, 64 in 35, 16 in 17; 240, 66 and 22 in the form before (16x16 tiles gathered as single elements, 1.31 times
// the products, outputs exchanged through LDS for the pooling).
constexpr int kStemPitch = 1664;                 // bytes of a ring row: 63 pooled columns' input and the window's rest
constexpr int kStemRing = 16;
constexpr int kStemPieces = kStemPitch / 16 - 1; // 16-byte pieces of a row
constexpr int kStemCols = 31;                    // pooled columns of a fragment, at most

struct StemArgs {
  const uint16_t* x;
  const uint16_t* w;
  const float* scale;
  const float* shift;
  uint16_t* y;
  int h, wd, c_out, pad, ho, wo, relu;
  int oh, ow;                                    // output of the kernel: pooled, or column pairs and row pairs of the layer's
  int cpf, col_wgs;                              // pooled columns per wavefront; workgroups across the columns
  int band, bands;                               // pooled rows per workgroup; workgroups across the rows
};

struct __attribute__((packed, aligned(2))) StemPiece {
  stem_i32x4 v;
};

// RAGGED: rows that are not whole 16-byte pieces (the others have no instruction for it: one image of 224x224 6.6 us with, 6.1 without)
template <bool POOL, int NFC, bool RAGGED>
__global__ __launch_bounds__(128, 2) void conv7x7s2c3_kernel(StemArgs a) {
  constexpr int K = 7, CI = 3, TAPS = K * K * CI, ST = 11, CB = 32 * NFC;
  __shared__ __align__(16) char ring[kStemRing * kStemPitch];   // first the weights, then input rows
  __shared__ __align__(16) float tab[2 * CB];                  // |scale|, shift
  __shared__ __align__(16) int fillers[2][4];                   // the 22nd chunk of a pixel: zeros; -inf, zeros
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lj = lane & 31, lh = lane >> 5;
  const int cb = blockIdx.y;
  int b = blockIdx.x;
  const int cw = b % a.col_wgs;
  b /= a.col_wgs;
  const int p0 = (b % a.bands) * a.band, img = b / a.bands;
  const int p1 = p0 + a.band < a.oh ? p0 + a.band : a.oh;

  // ---- rows of the input: 16-byte piece t of row `hi` by thread t.  A ring row starts (16 bytes in) with element el0 of
  // the image's row; pieces start at multiples of eight elements, so that no piece straddles the image's left edge.
  const int lead = a.pad & 1;                    // elements before the window
  const int first = cw * 2 * a.cpf;              // first pooled column of the workgroup
  const int el0 = (4 * (first - 1) - a.pad) * CI - lead, row_els = a.wd * CI;
  const int piece0 = (el0 & ~7) + tid * 8;       // first element of this thread's piece
  const uint16_t* const ximg = a.x + (long long)img * a.h * row_els;
  const bool in_row = tid < kStemPieces && piece0 >= 0 && piece0 + 8 <= row_els;
  // The piece that a row ends in (rows of whole pieces have none) is taken from the row's last eight elements and moved down when it is kept; rows of
  // fewer are put together from single ones.  (Every such piece from single ones, each waited for, us: 64 images of 223x223 47.8, now 35.4; 140 of
  // 201x201 98.4, now 68.4; 8 of 97x97 11.4, now 8.3.)
  const bool cut = RAGGED && tid < kStemPieces && piece0 < row_els && piece0 + 8 > row_els;
  const bool whole = in_row || (cut && row_els >= 8);
  const int from = cut ? row_els - 8 : piece0, down = cut && row_els >= 8 ? 8 - (row_els & 7) : 0;
  auto load_piece = [&](int hi) __attribute__((always_inline)) {
    stem_i32x4 v = {0, 0, 0, 0};
    if ((unsigned)hi < (unsigned)a.h) {
      const uint16_t* const row = ximg + (long long)hi * row_els;
      if (whole) v = ((const StemPiece*)(row + from))->v;
      if (RAGGED && row_els < 8 && cut) {
#pragma nounroll
        for (int e = 0; e < row_els; ++e) {
          const int bits = (int)((uint32_t)row[e] << (16 * (e & 1)));
#pragma unroll
          for (int d = 0; d < 4; ++d) v[d] |= e >> 1 == d ? bits : 0;
        }
      }
    }
    return v;
  };
  auto keep_piece = [&](int hi, stem_i32x4 v) __attribute__((always_inline)) {
    if constexpr (RAGGED) {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = down & 4 ? (e < 2 ? v[e + 2] : 0) : v[e];
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = down & 2 ? (e < 3 ? v[e + 1] : 0) : v[e];
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = down & 1 ? (int)__builtin_amdgcn_alignbit(e < 3 ? (uint32_t)v[e + 1] : 0u, (uint32_t)v[e], 16) : v[e];
    }
    if (tid < kStemPieces) {                     // (el0 is even)
      int* dst = (int*)(ring + ((hi + 64) & (kStemRing - 1)) * kStemPitch + 16 + (piece0 - el0) * 2);
#pragma unroll
      for (int e = 0; e < 4; ++e) dst[e] = v[e];
    }
  };
  // output row r of the layer reads input rows 2r - pad .. + 6; the first step's rows start at r = 2*p0 - 1
  const int hi0 = (POOL ? 4 * p0 - 2 : 4 * p0) - a.pad;
  constexpr int NFIRST = POOL ? 11 : 9;
  stem_i32x4 fill[NFIRST];
#pragma unroll
  for (int k = 0; k < NFIRST; ++k) fill[k] = load_piece(hi0 + k);

  // ---- weights through LDS: [chunk][row][8 elements]; a thread lays out a kernel row of a channel at a time (three
  // chunks from 24 elements of which the first and last ones may be its neighbours': those become zero)
  {
    constexpr int ROWS = CB * K, PER = (ROWS + 127) / 128;
    const uint16_t* wsrc = a.w + (long long)cb * CB * TAPS - lead;
    stem_i32x4 v[PER][3];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int pr = tid + 128 * u;              // = channel * 7 + kernel row
#pragma unroll
      for (int part = 0; part < 3; ++part) v[u][part] = stem_i32x4{0, 0, 0, 0};
      if (pr > 0 && pr < ROWS - 1) {
#pragma unroll
        for (int part = 0; part < 3; ++part) v[u][part] = ((const StemPiece*)(wsrc + pr * (K * CI) + part * 8))->v;
      } else if (pr < ROWS) {                    // the ends of the array
#pragma unroll
        for (int e = 0; e < K * CI; ++e) {
          const uint32_t el = (uint32_t)wsrc[pr * (K * CI) + e + lead];
          const uint32_t even = el << (16 * (e & 1)), odd = el << (16 * ((e + 1) & 1));   // without and with the lead
          v[u][e / 8][e % 8 / 2] |= lead ? 0 : (int)even;
          v[u][(e + 1) / 8][(e + 1) % 8 / 2] |= lead ? (int)odd : 0;
        }
      }
    }
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int pr = tid + 128 * u;
      if (pr >= ROWS) break;
      const int co = pr / K, kr = pr - co * K, ch = co & 31;
      const int row = (co & 32) + 8 * ((ch & 15) >> 2) + 4 * (ch >> 4) + (ch & 3);   // inverse of the row permutation
      const int flip = a.scale && a.scale[cb * CB + co] < 0.0f ? (int)0x80008000u : 0;
      v[u][0][0] &= lead ? (int)0xffff0000u : -1;
      v[u][2][2] &= lead ? -1 : 0xffff;          // elements 21 + lead and on
      v[u][2][3] = 0;
#pragma unroll
      for (int part = 0; part < 3; ++part) {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[u][part][e] ^= flip;
        *(stem_i32x4*)(ring + ((3 * kr + part) * CB + row) * 16) = v[u][part];
      }
    }
    if (tid < CB) {
      tab[tid] = a.scale ? fabsf(a.scale[cb * CB + tid]) : 1.0f;
      tab[CB + tid] = a.shift ? a.shift[cb * CB + tid] : 0.0f;
    }
    if (tid < 8) fillers[tid >> 2][tid & 3] = tid == 4 ? 0xff80 : 0;
  }
  __syncthreads();
  stem_i32x4 wf[ST][NFC];
#pragma unroll
  for (int st = 0; st < ST; ++st)
#pragma unroll
    for (int fc = 0; fc < NFC; ++fc) {
      // this lane half's chunk: kernel rows 0..2 and 3..5 side by side, then row 6; the 22nd chunk is 1, 0, 0, ...
      const int q = st < 9 ? st + 9 * lh : st == 9 ? 18 + 2 * lh : 19;
      wf[st][fc] = *(const stem_i32x4*)(ring + (q * CB + 32 * fc + lj) * 16);
      if (st == ST - 1 && lh) wf[st][fc] = stem_i32x4{0x3f80, 0, 0, 0};
    }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < NFIRST; ++k) keep_piece(hi0 + k, fill[k]);
  __syncthreads();

  const int pc = first + wave * a.cpf - 1 + lj;  // this lane's pooled column
  const int pcc = pc < a.ow ? pc : a.ow - 1;     // (lanes past the last one read its input)
  const int col = 16 + (pcc - first + 1) * (4 * CI * 2);        // bytes from the ring row's start to the even column's window
  const bool odd_in = 2 * pc + 1 >= 0 && 2 * pc + 1 < a.wo;     // the odd column lies inside the layer's output
  const bool mine = lj >= 1 && lj <= a.cpf && pc < a.ow;        // this lane writes

  // sums of row r: even and odd columns
  auto row_sums = [&](int r, stem_f32x16 (&acc)[2][NFC]) __attribute__((always_inline)) {
#pragma unroll
    for (int o = 0; o < 2; ++o)
#pragma unroll
      for (int fc = 0; fc < NFC; ++fc)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[o][fc][i] = 0.0f;
    const int top = 2 * r - a.pad + 64;
    auto row_at = [&](int kr) __attribute__((always_inline)) { return ((top + kr) & (kStemRing - 1)) * kStemPitch; };
    // (the odd columns' addresses are hidden from the compiler: it would read what the two have in common once and copy
    // it into place, which needs the value at once)
    unsigned at[4], at1[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      at[k] = (unsigned)(col + (k == 3 ? row_at(6) : lh ? row_at(k + 3) : row_at(k)));
      at1[k] = at[k] + 2 * CI * 2;
      asm("" : "+v"(at1[k]));
    }
    // operands of two K steps ahead are on their way while a step is multiplied
    stem_i32x4 even[3], odd[3];
    auto read_step = [&](int st) __attribute__((always_inline)) {
      const int k = st / 3 < 3 ? st / 3 : 3, ofs = st < 9 ? st % 3 * 16 : st == 9 ? 32 * lh : 16;
      const char *src = ring + at[k] + ofs, *src1 = ring + at1[k] + ofs;
      if (st == ST - 1) {
        src = lh ? (const char*)fillers[0] : src;
        src1 = lh ? (const char*)fillers[odd_in ? 0 : 1] : src1;
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        even[st % 3][e] = ((const int*)src)[e];
        odd[st % 3][e] = ((const int*)src1)[e];
      }
    };
    read_step(0);
    read_step(1);
#pragma unroll
    for (int st = 0; st < ST; ++st) {
      if (st + 2 < ST) read_step(st + 2);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int fc = 0; fc < NFC; ++fc) {
        acc[0][fc] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(stem_bf16x8, wf[st][fc]),
                                                             __builtin_bit_cast(stem_bf16x8, even[st % 3]), acc[0][fc], 0, 0, 0);
        acc[1][fc] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(stem_bf16x8, wf[st][fc]),
                                                             __builtin_bit_cast(stem_bf16x8, odd[st % 3]), acc[1][fc], 0, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto write = [&](const stem_f32x16 (&v)[NFC], uint16_t* dst) __attribute__((always_inline)) {
#pragma unroll
    for (int fc = 0; fc < NFC; ++fc) {
      uint32_t o[8];
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        const float4 sc = *(const float4*)(tab + 32 * fc + 16 * lh + 4 * q4);
        const float4 sh = *(const float4*)(tab + CB + 32 * fc + 16 * lh + 4 * q4);
        float r[4] = {fmaf(v[fc][4 * q4], sc.x, sh.x), fmaf(v[fc][4 * q4 + 1], sc.y, sh.y),
                      fmaf(v[fc][4 * q4 + 2], sc.z, sh.z), fmaf(v[fc][4 * q4 + 3], sc.w, sh.w)};
        if (a.relu) {
#pragma unroll
          for (int e = 0; e < 4; ++e) r[e] = fmaxf(r[e], 0.0f);
        }
        o[2 * q4] = bf16_pair(r[0], r[1]);
        o[2 * q4 + 1] = bf16_pair(r[2], r[3]);
      }
      ((uint4*)(dst + 32 * fc))[0] = uint4{o[0], o[1], o[2], o[3]};
      ((uint4*)(dst + 32 * fc))[1] = uint4{o[4], o[5], o[6], o[7]};
    }
  };
  // MFMA results may be read by inline assembly some wait states after the last one
  auto settle = [&]() __attribute__((always_inline)) {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  // the larger one of an odd column's sum and its left neighbour's (lane - 1; anything in lanes 0 and 32)
  auto with_left = [&](float odd) __attribute__((always_inline)) {
    float r;
    asm("v_max_f32_dpp %0, %1, %1 wave_shr:1 row_mask:0xf bank_mask:0xf" : "=v"(r) : "v"(odd));
    return r;
  };
  auto max2 = [&](float u, float v) __attribute__((always_inline)) {
    float r;
    asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(u), "v"(v));
    return r;
  };
  auto max3 = [&](float u, float v, float w) __attribute__((always_inline)) {
    float r;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(u), "v"(v), "v"(w));
    return r;
  };

  stem_f32x16 above[NFC];                        // the maxima of the row above the next pooled row's first own one
  stem_f32x16 acc[2][NFC];
  if constexpr (POOL) {
    if (p0 > 0) {
      row_sums(2 * p0 - 1, acc);
      settle();
#pragma unroll
      for (int fc = 0; fc < NFC; ++fc)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const float even = acc[0][fc][i], odd = acc[1][fc][i];
          above[fc][i] = max2(even, with_left(odd));
        }
    } else {
#pragma unroll
      for (int fc = 0; fc < NFC; ++fc)
#pragma unroll
        for (int i = 0; i < 16; ++i) above[fc][i] = -__builtin_inff();
    }
  }
  // No load is in flight from here on nor at the end of a step, as far as the compiler knows: those that only some of the threads keep were to it, and
  // it waited for the next rows' loads, or for a step's stores, before a step's first product.
  constexpr int kVmcnt0 = 0x0f70;
  __builtin_amdgcn_s_waitcnt(kVmcnt0);
#pragma nounroll
  for (int p = p0; p < p1; ++p) {
    stem_i32x4 next[4];
    const bool more = p + 1 < p1;
    if (more) {
#pragma unroll
      for (int k = 0; k < 4; ++k) next[k] = load_piece(4 * p + 9 - a.pad + k);
    }
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const int r = 2 * p + half;
      if (half == 1 && r >= a.ho) break;         // (the last pooled row of an odd height)
      row_sums(r, acc);
      // The next step's rows are kept here, ahead of this step's outputs, whose stores a wait for the loads would wait for too; their places are those
      // of rows 7 to 4 above this step's first, which nothing reads any more.
      if (half == 0) {
        __builtin_amdgcn_s_waitcnt(kVmcnt0);
        if (more) {
#pragma unroll
          for (int k = 0; k < 4; ++k) keep_piece(4 * p + 9 - a.pad + k, next[k]);
        }
      }
      if constexpr (POOL) {
        settle();
        const bool last = half == 1 || r + 1 >= a.ho;
        stem_f32x16 here[NFC];
#pragma unroll
        for (int fc = 0; fc < NFC; ++fc)
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            const float even = acc[0][fc][i], odd = acc[1][fc][i], up = above[fc][i];
            if (half == 0) {
              above[fc][i] = max3(up, even, with_left(odd));
            } else {
              const float m = max2(even, with_left(odd));
              here[fc][i] = m;
              above[fc][i] = max2(up, m);
            }
          }
        if (last) {
          if (mine) write(above, a.y + (((long long)img * a.oh + p) * a.ow + pc) * a.c_out + cb * CB + 16 * lh);
          if (half == 1) {
#pragma unroll
            for (int fc = 0; fc < NFC; ++fc) above[fc] = here[fc];
          }
        }
      } else {
        uint16_t* dst = a.y + (((long long)img * a.ho + r) * a.wo + 2 * pc) * a.c_out + cb * CB + 16 * lh;
        if (mine) write(acc[0], dst);
        if (mine && odd_in) write(acc[1], dst + a.c_out);
      }
    }
    if (more) __syncthreads();
  }
}

int launch_conv7x7s2c3(bool pool, const char* who, const void* x, const void* w, const float* scale, const float* shift,
                       void* y, int n, int h, int wd, int c_out, int pad, int relu, hipStream_t s) {
  StemArgs a{};
  a.x = (const uint16_t*)x;
  a.w = (const uint16_t*)w;
  a.scale = scale;
  a.shift = shift;
  a.y = (uint16_t*)y;
  a.h = h;
  a.wd = wd;
  a.c_out = c_out;
  a.pad = pad;
  a.relu = relu;
  a.ho = (h + 2 * pad - 7) / 2 + 1;
  a.wo = (wd + 2 * pad - 7) / 2 + 1;
  a.oh = pool ? (a.ho - 1) / 2 + 1 : (a.ho + 1) / 2;
  a.ow = pool ? (a.wo - 1) / 2 + 1 : (a.wo + 1) / 2;
  const int frags = (a.ow + kStemCols - 1) / kStemCols;
  a.cpf = (a.ow + frags - 1) / frags;
  a.col_wgs = (frags + 1) / 2;
  // Bands: a band computes one row more than it writes and lays out the weights anew, so long ones are better, as long as
  // the chip is full: a compute unit holds four workgroups.
  const long long per_row = (long long)n * a.col_wgs * (c_out / kCb), want = 4ll * cg::cu_count();
  long long bands = (want + per_row - 1) / per_row;
  if (bands > a.oh) bands = a.oh;
  a.band = (int)((a.oh + bands - 1) / bands);
  a.bands = (a.oh + a.band - 1) / a.band;
  const long long blocks = (long long)n * a.bands * a.col_wgs;
  if (blocks > 0x7fffffffll) return cg::set_error(CG_EUNSUPPORTED, "%s: too many tiles", who);
  // 32 channels a workgroup instead of 64, half of the products for a wavefront, where 64 would leave half of the chip idle:
  // images of 224x224 with pooling, one 8.8 -> 6.2 us, four 9.0 -> 8.0, eight 11.8 -> 11.1 (twelve are past the line).
  const bool narrow = 2 * blocks * (c_out / kCb) <= want, ragged = wd * 3 % 8 != 0;
  const auto kernel = narrow ? (pool ? (ragged ? conv7x7s2c3_kernel<true, 1, true> : conv7x7s2c3_kernel<true, 1, false>)
                                     : (ragged ? conv7x7s2c3_kernel<false, 1, true> : conv7x7s2c3_kernel<false, 1, false>))
                             : (pool ? (ragged ? conv7x7s2c3_kernel<true, 2, true> : conv7x7s2c3_kernel<true, 2, false>)
                                     : (ragged ? conv7x7s2c3_kernel<false, 2, true> : conv7x7s2c3_kernel<false, 2, false>));
  hipLaunchKernelGGL(kernel, dim3((unsigned)blocks, (unsigned)(c_out / (narrow ? 32 : kCb))), dim3(128), 0, s, a);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return cg::set_error(CG_EHIP, "%s: %s", who, hipGetErrorString(e));
  return CG_OK;
}

using cg::PointArgs;
using cg::point_pixel;
constexpr int kPointPx = 64;                       // pixels of a workgroup of pointwise_tile_kernel

// Few pixels: a workgroup of one wavefront does a piece (point_piece.h), all of up to eight K steps (256 channels) at once.
__global__ __launch_bounds__(64) void pointwise_small_kernel(PointArgs a) { cg::point_piece<8>(a, blockIdx.x, (int)blockIdx.y); }

// Many pixels: a workgroup of four wavefronts owns 64 pixels x 128 channels, a wavefront 32 of the channels.  The pixels go to LDS by
// direct loads, [K step of 32][pixel][four 16-byte chunks], all K steps at once; a wavefront's weights come straight from memory into
// registers, in batches of eight K steps (the compiler waits for all loads so far, the pixels' too, behind the second of a batch's; with all eight in flight
// the kernel takes 176 registers instead of 124).  Several workgroups fit a compute unit, so one's loads run under another's products.
// Chunk q of pixel p sits at position q ^ f(p / 4 % 4), f = 0, 2, 3, 1: each of the four groups of lanes that a 16-byte read is served in
// ({0-3, 12-15, 20-27}, the rest of the first 32, the same 32 lanes on) then covers every bank once.  Bound by the vector-memory path (weights and
// pixels in pieces of 64 bytes) and, with few channels, by memory.  ResNet-18's three shortcuts, 256 images 29.0, 20.8, 19.4 -> 22.6, 17.6, 15.1 us,
// 64 images 10.7, 8.8, 8.6 -> 8.6, 6.7, 6.1; 512 to 512 channels at 28x28, 256 images 112 -> 71.  (Before: 128 pixels x 64 channels a workgroup, the
// pixels in pieces of 32 bytes straight into registers, the weights in LDS, outputs in pieces of 32 bytes.)
__global__ __launch_bounds__(256) void pointwise_tile_kernel(PointArgs a) {
  constexpr int U = 8, PB = kPointPx / 16;
  extern __shared__ __align__(16) char point_lds[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lj = lane & 15, lg = lane >> 4;
  // block id mod 8 is the XCD: one takes a run of tiles with all their channel blocks, so that its L2 holds a tile's pixels once
  const unsigned rank = (blockIdx.x & 7) * (unsigned)a.per_xcd + (blockIdx.x >> 3);
  if (rank >= (unsigned)a.blocks) return;
  const unsigned tile = cg::quot(rank, a.d_ncb);
  const int c0 = (int)(rank - tile * (unsigned)a.ncb) * 128 + wave * 32;
  const unsigned m0 = tile * kPointPx;
  const int nq = a.c_in >> 3, steps = (nq + 3) >> 2;
  auto swap_of = [](int t) { return (t >> 1) | (((t ^ (t >> 1)) & 1) << 1); };
  {
    const unsigned m = m0 + 16 * wave + (lane >> 2);
    const char* const src = a.x + point_pixel(a, m < (unsigned)a.m_total ? m : m0);
    const int chunk = (lane & 3) ^ swap_of(lane >> 4);
    char* const dst = point_lds + wave * 1024;
    for (int st = 0; st < steps; ++st) {
      const int q = 4 * st + chunk < nq ? 4 * st + chunk : nq - 1;       // (chunks past the end: dropped where they are read)
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) unsigned*)(src + q * 16),
                                       (__attribute__((address_space(3))) unsigned*)(dst + st * (kPointPx * 64)), 16, 0, 0);
    }
  }
  const bool mine = c0 < a.c_out;                  // (c_out is a multiple of 64: the last block may have two idle wavefronts)
  // row r of block i holds channel 8 * (r / 4) + 4 * i + r % 4: a lane ends up with eight consecutive ones
  const char* const wr = a.w + (long long)((mine ? c0 : 0) + 8 * (lj >> 2) + (lj & 3)) * (a.c_in * 2) + lg * 16;
  const int w4 = 4 * a.c_in * 2;
  stem_i32x4 wv[U][2];
  auto fetch = [&](int s0) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      wv[u][0] = wv[u][1] = stem_i32x4{0, 0, 0, 0};
      if (4 * (s0 + u) + lg < nq) {                // (a last step of two chunks)
        wv[u][0] = *(const stem_i32x4*)(wr + (s0 + u) * 64);
        wv[u][1] = *(const stem_i32x4*)(wr + w4 + (s0 + u) * 64);
      }
    }
  };
  fetch(0);
  cg::f32x4 acc[PB][2], sc[2], sh[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int at = (mine ? c0 : 0) + 8 * lg + 4 * i;
    sc[i] = a.scale ? *(const cg::f32x4*)(a.scale + at) : cg::f32x4{1.0f, 1.0f, 1.0f, 1.0f};
    sh[i] = a.shift ? *(const cg::f32x4*)(a.shift + at) : cg::f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int b = 0; b < PB; ++b) acc[b][i] = cg::f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  }
  __syncthreads();
  if (!mine) return;
  const char* const at = point_lds + lj * 64 + (lg ^ swap_of(lj >> 2)) * 16;
  for (int s0 = 0; s0 < steps; s0 += U) {
    if (s0 > 0) fetch(s0);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (s0 + u >= steps) break;
      const bool on = 4 * (s0 + u) + lg < nq;
#pragma unroll
      for (int b = 0; b < PB; ++b) {
        stem_i32x4 xv = *(const stem_i32x4*)(at + (s0 + u) * (kPointPx * 64) + b * 1024);
        if (!on) xv = stem_i32x4{0, 0, 0, 0};
#pragma unroll
        for (int i = 0; i < 2; ++i)
          acc[b][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(stem_bf16x8, wv[u][i]), __builtin_bit_cast(stem_bf16x8, xv),
                                                              acc[b][i], 0, 0, 0);
      }
    }
  }
#pragma unroll
  for (int b = 0; b < PB; ++b) {
    const unsigned m = m0 + 16 * b + lj;
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      v[e] = acc[b][e >> 2][e & 3] * sc[e >> 2][e & 3] + sh[e >> 2][e & 3];
      if (a.relu) v[e] = fmaxf(v[e], 0.0f);
    }
    if (m < (unsigned)a.m_total)
      *(uint4*)(a.y + ((long long)m * a.c_out + c0 + 8 * lg) * 2) =
          uint4{bf16_pair(v[0], v[1]), bf16_pair(v[2], v[3]), bf16_pair(v[4], v[5]), bf16_pair(v[6], v[7])};
  }
}

// As many pixels where the kernel above would leave half of a last block's wavefronts idle (64 channels beyond a multiple of 128): a workgroup owns
// 128 pixels x 64 channels, a wavefront 32 of the pixels, which it takes straight from memory (16 bytes per lane and K step); the weights are in LDS,
// rows permuted so that a lane ends up with sixteen consecutive channels.
__global__ __launch_bounds__(256) void pointwise_conv_kernel(const uint16_t* __restrict__ x, const uint16_t* __restrict__ w,
                                                             const float* __restrict__ scale,
                                                             const float* __restrict__ shift, uint16_t* __restrict__ y,
                                                             long long m_total, int h, int wd, int c_in, int c_out,
                                                             int stride, int ho, int wo, int relu) {
  extern __shared__ __align__(16) uint16_t wlp[];          // [c_in/8 chunks][64 rows][8]
  const int tid = threadIdx.x;
  const int cb = blockIdx.y;
  const int nq = c_in >> 3;
  for (int i = tid; i < nq * kCb; i += 256) {
    const int col = i / nq, q = i - col * nq;            // consecutive threads read consecutive 16-byte pieces
    const int ch = col & 31;
    const int row = (col & 32) + 8 * ((ch & 15) >> 2) + 4 * (ch >> 4) + (ch & 3);
    *(uint4*)(wlp + ((q * kCb + row) << 3)) = *(const uint4*)(w + ((long long)(cb * kCb + col) * c_in + q * 8));
  }
  __syncthreads();
  const int lane = tid & 63, wave = tid >> 6;
  const int lj = lane & 31, lh = lane >> 5;
  const long long m = (long long)blockIdx.x * 128 + wave * 32 + lj;
  const bool valid = m < m_total;
  const long long mm = valid ? m : 0;
  const int ox = (int)(mm % wo);
  const long long t2 = mm / wo;
  const int oy = (int)(t2 % ho);
  const long long img = t2 / ho;
  const uint16_t* src = x + ((img * h + (long long)oy * stride) * wd + (long long)ox * stride) * c_in + lh * 8;
  stem_f32x16 acc[2];
#pragma unroll
  for (int fc = 0; fc < 2; ++fc)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[fc][i] = 0.0f;
  const int steps = c_in >> 4;
#pragma unroll 4
  for (int st = 0; st < steps; ++st) {
    stem_i32x4 b = {0, 0, 0, 0};
    if (valid) b = *(const stem_i32x4*)(src + st * 16);
    const int q = 2 * st + lh;
#pragma unroll
    for (int fc = 0; fc < 2; ++fc) {
      const stem_i32x4 a = *(const stem_i32x4*)(wlp + ((q * kCb + 32 * fc + lj) << 3));
      acc[fc] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(stem_bf16x8, a), __builtin_bit_cast(stem_bf16x8, b),
                                                        acc[fc], 0, 0, 0);
    }
  }
  if (!valid) return;
#pragma unroll
  for (int fc = 0; fc < 2; ++fc) {
    const int co0 = cb * kCb + 32 * fc + 16 * lh;
    uint16_t out[16];
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      const float4 a4 = scale ? *(const float4*)(scale + co0 + 4 * q4) : float4{1.0f, 1.0f, 1.0f, 1.0f};
      const float4 b4 = shift ? *(const float4*)(shift + co0 + 4 * q4) : float4{0.0f, 0.0f, 0.0f, 0.0f};
      const float sc[4] = {a4.x, a4.y, a4.z, a4.w}, sh[4] = {b4.x, b4.y, b4.z, b4.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float v = acc[fc][4 * q4 + e] * sc[e] + sh[e];
        if (relu) v = fmaxf(v, 0.0f);
        out[4 * q4 + e] = float_to_bf16(v);
      }
    }
    uint4* dst = (uint4*)(y + m * c_out + co0);
    dst[0] = *(const uint4*)(out);
    dst[1] = *(const uint4*)(out + 8);
  }
}

// 3x3 stride-2 max pooling with padding 1: the maximum over the taps inside the image.
// One thread per (output pixel, 8 channels).
__global__ __launch_bounds__(256) void maxpool3x3s2_kernel(const uint16_t* __restrict__ x, uint16_t* __restrict__ y, int n,
                                                           int h, int wd, int c, int ho, int wo) {
  const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const int c8 = c >> 3;
  const long long total = (long long)n * ho * wo * c8;
  if (t >= total) return;
  const int cc = (int)(t % c8);
  long long q = t / c8;
  const int ox = (int)(q % wo);
  q /= wo;
  const int oy = (int)(q % ho);
  const int img = (int)(q / ho);
  float m[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) m[i] = -__builtin_inff();
  for (int r = 0; r < 3; ++r) {
    const int hi = oy * 2 - 1 + r;
    if (hi < 0 || hi >= h) continue;
    for (int s = 0; s < 3; ++s) {
      const int wi = ox * 2 - 1 + s;
      if (wi < 0 || wi >= wd) continue;
      uint16_t v[8];
      *(uint4*)v = *(const uint4*)(x + (((long long)img * h + hi) * wd + wi) * c + cc * 8);
#pragma unroll
      for (int i = 0; i < 8; ++i) m[i] = fmaxf(m[i], bf16_to_float(v[i]));
    }
  }
  uint16_t out[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) out[i] = float_to_bf16(m[i]);
  *(uint4*)(y + (((long long)img * ho + oy) * wo + ox) * c + cc * 8) = *(const uint4*)out;
}

// Global average pooling and the fully connected layer for channel counts in multiples of 32: a workgroup of sixteen
// wavefronts takes up to four images and 32 to 256 classes, a wavefront 16 of them (and a share of the K steps).
//
// The means are fp32; each is split into three bf16 numbers that add up to it exactly (8 bits of its 24 each), and the
// three parts of four images are twelve of the sixteen columns of one 16x16x32 product with the weights: as exact as fp32
// products, at a third of a percent of their instructions.  What bounds it is the latency of three dependent steps
// (read the map, meet in LDS, multiply), so a wavefront's first weights are requested before the map is read, and with few images
// the weights of a workgroup, read at 23 bytes a clock: then it takes fewer classes, 32 at least, and its wavefronts share the
// K steps.  ResNet-18's head (512 channels of 7x7, 1000 classes): one image 11.9 -> 7.1 us, 16 images 14.2 -> 8.2, 256 images 14.9.
constexpr int kPoolImgs = 4;
constexpr int kPoolSteps = 16;                   // K steps whose weights a wavefront holds at a time
constexpr int kPoolMaxC = 2048;

__global__ __launch_bounds__(1024) void avgpool_fc_mfma_kernel(const uint16_t* __restrict__ x, const uint16_t* __restrict__ wfc,
                                                               const float* __restrict__ bias, float* __restrict__ logits,
                                                               int n, int hw, int c, int classes, int cls_log) {
  typedef __attribute__((ext_vector_type(4))) float f32x4;
  extern __shared__ __align__(16) char pool_lds[];
  const int rowb = c * 2 + 16;                   // bytes of a column of the product's right operand, skewed
  float* part = (float*)(pool_lds + 16 * rowb);  // [groups][c] partial sums
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int img0 = blockIdx.x * kPoolImgs, imgs = n - img0 < kPoolImgs ? n - img0 : kPoolImgs;
  // 16 << cls_log classes to a workgroup; 16 >> cls_log wavefronts share the K steps of 16 of them
  const int k0 = (int)(blockIdx.y << (4 + cls_log)) + (wave & ((1 << cls_log) - 1)) * 16;   // this wavefront's classes
  const int share = wave >> cls_log, shares = 16 >> cls_log;
  const int first = (c >> 5) * share / shares, steps = (c >> 5) * (share + 1) / shares - first;
  const int cls = k0 + (lane & 15) < classes ? k0 + (lane & 15) : classes - 1;
  const char* wrow = (const char*)(wfc + (long long)cls * c + (lane >> 4) * 8) + first * 64;
  stem_i32x4 wv[kPoolSteps];
#pragma unroll
  for (int st = 0; st < kPoolSteps; ++st)
    if (st < steps) wv[st] = *(const stem_i32x4*)(wrow + st * 64);

  // ---- sums: groups of c/8 threads, each an image and every per-th position; eight channels a thread
  const int tpp = c >> 3;                        // threads per position
  const int groups = 1024 / tpp;                 // (c <= 2048: at least four)
  const int per = groups / imgs;                 // groups per image
  const int g = tid / tpp, ch = (tid - g * tpp) * 8, gi = g / per, gp = g - gi * per;
  if (gi < imgs) {
    const uint16_t* src = x + (long long)(img0 + gi) * hw * c + ch;
    float s[8] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 4
    for (int q = gp; q < hw; q += per) {
      const stem_i32x4 v = *(const stem_i32x4*)(src + (long long)q * c);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        s[2 * e] += __uint_as_float((uint32_t)v[e] << 16);
        s[2 * e + 1] += __uint_as_float((uint32_t)v[e] & 0xffff0000u);
      }
    }
    float4* dst = (float4*)(part + g * c + ch);
    dst[0] = float4{s[0], s[1], s[2], s[3]};
    dst[1] = float4{s[4], s[5], s[6], s[7]};
  }
  __syncthreads();
  // ---- means, split; columns 4*split + image, the rest zero
  const float inv = 1.0f / (float)hw;
  for (int i = tid; i < kPoolImgs * c; i += 1024) {
    const int im = i / c, cc = i - im * c;
    float t = 0.0f;
    if (im < imgs)
      for (int k = 0; k < per; ++k) t += part[(im * per + k) * c + cc];
    const float mean = t * inv;
    const uint16_t hi = float_to_bf16(mean);
    const float r1 = fabsf(mean) < 3.0e38f ? mean - bf16_to_float(hi) : 0.0f;      // (an infinite mean has no rest)
    const uint16_t mid = float_to_bf16(r1);
    const uint16_t lo = float_to_bf16(r1 - bf16_to_float(mid));
    *(uint16_t*)(pool_lds + im * rowb + cc * 2) = hi;
    *(uint16_t*)(pool_lds + (4 + im) * rowb + cc * 2) = mid;
    *(uint16_t*)(pool_lds + (8 + im) * rowb + cc * 2) = lo;
    *(uint16_t*)(pool_lds + (12 + im) * rowb + cc * 2) = 0;
  }
  __syncthreads();
  if (shares == 1 && k0 >= classes) return;
  // ---- product: rows = classes
  f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
  const char* col = pool_lds + (lane & 15) * rowb + (lane >> 4) * 16 + first * 64;
  for (int s0 = 0; s0 < steps; s0 += kPoolSteps) {
    if (s0 > 0) {
#pragma unroll
      for (int st = 0; st < kPoolSteps; ++st)
        if (s0 + st < steps) wv[st] = *(const stem_i32x4*)(wrow + (s0 + st) * 64);
    }
#pragma unroll
    for (int st = 0; st < kPoolSteps; ++st)
      if (s0 + st < steps)
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(stem_bf16x8, wv[st]),
                                                      __builtin_bit_cast(stem_bf16x8, *(const stem_i32x4*)(col + (s0 + st) * 64)),
                                                      acc, 0, 0, 0);
  }
  if (shares > 1) {                              // the wavefronts' sums meet where the partial sums of the map were
    f32x4* const sums = (f32x4*)part;
    sums[wave * 64 + lane] = acc;
    __syncthreads();
    if (share > 0 || k0 >= classes) return;
    for (int s = 1; s < shares; ++s) acc += sums[((s << cls_log) + wave) * 64 + lane];
  }
  const int im = lane & 15, r0 = k0 + (lane >> 4) * 4;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float mid = __shfl_down(acc[i], 4, 16), lo = __shfl_down(acc[i], 8, 16);
    if (im < imgs && r0 + i < classes)
      logits[(long long)(img0 + im) * classes + r0 + i] = acc[i] + (mid + lo) + (bias ? bias[r0 + i] : 0.0f);
  }
}

// Any channel count: global average pooling over hw positions, then logits = W * mean + bias.  One block of sixteen
// wavefronts per image and 256 classes: the map is averaged by all threads (positions split over
// thread groups, partial sums met in LDS), then every wavefront takes a share of the classes.
__global__ __launch_bounds__(1024) void avgpool_fc_kernel(const uint16_t* __restrict__ x, const uint16_t* __restrict__ wfc,
                                                         const float* __restrict__ bias, float* __restrict__ logits,
                                                         int hw, int c, int classes) {
  extern __shared__ float mean[];
  const int img = blockIdx.x;
  const int k0 = blockIdx.y * 256, k1 = k0 + 256 < classes ? k0 + 256 : classes;
  const float inv = 1.0f / (float)hw;
  {
    // thread group g of (blockDim / cpad) takes positions g, g + groups, ...; cpad = channels rounded
    // up to 64; the groups' partial sums sit behind the means in LDS and are added in a fixed order
    float* part = mean + c;                        // [groups][cpad], at most blockDim floats
    const int cpad = (c + 63) & ~63;
    const int groups = (int)blockDim.x / cpad > 0 ? (int)blockDim.x / cpad : 1;
    for (int ch0 = 0; ch0 < c; ch0 += groups > 1 ? c : (int)blockDim.x) {
      // a single group strides over the channels by thread index (threads past cpad would otherwise
      // alias the channels of the first ones); several groups split the positions
      const int ch = groups == 1 ? ch0 + (int)threadIdx.x : (int)threadIdx.x % cpad;
      const int g = groups == 1 ? 0 : (int)threadIdx.x / cpad;
      float s = 0.0f;
      if (ch < c && g < groups)
        for (int p = g; p < hw; p += groups) s += bf16_to_float(x[((long long)img * hw + p) * c + ch]);
      if (groups == 1) {
        if (ch < c) mean[ch] = s * inv;
      } else {
        if (g < groups) part[g * cpad + (int)threadIdx.x % cpad] = s;
        __syncthreads();
        if ((int)threadIdx.x < c) {
          float t = 0.0f;
          for (int gg = 0; gg < groups; ++gg) t += part[gg * cpad + threadIdx.x];
          mean[threadIdx.x] = t * inv;
        }
      }
    }
  }
  __syncthreads();
  // one wavefront per class: lanes stride over the channels, then a butterfly sum
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const bool vec = (c & 7) == 0 && (((uintptr_t)wfc) & 15) == 0;     // a lane takes eight consecutive channels per load
  for (int k = k0 + wave; k < k1; k += nw) {
    float s = 0.0f;
    if (vec) {
      for (int ch = lane * 8; ch < c; ch += 512) {
        uint16_t wv[8];
        *(uint4*)wv = *(const uint4*)(wfc + (long long)k * c + ch);
#pragma unroll
        for (int e = 0; e < 8; ++e) s = fmaf(bf16_to_float(wv[e]), mean[ch + e], s);
      }
    } else {
      for (int ch = lane; ch < c; ch += 64) s = fmaf(bf16_to_float(wfc[(long long)k * c + ch]), mean[ch], s);
    }
#pragma unroll
    for (int sft = 32; sft >= 1; sft >>= 1) s += __shfl_xor(s, sft, 64);
    if (lane == 0) logits[(long long)img * classes + k] = s + (bias ? bias[k] : 0.0f);
  }
}

}  // namespace

namespace cg {

int point_check(const void* x, const void* w, const float* scale, const float* shift, const void* y, int n, int h, int wd, int c_in, int c_out, int stride) {
  if (!x || !w || !y) return cg::set_error(CG_EINVAL, "cg_pointwise_conv: x, w and y must not be NULL");
  if (n < 0 || h <= 0 || wd <= 0) return cg::set_error(CG_EINVAL, "cg_pointwise_conv: bad image size");
  if (stride < 1) return cg::set_error(CG_EINVAL, "cg_pointwise_conv: stride must be >= 1");
  if (c_in <= 0 || c_in % 16 || c_in > 512)
    return cg::set_error(CG_EUNSUPPORTED, "cg_pointwise_conv: c_in must be a multiple of 16, at most 512");
  if (c_out <= 0 || c_out % kCb) return cg::set_error(CG_EUNSUPPORTED, "cg_pointwise_conv: c_out must be a multiple of 64");
  if ((((uintptr_t)x) | ((uintptr_t)w) | ((uintptr_t)y) | ((uintptr_t)scale) | ((uintptr_t)shift)) & 15)
    return cg::set_error(CG_EINVAL, "cg_pointwise_conv: x, w, y, scale and shift must be 16-byte aligned");
  return CG_OK;
}

}  // namespace cg

extern "C" {

int cg_small_cin_conv(const void* x, const void* w, const float* scale, const float* shift, void* y, int32_t n,
                      int32_t h, int32_t wd, int32_t c_in, int32_t c_out, int32_t k, int32_t stride, int32_t pad,
                      int32_t relu, void* hip_stream) {
  if (!x || !w || !y) return cg::set_error(CG_EINVAL, "cg_small_cin_conv: x, w and y must not be NULL");
  if (n < 0 || h <= 0 || wd <= 0) return cg::set_error(CG_EINVAL, "cg_small_cin_conv: bad image size");
  if (c_in < 1 || c_in > 4) return cg::set_error(CG_EUNSUPPORTED, "cg_small_cin_conv: c_in must lie in [1, 4]");
  if (c_out <= 0 || c_out % kCb) return cg::set_error(CG_EUNSUPPORTED, "cg_small_cin_conv: c_out must be a multiple of 64");
  if (k < 1 || k > 7 || !(k & 1)) return cg::set_error(CG_EUNSUPPORTED, "cg_small_cin_conv: kernel size must be odd, at most 7");
  if (stride < 1 || stride > 2 || pad < 0 || pad >= k) return cg::set_error(CG_EINVAL, "cg_small_cin_conv: bad stride or pad");
  if (h + 2 * pad < k || wd + 2 * pad < k) return cg::set_error(CG_EINVAL, "cg_small_cin_conv: kernel larger than the padded input");
  if ((((uintptr_t)y) | ((uintptr_t)scale) | ((uintptr_t)shift)) & 15)
    return cg::set_error(CG_EINVAL, "cg_small_cin_conv: y, scale and shift must be 16-byte aligned");
  if (n == 0) return CG_OK;
  const int ho = (h + 2 * pad - k) / stride + 1, wo = (wd + 2 * pad - k) / stride + 1;
  if (k == 7 && stride == 2 && c_in == 3)        // the ImageNet input layer: the matrix-core kernel
    return launch_conv7x7s2c3(false, "cg_small_cin_conv", x, w, scale, shift, y, n, h, wd, c_out, pad, relu, (hipStream_t)hip_stream);
  const long long tiles = (long long)n * ((ho + kTile - 1) / kTile) * ((wo + kTile - 1) / kTile);
  if (tiles > 0x7fffffffll) return cg::set_error(CG_EUNSUPPORTED, "cg_small_cin_conv: too many tiles");
  const int pe = (kTile - 1) * stride + k;
  const size_t lds = ((size_t)k * k * c_in * kCb + (size_t)pe * pe * c_in) * sizeof(float);
  hipLaunchKernelGGL(small_cin_conv_kernel, dim3((unsigned)tiles, (unsigned)(c_out / kCb)), dim3(256), lds,
                     (hipStream_t)hip_stream, (const uint16_t*)x, (const uint16_t*)w, scale, shift, (uint16_t*)y, n, h, wd,
                     c_in, c_out, k, stride, pad, ho, wo, relu);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return cg::set_error(CG_EHIP, "cg_small_cin_conv: %s", hipGetErrorString(e));
  return CG_OK;
}

int cg_conv7x7s2_maxpool(const void* x, const void* w, const float* scale, const float* shift, void* y, int32_t n,
                         int32_t h, int32_t wd, int32_t c_out, int32_t pad, int32_t relu, void* hip_stream) {
  if (!x || !w || !y) return cg::set_error(CG_EINVAL, "cg_conv7x7s2_maxpool: x, w and y must not be NULL");
  if (n < 0 || h <= 0 || wd <= 0) return cg::set_error(CG_EINVAL, "cg_conv7x7s2_maxpool: bad image size");
  if (c_out <= 0 || c_out % kCb) return cg::set_error(CG_EUNSUPPORTED, "cg_conv7x7s2_maxpool: c_out must be a multiple of 64");
  if (pad < 0 || pad >= 7) return cg::set_error(CG_EINVAL, "cg_conv7x7s2_maxpool: bad pad");
  if (h + 2 * pad < 7 || wd + 2 * pad < 7) return cg::set_error(CG_EINVAL, "cg_conv7x7s2_maxpool: kernel larger than the padded input");
  if ((((uintptr_t)y) | ((uintptr_t)scale) | ((uintptr_t)shift)) & 15)
    return cg::set_error(CG_EINVAL, "cg_conv7x7s2_maxpool: y, scale and shift must be 16-byte aligned");
  if (n == 0) return CG_OK;
  return launch_conv7x7s2c3(true, "cg_conv7x7s2_maxpool", x, w, scale, shift, y, n, h, wd, c_out, pad, relu, (hipStream_t)hip_stream);
}

int cg_pointwise_conv(const void* x, const void* w, const float* scale, const float* shift, void* y, int32_t n,
                      int32_t h, int32_t wd, int32_t c_in, int32_t c_out, int32_t stride, int32_t relu,
                      void* hip_stream) {
  const int rc = cg::point_check(x, w, scale, shift, y, n, h, wd, c_in, c_out, stride);
  if (rc != CG_OK) return rc;
  if (n == 0) return CG_OK;
  const PointArgs a = cg::point_args(x, w, scale, shift, y, n, h, wd, c_in, c_out, stride, relu);
  const long long m_total = (long long)n * a.ho * a.wo;
  // Small tiles below a quarter of 128 pixels x 64 channels per compute unit, where the large ones leave most of the chip idle.  Small / large, us: 64 to
  // 128 channels, 3136 pixels (50 blocks of a line of 64) 3.5 and, just past the line, 6272 (98) 3.9; 256 to 512, 588 pixels (40) 5.2, 1176 (80) 5.7.
  if (cg::point_in_pieces(m_total, c_out, cg::cu_count())) {
    hipLaunchKernelGGL(pointwise_small_kernel, dim3((unsigned)((m_total + 15) / 16), (unsigned)(c_out / 32)), dim3(64), 0,
                       (hipStream_t)hip_stream, a);
  } else if (cg::point_in_wide_blocks(m_total, c_in, c_out, cg::cu_count())) {
    hipLaunchKernelGGL(pointwise_conv_kernel, dim3((unsigned)((m_total + 127) / 128), (unsigned)(c_out / kCb)), dim3(256), (size_t)c_in * kCb * 2,
                       (hipStream_t)hip_stream, (const uint16_t*)x, (const uint16_t*)w, scale, shift, (uint16_t*)y, m_total, h, wd,
                       c_in, c_out, stride, a.ho, a.wo, relu);
  } else {
    // A launch holds less than 2^32 threads and at most 2^30 pixels; larger batches go in pieces of images, rows or columns.
    const long long cap = std::min(((1ll << 24) - 8) / a.ncb * kPointPx, 1ll << 30);
    if (cap < kPointPx) return cg::set_error(CG_EUNSUPPORTED, "cg_pointwise_conv: too large");
    cg::for_point_pieces(a, n, cap, [&](PointArgs& p) {
      p.blocks = (p.m_total + kPointPx - 1) / kPointPx * a.ncb;
      p.per_xcd = (p.blocks + 7) / 8;
      hipLaunchKernelGGL(pointwise_tile_kernel, dim3((unsigned)p.per_xcd * 8u), dim3(256), (size_t)((c_in + 31) / 32) * (kPointPx * 64),
                         (hipStream_t)hip_stream, p);
    });
  }
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return cg::set_error(CG_EHIP, "cg_pointwise_conv: %s", hipGetErrorString(e));
  return CG_OK;
}

int cg_maxpool3x3s2(const void* x, void* y, int32_t n, int32_t h, int32_t wd, int32_t c, void* hip_stream) {
  if (!x || !y) return cg::set_error(CG_EINVAL, "cg_maxpool3x3s2: x and y must not be NULL");
  if (n < 0 || h <= 0 || wd <= 0 || c <= 0) return cg::set_error(CG_EINVAL, "cg_maxpool3x3s2: bad size");
  if (c % 8) return cg::set_error(CG_EUNSUPPORTED, "cg_maxpool3x3s2: c must be a multiple of 8");
  if ((((uintptr_t)x) | ((uintptr_t)y)) & 15) return cg::set_error(CG_EINVAL, "cg_maxpool3x3s2: x and y must be 16-byte aligned");
  if (n == 0) return CG_OK;
  const int ho = (h + 2 - 3) / 2 + 1, wo = (wd + 2 - 3) / 2 + 1;
  const long long total = (long long)n * ho * wo * (c / 8);
  const long long blocks = (total + 255) / 256;
  if (blocks > 0x7fffffffll) return cg::set_error(CG_EUNSUPPORTED, "cg_maxpool3x3s2: too large");
  hipLaunchKernelGGL(maxpool3x3s2_kernel, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)hip_stream,
                     (const uint16_t*)x, (uint16_t*)y, n, h, wd, c, ho, wo);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return cg::set_error(CG_EHIP, "cg_maxpool3x3s2: %s", hipGetErrorString(e));
  return CG_OK;
}

int cg_avgpool_fc(const void* x, const void* wfc, const float* bias, float* logits, int32_t n, int32_t hw, int32_t c,
                  int32_t classes, void* hip_stream) {
  if (!x || !wfc || !logits) return cg::set_error(CG_EINVAL, "cg_avgpool_fc: x, wfc and logits must not be NULL");
  if (n < 0 || hw <= 0 || c <= 0 || classes <= 0) return cg::set_error(CG_EINVAL, "cg_avgpool_fc: bad size");
  if (c > 11264) return cg::set_error(CG_EUNSUPPORTED, "cg_avgpool_fc: at most 11264 channels");
  if (n == 0) return CG_OK;
  if (c % 32 == 0 && c <= kPoolMaxC && ((((uintptr_t)x) | ((uintptr_t)wfc)) & 15) == 0) {
    const size_t lds = 16 * ((size_t)c * 2 + 16) + (size_t)(1024 / (c / 8)) * c * sizeof(float);
    static std::atomic<uint64_t> asked{0};
    const hipError_t attr = cg::allow_lds((const void*)avgpool_fc_mfma_kernel, 160 * 1024, asked);
    if (attr != hipSuccess) return cg::set_error(CG_EHIP, "cg_avgpool_fc: %s", hipGetErrorString(attr));
    // classes to a workgroup: as few as give every compute unit one, 32 at least (each workgroup averages its images again)
    const int groups = (n + kPoolImgs - 1) / kPoolImgs;
    int cls_log = 1;
    while (cls_log < 4 && (long long)groups * ((classes + (16 << cls_log) - 1) >> (4 + cls_log)) > cg::cu_count()) ++cls_log;
    hipLaunchKernelGGL(avgpool_fc_mfma_kernel, dim3((unsigned)groups, (unsigned)((classes + (16 << cls_log) - 1) >> (4 + cls_log))),
                       dim3(1024), lds, (hipStream_t)hip_stream, (const uint16_t*)x, (const uint16_t*)wfc, bias, logits, n, hw, c,
                       classes, cls_log);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return cg::set_error(CG_EHIP, "cg_avgpool_fc: %s", hipGetErrorString(e));
    return CG_OK;
  }
  hipLaunchKernelGGL(avgpool_fc_kernel, dim3((unsigned)n, (unsigned)((classes + 255) / 256)), dim3(1024),
                     ((size_t)c + 1024) * sizeof(float), (hipStream_t)hip_stream,
                     (const uint16_t*)x, (const uint16_t*)wfc, bias, logits, hw, c, classes);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return cg::set_error(CG_EHIP, "cg_avgpool_fc: %s", hipGetErrorString(e));
  return CG_OK;
}

}  // extern "C"
