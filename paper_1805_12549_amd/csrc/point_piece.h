// 1x1 convolution with stride (the ResNet shortcut) on the matrix cores, in pieces of one wavefront: a launch of its own (kernels_dense.hip)
// or further workgroups of the block's first layer (kernels_direct.hip).
#pragma once

#include "cg_device.h"

namespace cg {

struct PointArgs {
  const char* x;
  const char* w;
  const float* scale;
  const float* shift;
  char* y;
  int m_total, h, wd, c_in, c_out, stride, ho, wo, relu;
  Div d_wo, d_ho;
  int blocks, per_xcd, ncb;                        // pointwise_tile_kernel: its workgroups, those of an XCD, blocks of 128 channels
  Div d_ncb;
  int waves;                                       // gated_conv_beside_kernel: wavefronts of a workgroup that do a piece
};

inline PointArgs point_args(const void* x, const void* w, const float* scale, const float* shift, void* y, int n, int h, int wd, int c_in, int c_out,
                            int stride, int relu) {
  const int ho = (h - 1) / stride + 1, wo = (wd - 1) / stride + 1, ncb = (c_out + 127) / 128;
  return PointArgs{(const char*)x, (const char*)w, scale, shift, (char*)y, (int)((long long)n * ho * wo), h, wd, c_in, c_out, stride, ho, wo, relu,
                   div_of(wo), div_of(ho), 0, 0, ncb, div_of(ncb), 0};
}

// A 1x1 convolution that a layer's launch may do too; done: it has.
struct Beside {
  PointArgs what;
  bool done;
};

// Whether the small pieces are taken: below a quarter of 128 pixels x 64 channels per compute unit (see cg_pointwise_conv).
inline bool point_in_pieces(long long m_total, int c_out, int n_cu) { return (m_total + 127) / 128 * (c_out / 64) * 4 < n_cu; }

// Pieces to a workgroup of `most` wavefronts in the launch of a layer of `layer` workgroups that takes some `est` clocks (as a call).  A piece of 256 channels is
// 24 KB through its compute unit's memory path: a workgroup of k pieces takes 2.7 us and 5.1 more for k * channels = 2048.  As few as let layer and pieces have
// a compute unit to a workgroup, if they are done with the layer then; else as few as come to two and a half workgroups to a compute unit, from 256
// channels to a workgroup on (fewer gain nothing there).
//   Eight everywhere, before, and now: 256 to 512 channels, one image of 14x14 7.8 -> 5.2 us (two launches 7.4), five 10.8 -> 6.3 (8.0), ten 11.8 -> 8.1 (10.0);
// 512 to 512 at 7x7 13.0 -> 7.2 (10.3); 128 to 256, five images of 28x28 7.5 -> 5.6 (7.4); 64 to 128, five of 56x56 6.0 -> 5.7 (7.4).  Where eight are still
// taken 4.9 (64 to 128, three of 56x56) and 9.0 (256 to 512, twelve of 14x14); four there 5.4 and 11.0.
inline int pieces_to_workgroup(long long layer, long long pieces, int c_in, int most, double est, int n_cu) {
  auto workgroups = [&](int k) { return layer + (pieces + k - 1) / k; };
  int k = 1;
  while (k < most && workgroups(k) > n_cu) k *= 2;
  if (workgroups(k) > n_cu || 6100.0 + 5.6 * k * c_in > est - 3400.0) {
    k = c_in < 256 ? 256 / c_in : 1;
    while (k < most && 2 * workgroups(k) > 5ll * n_cu) k *= 2;
  }
  return k < most ? k : most;
}

// Whether 128 pixels x 64 channels a workgroup are taken instead of 64 x 128 (cg_pointwise_conv): where the last block of 128 channels is half empty and the
// other form comes to at least 5/3 as many workgroups to a compute unit, if these are all on the chip at once (the weights of 64 channels in LDS; beyond
// 384 channels two, as one alone has too few loads in flight) and the channels are whole rounds of that kernel's loop of four steps of 16.
//   64 x 128 and 128 x 64, us: 256 to 64 channels, 20000 pixels 8.2 and 7.4, 65536 14.7 and 12.6; 512 to 64, 55000 23.5 and 20.7; 256 to 320, 5441 8.2 and 7.5;
// 128 to 64, 120000 15.2 and 14.2.  Outside: 256 to 64, 33000 pixels (516 workgroups and 258) 10.4 and 11.0; 512 to 64, 20000 10.7 and 13.9; 208 to 64,
// 55000 9.7 and 11.2.
inline bool point_in_wide_blocks(long long m_total, int c_in, int c_out, int n_cu) {
  const long long tiles = (m_total + 63) / 64 * ((c_out + 127) / 128), wide = (m_total + 127) / 128 * (c_out / 64);
  const long long rounds = (tiles + n_cu - 1) / n_cu, each = (wide + n_cu - 1) / n_cu;
  return c_out % 128 != 0 && c_in % 64 == 0 && 3 * rounds >= 5 * each && each <= 4 && each * c_in <= 1152 && (each > 1 || c_in <= 384);
}

// What cg_pointwise_conv refuses (kernels_dense.hip).
int point_check(const void* x, const void* w, const float* scale, const float* shift, const void* y, int n, int h, int wd, int c_in, int c_out, int stride);

// The convolution `a` of n images in pieces of at most `cap` output pixels (cap >= 1): whole images, else whole rows of one image, else columns of one row.
template <typename Launch>
void for_point_pieces(const PointArgs& a, int n, long long cap, Launch&& launch) {
  const long long cols = a.wo < cap ? a.wo : cap;
  const long long rows = cols < a.wo ? 1 : cap / a.wo < a.ho ? cap / a.wo : a.ho;
  const long long px = (long long)a.ho * a.wo, imgs = cols < a.wo || rows < a.ho ? 1 : cap / px < n ? cap / px : n;
  for (long long i = 0; i < n; i += imgs)
    for (long long r = 0; r < a.ho; r += rows)
      for (long long c = 0; c < a.wo; c += cols) {
        PointArgs p = a;
        p.x = a.x + ((i * a.h + r * a.stride) * a.wd + c * a.stride) * (a.c_in * 2ll);
        p.y = a.y + ((i * a.ho + r) * a.wo + c) * (a.c_out * 2ll);
        p.ho = (int)(rows < a.ho - r ? rows : a.ho - r);
        p.wo = (int)(cols < a.wo - c ? cols : a.wo - c);
        p.m_total = (int)((imgs < n - i ? imgs : n - i) * p.ho * p.wo);
        p.d_wo = div_of(p.wo);
        p.d_ho = div_of(p.ho);
        launch(p);
      }
}

// byte offset of the input pixel of output pixel m
__device__ __forceinline__ long long point_pixel(const PointArgs& a, unsigned m) {
  const unsigned q = quot(m, a.d_wo), img = quot(q, a.d_ho);
  const long long row = (long long)img * a.h + (q - img * (unsigned)a.ho) * (unsigned)a.stride;
  return (row * a.wd + (m - q * (unsigned)a.wo) * (unsigned)a.stride) * (a.c_in * 2);
}

// Sixteen pixels (number `px` of them) x 32 channels by one wavefront, which takes both operands straight from memory in 64-byte pieces.  With U = 8 and 128
// registers free (a launch of its own) all loads of eight K steps are in flight at once: what bounds it is one latency.  ResNet-18's three shortcuts of
// one image 3.1, 3.5 and 4.0 us.  With U = 4, beside a layer, the compiler waits after each step's loads (they are under a lane's condition): four short latencies a
// batch.  Without that condition all are in flight there too, which gained nothing: layer and 1x1 in one launch, eight pieces to a workgroup, 4.1, 5.4
// and 7.8 -> 3.9, 5.2 and 7.9, and in two 5.6, 6.0 and 7.4 -> 5.5, 6.1 and 7.7.
template <int U>
__device__ __forceinline__ void point_piece(const PointArgs& a, unsigned px, int block) {
  typedef __attribute__((ext_vector_type(4))) int chunk_t;
  typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
  typedef __attribute__((ext_vector_type(4))) float sums_t;
  const int lane = threadIdx.x & 63, lj = lane & 15, lg = lane >> 4;
  const int c0 = block * 32, nq = a.c_in >> 3, steps = (nq + 3) >> 2;
  const unsigned m = px * 16 + lj;
  const bool valid = m < (unsigned)a.m_total;
  const char* const wr = a.w + (long long)(c0 + lj) * (a.c_in * 2) + lg * 16;
  const int w16 = 16 * a.c_in * 2;
  chunk_t wv[U][2], xv[U];
  sums_t acc[2] = {{0.0f, 0.0f, 0.0f, 0.0f}, {0.0f, 0.0f, 0.0f, 0.0f}}, sc[2], sh[2];
  const char* const xr = a.x + point_pixel(a, valid ? m : 0u) + lg * 16;
  for (int s0 = 0; s0 < steps; s0 += U) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool on = 4 * (s0 + u) + lg < nq;        // (a last step of two chunks)
      xv[u] = wv[u][0] = wv[u][1] = chunk_t{0, 0, 0, 0};
      if (on) {
        wv[u][0] = *(const chunk_t*)(wr + (s0 + u) * 64);
        wv[u][1] = *(const chunk_t*)(wr + w16 + (s0 + u) * 64);
        xv[u] = *(const chunk_t*)(xr + (s0 + u) * 64);
      }
    }
    if (s0 == 0) {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        sc[i] = a.scale ? *(const sums_t*)(a.scale + c0 + 16 * i + 4 * lg) : sums_t{1.0f, 1.0f, 1.0f, 1.0f};
        sh[i] = a.shift ? *(const sums_t*)(a.shift + c0 + 16 * i + 4 * lg) : sums_t{0.0f, 0.0f, 0.0f, 0.0f};
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int i = 0; i < 2; ++i)
        acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, wv[u][i]), __builtin_bit_cast(bf16x8_t, xv[u]), acc[i], 0, 0, 0);
  }
  if (!valid) return;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    float v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      v[e] = acc[i][e] * sc[i][e] + sh[i][e];
      if (a.relu) v[e] = fmaxf(v[e], 0.0f);
    }
    uint2 out;
    out.x = (uint32_t)float_to_bf16(v[0]) | (uint32_t)float_to_bf16(v[1]) << 16;
    out.y = (uint32_t)float_to_bf16(v[2]) | (uint32_t)float_to_bf16(v[3]) << 16;
    *(uint2*)(a.y + ((long long)m * a.c_out + c0 + 16 * i + 4 * lg) * 2) = out;
  }
}

}  // namespace cg
