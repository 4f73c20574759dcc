// Which kernel a forward call launches, without a GPU: this program defines the HIP runtime calls the library makes, which the
// loader finds before the runtime's own, keeps the kernels' names as they are registered and "launches" nothing.
// One layer a line on standard input: in_dtype out_dtype n_max n h w c_in c_out c_base k stride pad groups shuffle epilogue
// variant rq_shift; a line with the kernel's name and its threads to a workgroup for each.  Run by tests/test_kernels_of_calls_cpu.py.
//   "pointwise": n h w c_in c_out stride a line, for cg_pointwise_conv; "cut": the same and the pixels to a piece, for the cutting alone.  A line with the pieces,
// x (bytes) y (bytes) m_total ho wo each, or the kernel's name where it has no pieces.
//   "beside": n h w c_in c_out c_base k stride c_out1 groups a line, for cg_conv_call_beside on a bf16 layer.  A line with all launches: name, threads to a
// workgroup and workgroups each, with a semicolon behind.
#include <cxxabi.h>
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <limits>
#include <map>
#include <string>
#include <vector>

#include "cg_calls.h"
#include "cg_conv.h"
#include "point_piece.h"

static std::map<const void*, std::string>& names() {      // (the library registers its kernels before main)
  static std::map<const void*, std::string> m;
  return m;
}
struct Launch { const void* kernel; unsigned threads, blocks; cg::PointArgs piece; };
static const char *const kX = (const char*)0x200000000ull, *const kY = (const char*)0x1000000000000ull;
static std::vector<Launch> launches;
static dim3 config_grid, config_block;

extern "C" {
void** __hipRegisterFatBinary(const void*) {
  static void* handle[16];
  return handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* device, unsigned, void*, void*, void*, void*, int*) {
  int status = 0;
  char* d = abi::__cxa_demangle(device, nullptr, nullptr, &status);
  names()[host] = status == 0 && d ? d : device;
  std::free(d);
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int) {
  *v = a == hipDeviceAttributeMultiprocessorCount ? 256 : 0;
  return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) { *p = (void*)0x700000000000ull; return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t bytes, unsigned) { *p = std::calloc(1, bytes); return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t, hipStream_t) {
  config_grid = grid;
  config_block = block;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* s) {
  *grid = *block = dim3(1);
  *lds = 0;
  *s = nullptr;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3, dim3, void** args, size_t, hipStream_t) {
  launches.push_back({f, config_block.x, config_grid.x * config_grid.y * config_grid.z, {}});
  if (names()[f].find("pointwise_tile_kernel") != std::string::npos) launches.back().piece = *(const cg::PointArgs*)args[0];
  if (launches.size() > 10000) {
    std::fprintf(stderr, "a call that does not stop launching\n");
    std::exit(3);
  }
  return hipSuccess;
}
}

static void print_piece(const cg::PointArgs& p) { std::printf("%lld %lld %d %d %d ", (long long)(p.x - kX), (long long)(p.y - kY), p.m_total, p.ho, p.wo); }

static int pointwise_calls(bool cut) {
  int n, h, w, c_in, c_out, stride;
  long long cap;
  while (std::scanf("%d %d %d %d %d %d", &n, &h, &w, &c_in, &c_out, &stride) == 6) {
    if (cut) {
      if (std::scanf("%lld", &cap) != 1) return 2;
      cg::for_point_pieces(cg::point_args(kX, kX, nullptr, nullptr, (void*)kY, n, h, w, c_in, c_out, stride, 0), n, cap, print_piece);
    } else {
      launches.clear();
      if (cg_pointwise_conv(kX, kX, nullptr, nullptr, (void*)kY, n, h, w, c_in, c_out, stride, 0, nullptr) != CG_OK) std::printf("%s", cg_last_error());
      for (const Launch& l : launches) {
        if (l.piece.x) print_piece(l.piece);
        else std::printf("%s ", names()[l.kernel].c_str());
      }
    }
    std::printf("\n");
  }
  return 0;
}

static int beside_calls() {
  int n, h, w, c_in, c_out, c_base, k, stride, c_out1, groups;
  while (std::scanf("%d %d %d %d %d %d %d %d %d %d", &n, &h, &w, &c_in, &c_out, &c_base, &k, &stride, &c_out1, &groups) == 10) {
    const std::vector<float> zero(c_out, 0.0f), one(c_out, 1.0f);
    cg_conv_desc d;
    std::memset(&d, 0, sizeof d);
    d.struct_size = sizeof d;
    d.n_max = n; d.h = h; d.w = w; d.c_in = c_in; d.c_out = c_out; d.c_base = c_base; d.kh = d.kw = k; d.stride = stride; d.pad = k / 2;
    d.in_dtype = d.out_dtype = CG_BF16; d.groups = groups;
    d.gate_mean = d.delta = zero.data();
    d.gate_var = one.data();
    d.w_base = (const void*)0x1000;
    d.w_cond = c_base < c_in ? (const void*)0x2000 : nullptr;
    d.packed = (void*)0x100000;
    d.packed_bytes = cg_conv_packed_bytes(&d);
    cg_conv* layer = nullptr;
    if (cg_conv_create(&layer, &d, nullptr) != CG_OK) {
      std::printf("%s\n", cg_last_error());
      continue;
    }
    launches.clear();
    if (cg_conv_call_beside(layer, n, kX, (void*)0x300000000ull, kX, nullptr, nullptr, (void*)kY, c_out1, 0, nullptr) != CG_OK) std::printf("%s", cg_last_error());
    for (const Launch& l : launches) std::printf("%s %u %u;", names()[l.kernel].c_str(), l.threads, l.blocks);
    std::printf("\n");
    cg_conv_destroy(layer);
  }
  return 0;
}

int main(int argc, char** argv) {
  if (argc > 1 && !std::strcmp(argv[1], "beside")) return beside_calls();
  if (argc > 1) return pointwise_calls(!std::strcmp(argv[1], "cut"));
  int in_dtype, out_dtype, n_max, n, h, w, c_in, c_out, c_base, k, stride, pad, groups, shuffle, variant, rq_shift;
  unsigned epilogue;
  while (std::scanf("%d %d %d %d %d %d %d %d %d %d %d %d %d %d %u %d %d", &in_dtype, &out_dtype, &n_max, &n, &h, &w, &c_in, &c_out, &c_base, &k,
                    &stride, &pad, &groups, &shuffle, &epilogue, &variant, &rq_shift) == 17) {
    const std::vector<float> zero(c_out, 0.0f), one(c_out, 1.0f);
    const std::vector<int32_t> thr(c_out, 0);
    cg_conv_desc d;
    std::memset(&d, 0, sizeof d);
    d.struct_size = sizeof d;
    d.n_max = n_max; d.h = h; d.w = w; d.c_in = c_in; d.c_out = c_out; d.c_base = c_base; d.kh = d.kw = k; d.stride = stride; d.pad = pad;
    d.in_dtype = in_dtype; d.out_dtype = out_dtype; d.epilogue = epilogue; d.variant = variant; d.groups = groups; d.shuffle = shuffle;
    d.rq_shift = rq_shift;
    if (in_dtype == CG_I8) {
      d.gate_thr_i32 = thr.data();
    } else {
      d.gate_mean = d.delta = zero.data();
      d.gate_var = one.data();
    }
    d.w_base = (const void*)0x1000;
    d.w_cond = c_base < c_in ? (const void*)0x2000 : nullptr;
    d.packed = (void*)0x100000;
    d.packed_bytes = cg_conv_packed_bytes(&d);
    cg_conv* layer = nullptr;
    const char* said = "";
    launches.clear();
    if (cg_conv_create(&layer, &d, nullptr) != CG_OK) {
      said = cg_last_error();
    } else {
      launches.clear();
      if (cg_conv_forward(layer, n, (void*)0x200000000ull, (epilogue & CG_EPI_RESIDUAL) ? (void*)0x600000000ull : nullptr, (void*)0x300000000ull,
                          nullptr, nullptr, (void*)0x500000000ull, cg_conv_workspace_bytes(layer, n), nullptr) != CG_OK)
        said = cg_last_error();
      cg_conv_destroy(layer);
    }
    if (launches.empty())
      std::printf("none: %s\n", said);
    else
      std::printf("%s %u\n", names()[launches[0].kernel].c_str(), launches[0].threads);
  }
  return 0;
}
