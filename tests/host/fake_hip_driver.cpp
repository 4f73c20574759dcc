// Host side of forward calls without a GPU: this program defines the HIP runtime calls the library makes, which the loader
// finds before the runtime's own, notes them and "launches" nothing.  Run by tests/test_host_calls_cpu.py.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <set>
#include <utility>
#include <vector>

#include "cg_conv.h"

static int device = 0, failures = 0, device_asked = 0;
static int compute_units[2] = {256, 64};
static std::vector<void*> host_blocks;
struct Launch { const void* kernel; int device; unsigned blocks; size_t lds; };
static std::vector<Launch> launches;
static std::set<std::pair<const void*, int>> large_lds;      // (kernel, device) that may use more LDS than the default
static Launch config;
#define EXPECT(c) do { if (!(c)) { std::printf("FAILED line %d: %s  [%s]\n", __LINE__, #c, cg_last_error()); ++failures; } } while (0)

extern "C" {
hipError_t hipGetDevice(int* d) { *d = device; ++device_asked; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int d) {
  *v = a == hipDeviceAttributeMultiprocessorCount ? compute_units[d] : 0;
  return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void* f, hipFuncAttribute, int) {
  large_lds.insert({f, device});
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) { *p = (void*)0x700000000000ull; return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t bytes, unsigned) {
  *p = std::calloc(1, bytes);
  host_blocks.push_back(*p);
  return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t __hipPushCallConfiguration(dim3 grid, dim3, size_t lds, hipStream_t) {
  config = Launch{nullptr, device, grid.x * grid.y * grid.z, lds};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* s) {
  *grid = *block = dim3(1);
  *lds = 0;
  *s = nullptr;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3, dim3, void**, size_t, hipStream_t) {
  config.kernel = f;
  launches.push_back(config);
  return hipSuccess;
}
}

// a handle of 128 channels at 28x28 on the row-tiled kernel; its buffers exist in name only
static cg_conv* make(int n_max, unsigned epilogue = CG_EPI_RELU) {
  static int32_t thr[128];
  cg_conv_desc d;
  std::memset(&d, 0, sizeof d);
  d.struct_size = sizeof d;
  d.n_max = n_max; d.h = d.w = 28; d.c_in = d.c_out = 128; d.c_base = 32; d.kh = d.kw = 3; d.stride = d.pad = 1;
  d.in_dtype = d.out_dtype = CG_I8; d.epilogue = epilogue; d.rq_shift = 8; d.gate_thr_i32 = thr;
  d.w_base = (const void*)0x1000; d.w_cond = (const void*)0x2000;
  d.packed = (void*)0x100000; d.packed_bytes = cg_conv_packed_bytes(&d);
  cg_conv* h = nullptr;
  EXPECT(cg_conv_create(&h, &d, nullptr) == CG_OK);
  return h;
}

static int forward(cg_conv* h, int n) {
  return cg_conv_forward(h, n, (void*)0x200000000ull, nullptr, (void*)0x300000000ull, (uint32_t*)0x400000000ull, nullptr,
                         (void*)0x500000000ull, cg_conv_workspace_bytes(h, n), nullptr);
}

// A kernel that gave up a bounded wait sets a word of host memory; every later call fails.
static void gave_up_wait_is_reported() {
  cg_conv *a = make(32), *b = make(4);
  EXPECT(host_blocks.size() == 1);
  EXPECT(forward(a, 32) == CG_OK && forward(b, 4) == CG_OK);
  if (host_blocks.size() == 1) {
    *(volatile uint32_t*)host_blocks[0] = 1u;
    const size_t before = launches.size();
    EXPECT(forward(a, 32) == CG_EHIP && std::strstr(cg_last_error(), "gave up") != nullptr);
    EXPECT(forward(b, 4) == CG_EHIP && launches.size() == before);
    *(volatile uint32_t*)host_blocks[0] = 0u;
    EXPECT(forward(a, 32) == CG_OK);
  }
  cg_conv_destroy(a);
  cg_conv_destroy(b);
}

// Plans are made once per batch size (a plan asks for the device's compute units; a launch alone asks for the device once).
static void plans_are_kept() {
  cg_conv* h = make(64);
  for (int round = 0; round < 2; ++round)
    for (int n = 1; n <= 40; ++n) {
      device_asked = 0;
      EXPECT(forward(h, n) == CG_OK);
      EXPECT(round == 0 || device_asked <= 1);
    }
  cg_conv_destroy(h);
  // two fragments per wavefront, y over the residual: another plan, kept as well
  static float stat[256], one[256];
  for (float& v : one) v = 1.0f;
  cg_conv_desc d;
  std::memset(&d, 0, sizeof d);
  d.struct_size = sizeof d;
  d.n_max = 256; d.h = d.w = 14; d.c_in = d.c_out = 256; d.c_base = 64; d.kh = d.kw = 3; d.stride = d.pad = 1;
  d.in_dtype = d.out_dtype = CG_BF16; d.epilogue = CG_EPI_RELU | CG_EPI_RESIDUAL; d.gate_mean = d.delta = stat; d.gate_var = one;
  d.w_base = (const void*)0x1000; d.w_cond = (const void*)0x2000;
  d.packed = (void*)0x100000; d.packed_bytes = cg_conv_packed_bytes(&d);
  EXPECT(cg_conv_create(&h, &d, nullptr) == CG_OK);
  const void* kernel[2];
  for (int n = 256; n >= 200; n -= 56)
    for (int round = 0; round < 2; ++round)
      for (int over = 0; over < 2; ++over) {
        device_asked = 0;
        char *y = (char*)0x300000000ull, *res = over ? y : (char*)0x600000000ull;
        EXPECT(cg_conv_forward(h, n, (void*)0x200000000ull, res, y, nullptr, nullptr, (void*)0x500000000ull,
                               cg_conv_workspace_bytes(h, n), nullptr) == CG_OK);
        EXPECT((round == 0 && !over) || device_asked <= 1);
        kernel[over] = launches.back().kernel;
        EXPECT(!over || kernel[0] != kernel[1]);
      }
  cg_conv_destroy(h);
}

// What a launch depends on is asked of the device it goes to: the LDS beyond the default, the compute units.
static void devices_are_asked_one_by_one() {
  const size_t first = launches.size();
  unsigned blocks[2][2];
  for (device = 0; device < 2; ++device) {
    cg_conv* h = make(64);
    size_t at = launches.size();
    EXPECT(forward(h, 64) == CG_OK && launches.size() == at + 1);
    blocks[device][0] = launches.back().blocks;
    cg_conv_destroy(h);
    at = launches.size();
    EXPECT(cg_conv7x7s2_maxpool((void*)16, (void*)16, nullptr, nullptr, (void*)16, 16, 224, 224, 64, 3, 1, nullptr) == CG_OK);
    EXPECT(launches.size() == at + 1);
    blocks[device][1] = launches.back().blocks;
    EXPECT(cg_avgpool_fc((void*)16, (void*)16, nullptr, (float*)16, 4, 49, 2048, 1000, nullptr) == CG_OK);
  }
  device = 0;
  int large = 0;
  for (size_t i = first; i < launches.size(); ++i) {
    if (launches[i].lds <= 65536) continue;
    ++large;
    EXPECT(large_lds.count({launches[i].kernel, launches[i].device}) == 1);
  }
  EXPECT(large == 4);
  EXPECT(blocks[0][0] == 256 && blocks[1][0] == 64);
  EXPECT(blocks[0][1] == 896 && blocks[1][1] == 224);
}

int main() {
  devices_are_asked_one_by_one();
  plans_are_kept();
  gave_up_wait_is_reported();
  if (failures) { std::printf("%d checks failed\n", failures); return 1; }
  std::printf("host calls driver: ok\n");
  return 0;
}
