// The launches that libsppo's launchers would make, printed without making
// them: hipLaunchKernel is replaced by one that records.  Runs without a GPU
// (the library then counts 256 compute units).  One case a line on stdin:
//   fwd|pre|dkdv|dq|pair  bf16|f32  B Hq Hkv D S c0 c1 [kv0 kv1]
//   gemm  tn epi M N K
// For each, a line of "kernel gx gy gz threads [kv0 kv1]" groups separated by
// " ; " (kv0 kv1 of the fp32 dK/dV), "none" for a pair that is not taken, or
// "error".
#include <hip/hip_runtime.h>
#include <cstdio>
#include <cstring>
#include <iostream>
#include <map>
#include <sstream>
#include <string>

#include "sppo_kernels.h"

static std::map<const void*, std::string>& names() {
  static std::map<const void*, std::string> m;
  return m;
}
static std::string launched;

extern "C" void __hipRegisterFunction(void**, const void* host, char* device, const char*, unsigned, void*, void*, void*,
                                      void*, int*) {
  names()[host] = device;
}
static dim3 conf_grid, conf_block;
extern "C" hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t, hipStream_t) {
  conf_grid = g;
  conf_block = b;
  return hipSuccess;
}
extern "C" hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* shmem, hipStream_t* s) {
  *g = conf_grid;
  *b = conf_block;
  *shmem = 0;
  *s = nullptr;
  return hipSuccess;
}
extern "C" hipError_t hipGetLastError(void) { return hipSuccess; }
extern "C" hipError_t hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t, hipStream_t) {
  char line[256];
  std::string extra;
  if (names()[f].find("dkdv_f32_kernel") != std::string::npos) {
    const auto* a = static_cast<const sppo::ChunkArgs*>(args[0]);
    extra = " " + std::to_string(a->kv0) + " " + std::to_string(a->kv1);
  }
  std::snprintf(line, sizeof line, "%s %u %u %u %u%s", names()[f].c_str(), g.x, g.y, g.z, b.x, extra.c_str());
  launched += (launched.empty() ? "" : " ; ") + std::string(line);
  return hipSuccess;
}

int main() {
  std::string line;
  static int tiles[sppo::kTileQueueInts];
  while (std::getline(std::cin, line)) {
    std::istringstream in(line);
    std::string op, dt;
    in >> op;
    launched.clear();
    hipError_t e = hipSuccess;
    bool none = false;
    if (op == "gemm") {
      sppo::GemmArgs g{};
      in >> g.tn >> g.epi >> g.M >> g.N >> g.K;
      e = sppo::launch_gemm_bf16(g, nullptr);
    } else {
      sppo::ChunkArgs a{};
      in >> dt >> a.B >> a.Hq >> a.Hkv >> a.D >> a.S >> a.c0 >> a.c1;
      a.kv1 = a.c1;
      int64_t lo, hi;
      if (in >> lo >> hi) a.kv0 = lo, a.kv1 = hi;
      a.tiles = tiles;
      a.n_cu = sppo::device_cus();
      // buffers apart from each other, as a caller's are; nothing is read
      const int64_t q = a.B * a.S * a.Hq * a.D * 4;
      const void** in_ptr[] = {&a.q, &a.k, &a.v, &a.dout};
      int64_t at = 1 << 20;
      for (const void** p : in_ptr) *p = reinterpret_cast<const void*>(at), at += q;
      a.dq = reinterpret_cast<void*>(at);
      const bool b = dt == "bf16";
      if (op == "fwd") e = b ? sppo::launch_fwd_bf16(a, nullptr) : sppo::launch_fwd_f32(a, nullptr);
      else if (op == "pre") e = b ? sppo::launch_bwd_pre_bf16(a, nullptr) : sppo::launch_bwd_pre_f32(a, nullptr);
      else if (op == "dkdv") e = b ? sppo::launch_bwd_dkdv_bf16(a, nullptr) : sppo::launch_bwd_dkdv_f32(a, nullptr);
      else if (op == "dq") e = b ? sppo::launch_bwd_dq_bf16(a, nullptr) : sppo::launch_bwd_dq_f32(a, nullptr);
      else if (!(b ? sppo::bwd_pair_bf16(a) : sppo::bwd_pair_f32(a))) none = true;
      else e = b ? sppo::launch_bwd_pair_bf16(a, nullptr) : sppo::launch_bwd_pair_f32(a, nullptr);
    }
    std::puts(none ? "none" : e != hipSuccess ? "error" : launched.c_str());
  }
  return 0;
}
