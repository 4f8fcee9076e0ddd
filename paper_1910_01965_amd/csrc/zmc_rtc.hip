// zmc_rtc.hip -- user integrands compiled at run time (include/zmc.h).
//
// A handle keeps the user's source.  A scan of family ZMC_USER needs the
// kernels for its (precision, N, M): the first such scan builds a program
// from the library's own device headers (embedded in the library at build
// time), the user's source and four extern "C" kernels that instantiate the
// same point-major, sample-major, per-sample-value and persistent batch bodies
// as the compiled-in families, compiles it with hipRTC for gfx950, and keeps
// the code object; each device loads it once as a module.  The split merges
// are the library's compiled-in kernels.
#include <hip/hip_runtime.h>
#include <hip/hiprtc.h>
#include <string.h>

#include <algorithm>
#include <chrono>
#include <map>
#include <mutex>
#include <new>
#include <string>
#include <tuple>
#include <vector>

#include "zmc.h"
#include "zmc_device.hpp"
#include "zmc_internal.hpp"
#include "zmc_trace.hpp"

using zmc::fail;
using zmc::ok;

namespace {

// The device headers as text: kRtcHeaderCount, kRtcHeaderNames[],
// kRtcHeaderTexts[] (generated by the build from csrc/).
#include "zmc_rtc_headers.inc"

constexpr size_t kMaxSourceBytes = (size_t)1 << 20;
constexpr size_t kMaxLogInError = 4000;

struct Loaded {
  hipModule_t module = nullptr;
  hipFunction_t pm = nullptr, sm = nullptr, values = nullptr, batch = nullptr;
};

// The kernels of one variant; `big`: the sample-major kernel for blocks of more than
// 256 threads alone.
std::string program_text(const std::string& user, int precision, int N, int M, bool big) {
  const char* T = precision == ZMC_FP64 ? "double" : "float";
  std::string s;
  s += "#include \"zmc_scan.hpp\"\n";
  s += "#line 1 \"integrand\"\n";
  s += user;
  s += "\n#line 1 \"zmc_user_kernels\"\n#include \"zmc_user.hpp\"\n";
  const std::string fam = std::string("zmc::UserFamily<") + T + ", " + std::to_string(N) + ", " +
                          std::to_string(M) + ">, " + T + ", " + std::to_string(N);
  // sample-major blocks of up to 256 threads (every automatic plan and all of
  // N > 8), and of up to 1024 for explicit plans, whose bound of 128 VGPRs a lane
  // can make FP64 integrands spill: that kernel is built when a plan asks for it,
  // since each kernel is a fifth of a variant's build time
  s += std::string("extern \"C\" __global__ __launch_bounds__(") + (big ? "1024" : "256") +
       ") void zmc_user_sample_major(zmc::ScanParams p) {\n";
  s += "  __shared__ double lds[zmc::kSmLds];\n  zmc::sample_major_body<" + fam + ">(p, lds);\n}\n";
  if (big) return s;
  s += "extern \"C\" __global__ __launch_bounds__(256) void zmc_user_point_major(zmc::ScanParams p) {\n";
  s += "  zmc::point_major_body<" + fam + ">(p);\n}\n";
  s += "extern \"C\" __global__ __launch_bounds__(256) void zmc_user_values(zmc::ScanParams p, "
       "uint64_t g, uint64_t s0, int64_t count, double* out) {\n";
  s += "  zmc::debug_values_body<" + fam + ">(p, g, s0, count, out);\n}\n";
  s += "extern \"C\" __global__ __launch_bounds__(256) void zmc_user_batch("
       "const zmc::ScanParams* __restrict__ scans, const zmc::Tile* __restrict__ tiles, "
       "uint32_t begin, uint32_t end, uint32_t* counter) {\n";
  s += "  __shared__ uint32_t next;\n  __shared__ double lds[zmc::kSmLds];\n";
  s += "  zmc::batch_body<" + fam + ">(scans, tiles, begin, end, counter, &next, lds);\n}\n";
  return s;
}

}  // namespace

struct zmc_integrand {
  std::string source;
  uint32_t flags = 0;  // ZMC_INTEGRAND_* bits
  std::mutex mu;
  std::string log;
  std::map<std::tuple<int, int, int, bool>, std::vector<char>> code;  // (precision, N, M, big)
  std::map<std::tuple<int, int, int, int, bool>, Loaded> loaded;      // (device, precision, N, M, big)
};

namespace {

// Compiles one variant into h->code; the caller holds h->mu.
zmc_status compile_variant(zmc_integrand* h, int precision, int N, int M, bool big = false) {
  zmc::TraceRange trace_range("zmc_integrand compile");
  const auto key = std::make_tuple(precision, N, M, big);
  if (h->code.count(key)) return ZMC_OK;
  const std::string text = program_text(h->source, precision, N, M, big);
  const auto t0 = std::chrono::steady_clock::now();
  hiprtcProgram prog = nullptr;
  hiprtcResult r = hiprtcCreateProgram(&prog, text.c_str(), "zmc_user.hip", kRtcHeaderCount,
                                       kRtcHeaderTexts, kRtcHeaderNames);
  if (r != HIPRTC_SUCCESS) return fail(ZMC_E_DEVICE, "hiprtcCreateProgram: %s", hiprtcGetErrorString(r));
  std::vector<const char*> opts = {"--offload-arch=gfx950", "-O3", "-std=c++17",
                                   "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"};
  if ((h->flags & ZMC_INTEGRAND_FAST_MATH) && precision == ZMC_FP32_MERGE64) {
    opts.push_back("-fgpu-approx-transcendentals");
    opts.push_back("-fapprox-func");
  }
  r = hiprtcCompileProgram(prog, (int)opts.size(), opts.data());
  size_t n = 0;
  h->log.clear();
  if (hiprtcGetProgramLogSize(prog, &n) == HIPRTC_SUCCESS && n > 1) {
    h->log.resize(n);
    if (hiprtcGetProgramLog(prog, &h->log[0]) != HIPRTC_SUCCESS) h->log.clear();
    while (!h->log.empty() && h->log.back() == '\0') h->log.pop_back();
  }
  if (r != HIPRTC_SUCCESS) {
    (void)hiprtcDestroyProgram(&prog);
    return fail(ZMC_E_INVALID, "user integrand (precision %d, N = %d, M = %d) does not compile: %s\n%.*s",
                precision, N, M, hiprtcGetErrorString(r), (int)std::min(h->log.size(), kMaxLogInError),
                h->log.c_str());
  }
  std::vector<char> co;
  r = hiprtcGetCodeSize(prog, &n);
  if (r == HIPRTC_SUCCESS) {
    co.resize(n);
    r = hiprtcGetCode(prog, co.data());
  }
  (void)hiprtcDestroyProgram(&prog);
  zmc::log(1, "user integrand: compiled the (precision %d, N = %d, M = %d)%s variant in %.2f s",
           precision, N, M, big ? " large-block" : "",
           std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count());
  if (r != HIPRTC_SUCCESS) return fail(ZMC_E_DEVICE, "hiprtcGetCode: %s", hiprtcGetErrorString(r));
  h->code[key] = std::move(co);
  return ZMC_OK;
}

// Compiles and loads one variant on the current device; the caller holds h->mu.
zmc_status load_variant(zmc_integrand* h, int dev, int precision, int N, int M, bool big, Loaded* out) {
  const zmc_status st = compile_variant(h, precision, N, M, big);
  if (st != ZMC_OK) return st;
  Loaded& L = h->loaded[std::make_tuple(dev, precision, N, M, big)];
  if (L.module == nullptr) {
    const std::vector<char>& co = h->code[std::make_tuple(precision, N, M, big)];
    hipModule_t mod = nullptr;
    hipError_t e = hipModuleLoadData(&mod, co.data());
    if (e == hipSuccess) e = hipModuleGetFunction(&L.sm, mod, "zmc_user_sample_major");
    if (e == hipSuccess && !big) e = hipModuleGetFunction(&L.pm, mod, "zmc_user_point_major");
    if (e == hipSuccess && !big) e = hipModuleGetFunction(&L.values, mod, "zmc_user_values");
    if (e == hipSuccess && !big) e = hipModuleGetFunction(&L.batch, mod, "zmc_user_batch");
    if (e != hipSuccess) {
      if (mod != nullptr) (void)hipModuleUnload(mod);
      L = Loaded{};
      return fail(ZMC_E_DEVICE, "loading the user integrand's kernels: %s", hipGetErrorString(e));
    }
    L.module = mod;
  }
  *out = L;
  return ZMC_OK;
}

}  // namespace

namespace zmc {

zmc_status user_kernels(const zmc_integrand* hc, int precision, int N, int M, UserKernels* out, int block) {
  zmc_integrand* h = const_cast<zmc_integrand*>(hc);
  std::lock_guard<std::mutex> lk(h->mu);
  int dev = 0;
  const hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return fail(ZMC_E_DEVICE, "hipGetDevice: %s", hipGetErrorString(e));
  Loaded L, B;
  zmc_status st = load_variant(h, dev, precision, N, M, false, &L);
  if (st == ZMC_OK && block > 256) st = load_variant(h, dev, precision, N, M, true, &B);
  if (st != ZMC_OK) return st;
  out->pm = L.pm;
  out->sm = L.sm;
  out->sm_big = B.sm;
  out->values = L.values;
  out->batch = L.batch;
  return ok();
}

hipError_t user_batch_occupancy(const UserKernels& k, int* blocks_per_cu) {
  return hipModuleOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, k.batch, 256, 0);
}

hipError_t launch_user_batch(const UserKernels& k, const ScanParams* scans, const Tile* tiles,
                             uint32_t begin, uint32_t end, uint32_t* counter, unsigned blocks,
                             hipStream_t stream) {
  void* args[] = {&scans, &tiles, &begin, &end, &counter};
  return hipModuleLaunchKernel(k.batch, blocks, 1, 1, 256, 1, 1, 0, stream, args, nullptr);
}

hipError_t launch_user_scan(const UserKernels& k, const ScanParams& p, const Plan& plan,
                            hipStream_t stream, hipEvent_t ev_begin, hipEvent_t ev_end) {
  hipError_t e = hipSuccess;
  if (ev_begin != nullptr) e = hipEventRecord(ev_begin, stream);
  ScanParams arg = p;
  void* args[] = {&arg};
  const hipFunction_t f = plan.mode == ZMC_MODE_POINT_MAJOR ? k.pm : plan.block > 256 ? k.sm_big : k.sm;
  if (f == nullptr) return hipErrorInvalidValue;  // user_kernels was not told of such a block
  if (e == hipSuccess)
    e = hipModuleLaunchKernel(f, (unsigned)plan.grid_x, (unsigned)plan.splits, 1, (unsigned)plan.block,
                              1, 1, 0, stream, args, nullptr);
  if (e == hipSuccess && ev_end != nullptr) e = hipEventRecord(ev_end, stream);
  if (e != hipSuccess || p.splits == 1) return e;
  return launch_merge_splits(p, stream);
}

hipError_t launch_user_values(const UserKernels& k, const ScanParams& p, uint64_t g, uint64_t s0,
                              int64_t count, double* out, hipStream_t stream) {
  if (count <= 0) return hipSuccess;
  ScanParams arg = p;
  void* args[] = {&arg, &g, &s0, &count, &out};
  return hipModuleLaunchKernel(k.values, (unsigned)((count + 255) / 256), 1, 1, 256, 1, 1, 0, stream,
                               args, nullptr);
}

}  // namespace zmc

extern "C" {

zmc_status zmc_integrand_create(const char* source, zmc_integrand** out) {
  return zmc_integrand_create_ex(source, 0, out);
}

zmc_status zmc_integrand_create_ex(const char* source, uint32_t flags, zmc_integrand** out) {
  if (out == nullptr) return fail(ZMC_E_INVALID, "out is NULL");
  *out = nullptr;
  if (source == nullptr) return fail(ZMC_E_INVALID, "source is NULL");
  if (flags & ~ZMC_INTEGRAND_FAST_MATH) return fail(ZMC_E_INVALID, "unknown flags 0x%x", flags);
  const size_t len = strnlen(source, kMaxSourceBytes + 1);
  if (len == 0 || len > kMaxSourceBytes) return fail(ZMC_E_INVALID, "source is empty or longer than 1 MiB");
  zmc_integrand* h = new (std::nothrow) zmc_integrand();
  if (h == nullptr) return fail(ZMC_E_NOMEM, "host allocation failed");
  h->source.assign(source, len);
  h->flags = flags;
  zmc_status st;
  {
    std::lock_guard<std::mutex> lk(h->mu);
    st = compile_variant(h, ZMC_FP64, 1, 0);  // reports errors now
    // a fast-math handle also compiles an FP32 variant now, so that an error
    // only the approximate functions would raise is reported here too
    if (st == ZMC_OK && (flags & ZMC_INTEGRAND_FAST_MATH)) st = compile_variant(h, ZMC_FP32_MERGE64, 1, 0);
  }
  if (st != ZMC_OK) {
    delete h;
    return st;
  }
  *out = h;
  return ok();
}

const char* zmc_integrand_log(const zmc_integrand* h) {
  return h == nullptr ? "" : h->log.c_str();
}

zmc_status zmc_integrand_destroy(zmc_integrand* h) {
  if (h == nullptr) return ok();
  int dev = 0;
  const bool have_dev = hipGetDevice(&dev) == hipSuccess;
  for (auto& kv : h->loaded) {
    if (kv.second.module == nullptr) continue;
    (void)hipSetDevice(std::get<0>(kv.first));  // a module belongs to its device
    (void)hipDeviceSynchronize();               // no kernel of it may still run
    (void)hipModuleUnload(kv.second.module);
  }
  if (have_dev) (void)hipSetDevice(dev);
  delete h;
  return ok();
}

}  // extern "C"
