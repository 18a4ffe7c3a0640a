// zmc_rtc.hip -- user-defined integrands compiled at run time with hipRTC.
//
// The paper's package integrates general user-defined functions written in
// Python/Numba (abstract, Sec. 3.3).  Here the user supplies the body of a
// device function in C++ syntax,
//
//     template <typename real> real f(const real* x, const double* p)
//     { constexpr int D = <dim>;  <body> }
//
// using x[0..D-1] (the point, `real` is double or float), p[0..n_params-1]
// (the request's params) and D.  The body is compiled once per (D, eval) on
// first use, around the same sampling body as the precompiled registry
// (zmc_sample_core.hpp), and once more with the sums of squares kept if a level
// is traced (a conversion and an FP64 FMA per point: FP32 Gaussian bodies of 1
// to 16 dimensions run 1-7% faster without, FP64 ones 0-2%);
// the device headers are embedded in the library at
// build time, so nothing is read from disk at run time.
#include <hip/hip_runtime.h>
#include <hip/hiprtc.h>

#include <map>
#include <mutex>
#include <string>
#include <tuple>
#include <vector>

#include "zmc_engine.hpp"
#include "zmc_rtc.hpp"
#include "zmc_rtc_embed.inc" // kRtcHeaderNames / kRtcHeaderSources / kRtcHeaderCount

namespace zmc {

namespace {

struct UserDef {
    std::string body;
    int n_params;
};

struct Compiled {
    hipModule_t module = nullptr;
    hipFunction_t fn = nullptr;
    int capacity = 0;
};

// FP32 kernels run four waves per SIMD at least: always from kFourWavesMinD
// dimensions on, below where the compiler's free choice takes more than
// kFourWavesRegs registers, which leaves three.  Against the free choice, in
// 1e9 points/s: Gaussian bodies at D = 9, 10 and 12 283 -> 292, 274 -> 284,
// 236 -> 242; a body of three D x D products, which spills by the bound (128
// registers and up to 720 bytes a lane, for up to 256 registers), at D = 9,
// 12, 14 and 16 19.8 -> 20.5, 12.2 -> 12.9, 4.1 -> 4.8, 7.0 -> 6.9, and at
// D = 3 and 7 157 -> 181 and 33.6 -> 35.5.  A body that fits anyway can lose:
// 1.4% with a Gaussian of 67 registers at D = 3.
constexpr int kFourWavesMinD = 8;
constexpr int kFourWavesRegs = 128;
// From kHalvesMinD dimensions on the words of a whole group take too many
// registers under the compiler's own schedule: in halves the FP32 Gaussian
// body at D = 14 takes 126 of them for 146 (198 -> 207e9 points/s), at D = 16
// spills 20 bytes for 84 (154 -> 158), and the same at D = 12 in FP64 140 for
// 150 (180, 180); a body of D (D - 1) / 2 quotients at D = 16 22.3 -> 22.6.
// At D = 8 and 9 halves gain 0-4% with bodies that spill and lose 0-3% with others.
// An odd number of dimensions leaves words of the first half to the second, and
// an FP32 body that spills under the bound is then tried once more with the
// halves kept apart; the build that spills nothing is kept.  11- and 13-D
// Gaussian bodies spill 28 and 64 bytes a lane one way and nothing the other,
// 247 -> 255 and 211 -> 222, 11- and 13-D products of D factors 305 -> 312 and
// 257 -> 266.  Kept apart at even D they lose 2-4% though the spills go
// (Gaussian at 10-D 286 -> 276, at 12-D 244 -> 234), and so do bodies that
// spill nothing (damped wave at 11- and 13-D 3% and 2%).
constexpr int kHalvesMinD = 10;

std::mutex g_mu;
std::vector<UserDef> g_defs;
std::map<std::tuple<int, int, int, bool>, Compiled> g_cache; // (id, D, eval, sums of squares kept)

const char* kPrelude = R"ZMCRTC(
typedef __hip_internal::uint64_t uint64_t;
typedef __hip_internal::int64_t int64_t;
typedef __hip_internal::uint32_t uint32_t;
typedef __hip_internal::int32_t int32_t;
typedef __hip_internal::uint8_t uint8_t;
)ZMCRTC";

std::string program_source(const std::string& body, int dim, bool fp32, bool keep_s2, bool four_waves, int halves)
{
    std::string s = kPrelude;
    s += "#define ZMC_D " + std::to_string(dim) + "\n";
    s += "#define ZMC_FP32 " + std::string(fp32 ? "true" : "false") + "\n";
    s += "#define ZMC_OCCUPANCY " + std::string(four_waves ? "__attribute__((amdgpu_waves_per_eu(4)))" : "") + "\n";
    s += "#define ZMC_HALVES " + std::to_string(halves) + "\n";
    s += "#define ZMC_KEEP_S2 " + std::string(keep_s2 ? "true" : "false") + "\n";
    s += R"ZMCRTC(
#include "zmc_sample_core.hpp"
#include "zmc_trig.hpp"
namespace zmc_user {
// sin and cos of a double in the user's body are the registry's (other
// argument types keep the library's)
template <typename T> struct IsDouble { static constexpr bool value = false; };
template <> struct IsDouble<double> { static constexpr bool value = true; };
template <typename T>
__device__ __forceinline__ auto sin(T t) -> decltype(::sin(t))
{
    if constexpr (IsDouble<T>::value) return zmc::sin_f64(t);
    else return ::sin(t);
}
template <typename T>
__device__ __forceinline__ auto cos(T t) -> decltype(::cos(t))
{
    if constexpr (IsDouble<T>::value) return zmc::cos_f64(t);
    else return ::cos(t);
}
template <typename real>
__device__ __forceinline__ real f(const real* x, const double* p)
{
    constexpr int D = ZMC_D;
    (void)D;
    (void)p;
#line 1 "user integrand"
)ZMCRTC";
    s += body;
    s += R"ZMCRTC(
}
} // namespace zmc_user
namespace zmc {
// Adapter to the sampling body: FP64 from the absolute point; FP32 from the
// cell values v in [1, 2), x_i = (lo_i - h_i (1 - 2^-24)) + h_i v_i.
template <int D>
struct UserIntegrand {
    static constexpr bool kRangeCheck = true;
    static constexpr bool kProduct = true; // it may be
    struct P64 {
        const double* prm;
    };
    struct P32 {
        float b[D], m[D];
        const double* prm;
        double scale;
    };
    __device__ static void prep64(const SlotDesc& sd, P64& p) { p.prm = sd.params; }
    __device__ static double f64(const P64& p, const double* x) { return zmc_user::f<double>(x, p.prm); }
    __device__ static void prep32(const SlotDesc& sd, const double* lo, const double* h, P32& p)
    {
        for (int i = 0; i < D; ++i) {
            p.b[i] = (float)(lo[i] - h[i] * (1.0 - 0x1p-24));
            p.m[i] = (float)h[i];
        }
        p.prm = sd.params;
        p.scale = 1.0;
    }
    __device__ static float f32(const P32& p, const float* v)
    {
        float x[D];
#pragma unroll
        for (int i = 0; i < D; ++i) x[i] = __builtin_fmaf(p.m[i], v[i], p.b[i]);
        return zmc_user::f<float>(x, p.prm);
    }
};
} // namespace zmc
extern "C" __global__ __launch_bounds__(256) ZMC_OCCUPANCY void zmc_user_kernel(const zmc::SampleArgs a)
{
    zmc::sample_units<zmc::UserIntegrand<ZMC_D>, ZMC_D, ZMC_FP32, ZMC_KEEP_S2, ZMC_HALVES>(a);
}
)ZMCRTC";
    return s;
}

// Compile one variant to a code object; returns 0 and fills `code`, or -1
// with the compiler log in `log`.
int compile(const std::string& body, int dim, bool fp32, bool keep_s2, bool four_waves, int halves,
            std::vector<char>& code, std::string& log)
{
    const std::string src = program_source(body, dim, fp32, keep_s2, four_waves, halves);
    hiprtcProgram prog;
    if (hiprtcCreateProgram(&prog, src.c_str(), "zmc_user.hip", kRtcHeaderCount, kRtcHeaderSources,
                            kRtcHeaderNames) != HIPRTC_SUCCESS) {
        log = "hiprtcCreateProgram failed";
        return -1;
    }
    // no packed FP32 instructions (v_pk_*_f32) and aligned loop headers, as in
    // the precompiled kernels (not their scheduling strategy, which has been
    // seen through on known integrands only)
    const char* opts[] = {"--gpu-architecture=gfx950", "-O3", "-std=c++17",
                          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-falign-loops=64"};
    const hiprtcResult rc = hiprtcCompileProgram(prog, (int)(sizeof(opts) / sizeof(opts[0])), opts);
    size_t ls = 0;
    hiprtcGetProgramLogSize(prog, &ls);
    if (ls > 1) {
        std::vector<char> b(ls + 1, 0);
        hiprtcGetProgramLog(prog, b.data());
        log = b.data();
    }
    if (rc != HIPRTC_SUCCESS) {
        hiprtcDestroyProgram(&prog);
        if (log.empty()) log = hiprtcGetErrorString(rc);
        return -1;
    }
    size_t cs = 0;
    hiprtcGetCodeSize(prog, &cs);
    code.resize(cs);
    hiprtcGetCode(prog, code.data());
    hiprtcDestroyProgram(&prog);
    return 0;
}

} // namespace

int rtc_register(const char* body, int n_params, int* id)
{
    if (!body || !id || n_params < 0 || n_params > ZMC_MAX_PARAMS) {
        set_error("register_integrand: bad arguments");
        return ZMC_EINVAL;
    }
    // compile once (D = 4, FP64) so that syntax errors surface now
    std::vector<char> code;
    std::string log;
    if (compile(body, 4, false, false, false, 0, code, log) != 0) {
        set_error("user integrand does not compile:\n" + log);
        return ZMC_EINVAL;
    }
    std::lock_guard<std::mutex> lk(g_mu);
    if ((int)g_defs.size() >= kMaxUserIntegrands) {
        set_error("too many user integrands");
        return ZMC_EINVAL;
    }
    g_defs.push_back(UserDef{body, n_params});
    *id = kUserBase + (int)g_defs.size() - 1;
    return ZMC_OK;
}

int rtc_n_params(int id)
{
    std::lock_guard<std::mutex> lk(g_mu);
    const int k = id - kUserBase;
    if (k < 0 || k >= (int)g_defs.size()) return -1;
    return g_defs[k].n_params;
}

// The kernel for (id, D, eval) on the current device, compiled on first use.
// The compiler runs outside the lock, so launches of kernels already built
// never wait behind a compilation.
static int rtc_get(int id, int dim, int eval, bool keep_s2, Compiled& out)
{
    const auto key = std::make_tuple(id, dim, eval, keep_s2);
    std::string body;
    {
        std::lock_guard<std::mutex> lk(g_mu);
        auto it = g_cache.find(key);
        if (it != g_cache.end()) {
            out = it->second;
            return ZMC_OK;
        }
        const int k = id - kUserBase;
        if (k < 0 || k >= (int)g_defs.size()) {
            set_error("unknown user integrand");
            return ZMC_EINVAL;
        }
        body = g_defs[k].body;
    }
    const bool fp32 = eval == ZMC_EVAL_FP32;
    auto load = [&](bool four_waves, int halves, Compiled& k) -> int {
        std::vector<char> code;
        std::string log;
        if (compile(body, dim, fp32, keep_s2, four_waves, halves, code, log) != 0) {
            set_error("user integrand does not compile:\n" + log);
            return ZMC_EINVAL;
        }
        hipError_t e = hipModuleLoadData(&k.module, code.data());
        if (e == hipSuccess) e = hipModuleGetFunction(&k.fn, k.module, "zmc_user_kernel");
        if (e != hipSuccess) {
            set_error(std::string("loading the user kernel: ") + hipGetErrorString(e));
            return ZMC_EDEVICE;
        }
        return ZMC_OK;
    };
    auto attribute = [](const Compiled& k, hipFunction_attribute a) {
        int v = 0;
        return hipFuncGetAttribute(&v, a, k.fn) == hipSuccess ? v : 0;
    };
    const int halves = dim >= kHalvesMinD ? 1 : 0;
    Compiled c;
    const int rc = load(fp32 && dim >= kFourWavesMinD, halves, c);
    if (rc != ZMC_OK) return rc;
    // a second build, kept where it serves; should it fail, the first stands
    const bool bound = fp32 && dim < kFourWavesMinD && attribute(c, HIP_FUNC_ATTRIBUTE_NUM_REGS) > kFourWavesRegs;
    const bool apart =
        fp32 && halves && dim % 2 == 1 && attribute(c, HIP_FUNC_ATTRIBUTE_LOCAL_SIZE_BYTES) > 0;
    Compiled b;
    if ((bound || apart) && load(true, apart ? 2 : halves, b) == ZMC_OK) {
        if (apart && attribute(b, HIP_FUNC_ATTRIBUTE_LOCAL_SIZE_BYTES) > 0) std::swap(b, c);
        (void)hipModuleUnload(c.module);
        c = b;
    }
    std::lock_guard<std::mutex> lk(g_mu);
    auto it = g_cache.find(key);
    if (it != g_cache.end()) { // built meanwhile by another thread
        (void)hipModuleUnload(c.module);
        out = it->second;
        return ZMC_OK;
    }
    int nb = 0, dev = 0, ncu = 0;
    if (hipModuleOccupancyMaxActiveBlocksPerMultiprocessor(&nb, c.fn, kSampleThreads, 0) != hipSuccess || nb < 1)
        nb = 1;
    (void)hipGetDevice(&dev);
    (void)hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev);
    c.capacity = nb * (ncu > 0 ? ncu : 1);
    g_cache[key] = c;
    out = c;
    return ZMC_OK;
}

int rtc_launch(int id, int dim, int eval, bool keep_s2, hipStream_t st, const SampleArgs& a)
{
    Compiled c;
    const int rc = rtc_get(id, dim, eval, keep_s2, c);
    if (rc != ZMC_OK) return rc;
    const unsigned grid = (unsigned)std::min<int64_t>(a.total_units, c.capacity);
    SampleArgs arg = a;
    void* params[] = {&arg};
    const hipError_t e = hipModuleLaunchKernel(c.fn, grid, 1, 1, kSampleThreads, 1, 1, 0, st, params, nullptr);
    if (e != hipSuccess) {
        set_error(std::string("launching the user kernel: ") + hipGetErrorString(e));
        return ZMC_EDEVICE;
    }
    return ZMC_OK;
}

} // namespace zmc
