// device_math.hip -- the device header's shortened quotients and roots over whole
// ranges and on given operands, for tests/test_gpu_math.py (built by the package's
// build module with the library's flags into tests/libdevice_math.so).
#include "../paper_2308_09209_amd/csrc/vs_device.h"

using namespace vs;

namespace {

enum { RCP = 0, HALF_RSQRT = 1 };

__device__ __forceinline__ float shortened(int what, float x) { return what == RCP ? div_rcp(x) : half_rsqrt(x); }
__device__ __forceinline__ float operators(int what, float x) { return what == RCP ? 1.0f / x : 0.5f / sqrtf(x); }

// floats of the bit patterns [lo, lo + n): out[0] those whose shortened form has other
// bits than the operators', out[1] the least such pattern
__global__ __launch_bounds__(256) void k_sweep(int what, uint32_t lo, uint32_t n, unsigned long long* out)
{
    for (uint32_t i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) {
        const float x = __uint_as_float(lo + i);
        if (__float_as_uint(shortened(what, x)) != __float_as_uint(operators(what, x))) {
            atomicAdd(out, 1ull);
            atomicMin(out + 1, (unsigned long long)(lo + i));
        }
    }
}

// what 0, 1: the shortened forms; 2, 3: the operators
__global__ __launch_bounds__(256) void k_unary(int what, const float* x, float* y, int n)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) y[i] = what < 2 ? shortened(what, x[i]) : operators(what - 2, x[i]);
}

__global__ __launch_bounds__(256) void k_div(const float* a, const float* d, float* q, int n)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) q[i] = div_by(a[i], d[i], div_rcp(d[i]));
}

__global__ __launch_bounds__(256) void k_hom_div(const float* nu, const float* nv, const float* w, float* u, float* v,
                                                 int* ok, int n)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    float a, b;
    ok[i] = hom_div(nu[i], nv[i], w[i], a, b);
    u[i] = a;
    v[i] = b;
}

}  // namespace

extern "C" {

// n up to 2^31, lo + n - 1 a valid pattern; out two words on the device, 0 and ~0 before
int dm_sweep(int what, uint32_t lo, uint32_t n, unsigned long long* out)
{
    if (what < 0 || what > 1 || n == 0 || n > 0x80000000u || lo > 0xffffffffu - n) return -1;
    hipLaunchKernelGGL(k_sweep, dim3(8192), dim3(256), 0, nullptr, what, lo, n, out);
    return (int)hipGetLastError();
}

int dm_unary(int what, const float* x, float* y, int n)
{
    if (what < 0 || what > 3 || n < 1 || n > 1 << 30) return -1;
    hipLaunchKernelGGL(k_unary, dim3((n + 255) / 256), dim3(256), 0, nullptr, what, x, y, n);
    return (int)hipGetLastError();
}

int dm_div(const float* a, const float* d, float* q, int n)
{
    if (n < 1 || n > 1 << 30) return -1;
    hipLaunchKernelGGL(k_div, dim3((n + 255) / 256), dim3(256), 0, nullptr, a, d, q, n);
    return (int)hipGetLastError();
}

int dm_hom_div(const float* nu, const float* nv, const float* w, float* u, float* v, int* ok, int n)
{
    if (n < 1 || n > 1 << 30) return -1;
    hipLaunchKernelGGL(k_hom_div, dim3((n + 255) / 256), dim3(256), 0, nullptr, nu, nv, w, u, v, ok, n);
    return (int)hipGetLastError();
}

}
