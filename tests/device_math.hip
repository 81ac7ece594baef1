// The library's FP64 noise arithmetic (lb_rng.h) evaluated on the device and, from the same header, on the
// host: each function over arrays, for tests/test_gpu_device_math.py.
#include "lb_rng.h"

enum { LN, SIN, COS, RCP, DIV, SQRT, ROOT, RROOT };

// v: the argument (the 21-bit integer for LN, SIN, COS); a: the numerator for DIV
__host__ __device__ static double eval(int what, double a, double v)
{
    double s, c;
    switch (what) {
    case LN: return lbf::u21_ln((uint32_t)v);
    case SIN: lbf::u21_sincos_turn((uint32_t)v, s, c); return s;
    case COS: lbf::u21_sincos_turn((uint32_t)v, s, c); return c;
    case RCP: return lbf::rcp64(v);
    case DIV: return lbf::div64(a, v);
    case SQRT: return lbf::sqrt64(v);
    case ROOT: lbf::sqrt_rsqrt64(v, s, c); return s;
    default: lbf::sqrt_rsqrt64(v, s, c); return c;
    }
}

__global__ void k_eval(int what, const double *a, const double *v, double *out, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = eval(what, a[i], v[i]);
}

extern "C" int device_eval(int what, const double *a, const double *v, double *out, int n, void *stream)
{
    if (n < 1) return 1;
    hipLaunchKernelGGL(k_eval, dim3((n + 255) / 256), dim3(256), 0, (hipStream_t)stream, what, a, v, out, n);
    return (int)hipGetLastError();
}

extern "C" void host_eval(int what, const double *a, const double *v, double *out, int n)
{
    for (int i = 0; i < n; ++i) out[i] = eval(what, a[i], v[i]);
}
