// The short root and division of the model terms (mg_device.h) beside the
// compiler's, for tests/test_gpu_rounding.py.
#include "../../paper_2110_00566_amd/csrc/mg_device.h"

template <typename T>
__global__ void k_rounding(const T *a, const T *b, size_t n, T *root, T *root_ref, T *quot,
                           T *quot_ref) {
    const size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n) return;
    root[t] = mgk::sqrt_normal(a[t]);
    root_ref[t] = sqrt(a[t]);
    quot[t] = mgk::div_normal(a[t], b[t]);
    quot_ref[t] = a[t] / b[t];
}

// a, b, out: device arrays, out of 4 n values (short root, root, short quotient,
// quotient); returns a hipError_t
template <typename T>
static int run(const T *a, const T *b, size_t n, T *out) {
    if (!a || !b || !out || n == 0 || n > (size_t)1 << 28) return (int)hipErrorInvalidValue;
    k_rounding<T><<<(unsigned)((n + 255) / 256), 256>>>(a, b, n, out, out + n, out + 2 * n,
                                                        out + 3 * n);
    const hipError_t e = hipGetLastError();
    return (int)(e == hipSuccess ? hipDeviceSynchronize() : e);
}

extern "C" int rounding_f32(const float *a, const float *b, size_t n, float *out) {
    return run(a, b, n, out);
}
extern "C" int rounding_f64(const double *a, const double *b, size_t n, double *out) {
    return run(a, b, n, out);
}
