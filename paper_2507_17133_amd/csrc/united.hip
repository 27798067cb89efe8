// United experts (United Expert Model): parameter mean of each group of `way` consecutive experts,
// and helpers to evaluate the distillation loss of that section on calibration tokens.
#include "internal.h"

#include <algorithm>

namespace bmoe {

// Round a double to bf16 (8 significant bits), to nearest, ties to even, in one step.
__device__ __forceinline__ unsigned short f64_to_bf16_bits(double v)
{
    const float f = (float)v;                       // nearest float
    unsigned int u = __float_as_uint(f);
    const unsigned int low = u & 0xFFFFu;
    unsigned int up = 0;
    if (low > 0x8000u) up = 1;
    else if (low == 0x8000u) {
        // f sits on a bf16 midpoint; the double may lie to either side of it
        const double rest = fabs(v) - fabs((double)f);
        if (rest > 0.0) up = 1;
        else if (rest < 0.0) up = 0;
        else up = (u >> 16) & 1u;
    }
    return (unsigned short)((u >> 16) + up);
}

// u[g] = mean of the group's members, 8 elements per thread: every member's 16 bytes are read once, four members'
// loads in flight; sums in fp64, in member order.  (2-byte loads: 43 us for 12 experts of 5.8 MB per matrix; so 23.)
__global__ void __launch_bounds__(256) united_mean_kernel(const unsigned short* __restrict__ w, int m, int way,
                                                          size_t n8, unsigned short* __restrict__ u)
{
    const int g = blockIdx.y;
    const int lo = g * way, hi = min(m, lo + way);
    const double k = (double)(hi - lo);
    const size_t n_elem = n8 * 8;
    for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < n8; e += (size_t)gridDim.x * 256) {
        double s[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
        const unsigned short* src = w + (size_t)lo * n_elem + e * 8;
#pragma unroll 4
        for (int i = lo; i < hi; ++i, src += n_elem) {
            const uint4 q = *reinterpret_cast<const uint4*>(src);
            const unsigned v[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                s[2 * c] += (double)__uint_as_float(v[c] << 16);
                s[2 * c + 1] += (double)__uint_as_float(v[c] & 0xFFFF0000u);
            }
        }
        unsigned o[4];
#pragma unroll
        for (int c = 0; c < 4; ++c)
            o[c] = (unsigned)f64_to_bf16_bits(s[2 * c] / k) | ((unsigned)f64_to_bf16_bits(s[2 * c + 1] / k) << 16);
        *reinterpret_cast<uint4*>(u + (size_t)g * n_elem + e * 8) = make_uint4(o[0], o[1], o[2], o[3]);
    }
}

hipError_t launch_united_mean(const bf16_t* w, int m, int way, size_t n_elem, bf16_t* u, hipStream_t s)
{
    const int G = ceil_div(m, way);
    const int bx = (int)std::min<size_t>((n_elem / 8 + 255) / 256, 4096);
    united_mean_kernel<<<dim3(bx, G), 256, 0, s>>>(reinterpret_cast<const unsigned short*>(w), m, way, n_elem / 8,
                                                   reinterpret_cast<unsigned short*>(u));
    return hipGetLastError();
}

// GEMM tile table (see tiles.h) of units that all hold n rows, the k-th of them the rows (first_slot + k) * n ...
__global__ void __launch_bounds__(256) uniform_units_kernel(int u0, int n_units0, int u1, int n_units1, int first_slot, int n,
                                                            int bm, int32_t* __restrict__ table)
{
    const int per = (n + bm - 1) / bm, total = per * (n_units0 + n_units1);
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i == 0) { table[0] = total; table[1] = bm; table[2] = 0; table[3] = 0; }
    if (i >= total) return;
    const int k = i / per, r = (i - k * per) * bm;
    const int unit = k < n_units0 ? u0 + k : u1 + (k - n_units0);
    reinterpret_cast<int4*>(table + 4)[i] = make_int4(unit, (first_slot + k) * n + r, min(bm, n - r), 0);
}

hipError_t launch_uniform_units(int u0, int n_units0, int u1, int n_units1, int first_slot, int n, int bm, int32_t* table,
                                hipStream_t s)
{
    const int total = ceil_div(n, bm) * (n_units0 + n_units1);
    uniform_units_kernel<<<ceil_div(total, 256), 256, 0, s>>>(u0, n_units0, u1, n_units1, first_slot, n, bm, table);
    return hipGetLastError();
}

__global__ void __launch_bounds__(256) repeat_tokens_kernel(int32_t* __restrict__ row_token, int n, int total)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < total) row_token[i] = i % n;
}

hipError_t launch_repeat_tokens(int32_t* row_token, int n, int slots, hipStream_t s)
{
    repeat_tokens_kernel<<<ceil_div(n * slots, 256), 256, 0, s>>>(row_token, n, n * slots);
    return hipGetLastError();
}

// Sum over the block (256 threads) in a fixed order, valid in every thread.
__device__ __forceinline__ double block_sum(double s, double* red)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    return red[0] + red[1] + red[2] + red[3];
}

// Sums of squared differences between the student's rows and those of b teachers (half precision, 8 per thread):
// the student's values are read once per batch of teachers; fp64 partial sums per block.  (As one block per teacher
// this sum alone took 1.2 ms for 2048 tokens of width 2048.)
__global__ void __launch_bounds__(256) sqdiff_kernel(const unsigned short* __restrict__ yu, const unsigned short* __restrict__ yo,
                                                     int b, size_t n8, int first, double* __restrict__ part)
{
    typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
    __shared__ double red[4];
    double s = 0.0;
    for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < n8; e += (size_t)gridDim.x * 256) {
        const f16x8 a = *reinterpret_cast<const f16x8*>(yu + e * 8);
        for (int i = 0; i < b; ++i) {
            const f16x8 c = *reinterpret_cast<const f16x8*>(yo + ((size_t)i * n8 + e) * 8);
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const float df = (float)a[q] - (float)c[q];
                s += (double)df * (double)df;
            }
        }
    }
    const double t = block_sum(s, red);
    if (threadIdx.x == 0) part[blockIdx.x] = first ? t : part[blockIdx.x] + t;
}

__global__ void __launch_bounds__(256) sqdiff_sum_kernel(const double* __restrict__ part, int n, double scale,
                                                         float* __restrict__ loss)
{
    __shared__ double red[4];
    double s = 0.0;
    for (int i = threadIdx.x; i < n; i += 256) s += part[i];
    const double t = block_sum(s, red);
    if (threadIdx.x == 0) *loss = (float)(t * scale);
}

hipError_t launch_sqdiff(const bf16_t* yu, const bf16_t* yo, int b, size_t n, int blocks, bool first, bool last, double scale,
                         double* part, float* loss, hipStream_t s)
{
    sqdiff_kernel<<<blocks, 256, 0, s>>>(reinterpret_cast<const unsigned short*>(yu), reinterpret_cast<const unsigned short*>(yo),
                                         b, n / 8, first, part);
    if (last) sqdiff_sum_kernel<<<1, 256, 0, s>>>(part, blocks, scale, loss);
    return hipGetLastError();
}

}  // namespace bmoe
