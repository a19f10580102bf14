// Thresholds of Algorithm 2 from the captured curve (Eq. 1 with a / x^e, or the MLP of Appendix A.3), in binary64 with
// + - * / in a fixed order, so that a CPU reference that performs the same operations gets the same bits.
#ifndef FASTPOINT_ESTIMATOR_H_
#define FASTPOINT_ESTIMATOR_H_

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels.h"

#pragma clang fp contract(off)

namespace fastpoint {
namespace {

// x^e for an integer x >= 1 in binary64 using only + - * / (each correctly rounded
// by IEEE 754), in a fixed order: ln x from the atanh series after scaling x into
// [sqrt(1/2), sqrt(2)), then exp by its Taylor series after removing a multiple of ln 2.
// A CPU reference that performs the same operations in the same order gets the same bits.
__device__ __noinline__ double pow_int_base(int64_t x, double e)
{
    const double LN2 = 0.6931471805599453;
    int k = 63 - __builtin_clzll((unsigned long long)x);
    double f = (double)x * __longlong_as_double((long long)(1023 - k) << 52);   // exact, in [1,2)
    if (f > 1.4142135623730951) {
        f = f * 0.5;
        k = k + 1;
    }
    const double s = (f - 1.0) / (f + 1.0);
    const double s2 = s * s;
    double sum = 0.0;
    // unrolled: the quotients 1/(2t+1) are then constants (rounded correctly when the compiler folds
    // them, the bits the division gives at run time), and thirteen divisions go away
#pragma unroll
    for (int t = 12; t >= 0; --t) sum = sum * s2 + 1.0 / (double)(2 * t + 1);
    const double lnx = ((double)k * LN2) + ((2.0 * s) * sum);
    const double y = e * lnx;
    const double q = floor(y / LN2 + 0.5);
    const double r = y - q * LN2;
    double acc = 1.0;
#pragma unroll 1
    for (int t = 20; t >= 1; --t) acc = 1.0 + acc * (r / (double)t);
    return acc * __longlong_as_double((long long)(1023 + (int)q) << 52);
}

// ln v for a normal positive binary64 v and exp y, with + - * / only in a fixed order (the steps
// pow_int_base is made of): a CPU reference performing the same operations gets the same bits.
__device__ __noinline__ double ln_fixed(double v)
{
    const double LN2 = 0.6931471805599453;
    const long long bits = __double_as_longlong(v);
    int k = (int)((bits >> 52) & 0x7FF) - 1023;
    double f = __longlong_as_double((bits & 0x000FFFFFFFFFFFFFll) | (1023ll << 52));   // in [1,2)
    if (f > 1.4142135623730951) {
        f = f * 0.5;
        k = k + 1;
    }
    const double s = (f - 1.0) / (f + 1.0);
    const double s2 = s * s;
    double sum = 0.0;
    // unrolled: the quotients 1/(2t+1) are then constants (rounded correctly when the compiler folds
    // them, the bits the division gives at run time), and thirteen divisions go away
#pragma unroll
    for (int t = 12; t >= 0; --t) sum = sum * s2 + 1.0 / (double)(2 * t + 1);
    return ((double)k * LN2) + ((2.0 * s) * sum);
}
__device__ __noinline__ double exp_fixed(double y)
{
    const double LN2 = 0.6931471805599453;
    if (!(y >= -700.0)) y = -700.0;
    if (y > 700.0) y = 700.0;
    const double q = floor(y / LN2 + 0.5);
    const double r = y - q * LN2;
    double acc = 1.0;
#pragma unroll 1
    for (int t = 20; t >= 1; --t) acc = 1.0 + acc * (r / (double)t);
    return acc * __longlong_as_double((long long)(1023 + (int)q) << 52);
}

// One layer of the MLP estimator: neuron `o` (of NOUT) starts from its bias and adds the products
// with the NIN inputs in ascending order; weights input-major, so the threads of a wave read
// adjacent words.
template <int NIN, int NOUT, bool RELU>
__device__ __forceinline__ void mlp_layer(const float* __restrict__ w, const float* __restrict__ bias,
                                          const double* in, double* out, int o)
{
    if (o >= NOUT) return;
    double acc = (double)bias[o];
#pragma unroll 4
    for (int k = 0; k < NIN; ++k) acc = acc + (double)w[k * NOUT + o] * in[k];
    out[o] = (RELU && !(acc > 0.0)) ? 0.0 : acc;
}

// segment boundary b_l (curve index whose value becomes R_l), l = 1..nseg
__device__ __forceinline__ int boundary_index(int n, int nseg, int l)
{
    int64_t b = ((int64_t)n * l) / nseg;
    b = b < 1 ? 1 : b;
    b = b > n - 1 ? n - 1 : b;
    return (int)b;
}

// What a workgroup works the thresholds out in: S has ring (the curve's last values, place i & 63), thr_meas (its value at
// the levels' boundaries, where it has got there), mlp_val (its values at the network's inputs), the results thr, and
// the intermediate terms, powb, mlp_a, mlp_b.  Called by all threads; the results are there after the next barrier.
template <class S>
__device__ __forceinline__ void predict_thresholds(const SamplerArgs& a, S& sh, int tid)
{
    [[maybe_unused]] const int n = a.n, m = a.m;
    if (a.use_override) {
        if (tid < a.nseg) sh.thr[tid] = a.thr_override[tid];
    } else if (a.mlp) {
        // ---- MLP estimator (Appendix A.3): 32 log-ratios of the prefix curve in, 64 log-ratios
        //      of the rest of the curve out; every workgroup of the cloud computes the same
        const float* __restrict__ W1 = a.mlp;
        const float* __restrict__ b1 = W1 + 32 * 128;
        const float* __restrict__ W2 = b1 + 128;
        const float* __restrict__ b2 = W2 + 128 * 128;
        const float* __restrict__ W3 = b2 + 128;
        const float* __restrict__ b3 = W3 + 128 * 64;
        const double last = (double)sh.ring[m & 63];
        if (tid < 32) {
            const double ratio = (double)sh.mlp_val[tid] / last;
            sh.mlp_a[tid] = (ratio >= 1.0 && ratio <= 1e300) ? ln_fixed(ratio) : 0.0;
        }
        __syncthreads();
        mlp_layer<32, 128, true>(W1, b1, sh.mlp_a, sh.mlp_b, tid);
        __syncthreads();
        mlp_layer<128, 128, true>(W2, b2, sh.mlp_b, sh.mlp_a, tid);
        __syncthreads();
        mlp_layer<128, 64, false>(W3, b3, sh.mlp_a, sh.mlp_b, tid);
        __syncthreads();
        if (tid < a.nseg) {
            // the estimated curve at this level's boundary: the outputs interpolated linearly
            const int l = tid;
            const int64_t b = boundary_index(n, a.nseg, l + 1);
            float r;
            if (b <= m) {
                r = sh.thr_meas[l];
            } else {
                const double u = ((double)(b - m) * 64.0) / (double)(n - 1 - m);
                int j0 = (int)floor(u);
                if (j0 > 64) j0 = 64;
                const double frac = u - (double)j0;
                const double v0 = j0 == 0 ? 0.0 : sh.mlp_b[j0 - 1];
                const double v1 = j0 >= 64 ? sh.mlp_b[63] : sh.mlp_b[j0];
                const double y = v0 + frac * (v1 - v0);
                r = (float)((a.bias2 * (double)a.level_scale[l]) * (last * exp_fixed(y)));
            }
            if (!(r >= 1.17549435e-38f)) r = 1.17549435e-38f;
            sh.thr[l] = r;
        }
        __syncthreads();
        if (tid == 0)
            for (int l = 1; l < a.nseg; ++l)
                if (sh.thr[l] > sh.thr[l - 1]) sh.thr[l] = sh.thr[l - 1];
    } else {
        const int W = a.fit_window < m ? a.fit_window : m;
        if (tid < W) {
            const int ii = m - W + 1 + tid;
            sh.terms[tid] = (double)sh.ring[ii & 63] * pow_int_base(ii, a.exponent);
        } else if (tid >= 64 && tid < 64 + a.nseg) {
            const int l = tid - 64;
            sh.powb[l] = pow_int_base(boundary_index(n, a.nseg, l + 1), a.exponent);
        }
        __syncthreads();
        if (tid == 0) {
            double acc = 0.0;
            for (int t = 0; t < W; ++t) acc += sh.terms[t];
            acc = acc / (double)W;
            float prev = 0.0f;
            for (int l = 0; l < a.nseg; ++l) {
                float r;
                if (boundary_index(n, a.nseg, l + 1) <= m) r = sh.thr_meas[l];
                else r = (float)(((a.bias2 * (double)a.level_scale[l]) * acc) / sh.powb[l]);
                if (!(r >= 1.17549435e-38f)) r = 1.17549435e-38f;
                if (l >= 1 && r > prev) r = prev;
                sh.thr[l] = r;
                prev = r;
            }
        }
    }
}

}  // namespace
}  // namespace fastpoint
#endif
