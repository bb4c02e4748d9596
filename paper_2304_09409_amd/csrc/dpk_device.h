// dpk_device.h -- device helpers shared by the embedding (network and table paths) and fitting kernels.
#pragma once
#include <hip/hip_runtime.h>

namespace dpk {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));

// Wave-scope ordering of LDS traffic between lanes of one wave.
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// No vector memory access moves across this point in the instruction schedule (everything else may):
// the scheduler otherwise sinks a load that fills a register ring ahead of its use down to that use,
// to save registers, and the wave waits for its whole latency.
__device__ __forceinline__ void keep_loads() { __builtin_amdgcn_sched_barrier(0x78f); }

// Switching function of Sec. II.A.1 (eq. switch) and its derivative, FP64, from r, ir = 1/r and
// inv_w = 1/(rc - rs) (no division here: the caller's 1/r is the only one per neighbour).
__device__ __forceinline__ void switch_fn(double r, double ir, double rs, double rc, double inv_w, double& s,
                                          double& ds)
{
    if (r < rs) {
        s = ir;
        ds = -ir * ir;
    } else if (r < rc) {
        // u = x^3 (-6 x^2 + 15 x - 10) + 1 as (1 - x)^3 (1 + 3 x + 6 x^2): no cancellation near
        // r_c, so s >= 0 (a table counts negative inputs as out of range)
        double x = (r - rs) * inv_w;
        double y = 1.0 - x;
        double u = y * y * y * (1.0 + x * (3.0 + 6.0 * x));
        double du = -30.0 * x * x * y * y;
        s = u * ir;
        ds = du * ir * inv_w - u * ir * ir;
    } else {
        s = 0.0;
        ds = 0.0;
    }
}

// FP64 hyperbolic tangent from a table in LDS (the embedding passes evaluate 49 of these per lane
// and 16-pair chunk and share the FP64 unit with their matrix products). With x0 = k / 32 the node nearest to
// |x| and d = |x| - x0 (exact, |d| <= 1/64), t = tanh x0 from the table (the device library's tanh),
// u = tanh d = d - d^3/3 + 2 d^5/15 - 17 d^7/315 (next term below 1e-16 relative):
//   tanh |x| = (t + u) / (1 + t u) = t + u (1 - t^2) / (1 + t u),
// and, with e = t u (|e| < 1/64), 1 / (1 + e) = (1 - e)(1 + e^2)(1 + e^4) up to e^8 < 4e-15, which
// the factor u scales below 1e-16. 19 FP64 operations and an LDS read; (e^2x - 1) / (e^2x + 1) by a
// degree-13 series and two Newton steps took 41 and a reciprocal (12,288-atom water box, forward 677
// against 548 us, backward 1050 against 894, with the padded registers left out). |x| is clamped to
// TH_MAX, past which tanh is +-1 in double; NaN propagates (the index is bounded). Against the 80-bit C
// library at 4.2 million points over [-25, 25] and down to 1e-15: within 1.9 ulp relative and 1.15e-16
// absolute (the series: 3 ulp, 1.5 ulp(1)).
constexpr int TH_STEP = 32;
constexpr double TH_MAX = 19.5;
constexpr int TH_N = (int)(TH_MAX * TH_STEP) + 1;
__device__ __forceinline__ double tanh_tab(double x, const double* th)
{
    const double ax = __builtin_fabs(x), xa = ax > TH_MAX ? TH_MAX : ax;
    // adding 1.5 x 2^52 rounds to the nearest integer and leaves it in the low word
    const double kb = __builtin_fma(xa, (double)TH_STEP, 6755399441055744.0);
    const unsigned k = min((unsigned)__double_as_longlong(kb), (unsigned)(TH_N - 1));
    const double d = __builtin_fma(kb - 6755399441055744.0, -1.0 / TH_STEP, xa);
    const double t = th[k];
    const double q = d * d;
    double p = __builtin_fma(q, -17.0 / 315.0, 2.0 / 15.0);
    p = __builtin_fma(q, p, -1.0 / 3.0);
    const double u = __builtin_fma(d * q, p, d);
    const double e = t * u, e2 = e * e, e4 = e2 * e2;
    double v = u * __builtin_fma(-t, t, 1.0);
    v = __builtin_fma(-e, v, v);
    v = __builtin_fma(e2, v, v);
    return __builtin_copysign(t + __builtin_fma(e4, v, v), x);
}
__device__ __forceinline__ void tanh_tab_fill(double* th)
{
    for (int i = threadIdx.x; i < TH_N; i += blockDim.x) th[i] = tanh((double)i / TH_STEP);
}

// FP32 hyperbolic tangent: 1 - 2 / (exp(2x) + 1), with exp(2x) = 2^(K x), K = 2 log2 e, on the
// hardware exp2 and the hardware reciprocal. Saturates to +-1 without overflow trouble (2^inf =
// inf, 1/inf = 0). Absolute error about 1e-7. tanh_scaled takes y = K x, so that a bias staged as
// K b folds into one FMA: tanh(x + b) = tanh_scaled(K x + K b).
constexpr float TANH_K = 2.885390081777927f;
__device__ __forceinline__ float tanh_scaled(float y)
{
    return 1.0f - 2.0f * __builtin_amdgcn_rcpf(__builtin_amdgcn_exp2f(y) + 1.0f);
}
__device__ __forceinline__ float tanh_fast(float x) { return tanh_scaled(x * TANH_K); }

// Cross-lane sums over the four 16-lane groups of a wave on v_permlane32_swap (exchanges the
// upper half of one register with the lower half of another: pairs groups g, g + 2) and
// v_permlane16_swap (odd rows of one with even rows of the other: pairs g, g + 1).
__device__ __forceinline__ void swap_halves(float& a, float& b, bool rows16)
{
    const auto r = rows16 ? __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false)
                          : __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
}
__device__ __forceinline__ void swap_halves(double& a, double& b, bool rows16)
{
    const unsigned long long ua = __double_as_longlong(a), ub = __double_as_longlong(b);
    unsigned alo = (unsigned)ua, ahi = (unsigned)(ua >> 32), blo = (unsigned)ub, bhi = (unsigned)(ub >> 32);
    const auto rl = rows16 ? __builtin_amdgcn_permlane16_swap(alo, blo, false, false)
                           : __builtin_amdgcn_permlane32_swap(alo, blo, false, false);
    const auto rh = rows16 ? __builtin_amdgcn_permlane16_swap(ahi, bhi, false, false)
                           : __builtin_amdgcn_permlane32_swap(ahi, bhi, false, false);
    a = __longlong_as_double((long long)(((unsigned long long)rh[0] << 32) | rl[0]));
    b = __longlong_as_double((long long)(((unsigned long long)rh[1] << 32) | rl[1]));
}
// Every lane receives the sum of v over the four lanes of its column (lane & 15).
template <class T> __device__ __forceinline__ T sum_groups(T v)
{
    T a = v, b = v;
    swap_halves(a, b, false);
    v = a + b;
    a = v;
    b = v;
    swap_halves(a, b, true);
    return a + b;
}
// Lane group G receives the column sum of p[ksel(G)], ksel = {0, 2, 1, 3}.
__device__ __forceinline__ int ksel(int g) { return ((g & 1) << 1) | (g >> 1); }
template <class T> __device__ __forceinline__ T sum_groups4(const T* p)
{
    T a = p[0], b = p[1], c = p[2], d = p[3];
    swap_halves(a, b, false);
    swap_halves(c, d, false);
    T q0 = a + b, q1 = c + d;
    swap_halves(q0, q1, true);
    return q0 + q1;
}

}  // namespace dpk
