// Device helpers shared by the forward solver and the adjoint kernels, and
// the launch of their persistent kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <string.h>

namespace fmm {

#define FMM_INF __builtin_huge_val()

// ---------------------------------------------------------------------------
// Correctly rounded square root and division by 3 for the local solver, in
// fewer instructions than the general library sequences.
//
// solver_sqrt: the hardware reciprocal square root estimate y ~ 1/sqrt(x),
// one coupled Newton step on s ~ sqrt(x) and h ~ 1/(2 sqrt(x)) (Goldschmidt's
// iteration), then two residual corrections s += (x - s^2) h; the last one
// rounds correctly.  The general routine additionally rescales tiny inputs
// and patches 0 and +inf.  Here inputs below 2^-767 (0 included) take the
// library routine on a branch that the solver's discriminants practically
// never reach; +inf (only when r = +inf, where the solver returns +inf from
// its first root) gives NaN, which the root comparisons reject.
__device__ __forceinline__ double solver_sqrt_normal(double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    double s = x * y, h = y * 0.5;
    const double e = __builtin_fma(-h, s, 0.5);
    s = __builtin_fma(s, e, s);
    h = __builtin_fma(h, e, h);
    double d = __builtin_fma(-s, s, x);
    s = __builtin_fma(d, h, s);
    d = __builtin_fma(-s, s, x);
    return __builtin_fma(d, h, s);
}

__device__ __forceinline__ double solver_sqrt(double x)
{
    double s = solver_sqrt_normal(x);
    if (__builtin_expect(x < 0x1p-767, 0)) {
        asm volatile("");  // keeps the rare path a branch (not computed and selected)
        s = sqrt(x);
    }
    return s;
}

// x / 3, correctly rounded: q = x * RN(1/3) is within one ulp, and one
// remainder step q + (x - 3 q) RN(1/3) rounds correctly (Markstein's
// theorem; x / 3 is never a tie).
__device__ __forceinline__ double div3(double x)
{
    const double third = 1.0 / 3.0;
    const double q = x * third;
    return __builtin_fma(__builtin_fma(-q, 3.0, x), third, q);
}

// h / f for the march's r = h / F: a reciprocal estimate refined by two
// Newton steps, the quotient, and one remainder correction.  For operands of
// moderate exponents this is the correctly rounded quotient (the general
// routine additionally rescales extreme exponents and patches special
// values).  f must be positive and finite (the tile load keeps an infinite
// FP32 speed as the largest finite one).
__device__ __forceinline__ double solver_div(double h, double f)
{
    double y = __builtin_amdgcn_rcp(f);
    y = __builtin_fma(y, __builtin_fma(-f, y, 1.0), y);
    y = __builtin_fma(y, __builtin_fma(-f, y, 1.0), y);
    const double q = h * y;
    return __builtin_fma(__builtin_fma(-f, q, h), y, q);
}

// a / S, correctly rounded for ordinary operands: a refined reciprocal, the
// quotient and a remainder step (the library's sequence without its scaling).
__device__ __forceinline__ double quick_div(double a, double S)
{
    double y = __builtin_amdgcn_rcp(S);
    y = __builtin_fma(y, __builtin_fma(-S, y, 1.0), y);
    y = __builtin_fma(y, __builtin_fma(-S, y, 1.0), y);
    const double q = a * y;
    return __builtin_fma(__builtin_fma(-q, S, a), y, q);
}

// The same for all operands.  Where a step overflows or a value is infinite the quotient comes out infinite
// or NaN, and where it underflows subnormal; below 2^-960 the remainder itself
// may underflow.  There the division itself is taken, unless the caller has no
// use for the result (ok false).
__device__ __forceinline__ double fast_div(double a, double S, bool ok = true)
{
    double q = quick_div(a, S);
    // signalling and quiet NaN, both infinities, both subnormals
    const bool odd = __builtin_amdgcn_class(q, 0x1 | 0x2 | 0x4 | 0x10 | 0x80 | 0x200);
    if (__builtin_expect((int)ok & ((int)odd | ((int)(fabs(a) < 0x1p-960) & (int)(a != 0.0))), 0)) {
        asm volatile("");
        q = a / S;
    }
    return q;
}

// ---------------------------------------------------------------------------
// Local solver (Alg. 11 with Eqs. 4-7).  a = per-axis upwind values (+inf when
// an axis has no upwind neighbour), r = h / F.  With a1 <= a2 <= a3:
//   u1 = a1 + r
//   u2 = ((a1 + a2) + sqrt(2 r^2 - (a2 - a1)^2)) * 0.5          causal iff u2 > a2
//   u3 = (((a1 + a2) + a3) + sqrt(3 r^2 - (((a2-a1)^2 + (a3-a1)^2) + (a3-a2)^2))) / 3
//                                                                causal iff u3 > a3
// and G is the smallest causal root (discriminants must be >= 0).  This is the
// paper's quadratic with the identity (sum a)^2 - k sum a^2 = -sum_{i<j}(a_i-a_j)^2
// applied, so nothing of size T^2/h^2 cancels.  *k receives how many of the
// sorted values the returned root uses (0 when there is no upwind value).
__device__ __forceinline__ double godunov_sel(double x, double y, double z, double r, int *k)
{
    double lo = fmin(x, y), hi = fmax(x, y);
    double a3 = fmax(hi, z), m = fmin(hi, z);
    double a1 = fmin(lo, m), a2 = fmax(lo, m);
    // no upwind value: a1 = +inf makes the first root +inf (r >= 0), with
    // no branch ahead of the one on a2
    *k = a1 < FMM_INF ? 1 : 0;
    double r2 = r * r;
    double best = a1 + r;
    if (a2 < FMM_INF) {
        double d12 = a2 - a1;
        double D2 = 2.0 * r2 - d12 * d12;
        if (D2 >= 0.0) {
            double u2 = ((a1 + a2) + solver_sqrt(D2)) * 0.5;
            if (u2 > a2 && u2 < best) {
                best = u2;
                *k = 2;
            }
        }
        if (a3 < FMM_INF) {
            double d13 = a3 - a1, d23 = a3 - a2;
            double D3 = 3.0 * r2 - ((d12 * d12 + d13 * d13) + d23 * d23);
            if (D3 >= 0.0) {
                double u3 = div3(((a1 + a2) + a3) + solver_sqrt(D3));
                if (u3 > a3 && u3 < best) {
                    best = u3;
                    *k = 3;
                }
            }
        }
    }
    return best;
}

// The same root for r >= 0 with one square root.  In exact arithmetic the candidate of k
// values is causal iff the sum of (a_k - a_i)^2 over them is below r^2, and
// more values give a smaller root, so the sums decide which root to form.
// Rounding can decide otherwise only where a sum is close to r^2: the two roots
// then differ by about (u - a)^2 / (4 r), which exceeds a few ulps of the values
// once |r^2 - sum| > r^2 2^-22 sqrt(a1 / r), and t bounds twice that without a
// root.  Closer calls, and r^2 near the ends of the exponent range (r = +inf
// too), take godunov_sel(): bitwise the same result everywhere (the tests compare
// random triples, both decisions, ties and the ends of the range).  NaN sums,
// from absent values, compare false and leave the first root.
__device__ __forceinline__ double godunov(double x, double y, double z, double r)
{
    const double lo = fmin(x, y), hi = fmax(x, y);
    const double a3 = fmax(hi, z), m = fmin(hi, z);
    const double a1 = fmin(lo, m), a2 = fmax(lo, m);
    const double r2 = r * r;
    const double d12 = a2 - a1, d13 = a3 - a1, d23 = a3 - a2;
    const double q12 = d12 * d12, q13 = d13 * d13, q23 = d23 * d23;
    const double f3 = q13 + q23;
    const double t = __builtin_fma(r2, 0x1p-16, (r * fabs(a1)) * 0x1p-28);
    const uint32_t e = (uint32_t)((unsigned long long)__double_as_longlong(r2) >> 52);  // r2 >= 0
    const bool three = f3 < r2, two = q12 < r2;
    // selects and a single test (the lanes differ: no branch is saved)
    const double D2 = 2.0 * r2 - q12, D3 = 3.0 * r2 - ((q12 + q13) + q23);
    const double D = __builtin_unpredictable(three) ? D3 : D2;
    const double s12 = a1 + a2, s123 = s12 + a3;
    const double v = (__builtin_unpredictable(three) ? s123 : s12) + solver_sqrt_normal(D);
    const double v3 = div3(v), v2 = v * 0.5;
    const double root = __builtin_unpredictable(three) ? v3 : v2, u1 = a1 + r;
    double best = __builtin_unpredictable(two) ? root : u1;
    const int close = (int)(fabs(r2 - q12) <= t) | (int)(fabs(r2 - f3) <= t) | (int)(e - (1023u - 760u) > 760u + 990u);
    if (__builtin_expect(close, 0)) {
        asm volatile("");  // a branch, not computed and selected
        int k;
        best = godunov_sel(x, y, z, r, &k);
    }
    return best;
}

// The local solver with per-axis spacing h s_i (weights w_i = 1 / s_i^2):
// sum_i w_i max(u - a_i, 0)^2 = r^2, r = h / F.  For the k smallest values,
// sorted together with their scales (ties keep axis order),
//   u1 = a1 + r s1
//   u2 = ((w1 a1 + w2 a2) + sqrt((w1+w2) r^2 - (w1 w2)(a2-a1)^2)) / (w1+w2)
//   u3 = (((w1 a1 + w2 a2) + w3 a3) + sqrt(((w1+w2)+w3) r^2
//          - (((w1 w2)(a2-a1)^2 + (w1 w3)(a3-a1)^2) + (w2 w3)(a3-a2)^2))) / ((w1+w2)+w3)
// with the same causality rule and minimum.  With unit scales every
// operation is the one of godunov_sel().  Both roots are formed without a
// branch, with the short root and quotient and the weights of the axes instead
// of those of the sorted scales: the same operations, so the same bits (the tests
// compare ties, both decisions and wide ranges of values, r and scales).  A march is
// bound by its instructions, and this took five divisions and two roots of the
// library: 101x87x118, 3 spacings, 6.49 -> 5.81 ms.
__device__ __forceinline__ double godunov_w_sel(double x, double y, double z, double sx, double sy, double sz,
                                                double r, int *k)
{
    // the weights of the axes are the same for all points and leave the loop
    double a1 = x, a2 = y, a3 = z, s1 = sx, s2 = sy, s3 = sz;
    double w1 = 1.0 / (sx * sx), w2 = 1.0 / (sy * sy), w3 = 1.0 / (sz * sz);
    auto order = [](double &a, double &b, double &s, double &t, double &w, double &v) {
        const bool c = __builtin_unpredictable(a > b);
        const double a0 = a, s0 = s, w0 = w;
        a = c ? b : a;
        b = c ? a0 : b;
        s = c ? t : s;
        t = c ? s0 : t;
        w = c ? v : w;
        v = c ? w0 : v;
    };
    order(a1, a2, s1, s2, w1, w2);
    order(a2, a3, s2, s3, w2, w3);
    order(a1, a2, s1, s2, w1, w2);
    // (sum + sqrt(D)) / W for a finite D >= 0, NaN (which no comparison below
    // takes) for another D: the library's results bit for bit
    auto root = [](double sum, double D, double W) {
        const bool ok = __builtin_amdgcn_class(D, 0x20 | 0x40 | 0x80 | 0x100);  // +-0, positive and finite
        double q = solver_sqrt_normal(D);
        if (__builtin_expect((int)ok & (int)(D < 0x1p-767), 0)) {
            asm volatile("");
            q = sqrt(D);
        }
        return fast_div(sum + q, W, ok);
    };
    const double r2 = r * r;
    double best = a1 + r * s1;
    int n = 1;
    const double d12 = a2 - a1, d13 = a3 - a1, d23 = a3 - a2;
    const double q12 = (w1 * w2) * (d12 * d12), W2 = w1 + w2, W3 = W2 + w3, m2 = w1 * a1 + w2 * a2;
    // an absent value (+inf) makes its D -inf or NaN
    const double u2 = root(m2, W2 * r2 - q12, W2);
    if (u2 > a2 && u2 < best) {
        best = u2;
        n = 2;
    }
    const double u3 = root(m2 + w3 * a3, W3 * r2 - ((q12 + (w1 * w3) * (d13 * d13)) + (w2 * w3) * (d23 * d23)), W3);
    if (u3 > a3 && u3 < best) {
        best = u3;
        n = 3;
    }
    const bool any = a1 < FMM_INF;
    *k = any ? n : 0;
    return any ? best : FMM_INF;
}

// Per-axis grid spacing factors of a solve (spacing h * s[a] along axis a).
struct Spacing {
    double s[3];
    int aniso;  // 0: all factors are 1 (the isotropic solver is used)
};

__device__ __forceinline__ double local_solve(const Spacing &sp, double x, double y, double z, double r, int *k)
{
    if (sp.aniso) {
        // opaque here, so that the weights are not formed ahead of the branch
        double s0 = sp.s[0], s1 = sp.s[1], s2 = sp.s[2];
        asm volatile("" : "+v"(s0), "+v"(s1), "+v"(s2));
        return godunov_w_sel(x, y, z, s0, s1, s2, r, k);
    }
    return godunov_sel(x, y, z, r, k);
}

// ---------------------------------------------------------------------------
// Small helpers.

__device__ __forceinline__ unsigned long long bits_of(double x) { return (unsigned long long)__double_as_longlong(x); }
__device__ __forceinline__ double bitsd(unsigned long long b) { return __longlong_as_double((long long)b); }

__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <typename T> __device__ __forceinline__ T bcast0(T v) { return __shfl(v, 0); }

// One step of a wavefront reduction: the minimum with the value of another lane
// (DPP control CTRL, rows ROWS; lanes without a source keep their own).
template <int CTRL, int ROWS> __device__ __forceinline__ double dpp_min(double v)
{
    const unsigned long long b = bits_of(v);
    const int lo = (int)(uint32_t)b, hi = (int)(uint32_t)(b >> 32);
    const uint32_t lo2 = (uint32_t)__builtin_amdgcn_update_dpp(lo, lo, CTRL, ROWS, 0xf, false);
    const uint32_t hi2 = (uint32_t)__builtin_amdgcn_update_dpp(hi, hi, CTRL, ROWS, 0xf, false);
    return fmin(v, bitsd((unsigned long long)lo2 | ((unsigned long long)hi2 << 32)));
}

// Minimum over the wavefront (uniform result; all lanes active): shifts within
// rows of 16 lanes, then row broadcasts; lane 63 ends with the minimum.  Six
// exchanges through LDS took six round trips in a row (64^3 shells 6.17 and
// 6.08 ms, 1024^3 at 3.5h 184.5 and 183.0).
__device__ __forceinline__ double wave_min(double v)
{
    v = dpp_min<0x111, 0xf>(v);  // row_shr:1
    v = dpp_min<0x112, 0xf>(v);
    v = dpp_min<0x114, 0xf>(v);
    v = dpp_min<0x118, 0xf>(v);
    v = dpp_min<0x142, 0xa>(v);  // row_bcast:15
    v = dpp_min<0x143, 0xc>(v);  // row_bcast:31
    const unsigned long long b = bits_of(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, 63);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), 63);
    return bitsd((unsigned long long)lo | ((unsigned long long)hi << 32));
}

__device__ __forceinline__ unsigned long long wave_sum(unsigned long long v)
{
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

__device__ __forceinline__ uint32_t ld_acq(uint32_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long ld_acq64(unsigned long long *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Device-wide barrier of a persistent launch whose workgroups are all
// resident: a monotonic arrival counter (`bar`), agent-scope release and
// acquire fences, and a bounded wait.  A timeout (20 s) or an abort raised
// elsewhere sets `abort` (and `timeout_bit` in *err), so every workgroup
// leaves and the kernel always terminates.  Returns false on abort.
// The workgroup barrier first orders every wavefront's writes before thread
// 0's agent-scope release, which publishes them (release is cumulative), and
// thread 0's acquire, which invalidates the CU's and the XCD's caches, comes
// before the barrier that lets the other wavefronts read: one cache
// write-back and one invalidation per workgroup instead of one per wavefront.
__device__ __forceinline__ bool grid_sync(uint32_t *bar, uint32_t *abort, uint32_t *err, uint32_t timeout_bit,
                                          uint32_t &gen, uint32_t nwg, uint32_t *s_ok)
{
    __syncthreads();
    if (threadIdx.x == 0) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        gen++;
        uint32_t target = gen * nwg;
        uint32_t ok = 1;
        __hip_atomic_fetch_add(bar, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        unsigned long long t0 = wall_clock64();
        while (ld_acq(bar) < target) {
            if (ld_acq(abort)) {
                ok = 0;
                break;
            }
            __builtin_amdgcn_s_sleep(2);
            if (wall_clock64() - t0 > 2000000000ull) {  // 20 s at the 100 MHz constant clock
                atomicOr(err, timeout_bit);
                atomicExch(abort, 1u);
                ok = 0;
                break;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        *s_ok = ok;
    }
    __syncthreads();
    return *s_ok != 0;
}

// ---------------------------------------------------------------------------
// Host side, shared by the forward driver and the adjoint sweep.

// Launch a persistent kernel whose workgroups must all be resident at once
// (its device-wide barriers wait for every workgroup): a cooperative launch.
// Stream capture records the launch as an ordinary kernel node, so the
// cooperative attribute is set on the node the launch just added (the
// stream's only capture dependency), and a replay of the graph keeps the
// guarantee.
inline hipError_t launch_coresident(const void *kern, dim3 grid, dim3 block, void **args, hipStream_t s)
{
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    hipError_t e = hipStreamIsCapturing(s, &cs);
    if (e != hipSuccess) return e;
    if ((e = hipLaunchCooperativeKernel(kern, grid, block, args, 0, s)) != hipSuccess) return e;
    if (cs != hipStreamCaptureStatusActive) return hipSuccess;
    const hipGraphNode_t *deps = nullptr;
    size_t nd = 0;
    hipGraph_t g = nullptr;
    unsigned long long id = 0;
    if ((e = hipStreamGetCaptureInfo_v2(s, &cs, &id, &g, &deps, &nd)) != hipSuccess) return e;
    if (nd != 1 || !deps) return hipErrorStreamCaptureUnsupported;
    hipGraphNodeType ty = hipGraphNodeTypeEmpty;
    if ((e = hipGraphNodeGetType(deps[0], &ty)) != hipSuccess) return e;
    if (ty != hipGraphNodeTypeKernel) return hipErrorStreamCaptureUnsupported;
    hipLaunchAttributeValue v;
    memset(&v, 0, sizeof v);
    v.cooperative = 1;
    return hipGraphKernelNodeSetAttribute(deps[0], hipLaunchAttributeCooperative, &v);
}

}  // namespace fmm
