// sample.hip -- Gaussian initial phase-space points (Eq. (7) of
// arXiv:2212.04352, amplitude from the covariance of Appendix A.3; for a
// thermal initial state also the diagonal fluctuation of that covariance).
//
// One thread per (spin, packed element, trajectory); the trajectory index is
// the fastest grid dimension so that every wave stores 64 consecutive
// trajectories of one element (the packed layout keeps them contiguous).
#include "device_common.h"
#include "ftwa_internal.h"
#include "philox.h"

namespace ftwa {

namespace {

// The kernel is bound by the FP64 and integer arithmetic of a draw, not by the
// stores (the 198-site FP32 states of 8192 trajectories are 2.6 GB, 0.4 ms at
// the fill rate of 6.9 TB/s), so the logarithm, square root, sine and cosine
// are written for the ranges they meet here: no special values, no large
// argument reduction.  A draw of those states takes 1.9 ms (3.2 ms with the
// general device functions), about 230 instruction slots per element, a third
// of them Philox's 64-bit products; the error of an element against 80-bit
// values is 1.1e-16 of its norm (2.5e-16 before: the angle is reduced
// exactly, not from a rounded 2 pi u).

// a * b + c with the constant c in scalar registers (as a compiled fma chain,
// every coefficient is first copied into a vector register pair: a sixth of
// the kernel's instructions).
__device__ __forceinline__ double fma_k(double a, double b, double c) {
    double r;
    __asm__("v_fma_f64 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "s"(c));
    return r;
}

// sqrt(w) for w = 0 or 1e-17 < w < 1e3 (no scaling needed): reciprocal square
// root estimate, one Goldschmidt step, two residual corrections.
__device__ __forceinline__ double sqrt_pos(double w) {
    const double r = __builtin_amdgcn_rsq(w);
    double g = w * r, h = 0.5 * r;
    const double e = __builtin_fma(-h, g, 0.5);
    g = __builtin_fma(g, e, g);
    h = __builtin_fma(h, e, h);
    g = __builtin_fma(__builtin_fma(-g, g, w), h, g);
    g = __builtin_fma(__builtin_fma(-g, g, w), h, g);
    return w == 0.0 ? 0.0 : g;
}

// -ln(k 2^-53) for an integer 1 <= k <= 2^53.  k = 2^e m with m in
// [sqrt(1/2), sqrt(2)); with x = m - 1 (exact), f = x / (2 + x), s = f^2,
//   ln m = 2 atanh f = x - f (x - s L(s)),  L(s) = sum_j 2 s^j / (2j + 3),
// and (53 - e) ln 2 - ln m is one fused sum, accurate also next to k = 2^53
// where it tends to zero.  L: interpolated at the Chebyshev nodes of
// [0, 0.0295], s L(s) within 1e-17.
__device__ __forceinline__ double neg_log_u53(uint64_t k) {
    const double v = (double)k;
    int e = __builtin_amdgcn_frexp_exp(v);
    double m = __builtin_amdgcn_frexp_mant(v);
    const bool small = m < 0.70710678118654752;
    m = small ? 2.0 * m : m;
    e = small ? e - 1 : e;
    const double x = m - 1.0, d = 2.0 + x;
    double r = __builtin_amdgcn_rcp(d);
    r = __builtin_fma(r, __builtin_fma(-d, r, 1.0), r);
    r = __builtin_fma(r, __builtin_fma(-d, r, 1.0), r);
    double f = x * r;
    f = __builtin_fma(__builtin_fma(-d, f, x), r, f);
    const double s = f * f;
    double L = 0.14616449685043406;
    L = fma_k(L, s, 0.15331721600556042);
    L = fma_k(L, s, 0.18182889125261723);
    L = fma_k(L, s, 0.2222221113479508);
    L = fma_k(L, s, 0.28571428625975487);
    L = fma_k(L, s, 0.39999999999899505);
    L = fma_k(L, s, 0.666666666666667);
    const double lnm = __builtin_fma(-f, __builtin_fma(-s, L, x), x);
    const double n = (double)(53 - e);
    // ln 2 = 0.6931471805599453 + 2.3190468138462996e-17
    return __builtin_fma(n, 0.6931471805599453,
                         __builtin_fma(n, 2.3190468138462996e-17, -lnm));
}

// cos and sin of 2 pi u, u = k 2^-53 in [0, 1): 4u = q + r with q = 0..4 and
// |r| <= 1/2 exactly, then sin(pi/2 r) and cos(pi/2 r) as polynomials in r
// (Chebyshev nodes on r^2 <= 1/4, within 2e-17; the linear term pi/2 in two
// parts) and the quarter turn by q.
__device__ __forceinline__ void sincos_turn(uint64_t k, double* sn, double* cs) {
    const double t = (double)k * (4.0 / 9007199254740992.0);
    const double qd = __builtin_rint(t);
    const double r = t - qd;
    const int q = (int)qd;
    const double z = r * r;
    double S = 5.642225369163528e-08;
    S = fma_k(S, z, -3.5987029509735105e-06);
    S = fma_k(S, z, 0.00016044116661409423);
    S = fma_k(S, z, -0.004681754134254207);
    S = fma_k(S, z, 0.07969262624614423);
    S = fma_k(S, z, -0.6459640975062462);
    S = fma_k(S, z, 6.123233995736766e-17);
    const double s0 = __builtin_fma(r, 1.5707963267948966, r * S);
    double C = -6.329396344967424e-09;
    C = fma_k(C, z, 4.710678405505227e-07);
    C = fma_k(C, z, -2.5202039028029178e-05);
    C = fma_k(C, z, 0.0009192602745468447);
    C = fma_k(C, z, -0.020863480763340773);
    C = fma_k(C, z, 0.2536695079010478);
    C = fma_k(C, z, -1.2337005501361697);
    const double c0 = __builtin_fma(C, z, 1.0);
    const double a = (q & 1) ? c0 : s0, b = (q & 1) ? s0 : c0;
    *sn = (q & 2) ? -a : a;
    *cs = ((q + 1) & 2) ? -b : b;
}

template <typename T>
__global__ __launch_bounds__(256) void sample_kernel(int N, int64_t P, int64_t n_traj,
                                                     int64_t traj_offset, uint32_t instance,
                                                     uint64_t seed, const double* __restrict__ n0,
                                                     const double* __restrict__ shift,
                                                     const uint32_t* __restrict__ elem,
                                                     cplx_t<T>* __restrict__ rho, int thermal) {
    const int64_t m = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (m >= n_traj) return;
    const int64_t row = blockIdx.y;  // s * P + p
    const int s = row >= P ? 1 : 0;
    const int64_t p = row - (int64_t)s * P;
    const uint32_t ij = elem[p];
    const int i = (int)(ij & 0xffffu), j = (int)(ij >> 16);
    const double ni = n0[s * N + i], nj = n0[s * N + j];
    double re = 0.0, im = 0.0;
    if (i == j) {
        re = ni - 0.5;
        if (shift) re += shift[s * N + i];
        const double var = ni * (1.0 - ni);  // thermal state: Var rho_ii (Appendix A.3)
        if (thermal && var != 0.0) {
            const PhiloxBlock b = philox4x32_10(
                {(uint32_t)i, (instance << 1) | (uint32_t)s, (uint32_t)(traj_offset + m), 2u}, seed);
            double sn, cs;
            sincos_turn(b.bits53_second(), &sn, &cs);
            const double g = sqrt_pos(2.0 * neg_log_u53(b.bits53_first() + 1u)) * cs;
            re += sqrt(var) * g;
        }
    } else {
        const double var = 0.5 * ((ni + nj) - (2.0 * ni) * nj);
        if (var != 0.0) {
            const uint32_t pair = (uint32_t)(i * N - (i * (i + 1)) / 2 + (j - i - 1));
            const PhiloxBlock b = philox4x32_10(
                {pair, (instance << 1) | (uint32_t)s, (uint32_t)(traj_offset + m), 0u}, seed);
            const double radius = sqrt_pos(neg_log_u53(b.bits53_first() + 1u));
            double sn, cs;
            sincos_turn(b.bits53_second(), &sn, &cs);
            const double amp = sqrt(var);
            re = amp * (radius * cs);
            im = amp * (radius * sn);
        }
    }
    cplx_t<T> v;
    v.x = (T)re;
    v.y = (T)im;
    rho[row * n_traj + m] = v;
}

}  // namespace

ftwa_status launch_sample(const ftwa_instance& in, const DeviceTables& tab, uint64_t seed,
                          ftwa_dtype dtype, bool thermal, hipStream_t stream) {
    const int N = in.lat->N;
    const int64_t P = packed_count(N);
    if (in.n_traj == 0) return FTWA_OK;
    const dim3 block(256);
    const dim3 grid((unsigned)((in.n_traj + 255) / 256), (unsigned)(2 * P));
    if (dtype == FTWA_F64)
        hipLaunchKernelGGL(sample_kernel<double>, grid, block, 0, stream, N, P, in.n_traj,
                           in.traj_offset, in.instance, seed, in.n0, in.n_shift, tab.elem,
                           static_cast<double2*>(in.rho), thermal ? 1 : 0);
    else
        hipLaunchKernelGGL(sample_kernel<float>, grid, block, 0, stream, N, P, in.n_traj,
                           in.traj_offset, in.instance, seed, in.n0, in.n_shift, tab.elem,
                           static_cast<float2*>(in.rho), thermal ? 1 : 0);
    FTWA_LAUNCH_CHECK("sample_kernel");
    return FTWA_OK;
}

}  // namespace ftwa
