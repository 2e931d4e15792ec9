// Laguerre series helpers (§4.1 eqs. (34)-(35)): coefficients of the source
// pulse, right-hand sides of the harmonics (alpha = 0 and general integer
// alpha), receiver samples and the synthesis of time traces.
#include <cmath>
#include <mutex>

#include "kernels.h"

namespace axipcg {
namespace {

// Normalised generalized Laguerre functions by their recurrence:
// ell_m(x) = sqrt(eta) rt_m e^{-x/2} L^alpha_m(x), rt_m = sqrt(m!/(m+alpha)!),
// stepped as ell_{m+1} = (k_m - x) b_m ell_m - c_m ell_{m-1} with
// k_m = 2m + 1 + alpha, b_m = s1 / (m+1), c_m = (m + alpha) s2 / (m+1),
// s1 = rt_{m+1}/rt_m, s2 = rt_{m+1}/rt_{m-1} (no factorial is formed).  With
// alpha = 0 the same step takes the plain L_m.  The coefficients depend on m
// alone, so a workgroup is two waves: the second computes the coefficients
// of the next LC harmonics, one per lane, while every lane of the first steps
// its own x through the current ones.  A step is then three multiplies and one
// dependent multiply-add instead of two square roots and three divisions.
constexpr int LC = 64;   // harmonics per round

struct LagCoefs {
    double2 kb[LC];
    double c[LC];
    __device__ void fill(int m0, int lane, int alpha)
    {
        const int m = m0 + lane;
        const double m1 = m + 1.0;
        const double s1 = sqrt(m1 / (m1 + alpha));
        const double s2 = (m > 0) ? s1 * sqrt(m / (m + (double)alpha)) : 0.0;
        kb[lane] = make_double2(2.0 * m + 1.0 + alpha, s1 / m1);
        c[lane] = (m + alpha) * s2 / m1;
    }
    __device__ double next(int t, double x, double prev, double cur) const
    {
        return fma((kb[t].x - x) * kb[t].y, cur, -(c[t] * prev));
    }
};

// Harmonics stepped in round c of n: LC, in the last round what is left, up to
// the next multiple of 16 (the unrolled steps).  (All LC of them: 674 us instead
// of 269 for the synthesis of 4096 traces of 20001 samples from one harmonic.)
__device__ inline int lag_steps(int n, int c)
{
    const int left = n - c * LC;
    return left < LC ? (left + 15) & ~15 : LC;
}

__device__ inline double lag_start(double x, double eta, int alpha)
{
    double r0 = 1.0;   // rt_0 = 1/sqrt(alpha!)
    for (int k = 2; k <= alpha; ++k) r0 /= sqrt((double)k);
    return sqrt(eta) * r0 * exp(-0.5 * x);
}

// f_m = int f(t) psi_m(t) dt for every m < n by the trapezoid rule on the
// uniform samples, psi_m(t) = ell_m(eta t) (the projection kernel of
// eq. (34)); `plain` (alpha = 0): psi_m = sqrt(eta) e^{-eta t/2} L_m(eta t)
// with the recurrence on L_m itself.
// A workgroup steps 64 samples through all harmonics: n nt steps in all (a
// workgroup per harmonic, each stepping every sample from 0 to its m, is
// n^2 nt / 2).  Bound by the serial chain of the recurrence, so a stepping
// wave per 64 samples is all the parallelism there is.  Its products of LC
// harmonics go through LDS (pitch 65: rows and columns free of bank
// conflicts), and the second wave sums the previous round's, lane t those of
// harmonic t over the 64 samples: one write, one read and one add per step
// instead of a shuffle reduction per harmonic.  One partial sum per workgroup
// and harmonic; those with more than one group of samples add to their own.
// n = 2000, nt = 4001, alpha = 5: 64 us with the sum, where a workgroup per
// harmonic took 25.5 ms (and one wave doing both parts of the work 83 us).
__global__ void __launch_bounds__(128)
k_laguerre_coeffs(const double *__restrict__ f, int nt, double dt, double eta, int alpha, bool plain, int n,
                  double *__restrict__ part)
{
    __shared__ LagCoefs lc[2];
    __shared__ double prod[2][LC][65];
    const int lane = threadIdx.x & 63;
    const bool steps = threadIdx.x < 64;
    double *out = part + (size_t)blockIdx.x * n;
    const int groups = (nt + 63) / 64, rounds = (n + LC - 1) / LC;
    for (int gr = blockIdx.x; gr < groups; gr += gridDim.x) {
        const int j = gr * 64 + lane;
        const bool in = j < nt;
        const double x = in ? eta * (j * dt) : 0.0;
        double w = in ? ((j == 0 || j == nt - 1) ? 0.5 * dt : dt) * f[j] : 0.0;
        double prev = 0.0, cur = 1.0;
        if (plain) w = w * sqrt(eta) * exp(-0.5 * x);
        else cur = lag_start(x, eta, alpha);
        if (!steps) lc[0].fill(0, lane, alpha);
        // round c: harmonics [LC c, LC c + LC) are stepped while round c - 1 is summed
        for (int c = 0; c <= rounds; ++c) {
            __syncthreads();
            if (steps) {
                if (c == rounds) continue;
                const LagCoefs &l = lc[c & 1];
                for (int t0 = 0, nt_c = lag_steps(n, c); t0 < nt_c; t0 += 16)
#pragma unroll
                    for (int t = t0; t < t0 + 16; ++t) {
                        prod[c & 1][t][lane] = w * cur;
                        const double nx = l.next(t, x, prev, cur);
                        prev = cur;
                        cur = nx;
                    }
            } else {
                if (c + 1 < rounds) lc[(c + 1) & 1].fill((c + 1) * LC, lane, alpha);
                const int m = (c - 1) * LC + lane;
                if (c == 0 || m >= n) continue;   // rows past n are not written
                double s[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
                for (int i = 0; i < 64; i += 4)
#pragma unroll
                    for (int u = 0; u < 4; ++u) s[u] += prod[(c - 1) & 1][lane][i + u];
                const double t = (s[0] + s[1]) + (s[2] + s[3]);
                out[m] = (gr == (int)blockIdx.x) ? t : out[m] + t;
            }
        }
        __syncthreads();
    }
}

// g[m] = the sum of the workgroups' partials, in order.
__global__ void __launch_bounds__(64) k_laguerre_sum(const double *__restrict__ part, int np, int n, double *__restrict__ g)
{
    const int m = blockIdx.x * blockDim.x + threadIdx.x;
    if (m >= n) return;
    double s = 0.0;
#pragma unroll 8
    for (int p = 0; p < np; ++p) s += part[(size_t)p * n + m];
    g[m] = s;
}

// S1 += du u_prev; S2 += S1; b = r (g delta - c cs S2), c = coef or 4 q.
// (alpha = 0: du = cs = 1, and the products are exact.)
__global__ void __launch_bounds__(256)
k_laguerre_rhs(const double *__restrict__ u_prev, double *__restrict__ S1, double *__restrict__ S2,
               double *__restrict__ b, const double *__restrict__ coef, const double *__restrict__ W,
               const double *__restrict__ rw, int nr, int nz, int si, int sk, double src, double du, double cs)
{
    const size_t n = (size_t)nr * nz;
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (size_t)gridDim.x * blockDim.x) {
        double s1 = S1[e];
        if (u_prev) {
            s1 += du * u_prev[e];
            S1[e] = s1;
        }
        const double s2 = S2[e] + s1;
        S2[e] = s2;
        const int i = (int)(e / nz);
        const double cr = coef ? coef[e] * rw[i] : 4.0 * W[e];
        double v = -cr * (cs * s2);
        if (e == (size_t)si * nz + sk) v += src;
        b[e] = v;
    }
}

// out[j] = u[idx[j]] for the receivers (NaN for an index outside the grid)
__global__ void __launch_bounds__(64)
k_gather(const double *__restrict__ u, const long long *__restrict__ idx, int n, long long total,
         double *__restrict__ out)
{
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= n) return;
    const long long q = idx[j];
    out[j] = (q >= 0 && q < total) ? u[q] : __builtin_nan("");
}

// traces[r][j] = sum_m Q[m][r] phi_m(t_j), phi_m(t) = (eta t)^alpha psi_m(t)
// (eq. (34)): a lane of the first wave steps the recurrence at its time sample
// and adds RB receivers' terms; the second wave puts the coefficients and the
// receivers' values of the next LC harmonics into LDS.  Bound by the
// recurrence's serial chain over m, so the receivers are split over workgroups
// (synth_rb) until each SIMD of the chip has a stepping wave.
// n = 2000, 16 receivers, nt = 1001, alpha = 5: 48 us (1642 us with 16
// receivers and the coefficients in every thread, 75 us in one wave).
template <int RB>
__global__ void __launch_bounds__(128)
k_laguerre_synth(const double *__restrict__ Q, int n, int nrec, int nt, double dt, double eta, int alpha,
                 double *__restrict__ traces)
{
    __shared__ LagCoefs lc[2];
    __shared__ double qs[2][LC][RB];
    const int lane = threadIdx.x & 63;
    const int j = blockIdx.x * 64 + lane, r0 = blockIdx.y * RB;
    const int rounds = (n + LC - 1) / LC;
    if (threadIdx.x >= 64) {
        // values past the last harmonic are zero: their (bounded) terms add nothing
        auto stage = [&](int c) {
            const int m = c * LC + lane;
            double v[RB];
#pragma unroll
            for (int q = 0; q < RB; ++q) v[q] = (m < n && r0 + q < nrec) ? Q[(size_t)m * nrec + r0 + q] : 0.0;
            lc[c & 1].fill(c * LC, lane, alpha);
#pragma unroll
            for (int q = 0; q < RB; ++q) qs[c & 1][lane][q] = v[q];
        };
        stage(0);
        for (int c = 0; c < rounds; ++c) {
            __syncthreads();
            if (c + 1 < rounds) stage(c + 1);
        }
        return;
    }
    const double x = eta * (j * dt);   // lanes past nt run along and store nothing
    double xa = 1.0;
    for (int k = 0; k < alpha; ++k) xa *= x;
    double prev = 0.0, cur = lag_start(x, eta, alpha), acc[RB];
#pragma unroll
    for (int q = 0; q < RB; ++q) acc[q] = 0.0;
    for (int c = 0; c < rounds; ++c) {
        __syncthreads();
        const LagCoefs &l = lc[c & 1];
        for (int t0 = 0, nt_c = lag_steps(n, c); t0 < nt_c; t0 += 16)
#pragma unroll
            for (int t = t0; t < t0 + 16; ++t) {
#pragma unroll
                for (int q = 0; q < RB; ++q) acc[q] += qs[c & 1][t][q] * cur;
                const double nx = l.next(t, x, prev, cur);
                prev = cur;
                cur = nx;
            }
    }
    if (j >= nt) return;
#pragma unroll
    for (int q = 0; q < RB; ++q)
        if (r0 + q < nrec) traces[(size_t)(r0 + q) * nt + j] = xa * acc[q];
}

// Receivers per stepping wave: the fewest (a power of two up to 8) whose waves
// still fit the chip's 1024 SIMDs at one wave each.  A step costs some 16 issue
// cycles for the recurrence and 4 per receiver, so fewer receivers per wave
// shorten it only while there are idle SIMDs.
int synth_rb(int nt, int nrec)
{
    int rb = 1;
    while (rb < 8 && (long)((nt + 63) / 64) * ((nrec + rb - 1) / rb) > 1024) rb *= 2;
    return rb;
}

// Workgroups (= partial sums) of the projection: one per 64 samples, fewer for
// so many harmonics that their partials would take more than LAG_PARTS doubles.
constexpr size_t LAG_PARTS = size_t(1) << 19;
int coeff_parts(int n, int nt)
{
    const size_t groups = ((size_t)nt + 63) / 64, cap = LAG_PARTS / (size_t)n;
    return (int)(groups < cap ? groups : cap);
}

// g_host = the projections of the samples, through device buffers d_f [nt],
// d_g [n] and d_p [coeff_parts(n, nt) n]; synchronises the stream.
void project(const double *f_host, double *g_host, int n, int nt, double t_max, double eta, int alpha, bool plain,
             double *d_f, double *d_g, double *d_p, hipStream_t s)
{
    const int np = coeff_parts(n, nt);
    AXI_CHECK_HIP(hipMemcpyAsync(d_f, f_host, sizeof(double) * nt, hipMemcpyHostToDevice, s));
    hipLaunchKernelGGL(k_laguerre_coeffs, dim3(np), dim3(128), 0, s, d_f, nt, t_max / (nt - 1), eta, alpha, plain, n,
                       d_p);
    AXI_CHECK_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_laguerre_sum, dim3((n + 63) / 64), dim3(64), 0, s, d_p, np, n, d_g);
    AXI_CHECK_HIP(hipGetLastError());
    AXI_CHECK_HIP(hipMemcpyAsync(g_host, d_g, sizeof(double) * n, hipMemcpyDeviceToHost, s));
    AXI_CHECK_HIP(hipStreamSynchronize(s));
}

// The same through one temporary device buffer.
void project_alloc(const double *f_host, double *g_host, int n, int nt, double t_max, double eta, int alpha,
                   bool plain, hipStream_t s)
{
    struct Tmp {
        double *p = nullptr;
        ~Tmp() { if (p) (void)hipFree(p); }
    } tmp;
    const size_t parts = (size_t)coeff_parts(n, nt) * n;
    AXI_CHECK_HIP(hipMalloc((void **)&tmp.p, sizeof(double) * ((size_t)nt + n + parts)));
    project(f_host, g_host, n, nt, t_max, eta, alpha, plain, tmp.p, tmp.p + nt, tmp.p + nt + n, s);
}

}  // namespace
}  // namespace axipcg

using namespace axipcg;

extern "C" int axipcg_laguerre_coeffs(int n, double eta, int nt, double t_max, const double *f_host,
                                      double *g_host, void *stream)
{
    return guarded([&] {
        AXI_REQUIRE(n >= 1 && n <= 100000, "n must be in [1, 100000]");
        AXI_REQUIRE(nt >= 3, "nt must be >= 3");
        AXI_REQUIRE(std::isfinite(eta) && eta > 0 && std::isfinite(t_max) && t_max > 0, "eta, t_max must be > 0");
        AXI_REQUIRE(f_host && g_host, "NULL argument");
        for (int j = 0; j < nt; ++j) AXI_REQUIRE(std::isfinite(f_host[j]), "f has non-finite values");
        project_alloc(f_host, g_host, n, nt, t_max, eta, 0, true, (hipStream_t)stream);
        return AXIPCG_OK;
    });
}

extern "C" int axipcg_laguerre_rhs(axipcg_op_t h, double g_m, int src_i, int src_k, const double *coef,
                                   const double *u_prev, double *S1, double *S2, double *b, void *stream)
{
    return guarded([&] {
        const Operator *op = reinterpret_cast<const Operator *>(h);
        AXI_REQUIRE(op && S1 && S2 && b, "NULL argument");
        AXI_REQUIRE(std::isfinite(g_m), "g_m must be finite");
        AXI_REQUIRE(src_i >= 0 && src_i < op->nr && src_k >= 0 && src_k < op->nz, "source cell out of range");
        AXI_REQUIRE(S1 != S2 && S1 != b && S2 != b, "S1, S2 and b must be distinct");
        AXI_REQUIRE(!u_prev || (u_prev != S1 && u_prev != S2 && u_prev != b), "u_prev aliases an output");
        const size_t n = (size_t)op->nr * op->nz;
        const double src = g_m / (op->hr * op->hz);
        hipLaunchKernelGGL(k_laguerre_rhs, dim3(pointwise_blocks(n)), dim3(256), 0, (hipStream_t)stream, u_prev, S1,
                           S2, b, coef, op->W, op->rw64, op->nr, op->nz, src_i, src_k, src, 1.0, 1.0);
        AXI_CHECK_HIP(hipGetLastError());
        return AXIPCG_OK;
    });
}

// sqrt((k + alpha)! / k!) in FP64 through lgamma (k, alpha >= 0)
static double lag_ratio(int k, int alpha)
{
    return std::exp(0.5 * (std::lgamma(k + alpha + 1.0) - std::lgamma(k + 1.0)));
}

extern "C" int axipcg_laguerre_coeffs_alpha(int n, int alpha, double eta, int nt, double t_max, const double *f_host,
                                            double *g_host, void *stream)
{
    return guarded([&] {
        AXI_REQUIRE(n >= 1 && n <= 100000, "n must be in [1, 100000]");
        AXI_REQUIRE(alpha >= 0 && alpha <= 64, "alpha must be in [0, 64]");
        AXI_REQUIRE(nt >= 3, "nt must be >= 3");
        AXI_REQUIRE(std::isfinite(eta) && eta > 0 && std::isfinite(t_max) && t_max > 0, "eta, t_max must be > 0");
        AXI_REQUIRE(f_host && g_host, "NULL argument");
        for (int j = 0; j < nt; ++j) AXI_REQUIRE(std::isfinite(f_host[j]), "f has non-finite values");
        project_alloc(f_host, g_host, n, nt, t_max, eta, alpha, false, (hipStream_t)stream);
        return AXIPCG_OK;
    });
}

// ---- allocation-free variant of axipcg_laguerre_coeffs_alpha ---------------
// The staged pulse samples, the coefficients and the waves' partial sums live
// in one file-scope device array instead of a hipMalloc'd buffer.  Each device holds its own copy;
// host code reaches it only through the address hipGetSymbolAddress returns
// for that device (the array's name in host code is a stand-in, not a device
// address).
namespace {

constexpr size_t NOALLOC_DOUBLES = size_t(1) << 17;   // nt + n <= 131072; 5 MiB per device with the partials
constexpr int NOALLOC_MAX_DEVICES = 64;

__device__ __align__(256) double scratch[NOALLOC_DOUBLES + LAG_PARTS];

std::mutex g_scratch_mu;
double *g_scratch_ptr[NOALLOC_MAX_DEVICES] = {};

// Address of `scratch` on the current device, looked up once per device.
double *scratch_on_current_device()
{
    int dev = -1;
    AXI_CHECK_HIP(hipGetDevice(&dev));
    AXI_REQUIRE(dev >= 0 && dev < NOALLOC_MAX_DEVICES, "device index beyond the scratch table");
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        AXI_CHECK_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
        AXI_REQUIRE(ptr != nullptr, "hipGetSymbolAddress returned NULL for the scratch array");
        g_scratch_ptr[dev] = static_cast<double *>(ptr);
    }
    return g_scratch_ptr[dev];
}

}  // namespace

extern "C" int axipcg_laguerre_coeffs_alpha_noalloc(int n, int alpha, double eta, int nt, double t_max,
                                                    const double *f_host, double *g_host, void *stream)
{
    return guarded([&] {
        AXI_REQUIRE(n >= 1 && n <= 100000, "n must be in [1, 100000]");
        AXI_REQUIRE(alpha >= 0 && alpha <= 64, "alpha must be in [0, 64]");
        AXI_REQUIRE(nt >= 3, "nt must be >= 3");
        AXI_REQUIRE((size_t)nt + (size_t)n <= NOALLOC_DOUBLES,
                    "nt + n exceeds the 131072 doubles of the allocation-free scratch");
        AXI_REQUIRE(std::isfinite(eta) && eta > 0 && std::isfinite(t_max) && t_max > 0, "eta, t_max must be > 0");
        AXI_REQUIRE(f_host && g_host, "NULL argument");
        for (int j = 0; j < nt; ++j) AXI_REQUIRE(std::isfinite(f_host[j]), "f has non-finite values");
        double *d_f = scratch_on_current_device();
        project(f_host, g_host, n, nt, t_max, eta, alpha, false, d_f, d_f + nt, d_f + NOALLOC_DOUBLES,
                (hipStream_t)stream);
        return AXIPCG_OK;
    });
}

extern "C" int axipcg_laguerre_rhs_alpha(axipcg_op_t h, int m, int alpha, double g_m, int src_i, int src_k,
                                         const double *coef, const double *u_prev, double *S1, double *S2, double *b,
                                         void *stream)
{
    return guarded([&] {
        const Operator *op = reinterpret_cast<const Operator *>(h);
        AXI_REQUIRE(op && S1 && S2 && b, "NULL argument");
        AXI_REQUIRE(m >= 0 && alpha >= 0 && alpha <= 64, "need m >= 0 and alpha in [0, 64]");
        AXI_REQUIRE((m == 0) == (u_prev == nullptr), "u_prev is NULL exactly when m = 0");
        AXI_REQUIRE(std::isfinite(g_m), "g_m must be finite");
        AXI_REQUIRE(src_i >= 0 && src_i < op->nr && src_k >= 0 && src_k < op->nz, "source cell out of range");
        AXI_REQUIRE(S1 != S2 && S1 != b && S2 != b, "S1, S2 and b must be distinct");
        AXI_REQUIRE(!u_prev || (u_prev != S1 && u_prev != S2 && u_prev != b), "u_prev aliases an output");
        const size_t n = (size_t)op->nr * op->nz;
        const double src = g_m / (op->hr * op->hz);
        const double du = (m > 0) ? lag_ratio(m - 1, alpha) : 0.0;   // d_{m-1}
        const double cs = 1.0 / lag_ratio(m, alpha);                  // c_m
        hipLaunchKernelGGL(k_laguerre_rhs, dim3(pointwise_blocks(n)), dim3(256), 0, (hipStream_t)stream, u_prev, S1,
                           S2, b, coef, op->W, op->rw64, op->nr, op->nz, src_i, src_k, src, du, cs);
        AXI_CHECK_HIP(hipGetLastError());
        return AXIPCG_OK;
    });
}

extern "C" int axipcg_gather(axipcg_op_t h, const double *u, const long long *idx, int n, double *out, void *stream)
{
    return guarded([&] {
        const Operator *op = reinterpret_cast<const Operator *>(h);
        AXI_REQUIRE(op && u && idx && out, "NULL argument");
        AXI_REQUIRE(n >= 1 && n <= 65536, "n must be in [1, 65536]");
        hipLaunchKernelGGL(k_gather, dim3((n + 63) / 64), dim3(64), 0, (hipStream_t)stream, u, idx, n,
                           (long long)op->nr * op->nz, out);
        AXI_CHECK_HIP(hipGetLastError());
        return AXIPCG_OK;
    });
}

extern "C" int axipcg_laguerre_synth(int n, int alpha, double eta, int nrec, const double *Q, int nt, double t_max,
                                     double *traces, void *stream)
{
    return guarded([&] {
        AXI_REQUIRE(n >= 1 && n <= 100000 && nrec >= 1 && nrec <= 4096, "need 1 <= n <= 100000, 1 <= nrec <= 4096");
        AXI_REQUIRE(alpha >= 0 && alpha <= 64, "alpha must be in [0, 64]");
        AXI_REQUIRE(nt >= 2 && std::isfinite(eta) && eta > 0 && std::isfinite(t_max) && t_max > 0,
                    "need nt >= 2 and eta, t_max > 0");
        AXI_REQUIRE(Q && traces, "NULL argument");
        const int rb = synth_rb(nt, nrec);
        const dim3 grid((nt + 63) / 64, (nrec + rb - 1) / rb);
#define AXI_SYNTH(RBV)                                                                                          \
    hipLaunchKernelGGL(k_laguerre_synth<RBV>, grid, dim3(128), 0, (hipStream_t)stream, Q, n, nrec, nt,           \
                       t_max / (nt - 1), eta, alpha, traces)
        if (rb == 1) AXI_SYNTH(1);
        else if (rb == 2) AXI_SYNTH(2);
        else if (rb == 4) AXI_SYNTH(4);
        else AXI_SYNTH(8);
#undef AXI_SYNTH
        AXI_CHECK_HIP(hipGetLastError());
        return AXIPCG_OK;
    });
}
