// Strip-partitioned preconditioner z = B^{-1} r (§4.2 eqs. (36)-(39)) with
// the partition idea of §3: the grid is cut into strips of R consecutive
// r-rows, one workgroup each, the interior of every strip is eliminated in
// terms of the strips' boundary rows (the "preparatory" solutions of
// eqs. (18)-(22)), and only one reduced equation per strip and z-mode crosses
// workgroups.  Three launches:
//
//  K1 (forward + local elimination): each wave z-transforms one row of the
//     strip into the workgroup's LDS tile; then, per mode, the strip's
//     interior rows are swept forward (Thomas) and the forward-eliminated
//     data f' is written back row by row, together with two values per
//     (strip, mode) that the reduced equations need (E1, G0 below).
//  K2 (reduced systems): per mode, the tridiagonal system in the strips'
//     last rows X_s (G = nr / R unknowns), solved by one wavefront (segments
//     per lane, parallel cyclic reduction across lanes).  In PCG mode it
//     first runs the stop test.
//  K3 (back substitution + inverse): each strip rebuilds its interior rows
//     from f', X_{s-1} and X_s in the LDS tile, and each wave inverse-
//     transforms one row to z.
//
// Every global access is along z (whole rows), so no kernel gathers or
// scatters the strided [nr][modes] tiles a per-mode r-solve needs; the
// spectral data crosses HBM once each way as f' (4 + 4 bytes per point in
// FP32), and the reduced data is 3 values per strip and mode.
//
// Notation for strip s (rows i0 = s R + t, t < R; n = R - 1 interior rows,
// interface row j = i0 + n), mode l with lam = kbar mu_l + qbar:
//   row equation  -cb[i-1] y[i-1] + (db[i] + rw[i] lam) y[i] - cb[i] y[i+1] = f[i];
//   interior sweep  den_t = D_t - L_t c'_{t-1},  c'_t = cb[i0+t] / den_t,
//                   f'_t = (f_t + L_t f'_{t-1}) / den_t,
//                   v'_t = (t = 0 ? cb[i0-1] : L_t v'_{t-1}) / den_t,
//     with L_t = cb[i0+t-1] (t >= 1), so that
//                   y_t = f'_t + v'_t X_{s-1} + c'_t y_{t+1},  y_n = X_s;
//   back to the first interior row: y_0 = G0 + v_0 X_{s-1} + w_0 X_s and
//   y_{n-1} = f'_{n-1} + v'_{n-1} X_{s-1} + c'_{n-1} X_s;
//   reduced equation of strip s (the interface row with both neighbours
//   eliminated):
//     a_s = -cb[j-1] v'_{n-1},  b_s = D_j - cb[j-1] c'_{n-1} - cb[j] v_0(s+1),
//     c_s = -cb[j] w_0(s+1),    e_s = E1_s + cb[j] G0_{s+1},
//     E1_s = f_j + cb[j-1] f'_{n-1}.
// When R does not divide nr the last strip's missing rows are uncoupled lines
// with a zero right-hand side (the r-line arrays are padded so), which changes
// no other row.
// The coefficient-only quantities (c', v', v_0, w_0) are recomputed where
// needed from the O(nr) r-line arrays instead of being stored.
#include "strip.h"

namespace axipcg {
namespace {

template <typename T, int BC, bool FUSED, int R2, int R>
__global__ void __launch_bounds__(64 * R)
k_strip_fwd(const double *__restrict__ rin, double *__restrict__ r, const double *__restrict__ q, PcgState *st,
            double *__restrict__ partials, int n_pq, T *__restrict__ fprime, T *__restrict__ red_e, T *__restrict__ red_g,
            const typename vec2_of<T>::type *__restrict__ tw, const typename vec2_of<T>::type *__restrict__ pt,
            Lines<T> ln, int nr)
{
    extern __shared__ char smem_raw[];
    strip_phase1<T, BC, FUSED, R2, R>(rin, r, q, st, partials, n_pq, fprime, red_e, red_g, tw, pt, ln, nr,
                                      blockIdx.x, reinterpret_cast<T *>(smem_raw));
}

// MT modes per workgroup (one wave each)
template <typename T, int R, int LMAX, int MT>
__global__ void __launch_bounds__(64 * MT)
k_strip_reduced(const T *__restrict__ red_e, const T *__restrict__ red_g, T *__restrict__ red_x, Lines<T> ln,
                PcgState *st, const double *__restrict__ partials, TriGate g, int nr, int N, int G)
{
    __shared__ double red[RED_SLOTS];
    extern __shared__ char smem_raw[];
    T *base = reinterpret_cast<T *>(smem_raw);
    const int l0 = xcd_swizzle(blockIdx.x, N / MT) * MT;
    constexpr bool VEC = MT % (16 / (int)sizeof(T)) == 0;   // 16-byte staging loads
    GatePre pre;
    if (g.mode == 1) gate_issue(st, partials, g, pre);
    strip_stage2<T, VEC>(red_e, red_g, ln, nr, N, G, l0, MT, base);
    if (g.mode != 0 && tridiag_gate(st, partials, g, red, blockIdx.x, g.mode == 1 ? &pre : nullptr) != ST_RUN)
        return;
    __syncthreads();
    strip_solve2<T, R, LMAX, VEC>(red_x, ln, nr, N, G, l0, MT, base);
}

// The same for strips of four rows with the factored coefficients, each wave's
// factors on their way before the stop test.  Bound by its chain of latencies
// (stop test, staging, the wave's solve); against recomputing the coefficients:
// 8.2 -> 6.6 us at 1024^2 FP32, 6.8 -> 5.0 us at 512^2 FP32, 10.1 -> 6.9 us at
// 1021 x 512 FP64, for 6 MB of factors read at 1024^2 FP32.
template <typename T, int LMAX, int MT>
__global__ void __launch_bounds__(64 * MT)
k_strip_reduced_f(const T *__restrict__ red_e, const T *__restrict__ red_g, T *__restrict__ red_x,
                  const T *__restrict__ fac, const T *__restrict__ cb, PcgState *st,
                  const double *__restrict__ partials, TriGate g, int N, int G)
{
    __shared__ double red[RED_SLOTS];
    extern __shared__ char smem_raw[];
    T *te = reinterpret_cast<T *>(smem_raw);
    const int l0 = xcd_swizzle(blockIdx.x, N / MT) * MT;
    constexpr bool VEC = MT % (16 / (int)sizeof(T)) == 0;   // 16-byte staging loads
    GatePre pre;
    if (g.mode == 1) gate_issue(st, partials, g, pre);
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    int S, lo, m;
    red_lane(G, lane, S, lo, m);
    RedFac<T, LMAX> f;
    f.template load<(LMAX > 1)>(fac, l0 + w, LMAX, cb, lo, m, S, lane);   // (two rows a lane: more than 64 strips)
    stage_red<T, VEC>(red_e, red_g, N, G, l0, MT, te);
    if (g.mode != 0 && tridiag_gate(st, partials, g, red, blockIdx.x, g.mode == 1 ? &pre : nullptr) != ST_RUN)
        return;
    __syncthreads();
    f.solve(te + w * G, te + (MT + w) * G, G, lo, m, S, lane);
    store_red<T, VEC>(red_x, N, G, l0, MT, te);
}

// The factors (RedFac), one wave per mode, in FP64 from the r-line arrays of
// precision T: the strips' preparatory solutions (strip_coefs), the reduced
// rows, the elimination of each lane's rows and the cyclic reduction of
// wave_tri, all without their right-hand sides.
template <typename T, int LMAX>
__global__ void __launch_bounds__(64)
k_strip_factors(Lines<T> ln, T *__restrict__ fac, int G)
{
    constexpr int R = 4, n = R - 1;
    const int l = blockIdx.x, lane = threadIdx.x;
    int S, lo, m;
    red_lane(G, lane, S, lo, m);
    const bool active = lane < S;
    const double lam = ln.lam[l];
    double a[LMAX], b[LMAX], c[LMAX];
    // strip s: its first row's response (v0, w0) to the interface rows on either
    // side and its last interior row's (vL, wL)
    auto coefs = [&](int s, double &vL, double &wL, double &v0, double &w0) {
        const int i0 = s * R;
        double cp[R], vp[R], cprev = 0, vprev = 0;
#pragma unroll
        for (int t = 0; t < n; ++t) {
            const double L = t > 0 ? (double)ln.cb[i0 + t - 1] : 0.0;
            const double inv = 1.0 / ((double)ln.db[i0 + t] + (double)ln.rw[i0 + t] * lam - L * cprev);
            cprev = (double)ln.cb[i0 + t] * inv;
            vprev = (t == 0 ? (s > 0 ? (double)ln.cb[i0 - 1] : 0.0) : L * vprev) * inv;
            cp[t] = cprev;
            vp[t] = vprev;
        }
        vL = v0 = vp[n - 1];
        wL = w0 = cp[n - 1];
#pragma unroll
        for (int t = n - 2; t >= 0; --t) {
            v0 = vp[t] + cp[t] * v0;
            w0 = cp[t] * w0;
        }
    };
#pragma unroll
    for (int k = 0; k < LMAX; ++k) {
        a[k] = c[k] = 0;
        b[k] = 1;
        if (k < m) {
            const int s = lo + k, j = s * R + n;
            double vL, wL, v0, w0, vn = 0, wn = 0, x, y;
            coefs(s, vL, wL, v0, w0);
            const double cjm = ln.cb[j - 1], cj = s + 1 < G ? (double)ln.cb[j] : 0.0;
            if (s + 1 < G) coefs(s + 1, x, y, vn, wn);
            a[k] = -cjm * vL;
            b[k] = (double)ln.db[j] + (double)ln.rw[j] * lam - cjm * wL - cj * vn;
            c[k] = -cj * wn;
        }
    }
    T *f = fac + (size_t)l * red_items(LMAX) * S + lane;   // (lanes < S store)
    double vl = 0, wl = 0, v0 = 0, w0 = 1, vp[LMAX], cq[LMAX];
#pragma unroll
    for (int t = 0; t < LMAX; ++t) {
        double inv = 0;
        if (t < m - 1) {
            inv = 1.0 / (t == 0 ? b[0] : b[t] + a[t] * cq[t - 1]);
            vp[t] = -(t == 0 ? a[0] : a[t] * vp[t - 1]) * inv;
            cq[t] = -c[t] * inv;
            vl = vp[t];
            wl = cq[t];
        }
        if (active && t < LMAX - 1) f[t * S] = (T)inv;
        if (active) f[(LMAX - 1 + t) * S] = (T)c[t];
    }
    f += (2 * LMAX - 1) * S;
    if (active) f[0] = (T)a[0];
    if (m >= 2) {
        v0 = vl;
        w0 = wl;
#pragma unroll
        for (int t = LMAX - 1; t >= 0; --t)
            if (t < m - 2) {
                v0 = vp[t] + cq[t] * v0;
                w0 = cq[t] * w0;
            }
    }
    if (!active) v0 = w0 = 0;
    const double V0n = __shfl_down(v0, 1, 64), W0n = __shfl_down(w0, 1, 64);
    double ra = 0, rb = 1, rc = 0;
    if (active) {
        double am = 0, bm = 0, cm = 0;
#pragma unroll
        for (int t = 0; t < LMAX; ++t)
            if (t == m - 1) { am = a[t]; bm = b[t]; cm = c[t]; }
        const bool next = lane + 1 < S;
        ra = m >= 2 ? am * vl : am;
        rb = bm + (m >= 2 ? am * wl : 0.0) + (next ? cm * V0n : 0.0);
        rc = next ? cm * W0n : 0.0;
    }
#pragma unroll
    for (int q = 0; q < 6; ++q) {
        const int k = 1 << q;
        const double am = __shfl_up(ra, k, 64), bm = __shfl_up(rb, k, 64), cm = __shfl_up(rc, k, 64);
        const double ap = __shfl_down(ra, k, 64), bp = __shfl_down(rb, k, 64), cp = __shfl_down(rc, k, 64);
        const bool hm = active && k < S && lane >= k, hp = active && k < S && lane + k < S;
        const double al = hm ? -ra / bm : 0.0, ga = hp ? -rc / bp : 0.0;
        if (active && k < S) {
            rb += (hm ? al * cm : 0.0) + (hp ? ga * ap : 0.0);
            ra = hm ? al * am : 0.0;
            rc = hp ? ga * cp : 0.0;
        }
        if (active) {
            f[(1 + q) * S] = (T)al;
            f[(7 + q) * S] = (T)ga;
        }
    }
    if (active) f[13 * S] = (T)(1.0 / rb);
}

template <typename T, int BC, int MODE, int R2, int R>
__global__ void __launch_bounds__(64 * R)
k_strip_inv(const T *__restrict__ fprime, const T *__restrict__ red_x, ZOut<T, MODE> *__restrict__ zout,
            const double *__restrict__ r, const PcgState *st, double *__restrict__ partials, bool pr,
            const typename vec2_of<T>::type *__restrict__ tw, const typename vec2_of<T>::type *__restrict__ pt,
            Lines<T> ln, int nr, double *__restrict__ dinc, double tau, double rho2, XFin fin)
{
    extern __shared__ char smem_raw[];
    strip_phase3<T, BC, MODE, R2, R>(fprime, red_x, zout, r, st, partials, pr, tw, pt, ln, nr, dinc, tau, rho2,
                                     blockIdx.x, reinterpret_cast<T *>(smem_raw), fin);
}

inline int strip_count(int nr, int R) { return (nr + R - 1) / R; }

template <typename T>
Lines<T> lines_of(const Operator &op);
template <>
Lines<float> lines_of<float>(const Operator &op) { return {op.cb32, op.db32, op.rw32, op.lam32}; }
template <>
Lines<double> lines_of<double>(const Operator &op) { return {op.cb64, op.db64, op.rw64, op.lam64}; }

template <typename T>
const typename vec2_of<T>::type *tw_of(const Operator &op);
template <>
const float2 *tw_of<float>(const Operator &op) { return op.tw32; }
template <>
const double2 *tw_of<double>(const Operator &op) { return op.tw64; }
template <typename T>
const typename vec2_of<T>::type *pt_of(const Operator &op);
template <>
const float2 *pt_of<float>(const Operator &op) { return op.pt32; }
template <>
const double2 *pt_of<double>(const Operator &op) { return op.pt64; }

template <typename T>
T *fac_of(const Operator &op);
template <>
float *fac_of<float>(const Operator &op) { return op.red_fac32; }
template <>
double *fac_of<double>(const Operator &op) { return op.red_fac64; }

template <typename T>
struct RedBufs {
    T *e, *g, *x;
};
template <typename T>
RedBufs<T> red_bufs(const Operator &op, int R)
{
    T *b = static_cast<T *>(op.strip_red);
    const size_t gn = (size_t)strip_count(op.nr, R) * op.nz;
    return {b, b + gn, b + 2 * gn};
}

// modes per reduced-system workgroup: 32 bytes of each strip's row
template <typename T>
constexpr int red_mt() { return 32 / (int)sizeof(T); }
// They fit LDS on every grid that strips take: the reduced data alone in strips of
// four rows, with the r-line arrays in strips of eight.  (Fewer modes per workgroup
// made PCG iterations slower at 1024^2.)
static_assert(strip_fac_lds<float>(1024, red_mt<float>()) <= 65536 && strip_fac_lds<double>(1024, red_mt<double>()) <= 65536);
static_assert(strip_red_lds<float>(4096, 512, red_mt<float>()) <= 159 * 1024 &&
              strip_red_lds<double>(4096, 512, red_mt<double>()) <= 159 * 1024);

template <typename T, int BC, int R2, int R>
void fwd_r(const Operator &op, const ZfwdArgs &a, hipStream_t s)
{
    const RedBufs<T> rb = red_bufs<T>(op, R);
    const dim3 grid(strip_count(op.nr, R)), block(64 * R);
    const size_t shm = (size_t)R * wfft::Geo<R2>::LB * sizeof(cx<T>);
    if (a.fused)
        hipLaunchKernelGGL((k_strip_fwd<T, BC, true, R2, R>), grid, block, shm, s, nullptr, a.r, a.q, a.state, op.partials, a.n_pq, (T *)op.spec, rb.e, rb.g, tw_of<T>(op), pt_of<T>(op),
                           lines_of<T>(op), op.nr);
    else
        hipLaunchKernelGGL((k_strip_fwd<T, BC, false, R2, R>), grid, block, shm, s, a.rin, nullptr, nullptr, a.state, op.partials, 0, (T *)op.spec, rb.e, rb.g, tw_of<T>(op),
                           pt_of<T>(op), lines_of<T>(op), op.nr);
    AXI_CHECK_HIP(hipGetLastError());
}

template <typename T, int BC, int R2, int R>
void inv_r(const Operator &op, const ZinvArgs &a, hipStream_t s)
{
    const RedBufs<T> rb = red_bufs<T>(op, R);
    const dim3 grid(strip_count(op.nr, R)), block(64 * R);
    const size_t shm = (size_t)R * wfft::Geo<R2>::LB * sizeof(cx<T>);
    const T *fp = (const T *)op.spec;
    const auto tw = tw_of<T>(op);
    const auto pt = pt_of<T>(op);
    const Lines<T> ln = lines_of<T>(op);
#define AXI_SINV(MD, Z, RR, ST, PR, D)                                                                           \
    hipLaunchKernelGGL((k_strip_inv<T, BC, MD, R2, R>), grid, block, shm, s, fp, rb.x, (ZOut<T, MD> *)(Z), RR,  \
                       ST, op.partials,                                                                         \
                       PR, tw, pt, ln, op.nr, D, a.tau, a.rho2, a.fin)
    switch (a.mode) {
    case 0: AXI_SINV(0, a.zout, nullptr, nullptr, false, nullptr); break;
    case 1: AXI_SINV(1, a.zout, a.r, a.state, a.pr, nullptr); break;
    case 2: AXI_SINV(2, a.zout, a.r, a.state, false, nullptr); break;
    case 3: AXI_SINV(3, nullptr, nullptr, a.state, false, a.d); break;
    default: AXI_SINV(4, nullptr, nullptr, a.state, false, a.d); break;
    }
#undef AXI_SINV
    AXI_CHECK_HIP(hipGetLastError());
}

template <typename T, int LM, int MT>
void red_launch_f(const Operator &op, const TriGate &g, hipStream_t s)
{
    const RedBufs<T> rb = red_bufs<T>(op, 4);
    const int G = strip_count(op.nr, 4);
    const size_t shm = strip_fac_lds<T>(G, MT);
    static LdsLimit limit;
    limit.raise(reinterpret_cast<const void *>(&k_strip_reduced_f<T, LM, MT>), shm, 159 * 1024);
    hipLaunchKernelGGL((k_strip_reduced_f<T, LM, MT>), dim3(op.nz / MT), dim3(64 * MT), shm, s, rb.e, rb.g, rb.x,
                       fac_of<T>(op), lines_of<T>(op).cb, g.state, op.partials, g, op.nz, G);
    AXI_CHECK_HIP(hipGetLastError());
}

template <typename T, int R, int LM>
void red_launch(const Operator &op, const TriGate &g, hipStream_t s)
{
    constexpr int MT = red_mt<T>();
    const RedBufs<T> rb = red_bufs<T>(op, R);
    const int G = strip_count(op.nr, R), rows = G * R;
    const size_t shm = strip_red_lds<T>(rows, G, MT);
    static LdsLimit limit;
    limit.raise(reinterpret_cast<const void *>(&k_strip_reduced<T, R, LM, MT>), shm, 159 * 1024);
    hipLaunchKernelGGL((k_strip_reduced<T, R, LM, MT>), dim3(op.nz / MT), dim3(64 * MT), shm, s, rb.e, rb.g, rb.x,
                       lines_of<T>(op), g.state, op.partials, g, rows, op.nz, G);
    AXI_CHECK_HIP(hipGetLastError());
}

template <typename T, int R>
void red_r(const Operator &op, const TriGate &g, hipStream_t s)
{
    if constexpr (R == 4) {
        switch (red_rows(strip_count(op.nr, 4))) {
        case 1: return red_launch_f<T, 1, red_mt<T>()>(op, g, s);
        case 2: return red_launch_f<T, 2, red_mt<T>()>(op, g, s);
        case 4: return red_launch_f<T, 4, red_mt<T>()>(op, g, s);
        case 8: return red_launch_f<T, 8, red_mt<T>()>(op, g, s);
        default: return red_launch_f<T, 16, red_mt<T>()>(op, g, s);
        }
    } else {   // at most 512 strips of eight rows
        const int per = (strip_count(op.nr, R) + 63) / 64;
        if (per <= 1) red_launch<T, R, 1>(op, g, s);
        else if (per <= 2) red_launch<T, R, 2>(op, g, s);
        else if (per <= 4) red_launch<T, R, 4>(op, g, s);
        else red_launch<T, R, 8>(op, g, s);
    }
}

template <typename T>
int strip_r2(int nz)
{
    switch (nz) {
    case 256: return 2;
    case 512: return 4;
    case 1024: return 8;
    case 2048: return sizeof(T) == 4 ? 16 : 0;   // FP64 at 2048 would spill
    default: return 0;
    }
}

template <typename T, int BC, int R>
void fwd_rb(const Operator &op, const ZfwdArgs &a, hipStream_t s)
{
    switch (op.nz) {
    case 256: fwd_r<T, BC, 2, R>(op, a, s); break;
    case 512: fwd_r<T, BC, 4, R>(op, a, s); break;
    case 1024: fwd_r<T, BC, 8, R>(op, a, s); break;
    default:
        if constexpr (sizeof(T) == 4) fwd_r<T, BC, 16, R>(op, a, s);
        break;
    }
}

template <typename T, int BC, int R>
void inv_rb(const Operator &op, const ZinvArgs &a, hipStream_t s)
{
    switch (op.nz) {
    case 256: inv_r<T, BC, 2, R>(op, a, s); break;
    case 512: inv_r<T, BC, 4, R>(op, a, s); break;
    case 1024: inv_r<T, BC, 8, R>(op, a, s); break;
    default:
        if constexpr (sizeof(T) == 4) inv_r<T, BC, 16, R>(op, a, s);
        break;
    }
}

template <typename T>
void fwd_t(const Operator &op, int rows, const ZfwdArgs &a, hipStream_t s)
{
    const bool dir = op.bc_z == DIR;
    if (rows == 8) {
        if (dir) fwd_rb<T, DIR, 8>(op, a, s);
        else fwd_rb<T, AXIPCG_Z_NEUMANN, 8>(op, a, s);
    } else {
        if (dir) fwd_rb<T, DIR, 4>(op, a, s);
        else fwd_rb<T, AXIPCG_Z_NEUMANN, 4>(op, a, s);
    }
}

template <typename T>
void inv_t(const Operator &op, int rows, const ZinvArgs &a, hipStream_t s)
{
    const bool dir = op.bc_z == DIR;
    if (rows == 8) {
        if (dir) inv_rb<T, DIR, 8>(op, a, s);
        else inv_rb<T, AXIPCG_Z_NEUMANN, 8>(op, a, s);
    } else {
        if (dir) inv_rb<T, DIR, 4>(op, a, s);
        else inv_rb<T, AXIPCG_Z_NEUMANN, 4>(op, a, s);
    }
}

template <typename T>
bool usable_t(const Operator &op, int R)
{
    if (R != 4 && R != 8) return false;
    if (strip_r2<T>(op.nz) == 0) return false;
    return strip_count(op.nr, R) <= 1024;
}

}  // namespace

// The strip path serves an operator and precision with strips of `rows`
// rows (4 or 8) when the one-wave transforms cover nz and the reduced system fits
// one wavefront's registers (at most 1024 strips).
bool strip_usable(const Operator &op, int prec, int rows)
{
    if (!op.strip_red) return false;
    return prec == AXIPCG_PREC_FP32 ? usable_t<float>(op, rows) : usable_t<double>(op, rows);
}

// The factors of the reduced systems (strips of four rows), for each precision
// whose transforms the strips take.
template <typename T>
static void factors_t(const Operator &op, T **fac, hipStream_t s)
{
    if (strip_r2<T>(op.nz) == 0 || strip_count(op.nr, 4) > 1024) return;
    const int G = strip_count(op.nr, 4), L = red_rows(G);
    void *p = nullptr;
    const hipError_t e = hipMalloc(&p, sizeof(T) * (size_t)op.nz * red_items(L) * red_lanes(G));
    if (e != hipSuccess) throw Error{AXIPCG_ENOMEM, std::string("hipMalloc: ") + hipGetErrorString(e)};
    *fac = static_cast<T *>(p);
#define AXI_FAC(LM) hipLaunchKernelGGL((k_strip_factors<T, LM>), dim3(op.nz), dim3(64), 0, s, lines_of<T>(op), *fac, G)
    if (L == 1) AXI_FAC(1);
    else if (L == 2) AXI_FAC(2);
    else if (L == 4) AXI_FAC(4);
    else if (L == 8) AXI_FAC(8);
    else AXI_FAC(16);
#undef AXI_FAC
    AXI_CHECK_HIP(hipGetLastError());
}

void strip_factors(Operator &op, hipStream_t s)
{
    factors_t<float>(op, &op.red_fac32, s);
    factors_t<double>(op, &op.red_fac64, s);
}

// Reduced data for strips of 4 rows (the larger of the two heights' needs).
size_t strip_red_bytes(int nr, int nz)
{
    return 3 * (size_t)strip_count(nr, 4) * nz * sizeof(double);
}

void strip_fwd(const Operator &op, int prec, int rows, const ZfwdArgs &a, hipStream_t s)
{
    if (prec == AXIPCG_PREC_FP32) fwd_t<float>(op, rows, a, s);
    else fwd_t<double>(op, rows, a, s);
}

void strip_reduced(const Operator &op, int prec, int rows, const TriGate &g, hipStream_t s)
{
    if (prec == AXIPCG_PREC_FP32) {
        if (rows == 8) red_r<float, 8>(op, g, s);
        else red_r<float, 4>(op, g, s);
    } else {
        if (rows == 8) red_r<double, 8>(op, g, s);
        else red_r<double, 4>(op, g, s);
    }
}

void strip_inv(const Operator &op, int prec, int rows, const ZinvArgs &a, hipStream_t s)
{
    if (prec == AXIPCG_PREC_FP32) inv_t<float>(op, rows, a, s);
    else inv_t<double>(op, rows, a, s);
}

}  // namespace axipcg
