// PCG for a small grid in one launch of one workgroup (§2.2 eq. (8) with
// conjugate-gradient parameters, the preconditioner of §4.2).
//
// A grid of up to 4096 points cannot fill the chip, and its solve is a chain of
// launches of some 5 us each, four per iteration, that do well under 1 us of
// work: what they wait for is memory they have just written.  Here one
// workgroup of 1024 threads keeps everything but the scheme coefficients in its
// CU: x, r and p in registers (four points a thread), p (for its neighbours),
// the spectra and the r-solves' pivots in LDS.  Per iteration:
//   - the SpMV from LDS; three block-wide sums (p.q, ||r||^2, r.z);
//   - the z-transforms of all rows at once through complex radix-8 FFTs, two rows
//     each in FP64 and one in FP32 (the pairing and scalings of zfwd_body /
//     zinv_body), eight values a thread;
//   - one r-system per z-mode, two threads to a mode: both ends are eliminated
//     towards the middle row, whose value then runs back to both ends (pivots
//     formed once per solve, so that a step is one dependent multiply-add).
// What bounds it is latency inside one CU.  An iteration at 64 x 64 FP64 takes some
// 30 000 clocks (13.8 us): the r-solves' serial chains 8000, the two FFTs 4800, the
// passes that bring rows to them and spectra from them 8400, the three block-wide
// sums 5900 (with the coefficients' way from L2 during the first), the SpMV and p
// 2800; eighteen workgroup barriers are in these.  At 250 x 16 the r-solves are
// 24 000 of 46 000.  A whole solve, as launches and here (us):
//   64 x 64 FP64 531 -> 331, FP32 509 -> 296      32 x 128 FP32 542 -> 309, FP64 566 -> 365
//   128 x 32 FP64 535 -> 391, FP32 511 -> 354     250 x 16 FP32 534 -> 432, FP64 576 -> 482
#include "xform.h"

namespace axipcg {
namespace {

constexpr int TINY_POINTS = 4096, TINY_THREADS = 1024, TINY_PPT = TINY_POINTS / TINY_THREADS;
constexpr int TINY_NZ_MIN = 16, TINY_NZ_MAX = 128, TINY_NR_MAX = 256;

template <typename T>
struct TinyArgs {
    const double *b;
    double *x;
    const double *D, *CR, *CZ;
    const T *cb, *db, *rw, *lam;
    const typename vec2_of<T>::type *tw, *pt;
    int nr, nz, bc;
    double rtol2;
    int maxit, flags;
    PcgState *st;
    HostMirror *mirror;
    unsigned seq;
};

// Rows to a complex FFT: two in FP64.  FP32 rows take one each, as rounding of the
// larger one's size could be all of a smaller partner.
template <typename T>
__host__ __device__ constexpr int tiny_pair() { return sizeof(T) == 8 ? 2 : 1; }
template <typename T>
__host__ __device__ constexpr int tiny_ffts(int nr) { return (nr + tiny_pair<T>() - 1) / tiny_pair<T>(); }

// Complex slots of an FFT: slot i at i + i / 8, which spreads a pass's strided
// writes over the banks.
template <int N>
constexpr int tiny_row() { return N + N / 8; }

// LDS: p, the FFT buffers, the spectra, the pivots, the tables and the r-line
// couplings.
template <typename T, int N>
size_t tiny_lds(int nr)
{
    return sizeof(double) * nr * N + sizeof(cx<T>) * ((size_t)tiny_ffts<T>(nr) * tiny_row<N>() + 2 * N) +
           sizeof(T) * (2 * (size_t)nr * N + nr);
}

// v plus its value at another lane of the same 16 (a DPP move, no trip
// through LDS as a shuffle takes).
template <int CTRL>
__device__ inline double dpp_add(double v)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, true);
    return v + __hiloint2double(hi, lo);
}
// Sum over each 16 lanes, in all of them: neighbours, pairs, then mirrored
// halves and rows, whose lanes already agree in groups of 4 and 8.
__device__ inline double row_sum(double v)
{
    v = dpp_add<0xB1>(v);    // quad_perm 1,0,3,2
    v = dpp_add<0x4E>(v);    // quad_perm 2,3,0,1
    v = dpp_add<0x141>(v);   // row_half_mirror
    return dpp_add<0x140>(v);   // row_mirror
}
__device__ inline double lane_value(double v, int lane)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                            __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// Sum over the workgroup, returned in every thread; `sm` (16 doubles) is this
// sum's alone until the next barrier but one.
__device__ inline double tiny_sum(double v, double *sm)
{
    v = row_sum(v);
    v = (lane_value(v, 0) + lane_value(v, 16)) + (lane_value(v, 32) + lane_value(v, 48));
    if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = v;
    __syncthreads();
    return lane_value(row_sum(sm[threadIdx.x & 15]), 0);
}

// All FFTs in place, N / 8 threads to each; the threads past the last one take part
// in the barriers.  The buffer is complete on entry and
// on exit (barriers included).
template <typename T, int N>
struct TinyFft {
    __device__ static int at(int i) { return i + (i >> 3); }
    static constexpr int NT = N / 8;
    template <int RAD, int NS>
    __device__ __forceinline__ static void pass(cx<T> *a, const cx<T> *tw, int j0, bool act)
    {
        constexpr int Q = N / RAD, PER = 8 / RAD;   // butterflies in all, and of a thread
        cx<T> v[8];
        if (act) {
#pragma unroll
            for (int h = 0; h < PER; ++h) {
                const int j = j0 + h * NT, jm = j & (NS - 1);
                cx<T> *u = v + h * RAD;
#pragma unroll
                for (int r = 0; r < RAD; ++r) u[r] = a[at(j + r * Q)];
                if constexpr (NS > 1) {
#pragma unroll
                    for (int r = 1; r < RAD; ++r) u[r] = cmul(u[r], tw[r * jm * (N / (NS * RAD))]);
                }
                wfft::Dft<T, RAD>::run(u);
            }
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                in_register(v[r].x);
                in_register(v[r].y);
            }
        }
        __syncthreads();
        if (act) {
#pragma unroll
            for (int h = 0; h < PER; ++h) {
                const int j = j0 + h * NT, jm = j & (NS - 1), o = (j - jm) * RAD + jm;
#pragma unroll
                for (int r = 0; r < RAD; ++r) a[at(o + r * NS)] = v[h * RAD + r];
            }
        }
        __syncthreads();
    }
    __device__ __forceinline__ static void run(cx<T> *buf, const cx<T> *tw, int nfft, int t)
    {
        const int q = t / NT, j = t & (NT - 1);
        const bool act = q < nfft;
        cx<T> *a = buf + (act ? q : 0) * tiny_row<N>();
        pass<8, 1>(a, tw, j, act);
        if constexpr (N == 16) pass<2, 8>(a, tw, j, act);
        else if constexpr (N == 32) pass<4, 8>(a, tw, j, act);
        else pass<8, 8>(a, tw, j, act);
        if constexpr (N == 128) pass<2, 64>(a, tw, j, act);
    }
};

template <typename T, int N>
__global__ void __launch_bounds__(TINY_THREADS) k_pcg_tiny(TinyArgs<T> A)
{
    extern __shared__ __attribute__((aligned(16))) char smem_raw[];
    __shared__ double sums[4][16];
    constexpr int ROW = tiny_row<N>(), PAIR = tiny_pair<T>();
    using F = TinyFft<T, N>;
    const int nr = A.nr, n = nr * N, t = threadIdx.x, nfft = tiny_ffts<T>(nr);
    const bool dir = A.bc == DIR;
    double *ps = reinterpret_cast<double *>(smem_raw);
    cx<T> *buf = reinterpret_cast<cx<T> *>(ps + n);
    cx<T> *twl = buf + nfft * ROW, *ptl = twl + N;
    T *f = reinterpret_cast<T *>(ptl + N), *piv = f + n, *cb = piv + n;   // f: spectra [nr][N]

    // this thread's points e = t + 1024 j, row i = e / N, column k = e % N; the
    // scheme coefficients are read (from L2) for each SpMV, as registers for
    // them would be spilled around the transforms
    double x[TINY_PPT], r[TINY_PPT], p[TINY_PPT];
    struct Coefs {
        double D[TINY_PPT], CR[TINY_PPT], CRm[TINY_PPT], CZ[TINY_PPT], CZm[TINY_PPT];
    };
    auto coefs = [&](Coefs &c, int t) {
#pragma unroll
        for (int j = 0; j < TINY_PPT; ++j) {
            const int e = t + TINY_THREADS * j;
            const bool in = e < n;
            c.D[j] = in ? A.D[e] : 0.0;
            c.CR[j] = in ? A.CR[e] : 0.0;   // (0 in the last row, CZ in the last column)
            c.CRm[j] = in && e >= N ? A.CR[e - N] : 0.0;
            c.CZ[j] = in ? A.CZ[e] : 0.0;
            c.CZm[j] = in && e > 0 ? A.CZ[e - 1] : 0.0;
        }
    };
    Coefs c0;
    coefs(c0, t);
    double bb = 0.0;
#pragma unroll
    for (int j = 0; j < TINY_PPT; ++j) {
        const int e = t + TINY_THREADS * j;
        const bool in = e < n;
        x[j] = in ? A.x[e] : 0.0;
        r[j] = in ? A.b[e] : 0.0;
        p[j] = 0.0;
        bb += r[j] * r[j];
        if (in) ps[e] = x[j];
    }
    for (int k = t; k < N; k += TINY_THREADS) {
        twl[k] = ld_tw<T>(A.tw, k);
        ptl[k] = ld_tw<T>(A.pt, k);
    }
    for (int i = t; i < nr; i += TINY_THREADS) cb[i] = A.cb[i];
    __syncthreads();
    // y = A v of the vector in ps (v: this thread's own values)
    auto stencil_at = [&](const Coefs &c, int j, double v, int t) {
        const int e = t + TINY_THREADS * j;
        if (e >= n) return 0.0;
        double y = c.D[j] * v;
        if (e + N < n) y -= c.CR[j] * ps[e + N];
        if (e >= N) y -= c.CRm[j] * ps[e - N];
        if (e + 1 < n) y -= c.CZ[j] * ps[e + 1];
        if (e > 0) y -= c.CZm[j] * ps[e - 1];
        return y;
    };
    double rr = 0.0;
#pragma unroll
    for (int j = 0; j < TINY_PPT; ++j) {
        r[j] -= stencil_at(c0, j, x[j], t);
        rr += r[j] * r[j];
    }
    // pivots: mode l by threads l (rows 0 .. mid - 1, downwards) and N + l (rows
    // nr - 1 .. mid + 1, upwards), then row mid
    const int mid = nr / 2;
    const int l = t & (N - 1);
    const bool top = t < N, solver = t < 2 * N;
    if (solver) {
        const T lam = A.lam[l];
        const int m = top ? mid : nr - 1 - mid;
        T inv = 0;
        for (int s = 0; s < m; ++s) {
            const int i = top ? s : nr - 1 - s;
            const T c = s == 0 ? (T)0 : cb[top ? i - 1 : i];   // coupling to the row eliminated before
            inv = (T)1 / (A.db[i] + A.rw[i] * lam - c * c * inv);
            piv[i * N + l] = inv;
        }
    }
    bb = tiny_sum(bb, sums[0]);
    rr = tiny_sum(rr, sums[1]);   // (its barrier also publishes the pivots)
    if (t < N) {
        T d = A.db[mid] + A.rw[mid] * A.lam[l];
        if (mid > 0) d -= cb[mid - 1] * cb[mid - 1] * piv[(mid - 1) * N + l];
        if (mid + 1 < nr) d -= cb[mid] * cb[mid] * piv[(mid + 1) * N + l];
        piv[mid * N + l] = (T)1 / d;
    }
    const T nrm = (T)sqrt(2.0 / N), half = (T)0.70710678118654752440;
    const T isc = (T)sqrt(0.5 * N), sq2 = (T)1.41421356237309504880, invN = (T)1 / (T)N;

    // z = B^{-1} r into `z`
    auto precond = [&](double (&z)[TINY_PPT], int t) {
#pragma unroll
        for (int j = 0; j < TINY_PPT; ++j) {
            const int e = t + TINY_THREADS * j, i = e / N, k = e & (N - 1);
            if (e >= n) continue;
            cx<T> *slot = buf + i / PAIR * ROW + F::at((k & 1) ? N - 1 - (k >> 1) : k >> 1);
            const T v = (dir && (k & 1)) ? -(T)r[j] : (T)r[j];
            if constexpr (PAIR == 1) *slot = {v, (T)0};
            else if (i & 1) slot->y = v;
            else slot->x = v;
        }
        if (PAIR == 2 && (nr & 1) && t < N) buf[(nfft - 1) * ROW + F::at(t)].y = (T)0;
        __syncthreads();
        F::run(buf, twl, nfft, t);
        for (int e = t; e < nfft * N; e += TINY_THREADS) {
            const int q = e / N, j = e & (N - 1);
            const int m = dir ? N - 1 - j : j;
            const cx<T> zm = buf[q * ROW + F::at(m)], w = ptl[m];
            const T sc = nrm * (m == 0 ? half : (T)1);
            if constexpr (PAIR == 1) {
                f[e] = sc * (zm.x * w.x - zm.y * w.y);
                continue;
            }
            const cx<T> zc = buf[q * ROW + F::at((N - m) & (N - 1))];
            f[2 * q * N + j] = sc * ((T)0.5 * (zm.x + zc.x) * w.x - (T)0.5 * (zm.y - zc.y) * w.y);
            if (2 * q + 1 < nr)
                f[(2 * q + 1) * N + j] = sc * ((T)0.5 * (zm.y + zc.y) * w.x - (T)0.5 * (zc.x - zm.x) * w.y);
        }
        __syncthreads();
        const int l = t & (N - 1);
        const bool top = t < N, solver = t < 2 * N;
        const int m = top ? mid : nr - 1 - mid, step = top ? N : -N;
        T *fe = f + (top ? 0 : nr - 1) * N + l;            // row s of this end at fe + s step
        const T *pe = piv + (top ? 0 : nr - 1) * N + l;
        const int cs = top ? 1 : -1;                       // coupling of rows s - 1, s of this end: ce[s cs]
        const T *ce = cb + (top ? -1 : nr - 1);
        if (solver) {
            // eight rows' values at a time, on their way together (row 0 has no
            // coupling: whatever ce[0] holds meets g = 0)
            T g = 0;
            int s = 0;
            for (; s + 8 <= m; s += 8) {
                T fv[8], iv[8], cv[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    fv[u] = fe[(s + u) * step];
                    iv[u] = pe[(s + u) * step];
                    cv[u] = ce[(s + u) * cs];
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    g = fv[u] * iv[u] + (cv[u] * iv[u]) * g;
                    fe[(s + u) * step] = g;
                }
            }
            for (; s < m; ++s) {
                const T iv = pe[s * step];
                g = fe[s * step] * iv + (ce[s * cs] * iv) * g;
                fe[s * step] = g;
            }
        }
        __syncthreads();
        T y = 0;
        if (solver) {
            T v = f[mid * N + l];
            if (mid > 0) v += cb[mid - 1] * f[(mid - 1) * N + l];
            if (mid + 1 < nr) v += cb[mid] * f[(mid + 1) * N + l];
            y = v * piv[mid * N + l];
            in_register(y);
        }
        __syncthreads();
        if (solver) {
            if (top) f[mid * N + l] = y;
            int s = m - 1;
            for (; s >= 7; s -= 8) {
                T fv[8], cv[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    fv[u] = fe[(s - u) * step];
                    cv[u] = ce[(s - u + 1) * cs] * pe[(s - u) * step];
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    y = fv[u] + cv[u] * y;
                    fe[(s - u) * step] = y;
                }
            }
            for (; s >= 0; --s) {
                y = fe[s * step] + (ce[(s + 1) * cs] * pe[s * step]) * y;
                fe[s * step] = y;
            }
        }
        __syncthreads();
        for (int e = t; e < nfft * N; e += TINY_THREADS) {
            const int q = e / N, m1 = e & (N - 1), m2 = (N - m1) & (N - 1);
            const int j1 = dir ? N - 1 - m1 : m1, j2 = dir ? N - 1 - m2 : m2;
            const T *f0 = f + PAIR * q * N;
            const T s1 = isc * (m1 == 0 ? sq2 : (T)1), s2 = m1 == 0 ? (T)0 : isc;
            const T a0 = f0[j1] * s1, b0 = f0[j2] * s2;
            const cx<T> w = ptl[m1];
            if constexpr (PAIR == 1) {
                buf[q * ROW + F::at(m1)] = {w.x * a0 - w.y * b0, w.x * b0 + w.y * a0};
                continue;
            }
            const bool two = 2 * q + 1 < nr;
            const T *f1 = two ? f0 + N : f0;
            const T a1 = two ? f1[j1] * s1 : (T)0, b1 = two ? f1[j2] * s2 : (T)0;
            buf[q * ROW + F::at(m1)] = {(w.x * a0 - w.y * b0) - (w.x * b1 + w.y * a1),
                                        (w.x * b0 + w.y * a0) + (w.x * a1 - w.y * b1)};
        }
        __syncthreads();
        F::run(buf, twl, nfft, t);
#pragma unroll
        for (int j = 0; j < TINY_PPT; ++j) {
            const int e = t + TINY_THREADS * j, i = e / N, k = e & (N - 1);
            z[j] = 0.0;
            if (e >= n) continue;
            const cx<T> v = buf[i / PAIR * ROW + F::at((k & 1) ? N - 1 - (k >> 1) : k >> 1)];
            const T s = (PAIR == 2 && (i & 1) ? v.y : v.x) * invN;
            z[j] = (double)((dir && (k & 1)) ? -s : s);
        }
    };

    const double tol2 = A.rtol2 * bb;
    int status = ST_RUN, it = 0;
    if (bb == 0.0) status = ST_BZERO;
    else if (!(rr == rr) || rr > 1e300) status = ST_BREAK;
    else if (rr <= tol2) status = ST_CONV;
    double rho = 0.0;
    while (status == ST_RUN) {
        // the thread's index anew, so that the loop's addresses are formed where
        // they are used instead of being held in registers across the loop
        int ti = t;
        in_register(ti);
        double z[TINY_PPT], s = 0.0;
        precond(z, ti);
#pragma unroll
        for (int j = 0; j < TINY_PPT; ++j) s += r[j] * z[j];
        Coefs c;   // on their way during the sum
        coefs(c, ti);
        const double rn = tiny_sum(s, sums[2]);
        const double beta = it > 0 ? rn / rho : 0.0;
        rho = rn;
#pragma unroll
        for (int j = 0; j < TINY_PPT; ++j) {
            const int e = ti + TINY_THREADS * j;
            p[j] = it > 0 ? z[j] + beta * p[j] : z[j];
            if (e < n) ps[e] = p[j];
        }
        __syncthreads();
        double q[TINY_PPT];
        s = 0.0;
#pragma unroll
        for (int j = 0; j < TINY_PPT; ++j) {
            q[j] = stencil_at(c, j, p[j], ti);
            s += p[j] * q[j];
        }
        const double pq = tiny_sum(s, sums[3]);
        if (!(pq > 0.0) || !(pq < 1e308)) {
            status = ST_BREAK;
            break;
        }
        const double alpha = rho / pq;
        s = 0.0;
#pragma unroll
        for (int j = 0; j < TINY_PPT; ++j) {
            x[j] += alpha * p[j];
            r[j] -= alpha * q[j];
            s += r[j] * r[j];
        }
        rr = tiny_sum(s, sums[1]);
        ++it;
        if (!(rr == rr) || rr > 1e300) status = ST_BREAK;
        else if (rr <= tol2) status = ST_CONV;
        else if (it >= A.maxit) status = ST_MAXIT;
    }
#pragma unroll
    for (int j = 0; j < TINY_PPT; ++j) {
        const int e = t + TINY_THREADS * j;
        if (e < n) A.x[e] = status == ST_BZERO ? 0.0 : x[j];
    }
    // the host may go on as soon as it sees the record: the solution first
    __threadfence_system();
    __syncthreads();
    if (t == 0) {
        A.st->rr = rr;
        A.st->bb = bb;
        A.st->tol2 = tol2;
        A.st->iters = it;
        A.st->done = status;
        A.st->maxit = A.maxit;
        A.st->flags = A.flags;
        A.st->step = {0.0, it, 0};
        publish(A.mirror, A.seq, rr, bb, it, status);
    }
}

template <typename T, int N>
void tiny_launch_n(const TinyArgs<T> &a, hipStream_t s)
{
    const size_t shm = tiny_lds<T, N>(a.nr);
    static LdsLimit limit;
    limit.raise(reinterpret_cast<const void *>(&k_pcg_tiny<T, N>), shm, 159 * 1024);   // (512 bytes are the static sums)
    hipLaunchKernelGGL((k_pcg_tiny<T, N>), dim3(1), dim3(TINY_THREADS), shm, s, a);
    AXI_CHECK_HIP(hipGetLastError());
}

template <typename T>
void tiny_launch(const TinyArgs<T> &a, hipStream_t s)
{
    switch (a.nz) {
    case 16: return tiny_launch_n<T, 16>(a, s);
    case 32: return tiny_launch_n<T, 32>(a, s);
    case 64: return tiny_launch_n<T, 64>(a, s);
    default: return tiny_launch_n<T, 128>(a, s);
    }
}

}  // namespace

// Grids the one-workgroup solve takes: up to 4096 points (four a thread, whose
// vectors then fit registers and LDS), rows of 16 .. 128 points (shorter ones
// leave the r-solves to a few threads) and lines of up to 256 rows, what 4096
// points of such rows hold.  A solve of 4096 points takes 296 .. 482 us here
// and 509 .. 576 us as launches; above 4096 the launches' work begins to count
// and one CU's registers no longer hold the vectors.
bool tiny_usable(const Operator &op)
{
    return op.nr * op.nz <= TINY_POINTS && op.nz >= TINY_NZ_MIN && op.nz <= TINY_NZ_MAX && op.nr <= TINY_NR_MAX;
}

void tiny_pcg(const Operator &op, const double *b, double *x, double rtol2, int maxit, int prec, int flags,
              unsigned seq, hipStream_t s)
{
    if (prec == AXIPCG_PREC_FP32)
        tiny_launch(TinyArgs<float>{b, x, op.D, op.CR, op.CZ, op.cb32, op.db32, op.rw32, op.lam32, op.tw32, op.pt32, op.nr,
                                    op.nz, op.bc_z, rtol2, maxit, flags, op.state, op.mirror_dev, seq}, s);
    else
        tiny_launch(TinyArgs<double>{b, x, op.D, op.CR, op.CZ, op.cb64, op.db64, op.rw64, op.lam64, op.tw64, op.pt64,
                                     op.nr, op.nz, op.bc_z, rtol2, maxit, flags, op.state, op.mirror_dev, seq}, s);
}

}  // namespace axipcg
