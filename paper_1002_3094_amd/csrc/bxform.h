// Block-wide z-transforms of long rows (§4.2 eq. (38); N = 2048 and 4096) that
// one wave cannot hold: one workgroup of N / 8 threads per ROWS rows, a
// radix-8 Stockham FFT of length N (one radix-4 pass where log2 N is no
// multiple of 3) whose butterflies live in registers and whose passes exchange
// through ONE padded LDS buffer.
//
// The reorderings, the split of two real rows out of one complex FFT and the
// scalings are those of zfwd_body / zinv_body (xform.h).  What bounds these
// kernels is LDS passes and barriers, so:
//  - radix 8 takes 4 passes over LDS instead of the radix-4 form's 6, with 21
//    twiddle reads per thread instead of 30;
//  - a pass reads all its values before the barrier that lets it write, so a
//    single buffer serves (N 9/8 values) and twice the workgroups fit a CU;
//  - the inverse's first pass takes its inputs from the pre-twiddle directly,
//    and the rows enter and leave as 16-byte pairs of both rows at once.
// Measured against the radix-4 form: FP64 rows of 2048, forward 33.4 -> 21.3 us
// and inverse 40.3 -> 20.9 us at 2048^2 (3.2 TB/s); FP32 rows of 4096 at 4096^2,
// PCG forward 143 -> 122 us (3.9 TB/s), PCG inverse 104 -> 64 us (4.2 TB/s).
// Slot i of the buffer sits at i + i / 8: a pass writes with strides of 1, 8,
// 64 or 512 butterflies of 8, and the gap puts 16 consecutive lanes' 16-byte
// values (32 lanes' 8-byte ones) in distinct banks for each of them.
#pragma once

#include "kernels.h"
#include "wfft.h"
#include "wxform.h"

namespace axipcg {
namespace {

template <typename T, int N>
struct BlockFft {
    static constexpr int NT = N / 8;   // threads
    static constexpr size_t LDS = (size_t)(N + N / 8) * sizeof(cx<T>);
    using V2 = typename vec2_of<T>::type;
    __device__ static int at(int i) { return i + (i >> 3); }

    // One radix-8 pass on the values v[r] = element j + r N/8 (j the thread):
    // twiddles, DFT, and the store after every thread has read its values.
    template <int NS>
    __device__ static void pass8(cx<T> (&v)[8], cx<T> *buf, const V2 *__restrict__ tw)
    {
        const int j = threadIdx.x, jm = j & (NS - 1);
        if constexpr (NS > 1) {
            constexpr int stride = N / (NS * 8);
#pragma unroll
            for (int r = 1; r < 8; ++r) v[r] = cmul(v[r], ld_tw<T>(tw, r * jm * stride));
        }
        wfft::Dft<T, 8>::run(v);
        __syncthreads();
        const int o = ((j - jm) << 3) + jm;
#pragma unroll
        for (int r = 0; r < 8; ++r) buf[at(o + r * NS)] = v[r];
        __syncthreads();
    }
    __device__ static void read8(cx<T> (&v)[8], const cx<T> *buf)
    {
#pragma unroll
        for (int r = 0; r < 8; ++r) v[r] = buf[at((int)threadIdx.x + r * NT)];
    }
    // The FFT: in, v[r] = element threadIdx.x + r N/8 (read from buf or made
    // by the caller; every thread may still be reading buf); out, the spectrum
    // in natural order in buf.
    __device__ static void run(cx<T> (&v)[8], cx<T> *buf, const V2 *__restrict__ tw)
    {
        pass8<1>(v, buf, tw);
        read8(v, buf);
        pass8<8>(v, buf, tw);
        read8(v, buf);
        pass8<64>(v, buf, tw);
        if constexpr (N == 4096) {
            read8(v, buf);
            pass8<512>(v, buf, tw);
        } else {
            static_assert(N == 2048, "rows of 2048 or 4096 points");
            // radix 4 at 512: butterflies j = thread and thread + 256
            constexpr int NS = 512, Q = N / 4;
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int r = 0; r < 4; ++r) v[4 * h + r] = buf[at((int)threadIdx.x + h * NT + r * Q)];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int jm = (int)threadIdx.x + h * NT;   // < NS
#pragma unroll
                for (int r = 1; r < 4; ++r) v[4 * h + r] = cmul(v[4 * h + r], ld_tw<T>(tw, r * jm));
                wfft::Dft<T, 4>::run(&v[4 * h]);
            }
            __syncthreads();
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int r = 0; r < 4; ++r) buf[at((int)threadIdx.x + h * NT + r * NS)] = v[4 * h + r];
            __syncthreads();
        }
    }
};

// Spectra of one row (ROWS 1) or of two, both real, through one complex FFT
// (the second row in the imaginary parts, zero unless `two`): v0, v1 hold the
// thread's pairs (2 (t + j NT), + 1), s0, s1 receive modes t + e NT.  The
// buffer is free on entry and may still be read by others on exit, this
// thread's reads done.
template <typename T, int BC, int N, int ROWS>
__device__ __forceinline__ void pair_spectra(const double2 (&v0)[4], const double2 (&v1)[4], bool two, cx<T> *buf,
                                             const typename vec2_of<T>::type *__restrict__ tw,
                                             const typename vec2_of<T>::type *__restrict__ pt, T (&s0)[8], T (&s1)[8])
{
    using F = BlockFft<T, N>;
    constexpr int NT = F::NT;
    const int t = threadIdx.x;
    // even k -> v[k/2], odd k -> v[N-1-(k-1)/2] (sine: y_k = (-1)^k x_k)
    const T sg = (BC == DIR) ? (T)-1 : (T)1;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int n = t + j * NT;
        buf[F::at(n)] = {(T)v0[j].x, two ? (T)v1[j].x : (T)0};
        buf[F::at(N - 1 - n)] = {sg * (T)v0[j].y, two ? sg * (T)v1[j].y : (T)0};
    }
    __syncthreads();
    cx<T> v[8];
    F::read8(v, buf);
    F::run(v, buf, tw);
    const T nrm = (T)sqrt(2.0 / N);
    const T half = (T)0.70710678118654752440;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int j = t + e * NT;
        const int m = (BC == DIR) ? N - 1 - j : j;
        const cx<T> zm = buf[F::at(m)];
        const cx<T> w = ld_tw<T>(pt, m);
        const T sc = nrm * (m == 0 ? half : (T)1);
        if constexpr (ROWS == 2) {
            // Z = V0 + i V1: V0_m = (Z_m + conj Z_{N-m}) / 2, V1_m = (Z_m - conj Z_{N-m}) / 2i
            const cx<T> zc = buf[F::at((N - m) & (N - 1))];
            const T v0x = (T)0.5 * (zm.x + zc.x), v0y = (T)0.5 * (zm.y - zc.y);
            const T v1x = (T)0.5 * (zm.y + zc.y), v1y = (T)0.5 * (zc.x - zm.x);
            s0[e] = sc * (v0x * w.x - v0y * w.y);
            s1[e] = sc * (v1x * w.x - v1y * w.y);
        } else {
            s0[e] = sc * (zm.x * w.x - zm.y * w.y);
            s1[e] = (T)0;
        }
        in_register(s0[e]);
        in_register(s1[e]);
    }
}

// Forward transform of rows i0 .. i0 + ROWS - 1 (the last workgroup of an odd
// nr has one): fused PCG step or plain, as zfwd_body.
template <typename T, int BC, bool FUSED, int N, int ROWS>
__device__ __forceinline__ void zfwd8_body(const double *__restrict__ rin, double *__restrict__ r,
                                           const double *__restrict__ q, PcgState *st, double *__restrict__ partials,
                                           int n_pq, T *__restrict__ spec,
                                           const typename vec2_of<T>::type *__restrict__ tw,
                                           const typename vec2_of<T>::type *__restrict__ pt, int nr, int vb)
{
    using F = BlockFft<T, N>;
    constexpr int NT = F::NT;
    extern __shared__ char smem_raw[];
    cx<T> *buf = reinterpret_cast<cx<T> *>(smem_raw);
    __shared__ double red[RED_SLOTS];
    const int i0 = xcd_swizzle(vb, (nr + ROWS - 1) / ROWS) * ROWS;
    const int t = threadIdx.x;
    const bool two = ROWS == 2 && i0 + 1 < nr;
    int done = 0, k_it = 0;
    double rho_slot[2] = {0.0, 0.0};
    TotalLoads<2> pq_pre;
    if constexpr (FUSED) {
        done = st->done;
        k_it = st->iters;
        rho_slot[0] = st->rho[0];
        rho_slot[1] = st->rho[1];
        total_issue(partials + SLOT_PQ * MAX_PARTIALS, n_pq, pq_pre);
    } else {
        if (st && st->done) return;
    }
    // pairs (2 (t + j NT), + 1), j < 4, of each row
    double2 rv[ROWS][4], qv[ROWS][4];
#pragma unroll
    for (int s = 0; s < ROWS; ++s) {
        const size_t base = (size_t)(i0 + (s && !two ? 0 : s)) * N + 2 * t;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            rv[s][j] = *reinterpret_cast<const double2 *>((FUSED ? r : rin) + base + 2 * j * NT);
            if (FUSED) qv[s][j] = *reinterpret_cast<const double2 *>(q + base + 2 * j * NT);
        }
    }
    double rr = 0.0;
    if constexpr (FUSED) {
        if (done) return;
        const double pq = total_finish(partials + SLOT_PQ * MAX_PARTIALS, n_pq, pq_pre, red);
        if (!(pq > 0.0) || !(pq < 1e308)) {
            if (vb == 0 && threadIdx.x == 0) st->done = ST_BREAK;
            return;
        }
        const double alpha = rho_slot[k_it & 1] / pq;
        if (vb == 0 && threadIdx.x == 0) st->step = {alpha, k_it, 0};
#pragma unroll
        for (int s = 0; s < ROWS; ++s) {
            if (s && !two) continue;
            const size_t base = (size_t)(i0 + s) * N + 2 * t;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                double2 &v = rv[s][j];
                v.x -= alpha * qv[s][j].x;
                v.y -= alpha * qv[s][j].y;
                *reinterpret_cast<double2 *>(r + base + 2 * j * NT) = v;
                rr += v.x * v.x + v.y * v.y;
            }
        }
    }
    T s0[8], s1[8];
    pair_spectra<T, BC, N, ROWS>(rv[0], rv[ROWS - 1], two, buf, tw, pt, s0, s1);
    T *row0 = spec + (size_t)i0 * N;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        row0[t + e * NT] = s0[e];
        if (two) row0[N + t + e * NT] = s1[e];
    }
    if (FUSED) {
        const double s = block_sum(rr, red);
        if (threadIdx.x == 0) partials[SLOT_RR * MAX_PARTIALS + vb] = s;
    }
}

// The inverse FFT of one row's or two rows' spectra: pair_stage puts them
// (modes t + e NT in y0, y1) into the free buffer as unnormalised DCT-II
// coefficients Y_m; pair_inverse leaves N times the rows, reordered, in the
// buffer's real and imaginary parts.
template <typename T, int BC, int N>
__device__ __forceinline__ void pair_stage(const T (&y0)[8], const T (&y1)[8], cx<T> *buf)
{
    using F = BlockFft<T, N>;
    const T isc = (T)sqrt(0.5 * N);      // 1 / sqrt(2/N)
    const T sq2 = (T)1.41421356237309504880;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int j = (int)threadIdx.x + e * F::NT;
        const int m = (BC == DIR) ? N - 1 - j : j;
        const T sc = isc * (m == 0 ? sq2 : (T)1);
        buf[F::at(m)] = {y0[e] * sc, y1[e] * sc};
    }
}

template <typename T, int N, int ROWS>
__device__ __forceinline__ void pair_inverse(cx<T> *buf, const typename vec2_of<T>::type *__restrict__ tw,
                                             const typename vec2_of<T>::type *__restrict__ pt)
{
    using F = BlockFft<T, N>;
    constexpr int NT = F::NT;
    const int t = threadIdx.x;
    __syncthreads();
    // the FFT of conj(V0) + i conj(V1), conj(V)_m = w_m (Y_m + i Y_{N-m})
    cx<T> v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int m = t + e * NT;
        const cx<T> y = buf[F::at(m)];
        const cx<T> yn = (m == 0) ? cx<T>{(T)0, (T)0} : buf[F::at((N - m) & (N - 1))];
        const cx<T> w = ld_tw<T>(pt, m);
        const cx<T> q0 = {w.x * y.x - w.y * yn.x, w.x * yn.x + w.y * y.x};
        if constexpr (ROWS == 2) {
            const cx<T> q1 = {w.x * y.y - w.y * yn.y, w.x * yn.y + w.y * y.y};
            v[e] = {q0.x - q1.y, q0.y + q1.x};
        } else {
            v[e] = q0;
        }
    }
    F::run(v, buf, tw);
}

// What an inverse transform of a row or a pair of rows reads besides its
// spectra (r and the old z, or the increment; in flight during the FFT) and
// its results' way out of the buffer (pair_inverse), as pairs of columns.
template <typename T, int MODE, int N>
struct RowPair {
    static constexpr bool PCGM = (MODE == 1 || MODE == 2);
    static constexpr bool CHEB = (MODE == 3 || MODE == 4);
    static constexpr int NT = N / 8;
    double2 rv[2][4], zo[2][4];
    __device__ __forceinline__ void load(const ZOut<T, MODE> *zout, const double *r, const double *dinc, bool pr, int i,
                                         bool two)
    {
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            if (s && !two) continue;
            const size_t base = (size_t)(i + s) * N + 2 * threadIdx.x;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (PCGM) {
                    rv[s][j] = *reinterpret_cast<const double2 *>(r + base + 2 * j * NT);
                    if (pr) zo[s][j] = ld_pair(zout + base + 2 * j * NT);
                }
                if (MODE == 3) rv[s][j] = *reinterpret_cast<const double2 *>(dinc + base + 2 * j * NT);
            }
        }
    }
    template <int BC, int ROWS>
    __device__ __forceinline__ void store(const cx<T> *buf, ZOut<T, MODE> *zout, double *dinc, bool pr, int i, bool two,
                                          double c1, double c2, double &rz, double &rzo) const
    {
        using F = BlockFft<T, N>;
        const int t = threadIdx.x;
        const T invN = (T)1 / (T)N;
        const T sg = (BC == DIR) ? -invN : invN;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int n = t + j * NT;
            const cx<T> ev = buf[F::at(n)], od = buf[F::at(N - 1 - n)];
#pragma unroll
            for (int s = 0; s < ROWS; ++s) {
                if (s && !two) continue;
                const double2 zv = make_double2((double)((s ? ev.y : ev.x) * invN), (double)((s ? od.y : od.x) * sg));
                const size_t base = (size_t)(i + s) * N + 2 * t + 2 * j * NT;
                if (PCGM) {
                    if (pr) rzo += rv[s][j].x * zo[s][j].x + rv[s][j].y * zo[s][j].y;
                    rz += rv[s][j].x * zv.x + rv[s][j].y * zv.y;
                }
                if (CHEB) {
                    const double2 d = rv[s][j];
                    *reinterpret_cast<double2 *>(dinc + base) =
                        (MODE == 4) ? make_double2(c2 * zv.x, c2 * zv.y)
                                    : make_double2(c1 * d.x + c2 * zv.x, c1 * d.y + c2 * zv.y);
                } else {
                    st_pair(zout + base, zv);
                }
            }
        }
    }
};

// Inverse transform of the same rows, modes as zinv_body.
template <typename T, int BC, int MODE, int N, int ROWS>
__device__ __forceinline__ void zinv8_body(const T *__restrict__ spec, ZOut<T, MODE> *__restrict__ zout,
                                           const double *__restrict__ r, const PcgState *st,
                                           double *__restrict__ partials, bool pr,
                                           const typename vec2_of<T>::type *__restrict__ tw,
                                           const typename vec2_of<T>::type *__restrict__ pt, int nr, int vb,
                                           double *__restrict__ dinc, double tau, double rho2, const XFin &fin)
{
    constexpr bool PCGM = (MODE == 1 || MODE == 2);
    constexpr bool CHEB = (MODE == 3 || MODE == 4);
    using F = BlockFft<T, N>;
    constexpr int NT = F::NT;
    extern __shared__ char smem_raw[];
    cx<T> *buf = reinterpret_cast<cx<T> *>(smem_raw);
    __shared__ double red[RED_SLOTS];
    const int i0 = xcd_swizzle(vb, (nr + ROWS - 1) / ROWS) * ROWS;
    const int t = threadIdx.x;
    const bool two = ROWS == 2 && i0 + 1 < nr;
    const int done = MODE != 0 ? st->done : 0;
    T y0[8], y1[8];
    const T *s0 = spec + (size_t)i0 * N, *s1 = s0 + (two ? N : 0);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        y0[e] = s0[t + e * NT];
        y1[e] = ROWS == 2 ? s1[t + e * NT] : (T)0;
    }
    pair_stage<T, BC, N>(y0, y1, buf);
    RowPair<T, MODE, N> io;
    io.load(zout, r, dinc, pr, i0, two);
    if (done) {   // every workgroup alike
        if (MODE == 1) x_finish(fin, st, (size_t)i0 * N, (two ? 2 : 1) * N, t, NT);
        return;
    }
    double c1 = 0.0, c2 = 0.0;
    if (CHEB) {
        const double alpha = cheb_alpha(st->iters + 1, rho2);
        c1 = alpha - 1.0;
        c2 = alpha * tau;
    }
    pair_inverse<T, N, ROWS>(buf, tw, pt);
    double rz = 0.0, rzo = 0.0;
    io.template store<BC, ROWS>(buf, zout, dinc, pr, i0, two, c1, c2, rz, rzo);
    if (PCGM) {
        const double s = block_sum(rz, red);
        if (threadIdx.x == 0) partials[SLOT_RZ * MAX_PARTIALS + vb] = s;
        if (pr) {
            const double so = block_sum(rzo, red);
            if (threadIdx.x == 0) partials[SLOT_RZOLD * MAX_PARTIALS + vb] = so;
        }
    }
}

}  // namespace
}  // namespace axipcg
