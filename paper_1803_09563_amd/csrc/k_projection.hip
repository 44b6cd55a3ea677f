// Pressure projection, Sec. 3.2.2 Eqs. (var poisson) and (projection) with constant rho:
//   r = rho (D_h u*) / dt;  L_h p = r (zero-mean p);  u^{n+1} = u* - (dt/rho) G_h p.
// The 7-point Laplacian L_h = D_h G_h is diagonalised by discrete Fourier transforms in periodic
// directions (eigenvalues -(4/h^2) sin^2(pi k/N)); across walls (homogeneous Neumann rows) each
// (kx, kz) mode is a tridiagonal system in y solved by a Thomas sweep.
//
// Passes over the half spectrum S[kz][j][kx] (kx < nx/2+1, FP64 complex; rows padded to a
// multiple of 8 values, 128 bytes):
//   periodic: div+fft(x) | fft(y) | fft(z), divide, ifft(z) | ifft(y) | ifft(x) -> p | correct
//   walls:    div+fft(x) | fft(z) | Thomas(y)                | ifft(z) | ifft(x) -> p | correct
// Real x-lines are transformed two at a time as one complex line (a + i b).  Periodic grids with
// nx == ny up to 64, and 96 or 128 in batches with a z plane for every CU, fuse the first two and the last
// two periodic passes into one block per z plane, whose half-spectrum plane stays in LDS.
#include "evp_internal.h"
#include "fft_lds.h"

namespace evp {

namespace {

constexpr int NT = 256;    // threads per block of the line-transform kernels
constexpr int TK = 16;     // consecutive kx per block in the strided passes

__device__ __forceinline__ int wrapi(int i, int n) { return i < 0 ? i + n : (i >= n ? i - n : i); }
// sc (D_h u*) of a cell from a = u, u(i-1), v, -, w, w(k-1) and vm = v(j-1), in the same operations in
// every kernel
__device__ __forceinline__ double divergence(const double* a, double vm, double idx, double idy, double idz, double sc)
{
    return sc * fma(a[4] - a[5], idz, fma(a[2] - vm, idy, (a[0] - a[1]) * idx));
}

// ---------------------------------------------------------------------------------------------
// div + forward x transform
// ---------------------------------------------------------------------------------------------
template <int N>
__global__ __launch_bounds__(NT) void k_div_fftx(Batch B)
{
    constexpr int T = fft_threads<N>();
    constexpr int LP = NT / T;                 // complex lines (= real line pairs) per block
    constexpr int NHF = N / 2 + 1;
    __shared__ double2 buf[LP * N];
    __shared__ double2 tw[N];
    const Desc& D = *B.d[blockIdx.y];
    const double sc = D.rho / B.dt[blockIdx.y];
    const int tid = threadIdx.x;
    for (int n = tid; n < N; n += NT) tw[n] = gload2((gptr<const double2>)D.twx + n);
    const bool from_u = (B.state[blockIdx.y] & ST_FROM_U) != 0;
    const gptr<const double> us = (gptr<const double>)(from_u ? D.u : D.us);
    const gptr<const double> vs = (gptr<const double>)(from_u ? D.v : D.vs);
    const gptr<const double> ws = (gptr<const double>)(from_u ? D.w : D.ws);
    const gptr<double2> spec = (gptr<double2>)D.spec;
    const int ny = D.ny, nz = D.nz;
    const int nlines = ny * nz;
    const int npairs = (nlines + 1) >> 1;
    const int pair0 = blockIdx.x * LP;
    const double idx = D.idx, idy = D.idy, idz = D.idz;
    const long long sxy = (long long)N * ny;
    // divergence of u* at the inputs of the thread's first butterflies, on the two lines of its pair;
    // the loads of up to four elements (48 values) are issued before their arithmetic
    const bool walls = D.walls != 0;
    const int lp = tid / T, t = tid - (tid / T) * T;
    const bool active = lp < LP;
    constexpr int R0 = fft_radix<N, false>(0), NB = N / R0, MB = fft_per_thread<N, T, R0>();
    long long q0[2];
    int j0[2], k0[2];
    bool ok[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int l = 2 * (pair0 + lp) + h;
        ok[h] = active && l < nlines;
        const int ll = ok[h] ? l : 0;
        k0[h] = ll / ny;
        j0[h] = ll - k0[h] * ny;
        q0[h] = (long long)ll * N;
    }
    double2 v[MB][R0];
    constexpr int G = R0 % 4 == 0 ? 4 : R0;
#pragma unroll
    for (int m = 0; m < MB; ++m) {
        const int jb = t + m * T < NB ? t + m * T : 0;
#pragma unroll
        for (int g0 = 0; g0 < R0; g0 += G) {
            double ld[G][2][6];
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const int i = jb + (g0 + g) * NB;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const long long q = q0[h] + i;
                    ld[g][h][0] = us[q];
                    ld[g][h][1] = us[q0[h] + wrapi(i - 1, N)];
                    ld[g][h][2] = vs[q];
                    ld[g][h][3] = (j0[h] > 0) ? vs[q - N] : vs[q + (long long)(ny - 1) * N];
                    ld[g][h][4] = ws[q];
                    ld[g][h][5] = (k0[h] > 0) ? ws[q - sxy] : ws[q + (long long)(nz - 1) * sxy];
                }
            }
#pragma unroll
            for (int g = 0; g < G; ++g) {
                double r2[2];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const double* a = ld[g][h];
                    const double vm = (walls && j0[h] == 0) ? 0.0 : a[3];        // wall: v = 0 below row 0
                    r2[h] = ok[h] ? divergence(a, vm, idx, idy, idz, sc) : 0.0;
                }
                v[m][g0 + g] = make_double2(r2[0], r2[1]);
            }
        }
    }
    double2* const line = buf + (active ? lp : 0) * N;
    constexpr int RL = fft_radix<N, false>(make_plan(N).nst - 1), ML = fft_per_thread<N, T, RL>();
    double2 z[ML][RL];
    fft_from<N, T, false, 0, 1, true>(v, line, 1, t, active, tw, [&](int, double2 x, int m, int r) { z[m][r] = x; });
    __syncthreads();
#pragma unroll
    for (int m = 0; m < ML; ++m)
#pragma unroll
        for (int r = 0; r < RL; ++r)
            if (active && t + m * T < N / RL) line[t + m * T + r * (N / RL)] = z[m][r];
    __syncthreads();
    const int sh = D.sh;
    for (int e = tid; e < LP * NHF; e += NT) {
        const int l2 = e / NHF, k = e - l2 * NHF;
        const int pair = pair0 + l2;
        if (pair >= npairs) continue;
        const double2 Z = buf[l2 * N + k];
        const double2 Zc = cconj(buf[l2 * N + (k == 0 ? 0 : N - k)]);
        const double2 s = cadd(Z, Zc), d = csub(Z, Zc);
        const int la = 2 * pair;
        gstore2(spec + (long long)la * sh + k, make_double2(0.5 * s.x, 0.5 * s.y));
        if (la + 1 < nlines)
            gstore2(spec + (long long)(la + 1) * sh + k, make_double2(0.5 * d.y, -0.5 * d.x));
    }
}

// ---------------------------------------------------------------------------------------------
// periodic grids whose x-y half-spectrum plane fits in LDS: one block per z plane does the
// divergence and the forward x and y transforms in one pass, and the inverse y and x transforms
// in another (the same line transforms, twiddles and two-for-one formulas as the separate
// passes, so the same numbers, with two spectrum round trips and two launches fewer)
// ---------------------------------------------------------------------------------------------
// Threads of the plane kernels: a small plane keeps few busy, and a block of fewer waves starts and passes
// its barriers sooner (projection of 8^3: 18.0 us with 1024 threads, 13.5 with 128; 24^3: 20.2 and 17.2)
template <int N> constexpr int plane_block() { return N <= 12 ? 128 : N <= 24 ? 256 : N <= 48 ? 512 : 1024; }

// threads per y column: the largest of N/8, N/16, N/32 (at least 1) that lets all N/2 + 1 columns
// of the plane be transformed at once
template <int N>
constexpr int plane_y_threads()
{
    int t = fft_threads<N>();
    while (t > 1 && (N / 2 + 1) * t > plane_block<N>()) t /= 2;
    return t;
}

// y transforms of all nh columns of the plane in LDS (stride nh)
template <int N>
__device__ __forceinline__ void plane_y_fft(double2* buf, const double2* tw, int tid)
{
    constexpr int NH = N / 2 + 1, TY = plane_y_threads<N>();
    static_assert(NH * TY <= plane_block<N>(), "one pass of y transforms");
    const int col = tid / TY, t = tid - (tid / TY) * TY;
    fft_stages<N, TY, 0, 1>(buf + (col < NH ? col : 0), NH, t, col < NH, tw);
}

template <int N>
__global__ __launch_bounds__(plane_block<N>()) void k_div_fftxy(Batch B)
{
    constexpr int NH = N / 2 + 1, L = N / 2, TX = fft_threads<N>(), NTP = plane_block<N>();
    static_assert(L * TX <= NTP, "one pass of x transforms");
    __shared__ double2 buf[N * NH];
    __shared__ double2 twx[N], twy[N];
    const Desc& D = *B.d[blockIdx.y];
    const int tid = threadIdx.x, k = blockIdx.x;
    for (int n = tid; n < N; n += NTP) {
        twx[n] = gload2((gptr<const double2>)D.twx + n);
        twy[n] = gload2((gptr<const double2>)D.twy + n);
    }
    const double sc = D.rho / B.dt[blockIdx.y];
    const bool from_u = (B.state[blockIdx.y] & ST_FROM_U) != 0;
    const gptr<const double> us = (gptr<const double>)(from_u ? D.u : D.us);
    const gptr<const double> vs = (gptr<const double>)(from_u ? D.v : D.vs);
    const gptr<const double> ws = (gptr<const double>)(from_u ? D.w : D.ws);
    const int nz = D.nz;
    const long long sxy = (long long)N * N;
    const double idx = D.idx, idy = D.idy, idz = D.idz;
    // divergence of u* on the plane; complex line p holds rows 2p (real) and 2p + 1 (imaginary).
    // Loads of four elements (48 values) are issued before their arithmetic and LDS stores.
    constexpr int MD = (L * N + NTP - 1) / NTP, GD = MD < 4 ? MD : 4;
#pragma unroll
    for (int g0 = 0; g0 < MD; g0 += GD) {
        double ld[GD][2][6];
#pragma unroll
        for (int m = 0; m < GD; ++m) {
            const int e = tid + (g0 + m) * NTP;
            const int ee = (g0 + m < MD && e < L * N) ? e : 0;
            const int p = ee / N, i = ee - (ee / N) * N;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int j = 2 * p + h;
                const long long q = ((long long)k * N + j) * N + i;
                ld[m][h][0] = us[q];
                ld[m][h][1] = us[q - i + wrapi(i - 1, N)];
                ld[m][h][2] = vs[q];
                ld[m][h][3] = (j > 0) ? vs[q - N] : vs[q + (long long)(N - 1) * N];
                ld[m][h][4] = ws[q];
                ld[m][h][5] = (k > 0) ? ws[q - sxy] : ws[q + (long long)(nz - 1) * sxy];
            }
        }
#pragma unroll
        for (int m = 0; m < GD; ++m) {
            const int e = tid + (g0 + m) * NTP;
            if (g0 + m >= MD || e >= L * N) continue;
            double r2[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const double* a = ld[m][h];
                r2[h] = divergence(a, a[3], idx, idy, idz, sc);
            }
            buf[e] = make_double2(r2[0], r2[1]);
        }
    }
    __syncthreads();
    {
        const int lp = tid / TX, t = tid - (tid / TX) * TX;
        fft_stages<N, TX, 0, 1>(buf + (lp < L ? lp : 0) * N, 1, t, lp < L, twx);
    }
    // two real spectra from each complex line, into rows j of the plane's half spectrum [j][kx]
    constexpr int MS = (L * NH + NTP - 1) / NTP;
    double2 za[MS], zb[MS];
#pragma unroll
    for (int m = 0; m < MS; ++m) {
        const int e = tid + m * NTP;
        if (e < L * NH) {
            const int p = e / NH, kx = e - (e / NH) * NH;
            const double2 Z = buf[p * N + kx];
            const double2 Zc = cconj(buf[p * N + (kx == 0 ? 0 : N - kx)]);
            const double2 sm = cadd(Z, Zc), d = csub(Z, Zc);
            za[m] = make_double2(0.5 * sm.x, 0.5 * sm.y);
            zb[m] = make_double2(0.5 * d.y, -0.5 * d.x);
        }
    }
    __syncthreads();
#pragma unroll
    for (int m = 0; m < MS; ++m) {
        const int e = tid + m * NTP;
        if (e < L * NH) {
            const int p = e / NH, kx = e - (e / NH) * NH;
            buf[(2 * p) * NH + kx] = za[m];
            buf[(2 * p + 1) * NH + kx] = zb[m];
        }
    }
    __syncthreads();
    plane_y_fft<N>(buf, twy, tid);
    const int sh = D.sh;
    const gptr<double2> spec = (gptr<double2>)D.spec + (long long)k * N * sh;
    for (int e = tid; e < N * NH; e += NTP) {
        const int row = e / NH, kx = e - row * NH;
        gstore2(spec + row * sh + kx, buf[e]);
    }
}

template <int N>
__global__ __launch_bounds__(plane_block<N>()) void k_ifftxy(Batch B)
{
    constexpr int NH = N / 2 + 1, L = N / 2, TX = fft_threads<N>(), NTP = plane_block<N>();
    static_assert(L * TX <= NTP, "one pass of x transforms");
    __shared__ double2 buf[N * NH];
    __shared__ double2 twx[N], twy[N];
    const Desc& D = *B.d[blockIdx.y];
    const int tid = threadIdx.x, k = blockIdx.x;
    for (int n = tid; n < N; n += NTP) {
        twx[n] = gload2((gptr<const double2>)D.twx + n);
        twy[n] = gload2((gptr<const double2>)D.twy + n);
    }
    // inverse y transform by conjugation on the way in and out
    const int sh = D.sh;
    const gptr<const double2> spec = (gptr<const double2>)D.spec + (long long)k * N * sh;
    {
        constexpr int MS = (N * NH + NTP - 1) / NTP;
        double2 v[MS];
#pragma unroll
        for (int m = 0; m < MS; ++m) {
            const int e0 = tid + m * NTP, e = e0 < N * NH ? e0 : 0;
            const int row = e / NH, kx = e - row * NH;
            v[m] = gload2(spec + row * sh + kx);
        }
#pragma unroll
        for (int m = 0; m < MS; ++m) {
            const int e = tid + m * NTP;
            if (e < N * NH) buf[e] = cconj(v[m]);
        }
    }
    __syncthreads();
    plane_y_fft<N>(buf, twy, tid);
    // Hermitian extension of rows 2p and 2p + 1 into complex line p (a + i b)
    constexpr int ME = (L * N + NTP - 1) / NTP;
    double2 ze[ME];
#pragma unroll
    for (int m = 0; m < ME; ++m) {
        const int e = tid + m * NTP;
        if (e < L * N) {
            const int p = e / N, n = e - (e / N) * N;
            const int kx = n <= N / 2 ? n : N - n;
            double2 a = cconj(buf[(2 * p) * NH + kx]), b = cconj(buf[(2 * p + 1) * NH + kx]);
            if (n > N / 2) { a = cconj(a); b = cconj(b); }
            ze[m] = cconj(make_double2(a.x - b.y, a.y + b.x));
        }
    }
    __syncthreads();
#pragma unroll
    for (int m = 0; m < ME; ++m) {
        const int e = tid + m * NTP;
        if (e < L * N) buf[e] = ze[m];
    }
    __syncthreads();
    {
        const int lp = tid / TX, t = tid - (tid / TX) * TX;
        fft_stages<N, TX, 0, 1>(buf + (lp < L ? lp : 0) * N, 1, t, lp < L, twx);
    }
    const gptr<double> p = (gptr<double>)D.p + (long long)k * N * N;
    for (int e = tid; e < L * N; e += NTP) {
        const int pr = e / N, n = e - (e / N) * N;
        const double2 z = cconj(buf[e]);
        p[(long long)(2 * pr) * N + n] = z.x;
        p[(long long)(2 * pr + 1) * N + n] = z.y;
    }
}

// ---------------------------------------------------------------------------------------------
// strided forward / inverse transform along y (axis 1) or z (axis 2), in place
// ---------------------------------------------------------------------------------------------
// A tile is TK consecutive kx of one y or z line bundle, T threads per column; lines so short that a
// tile has less than a wave take several tiles per block.  A thread loads the inputs of its first
// butterflies straight into registers and stores its last results from them, so a line passes
// through LDS only between the stages (one exchange for lengths of two radices, two for three).  Against
// staging the tile through LDS before and after the transform, with every stage from LDS to LDS:
// forward y 12.2 -> 11.1 us, solve 19.9 -> 16.8, inverse 14.9 -> 13.5, x inverse 13.7 -> 11.1 at 128^3;
// forward z 20.0 -> 17.7, inverse z 17.5 -> 17.2, x inverse 20.7 -> 17.2 on the 256 x 128 x 128 channel; no change at 512 x 256 x 256,
// where each pass is at the rate of memory (93 us for 538 MB).
template <int N>
constexpr int strided_threads() { return fft_threads<N>() < NT / TK ? fft_threads<N>() : NT / TK; }
template <int N>
constexpr int strided_tiles() { return strided_threads<N>() * TK >= 64 ? 1 : 64 / (strided_threads<N>() * TK); }
template <int N>
constexpr int strided_block() { return strided_threads<N>() * TK * strided_tiles<N>(); }

template <int N, bool INV>
__global__ __launch_bounds__(strided_block<N>()) void k_fft_strided(Batch B, int axis)
{
    constexpr int T = strided_threads<N>(), NTL = strided_tiles<N>();
    __shared__ double2 buf[NTL][N * TK];
    __shared__ double2 tw[N];
    const Desc& D = *B.d[blockIdx.y];
    const int tid = threadIdx.x;
    const gptr<const double2> twg = (gptr<const double2>)(axis == 1 ? D.twy : D.twz);
    for (int n = tid; n < N; n += strided_block<N>()) tw[n] = gload2(twg + n);
    const int nh = D.nh, sh = D.sh, ny = D.ny;
    const int ntk = (nh + TK - 1) / TK;
    const int c = tid % TK, t = (tid / TK) % T, sub = tid / (TK * T);
    const int id = blockIdx.x * NTL + sub;
    const int tile = id % ntk, other = id / ntk;
    const int kx = tile * TK + c;
    const bool active = kx < nh && other < (axis == 1 ? D.nz : ny);
    long long base, es;
    if (axis == 1) { base = (long long)other * ny * sh + kx; es = sh; }
    else { base = (long long)other * sh + kx; es = (long long)sh * ny; }
    const gptr<double2> line = (gptr<double2>)D.spec + (active ? base : 0);
    constexpr int R0 = fft_radix<N, false>(0), NB = N / R0, MB = fft_per_thread<N, T, R0>();
    double2 v[MB][R0];
#pragma unroll
    for (int m = 0; m < MB; ++m) {
        const int j = t + m * T < NB ? t + m * T : 0;
#pragma unroll
        for (int r = 0; r < R0; ++r) v[m][r] = gload2(line + (j + r * NB) * es);
    }
    if (INV) {
#pragma unroll
        for (int m = 0; m < MB; ++m)
#pragma unroll
            for (int r = 0; r < R0; ++r) v[m][r] = cconj(v[m][r]);
    }
    fft_from<N, T, false, 0, 1, true>(v, buf[sub] + c, TK, t, active, tw,
                                      [&](int k, double2 x, int, int) { gstore2(line + k * es, INV ? cconj(x) : x); });
}

// ---------------------------------------------------------------------------------------------
// periodic: transform along z, divide by the Laplacian eigenvalue, transform back (in place).  The way
// back takes the radices in reverse order and so starts on the results where they are.
// ---------------------------------------------------------------------------------------------
template <int N>
__global__ __launch_bounds__(strided_block<N>()) void k_solve_periodic(Batch B)
{
    constexpr int T = strided_threads<N>(), NTL = strided_tiles<N>();
    __shared__ double2 buf[NTL][N * TK];
    __shared__ double2 tw[N];
    __shared__ double ez[N];        // Laplacian eigenvalues along z
    const Desc& D = *B.d[blockIdx.y];
    const int tid = threadIdx.x;
    for (int n = tid; n < N; n += strided_block<N>()) {
        tw[n] = gload2((gptr<const double2>)D.twz + n);
        ez[n] = ((gptr<const double>)D.eigz)[n];
    }
    const int nh = D.nh, sh = D.sh, ny = D.ny;
    const int ntk = (nh + TK - 1) / TK;
    const int c = tid % TK, t = (tid / TK) % T, sub = tid / (TK * T);
    const int id = blockIdx.x * NTL + sub;
    const int kx = (id % ntk) * TK + c, ky = id / ntk;
    const bool active = kx < nh && ky < ny;
    const long long es = (long long)sh * ny;
    const gptr<double2> line = (gptr<double2>)D.spec + (active ? (long long)ky * sh + kx : 0);
    const double exy = active ? ((gptr<const double>)D.eigx)[kx] + ((gptr<const double>)D.eigy)[ky] : 1.0;
    const double scale = 1.0 / ((double)D.nx * ny * N);
    constexpr int NS = make_plan(N).nst;
    constexpr int R0 = fft_radix<N, false>(0), NB = N / R0, MB = fft_per_thread<N, T, R0>();
    constexpr int RL = fft_radix<N, false>(NS - 1), ML = fft_per_thread<N, T, RL>();
    double2 v[MB][R0];
#pragma unroll
    for (int m = 0; m < MB; ++m) {
        const int j = t + m * T < NB ? t + m * T : 0;
#pragma unroll
        for (int r = 0; r < R0; ++r) v[m][r] = gload2(line + (j + r * NB) * es);
    }
    double2 z[ML][RL];
    fft_from<N, T, false, 0, 1, true>(v, buf[sub] + c, TK, t, active, tw, [&](int, double2 x, int m, int r) { z[m][r] = x; });
    if constexpr (NS == 1) __syncthreads();      // ez is there (longer lines have passed a barrier)
#pragma unroll
    for (int m = 0; m < ML; ++m)
#pragma unroll
        for (int r = 0; r < RL; ++r) {
            const int kz = (t + m * T < N / RL ? t + m * T : 0) + r * (N / RL);
            const double f = (kx == 0 && ky == 0 && kz == 0) ? 0.0 : scale / (exy + ez[kz]);
            z[m][r] = cconj(cscale(z[m][r], f));        // inverse transform by conjugation
        }
    fft_from<N, T, true, 0, 1, false>(z, buf[sub] + c, TK, t, active, tw,
                                      [&](int k, double2 x, int, int) { gstore2(line + k * es, cconj(x)); });
}

// ---------------------------------------------------------------------------------------------
// walls: tridiagonal solve in y for every (kx, kz), pivots precomputed per (kx, |kz|)
// ---------------------------------------------------------------------------------------------
// A block holds TS_M modes, and each group of TS_M lanes holds TS_L rows of them in registers
// (segment w of a block: rows [TS_L w, TS_L w + TS_L)), so the spectrum is read once and written
// once.  Both sweeps are first-order linear recurrences,
//   forward   d'_j = s r_j iv_j + g_j d'_{j-1},
//   backward  x_j  = d'_j + g_j x_{j+1}  (j <= ny-2; x_{ny-1} = d'_{ny-1}),  g_j = -a iv_j,
// with |g_j| <= 1 (diagonally dominant rows).  Each segment runs its rows with a zero
// value coming in and keeps the product of its coefficients; the segments' (product, last value)
// pairs go through LDS, each segment composes those of the segments before it (after it,
// backward) into its incoming value, and adds that value times the running product of its
// coefficients to its rows.  Mathematically the sequential sweep; the sums are associated
// differently.  Against one lane per mode sweeping sequentially (the spectrum read and written
// twice, a chain of 2 ny dependent steps in few waves): 208 -> 96 us at 512x256x256, 82 -> 15 us at
// 96x400x64.  Up to 256 rows, blocks of 16 modes (256 threads) let three of them share a CU at the
// kernel's 166 registers; 32 modes (two per CU) took 114 us, 8 modes 99 us.  Taller channels take 8
// modes (128 contiguous bytes of a row) in up to 64 segments, 512 threads at 1024 rows.
constexpr int TS_L = 16;     // rows per lane
constexpr int kRawWord3 = 0x00020000;   // raw-buffer format word of CDNA: 32-bit data, no swizzle
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
template <int TS_M, int TS_SEG>   // modes per block, segments per block at most
__global__ __launch_bounds__(TS_M * TS_SEG) void k_thomas_seg(Batch B)
{
    __shared__ double fwd[3][TS_SEG][TS_M];    // forward: product, last d'.x, last d'.y
    __shared__ double bwd[3][TS_SEG][TS_M];    // backward: product, first x.x, first x.y
    __shared__ double gsum[TS_SEG];
    const Desc& D = *B.d[blockIdx.y];
    const int nh = D.nh, sh = D.sh, ny = D.ny, nz = D.nz;
    const int lane = threadIdx.x % TS_M, seg = threadIdx.x / TS_M, nseg = blockDim.x / TS_M;
    // modes run over the padded rows (a block's modes start on a 128-byte line); lanes past the
    // last mode take part in the barriers and load only in-bounds lines they discard
    const int col = blockIdx.x * TS_M + lane;
    const int kz = col / sh, kx = col - kz * sh;
    const bool live = kz < nz && kx < nh;
    const int kzc = live ? kz : 0, kzr = live ? kz - (TS_SEG > 16 ? (blockIdx.x * TS_M) / sh : 0) : 0;
    const int kzs = kzc <= nz - kzc ? kzc : nz - kzc;
    const double a = D.idy * D.idy;
    const double scale = 1.0 / ((double)D.nx * nz);
    // From row jc on (up to row ny-2) the pivot recurrence of every mode of these 64 has reached its
    // fixed point in floating point: those rows use the mode's pivot of row ny-2, loaded once,
    // instead of a load per row (the same numbers)
    const int jc = ((gptr<const int>)D.pvj)[blockIdx.x * TS_M / 64];
    const int j0 = seg * TS_L;
    // raw buffer accesses: the lane's byte offset of its first row in one register, the row step
    // m sh as the wave-uniform offset (no per-row 64-bit addresses held for the stores)
    // (offsets from the start of the spectrum up to 256 rows; the taller spectra pass 2^31 bytes, and
    // count from the plane of the block's first mode)
    const int kzb = TS_SEG > 16 ? (blockIdx.x * TS_M) / sh : 0;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((EVP_GLOBAL void*)(D.spec + (long long)kzb * ny * sh), (short)0, 0x7fffffff, kRawWord3);
    const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc((EVP_GLOBAL void*)D.piv, (short)0, 0x7fffffff, kRawWord3);
    const unsigned vs = (unsigned)((((long long)kzr * ny + j0) * sh + kx) * 16);
    const unsigned vp = (unsigned)((((long long)kzs * ny + j0) * sh + kx) * 8);
    // v: the right-hand side scaled by the row's pivot, then d', then x; g: -a iv_j.  All loads
    // are issued before any is used: a row past ny, a lane past the last mode and a converged
    // pivot read row m of the first mode instead (in bounds, the same few lines for the whole
    // grid) and discard it, so that no load sits behind a branch.
    double2 v[TS_L];
    double g[TS_L];
    {
        const unsigned plast = (unsigned)((((long long)kzs * ny + ny - 2) * sh + kx) * 8);
        const double pinf = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rp, live ? plast : 0u, 0, 0));
        dvec2 t[TS_L];
        double pl[TS_L];
#pragma unroll
        for (int m = 0; m < TS_L; ++m) {
            const int j = j0 + m;
            const bool in = live && j < ny;
            const bool need = in && (j < jc || j == ny - 1);
            t[m] = __builtin_bit_cast(dvec2, __builtin_amdgcn_raw_buffer_load_b128(rs, in ? vs : 0u, (unsigned)(m * sh * 16), 0));
            pl[m] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rp, need ? vp : 0u, (unsigned)(m * sh * 8), 0));
        }
#pragma unroll
        for (int m = 0; m < TS_L; ++m) {
            const int j = j0 + m;
            const bool in = live && j < ny;
            const double iv = in ? ((j < jc || j == ny - 1) ? pl[m] : pinf) : 0.0;
            v[m] = make_double2(scale * iv * t[m].x, scale * iv * t[m].y);
            g[m] = -a * iv;
        }
    }
    // forward sweep of the segment from a zero incoming value (rows past ny have iv = 0 and stay 0)
    {
        double2 dp = make_double2(0.0, 0.0);
        double pr = 1.0;
#pragma unroll
        for (int m = 0; m < TS_L; ++m) {
            dp = make_double2(v[m].x + g[m] * dp.x, v[m].y + g[m] * dp.y);
            v[m] = dp;
            pr *= g[m];
        }
        fwd[0][seg][lane] = pr;
        fwd[1][seg][lane] = dp.x;
        fwd[2][seg][lane] = dp.y;
    }
    __syncthreads();
    if (seg > 0) {
        double2 in = make_double2(0.0, 0.0);
#pragma unroll 2
        for (int q = 0; q < seg; ++q) {
            const double p = fwd[0][q][lane];
            in = make_double2(fwd[1][q][lane] + p * in.x, fwd[2][q][lane] + p * in.y);
        }
        double pr = 1.0;
#pragma unroll
        for (int m = 0; m < TS_L; ++m) {
            pr *= g[m];
            v[m] = make_double2(v[m].x + pr * in.x, v[m].y + pr * in.y);
        }
    }
    // backward sweep of the segment from a zero incoming value x_{j0 + TS_L}
    {
        double2 x = make_double2(0.0, 0.0);
        double pr = 1.0;
#pragma unroll
        for (int m = TS_L - 1; m >= 0; --m) {
            const double gb = j0 + m <= ny - 2 ? g[m] : 0.0;
            x = make_double2(v[m].x + gb * x.x, v[m].y + gb * x.y);
            v[m] = x;
            pr *= gb;
        }
        bwd[0][seg][lane] = pr;
        bwd[1][seg][lane] = x.x;
        bwd[2][seg][lane] = x.y;
    }
    __syncthreads();
    if (seg < nseg - 1) {
        double2 in = make_double2(0.0, 0.0);
#pragma unroll 2
        for (int q = nseg - 1; q > seg; --q) {
            const double p = bwd[0][q][lane];
            in = make_double2(bwd[1][q][lane] + p * in.x, bwd[2][q][lane] + p * in.y);
        }
        double pr = 1.0;
#pragma unroll
        for (int m = TS_L - 1; m >= 0; --m) {
            pr *= j0 + m <= ny - 2 ? g[m] : 0.0;
            v[m] = make_double2(v[m].x + pr * in.x, v[m].y + pr * in.y);
        }
    }
    double sum = 0.0;
#pragma unroll
    for (int m = 0; m < TS_L; ++m) {
        const int j = j0 + m;
        if (live && j < ny) {
            dvec2 t;
            t.x = v[m].x;
            t.y = v[m].y;
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, t), rs, vs, (unsigned)(m * sh * 16), 0);
            sum += v[m].x;
        }
    }
    // gauge from the (0, 0) mode (lane 0 of block 0): segment sums added in segment order
    if (blockIdx.x == 0) {
        if (lane == 0) gsum[seg] = sum;
        __syncthreads();
        if (threadIdx.x == 0) {
            double t = 0.0;
            for (int q = 0; q < nseg; ++q) t += gsum[q];
            ((gptr<double>)D.gauge)[0] = t / ny;
        }
    }
}

// ---------------------------------------------------------------------------------------------
// inverse x transform of two half spectra -> two real lines of p
// ---------------------------------------------------------------------------------------------
template <int N>
__global__ __launch_bounds__(NT) void k_ifftx(Batch B)
{
    constexpr int T = fft_threads<N>();
    constexpr int LP = NT / T;
    __shared__ double2 buf[LP * N];
    __shared__ double2 tw[N];
    const Desc& D = *B.d[blockIdx.y];
    const int tid = threadIdx.x;
    for (int n = tid; n < N; n += NT) tw[n] = gload2((gptr<const double2>)D.twx + n);
    const gptr<const double2> spec = (gptr<const double2>)D.spec;
    const gptr<double> p = (gptr<double>)D.p;
    const int nlines = D.ny * D.nz;
    const int npairs = (nlines + 1) >> 1;
    const int pair0 = blockIdx.x * LP;
    const int sh = D.sh;
    // Hermitian extension of two half spectra into one complex line a + i b, at the inputs of the
    // thread's first butterflies
    const int lp = tid / T, t = tid - (tid / T) * T;
    const int pair = pair0 + lp;
    const bool active = lp < LP && pair < npairs;
    const int la = active ? 2 * pair : 0;
    const bool two = active && la + 1 < nlines;
    const gptr<const double2> sa = spec + (long long)la * sh, sb = spec + (long long)(two ? la + 1 : la) * sh;
    constexpr int R0 = fft_radix<N, false>(0), NB = N / R0, MB = fft_per_thread<N, T, R0>();
    double2 v[MB][R0];
#pragma unroll
    for (int m = 0; m < MB; ++m) {
        const int j = t + m * T < NB ? t + m * T : 0;
        double2 av[R0], bv[R0];
#pragma unroll
        for (int r = 0; r < R0; ++r) {
            const int n = j + r * NB, k = n <= N / 2 ? n : N - n;
            av[r] = gload2(sa + k);
            bv[r] = gload2(sb + k);
        }
#pragma unroll
        for (int r = 0; r < R0; ++r) {
            double2 a = av[r], b = two ? bv[r] : make_double2(0.0, 0.0);
            if (j + r * NB > N / 2) { a = cconj(a); b = cconj(b); }
            v[m][r] = make_double2(a.x - b.y, -(a.y + b.x));        // conjugated: inverse transform
        }
    }
    // walls: zero-mean gauge (the mean of the Neumann solution, from the tridiagonal solve)
    const double pm = D.walls ? ((gptr<const double>)D.gauge)[0] : 0.0;
    const gptr<double> pa = p + (long long)la * N;
    fft_from<N, T, false, 0, 1, true>(v, buf + (lp < LP ? lp : 0) * N, 1, t, active, tw, [&](int n, double2 x, int, int) {
        pa[n] = x.x - pm;
        if (two) pa[N + n] = -x.y - pm;
    });
}

// ---------------------------------------------------------------------------------------------
// velocity correction u = u* - (dt/rho) G_h p; copy of u* to u
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_correct(Batch B)
{
    const Desc& D = *B.d[blockIdx.y];
    const int nx = D.nx, ny = D.ny, nz = D.nz;
    // consecutive blocks on one XCD (the hardware deals blocks round-robin over the eight XCDs),
    // so the rows j + 1 and the plane k + 1 whose p this block reads are read by blocks of the
    // same XCD's L2
    const int nb = gridDim.x;
    int bid = blockIdx.x;
    if ((nb & 7) == 0) bid = (bid & 7) * (nb >> 3) + (bid >> 3);
    const long long q = (long long)bid * 256 + threadIdx.x;
    if (q >= D.ncell) return;
    const int i = (int)(q % nx);
    const long long r = q / nx;
    const int j = (int)(r % ny), k = (int)(r / ny);
    const double c = B.dt[blockIdx.y] * D.inv_rho;
    const gptr<const double> p = (gptr<const double>)D.p;
    const bool from_u = (B.state[blockIdx.y] & ST_FROM_U) != 0;      // in place, cell by cell
    const gptr<const double> us = (gptr<const double>)(from_u ? D.u : D.us), vs = (gptr<const double>)(from_u ? D.v : D.vs),
                             ws = (gptr<const double>)(from_u ? D.w : D.ws);
    const gptr<double> u = (gptr<double>)D.u, v = (gptr<double>)D.v, w = (gptr<double>)D.w;
    const double p0 = p[q];
    const double px = p[q - i + (i + 1 == nx ? 0 : i + 1)];
    const long long sxy = (long long)nx * ny;
    const double pz = p[k + 1 == nz ? q - (long long)(nz - 1) * sxy : q + sxy];
    u[q] = us[q] - c * (px - p0) * D.idx;
    w[q] = ws[q] - c * (pz - p0) * D.idz;
    if (j + 1 == ny) {
        v[q] = D.walls ? 0.0 : vs[q] - c * (p[q - (long long)(ny - 1) * nx] - p0) * D.idy;
    } else {
        v[q] = vs[q] - c * (p[q + nx] - p0) * D.idy;
    }
}

__global__ __launch_bounds__(256) void k_copy_ustar(Batch B)
{
    const Desc& D = *B.d[blockIdx.y];
    const long long ncell = D.ncell;
    const gptr<double> u = (gptr<double>)D.u, v = (gptr<double>)D.v, w = (gptr<double>)D.w;
    const gptr<const double> us = (gptr<const double>)D.us, vs = (gptr<const double>)D.vs, ws = (gptr<const double>)D.ws;
    const long long q = (long long)blockIdx.x * 256 + threadIdx.x;
    if (q >= ncell) return;
    const double a = us[q], b = vs[q], c = ws[q];
    u[q] = a; v[q] = b; w[q] = c;
}

}  // namespace

bool fft_size_supported(int n)
{
    switch (n) {
    case 8: case 12: case 16: case 24: case 32: case 48: case 64: case 96: case 128: case 192:
    case 256: case 384: case 512:
    case 10: case 20: case 30: case 40: case 60: case 80: case 120: case 160: case 240: case 320:
    case 480:
        return true;
    default:
        return false;
    }
}

#define EVP_FFT_SWITCH(n, CALL)                                                                  \
    switch (n) {                                                                                 \
    case 8: CALL(8); break;                                                                      \
    case 12: CALL(12); break;                                                                    \
    case 16: CALL(16); break;                                                                    \
    case 24: CALL(24); break;                                                                    \
    case 32: CALL(32); break;                                                                    \
    case 48: CALL(48); break;                                                                    \
    case 64: CALL(64); break;                                                                    \
    case 96: CALL(96); break;                                                                    \
    case 128: CALL(128); break;                                                                  \
    case 192: CALL(192); break;                                                                  \
    case 256: CALL(256); break;                                                                  \
    case 384: CALL(384); break;                                                                  \
    case 512: CALL(512); break;                                                                  \
    case 10: CALL(10); break;                                                                    \
    case 20: CALL(20); break;                                                                    \
    case 30: CALL(30); break;                                                                    \
    case 40: CALL(40); break;                                                                    \
    case 60: CALL(60); break;                                                                    \
    case 80: CALL(80); break;                                                                    \
    case 120: CALL(120); break;                                                                  \
    case 160: CALL(160); break;                                                                  \
    case 240: CALL(240); break;                                                                  \
    case 320: CALL(320); break;                                                                  \
    case 480: CALL(480); break;                                                                  \
    default: return hipErrorInvalidValue;                                                        \
    }

hipError_t launch_div_fftx(const Batch& b, int nx, int ny, int nz, hipStream_t s)
{
    const int npairs = (ny * nz + 1) / 2;
#define CALL(N)                                                                                  \
    {                                                                                            \
        constexpr int LP = NT / fft_threads<N>();                                                \
        dim3 grid((npairs + LP - 1) / LP, b.count);                                              \
        hipLaunchKernelGGL(k_div_fftx<N>, grid, dim3(NT), 0, s, b);                              \
    }
    EVP_FFT_SWITCH(nx, CALL)
#undef CALL
    return hipGetLastError();
}

hipError_t launch_ifftx(const Batch& b, int nx, int ny, int nz, hipStream_t s)
{
    const int npairs = (ny * nz + 1) / 2;
#define CALL(N)                                                                                  \
    {                                                                                            \
        constexpr int LP = NT / fft_threads<N>();                                                \
        dim3 grid((npairs + LP - 1) / LP, b.count);                                              \
        hipLaunchKernelGGL(k_ifftx<N>, grid, dim3(NT), 0, s, b);                                 \
    }
    EVP_FFT_SWITCH(nx, CALL)
#undef CALL
    return hipGetLastError();
}

// sides of the square planes that the fused kernels are built for
#define EVP_PLANE_LENGTHS                                                                        \
    CALL(8) CALL(10) CALL(12) CALL(16) CALL(20) CALL(24) CALL(30) CALL(32) CALL(40) CALL(48)     \
    CALL(60) CALL(64) CALL(96) CALL(128)

bool plane_transforms(int nx, int ny, int nz, int count)
{
    // One block per z plane.  Up to 64^2 a plane's block takes little longer than the blocks of the
    // separate passes, and two launches fewer count: a step of one 32^3 grid 39 -> 28 us, 48^3 49 -> 41.5,
    // 64^3 59 -> 56; a projection of 12^3 27.5 -> 16, 30^3 35 -> 21.5, 60^3 39 -> 32.  Above, one block per CU
    // and as many planes as the chip has CUs are needed: one 96^3 grid 121 us a step separately and 132
    // fused, 128^3 237 and 254; with at least 256 planes the fused passes save 2-11 % of the step
    // (batches of 96^3 and 128^3 grids).
    switch (nx == ny ? nx : 0) {
#define CALL(N) case N: return N <= 64 || (long long)nz * count >= 256;
    EVP_PLANE_LENGTHS
#undef CALL
    default: return false;
    }
}

hipError_t launch_div_fftxy(const Batch& b, int n, int nz, hipStream_t s)
{
    dim3 grid(nz, b.count);
    switch (n) {
#define CALL(N) case N: hipLaunchKernelGGL(k_div_fftxy<N>, grid, dim3(plane_block<N>()), 0, s, b); break;
    EVP_PLANE_LENGTHS
#undef CALL
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_ifftxy(const Batch& b, int n, int nz, hipStream_t s)
{
    dim3 grid(nz, b.count);
    switch (n) {
#define CALL(N) case N: hipLaunchKernelGGL(k_ifftxy<N>, grid, dim3(plane_block<N>()), 0, s, b); break;
    EVP_PLANE_LENGTHS
#undef CALL
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_fft_strided(const Batch& b, int nx, int ny, int nz, int axis, bool inverse,
                              hipStream_t s)
{
    const int nh = nx / 2 + 1;
    const int ntk = (nh + TK - 1) / TK;
    const int n = axis == 1 ? ny : nz;
    const int other = axis == 1 ? nz : ny;
#define CALL(N)                                                                                  \
    {                                                                                            \
        dim3 grid((ntk * other + strided_tiles<N>() - 1) / strided_tiles<N>(), b.count);         \
        if (inverse) hipLaunchKernelGGL((k_fft_strided<N, true>), grid, dim3(strided_block<N>()), 0, s, b, axis); \
        else hipLaunchKernelGGL((k_fft_strided<N, false>), grid, dim3(strided_block<N>()), 0, s, b, axis); \
    }
    EVP_FFT_SWITCH(n, CALL)
#undef CALL
    return hipGetLastError();
}

hipError_t launch_solve_periodic(const Batch& b, int nx, int ny, int nz, hipStream_t s)
{
    const int nh = nx / 2 + 1;
    const int ntk = (nh + TK - 1) / TK;
#define CALL(N)                                                                                  \
    {                                                                                            \
        dim3 grid((ntk * ny + strided_tiles<N>() - 1) / strided_tiles<N>(), b.count);            \
        hipLaunchKernelGGL(k_solve_periodic<N>, grid, dim3(strided_block<N>()), 0, s, b);        \
    }
    EVP_FFT_SWITCH(nz, CALL)
#undef CALL
    return hipGetLastError();
}

hipError_t launch_thomas(const Batch& b, int nx, int ny, int nz, hipStream_t s)
{
    const int cols = (int)((nx / 2 + 1 + 7) / 8 * 8) * nz;   // padded rows (Desc::sh)
    const int nseg = (ny + TS_L - 1) / TS_L;
    if (nseg <= 16) {
        dim3 grid((cols + 15) / 16, b.count);
        hipLaunchKernelGGL((k_thomas_seg<16, 16>), grid, dim3(16 * nseg), 0, s, b);
    } else {
        dim3 grid((cols + 7) / 8, b.count);
        hipLaunchKernelGGL((k_thomas_seg<8, 64>), grid, dim3(8 * nseg), 0, s, b);
    }
    return hipGetLastError();
}

hipError_t launch_correct(const Batch& b, int nx, int ny, int nz, hipStream_t s)
{
    const long long n = (long long)nx * ny * nz;
    dim3 grid((unsigned)((n + 255) / 256), b.count);
    hipLaunchKernelGGL(k_correct, grid, dim3(256), 0, s, b);
    return hipGetLastError();
}

hipError_t launch_copy_ustar(const Batch& b, int nx, int ny, int nz, hipStream_t s)
{
    const long long n = (long long)nx * ny * nz;
    dim3 grid((unsigned)((n + 255) / 256), b.count);
    hipLaunchKernelGGL(k_copy_ustar, grid, dim3(256), 0, s, b);
    return hipGetLastError();
}

}  // namespace evp
