// Predictor of the Adams-Bashforth step (Sec. 3.2.2, Eqs. (rt), (ab2tau), (ru), (ab2)) or of
// one Runge-Kutta substep (Sec. 3.3.1), periodic or between walls, with asynchronously staged
// planes, in FP64 and in the mixed form (stresses, histories and arithmetic FP32, velocities FP64).
//
// A block owns a TX x TY column of cells and marches along z.  Two threads share a cell: half 0 of
// the block advances B_xx, B_xy, B_xz and the x-momentum, half 1 B_yy, B_yz, B_zz and the y- and
// z-momentum, so that a thread's z window is three components and four FP64 waves fit a SIMD (128
// registers) and six mixed ones.  Per plane k:
//   top     the halo of plane k+1 of B - I and the velocities of plane k+1 start on their way from
//           memory straight into LDS (global_load_lds, 16 bytes a lane, no registers), then the
//           results of plane k-1 are stored; the thread's own cell of plane k+1 goes to LDS from its
//           register window
//   first   closure and the 18 upwind derivatives of plane k, from the plane's LDS buffer and the
//           window; the requests and the stores above are in flight meanwhile
//   middle  wait for the requests only (the stores were issued after them), barrier; beside a wall
//           the ghost rows are extrapolated in LDS (barrier); plane k+4 of the window and the cell's
//           history are asked for
//   second  velocity gradient, upper-convected terms, momentum (it needs plane k+1 beside plane k)
//
// In the mixed form the velocities of plane k+1 arrive in FP64 and the lanes that asked for them round
// them into the ring before the barrier of the middle; the cell's own FP64 velocity is kept from there
// for the update of the plane after.
//
// What bounds it: in FP64 at 512x256x256 the vector ALU (1.4k instructions per cell and plane, busy 0.6 of
// the cycles at the 2.1 GHz the chip holds under this load) and memory (12.3 GB a launch, 4.9 TB/s, a plain
// copy's rate) are about equal, and neither hides fully behind the other.  The mixed form is bound by
// the vector ALU (1.4k instructions, FP32 runs at the rate of FP64 here; busy all the time).  Against the synchronously
// staged form before it (one thread per cell, FP64: two waves per SIMD and three exposed memory round
// trips a plane; mixed: four waves, the rows beside a wall in a kernel of their own on a second stream):
// FP64 Saramito 2970 -> 2510 us at 512x256x256, 457 -> 309 at 256x128x128 (a Runge-Kutta substep), 180 -> 154
// at 128^3, 32 -> 12 at 32^3; mixed Saramito 1700 -> 1454 at 512x256x256, 116 -> 108 at 128^3, 29 -> 11 at
// 32^3, FENE-P 291 -> 239 at 256x128x128.
#pragma once

#include <cmath>

#include "evp_internal.h"
#include "weno.h"

namespace evp {

namespace {

// A tile of TX x TY cells; two threads per cell.
// W: values of B that a lane stages at a time (16 bytes, or one value where rows are not aligned to 16)
template <int TX, int TY, int W> struct Tile {
    static constexpr int NC = TX * TY, NT = 2 * NC, NW = NT / 64;     // cells, threads, waves
    // B plane: 3-cell cross halo, 4 columns left and right so that groups of W are aligned
    static constexpr int BR = TY + 6, BP = TX + 8;
    // velocity plane: 1-cell ring, 2 columns left and right
    static constexpr int VR = TY + 2, VP = TX + 4;
    static constexpr int NB = BR * BP / W;              // groups of a B plane
    static constexpr int PB = (NB + NC - 1) / NC;       // groups per thread of a half
    static constexpr int NV = VR * VP / 2;              // pairs of a velocity plane
    static constexpr int SEG = (NV + 63) / 64;          // wave loads per velocity plane
    static_assert(3 * SEG <= 2 * NW, "at most two velocity loads per wave");
};

// Between z-planes: T is the type of the stresses (B, RT, RU) and of the arithmetic.
template <typename T, int TX, int TY, bool FENE> struct __align__(16) SmemA {
    using TL = Tile<TX, TY, 1>;
    static constexpr bool MIXED = sizeof(T) == 4;
    T B[2][6][TL::BR][TL::BP];          // B - I of planes k and k+1
    T V[3][3][TL::VR][TL::VP];          // u, v, w of planes k-1, k, k+1
    double W[MIXED ? 3 : 1][MIXED ? TL::VR : 1][MIXED ? TL::VP : 1];   // u, v, w of plane k+1 in FP64 (mixed form)
    T F[FENE ? 2 : 1][FENE ? TL::VR : 1][FENE ? TL::VP : 1];   // FENE-P factor F
};

__device__ __forceinline__ int modp(int i, int n)
{
    int r = i % n;
    return r < 0 ? r + n : r;
}

// The descriptor in the constant address space: its fields come by scalar loads.  again() hides
// where the pointer comes from, so that a stage of the loop loads its own constants (scalar cache)
// instead of holding every stage's in registers along the march.
typedef const __attribute__((address_space(4))) Desc CDesc;
__device__ __forceinline__ const CDesc& again(const CDesc* p)
{
    __asm__ volatile("" : "+s"(p));
    return *p;
}
template <typename T> __device__ __forceinline__ const __attribute__((address_space(4))) StageConst<T>& constants(const CDesc& C)
{
    if constexpr (sizeof(T) == 4) return C.kf;
    else return C.kd;
}
#define EVP_STAGE_CONSTANTS                                                                        \
    const auto& C = constants<T>(again(Dp));                                                       \
    [[maybe_unused]] const T idx = C.idx, idy = C.idy, idz = C.idz, qx = C.qx, qy = C.qy, qz = C.qz; \
    [[maybe_unused]] const T idx2 = C.idx2, idy2 = C.idy2, idz2 = C.idz2, e2x = C.e2x, e2y = C.e2y, e2z = C.e2z; \
    [[maybe_unused]] const T G = C.G, L2 = C.L2, il = C.inv_lam, ms = C.mu_s, irho = C.inv_rho
// a wave-uniform pointer, in scalar registers
__device__ __forceinline__ gptr<const double> uniform(gptr<const double> p)
{
    const unsigned long long a = (unsigned long long)p;
    const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)a);
    const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(a >> 32));
    return (gptr<const double>)((unsigned long long)hi << 32 | lo);
}
// BYTES per active lane from base + off (per lane) to the LDS bytes lds + BYTES lane.  Counted by
// vmcnt; arrive() is the only wait for it.  The wait states cover a base in scalar
// registers just written by the vector ALU and the use of m0.
template <int BYTES, typename T>
__device__ __forceinline__ void load_lds(unsigned lds, gptr<const T> base, unsigned off)
{
    static_assert(BYTES == 16 || BYTES == 4, "the widths below");
    if constexpr (BYTES == 16)
        __asm__ volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tglobal_load_lds_dwordx4 %1, %2"
                         ::"s"(lds), "v"(off), "s"(base) : "memory", "m0");
    else
        __asm__ volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tglobal_load_lds_dword %1, %2"
                         ::"s"(lds), "v"(off), "s"(base) : "memory", "m0");
}
// The requests of this wave have arrived.  vmcnt counts a wave's loads and stores in order; LATER of
// them may still be in flight (issued after the requests).
template <int LATER>
__device__ __forceinline__ void arrive()
{
    static_assert(LATER == 0 || LATER == 8 || LATER == 10, "the waits below");
    if constexpr (LATER == 0) __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");
    else if constexpr (LATER == 8) __asm__ volatile("s_waitcnt vmcnt(8)" ::: "memory");
    else __asm__ volatile("s_waitcnt vmcnt(10)" ::: "memory");
}
// block barrier for LDS accesses only: loads and stores to memory stay in flight
__device__ __forceinline__ void lds_barrier()
{
    __asm__ volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// The cell's own values: raw buffer accesses at a wave-uniform plane base (descriptor in scalar
// registers) plus the cell's byte offset in a plane, so that an access takes no vector arithmetic.
// STREAM: data only this cell touches (history, results), non-temporal, so L2 keeps the halo lines.
// A load at or past `bytes` touches no memory and gives 0.
constexpr int kRawBufferWord3 = 0x00020000, kNonTemporal = 2, kAllBytes = 0x7fffffff;
template <bool STREAM, typename T>
__device__ __forceinline__ T ld_cell(gptr<const T> base, unsigned off, int bytes = kAllBytes)
{
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((EVP_GLOBAL void*)base, (short)0, bytes, kRawBufferWord3);
    if constexpr (sizeof(T) == 4) return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, STREAM ? kNonTemporal : 0));
    else return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, STREAM ? kNonTemporal : 0));
}
template <typename T>
__device__ __forceinline__ void st_stream(gptr<T> base, unsigned off, T v)
{
    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((EVP_GLOBAL void*)base, (short)0, kAllBytes, kRawBufferWord3);
    if constexpr (sizeof(T) == 4) __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, off, 0, kNonTemporal);
    else __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, off, 0, kNonTemporal);
}

// upwind derivative (times h) from six values in upwind order (mirrored for a negative velocity)
template <bool HOUC, typename T>
__device__ __forceinline__ T upwind(T g0, T g1, T g2, T g3, T g4, T g5, T eps2)
{
    const T v1 = g1 - g0, v2 = g2 - g1, v3 = g3 - g2, v4 = g4 - g3, v5 = g5 - g4;
    if constexpr (HOUC)
        return (T)(2.0 / 60.0) * v1 - (T)(13.0 / 60.0) * v2 + (T)(47.0 / 60.0) * v3 + (T)(27.0 / 60.0) * v4 - (T)(3.0 / 60.0) * v5;
    else
        return weno5u<T>(v1, v2, v3, v4, v5, eps2);
}

// The march of one half of the block: half 0 advances B_xx, B_xy, B_xz and the x-momentum, half 1
// B_yy, B_yz, B_zz and the y- and z-momentum of the same cells.
template <typename T, int W, int HALF, int TX, int TY, int MODEL, bool RK3, bool HOUC>
__device__ __forceinline__ void march(SmemA<T, TX, TY, MODEL == EVP_FENE_P>& S, const Batch& B, int freeze, int kc)
{
    using TL = Tile<TX, TY, W>;
    constexpr bool MIXED = sizeof(T) == 4;
    constexpr bool fene = MODEL == EVP_FENE_P, sara = MODEL == EVP_SARAMITO, neo = MODEL == EVP_NEO_HOOKEAN;
    constexpr int C0 = 3 * HALF;                        // first component of this half
    constexpr int NF = HALF == 0 ? 1 : 2;               // momentum faces of this half
    constexpr int kResults = 6 + 2 * NF;
    const int b = blockIdx.y;
    // the descriptor in the constant address space: its fields come by scalar loads anywhere below
    const CDesc& D = *(const CDesc*)B.d[b];
    const CDesc* const Dp = &D;
    const int nx = D.nx, ny = D.ny, nz = D.nz;
    const int sxy = nx * ny;
    const int ps = (int)D.ps;
    const bool walls = D.walls != 0;
    const int ntx = (nx + TX - 1) / TX, nty = (ny + TY - 1) / TY;
    const int nblk = gridDim.x;
    int bid = blockIdx.x;
    if ((nblk & 7) == 0) bid = (bid & 7) * (nblk >> 3) + (bid >> 3);     // XCD-contiguous tiles
    const int i0 = (bid % ntx) * TX, j0 = ((bid / ntx) % nty) * TY, k0 = (bid / (ntx * nty)) * kc;
    const int k1 = min(k0 + kc, nz);
    const int t = threadIdx.x & (TL::NC - 1), tx = t % TX, ty = t / TX;
    const int i = i0 + tx, j = j0 + ty;
    const bool valid = i < nx && j < ny;
    const int oij = min(j, ny - 1) * nx + min(i, nx - 1);
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = t & 63;
    const int hwave = wave & (TL::NC / 64 - 1);          // wave of this half
    const unsigned o8 = (unsigned)oij * 8u, oT = (unsigned)oij * (unsigned)sizeof(T);

    const int st = B.state[b];
    // fields of this half: its components of B and RT, its rows of RU, its predicted velocities
    const gptr<const T> Bin = (gptr<const T>)D.Bt[st & 1] + (long long)C0 * ps;
    const bool euler = (st & ST_EULER) != 0;
    const T dt = (T)B.dt[b];
    // history weights: AB2 (3/2, -1/2; Euler start 1, 0) or the substep's (zeta, xi)
    const T c1 = RK3 ? (T)B.rk[0] : (euler ? (T)1 : (T)1.5);
    const T c2 = euler ? (T)0 : (RK3 ? (T)B.rk[1] : (T)-0.5);
    // ---- staging maps, fixed along the march ----
    // B planes of this half's components: thread t stages groups t + NC q of the padded plane
    // (row-major, W values each), unless the group lies in the block's own cells (written from the window), outside
    // the cross, or beyond a wall (extrapolated later).  nx and i0 are multiples of W, so a group never
    // straddles the wrap.
    unsigned boff[TL::PB];
    bool bload[TL::PB];
#pragma unroll
    for (int q = 0; q < TL::PB; ++q) {
        const int e = t + q * TL::NC;
        const int r = e / (TL::BP / W) - 3, c = W * (e % (TL::BP / W)) - 4;
        const int jj = j0 + r;
        const bool inrow = r >= 0 && r < TY;
        const bool cross = inrow || (c >= 0 && c < TX) || ((r == -1 || r == TY) && ((c <= -1 && c + W > -1) || c == TX));
        const bool own = inrow && jj < ny && c >= 0 && c < TX && i0 + c < nx;
        bload[q] = e < TL::NB && cross && !own && !(walls && (jj < 0 || jj >= ny));
        boff[q] = (unsigned)(modp(jj, ny) * nx + modp(i0 + c, nx)) * (unsigned)sizeof(T);
    }
    const unsigned lds0 = (unsigned)(unsigned long long)(__attribute__((address_space(3))) char*)(&S.B[0][0][0][0]);
    const unsigned ldsv = (unsigned)(unsigned long long)(__attribute__((address_space(3))) char*)(MIXED ? (void*)&S.W[0][0][0] : (void*)&S.V[0][0][0][0]);
    constexpr unsigned BPL = TL::BR * TL::BP * sizeof(T), VPL = TL::VR * TL::VP * 8u;
    auto stage_b = [&](int kk, int buf) {
#pragma unroll
        for (int q = 0; q < TL::PB; ++q) {
            if (!bload[q]) continue;
#pragma unroll
            for (int cc = 0; cc < 3; ++cc)
                load_lds<W * (int)sizeof(T)>(lds0 + (unsigned)(buf * 6 + C0 + cc) * BPL + (unsigned)(hwave + q * (TL::NC / 64)) * (64u * W * (unsigned)sizeof(T)),
                                             Bin + (kk * sxy + cc * ps), boff[q]);
        }
    };
    // velocity planes: wave load q = wave + NW m covers pairs 64 (q % SEG) + lane of component q / SEG; in
    // the mixed form they arrive in S.W and the lane that asked for a pair then rounds it into the ring
    unsigned voff[2];
    bool vload[2];
    gptr<const double> vsrc[2];
#pragma unroll
    for (int m = 0; m < 2; ++m) {
        const int q = wave + TL::NW * m, e = (q % TL::SEG) * 64 + lane;
        const int jj = j0 + e / (TL::VP / 2) - 1, ii = i0 + 2 * (e % (TL::VP / 2)) - 2;
        vload[m] = q < 3 * TL::SEG && e < TL::NV && !(walls && (jj < 0 || jj >= ny));
        voff[m] = (unsigned)(modp(jj, ny) * nx + modp(ii, nx)) * 8u;
        vsrc[m] = uniform((gptr<const double>)(q / TL::SEG == 0 ? D.u : q / TL::SEG == 1 ? D.v : D.w));
    }
    auto stage_v = [&](int kk, int slot) {
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            const int q = wave + TL::NW * m, comp = q / TL::SEG;
            if (vload[m])
                load_lds<16>(ldsv + (unsigned)((MIXED ? 0 : slot * 3) + comp) * VPL + (unsigned)(q % TL::SEG) * 1024u,
                             vsrc[m] + kk * sxy, voff[m]);
        }
    };
    auto round_v = [&](int slot) {
        if constexpr (MIXED) {
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                const int q = wave + TL::NW * m, comp = q / TL::SEG, e = (q % TL::SEG) * 64 + lane;
                if (vload[m]) {
                    const double2 x = ((const double2*)&S.W[comp][0][0])[e];
                    ((float2*)&S.V[slot][comp][0][0])[e] = make_float2((float)x.x, (float)x.y);
                }
            }
        }
    };
    const int rB = ty + 3, cB = tx + 4, rV = ty + 1, cV = tx + 2;
    auto stage_own = [&](int buf, const T* own) {
        if (valid) {
#pragma unroll
            for (int cc = 0; cc < 3; ++cc) S.B[buf][C0 + cc][rB][cB] = own[cc];
        }
    };
    // beside a wall: ghost rows of the plane in B buffer buf (this half's components) and velocity
    // slot (half 0; B extrapolated linearly, u and w reflected about the wall velocity, v = 0), from
    // rows already in LDS
    const bool wall_tile = walls && (j0 < 3 || j0 + TY + 2 >= ny);
    auto ghosts = [&](int buf, int slot, bool velocities) {
        for (int e = t; e < 6 * TL::BP; e += TL::NC) {
            const int g = e / TL::BP, c = e % TL::BP;       // ghost row 0..2 below, 3..5 above
            const int m = g < 3 ? g + 1 : g - 2;            // distance beyond the wall row
            const int ra = (g < 3 ? 0 : ny - 1) - j0 + 3, rb = g < 3 ? ra + 1 : ra - 1;
            const int r = g < 3 ? ra - m : ra + m;
            if (r < 0 || r >= TL::BR || ra < 0 || ra >= TL::BR || rb < 0 || rb >= TL::BR) continue;
#pragma unroll
            for (int cc = 0; cc < 3; ++cc)
                S.B[buf][C0 + cc][r][c] = (T)(1 + m) * S.B[buf][C0 + cc][ra][c] - (T)m * S.B[buf][C0 + cc][rb][c];
        }
        if (HALF == 0 && velocities && t < 2 * TL::VP) {
            const bool bot = t < TL::VP;
            const int cv = bot ? t : t - TL::VP;
            const int ra = (bot ? 0 : ny - 1) - j0 + 1, r = bot ? ra - 1 : ra + 1;
            if (r >= 0 && r < TL::VR && ra >= 0 && ra < TL::VR) {
                double uu, ww;
                if constexpr (MIXED) { uu = S.W[0][ra][cv]; ww = S.W[2][ra][cv]; }
                else { uu = S.V[slot][0][ra][cv]; ww = S.V[slot][2][ra][cv]; }
                S.V[slot][0][r][cv] = (T)(2.0 * (bot ? D.u_bot : D.u_top) - uu);
                S.V[slot][1][r][cv] = (T)0;
                S.V[slot][2][r][cv] = (T)(2.0 * (bot ? D.w_bot : D.w_top) - ww);
            }
        }
    };
    // FENE-P: F on the block's cells (half 0) and the ring around them (half 1)
    auto factor = [&](int buf, int r, int c) {
        const T L2 = constants<T>(again(Dp)).L2;
        return L2 / (L2 - (S.B[buf][0][r][c] + S.B[buf][3][r][c] + S.B[buf][5][r][c] + (T)3));
    };
    int ring_r = -1, ring_c = 0;
    if (fene && HALF == 1 && t < 2 * (TX + 2) + 2 * TY) {
        if (t < 2 * (TX + 2)) { ring_r = t < TX + 2 ? -1 : TY; ring_c = t % (TX + 2) - 1; }
        else { const int u = t - 2 * (TX + 2); ring_r = u / 2; ring_c = (u & 1) ? TX : -1; }
        ring_r += 1;
    }
    auto stage_f = [&](int buf, int slot) {
        if (HALF == 0) S.F[slot][rV][cV] = factor(buf, rB, cB);
        else if (ring_r >= 0) S.F[slot][ring_r][ring_c + 2] = factor(buf, ring_r + 2, ring_c + 4);
    };

    // forcing on this thread's x-face row
    T fx = (T)0;
    if (HALF == 0) {
        if (D.force_kind == EVP_FORCE_CONST_X) fx = (T)D.force_amp;
        else if (D.force_kind == EVP_FORCE_SIN_X_OF_Y) fx = (T)(D.force_amp * sin(D.force_ky * (D.y0 + (min(j, ny - 1) + 0.5) * D.dy)));
    }

    // ---- prologue: window, B of planes k0-1 (buffer 1) and k0 (buffer 0), velocities of planes
    // k0-1 and k0 ----
    const int km = modp(k0 - 1, nz);
    stage_b(km, 1);
    stage_b(k0, 0);
    if constexpr (!MIXED) stage_v(km, (k0 + 2) % 3);
    stage_v(k0, k0 % 3);
    if constexpr (MIXED) {
        // S.W holds one plane: plane k0-1 comes through registers, ghost rows with it
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            const int q = wave + TL::NW * m, comp = q / TL::SEG, e = (q % TL::SEG) * 64 + lane;
            if (q < 3 * TL::SEG && e < TL::NV) {
                const int jj = j0 + e / (TL::VP / 2) - 1, ii = i0 + 2 * (e % (TL::VP / 2)) - 2;
                const bool bot = walls && jj < 0, top = walls && jj >= ny;
                const int js = bot ? min(-1 - jj, ny - 1) : top ? max(2 * ny - 1 - jj, 0) : modp(jj, ny);
                const gptr<const double> a = vsrc[m] + (km * sxy + js * nx + modp(ii, nx));
                double x = a[0], y = a[1];
                if (bot || top) {
                    const double twice = 2.0 * (comp == 0 ? (bot ? D.u_bot : D.u_top) : (bot ? D.w_bot : D.w_top));
                    x = comp == 1 ? 0.0 : twice - x;
                    y = comp == 1 ? 0.0 : twice - y;
                }
                ((float2*)&S.V[(k0 + 2) % 3][comp][0][0])[e] = make_float2((float)x, (float)y);
            }
        }
    }
    // register window of the thread's own cell: planes k-3..k-1 (wm) and k+1..k+3 (wp); plane k, and
    // plane k+1 from the top of its iteration on, are read from LDS
    T wm[3][3], wp[3][3];
    auto load_own = [&](int kk, T* o) {
        const gptr<const T> p = Bin + modp(kk, nz) * sxy;
#pragma unroll
        for (int cc = 0; cc < 3; ++cc) o[cc] = ld_cell<false, T>(p + cc * ps, oT);
    };
    {
        T w0[3];
        load_own(k0, w0);
#pragma unroll
        for (int m = 0; m < 3; ++m) {
            load_own(k0 - 3 + m, wm[m]);
            load_own(k0 + 1 + m, wp[m]);
        }
        stage_own(1, wm[2]);
        stage_own(0, w0);
    }
    // the grid's note that its history is zero: a plain load, and the only one, because another block clears
    // the note later in this launch (the high word of 0.0 or 1.0); it travels with the requests above
    int note = *(gptr<const volatile int>)((gptr<const int>)hist_zero(B.d[b]) + 1);
    arrive<0>();
    __asm__ volatile("" : "+v"(note));
    round_v(k0 % 3);
    // no history: zeros are taken, the histories' memory may hold anything
    const bool none = euler || __builtin_amdgcn_readfirstlane(note) != 0;
    const int hist_bytes = none ? 0 : kAllBytes;
    lds_barrier();
    // this launch writes the histories, so the note goes: at an Euler step, where no block reads it, at
    // once, otherwise when the last block has read it
    if (HALF == 0 && threadIdx.x == 0 && none) {
        if (euler) {
            if (blockIdx.x == 0) *(gptr<double>)hist_zero(B.d[b]) = 0.0;
        } else {
            const gptr<unsigned> readers = (gptr<unsigned>)hist_readers(B.d[b]);
            if (__hip_atomic_fetch_add(readers, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1) {
                *readers = 0u;
                *(gptr<double>)hist_zero(B.d[b]) = 0.0;
            }
        }
    }
    if (wall_tile) {
        if constexpr (!MIXED) ghosts(1, (k0 + 2) % 3, true);
        else ghosts(1, 0, false);
        ghosts(0, k0 % 3, true);
        lds_barrier();
    }
    // the cell's velocities of plane k in FP64 (mixed form): u (half 0) or v and w
    double vd[NF];
    auto keep_v = [&]() {
        if constexpr (MIXED) {
#pragma unroll
            for (int f = 0; f < NF; ++f) vd[f] = S.W[HALF + f][rV][cV];
        }
    };
    keep_v();
    // tau_xz(i) + tau_xz(i+1) (half 0) or tau_yz(j) + tau_yz(j+1) (half 1) of the plane below, over G
    // (the same operations as in the loop, so that a grid's numbers do not depend on its z-chunks)
    T sz;
    {
        constexpr int c = HALF == 0 ? 2 : 4, dj = HALF == 0 ? 0 : 1, di = 1 - dj;
        if constexpr (fene) sz = fma(factor(1, rB + dj, cB + di), S.B[1][c][rB + dj][cB + di], factor(1, rB, cB) * S.B[1][c][rB][cB]);
        else sz = S.B[1][c][rB][cB] + S.B[1][c][rB + dj][cB + di];
    }
    if constexpr (fene) stage_f(0, k0 & 1);
    lds_barrier();

    const T h = (T)0.5;
    const bool vwall = walls && j == ny - 1;
    // results of a plane: stored after the requests for the next plane, so that the wait for those
    // does not wait for the stores too
    T rb[3], rt[3], ru[NF];
    double rs[NF];
    auto store_results = [&](int kk) {
        const CDesc& C = again(Dp);
        const int kq = kk * sxy;
        const gptr<T> RU = (gptr<T>)C.RU + kq;
        if constexpr (HALF == 0) {
            st_stream((gptr<double>)C.us + kq, o8, rs[0]);
            st_stream(RU, oT, ru[0]);
        } else {
            st_stream((gptr<double>)C.vs + kq, o8, rs[0]);
            st_stream((gptr<double>)C.ws + kq, o8, rs[NF - 1]);
            st_stream(RU + ps, oT, ru[0]);
            st_stream(RU + 2 * ps, oT, ru[NF - 1]);
        }
        const gptr<T> Bout = (gptr<T>)C.Bt[(st & 1) ^ 1] + kq, RT = (gptr<T>)C.RT + kq;
#pragma unroll
        for (int cc = 0; cc < 3; ++cc) {
            st_stream(Bout + (C0 + cc) * ps, oT, rb[cc]);
            st_stream(RT + (C0 + cc) * ps, oT, rt[cc]);
        }
    };
    const bool wave_stores = __ballot(valid) != 0;

    for (int k = k0; k < k1; ++k) {
        const int cur = (k - k0) & 1, nxt = cur ^ 1;
        const int sm = (k + 2) % 3, s0 = k % 3, sp = (k + 1) % 3;
        const int kq = k * sxy;
        const int kp = k + 1 == nz ? 0 : k + 1;
        stage_b(kp, nxt);
        stage_v(kp, sp);
        stage_own(nxt, wp[0]);
        if (k > k0 && valid) store_results(k - 1);
#define VU(s, di, dj) S.V[s][0][rV + (dj)][cV + (di)]
#define VV(s, di, dj) S.V[s][1][rV + (dj)][cV + (di)]
#define VW(s, di, dj) S.V[s][2][rV + (dj)][cV + (di)]
        // ---- first part: closure, relaxation and advection (each fence bounds live ranges: its
        // operands are done before anything below is read) ----
        {
            EVP_STAGE_CONSTANTS;
            T bt[6];
#pragma unroll
            for (int cc = 0; cc < 6; ++cc) bt[cc] = S.B[cur][cc][rB][cB];
            T F = (T)1, a = (T)1;
            if (fene) {
                F = S.F[k & 1][rV][cV];
                a = C.a_fene;
            } else if (sara) {
                // in units of a power of two near G, so that no choice of units brings the squares near the
                // ends of the type's range (the yield factor is a ratio of stresses)
                const T g = C.G_unit, tyld = C.tau_y_unit;
                const T t3 = g * (bt[0] + bt[3] + bt[5]) * (T)(1.0 / 3.0);
                const T dxx = g * bt[0] - t3, dyy = g * bt[3] - t3, dzz = g * bt[5] - t3;
                const T txy = g * bt[1], txz = g * bt[2], tyz = g * bt[4];
                const T n2 = (T)0.5 * (dxx * dxx + dyy * dyy + dzz * dzz) + txy * txy + txz * txz + tyz * tyz;
                // 1 - tau_y / |tau_d| above the yield stress; rounding leaves it in [0, 1]
                F = n2 > tyld * tyld ? min(max((T)1 - tyld * fast_rsqrt(n2), (T)0), (T)1) : (tyld == (T)0 ? (T)1 : (T)0);
                a = F;
            } else if (neo) {
                F = (T)0;
                a = (T)0;
            }
#pragma unroll
            for (int cc = 0; cc < 3; ++cc) {
                const bool diag = C0 + cc == 0 || C0 + cc == 3 || C0 + cc == 5;
                rt[cc] = ((diag ? (a - F) : (T)0) - F * bt[C0 + cc]) * il;
            }
            __asm__ volatile("" ::"v"(rt[0]), "v"(rt[1]), "v"(rt[2]) : "memory");
        }
        const T* const bx = &S.B[cur][C0][rB][cB];
        // x and y stencils are read from LDS in upwind order: element m of the x stencil is column
        // cB + s (m - 3), of the y stencil row rB + s (m - 3), s = +1 for a non-negative velocity and -1
        // otherwise; the sign of the derivative comes with |velocity|
        {
            EVP_STAGE_CONSTANTS;
            const T uc = h * (VU(s0, 0, 0) + VU(s0, -1, 0)), auc = fabs(uc) * idx;
            const int sx = uc >= (T)0 ? 1 : -1;
#pragma unroll
            for (int cc = 0; cc < 3; ++cc) {
                const T* const pc = bx + cc * (TL::BR * TL::BP);
                rt[cc] -= auc * upwind<HOUC>(pc[-3 * sx], pc[-2 * sx], pc[-sx], pc[0], pc[sx], pc[2 * sx], e2x);
                __asm__ volatile("" ::"v"(rt[cc]) : "memory");
            }
        }
        {
            EVP_STAGE_CONSTANTS;
            const T vc = h * (VV(s0, 0, 0) + VV(s0, 0, -1)), avc = fabs(vc) * idy;
            const int sy = vc >= (T)0 ? TL::BP : -TL::BP;
#pragma unroll
            for (int cc = 0; cc < 3; ++cc) {
                const T* const pc = bx + cc * (TL::BR * TL::BP);
                rt[cc] -= avc * upwind<HOUC>(pc[-3 * sy], pc[-2 * sy], pc[-sy], pc[0], pc[sy], pc[2 * sy], e2y);
                __asm__ volatile("" ::"v"(rt[cc]) : "memory");
            }
        }
        // the z stencils come last: plane k+3 was asked for in the second part of plane k-1
        {
            EVP_STAGE_CONSTANTS;
            const T wc = h * (VW(s0, 0, 0) + VW(sm, 0, 0)), awc = fabs(wc) * idz;
            const bool up = wc >= (T)0;
#pragma unroll
            for (int cc = 0; cc < 3; ++cc) {
                const T n = S.B[nxt][C0 + cc][rB][cB], m3 = wm[0][cc], m2 = wm[1][cc], m1 = wm[2][cc], p2 = wp[1][cc], p3 = wp[2][cc];
                rt[cc] -= awc * upwind<HOUC>(up ? m3 : p3, up ? m2 : p2, up ? m1 : n, bx[cc * (TL::BR * TL::BP)], up ? n : m1, up ? p2 : m2, e2z);
                __asm__ volatile("" ::"v"(rt[cc]) : "memory");
            }
        }
        {
            EVP_STAGE_CONSTANTS;
            const T kap = C.kappa;
            // local artificial diffusion (Sec. 3.1): det B < 0, or tr B >= 0.95 L^2 (FENE-P)
            if (kap > (T)0) {
                T bt[6];
#pragma unroll
                for (int cc = 0; cc < 6; ++cc) bt[cc] = S.B[cur][cc][rB][cB];
                const T b0 = bt[0] + (T)1, b3 = bt[3] + (T)1, b5 = bt[5] + (T)1;
                const T det = b0 * (b3 * b5 - bt[4] * bt[4]) - bt[1] * (bt[1] * b5 - bt[4] * bt[2])
                                 + bt[2] * (bt[1] * bt[4] - b3 * bt[2]);
                if (det < (T)0 || (fene && b0 + b3 + b5 >= (T)0.95 * L2)) {
#pragma unroll
                    for (int cc = 0; cc < 3; ++cc) {
                        const int c = C0 + cc;
                        rt[cc] += kap * ((S.B[cur][c][rB][cB - 1] - (T)2 * bt[c] + S.B[cur][c][rB][cB + 1]) * idx2
                                         + (S.B[cur][c][rB - 1][cB] - (T)2 * bt[c] + S.B[cur][c][rB + 1][cB]) * idy2
                                         + (wm[2][cc] - (T)2 * bt[c] + S.B[nxt][c][rB][cB]) * idz2);
                    }
                }
            }
        }
        // ---- middle: plane k+1 is complete ----
        if (k > k0 && wave_stores) arrive<kResults>();
        else arrive<0>();
        round_v(sp);
        lds_barrier();
        if (wall_tile) {
            ghosts(nxt, sp, true);
            lds_barrier();
        }
        if constexpr (fene) {
            stage_f(nxt, (k + 1) & 1);
            lds_barrier();
        }
        // window: drop plane k-3, load plane k+4
#pragma unroll
        for (int cc = 0; cc < 3; ++cc) {
            wm[0][cc] = wm[1][cc];
            wm[1][cc] = wm[2][cc];
            wp[0][cc] = wp[1][cc];
            wp[1][cc] = wp[2][cc];
            // in place before the load below overwrites the registers of plane k+3
            __asm__ volatile("" : "+v"(wm[0][cc]), "+v"(wm[1][cc]), "+v"(wp[0][cc]), "+v"(wp[1][cc])::"memory");
        }
        load_own(k + 4, wp[2]);
        // the cell's history, consumed at the end of the plane
        T old[3], oru[NF];
        {
            const CDesc& C = again(Dp);
#pragma unroll
            for (int cc = 0; cc < 3; ++cc) old[cc] = ld_cell<true, T>((gptr<const T>)C.RT + (kq + (C0 + cc) * ps), oT, hist_bytes);
#pragma unroll
            for (int f = 0; f < NF; ++f) oru[f] = ld_cell<true, T>((gptr<const T>)C.RU + (kq + (HALF + f) * ps), oT, hist_bytes);
        }
        // ---- second part: upper-convected terms, momentum (every lane; only valid cells are
        // stored).  e, w, n, s, f, b: the +x, -x, +y, -y, +z, -z neighbours ----
        const int f0 = k & 1, f1 = (k + 1) & 1;
#define TAU(buf, ff, cc, di, dj) (fene ? (((cc) == 0 || (cc) == 3 || (cc) == 5) \
                                      ? fma(S.F[ff][rV + (dj)][cV + (di)], S.B[buf][cc][rB + (dj)][cB + (di)], S.F[ff][rV + (dj)][cV + (di)] - C.a_fene) \
                                      : S.F[ff][rV + (dj)][cV + (di)] * S.B[buf][cc][rB + (dj)][cB + (di)]) \
                                       : S.B[buf][cc][rB + (dj)][cB + (di)])
        // sum of an off-diagonal component of the cell and of its neighbour
#define TSUM(buf, ff, cc, di, dj) (fene ? fma(S.F[ff][rV + (dj)][cV + (di)], S.B[buf][cc][rB + (dj)][cB + (di)], S.F[ff][rV][cV] * S.B[buf][cc][rB][cB]) \
                                        : S.B[buf][cc][rB][cB] + S.B[buf][cc][rB + (dj)][cB + (di)])
        // stress over G of plane k (TK) and of plane k+1 (TP): F (B - I), and F - a on the FENE-P diagonal
        // (not F B - a: B itself in 32 bits has lost the digits of a small B - I)
#define TK(cc, di, dj) TAU(cur, f0, cc, di, dj)
#define TP(cc, di, dj) TAU(nxt, f1, cc, di, dj)
        T u0, v0, w0;
        {
            EVP_STAGE_CONSTANTS;
            T bt[6], L[3][3];
#pragma unroll
            for (int cc = 0; cc < 6; ++cc) bt[cc] = S.B[cur][cc][rB][cB];
            u0 = VU(s0, 0, 0);
            v0 = VV(s0, 0, 0);
            w0 = VW(s0, 0, 0);
            if constexpr (HALF == 0) {
                L[0][0] = (u0 - VU(s0, -1, 0)) * idx;
                L[0][1] = (VU(s0, 0, 1) + VU(s0, -1, 1) - VU(s0, 0, -1) - VU(s0, -1, -1)) * qy;
                L[0][2] = (VU(sp, 0, 0) + VU(sp, -1, 0) - VU(sm, 0, 0) - VU(sm, -1, 0)) * qz;
            }
            L[1][0] = (VV(s0, 1, 0) + VV(s0, 1, -1) - VV(s0, -1, 0) - VV(s0, -1, -1)) * qx;
            L[1][1] = (v0 - VV(s0, 0, -1)) * idy;
            L[1][2] = (VV(sp, 0, 0) + VV(sp, 0, -1) - VV(sm, 0, 0) - VV(sm, 0, -1)) * qz;
            L[2][0] = (VW(s0, 1, 0) + VW(sm, 1, 0) - VW(s0, -1, 0) - VW(sm, -1, 0)) * qx;
            L[2][1] = (VW(s0, 0, 1) + VW(sm, 0, 1) - VW(s0, 0, -1) - VW(sm, 0, -1)) * qy;
            L[2][2] = (w0 - VW(sm, 0, 0)) * idz;
            const int pa[6] = {0, 0, 0, 1, 1, 2}, pb[6] = {0, 1, 2, 1, 2, 2};
            const int cm[3][3] = {{0, 1, 2}, {1, 3, 4}, {2, 4, 5}};
#pragma unroll
            for (int cc = 0; cc < 3; ++cc) {
                const int p = pa[C0 + cc], rr = pb[C0 + cc];
                T ucv = L[p][rr] + L[rr][p];
#pragma unroll
                for (int m = 0; m < 3; ++m) ucv += L[p][m] * bt[cm[m][rr]] + bt[cm[p][m]] * L[rr][m];
                rt[cc] += ucv;
                wm[2][cc] = bt[C0 + cc];
            }
        }
        // (each fence bounds live ranges: its operands are done before anything below is read)
        __asm__ volatile("" ::"v"(rt[0]), "v"(rt[1]), "v"(rt[2]) : "memory");
        const T cal = RK3 ? (T)B.rk[2] : (T)0;
        // what the increments are added to: the velocity in FP64
#define U0 (MIXED ? vd[0] : (double)u0)
#define V0 (MIXED ? vd[0] : (double)v0)
#define W0 (MIXED ? vd[NF - 1] : (double)w0)
        if constexpr (HALF == 0) {
            // x-face (i+1/2, j, k)
            T ax, lx;
            {
                EVP_STAGE_CONSTANTS;
                const T ue = VU(s0, 1, 0), uw = VU(s0, -1, 0), un = VU(s0, 0, 1), us = VU(s0, 0, -1), uf = VU(sp, 0, 0), ub = VU(sm, 0, 0);
                // twice the face means; their products are divided by 4 h
                const T cR = u0 + ue, cL = uw + u0, vT = v0 + VV(s0, 1, 0), vB = VV(s0, 0, -1) + VV(s0, 1, -1);
                const T wF = w0 + VW(s0, 1, 0), wB = VW(sm, 0, 0) + VW(sm, 1, 0);
                ax = (cR * cR - cL * cL) * qx + (vT * (u0 + un) - vB * (us + u0)) * qy + (wF * (u0 + uf) - wB * (ub + u0)) * qz;
                lx = (ue - (T)2 * u0 + uw) * idx2 + (un - (T)2 * u0 + us) * idy2 + (uf - (T)2 * u0 + ub) * idz2;
            }
            __asm__ volatile("" ::"v"(ax), "v"(lx) : "memory");
            EVP_STAGE_CONSTANTS;
            const T zx = TSUM(cur, f0, 2, 1, 0), px = TSUM(nxt, f1, 2, 1, 0);
            const T tt = G * ((TK(0, 1, 0) - TK(0, 0, 0)) * idx
                                   + (TK(1, 0, 1) + TK(1, 1, 1) - TK(1, 0, -1) - TK(1, 1, -1)) * qy + (px - sz) * qz);
            sz = zx;
            if constexpr (RK3) {
                // RK3 keeps the advection as the history; the stress divergence at B^k and any solid
                // penalisation follow in k_stress_div
                ru[0] = ax;
                rs[0] = U0 + (double)(dt * (((T)2 * cal * (ms * lx + fx) + cal * tt) * irho - c1 * ax - c2 * oru[0]));
            } else {
                // a solid, if any, is applied by k_penalise once u* is complete
                ru[0] = -ax + (ms * lx + tt + fx) * irho;
                rs[0] = U0 + (double)(dt * fma(c1, ru[0], c2 * oru[0]));
            }
            if (freeze) { rs[0] = U0; ru[0] = (T)0; }
        } else {
            // y-face (i, j+1/2, k)
            T ay, ly, az, lz;
            {
                EVP_STAGE_CONSTANTS;
                const T ve = VV(s0, 1, 0), vw = VV(s0, -1, 0), vn = VV(s0, 0, 1), vs = VV(s0, 0, -1), vf = VV(sp, 0, 0), vb = VV(sm, 0, 0);
                const T cT = v0 + vn, cS = vs + v0, uR = u0 + VU(s0, 0, 1), uL = VU(s0, -1, 0) + VU(s0, -1, 1);
                const T wF = w0 + VW(s0, 0, 1), wB = VW(sm, 0, 0) + VW(sm, 0, 1);
                ay = (uR * (v0 + ve) - uL * (vw + v0)) * qx + (cT * cT - cS * cS) * qy + (wF * (v0 + vf) - wB * (vb + v0)) * qz;
                ly = (ve - (T)2 * v0 + vw) * idx2 + (vn - (T)2 * v0 + vs) * idy2 + (vf - (T)2 * v0 + vb) * idz2;
            }
            __asm__ volatile("" ::"v"(ay), "v"(ly) : "memory");
            // z-face (i, j, k+1/2)
            {
                EVP_STAGE_CONSTANTS;
                const T we = VW(s0, 1, 0), ww = VW(s0, -1, 0), wn = VW(s0, 0, 1), ws = VW(s0, 0, -1), wf = VW(sp, 0, 0), wb = VW(sm, 0, 0);
                const T cF = w0 + wf, cK = wb + w0, uR = u0 + VU(sp, 0, 0), uL = VU(s0, -1, 0) + VU(sp, -1, 0);
                const T vT = v0 + VV(sp, 0, 0), vB = VV(s0, 0, -1) + VV(sp, 0, -1);
                az = (uR * (w0 + we) - uL * (ww + w0)) * qx + (vT * (w0 + wn) - vB * (ws + w0)) * qy + (cF * cF - cK * cK) * qz;
                lz = (we - (T)2 * w0 + ww) * idx2 + (wn - (T)2 * w0 + ws) * idy2 + (wf - (T)2 * w0 + wb) * idz2;
            }
            __asm__ volatile("" ::"v"(az), "v"(lz) : "memory");
            EVP_STAGE_CONSTANTS;
            const T zy1 = TK(4, 0, 1), py1 = TP(4, 0, 1), zy = TSUM(cur, f0, 4, 0, 1), py = TSUM(nxt, f1, 4, 0, 1);
            const T ty_ = G * ((TK(1, 1, 0) + TK(1, 1, 1) - TK(1, -1, 0) - TK(1, -1, 1)) * qx
                                    + (TK(3, 0, 1) - TK(3, 0, 0)) * idy + (py - sz) * qz);
            const T tz_ = G * ((TK(2, 1, 0) + TP(2, 1, 0) - TK(2, -1, 0) - TP(2, -1, 0)) * qx
                                    + (zy1 + py1 - TK(4, 0, -1) - TP(4, 0, -1)) * qy + (TP(5, 0, 0) - TK(5, 0, 0)) * idz);
            sz = zy;
            if constexpr (RK3) {
                ru[0] = ay;
                ru[NF - 1] = az;
                rs[0] = V0 + (double)(dt * (((T)2 * cal * (ms * ly) + cal * ty_) * irho - c1 * ay - c2 * oru[0]));
                rs[NF - 1] = W0 + (double)(dt * (((T)2 * cal * (ms * lz) + cal * tz_) * irho - c1 * az - c2 * oru[NF - 1]));
            } else {
                ru[0] = -ay + (ms * ly + ty_) * irho;
                ru[NF - 1] = -az + (ms * lz + tz_) * irho;
                rs[0] = V0 + (double)(dt * fma(c1, ru[0], c2 * oru[0]));
                rs[NF - 1] = W0 + (double)(dt * fma(c1, ru[NF - 1], c2 * oru[NF - 1]));
            }
            if (vwall) { rs[0] = 0.0; ru[0] = (T)0; }
            if (freeze) {
                rs[0] = V0;
                rs[NF - 1] = W0;
                ru[0] = ru[NF - 1] = (T)0;
            }
        }
#pragma unroll
        for (int cc = 0; cc < 3; ++cc) {
            rb[cc] = wm[2][cc] + dt * fma(c1, rt[cc], c2 * old[cc]);
        }
        keep_v();
#undef U0
#undef V0
#undef W0
#undef TK
#undef TP
#undef TAU
#undef TSUM
#undef VU
#undef VV
#undef VW
        // the plane's LDS reads are done before its buffers are staged into again
        lds_barrier();
    }
    if (valid) store_results(k1 - 1);
}

constexpr int kAnyModel = -1;      // several models in one launch

// Waves per SIMD the registers are to allow.  Mixed form, wide tiles: three blocks fit a CU's LDS, and six
// waves in 80 registers (10 to 12 spilled) beat four in 90 where a grid fills them (512x256x256 Saramito:
// 1446 against 1580 us; 128^3: 105 against 107); FENE-P alone, with 28 spilled, loses (256x128x128: 249
// against 222 us).  The kernel for several models gains although it holds the FENE-P march (61 spilled, 84
// bytes of scratch a lane; none at four waves): 16 grids of 48^3, a third of them FENE-P, 123 against 139
// us, 32 of 32^3 66 against 73, 16 of 64^3 227 against 246, 8 of 96^3 386 against 400.
template <typename T, int TX, int MODEL> constexpr int min_waves()
{
    return sizeof(T) == 4 && TX == 32 && MODEL != EVP_FENE_P ? 6 : 4;
}

template <typename T, int W, int TX, int TY, int MODEL, bool RK3, bool HOUC>
__global__ __launch_bounds__(2 * TX * TY, (min_waves<T, TX, MODEL>())) void k_pred_async(Batch B, int freeze, int kc)
{
    __shared__ SmemA<T, TX, TY, MODEL == EVP_FENE_P> S;
    // whole waves take either branch; both run the same sequence of barriers
    if (__builtin_amdgcn_readfirstlane((int)threadIdx.x / (TX * TY)) == 0) march<T, W, 0, TX, TY, MODEL, RK3, HOUC>(S, B, freeze, kc);
    else march<T, W, 1, TX, TY, MODEL, RK3, HOUC>(S, B, freeze, kc);
}

// Grids of several models in one launch (Adams-Bashforth): a block takes the march of its grid's model.
template <typename T, int W, int TX, int TY, bool HOUC>
__global__ __launch_bounds__(2 * TX * TY, (min_waves<T, TX, EVP_SARAMITO>())) void k_pred_async_models(Batch B, int freeze, int kc)
{
    __shared__ __align__(16) char mem[sizeof(SmemA<T, TX, TY, true>)];
    const bool first = __builtin_amdgcn_readfirstlane((int)threadIdx.x / (TX * TY)) == 0;
#define EVP_MARCH(MM)                                                                              \
    do {                                                                                           \
        auto& S = *(SmemA<T, TX, TY, (MM) == EVP_FENE_P>*)mem;                                     \
        if (first) march<T, W, 0, TX, TY, MM, false, HOUC>(S, B, freeze, kc);                      \
        else march<T, W, 1, TX, TY, MM, false, HOUC>(S, B, freeze, kc);                            \
    } while (0)
    switch (((const CDesc*)B.d[blockIdx.y])->model) {
    case EVP_FENE_P: EVP_MARCH(EVP_FENE_P); break;
    case EVP_SARAMITO: EVP_MARCH(EVP_SARAMITO); break;
    case EVP_NEO_HOOKEAN: EVP_MARCH(EVP_NEO_HOOKEAN); break;
    default: EVP_MARCH(EVP_OLDROYD_B); break;
    }
#undef EVP_MARCH
}

// Planes per block and its cost, for tiles of which `slots` fill the chip.  In units of one plane of
// a full chip (`idle` of one where a CU is nearly empty): rounds of resident blocks (a last round that is partly empty runs about half as much
// faster as it is empty) times the block's planes, plus one for its prologue.  Chunk heights that
// are a multiple of 16 put the planes that the chunks work on at the same time at equal places of
// the memory interleave once there are several chunks per resident block; they measured 1-10 %
// slower there (512x256x256 channel, 32 x 8 tiles: 2598 us with 64 planes, 2567 us with 43;
// 16 x 8: 3020 us with 32 planes, 2718 us with 43).
struct Chunk { int kc; double cost; };
inline Chunk chunk_planes(long long tiles, int nz, int slots, double idle)
{
    Chunk best{1, 1e300};
    for (int kc = 1; kc <= min(nz, 64); ++kc) {
        const double full = (double)(tiles * ((nz + kc - 1) / kc)) / slots;
        double c = (full <= 1.0 ? idle + (1.0 - idle) * std::ceil(full * slots / 256) * 256 / slots : 0.5 * (full + std::ceil(full))) * (kc + 1);
        if (full > 1.0 && kc % 16 == 0) c *= 1.03;
        if (c < best.cost) best = {kc, c};
    }
    return best;
}

template <typename T, int W, int TX, int TY>
hipError_t launch_tile(const Batch& b, int nx, int ny, int nz, int kc, int fz, hipStream_t s, int model, bool rk3, bool houc)
{
    const int tiles = ((nx + TX - 1) / TX) * ((ny + TY - 1) / TY);
    dim3 grid(tiles * ((nz + kc - 1) / kc), b.count);
#define EVP_L(MM, RR, HH) hipLaunchKernelGGL((k_pred_async<T, W, TX, TY, MM, RR, HH>), grid, dim3(2 * TX * TY), 0, s, b, fz, kc)
#define EVP_M(MM)                                                                                  \
    do {                                                                                           \
        if (rk3) { if (houc) EVP_L(MM, true, true); else EVP_L(MM, true, false); }                 \
        else { if (houc) EVP_L(MM, false, true); else EVP_L(MM, false, false); }                   \
    } while (0)
    switch (model) {
    case kAnyModel:
        if constexpr (sizeof(T) == 4) {
            if (rk3) return hipErrorInvalidValue;
            if (houc) hipLaunchKernelGGL((k_pred_async_models<T, W, TX, TY, true>), grid, dim3(2 * TX * TY), 0, s, b, fz, kc);
            else hipLaunchKernelGGL((k_pred_async_models<T, W, TX, TY, false>), grid, dim3(2 * TX * TY), 0, s, b, fz, kc);
            break;
        } else return hipErrorInvalidValue;
    case EVP_FENE_P:
        if constexpr (TX == 16 || sizeof(T) == 4) { EVP_M(EVP_FENE_P); break; }
        else return hipErrorInvalidValue;
    case EVP_SARAMITO: EVP_M(EVP_SARAMITO); break;
    case EVP_NEO_HOOKEAN: EVP_M(EVP_NEO_HOOKEAN); break;
    default: EVP_M(EVP_OLDROYD_B); break;
    }
#undef EVP_M
#undef EVP_L
    return hipGetLastError();
}

}  // namespace

}  // namespace evp
