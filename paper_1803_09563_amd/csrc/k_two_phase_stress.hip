// Stress part of the two-phase step (Sec. 3.2, FP64, AB2; Eqs. (rt), (ab2tau)) as a z-marching
// LDS-tiled kernel (the single-phase predictor is predictor_async.h, the two-phase momentum
// k_two_phase.hip):
//   * a block of 32 x 8 threads owns a 32 x 8 column of cells and marches along z over a chunk of
//     planes, so every field is read from HBM about once;
//   * the seven planes k-3..k+3 that the z-direction WENO needs for the thread's own cell live in
//     registers (a sliding window);
//   * plane k of B - I, with the 3-cell cross halo of the x/y WENO stencils (ghost rows beyond a
//     wall extrapolated at load time), sits in LDS;
//   * three-plane rings in LDS hold the velocities and the stress components tau_xz, tau_yz,
//     tau_zz of planes k-1, k, k+1 on the tile plus a 1-cell halo;
//   * FENE-P stress factors G F and G (F - a) of plane k are staged once per cell.
// Block ids are remapped so consecutive tiles land on the same XCD (shared L2 for halo reads).
#include "evp_internal.h"
#include "weno.h"

namespace evp {

namespace {

constexpr int TX = 32, TY = 8, NTH = TX * TY;
constexpr int RW = TX + 6, RH = TY + 6;    // B plane with a 3-cell halo
constexpr int BW = TX + 2, BH = TY + 2;    // 1-cell halo box
constexpr int BOX = BW * BH;

// The tile rows (in y) one launch covers: rows.first + r for r < rows.count, shifted up by
// rows.skip once they reach rows.skip_from (so one launch can take the bottom and top rows of a
// channel and leave out the interior ones).
struct Rows { int first, count, skip_from, skip; };

__device__ __forceinline__ int modp(int i, int n)
{
    int r = i % n;
    return r < 0 ? r + n : r;
}

// Loads and stores at a wave-uniform base plus a per-thread byte offset that fits 32 bits
// (within one plane of one field).  BUF: as raw buffer instructions, whose descriptor (base, no
// stride, 2^31 - 1 bytes; fourth word the raw-buffer format of CDNA, 32-bit data, no swizzle)
// lives in scalar registers, so an access costs no vector arithmetic and no 64-bit address
// registers; otherwise as global instructions on the base plus the zero-extended offset (measured
// faster for the periodic kernel).
constexpr int kRawBufferWord3 = 0x00020000;
// Cache policy of an access.  kKeep: data that neighbouring tiles read again as their halo
// (B - I, u, v, w).  kStream: data that only this cell touches in this kernel (the history it
// reads, every result it writes); the non-temporal bit lets L2 evict those lines first, so the
// halo lines of a plane survive until the neighbouring tiles have read them.  The value is the
// non-temporal bit of the buffer instructions' cache-policy operand.
constexpr int kKeep = 0, kStream = 2;
template <bool BUF, typename T, int POL = kKeep>
__device__ __forceinline__ T ldx(gptr<const T> base, unsigned boff)
{
    if constexpr (BUF) {
        const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((EVP_GLOBAL void*)base, (short)0, 0x7fffffff, kRawBufferWord3);
        return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, boff, 0, POL));
    } else {
        const gptr<const T> a = (gptr<const T>)((gptr<const char>)base + boff);
        if constexpr (POL == kStream) return __builtin_nontemporal_load(a);
        else return *a;
    }
}
template <bool BUF, typename T, int POL = kStream>
__device__ __forceinline__ void stx(gptr<T> base, unsigned boff, T v)
{
    if constexpr (BUF) {
        typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
        const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((EVP_GLOBAL void*)base, (short)0, 0x7fffffff, kRawBufferWord3);
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, boff, 0, POL);
    } else {
        const gptr<T> a = (gptr<T>)((gptr<char>)base + boff);
        if constexpr (POL == kStream) __builtin_nontemporal_store(v, a);
        else *a = v;
    }
}

template <typename T> struct Smem {
    T B[6][RH][RW];      // B - I of plane k
    T gf[BH][BW];        // G F of plane k (G for Oldroyd-B / Saramito)
    T ga[BH][BW];        // G (F - a) of plane k (0 for Oldroyd-B / Saramito)
    T Z[3][3][BH][BW];   // ring slot, (tau_xz, tau_yz, tau_zz)
    T V[3][3][BH][BW];   // ring slot, (u, v, w)
};

// upwind derivative (times h) at the middle of f0..f6: WENO5, or HOUC5 (the fifth-order linear
// upwind-biased combination)
template <typename T, bool HOUC>
__device__ __forceinline__ T weno_up(T f0, T f1, T f2, T f3, T f4, T f5, T f6, T vel, T eps2)
{
    const T d0 = f1 - f0, d1 = f2 - f1, d2 = f3 - f2, d3 = f4 - f3, d4 = f5 - f4, d5 = f6 - f5;
    // pick the upwind-side differences with selects, then evaluate one WENO (no divergence)
    const bool pos = vel >= (T)0;
    const T v1 = pos ? d0 : d5, v2 = pos ? d1 : d4, v3 = pos ? d2 : d3;
    const T v4 = pos ? d3 : d2, v5 = pos ? d4 : d1;
    if constexpr (HOUC)
        return (T)(2.0 / 60.0) * v1 - (T)(13.0 / 60.0) * v2 + (T)(47.0 / 60.0) * v3
             + (T)(27.0 / 60.0) * v4 - (T)(3.0 / 60.0) * v5;
    else
        return weno5u<T>(v1, v2, v3, v4, v5, eps2);
}

// upwind derivative (times h) from six values g0..g5 already in upwind order (for a negative
// velocity the caller passes the stencil mirrored, f6..f1, and gets minus the derivative: the
// scheme is odd in its differences, and every step of it is sign-symmetric in floating point)
template <typename T, bool HOUC>
__device__ __forceinline__ T weno_dir(T g0, T g1, T g2, T g3, T g4, T g5, T eps2)
{
    const T v1 = g1 - g0, v2 = g2 - g1, v3 = g3 - g2, v4 = g4 - g3, v5 = g5 - g4;
    if constexpr (HOUC)
        return (T)(2.0 / 60.0) * v1 - (T)(13.0 / 60.0) * v2 + (T)(47.0 / 60.0) * v3
             + (T)(27.0 / 60.0) * v4 - (T)(3.0 / 60.0) * v5;
    else
        return weno5u<T>(v1, v2, v3, v4, v5, eps2);
}

// HOUC: fifth-order upstream-central advection instead of WENO5 (a separate instantiation, so
// the WENO kernel's register allocation is not shared with the other scheme).
// lambda and G = mu_p/lambda of the cell come from the mixture at phi^{n+1}; only the stress is
// advanced (the momentum has its own kernel).
// The block's work: tile `bid` of the tile rows `rows`, z-chunks of kc planes.
template <bool WALLS, int MODEL, bool HOUC>
__device__ __forceinline__ void stress_block(Smem<double>& S, const Batch& B, int kc, Rows rows, int bid)
{
    using T = double;
    // buffer-instruction accesses in the wall kernel (which then keeps its ghost-row state in
    // registers with less spilling)
    constexpr bool BUF = WALLS;
    const int b = blockIdx.y;
    const Desc& D = *B.d[b];
    const int nx = D.nx, ny = D.ny, nz = D.nz;
    const int sxy = nx * ny;
    const int ps = (int)D.ps;
    const int ntx = (nx + TX - 1) / TX, nty = rows.count, nch = (nz + kc - 1) / kc;
    const int nblk = ntx * nty * nch;
    if ((nblk & 7) == 0) bid = (bid & 7) * (nblk >> 3) + (bid >> 3);     // XCD-contiguous tiles
    const int tile_x = bid % ntx, ch = bid / (ntx * nty);
    int tile_y = rows.first + (bid / ntx) % nty;
    if (tile_y >= rows.skip_from) tile_y += rows.skip;
    const int i0 = tile_x * TX, j0 = tile_y * TY, k0 = ch * kc;
    const int k1 = min(k0 + kc, nz);
    const int tx = threadIdx.x % TX, ty = threadIdx.x / TX;
    const int i = i0 + tx, j = j0 + ty;
    const bool valid = i < nx && j < ny;
    const int ic = min(i, nx - 1), jc = min(j, ny - 1);
    const int oij = jc * nx + ic;

    const int st = B.state[b];
    const gptr<const T> __restrict__ Bin = (gptr<const T>)D.Bt[st & 1];
    const gptr<T> __restrict__ Bout = (gptr<T>)D.Bt[(st & 1) ^ 1];
    const gptr<T> __restrict__ RT = (gptr<T>)D.RT;
    const bool euler = (st & ST_EULER) != 0;
    const T dt = (T)B.dt[b];
    // history weights: AB2 (3/2, -1/2; Euler start 1, 0)
    const T c1 = euler ? (T)1 : (T)1.5;
    const T c2 = euler ? (T)0 : (T)-0.5;
    constexpr bool fene = MODEL == EVP_FENE_P, sara = MODEL == EVP_SARAMITO, neo = MODEL == EVP_NEO_HOOKEAN;
    const T kap = (T)D.kappa;
    const T G = (T)D.G, L2 = (T)D.L2, afene = (T)D.a_fene, tyld = (T)D.tau_y;
    const T idx = (T)D.idx, idy = (T)D.idy, idz = (T)D.idz;
    const T e2x = (T)(1e-6 * D.dx * D.dx), e2y = (T)(1e-6 * D.dy * D.dy), e2z = (T)(1e-6 * D.dz * D.dz);
    const gptr<const double> __restrict__ gu = (gptr<const double>)D.u;
    const gptr<const double> __restrict__ gv = (gptr<const double>)D.v;
    const gptr<const double> __restrict__ gw = (gptr<const double>)D.w;

    // ---- staging descriptors, computed once: the per-plane offsets do not depend on k ----
    // Interior slots (the block's own cells) are filled from the thread's register window; only
    // halo slots, and interior slots of threads whose cell lies outside the domain (ragged
    // tiles: periodic image or wall ghost), are read from global memory.
    // B-plane halo: rows j0-1 and j0+TY over the full width, columns i0-3..i0-1 and
    // i0+TX..i0+TX+2 of the tile's rows, and the arm rows j0-3, j0-2, j0+TY+1, j0+TY+2 over the
    // tile's columns.  Box halo: the 1-cell ring.
    constexpr int NHB = 2 * RW + 6 * TY + 4 * TX;
    constexpr int NHX = 2 * BW + 2 * TY;
    static_assert(NHB <= NTH && NHX <= NTH, "one halo slot per thread");
    // row map of a (possibly ghost) centre row jg: value = wa B[ja] + wb B[jb]
    auto rowmap = [&](int jg, int& ja, int& jb, T& wa, T& wb) {
        if (!WALLS) { ja = modp(jg, ny); jb = ja; wa = (T)1; wb = (T)0; return; }
        if (jg < 0) { const T g = (T)(-jg); ja = 0; jb = 1; wa = (T)1 + g; wb = -g; return; }
        if (jg >= ny) { const T g = (T)(jg - ny + 1); ja = ny - 1; jb = ny - 2; wa = (T)1 + g; wb = -g; return; }
        ja = jg; jb = jg; wa = (T)1; wb = (T)0;
    };
    struct Src { int a, b; T wa, wb; };          // B value = wa B[a] + wb B[b] (plane-relative)
    struct VSrc { int o, kind; };                  // velocity row offset; 0 inner, 1/2 ghost, 3 top v-face
    auto bsrc = [&](int ig, int jg) {
        Src q; int ja, jb; rowmap(jg, ja, jb, q.wa, q.wb);
        q.a = ja * nx + ig; q.b = jb * nx + ig; return q;
    };
    auto vsrc = [&](int ig, int jg) {
        VSrc q;
        if (!WALLS) { q.o = modp(jg, ny) * nx + ig; q.kind = 0; }
        else if (jg < 0) { q.o = min(-1 - jg, ny - 1) * nx + ig; q.kind = 1; }
        else if (jg >= ny) { q.o = max(2 * ny - 1 - jg, 0) * nx + ig; q.kind = 2; }
        else { q.o = jg * nx + ig; q.kind = (jg == ny - 1) ? 3 : 0; }
        return q;
    };
    const int t = threadIdx.x;
    int hb_l = -1;
    Src hb{0, 0, (T)1, (T)0};
    if (t < NHB) {
        int r, c;
        if (t < 2 * RW) { r = t < RW ? 2 : TY + 3; c = t % RW; }
        else if (t < 2 * RW + 6 * TY) { const int u = t - 2 * RW, c6 = u % 6; r = 3 + u / 6; c = c6 < 3 ? c6 : TX + c6; }
        else { const int u = t - 2 * RW - 6 * TY, qq = u / TX; r = qq < 2 ? qq : TY + 2 + qq; c = 3 + u % TX; }
        hb_l = r * RW + c;
        hb = bsrc(modp(i0 + c - 3, nx), j0 + r - 3);
    }
    int hx_l = -1;
    Src hx{0, 0, (T)1, (T)0};
    VSrc hv{0, 0};
    if (t < NHX) {
        int r, c;
        if (t < 2 * BW) { r = t < BW ? 0 : TY + 1; c = t % BW; }
        else { const int u = t - 2 * BW; r = 1 + u / 2; c = (u & 1) ? TX + 1 : 0; }
        hx_l = r * BW + c;
        hx = bsrc(modp(i0 + c - 1, nx), j0 + r - 1);
        hv = vsrc(modp(i0 + c - 1, nx), j0 + r - 1);
    }
    const int own_b = (ty + 3) * RW + (tx + 3), own_x = (ty + 1) * BW + (tx + 1);
    const Src os = bsrc(modp(i, nx), j);           // used only when the cell is outside the domain
    const VSrc ov = vsrc(modp(i, nx), j);

    constexpr unsigned TS = sizeof(T);
    auto bload = [&](gptr<const T> p, int cc, const Src& q) {
        T x = ldx<BUF, T>(p + cc * ps, (unsigned)q.a * TS);
        if (WALLS) x = q.wa * x + q.wb * ldx<BUF, T>(p + cc * ps, (unsigned)q.b * TS);
        return x;
    };
    auto vload = [&](int kv, const VSrc& q, T* out) {
        const unsigned o8 = (unsigned)q.o * 8u;
        const double uu = ldx<BUF, double>(gu + kv, o8), vv = ldx<BUF, double>(gv + kv, o8), ww = ldx<BUF, double>(gw + kv, o8);
        if (!WALLS || q.kind == 0) { out[0] = (T)uu; out[1] = (T)vv; out[2] = (T)ww; }
        else if (q.kind == 3) { out[0] = (T)uu; out[1] = (T)0; out[2] = (T)ww; }
        else {
            const bool bot = q.kind == 1;
            out[0] = (T)(2.0 * (bot ? D.u_bot : D.u_top) - uu);
            out[1] = (T)0;
            out[2] = (T)(2.0 * (bot ? D.w_bot : D.w_top) - ww);
        }
    };
    // stress factors G F, G (F - a) of a B - I value set
    auto factors = [&](T b0, T b3, T b5, T& gfo, T& gao) {
        gfo = G; gao = (T)0;
        if (fene) {
            const T F = L2 / (L2 - (b0 + b3 + b5 + (T)3));
            gfo = G * F; gao = G * (F - afene);
        }
    };

    T* const sB = &S.B[0][0][0];
    // B - I of plane kk with the cross halo into S.B (own value: the window entry of plane kk)
    auto load_bplane = [&](int kk, const T* own) {
        const gptr<const T> bk = Bin + kk * sxy;
        T hvv[6], ovv[6];
#pragma unroll
        for (int cc = 0; cc < 6; ++cc) {
            hvv[cc] = (hb_l >= 0) ? bload(bk, cc, hb) : (T)0;
            ovv[cc] = valid ? own[cc] : bload(bk, cc, os);
        }
#pragma unroll
        for (int cc = 0; cc < 6; ++cc) {
            if (hb_l >= 0) sB[cc * (RH * RW) + hb_l] = hvv[cc];
            sB[cc * (RH * RW) + own_b] = ovv[cc];
        }
    };

    // ring slot sl <- tau_xz, tau_yz, tau_zz and u, v, w of plane kz (own B - I values: ownz);
    // if ownk != nullptr also the stress factors of plane k (own values: ownk)
    auto load_box = [&](int kz, const T* ownz, int sl, int kg, const T* ownk) {
        const gptr<const T> bz = Bin + kz * sxy;
        const gptr<const T> bg = Bin + kg * sxy;
        const int kv = kz * sxy;
        // halo slot
        T hz[3], hvel[3], hgf = G, hga = (T)0;
        if (hx_l >= 0) {
            T gf, ga;
            if (fene) factors(bload(bz, 0, hx), bload(bz, 3, hx), bload(bz, 5, hx), gf, ga);
            else { gf = G; ga = (T)0; }
            hz[0] = gf * bload(bz, 2, hx); hz[1] = gf * bload(bz, 4, hx); hz[2] = gf * bload(bz, 5, hx) + ga;
            vload(kv, hv, hvel);
            if (ownk && fene) factors(bload(bg, 0, hx), bload(bg, 3, hx), bload(bg, 5, hx), hgf, hga);
        }
        // own slot
        T oz[3], ovel[3], ogf = G, oga = (T)0;
        {
            T zb[6];
#pragma unroll
            for (int cc = 0; cc < 6; ++cc) zb[cc] = (cc == 1) ? (T)0 : (valid ? ownz[cc] : bload(bz, cc, os));
            T gf, ga;
            factors(zb[0], zb[3], zb[5], gf, ga);
            oz[0] = gf * zb[2]; oz[1] = gf * zb[4]; oz[2] = gf * zb[5] + ga;
            vload(kv, ov, ovel);
            if (ownk && fene) {
                if (valid) factors(ownk[0], ownk[3], ownk[5], ogf, oga);
                else factors(bload(bg, 0, os), bload(bg, 3, os), bload(bg, 5, os), ogf, oga);
            }
        }
        T* zs = &S.Z[sl][0][0][0];
        T* vs = &S.V[sl][0][0][0];
        if (hx_l >= 0) {
            zs[hx_l] = hz[0]; zs[BOX + hx_l] = hz[1]; zs[2 * BOX + hx_l] = hz[2];
            vs[hx_l] = hvel[0]; vs[BOX + hx_l] = hvel[1]; vs[2 * BOX + hx_l] = hvel[2];
            if (ownk) { (&S.gf[0][0])[hx_l] = hgf; (&S.ga[0][0])[hx_l] = hga; }
        }
        zs[own_x] = oz[0]; zs[BOX + own_x] = oz[1]; zs[2 * BOX + own_x] = oz[2];
        vs[own_x] = ovel[0]; vs[BOX + own_x] = ovel[1]; vs[2 * BOX + own_x] = ovel[2];
        if (ownk) { (&S.gf[0][0])[own_x] = ogf; (&S.ga[0][0])[own_x] = oga; }
    };

    // prologue: register window planes k0-3..k0+2, rings for planes k0-1 and k0
    T win[7][6];
#pragma unroll
    for (int m = 0; m < 6; ++m) {
        const gptr<const T> p = Bin + modp(k0 - 3 + m, nz) * sxy;
#pragma unroll
        for (int cc = 0; cc < 6; ++cc) win[m][cc] = ldx<BUF, T>(p + cc * ps, (unsigned)oij * TS);
    }
    load_box(modp(k0 - 1, nz), win[2], (k0 + 2) % 3, 0, nullptr);
    load_box(k0, win[3], (k0 + 3) % 3, 0, nullptr);

    const T h = (T)0.5, qt = (T)0.25;

    for (int k = k0; k < k1; ++k) {
        const int kp = modp(k + 1, nz);
        {
            const gptr<const T> p = Bin + modp(k + 3, nz) * sxy;
#pragma unroll
            for (int cc = 0; cc < 6; ++cc) win[6][cc] = ldx<BUF, T>(p + cc * ps, (unsigned)oij * TS);
        }
        load_bplane(k, win[3]);
        load_box(kp, win[4], (k + 4) % 3, k, win[3]);
        __syncthreads();

        if (valid) {
            const int q = k * sxy + j * nx + i;
            const int r = ty + 3, c = tx + 3, rb = ty + 1, cb = tx + 1;
            const int sm = (k + 2) % 3, s0 = (k + 3) % 3, sp = (k + 4) % 3;
#define VU(s, di, dj) S.V[s][0][rb + (dj)][cb + (di)]
#define VV(s, di, dj) S.V[s][1][rb + (dj)][cb + (di)]
#define VW(s, di, dj) S.V[s][2][rb + (dj)][cb + (di)]
            // velocity gradient L_ab = du_a/dx_b at the centre, and the centre velocity
            T L[3][3];
            L[0][0] = (VU(s0, 0, 0) - VU(s0, -1, 0)) * idx;
            L[0][1] = (VU(s0, 0, 1) + VU(s0, -1, 1) - VU(s0, 0, -1) - VU(s0, -1, -1)) * (qt * idy);
            L[0][2] = (VU(sp, 0, 0) + VU(sp, -1, 0) - VU(sm, 0, 0) - VU(sm, -1, 0)) * (qt * idz);
            L[1][0] = (VV(s0, 1, 0) + VV(s0, 1, -1) - VV(s0, -1, 0) - VV(s0, -1, -1)) * (qt * idx);
            L[1][1] = (VV(s0, 0, 0) - VV(s0, 0, -1)) * idy;
            L[1][2] = (VV(sp, 0, 0) + VV(sp, 0, -1) - VV(sm, 0, 0) - VV(sm, 0, -1)) * (qt * idz);
            L[2][0] = (VW(s0, 1, 0) + VW(sm, 1, 0) - VW(s0, -1, 0) - VW(sm, -1, 0)) * (qt * idx);
            L[2][1] = (VW(s0, 0, 1) + VW(sm, 0, 1) - VW(s0, 0, -1) - VW(sm, 0, -1)) * (qt * idy);
            L[2][2] = (VW(s0, 0, 0) - VW(sm, 0, 0)) * idz;
            const T uc = h * (VU(s0, 0, 0) + VU(s0, -1, 0));
            const T vc = h * (VV(s0, 0, 0) + VV(s0, 0, -1));
            const T wc = h * (VW(s0, 0, 0) + VW(sm, 0, 0));

            // Table 1 closure of this cell
            const T* bt = win[3];
            const double hh = heaviside(((gptr<const double>)D.phi)[q], D.eps_if);
            const double lam = D.lam1 * hh + D.lam2 * (1.0 - hh), mup = D.mup1 * hh + D.mup2 * (1.0 - hh);
            const T Gc = mup / lam, ilc = 1.0 / lam;
            T F = (T)1, a = (T)1;
            if (fene) {
                F = L2 / (L2 - (bt[0] + bt[3] + bt[5] + (T)3));
                a = afene;
            } else if (sara) {
                const T t3 = Gc * (bt[0] + bt[3] + bt[5]) * (T)(1.0 / 3.0);
                const T dxx = Gc * bt[0] - t3, dyy = Gc * bt[3] - t3, dzz = Gc * bt[5] - t3;
                const T txy = Gc * bt[1], txz = Gc * bt[2], tyz = Gc * bt[4];
                const T nrm = sqrt((T)0.5 * (dxx * dxx + dyy * dyy + dzz * dzz)
                                   + txy * txy + txz * txz + tyz * tyz);
                F = (tyld == (T)0) ? (T)1 : (nrm > tyld ? (T)1 - tyld / nrm : (T)0);
                a = F;
            } else if (neo) {
                F = (T)0;
                a = (T)0;
            }
            // local artificial diffusion (Sec. 3.1): det B < 0, or tr B >= 0.95 L^2 (FENE-P)
            bool diffon = false;
            if (kap > (T)0) {
                const T b0 = bt[0] + (T)1, b3 = bt[3] + (T)1, b5 = bt[5] + (T)1;
                const T det = b0 * (b3 * b5 - bt[4] * bt[4]) - bt[1] * (bt[1] * b5 - bt[4] * bt[2])
                            + bt[2] * (bt[1] * bt[4] - b3 * bt[2]);
                diffon = det < (T)0 || (fene && b0 + b3 + b5 >= (T)0.95 * L2);
            }

            // stress right-hand side (Eq. rt) and AB2 update (Eq. ab2tau)
            const int pa[6] = {0, 0, 0, 1, 1, 2}, pb[6] = {0, 1, 2, 1, 2, 2};
            const int cm[3][3] = {{0, 1, 2}, {1, 3, 4}, {2, 4, 5}};
            T rtv[6];
            {
                // x and y stencils read from LDS in upwind order: element m of the x stencil
                // is column c + sx (m - 3), of the y stencil row r + sy (m - 3), with s = +1 for a
                // non-negative velocity and -1 otherwise; the sign of the derivative then comes
                // with |velocity| in the advection term (no selects; bitwise the same numbers).
                const int sx = uc >= (T)0 ? 1 : -1, sy = vc >= (T)0 ? RW : -RW;
                const T* const bx = &S.B[0][r][c];
                const T auc = uc >= (T)0 ? uc : -uc, avc = vc >= (T)0 ? vc : -vc;
#pragma unroll
                for (int cc = 0; cc < 6; ++cc) {
                    const T* const pc = bx + cc * (RH * RW);
                    const T gx = weno_dir<T, HOUC>(pc[-3 * sx], pc[-2 * sx], pc[-sx], pc[0], pc[sx], pc[2 * sx], e2x);
                    const T gy = weno_dir<T, HOUC>(pc[-3 * sy], pc[-2 * sy], pc[-sy], pc[0], pc[sy], pc[2 * sy], e2y);
                    const T gz = weno_up<T, HOUC>(win[0][cc], win[1][cc], win[2][cc], win[3][cc], win[4][cc],
                                                  win[5][cc], win[6][cc], wc, e2z);
                    const T adv = auc * gx * idx + avc * gy * idy + wc * gz * idz;
                    const int p = pa[cc], rr = pb[cc];
                    T ucv = L[p][rr] + L[rr][p];
#pragma unroll
                    for (int m = 0; m < 3; ++m) ucv += L[p][m] * bt[cm[m][rr]] + bt[cm[p][m]] * L[rr][m];
                    const T relax = (((p == rr) ? (a - F) : (T)0) - F * bt[cc]) * ilc;
                    rtv[cc] = relax - adv + ucv;
                    // bound live ranges: finish this component before the next one's LDS reads
                    __asm__ volatile("" ::"v"(rtv[cc]) : "memory");
                }
            }
            if (diffon) {
#pragma unroll
                for (int cc = 0; cc < 6; ++cc)
                    rtv[cc] += kap * ((S.B[cc][r][c - 1] - (T)2 * bt[cc] + S.B[cc][r][c + 1]) * (idx * idx)
                                      + (S.B[cc][r - 1][c] - (T)2 * bt[cc] + S.B[cc][r + 1][c]) * (idy * idy)
                                      + (win[2][cc] - (T)2 * bt[cc] + win[4][cc]) * (idz * idz));
            }
            // every load of this cell's history and velocity is issued before any store: the
            // compiler cannot move a load above a store it cannot prove disjoint, and a wait for
            // a load also waits for the stores issued before it
            // plane bases (uniform) and this cell's byte offsets within a plane
            const int kq = k * sxy;
            const unsigned ob = (unsigned)(j * nx + i) * TS;
            T old[6];
#pragma unroll
            for (int cc = 0; cc < 6; ++cc) old[cc] = euler ? (T)0 : ldx<BUF, T, kStream>(RT + (kq + cc * ps), ob);
#pragma unroll
            for (int cc = 0; cc < 6; ++cc) {
                stx<BUF, T>(Bout + (kq + cc * ps), ob, bt[cc] + dt * (c1 * rtv[cc] + c2 * old[cc]));
                stx<BUF, T>(RT + (kq + cc * ps), ob, rtv[cc]);
            }
#undef VU
#undef VV
#undef VW
        }
        __syncthreads();
#pragma unroll
        for (int m = 0; m < 6; ++m)
#pragma unroll
            for (int cc = 0; cc < 6; ++cc) win[m][cc] = win[m + 1][cc];
    }
}

template <bool WALLS, int MODEL, bool HOUC>
__global__ __launch_bounds__(NTH, 2) void k_stress_two_phase(Batch B, int kc, Rows rows)
{
    __shared__ Smem<double> S;
    stress_block<WALLS, MODEL, HOUC>(S, B, kc, rows, blockIdx.x);
}

}  // namespace

// planes per block: `target` blocks per grid in total, at least 4 planes per block (periodic grids: one
// round of resident blocks; channels: shorter chunks, which leave a shorter last round)
static int chunk_planes(int tiles, int nz, int target)
{
    int nch = (target + tiles - 1) / tiles;
    nch = max(1, min(nch, nz / 4));
    return (nz + nch - 1) / nch;
}

hipError_t launch_stress_two_phase(const Batch& b, int nx, int ny, int nz, hipStream_t s, bool walls, int model, bool houc)
{
    const int ntx = (nx + TX - 1) / TX, nty = (ny + TY - 1) / TY;
    // Channel: tile rows whose whole stencil (B rows j0-3 .. j0+TY+2, velocity rows j0-1 ..
    // j0+TY) lies in rows 0 .. ny-3 never see a ghost row or the top wall face; they run the
    // periodic instantiation (same arithmetic there, and no spills of the ghost-row state), the
    // rows next to the walls the wall instantiation.
    int in_lo = 1, in_hi = walls ? (ny - 3) / TY : 0;
    if (in_hi <= in_lo) in_lo = in_hi = 0;
    struct Part { bool w; Rows rows; };
    Part parts[2];
    int np = 0;
    if (!walls) parts[np++] = {false, {0, nty, 1 << 30, 0}};
    else {
        if (in_hi > in_lo) parts[np++] = {false, {in_lo, in_hi - in_lo, 1 << 30, 0}};
        if (in_hi > in_lo) parts[np++] = {true, {0, nty - (in_hi - in_lo), in_lo, in_hi - in_lo}};
        else parts[np++] = {true, {0, nty, 1 << 30, 0}};
    }
    for (int ip = 0; ip < np; ++ip) {
        const Rows rows = parts[ip].rows;
        const int kc = chunk_planes(ntx * rows.count, nz, walls ? 2048 : 512);
        dim3 grid(ntx * rows.count * ((nz + kc - 1) / kc), b.count);
#define EVP_LAUNCH(WW, MM)                                                                         \
    do {                                                                                           \
        if (houc) hipLaunchKernelGGL((k_stress_two_phase<WW, MM, true>), grid, dim3(NTH), 0, s, b, kc, rows); \
        else hipLaunchKernelGGL((k_stress_two_phase<WW, MM, false>), grid, dim3(NTH), 0, s, b, kc, rows);   \
    } while (0)
#define EVP_BY_MODEL(WW)                                                                           \
    switch (model) {                                                                               \
    case EVP_FENE_P: EVP_LAUNCH(WW, EVP_FENE_P); break;                                           \
    case EVP_SARAMITO: EVP_LAUNCH(WW, EVP_SARAMITO); break;                                       \
    case EVP_NEO_HOOKEAN: EVP_LAUNCH(WW, EVP_NEO_HOOKEAN); break;                                 \
    default: EVP_LAUNCH(WW, EVP_OLDROYD_B); break;                                                \
    }
        if (parts[ip].w) { EVP_BY_MODEL(true) } else { EVP_BY_MODEL(false) }
#undef EVP_BY_MODEL
#undef EVP_LAUNCH
    }
    return hipGetLastError();
}

}  // namespace evp
