// Fused thread-safe LB step for gfx950: one kernel reads the raw moments and
// phase field of step t once from HBM and writes those of step t+1 once.
//
// Work decomposition.  A workgroup owns a 32 x 16 (or 32 x 20) tile of (x, y)
// destination columns and marches through a chunk of z planes.  Its waves have
// fixed roles: destination columns (each also the source of that column), columns
// of the one-node halo ring (sources only) and, with two components, the geometry
// of the interface (columns of a one- and a two-node halo, two rows at a time).
// For every z plane the workgroup
//   S1  stages the fixed-point phase field of a plane (3-node halo) in LDS,
//   S2  computes G = grad(phi) and n = G/(|G| + eps) (2-node halo) from the plane's
//       nine values around a column and sums kept of the planes before it,
//   S3  computes kappa = div n and F = -sigma kappa G (1-node halo),
//   S4  expands at every source the post-collision populations (as brackets
//       t_i = f_i/w_i - 1) in c_z: t(c) = T0 + c_z T1 + (c_z^2 - 1/3) T2, each T on the
//       nine (c_x, c_y), and the 7 phase populations,
//   S5  moves them across columns through LDS,
//   S6  sums the three T over (c_x, c_y) at the destination, forms from the sums what
//       c_z = -1, 0, +1 carry to the planes below, at and above (kept in registers),
//       finishes the plane below and stores it.
// Each destination node is written by exactly one thread and every read is of
// step t, so the update is race-free (the thread-safe property of the method).
//
// What bounds it.  Vector instructions (75 % of the SIMDs' cycles on a 128 x 128 x 512
// jet, 70 % at 512 x 512 x 2048, 54 % with one component) and the latency of two
// dependent phases per plane, not HBM; on large lattices with every node moving the
// chip also lowers its clock, so instructions and LDS words cost time twice.  What the
// choices below bought, each timed on a 128 x 128 x 512 jet in motion in turn with the
// one before (us a step; from process to process the last varies from 180 to 189):
//   252  populations exchanged per c_z, G from 13 differences per column and plane
//   226  the T exchanged instead (the c_z expansion and the neighbour density
//        difference then act on 6 sums and on T0 instead of on 27 populations), 16-byte
//        LDS records per direction, G and kappa from running sums (9 LDS reads of phi
//        a column instead of 26), state accesses with a scalar base, the memory wait
//        after the destination's arithmetic
//   195  geometry in waves of its own (six beside ten, or four beside twelve).  Spread
//        over the source waves its work stood in the same chain: phase A was a source
//        and a geometry item one after the other, phase B a destination and a curvature
//        item, on 10 waves (2.5 a SIMD, so the third wave of two SIMDs set the pace).
//        Now both run side by side on 16 waves, the geometry one plane ahead; two rows
//        of an item share their 12 values of phi (instead of 9 each) and their sums of
//        n.  256^3 vortex (one component, only the first moment load moved) 266 as before,
//        variable density 237 -> 201, 512 x 512 x 2048 jet 14.1 -> 12.8 ms.
//   182  wall lanes served by register moves (at `edge` below), and the moments no longer
//        one register tuple (at `each`); 512 x 512 x 2048 jet 12.3 -> 11.5 ms
// and the same here, but 32^3 droplet 15.4 -> 14.6, 96^3 29.6 -> 28.5, 128^3 48.7 -> 47.1,
// 200 x 200 x 400 FP16Q jet 449 -> 433: the first geometry planes in a prologue of three
// barriers instead of three iterations, and LDS reads around one address (at lds_base; a
// geometry wave's vector instructions a plane 162 -> 153, 233 -> 207 with 16-bit moments).
//
// Arithmetic (Eqs. 5-8, 15-19 with Guo forcing; Eqs. 20-24):
//   source:  u = ubar + F/(2 rho), P = Q + F F/(4 rho), J = rho u + F/2,
//            a2 = rho u u + (1-omega) P + (u F + F u)/2,
//            a3_aab = rho u_a^2 u_b + (1-omega)(2 u_a P_ab + u_b P_aa),
//            a3_xyz = rho u_x u_y u_z + (1-omega)(u_x P_yz + u_y P_xz + u_z P_xy),
//            t(c) = rho' + 3 c.J + 4.5 H2(c):a2 + 4.5 H3(c):a3, evaluated as a tensor
//            product of 1-D quadratics in c_x, c_y, c_z;
//   destination: moments sum_i w_i H(c_i) t_i(x - c_i) as a tensor product of
//            1-D three-point transforms written relative to the middle value, so
//            the large isotropic part cancels before rounding.
// 16-bit stored moments (FP16, BF16, FP16Q) keep an earlier order of this arithmetic:
// populations instead of the T are exchanged, G comes from 13 pairs of neighbours, and
// sums carry their factors.  A
// change of rounding in binary32 turns into other roundings of stored moments, and
// those travel: ten steps of a jet with BF16 moments then differ by 5e-3 in the
// stress, as much as from the exact result.  Waves, tiles and the LDS records are the
// same.  It takes 25 % more vector instructions (735 a node, 589 in binary32; 128 x 128 x
// 512 jet, FP16, 188 us a step; 248 with its geometry spread over the source waves).
// Variable density and viscosity (VD): the velocity-based form of the phase-field
// scheme for components of different density.  The stored rho' is then the
// normalised pressure p*, the velocity terms of the rebuild take unit density,
// omega follows nu(phi) per source, and F is replaced by the acceleration
//   a = (-sigma kappa G - p* c_s^2 drho G - (1 - omega/2) drho Q.G) / rho(phi) + g
// (surface tension, pressure and viscous forces over rho(phi) = rho_b + drho phi,
// plus gravity; zero on boundary layers), so that at the destination
// ubar = j and Q = Pi - rho c_s^2 I - j j.
// Precision: the source builds tau = t - rho' (no density part) and publishes its
// rho' beside it; the destination forms t - rho'(own column, same plane) as
// tau + (rho'(source) - rho'(own column)), exact differences of neighbours, and
// puts rho'(own column) back into the zeroth moment only; in binary32 it takes the
// differences of tau and of rho' apart (xy_moments).  No sum is rounded at the magnitude
// of rho' except in z and in the final density itself.
#include <algorithm>
#include <type_traits>
#include <utility>

#include "tslb_internal.h"

namespace tslb {
namespace fused {

// Tile shapes.  A workgroup owns TX x TY destination columns; its sources, the
// geometry and the staged phase field cover the tile plus a halo of 1, 2 and 3
// columns.  Two heights: 16 rows (10 waves with a source, 6 of geometry) and 20
// rows (12 and 4: about 1.25 times the time a plane for 1.25 times the columns, but fewer
// workgroups where that saves a round), chosen
// per lattice by the host (fused_plan); the one-component and variable-density
// steps take 16 rows, the former without geometry waves.
template <int ROWS> struct Tile {
    static constexpr int TX = 32, TY = ROWS;
    static constexpr int SX = TX + 2, SY = TY + 2, NSRC = SX * SY;   // sources: 34 x 18 or 34 x 22
    static constexpr int GX = TX + 4, GY = TY + 4, NGEO = GX * GY;   // geometry: 36 x 20 or 36 x 24
    static constexpr int PX = TX + 6, PY = TY + 6, NPHI = PX * PY;   // phase field: 38 x 22 or 38 x 26
    static constexpr int NDST = TX * TY;                              // 512 or 640
    static constexpr int NST = ROWS == 16 ? 640 : 768;                // threads with a source or destination
    static constexpr int NGT = ROWS == 16 ? 384 : 256;                // threads of the geometry waves (two components)
    static constexpr int REC = 36;                                    // words of a source's exchange record
    static_assert(ROWS == 16 || ROWS == 20, "tile heights: 16 or 20 rows");
    static_assert(NSRC <= NST && NDST <= NSRC && NST + NGT <= 1024, "tile does not fit the workgroup");
    static constexpr int threads(bool phase) { return phase ? NST + NGT : NST; }
};
typedef float vec4 __attribute__((ext_vector_type(4)));
typedef int32_t ivec4 __attribute__((ext_vector_type(4)));

// LDS of a workgroup: PH = two components (with the phase field), else one.
// The gradient ring holds G itself for the variable-density step (its forces
// take G directly), else only |G| + eps: the force is rebuilt as n (|G| + eps)
// from the stored normal, which keeps the 20-row tile within 160 KB of LDS.
// One component has no phase field to publish.  Its exchange buffer is laid out by
// direction (DIR) where that was the faster, 10 KB less: two workgroups share a compute
// unit where a launch has more of them than units, as before the records (186 x 6 x 853
// BF16 46.1 us a step, 47.3 with records; 256^3 vortex 265.6 and 267.9, FP16 249 and 257,
// BF16 258 and 261).  FP16Q keeps the records of two components (267 us, 275 by direction).
template <int ST, bool PH> constexpr bool by_direction = !PH && ST != ST_FP16Q;
template <bool PH, bool VD, int ROWS, bool DIR> struct alignas(16) Smem {
    using T = Tile<ROWS>;
    float xch[T::NSRC][T::REC];        // populations crossing columns
    int32_t phi[4][T::NPHI];           // fixed-point phase field, ring of 4 planes
    float n[2][3][T::NGEO];            // unit normal, ring of 2 planes
    float G[2][VD ? 3 : 1][T::NSRC];   // gradient (VD) or |G| + eps on the source region, ring of 2 planes
    float kap[T::NSRC];                // 72 kappa of the next source plane
};
template <bool VD, int ROWS> struct alignas(16) Smem<false, VD, ROWS, false> {
    float xch[Tile<ROWS>::NSRC][Tile<ROWS>::REC];  // populations crossing columns
};
template <bool VD, int ROWS> struct alignas(16) Smem<false, VD, ROWS, true> {
    vec4 xch[8][Tile<ROWS>::NSRC];  // populations crossing columns
};
static_assert(sizeof(Smem<true, false, 20, false>) <= 160 * 1024 && sizeof(Smem<true, true, 16, false>) <= 160 * 1024,
              "LDS of one workgroup");
static_assert(2 * sizeof(Smem<false, false, 16, true>) <= 160 * 1024, "LDS of two workgroups");
// Waves a SIMD holds: of one workgroup of 16 waves, or of two of ten.
template <int ST, bool PH> constexpr int waves_per_simd = by_direction<ST, PH> ? 5 : PH ? 4 : 3;

// f(0), ..., f(N - 1) with compile-time indices.  An unrolled loop over an array that
// lives across branches or iterations is too late: the compiler has made the array one
// wide register tuple by then, which it copies as a whole (ten moves a plane for the
// moments, and a tuple carried through the loop).
template <class F, int... I> __device__ __forceinline__ void each_of(F &&f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F> __device__ __forceinline__ void each(F &&f) { each_of(f, std::make_integer_sequence<int, N>{}); }

// Values formed here, in program order with the other pins (an empty asm statement).
__device__ __forceinline__ void keep_here(float &a) { __asm__ volatile("" : "+v"(a)); }
__device__ __forceinline__ void keep_here(float &a, float &b) { __asm__ volatile("" : "+v"(a), "+v"(b)); }
__device__ __forceinline__ void keep_here(float &a, float &b, float &c) { __asm__ volatile("" : "+v"(a), "+v"(b), "+v"(c)); }

// 1-D three-point transform of (a_-, a_0, a_+) with weights (1/6, 2/3, 1/6):
// m0 = sum w a, 6 m1 = 6 sum w c a, 9 m2 = 9 sum w (c^2 - 1/3) a, written relative to
// a_0.  The factors of the first and second moments are left to the constants of
// the multiply-adds that take them (in z, and where the new moments are formed).
struct Tr3 {
    float m0, m1, m2;
};
__device__ __forceinline__ Tr3 tr3(float am, float a0, float ap) {
    const float dm = am - a0, dp = ap - a0;
    Tr3 r;
    r.m2 = dm + dp;
    r.m0 = fmaf(r.m2, 1.0f / 6.0f, a0);
    r.m1 = dp - dm;
    return r;
}
__device__ __forceinline__ float tr3_m0(float am, float a0, float ap) {
    return fmaf((am - a0) + (ap - a0), 1.0f / 6.0f, a0);
}

// 1/x for a normal x (a density near 1, or |G| + eps): the hardware reciprocal
// refined by one Newton-Raphson step, e = 1 - x r, r' = r + r e, within an ulp.
__device__ __forceinline__ float recip(float x) {
    const float r = __builtin_amdgcn_rcpf(x);
    return fmaf(r, fmaf(-x, r, 1.0f), r);
}

// Quadratic A + B c + C (c^2 - 1/3) at c = -1, 0, +1.
__device__ __forceinline__ void quad3(float A, float B, float C, float &vm, float &v0, float &vp) {
    const float m = fmaf(C, 2.0f / 3.0f, A);
    v0 = fmaf(C, -1.0f / 3.0f, A);
    vm = m - B;
    vp = m + B;
}

// The T of t(c) = T0 + c_z T1 + (c_z^2 - 1/3) T2 from the Hermite coefficients, without
// the density (tau = t - rho'): put(ix, iy, T0, T1, T2) for each of the nine (c_x, c_y) =
// (ix - 1, iy - 1).  H: the roundings that 16-bit stored moments keep (9 a2_yz unrounded).
template <bool H, class Put>
__device__ __forceinline__ void expand_c(float Jx, float Jy, float Jz, float a2xx, float a2yy, float a2zz, float a2xy,
                                         float a2xz, float a2yz, float a3xxy, float a3xxz, float a3yyx, float a3yyz,
                                         float a3zzx, float a3zzy, float a3xyz, Put &&put) {
#pragma clang fp contract(off)
    // The scale factors of the coefficients (3 J, 4.5 a2_aa, 9 a2_ab, 13.5 a3_aab,
    // 27 a3_xyz) are folded into the constants of the multiply-adds that take
    // a coefficient as a slope or curvature term; only the five that enter as
    // an addend are scaled explicitly.
    const float K1y = 3.0f * Jy, K1z = 3.0f * Jz;
    const float K2yy = 4.5f * a2yy, K2zz = 4.5f * a2zz, K2yz = 9.0f * a2yz;
    // t = T0 + cz T1 + h(cz) T2; T0 = U0 + cy U1 + h(cy) U2 (per cx), etc.
    float U0[3], U1[3], V0[3], W0[3];
    {   // U0 = quad3(0, 3 Jx, 4.5 a2xx): tau = t - rho'
        const float m = 3.0f * a2xx;
        U0[1] = -1.5f * a2xx;
        U0[0] = fmaf(-3.0f, Jx, m);
        U0[2] = fmaf(3.0f, Jx, m);
    }
    {   // U1 = quad3(3 Jy, 9 a2xy, 13.5 a3xxy)
        const float m = fmaf(9.0f, a3xxy, K1y);
        U1[1] = fmaf(-4.5f, a3xxy, K1y);
        U1[0] = fmaf(-9.0f, a2xy, m);
        U1[2] = fmaf(9.0f, a2xy, m);
    }
    {   // V0 = quad3(3 Jz, 9 a2xz, 13.5 a3xxz)
        const float m = fmaf(9.0f, a3xxz, K1z);
        V0[1] = fmaf(-4.5f, a3xxz, K1z);
        V0[0] = fmaf(-9.0f, a2xz, m);
        V0[2] = fmaf(9.0f, a2xz, m);
    }
    W0[0] = fmaf(-13.5f, a3zzx, K2zz);
    W0[1] = K2zz;
    W0[2] = fmaf(13.5f, a3zzx, K2zz);
#pragma unroll
    for (int ix = 0; ix < 3; ++ix) {
        const float cx = (float)(ix - 1);
        const float U2 = ix == 1 ? K2yy : fmaf(13.5f * cx, a3yyx, K2yy);  // linear in cx
        const float V1 = ix == 1 ? K2yz : fmaf(27.0f * cx, a3xyz, K2yz);
        float T0[3], T1[3], T2[3];
        quad3(U0[ix], U1[ix], U2, T0[0], T0[1], T0[2]);
        {   // T1 = quad3(V0, V1, 13.5 a3yyz)
            const float m = fmaf(9.0f, a3yyz, V0[ix]);
            T1[1] = fmaf(-4.5f, a3yyz, V0[ix]);
            T1[0] = H && ix == 1 ? fmaf(-9.0f, a2yz, m) : m - V1;
            T1[2] = H && ix == 1 ? fmaf(9.0f, a2yz, m) : m + V1;
        }
        T2[0] = fmaf(-13.5f, a3zzy, W0[ix]);
        T2[1] = W0[ix];
        T2[2] = fmaf(13.5f, a3zzy, W0[ix]);
#pragma unroll
        for (int iy = 0; iy < 3; ++iy) put(ix, iy, T0[iy], T1[iy], T2[iy]);
    }
}

// Slot of direction (cx, cy) != (0, 0) in the exchange buffer of one z group.
__device__ __forceinline__ constexpr int xy_slot(int cx, int cy) {
    return ((cx + 1) + 3 * (cy + 1)) < 4 ? ((cx + 1) + 3 * (cy + 1)) : ((cx + 1) + 3 * (cy + 1)) - 1;
}

__device__ __forceinline__ int wrap_or_clamp(int v, int n, int periodic) {
    if (periodic) {
        v %= n;
        return v < 0 ? v + n : v;
    }
    return v < 0 ? 0 : (v >= n ? n - 1 : v);
}

// Column i of a W x H region (W > 32) in the order in which lanes take them: first
// columns 0-31, one row per half-wave (32 neighbouring LDS words: no bank conflict),
// then the remaining W - 32 columns, row by row.
struct Item {
    int x, y;
};
template <int W, int H> __device__ __forceinline__ Item item_of(int i) {
    static_assert(W > 32 && W < 64, "rows are split into 32 + (W - 32) columns");
    if (i < 32 * H) return {i & 31, i >> 5};
    return {32 + (i - 32 * H) % (W - 32), (i - 32 * H) / (W - 32)};
}

// The six 2-D moments X_pq = sum_{cx,cy} w(cx) w(cy) h_p(cx) h_q(cy) t(cx, cy) of
// one z group, p, q in {00, 10, 01, 20, 02, 11} (order of the output array), times
// 1, 6, 6, 9, 9 and 36.
__device__ __forceinline__ void xy_moments(const float t[9], float X[6]) {
    // y stage, per c_x: t[(cx+1) + 3(cy+1)]
    Tr3 y0 = tr3(t[0], t[3], t[6]);   // c_x = -1
    Tr3 y1 = tr3(t[1], t[4], t[7]);   // c_x = 0
    Tr3 y2 = tr3(t[2], t[5], t[8]);   // c_x = +1
    Tr3 a = tr3(y0.m0, y1.m0, y2.m0);
    X[0] = a.m0;                       // 00
    X[1] = a.m1;                       // 10
    X[3] = a.m2;                       // 20
    Tr3 b = tr3(y0.m1, y1.m1, y2.m1);
    X[2] = b.m0;                       // 01
    X[5] = b.m1;                       // 11
    X[4] = tr3_m0(y0.m2, y1.m2, y2.m2);  // 02
}

// The same of t + (w - w[4]), the brackets t without their density and the densities w.
// Differences of t and of w are taken before the two are added, so that the sums of
// three columns are not rounded at the magnitude of a population (the velocity's) for
// the sake of a difference of densities.
__device__ __forceinline__ void xy_moments(const float t[9], const float w[9], float X[6]) {
    const float m0 = (t[0] - t[3]) + (w[0] - w[3]), p0 = (t[6] - t[3]) + (w[6] - w[3]);
    const float m1 = t[1] - (t[4] - (w[1] - w[4])), p1 = t[7] - (t[4] - (w[7] - w[4]));
    const float m2 = (t[2] - t[5]) + (w[2] - w[5]), p2 = (t[8] - t[5]) + (w[8] - w[5]);
    const float s0 = m0 + p0, s1 = m1 + p1, s2 = m2 + p2;
    const float a0 = fmaf(s0, 1.0f / 6.0f, t[3]), a1 = fmaf(s1, 1.0f / 6.0f, t[4]), a2 = fmaf(s2, 1.0f / 6.0f, t[5]);
    const float dm = a0 - (a1 - (w[3] - w[4])), dp = a2 - (a1 - (w[5] - w[4]));
    X[3] = dm + dp;
    X[0] = fmaf(X[3], 1.0f / 6.0f, a1);
    X[1] = dp - dm;
    const Tr3 b = tr3(p0 - m0, p1 - m1, p2 - m2);
    X[2] = b.m0;
    X[5] = b.m1;
    X[4] = tr3_m0(s0, s1, s2);
}

// The forms of the arithmetic that 16-bit stored moments keep (see the header): the
// transforms with their factors multiplied out, and the weighted three-point sum
// (1/6) m + (2/3) z + (1/6) p.
__device__ __forceinline__ Tr3 tr3_scaled(float am, float a0, float ap) {
    const float dm = am - a0, dp = ap - a0;
    const float s = dm + dp;
    Tr3 r;
    r.m0 = fmaf(s, 1.0f / 6.0f, a0);
    r.m1 = (dp - dm) * (1.0f / 6.0f);
    r.m2 = s * (1.0f / 9.0f);
    return r;
}
__device__ __forceinline__ void xy_moments_scaled(const float t[9], float X[6]) {
    const Tr3 y0 = tr3_scaled(t[0], t[3], t[6]), y1 = tr3_scaled(t[1], t[4], t[7]), y2 = tr3_scaled(t[2], t[5], t[8]);
    const Tr3 a = tr3_scaled(y0.m0, y1.m0, y2.m0);
    X[0] = a.m0;
    X[1] = a.m1;
    X[3] = a.m2;
    const Tr3 b = tr3_scaled(y0.m1, y1.m1, y2.m1);
    X[2] = b.m0;
    X[5] = b.m1;
    X[4] = tr3_m0(y0.m2, y1.m2, y2.m2);
}
__device__ __forceinline__ float w1sum(float m, float z, float p) { return fmaf(z, 2.0f / 3.0f, (m + p) * (1.0f / 6.0f)); }

// Workgroups are dispatched round-robin over the 8 XCDs, each with its own L2.
// Work item w is assigned so that every XCD receives a contiguous range of w:
// the tiles of one z chunk then run side by side on one XCD and their
// overlapping halos are served by that XCD's L2 instead of HBM.
__device__ __forceinline__ int xcd_work_item(int b, int nb) {
    const int q8 = nb >> 3, rem8 = nb & 7;
    const int xcd = b & 7, slot = b >> 3;
    return (xcd < rem8 ? xcd * (q8 + 1) : rem8 * (q8 + 1) + (xcd - rem8) * q8) + slot;
}

// A pointer that is the same in every lane, kept in scalar registers, and a
// 32-bit lane offset in bytes.  The empty asm statements hide how the two were
// formed, so that an access through them takes the scalar-base form of the memory
// instructions.  Without them the compiler shares base + lane offset between the
// planes and adds each plane's stride in 64-bit vector arithmetic (one
// v_lshl_add_u64 per access, 22 of them per node), or keeps every plane's base in
// scalar registers, which do not suffice for that.
__device__ __forceinline__ global_t<char> *uniform(global_t<char> *p) {
    __asm__ volatile("" : "+s"(p));
    return p;
}
__device__ __forceinline__ uint32_t lane_offset(uint32_t off) {
    __asm__ volatile("" : "+v"(off));
    return off;
}

// An LDS address kept in one register: reads around it then take their offsets in the
// instruction.  Else every pair of words (ds_read2, whose offsets span 1 KB) gets an
// address of its own, the position in LDS folded into each.
template <class T> using lds_t = __attribute__((address_space(3))) T;
template <class T> __device__ __forceinline__ const lds_t<T> *lds_base(const T *p) {
    const lds_t<T> *q = (const lds_t<T> *)p;
    __asm__ volatile("" : "+v"(q));
    return q;
}

// Bytes of a word of moment plane p.
template <int ST> __device__ __forceinline__ constexpr int moment_size(int p) {
    return ST == ST_FP32 || (ST == ST_FP16Q && p < 4) ? 4 : 2;
}

// Stored words of the ten moments of the node at element `off` of the z plane that
// starts `zoff` elements into each moment plane (zoff uniform).
template <int ST>
__device__ __forceinline__ void load_plane(const void *mom, long long ld, long long zoff, uint32_t off, uint32_t m[10]) {
    global_t<char> *q = (global_t<char> *)mom + moment_size<ST>(0) * zoff;
    uint32_t o = lane_offset(off * moment_size<ST>(0));
    each<10>([&](auto i_) {
        constexpr int p = i_;
        const int sz = moment_size<ST>(p);
        q = uniform(q);
        if (sz == 4)
            m[p] = *(const global_t<uint32_t> *)(q + o);
        else
            m[p] = *(const global_t<uint16_t> *)(q + o);
        q += sz * ld;
        if (p < 9 && moment_size<ST>(p + 1) != sz) {  // from the binary32 to the binary16 planes
            q -= (sz - moment_size<ST>(p + 1)) * zoff;
            o = lane_offset(off * moment_size<ST>(p + 1));
        }
    });
}

// One word of a new state: with the non-temporal hint or without (fused_stream_stores;
// a template parameter, since the choice at run time cost 1 to 3 % of a step).
template <bool NT, class T> __device__ __forceinline__ void store_word(global_t<char> *q, T v) {
    if constexpr (NT)
        __builtin_nontemporal_store(v, (global_t<T> *)q);
    else
        *(global_t<T> *)q = v;
}

template <int ST, bool PH, bool NT>
__device__ __forceinline__ void store_plane(const StateView &out, long long ld, long long zoff, uint32_t off,
                                               const float m[10], int32_t phi, const Scales &sc) {
    global_t<char> *q = (global_t<char> *)out.mom + moment_size<ST>(0) * zoff;
    uint32_t o = lane_offset(off * moment_size<ST>(0));
    each<10>([&](auto i_) {
        constexpr int p = i_;
        const int sz = moment_size<ST>(p);
        q = uniform(q);
        if (sz == 4)
            store_word<NT>(q + o, m[p]);
        else
            store_word<NT>(q + o, half_bits<ST>(m[p], p, sc));
        q += sz * ld;
        if (p < 9 && moment_size<ST>(p + 1) != sz) {
            q -= (sz - moment_size<ST>(p + 1)) * zoff;
            o = lane_offset(off * moment_size<ST>(p + 1));
        }
    });
    if constexpr (PH) {
        q = uniform((global_t<char> *)out.phi + 4 * zoff);
        store_word<NT>(q + lane_offset(off * 4u), phi);
    }
}
// The moments and phase of each wall lane from the lane of its nearest interior node:
// edge & 1, 2: columns 0 and 31 of each half-wave from columns 1 and 30; edge & 4, 8:
// the lower from the upper half-wave or the reverse; edge & 16: from lane lane_f.
__device__ __forceinline__ void take_over(int edge, int lane_f, float m[10], int32_t &phi) {
    auto move = [&](auto f) {
        each<10>([&](auto i_) {
            constexpr int k = i_;
            m[k] = __uint_as_float(f(__float_as_uint(m[k])));
        });
        phi = (int32_t)f((uint32_t)phi);
    };
    // quads 1, 1, 2, 3 in the first quad of rows (16 lanes) 0 and 2; 0, 1, 2, 2 in the last of 1 and 3
    if (edge & 1) move([](uint32_t v) { return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0xE5, 0x5, 0x1, false); });
    if (edge & 2) move([](uint32_t v) { return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0xA4, 0xA, 0x8, false); });
    // swap of one operand's upper half with the other's lower half: both halves lower, both upper
    if (edge & 4) move([](uint32_t v) { return (uint32_t)__builtin_amdgcn_permlane32_swap(v, v, false, false)[1]; });
    if (edge & 8) move([](uint32_t v) { return (uint32_t)__builtin_amdgcn_permlane32_swap(v, v, false, false)[0]; });
    if (edge & 16) move([=](uint32_t v) { return (uint32_t)__shfl((int)v, lane_f); });
}

// The lattice's parameters in memory: what only the inlet rule needs is read where
// an inlet node is written (loaded at kernel entry it would sit in scalar registers
// through the whole loop).
using PhysMem = const __attribute__((address_space(4))) Phys *;

// One work item (a tile and a z chunk) of one lattice.
// MULTI marks the multi-lattice kernel's instantiation: it keeps that kernel's
// copy of the step apart from the single-lattice kernel's, whose code is
// otherwise changed (and slowed) by the second user of the same instantiation.
template <int ST, bool PH, bool MULTI, bool VD, int ROWS, bool NT>
__device__ __forceinline__ void step_fused(Smem<PH, VD, ROWS, by_direction<ST, PH>> &sm, const Geo &g, const Phys &ph, PhysMem walls,
                                           const Scales &sc, const StateView &in, const StateView &out, int lz,
                                           int tiles_x, int tiles_y, unsigned long long step_next, int w) {
// multiply-adds are written out: every instantiation rounds alike
#pragma clang fp contract(off)
    using T = Tile<ROWS>;
    constexpr int TX = T::TX, TY = T::TY, SX = T::SX, SY = T::SY, NSRC = T::NSRC, GX = T::GX, GY = T::GY,
                  NGEO = T::NGEO, PX = T::PX, NPHI = T::NPHI, NDST = T::NDST;
    const int tile = w % (tiles_x * tiles_y);
    const int chunk = w / (tiles_x * tiles_y);
    // The tile owns columns [xo, xo + TX) x [yo, yo + TY); its origin (x0, y0) is
    // pulled inward at the high edge so that all TX x TY columns lie in the
    // lattice (a wall column's nearest interior node is then always in the tile).
    const int xo = (tile % tiles_x) * TX, yo = (tile / tiles_x) * TY;
    const int x0 = g.nx > TX ? min(xo, g.nx - TX) : 0;
    const int y0 = g.ny > TY ? min(yo, g.ny - TY) : 0;
    const int z0 = chunk * lz;
    const int z1 = min(z0 + lz, g.nz);  // destination planes [z0, z1)
    // Roles.  Waves are placed on the four SIMDs round-robin (wave w on SIMD w % 4).
    // The first NDST / 64 waves hold the destination columns (and their sources), the
    // next two the halo sources, the rest the geometry.  With 20 rows ten waves finish
    // destinations, three of them on SIMDs 0 and 1 and two on SIMDs 2 and 3: the halo
    // waves go to SIMDs 0 and 1 (waves 12 and 13), the geometry waves to 2 and 3, which
    // evens out both phases.
    int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    if constexpr (PH && ROWS == 20) wave = wave < 10 ? wave : (wave < 12 ? wave + 2 : (wave < 14 ? wave - 2 : wave));
    const int t = wave * 64 + ((int)threadIdx.x & 63);
    const long long plane = (long long)g.nx * g.ny;

    // ---- this thread's source column (local sx, sy in the 34 x 18 or 34 x 22 region) ----
    int sx = 0, sy = 0;
    const bool is_dst = t < NDST;
    const bool is_src = t < NSRC;
    static_assert(NDST % 64 == 0, "a wave has destinations in all lanes or in none");
    const bool dst_wave = wave < NDST / 64, source_wave = wave < T::NST / 64;
    if (is_dst) {
        sx = t % TX + 1;
        sy = t / TX + 1;
    } else if (is_src) {
        const int r = t - NDST;
        if (r < SX) { sx = r; sy = 0; }
        else if (r < 2 * SX) { sx = r - SX; sy = SY - 1; }
        else if (r < 2 * SX + TY) { sx = 0; sy = r - 2 * SX + 1; }
        else { sx = SX - 1; sy = r - 2 * SX - TY + 1; }
    }
    const int sidx = sy * SX + sx;
    const int gxs = x0 + sx - 1, gys = y0 + sy - 1;          // unwrapped global source column
    const int cxs = wrap_or_clamp(gxs, g.nx, g.per[0]);
    const int cys = wrap_or_clamp(gys, g.ny, g.per[1]);
    const uint32_t off_src = (uint32_t)cxs + (uint32_t)g.nx * (uint32_t)cys;  // nx ny < 2^30
    const bool src_bnd_xy = (!g.per[0] && (gxs <= 0 || gxs >= g.nx - 1)) ||
                            (!g.per[1] && (gys <= 0 || gys >= g.ny - 1));
    // Destination columns: every owned column, walls included.  A node on an x or y
    // wall takes the moments of its nearest interior node x_F through its face rule
    // (Eqs. 9, 10).  Each lane finishes its own column; where the tile has walls, a
    // wall lane then takes the moments of x_F from the lane that finished it.  The two
    // are in one wave (a wave holds two rows of 32 columns, walls lie at the tile's
    // edges and its height is even), but for the last row of a lattice of odd height
    // below a tile's: that row is written as an image of the row before it (y_image).
    const bool owned = is_dst && gxs >= xo && gxs < xo + TX && gxs < g.nx && gys >= yo && gys < yo + TY &&
                       gys < g.ny;
    const int dxf = (!g.per[0] && gxs == 0) ? 1 : ((!g.per[0] && gxs == g.nx - 1) ? -1 : 0);
    const int dyf = (!g.per[1] && gys == 0) ? 1 : ((!g.per[1] && gys == g.ny - 1) ? -1 : 0);
    const bool y_image = !g.per[1] && g.ny < TY && (g.ny & 1);
    const bool own = owned && !(y_image && gys == g.ny - 1);
    const int lane_f = (t & 63) + dxf + TX * (y_image && dyf < 0 ? 0 : dyf);  // lane of x_F
    uint32_t rules = 0;  // four bits per face
#pragma unroll
    for (int f = 0; f < 6; ++f) rules |= (uint32_t)ph.bc[f] << (4 * f);
    // `edge` says which walls this wave's columns meet: x walls are columns 0 and 31 of
    // its half-waves (in a lattice at least a tile wide), y walls its lower (y = 0) or
    // upper half-wave.  `keep`: the moments that the column's x or y rule leaves (bit k;
    // the inlet is a z face).  Moved within quads and between half-waves in place of
    // 11 LDS permutes in each wave of a tile with walls, a 128 x 128 x 512 jet takes
    // 182 us a step instead of 190 (periodic: 176).
    const int edge = __builtin_amdgcn_readfirstlane(!g.per[0] && g.nx < TX ? 16 :
        (!g.per[0] && x0 == 0 ? 1 : 0) | (!g.per[0] && x0 + TX >= g.nx ? 2 : 0) |
        (!g.per[1] && y0 + 2 * wave == 0 ? 4 : 0) | (!g.per[1] && y0 + 2 * wave + 1 == g.ny - 1 ? 8 : 0));
    uint32_t keep = ~0u;
    if (edge) {
        const int face = boundary_face(g, gxs, gys, 1);
        const uint32_t rule = face < 0 ? 0u : (rules >> (4 * face)) & 15u;
        if (rule == 1u) keep = face < 2 ? ~(1u << 1 | 1u << 7 | 1u << 8) : ~(1u << 2 | 1u << 7 | 1u << 9);
        if (rule == 4u) keep = ~(7u << 1);
        if (rule == 3u) keep = ~1u;
    }
    const uint32_t off_dst = (uint32_t)gxs + (uint32_t)g.nx * (uint32_t)gys;  // used where owned

    constexpr bool H = ST != ST_FP32;  // the arithmetic of 16-bit stored moments
    const float omega1 = 1.0f - ph.omega;
    const float sigma72 = ph.sigma * (1.0f / 72.0f), gamma = ph.gamma;

    // carried destination state (see S6)
    float ZA[3], ZD[3], ZQ[3], ZP[6], ZR = 0.f;
    each<3>([&](auto i_) {
        constexpr int k = i_;
        ZA[k] = ZD[k] = ZQ[k] = 0.f;
    });
    each<6>([&](auto i_) {
        constexpr int k = i_;
        ZP[k] = 0.f;
    });
    float XA[6], XB[6], XC[6];  // with 16-bit moments: X(+1) and X(0) of plane r - 1, X(+1) of plane r
    each<6>([&](auto i_) {
        constexpr int k = i_;
        XA[k] = XB[k] = XC[k] = 0.f;
    });
    int32_t PA = 0, PC = 0;    // phase partial sums of planes r - 1 and r
    float own_n[3] = {0.f, 0.f, 0.f}, own_G[3] = {0.f, 0.f, 0.f};  // n, |G| + eps (or G) and phi of the
    int32_t own_phi = 0;                                           // next source plane (own column)

    // prefetched moments of the next source plane (own column)
    uint32_t mom[10] = {};  // defined before the first prefetch (decoded but unused until then)

    // z is uniform and at most a few planes outside [0, nz): wrapped by whole
    // periods, or clamped.  In the loop each index follows from the one before.
    auto plane_of = [&](int z) {
        if (g.per[2]) {
            while (z < 0) z += g.nz;
            while (z >= g.nz) z -= g.nz;
            return z;
        }
        return z < 0 ? 0 : (z >= g.nz ? g.nz - 1 : z);
    };
    auto plane_after = [&](int z, int k) {  // plane_of(z) from k = plane_of(z - 1)
        const int n = g.per[2] ? 0 : g.nz - 1;
        return (!g.per[2] && z <= 0) ? 0 : (k + 1 >= g.nz ? n : k + 1);
    };
    const int nit = (z1 - z0) + 6;

    // ---- geometry waves (two components): waves NST / 64 and up ----
    // They stage the phase field and hand the sources n, G and kappa in LDS, each a
    // phase or more before it is used.
    if constexpr (PH) {
        if (!source_wave) {
            constexpr int NGT = T::NGT;
            constexpr int NP = (NPHI + NGT - 1) / NGT;
            // geometry and curvature go by pairs of rows, which share the values between them
            constexpr int NGP = GX * GY / 2, NCP = SX * SY / 2, NG = (NGP + NGT - 1) / NGT, NC = (NCP + NGT - 1) / NGT;
            static_assert(GY % 2 == 0 && SY % 2 == 0, "rows come in pairs");
            const int l = t - T::NST;
            // staged columns of the phase field, geometry and source columns of
            // this thread (the same ones on every plane; a surplus item repeats the last
            // column and writes nothing)
            uint32_t off_phi[NP];
#pragma unroll
            for (int k = 0; k < NP; ++k) {
                const int i = min(l + k * NGT, NPHI - 1);
                const int px = i % PX, py = i / PX;
                const int gx = wrap_or_clamp(x0 - 3 + px, g.nx, g.per[0]);
                const int gy = wrap_or_clamp(y0 - 3 + py, g.ny, g.per[1]);
                off_phi[k] = (uint32_t)gx + (uint32_t)g.nx * (uint32_t)gy;
            }
            int gc[NG], gi[NG], gs[NG];  // lower column's position in the phi, geometry and source regions
            bool gin[NG][2];             // the two columns lie in the source region
#pragma unroll
            for (int k = 0; k < NG; ++k) {
                const Item i = item_of<GX, GY / 2>(min(l + k * NGT, NGP - 1));
                const int gxl = i.x, gyl = 2 * i.y;
                gi[k] = gyl * GX + gxl;
                gc[k] = (gyl + 1) * PX + (gxl + 1);
                gs[k] = (gyl - 1) * SX + (gxl - 1);
                for (int j = 0; j < 2; ++j) gin[k][j] = gxl >= 1 && gxl <= SX && gyl + j >= 1 && gyl + j <= SY;
            }
            int cs[NC], cg[NC];  // source index, corner (x-1, y-1) in the geometry region
#pragma unroll
            for (int k = 0; k < NC; ++k) {
                const Item i = item_of<SX, SY / 2>(min(l + k * NGT, NCP - 1));
                const int cx = i.x, cy = 2 * i.y;
                cs[k] = cy * SX + cx;
                cg[k] = cy * GX + cx;
            }
            const float eps = ph.eps;
            float gSx[2 * NG], gAx[2 * NG], gSy[2 * NG], gAy[2 * NG], gR0[2 * NG], gR1[2 * NG];  // gradient partial sums (S2)
            int32_t gc0[2 * NG], gc1[2 * NG];
#pragma unroll
            for (int k = 0; k < 2 * NG; ++k) {
                gSx[k] = gAx[k] = gSy[k] = gAy[k] = gR0[k] = gR1[k] = 0.f;
                gc0[k] = gc1[k] = 0;
            }
            float k1[2 * NC], k2[2 * NC], e1[2 * NC], e2[2 * NC];  // curvature partial sums (S3a)
#pragma unroll
            for (int k = 0; k < 2 * NC; ++k) k1[k] = k2[k] = e1[k] = e2[k] = 0.f;
            auto load_phi = [&](int z, int32_t v[NP]) {
                global_t<char> *q = uniform((global_t<char> *)in.phi + 4 * (plane * z));
#pragma unroll
                for (int k = 0; k < NP; ++k) v[k] = *(const global_t<int32_t> *)(q + lane_offset(off_phi[k] * 4u));
            };
            auto stage_phi = [&](int slot, const int32_t v[NP]) {
#pragma unroll
                for (int k = 0; k < NP; ++k)
                    if (l + k * NGT < NPHI) sm.phi[slot & 3][l + k * NGT] = v[k];
            };
            // ---- S2: G and n of plane p at geometry column k ----
            // G = 3 sum_i w_i c_i phi(y + c_i) with the factorised weights (1, 4, 1)/6 per
            // axis: G_x = (1/72) sum_z (1,4,1) sum_y (1,4,1) [phi(x+1) - phi(x-1)], G_y
            // likewise, and G_z = (1/72) [36 (c(z+1) - c(z-1)) + R(z+1) - R(z-1)] with c the
            // column's own value and R = sum_xy (1,4,1)(1,4,1) (phi - c).  So one plane of
            // phi enters through nine values, and the column keeps its sums of the planes
            // before it.  Differences of phi are exact integers, rounded once when they
            // become binary32, so a uniform field gives exactly G = 0.
            auto absorb_plane = [&](int k, const int32_t *q, float &Gx, float &Gy, float &Gz) {
                const int32_t c = q[4], e = q[5], v = q[3], n = q[7], d = q[1];
                const int32_t ne = q[8], sw = q[0], se = q[2], nw = q[6];
                const float ew = (float)(e - v), ns = (float)(n - d), d1 = (float)(ne - sw), d2 = (float)(se - nw);
                const float wc = (float)(v - c), sc = (float)(d - c), swc = (float)(sw - c), nwc = (float)(nw - c);
                const float dd = d1 + d2;
                const float A = fmaf(4.0f, ew, dd), B = fmaf(4.0f, ns, d1 - d2);
                const float R = fmaf(4.0f, fmaf(2.0f, wc + sc, ew + ns), fmaf(2.0f, swc + nwc, dd));
                Gx = gSx[k] + A;
                Gy = gSy[k] + B;
                Gz = fmaf(36.0f, (float)(c - gc0[k]), R - gR0[k]);
                gSx[k] = fmaf(4.0f, A, gAx[k]);
                gAx[k] = A;
                gSy[k] = fmaf(4.0f, B, gAy[k]);
                gAy[k] = B;
                gR0[k] = gR1[k];
                gR1[k] = R;
                gc0[k] = gc1[k];
                gc1[k] = c;
            };
            auto read_phi = [&](int k, int slot, int32_t q[12]) {  // rows y - 1 .. y + 2, columns x - 1 .. x + 1
                const lds_t<int32_t> *b = lds_base(sm.phi[slot & 3] + gc[k] - PX - 1);
#pragma unroll
                for (int j = 0; j < 12; ++j) q[j] = b[(j / 3) * PX + j % 3];
            };
            // G of the middle column of q0 from 13 pairs of opposite neighbours (16-bit
            // moments), planes p - 1, p and p + 1 in qm, q0 and qp
            auto pair_gradient = [&](const int32_t *qm, const int32_t *q0, const int32_t *qp, float &Gx, float &Gy, float &Gz) {
                Gx = Gy = Gz = 0.f;
#pragma unroll
                for (int cz = -1; cz <= 1; ++cz)
#pragma unroll
                    for (int cy = -1; cy <= 1; ++cy)
#pragma unroll
                        for (int cx = -1; cx <= 1; ++cx) {
                            const bool lead = cx > 0 || (cx == 0 && (cy > 0 || (cy == 0 && cz > 0)));
                            if (!lead) continue;
                            const int32_t *qa = cz > 0 ? qp : (cz < 0 ? qm : q0), *qb = cz > 0 ? qm : (cz < 0 ? qp : q0);
                            const float d = (float)(qa[4 + 3 * cy + cx] - qb[4 - 3 * cy - cx]);
                            const float w = 3.0f * w27(cx, cy, cz) * kPhiUlp;
                            if (cx) Gx = fmaf(w * cx, d, Gx);
                            if (cy) Gy = fmaf(w * cy, d, Gy);
                            if (cz) Gz = fmaf(w * cz, d, Gz);
                        }
            };
            // G and n of the plane of iteration it (see below), from the phase planes around it
            auto geometry = [&](int it) {
                constexpr float kS = kPhiUlp / 72.0f;
#pragma unroll
                for (int k = 0; k < NG; ++k) {
                    if (k && l + k * NGT >= NGP) break;  // 20 rows: the last waves have no second pair, one has some
                    int32_t q[12], q0[12], qm[12];
                    read_phi(k, it + 1, q);
                    if constexpr (H) {
                        read_phi(k, it, q0);
                        read_phi(k, it + 3, qm);
                    }
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        float Gx, Gy, Gz, den, inv;
                        // hardware square root (1 ulp) and a refined reciprocal: |G| + eps >= eps
                        if constexpr (H) {
                            pair_gradient(qm + 3 * j, q0 + 3 * j, q + 3 * j, Gx, Gy, Gz);
                            den = __builtin_amdgcn_sqrtf(fmaf(Gx, Gx, fmaf(Gy, Gy, Gz * Gz))) + eps;
                            inv = recip(den);
                        } else {
                            absorb_plane(2 * k + j, q + 3 * j, Gx, Gy, Gz);
                            den = fmaf(__builtin_amdgcn_sqrtf(fmaf(Gx, Gx, fmaf(Gy, Gy, Gz * Gz))), kS, eps);
                            inv = recip(den) * kS;
                        }
                        if (l + k * NGT < NGP) {
                            const int i = gi[k] + j * GX, si = gs[k] + j * SX;
                            sm.n[it & 1][0][i] = Gx * inv;
                            sm.n[it & 1][1][i] = Gy * inv;
                            sm.n[it & 1][2][i] = Gz * inv;
                            if (gin[k][j]) {
                                if constexpr (VD) {
                                    sm.G[it & 1][0][si] = Gx * kS;
                                    sm.G[it & 1][1][si] = Gy * kS;
                                    sm.G[it & 1][2][si] = Gz * kS;
                                } else {
                                    sm.G[it & 1][0][si] = den;
                                }
                            }
                        }
                    }
                }
            };
            // and its share of the curvature sums
            auto curvature = [&](int it) {
                // ---- S3a: per-column partial sums of the curvature stencil (plane p) ----
                // With w_i = w1(c_x) w1(c_y) w1(c_z), w1 = (1, 4, 1)/6, the stencil
                // kappa = 3 sum_i w_i c_i . n(x + c_i) factorises into sums over one plane:
                //   72 kappa(q) = C(q-1) + 4 C(q) + C(q+1) + E(q+1) - E(q-1),
                //   C = sum_cy (1,4,1) (n_x(x+1, y+cy) - n_x(x-1, y+cy))
                //     + sum_cx (1,4,1) (n_y(x+cx, y+1) - n_y(x+cx, y-1)),
                //   E = sum_{cx,cy} (1,4,1)(1,4,1) n_z(x+cx, y+cy),
                // so each column keeps k1 = C(q-1) + 4 C(q), k2 = C(q), e1 = E(q-1) and e2 = E(q)
                // (E apart: it is of order 36 where C, a sum of differences, is small).
                // The kappa of plane p - 1 is then complete and goes out.
#pragma unroll
                for (int k = 0; k < NC; ++k) {
                    if (k && l + k * NGT >= NCP) break;
                    const lds_t<float> *bx = lds_base(sm.n[it & 1][0] + cg[k]), *by = lds_base(sm.n[it & 1][1] + cg[k]),
                                       *bz = lds_base(sm.n[it & 1][2] + cg[k]);
                    float ny[4][3], nz[4][3], D[4], e[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        D[j] = bx[j * GX + 2] - bx[j * GX];
#pragma unroll
                        for (int i = 0; i < 3; ++i) {
                            ny[j][i] = by[j * GX + i];
                            nz[j][i] = bz[j * GX + i];
                        }
                        e[j] = H ? w1sum(nz[j][0], nz[j][1], nz[j][2]) : fmaf(4.0f, nz[j][1], nz[j][0] + nz[j][2]);
                    }
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        const int m = 2 * k + j, si = cs[k] + j * SX;
                        if constexpr (H) {  // kappa itself, its weights multiplied out
                            const float C = w1sum(D[j], D[j + 1], D[j + 2]) +
                                            w1sum(ny[j + 2][0] - ny[j][0], ny[j + 2][1] - ny[j][1], ny[j + 2][2] - ny[j][2]);
                            const float E = w1sum(e[j], e[j + 1], e[j + 2]);
                            const float kap = 0.5f * (w1sum(k1[m], k2[m], C) + (E - e1[m]));
                            k1[m] = k2[m];
                            k2[m] = C;
                            e1[m] = e2[m];
                            e2[m] = E;
                            if (l + k * NGT < NCP) sm.kap[si] = kap;
                            continue;
                        }
                        const float Cx = fmaf(4.0f, D[j + 1], D[j] + D[j + 2]);
                        const float Cy = fmaf(4.0f, ny[j + 2][1] - ny[j][1], (ny[j + 2][0] - ny[j][0]) + (ny[j + 2][2] - ny[j][2]));
                        const float C = Cx + Cy, E = fmaf(4.0f, e[j + 1], e[j] + e[j + 2]);
                        const float kap = (k1[m] + C) + (E - e1[m]);
                        k1[m] = fmaf(4.0f, C, k2[m]);
                        k2[m] = C;
                        e1[m] = e2[m];
                        e2[m] = E;
                        if (l + k * NGT < NCP) sm.kap[si] = kap;
                    }
                }
            };
            // Prologue: what iterations 1 and 2 would do, whose planes have no source yet,
            // between two barriers instead of four (iteration 0 has nothing that is used).
            // Phase planes z0 - 3 .. z0 are staged at once (slots 0 - 3), z0 + 1 after them.
            {
                int32_t first[5][NP];
#pragma unroll
                for (int j = 0; j < 5; ++j) load_phi(plane_of(z0 - 3 + j), first[j]);
#pragma unroll
                for (int j = 0; j < 4; ++j) stage_phi(j, first[j]);
                __syncthreads();
#pragma unroll
                for (int k = 0; k < NG; ++k) {
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        float gx, gy, gz;
                        int32_t q[12];
                        read_phi(k, j, q);
                        absorb_plane(2 * k, q, gx, gy, gz);
                        absorb_plane(2 * k + 1, q + 3, gx, gy, gz);
                    }
                }
#pragma unroll 1
                for (int it = 1; it < 3; ++it) geometry(it);
                __syncthreads();
#pragma unroll 1
                for (int it = 1; it < 3; ++it) curvature(it);
                stage_phi(4, first[4]);
                __syncthreads();
            }
            int32_t v[NP];
            int kphi = plane_of(z0 + 1);
            for (int it = 3; it < nit; ++it) {
                kphi = plane_after(z0 - 1 + it, kphi);
                load_phi(kphi, v);
                // ================= phase A =================
                geometry(it);
                __syncthreads();
                // ================= phase B =================
                curvature(it);
                // slot of plane p - 2, whose last readers (own_phi, phase B of it - 1) are done
                stage_phi(it + 2, v);
                __syncthreads();
            }
            return;
        }
    }
    if constexpr (PH) {  // the geometry waves' prologue
        __syncthreads();
        __syncthreads();
        __syncthreads();
    }

    int kmom = plane_of(z0 - 1);  // z plane of the last load
    // Iteration it works on three planes: p = z0 - 3 + it (geometry), q = p - 1
    // (normal of the curvature sums) and r = p - 2 (sources), and finishes
    // destination plane r - 1.  Rings: phi plane p at slot it mod 4, n and G of
    // plane p at slot it mod 2.  Phase A (sources; G and n) and phase B
    // (destinations; kappa and the staging of phi) are separated by barriers.
    constexpr int IT0 = 3;  // the first source plane is loaded; it is expanded at 4
    for (int it = IT0; it < nit; ++it) {
        const int p = z0 - 3 + it;
        const int r = p - 2;

        float kap = 0.f;
        if constexpr (PH) kap = sm.kap[sidx];  // read ahead of the loads' address work
        // moments of source plane r + 1 for the next iteration
        float mom_cur[10], rho_cur = 0.f;
        if constexpr (ST == ST_FP16) {  // 1 + rho' with one rounding
            rho_cur = fmaf((float)__builtin_bit_cast(_Float16, (uint16_t)mom[0]), sc.s2, 1.0f);
            __asm__ volatile("" : "+v"(rho_cur));
        }
        each<10>([&](auto i_) {
            constexpr int k = i_;
            mom_cur[k] = ST == ST_BF16 && k == 0 ? __uint_as_float(mom[0] << 16) : decode_moment<ST>(mom[k], k, sc);
            if (!VD && !H && k >= 4) mom_cur[k] *= omega1;  // (1 - omega) Q
            // formed before the loads below, which then reuse the words' registers
            keep_here(mom_cur[k]);
        });
        // (the first source plane is z0 - 1, loaded at the first iteration; lanes without
        // a source load a column of the lattice and drop it)
        if (it > IT0) kmom = plane_after(r + 1, kmom);
        load_plane<ST>(in.mom, g.ld, plane * kmom, off_src, mom);
        // ================= phase A =================
        // what the source's own column takes of its populations (used in phase B)
        float T0c, T1c, T2c, rpc;
        int32_t prest, pup, pdown;
        if (it >= 4 && is_src) {
            // ---- S3: kappa and F at the source (plane r = q - 1) ----
            float F0 = 0.f, F1 = 0.f, F2 = 0.f, n0 = 0.f, n1 = 0.f, n2 = 0.f;
            float Gx = 0.f, Gy = 0.f, Gz = 0.f;  // grad(phi) at the source (VD)
            bool sbnd = false;                   // the source is a boundary-layer node (VD)
            int32_t phis = 0;
            if constexpr (PH) {
                const bool bnd = src_bnd_xy || (!g.per[2] && (r <= 0 || r >= g.nz - 1));
                const float a = bnd ? 0.f : -(H ? ph.sigma : sigma72) * kap;
                n0 = own_n[0];
                n1 = own_n[1];
                n2 = own_n[2];
                phis = own_phi;
                if constexpr (VD) {
                    Gx = own_G[0];
                    Gy = own_G[1];
                    Gz = own_G[2];
                    sbnd = bnd;
                    F0 = a * Gx;
                    F1 = a * Gy;
                    F2 = a * Gz;
                } else {
                    const float ag = a * own_G[0];  // G = n (|G| + eps)
                    F0 = ag * n0;
                    F1 = ag * n1;
                    F2 = ag * n2;
                }
            }

            // ---- S4: post-collision populations of the source ----
            float rp = mom_cur[0];
            if constexpr (ST == ST_BF16) {  // scaled here, from the word: one register less over the loads, 5 % (256^3 vortex)
                rho_cur = fmaf(rp, sc.s2, 1.0f);
                rp *= sc.s2;
                keep_here(rp);
            }
            float om1 = omega1;
            if constexpr (VD) {
                // rho(phi), omega(phi) and the acceleration that replaces F
                const float pc = fminf(fmaxf(phi_to_float(phis), 0.0f), 1.0f);
                const float om = recip(fmaf(3.0f, fmaf(ph.dnu, pc, ph.nu_b), 0.5f));
                om1 = 1.0f - om;
                if (sbnd) {
                    F0 = F1 = F2 = 0.f;
                } else {
                    const float ir = recip(fmaf(ph.drho, pc, ph.rho_b));
                    const float cp = (-1.0f / 3.0f) * ph.drho * rp;     // pressure force / G
                    const float cm = (0.5f * om - 1.0f) * ph.drho;      // viscous force / (Q.G)
                    const float QG0 = fmaf(mom_cur[4], Gx, fmaf(mom_cur[7], Gy, mom_cur[8] * Gz));
                    const float QG1 = fmaf(mom_cur[7], Gx, fmaf(mom_cur[5], Gy, mom_cur[9] * Gz));
                    const float QG2 = fmaf(mom_cur[8], Gx, fmaf(mom_cur[9], Gy, mom_cur[6] * Gz));
                    F0 = fmaf(fmaf(cm, QG0, fmaf(cp, Gx, F0)), ir, ph.grav[0]);
                    F1 = fmaf(fmaf(cm, QG1, fmaf(cp, Gy, F1)), ir, ph.grav[1]);
                    F2 = fmaf(fmaf(cm, QG2, fmaf(cp, Gz, F2)), ir, ph.grav[2]);
                }
#pragma unroll
                for (int k = 4; k < 10; ++k) mom_cur[k] *= om1;
            }
            const float rho = VD ? 1.0f : ST == ST_FP16 || ST == ST_BF16 ? rho_cur : 1.0f + rp;  // density of the velocity terms
            float u0 = mom_cur[1], u1 = mom_cur[2], u2 = mom_cur[3];
            auto rec = [&](int slot) -> vec4 & {  // where this source publishes `slot`
                if constexpr (by_direction<ST, PH>)
                    return sm.xch[slot][sidx];
                else
                    return ((vec4 *)&sm.xch[sidx][0])[slot];
            };
            rpc = rp;
            if constexpr (H) {
                // populations of c_z = -1, 0, +1 in place of the three T
#pragma clang fp contract(fast)
                float tm[9], t0[9], tp[9];
                const float inv = recip(rho);
                const float hF = 0.5f * inv, qF = 0.25f * inv;
                u0 = fmaf(hF, F0, u0);
                u1 = fmaf(hF, F1, u1);
                u2 = fmaf(hF, F2, u2);
                const float Pxx = fmaf(qF * F0, F0, mom_cur[4]), Pyy = fmaf(qF * F1, F1, mom_cur[5]);
                const float Pzz = fmaf(qF * F2, F2, mom_cur[6]), Pxy = fmaf(qF * F0, F1, mom_cur[7]);
                const float Pxz = fmaf(qF * F0, F2, mom_cur[8]), Pyz = fmaf(qF * F1, F2, mom_cur[9]);
                // Hermite coefficients, pre-scaled: t(c) = K0 + sum K1 c + ... (see header)
                const float Jx = fmaf(rho, u0, 0.5f * F0), Jy = fmaf(rho, u1, 0.5f * F1), Jz = fmaf(rho, u2, 0.5f * F2);
                const float mxx = omega1 * Pxx, myy = omega1 * Pyy, mzz = omega1 * Pzz;
                const float mxy = omega1 * Pxy, mxz = omega1 * Pxz, myz = omega1 * Pyz;
                const float ru0 = rho * u0, ru1 = rho * u1, ru2 = rho * u2;
                const float a2xx = fmaf(ru0, u0, mxx) + u0 * F0;
                const float a2yy = fmaf(ru1, u1, myy) + u1 * F1;
                const float a2zz = fmaf(ru2, u2, mzz) + u2 * F2;
                const float a2xy = fmaf(ru0, u1, mxy) + 0.5f * (u0 * F1 + F0 * u1);
                const float a2xz = fmaf(ru0, u2, mxz) + 0.5f * (u0 * F2 + F0 * u2);
                const float a2yz = fmaf(ru1, u2, myz) + 0.5f * (u1 * F2 + F1 * u2);
                // a3_aab = u_a (rho u_a u_b + 2 m_ab) + u_b m_aa
                const float a3xxy = fmaf(u0, fmaf(ru0, u1, 2.0f * mxy), u1 * mxx);
                const float a3xxz = fmaf(u0, fmaf(ru0, u2, 2.0f * mxz), u2 * mxx);
                const float a3yyx = fmaf(u1, fmaf(ru1, u0, 2.0f * mxy), u0 * myy);
                const float a3yyz = fmaf(u1, fmaf(ru1, u2, 2.0f * myz), u2 * myy);
                const float a3zzx = fmaf(u2, fmaf(ru2, u0, 2.0f * mxz), u0 * mzz);
                const float a3zzy = fmaf(u2, fmaf(ru2, u1, 2.0f * myz), u1 * mzz);
                const float a3xyz = fmaf(ru0 * u1, u2, fmaf(u0, myz, fmaf(u1, mxz, u2 * mxy)));
                expand_c<true>(Jx, Jy, Jz, a2xx, a2yy, a2zz, a2xy, a2xz, a2yz, a3xxy, a3xxz, a3yyx, a3yyz, a3zzx, a3zzy,
                               a3xyz, [&](int ix, int iy, float T0, float T1, float T2) {
                                   const int k = ix + 3 * iy;
                                   const float mid = fmaf(T2, 2.0f / 3.0f, T0);
                                   t0[k] = fmaf(T2, -1.0f / 3.0f, T0);
                                   tm[k] = mid - T1;
                                   tp[k] = mid + T1;
                               });
                T0c = tm[4];
                T1c = t0[4];
                T2c = tp[4];
#pragma unroll
                for (int k = 0; k < 9; ++k)
                    if (k != 4) rec(xy_slot(k % 3 - 1, k / 3 - 1)) = vec4{tm[k], t0[k], tp[k], rp};
            } else {
            // m = (1 - omega) P and a2 of the header, with g = F/rho, v = ubar + g, J = rho v
            // (formed from ubar and F: one rounding):
            //   a2_ab = J_a v_b + (1 - omega) Q_ab - (omega/4) F_a g_b
            float mxx = mom_cur[4], myy = mom_cur[5], mzz = mom_cur[6], mxy = mom_cur[7], mxz = mom_cur[8],
                  myz = mom_cur[9];
            float Jx, Jy, Jz, a2xx, a2yy, a2zz, a2xy, a2xz, a2yz;
            if constexpr (PH) {
                const float inv = VD ? 1.0f : recip(rho);
                const float g0 = F0 * inv, g1 = F1 * inv, g2 = F2 * inv;
                const float v0 = u0 + g0, v1 = u1 + g1, v2 = u2 + g2;
                Jx = fmaf(rho, u0, F0);
                Jy = fmaf(rho, u1, F1);
                Jz = fmaf(rho, u2, F2);
                u0 = fmaf(0.5f, g0, u0);
                u1 = fmaf(0.5f, g1, u1);
                u2 = fmaf(0.5f, g2, u2);
                const float hs = 0.25f * (om1 - 1.0f), ks = 0.25f * om1;
                const float h0 = hs * F0, h1 = hs * F1, h2 = hs * F2;
                const float q0 = ks * F0, q1 = ks * F1, q2 = ks * F2;
                a2xx = fmaf(Jx, v0, fmaf(h0, g0, mxx));
                a2yy = fmaf(Jy, v1, fmaf(h1, g1, myy));
                a2zz = fmaf(Jz, v2, fmaf(h2, g2, mzz));
                a2xy = fmaf(Jx, v1, fmaf(h0, g1, mxy));
                a2xz = fmaf(Jx, v2, fmaf(h0, g2, mxz));
                a2yz = fmaf(Jy, v2, fmaf(h1, g2, myz));
                mxx = fmaf(q0, g0, mxx);
                myy = fmaf(q1, g1, myy);
                mzz = fmaf(q2, g2, mzz);
                mxy = fmaf(q0, g1, mxy);
                mxz = fmaf(q0, g2, mxz);
                myz = fmaf(q1, g2, myz);
            } else {
                Jx = rho * u0;
                Jy = rho * u1;
                Jz = rho * u2;
                a2xx = fmaf(Jx, u0, mxx);
                a2yy = fmaf(Jy, u1, myy);
                a2zz = fmaf(Jz, u2, mzz);
                a2xy = fmaf(Jx, u1, mxy);
                a2xz = fmaf(Jx, u2, mxz);
                a2yz = fmaf(Jy, u2, myz);
            }
            const float ru0 = PH ? rho * u0 : Jx, ru1 = PH ? rho * u1 : Jy;
            const float rxy = ru0 * u1, rxz = ru0 * u2, ryz = ru1 * u2;
            // a3_aab = u_a (rho u_a u_b + 2 m_ab) + u_b m_aa
            const float sxy = fmaf(2.0f, mxy, rxy), sxz = fmaf(2.0f, mxz, rxz), syz = fmaf(2.0f, myz, ryz);
            const float a3xxy = fmaf(u0, sxy, u1 * mxx), a3xxz = fmaf(u0, sxz, u2 * mxx);
            const float a3yyx = fmaf(u1, sxy, u0 * myy), a3yyz = fmaf(u1, syz, u2 * myy);
            const float a3zzx = fmaf(u2, sxz, u0 * mzz), a3zzy = fmaf(u2, syz, u1 * mzz);
            const float a3xyz = fmaf(rxy, u2, fmaf(u0, myz, fmaf(u1, mxz, u2 * mxy)));
            // ---- S5a: publish what crosses columns ----
            expand_c<false>(Jx, Jy, Jz, a2xx, a2yy, a2zz, a2xy, a2xz, a2yz, a3xxy, a3xxz, a3yyx, a3yyz, a3zzx, a3zzy, a3xyz,
                            [&](int ix, int iy, float T0, float T1, float T2) {
                                if (ix == 1 && iy == 1) {
                                    T0c = T0;
                                    T1c = T1;
                                    T2c = T2;
                                } else {
                                    rec(xy_slot(ix - 1, iy - 1)) = vec4{T0, T1, T2, rp};
                                }
                            });
            }
            if constexpr (PH) {
                // phase: base to every axis neighbour, +-a_e along +-e, phi - 6 base stays
                const float phif = phi_to_float(phis);
                const float omphi = (float)(kPhiOne - phis) * kPhiUlp;
                const float gph = gamma * omphi;
                const float h8 = 0.125f * phif * kPhiInvUlp;
                const int32_t base = (phis + 4) >> 3;
                const int32_t ax = __float2int_rn(h8 * fmaf(4.0f, u0, gph * n0));
                const int32_t ay = __float2int_rn(h8 * fmaf(4.0f, u1, gph * n1));
                const int32_t az = __float2int_rn(h8 * fmaf(4.0f, u2, gph * n2));
                *(ivec4 *)&rec(8) = ivec4{base + ax, base - ax, base + ay, base - ay};  // +x, -x, +y, -y
                // phi - 6 base, kept from becoming a 64-bit multiply-add (whose unused upper
                // addend may be a register that a prefetch is still loading: its wait)
                int32_t base2 = 2 * base, base4 = 4 * base;
                __asm__("" : "+v"(base2), "+v"(base4));
                prest = phis - base2 - base4;
                pup = base + az;
                pdown = base - az;
            }
        }

        __syncthreads();

        // ================= phase B =================
        // what the next iteration's source (plane p - 1) takes of the geometry at its own
        // column (the slots are free for plane p + 1 from the next phase A on)
        if constexpr (PH) {
            const float *nq = &sm.n[(it + 1) & 1][0][0] + (sy + 1) * GX + (sx + 1);
            const float *Gq = &sm.G[(it + 1) & 1][0][0] + sidx;
            each<3>([&](auto i_) {
                constexpr int k = i_;
                own_n[k] = nq[k * NGEO];
            });
#pragma unroll
            for (int k = 0; k < (VD ? 3 : 1); ++k) own_G[k] = Gq[k * NSRC];
            own_phi = sm.phi[(it - 1) & 3][(sy + 2) * PX + (sx + 2)];
        }
        const bool finish = it >= 4 && dst_wave;
        float m[10];
        int32_t phin;
        if (finish) {
            // ---- S5b/S6: gather at the destination and finish plane r - 1 ----
            float t0[9], t1[9], t2[9], w[9];
            w[4] = rpc;
            t0[4] = T0c;
            t1[4] = T1c;
            t2[4] = T2c;
            auto arrived = [&](int dx, int dy, int slot) -> const vec4 & {  // from the source at (x + dx, y + dy)
                if constexpr (by_direction<ST, PH>)
                    return sm.xch[slot][sidx + dy * SX + dx];
                else
                    return ((const vec4 *)&sm.xch[sidx - SX - 1][0] + ((1 + dy) * SX + 1 + dx) * (T::REC / 4))[slot];
            };
#pragma unroll
            for (int cy = -1; cy <= 1; ++cy)
#pragma unroll
                for (int cx = -1; cx <= 1; ++cx) {
                    if (!cx && !cy) continue;
                    const int k = (cx + 1) + 3 * (cy + 1);
                    const vec4 v = arrived(-cx, -cy, xy_slot(cx, cy));
                    if constexpr (H) {
                        const float drp = v.w - rpc;
                        t0[k] = v.x + drp;
                        t1[k] = v.y + drp;
                        t2[k] = v.z + drp;
                    } else {
                        t0[k] = v.x;
                        t1[k] = v.y;
                        t2[k] = v.z;
                        w[k] = v.w;
                    }
                }
            float X0[6], X1[6], X2[6];
            if constexpr (H) {
                xy_moments_scaled(t0, X0);
                xy_moments_scaled(t1, X1);
                xy_moments_scaled(t2, X2);
            } else {
                xy_moments(t0, w, X0);
                xy_moments(t1, X1);
                xy_moments(t2, X2);
            }
            int32_t pin = 0;
            if constexpr (PH) {
                const int32_t(*xi)[T::REC] = (const int32_t(*)[T::REC])&sm.xch[sidx - SX - 1];
                pin = xi[SX][32] + xi[SX + 2][33] + xi[1][34] + xi[2 * SX + 1][35];
            }
            float dr = 0.f;
            if constexpr (H) {
                // X0, X1, X2 are the sums of the populations of c_z = -1, 0, +1
#pragma clang fp contract(fast)
                X0[0] += rpc;
                X1[0] += rpc;
                X2[0] += rpc;
                const Tr3 m00 = tr3_scaled(X0[0], XB[0], XA[0]);  // rho', j_z, H_zz
                const Tr3 m10 = tr3_scaled(X0[1], XB[1], XA[1]);  // j_x, H_xz
                const Tr3 m01 = tr3_scaled(X0[2], XB[2], XA[2]);  // j_y, H_yz
                const float Hxx = tr3_m0(X0[3], XB[3], XA[3]);
                const float Hyy = tr3_m0(X0[4], XB[4], XA[4]);
                const float Hxy = tr3_m0(X0[5], XB[5], XA[5]);
                const float jx = m10.m0, jy = m01.m0, jz = m00.m1;
                const float inv = recip(1.0f + m00.m0);
                m[0] = m00.m0;
                m[1] = jx * inv;
                m[2] = jy * inv;
                m[3] = jz * inv;
                m[4] = fmaf(-m[1], jx, Hxx);
                m[5] = fmaf(-m[2], jy, Hyy);
                m[6] = fmaf(-m[3], jz, m00.m2);
                m[7] = fmaf(-m[1], jy, Hxy);
                m[8] = fmaf(-m[1], jz, m10.m1);
                m[9] = fmaf(-m[2], jz, m01.m1);
                each<6>([&](auto i_) {
                    constexpr int k = i_;
                    XA[k] = XC[k];
                    XB[k] = X1[k];
                    XC[k] = X2[k];
                });
            } else {
            // The populations of c_z = -1, 0, +1 sum to M, Z, P (X = X0 + c_z X1 +
            // (c_z^2 - 1/3) X2) and belong to planes r - 1, r, r + 1.  The plane r still
            // lacks the M of plane r + 1.  Kept for it: of rho', which needs all three z
            // moments, Z (ZA[0]) and P(r - 1) - Z (ZD[0]); of the others the weighted sum of
            // Z and P(r - 1) (ZA[1], ZA[2], ZQ), and of j_x and j_y, whose first z moment is
            // needed too, P(r - 1) itself (ZD[1], ZD[2]).  For the plane above: P (ZP).
            // rho' of the own column comes back last, one rounding at its magnitude, which
            // also keeps the density of a uniform stream from creeping by rounding (a
            // tenth of an ulp a step stays below what the sum resolves).  With variable
            // density p* is larger than the stress by far: there the sums stay without it
            // and the exact differences between planes (dr, from ZR) enter, with which a
            // droplet at density ratio 1:10 keeps its stress within 5.7e-6 of the oracle
            // after 200 steps (1.1e-5 with p* added in, in an earlier form).
            // Elsewhere the large term comes in last, so that M, P and the weighted sums are
            // rounded once at its magnitude.  With that, the differences of xy_moments and J rounded
            // once, the rms error of the stress against binary64 is, after ten steps of a
            // 256^3 vortex 8.3e-10 (9.2e-10 with Z, P - Z and a rounding more in each of M,
            // P and J; 8.5e-10 where 27 populations are summed), of a 128 x 128 x 256 jet
            // 2.26e-10 (2.33e-10, 2.28e-10); of the velocity 2.5e-9 and 1.11e-9 (5.7e-9 and
            // 1.16e-9, 5.7e-9 and 1.20e-9).
            // In this order (held by the empty asm statements) each carried value is
            // formed in the register of the one it replaces.
            float M[6];
            each<6>([&](auto i_) {
                constexpr int k = i_;
                M[k] = k ? X0[k] + fmaf(X2[k], 2.0f / 3.0f, -X1[k]) : fmaf(X2[k], 2.0f / 3.0f, X0[k]) - X1[k];
            });
            if constexpr (VD)
                dr = rpc - ZR;
            else
                M[0] += rpc;
            // (X carries the factors 1, 6, 6, 9, 9, 36 of xy_moments)
            const float d00 = VD ? (M[0] - ZA[0]) + dr : M[0] - ZA[0];
            const float s00 = d00 + ZD[0];
            const float drho = VD ? ZR + fmaf(s00, 1.0f / 6.0f, ZA[0]) : fmaf(s00, 1.0f / 6.0f, ZA[0]);
            const float jz = (ZD[0] - d00) * (1.0f / 6.0f), Hzz = s00 * (1.0f / 9.0f);
            const float jx = fmaf(M[1], 1.0f / 36.0f, ZA[1]), Hxz = (ZD[1] - M[1]) * (1.0f / 36.0f);
            const float jy = fmaf(M[2], 1.0f / 36.0f, ZA[2]), Hyz = (ZD[2] - M[2]) * (1.0f / 36.0f);
            const float Hxx = fmaf(M[3], 1.0f / 54.0f, ZQ[0]);
            const float Hyy = fmaf(M[4], 1.0f / 54.0f, ZQ[1]);
            const float Hxy = fmaf(M[5], 1.0f / 216.0f, ZQ[2]);
            const float inv = VD ? 1.0f : recip(1.0f + drho);
            m[0] = drho;
            m[1] = jx * inv;
            m[2] = jy * inv;
            m[3] = jz * inv;
            m[4] = fmaf(-m[1], jx, Hxx);
            m[5] = fmaf(-m[2], jy, Hyy);
            m[6] = fmaf(-m[3], jz, Hzz);
            m[7] = fmaf(-m[1], jy, Hxy);
            m[8] = fmaf(-m[1], jz, Hxz);
            m[9] = fmaf(-m[2], jz, Hyz);
            }
            // streamed phase, held to the clamp range (a stable run never reaches it)
            phin = PH ? phi_clamp(PA + pdown) : 0;
            each<10>([&](auto i_) {
                constexpr int k = i_;
                keep_here(m[k]);
            });
            __asm__ volatile("" : "+v"(phin));
            if constexpr (PH) {
                PA = PC + prest + pin;
                PC = pup;
            }
            if constexpr (!H) {
            each<6>([&](auto i_) {
                constexpr int k = i_;
                keep_here(X0[k], X2[k]);
            });
            ZA[0] = fmaf(X2[0], -1.0f / 3.0f, X0[0]);
            if (!VD) ZA[0] += rpc;
            ZD[0] = VD ? (ZP[0] - ZA[0]) - dr : ZP[0] - ZA[0];
            keep_here(ZA[0], ZD[0]);
            each<5>([&](auto i_) {
                constexpr int k = i_ + 1;  // weights (1, 4, 1)/6 over the factor of X
                constexpr float c = k < 3 ? 1.0f / 36.0f : k < 5 ? 1.0f / 54.0f : 1.0f / 216.0f;
                constexpr float c3 = k < 3 ? 1.0f / 27.0f : k < 5 ? 2.0f / 81.0f : 1.0f / 162.0f;  // 4 c / 3
                float &sum = k < 3 ? ZA[k % 3] : ZQ[k % 3];
                sum = fmaf(X0[k], 4.0f * c, fmaf(X2[k], -c3, ZP[k] * c));
                keep_here(sum);
                if constexpr (k < 3) {
                    ZD[k] = ZP[k];
                    keep_here(ZD[k]);
                }
            });
            each<6>([&](auto i_) {
                constexpr int k = i_;
                keep_here(X2[k]);
                ZP[k] = k ? X0[k] + fmaf(X2[k], 2.0f / 3.0f, X1[k]) : fmaf(X2[k], 2.0f / 3.0f, X0[k]) + X1[k];
            });
            if constexpr (VD)
                ZR = rpc;
            else
                ZP[0] += rpc;
            }
        }
        // After the destinations' arithmetic and before any store of the iteration:
        // wait for the loads issued at its top (vmcnt 0; expcnt and lgkmcnt fields at
        // their maxima, i.e. not waited for).
        // Loads and stores share one in-order counter, and the stores are conditional,
        // so a wait placed after them could only be vmcnt(0) and would also wait until
        // every store of the iteration has been acknowledged.  Here the loads have had
        // nearly the whole iteration to arrive, and the stores drain during the next one.
        __builtin_amdgcn_s_waitcnt(0x0F70);
        // (an opaque copy: with the same condition the two blocks are joined into one, the
        // wait is doubled, and a path without it is left on paper, for which the compiler
        // then waits at the top of the loop, stores included)
        int storing = __builtin_amdgcn_readfirstlane((int)finish);
        __asm__ volatile("" : "+s"(storing));
        if (storing) {
            const int zd = r - 1;
            const bool z_image = !g.per[2] && (zd == 1 || zd == g.nz - 2);
            if (zd >= z0 && zd < z1 && (g.per[2] || (zd > 0 && zd < g.nz - 1))) {
                int e = __builtin_amdgcn_readfirstlane(edge);
                __asm__ volatile("" : "+s"(e));  // tested here, not kept as four masks
                const bool images = z_image || y_image;
                if (e) {
                    take_over(e, lane_f, m, phin);
                    if (!images)
                        each<10>([&](auto i_) {
                            constexpr int k = i_;
                            if (k < 4 || k > 6)
                                m[k] = __uint_as_float(__float_as_uint(m[k]) & (uint32_t)((int32_t)(keep << (31 - k)) >> 31));
                        });
                }
                if (!images) {
                    if (own) {
                        store_plane<ST, PH, NT>(out, g.ld, plane * zd, off_dst, m, phin, sc);
                    }
                } else {
                    // the node itself (v = 0) and its images: on the z wall next to plane
                    // zd (v & 1) and in the last row of an odd low lattice (v & 2).  x_F of
                    // an edge node is interior in every coordinate, so each is made from
                    // the moments before any rule.
                    const bool yi = y_image && gys == g.ny - 2;
#pragma unroll 1
                    for (int v = 0; v < (y_image ? 4 : 2); ++v) {
                        if ((v & 1) && !z_image) continue;
                        if (!own || ((v & 2) && !yi)) continue;
                        const int Y = (v & 2) ? g.ny - 1 : gys;
                        const int Zp = !(v & 1) ? zd : (zd == 1 ? 0 : g.nz - 1);
                        float mb[10];
                        each<10>([&](auto i_) {
                            constexpr int k = i_;
                            mb[k] = m[k];
                        });
                        int32_t pb = phin;
                        const int face = boundary_face(g, gxs, Y, Zp);
                        const uint32_t rule = face < 0 ? 0u : (rules >> (4 * face)) & 15u;
                        if (rule == 2u)
                            apply_inlet(*walls, g, gxs, Y, step_next, mb, pb);
                        else
                            apply_rule(rule, face >> 1, mb);
                        const uint32_t off = (uint32_t)gxs + (uint32_t)g.nx * (uint32_t)Y;
                        store_plane<ST, PH, NT>(out, g.ld, plane * Zp, off, mb, pb, sc);
                    }
                }
            }
        }
        __syncthreads();
    }
}


static_assert(sizeof(Geo) % alignof(Phys) == 0 && alignof(Geo) == alignof(Phys), "ph follows g directly");
// `first` is the first work item of a launch that is one of several.  PART: it is used.
// As an argument of every launch it moved the compiler's registers about in the other
// loops: two components FP16Q 2 % and FP16 1 to 2 % slower (128^3 droplet 52.2 and 53.4 us
// a step, 100 x 100 x 200 jet 72.8 and 74.4), BF16 2 % faster (131 x 77 x 301 jet 98.1 and
// 100.1), one component up to 4 % faster.  So it always is for the latter two, and a kernel
// of its own does the rest.
template <int ST, bool PH> constexpr bool takes_first = !PH || ST == ST_BF16;
template <int ST, bool PH, bool VD, int ROWS, bool NT, bool PART>
__global__ __launch_bounds__(Tile<ROWS>::threads(PH), (waves_per_simd<ST, PH>)) void k_step_fused(Geo g, Phys ph, Scales sc, StateView in, StateView out,
                                                               int lz, int tiles_x, int tiles_y,
                                                               unsigned long long step_next, int first) {
    __shared__ Smem<PH, VD, ROWS, by_direction<ST, PH>> sm;
    // ph sits behind g in the kernel's argument segment
    const PhysMem walls = (PhysMem)((const __attribute__((address_space(4))) char *)__builtin_amdgcn_kernarg_segment_ptr() +
                                    sizeof(Geo));
    step_fused<ST, PH, false, VD, ROWS, NT>(sm, g, ph, walls, sc, in, out, lz, tiles_x, tiles_y, step_next,
                                               (PART ? first : 0) + xcd_work_item(blockIdx.x, gridDim.x));
}

// Several lattices in one launch: the work items of domain k are
// [work_begin, work_begin + tiles * chunks); domains are sorted by work_begin.
template <int ST, bool PH, bool VD, int ROWS, bool NT>
__global__ __launch_bounds__(Tile<ROWS>::threads(PH), (waves_per_simd<ST, PH>)) void k_step_fused_multi(const FusedDomain *__restrict__ doms, int ndom, int first) {
    __shared__ Smem<PH, VD, ROWS, by_direction<ST, PH>> sm;
    const int w = first + xcd_work_item(blockIdx.x, gridDim.x);
    int lo = 0, hi = ndom - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (doms[mid].work_begin <= w)
            lo = mid;
        else
            hi = mid - 1;
    }
    const FusedDomain &d = doms[lo];
    // Every field is read once, here, into fresh local objects.  Used through the
    // reference instead, the record's fields are loaded where the step needs them,
    // inside the plane loop (the loads sit in conditional code, so the compiler
    // does not hoist them), together with the 64-bit products derived from them;
    // copied as a whole, the record stays in scratch memory.  Field by field, the
    // step compiles to the same loop as the single-lattice kernel.
    Geo g;
    g.nx = d.g.nx; g.ny = d.g.ny; g.nz = d.g.nz;
    g.per[0] = d.g.per[0]; g.per[1] = d.g.per[1]; g.per[2] = d.g.per[2];
    g.N = d.g.N; g.ld = d.g.ld;
    Phys ph;
    ph.omega = d.ph.omega; ph.sigma = d.ph.sigma; ph.gamma = d.ph.gamma; ph.eps = d.ph.eps;
    ph.bc[0] = d.ph.bc[0]; ph.bc[1] = d.ph.bc[1]; ph.bc[2] = d.ph.bc[2];
    ph.bc[3] = d.ph.bc[3]; ph.bc[4] = d.ph.bc[4]; ph.bc[5] = d.ph.bc[5];
    if constexpr (VD) {
        ph.rho_b = d.ph.rho_b; ph.drho = d.ph.drho; ph.nu_b = d.ph.nu_b; ph.dnu = d.ph.dnu;
        ph.grav[0] = d.ph.grav[0]; ph.grav[1] = d.ph.grav[1]; ph.grav[2] = d.ph.grav[2];
    }
    Scales sc;
    sc.s2 = d.sc.s2; sc.s1 = d.sc.s1; sc.inv_s2 = d.sc.inv_s2; sc.inv_s1 = d.sc.inv_s1;
    StateView in, out;
    in.mom = d.in.mom; in.phi = d.in.phi; out.mom = d.out.mom; out.phi = d.out.phi;
    const int lz = d.lz, tx = d.tiles_x, ty = d.tiles_y, wb = d.work_begin;
    const unsigned long long sn = d.step_next;
    step_fused<ST, PH, true, VD, ROWS, NT>(sm, g, ph, (PhysMem)&d.ph, sc, in, out, lz, tx, ty, sn, w - wb);
}

}  // namespace fused

bool fused_wide_allowed(const tslb_ctx *c) { return c->phase && !c->vd; }

namespace {

PlanShape shape_of(const tslb_ctx *c) {
    static_assert(fused::Tile<16>::TX == kTileX && fused::Tile<20>::TX == kTileX, "tiles of the plan");
    return {c->geo.nx, c->geo.ny, c->geo.nz, c->phase, fused_wide_allowed(c), c->storage != ST_FP32, c->cu_count};
}

}  // namespace

FusedPlan fused_plan(const tslb_ctx *c) { return plan_fused(shape_of(c), c->chunk_z, c->tile_rows); }

long long fused_walk2(const tslb_ctx *c, int lz) { return fused_walk2(shape_of(c), lz); }

bool fused_stream_stores(const tslb_ctx *c, size_t launch_bytes) { return stream_stores(shape_of(c), launch_bytes); }

int fused_chunk(const tslb_ctx *c) { return c->plan_lz; }

int fused_rows(const tslb_ctx *c) { return c->plan_rows; }

int fused_work_items(const tslb_ctx *c, int lz) {
    return (int)(fused_tiles(shape_of(c), fused_rows(c)) * chunk_count(c->geo.nz, lz));
}

FusedDomain fused_domain(const tslb_ctx *c, StateView in, StateView out, int64_t step_next, int work_begin,
                         int lz) {
    FusedDomain d;
    d.g = c->geo;
    d.ph = c->phys;
    d.sc = c->scales;
    d.in = in;
    d.out = out;
    d.step_next = (unsigned long long)step_next;
    d.lz = lz > 0 ? lz : c->plan_lz;
    d.tiles_x = (c->geo.nx + fused::Tile<16>::TX - 1) / fused::Tile<16>::TX;
    d.tiles_y = (c->geo.ny + c->plan_rows - 1) / c->plan_rows;
    d.work_begin = work_begin;
    d.work_count = fused_work_items(c, d.lz);
    return d;
}

// Launch the fused step over the whole lattice, in as many launches as its work items
// need (launch_blocks).
namespace {

template <int ST, bool PH, bool VD, int ROWS>
void launch_one(long long items, hipStream_t s, const tslb_ctx *c, StateView in, StateView out, int lz, int tiles_x,
                int tiles_y, unsigned long long sn) {
    using namespace fused;
    constexpr int threads = Tile<ROWS>::threads(PH);
    constexpr bool part = takes_first<ST, PH>;
    const bool nt = fused_stream_stores(c, c->buffer_bytes), several = launch_blocks(items, threads) < items;
    const auto kernel = several && !part ? k_step_fused<ST, PH, VD, ROWS, true, true>
                        : nt             ? k_step_fused<ST, PH, VD, ROWS, true, part>
                                         : k_step_fused<ST, PH, VD, ROWS, false, part>;
    for (long long first = 0, n; first < items; first += n) {
        n = launch_blocks(items - first, threads);
        hipLaunchKernelGGL(kernel, dim3((unsigned)n), dim3(threads), 0, s, c->geo, c->phys, c->scales, in, out, lz,
                           tiles_x, tiles_y, sn, (int)first);
    }
}

template <int ST, bool PH, bool VD, int ROWS>
void launch_multi(long long items, hipStream_t s, const FusedDomain *doms, int ndom, bool nt) {
    using namespace fused;
    constexpr int threads = Tile<ROWS>::threads(PH);
    for (long long first = 0, n; first < items; first += n) {
        n = launch_blocks(items - first, threads);
        hipLaunchKernelGGL((nt ? k_step_fused_multi<ST, PH, VD, ROWS, true> : k_step_fused_multi<ST, PH, VD, ROWS, false>),
                           dim3((unsigned)n), dim3(threads), 0, s, doms, ndom, (int)first);
    }
}

}  // namespace

hipError_t launch_step_fused(const tslb_ctx *c, StateView in, StateView out, int lz, int64_t step_next,
                             hipStream_t s) {
    const int rows = fused_rows(c);
    const int tiles_x = (c->geo.nx + fused::Tile<16>::TX - 1) / fused::Tile<16>::TX;
    const int tiles_y = (c->geo.ny + rows - 1) / rows;
    const long long items = fused_work_items(c, lz);
    const unsigned long long sn = (unsigned long long)step_next;
    if (c->vd) {  // variable density: two components, 16 rows (validated at creation)
        if (!c->phase || rows != 16) return hipErrorInvalidValue;
        launch_one<ST_FP32, true, true, 16>(items, s, c, in, out, lz, tiles_x, tiles_y, sn);
        return hipGetLastError();
    }
#define TSLB_FUSED_CASE(ST)                                                                            \
    case ST:                                                                                           \
        if (!c->phase)                                                                                 \
            launch_one<ST, false, false, 16>(items, s, c, in, out, lz, tiles_x, tiles_y, sn);         \
        else if (rows == 20)                                                                           \
            launch_one<ST, true, false, 20>(items, s, c, in, out, lz, tiles_x, tiles_y, sn);          \
        else                                                                                           \
            launch_one<ST, true, false, 16>(items, s, c, in, out, lz, tiles_x, tiles_y, sn);          \
        break;
    switch (c->storage) {
        TSLB_FUSED_CASE(ST_FP32)
        TSLB_FUSED_CASE(ST_FP16)
        TSLB_FUSED_CASE(ST_BF16)
        TSLB_FUSED_CASE(ST_FP16Q)
    default:
        return hipErrorInvalidValue;
    }
#undef TSLB_FUSED_CASE
    return hipGetLastError();
}

hipError_t launch_step_fused_multi(const FusedDomain *doms, int ndom, int total_work, int storage, bool phase,
                                   bool vd, int rows, bool nt, hipStream_t s) {
    if (ndom <= 0 || total_work <= 0) return hipSuccess;
    if (vd) {
        if (!phase || rows != 16 || storage != ST_FP32) return hipErrorInvalidValue;
        launch_multi<ST_FP32, true, true, 16>(total_work, s, doms, ndom, nt);
        return hipGetLastError();
    }
    if (rows != 16 && (rows != 20 || !phase)) return hipErrorInvalidValue;
#define TSLB_MULTI_CASE(ST)                                                                            \
    case ST:                                                                                           \
        if (!phase)                                                                                    \
            launch_multi<ST, false, false, 16>(total_work, s, doms, ndom, nt);                                 \
        else if (rows == 20)                                                                           \
            launch_multi<ST, true, false, 20>(total_work, s, doms, ndom, nt);                                  \
        else                                                                                           \
            launch_multi<ST, true, false, 16>(total_work, s, doms, ndom, nt);                                  \
        break;
    switch (storage) {
        TSLB_MULTI_CASE(ST_FP32)
        TSLB_MULTI_CASE(ST_FP16)
        TSLB_MULTI_CASE(ST_BF16)
        TSLB_MULTI_CASE(ST_FP16Q)
    default:
        return hipErrorInvalidValue;
    }
#undef TSLB_MULTI_CASE
    return hipGetLastError();
}

}  // namespace tslb
