// pond_stream.h -- the predictor-corrector passes of the semi-Lagrangian streaming
// (eqs. 1-4, App. C-D) and the store of the streamed state, shared by the two-kernel
// streaming kernel (k_stream) and the fused step kernel (k_step).  The moment fields of
// a tile and its 2-node halo sit in LDS as written by the kernels' fill stages, field
// (m, n) of both sets at window node li at pair_at<DIM, LdsT, LN>(3 m + n, li).
//
// A receiver has one lane, or two (lanes i and i + 32 of a wave, half 0 and 1).  In two
// dimensions a lane works on both sets, so a window value of f and g is one LDS read; two
// lanes take half of the window's rows each, and half 0 then keeps the finished f
// populations, half 1 g's.
#pragma once

#include <type_traits>
#include <utility>

#include "pond_collide.h"
#include "pond_device.h"

namespace pond {

// f(0), f(1), .. f(N - 1) with the index as a type: unrolled whatever the size of the body
template <typename F, int... I> __device__ __forceinline__ void unrolled(std::integer_sequence<int, I...>, F f)
{
    (f(std::integral_constant<int, I>{}), ...);
}

// ---------------------------------------------------------------------------
// lanes and receivers: 32 lanes hold 32 consecutive receivers of the tile (x fastest).  A
// 16-byte LDS read serves them in two groups, lanes 0-3, 12-15, 20-27 and the others (even
// and odd parity of lane bits 2-4; measured), and each group takes sixteen neighbouring
// receivers, whose reads touch every bank once: with the receivers in lane order, rows of
// sixteen nodes cost half the LDS time in bank conflicts.
// ---------------------------------------------------------------------------
template <int LANES> __device__ __forceinline__ int lane_receiver(int tid)
{
    const int group = ((tid >> 2) ^ (tid >> 3) ^ (tid >> 4)) & 1;
    return (LANES == 2 ? tid >> 6 : tid >> 5) * 32 + group * 16 + ((tid >> 3) & 3) * 4 + (tid & 3);
}
template <int LANES> __device__ __forceinline__ int lane_half(int tid) { return LANES == 2 ? (tid >> 5) & 1 : 0; }

// a = [a of half 0 | b of half 0], b = [a of half 1 | b of half 1]
__device__ __forceinline__ void swap_halves(double &a, double &b)
{
    const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(a), __double2loint(b), false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(a), __double2hiint(b), false, false);
    a = __hiloint2double(hi[0], lo[0]);
    b = __hiloint2double(hi[1], lo[1]);
}
// the value of half 0 and of half 1, in both
__device__ __forceinline__ void both_halves(double v, double &v0, double &v1)
{
    v0 = v1 = v;
    swap_halves(v0, v1);
}
__device__ __forceinline__ double sum_halves(double v)
{
    double w = v;
    swap_halves(v, w);
    return v + w;
}

// ---------------------------------------------------------------------------
// LDS layout of the moment fields.  FP64 and 1D: (f, g) pairs, field by field; FP32: (f_0, g_0,
// f_1, g_1) and (f_2, g_2) of each n (index m).  So a lane reads 16 bytes at a time (8 for
// the last field in FP32), the lanes of a half wave side by side: 240 bytes a clock and CU,
// where 8-byte reads move 125.
// ---------------------------------------------------------------------------
template <int DIM, typename T, int LN> __device__ __forceinline__ constexpr int pair_at(int i, int li)
{
    if (DIM == 1 || sizeof(T) == 8) return (i * LN + li) * 2;
    const int m = i / 3, n = i % 3;
    return m < 2 ? (n * LN + li) * 4 + 2 * m : 12 * LN + (n * LN + li) * 2;
}
// the three fields of window column `off` nodes from a row base (n, node)
template <typename T, int LN> struct PairRow;
template <int LN> struct PairRow<double, LN> {
    const double2 *p;
    __device__ __forceinline__ PairRow(const double *lds, int n, int node) : p((const double2 *)lds + (n * LN + node)) {}
    __device__ __forceinline__ void load(int off, double f[3], double g[3]) const
    {
#pragma unroll
        for (int m = 0; m < 3; ++m) {
            const double2 v = p[3 * m * LN + off];
            f[m] = v.x;
            g[m] = v.y;
        }
    }
};
template <int LN> struct PairRow<float, LN> {
    const float4 *p01;
    const float2 *p2;
    __device__ __forceinline__ PairRow(const float *lds, int n, int node)
        : p01((const float4 *)lds + (n * LN + node)), p2((const float2 *)(lds + 12 * LN) + (n * LN + node))
    {
    }
    __device__ __forceinline__ void load(int off, float f[3], float g[3]) const
    {
        const float4 v = p01[off];
        const float2 w = p2[off];
        f[0] = v.x, g[0] = v.y, f[1] = v.z, g[1] = v.w, f[2] = w.x, g[2] = w.y;
    }
};

// Keeps the arithmetic of a window in front of the closure that uses its results: the
// compiler would otherwise sink it into the closure's branches, away from its LDS reads
// (618 registers to scratch in an isothermal kernel).
template <int N> __device__ __forceinline__ void pin(double (&v)[N])
{
#pragma unroll
    for (int i = 0; i < N; ++i) asm volatile("" : "+v"(v[i]));
}

// The rows of a lane.  One lane a receiver: fifteen, the five of n = 0, 1, 2.  Two: the five
// rows of n = 0 (half 1: n = 2), then rows 0..2 (half 1: 2..4) of n = 1, whose middle row
// both halves take with half its weight.
template <int LANES> constexpr int kLaneRows = LANES == 2 ? 8 : 15;

// Calls use(row, column, f, g) for the columns of a lane's rows in order; each is read three
// columns ahead of its use, since the compiler by itself reads a column just before it
// needs it and waits, and two waves a SIMD do not cover that.  (Two ahead for one FP64 lane a
// receiver, whose registers are short: 2048^2 896 -> 862 us.)
template <int LANES, typename T, int LN, int LX, typename Use>
__device__ __forceinline__ void walk_rows(const T *lds, int node, int half, Use use)
{
    constexpr int kAhead = sizeof(T) == 8 && LANES == 1 ? 2 : 3, kColumns = 5 * kLaneRows<LANES>;
    const PairRow<T, LN> A(lds, half ? 2 : 0, node), B(lds, 1, node + (half ? 2 * LX : 0)), C(lds, 2, node);
    T f[kAhead][3], g[kAhead][3];
    auto load = [&](int i) {
        const int r = i / 5 % 5, c = i % 5;
        (i < 25 ? A : i < 50 ? B : C).load(r * LX + c, f[i % kAhead], g[i % kAhead]);
    };
#pragma unroll
    for (int i = 0; i < kAhead; ++i) load(i);
    unrolled(std::make_integer_sequence<int, kColumns>{}, [&](auto ii) __attribute__((always_inline)) {
        constexpr int i = decltype(ii)::value;
        use(std::integral_constant<int, i / 5>{}, std::integral_constant<int, i % 5>{}, f[i % kAhead], g[i % kAhead]);
        if constexpr (i + kAhead < kColumns) load(i + kAhead);
        __builtin_amdgcn_sched_barrier(0);
    });
}

// The y taps and Lagrange coefficients of a lane's rows
template <int LANES> struct LaneRows;
template <> struct LaneRows<1> {
    const double (&w)[3][5];
    const double (&C)[3][3];
    __device__ __forceinline__ LaneRows(int, const double (&wy)[3][5], const double (&Cy)[3][3]) : w(wy), C(Cy) {}
    __device__ __forceinline__ double tap(int j, int l) const { return w[l][j % 5]; }
    __device__ __forceinline__ double weight(int j, int l) const { return C[l][j / 5] * w[l][j % 5]; }
};
template <> struct LaneRows<2> {
    double w[3][5], wb[3][3], B[3], B1[3]; // [l][row]; C of n = 0 (half 1: n = 2), of n = 1
    double share[3];
    __device__ __forceinline__ LaneRows(int half, const double (&wy)[3][5], const double (&C)[3][3])
    {
        share[0] = half ? 0.5 : 1.0;
        share[1] = 1.0;
        share[2] = half ? 1.0 : 0.5;
#pragma unroll
        for (int l = 0; l < 3; ++l) {
#pragma unroll
            for (int j = 0; j < 5; ++j) w[l][j] = wy[l][j];
#pragma unroll
            for (int j = 0; j < 3; ++j) wb[l][j] = half ? wy[l][2 + j] : wy[l][j];
            B[l] = half ? C[l][2] : C[l][0];
            B1[l] = C[l][1];
        }
    }
    // tap of row j, and its product with the coefficient of its n
    __device__ __forceinline__ double tap(int j, int l) const
    {
        return j < 5 ? w[l][j] : j == 6 ? wb[l][1] : share[j - 5] * wb[l][j - 5];
    }
    __device__ __forceinline__ double weight(int j, int l) const
    {
        return j < 5 ? B[l] * w[l][j] : j == 6 ? B1[l] * wb[l][1] : (share[j - 5] * B1[l]) * wb[l][j - 5];
    }
};

// Populations of both sets at the departure points, this lane's rows:
//   f_kl += sum_n B_ln sum_r wy_l[r] sum_m A_km sum_c wx_k[c] M_mn[r][c]
// FAST leaves out the zero taps: each cubic stencil covers four of the five window columns,
// and for the directions c = -1 and +1 the unused one is the first (k = 0) or the last (k =
// 2) whenever the gauge velocity lies in (-s, s].  FP64 rows go straight into the
// accumulators; FP32 rows of one n are summed in FP32 and then added in FP64.
// The coefficients A_km stay outside the taps: folded into them the window has nine FMA a
// row less, but their FP32 products, each rounded by itself, no longer cancel over the
// directions as the A_km do (a 256^2 droplet after 20 000 steps was 4e-5 off in rho instead
// of 7e-6), and in FP64 it ran no faster (1.5% slower at 2048^2, 7% at 256^2).
template <int LANES, bool FAST, typename T, int LN, int LX>
__device__ __forceinline__ void window_pops(const T *lds, int node, int half, const double (&wx)[3][5],
                                            const double (&wy)[3][5], const double (&A)[3][3],
                                            const double (&B)[3][3], double dy, double s, double (&f)[9],
                                            double (&g)[9])
{
    constexpr bool kF32 = sizeof(T) == 4;
    const LaneRows<LANES> rows(half, wy, B);
    T w[3][5], a[3][3], tf[3][3], tg[3][3], zf[3], zg[3], F[9], G[9];
    // FP32: the taps, rounded once; two lanes in FP64: the products, fewer than their factors
    constexpr bool kKeep = kF32 || LANES == 2;
    T taps[kKeep ? kLaneRows<LANES> : 1][3];
    if constexpr (kKeep) {
#pragma unroll
        for (int j = 0; j < kLaneRows<LANES>; ++j)
#pragma unroll
            for (int l = 0; l < 3; ++l) taps[j][l] = (T)(kF32 ? rows.tap(j, l) : rows.weight(j, l));
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
#pragma unroll
        for (int c = 0; c < 5; ++c) w[k][c] = (T)wx[k][c];
#pragma unroll
        for (int m = 0; m < 3; ++m) a[k][m] = (T)A[k][m];
    }
    walk_rows<LANES, T, LN, LX>(lds, node, half, [&](auto jj, auto cc, const T(&vf)[3], const T(&vg)[3]) __attribute__((always_inline)) {
        constexpr int j = decltype(jj)::value, c = decltype(cc)::value;
        constexpr int n = j / 5, r = j % 5;
        constexpr bool whole = LANES == 1 || n == 0; // all five rows of an n: its zero taps are known
#pragma unroll
        for (int m = 0; m < 3; ++m)
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                if (FAST && ((k == 0 && c == 0) || (k == 2 && c == 4))) continue; // zero taps
                const bool first = FAST && k == 0 ? c == 1 : c == 0;
                tf[k][m] = first ? w[k][c] * vf[m] : tf[k][m] + w[k][c] * vf[m];
                tg[k][m] = first ? w[k][c] * vg[m] : tg[k][m] + w[k][c] * vg[m];
            }
        if constexpr (c != 4) return;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            zf[k] = a[k][0] * tf[k][0] + a[k][1] * tf[k][1] + a[k][2] * tf[k][2];
            zg[k] = a[k][0] * tg[k][0] + a[k][1] * tg[k][1] + a[k][2] * tg[k][2];
        }
#pragma unroll
        for (int l = 0; l < 3; ++l) {
            if (FAST && whole && ((l == 0 && r == 0) || (l == 2 && r == 4))) continue; // zero taps
            const T q = kKeep ? taps[kKeep ? j : 0][l] : (T)rows.weight(j, l);
            const bool first = (FAST && whole && l == 0 ? r == 1 : r == 0) && (kF32 || n == 0);
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                F[3 * k + l] = first ? q * zf[k] : F[3 * k + l] + q * zf[k];
                G[3 * k + l] = first ? q * zg[k] : G[3 * k + l] + q * zg[k];
            }
        }
        // FP32: the rows of an n, complete, into the FP64 sums.  Its coefficients are computed
        // here (the inputs pass an empty asm) rather than kept through the window
        if constexpr (kF32 && (r == 4 || j + 1 == kLaneRows<LANES>)) {
            double d = dy, v = s, C[3][3], b[3];
            asm volatile("" : "+v"(d), "+v"(v));
            lagrange_coeffs(d, v, C);
#pragma unroll
            for (int l = 0; l < 3; ++l) b[l] = LANES == 1 ? C[l][n] : n == 1 ? C[l][1] : half ? C[l][2] : C[l][0];
#pragma unroll
            for (int i = 0; i < 9; ++i) {
                f[i] = n == 0 ? b[i % 3] * (double)F[i] : f[i] + b[i % 3] * (double)F[i];
                g[i] = n == 0 ? b[i % 3] * (double)G[i] : g[i] + b[i % 3] * (double)G[i];
            }
        }
    });
    if constexpr (!kF32) {
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            f[i] = F[i];
            g[i] = G[i];
        }
    }
}

// Sums of the populations at the departure points, this lane's rows: S = rho, J_x, J_y
// (J = sum f c, c the direction: the momentum is U rho + s J) and 2 rho E = sum g.  They
// separate: with the x weights folded over the directions,
//   a0_m[c] = sum_k A_km wx_k[c],  a1_m[c] = sum_k (k - 1) A_km wx_k[c],
// and b0, b1 likewise in y, rho = sum M b0 a0, J_x = sum M b0 a1, J_y = sum M b1 a0: 49 FMA
// a row for both sets where the populations take 114.  Rows are added in FP64.  A further pass
// of 256^2 in FP64 so costs 4.3 us where one of populations cost 5.9.
template <int LANES, typename T, int LN, int LX>
__device__ __forceinline__ void window_sums(const T *lds, int node, int half, const double (&wx)[3][5],
                                            const double (&wy)[3][5], const double (&A)[3][3],
                                            const double (&B)[3][3], double (&S)[4])
{
    const LaneRows<LANES> rows(half, wy, B);
    T a0[3][5], a1[3][5], x0, x1, xg;
#pragma unroll
    for (int m = 0; m < 3; ++m)
#pragma unroll
        for (int c = 0; c < 5; ++c) {
            const double lo = A[0][m] * wx[0][c], hi = A[2][m] * wx[2][c];
            a0[m][c] = (T)(lo + A[1][m] * wx[1][c] + hi);
            a1[m][c] = (T)(hi - lo);
        }
    walk_rows<LANES, T, LN, LX>(lds, node, half, [&](auto jj, auto cc, const T(&vf)[3], const T(&vg)[3]) __attribute__((always_inline)) {
        constexpr int j = decltype(jj)::value, c = decltype(cc)::value;
#pragma unroll
        for (int m = 0; m < 3; ++m) {
            const bool first = c == 0 && m == 0;
            x0 = first ? a0[m][c] * vf[m] : x0 + a0[m][c] * vf[m];
            x1 = first ? a1[m][c] * vf[m] : x1 + a1[m][c] * vf[m];
            xg = first ? a0[m][c] * vg[m] : xg + a0[m][c] * vg[m];
        }
        if constexpr (c != 4) return;
        const double q0 = rows.weight(j, 0), q1 = rows.weight(j, 1), q2 = rows.weight(j, 2);
        const double b0 = q0 + q1 + q2, b1 = q2 - q0;
        S[0] = j == 0 ? b0 * (double)x0 : S[0] + b0 * (double)x0;
        S[1] = j == 0 ? b0 * (double)x1 : S[1] + b0 * (double)x1;
        S[2] = j == 0 ? b1 * (double)x0 : S[2] + b1 * (double)x0;
        S[3] = j == 0 ? b0 * (double)xg : S[3] + b0 * (double)xg;
    });
}

// The passes of one receiver lane: interpolate the moment fields at the departure points
// of the receiver's gauge (Ux, Uy, th), contract them into populations in that gauge, and
// close their moments through the EoS for the next gauge, n_pass times; in two dimensions
// the passes before the last take the sums only.  `node` is the window corner (gx - 2, gy -
// 2).  FP32 windows (LdsT = float) hold deviations from the tile's reference moment vector
// R (1, v, v, v^2) (refR0, refR1 and refT = v, the per-axis second moment theta T_L of the
// centre's gauge).  On return f and g hold the populations in the gauge (sUx, sUy, sS) of the
// last pass (two lanes a receiver: f those of this half's set, f or g), and (Ux, Uy, th) the
// gauge it produced; returns the error bits.
template <int DIM, int LANES, typename LdsT, int LN, int LX, int NT, int LAW>
__device__ __forceinline__ int stream_passes(const POND_GLOBAL DevParams &P, const LdsT *lds, int node, int tid, int half,
                                             double rx, double ry, double refR0, double refR1, double refT, double &Ux,
                                             double &Uy, double &th, double Fpx, double Fpy,
                                             double (&f)[Layout<DIM>::Q], double (&g)[Layout<DIM>::Q], double &rho,
                                             double &sUx, double &sUy, double &sS)
{
    constexpr int Q = Layout<DIM>::Q;
    constexpr bool kDevI = sizeof(LdsT) == 4;
    static_assert(DIM == 2 || LANES == 2, "one dimension: a lane for each set");
    const double dt = P.dt;
    int err = 0;
    // closure of the sums (eq. 2) of a pass in the gauge (Ux, Uy, s): the next gauge
    auto close = [&](double s, double r0, double jx, double jy, double G2) {
        rho = r0;
        // one reciprocal of rho serves every quotient by it (FP64 division is a
        // long dependent sequence on this hardware); the lean van der Waals closure
        // takes it and 1 / (1 - b rho) from one division
        const double q = 1.0 - P.b * rho;
        const double i_rq = LAW != kLean ? 0.0 : 1.0 / (rho * q);
        const double i_rho = LAW != kLean ? 1.0 / rho : q * i_rq;
        const double E = 0.5 * G2 * i_rho;
        const double ux = jx * i_rho;
        const double uy = DIM == 2 ? jy * i_rho : 0.0;
        const double uhx = ux + 0.5 * Fpx * dt * i_rho;
        const double uhy = DIM == 2 ? uy + 0.5 * Fpy * dt * i_rho : 0.0;
        const double e = E - 0.5 * (uhx * uhx + uhy * uhy);
        const double T = eos_T_of_e<LAW>(P, rho, e);
        const double p = LAW != kLean ? eos_p<LAW>(P, rho, T) : vdw_p_lean(P, rho, T, i_rq);
        err |= eos_bad<LAW>(P, rho, p);
        sUx = Ux;
        sUy = Uy;
        sS = s;
        Ux = ux;
        Uy = uy;
        th = p * i_rho * kInvTL;
    };
    // When the grid is one workgroup per CU (512 lanes, two waves per SIMD), the SIMD
    // issues for the older wave first, the younger one falls behind and finishes its
    // last pass alone, with nothing to hide its latencies.  Favouring the younger wave
    // in the first pass lets both finish at about the same time.
    const int young = __builtin_amdgcn_readfirstlane((tid >> 6) >= NT / 128 && NT == 512 && gridDim.x <= kCUs ? 1 : 0);
    if (DIM == 2 && young) __builtin_amdgcn_s_setprio(1);
    // the passes before the last (one dimension takes populations in all of them: folding
    // its weights costs more than its fifteen taps)
#pragma unroll 1
    for (int pass = 0; DIM == 2 && pass + 1 < P.n_pass; ++pass) {
        const double s = sqrt(th);
        double wx[3][5], wy[3][5], A[3][3], B[3][3], S[4];
        err |= window_weights<double>(Ux, s, dt, wx) | window_weights<double>(Uy, s, dt, wy);
        lagrange_coeffs(Ux - rx, s, A);
        lagrange_coeffs(Uy - ry, s, B);
        window_sums<LANES, LdsT, LN, LX>(lds, node, half, wx, wy, A, B, S);
        pin(S);
#pragma unroll
        for (int i = 0; i < 4 && LANES == 2; ++i) S[i] = sum_halves(S[i]);
        // the reference's own sums: R at the velocity (rx, ry)
        const double r0 = kDevI ? refR0 + S[0] : S[0], G2 = kDevI ? refR1 + S[3] : S[3];
        const double jx = Ux * S[0] + s * S[1] + (kDevI ? rx * refR0 : 0.0);
        const double jy = Uy * S[0] + s * S[2] + (kDevI ? ry * refR0 : 0.0);
        close(s, r0, jx, jy, G2);
        __builtin_amdgcn_s_setprio(0);
    }
    int pass = DIM == 2 ? P.n_pass - 1 : 0;
    do {
        const double s = sqrt(th);
        double wx[3][5], wy[3][5], Ad[3][3], Bd[3][3];
        err |= window_weights<double>(Ux, s, dt, wx);
        lagrange_coeffs(Ux - rx, s, Ad);
        if constexpr (DIM == 2) {
            err |= window_weights<double>(Uy, s, dt, wy);
            lagrange_coeffs(Uy - ry, s, Bd);
            if (__all(wx[0][0] == 0.0 && wx[2][4] == 0.0 && wy[0][0] == 0.0 && wy[2][4] == 0.0))
                window_pops<LANES, true, LdsT, LN, LX>(lds, node, half, wx, wy, Ad, Bd, Uy - ry, s, f, g);
            else
                window_pops<LANES, false, LdsT, LN, LX>(lds, node, half, wx, wy, Ad, Bd, Uy - ry, s, f, g);
            pin(f);
            pin(g);
            // the reference part (see the fill), R a_k b_l, from coefficients computed again
            double ra[3], rb[3];
            if constexpr (kDevI) {
                double dx = Ux - rx, dy = Uy - ry, v = s, C[3][3];
                asm volatile("" : "+v"(dx), "+v"(dy), "+v"(v));
                lagrange_coeffs(dx, v, C);
#pragma unroll
                for (int k = 0; k < 3; ++k) ra[k] = C[k][0] + refT * C[k][2];
                lagrange_coeffs(dy, v, C);
#pragma unroll
                for (int k = 0; k < 3; ++k) rb[k] = C[k][0] + refT * C[k][2];
            }
#pragma unroll
            for (int q = 0; q < 9; ++q) {
                if constexpr (LANES == 2) { // half 0 completes f, half 1 g
                    swap_halves(f[q], g[q]);
                    f[q] += g[q];
                }
                if constexpr (kDevI) {
                    f[q] += (half ? refR1 : refR0) * ra[q / 3] * rb[q % 3];
                    if (LANES == 1) g[q] += refR1 * ra[q / 3] * rb[q % 3];
                }
            }
        } else {
#pragma unroll
            for (int k = 0; k < 3; ++k) f[k] = kDevI ? (half ? refR1 : refR0) * (Ad[k][0] + refT * Ad[k][2]) : 0.0;
#pragma unroll
            for (int m = 0; m < 3; ++m) {
                LdsT v[5];
#pragma unroll
                for (int c = 0; c < 5; ++c) v[c] = lds[pair_at<DIM, LdsT, LN>(m, node + c) + half];
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    const LdsT xk = (LdsT)wx[k][0] * v[0] + (LdsT)wx[k][1] * v[1] + (LdsT)wx[k][2] * v[2] +
                                    (LdsT)wx[k][3] * v[3] + (LdsT)wx[k][4] * v[4];
                    f[k] += Ad[k][m] * (double)xk;
                }
            }
        }
        // moments of the populations (eq. 2); two lanes: of this half's set, exchanged
        double r0 = 0.0, jx = 0.0, jy = 0.0, G2 = 0.0;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const double cx = DIM == 2 ? (double)(q / 3 - 1) : (double)(q - 1);
            const double cy = DIM == 2 ? (double)(q % 3 - 1) : 0.0;
            r0 += f[q];
            jx += f[q] * (Ux + s * cx);
            if (DIM == 2) jy += f[q] * (Uy + s * cy);
            if (LANES == 1) G2 += g[q];
        }
        if constexpr (LANES == 2) {
            double unused;
            both_halves(r0, r0, G2);
            both_halves(jx, jx, unused);
            if (DIM == 2) both_halves(jy, jy, unused);
        }
        close(s, r0, jx, jy, G2);
        if (DIM == 1) __builtin_amdgcn_s_setprio(0);
    } while (DIM == 1 && ++pass < P.n_pass);
    return err;
}

// Store the streamed state of a receiver for the collision, gauge free: rho and u (the f
// lane), and the central moments of the lane's set about u (moment planes of
// pond_internal.h, in FP64 or the mixed FP32 form).
template <int DIM, bool MIXED>
__device__ __forceinline__ void store_streamed(void *mom, size_t N, size_t node, int myset, const double *pq,
                                               double rho, double Ux, double Uy, double sUx, double sUy, double sS)
{
    using L = Layout<DIM>;
    using MIO = MomIO<DIM, MIXED>;
    constexpr int NF = L::NF;
    double mq[NF];
    moments_about<DIM>(pq, sUx - Ux, sUy - Uy, sS, mq);
    if (myset == 0) {
        MIO::store(mom, N, node, L::kRho, rho);
        MIO::store(mom, N, node, L::kUx, Ux);
        if constexpr (DIM == 2) {
            MIO::store(mom, N, node, L::kUy, Uy);
            MIO::store(mom, N, node, (L::kF + 0), mq[4]); // (1,1)
            MIO::store(mom, N, node, (L::kF + 1), mq[6]); // (2,0)
            MIO::store(mom, N, node, (L::kF + 2), mq[2]); // (0,2)
            MIO::store(mom, N, node, (L::kF + 3), mq[7]); // (2,1)
            MIO::store(mom, N, node, (L::kF + 4), mq[5]); // (1,2)
            MIO::store(mom, N, node, (L::kF + 5), mq[8]); // (2,2)
        } else {
            MIO::store(mom, N, node, L::kF, mq[2]);
        }
    } else {
#pragma unroll
        for (int i = 0; i < NF; ++i) MIO::store(mom, N, node, (L::kG + i), mq[i]);
    }
}

} // namespace pond
