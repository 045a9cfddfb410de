// Per-lane stepping logic of the field-line tracer (host + device).
//
// One call of lane_iterate() makes one trial step of one half line inside its
// current grid cell; the caller owns the cell coefficients and refetches them when
// the call reports a cell change. The same function runs in the tracer kernel and
// in the adjoint's replays of recorded segments (which capture the accepted steps
// through the event sink).
//
// Method: RKF45 (Fehlberg's 4(5) pair, fifth-order solution kept; Section 2.3) on
// dr/ds = B/|B| (Section 2.1, Eq. rb) with the Eq. tw integrand (Section 1) and the
// length as extra components. B and curl B come from the cell's trilinear
// interpolant (Section 2.2, Eq. interp) in monomial form. Position = cell index +
// local coordinates in [0,1]. A step whose straight-line guess reaches a face is
// taken with that face's normal coordinate as the independent variable, so it ends
// exactly on the face.
#pragma once

#include <float.h>
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

namespace fq {

template <typename T> struct Num;
template <> struct Num<float> {
    static __host__ __device__ __forceinline__ float fma_(float a, float b, float c)
    {
        return __builtin_fmaf(a, b, c);
    }
    static __host__ __device__ __forceinline__ float rsq(float x)
    {
#if defined(__HIP_DEVICE_COMPILE__)
        return __builtin_amdgcn_rsqf(x);
#else
        return 1.0f / sqrtf(x);
#endif
    }
    static __host__ __device__ __forceinline__ float rcp(float x)
    {
#if defined(__HIP_DEVICE_COMPILE__)
        return __builtin_amdgcn_rcpf(x);
#else
        return 1.0f / x;
#endif
    }
    static __host__ __device__ __forceinline__ float min_(float a, float b) { return __builtin_fminf(a, b); }
    static constexpr float ov = 1e-5f;        // overshoot of a step past a face that is kept
    // Method II: the gradient of the trilinear B/B jumps across a cell face, so an
    // overshoot d kept there moves U and V by d times that jump (first order, where
    // positions err by d^2): about two ulp of a local coordinate
    static constexpr float ov_tan = 1.2e-7f;
    static constexpr float tau = 1e-4f;       // |direction component| below this is tangent
    static constexpr float null_rel = 1e-30f; // |B|^2 below null_rel * max|B|^2 is a null
    static constexpr float gmin = 1e-4f;      // smallest usable d(coordinate)/ds on a landing
    static constexpr float hmin = 1e-6f;      // smallest plain step (reference lengths)
};
template <> struct Num<double> {
    static __host__ __device__ __forceinline__ double fma_(double a, double b, double c)
    {
        return __builtin_fma(a, b, c);
    }
    // 1/sqrt(x) and 1/x: the hardware estimates (relative error about 5e-8) refined
    // by one Newton-Raphson iteration each (to about 5e-15 relative, measured on
    // gfx950) instead of the IEEE division and square root sequences. Arguments are
    // positive normal |B|^2 values and direction components bounded away from zero
    // by the callers.
    static __host__ __device__ __forceinline__ double rsq(double x)
    {
#if defined(__HIP_DEVICE_COMPILE__)
        const double y = __builtin_amdgcn_rsq(x);
        return y * __builtin_fma(-0.5 * x * y, y, 1.5);
#else
        return 1.0 / sqrt(x);
#endif
    }
    static __host__ __device__ __forceinline__ double rcp(double x)
    {
#if defined(__HIP_DEVICE_COMPILE__)
        const double y = __builtin_amdgcn_rcp(x);
        return __builtin_fma(y, __builtin_fma(-x, y, 1.0), y);
#else
        return 1.0 / x;
#endif
    }
    static __host__ __device__ __forceinline__ double min_(double a, double b) { return __builtin_fmin(a, b); }
    static constexpr double ov = 1e-9;
    static constexpr double ov_tan = 1e-9;
    static constexpr double tau = 1e-9;
    static constexpr double null_rel = 1e-60;
    static constexpr double gmin = 1e-9;
    static constexpr double hmin = 1e-12;
};

// x^(1/10) for the step controller, which works on squared errors (accuracy of a
// few ulp is plenty: it only scales the next trial step)
__host__ __device__ __forceinline__ float pow01(float x)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_exp2f(0.1f * __builtin_amdgcn_logf(x));
#else
    return powf(x, 0.1f);
#endif
}

// x is computed where this stands. (The twist sum is used only where a step is accepted;
// left to itself the compiler moves the whole twist integrand there and holds every
// stage's position and field in registers until then.)
template <typename T> __host__ __device__ __forceinline__ void here_and_now(T &x)
{
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("" : "+v"(x));
#endif
}

template <typename T> __host__ __device__ __forceinline__ T mn(T a, T b) { return a < b ? a : b; }
template <typename T> __host__ __device__ __forceinline__ T mx(T a, T b) { return a > b ? a : b; }
template <typename T> __host__ __device__ __forceinline__ bool finite_(T x)
{
    return __builtin_isfinite(x);
}

// P(u,v,w) = c0 + c1 u + c2 v + c3 w + c4 uv + c5 uw + c6 vw + c7 uvw, 7 FMAs.
template <typename T>
__host__ __device__ __forceinline__ T poly(const T c[8], T u, T v, T w)
{
    using N = Num<T>;
    T a = N::fma_(c[5], w, c[1]);
    T b = N::fma_(c[6], w, c[2]);
    T d = N::fma_(c[7], w, c[4]);
    T e = N::fma_(c[3], w, c[0]);
    b = N::fma_(u, d, b);
    e = N::fma_(u, a, e);
    return N::fma_(v, b, e);
}

// Monomial coefficients from the 8 corner values f[x + 2y + 4z].
template <typename T>
__host__ __device__ __forceinline__ void coeffs(const T f[8], T c[8])
{
    c[0] = f[0];
    c[1] = f[1] - f[0];
    c[2] = f[2] - f[0];
    c[3] = f[4] - f[0];
    c[4] = (f[3] - f[1]) - (f[2] - f[0]);
    c[5] = (f[5] - f[1]) - (f[4] - f[0]);
    c[6] = (f[6] - f[2]) - (f[4] - f[0]);
    c[7] = ((f[7] - f[6]) - (f[5] - f[4])) - ((f[3] - f[2]) - (f[1] - f[0]));
}

// Direction (local units per reference length), twist integrand per reference
// length and |B|^2 at local point (u,v,w).
template <typename T, bool TW>
__host__ __device__ __forceinline__ void rhs(const T cb[3][8], const T cj[3][8], T u, T v, T w,
                                             T sgn, T rx, T ry, T rz, T twk, T &f0, T &f1, T &f2,
                                             T &ft, T &b2)
{
    using N = Num<T>;
    const T bx = poly<T>(cb[0], u, v, w);
    const T by = poly<T>(cb[1], u, v, w);
    const T bz = poly<T>(cb[2], u, v, w);
    b2 = N::fma_(bx, bx, N::fma_(by, by, bz * bz));
    const T inv = N::rsq(b2);
    const T s = sgn * inv;
    f0 = s * bx * rx;
    f1 = s * by * ry;
    f2 = s * bz * rz;
    if (TW) {
        const T jx = poly<T>(cj[0], u, v, w);
        const T jy = poly<T>(cj[1], u, v, w);
        const T jz = poly<T>(cj[2], u, v, w);
        const T jb = N::fma_(jx, bx, N::fma_(jy, by, jz * bz));
        ft = jb * (inv * inv) * twk;
    } else {
        ft = T(0);
    }
}

// State of one half line.
template <typename T> struct Lane {
    int c0, c1, c2;  // cell
    T p0, p1, p2;    // local coordinates in [0,1]
    T h, tol, sgn;   // step (reference lengths), error bound (grid spacings), direction
    double tw, len;  // twist and length (reference lengths) so far
    uint32_t trials;
    int force;       // 2*axis + (direction > 0) of a landing to try next, -1 = none
};

template <typename T> struct LaneConst {
    T rx, ry, rz;    // reference length / spacing per axis
    T twk;           // reference length / (4 pi)
    T bnull2;        // null-field threshold on |B|^2
    int nx, ny, nz;  // nodes per axis
    uint32_t max_steps;
};

// Method II (Section 2.1, Eq. rb2): the two tangent vectors U, V carried along the
// line, in local grid units (component a in units of the spacing of axis a), so
// that dU/ds = J U with J the Jacobian of the local direction field
// f = sgn R B/|B| (R = diag(rx, ry, rz)) with respect to the local coordinates.
template <typename T> struct Tan {
    T u[3], v[3];
};

// d/du, d/dv, d/dw of the cell polynomial P (see poly).
template <typename T>
__host__ __device__ __forceinline__ void dpoly(const T c[8], T u, T v, T w, T &du, T &dv, T &dw)
{
    using N = Num<T>;
    du = N::fma_(v, N::fma_(c[7], w, c[4]), N::fma_(c[5], w, c[1]));
    dv = N::fma_(u, N::fma_(c[7], w, c[4]), N::fma_(c[6], w, c[2]));
    dw = N::fma_(u, N::fma_(c[7], v, c[5]), N::fma_(c[6], v, c[3]));
}

// The rates of U and V at local point (u,v,w), per reference length: J U and J V
// with J = sgn R (I - b b^T) (dB/dp) / |B| and b = B/|B| (B given, inv = 1/|B|).
// The gradient of B/B is taken analytically on the cell's interpolant.
template <typename T>
__host__ __device__ __forceinline__ void tan_rates(const T cb[3][8], T u, T v, T w, T bx, T by,
                                                   T bz, T inv, T sgn, T rx, T ry, T rz,
                                                   const T U[3], const T V[3], T kU[3], T kV[3])
{
    using N = Num<T>;
    T d[3][3];  // d[i][j] = dB_i / dp_j
#pragma unroll
    for (int i = 0; i < 3; i++) dpoly<T>(cb[i], u, v, w, d[i][0], d[i][1], d[i][2]);
    const T b0 = bx * inv, b1 = by * inv, b2 = bz * inv;
    const T s = sgn * inv;
#pragma unroll
    for (int m = 0; m < 2; m++) {
        const T *X = m ? V : U;
        T *K = m ? kV : kU;
        T g[3];
#pragma unroll
        for (int i = 0; i < 3; i++) g[i] = N::fma_(d[i][0], X[0], N::fma_(d[i][1], X[1], d[i][2] * X[2]));
        const T bg = N::fma_(b0, g[0], N::fma_(b1, g[1], b2 * g[2]));
        K[0] = s * rx * N::fma_(-b0, bg, g[0]);
        K[1] = s * ry * N::fma_(-b1, bg, g[1]);
        K[2] = s * rz * N::fma_(-b2, bg, g[2]);
    }
}

// What the adjoint's replay captures of an accepted step: landing axis (-1 for a plain
// step), its signed length in the independent variable (arc length for a plain step,
// the axis coordinate for a landing) and the coordinates (bit q) it left past a box
// face and that were clamped onto it.
struct NoEvents {
    template <typename T> __host__ __device__ __forceinline__ void accepted(int, T, int) const {}
};

// Carry a coordinate that left [0,1] by a small amount into the neighbouring cell
// (on a box face it is clamped to the face, and `bit` is set in `clamped`). Returns
// true if the cell changed.
template <typename T>
__host__ __device__ __forceinline__ bool carry(int &c, T &p, int n, int &clamped, int bit)
{
    if (p > T(1)) {
        if (c < n - 2) {
            c++;
            p -= T(1);
            return true;
        }
        p = T(1);
        clamped |= bit;
    } else if (p < T(0)) {
        if (c > 0) {
            c--;
            p += T(1);
            return true;
        }
        p = T(0);
        clamped |= bit;
    }
    return false;
}

// Did the step leave [-ov, 1+ov] along this axis and come back? The coordinate
// along the step is modelled by the quadratic through its start (slope s1 = H k1)
// and its end (displacement D, s2 = D - s1); true if it has an interior extremum
// beyond the cell (its maximum if s2 < 0, else its minimum).
template <typename T>
__host__ __device__ __forceinline__ bool excursion(T p, T s1, T s2, T ov)
{
    // x(t) = p + s1 t + s2 t^2 on t in [0,1]; an interior extremum needs s1 s2 < 0 and
    // t* = -s1 / (2 s2) < 1, and lies at x* = p - s1^2 / (4 s2). Written without
    // divisions: with a = |s2| the conditions are |s1| < 2a and, for a maximum
    // (s2 < 0), s1^2 > 4a (1 + ov - p); for a minimum, s1^2 > 4a (p + ov).
    const T a = fabs(s2);
    const T room = s2 < T(0) ? (T(1) + ov) - p : p + ov;
    return (s1 * s2 < T(0)) & (fabs(s1) < T(2) * a) & (s1 * s1 > (T(4) * a) * room);
}

// One trial step. On return: fin_st >= 0 if the half line ended (status bits,
// fin_face = exit face or -1), need_load if the cell changed. n_acc counts
// accepted steps.
// Integration schemes (Section 2.3). RKF45 is adaptive; the two RK4 rules take a
// fixed step (L.tol holds it; the error bound is not used), cut short only by cell
// faces like every step here.
enum Scheme : int { SCH_RKF45 = 0, SCH_RK4 = 1, SCH_RK4_38 = 2 };

// M2: carry Method II's tangent vectors tn along (RKF45 only).
//
// The trial is one straight line of arithmetic: every case (a face crossed before the
// step, a landing not possible yet, a rejected step, a step that leaves the cell, an
// accepted one) is a predicate, and the state is written once at the end. The lanes of a
// wave take all the cases at once in almost every iteration, so a branch per case saved
// nothing and cost the copies of the lane state at each join. Branches remain only where
// a whole wave usually skips them: the box faces, a step that left its cell, a carried
// overshoot, the end of a line.
// Against a branch per case, bit for bit the same lines: a 1024 x 1024 map of a
// 256x256x128 FP32 cube 6.97 -> 5.47 ms (FP64 11.9 -> 8.46 ms, Method II at 512 x 512
// 7.57 -> 5.60 ms), a 256x256x128 voxel map of a 512x512x256 cube 238 -> 189 ms: the
// tracer is bound by vector issue, and the FP32 loop lost about a third of its vector
// and two thirds of its scalar instructions.
template <typename T, bool TW, typename EvSink = NoEvents, int SCH = SCH_RKF45, bool M2 = false>
__host__ __device__ __forceinline__ void lane_iterate(Lane<T> &L, const T cb[3][8],
                                                      const T cj[3][8], const LaneConst<T> &K,
                                                      int &fin_st, int &fin_face, bool &need_load,
                                                      unsigned &n_acc, EvSink ev = EvSink(),
                                                      Tan<T> *tn = nullptr)
{
// products and sums round as written (a fused one is an fma_)
#pragma clang fp contract(off)
    static_assert(!M2 || SCH == 0, "Method II is traced with RKF45");
    constexpr bool FIXED = SCH != SCH_RKF45;
    constexpr int NS = FIXED ? 4 : 6;  // stages
    using N = Num<T>;
    constexpr int kNull = 2, kMaxSteps = 4, kNonFinite = 8;  // FQ_ST_* bits
    const bool over = ++L.trials > K.max_steps;
    T f0, f1, f2, ft, b2;
    rhs<T, TW>(cb, cj, L.p0, L.p1, L.p2, L.sgn, K.rx, K.ry, K.rz, K.twk, f0, f1, f2, ft, b2);
    const bool live = !(over | !finite_(b2) | (b2 <= K.bnull2));

    // Per axis: the face ahead, whether it is a box face, the distance to it, and
    // whether the point sits on it and moves out through it. Such a point changes cell
    // first (on a box face the line ends). Between two cells a direction within tau of
    // the face plane counts as tangent: the two cells' polynomials agree on the face
    // only to rounding, so the sign of a tiny normal component may differ between them.
    // On a box face the sign alone decides, as for the exact line.
    const T tau = N::tau;
    const bool u0 = f0 > T(0), u1 = f1 > T(0), u2 = f2 > T(0);
    const T w0 = u0 ? T(1) : T(0), w1 = u1 ? T(1) : T(0), w2 = u2 ? T(1) : T(0);
    const bool e0 = L.c0 == (u0 ? K.nx - 2 : 0), e1 = L.c1 == (u1 ? K.ny - 2 : 0),
               e2 = L.c2 == (u2 ? K.nz - 2 : 0);
    const bool o0 = (L.p0 == w0) & (fabs(f0) > (e0 ? T(0) : tau)),
               o1 = (L.p1 == w1) & (fabs(f1) > (e1 ? T(0) : tau)),
               o2 = (L.p2 == w2) & (fabs(f2) > (e2 ? T(0) : tau));
    const bool cross = o0 | o1 | o2;

    // the straight-line distance to the faces ahead, and the landing it asks for
    const T d0 = w0 - L.p0, d1 = w1 - L.p1, d2 = w2 - L.p2;
    const T t0 = fabs(f0) > tau ? d0 * N::rcp(f0) : T(FLT_MAX),
            t1 = fabs(f1) > tau ? d1 * N::rcp(f1) : T(FLT_MAX),
            t2 = fabs(f2) > tau ? d2 * N::rcp(f2) : T(FLT_MAX);
    const bool first1 = t1 < t0;
    const T t01 = first1 ? t1 : t0;
    const bool first2 = t2 < t01;
    const T t_exit = first2 ? t2 : t01;
    const bool forced = L.force >= 0, reach = !forced & (L.h >= t_exit);
    const int fa = L.force >> 1;
    const bool l0 = (fa == 0) | (reach & !first1 & !first2), l1 = (fa == 1) | (reach & first1 & !first2),
               l2 = (fa == 2) | (reach & first2);
    const bool land = l0 | l1 | l2;
    const T g0 = land ? (l0 ? f0 : (l1 ? f1 : f2)) : T(1);
    const T H = land ? (l0 ? d0 : (l1 ? d1 : d2)) : L.h;
    const bool wrong_way = forced & ((g0 > T(0)) != ((L.force & 1) != 0));
    // not heading to that face yet: approach it with a plain step
    const bool noland = land & (wrong_way | !(fabs(g0) > N::gmin) | (H == T(0)));
    const bool step = live & !cross & !noland;
    const bool hneg = !(H >= T(0));
    const T ig0 = N::rcp(g0);

    // Fehlberg 4(5), or classic / 3/8-rule RK4 (Kutta). Stage positions need only
    // the position parts of earlier stages; the twist and length parts go straight
    // into the weighted sums of the solution.
    constexpr T A10 = T(1.0 / 4.0);
    constexpr T A20 = T(3.0 / 32.0), A21 = T(9.0 / 32.0);
    constexpr T A30 = T(1932.0 / 2197.0), A31 = T(-7200.0 / 2197.0), A32 = T(7296.0 / 2197.0);
    constexpr T A40 = T(439.0 / 216.0), A41 = T(-8.0), A42 = T(3680.0 / 513.0),
                A43 = T(-845.0 / 4104.0);
    constexpr T A50 = T(-8.0 / 27.0), A51 = T(2.0), A52 = T(-3544.0 / 2565.0),
                A53 = T(1859.0 / 4104.0), A54 = T(-11.0 / 40.0);
    constexpr T B0 = T(16.0 / 135.0), B2 = T(6656.0 / 12825.0), B3 = T(28561.0 / 56430.0),
                B4 = T(-9.0 / 50.0), B5 = T(2.0 / 55.0);
    constexpr T E0 = T(1.0 / 360.0), E2 = T(-128.0 / 4275.0), E3 = T(-2197.0 / 75240.0),
                E4 = T(1.0 / 50.0), E5 = T(2.0 / 55.0);
    // classic RK4: c = (0, 1/2, 1/2, 1), b = (1, 2, 2, 1) / 6;
    // 3/8 rule: c = (0, 1/3, 2/3, 1), a = (1/3; -1/3, 1; 1, -1, 1), b = (1, 3, 3, 1) / 8
    constexpr T W0 = SCH == SCH_RK4 ? T(1.0 / 6.0) : SCH == SCH_RK4_38 ? T(1.0 / 8.0) : B0;
    T k[6][3];
    k[0][0] = f0 * ig0;
    k[0][1] = f1 * ig0;
    k[0][2] = f2 * ig0;
    T ku[M2 ? 6 : 1][3], kv[M2 ? 6 : 1][3];
    if constexpr (M2) {
        // the rates at the start need B there; one more evaluation of it
        const T bx = poly<T>(cb[0], L.p0, L.p1, L.p2), by = poly<T>(cb[1], L.p0, L.p1, L.p2),
                bz = poly<T>(cb[2], L.p0, L.p1, L.p2);
        tan_rates<T>(cb, L.p0, L.p1, L.p2, bx, by, bz, N::rsq(b2), L.sgn, K.rx, K.ry, K.rz,
                     tn->u, tn->v, ku[0], kv[0]);
#pragma unroll
        for (int q = 0; q < 3; q++) {
            ku[0][q] *= ig0;
            kv[0][q] *= ig0;
        }
    }
    T stw = W0 * (ft * ig0), slen = W0 * ig0;
    bool ok = true;
    T b2min = b2;
    T fe[3] = {T(0), T(0), T(0)}, ige = T(0);  // the last stage's rate (RK4)
#pragma unroll
    for (int st = 1; st < NS; st++) {
        T y[3];
#pragma unroll
        for (int q = 0; q < 3; q++) {
            T acc;
            if (SCH == SCH_RK4) {
                acc = st == 3 ? k[2][q] : T(0.5) * k[st - 1][q];
            } else if (SCH == SCH_RK4_38) {
                if (st == 1) acc = T(1.0 / 3.0) * k[0][q];
                else if (st == 2) acc = N::fma_(fe[q], ige, -(T(1.0 / 3.0) * k[0][q]));
                else acc = N::fma_(fe[q], ige, k[0][q] - k[1][q]);
            } else if (st == 1) acc = A10 * k[0][q];
            else if (st == 2) acc = N::fma_(A21, k[1][q], A20 * k[0][q]);
            else if (st == 3) acc = N::fma_(A32, k[2][q], N::fma_(A31, k[1][q], A30 * k[0][q]));
            else if (st == 4)
                acc = N::fma_(A43, k[3][q],
                              N::fma_(A42, k[2][q], N::fma_(A41, k[1][q], A40 * k[0][q])));
            else
                acc = N::fma_(A54, k[4][q],
                              N::fma_(A53, k[3][q],
                                      N::fma_(A52, k[2][q], N::fma_(A51, k[1][q], A50 * k[0][q]))));
            y[q] = N::fma_(H, acc, q == 0 ? L.p0 : (q == 1 ? L.p1 : L.p2));
        }
        T uy[3], vy[3];
        if constexpr (M2) {
#pragma unroll
            for (int q = 0; q < 3; q++) {
                T au, av;
                if (st == 1) au = A10 * ku[0][q], av = A10 * kv[0][q];
                else if (st == 2) {
                    au = N::fma_(A21, ku[1][q], A20 * ku[0][q]);
                    av = N::fma_(A21, kv[1][q], A20 * kv[0][q]);
                } else if (st == 3) {
                    au = N::fma_(A32, ku[2][q], N::fma_(A31, ku[1][q], A30 * ku[0][q]));
                    av = N::fma_(A32, kv[2][q], N::fma_(A31, kv[1][q], A30 * kv[0][q]));
                } else if (st == 4) {
                    au = N::fma_(A43, ku[3][q], N::fma_(A42, ku[2][q], N::fma_(A41, ku[1][q], A40 * ku[0][q])));
                    av = N::fma_(A43, kv[3][q], N::fma_(A42, kv[2][q], N::fma_(A41, kv[1][q], A40 * kv[0][q])));
                } else {
                    au = N::fma_(A54, ku[4][q], N::fma_(A53, ku[3][q],
                         N::fma_(A52, ku[2][q], N::fma_(A51, ku[1][q], A50 * ku[0][q]))));
                    av = N::fma_(A54, kv[4][q], N::fma_(A53, kv[3][q],
                         N::fma_(A52, kv[2][q], N::fma_(A51, kv[1][q], A50 * kv[0][q]))));
                }
                uy[q] = N::fma_(H, au, tn->u[q]);
                vy[q] = N::fma_(H, av, tn->v[q]);
            }
        }
        T g0s, g1s, g2s, gts, b2s;
        // the twist integrand of Fehlberg's stage 1 has weight zero in the
        // fifth-order sum
        if (!FIXED && st == 1)
            rhs<T, false>(cb, cj, y[0], y[1], y[2], L.sgn, K.rx, K.ry, K.rz, K.twk, g0s, g1s, g2s,
                          gts, b2s);
        else
            rhs<T, TW>(cb, cj, y[0], y[1], y[2], L.sgn, K.rx, K.ry, K.rz, K.twk, g0s, g1s, g2s,
                       gts, b2s);
        // (a NaN at one stage is a NaN at the last, and no null)
        b2min = st < NS - 1 ? N::min_(b2min, b2s) : mn(b2min, b2s);
        ok = ok & finite_(b2s);
        // A landing whose face coordinate turns within the step is given up. A
        // fixed-step scheme has no error estimate to catch one that turns badly (a line
        // meeting the face at a small angle): it approaches with shorter plain steps
        // until the face coordinate's rate changes by at most a tenth.
        T g = l0 ? g0s : (l1 ? g1s : g2s);
        bool turned = !((hneg ? -g : g) > N::gmin);
        if (FIXED) turned = turned | (fabs(g - g0) > T(0.1) * fabs(g0));
        ok = ok & !(land & turned);
        g = land & !turned ? g : g0;  // g0 = 1 for a plain step
        const T ig = N::rcp(g);
        k[st][0] = g0s * ig;
        k[st][1] = g1s * ig;
        k[st][2] = g2s * ig;
        if (FIXED) fe[0] = g0s, fe[1] = g1s, fe[2] = g2s, ige = ig;
        if constexpr (M2) {
            const T bx = poly<T>(cb[0], y[0], y[1], y[2]), by = poly<T>(cb[1], y[0], y[1], y[2]),
                    bz = poly<T>(cb[2], y[0], y[1], y[2]);
            tan_rates<T>(cb, y[0], y[1], y[2], bx, by, bz, N::rsq(b2s), L.sgn, K.rx, K.ry, K.rz,
                         uy, vy, ku[st], kv[st]);
#pragma unroll
            for (int q = 0; q < 3; q++) {
                ku[st][q] *= ig;
                kv[st][q] *= ig;
            }
        }
        T bs;
        if (SCH == SCH_RK4) bs = st == 3 ? T(1.0 / 6.0) : T(1.0 / 3.0);
        else if (SCH == SCH_RK4_38) bs = st == 3 ? T(1.0 / 8.0) : T(3.0 / 8.0);
        else bs = st == 2 ? B2 : st == 3 ? B3 : st == 4 ? B4 : st == 5 ? B5 : T(0);
        if (FIXED || st != 1) stw = N::fma_(bs, gts * ig, stw);
        if (FIXED || st != 1) slen = N::fma_(bs, ig, slen);
        if (TW) here_and_now(stw);
    }
    // displacement and new position (the sum of the two rounded once), error
    T dy[3], e[3], nw[3];
#pragma unroll
    for (int q = 0; q < 3; q++) {
        T acc;
        if (SCH == SCH_RK4) {
            acc = N::fma_(T(1.0 / 3.0), k[1][q] + k[2][q], T(1.0 / 6.0) * N::fma_(fe[q], ige, k[0][q]));
            e[q] = T(0);
        } else if (SCH == SCH_RK4_38) {
            acc = N::fma_(T(3.0 / 8.0), k[1][q] + k[2][q], T(1.0 / 8.0) * N::fma_(fe[q], ige, k[0][q]));
            e[q] = T(0);
        } else {
            acc = N::fma_(B5, k[5][q], N::fma_(B4, k[4][q],
                  N::fma_(B3, k[3][q], N::fma_(B2, k[2][q], B0 * k[0][q]))));
            const T ea = N::fma_(E5, k[5][q], N::fma_(E4, k[4][q],
                         N::fma_(E3, k[3][q], N::fma_(E2, k[2][q], E0 * k[0][q]))));
            e[q] = H * ea;
        }
        dy[q] = H * acc;
        nw[q] = N::fma_(H, acc, q == 0 ? L.p0 : (q == 1 ? L.p1 : L.p2));
    }
    const bool null_in = b2min <= K.bnull2;
    T err2 = N::fma_(e[0], e[0], N::fma_(e[1], e[1], e[2] * e[2]));
    T du[3], dvv[3];
    if constexpr (M2) {
        // the tangent vectors' errors join the norm relative to their size (at
        // least one grid unit), as their 5th-order updates are formed
        T eu2 = T(0), ev2 = T(0);
#pragma unroll
        for (int q = 0; q < 3; q++) {
            du[q] = H * N::fma_(B5, ku[5][q], N::fma_(B4, ku[4][q],
                        N::fma_(B3, ku[3][q], N::fma_(B2, ku[2][q], B0 * ku[0][q]))));
            dvv[q] = H * N::fma_(B5, kv[5][q], N::fma_(B4, kv[4][q],
                         N::fma_(B3, kv[3][q], N::fma_(B2, kv[2][q], B0 * kv[0][q]))));
            const T a = H * N::fma_(E5, ku[5][q], N::fma_(E4, ku[4][q],
                            N::fma_(E3, ku[3][q], N::fma_(E2, ku[2][q], E0 * ku[0][q]))));
            const T b = H * N::fma_(E5, kv[5][q], N::fma_(E4, kv[4][q],
                            N::fma_(E3, kv[3][q], N::fma_(E2, kv[2][q], E0 * kv[0][q]))));
            eu2 = N::fma_(a, a, eu2);
            ev2 = N::fma_(b, b, ev2);
        }
        const T uu = mx(T(1), N::fma_(tn->u[0], tn->u[0], N::fma_(tn->u[1], tn->u[1], tn->u[2] * tn->u[2])));
        const T vv = mx(T(1), N::fma_(tn->v[0], tn->v[0], N::fma_(tn->v[1], tn->v[1], tn->v[2] * tn->v[2])));
        err2 = N::fma_(ev2, N::rcp(vv), N::fma_(eu2, N::rcp(uu), err2));
    }
    const T tol2 = L.tol * L.tol;
    const T s_abs = fabs(H * ig0);  // arc length of the step, reference lengths
    // a NaN/Inf in the field, or a landing parametrisation that broke down (the line
    // turns within the step)
    const bool broke = !ok | !finite_(err2);
    const bool over_tol = !FIXED & (err2 > tol2);
    const float ratio = 0.9f * pow01((float)tol2 * Num<float>::rcp((float)err2));
    const T ov = M2 ? N::ov_tan : N::ov;
    const bool inerr = step & !null_in & !broke & !over_tol;

    // Past a box face the line ends on that face, and clamping an overshoot d onto
    // it moves the end by d over the line's slope to the face: a first-order
    // error, not the second-order kink error of an interior face. So a step that
    // ends past a box face the line crosses keeps no overshoot: it lands on that
    // face instead (`bp`, its face code 2*axis + (high side)), or, where the line is not
    // heading out steeply enough at the step's start to take the face coordinate as the
    // independent variable, approaches it with shorter plain steps first. Only
    // a line tangent to the box face at both ends of the step keeps the
    // allowance: one that turns over within the step and leaves at a small angle alpha
    // would otherwise be clamped onto the face up to ov / alpha away from its crossing
    // (near a polarity inversion line on a box face, alpha is the seed's distance from
    // that line). The start direction is k1 times g0; stage 5 sits at the end
    // of the step, so k5 times g0 stands for the end direction (its sign is
    // exact, its size is scaled by that stage's own g on a landing).
    constexpr int KE = FIXED ? 3 : 4;  // the stage at the end of the step (c = 1)
    const bool h0 = nw[0] > T(1), h1 = nw[1] > T(1), h2 = nw[2] > T(1);
    const bool p0 = !l0 & (h0 | (nw[0] < T(0))), p1 = !l1 & (h1 | (nw[1] < T(0))),
               p2 = !l2 & (h2 | (nw[2] < T(0)));  // past a face
    const bool x0 = p0 & (L.c0 == (h0 ? K.nx - 2 : 0)), x1 = p1 & (L.c1 == (h1 ? K.ny - 2 : 0)),
               x2 = p2 & (L.c2 == (h2 ? K.nz - 2 : 0));  // past a box face
    int bp = -1;
    if (inerr & (x0 | x1 | x2)) {
        // heading out through the face at the start or at the end of the step
        const T s0 = h0 ? g0 : -g0, s1 = h1 ? g0 : -g0, s2 = h2 ? g0 : -g0;
        if (x2 & ((k[0][2] * s2 > N::gmin) | (k[KE][2] * s2 > N::gmin))) bp = 4 + (h2 ? 1 : 0);
        if (x1 & ((k[0][1] * s1 > N::gmin) | (k[KE][1] * s1 > N::gmin))) bp = 2 + (h1 ? 1 : 0);
        if (x0 & ((k[0][0] * s0 > N::gmin) | (k[KE][0] * s0 > N::gmin))) bp = h0 ? 1 : 0;
    }
    // a brief excursion over a face inside the step (the end may be back inside)
    const T v0 = N::fma_(-H, k[0][0], dy[0]), v1 = N::fma_(-H, k[0][1], dy[1]),
            v2 = N::fma_(-H, k[0][2], dy[2]);
    const bool q0 = !l0 & excursion(L.p0, H * k[0][0], v0, ov),
               q1 = !l1 & excursion(L.p1, H * k[0][1], v1, ov),
               q2 = !l2 & excursion(L.p2, H * k[0][2], v2, ov);
    // A step that ends inside, or past a face by at most ov, is kept: straddling a face
    // by d it errs by O(d^2), and the overshoot is carried into the neighbouring cell
    // (on a box face, clamped to it).
    const bool b0 = !l0 & ((nw[0] < -ov) | (nw[0] > T(1) + ov)),
               b1 = !l1 & ((nw[1] < -ov) | (nw[1] > T(1) + ov)),
               b2n = !l2 & ((nw[2] < -ov) | (nw[2] > T(1) + ov));
    const bool leaves = (bp >= 0) | q0 | q1 | q2 | b0 | b1 | b2n;
    const bool acc = inerr & !leaves;

    // the next step when this one is not kept: half the shorter of h and the step tried
    // (or of the distance to the face), or as the error asks, or as far as the line
    // stayed in the cell. Every failure shrinks h below both the current h and the step
    // just tried, so the plain-step fallback always makes progress.
    T shrink = over_tol & !broke & !noland ? mx((T)ratio, (T)0.1f) : T(0.5);
    int force = -1;
    if (inerr & leaves) {
        int xf = -1;
        if (q2) xf = v2 < T(0) ? 5 : 4;
        if (q1) xf = v1 < T(0) ? 3 : 2;
        if (q0) xf = v0 < T(0) ? 1 : 0;
        if (land) {
            // another face comes first: land there next, unless this already was a
            // forced landing (then approach with plain steps, which always progress)
            int fb = bp >= 0 ? bp : xf;
            if (b0) fb = h0 ? 1 : 0;
            if (b1) fb = h1 ? 3 : 2;
            if (b2n) fb = h2 ? 5 : 4;
            if (!forced) force = fb;
        } else {
            // the line curved out of the cell before the straight-line guess: land
            // next on the face its chord crossed first
            T th = T(2);
            if (p0) {
                const T tq = ((h0 ? T(1) : T(0)) - L.p0) / (nw[0] - L.p0);
                if (tq < th) th = tq, force = h0 ? 1 : 0;
            }
            if (p1) {
                const T tq = ((h1 ? T(1) : T(0)) - L.p1) / (nw[1] - L.p1);
                if (tq < th) th = tq, force = h1 ? 3 : 2;
            }
            if (p2) {
                const T tq = ((h2 ? T(1) : T(0)) - L.p2) / (nw[2] - L.p2);
                if (tq < th) th = tq, force = h2 ? 5 : 4;
            }
            if (force < 0) force = xf, th = T(0.5);
            shrink = mn(mx(th, T(0.5)), T(1));
        }
    }
    const T tried = noland ? t_exit : s_abs;
    const T from = land ? mn(L.h, tried) : L.h;
    T hn = mx(from * shrink, N::hmin);
    // ... and when it is: a landing is cut short by the face, not by the error bound:
    // unless the error asks for a smaller step, keep the step the controller had before
    // the cut
    if (FIXED) {
        hn = acc ? L.tol : hn;
    } else {
        const float grow = err2 > T(0) ? fminf(ratio, 5.0f) : 5.0f;
        const T g1 = (land ? s_abs : L.h) * (T)grow;
        const T g2 = mn(land ? mx(g1, L.h) : g1, T(4));
        hn = acc ? (land & !(grow >= 1.0f) ? g1 : g2) : hn;
    }
    const bool again = (hn == L.h) & (force == L.force);
    if (!cross) {
        L.h = hn;
        L.force = force;
    }

    bool moved = false;
    if (acc) {
        L.p0 = nw[0];
        L.p1 = nw[1];
        L.p2 = nw[2];
        if constexpr (M2)
#pragma unroll
            for (int q = 0; q < 3; q++) {
                tn->u[q] += du[q];
                tn->v[q] += dvv[q];
            }
        if constexpr (sizeof(T) == 8) {
            L.tw = N::fma_(H, stw, L.tw);
            L.len = N::fma_(H, slen, L.len);
        } else {
            L.tw += (double)(H * stw);
            L.len += (double)(H * slen);
        }
        n_acc++;
        int cl = 0;
        if (p0 | p1 | p2) {
            if (p0) moved |= carry(L.c0, L.p0, K.nx, cl, 1);
            if (p1) moved |= carry(L.c1, L.p1, K.ny, cl, 2);
            if (p2) moved |= carry(L.c2, L.p2, K.nz, cl, 4);
        }
        ev.accepted(l0 ? 0 : (l1 ? 1 : (l2 ? 2 : -1)), H, cl);
    }
    // cross the face reached: the next cell, or the end of the line
    const bool x = live & cross, xl = acc & land;
    const bool a0 = (x & o0) | (xl & l0), a1 = (x & o1 & !o0) | (xl & l1),
               a2 = (x & o2 & !o1 & !o0) | (xl & l2);
    const bool at_box = (a0 & e0) | (a1 & e1) | (a2 & e2);
    const bool upx = (a0 & u0) | (a1 & u1) | (a2 & u2);
    const bool on = (x | xl) & !at_box;
    const T pf = upx != on ? T(1) : T(0);
    L.p0 = a0 ? pf : L.p0;
    L.p1 = a1 ? pf : L.p1;
    L.p2 = a2 ? pf : L.p2;
    L.c0 += (a0 & on) ? (u0 ? 1 : -1) : 0;
    L.c1 += (a1 & on) ? (u1 ? 1 : -1) : 0;
    L.c2 += (a2 & on) ? (u2 ? 1 : -1) : 0;
    need_load = need_load | moved | on;
    const bool dead = !live | (step & (null_in | (broke & !land)));
    // A trial that moves nothing and asks for the step it had (the smallest one, rejected)
    // will be the same trial for good: the line's other trials are taken as done. (A layer
    // of zero field under 700 x 700 points holds 28 000 such half lines, max_steps trials
    // each: 1.42 -> 0.58 s. Not in the step with four lanes to a half line, whose longest
    // chain the test would cost 3%.)
    if (!FIXED && (again & !(dead | cross | acc))) L.trials = K.max_steps;
    if (dead | at_box) {
        fin_st = at_box ? 0
                 : over ? kMaxSteps
                 : !finite_(b2) ? kNonFinite
                 : (b2 <= K.bnull2) | null_in ? kNull : kNonFinite;
        if (at_box) fin_face = (a0 ? 0 : (a1 ? 2 : 4)) + (upx ? 1 : 0);
    }
}

}  // namespace fq
