// The trial step of lane_iterate (trace_core.h) with four lanes to a half line.
//
// Where a launch has few lines, what it takes is the longest line's chain of trial
// steps, while most issue slots of the chip stay empty. Here lane c < 3 of a quad holds
// component c of the cell's polynomials of B (and curl B), of the stage derivatives, of
// the position's error and of Method II's tangent vectors, and does the tests of axis c;
// the lanes exchange the three values they share (the stage position, B, the twist's
// curl B) by quad permutes. Lane 3 carries a zero component that never meets a face. The
// step, the twist and the length are computed by all four alike. Every sum is formed in
// the order and with the roundings of lane_iterate, so a line comes out bit for bit the
// same either way.
#pragma once

#include "trace_core.h"
#include "trace_dev.h"

namespace fq {
namespace quad {

// x of the quad's lane I / of the lane the permutation CTRL names
template <int CTRL> __device__ __forceinline__ int perm(int x)
{
    return __builtin_amdgcn_mov_dpp(x, CTRL, 0xf, 0xf, true);
}
template <int CTRL> __device__ __forceinline__ float perm(float x)
{
    return __builtin_bit_cast(float, perm<CTRL>(__builtin_bit_cast(int, x)));
}
struct Halves {
    int lo, hi;
};
template <int CTRL> __device__ __forceinline__ double perm(double x)
{
    Halves h = __builtin_bit_cast(Halves, x);
    h.lo = perm<CTRL>(h.lo);
    h.hi = perm<CTRL>(h.hi);
    return __builtin_bit_cast(double, h);
}
template <int I, typename T> __device__ __forceinline__ T from(T x) { return perm<I * 0x55>(x); }
constexpr int kSwap1 = 0xb1, kSwap2 = 0x4e;  // lanes 1,0,3,2 and 2,3,0,1

// all three components in every lane
template <typename T> __device__ __forceinline__ void all3(T x, T v[3])
{
    v[0] = from<0>(x);
    v[1] = from<1>(x);
    v[2] = from<2>(x);
}
__device__ __forceinline__ int any(int x)
{
    x |= perm<kSwap1>(x);
    return x | perm<kSwap2>(x);
}
template <typename T> __device__ __forceinline__ T least(T x)
{
    x = Num<T>::min_(x, perm<kSwap1>(x));
    return Num<T>::min_(x, perm<kSwap2>(x));
}
// the value of the one lane of the quad where `on` (0 if there is none)
__device__ __forceinline__ float one(float x, bool on)
{
    return __builtin_bit_cast(float, any(on ? __builtin_bit_cast(int, x) : 0));
}
__device__ __forceinline__ double one(double x, bool on)
{
    Halves h = __builtin_bit_cast(Halves, x);
    h.lo = any(on ? h.lo : 0);
    h.hi = any(on ? h.hi : 0);
    return __builtin_bit_cast(double, h);
}
// lowest / highest axis of a 3-bit set (-1 if empty)
__device__ __forceinline__ int lowest(int set) { return __builtin_ffs(set) - 1; }
__device__ __forceinline__ int highest(int set) { return 31 - __builtin_clz(set | 1) - (set == 0); }

// One half line: replicated state, and this lane's axis.
template <typename T> struct Line {
    T P[3];          // local position (all lanes)
    T h, tol, sgn;
    double tw, len;
    uint32_t trials;
    int force;
    int c;           // this lane's axis (3: none; sets of axes hold it in a bit nobody reads)
    int cell, n;     // cell and nodes along it
    T p, r;          // coordinate and direction scale along it
    T u, v;          // Method II: its components of U and V
};

template <typename T> struct Const {
    T twk, bnull2;
    uint32_t max_steps;
};

// B (and curl B) at Y: this lane's component b, all three in B; direction component f,
// twist rate ft, |B|^2, 1/|B|.
template <typename T, bool TW>
__device__ __forceinline__ void rates(const T cb[8], const T cj[8], const T Y[3], const Line<T> &L,
                                      T twk, T B[3], T &f, T &ft, T &b2, T &inv)
{
    using N = Num<T>;
    const T b = poly<T>(cb, Y[0], Y[1], Y[2]);
    all3(b, B);
    b2 = N::fma_(B[0], B[0], N::fma_(B[1], B[1], B[2] * B[2]));
    inv = N::rsq(b2);
    const T s = L.sgn * inv;
    f = s * b * L.r;
    ft = T(0);
    if (TW) {
        T J[3];
        all3(poly<T>(cj, Y[0], Y[1], Y[2]), J);
        const T jb = N::fma_(J[0], B[0], N::fma_(J[1], B[1], J[2] * B[2]));
        ft = jb * (inv * inv) * twk;
    }
}

// Method II's rates of this lane's components of U and V (see tan_rates).
template <typename T>
__device__ __forceinline__ void tangent(const T cb[8], const T Y[3], const Line<T> &L, const T B[3],
                                        T inv, T u, T v, T &ku, T &kv)
{
    using N = Num<T>;
    T d0, d1, d2;
    dpoly<T>(cb, Y[0], Y[1], Y[2], d0, d1, d2);
    const T b0 = B[0] * inv, b1 = B[1] * inv, b2 = B[2] * inv;
    const T own = L.c == 0 ? b0 : (L.c == 1 ? b1 : (L.c == 2 ? b2 : T(0)));
    const T s = L.sgn * inv;
#pragma unroll
    for (int m = 0; m < 2; m++) {
        T X[3], g[3];
        all3(m ? v : u, X);
        const T go = N::fma_(d0, X[0], N::fma_(d1, X[1], d2 * X[2]));
        all3(go, g);
        const T bg = N::fma_(b0, g[0], N::fma_(b1, g[1], b2 * g[2]));
        const T k = s * L.r * N::fma_(-own, bg, go);
        if (m) kv = k;
        else ku = k;
    }
}

// One trial step (RKF45): lane_iterate's cases and results, its event sink too.
template <typename T, bool TW, bool M2, typename EV = NoEvents>
__device__ __forceinline__ void iterate(Line<T> &L, const T cb[8], const T cj[8], const Const<T> &K,
                                        int &fin_st, int &fin_face, bool &need_load, unsigned &n_acc,
                                        const EV &ev = EV{})
{
// products and sums round as written (a fused one is an fma_)
#pragma clang fp contract(off)
    using N = Num<T>;
    constexpr int kNull = 2, kMaxSteps = 4, kNonFinite = 8;  // FQ_ST_* bits
    const bool over = ++L.trials > K.max_steps;
    T B[3], f, ft, b2, inv;
    rates<T, TW>(cb, cj, L.P, L, K.twk, B, f, ft, b2, inv);
    const bool live = !(over | !finite_(b2) | (b2 <= K.bnull2));

    // this axis: the face ahead, whether it is a box face, whether the point sits on it
    // and moves out through it, the straight-line distance to it
    const T tau = N::tau;
    const bool up = f > T(0);
    const T w = up ? T(1) : T(0);
    const bool edge = L.cell == (up ? L.n - 2 : 0);
    const bool out = (L.p == w) & (fabs(f) > (edge ? T(0) : tau));
    const T d = w - L.p;
    const T t = fabs(f) > tau ? d * N::rcp(f) : T(FLT_MAX);
    const T t_exit = least(t);
    // bits 0-2 out, 4-6 first face ahead, 8-10 up, 12-14 edge
    const int F = any(((out ? 1 : 0) | (t == t_exit ? 1 << 4 : 0) | (up ? 1 << 8 : 0) | (edge ? 1 << 12 : 0))
                      << L.c);
    const bool cross = (F & 7) != 0;
    const bool forced = L.force >= 0, reach = !forced & (L.h >= t_exit), land = forced | reach;
    const int lax = forced ? L.force >> 1 : lowest((F >> 4) & 7);
    const bool lnd = land & (lax == L.c);
    const T g0 = land ? one(f, lnd) : T(1);
    const T H = land ? one(d, lnd) : L.h;
    const bool wrong_way = forced & ((g0 > T(0)) != ((L.force & 1) != 0));
    const bool noland = land & (wrong_way | !(fabs(g0) > N::gmin) | (H == T(0)));
    const bool step = live & !cross & !noland;
    const bool hneg = !(H >= T(0));
    const T ig0 = N::rcp(g0);

    constexpr T A10 = T(1.0 / 4.0);
    constexpr T A20 = T(3.0 / 32.0), A21 = T(9.0 / 32.0);
    constexpr T A30 = T(1932.0 / 2197.0), A31 = T(-7200.0 / 2197.0), A32 = T(7296.0 / 2197.0);
    constexpr T A40 = T(439.0 / 216.0), A41 = T(-8.0), A42 = T(3680.0 / 513.0), A43 = T(-845.0 / 4104.0);
    constexpr T A50 = T(-8.0 / 27.0), A51 = T(2.0), A52 = T(-3544.0 / 2565.0), A53 = T(1859.0 / 4104.0),
                A54 = T(-11.0 / 40.0);
    constexpr T B0 = T(16.0 / 135.0), B2 = T(6656.0 / 12825.0), B3 = T(28561.0 / 56430.0),
                B4 = T(-9.0 / 50.0), B5 = T(2.0 / 55.0);
    constexpr T E0 = T(1.0 / 360.0), E2 = T(-128.0 / 4275.0), E3 = T(-2197.0 / 75240.0),
                E4 = T(1.0 / 50.0), E5 = T(2.0 / 55.0);
    auto stage = [&](int st, const T k[6]) -> T {
        return st == 1   ? A10 * k[0]
               : st == 2 ? N::fma_(A21, k[1], A20 * k[0])
               : st == 3 ? N::fma_(A32, k[2], N::fma_(A31, k[1], A30 * k[0]))
               : st == 4 ? N::fma_(A43, k[3], N::fma_(A42, k[2], N::fma_(A41, k[1], A40 * k[0])))
                         : N::fma_(A54, k[4], N::fma_(A53, k[3], N::fma_(A52, k[2], N::fma_(A51, k[1], A50 * k[0]))));
    };
    auto solution = [&](const T k[6]) -> T {
        return N::fma_(B5, k[5], N::fma_(B4, k[4], N::fma_(B3, k[3], N::fma_(B2, k[2], B0 * k[0]))));
    };
    auto error = [&](const T k[6]) -> T {
        return N::fma_(E5, k[5], N::fma_(E4, k[4], N::fma_(E3, k[3], N::fma_(E2, k[2], E0 * k[0]))));
    };

    T k[6], ku[6], kv[6];
    k[0] = f * ig0;
    if constexpr (M2) {
        tangent<T>(cb, L.P, L, B, inv, L.u, L.v, ku[0], kv[0]);
        ku[0] *= ig0;
        kv[0] *= ig0;
    }
    T stw = B0 * (ft * ig0), slen = B0 * ig0;
    bool ok = true;
    T b2min = b2;
#pragma unroll
    for (int st = 1; st < 6; st++) {
        T Y[3];
        all3(N::fma_(H, stage(st, k), L.p), Y);
        T uy, vy;
        if constexpr (M2) {
            uy = N::fma_(H, stage(st, ku), L.u);
            vy = N::fma_(H, stage(st, kv), L.v);
        }
        T fs, fts, b2s, invs;
        if (st == 1) rates<T, false>(cb, cj, Y, L, K.twk, B, fs, fts, b2s, invs);
        else rates<T, TW>(cb, cj, Y, L, K.twk, B, fs, fts, b2s, invs);
        b2min = st < 5 ? N::min_(b2min, b2s) : mn(b2min, b2s);
        ok = ok & finite_(b2s);
        T g = one(fs, lnd);
        const bool turned = !((hneg ? -g : g) > N::gmin);
        ok = ok & !(land & turned);
        g = land & !turned ? g : g0;
        const T ig = N::rcp(g);
        k[st] = fs * ig;
        if constexpr (M2) {
            tangent<T>(cb, Y, L, B, invs, uy, vy, ku[st], kv[st]);
            ku[st] *= ig;
            kv[st] *= ig;
        }
        const T bs = st == 2 ? B2 : st == 3 ? B3 : st == 4 ? B4 : B5;
        if (st != 1) {
            stw = N::fma_(bs, fts * ig, stw);
            slen = N::fma_(bs, ig, slen);
            if (TW) here_and_now(stw);
        }
    }
    const T sol = solution(k);
    const T dy = H * sol, nw = N::fma_(H, sol, L.p);
    T e[3];
    all3(H * error(k), e);
    const bool null_in = b2min <= K.bnull2;
    T err2 = N::fma_(e[0], e[0], N::fma_(e[1], e[1], e[2] * e[2]));
    T du, dv;
    if constexpr (M2) {
        du = H * solution(ku);
        dv = H * solution(kv);
        T a[3], b[3], uu[3], vv[3];
        all3(H * error(ku), a);
        all3(H * error(kv), b);
        all3(L.u, uu);
        all3(L.v, vv);
        T eu2 = T(0), ev2 = T(0);
#pragma unroll
        for (int q = 0; q < 3; q++) {
            eu2 = N::fma_(a[q], a[q], eu2);
            ev2 = N::fma_(b[q], b[q], ev2);
        }
        const T u2 = mx(T(1), N::fma_(uu[0], uu[0], N::fma_(uu[1], uu[1], uu[2] * uu[2])));
        const T v2 = mx(T(1), N::fma_(vv[0], vv[0], N::fma_(vv[1], vv[1], vv[2] * vv[2])));
        err2 = N::fma_(ev2, N::rcp(v2), N::fma_(eu2, N::rcp(u2), err2));
    }
    const T tol2 = L.tol * L.tol;
    const T s_abs = fabs(H * ig0);
    const bool broke = !ok | !finite_(err2);
    const bool over_tol = err2 > tol2;
    const float ratio = 0.9f * pow01((float)tol2 * Num<float>::rcp((float)err2));
    const T ov = M2 ? N::ov_tan : N::ov;
    const bool inerr = step & !null_in & !broke & !over_tol;

    // this axis at the end of the step: past a face, past a box face, an excursion inside
    // the step, past by more than ov
    const bool hi = nw > T(1);
    const bool past = !lnd & (hi | (nw < T(0)));
    const bool xb = past & (L.cell == (hi ? L.n - 2 : 0));
    const T v2 = N::fma_(-H, k[0], dy);
    const bool exc = !lnd & excursion(L.p, H * k[0], v2, ov);
    const bool bey = !lnd & ((nw < -ov) | (nw > T(1) + ov));
    // bits 0-2 past, 4-6 past a box face, 8-10 excursion, 12-14 beyond, 16-18 high side,
    // 20-22 the excursion's side
    const int G = any(((past ? 1 : 0) | (xb ? 1 << 4 : 0) | (exc ? 1 << 8 : 0) | (bey ? 1 << 12 : 0) |
                       (hi ? 1 << 16 : 0) | (v2 < T(0) ? 1 << 20 : 0))
                      << L.c);
    auto code = [](int ax, int sides) { return 2 * ax + ((sides >> ax) & 1); };
    int bp = -1;
    if (inerr & ((G & 0x70) != 0)) {
        const T s = hi ? g0 : -g0;
        const int hit = any((xb & ((k[0] * s > N::gmin) | (k[4] * s > N::gmin))) ? 1 << L.c : 0);
        if (hit) bp = code(lowest(hit), G >> 16);
    }
    const bool leaves = (bp >= 0) | ((G & 0x7700) != 0);
    const bool acc = inerr & !leaves;
    T shrink = over_tol & !broke & !noland ? mx((T)ratio, (T)0.1f) : T(0.5);
    int force = -1;
    if (inerr & leaves) {
        const int xf = (G & 0x700) ? code(lowest((G >> 8) & 7), G >> 20) : -1;
        if (land) {
            int fb = bp >= 0 ? bp : xf;
            if (G & 0x7000) fb = code(highest((G >> 12) & 7), G >> 16);
            if (!forced) force = fb;
        } else {
            const T tq = past ? ((hi ? T(1) : T(0)) - L.p) / (nw - L.p) : T(2);
            T th = least(tq);
            const int first = any((past & (tq == th)) ? 1 << L.c : 0);
            if (first) force = code(lowest(first), G >> 16);
            else force = xf, th = T(0.5);
            shrink = mn(mx(th, T(0.5)), T(1));
        }
    }
    const T tried = noland ? t_exit : s_abs;
    const T base = land ? mn(L.h, tried) : L.h;
    T hn = mx(base * shrink, N::hmin);
    const float grow = err2 > T(0) ? fminf(ratio, 5.0f) : 5.0f;
    const T g1 = (land ? s_abs : L.h) * (T)grow;
    const T g2 = mn(land ? mx(g1, L.h) : g1, T(4));
    hn = acc ? (land & !(grow >= 1.0f) ? g1 : g2) : hn;
    if (!cross) {
        L.h = hn;
        L.force = force;
    }

    int moved = 0;
    if (acc) {
        L.p = nw;
        if constexpr (M2) {
            L.u += du;
            L.v += dv;
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
        if (G & 7) {
            if (past) moved = carry(L.cell, L.p, L.n, cl, 1);
            moved = any(moved);
            cl = any(cl << L.c);
        }
        ev.accepted(land ? lax : -1, H, cl);
    }
    // cross the face reached: the next cell, or the end of the line
    const bool x = live & cross, xl = acc & land;
    const int cax = (x ? lowest(F & 7) : lax) & 3;
    const bool upx = ((F >> 8 >> cax) & 1) != 0;
    const bool at_box = (x | xl) & (((F >> 12 >> cax) & 1) != 0);
    const bool on = (x | xl) & !at_box;
    if ((x | xl) & (cax == L.c)) {
        L.p = upx != on ? T(1) : T(0);
        L.cell += on ? (upx ? 1 : -1) : 0;
    }
    all3(L.p, L.P);
    need_load = need_load | (moved != 0) | on;
    const bool dead = !live | (step & (null_in | (broke & !land)));
    if (dead | at_box) {
        fin_st = at_box ? 0
                 : over ? kMaxSteps
                 : !finite_(b2) ? kNonFinite
                 : (b2 <= K.bnull2) | null_in ? kNull : kNonFinite;
        if (at_box) fin_face = 2 * cax + (upx ? 1 : 0);
    }
}

// This lane's component of the cell's polynomials: 8 corner values each, from records of
// type S. Lane 3 reads the records' zero padding.
template <typename T, typename S, bool TW, bool WIDE>
__device__ __forceinline__ void load_cell(const void *nodes, int nx, int ny, const Line<T> &L, T cb[8], T cj[8])
{
    const int c0 = from<0>(L.cell), c1 = from<1>(L.cell), c2 = from<2>(L.cell);
    constexpr unsigned kRec = (WIDE ? 8 : 4) * sizeof(S);
    const unsigned row = __umul24((unsigned)c2, (unsigned)ny) + (unsigned)c1;
    const unsigned ob = (WIDE && L.c == 3 ? 6 : L.c) * sizeof(S), oj = (L.c == 3 ? 7 : 3 + L.c) * sizeof(S);
    const FQ_GLOBAL char *A = dev::gptr((const char *)nodes) + ((uint64_t)row * (unsigned)nx + (unsigned)c0) * kRec;
    const int64_t sy = (int64_t)nx * kRec, sz = (int64_t)ny * sy;
    T fb[8], fj[8];
#pragma unroll
    for (int q = 0; q < 8; q++) {
        const FQ_GLOBAL char *r = A + ((q & 2) ? sy : 0) + ((q & 4) ? sz : 0) + ((q & 1) ? kRec : 0);
        fb[q] = (T) * (const FQ_GLOBAL S *)(r + ob);
        if (TW) fj[q] = (T) * (const FQ_GLOBAL S *)(r + oj);
    }
    coeffs<T>(fb, cb);
    if (TW) coeffs<T>(fj, cj);
}

}  // namespace quad
}  // namespace fq
