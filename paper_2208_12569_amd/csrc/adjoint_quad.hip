// trace_backward (adjoint.hip) for RKF45 in FP64 with four lanes to a half line, as the tracer's
// trace_quad.h: lane c < 3 holds component c of the cell's polynomials, of the stages, of
// the adjoint and of the cell's gradient sums.
//
// Bound by instruction issue: about 1500 vector instructions for the adjoint of an
// accepted step and 900 for each trial of its replay, with two waves per SIMD. At that
// (256 registers) the form with twist spills 94 registers, 240 bytes of scratch a lane; the
// one without takes 216 and spills none. The atomic
// adds of the cells' sums to the nodes cost 1.9 ms of 5.7 while each component had a plane
// of its own, and 0.5 ms since a node's values lie side by side, where the three lanes of a
// half line add to one cache line. One lane to a line
// needs 510 registers, so one wave per SIMD, and the replay buffer, sized by half lines,
// gave it 512 waves for 1024 SIMDs; four lanes make that 2048 waves at two per SIMD. The
// map, loss and gradient of a 256 x 256 plane on a 128x128x96 field in FP64 9.43 -> 7.68 -> 6.24 ms.
#include <math.h>

#include "adjoint_dev.h"
#include "fq_internal.h"
#include "stencil_dev.h"
#include "trace_quad.h"

namespace fq {
namespace {

using namespace adj;
using namespace dev;
using quad::all3;
using quad::any;
using quad::from;

// Fehlberg 4(5): stages, and the weights of the fifth-order solution.
constexpr double kA[6][5] = {{0.0, 0.0, 0.0, 0.0, 0.0},
                             {1.0 / 4.0, 0.0, 0.0, 0.0, 0.0},
                             {3.0 / 32.0, 9.0 / 32.0, 0.0, 0.0, 0.0},
                             {1932.0 / 2197.0, -7200.0 / 2197.0, 7296.0 / 2197.0, 0.0, 0.0},
                             {439.0 / 216.0, -8.0, 3680.0 / 513.0, -845.0 / 4104.0, 0.0},
                             {-8.0 / 27.0, 2.0, -3544.0 / 2565.0, 1859.0 / 4104.0, -11.0 / 40.0}};
constexpr double kB[6] = {16.0 / 135.0, 0.0, 6656.0 / 12825.0, 28561.0 / 56430.0, -9.0 / 50.0, 2.0 / 55.0};

// One accepted step found by a replay. Every lane writes and reads its own slots: its
// coordinate before the step and its cell index; lane 3 the step length and the landing
// axis + 1 (bits 0-1) and clamped coordinates (bits 2-4).
struct QuadRec {
    double v[4];
    int32_t w[4];
};
static_assert(sizeof(QuadRec) <= sizeof(StepRec), "the replay buffer is sized for StepRec");

template <typename T> __device__ __forceinline__ T sum3(T x)
{
    T v[3];
    all3(x, v);
    return v[0] + v[1] + v[2];
}

// The adjoint of one accepted step, in the terms of step_adjoint (adjoint.hip): p, lam
// this lane's coordinate and adjoint. B, curl B and 1/|B| of the stages are kept from the
// forward stages to their adjoints.
template <typename T, bool TW>
__device__ __forceinline__ void step_adjoint(const T cb[8], const T cj[8], const quad::Line<T> &L, T twk, T p,
                                             T H, int ax, int clamp, int endb, T &lam, T ltw, T gB[8], T gJ[8])
{
    const int c = L.c;
    const bool landing = ax >= 0, mine = ax == c;
    T y[6], k[6], b[6], j[6], inv[6], ig[6], jb[6];
#pragma unroll
    for (int st = 0; st < 6; st++) {
        T acc = T(0), Y[3], B[3];
#pragma unroll
        for (int q = 0; q < st; q++) acc += (T)kA[st][q] * k[q];
        y[st] = p + H * acc;
        all3(y[st], Y);
        b[st] = poly<T>(cb, Y[0], Y[1], Y[2]);
        all3(b[st], B);
        inv[st] = T(1) / sqrt(B[0] * B[0] + B[1] * B[1] + B[2] * B[2]);
        const T F = L.sgn * inv[st] * b[st] * L.r;
        j[st] = TW && kB[st] != 0.0 ? poly<T>(cj, Y[0], Y[1], Y[2]) : T(0);
        jb[st] = TW && kB[st] != 0.0 ? sum3(j[st] * b[st]) : T(0);
        k[st] = F;
        ig[st] = T(1);
        if (landing) {
            const T g = quad::one(F, mine);
            k[st] = F / g;
            ig[st] = T(1) / g;
        }
    }
    T lo = mine ? T(0) : lam;
    int bx = -1;
    if (endb >= 0 && endb != ax) bx = endb;
    else if (endb < 0 && clamp) bx = (clamp & 1) ? 0 : ((clamp & 2) ? 1 : 2);
    if (bx >= 0) {
        // ends on box face bx without landing there: slide along the line onto the face
        T dy = T(0), P[3], B[3];
#pragma unroll
        for (int st = 0; st < 6; st++) dy += (T)kB[st] * k[st];
        all3(p + H * dy, P);
        const T be = poly<T>(cb, P[0], P[1], P[2]);
        all3(be, B);
        const T ie = T(1) / sqrt(B[0] * B[0] + B[1] * B[1] + B[2] * B[2]);
        const T Fe = L.sgn * ie * be * L.r;
        T s = sum3(c == bx ? T(0) : lam * Fe);
        if (TW) s += ltw * twk * sum3(poly<T>(cj, P[0], P[1], P[2]) * be) * ie * ie;
        lo = c == bx ? -s / Fe : lam;
    }
    // dL/dH: this lane's share, and the twist's
    T mu[6], dh = T(0), dht = T(0);
#pragma unroll
    for (int st = 0; st < 6; st++) {
        mu[st] = H * (T)kB[st] * lo;
        dh += (T)kB[st] * k[st] * lo;
        if (TW) dht += ltw * (T)kB[st] * (twk * jb[st] * inv[st] * inv[st]) * ig[st];
    }
    T ln = lo;
#pragma unroll
    for (int st = 5; st >= 0; st--) {
        const bool tw = TW && kB[st] != 0.0;
        T Y[3];
        all3(y[st], Y);
        const T i2 = inv[st] * inv[st];
        const T tau = tw ? H * (T)kB[st] * ltw : T(0);
        T Fb = mu[st], Gb = tau;
        if (landing) {
            const T mk = sum3(mu[st] * k[st]);
            Fb *= ig[st];
            Gb *= ig[st];
            if (mine) Fb += -mk * ig[st] - tau * (twk * jb[st] * i2) * ig[st] * ig[st];
        }
        const T d = b[st] * inv[st], db = L.sgn * L.r * Fb;
        T Bb = (db - sum3(db * d) * d) * inv[st], Jb = T(0);
        if (tw) {
            // G = twk (J.B) / |B|^2
            Jb = twk * Gb * b[st] * i2;
            Bb += twk * Gb * (j[st] * i2 - T(2) * jb[st] * i2 * i2 * b[st]);
        }
        T e[3], g[3];
        poly_grad(cb, Y[0], Y[1], Y[2], g);
#pragma unroll
        for (int a = 0; a < 3; a++) e[a] = Bb * g[a];
        if (tw) {
            poly_grad(cj, Y[0], Y[1], Y[2], g);
#pragma unroll
            for (int a = 0; a < 3; a++) e[a] += Jb * g[a];
        }
        const T s0 = sum3(e[0]), s1 = sum3(e[1]), s2 = sum3(e[2]);
        const T yb = c == 0 ? s0 : (c == 1 ? s1 : (c == 2 ? s2 : T(0)));
#pragma unroll
        for (int q = 0; q < 8; q++) {
            const T wq = tri_w(q, Y[0], Y[1], Y[2]);
            gB[q] += Bb * wq;
            if (tw) gJ[q] += Jb * wq;
        }
        ln += yb;
#pragma unroll
        for (int q = 0; q < st; q++) {
            mu[q] += H * (T)kA[st][q] * yb;
            dh += (T)kA[st][q] * (yb * k[q]);
        }
    }
    const T dH = sum3(dh) + dht;
    if (mine && bx < 0) ln -= dH;  // H = face - p_axis
    lam = ln;
}

// This lane's component of the cell's sums to the nodes.
template <typename T, bool TW>
__device__ __forceinline__ void flush_cell(double *gnode, int nx, int ny, int c, int cell, T gB[8], T gJ[8])
{
    const int c0 = from<0>(cell), c1 = from<1>(cell), c2 = from<2>(cell);
    constexpr int kNode = TW ? 6 : 3;
    const int64_t sy = (int64_t)nx * kNode, sz = sy * ny;
    double *g = gnode + (c2 * sz + c1 * sy + c0 * kNode + c);
#pragma unroll
    for (int q = 0; q < 8; q++) {
        double *o = g + (q & 1) * kNode + ((q >> 1) & 1) * sy + ((q >> 2) & 1) * sz;
        if (c < 3 && gB[q] != T(0)) atomicAdd(o, (double)gB[q]);
        gB[q] = T(0);
        if (TW) {
            if (c < 3 && gJ[q] != T(0)) atomicAdd(o + 3, (double)gJ[q]);
            gJ[q] = T(0);
        }
    }
}

template <typename T, typename S, bool TW>
__global__ __launch_bounds__(64, 2) void trace_backward_quad_kernel(const TraceJob *__restrict__ jobs, BwdParams bp)
{
    const TraceJob &J = jobs[0];
    const int c = (int)threadIdx.x & 3;
    const int64_t slot = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 2;
    if (slot >= bp.nslots) return;
    QuadRec *buf = (QuadRec *)(bp.buf + slot * bp.seg);
    const int nx = J.n[0], ny = J.n[1];
    quad::Const<T> K;
    K.twk = (T)J.twk;
    K.bnull2 = (T)((double)Num<T>::null_rel * (double)(*J.bmax2));
    K.max_steps = (uint32_t)(bp.max_steps < 0xfffffffell ? bp.max_steps : 0xfffffffell);
    const bool str = J.geo != nullptr;
    const double dref = str ? J.geo->dref : 0.0;
    if (str) K.twk = (T)(dref * (0.25 / M_PI));
    quad::Line<T> L{};
    L.c = c;
    L.n = c < 3 ? J.n[c] : 4;
    L.r = c < 3 ? (T)J.rscale[c] : T(0);
    T cb[8], cj[8], gB[8], gJ[8];
#pragma unroll
    for (int q = 0; q < 8; q++) gB[q] = gJ[q] = T(0);
    auto fetch = [&]() {
        quad::load_cell<T, S, TW, TW>(J.nodes, nx, ny, L, cb, cj);
        if (str && c < 3) L.r = (T)(dref * J.iw[c][L.cell]);
    };
    auto pick = [&](auto a0, auto a1, auto a2, auto a3) { return c == 0 ? a0 : (c == 1 ? a1 : (c == 2 ? a2 : a3)); };
    unsigned long long n_half = 0, n_steps = 0, n_bad = 0, n_drop = 0;
    // A quad reverses its half line one segment per iteration and takes the next half
    // line as soon as its own is done.
    int64_t h = -1;       // the quad's half line, -1 = none
    bool drained = false; // the queue is empty
    T lam = T(0), ltw = T(0);
    int endax = -1, ckslot = -1, next = -1, ck = -1, nck = 0, nacc = 0, rj = 0;
    bool bad = false;
    for (;;) {
        while (h < 0 && !drained) {
            unsigned long long hq = 0;
            if (c == 0) hq = atomicAdd(bp.counter, 1ull);
            hq = (unsigned long long)(unsigned)from<0>((int)hq) |
                 ((unsigned long long)(unsigned)from<0>((int)(hq >> 32)) << 32);
            if (hq >= (unsigned long long)bp.nhalves) {
                drained = true;
                break;
            }
            // long half lines first: they set the end of the launch
            const int64_t hh = bp.order ? (int64_t)bp.order[hq] : (int64_t)hq;
            // the half's own job (a rotated-S0 job's halves follow the plane's) and
            // its record there
            rj = hh >= bp.nhalf0 ? 1 : 0;
            const TraceJob &Jh = jobs[rj];
            const int64_t lh = hh - (rj ? bp.nhalf0 : 0);
            // in physical units here; in local units (times the end cell's widths) once
            // the replay of the last segment has found that cell
            lam = c < 3 ? (T)bp.lam_end[3 * hh + c] : T(0);
            // the end lies on its box face: only its in-face coordinates can move
            const int fe = Jh.rec.face[lh];
            endax = fe >= 0 ? (fe >> 1) : -1;
            if (endax == c) lam = T(0);
            ltw = TW ? (T)bp.lam_tw[hh] : T(0);
            if (any(lam != T(0)) == 0 && ltw == T(0)) continue;
            const uint16_t st = Jh.rec.st[lh];
            nck = bp.tape_n[hh];
            nacc = bp.tape_acc[hh];
            if (st & sten::kFatal) {
                n_drop++;  // a line the forward map has but this pass could not keep
                continue;
            }
            if (nck <= 0 || nacc <= 0) continue;  // no step taken (a seed on its exit face)
            L.sgn = lh >= Jh.nlines ? T(1) : T(-1);
            n_half++;
            bad = false;
            ckslot = bp.tape_last[hh];
            next = -1;
            ck = nck - 1;
            h = hh;
        }
        if (__ballot(h >= 0) == 0) break;  // every quad is drained
        if (h < 0) continue;
        {
            // replay the segment from its checkpoint
            const Ckpt &cp = bp.tape[ckslot];
            const int prev = cp.prev;
            const int seedcell = pick(cp.c0, cp.c1, cp.c2, 0);
            L.cell = seedcell;
            L.P[0] = (T)cp.p0, L.P[1] = (T)cp.p1, L.P[2] = (T)cp.p2;
            L.p = pick(L.P[0], L.P[1], L.P[2], T(0.5));
            L.h = (T)cp.h, L.tol = (T)cp.tol;
            L.tw = 0.0, L.len = 0.0;
            L.trials = cp.trials;
            L.force = cp.force;
            const bool last = ck == nck - 1;
            const int target = last ? nacc - ck * bp.seg : bp.seg;
            if (target < 0 || target > bp.seg || (target == 0 && !last)) bad = true;
            int nrec = 0;
            if (!bad) {
                fetch();
                unsigned acc = 0;
                int cap_axis = -1, cap_clamp = 0;
                double cap_H = 0.0;
                const Capture capture{&cap_axis, &cap_H, &cap_clamp};
                for (;;) {
                    if (nrec == target && !last) break;
                    const T p = L.p;
                    const int cell = L.cell;
                    int fin_st = -1, fin_face = -1;
                    bool need_load = false;
                    const unsigned before = acc;
                    quad::iterate<T, TW, false, Capture>(L, cb, cj, K, fin_st, fin_face, need_load, acc, capture);
                    if (acc != before) {
                        if (nrec >= target) {
                            bad = true;
                            break;
                        }
                        buf[nrec].v[c] = c < 3 ? (double)p : cap_H;
                        buf[nrec].w[c] = c < 3 ? cell : ((cap_axis + 1) | (cap_clamp << 2));
                        nrec++;
                    }
                    if (fin_st >= 0) {
                        if (fin_st != 0 || nrec != target || !last) bad = true;
                        break;
                    }
                    if (need_load) fetch();
                }
                if (!bad && last && c < 3) {
                    // the end's adjoint into the local units of the cell it ends in
                    lam *= (T)(str ? 1.0 / J.iw[c][L.cell] : J.spacing[c]);
                }
                if (!bad && !last) {
                    const Ckpt &nx_ = bp.tape[next];
                    const bool off = L.cell != pick(nx_.c0, nx_.c1, nx_.c2, L.cell) ||
                                     (double)L.p != pick(nx_.p0, nx_.p1, nx_.p2, (double)L.p) ||
                                     nx_.h != (double)L.h;
                    if (any(off)) bad = true;
                }
            }
            if (!bad) {
                // reverse sweep over the segment
                L.cell = -1;
                double v = 0.0;
                int w = 0;
                if (nrec > 0) v = buf[nrec - 1].v[c], w = buf[nrec - 1].w[c];
                for (int r = nrec - 1; r >= 0; r--) {
                    const T p = c < 3 ? (T)v : T(0.5);
                    const T H = (T)from<3>(v);
                    const int code = from<3>(w), cell = c < 3 ? w : 0;
                    if (r > 0) v = buf[r - 1].v[c], w = buf[r - 1].w[c];
                    if (any(cell != L.cell)) {
                        if (r != nrec - 1) flush_cell<T, TW>(bp.gnode, nx, ny, c, L.cell, gB, gJ);
                        L.cell = cell;
                        fetch();
                    }
                    const int endb = (last && r == nrec - 1) ? endax : -1;
                    step_adjoint<T, TW>(cb, cj, L, K.twk, p, H, (code & 3) - 1, code >> 2, endb, lam, ltw, gB, gJ);
                    n_steps++;
                }
                if (nrec > 0) flush_cell<T, TW>(bp.gnode, nx, ny, c, L.cell, gB, gJ);
                if (ck == 0 && rj == 1 && bp.lam_seed && c < 3) {
                    // a rotated-S0 line's adjoint at its seed, which depends on B0 (its
                    // offset along U or V): local units -> physical
                    const int64_t lh = h - bp.nhalf0;
                    bp.lam_seed[3 * lh + c] = (double)lam * (str ? J.iw[c][seedcell] : 1.0 / J.spacing[c]);
                }
                next = ckslot;
                ckslot = prev;
                ck--;
            }
        }
        if (bad || ckslot < 0 || ck < 0) {
            if (!bad && (ck != -1 || ckslot != -1)) bad = true;  // the chain and the count disagree
            if (bad) n_bad++;
            h = -1;
        }
    }
    if (bp.stats && c == 0) {
        if (n_half) atomicAdd(bp.stats + 0, n_half);
        if (n_steps) atomicAdd(bp.stats + 1, n_steps);
        if (n_bad) atomicAdd(bp.stats + 2, n_bad);
        if (n_drop) atomicAdd(bp.stats + 3, n_drop);
    }
}

}  // namespace

hipError_t launch_trace_backward_quad(int want_tw, const TraceJob *job_dev, const BwdParams &bp, hipStream_t s)
{
    const dim3 grid((unsigned)((4 * bp.nslots + 63) / 64)), blk(64);
    if (want_tw) hipLaunchKernelGGL((trace_backward_quad_kernel<double, double, true>), grid, blk, 0, s, job_dev, bp);
    else hipLaunchKernelGGL((trace_backward_quad_kernel<double, double, false>), grid, blk, 0, s, job_dev, bp);
    return hipGetLastError();
}

}  // namespace fq
