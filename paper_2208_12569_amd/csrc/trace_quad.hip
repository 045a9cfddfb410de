// Tracer with four lanes to a half line, for launches of few lines: RKF45, Method I and
// II, the adjoint's forward pass, uniform and stretched grids, any number of jobs
// (trace.hip has the queue, the records and everything else that the two kernels share in
// meaning; trace_quad.h the step). Results are those of trace_kernel, bit for bit.
//
// Bound by the latency of the longest line's trial steps, one after the other: a step is
// about 60 % of the one-lane step's instructions in a row, because each lane evaluates
// one component of the field and its curl instead of three, and a cell's records are
// fetched by three lanes, one component each. Against one lane to a line, whole calls: a
// 32 x 32 plane of 64^3 nodes 1097 -> 761 us, a 128 x 128 one in FP64 812 -> 676 (both
// without a tile order), an interior cut of 157 x 211 points 1612 -> 1224, 30001 seeds from
// a list 3352 -> 2895; through the FP64 re-trace of an FP32 pass also large calls, a 1024 x 1024 plane 4951 -> 4457, eight in a
// batch 32.7 -> 27.1 ms; the map, loss and gradient of a 256 x 256 plane, whose forward
// pass this is as well, 6.26 -> 6.12 ms.
#include "fq_internal.h"
#include "trace_quad.h"

namespace fq {
namespace {

using namespace dev;
using quad::all3;

// A checkpoint of the adjoint's forward pass (store_ckpt in trace.hip).
template <typename T> __device__ __forceinline__ bool store_ckpt(const TraceParams &tp, int &last, const quad::Line<T> &L)
{
    unsigned long long slot = 0;
    if (L.c == 0) slot = atomicAdd(tp.pool_ctr, 1ull);
    slot = (unsigned long long)(unsigned)quad::from<0>((int)slot) |
           ((unsigned long long)(unsigned)quad::from<0>((int)(slot >> 32)) << 32);
    if (slot >= (unsigned long long)tp.pool_cap) return false;  // the pool is exhausted
    const int c0 = quad::from<0>(L.cell), c1 = quad::from<1>(L.cell), c2 = quad::from<2>(L.cell);
    if (L.c == 0) {
        Ckpt c;
        c.p0 = (double)L.P[0];
        c.p1 = (double)L.P[1];
        c.p2 = (double)L.P[2];
        c.h = (double)L.h;
        c.tol = (double)L.tol;
        c.c0 = c0;
        c.c1 = c1;
        c.c2 = c2;
        c.force = L.force;
        c.trials = (int32_t)L.trials;
        c.prev = last;
        gptr(tp.tape)[slot] = c;
    }
    last = (int)slot;
    return true;
}

// TWM as trace_kernel's: 0 no twist (narrow records), 1 twist, 2 positions only on wide
// records. TAPE: the adjoint's forward pass. Runs only if the queue holds at most `most`
// items.
template <typename T, typename S, int TWM, bool M2, bool TAPE>
__global__ __launch_bounds__(256, sizeof(T) == 4 ? (M2 ? 3 : 4) : (M2 ? 2 : 3)) void trace_quad_kernel(
    const TraceJob *__restrict__ jobs, TraceParams tp, unsigned long long *__restrict__ counter, int64_t most)
{
    using N = Num<T>;
    constexpr bool TW = TWM == 1;
    const int lane = (int)threadIdx.x & 63;
    const int c = lane & 3;
    constexpr unsigned long long kFirst = 0x1111111111111111ull;  // lane 0 of every quad

    int64_t total = tp.static_items;
    if (tp.list) {
        total = (int64_t)(*tp.list_count);
        if (total > tp.list_cap) total = tp.list_cap;
    } else if (tp.dynamic_last) {
        total = *tp.total_dev;
    }
    if (total > most) return;
    // waves without an item end at once, ranked across the blocks first (see trace_kernel)
    if ((int64_t)((threadIdx.x >> 6) * gridDim.x + blockIdx.x) * 16 >= total) return;

    int jb = -1;
    bool exhausted = false, need_load = false, fresh = false, str = false;
    int64_t rec = 0;
    double dref_s = 0.0;
    const void *nodes = nullptr;
    int nx = 0, ny = 0;
    quad::Line<T> L{};
    quad::Const<T> K{};
    L.c = c;
    K.max_steps = (uint32_t)(tp.max_steps < 0xfffffffell ? tp.max_steps : 0xfffffffell);
    T cb[8], cj[8];
    unsigned n_trial = 0, n_acc = 0, n_fetch = 0, n_half = 0;
    int acc_half = 0, nck = 0, last_ck = -1;  // TAPE: steps, checkpoints, the last one's slot

    for (;;) {
        int fin_st = -1, fin_face = -1;

        // ---- refill idle quads: one atomic per wave -------------------------------------
        const bool need = (jb < 0) && !exhausted;
        unsigned long long m = __ballot(need) & kFirst;
        // (few lines: an idle quad waits for three more only while others run)
        if (m && __popcll(m) < 4 && __ballot(jb >= 0) != 0) m = 0;
        if (m) {
            const int leader = __ffsll((long long)m) - 1;
            unsigned long long base = 0;
            if (lane == leader) base = atomicAdd(counter, (unsigned long long)__popcll(m));
            base = shfl_u64(base, leader);
            if (need) {
                const int64_t it = (int64_t)(base + (unsigned long long)__popcll(m & ((1ull << (lane & ~3)) - 1ull)));
                if (it >= total) {
                    exhausted = true;
                } else {
                    int j = 0;
                    LineAt at;
                    bool forward;
                    if (tp.list) {
                        const FixEntry e = gptr(tp.list)[it];
                        j = e.job;
                        at = line_at(jobs[j], e.line);
                        forward = e.half != 0;
                    } else {
                        while (j + 1 < tp.njobs &&
                               !(it >= jobs[j].item_base && it < jobs[j].item_base + 2 * jobs[j].nitems))
                            j++;
                        const TraceJob &J = jobs[j];
                        const int64_t local = it - J.item_base;
                        if (seeds_on_grid(J)) {
                            forward = ((local >> 6) & 1) == 0;
                            at = line_of_item(J, ((local >> 7) << 6) | (local & 63));
                        } else {
                            forward = local < J.nitems;
                            at = line_of_item(J, forward ? local : local - J.nitems);
                        }
                    }
                    if (at.line >= 0) {
                        const TraceJob &J = jobs[j];
                        double r[3], nrm[3];
                        seed_of_line<false>(J, at, r, nrm);
                        jb = j;
                        nodes = J.nodes;
                        nx = J.n[0];
                        ny = J.n[1];
                        K.twk = (T)J.twk;
                        K.bnull2 = (T)((double)N::null_rel * (double)(*J.bmax2));
                        str = J.geo != nullptr;
                        if (str) {
                            dref_s = J.geo->dref;
                            K.twk = (T)(dref_s * (0.25 / M_PI));
                        }
                        rec = (forward ? J.nlines : 0) + at.line;
                        L.sgn = forward ? T(1) : T(-1);
                        L.tw = 0.0;
                        L.len = 0.0;
                        L.trials = 0;
                        L.force = -1;
                        if (TAPE) acc_half = 0, nck = 0, last_ck = -1;
                        bool in = !(str && J.geo->bad);
                        int cell[3] = {0, 0, 0};
                        for (int a = 0; a < 3; a++) {
                            const FQ_GLOBAL double *x = gptr(J.planes.coord[a]);
                            double q;
                            if (str) {
                                if (x) in = in && r[a] >= x[0] && r[a] <= x[J.n[a] - 1];
                                else in = in && r[a] >= J.origin[a] &&
                                          r[a] <= J.origin[a] + (J.n[a] - 1) * J.spacing[a];
                                cell[a] = in ? str_cell(J, a, r[a], q) : 0;
                                L.P[a] = in ? (T)q : T(0);
                            } else {
                                const double g = (r[a] - J.origin[a]) * J.inv_spacing[a];
                                in = in && g >= 0.0 && g <= (double)(J.n[a] - 1);
                                cell[a] = in ? min(max((int)floor(g), 0), J.n[a] - 2) : 0;
                                L.P[a] = (T)(g - cell[a]);
                            }
                        }
                        if (!in) {
                            fin_st = str && J.geo->bad ? FQ_ST_NONFINITE : FQ_ST_OUTSIDE;
                        } else {
                            L.cell = c == 0 ? cell[0] : (c == 1 ? cell[1] : (c == 2 ? cell[2] : 0));
                            L.p = c == 0 ? L.P[0] : (c == 1 ? L.P[1] : (c == 2 ? L.P[2] : T(0.5)));
                            L.n = c < 3 ? J.n[c] : 4;
                            L.r = c < 3 ? (T)J.rscale[c] : T(0);
                            need_load = true;
                            fresh = true;
                        }
                    }
                }
            }
        }

        // ---- fetch the cell --------------------------------------------------------------
        if (jb >= 0 && need_load) {
            quad::load_cell<T, S, TW, TWM != 0>(nodes, nx, ny, L, cb, cj);
            need_load = false;
            n_fetch++;
            if (str && c < 3) L.r = (T)(dref_s * gptr(jobs[jb].iw[c])[L.cell]);
            if (fresh) {
                // Eq. step and Eq. tol from the field angle |Bn0/B| at the seed (see
                // trace_kernel)
                fresh = false;
                const TraceJob &J = jobs[jb];
                T B[3], R[3];
                all3(poly<T>(cb, L.P[0], L.P[1], L.P[2]), B);
                all3(L.r, R);
                const float bx = (float)B[0], by = (float)B[1], bz = (float)B[2];
                const float b2 = bx * bx + by * by + bz * bz;
                const float n0 = (float)J.normal[0], n1 = (float)J.normal[1], n2 = (float)J.normal[2];
                const float bn = bx * n0 + by * n1 + bz * n2;
                const bool on_face = quad::any(c < 3 && ((L.cell == 0 && L.p == T(0)) ||
                                                         (L.cell == L.n - 2 && L.p == T(1)))) != 0;
                const float amin = on_face ? 1e-9f : 0.05f;
                float ang = (J.kind == SEED_ROTATED || M2) ? 1.0f : fabsf(bn) * Num<float>::rsq(b2);
                if (!(ang >= amin)) ang = amin;  // also catches NaN
                if (ang > 1.0f) ang = 1.0f;
                L.h = (T)fmaxf((float)tp.step_perp * ang, (float)tp.step_min);
                if (str) {
                    const float sx = bx * (float)R[0], sy = by * (float)R[1], sz = bz * (float)R[2];
                    const float w2 = sx * sx + sy * sy + sz * sz;
                    if (w2 > 0.0f) L.h = (T)((float)L.h * sqrtf(b2 / w2));
                }
                L.tol = (T)fmax(tp.tol_perp * (double)(ang * sqrtf(ang)), tp.tol_floor);
                if constexpr (M2) {
                    const T inv = N::rsq(N::fma_(B[0], B[0], N::fma_(B[1], B[1], B[2] * B[2])));
                    const T b[3] = {B[0] * inv, B[1] * inv, B[2] * inv};
                    int a = 0;
                    if (fabs(b[1]) < fabs(b[a])) a = 1;
                    if (fabs(b[2]) < fabs(b[a])) a = 2;
                    T u[3] = {a == 0 ? T(0) : (a == 1 ? b[2] : -b[1]),
                              a == 0 ? -b[2] : (a == 1 ? T(0) : b[0]),
                              a == 0 ? b[1] : (a == 1 ? -b[0] : T(0))};
                    const T iu = N::rsq(N::fma_(u[0], u[0], N::fma_(u[1], u[1], u[2] * u[2])));
                    for (int q = 0; q < 3; q++) u[q] *= iu;
                    const T v[3] = {b[1] * u[2] - b[2] * u[1], b[2] * u[0] - b[0] * u[2],
                                    b[0] * u[1] - b[1] * u[0]};
                    const T is = c < 3 ? (T)J.inv_spacing[c] : T(0);
                    L.u = (c == 0 ? u[0] : (c == 1 ? u[1] : u[2])) * is;
                    L.v = (c == 0 ? v[0] : (c == 1 ? v[1] : v[2])) * is;
                }
                if (TAPE) {
                    if (store_ckpt(tp, last_ck, L)) nck++;
                    else fin_st = FQ_ST_MAXSTEPS | FQ_ST_NOTAPE;  // no checkpoint space
                }
            }
        }

        // ---- one trial step ---------------------------------------------------------------
        if (jb >= 0 && fin_st < 0) {
            n_trial++;
            const unsigned acc_before = n_acc;
            quad::iterate<T, TW, M2>(L, cb, cj, K, fin_st, fin_face, need_load, n_acc);
            if (TAPE && n_acc != acc_before) {
                acc_half++;
                if (fin_st < 0 && acc_half % tp.seg == 0) {
                    if (store_ckpt(tp, last_ck, L)) {
                        nck++;
                    } else {
                        fin_st = FQ_ST_MAXSTEPS | FQ_ST_NOTAPE;  // no checkpoint space
                        fin_face = -1;
                    }
                }
            }
        }

        // ---- write the record of a finished half line -------------------------------------
        if (jb >= 0 && fin_st >= 0) {
            const TraceJob &J = jobs[jb];
            const bool bad = (fin_st & (FQ_ST_OUTSIDE | FQ_ST_NULLB | FQ_ST_MAXSTEPS | FQ_ST_NONFINITE)) != 0;
            if (c < 3) {
                double e = NAN;
                if (!bad && L.len == 0.0) {
                    // no step taken: the half line ends exactly at its seed
                    double r[3], nrm[3];
                    seed_of_line<false>(J, line_at(J, rec >= J.nlines ? rec - J.nlines : rec), r, nrm);
                    e = c == 0 ? r[0] : (c == 1 ? r[1] : r[2]);
                } else if (!bad && str) {
                    e = grid_pos(J, c, L.cell, (double)L.p);
                } else if (!bad) {
                    e = J.origin[c] + ((double)L.cell + (double)L.p) * J.spacing[c];
                }
                gptr(J.rec.end)[3 * rec + c] = e;
                if constexpr (M2) {
                    FQ_GLOBAL double *uv = gptr(J.rec.uv) + 6 * rec;
                    uv[c] = bad ? NAN : (double)L.u * J.spacing[c];
                    uv[3 + c] = bad ? NAN : (double)L.v * J.spacing[c];
                }
            }
            if (c == 0) {
                if (TWM != 2) gptr(J.rec.tw)[rec] = bad ? NAN : (TW ? L.tw : NAN);
                gptr(J.rec.len)[rec] = bad ? NAN : L.len * (str ? dref_s : J.dref);
                gptr(J.rec.face)[rec] = bad ? (int8_t)-1 : (int8_t)fin_face;
                gptr(J.rec.st)[rec] = (uint16_t)fin_st;
                if (TAPE) {
                    // a rotated-S0 job's halves follow the plane's
                    const int64_t trec = rec + (jb > 0 ? tp.tape_base1 : 0);
                    gptr(tp.tape_last)[trec] = last_ck;
                    gptr(tp.tape_n)[trec] = nck;
                    gptr(tp.tape_acc)[trec] = acc_half;
                }
            }
            jb = -1;
            need_load = false;
            n_half++;
        }

        if (__ballot(jb >= 0) == 0 && __ballot(!exhausted) == 0) break;
    }
    if (tp.stats) {
        const bool fix = tp.list != nullptr;
        unsigned long long v[5] = {n_trial, n_acc, n_fetch, fix ? 0u : n_half, fix ? n_half : 0u};
#pragma unroll
        for (int q = 0; q < 5; q++) {
            unsigned long long x = c == 0 ? v[q] : 0ull;
            for (int off = 32; off > 0; off >>= 1) {
                unsigned lo = __shfl_xor((unsigned)x, off), hi = __shfl_xor((unsigned)(x >> 32), off);
                x += ((unsigned long long)hi << 32) | lo;
            }
            if (lane == 0 && x) atomicAdd(tp.stats + q, x);
        }
    }
}

template <typename T, typename S> const void *pick(int twm, const TraceParams &tp)
{
    if constexpr (sizeof(T) == sizeof(S))
        if (tp.tape)
            return twm == 1 ? (const void *)trace_quad_kernel<T, S, 1, false, true>
                            : (const void *)trace_quad_kernel<T, S, 0, false, true>;
    if (tp.method == FQ_METHOD_II)
        return twm == 1 ? (const void *)trace_quad_kernel<T, S, 1, true, false>
                        : (const void *)trace_quad_kernel<T, S, 0, true, false>;
    if constexpr (sizeof(T) == 8)
        if (twm > 1) return (const void *)trace_quad_kernel<T, S, 2, false, false>;
    if constexpr (sizeof(T) == sizeof(S))
        if (twm == 1) return (const void *)trace_quad_kernel<T, S, 1, false, false>;
    return twm == 0 ? (const void *)trace_quad_kernel<T, S, 0, false, false> : nullptr;
}

}  // namespace

hipError_t launch_trace_quad(bool f64, bool s64, int twm, const TraceJob *jobs_dev, const TraceParams &tp,
                             unsigned long long *counter, int64_t most, int ncu, int block,
                             int waves_per_cu, hipStream_t s)
{
    const void *fn = !f64 ? pick<float, float>(twm, tp)
                     : s64 ? pick<double, double>(twm, tp) : pick<double, float>(twm, tp);
    if (!fn || tp.list_rev) return hipErrorInvalidValue;
    const int per_cu = tracer_blocks_per_cu(fn, block, waves_per_cu);
    TraceParams p = tp;
    void *args[4] = {&jobs_dev, &p, &counter, &most};
    return hipLaunchKernel(fn, dim3((unsigned)(per_cu * ncu)), dim3((unsigned)block), args, 0, s);
}

}  // namespace fq
