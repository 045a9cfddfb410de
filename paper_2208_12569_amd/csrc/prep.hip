// Field ingest and curl preparation.
//
// One streaming pass over the caller's Bx, By, Bz planes writes, per node, the
// record the tracer gathers: (Bx, By, Bz, Jx, Jy, Jz, 0, 0) in the compute type,
// J = curl B by second-order differences (central inside, the one-sided
// second-order formula on boundary nodes; the stencil of the paper's Eq. grad_B,
// Section 4; on a stretched axis the derivative of the quadratic through the same
// three nodes), or (Bx, By, Bz, 0) without the twist integrand. Interleaving the six
// values of a node in one aligned record lets one grid cell be fetched with 16
// vector loads from about 5 cache lines instead of 48 scalar gathers from six
// planes.
// The pass also reduces max |B|^2, the scale of the null-field test.
#include <float.h>

#include "fq_internal.h"

namespace fq {
namespace {

template <typename S>
__device__ __forceinline__ double ld(const S *p, int64_t i)
{
    return (double)p[i];
}

// d p / d axis at node (i,j,k) (stride = element distance along the axis).
template <typename S>
__device__ __forceinline__ double ddx(const S *p, int64_t q, int m, int n, int64_t stride,
                                      double inv_h)
{
    if (n < 3) return (ld(p, q - (int64_t)m * stride + stride) - ld(p, q - (int64_t)m * stride)) * inv_h;
    if (m == 0)
        return (-3.0 * ld(p, q) + 4.0 * ld(p, q + stride) - ld(p, q + 2 * stride)) * (0.5 * inv_h);
    if (m == n - 1)
        return (3.0 * ld(p, q) - 4.0 * ld(p, q - stride) + ld(p, q - 2 * stride)) * (0.5 * inv_h);
    return (ld(p, q + stride) - ld(p, q - stride)) * (0.5 * inv_h);
}

// The same on a stretched axis with node coordinates x: the derivative at node m of
// the quadratic through it and two other nodes (its neighbours inside, the next two
// inward on a boundary node), from the signed distances h1, h2 to them and the
// differences d1, d2 of p there: (d1 h2^2 - d2 h1^2) / (h1 h2 (h2 - h1)).
template <typename S>
__device__ __forceinline__ double ddx_s(const S *p, int64_t q, int m, int n, int64_t stride,
                                        const double *x)
{
    if (n < 3) return (ld(p, q - (int64_t)m * stride + stride) - ld(p, q - (int64_t)m * stride)) / (x[1] - x[0]);
    const int m1 = m == 0 ? 1 : (m == n - 1 ? n - 2 : m - 1);
    const int m2 = m == 0 ? 2 : (m == n - 1 ? n - 3 : m + 1);
    const double h1 = x[m1] - x[m], h2 = x[m2] - x[m];
    const double p0 = ld(p, q);
    const double d1 = ld(p, q + (int64_t)(m1 - m) * stride) - p0;
    const double d2 = ld(p, q + (int64_t)(m2 - m) * stride) - p0;
    return (d1 * h2 * h2 - d2 * h1 * h1) / (h1 * h2 * (h2 - h1));
}

template <typename S>
__device__ __forceinline__ double dax(const S *p, int64_t q, int m, int n, int64_t stride,
                                      double inv_h, const double *x)
{
    return x ? ddx_s(p, q, m, n, stride, x) : ddx(p, q, m, n, stride, inv_h);
}

template <typename T> struct V4;
template <> struct V4<float> { using t = float4; };
template <> struct V4<double> { using t = double4; };

// A block takes a 64 x 4 patch of x and z and marches along y through `depth` rows, kRows
// at a time: it asks for all of their values before it computes the first, since the pass
// waits on memory and what counts is how much a wave has on its way (with one row at a
// time it waited 90% of its time at 1.8 TB/s). A thread keeps its column's Bx and Bz of
// the rows below and at its node; the x and z neighbours are mostly other lanes' own
// values, in the caches: consecutive patches go to one XCD (blocks are dealt to the 8 XCDs
// in turn), x fastest, then z. A wave's records leave through LDS in the order they have
// in memory, 16 bytes a lane, so that every store fills whole lines.
// The bound is memory, 12 bytes read and 32 written per FP32 node. Against one row piece
// of 256 nodes per block iteration: 512x512x256 1.57 -> 0.70 ms (4.2 TB/s; a device copy
// reaches 5.1), 384^3 1.70 -> 0.60 ms, 256x256x128 0.19 -> 0.10 ms, 64^3 (where most lanes
// were past the row's end) 35 -> 19 us; FP32 planes to FP64 records of 384^3 2.39 -> 1.01 ms.
constexpr int kRows = 4;
constexpr int64_t kMostBlocks = 1 << 23;

// LDS that a wave's lanes exchange among themselves: what was written before is there for
// the other lanes after, and what was read before is read (no instruction, but the
// compiler moves no access across).
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The block's maximum to *bmax2, one atomic per block of 256 (non-negative floats order
// like ints).
__device__ __forceinline__ void block_max(float local, float *__restrict__ bmax2)
{
    for (int off = 32; off > 0; off >>= 1) {
        const float o = __shfl_xor(local, off);
        local = o > local ? o : local;
    }
    __shared__ float wmax[4];
    if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = local;
    __syncthreads();
    if (threadIdx.x == 0) {
        float m = 0.0f;
        for (int v = 0; v < 4; v++) m = wmax[v] > m ? wmax[v] : m;
        if (m > 0.0f) {
            if (m > FLT_MAX) m = FLT_MAX;
            // (most blocks see a larger maximum there already: thousands of atomics on one
            // word take longer than the pass)
            if (m > *(volatile float *)bmax2) atomicMax((int *)bmax2, __float_as_int(m));
        }
    }
}

template <typename S, typename T>
__global__ __launch_bounds__(256) void prep_kernel(const S *__restrict__ bx,
                                                   const S *__restrict__ by,
                                                   const S *__restrict__ bz, int nx, int ny,
                                                   int nz, double ihx, double ihy, double ihz,
                                                   const double *__restrict__ cx,
                                                   const double *__restrict__ cy,
                                                   const double *__restrict__ cz, int tx, int tz,
                                                   int depth, typename V4<T>::t *__restrict__ A,
                                                   float *__restrict__ bmax2)
{
// sums and differences round as written
#pragma clang fp contract(off)
    using V = typename V4<T>::t;
    // 16-byte pieces of the four waves' 64 records
    typedef float Piece __attribute__((ext_vector_type(4)));
    constexpr int kPieces = 2 * sizeof(V) / sizeof(Piece);
    __shared__ Piece out[4][64 * kPieces];
    const int lane = (int)threadIdx.x & 63, w = (int)threadIdx.x >> 6;
    const int64_t nxy = (int64_t)nx * ny;
    // patch of this block: gridDim.x / 8 consecutive ones per XCD (the grid is rounded up)
    const int64_t pt = (int64_t)(blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    const int64_t pxz = (int64_t)tx * tz;
    const int yc = (int)(pt / pxz);
    const int r = (int)(pt - yc * pxz);
    const int kb = r / tx, ib = r - kb * tx;
    const int i = ib * 64 + lane, k = kb * 4 + w;
    const int64_t j0 = (int64_t)yc * depth;
    const int j1 = (int)min((int64_t)ny, j0 + depth);
    const bool in = i < nx;
    float local = 0.0f;
    if (k < nz && j0 < ny) {  // uniform in a wave
        const int iq = in ? i : nx - 1;
        int64_t q = (int64_t)k * nxy + j0 * nx + iq;
        // interior nodes of uniform axes take the central differences from values loaded
        // here; the others go through dax (one-sided or unequal spacings)
        const bool zin = !cz && k > 0 && k < nz - 1, xin = !cx && iq > 0 && iq < nx - 1;
        const int64_t zs = zin ? nxy : 0, xs = xin ? 1 : 0;
        // Bx and Bz one row below and at the node
        S xm = S(0), zm = S(0), x0 = bx[q], z0 = bz[q];
        if (j0 > 0) xm = bx[q - nx], zm = bz[q - nx];
        for (int jr = (int)j0; jr < j1; jr += kRows) {
            // all of these rows' values first: the pass waits on memory, so what counts is
            // how much a wave has on its way at once
            S X[kRows + 2], Z[kRows + 2], Y[kRows], Xl[kRows], Xh[kRows], Yl[kRows], Yh[kRows], Zw[kRows], Ze[kRows],
                Yw[kRows], Ye[kRows];
            X[0] = xm, X[1] = x0, Z[0] = zm, Z[1] = z0;
#pragma unroll
            for (int v = 0; v < kRows; v++) {
                const int64_t p = q + (int64_t)min(v, ny - 1 - jr) * nx;
                const int64_t pn = q + (int64_t)min(v + 1, ny - 1 - jr) * nx;
                X[v + 2] = bx[pn];
                Z[v + 2] = bz[pn];
                Y[v] = by[p];
                Xl[v] = bx[p - zs], Xh[v] = bx[p + zs];
                Yl[v] = by[p - zs], Yh[v] = by[p + zs];
                Zw[v] = bz[p - xs], Ze[v] = bz[p + xs];
                Yw[v] = by[p - xs], Ye[v] = by[p + xs];
            }
#pragma unroll
            for (int v = 0; v < kRows; v++) {
                const int j = jr + v;
                if (j >= j1) break;
                const int64_t p = q + (int64_t)v * nx;
                const double dx0 = (double)X[v + 1], dy0 = (double)Y[v], dz0 = (double)Z[v + 1];
                V a, c;
                a.x = (T)dx0;
                a.y = (T)dy0;
                a.z = (T)dz0;
                double dyx = ((double)X[v + 2] - (double)X[v]) * (0.5 * ihy);
                double dyz = ((double)Z[v + 2] - (double)Z[v]) * (0.5 * ihy);
                double dzx = ((double)Xh[v] - (double)Xl[v]) * (0.5 * ihz);
                double dzy = ((double)Yh[v] - (double)Yl[v]) * (0.5 * ihz);
                double dxz = ((double)Ze[v] - (double)Zw[v]) * (0.5 * ihx);
                double dxy = ((double)Ye[v] - (double)Yw[v]) * (0.5 * ihx);
                if (cy || j == 0 || j == ny - 1) {
                    dyx = dax(bx, p, j, ny, nx, ihy, cy);
                    dyz = dax(bz, p, j, ny, nx, ihy, cy);
                }
                if (!zin) {
                    dzx = dax(bx, p, k, nz, nxy, ihz, cz);
                    dzy = dax(by, p, k, nz, nxy, ihz, cz);
                }
                if (!xin) {
                    dxz = dax(bz, p, iq, nx, 1, ihx, cx);
                    dxy = dax(by, p, iq, nx, 1, ihx, cx);
                }
                a.w = (T)(dyz - dzy);
                c.x = (T)(dzx - dxz);
                c.y = (T)(dxy - dyx);
                c.z = (T)0;
                c.w = (T)0;
                // the wave's 64 records in memory order (a wave's own rows: no block barrier)
                V *own = (V *)&out[w][kPieces * lane];
                own[0] = a;
                own[1] = c;
                wave_sync();
                Piece *row = (Piece *)(A + 2 * ((int64_t)k * nxy + (int64_t)j * nx + ib * 64));
                const int live = kPieces * min(64, nx - ib * 64);
#pragma unroll
                for (int u = 0; u < kPieces; u++)
                    if (lane + 64 * u < live) row[lane + 64 * u] = out[w][lane + 64 * u];
                wave_sync();
                const float fb2 = (float)(dx0 * dx0 + dy0 * dy0 + dz0 * dz0);
                if (in && fb2 > local) local = fb2;  // NaN compares false and is skipped
            }
            xm = X[kRows], zm = Z[kRows], x0 = X[kRows + 1], z0 = Z[kRows + 1];
            q += (int64_t)kRows * nx;
        }
    }
    block_max(local, bmax2);
}

// Records without twist need no neighbours: the three planes side by side, nodes in memory
// order whatever the rows are, four of a thread's on their way at once, a block's next to
// each other. Bound by memory, 12 bytes read and 16 written per FP32 node. By patches and
// rows as above, where the lanes past the ends of ragged rows wait too, FP32 planes to
// FP64 records of 65x400x400 nodes took 199 us for 110 here, 129x300x300 155 for 114, 256^3
// 173 for 163; FP32 records of 256x256x128 42 for 45. (Four nodes a grid apart: 256^3 from
// FP64 207 us for 188.)
template <typename S, typename T>
__global__ __launch_bounds__(256) void pack_kernel(const S *__restrict__ bx, const S *__restrict__ by,
                                                   const S *__restrict__ bz, int64_t nn,
                                                   typename V4<T>::t *__restrict__ A,
                                                   float *__restrict__ bmax2)
{
// sums and differences round as written
#pragma clang fp contract(off)
    constexpr int64_t step = 256;
    float local = 0.0f;
    for (int64_t q = (int64_t)blockIdx.x * kRows * step + threadIdx.x; q < nn;
         q += (int64_t)gridDim.x * kRows * step) {
        S X[kRows], Y[kRows], Z[kRows];
#pragma unroll
        for (int v = 0; v < kRows; v++) {
            const int64_t p = q + v * step < nn ? q + v * step : q;
            X[v] = bx[p], Y[v] = by[p], Z[v] = bz[p];
        }
#pragma unroll
        for (int v = 0; v < kRows; v++) {
            const int64_t p = q + v * step;
            if (p >= nn) break;
            const double x = (double)X[v], y = (double)Y[v], z = (double)Z[v];
            typename V4<T>::t a;
            a.x = (T)x;
            a.y = (T)y;
            a.z = (T)z;
            a.w = (T)0;
            A[p] = a;
            const float fb2 = (float)(x * x + y * y + z * z);
            if (fb2 > local) local = fb2;  // NaN compares false and is skipped
        }
    }
    block_max(local, bmax2);
}

// Stretched grids: 1 / width of every cell of every axis (a uniform axis repeats
// 1 / spacing), the smallest width, and whether all widths are positive and finite
// and the stretched axes span the box given by origin and spacing. One block of 256.
__global__ __launch_bounds__(256) void geometry_kernel(GeoIn g, double *__restrict__ iw0,
                                                       double *__restrict__ iw1,
                                                       double *__restrict__ iw2, Geo *__restrict__ geo)
{
    double wmin = INFINITY;
    int bad = 0;
    for (int a = 0; a < 3; a++) {
        double *iw = a == 0 ? iw0 : (a == 1 ? iw1 : iw2);
        const double *x = g.coord[a];
        for (int c = (int)threadIdx.x; c < g.n[a] - 1; c += (int)blockDim.x) {
            const double w = x ? x[c + 1] - x[c] : g.spacing[a];
            const bool ok = w > 0.0 && w <= DBL_MAX;  // false for NaN
            iw[c] = ok ? 1.0 / w : NAN;
            if (ok) wmin = w < wmin ? w : wmin;
            bad |= !ok;
        }
    }
    // the first and last nodes of a stretched axis are the box's extent
    if (threadIdx.x == 0)
        for (int a = 0; a < 3; a++) {
            const double *x = g.coord[a];
            if (!x) continue;
            const double lo = g.origin[a], hi = g.origin[a] + (g.n[a] - 1) * g.spacing[a];
            const double tol = 1e-12 * (hi - lo);
            if (!(fabs(x[0] - lo) <= tol) || !(fabs(x[g.n[a] - 1] - hi) <= tol)) bad = 1;
        }
    __shared__ double smin[256];
    __shared__ int sbad[256];
    smin[threadIdx.x] = wmin;
    sbad[threadIdx.x] = bad;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) {
            const double o = smin[threadIdx.x + h];
            smin[threadIdx.x] = o < smin[threadIdx.x] ? o : smin[threadIdx.x];
            sbad[threadIdx.x] |= sbad[threadIdx.x + h];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        geo->dref = smin[0];
        geo->bad = sbad[0];
        geo->pad = 0;
    }
}

__global__ void fill_u32_kernel(uint32_t *p, int64_t n, uint32_t v)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

template <typename S, typename T>
hipError_t run_prep(const fq_field &f, int want_tw, void *A, float *bmax2, hipStream_t s)
{
    using V = typename V4<T>::t;
    const S *const b[3] = {(const S *)f.b[0], (const S *)f.b[1], (const S *)f.b[2]};
    if (!want_tw) {
        const int64_t nn = f.n[0] * f.n[1] * f.n[2], need = (nn + 256 * kRows - 1) / (256 * kRows);
        const unsigned blocks = (unsigned)(need < 4096 ? need : 4096);
        hipLaunchKernelGGL((pack_kernel<S, T>), dim3(blocks), dim3(256), 0, s, b[0], b[1], b[2], nn, (V *)A,
                           bmax2);
        return hipGetLastError();
    }
    const int64_t tx = (f.n[0] + 63) / 64, tz = (f.n[2] + 3) / 4;
    // rows per block: about 4096 blocks where the grid has them (16 per CU), and no more
    // than 32 rows (the row before the first is read twice)
    int64_t depth = tx * tz * f.n[1] / 4096;
    depth = depth < 1 ? 1 : (depth > 32 ? 32 : depth);
    // (a launch has less than 2^32 threads, which thin grids of 4e9 nodes would pass)
    const int64_t pieces = kMostBlocks / (tx * tz);
    if (pieces * depth < f.n[1]) depth = pieces > 1 ? (f.n[1] + pieces - 1) / pieces : f.n[1];
    int64_t blocks = tx * tz * ((f.n[1] + depth - 1) / depth);
    blocks = (blocks + 7) / 8 * 8;
    hipLaunchKernelGGL((prep_kernel<S, T>), dim3((unsigned)blocks), dim3(256), 0, s, b[0], b[1], b[2],
                       (int)f.n[0], (int)f.n[1], (int)f.n[2], 1.0 / f.spacing[0], 1.0 / f.spacing[1],
                       1.0 / f.spacing[2], f.coord[0], f.coord[1], f.coord[2], (int)tx, (int)tz,
                       (int)depth, (V *)A, bmax2);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_geometry(const fq_field &f, double *const iw[3], Geo *geo, hipStream_t s)
{
    GeoIn g;
    for (int a = 0; a < 3; a++) {
        g.coord[a] = f.coord[a];
        g.n[a] = (int32_t)f.n[a];
        g.spacing[a] = f.spacing[a];
        g.origin[a] = f.origin[a];
    }
    hipLaunchKernelGGL(geometry_kernel, dim3(1), dim3(256), 0, s, g, iw[0], iw[1], iw[2], geo);
    return hipGetLastError();
}

hipError_t launch_fill_u32(uint32_t *p, int64_t n, uint32_t v, hipStream_t s)
{
    int64_t blocks = (n + 255) / 256;
    if (blocks < 1) blocks = 1;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(fill_u32_kernel, dim3((unsigned)blocks), dim3(256), 0, s, p, n, v);
    return hipGetLastError();
}

hipError_t launch_prep(const fq_field &f, int prec, int want_tw, void *A, float *bmax2,
                       hipStream_t s)
{
    if (f.dtype == FQ_DT_F32) {
        return prec == FQ_PREC_F64 ? run_prep<float, double>(f, want_tw, A, bmax2, s)
                                   : run_prep<float, float>(f, want_tw, A, bmax2, s);
    }
    return prec == FQ_PREC_F64 ? run_prep<double, double>(f, want_tw, A, bmax2, s)
                               : run_prep<double, float>(f, want_tw, A, bmax2, s);
}

}  // namespace fq
