// What the host layer (api.cpp) asks of the kernels for one call: linked with launcher
// stand-ins that only note their arguments, so that dispatch rules can be checked without
// a GPU and at sizes that no test would run. Device addresses are made up and never read.
//
// route_driver plane|voxels|fit|fit3 n0 n1 n2 nu nv nw precision method scheme in_flight
//              waves_per_cu height jobs
// prints "name value" lines.
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <vector>

#include "fq_internal.h"

namespace fq {

static int orders, traces, grad_form;
static TraceParams first_trace, last_trace;
static MapJob map_backward;

hipError_t launch_prep(const fq_field &, int, int, void *, float *, hipStream_t) { return hipSuccess; }
hipError_t launch_geometry(const fq_field &, double *const[3], Geo *, hipStream_t) { return hipSuccess; }
hipError_t launch_fill_u32(uint32_t *, int64_t, uint32_t, hipStream_t) { return hipSuccess; }
hipError_t launch_store_job(const TraceJob &, TraceJob *, hipStream_t) { return hipSuccess; }
hipError_t launch_trace(int, int, int, const TraceJob *, const TraceParams &tp, unsigned long long *, int, int,
                        hipStream_t)
{
    if (traces++ == 0) first_trace = tp;
    last_trace = tp;
    return hipSuccess;
}
hipError_t launch_bucket_order(int64_t, int32_t *, uint32_t *, int32_t *, hipStream_t) { return hipSuccess; }
hipError_t launch_tile_order(const TraceJob &, int, int, int32_t *, uint32_t *, int32_t *, hipStream_t)
{
    orders++;
    return hipSuccess;
}
hipError_t launch_voxel_order(const TraceJob &, int, int, int32_t *, uint32_t *, int32_t *, hipStream_t)
{
    orders++;
    return hipSuccess;
}
hipError_t launch_graze(const TraceJob *, int, int64_t, double, const double *, double, FixEntry *, uint32_t *,
                        uint32_t *, int64_t, int, int, hipStream_t)
{
    return hipSuccess;
}
hipError_t launch_fix_order(const TraceJob *, const FixEntry *, const uint32_t *, int64_t, int32_t *, uint32_t *,
                            FixEntry *, hipStream_t)
{
    return hipSuccess;
}
hipError_t launch_map_backward(const MapJob &m, const double *, const double *, const double *, const double *,
                               double *, double *, double *, int64_t, hipStream_t)
{
    map_backward = m;
    return hipSuccess;
}
hipError_t launch_rot_seed(const MapJob &, const RotEntry *, const uint32_t *, int64_t, const double *, double *,
                           hipStream_t)
{
    return hipSuccess;
}
hipError_t launch_bwd_order(const int32_t *, int64_t, int32_t *, uint32_t *, int32_t *, hipStream_t)
{
    return hipSuccess;
}
hipError_t launch_trace_backward(int, int, const TraceJob *, const BwdParams &, hipStream_t) { return hipSuccess; }
hipError_t launch_grad_planes(const fq_field &, const double *, int form, double *const[3], hipStream_t)
{
    grad_form = form;
    return hipSuccess;
}
hipError_t launch_classify(const MapJob &, int32_t *, RotEntry *, uint32_t *, int64_t, hipStream_t)
{
    return hipSuccess;
}
hipError_t launch_stencil(const MapJob &, hipStream_t) { return hipSuccess; }
hipError_t launch_m2_map(const MapJob &, hipStream_t) { return hipSuccess; }
hipError_t launch_rot_ranges(TraceJob *, int, int, int64_t, int64_t *, hipStream_t) { return hipSuccess; }
hipError_t launch_cyl_map(const MapJob &, hipStream_t) { return hipSuccess; }
hipError_t launch_perp_map(const MapJob &, int, hipStream_t) { return hipSuccess; }
hipError_t launch_lines_out(const MapJob &, const double *, hipStream_t) { return hipSuccess; }

}  // namespace fq

hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }

int main(int argc, char **argv)
{
    if (argc != 15) return 2;
    long long a[15];
    for (int i = 2; i < 13; i++) a[i] = atoll(argv[i]);
    const double height = atof(argv[13]);
    const int jobs = atoi(argv[14]);
    static double dev[16];
    fq_field f;
    memset(&f, 0, sizeof f);
    for (int q = 0; q < 3; q++) f.n[q] = a[2 + q], f.spacing[q] = 1.0 / (a[2] - 1), f.b[q] = dev;
    f.dtype = FQ_DT_F32;
    fq_plane pl;
    memset(&pl, 0, sizeof pl);
    pl.nu = a[5], pl.nv = a[6], pl.du = 0.9 / a[5], pl.dv = 0.9 / a[6];
    pl.u[0] = pl.v[1] = 1.0;
    pl.origin[2] = height;
    fq_voxels vx;
    memset(&vx, 0, sizeof vx);
    for (int q = 0; q < 3; q++) vx.n[q] = a[5 + q], vx.spacing[q] = 0.9 / a[5 + q];
    fq_params P;
    memset(&P, 0, sizeof P);
    P.want_tw = 1;
    P.precision = (int)a[8], P.method = (int)a[9], P.scheme = (int)a[10], P.in_flight = (int)a[11];
    P.waves_per_cu = (int)a[12];
    fq_map m;
    memset(&m, 0, sizeof m);
    m.q = m.tw = dev;
    m.status = (uint16_t *)dev;
    void *const ws = (void *)(uintptr_t)0x100000000ull;
    double *gb[3] = {dev, dev, dev};
    int rc;
    size_t need;
    if (!strcmp(argv[1], "voxels")) {
        need = fastqsl_q3d_workspace_size(&f, &vx, &P);
        rc = fastqsl_q3d(&f, &vx, &P, &m, ws, need, nullptr);
    } else if (!strcmp(argv[1], "fit")) {
        need = fastqsl_backward_workspace_size(&f, &pl, &P, 32);
        rc = fastqsl_backward(&f, &pl, &P, 32, dev, dev, nullptr, nullptr, gb, ws, need, nullptr);
    } else if (!strcmp(argv[1], "fit3")) {
        need = fastqsl_q3d_backward_workspace_size(&f, &vx, &P, 32);
        rc = fastqsl_q3d_backward(&f, &vx, &P, 32, dev, dev, nullptr, nullptr, gb, ws, need, nullptr);
    } else {
        std::vector<fq_field> fs(jobs, f);
        std::vector<fq_plane> ps(jobs, pl);
        std::vector<fq_map> ms(jobs, m);
        need = fastqsl_q2d_workspace_size(fs.data(), ps.data(), jobs, &P);
        rc = fastqsl_q2d(fs.data(), ps.data(), jobs, &P, ms.data(), ws, need, nullptr);
    }
    printf("rc %d\nneed %zu\ntraces %d\nfew %d\norders %d\n", rc, need, fq::traces, (int)fq::first_trace.few,
           fq::orders);
    printf("node_step %lld\nvalue_step %lld\ngrad_form %d\n", (long long)fq::map_backward.gstride,
           (long long)fq::map_backward.gplane, fq::grad_form);
    return rc == FQ_OK ? 0 : 1;
}
