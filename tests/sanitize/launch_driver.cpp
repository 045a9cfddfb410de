// What the launchers (host code of trace.hip, trace_quad.hip and prep.hip) start for given
// arguments: linked with stand-ins for the HIP runtime that note each launch, so that
// launch shapes and kernel choice can be checked without a GPU. A CU holds 2048 threads here.
//
// launch_driver trace precision store twm list list_rev few cyl scheme method jobs tape block waves
// launch_driver prep n0 n1 n2 dtype precision want_tw
// prints "status <error>" and a line "<grid> <block> <kernel>" per launch.
#include <cxxabi.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <map>
#include <string>

#include "fq_internal.h"

static std::map<const void *, std::string> &names()
{
    static std::map<const void *, std::string> m;
    return m;
}
static dim3 g_grid, g_block;

extern "C" {
void **__hipRegisterFatBinary(const void *) { return nullptr; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *,
                           int *)
{
    names()[host] = name;
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t, hipStream_t)
{
    g_grid = grid, g_block = block;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *shmem, hipStream_t *s)
{
    *grid = g_grid, *block = g_block, *shmem = 0, *s = nullptr;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *fn, dim3 grid, dim3 block, void **, size_t, hipStream_t)
{
    int st = 0;
    const std::string &name = names()[fn];
    char *d = abi::__cxa_demangle(name.c_str(), nullptr, nullptr, &st);
    printf("%llu %u %s\n", (unsigned long long)grid.x * grid.y * grid.z, block.x, st == 0 ? d : name.c_str());
    free(d);
    return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int block, size_t)
{
    *n = 2048 / block;
    return hipSuccess;
}
hipError_t hipGetDevice(int *d)
{
    *d = 0;
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int)
{
    *v = 256;
    return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
}

int main(int argc, char **argv)
{
    long long a[16] = {0};
    for (int i = 2; i < argc && i < 16; i++) a[i] = atoll(argv[i]);
    static double dev[16];
    hipError_t e = hipErrorInvalidValue;
    if (argc == 15 && !strcmp(argv[1], "trace")) {
        fq::TraceParams tp;
        memset(&tp, 0, sizeof tp);
        static fq::FixEntry list;
        static fq::Ckpt tape;
        static uint32_t count;
        if (a[5]) tp.list = &list, tp.list_count = &count;
        tp.list_rev = (int)a[6], tp.few = (int)a[7], tp.cyl = (int)a[8];
        tp.scheme = (int)a[9], tp.method = (int)a[10], tp.njobs = (int)a[11];
        if (a[12]) tp.tape = &tape, tp.seg = 32;
        e = fq::launch_trace((int)a[2], (int)a[3], (int)a[4], nullptr, tp, nullptr, (int)a[13], (int)a[14], nullptr);
    } else if (argc == 8) {
        fq_field f;
        memset(&f, 0, sizeof f);
        for (int q = 0; q < 3; q++) f.n[q] = a[2 + q], f.spacing[q] = 1.0, f.b[q] = dev;
        f.dtype = (int)a[5];
        e = fq::launch_prep(f, (int)a[6], (int)a[7], dev, (float *)dev, nullptr);
    }
    printf("status %d\n", (int)e);
    return 0;
}
