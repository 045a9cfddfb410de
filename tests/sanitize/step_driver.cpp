// The one-lane trial step (trace_core.h) on the host: half lines from random points of random
// cells, some of whose corners have no field. Where a trial leaves the lane's state as it
// was, the next one has to end the line as one that used up its trials.
// Prints: precision, lines that ran out of trials, those among them whose state stood still,
// trial steps computed, faults.
#include <float.h>
#include <math.h>
#include <stdio.h>

#include <random>

#include "trace_core.h"

using namespace fq;

template <typename T> static int run(const char *name)
{
    std::mt19937_64 rng(7);
    std::uniform_real_distribution<double> U(0.0, 1.0);
    std::normal_distribution<double> G;
    const uint32_t most = 5000;
    long out = 0, stood = 0, calls = 0, faults = 0;
    for (int line = 0; line < 20000; line++) {
        T f[3][8], cb[3][8], cj[3][8];
        const double w = U(rng);
        double bmax2 = 0.0;
        for (int q = 0; q < 8; q++) {
            const bool zero = U(rng) < w;
            double b2 = 0.0;
            for (int c = 0; c < 3; c++) f[c][q] = zero ? T(0) : (T)G(rng), b2 += (double)f[c][q] * f[c][q];
            bmax2 = fmax(bmax2, b2);
        }
        for (int c = 0; c < 3; c++) coeffs<T>(f[c], cb[c]), coeffs<T>(f[(c + 1) % 3], cj[c]);
        LaneConst<T> K{};
        K.rx = K.ry = K.rz = T(1);
        K.twk = T(0.1);
        K.bnull2 = (T)((double)Num<T>::null_rel * bmax2);
        K.nx = K.ny = K.nz = 3;
        K.max_steps = most;
        Lane<T> L{};
        L.p0 = (T)U(rng), L.p1 = (T)U(rng), L.p2 = (T)U(rng);
        L.h = T(0.5), L.tol = T(1e-6), L.sgn = T(line & 1 ? 1 : -1);
        L.force = -1;
        uint32_t trials = 0;
        for (bool still = false;;) {
            const Lane<T> b = L;
            int st = -1, face = -1;
            bool load = false;
            unsigned acc = 0;
            lane_iterate<T, true>(L, cb, cj, K, st, face, load, acc);
            calls++;
            trials += L.trials - b.trials;
            if (still && st != 4) faults++;
            if (st >= 0) {
                if (st == 4) out++, stood += still;
                if (st == 4 && trials != most + 1) faults++;
                break;
            }
            if (load) break;  // another cell
            still = acc == 0 && L.p0 == b.p0 && L.p1 == b.p1 && L.p2 == b.p2 && L.h == b.h && L.force == b.force &&
                    L.c0 == b.c0 && L.c1 == b.c1 && L.c2 == b.c2;
        }
    }
    printf("%s %ld %ld %ld %ld\n", name, out, stood, calls, faults);
    return 0;
}

int main() { return run<float>("f32") + run<double>("f64"); }
