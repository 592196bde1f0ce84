// Phase-table entries and rotation parameters of a set of angles: FP64
// products, sine and cosine, rounded to FP32.
#pragma once

#include "common.h"

namespace pq {

__device__ inline void cpow_d(double re, double im, int e, double& ore, double& oim)
{
    double r = 1.0, i = 0.0;
    for (int k = 0; k < e; ++k) {
        const double nr = r * re - i * im, ni = r * im + i * re;
        r = nr;
        i = ni;
    }
    ore = r;
    oim = i;
}

// e^{-i gamma c}
__device__ inline float2 lut_entry(int c, double gm)
{
    double sv, cv;
    sincos(gm * (double)c, &sv, &cv);
    return make_float2((float)cv, (float)(-sv));
}

// rotation parameters of one layer
__device__ inline RxCoef rx_coef(const SubDesc* sd, double bt)
{
    double s, c;
    sincos(bt, &s, &c);
    RxCoef rc;
    // e^{-i beta X} = c (I - i tan(beta) X)            when |cos| >= |sin|
    //               = -i s X (I + i cot(beta) X)       otherwise
    // i.e. f (I - i t X) X^flip with (f, t) = (c, tan) or (-i s, -cot)
    const bool tanm = fabs(c) >= fabs(s);
    rc.mode = tanm ? 0 : 1;
    rc.t = (float)(tanm ? s / c : -c / s);
    double f = tanm ? c : s;
    // On wide tiles the factor is that of the rounded t, which makes f (I - i t X)
    // unitary: the rounding of t otherwise changes the state's norm by as much for
    // every qubit. (The other tiles keep f, and with it their bits; see wide_allowed.)
    if (sd->wide) f = copysign(1.0 / sqrt(1.0 + (double)rc.t * rc.t), f);
    rc.fsq = (float)(f * f);
    // per-qubit factors: forward c or -i s, inverse c or +i s
    const double fr = tanm ? f : 0.0, fi_f = tanm ? 0.0 : -f, fi_i = tanm ? 0.0 : f;
    for (int g = 0; g < MAX_GROUPS; ++g) {
        const int nq = g < sd->ngroups ? sd->gsize[g] : 0;
        double r, i;
        cpow_d(fr, fi_f, nq, r, i);
        rc.Ff[g] = make_float2((float)r, (float)i);
        cpow_d(fr, fi_i, nq, r, i);
        rc.Fi[g] = make_float2((float)r, (float)i);
    }
    return rc;
}

}  // namespace pq
