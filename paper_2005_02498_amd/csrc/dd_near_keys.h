// Keys and bounding spheres of the exact band's search, made by a launch of
// their own or, for a single volume, in the one that makes its segment records.
#pragma once

#include <hip/hip_runtime.h>

#include "dd_common.h"

namespace dd {

namespace {

__device__ __forceinline__ int64_t inst_of(const NearArgs &A, int64_t s)
{
    return A.seg_inst ? A.seg_inst[s] : 0;
}

// x1 + x2 and |x2 - x1|^2 of segment s in the caller's units, written out
// without contraction (the near decision must match the oracle's bit for bit).
__device__ __forceinline__ void near_key(const double *xa, const double *xb, double *k)
{
#pragma clang fp contract(off)
    const double d0 = xb[0] - xa[0], d1 = xb[1] - xa[1], d2 = xb[2] - xa[2];
    k[0] = xa[0] + xb[0];
    k[1] = xa[1] + xb[1];
    k[2] = xa[2] + xb[2];
    k[3] = d0 * d0 + d1 * d1 + d2 * d2;
}

// One thread per segment s, consecutive over the wavefront's lanes: its key; the
// NEAR_GROUP lanes of a group (the last one may be partial) then form the group's
// sphere (centre C = key of its first segment, radius R = max |S_i - C| +
// sqrt(c2 |D_i|^2)), which holds S_j of every segment j that can be near one of
// them, since near(i, j) implies |S_i - S_j| < sqrt(c2 |D_i|^2) + sqrt(c2 |D_j|^2).
// The sphere is stored in FP32 with R widened by 4e-6 (|C|_1 + R), more than the
// rounding of the FP32 test can take away.
__device__ __forceinline__ void near_keys(const NearArgs &A, int64_t s)
{
    const int lane = threadIdx.x & 63, first = lane & ~(NEAR_GROUP - 1);
    if (s - (lane - first) >= A.ns) return;   // whole group past the end
    const bool live = s < A.ns;
    double k[4] = {0, 0, 0, 0};
    if (live) {
        const int64_t inst = inst_of(A, s);
        const int64_t n0 = A.node_off ? A.node_off[inst] : 0;
        const int64_t nn = A.node_off ? A.node_off[inst + 1] - n0 : A.nn;
        int64_t i1 = A.seg_nodes[s], i2 = A.seg_nodes[A.ns + s];
        // out-of-range indices are reported by the segment preparation; stay in bounds here
        if (i1 < 0 || i1 >= nn || i2 < 0 || i2 >= nn) i1 = i2 = 0;
        const double xa[3] = {A.x[n0 + i1], A.x[A.nn + n0 + i1], A.x[2 * A.nn + n0 + i1]};
        const double xb[3] = {A.x[n0 + i2], A.x[A.nn + n0 + i2], A.x[2 * A.nn + n0 + i2]};
        near_key(xa, xb, k);
        double *o = A.key + 4 * s;
        o[0] = k[0]; o[1] = k[1]; o[2] = k[2]; o[3] = k[3];
    }
    const double c0 = __shfl(k[0], first, 64), c1 = __shfl(k[1], first, 64), c2 = __shfl(k[2], first, 64);
    double r = 0.0;
    if (live) {
        const double e0 = k[0] - c0, e1 = k[1] - c1, e2 = k[2] - c2;
        r = sqrt(e0 * e0 + e1 * e1 + e2 * e2) + sqrt(A.c2 * k[3]);
    }
    for (int o = 1; o < NEAR_GROUP; o <<= 1) r = fmax(r, __shfl_xor(r, o, 64));
    if (lane == first) {
        r += 4e-6 * (fabs(c0) + fabs(c1) + fabs(c2) + r);
        A.sph[s / NEAR_GROUP] = make_float4((float)c0, (float)c1, (float)c2, (float)r);
    }
}

}  // namespace

}  // namespace dd
