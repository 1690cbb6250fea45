// a2, FP64 path: the all-pairs kernel k_pair64 and its launcher.
#include "dd_common.h"
#include "dd_pair64.h"

namespace dd {

// ------------------------------------------ a2: the all-pairs FP64 kernel --
// One workgroup = one work item: up to TILE target Gauss points (one per
// lane) against a contiguous source range.  Every lane of a wavefront works on
// the same source at the same time, so the source records are read with
// scalar loads into scalar registers (no LDS staging, no barriers) and enter
// the arithmetic as uniform operands.  Each lane accumulates sigma b_j / k2
// (3 values) over the range; the item's sums, scaled by k2, go to their own
// slot, reduced in a fixed order later.
//
// Sources come in runs that share nodes and the Burgers vector (loops stored
// in order): the inverse distance to a run's first node is computed once, then
// each source reuses the previous source's far-end value, and the cross
// products by the Burgers vector are taken once per run (pair_run_acc_f64).
// Only the part of the range that holds the wavefront's own segments tests for
// the excluded self pair.
//
// Bound by FP64 issue: 83 VALU instructions per source and wavefront (89 when
// every source forms rho x b), at 4.5 cycles each; 72 VGPRs.  A step of 16,384
// segments at 2 points 1.52 ms without the run form, 1.41 with it.  Measured and
// left out: two Gauss points of a segment per lane (t.b_j and t.g shared, 79
// instructions, 120 VGPRs), 0.3 % slower; six wavefronts per SIMD forced by launch
// bounds, 2 % slower.
// With few wavefronts per SIMD (up to a few thousand segments) the wait for a
// record's scalar load shows: the next record is therefore asked for before a
// source is evaluated, in a run and between runs.  Against records loaded when they
// are needed that takes 7 us off a step of 1,024 segments (28 us as it stands), 26 off
// one of 1,107 shuffled segments with close pairs exact (101), 7 off a step of 64
// volumes of 256 segments, 13 off one of 4,096 shuffled segments, and nothing off
// 16,384.  What is left there is the first wavefront's wait for each record to come
// into the L2: every lane asks for one of the range at once, 3 us off a step of
// 1,024 segments (with the wavefronts past a tile's end gone and the self test kept
// to a wavefront's own segments).
//
// Runs of fewer than RUN_MIN sources take the form that needs no set-up: the
// run form costs 15 instructions per run and saves 7 per source.
constexpr int RUN_MIN = 4;

// N consecutive words of a source's record, from the FIRST-th, in scalar registers.
template <int FIRST, int N>
struct RecWords {
    double v[N];
    __device__ __forceinline__ void load(const double *r)
    {
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = r[FIRST + i];
    }
    // What precedes this in the program is issued before these values are
    // waited for, loads that follow after it (scalar loads return in no order,
    // so a wait for one waits for all).
    __device__ __forceinline__ void arrived()
    {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < N; ++i) asm volatile("" : "+s"(v[i]) : : "memory");
    }
};

// What a run reads of a source: (x1, t, L) and c.
struct RunRec {
    RecWords<0, 7> p;
    RecWords<10, 3> c;
    __device__ __forceinline__ void load(const double *r)
    {
        p.load(r);
        c.load(r);
    }
    __device__ __forceinline__ void arrived()
    {
        p.arrived();
        c.arrived();
    }
};

template <bool SELF>
__device__ __forceinline__ void pair64_range(const double *__restrict__ ra, int64_t b, int64_t e,
                                             int64_t j, double xq0, double xq1, double xq2, double bj0,
                                             double bj1, double bj2, double kr, double nu, double ikr,
                                             double nukr, double &a0, double &a1, double &a2, double &ak)
{
    // Counted in 32 bits, so that the loop control stays on the scalar unit (a
    // volume of 2^31 segments does not fit the device's memory).
    const double *const c = ra + b * RECA;
    const int n = (int)(e - b), own = (int)(j - b);
    if (n <= 0) return;
    // A: the source to be evaluated; the next one asked for is never past the range's last
    RecWords<0, 14> A;
    A.load(c);
    double r1 = 0.0, r1c = 0.0;
    int left = 0;   // of the run being evaluated
    for (int k = 0; k < n;) {
        A.arrived();
        if (left == 0) {
            left = (int)min((int64_t)(n - k), (int64_t)__double_as_longlong(A.v[13]));
            const double R0 = xq0 - A.v[0], R1 = xq1 - A.v[1], R2 = xq2 - A.v[2];
            r1 = rsqrt64(fma(R2, R2, fma(R1, R1, fma(R0, R0, 1.0))));
            r1c = r1 * r1 * r1;
            if (!SELF && left >= RUN_MIN) {
                const double b0 = A.v[7], b1 = A.v[8], b2 = A.v[9];
                const double g0 = kr * fma(bj1, b2, -bj2 * b1), g1 = kr * fma(bj2, b0, -bj0 * b2),
                             g2 = kr * fma(bj0, b1, -bj1 * b0);
                double w0 = 0.0, w1 = 0.0, w2 = 0.0;
                // two sources per iteration: the second takes the first's far-end
                // values and leaves its own where the first's near-end values were,
                // so no register copy is made per source; while one is evaluated the
                // record of the next is on its way
                RunRec P, N;
#pragma unroll
                for (int i = 0; i < 7; ++i) P.p.v[i] = A.v[i];
#pragma unroll
                for (int i = 0; i < 3; ++i) P.c.v[i] = A.v[10 + i];
                do {
                    double r2, r2c;
                    P.arrived();
                    N.load(c + (k + 1) * (int64_t)RECA);
                    __builtin_amdgcn_sched_barrier(0);
                    pair_run_acc_f64(xq0, xq1, xq2, bj0, bj1, bj2, g0, g1, g2, P.p.v[0], P.p.v[1], P.p.v[2],
                                     P.p.v[3], P.p.v[4], P.p.v[5], P.p.v[6], P.c.v[0], P.c.v[1], P.c.v[2], ikr,
                                     nukr, r1, r1c, r2, r2c, a0, a1, a2, w0, w1, w2, ak);
                    N.arrived();
                    k += 2;
                    P.load(c + min(k, n - 1) * (int64_t)RECA);
                    __builtin_amdgcn_sched_barrier(0);
                    pair_run_acc_f64(xq0, xq1, xq2, bj0, bj1, bj2, g0, g1, g2, N.p.v[0], N.p.v[1], N.p.v[2],
                                     N.p.v[3], N.p.v[4], N.p.v[5], N.p.v[6], N.c.v[0], N.c.v[1], N.c.v[2], ikr,
                                     nukr, r2, r2c, r1, r1c, a0, a1, a2, w0, w1, w2, ak);
                    left -= 2;
                } while (left >= 2);
                A.load(c + min(k, n - 1) * (int64_t)RECA);
                a0 = fma(-kr, fma(w1, b2, -w2 * b1), a0);
                a1 = fma(-kr, fma(w2, b0, -w0 * b2), a1);
                a2 = fma(-kr, fma(w0, b1, -w1 * b0), a2);
                continue;
            }
        }
        double r2, r2c;
        RecWords<0, 14> B;
        B.load(c + min(k + 1, n - 1) * (int64_t)RECA);
        __builtin_amdgcn_sched_barrier(0);
        if (SELF) {
            double n0 = a0, n1 = a1, n2 = a2, nk = ak;
            pair_acc_f64(xq0, xq1, xq2, bj0, bj1, bj2, A.v[0], A.v[1], A.v[2], A.v[3], A.v[4], A.v[5], A.v[6],
                         A.v[7], A.v[8], A.v[9], A.v[10], A.v[11], A.v[12], kr, nu, r1, r1c, r2, r2c, n0, n1, n2,
                         nk);
            const bool self = k == own;
            a0 = self ? a0 : n0;
            a1 = self ? a1 : n1;
            a2 = self ? a2 : n2;
            ak = self ? ak : nk;
        } else {
            pair_acc_f64(xq0, xq1, xq2, bj0, bj1, bj2, A.v[0], A.v[1], A.v[2], A.v[3], A.v[4], A.v[5], A.v[6],
                         A.v[7], A.v[8], A.v[9], A.v[10], A.v[11], A.v[12], kr, nu, r1, r1c, r2, r2c, a0, a1, a2,
                         ak);
        }
        r1 = r2;
        r1c = r2c;
        B.arrived();
        A = B;
        ++k;
        --left;
    }
}

__global__ __launch_bounds__(TILE) void k_pair64(const Item *__restrict__ items,
                                                 const Tile *__restrict__ tiles,
                                                 const double *__restrict__ rec,
                                                 const double *__restrict__ ra, int64_t ns,
                                                 GaussRule g, double kr, double nu, double ikr, double nukr,
                                                 double k2,
                                                 double *__restrict__ partial)
{
    const Item it = items[blockIdx.x];
    const int lane = threadIdx.x;
    const int64_t b = it.src_begin, e = it.src_end;
    // a load per lane brings the first TILE records of the range into the L2 while
    // the rest is set up (the wavefronts read them one by one, and the first to
    // do so would wait for each)
    const double ahead = ra[min(b + lane, e - 1) * RECA];
    const Tile tl = tiles[it.tile];
    const int w0 = __builtin_amdgcn_readfirstlane(lane & ~63);   // the wavefront's first point
    if (w0 >= tl.n_points) return;   // none of them in the tile
    const bool valid = lane < tl.n_points;
    const int64_t p = tl.point_begin + (valid ? lane : 0);
    const int Q = g.n;
    const int64_t j = p / Q;
    const int q = (int)(p - j * Q);
    double sq = g.s[0];
    for (int k = 1; k < DD_MAX_GAUSS; ++k)
        if (k == q) sq = g.s[k];
    const double L = rec[6 * ns + j];
    const double xq0 = rec[0 * ns + j] + sq * L * rec[3 * ns + j];
    const double xq1 = rec[1 * ns + j] + sq * L * rec[4 * ns + j];
    const double xq2 = rec[2 * ns + j] + sq * L * rec[5 * ns + j];
    const double bj0 = rec[7 * ns + j], bj1 = rec[8 * ns + j], bj2 = rec[9 * ns + j];
    double a0 = 0.0, a1 = 0.0, a2 = 0.0, ak = 0.0;

    // the wavefront's own segments [jlo, jhi] split the range in three parts
    const int64_t jlo = (tl.point_begin + w0) / Q, jhi = (tl.point_begin + min(w0 + 63, (int)tl.n_points - 1)) / Q;
    const int64_t s0 = min(max(b, jlo), e), s1 = min(max(b, jhi + 1), e);
    pair64_range<false>(ra, b, s0, j, xq0, xq1, xq2, bj0, bj1, bj2, kr, nu, ikr, nukr, a0, a1, a2, ak);
    pair64_range<true>(ra, s0, s1, j, xq0, xq1, xq2, bj0, bj1, bj2, kr, nu, ikr, nukr, a0, a1, a2, ak);
    pair64_range<false>(ra, s1, e, j, xq0, xq1, xq2, bj0, bj1, bj2, kr, nu, ikr, nukr, a0, a1, a2, ak);
    asm volatile("" : : "v"(ahead));
    a0 = fma(ak, bj0, a0);   // the b_j terms of every source at once
    a1 = fma(ak, bj1, a1);
    a2 = fma(ak, bj2, a2);
    if (valid) {
        double *o = partial + it.slot * 3 * TILE;
        o[lane] = k2 * a0;
        o[TILE + lane] = k2 * a1;
        o[2 * TILE + lane] = k2 * a2;
    }
}

void launch_pair64(const Item *items, const Tile *tiles, const double *rec, int64_t ns, const GaussRule &g,
                   double k1, double k2, double *partial, int64_t n_items, hipStream_t st)
{
    const double kr = k1 / k2, nu = 1.0 - 2.0 * kr;
    hipLaunchKernelGGL(k_pair64, dim3((unsigned)n_items), dim3(TILE), 0, st, items, tiles, rec,
                       rec + (int64_t)REC64 * ns, ns, g, kr, nu, 1.0 / kr, nu / kr, k2, partial);
}

}  // namespace dd
