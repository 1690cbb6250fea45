// a2, mixed FP32/FP64 path: the all-pairs kernel k_pair_mixed and its launcher.
#include "dd_common.h"
#include "dd_pair32.h"
#include "dd_pair64.h"

namespace dd {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// A value that is the same in every lane, into a scalar register.
__device__ __forceinline__ float uniform(float v)
{
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}

// The first N groups of four of a staged record (broadcast reads from LDS: the
// FP32 quadrature then runs on vector-register operands, which issue faster than
// FP32 instructions with a scalar operand).
template <int N>
struct Staged {
    float f[4 * N];
    __device__ __forceinline__ explicit Staged(const f32x4 *s)
    {
#pragma unroll
        for (int g = 0; g < N; ++g) {
            const f32x4 q = s[g];
#pragma unroll
            for (int i = 0; i < 4; ++i) f[4 * g + i] = q[i];
        }
    }
};

// True when every target point within the sphere (centre c, radius r, both
// FP32; cm = |c|_1) lies outside the band and outside the collinear cone of the
// source whose FP32 record is s, with a margin above the rounding of this test
// and of the per-point ones.  A ball lies outside a cone of half-angle al
// (tan al = 1/16) when its centre's distance from the cone surface, (16 rho -
// |y|) / sqrt(257), exceeds its radius.  False on NaN.
__device__ __forceinline__ bool quad_safe(const f32x4 *s, const float (&c)[3], float r, float cm)
{
    const Staged<R32_QUAD_VECS> v(s);
    const float m0 = v.f[R32_XH], m1 = v.f[R32_XH + 1], m2 = v.f[R32_XH + 2];
    const float e0 = c[0] - m0, e1 = c[1] - m1, e2 = c[2] - m2;
    const float y = fmaf(e2, v.f[R32_T + 2], fmaf(e1, v.f[R32_T + 1], e0 * v.f[R32_T]));
    const float ee = fmaf(e2, e2, fmaf(e1, e1, e0 * e0));
    const float d = sqrtf(ee), rho = sqrtf(fmaxf(fmaf(-y, y, ee), 0.f));
    const float rm = r + 1e-6f * (cm + fabsf(m0) + fabsf(m1) + fabsf(m2) + d);
    const float lim = d * 0.9999f - rm;
    return lim > 0.f && lim * lim >= v.f[R32_BAND] &&
           (16.0f * rho - fabsf(y)) * (0.99f / 16.03121954f) > rm + 0.002f * d;
}

template <int QN>
__device__ __forceinline__ void quad_acc(float e0, float e1, float e2, float ee, float ym, const float *s, float ra0,
                                         float tw2, float tb, float cb, float bj0, float bj1, float bj2, float kr,
                                         float nu, float three, float &f0, float &f1, float &f2, float &fk)
{
    if (QN == 2)
        quad2_acc_f32(e0, e1, e2, ee, ym, s, ra0, tw2, tb, cb, bj0, bj1, bj2, kr, nu, three, f0, f1, f2, fk);
    else
        quad3_acc_f32(e0, e1, e2, ee, ym, s, ra0, tw2, tb, cb, bj0, bj1, bj2, kr, nu, three, f0, f1, f2, fk);
}

// A target point and the constants of its pairs, in FP32.
struct MixedTarget {
    float xh0, xh1, xh2, xl0, xl1, xl2, fb0, fb1, fb2, fkr, fnu, three;
};

// A source that every target point of the wavefront takes by quadrature: the
// offsets and the rule, as k_pair_mixed forms them where it tests.
template <int QN>
__device__ __forceinline__ void safe_quad(const MixedTarget &T, const float *r, float ra0, float tw2, float tb,
                                          float cb, float &f0, float &f1, float &f2, float &fk)
{
    const float e0 = (T.xh0 - r[R32_XH]) + (T.xl0 - r[R32_XL]);
    const float e1 = (T.xh1 - r[R32_XH + 1]) + (T.xl1 - r[R32_XL + 1]);
    const float e2 = (T.xh2 - r[R32_XH + 2]) + (T.xl2 - r[R32_XL + 2]);
    const float ym = fmaf(e2, r[R32_T + 2], fmaf(e1, r[R32_T + 1], e0 * r[R32_T]));
    const float ee = fmaf(e2, e2, fmaf(e1, e1, e0 * e0));
    quad_acc<QN>(e0, e1, e2, ee, ym, r, ra0, tw2, tb, cb, T.fb0, T.fb1, T.fb2, T.fkr, T.fnu, T.three, f0, f1, f2, fk);
}

// Mixed precision.  As in the FP64 kernel, every lane of a wavefront works on
// the same source at the same time.  FP64 records are read with scalar loads.
// QN = the source-quadrature points of the variant (0: none, 2 or 3).  With
// QN > 0 the FP32 records are staged through LDS TILE sources at a time (the
// quadrature's FP32 instructions issue faster with every operand in a vector
// register) and each source is first located in FP32 relative to its midpoint
// (positions split into FP32 high and low parts, so the offset carries no
// rounding of the absolute coordinates): when, for every target point of the
// wavefront, the midpoint lies outside the source's band (max(30 L, cutoff +
// L/2) for 2 points, max(6 L, cutoff + L/2) for 3), the source is evaluated by
// FP32 quadrature.  With QN = 0 the FP32 records are read with scalar loads.
// Other pairs get their axial and perpendicular parts in FP32 from the same
// midpoint offset: those closer than the cutoff (minimum distance from the
// Gauss point to the closed source segment), and nearly collinear ones (the
// target within an angle of about 1/16 of the source's axis, seen from its
// midpoint), are evaluated in FP64 from the FP64 record, the rest by the
// cancellation-free FP32 closed form.  Nearly collinear pairs never take the
// quadrature either: in FP32 their perpendicular part rho carries an absolute
// error of order |ym| 6e-8, which is large against rho itself there, and for a
// screw source (b along t) the field on its axis consists of terms linear in
// rho alone.  FP32 contributions are summed in FP32 over TILE sources
// at a time, then added to FP64 sums; all sums are in units of k2 and scaled
// once at the end.
//
// SAFE, for long source ranges.  Bound by FP32 issue and by broadcast reads from
// LDS (five 16-byte reads a source).  Per 64 sources a wavefront first finds, one
// source per lane, those that all its target points take by quadrature (quad_safe,
// 96-98 % of them in sparse volumes in order): a run of these goes through an inner
// loop without tests or branches, the rest through the loop with the tests.  When
// its target points share their Burgers vector (a loop of 32 segments at 2 points
// is one wavefront), t.b_j and c.b_j belong to the source and are formed once, in
// the same pass, instead of by every lane.  Neither changes a bit of the result.
// VALU instructions a source in that loop, 2-point rule: 98 with the tests, 94, and
// 89 with a shared Burgers vector.  The inner loop stands inside the loop with the
// tests: as two loops or a called function the latter copies the four sums for
// every source (12-16 v_mov), 5-15 % of a volume whose segments come in no order,
// where next to no source is safe for a whole wavefront.  After two groups of 64 in
// a row with fewer than 8 safe sources only the first group of a stage is looked at,
// until one has more: shuffled segments 1 % less.  Against the loop with the tests
// alone: 16,384 segments at 4 points 1.96 -> 1.84 ms, 65,536 at 2 points 15.1 -> 14.0
// ms; 16,384 and 65,536 shuffled segments at 2 points 1.25 -> 1.28 and 17.8 -> 17.9
// ms.  Five wavefronts per SIMD (92 VGPRs, no scratch).  Left out: the index of the next
// safe source in place of the mask (the copies come back, 14-19 % of shuffled segments).
template <int QN, bool SAFE>
__global__ __launch_bounds__(TILE, SAFE ? 5 : 1) void k_pair_mixed(
    const Item *__restrict__ items, const Tile *__restrict__ tiles, const double *__restrict__ rec,
    const double *__restrict__ ra, const float *__restrict__ rf, int64_t ns, GaussRule g, double kr, double nu,
    double k2, float cut, double *__restrict__ partial, unsigned long long *near_count)
{
    __shared__ f32x4 shr[QN ? TILE : 1][REC32A / 4];   // FP32 records of one stage of sources
    __shared__ f32x4 bsh[SAFE ? TILE : 1];             // per wavefront, of 64 sources: t.b_j, c.b_j, 1 + hq^2, 2 hq
    __shared__ unsigned n_near_block, n_quad_block;
    const Item it = items[blockIdx.x];
    const Tile tl = tiles[it.tile];
    const int lane = threadIdx.x;
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
    const float xh0 = (float)xq0, xh1 = (float)xq1, xh2 = (float)xq2;
    const float xl0 = (float)(xq0 - (double)xh0), xl1 = (float)(xq1 - (double)xh1),
                xl2 = (float)(xq2 - (double)xh2);
    const double bj0 = rec[7 * ns + j], bj1 = rec[8 * ns + j], bj2 = rec[9 * ns + j];
    const float fb0 = (float)bj0, fb1 = (float)bj1, fb2 = (float)bj2;
    const float fkr = (float)kr, fnu = (float)nu, cut2 = cut * cut;
    // constants of the FP32 arithmetic in vector registers (the empty asm keeps
    // them there): an FP32 instruction with a literal operand issues at half rate
    // kap = K^2 / (1 + K^2): the collinear test ym^2 (1 + K^2) <= K^2 (ee + 1)
    // as ym^2 <= kap (ee + 1), one instruction fewer
    float three = 3.0f, ck2 = COLLINEAR_K2, kap = COLLINEAR_K2 / (1.0f + COLLINEAR_K2);
    asm volatile("" : "+v"(three), "+v"(ck2), "+v"(kap));
    double a0 = 0.0, a1 = 0.0, a2 = 0.0;
    unsigned n_near = 0, n_quad_src = 0;
    if (lane == 0) {
        n_near_block = 0;
        n_quad_block = 0;
    }
    // a sphere around the wavefront's target points; do they share a Burgers vector?
    float sc[3] = {}, sr = 0.f, sm = 0.f;
    bool same_b = false;
    if (SAFE) {
        float lo[3] = {xh0, xh1, xh2}, hi[3] = {xh0, xh1, xh2};
#pragma unroll
        for (int off = 32; off > 0; off >>= 1)
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                lo[k] = fminf(lo[k], __shfl_xor(lo[k], off));
                hi[k] = fmaxf(hi[k], __shfl_xor(hi[k], off));
            }
#pragma unroll
        for (int k = 0; k < 3; ++k) sc[k] = uniform(0.5f * lo[k] + 0.5f * hi[k]);
        const float d0 = xh0 - sc[0], d1 = xh1 - sc[1], d2 = xh2 - sc[2];
        sr = fmaf(d2, d2, fmaf(d1, d1, d0 * d0));
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) sr = fmaxf(sr, __shfl_xor(sr, off));
        sr = uniform(sqrtf(sr));
        sm = fabsf(sc[0]) + fabsf(sc[1]) + fabsf(sc[2]);
        same_b =
            __builtin_amdgcn_ballot_w64(fb0 == uniform(fb0) && fb1 == uniform(fb1) && fb2 == uniform(fb2)) == ~0ull;
    }
    int misses = 0;   // groups of 64 sources in a row with next to none of them safe
    const MixedTarget T{xh0, xh1, xh2, xl0, xl1, xl2, fb0, fb1, fb2, fkr, fnu, three};
    __syncthreads();   // the counters are cleared before any wavefront adds to them

    for (int64_t base = it.src_begin; base < it.src_end; base += TILE) {
        const int n = (int)min(it.src_end - base, (int64_t)TILE);
        // the target's own segment as a source index of this stage (-1: not in it)
        const int self = j >= base && j < base + n ? (int)(j - base) : -1;
        float f0 = 0.f, f1 = 0.f, f2 = 0.f, fk = 0.f;
        if (QN) {
            __syncthreads();
            if (lane < n) {
                const f32x4 *g4 = reinterpret_cast<const f32x4 *>(rf + (base + lane) * REC32A);
#pragma unroll
                for (int f = 0; f < REC32A / 4; ++f) shr[lane][f] = g4[f];
            }
            __syncthreads();
        }
        const float *s = rf + base * REC32A;
        for (int k64 = 0; k64 < n; k64 += SAFE ? 64 : TILE) {
            const int kgrp = SAFE ? min(n, k64 + 64) : n;
            uint64_t safe = 0;
            if (SAFE && (misses < 2 || k64 == 0)) {
                // 64 sources at a time: those that every target point of the wavefront
                // takes by quadrature, tested one per lane
                const int ks = k64 + (lane & 63);
                bool ok = false;
                if (ks < n) {
                    ok = quad_safe(shr[ks], sc, sr, sm);
                    if (same_b) {
                        const Staged<R32_QUAD_VECS> q5(shr[ks]);
                        bsh[lane] = f32x4{record_tb(q5.f, fb0, fb1, fb2), record_cb(q5.f, fb0, fb1, fb2),
                                          q5.f[R32_RA0], q5.f[R32_TW]};
                    }
                }
                __builtin_amdgcn_wave_barrier();
                safe = __builtin_amdgcn_ballot_w64(ok);
                __builtin_amdgcn_wave_barrier();
                misses = __builtin_popcountll(safe) < 8 ? misses + 1 : 0;
            }
            for (int k = k64; k < kgrp; ++k, s += REC32A) {
                if (SAFE) {
                    if (safe & 1) {
                        const int run = ~safe ? __builtin_ctzll(~safe) : 64;
                        const int kend = k + run;
                        n_quad_src += (unsigned)run;
                        s += (run - 1) * REC32A;
                        safe = run < 64 ? safe >> run : 0;
                        if (same_b) {
                            const f32x4 *bw = bsh + (lane & ~63) + (k & 63);
                            for (; k < kend; ++k, ++bw) {
                                const Staged<4> q(shr[k]);
                                const f32x4 w = *bw;
                                safe_quad<QN ? QN : 2>(T, q.f, w[2], w[3], w[0], w[1], f0, f1, f2, fk);
                            }
                        } else {
                            for (; k < kend; ++k) {
                                const Staged<R32_QUAD_VECS> q(shr[k]);
                                safe_quad<QN ? QN : 2>(T, q.f, q.f[R32_RA0], q.f[R32_TW], record_tb(q.f, fb0, fb1, fb2),
                                                       record_cb(q.f, fb0, fb1, fb2), f0, f1, f2, fk);
                            }
                        }
                        --k;
                        continue;
                    }
                    safe >>= 1;
                }
                float r[REC32A];
                if (QN) {
                    // from LDS (broadcast reads): the FP32 quadrature then runs on
                    // vector-register operands, which issue faster than FP32
                    // instructions with a scalar operand; the fields only the
                    // other pairs use are read below, for those
    #pragma unroll
                    for (int f = 0; f < R32_QUAD_VECS; ++f) {
                        const f32x4 v = shr[k][f];
                        r[4 * f] = v[0];
                        r[4 * f + 1] = v[1];
                        r[4 * f + 2] = v[2];
                        r[4 * f + 3] = v[3];
                    }
                } else {
                    // straight from memory into scalar registers (two loads, one wait)
                    const f32x16 va = *reinterpret_cast<const f32x16 *>(s);
                    const f32x8 vb = *reinterpret_cast<const f32x8 *>(s + 16);
    #pragma unroll
                    for (int f = 0; f < 16; ++f) r[f] = va[f];
    #pragma unroll
                    for (int f = 0; f < 8; ++f) r[16 + f] = vb[f];
                }
                // offset from the source midpoint, from the split FP32 positions:
                // accurate to the rounding of its own size
                const float e0 = (xh0 - r[R32_XH]) + (xl0 - r[R32_XL]);
                const float e1 = (xh1 - r[R32_XH + 1]) + (xl1 - r[R32_XL + 1]);
                const float e2 = (xh2 - r[R32_XH + 2]) + (xl2 - r[R32_XL + 2]);
                // axial coordinate from the midpoint
                const float ym = fmaf(e2, r[R32_T + 2], fmaf(e1, r[R32_T + 1], e0 * r[R32_T]));
                const float ym2 = ym * ym;
                if (QN) {
                    const float ee = fmaf(e2, e2, fmaf(e1, e1, e0 * e0));
                    // outside the band and not nearly collinear (ym^2 > K^2 (rho^2 + 1)
                    // with rho^2 = ee - ym^2, see COLLINEAR_K2)
                    // every active lane passes both tests: the two comparison masks
                    // against exec, in scalar registers (a ballot of their
                    // conjunction would select and re-compare per lane)
                    const uint64_t quad = __builtin_amdgcn_ballot_w64(ee >= r[R32_BAND]) &
                                          __builtin_amdgcn_ballot_w64(ym2 <= fmaf(kap, ee, kap));
                    if (quad == __builtin_amdgcn_read_exec()) {
                        ++n_quad_src;
                        quad_acc<QN>(e0, e1, e2, ee, ym, r, r[R32_RA0], r[R32_TW], record_tb(r, fb0, fb1, fb2),
                                     record_cb(r, fb0, fb1, fb2), fb0, fb1, fb2, fkr, fnu, three, f0, f1, f2, fk);
                        continue;
                    }
                }
                if (QN) {
    #pragma unroll
                    for (int f = R32_QUAD_VECS; f < REC32A / 4; ++f) {
                        const f32x4 v = shr[k][f];
                        r[4 * f] = v[0];
                        r[4 * f + 1] = v[1];
                        r[4 * f + 2] = v[2];
                        r[4 * f + 3] = v[3];
                    }
                }
                // axial coordinate from the first node and perpendicular part
                const float Ls = r[R32_L];
                const float y = fmaf(0.5f, Ls, ym);
                const float h0 = fmaf(-ym, r[R32_T], e0), h1 = fmaf(-ym, r[R32_T + 1], e1),
                            h2 = fmaf(-ym, r[R32_T + 2], e2);
                const float hh = fmaf(h2, h2, fmaf(h1, h1, h0 * h0));
                const float ya = y - __builtin_amdgcn_fmed3f(y, 0.f, Ls);   // y clamped to [0, L]: one instruction
                // FP64: near pairs, and nearly collinear ones (rho carries an absolute
                // error of order |ym| eps32 in FP32)
                if (hh + ya * ya < cut2 || ym2 > fmaf(ck2, hh, ck2)) {
                    // k through an empty asm: the comparison stays in this branch
                    // instead of becoming a per-lane counter stepped every source
                    int ks = k;
                    asm volatile("" : "+s"(ks));
                    if (ks != self) {
                        n_near += valid ? 1u : 0u;
                        pair_acc_isolated_f64(xq0, xq1, xq2, bj0, bj1, bj2, ra + (base + k) * RECA, kr, nu, a0, a1, a2);
                    }
                } else {
                    // the record's b and c carry the quadrature weight (1 without a quadrature)
                    pair_acc_f32(y, h0, h1, h2, hh, fb0, fb1, fb2, r[R32_T], r[R32_T + 1], r[R32_T + 2], Ls, r[R32_B],
                                 r[R32_B + 1], r[R32_B + 2], r[R32_C], r[R32_C + 1], r[R32_C + 2],
                                 QN ? r[R32_IW] : 1.0f, fkr, fnu, f0, f1, f2, fk);
                }
            }
        }
        a0 += (double)fmaf(fk, fb0, f0);   // the b_j terms of the stage at once
        a1 += (double)fmaf(fk, fb1, f1);
        a2 += (double)fmaf(fk, fb2, f2);
    }
    if (valid) {
        double *o = partial + it.slot * 3 * TILE;
        o[lane] = k2 * a0;
        o[TILE + lane] = k2 * a1;
        o[2 * TILE + lane] = k2 * a2;
    }
    const unsigned n_quad = valid ? n_quad_src : 0u;
    if (n_near) atomicAdd(&n_near_block, n_near);
    if (n_quad) atomicAdd(&n_quad_block, n_quad);
    __syncthreads();
    if (lane == 0 && n_near_block) atomicAdd(near_count, (unsigned long long)n_near_block);
    if (lane == 0 && n_quad_block) atomicAdd(near_count + 1, (unsigned long long)n_quad_block);
}

// Source ranges from which the SAFE form is used: its set-up costs a wavefront
// the sphere around its targets and a test per 64 sources.  Ranges of 64 and 128
// sources (5,000 segments and fewer) lose up to 10 % with it, 256 about as much
// as they gain; 1,024 and 2,048 gain 6-8 % in order at 2 and 4 points.  With one
// Gauss point a wavefront holds two loops of 32, which lie apart and share no
// Burgers vector: 16,384 segments at ranges of 512 and 1,024 641 and 650 us, with the
// SAFE form 652 and 671, shuffled 734 and 755.
constexpr int64_t SAFE_MIN_RANGE = 512;
constexpr int SAFE_MIN_GAUSS = 2;

template <int QN>
static void launch_mixed(const Item *items, const Tile *tiles, const double *rec, const float *rec32, int64_t ns,
                         const GaussRule &g, double kr, double nu, double k2, float cut, double *partial,
                         unsigned long long *counters, int64_t n_items, int64_t range, hipStream_t st)
{
    const double *ra = rec + (int64_t)REC64 * ns;
    if (QN && range >= SAFE_MIN_RANGE && g.n >= SAFE_MIN_GAUSS)
        hipLaunchKernelGGL((k_pair_mixed<QN ? QN : 2, true>), dim3((unsigned)n_items), dim3(TILE), 0, st, items,
                           tiles, rec, ra, rec32, ns, g, kr, nu, k2, cut, partial, counters);
    else
        hipLaunchKernelGGL((k_pair_mixed<QN, false>), dim3((unsigned)n_items), dim3(TILE), 0, st, items, tiles, rec,
                           ra, rec32, ns, g, kr, nu, k2, cut, partial, counters);
}

void launch_pair_mixed(const Item *items, const Tile *tiles, const double *rec, const float *rec32, int64_t ns,
                       const GaussRule &g, double k1, double k2, float cut, double *partial,
                       unsigned long long *counters, int64_t n_items, int64_t range, int variant, hipStream_t st)
{
    const double kr = k1 / k2, nu = 1.0 - 2.0 * kr;
    const int qn = quad_points(variant);
    if (qn == 2)
        launch_mixed<2>(items, tiles, rec, rec32, ns, g, kr, nu, k2, cut, partial, counters, n_items, range, st);
    else if (qn == 3)
        launch_mixed<3>(items, tiles, rec, rec32, ns, g, kr, nu, k2, cut, partial, counters, n_items, range, st);
    else
        launch_mixed<0>(items, tiles, rec, rec32, ns, g, kr, nu, k2, cut, partial, counters, n_items, range, st);
}

}  // namespace dd
