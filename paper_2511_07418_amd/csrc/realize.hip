// Kinematics optimisation (Sec. 5.5, Eq. 7-8, Phase I and II) and the
// penetration part of the validity criterion (Sec. 3.2), in two kernels: the
// damped steps need every register (two waves per SIMD), the penetration test is
// bound by the SDF's scattered reads and wants as many waves as fit; in one kernel
// its reads waited at two waves per SIMD (470,724 accepted sets of 22 joints: 1.7
// of 3.1 ms).
//
// Lane layout of both: F lanes per accepted set, lane f realises finger f, so a
// wave covers 64 / F sets (the 64 mod F lanes left over idle) and the set-level
// reductions (max depth) read the set's lanes with shuffles.
// Everything per lane of the steps lives in registers; that kernel is templated
// on the largest finger DOF so the small dense solves unroll.
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "lg_internal.h"

namespace lg {

constexpr int kRealizeThreads = 256;

constexpr uint32_t kPurposeUnused = 15u;

// distance between segments [p1, q1] and [p2, q2]: the closest parameters
// (s, t) in [0,1]^2 in closed form (Ericson, Real-Time Collision Detection,
// Sec. 5.1.9)
__device__ inline float segment_distance(const float *p1, const float *q1, const float *p2, const float *q2)
{
    const float d1x = q1[0] - p1[0], d1y = q1[1] - p1[1], d1z = q1[2] - p1[2];
    const float d2x = q2[0] - p2[0], d2y = q2[1] - p2[1], d2z = q2[2] - p2[2];
    const float rx = p1[0] - p2[0], ry = p1[1] - p2[1], rz = p1[2] - p2[2];
    const float a = d1x * d1x + d1y * d1y + d1z * d1z, e = d2x * d2x + d2y * d2y + d2z * d2z;
    const float f = d2x * rx + d2y * ry + d2z * rz;
    float s, t;
    if (a <= 1e-20f && e <= 1e-20f) {
        s = t = 0.0f;
    } else if (a <= 1e-20f) {
        s = 0.0f;
        t = fminf(fmaxf(f / e, 0.0f), 1.0f);
    } else {
        const float c = d1x * rx + d1y * ry + d1z * rz;
        if (e <= 1e-20f) {
            t = 0.0f;
            s = fminf(fmaxf(-c / a, 0.0f), 1.0f);
        } else {
            const float b = d1x * d2x + d1y * d2y + d1z * d2z, den = a * e - b * b;
            s = den > 0.0f ? fminf(fmaxf((b * f - c * e) / den, 0.0f), 1.0f) : 0.0f;
            t = (b * s + f) / e;
            if (t < 0.0f) {
                t = 0.0f;
                s = fminf(fmaxf(-c / a, 0.0f), 1.0f);
            } else if (t > 1.0f) {
                t = 1.0f;
                s = fminf(fmaxf((b - c) / a, 0.0f), 1.0f);
            }
        }
    }
    const float x = rx + s * d1x - t * d2x, y = ry + s * d1y - t * d2y, z = rz + s * d1z - t * d2z;
    return sqrtf(x * x + y * y + z * z);
}

__device__ inline float dot3f(float ax, float ay, float az, float bx, float by, float bz)
{
    return fmaf(ax, bx, fmaf(ay, by, az * bz));
}

// unit vector of (x, y, z); a direction perpendicular to the axis if tiny
__device__ inline void unit_or_perp(float &x, float &y, float &z, float ax, float ay, float az)
{
    const float n2 = dot3f(x, y, z, x, y, z);
    if (n2 > 1e-30f) {
        const float r = 1.0f / sqrtf(n2);
        x *= r;
        y *= r;
        z *= r;
    } else {
        // Duff et al. basis, first tangent of the axis
        const float sign = copysignf(1.0f, az);
        const float a = -1.0f / (sign + az);
        x = 1.0f + sign * ax * ax * a;
        y = sign * ax * ay * a;
        z = -sign * ax;
    }
}

// Capsule point closest to (p, n) in |x - p|^2 + beta^2 |nt - n|^2.
__device__ inline void capsule_aligned(const float *A, const float *Bp, float r, const float *p, const float *n,
                                       float beta, float *pt, float *nt)
{
    float ab[3] = {Bp[0] - A[0], Bp[1] - A[1], Bp[2] - A[2]};
    const float L = sqrtf(dot3f(ab[0], ab[1], ab[2], ab[0], ab[1], ab[2]));
    float ax = 0.f, ay = 0.f, az = 1.f;
    if (L > 0.f) {
        ax = ab[0] / L;
        ay = ab[1] / L;
        az = ab[2] / L;
    }
    const float b2 = beta * beta;
    float best;
    {  // cylinder
        float s = dot3f(p[0] - A[0], p[1] - A[1], p[2] - A[2], ax, ay, az);
        s = fminf(fmaxf(s, 0.f), L);
        const float cx = fmaf(s, ax, A[0]), cy = fmaf(s, ay, A[1]), cz = fmaf(s, az, A[2]);
        float vx = fmaf(r, p[0] - cx, b2 * n[0]), vy = fmaf(r, p[1] - cy, b2 * n[1]), vz = fmaf(r, p[2] - cz, b2 * n[2]);
        const float va = dot3f(vx, vy, vz, ax, ay, az);
        vx = fmaf(-va, ax, vx);
        vy = fmaf(-va, ay, vy);
        vz = fmaf(-va, az, vz);
        unit_or_perp(vx, vy, vz, ax, ay, az);
        pt[0] = fmaf(r, vx, cx);
        pt[1] = fmaf(r, vy, cy);
        pt[2] = fmaf(r, vz, cz);
        nt[0] = vx;
        nt[1] = vy;
        nt[2] = vz;
        const float d0 = pt[0] - p[0], d1 = pt[1] - p[1], d2 = pt[2] - p[2];
        const float e0 = vx - n[0], e1 = vy - n[1], e2 = vz - n[2];
        best = dot3f(d0, d1, d2, d0, d1, d2) + b2 * dot3f(e0, e1, e2, e0, e1, e2);
    }
#pragma unroll
    for (int cap = 0; cap < 2; ++cap) {
        const float *c = cap == 0 ? Bp : A;
        const float sg = cap == 0 ? 1.0f : -1.0f;
        float vx = fmaf(r, p[0] - c[0], b2 * n[0]), vy = fmaf(r, p[1] - c[1], b2 * n[1]),
              vz = fmaf(r, p[2] - c[2], b2 * n[2]);
        const float n2 = dot3f(vx, vy, vz, vx, vy, vz);
        if (!(n2 > 1e-30f)) continue;
        const float rn = 1.0f / sqrtf(n2);
        vx *= rn;
        vy *= rn;
        vz *= rn;
        if (sg * dot3f(vx, vy, vz, ax, ay, az) < 0.f) continue;
        const float x0 = fmaf(r, vx, c[0]), x1 = fmaf(r, vy, c[1]), x2 = fmaf(r, vz, c[2]);
        const float d0 = x0 - p[0], d1 = x1 - p[1], d2 = x2 - p[2];
        const float e0 = vx - n[0], e1 = vy - n[1], e2 = vz - n[2];
        const float cost = dot3f(d0, d1, d2, d0, d1, d2) + b2 * dot3f(e0, e1, e2, e0, e1, e2);
        if (cost < best) {
            best = cost;
            pt[0] = x0;
            pt[1] = x1;
            pt[2] = x2;
            nt[0] = vx;
            nt[1] = vy;
            nt[2] = vz;
        }
    }
}

// Plain projection of p onto the capsule surface.
__device__ inline void capsule_project(const float *A, const float *Bp, float r, const float *p, float *pt, float *nt)
{
    const float ab0 = Bp[0] - A[0], ab1 = Bp[1] - A[1], ab2 = Bp[2] - A[2];
    const float L2 = dot3f(ab0, ab1, ab2, ab0, ab1, ab2);
    float t = L2 > 0.f ? dot3f(p[0] - A[0], p[1] - A[1], p[2] - A[2], ab0, ab1, ab2) / L2 : 0.f;
    t = fminf(fmaxf(t, 0.f), 1.f);
    const float c0 = fmaf(t, ab0, A[0]), c1 = fmaf(t, ab1, A[1]), c2 = fmaf(t, ab2, A[2]);
    float ax = 0.f, ay = 0.f, az = 1.f;
    if (L2 > 0.f) {
        const float rl = 1.0f / sqrtf(L2);
        ax = ab0 * rl;
        ay = ab1 * rl;
        az = ab2 * rl;
    }
    float vx = p[0] - c0, vy = p[1] - c1, vz = p[2] - c2;
    unit_or_perp(vx, vy, vz, ax, ay, az);
    nt[0] = vx;
    nt[1] = vy;
    nt[2] = vz;
    pt[0] = fmaf(r, vx, c0);
    pt[1] = fmaf(r, vy, c1);
    pt[2] = fmaf(r, vz, c2);
}


#define LG_REALIZE_ARGS                                                                                         \
    DevHand H, const int32_t *__restrict__ wit, const float *__restrict__ pts, const float *__restrict__ nrm,   \
        int N, const float *__restrict__ poses, const int32_t *__restrict__ set_pt,                             \
        const int8_t *__restrict__ set_link, int k, int D, int64_t n_sets,                                      \
        const int32_t *__restrict__ acc_list, const int32_t *__restrict__ n_acc_dev, int max_acc, IkDev ik,    \
        float *__restrict__ q_out, float *__restrict__ cerr, float *__restrict__ cang
#define LG_REALIZE_PASS                                                                                         \
    H, wit, pts, nrm, N, poses, set_pt, set_link, k, D, n_sets, acc_list, n_acc_dev, max_acc, ik, q_out, cerr,  \
        cang

// t / d, correctly rounded, from the correctly rounded r = 1 / d: the quotient's
// residual is exact in one fma, so one correction rounds it right (Markstein);
// the fix-up handles zeros, infinities and NaNs.  Four instructions, not ten.
__device__ inline float div_by(float t, float d, float r)
{
    const float q = t * r;
    return __builtin_amdgcn_div_fixupf(fmaf(fmaf(-q, d, t), r, q), d, t);
}

// LDS of a block of realize_sets: the bin centres and per joint its origin [12],
// axis [3] and limits [2] (read ten times per set; from memory each was a wait)
struct RealizeLds {
    float4 cb4[kMaxBins];
    __attribute__((aligned(16))) float jp[kMaxJoints][20];
};

// The joint values and contact errors of the accepted sets; block bid of nb
// (grid-stride).  What bounds it: VALU issue (470,724 sets of 22 joints: 0.60 G
// wave instructions in 0.92 ms; the same part took 1.2 ms with the joint data in
// memory, full divisions and the five-joint fingers padded to six).
template <int DM>
__device__ __forceinline__ void realize_sets(
    RealizeLds &L, int64_t bid, int64_t nb, const DevHand &H, const int32_t *__restrict__ wit,
    const float *__restrict__ pts, const float *__restrict__ nrm, int N, const float *__restrict__ poses,
    const int32_t *__restrict__ set_pt, const int8_t *__restrict__ set_link, int k, int D, int64_t n_sets,
    const int32_t *__restrict__ acc_list, const int32_t *__restrict__ n_acc_dev, int max_acc, const IkDev &ik,
    float *__restrict__ q_out, float *__restrict__ cerr, float *__restrict__ cang)
{
    for (int i = threadIdx.x; i < H.B; i += kRealizeThreads)
        L.cb4[i] = make_float4(H.bin_c[3 * i], H.bin_c[3 * i + 1], H.bin_c[3 * i + 2], 0.0f);
    for (int i = threadIdx.x; i < 17 * H.J; i += kRealizeThreads) {
        const int j = i / 17, c = i - 17 * j;
        L.jp[j][c] = c < 12 ? H.origin[12 * j + c] : c < 15 ? H.axis[3 * j + c - 12] : H.limits[2 * j + c - 15];
    }
    __syncthreads();
    const int64_t gt = bid * kRealizeThreads + threadIdx.x;
    const int spw = 64 / H.F;                    // sets per wave
    const int lane = threadIdx.x & 63, slot = lane / H.F;
    const int f = lane - slot * H.F;             // this lane's finger
    const int64_t nacc = min((int64_t)*n_acc_dev, (int64_t)max_acc);
    const int64_t stride = ((nb * kRealizeThreads) >> 6) * spw;
    // grid-stride over accepted sets; the F lanes of a set move together, the
    // lanes past spw * F do nothing
    for (int64_t a = slot < spw ? (gt >> 6) * spw + slot : nacc; a < nacc; a += stride) {
        const int64_t id = acc_list[a];
        if (id < 0 || id >= n_sets) {  // not a set id: no reads through it (uniform over the set's lanes)
            if (f < H.F)
                for (int t = 0; t < H.finger_dof[f]; ++t) q_out[a * H.J + H.finger_first[f] + t] = __builtin_nanf("");
            if (f < k) {
                cerr[a * k + f] = INFINITY;
                cang[a * k + f] = INFINITY;
            }
            continue;
        }
        const int64_t g = id / D;
        const int dr = (int)(id % D);
        float P[12];
#pragma unroll
        for (int i = 0; i < 12; ++i) P[i] = poses[12 * g + i];
        // contact layout: the finger of contact i is that of its link; the set is
        // realisable iff every link is a hand link, every point an object point
        // and the fingers increase strictly with i
        uint32_t used = 0;
        bool ok = true;
        int prev = -1;
        for (int i = 0; i < k; ++i) {
            const int l = set_link[id * k + i], idx = set_pt[id * k + i];
            int fl = -1;
            for (int ff = 0; ff < H.F; ++ff)
                if (l >= H.finger_first[ff] && l < H.finger_first[ff] + H.finger_dof[ff]) fl = ff;
            ok = ok && fl > prev && idx >= 0 && idx < N;
            prev = fl;
            if (fl >= 0) used |= 1u << fl;
        }
        if (!ok) used = 0;
        if (f < H.F) {
            float emax = 0.f, amax = 0.f;
            const int first = H.finger_first[f], d = H.finger_dof[f];
            const int ci = ((used >> f) & 1u) ? __popc(used & ((1u << f) - 1u)) : -1;  // this finger's contact
            float q[DM];
            int tl = -1;  // link index within the finger of the contact (-1: none)
            float p[3] = {0.f, 0.f, 0.f}, n[3] = {0.f, 0.f, 1.f};
            if (ci >= 0) {
                const int idx = set_pt[id * k + ci];
                const int l = set_link[id * k + ci];
                const float ox = pts[idx], oy = pts[N + idx], oz = pts[2 * N + idx];
                p[0] = fmaf(P[0], ox, fmaf(P[1], oy, fmaf(P[2], oz, P[3])));
                p[1] = fmaf(P[4], ox, fmaf(P[5], oy, fmaf(P[6], oz, P[7])));
                p[2] = fmaf(P[8], ox, fmaf(P[9], oy, fmaf(P[10], oz, P[11])));
                query_dir(P, nrm[idx], nrm[N + idx], nrm[2 * N + idx], n[0], n[1], n[2]);
                // reverse lookup: witness sample of (link, voxel(p), bin(n))
                int32_t w = kNoWitness;
                if (wit) {
                    const int v = finger_window_voxel(H, P, f, ox, oy, oz);
                    const int b = nearest_bin_any(H.bin_lut, L.cb4, H.B, n[0], n[1], n[2]);
                    if (v >= 0) w = wit[((int64_t)l * H.G * H.G * H.G + v) * H.B + b];
                }
                // the joint sample w (see joint_sample; one Philox block per four joints)
                uint32_t rw[8];
                philox4x32_10((uint32_t)w, (uint32_t)(8 * f), kPurposeJoint, 0u, H.seed_lo, H.seed_hi, rw);
                if (DM > 4 && d > 4)
                    philox4x32_10((uint32_t)w, (uint32_t)(8 * f + 1), kPurposeJoint, 0u, H.seed_lo, H.seed_hi, rw + 4);
#pragma unroll
                for (int t = 0; t < DM; ++t) {
                    q[t] = 0.f;
                    if (t < d) {
                        const float lo = L.jp[first + t][15], hi = L.jp[first + t][16];
                        q[t] = (w >= 0 && w < H.samples) ? fmaf(hi - lo, u01f(rw[t]), lo) : 0.5f * (lo + hi);
                    }
                }
                tl = l - first;
                const float *cap = H.capsule + 7 * l;
                const float r = cap[6];
                float loc_p[3] = {0.f, 0.f, 0.f}, loc_n[3] = {0.f, 0.f, 1.f};
                for (int it = 0; it < ik.iters; ++it) {
                    float o[DM][3], z[DM][3];
                    Tf T, Tl;
#pragma unroll
                    for (int t = 0; t < DM; ++t) {
                        if (t < d) {
                            const float *jp = L.jp[first + t];
                            T = joint_frame_at(jp, jp + 12, T, t > 0, q[t]);
                            o[t][0] = T.m[3];
                            o[t][1] = T.m[7];
                            o[t][2] = T.m[11];
                            tf_dir(T, jp[12], jp[13], jp[14], z[t][0], z[t][1], z[t][2]);
                            if (t == tl) Tl = T;
                        }
                    }
                    float pt[3], nt[3];
                    if (it == 0 || it >= ik.phase1) {
                        float A[3], Bq[3];
                        tf_point(Tl, cap[0], cap[1], cap[2], A[0], A[1], A[2]);
                        tf_point(Tl, cap[3], cap[4], cap[5], Bq[0], Bq[1], Bq[2]);
                        capsule_aligned(A, Bq, r, p, n, ik.beta, pt, nt);
                        const float dx = pt[0] - Tl.m[3], dy = pt[1] - Tl.m[7], dz = pt[2] - Tl.m[11];
#pragma unroll
                        for (int c = 0; c < 3; ++c) {
                            loc_p[c] = fmaf(Tl.m[c], dx, fmaf(Tl.m[4 + c], dy, Tl.m[8 + c] * dz));
                            loc_n[c] = fmaf(Tl.m[c], nt[0], fmaf(Tl.m[4 + c], nt[1], Tl.m[8 + c] * nt[2]));
                        }
                    } else {
                        tf_point(Tl, loc_p[0], loc_p[1], loc_p[2], pt[0], pt[1], pt[2]);
                        tf_dir(Tl, loc_n[0], loc_n[1], loc_n[2], nt[0], nt[1], nt[2]);
                    }
                    float x2[3], e[6];
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        x2[c] = fmaf(ik.beta, nt[c], pt[c]);
                        e[c] = p[c] - pt[c];
                        e[3 + c] = fmaf(ik.beta, n[c], p[c]) - x2[c];
                    }
                    float Jc[DM][6];
#pragma unroll
                    for (int t = 0; t < DM; ++t) {
                        const bool on = t < d && t <= tl;
#pragma unroll
                        for (int s = 0; s < 2; ++s) {
                            const float *x = s == 0 ? pt : x2;
                            const float vx = x[0] - o[t][0], vy = x[1] - o[t][1], vz = x[2] - o[t][2];
                            Jc[t][3 * s + 0] = on ? z[t][1] * vz - z[t][2] * vy : 0.f;
                            Jc[t][3 * s + 1] = on ? z[t][2] * vx - z[t][0] * vz : 0.f;
                            Jc[t][3 * s + 2] = on ? z[t][0] * vy - z[t][1] * vx : 0.f;
                        }
                    }
                    // normal equations (J^T J + lambda I) dq = J^T e, Cholesky in place
                    float M[DM][DM], gv[DM], Mi[DM];  // Mi: reciprocals of the factor's diagonal
#pragma unroll
                    for (int i = 0; i < DM; ++i) {
                        float acc = 0.f;
#pragma unroll
                        for (int rr = 0; rr < 6; ++rr) acc = fmaf(Jc[i][rr], e[rr], acc);
                        gv[i] = acc;
#pragma unroll
                        for (int j = 0; j < DM; ++j) {
                            float s2 = 0.f;
#pragma unroll
                            for (int rr = 0; rr < 6; ++rr) s2 = fmaf(Jc[i][rr], Jc[j][rr], s2);
                            M[i][j] = s2 + (i == j ? ik.lambda : 0.f);
                        }
                    }
                    bool ok = true;
#pragma unroll
                    for (int j = 0; j < DM; ++j) {
                        float s2 = M[j][j];
#pragma unroll
                        for (int kk = 0; kk < j; ++kk) s2 = fmaf(-M[j][kk], M[j][kk], s2);
                        ok &= s2 > 0.f;
                        const float dd = sqrtf(fmaxf(s2, 1e-30f));
                        M[j][j] = dd;
                        const float inv = 1.0f / dd;
                        Mi[j] = inv;
#pragma unroll
                        for (int i = j + 1; i < DM; ++i) {
                            float t2 = M[i][j];
#pragma unroll
                            for (int kk = 0; kk < j; ++kk) t2 = fmaf(-M[i][kk], M[j][kk], t2);
                            M[i][j] = t2 * inv;
                        }
                    }
                    if (!ok) break;
#pragma unroll
                    for (int i = 0; i < DM; ++i) {
                        float t2 = gv[i];
#pragma unroll
                        for (int kk = 0; kk < i; ++kk) t2 = fmaf(-M[i][kk], gv[kk], t2);
                        gv[i] = div_by(t2, M[i][i], Mi[i]);
                    }
#pragma unroll
                    for (int i = DM - 1; i >= 0; --i) {
                        float t2 = gv[i];
#pragma unroll
                        for (int kk = i + 1; kk < DM; ++kk) t2 = fmaf(-M[kk][i], gv[kk], t2);
                        gv[i] = div_by(t2, M[i][i], Mi[i]);
                    }
#pragma unroll
                    for (int t = 0; t < DM; ++t) {
                        if (t < d) q[t] = fminf(fmaxf(q[t] + gv[t], L.jp[first + t][15]), L.jp[first + t][16]);
                    }
                }
            } else {
                // a finger without contact takes uniform random joint values (Sec. 5.6)
                uint32_t w[8];
                philox4x32_10((uint32_t)(ik.pose_offset + g), (uint32_t)dr, kPurposeUnused | ((uint32_t)(2 * f) << 8),
                              ik.request_id, ik.seed_lo, ik.seed_hi, w);
                if (d > 4)
                    philox4x32_10((uint32_t)(ik.pose_offset + g), (uint32_t)dr,
                                  kPurposeUnused | ((uint32_t)(2 * f + 1) << 8), ik.request_id, ik.seed_lo,
                                  ik.seed_hi, w + 4);
#pragma unroll
                for (int t = 0; t < DM; ++t) {
                    q[t] = 0.f;
                    if (t < d) {
                        const float lo = L.jp[first + t][15], hi = L.jp[first + t][16];
                        q[t] = fmaf(hi - lo, u01f(w[t]), lo);
                    }
                }
            }
            // final configuration: contact quality
            Tf T;
#pragma unroll
            for (int t = 0; t < DM; ++t) {
                if (t < d) {
                    const int j = first + t;
                    q_out[a * H.J + j] = q[t];
                    if (t > tl) continue;  // no contact further out
                    T = joint_frame_at(L.jp[j], L.jp[j] + 12, T, t > 0, q[t]);
                    if (t == tl) {
                        const float *cj = H.capsule + 7 * j;
                        float A[3], Bq[3];
                        tf_point(T, cj[0], cj[1], cj[2], A[0], A[1], A[2]);
                        tf_point(T, cj[3], cj[4], cj[5], Bq[0], Bq[1], Bq[2]);
                        float pt[3], nt[3];
                        capsule_project(A, Bq, cj[6], p, pt, nt);
                        const float d0 = p[0] - pt[0], d1 = p[1] - pt[1], d2 = p[2] - pt[2];
                        emax = sqrtf(dot3f(d0, d1, d2, d0, d1, d2));
                        amax = acosf(fminf(fmaxf(dot3f(nt[0], nt[1], nt[2], n[0], n[1], n[2]), -1.f), 1.f));
                    }
                }
            }
            if (ci >= 0) {
                cerr[a * k + ci] = emax;
                cang[a * k + ci] = amax;
            }
        }
        if (!ok && f < k) {  // not realisable: no contact is met
            cerr[a * k + f] = INFINITY;
            cang[a * k + f] = INFINITY;
        }
    }
}

// Part [t0, t1] of a segment (parameter 0..1, ends yA, yB in SDF grid
// coordinates) that can lie in the grid [0, gm]^3, widened by 1e-3 of a cell;
// empty: t0 > t1.  A NaN constrains nothing.
__device__ inline void grid_part(const float *yA, const float *yB, float gm, float &t0, float &t1)
{
    t0 = 0.f;
    t1 = 1.f;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const float d = yB[c] - yA[c], lo = -1e-3f - yA[c], hi = gm + 1e-3f - yA[c];
        if (fabsf(d) < 1e-6f) {
            if (lo > 1e-3f || hi < -1e-3f) t0 = 2.f;
            continue;
        }
        const float r = 1.0f / d, a = lo * r, b = hi * r;
        t0 = fmaxf(t0, fminf(a, b));  // fmaxf / fminf drop a NaN
        t1 = fminf(t1, fmaxf(a, b));
    }
}

// Sets whose samples a wave takes side by side when it has kManySets or more: a
// hand's few samples in the grid then fill the lanes, and their reads overlap (65,536
// sets of 12 links in two fingers 209 -> 171 us with the joint steps, 262,144 of 22
// links 1,103 -> 1,047).  With fewer sets per wave one set after another over all lanes is the
// faster one (300 sets of 22 links 73 us, 96 with four side by side).
constexpr int kManySets = 8, kSideBySide = 4;

// A link of a set at its final configuration: axis ends (hand frame), the set's
// samples before it and its first sample in the grid.
struct __attribute__((aligned(16))) LinkSeg {
    float a[3], b[3];
    int pre, first;
};

// Sets per wave of the penetration test: a lane per finger, and no more than leave
// room for four blocks' segments in a CU's 160 KB, which is the launch's size and what
// the registers allow (1 finger of 8 links: 64 sets per wave leave room for two blocks,
// 8 x 8 links two, 2 x 6 three).  With the joint steps, 65,536 sets: 2 x 6 links 172 ->
// 136 us, 1 x 8 157 -> 127, 6 x 7 882 -> 714, 8 x 8 1,077 -> 922.
__host__ __device__ inline int penetrate_sets_per_wave(int F, int J)
{
    const int room = (40960 - J * (int)sizeof(float2)) / (kRealizeThreads / 64 * J * (int)sizeof(LinkSeg));
    return room < 64 / F ? room : 64 / F;  // J <= 64: room >= 4
}

// LDS of a block: a LinkSeg per (set, link) of each wave, and per link the
// sample spacing 1 / (M - 1) and the radius
__host__ __device__ inline size_t penetrate_lds(int F, int J)
{
    return (size_t)(kRealizeThreads / 64) * penetrate_sets_per_wave(F, J) * J * sizeof(LinkSeg) +
           (size_t)J * sizeof(float2);
}

__device__ inline void wave_fence()
{
    __builtin_amdgcn_wave_barrier();
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

// Penetration and validity of the realised sets (q_out, cerr, cang of
// realize_sets).  A wave takes 64 / F sets.  First each lane walks its finger's
// links, the joint frames from the joint values as realize_sets computes them,
// and leaves the axis ends and the number of axis samples that can lie in the
// SDF's grid in LDS (the others give no depth).  Then the lanes take the
// samples of one set after another, or of a few side by side: neighbouring lanes
// are 1 mm apart on one axis, so their corner reads fall in few cache lines.  With
// a lane per finger, 64 lanes read 64 unrelated cells each time: 2.6 ms at six waves
// per SIMD, 1.7 ms at two inside the step kernel (fewer lines evicted between a
// lane's samples); 470,724 sets of 22 joints now take 1.2 ms, bound by the lines the
// corner reads touch (28 per read, one a cycle) and by VALU issue.
// SC: the hand's self-collision too, a set's pairs of links over the same lanes (a
// finger's lane for its links took 448 pairs one after another at 8 fingers of 8
// links: 300 sets 503 us with the joint steps, now 122).
template <bool SC>
__device__ __forceinline__ void penetrate_sets(
    char *lds, int64_t bid, int64_t nb, const DevHand &H, const SdfDev &S, const float *__restrict__ poses, int k,
    int D, int64_t n_sets, const int32_t *__restrict__ acc_list, const int32_t *__restrict__ n_acc_dev, int max_acc,
    const IkDev &ik, const float *__restrict__ q_in, const float *__restrict__ cerr, const float *__restrict__ cang,
    float *__restrict__ depth_out, uint8_t *__restrict__ valid_out)
{
    const int J = H.J, F = H.F, spw = penetrate_sets_per_wave(F, J);
    const int tid = threadIdx.x, lane = tid & 63, slot = lane / F, f = lane - slot * F;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    LinkSeg *segs = reinterpret_cast<LinkSeg *>(lds) + (size_t)wave * spw * J;  // [set][link]
    float2 *link = reinterpret_cast<float2 *>(lds + (size_t)(kRealizeThreads / 64) * spw * J * sizeof(LinkSeg));
    for (int j = tid; j < J; j += kRealizeThreads)
        link[j] = make_float2(1.0f / (float)(H.axis_samples[j] - 1), H.capsule[7 * j + 6]);
    __syncthreads();
    const int64_t nacc = min((int64_t)*n_acc_dev, (int64_t)max_acc);
    const int first = H.finger_first[f], d = H.finger_dof[f];
    const float gm = (float)(S.G - 1);
    // few sets: fewer than spw per wave, so that every wave has some
    const int64_t waves = nb * (kRealizeThreads / 64);
    const int per = (int)max((int64_t)1, min((int64_t)spw, (nacc + waves - 1) / waves));
    for (int64_t a0 = (bid * (kRealizeThreads / 64) + wave) * per; a0 < nacc; a0 += waves * per) {
        const int64_t a = a0 + slot;
        const bool mine = slot < per && a < nacc;
        const int64_t id = mine ? acc_list[a] : -1;
        const bool live = id >= 0 && id < n_sets;  // uniform over a set's lanes
        const int g = live ? (int)(id / D) : 0;
        float dep = -INFINITY;
        int count = 0;  // samples of this lane's finger
        if (live) {
            float P[12];
#pragma unroll
            for (int i = 0; i < 12; ++i) P[i] = poses[12 * (int64_t)g + i];
            Tf T;
            for (int t = 0; t < d; ++t) {
                const int j = first + t;
                T = joint_frame(H, T, t > 0, j, q_in[a * J + j]);
                const float *cj = H.capsule + 7 * j;
                LinkSeg sg;
                tf_point(T, cj[0], cj[1], cj[2], sg.a[0], sg.a[1], sg.a[2]);
                tf_point(T, cj[3], cj[4], cj[5], sg.b[0], sg.b[1], sg.b[2]);
                const float M1 = (float)(H.axis_samples[j] - 1);
                // the axis in grid coordinates: R^T (x - t), less the origin, over h
                float y[2][3];
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const float *x = e ? sg.b : sg.a;
                    const float x0 = x[0] - P[3], x1 = x[1] - P[7], x2 = x[2] - P[11];
                    y[e][0] = (fmaf(P[0], x0, fmaf(P[4], x1, P[8] * x2)) - S.ox) * S.inv_h;
                    y[e][1] = (fmaf(P[1], x0, fmaf(P[5], x1, P[9] * x2)) - S.oy) * S.inv_h;
                    y[e][2] = (fmaf(P[2], x0, fmaf(P[6], x1, P[10] * x2)) - S.oz) * S.inv_h;
                }
                float t0, t1;
                grid_part(y[0], y[1], gm, t0, t1);
                // a sample more on either side covers the rounding of t
                sg.first = max(0, (int)(t0 * M1) - 1);
                const int last = t0 > t1 ? -1 : min((int)M1, (int)(t1 * M1) + 2);
                sg.pre = max(0, last - sg.first + 1);  // the link's samples; summed below
                count += sg.pre;
                segs[slot * J + j] = sg;
            }
        }
        // samples of the set before this lane's finger, and of the whole set
        int before = 0, total = 0;
        for (int q = 0; q < F; ++q) {
            const int n = __shfl(count, lane - f + q, 64);
            before += q < f ? n : 0;
            total += n;
        }
        if (live)
            for (int t = 0; t < d; ++t) {
                int &pre = segs[slot * J + first + t].pre;
                const int n = pre;
                pre = before;
                before += n;
            }
        wave_fence();
        const int n_slots = (int)min((int64_t)per, nacc - a0);
        // depths of the wave's sets, NS at a time, 64 / NS lanes for each
        auto depths = [&](auto at_a_time) {
            constexpr int NS = decltype(at_a_time)::value, kLanes = 64 / NS;
            for (int sl0 = 0; sl0 < n_slots; sl0 += NS) {
                const int sl = NS == 1 ? sl0 : sl0 + lane / kLanes, sub = lane % kLanes;  // this lane's set
                int n, gs;
                bool on;  // a set, and something to test
                if constexpr (NS == 1) {
                    n = __builtin_amdgcn_readlane(total, sl * F);
                    gs = __builtin_amdgcn_readlane(g, sl * F);
                    on = SC ? __builtin_amdgcn_readlane((int)live, sl * F) != 0 : n > 0;
                    if (!on) continue;
                } else {
                    const bool is = sl < n_slots;
                    n = __shfl(total, sl * F, 64);
                    gs = __shfl(g, sl * F, 64);
                    on = __shfl((int)live, sl * F, 64) != 0 && is;
                    n = is ? n : 0;
                    if (__ballot(SC ? on : n > 0) == 0) continue;
                }
                const float *P = poses + 12 * (int64_t)gs;
                const LinkSeg *sg = segs + sl * J;
                float dp = -INFINITY;
                // hand self-collision: the links of finger f1 against all of the later fingers
                if (SC && on)
                    for (int f1 = 0; f1 + 1 < F; ++f1) {
                        const int l0 = H.finger_first[f1], l1 = l0 + H.finger_dof[f1], m = J - l1;
                        const float rm = 1.0f / (float)m;
                        for (int i = sub; i < (l1 - l0) * m; i += kLanes) {
                            const int t = (int)(((float)i + 0.5f) * rm);  // i / m (i < 512: exact)
                            const int j1 = l0 + t, j2 = l1 + i - t * m;
                            dp = fmaxf(dp, link[j1].y + link[j2].y - segment_distance(sg[j1].a, sg[j1].b, sg[j2].a, sg[j2].b));
                        }
                    }
                int lo = 0;
                for (int i = sub; i < n; i += kLanes) {
                    while (lo + 1 < J && sg[lo + 1].pre <= i) ++lo;  // the link: the last one with pre <= i
                    const LinkSeg c = sg[lo];
                    const float2 l = link[lo];
                    const float ts = (float)(c.first + i - c.pre) * l.x;
                    const float x0 = fmaf(ts, c.b[0] - c.a[0], c.a[0]) - P[3];
                    const float x1 = fmaf(ts, c.b[1] - c.a[1], c.a[1]) - P[7];
                    const float x2 = fmaf(ts, c.b[2] - c.a[2], c.a[2]) - P[11];
                    // object frame: R^T (x - t)
                    const float y0 = fmaf(P[0], x0, fmaf(P[4], x1, P[8] * x2));
                    const float y1 = fmaf(P[1], x0, fmaf(P[5], x1, P[9] * x2));
                    const float y2 = fmaf(P[2], x0, fmaf(P[6], x1, P[10] * x2));
                    dp = fmaxf(dp, l.y - sdf_trilinear<true>(S, y0, y1, y2));
                }
                for (int off = kLanes / 2; off > 0; off >>= 1) dp = fmaxf(dp, __shfl_xor(dp, off, 64));
                if constexpr (NS > 1) dp = __shfl(dp, (slot - sl0) * kLanes, 64);  // of the finger lanes' set
                if (slot >= sl0 && slot < sl0 + NS) dep = fmaxf(dep, dp);
            }
        };
        if (per >= kManySets)
            depths(std::integral_constant<int, kSideBySide>());
        else
            depths(std::integral_constant<int, 1>());
        wave_fence();  // the segments are rewritten by the next sets
        // the set's depth over its F lanes
        float dm = dep;
        for (int q = 0; q < F; ++q) dm = fmaxf(dm, __shfl(dep, lane - f + q, 64));
        if (mine && f == 0) {
            if (!live) {  // not a set id
                depth_out[a] = __builtin_nanf("");
                valid_out[a] = 0;
                continue;
            }
            // worst contact (a finger without contact counts 0)
            float emax = k < F ? 0.f : cerr[a * k], amax = k < F ? 0.f : cang[a * k];
            for (int i = 0; i < k; ++i) {
                emax = fmaxf(emax, cerr[a * k + i]);
                amax = fmaxf(amax, cang[a * k + i]);
            }
            depth_out[a] = dm;
            valid_out[a] = (emax <= ik.tol_pos && amax <= ik.tol_ang && dm <= ik.margin) ? 1 : 0;
        }
    }
}

// up to 6 joints per finger: two waves per SIMD (at most 256 registers)
template <int DM>
__global__ void __launch_bounds__(kRealizeThreads) __attribute__((amdgpu_waves_per_eu(2)))
k_realize(LG_REALIZE_ARGS)
{
    __shared__ RealizeLds L;
    realize_sets<DM>(L, blockIdx.x, gridDim.x, LG_REALIZE_PASS);
}

// 7 or 8 joints per finger: one wave per SIMD rather than spilling
__global__ void __launch_bounds__(kRealizeThreads) k_realize_wide(LG_REALIZE_ARGS)
{
    __shared__ RealizeLds L;
    realize_sets<8>(L, blockIdx.x, gridDim.x, LG_REALIZE_PASS);
}

template <bool SC>
__global__ void __launch_bounds__(kRealizeThreads)
k_penetrate(DevHand H, SdfDev S, const float *__restrict__ poses, int k, int D, int64_t n_sets,
            const int32_t *__restrict__ acc_list, const int32_t *__restrict__ n_acc_dev, int max_acc, IkDev ik,
            const float *__restrict__ q, const float *__restrict__ cerr, const float *__restrict__ cang,
            float *__restrict__ depth, uint8_t *__restrict__ valid)
{
    extern __shared__ __attribute__((aligned(16))) char lds[];
    penetrate_sets<SC>(lds, blockIdx.x, gridDim.x, H, S, poses, k, D, n_sets, acc_list, n_acc_dev, max_acc, ik, q,
                       cerr, cang, depth, valid);
}

// The same over the accepted sets of several chunks (max_acc = the chunk's
// P * D); DM = 8 takes one wave per SIMD like k_realize_wide.
template <int DM>
__global__ void __launch_bounds__(kRealizeThreads) __attribute__((amdgpu_waves_per_eu(DM <= 6 ? 2 : 1)))
k_realize_batch(const ChunkDesc *__restrict__ d, const uint16_t *__restrict__ idx, const uint32_t *__restrict__ first,
                int n)
{
    __shared__ RealizeLds L;
    const int j = batch_member(first, n, blockIdx.x);
    const ChunkDesc &c = d[idx[j]];
    const int64_t n_sets = (int64_t)c.P * c.D;
    realize_sets<DM>(L, blockIdx.x - first[j], first[j + 1] - first[j], c.H, c.wit, c.pts, c.nrm, c.N, c.poses,
                     c.set_pt, c.set_link, c.k, c.D, n_sets, c.acc, c.n_acc, (int)n_sets, c.ik, c.q, c.err, c.ang);
}

template <bool SC>
__global__ void __launch_bounds__(kRealizeThreads) __attribute__((amdgpu_waves_per_eu(4)))
k_penetrate_batch(const ChunkDesc *__restrict__ d, const uint16_t *__restrict__ idx,
                  const uint32_t *__restrict__ first, int n)
{
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int j = batch_member(first, n, blockIdx.x);
    const ChunkDesc &c = d[idx[j]];
    const int64_t n_sets = (int64_t)c.P * c.D;
    penetrate_sets<SC>(lds, blockIdx.x - first[j], first[j + 1] - first[j], c.H, c.S, c.poses, c.k, c.D, n_sets,
                       c.acc, c.n_acc, (int)n_sets, c.ik, c.q, c.err, c.ang, c.depth, c.valid);
}

#undef LG_REALIZE_ARGS
#undef LG_REALIZE_PASS

}  // namespace lg

using namespace lg;

extern "C" lg_status lg_realize(const lg_field *field, const lg_sdf *sdf, const float *pts, const float *nrm,
                                int32_t n_points, const float *poses, int32_t n_poses, const int32_t *set_pt,
                                const int8_t *set_link, int32_t k, int32_t draws, const int32_t *acc_list,
                                const int32_t *n_acc_dev, int32_t max_acc, const lg_ik_params *p, float *q_out,
                                float *contact_err, float *contact_ang, float *depth, uint8_t *valid, void *stream)
{
    if (!field || !sdf || !p) return fail(LG_EINVAL, "null field, sdf or params");
    const DevHand &H = field->dh;
    if (k < 1 || k > H.F) return fail(LG_EINVAL, "need 1 <= k <= number of fingers");
    if (n_points <= 0 || n_poses <= 0 || draws <= 0 || max_acc < 0)
        return fail(LG_EINVAL, "bad sizes");
    if (sdf->dims < 2 || !(sdf->h > 0.f) || !sdf->values) return fail(LG_EINVAL, "bad sdf");
    if (p->iters < 0 || p->phase1 < 0 || !(p->lambda > 0.f)) return fail(LG_EINVAL, "need iters >= 0, lambda > 0");
    if (max_acc == 0) return LG_OK;
    if (!pts || !nrm || !poses || !set_pt || !set_link || !acc_list || !n_acc_dev || !q_out || !contact_err ||
        !contact_ang || !depth || !valid)
        return fail(LG_EINVAL, "null device buffer");
    SdfDev S{sdf->origin[0], sdf->origin[1], sdf->origin[2], sdf->h, 1.0f / sdf->h, sdf->dims, sdf->values};
    IkDev ik{p->iters, p->phase1, p->lambda, p->beta, p->tol_pos, p->tol_ang, p->margin, p->self_collision,
             (uint32_t)p->seed, (uint32_t)(p->seed >> 32), p->request_id, p->pose_offset};
    hipStream_t s = as_stream(stream);
    // grid-stride launch sized to the device, not to the max_acc upper bound
    int dev = 0, n_cu = 0;
    LG_HIP(hipGetDevice(&dev));
    LG_HIP(hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev));
    const dim3 grid(realize_blocks(max_acc, H.F, n_cu));
    const int32_t *wit = field->has_witness ? field->d_wit : nullptr;
    const int64_t n_sets = (int64_t)n_poses * draws;
#define LG_REALIZE(KERNEL)                                                                                      \
    hipLaunchKernelGGL(KERNEL, grid, dim3(kRealizeThreads), 0, s, H, wit, pts, nrm, n_points, poses, set_pt,     \
                       set_link, k, draws, n_sets, acc_list, n_acc_dev, max_acc, ik, q_out, contact_err, contact_ang)
    if (field->max_dof <= 4)
        LG_REALIZE(k_realize<4>);
    else if (field->max_dof <= 5)
        LG_REALIZE(k_realize<5>);
    else if (field->max_dof <= 6)
        LG_REALIZE(k_realize<6>);
    else
        LG_REALIZE(k_realize_wide);
#undef LG_REALIZE
    const size_t lds = penetrate_lds(H.F, H.J);
    const dim3 pgrid(penetrate_blocks(max_acc, n_cu));
    if (ik.self_collision)
        hipLaunchKernelGGL(k_penetrate<true>, pgrid, dim3(kRealizeThreads), lds, s, H, S, poses, k, draws, n_sets, acc_list,
                           n_acc_dev, max_acc, ik, q_out, contact_err, contact_ang, depth, valid);
    else
        hipLaunchKernelGGL(k_penetrate<false>, pgrid, dim3(kRealizeThreads), lds, s, H, S, poses, k, draws, n_sets, acc_list,
                           n_acc_dev, max_acc, ik, q_out, contact_err, contact_ang, depth, valid);
    LG_HIP(hipGetLastError());
    return LG_OK;
}

size_t lg::realize_lds_bytes(int F, int J) { return penetrate_lds(F, J); }

uint32_t lg::realize_blocks(int64_t max_acc, int F, int n_cu)
{
    const int64_t spw = 64 / F;  // sets per wave
    const int64_t threads = std::min<int64_t>((max_acc + spw - 1) / spw * 64, (int64_t)n_cu * 16 * kRealizeThreads);
    return (uint32_t)std::max<int64_t>(1, (threads + kRealizeThreads - 1) / kRealizeThreads);
}

// Blocks of the penetration test: at most what is resident (16 waves a CU), down to
// a set per wave (1,000 sets of 3 fingers: 40 us with 21 sets per wave).
uint32_t lg::penetrate_blocks(int64_t max_acc, int n_cu)
{
    return (uint32_t)std::max<int64_t>(1, std::min<int64_t>((max_acc + 3) / 4, (int64_t)n_cu * 4));
}

lg_status lg::realize_batch(const BatchLaunch &b, const BatchLaunch &pb, int max_dof, size_t lds, bool self_collision,
                            hipStream_t s)
{
    if (b.n <= 0 || b.blocks == 0) return LG_OK;
    if (max_dof <= 4)
        hipLaunchKernelGGL(k_realize_batch<4>, dim3(b.blocks), dim3(kRealizeThreads), 0, s, b.d, b.idx, b.first, b.n);
    else if (max_dof <= 5)
        hipLaunchKernelGGL(k_realize_batch<5>, dim3(b.blocks), dim3(kRealizeThreads), 0, s, b.d, b.idx, b.first, b.n);
    else if (max_dof <= 6)
        hipLaunchKernelGGL(k_realize_batch<6>, dim3(b.blocks), dim3(kRealizeThreads), 0, s, b.d, b.idx, b.first, b.n);
    else
        hipLaunchKernelGGL(k_realize_batch<8>, dim3(b.blocks), dim3(kRealizeThreads), 0, s, b.d, b.idx, b.first, b.n);
    if (self_collision)
        hipLaunchKernelGGL(k_penetrate_batch<true>, dim3(pb.blocks), dim3(kRealizeThreads), lds, s, pb.d, pb.idx,
                           pb.first, pb.n);
    else
        hipLaunchKernelGGL(k_penetrate_batch<false>, dim3(pb.blocks), dim3(kRealizeThreads), lds, s, pb.d, pb.idx,
                           pb.first, pb.n);
    LG_HIP(hipGetLastError());
    return LG_OK;
}
