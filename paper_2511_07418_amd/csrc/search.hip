// Contact-set draws (Sec. 5.3, Alg. 2 initialisation), reverse lookup of the
// hand link (Sec. 5.5), the contact-set criterion (Eq. 1-2 with a linearised
// friction cone, as an LP) and deterministic compaction of accepted sets.
#include <math.h>

#include <algorithm>
#include <mutex>
#include <string>

#include "lg_internal.h"

namespace lg {

constexpr int kDrawThreads = 256;
constexpr int kSuper = 8;           // words per rank superblock
constexpr int kChunkPerThread = 32; // compaction: sets per thread
constexpr int kCompactThreads = 256;
constexpr int kChunk = kChunkPerThread * kCompactThreads;

// select the r-th (0-based) set bit of x (r < popcount): halves by their popcounts
__device__ inline int select_in_word(uint32_t x, uint32_t r)
{
    int at = 0;
#pragma unroll
    for (int h = 16; h > 0; h >>= 1) {
        const uint32_t low = x & ((1u << h) - 1u), c = (uint32_t)__popc(low);
        const bool up = r >= c;
        at += up ? h : 0;
        r -= up ? c : 0u;
        x = up ? x >> h : low;
    }
    return at;
}

constexpr uint32_t kPurposeFingers = 13u;
constexpr uint32_t kPurposeExtFingers = 19u;  // second contact round: fingers
constexpr uint32_t kPurposeExtDraw = 21u;     // second contact round: points and links

// Contact fingers of set d of pose gg (global index) as a bit mask: k picks
// without replacement among the eligible fingers (non-empty domains), pick j
// taking the floor(w_j (c - j) / 2^32)-th remaining one in increasing finger
// order; contact i goes to the i-th lowest bit.  With c == k every eligible
// finger is picked whatever the words, so they are not drawn.
__device__ inline uint32_t choose_fingers(uint32_t elig, int k, uint32_t gg, int d, uint32_t request_id,
                                          uint32_t seed_lo, uint32_t seed_hi, uint32_t purpose = kPurposeFingers)
{
    const int c = __popc(elig);
    if (c <= k) return c == k ? elig : 0u;
    uint32_t w[8];
    philox4x32_10(gg, (uint32_t)d, purpose, request_id, seed_lo, seed_hi, w);
    if (k > 4) philox4x32_10(gg, (uint32_t)d, purpose | (1u << 8), request_id, seed_lo, seed_hi, w + 4);
    uint32_t left = elig, mask = 0;
    for (int j = 0; j < k; ++j) {
        uint32_t x = left;
        for (uint32_t r = __umulhi(w[j], (uint32_t)(c - j)); r > 0; --r) x &= x - 1u;
        const uint32_t bit = x & (0u - x);
        mask |= bit;
        left &= ~bit;
    }
    return mask;
}

// eligible fingers of pose g: those whose domain is non-empty
__device__ inline uint32_t eligible_fingers(const uint32_t *__restrict__ dom_count, int64_t g, int F)
{
    uint32_t e = 0;
    for (int f = 0; f < F; ++f) e |= (dom_count[g * F + f] > 0 ? 1u : 0u) << f;
    return e;
}

// inclusive prefix sum over the lanes (row shifts by 1, 2, 4, 8, then the row
// broadcasts); lanes without a source add 0
__device__ inline uint32_t wave_scan_incl(uint32_t x)
{
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, false);  // row_shr:1
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, false);  // row_shr:2
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, false);  // row_shr:4
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, false);  // row_shr:8
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xa, 0xf, false);  // row_bcast:15
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xc, 0xf, false);  // row_bcast:31
    return x;
}

// What the reverse lookup of a pose needs in LDS: the bin centres and the map of
// each finger's window (the lattice's in entry 0 for lattice windows).
struct LinkLds {
    float4 cb4[kMaxBins];
    Affine aff[kMaxFingers];
};

// fill it (the caller synchronises after)
__device__ inline void link_lds(LinkLds &L, const DevHand &H, const float *pose)
{
    for (int i = threadIdx.x; i < H.B; i += blockDim.x)
        L.cb4[i] = make_float4(H.bin_c[3 * i], H.bin_c[3 * i + 1], H.bin_c[3 * i + 2], 0.0f);
    if ((int)threadIdx.x < (H.lat ? 1 : H.F)) L.aff[threadIdx.x] = window_map(H, pose, threadIdx.x);
}

// Reverse lookup (Sec. 5.5): among the links of finger i whose own table is
// hit at point idx under the pose, the floor(r * count / 2^32)-th; -1 if none.
// aff: window_map of the finger.
__device__ inline int pick_link(const DevHand &H, const float4 *cb4,
                                const Affine &aff, const float *__restrict__ pts, const float *__restrict__ nrm, int N,
                                const float *pose, int i, int idx, uint32_t r)
{
    const int v = map_window_voxel(H, aff, i, pts[idx], pts[N + idx], pts[2 * N + idx]);
    float qx, qy, qz;
    query_dir(pose, nrm[idx], nrm[N + idx], nrm[2 * N + idx], qx, qy, qz);
    const int b = nearest_bin_any(H.bin_lut, cb4, H.B, qx, qy, qz);
    const int first = H.finger_first[i];
    const uint32_t mask = v >= 0 ? H.link_mask[((int64_t)i * H.G * H.G * H.G + v) * H.B + b] : 0u;
    const uint32_t pc = __popc(mask);
    return pc ? first + select_in_word(mask, __umulhi(r, pc)) : -1;
}

// Words [s kSuper, (s + 1) kSuper) of a domain of NW words (0 past its end), loaded together.
__device__ inline void load_super(const uint32_t *__restrict__ dom, int NW, int s, uint32_t (&w)[kSuper])
{
    static_assert(kSuper == 8, "two 16-byte loads");
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4), aligned(4)));
    const uint32_t *d = dom + s * kSuper;
    if ((s + 1) * kSuper <= NW) {
        const u32x4 a = *(const u32x4 *)d, b = *(const u32x4 *)(d + 4);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            w[i] = a[i];
            w[4 + i] = b[i];
        }
    } else {
#pragma unroll
        for (int i = 0; i < kSuper; ++i) w[i] = s * kSuper + i < NW ? d[i] : 0u;
    }
}

// The j-th (0-based) set bit of a domain of NW words through its superblock
// prefix pf (nsb + 1 exclusive popcounts of kSuper-word superblocks): binary
// search for the last superblock with pf <= j, then its words; -1 if the domain
// has no j-th bit.
__device__ inline int select_domain(const uint32_t *pf, int nsb, const uint32_t *__restrict__ dom, int NW, uint32_t j)
{
    int lo = 0, hi = nsb;  // invariant pf[lo] <= j < pf[hi]
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (pf[mid] <= j) lo = mid; else hi = mid;
    }
    uint32_t rem = j - pf[lo], w[kSuper], word = 0, left = 0;
    load_super(dom, NW, lo, w);
    int at = -1;
#pragma unroll
    for (int i = 0; i < kSuper; ++i) {
        const uint32_t pc = __popc(w[i]);
        if (at < 0 && rem < pc) {
            at = lo * kSuper + i;
            word = w[i];
            left = rem;
        }
        rem -= pc;
    }
    return at < 0 ? -1 : at * 32 + select_in_word(word, left);
}

// Superblock popcount prefixes of the F domains of one pose into LDS
// (prefix[f * (nsb + 1) + sb]); the caller synchronises after.  A wave takes a
// finger: 64 superblocks at a time, summed by a scan over the lanes (one thread
// per finger adding up its 256 counts took most of the draw).
__device__ inline void build_prefix(uint32_t *prefix, const uint32_t *__restrict__ dom, int F, int NW, int nsb)
{
    const int lane = threadIdx.x & 63, waves = blockDim.x >> 6;
    for (int f = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); f < F; f += waves) {
        const uint32_t *d = dom + (int64_t)f * NW;
        uint32_t *pf = prefix + f * (nsb + 1);
        uint32_t run = 0;
        if (lane == 0) pf[0] = 0;
        for (int s0 = 0; s0 < nsb; s0 += 64) {
            const int sb = s0 + lane;
            uint32_t c = 0;
            if (sb < nsb) {
                uint32_t w[kSuper];
                load_super(d, NW, sb, w);
#pragma unroll
                for (int q = 0; q < kSuper; ++q) c += __popc(w[q]);
            }
            const uint32_t incl = wave_scan_incl(c);
            if (sb < nsb) pf[sb + 1] = run + incl;
            run += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
        }
    }
}

// One workgroup per pose.  Rank structure: exclusive popcount prefix per
// superblock of 8 domain words, in LDS; a draw binary-searches it and scans
// at most 8 words.  A thread per contact of a set (each draws the words it needs);
// a thread per set walked its contacts' dependent reads one after another.  What
// bounds it: the latency of those reads (65,536 poses x 64 sets of 5, 30 % of the
// poses with draws: 0.88 -> 0.40 ms; 256 poses x 16 sets of 3: 21 -> 6 us).
// the D sets of pose g (one block); prefix: [F][nsb + 1] words of LDS
__device__ __forceinline__ void draw_pose(uint32_t *prefix, LinkLds &L, uint32_t *counts, const DevHand &H,
                                          const float *__restrict__ pts,
                                          const float *__restrict__ nrm, int N, const float *__restrict__ poses,
                                          const uint32_t *__restrict__ dom_bits, const uint32_t *__restrict__ dom_count,
                                          const int32_t *__restrict__ palm_pt, int D, int k, uint32_t seed_lo,
                                          uint32_t seed_hi, uint32_t request_id, int64_t pose_offset,
                                          int32_t *__restrict__ set_pt, int8_t *__restrict__ set_link,
                                          uint8_t *__restrict__ pose_valid, uint8_t *__restrict__ verdict,
                                          double *__restrict__ tstar, int g)
{
    const int F = H.F;
    const int NW = (N + 31) >> 5, nsb = (NW + kSuper - 1) / kSuper;
    const uint32_t *dom = dom_bits + (int64_t)g * F * NW;
    if (threadIdx.x < F) counts[threadIdx.x] = dom_count[(int64_t)g * F + threadIdx.x];
    __syncthreads();
    uint32_t elig = 0;
    for (int f = 0; f < F; ++f) elig |= (counts[f] > 0 ? 1u : 0u) << f;
    // fewer than k usable domains, or a palm placement that was rejected
    const bool empty = __popc(elig) < k || (palm_pt && palm_pt[g] == -2);
    if (threadIdx.x == 0) pose_valid[g] = empty ? 0 : 1;
    if (empty) {
        for (int64_t i = threadIdx.x; i < (int64_t)D * k; i += blockDim.x) {  // D k may exceed 2^31
            set_pt[(int64_t)g * D * k + i] = -1;
            set_link[(int64_t)g * D * k + i] = -1;
        }
        for (int64_t d = threadIdx.x; d < D; d += blockDim.x) {  // no LP for these sets
            verdict[(int64_t)g * D + d] = 0;
            tstar[(int64_t)g * D + d] = __builtin_nan("");
        }
        return;  // uniform over the block
    }
    const float *pose = poses + 12 * (int64_t)g;
    link_lds(L, H, pose);
    build_prefix(prefix, dom, F, NW, nsb);
    __syncthreads();
    const uint32_t gg = (uint32_t)(pose_offset + g);
    // contact i of set d, blockDim.x contacts apart (D k may exceed 2^31)
    const uint32_t step_d = blockDim.x / (uint32_t)k, step_i = blockDim.x - step_d * (uint32_t)k;
    uint32_t d = threadIdx.x / (uint32_t)k;
    for (uint32_t i = threadIdx.x - d * (uint32_t)k; d < (uint32_t)D; d += step_d, i += step_i) {
        if (i >= (uint32_t)k) {
            i -= (uint32_t)k;
            if (++d >= (uint32_t)D) break;
        }
        uint32_t w[4];
        auto word = [&](int q) {  // word q of the set's Philox blocks
            philox4x32_10(gg, 4u * d + ((uint32_t)q >> 2), kPurposeDraw, request_id, seed_lo, seed_hi, w);
            return (q & 2) ? ((q & 1) ? w[3] : w[2]) : ((q & 1) ? w[1] : w[0]);
        };
        const uint32_t fm = choose_fingers(elig, k, gg, (int)d, request_id, seed_lo, seed_hi);
        const int f = select_in_word(fm, i);  // its finger
        const int idx = select_domain(prefix + f * (nsb + 1), nsb, dom + (int64_t)f * NW, NW,
                                      __umulhi(word(i), counts[f]));
        const int64_t at = ((int64_t)g * D + d) * k + i;
        set_pt[at] = idx;
        set_link[at] = (int8_t)(idx >= 0 ? pick_link(H, L.cb4, L.aff[H.lat ? 0 : f], pts, nrm, N, pose, f, idx,
                                                     word(k + i))
                                         : -1);
    }
}

__global__ void __launch_bounds__(kDrawThreads)
k_draw(DevHand H, const float *__restrict__ pts, const float *__restrict__ nrm,
       int N, const float *__restrict__ poses, const uint32_t *__restrict__ dom_bits,
       const uint32_t *__restrict__ dom_count, const int32_t *__restrict__ palm_pt, int D, int k, uint32_t seed_lo,
       uint32_t seed_hi, uint32_t request_id, int64_t pose_offset, int32_t *__restrict__ set_pt,
       int8_t *__restrict__ set_link, uint8_t *__restrict__ pose_valid, uint8_t *__restrict__ verdict,
       double *__restrict__ tstar)
{
    extern __shared__ uint32_t prefix[];
    __shared__ LinkLds L;
    __shared__ uint32_t counts[kMaxFingers];
    draw_pose(prefix, L, counts, H, pts, nrm, N, poses, dom_bits, dom_count, palm_pt, D, k, seed_lo, seed_hi,
              request_id, pose_offset, set_pt, set_link, pose_valid, verdict, tstar, blockIdx.x);
}

// the same over the poses of several chunks (no palm contacts)
__global__ void __launch_bounds__(kDrawThreads)
k_draw_batch(const ChunkDesc *__restrict__ d, const uint16_t *__restrict__ idx, const uint32_t *__restrict__ first,
             int n)
{
    extern __shared__ uint32_t prefix[];
    __shared__ LinkLds L;
    __shared__ uint32_t counts[kMaxFingers];
    const int j = batch_member(first, n, blockIdx.x);
    const ChunkDesc &c = d[idx[j]];
    draw_pose(prefix, L, counts, c.H, c.pts, c.nrm, c.N, c.poses, c.dom_bits, c.dom_count, nullptr, c.D,
              c.k, c.seed_lo, c.seed_hi, c.request_id, c.pose_offset, c.set_pt, c.set_link, c.pose_valid, c.verdict,
              c.tstar, (int)(blockIdx.x - first[j]));
}

// ---- force-closure LP ---------------------------------------------------------
// Duff et al. (2017) branchless orthonormal basis of unit n.
__device__ inline double duff_a(double nz) { return -1.0 / (copysign(1.0, nz) + nz); }

// the basis from a = duff_a(nz), computed once per normal by the LP
__device__ inline void duff_basis_a(double nx, double ny, double nz, double a, double *x, double *y)
{
    const double sign = copysign(1.0, nz);
    const double b = nx * ny * a;
    x[0] = 1.0 + sign * nx * nx * a;
    x[1] = sign * b;
    x[2] = -sign * nx;
    y[0] = b;
    y[1] = sign + ny * ny * a;
    y[2] = -ny;
}

__device__ inline void duff_basis(double nx, double ny, double nz, double *x, double *y)
{
    const double sign = copysign(1.0, nz);
    const double a = duff_a(nz);
    const double b = nx * ny * a;
    x[0] = 1.0 + sign * nx * nx * a;
    x[1] = sign * b;
    x[2] = -sign * nx;
    y[0] = b;
    y[1] = sign + ny * ny * a;
    y[2] = -ny;
}

constexpr double kLpTol = 1e-12;  // reduced-cost and ratio-tie tolerance
constexpr double kLpPiv = 1e-9;   // smallest admissible pivot element
constexpr int kBlandAfter = 48;   // pivots priced by Dantzig's rule before Bland's
constexpr int kLpChecks = 4;      // residual corrections of one LP at most
// Lanes of a wave at a candidate optimum before they are served together: fewer
// run the refinement and the reloads more often, more let lanes wait (1.2 M LPs
// of 5 contacts: 8 lanes 0.82 ms, 16 0.67, 24 0.63, 32 0.65).
constexpr int kLpBatch = 24;

// contact data of each lane's set, lane-contiguous: cd[6 i + c][tid] (point,
// normal), da[i][tid] the reciprocal of contact i's tangent basis (up to 6
// contacts; beyond that it is recomputed, the LDS would cost occupancy)
template <int KM>
struct LpLds {
    static constexpr bool kDa = KM <= 6;
    float cd[KM * 6][256];
    double da[kDa ? KM : 1][256];
};

template <int KM>
__device__ inline void lp_load(LpLds<KM> &L, int tid, int ci, const float *__restrict__ pts,
                               const float *__restrict__ nrm, int N, int idx)
{
    L.cd[6 * ci + 0][tid] = pts[idx];
    L.cd[6 * ci + 1][tid] = pts[N + idx];
    L.cd[6 * ci + 2][tid] = pts[2 * N + idx];
    L.cd[6 * ci + 3][tid] = nrm[idx];
    L.cd[6 * ci + 4][tid] = nrm[N + idx];
    L.cd[6 * ci + 5][tid] = nrm[2 * N + idx];
    if constexpr (LpLds<KM>::kDa) L.da[ci][tid] = duff_a((double)L.cd[6 * ci + 5][tid]);
}

// ---- force-closure LP, one set per lane -------------------------------------
// Revised simplex with an explicit 7x7 basis inverse per lane.  Reduced
// costs are priced through the duals y = c_B^T B^-1: for wrench column
// (contact i, edge e),
//   y^T a_ie = u_i . d_ie + y_6,  u_i = y_f + (y_m x p_i) / rho,
//   u_i . d_ie = -u_i.n_i + mu (cos_e u_i.x_i + sin_e u_i.y_i).
// With the Duff basis (s = sign n_z, a = -1 / (s + n_z)) and
// h = a (n_x u_x + n_y u_y) - u_z, u.x = u_x + s n_x h and u.y = s u_y + n_y h,
// so a contact's three projections take six multiply-adds and no basis.  For
// the 8-edge cone (MC == 8) the best edge of a contact is the largest of
// |bx|, |by| and (|bx| + |by|) / sqrt 2 (b = (u.x, u.y)); its index is formed
// once, for the winning contact.  The slack pair of row r costs 1 - |y_r|.
// The duals are updated with the pivot row instead of recomputed (c_B^T B^-1
// is 49 multiply-adds), and a pivot is one multiply-add per entry of B^-1:
// row r loses (al_r - [r == lr]) / al_lr times the old pivot row.  Dantzig's
// rule for the first kBlandAfter pivots, then Bland's (lowest entering index,
// ratio ties to the lowest basic variable; no cycling); pivots below kLpPiv
// are not admissible.  Double precision: the verdict is a thresholded decision.
// At a candidate optimum x_B and y are refined against the original columns
// (one residual correction through the current B^-1) and the pricing is
// repeated, so drift in B^-1 or y cannot end the search early or bias t*.
// What bounds it: VALU issue, and the lanes of a wave that wait for the
// wave's slowest LP.  The pricing was half of a pivot's ~1,000 instructions
// (each edge's reduced cost and each basis written out), the row exchange
// with its selects a third.  Measured (65,536 poses x 64 sets of 5 contacts,
// 1.2 M LPs): 2.05 -> 0.63 ms with the lanes refilled as in lp_wave; 4,096 sets
// of 3 contacts 165 -> 55 us; Alg. 2's criteria of a contact step (8,192 poses)
// 1.57 -> 0.63 ms.
template <int KM, int MC>
struct Lp {
    double Bi[7][7], xB[7], y[7];
    int basis[7];
    int k, n, m;
    double mu, inv_rho;

    __device__ inline void basis_of(const LpLds<KM> &L, int tid, int ci, double &px, double &py, double &pz,
                                    double &nx, double &ny, double &nz, double &a) const
    {
        px = L.cd[6 * ci + 0][tid];
        py = L.cd[6 * ci + 1][tid];
        pz = L.cd[6 * ci + 2][tid];
        nx = L.cd[6 * ci + 3][tid];
        ny = L.cd[6 * ci + 4][tid];
        nz = L.cd[6 * ci + 5][tid];
        if constexpr (LpLds<KM>::kDa) a = L.da[ci][tid]; else a = duff_a(nz);
    }

    // original column j of [W^T -I I; 1 0 0]
    __device__ inline void column(const LpLds<KM> &L, int tid, const LpConst &cs, int j, double *a) const
    {
        if (j < n) {
            const int mm = MC > 0 ? MC : m;  // a constant divisor for the 8-edge kernels
            const int ci = j / mm, e = j - ci * mm;
            double px, py, pz, nx, ny, nz, ia, x[3], t[3];
            basis_of(L, tid, ci, px, py, pz, nx, ny, nz, ia);
            duff_basis_a(nx, ny, nz, ia, x, t);
            const double c = mu * cs.ce[e], s = mu * cs.se[e];
            const double dx = fma(s, t[0], fma(c, x[0], -nx));
            const double dy = fma(s, t[1], fma(c, x[1], -ny));
            const double dz = fma(s, t[2], fma(c, x[2], -nz));
            a[0] = dx;
            a[1] = dy;
            a[2] = dz;
            a[3] = (py * dz - pz * dy) * inv_rho;
            a[4] = (pz * dx - px * dz) * inv_rho;
            a[5] = (px * dy - py * dx) * inv_rho;
            a[6] = 1.0;
        } else {
            const int r0 = j < n + 6 ? j - n : j - n - 6;
            const double v = j < n + 6 ? -1.0 : 1.0;
#pragma unroll
            for (int r = 0; r < 6; ++r) a[r] = r == r0 ? v : 0.0;
            a[6] = 0.0;
        }
    }

    // initial basis: g_0 on the normalisation row, s-_r (w0_r <= 0) or s+_r
    __device__ inline void cold(const LpLds<KM> &L, int tid, const LpConst &cs)
    {
        double w0[7];
        column(L, tid, cs, 0, w0);
#pragma unroll
        for (int r = 0; r < 7; ++r)
#pragma unroll
            for (int c = 0; c < 7; ++c) Bi[r][c] = 0.0;
        y[6] = 0.0;
#pragma unroll
        for (int r = 0; r < 6; ++r) {
            const double sg = w0[r] <= 0.0 ? 1.0 : -1.0;
            basis[r] = w0[r] <= 0.0 ? n + 6 + r : n + r;
            Bi[r][r] = sg;
            Bi[r][6] = -sg * w0[r];
            xB[r] = -sg * w0[r];
            y[r] = sg;
            y[6] += xB[r];
        }
        Bi[6][6] = 1.0;
        basis[6] = 0;
        xB[6] = 1.0;
    }

    // entering column, -1 when no reduced cost is below -kLpTol; d: its reduced cost
    __device__ inline int price(const LpLds<KM> &L, int tid, const LpConst &cs, bool bland, double &d) const
    {
        const double m0 = y[3] * inv_rho, m1 = y[4] * inv_rho, m2 = y[5] * inv_rho;
        int e = -1;
        double best = -kLpTol;
        auto project = [&](int i, double &an, double &bx, double &by) {
            double px, py, pz, nx, ny, nz, a;
            basis_of(L, tid, i, px, py, pz, nx, ny, nz, a);
            // u = y_f + (y_m x p) / rho
            const double ux = fma(m1, pz, fma(-m2, py, y[0]));
            const double uy = fma(m2, px, fma(-m0, pz, y[1]));
            const double uz = fma(m0, py, fma(-m1, px, y[2]));
            const double t = fma(nx, ux, ny * uy), h = fma(a, t, -uz), sg = copysign(1.0, nz);
            an = fma(nz, uz, t);
            bx = fma(sg * nx, h, ux);
            by = fma(ny, h, sg * uy);
        };
        if (MC == 8 && !bland) {
            double sbx = 0.0, sby = 0.0;
            int ci = -1;
            for (int i = 0; i < k; ++i) {
                double an, bx, by;
                project(i, an, bx, by);
                const double ax = fabs(bx), ay = fabs(by);
                const double r = fmax(fmax(ax, ay), (ax + ay) * M_SQRT1_2);
                const double di = fma(-mu, r, an) - y[6];
                if (di < best) {
                    best = di;
                    ci = i;
                    sbx = bx;
                    sby = by;
                }
            }
            if (ci >= 0) {
                const double ax = fabs(sbx), ay = fabs(sby), dg = (ax + ay) * M_SQRT1_2;
                const bool xn = sbx < 0.0, yn = sby < 0.0;
                const int diag = yn ? (xn ? 5 : 7) : (xn ? 3 : 1), ex = xn ? 4 : 0, ey = yn ? 6 : 2;
                e = ci * 8 + (dg > fmax(ax, ay) ? diag : (ax >= ay ? ex : ey));
            }
        } else {
            for (int i = 0; i < k && !(bland && e >= 0); ++i) {
                double an, bx, by;
                project(i, an, bx, by);
                for (int ee = 0; ee < m; ++ee) {
                    const double di = fma(-mu, fma(cs.ce[ee], bx, cs.se[ee] * by), an) - y[6];
                    if (di < best) {
                        best = di;
                        e = i * m + ee;
                        if (bland) break;
                    }
                }
            }
        }
        if (bland) {
            for (int r = 0; r < 12 && e < 0; ++r) {
                double v = 0.0;
#pragma unroll
                for (int q = 0; q < 6; ++q)
                    if (q == r % 6) v = r < 6 ? 1.0 + y[q] : 1.0 - y[q];
                if (v < best) {
                    best = v;
                    e = n + r;
                }
            }
        } else {
#pragma unroll
            for (int r = 0; r < 6; ++r)
                if (1.0 - fabs(y[r]) < best) {
                    best = 1.0 - fabs(y[r]);
                    e = y[r] < 0.0 ? n + r : n + 6 + r;
                }
        }
        d = best;
        return e;
    }

    // al = B^-1 a
    __device__ inline void solve(const double *a, double *al) const
    {
#pragma unroll
        for (int r = 0; r < 7; ++r) {
            double s = 0.0;
#pragma unroll
            for (int c = 0; c < 7; ++c) s = fma(Bi[r][c], a[c], s);
            al[r] = s;
        }
    }

    // Ratio test min x_B[r] / al[r] without divisions: the current best is
    // kept as the fraction bx / ba (ba > 0) and ratios are compared by
    // cross-multiplication; the tie band is kLpTol (1 + |best|).
    __device__ inline int ratio(const double *al) const
    {
        int lr = -1, bb = 0;
        double bx = 0.0, ba = 1.0;
#pragma unroll
        for (int r = 0; r < 7; ++r) {
            if (al[r] > kLpPiv) {
                const double lhs = xB[r] * ba, rhs = bx * al[r];
                const double band = kLpTol * (ba + fabs(bx)) * al[r];
                if (lr < 0 || lhs < rhs - band || (fabs(lhs - rhs) <= band && basis[r] < bb)) {
                    lr = r;
                    bx = xB[r];
                    ba = al[r];
                    bb = basis[r];
                }
            }
        }
        return lr;
    }

    // replace the basic variable of row lr by column e (al = B^-1 a_e, d its reduced cost)
    __device__ inline void pivot(int lr, const double *al, int e, double d)
    {
        double oh[7], pv = 0.0, px = 0.0, prow[7];
#pragma unroll
        for (int r = 0; r < 7; ++r) {
            oh[r] = r == lr ? 1.0 : 0.0;
            pv = fma(oh[r], al[r], pv);
            px = fma(oh[r], xB[r], px);
        }
#pragma unroll
        for (int c = 0; c < 7; ++c) {
            prow[c] = oh[0] * Bi[0][c];
#pragma unroll
            for (int r = 1; r < 7; ++r) prow[c] = fma(oh[r], Bi[r][c], prow[c]);
        }
        double inv = __builtin_amdgcn_rcp(pv);
        inv = fma(fma(-pv, inv, 1.0), inv, inv);
        inv = fma(fma(-pv, inv, 1.0), inv, inv);
        const double dy = d * inv;
#pragma unroll
        for (int c = 0; c < 7; ++c) y[c] = fma(dy, prow[c], y[c]);
#pragma unroll
        for (int r = 0; r < 7; ++r) {
            const double f = (oh[r] - al[r]) * inv;
            xB[r] = fma(f, px, xB[r]);
            basis[r] = r == lr ? e : basis[r];
#pragma unroll
            for (int c = 0; c < 7; ++c) Bi[r][c] = fma(f, prow[c], Bi[r][c]);
        }
    }

    __device__ inline double cost(int j) const { return j >= n ? 1.0 : 0.0; }

    // residual corrections of x_B (B x = e_6) and y (B^T y = c_B); a rolled loop,
    // so that one column's registers are live at a time (unrolled it spills 68)
    __device__ inline void refine(const LpLds<KM> &L, int tid, const LpConst &cs)
    {
        double rx[7] = {0, 0, 0, 0, 0, 0, 1.0}, ry[7];
#pragma unroll 1
        for (int q = 0; q < 7; ++q) {
            int bq = basis[0];
            double xq = xB[0];
#pragma unroll
            for (int r = 1; r < 7; ++r) {
                bq = r == q ? basis[r] : bq;
                xq = r == q ? xB[r] : xq;
            }
            double a[7];
            column(L, tid, cs, bq, a);
            double res = cost(bq);
#pragma unroll
            for (int r = 0; r < 7; ++r) {
                rx[r] = fma(-a[r], xq, rx[r]);
                res = fma(-a[r], y[r], res);
            }
#pragma unroll
            for (int r = 0; r < 7; ++r) ry[r] = r == q ? res : ry[r];
        }
#pragma unroll
        for (int r = 0; r < 7; ++r) {
            double s = 0.0;
#pragma unroll
            for (int c = 0; c < 7; ++c) s = fma(Bi[r][c], rx[c], s);
            xB[r] += s;
        }
#pragma unroll
        for (int c = 0; c < 7; ++c) {
            double s = 0.0;
#pragma unroll
            for (int r = 0; r < 7; ++r) s = fma(ry[r], Bi[r][c], s);
            y[c] += s;
        }
    }

    __device__ inline bool basic(int j) const
    {
        bool in = false;
#pragma unroll
        for (int r = 0; r < 7; ++r) in |= basis[r] == j;
        return in;
    }

    __device__ inline double tstar() const
    {
        double ts = 0.0;
#pragma unroll
        for (int r = 0; r < 7; ++r)
            if (basis[r] >= n) ts += xB[r];
        return ts;
    }
};

// The LPs of a wave: lanes take LPs one after another instead of waiting for
// the slowest of 64.  fetch(tid, t): load LP t of the wave's share into the
// lane's column of L and set P.k, P.n (false: no LP, already written); done(t, ts,
// status, P): write a finished one.  status 0 = optimal, 1 = pivot cap,
// 2 = unbounded ratio test (not expected).  A lane at a candidate optimum waits
// until kLpBatch lanes of its wave are (or none is running); those are then
// refined, written and reloaded together, because that part (about two pivots'
// instructions, and dependent loads) would otherwise run for a lane or two at
// nearly every pivot.  Warm start (the "free lunch" of Sec. 5.4): warm(t, r) is
// column id r of the optimal basis of a neighbouring problem -- the same column
// ids, one contact's columns rebuilt from its new point -- or -1 at r = 0 for
// none.  The seven columns are brought into the cold basis one per step, each
// by a primal pivot with the usual ratio test (so the basis stays feasible; a
// column without an admissible pivot is left out); the simplex continues from
// there, near the optimum when the problems are close.  t* does not depend on
// the start.
template <int KM, int MC, bool WARM, class Fetch, class Warm, class Done>
__device__ __forceinline__ void lp_wave(LpLds<KM> &L, int64_t next, int64_t end, int m, double mu, double rho,
                                        int max_pivots, const LpConst &cs, Fetch fetch, Warm warm, Done done)
{
    const int tid = threadIdx.x, lane = tid & 63;
    enum { kIdle, kRun, kStop };
    Lp<KM, MC> P;
    P.m = m;
    P.mu = mu;
    P.inv_rho = 1.0 / rho;
    P.k = P.n = 0;
    int st = kIdle, status = 0, piv = 0, checks = 0, wi = 7;
    int64_t t = 0;
    for (;;) {
        const unsigned long long running = __ballot(st == kRun);
        if (running == 0 || __popcll(__ballot(st == kStop)) >= kLpBatch) {
            if (st == kStop) {
                bool fin = true;
                if (status == 0 && checks < kLpChecks) {
                    ++checks;
                    P.refine(L, tid, cs);
                    double d;
                    fin = P.price(L, tid, cs, piv >= kBlandAfter, d) < 0;
                }
                if (fin) done(t, P.tstar(), status, P);
                st = fin ? kIdle : kRun;
            }
            const unsigned long long need = __ballot(st == kIdle);
            if (next < end && need) {
                if (st == kIdle) {
                    t = next + __popcll(need & ((1ull << lane) - 1ull));
                    if (t < end && fetch(t, P)) {
                        P.cold(L, tid, cs);
                        piv = checks = status = 0;
                        if constexpr (WARM) wi = warm(t, 0) >= 0 ? 0 : 7;
                        st = kRun;
                    }
                }
                next += __popcll(need);
            }
            if (__ballot(st == kRun) == 0) {
                if (next >= end) break;
                continue;
            }
        }
        if (st == kRun) {
            int e = -1;
            double d = 0.0;
            if constexpr (WARM) {
                while (wi < 7) {
                    const int c = warm(t, wi++);
                    if (!P.basic(c)) {
                        e = c;
                        break;
                    }
                }
            }
            const bool forced = e >= 0;
            if (!forced) {
                e = P.price(L, tid, cs, piv >= kBlandAfter, d);
                if (e < 0) st = kStop;
                if (e >= 0 && piv >= max_pivots) {
                    status = 1;
                    st = kStop;
                }
            }
            if (st == kRun) {
                double a[7], al[7];
                P.column(L, tid, cs, e, a);
                if (WARM && forced) {
                    d = P.cost(e);
#pragma unroll
                    for (int r = 0; r < 7; ++r) d = fma(-a[r], P.y[r], d);
                }
                P.solve(a, al);
                const int lr = P.ratio(al);
                if (lr >= 0) {
                    P.pivot(lr, al, e, d);
                    if (!forced) ++piv;
                } else if (!forced) {
                    status = 2;
                    st = kStop;
                }
            }
        }
    }
}

// one LP per lane, every lane of the caller's own; warm[r][tid]: the column ids
// in (see lp_wave), the final basis out
template <int KM, int MC>
__device__ inline double lp_lane(LpLds<KM> &L, int tid, int k, int m, double mu, double rho, int max_pivots,
                                 const LpConst &cs, int &status, int (*warm)[256])
{
    Lp<KM, MC> P;
    P.k = k;
    P.m = m;
    P.n = k * m;
    P.mu = mu;
    P.inv_rho = 1.0 / rho;
    P.cold(L, tid, cs);
    int piv = 0, checks = 0, wi = warm[0][tid] >= 0 ? 0 : 7;
    status = 0;
    for (;;) {
        int e = -1;
        double d = 0.0;
        while (wi < 7 && e < 0) {
            const int c = warm[wi++][tid];
            if (!P.basic(c)) e = c;
        }
        const bool forced = e >= 0;
        if (!forced) {
            e = P.price(L, tid, cs, piv >= kBlandAfter, d);
            if (e < 0) {
                if (checks >= kLpChecks) break;
                ++checks;
                P.refine(L, tid, cs);
                e = P.price(L, tid, cs, piv >= kBlandAfter, d);
                if (e < 0) break;
            }
            if (piv >= max_pivots) {
                status = 1;
                break;
            }
        }
        double a[7], al[7];
        P.column(L, tid, cs, e, a);
        if (forced) {
            d = P.cost(e);
#pragma unroll
            for (int r = 0; r < 7; ++r) d = fma(-a[r], P.y[r], d);
        }
        P.solve(a, al);
        const int lr = P.ratio(al);
        if (lr >= 0) {
            P.pivot(lr, al, e, d);
            if (!forced) ++piv;
        } else if (!forced) {
            status = 2;
            break;
        }
    }
#pragma unroll
    for (int r = 0; r < 7; ++r) warm[r][tid] = P.basis[r];
    return P.tstar();
}

// waves of the nb blocks share n_work LPs in contiguous runs
__device__ inline void lp_share(int64_t bid, int64_t nb, int64_t n_work, int64_t &next, int64_t &end)
{
    const int64_t w = bid * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t per = (n_work + 4 * nb - 1) / (4 * nb);
    next = min(n_work, w * per);
    end = min(n_work, next + per);
}

// block bid of nb blocks: the verdicts of the sets of poses with at least k non-empty domains
template <int KM, int MC = 0>
__device__ __forceinline__ void verdict_sets(LpLds<KM> &L, int64_t bid, int64_t nb, const float *__restrict__ pts,
                                             const float *__restrict__ nrm, int N, const int32_t *__restrict__ set_pt,
                                             const int32_t *__restrict__ palm_pt,
                                             const int32_t *__restrict__ valid_poses,
                                             const int32_t *__restrict__ n_valid_poses, int D, int k, int m, double mu,
                                             double rho, double eps, int max_pivots, const LpConst &cs,
                                             uint8_t *__restrict__ verdict, double *__restrict__ tstar)
{
    const int tid = threadIdx.x;
    int64_t next, end;
    lp_share(bid, nb, (int64_t)(*n_valid_poses) * D, next, end);
    // n_poses * D < 2^31
    auto set_of = [&](int64_t t) {
        const uint32_t q = (uint32_t)t / (uint32_t)D;
        return (int64_t)valid_poses[q] * D + ((uint32_t)t - q * (uint32_t)D);
    };
    auto fetch = [&](int64_t t, Lp<KM, MC> &P) {
        const int64_t sid = set_of(t);
        // a palm contact (Sec. 5.1 static link) is one more, fixed, contact
        const int pc = palm_pt ? palm_pt[valid_poses[(uint32_t)t / (uint32_t)D]] : -1;
        const int kc = pc >= 0 ? k + 1 : k;
        bool valid = true;
        for (int i = 0; i < kc; ++i) {
            const int idx = i < k ? set_pt[sid * k + i] : pc;
            valid &= idx >= 0 && idx < N;
            lp_load(L, tid, i, pts, nrm, N, (idx >= 0 && idx < N) ? idx : 0);
        }
        if (!valid) {
            verdict[sid] = 0;
            tstar[sid] = __builtin_nan("");
        }
        P.k = kc;
        P.n = kc * m;
        return valid;
    };
    lp_wave<KM, MC, false>(
        L, next, end, m, mu, rho, max_pivots, cs, fetch, [](int64_t, int) { return -1; },
        [&](int64_t t, double ts, int status, const Lp<KM, MC> &) {
            const int64_t sid = set_of(t);
            verdict[sid] = (status == 0 && ts <= eps) ? 1 : 0;
            tstar[sid] = status == 0 ? ts : __builtin_nan("");
        });
}

template <int KM, int MC>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_verdict_lane(const float *__restrict__ pts, const float *__restrict__ nrm, int N, const int32_t *__restrict__ set_pt,
               const int32_t *__restrict__ palm_pt, const int32_t *__restrict__ valid_poses,
               const int32_t *__restrict__ n_valid_poses, int D, int k, int m, double mu, double rho, double eps,
               int max_pivots, LpConst cs, uint8_t *__restrict__ verdict, double *__restrict__ tstar)
{
    __shared__ LpLds<KM> L;
    verdict_sets<KM, MC>(L, blockIdx.x, gridDim.x, pts, nrm, N, set_pt, palm_pt, valid_poses, n_valid_poses, D, k, m,
                         mu, rho, eps, max_pivots, cs, verdict, tstar);
}

template <int KM, int MC>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_verdict_batch(const ChunkDesc *__restrict__ d, const uint16_t *__restrict__ idx, const uint32_t *__restrict__ first,
                int n)
{
    __shared__ LpLds<KM> L;
    const int j = batch_member(first, n, blockIdx.x);
    const ChunkDesc &c = d[idx[j]];
    verdict_sets<KM, MC>(L, blockIdx.x - first[j], first[j + 1] - first[j], c.pts, c.nrm, c.N, c.set_pt, nullptr,
                     c.valid_poses, c.n_valid_poses, c.D, c.k, c.m, c.mu, c.rho, c.eps, c.max_pivots, c.cs, c.verdict,
                     c.tstar);
}

// ---- contact-point optimisation (Sec. 5.4, Alg. 2) ---------------------------
// A cell grid over the object's points serves the projection of a candidate onto a
// contact domain (nearest domain point): rows of cells along x, of edge c across a
// row and c / 2 along it; a row's points are contiguous, so a search reads any
// stretch of a row as one range.  c = sigma / 2, at least 1.5 times the mean point
// spacing (some points per cell) and within kGridCells cells (k_grid_setup).
// Distances are FP64, ties go to the lowest point index.
constexpr int kGridMax = 64;
constexpr int kGridCells = (kGridMax + 1) * (kGridMax + 1) * (kGridMax + 1);
constexpr float kGridSpacing = 1.5f;
constexpr int kGridY = 128;  // cells across the rows, at most
constexpr uint32_t kPurposeOpt = 5u;
constexpr double kOptTau = 1e-9;  // candidates within kOptTau of the best criterion value tie

struct GridDev {
    float lo[3];
    float cell, inv_cell;  // across the rows; along them cells are half as long
    float slack;           // (m) what float binning and box tests may be off by, and more
    int dims[3];
    uint32_t used;         // records given to rows so far (k_grid_rows)
};

// start of cell (0, y, z) in the cell arrays: a row has an entry more than cells
__device__ inline int grid_row(const GridDev &g, int y, int z) { return (z * g.dims[1] + y) * (g.dims[0] + 1); }

__global__ void __launch_bounds__(1024)
k_grid_setup(const float *__restrict__ pts, int N, float sigma, GridDev *__restrict__ gd)
{
    __shared__ float red[6][1024];
    float mn[3] = {INFINITY, INFINITY, INFINITY}, mx[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (int i = threadIdx.x; i < N; i += blockDim.x)
        for (int a = 0; a < 3; ++a) {
            mn[a] = fminf(mn[a], pts[a * N + i]);
            mx[a] = fmaxf(mx[a], pts[a * N + i]);
        }
    for (int a = 0; a < 3; ++a) {
        red[a][threadIdx.x] = mn[a];
        red[3 + a][threadIdx.x] = mx[a];
    }
    __syncthreads();
    for (int w = 512; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w)
            for (int a = 0; a < 3; ++a) {
                red[a][threadIdx.x] = fminf(red[a][threadIdx.x], red[a][threadIdx.x + w]);
                red[3 + a][threadIdx.x] = fmaxf(red[3 + a][threadIdx.x], red[3 + a][threadIdx.x + w]);
            }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        float e[3], ext = 0.0f;
        for (int a = 0; a < 3; ++a) {
            e[a] = red[3 + a][0] - red[a][0];
            ext = fmaxf(ext, e[a]);
        }
        const float area = 2.0f * (e[0] * e[1] + e[1] * e[2] + e[2] * e[0]);  // the box's, about the object's
        float c = fmaxf(fmaxf(0.5f * sigma, kGridSpacing * sqrtf(area / (float)N)), fmaxf(ext / (float)kGridY, 1e-4f));
        GridDev g;
        for (int it = 0;; ++it) {
            g.cell = c;
            g.inv_cell = 1.0f / c;
            for (int a = 0; a < 3; ++a) {
                const float n = fminf(e[a] * g.inv_cell * (a == 0 ? 2.0f : 1.0f), (float)(a == 0 ? 2 * kGridY : kGridY));
                g.dims[a] = n > 0.0f ? (int)n + 1 : 1;
            }
            if ((int64_t)(g.dims[0] + 1) * g.dims[1] * g.dims[2] <= kGridCells || it == 64) break;
            c *= 1.25f;
        }
        if ((int64_t)(g.dims[0] + 1) * g.dims[1] * g.dims[2] > kGridCells) g.dims[0] = g.dims[1] = g.dims[2] = 1;
        for (int a = 0; a < 3; ++a) g.lo[a] = red[a][0];
        g.slack = 1e-6f + 4e-7f * ext;
        g.used = 0;
        *gd = g;
    }
}

// the cell array entry of point i
__device__ inline int point_cell(const GridDev &g, const float *pts, int N, int i)
{
    int c[3];
    for (int a = 0; a < 3; ++a) {
        const float u = (pts[a * N + i] - g.lo[a]) * g.inv_cell * (a == 0 ? 2.0f : 1.0f);
        c[a] = min(max((int)floorf(u), 0), g.dims[a] - 1);
    }
    return grid_row(g, c[1], c[2]) + c[0];
}

__global__ void k_fill_u32(uint32_t *__restrict__ a, int64_t n, uint32_t v)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) a[i] = v;
}

__global__ void k_grid_count(const float *__restrict__ pts, int N, const GridDev *__restrict__ gd,
                             uint32_t *__restrict__ cell_count)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < N) atomicAdd(&cell_count[point_cell(*gd, pts, N, i)], 1u);
}

// Wave per row: the starts of its cells' records, and of the end of its last one.
// Rows take their ranges in the order they come by (a search reads whole rows, and
// its result does not depend on the order of the points); one workgroup's scan of
// all cells took 21 us for 11,000, this takes 11 us for 95,000.
__global__ void __launch_bounds__(256)
k_grid_rows(uint32_t *__restrict__ cell_count, GridDev *__restrict__ gd, uint32_t *__restrict__ cell_start)
{
    const int dx = gd->dims[0], rows = gd->dims[1] * gd->dims[2], lane = threadIdx.x & 63;
    const int n_waves = gridDim.x * (blockDim.x >> 6);
    for (int row = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6); row < rows; row += n_waves) {
        const int r0 = row * (dx + 1);
        uint32_t sum = 0;
        for (int x = lane; x < dx; x += 64) sum += cell_count[r0 + x];
        for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
        uint32_t run = 0;
        if (lane == 0) run = sum ? atomicAdd(&gd->used, sum) : 0u;
        run = (uint32_t)__builtin_amdgcn_readfirstlane((int)run);
        for (int x0 = 0; x0 <= dx; x0 += 64) {
            const int x = x0 + lane;
            const uint32_t c = x < dx ? cell_count[r0 + x] : 0u;
            const uint32_t incl = wave_scan_incl(c);
            if (x <= dx) {
                cell_start[r0 + x] = run + incl - c;
                cell_count[r0 + x] = run + incl - c;  // becomes the scatter cursor
            }
            run += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
        }
    }
}

// the points of each cell, contiguous: (x, y, z, point index as bits)
__global__ void k_grid_scatter(const float *__restrict__ pts, int N, const GridDev *__restrict__ gd,
                               uint32_t *__restrict__ cursor, float4 *__restrict__ cell_pts)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < N)
        cell_pts[atomicAdd(&cursor[point_cell(*gd, pts, N, i)], 1u)] =
            make_float4(pts[i], pts[N + i], pts[2 * N + i], __int_as_float(i));
}

__device__ inline bool dom_has(const uint32_t *dom, int i) { return (dom[i >> 5] >> (i & 31)) & 1u; }

__device__ inline double wave_bcast(double v, int l)
{
    const long long b = __double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, l);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), l);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// DPP move of both halves of a double; lanes without a source keep v
template <int C, int RM = 0xf>
__device__ inline double dpp_d(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = (int)(uint32_t)b, hi = (int)(b >> 32);
    const int nlo = __builtin_amdgcn_update_dpp(lo, lo, C, RM, 0xf, false);
    const int nhi = __builtin_amdgcn_update_dpp(hi, hi, C, RM, 0xf, false);
    return __longlong_as_double((long long)(((uint64_t)(uint32_t)nhi << 32) | (uint32_t)nlo));
}

// minimum over the wave, valid in lane 63: quad swaps, row rotations by 4
// and 8, then rows 0+1 and 2+3 and the halves joined by the row broadcasts
__device__ inline double wave_min63(double v)
{
    v = fmin(v, dpp_d<0xB1>(v));        // quad_perm [1, 0, 3, 2]
    v = fmin(v, dpp_d<0x4E>(v));        // quad_perm [2, 3, 0, 1]
    v = fmin(v, dpp_d<0x124>(v));       // row_ror:4
    v = fmin(v, dpp_d<0x128>(v));       // row_ror:8
    v = fmin(v, dpp_d<0x142, 0xA>(v));  // row_bcast:15 into rows 1 and 3
    v = fmin(v, dpp_d<0x143, 0xC>(v));  // row_bcast:31 into rows 2 and 3
    return v;
}

// the minimum of (d2, i) over the lanes with `take` (lexicographic), folded
// into (best, bi); every lane returns the same result
__device__ inline void wave_lexmin(bool take, double d2, int i, double &best, int &bi)
{
    const unsigned long long m = __ballot(take);
    if (!m) return;
    double v;
    int ib;
    if (__popcll(m) == 1) {
        const int l = __builtin_ctzll(m);
        v = wave_bcast(d2, l);
        ib = __builtin_amdgcn_readlane(i, l);
    } else {
        v = wave_bcast(wave_min63(take ? d2 : INFINITY), 63);
        const unsigned long long t = __ballot(take && d2 == v);
        ib = __builtin_amdgcn_readlane(i, __builtin_ctzll(t));
        for (unsigned long long r = t & (t - 1); r; r &= r - 1)  // equal distances: the lowest index
            ib = min(ib, __builtin_amdgcn_readlane(i, __builtin_ctzll(r)));
    }
    if (v < best || (v == best && ib < bi)) {
        best = v;
        bi = ib;
    }
}

// LDS of one wave: what its lanes wrote before is there for all of them after it
__device__ inline void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// the ring of row position q >= 0 (ring R holds 8 R rows), and the row's offset
__device__ inline int row_ring(int q) { return (int)(0.5f * (1.0f + sqrtf((float)(q + 1)))); }

__device__ inline void row_offset(int R, int q, int &dy, int &dz)
{
    const int side = 2 * R, o = q - 4 * R * (R - 1), e = o / side, t = o - e * side;
    dy = e == 0 ? t - R : (e == 1 ? R : (e == 2 ? R - t : -R));
    dz = e == 0 ? -R : (e == 1 ? t - R : (e == 2 ? R : R - t));
}

// A candidate y waiting for its projection: its cell (i) and its place in it (r, in
// cells), the squared distance and index of the best domain point so far.
struct ProjSlot {
    double y[3], best;
    int64_t dom, out;  // its domain's first word; its entry of cands
    int bi, i[3];
    float r[3];
};
constexpr int kProjSets = 4;     // sets whose candidates a wave draws together
constexpr int kProjRows = 1024;  // row positions searched before the whole domain is
constexpr int kProjWindow = 2;   // cells along x to each side of y's in the first two searches

struct ProjLds {
    ProjSlot slot[64];
    int64_t set[kProjSets], pose[kProjSets];  // the drawn sets: rank, pose, chosen fingers
    uint32_t fingers[kProjSets];
    uint8_t cls[64], order[64];  // of the slots: what a search left to do; by that
};

// how far the search has to go, in cells across rows: a point at or below `best`
// lies within it (inflated by the slack and the rounding of the float tests)
__device__ inline float proj_limit(const GridDev &g, double best)
{
    return (sqrtf((float)best) + g.slack) * g.inv_cell * 1.0001f;
}

// distance (cells) from y to the slab of cells at offset o on one axis
__device__ inline float proj_slab(int o, float r) { return o > 0 ? (float)o - r : (o < 0 ? (float)(-o - 1) + r : 0.0f); }

// The records of row (iy + dy, iz + dz) within lim of y and, along x, at cell offsets
// lo .. hi of its own: [q0, q0 + cnt)
__device__ inline void proj_span(const GridDev &g, const uint32_t *__restrict__ cell_start, const ProjSlot &S, int dy,
                                 int dz, float lim, int lo, int hi, uint32_t &q0, uint32_t &cnt)
{
    q0 = cnt = 0;
    const float sy = proj_slab(dy, S.r[1]), sz = proj_slab(dz, S.r[2]), rest = lim * lim - (sy * sy + sz * sz);
    const int y = S.i[1] + dy, z = S.i[2] + dz;
    if (rest < 0.0f || y < 0 || y >= g.dims[1] || z < 0 || z >= g.dims[2]) return;
    const float hx = fminf(2.0f * sqrtf(rest) + 1e-3f, 1048576.0f);  // half width, in cells along x
    const int xa = max(S.i[0] + max((int)floorf(S.r[0] - hx), lo), 0);
    const int xb = min(S.i[0] + min((int)floorf(S.r[0] + hx), hi), g.dims[0] - 1);
    if (xa > xb) return;
    const uint32_t *row = cell_start + grid_row(g, y, z);
    q0 = row[xa];
    cnt = row[xb + 1] - q0;
}

// the better of (d, i) and its partner's under DPP control C
template <int C>
__device__ inline void dpp_lexmin(double &d, int &i)
{
    const double od = dpp_d<C>(d);
    const int oi = __builtin_amdgcn_update_dpp(i, i, C, 0xf, 0xf, false);
    const bool less = ((int)(od < d) | ((int)(od == d) & (int)(oi < i))) != 0;  // no branches
    d = less ? od : d;
    i = less ? oi : i;
}

// The search of one candidate by a group of 8 lanes.  Each lane keeps the best
// (distance, index) of the points it read; equal in the group's lanes at first.
struct ProjGroup {
    double yx, yy, yz, lb;
    int li, gl, g0;

    __device__ inline ProjGroup(const ProjSlot &S, int lane)
        : yx(S.y[0]), yy(S.y[1]), yz(S.y[2]), lb(S.best), li(S.bi), gl(lane & 7), g0(lane & 56)
    {
    }
    __device__ inline void scan(const float4 *__restrict__ cell_pts, const uint32_t *__restrict__ dom, uint32_t q,
                                uint32_t end)
    {
        for (q += gl; q < end; q += 8) {
            const float4 v = cell_pts[q];
            const int i = __float_as_int(v.w);
            const double ex = (double)v.x - yx, ey = (double)v.y - yy, ez = (double)v.z - yz;
            const double d2 = ex * ex + ey * ey + ez * ez;
            if (((int)(d2 < lb) | ((int)(d2 == lb) & (int)(i < li))) != 0) {
                const bool in = dom_has(dom, i);
                lb = in ? d2 : lb;
                li = in ? i : li;
            }
        }
    }
    // each lane's span, one after another
    __device__ inline void scan_spans(const float4 *__restrict__ cell_pts, const uint32_t *__restrict__ dom,
                                      uint32_t q0, uint32_t cnt)
    {
        for (uint32_t rows = (uint32_t)(__ballot(cnt > 0) >> g0) & 0xffu; rows; rows &= rows - 1) {
            const int l = g0 + __builtin_ctz(rows);
            const uint32_t q = (uint32_t)__shfl((int)q0, l, 64);
            scan(cell_pts, dom, q, q + (uint32_t)__shfl((int)cnt, l, 64));
        }
    }
    __device__ inline void best()
    {
        dpp_lexmin<0xB1>(lb, li);
        dpp_lexmin<0x4E>(lb, li);
        dpp_lexmin<0x141>(lb, li);
    }
};

// distance (cells) from y to the rows around its own
__device__ inline float proj_edge(const ProjSlot &S)
{
    return fminf(fminf(S.r[1], 1.0f - S.r[1]), fminf(S.r[2], 1.0f - S.r[2]));
}

// y's own row and the 8 around it, kProjWindow cells along x to each side, hold
// every point within lim
__device__ inline bool proj_inside(const ProjSlot &S, float lim)
{
    return lim < 1.0f + proj_edge(S) && 2.0f * lim <= (float)kProjWindow + fminf(S.r[0], 1.0f - S.r[0]) - 1e-3f;
}

// What the groups' searches leave, by the whole wave, a lane per stretch of cells:
// first the 18 ends of y's own row and the 8 around it, then the rows of ring 2 and
// on, 64 stretches per pass.  Their points are spread over the lanes, 64 per step, in
// the order of the lanes' running counts; a stretch that a better point has put out
// of reach since is left out.  Past kProjRows every domain point.
__device__ inline int project_wave(const GridDev &g, const uint32_t *__restrict__ cell_start,
                                   const float4 *__restrict__ cell_pts, const float *__restrict__ pts, int N,
                                   const uint32_t *__restrict__ dom, const ProjSlot &S, int lane)
{
    const double yx = S.y[0], yy = S.y[1], yz = S.y[2];
    double best = S.best;
    int bi = S.bi;
    const float edge = proj_edge(S);
    float lim = proj_limit(g, best);
    for (int p0 = 0; p0 < kProjRows; p0 += 64) {
        if (p0 > 0 && lim < (float)(row_ring(p0 - 10) - 1) + edge) return bi;  // no closer point from here on
        const int p = p0 + lane, q = p < 18 ? (p >> 1) - 1 : p - 10;
        int dy = 0, dz = 0, lo = -(1 << 20), hi = 1 << 20;
        if (q >= 0) row_offset(row_ring(q), q, dy, dz);
        float gap = 0.0f;  // along x
        if (p < 18) {
            if (p & 1) {
                lo = kProjWindow + 1;
                gap = 0.5f * ((float)lo - S.r[0]);
            } else {
                hi = -kProjWindow - 1;
                gap = 0.5f * ((float)kProjWindow + S.r[0]);
            }
        }
        const float sy = proj_slab(dy, S.r[1]), sz = proj_slab(dz, S.r[2]);
        const float near2 = sy * sy + sz * sz + gap * gap;
        uint32_t q0, cnt;
        proj_span(g, cell_start, S, dy, dz, lim, lo, hi, q0, cnt);
        // lane l's points are [ex, ex + cnt) of the pass's running count
        const uint32_t incl = wave_scan_incl(cnt), ex = incl - cnt;
        const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
        for (uint32_t b0 = 0; b0 < total; b0 += 64) {
            const uint32_t f = b0 + (uint32_t)lane;
            // the record of point f: the stretches that meet this step, in lane order
            uint32_t rec = 0, end = 0;
            for (unsigned long long km = __ballot(cnt > 0 && ex < b0 + 64u && incl > b0 && near2 <= lim * lim); km;
                 km &= km - 1) {
                const int l = __builtin_ctzll(km);
                const uint32_t lex = (uint32_t)__builtin_amdgcn_readlane((int)ex, l);
                const uint32_t lq0 = (uint32_t)__builtin_amdgcn_readlane((int)q0, l);
                if (f >= lex) {
                    rec = lq0 + (f - lex);
                    end = lq0 + (uint32_t)__builtin_amdgcn_readlane((int)cnt, l);
                }
            }
            bool take = false;
            double d2 = INFINITY;
            int i = INT_MAX;
            if (rec < end) {
                const float4 v = cell_pts[rec];
                i = __float_as_int(v.w);
                const double ex3 = (double)v.x - yx, ey3 = (double)v.y - yy, ez3 = (double)v.z - yz;
                d2 = ex3 * ex3 + ey3 * ey3 + ez3 * ez3;
                take = (d2 < best || (d2 == best && i < bi)) && dom_has(dom, i);
            }
            const double old = best;
            wave_lexmin(take, d2, i, best, bi);
            if (best != old) lim = proj_limit(g, best);
        }
    }
    if (lim < (float)(row_ring(kProjRows - 11) - 1) + edge) return bi;
    const int NW = (N + 31) >> 5;
    double lb = INFINITY;
    int li = INT_MAX;
    for (int w = lane; w < NW; w += 64) {
        uint32_t x = dom[w];
        while (x) {
            const int b = __ffs(x) - 1;
            x &= x - 1u;
            const int i = w * 32 + b;
            const double ex3 = (double)pts[i] - yx, ey3 = (double)pts[N + i] - yy, ez3 = (double)pts[2 * N + i] - yz;
            const double d2 = ex3 * ex3 + ey3 * ey3 + ez3 * ez3;
            if (d2 < lb || (d2 == lb && i < li)) {
                lb = d2;
                li = i;
            }
        }
    }
    wave_lexmin(li != INT_MAX, lb, li, best, bi);
    return bi;
}

// Alg. 2, the candidates of one round (Sec. 5.4): one candidate per
// (set, contact i, candidate j).  Contact i's candidates are drawn around its
// point at the start of the round (contact i moves only at its own step), so
// a round's projections are independent of its criterion evaluations and run
// here, before them: y = p_i + dx x_i + dy y_i with (dx, dy) = sigma *
// Box-Muller of Philox block (g + pose_offset, d, 5 | step << 8, request_id),
// step = (round k + i) n_inner + j, and cand = the nearest point of contact
// i's domain (incumbent p_i).  cands[((t k + i) n_inner + j)], t = the set's
// rank among the sets of valid poses; -1 for sets not drawn.  A wave takes
// kProjSets sets (few: 16 made 8,800 waves of 640 candidates, one and a half times
// what the chip holds, and 1.5 times the time), and where those would not fill the
// chip (fill waves) fewer, down to 8 candidates of one set (512 sets of 80 candidates
// each: 845 us with four sets per wave, 86 so, 301 with a wave per candidate).  It
// draws the candidates of the drawn ones 64 at a time, a lane each; a group of 8
// lanes then projects each: its own row kProjWindow cells to each side, then the 8
// rows around it so, first those candidates that surely end there, so that a group
// waits for groups with about its own work.  The few with nothing so near go on as a
// whole wave each (8 lanes took 3.4 ms for them, the wave 1.3).
// What bounds it: load latency and VALU issue about equally.  A wave per candidate
// with 4 mm cells of 34 points read 200 points and issued 515 instructions for each;
// with groups and cells of 2 mm x 1 mm it issues 212 (8,192 poses x 64 draws, 65,536
// points, 5.7 M candidates of drawn sets: 5.3 -> 2.9 ms).  Seven waves per SIMD: six
// are 2 % slower, eight 18 %; at seven 33 registers of the set-up live in scratch memory.
__global__ void __launch_bounds__(256, 7)
k_opt_project(const float *__restrict__ pts, const float *__restrict__ nrm, int N,
              const int32_t *__restrict__ valid_poses, const int32_t *__restrict__ n_valid_poses,
              const uint32_t *__restrict__ dom_bits, const uint32_t *__restrict__ dom_count,
              const int32_t *__restrict__ palm_pt, int F, int D, int k, int round, int n_inner, double sigma,
              uint32_t seed_lo, uint32_t seed_hi, uint32_t request_id, int64_t pose_offset,
              const GridDev *__restrict__ gdp, const uint32_t *__restrict__ cell_start,
              const float4 *__restrict__ cell_pts, const int32_t *__restrict__ set_pt, int fill,
              int32_t *__restrict__ cands)
{
    __shared__ ProjLds lds[4];
    ProjLds &L = lds[threadIdx.x >> 6];
    const GridDev g = *gdp;
    const int NW = (N + 31) >> 5;
    const int lane = threadIdx.x & 63, per_set = k * n_inner;
    const int64_t n_sets = (int64_t)(*n_valid_poses) * D;
    // a wave's unit: spw sets, or a part of one set's candidates
    const uint32_t n_waves = gridDim.x * 4, share = min(n_waves, (uint32_t)fill), sets = (uint32_t)n_sets;  // < 2^31
    const uint32_t spw = sets / kProjSets >= share ? (uint32_t)kProjSets : max(1u, (sets + share - 1) / share);
    const uint32_t parts = spw > 1 || sets == 0 ? 1u : min((uint32_t)(per_set + 7) >> 3, share / sets);
    const int part_n = (int)((per_set + parts - 1) / parts + 7) & ~7;  // candidates of a part
    const uint32_t units = (sets + spw - 1) / spw * parts;
    for (uint32_t u = (uint32_t)__builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + (threadIdx.x >> 6))); u < units;
         u += n_waves) {
        const uint32_t q = parts > 1 ? u / parts : u;
        const int part = (int)(u - q * parts);
        const int64_t t0 = (int64_t)q * spw;
        const int64_t t = t0 + lane;
        bool drawn = false;
        if (lane < (int)spw && t < n_sets) {
            const int64_t pg = valid_poses[t / D];
            const int d = (int)(t % D);
            const int pc = palm_pt ? palm_pt[pg] : -1;
            drawn = pc < N;
            for (int q = 0; q < k; ++q) {
                const int sp = set_pt[(pg * D + d) * k + q];
                drawn &= sp >= 0 && sp < N;
            }
            if (drawn) {
                const uint32_t fm = choose_fingers(eligible_fingers(dom_count, pg, F), k,
                                                   (uint32_t)(pose_offset + pg), d, request_id, seed_lo, seed_hi);
                drawn = fm != 0;
                L.set[lane] = t;
                L.pose[lane] = pg;
                L.fingers[lane] = fm;
            }
        }
        wave_lds_sync();
        const uint32_t dm = (uint32_t)__ballot(drawn);
        const int n_here = (int)min((int64_t)spw, n_sets - t0);
        if (__popc(dm) < n_here)
            for (int e = lane + 64 * part; e < n_here * per_set; e += 64 * (int)parts)
                if (!((dm >> (e / per_set)) & 1u)) cands[t0 * per_set + e] = -1;
        const int total = __popc(dm) * per_set, end = parts > 1 ? min(total, (part + 1) * part_n) : total;
        for (int c0 = part * part_n; c0 < end; c0 += 64) {
            const int nb = min(64, end - c0);
            if (lane < nb) {
                const int c = c0 + lane, nth = c / per_set, rem = c - nth * per_set, i = rem / n_inner;
                const int at = select_in_word(dm, (uint32_t)nth);
                const int64_t pg = L.pose[at], set = L.set[at];
                const int d = (int)(set % D);
                const int inc = set_pt[(pg * D + d) * k + i];
                ProjSlot S;
                const double px = pts[inc], py = pts[N + inc], pz = pts[2 * N + inc];
                double tx[3], ty[3];
                duff_basis(nrm[inc], nrm[N + inc], nrm[2 * N + inc], tx, ty);
                uint32_t w[4];
                philox4x32_10((uint32_t)(pose_offset + pg), (uint32_t)d,
                              kPurposeOpt | ((uint32_t)(round * per_set + rem) << 8), request_id, seed_lo, seed_hi, w);
                const double u1 = ((double)(w[0] >> 8) + 1.0) * (1.0 / 16777216.0);
                const double u2 = (double)(w[1] >> 8) * (1.0 / 16777216.0);
                const double rr = sqrt(-2.0 * log(u1));
                const double dx = sigma * rr * cos(2.0 * M_PI * u2), dy = sigma * rr * sin(2.0 * M_PI * u2);
                S.y[0] = px + dx * tx[0] + dy * ty[0];
                S.y[1] = py + dx * tx[1] + dy * ty[1];
                S.y[2] = pz + dx * tx[2] + dy * ty[2];
                const double ex = px - S.y[0], ey = py - S.y[1], ez = pz - S.y[2];
                S.best = ex * ex + ey * ey + ez * ez;
                S.bi = inc;
                S.dom = (pg * F + select_in_word(L.fingers[at], (uint32_t)i)) * NW;  // contact i's finger
                S.out = set * per_set + rem;
                for (int a = 0; a < 3; ++a) {
                    const double u = (S.y[a] - g.lo[a]) * (double)g.inv_cell * (a == 0 ? 2.0 : 1.0);
                    const double v = fmin(fmax(floor(u), -1048576.0), 1048576.0);  // far outside: any cell that is
                    S.i[a] = (int)v;
                    S.r[a] = (float)(u - v);
                }
                L.slot[lane] = S;
            }
            wave_lds_sync();
            // own row; 0: ended, 1: ends with the rows around it, 2: maybe further
            for (int b = 0; b < nb; b += 8) {
                const int sl = b + (lane >> 3);
                if (sl >= nb) continue;
                ProjSlot &S = L.slot[sl];
                ProjGroup G(S, lane);
                uint32_t q0, cnt;
                proj_span(g, cell_start, S, 0, 0, proj_limit(g, G.lb), -kProjWindow, kProjWindow, q0, cnt);
                G.scan(cell_pts, dom_bits + S.dom, q0, q0 + cnt);
                G.best();
                const float lim = proj_limit(g, G.lb);
                const int cls = !proj_inside(S, lim) ? 2 : lim < proj_edge(S) ? 0 : 1;
                if (G.gl == 0) {
                    S.best = G.lb;
                    S.bi = G.li;
                    L.cls[sl] = (uint8_t)cls;
                    if (cls == 0) cands[S.out] = G.li;
                }
            }
            wave_lds_sync();
            const int cls = lane < nb ? L.cls[lane] : 0;
            const unsigned long long m1 = __ballot(cls == 1), m2 = __ballot(cls == 2), below = (1ull << lane) - 1ull;
            const int n1 = __popcll(m1), n2 = __popcll(m2);
            if (cls == 1) L.order[__popcll(m1 & below)] = (uint8_t)lane;
            if (cls == 2) L.order[n1 + __popcll(m2 & below)] = (uint8_t)lane;
            wave_lds_sync();
            for (int b0 = 0; b0 < n1 + n2; b0 += 8) {
                const int b = b0 + (lane >> 3);
                bool open = false;
                if (b < n1 + n2) {
                    ProjSlot &S = L.slot[L.order[b]];
                    ProjGroup G(S, lane);
                    const int t = G.gl & 1, e = G.gl >> 1;  // row_offset(1, gl)
                    const int dy = e == 0 ? t - 1 : (e == 1 ? 1 : (e == 2 ? 1 - t : -1));
                    const int dz = e == 0 ? -1 : (e == 1 ? t - 1 : (e == 2 ? 1 : 1 - t));
                    uint32_t q0, cnt;
                    proj_span(g, cell_start, S, dy, dz, proj_limit(g, G.lb), -kProjWindow, kProjWindow, q0, cnt);
                    G.scan_spans(cell_pts, dom_bits + S.dom, q0, cnt);
                    G.best();
                    open = b >= n1 && !proj_inside(S, proj_limit(g, G.lb));
                    if (G.gl == 0) {
                        S.best = G.lb;
                        S.bi = G.li;
                        if (!open) cands[S.out] = G.li;
                    }
                }
                wave_lds_sync();
                for (unsigned long long todo = __ballot(open && (lane & 7) == 0); todo; todo &= todo - 1) {
                    const ProjSlot &S = L.slot[L.order[b0 + (__builtin_ctzll(todo) >> 3)]];
                    const int r = project_wave(g, cell_start, cell_pts, pts, N, dom_bits + S.dom, S, lane);
                    if (lane == 0) cands[S.out] = r;
                }
            }
            wave_lds_sync();
        }
        wave_lds_sync();
    }
}

// Alg. 2, the criterion side of one round: a group of GS = pow2 >= n_inner
// lanes per set (lane = candidate), grid-stride over the sets of poses with
// non-empty domains.  Contacts i = 0..k-1 in turn: each lane evaluates the LP
// of the set with contact i at its candidate (cands of k_opt_project), the
// group takes the minimum by xor-shuffles and the first lane within kOptTau
// of it by one ballot; contact i moves there.  The set's points are written
// back after the round; tstar (the last step's J) and, after the last round,
// the verdict.
template <int KM, int GS, int MC>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_optimize(const float *__restrict__ pts, const float *__restrict__ nrm, int N, const int32_t *__restrict__ valid_poses,
           const int32_t *__restrict__ n_valid_poses, const uint32_t *__restrict__ dom_count,
           const int32_t *__restrict__ palm_pt, int F, int D, int k, int m, double mu, double rho, double eps,
           int max_pivots, LpConst cs, int n_inner, bool last, uint32_t seed_lo, uint32_t seed_hi,
           uint32_t request_id, int64_t pose_offset, const int32_t *__restrict__ cands, int32_t *__restrict__ set_pt,
           uint8_t *__restrict__ verdict, double *__restrict__ tstar)
{
    __shared__ LpLds<KM> L;
    __shared__ int cur[KM][256];  // the set's current point indices (every lane of a group holds them)
    __shared__ int wbs[7][256];   // per lane: the warm basis of its LP in, its final basis out
    __shared__ int cbs[7][256];   // per lane: the current set's optimal basis (the last pick's)
    const int tid = threadIdx.x, lane = tid & 63, j = tid % GS, gbase = lane - j;
    const int wbase = tid - lane;  // first thread of this wave
    const int64_t n_work = (int64_t)(*n_valid_poses) * D;
    const int64_t groups = ((int64_t)gridDim.x * blockDim.x) / GS;
    auto load = [&](int ci, int idx) { lp_load(L, tid, ci, pts, nrm, N, idx); };
    for (int64_t t = ((int64_t)blockIdx.x * blockDim.x + tid) / GS; t < n_work; t += groups) {
        const int64_t pg = valid_poses[t / D];
        const int d = (int)(t % D);
        const int64_t sid = pg * D + d;
        int32_t *sp = set_pt + sid * k;
        const uint32_t fm = choose_fingers(eligible_fingers(dom_count, pg, F), k, (uint32_t)(pose_offset + pg), d,
                                           request_id, seed_lo, seed_hi);
        const int pc = palm_pt ? palm_pt[pg] : -1;  // fixed palm contact (-1: none)
        const int kc = pc >= 0 ? k + 1 : k;
        bool drawn = fm != 0 && pc < N;
        for (int i = 0; i < k; ++i) drawn &= sp[i] >= 0 && sp[i] < N;
        if (!drawn) {  // not a drawn set (inconsistent domain sizes): no criterion
            if (j == 0) {
                verdict[sid] = 0;
                tstar[sid] = __builtin_nan("");
            }
            continue;  // uniform over the group
        }
        for (int i = 0; i < k; ++i) {
            cur[i][tid] = sp[i];
            load(i, sp[i]);
        }
        if (pc >= 0) load(k, pc);
        double J = INFINITY;
        // optimal basis of the current set (the last pick's), the warm start of
        // the next contact's candidates; none before the round's first pick
        cbs[0][tid] = -1;
        for (int i = 0; i < k; ++i) {
            int cand = -1;
            double Jc = INFINITY;
#pragma unroll
            for (int r = 0; r < 7; ++r) wbs[r][tid] = cbs[r][tid];
            if (j < n_inner) {
                cand = cands[(t * k + i) * n_inner + j];
                if (cand >= 0) {  // always, for a drawn set (its domains are non-empty)
                    load(i, cand);
                    int st = 0;
                    Jc = lp_lane<KM, MC>(L, tid, kc, m, mu, rho, max_pivots, cs, st, wbs);
                    if (st != 0) Jc = INFINITY;
                }
            }
            double mn = Jc;
            for (int off = GS >> 1; off > 0; off >>= 1) mn = fmin(mn, __shfl_xor(mn, off, GS));
            const unsigned long long ok = __ballot(Jc <= mn + kOptTau);
            const int js = __ffsll((long long)((ok >> gbase) & ((GS == 64) ? ~0ull : ((1ull << GS) - 1)))) - 1;
            const int pick = __shfl(cand, gbase + js, 64);
            const double Jp = __shfl(Jc, gbase + js, 64);
            if (pick >= 0) {
                J = Jp;
                cur[i][tid] = pick;
                // the picked lane's final basis (written by that lane of this wave)
                if (!isinf(Jp)) {
#pragma unroll
                    for (int r = 0; r < 7; ++r) cbs[r][tid] = wbs[r][wbase + gbase + js];
                }
            }
            load(i, cur[i][tid]);
        }
        if (j == 0) {
            for (int i = 0; i < k; ++i) sp[i] = cur[i][tid];
            tstar[sid] = isinf(J) ? __builtin_nan("") : J;
            if (last) verdict[sid] = J <= eps ? 1 : 0;
        }
    }
}

// ---- Alg. 2 criteria, a contact step's LPs over all sets ----------------------
// k_optimize runs a contact step's candidate LPs side by side, so each wave
// waits for the slowest of its 64 LPs at every step.  With a workspace that
// holds a step's candidate results, each contact step takes two launches
// instead: every candidate's LP, the lanes of a wave taking one after another
// (k_opt_solve, see lp_wave), then each set's pick (k_opt_pick).  The LPs, their
// starting bases and the picks are those of k_optimize.
struct OptSplit {
    double *sJ;          // per set: criterion value of its last pick (INF before any)
    int32_t *sB;         // per set: 7 basis column ids of its last finite pick (-1: none yet)
    double *cJ;          // per candidate (set t, candidate j at t * n_inner + j): t*, INF if unsolved
    int32_t *cB;         // per candidate: the 7 column ids of its final basis
};

// Set t of the sets of poses with non-empty domains: its set id and whether it
// was drawn (the drawn-set test of k_optimize); kc = contacts with the palm's.
__device__ inline bool opt_set(int64_t t, const int32_t *__restrict__ valid_poses, const uint32_t *__restrict__ dom_count,
                               const int32_t *__restrict__ palm_pt, const int32_t *__restrict__ set_pt, int N, int F,
                               int D, int k, uint32_t seed_lo, uint32_t seed_hi, uint32_t request_id,
                               int64_t pose_offset, int64_t &sid, int &pc)
{
    const int64_t pg = valid_poses[t / D];
    const int d = (int)(t % D);
    sid = pg * D + d;
    const int32_t *sp = set_pt + sid * k;
    const uint32_t fm = choose_fingers(eligible_fingers(dom_count, pg, F), k, (uint32_t)(pose_offset + pg), d,
                                       request_id, seed_lo, seed_hi);
    pc = palm_pt ? palm_pt[pg] : -1;
    bool drawn = fm != 0 && pc < N;
    for (int i = 0; i < k; ++i) drawn &= sp[i] >= 0 && sp[i] < N;
    return drawn;
}

// LPs of the candidates at contact step i, each from the set's current points,
// warm-started from the set's last pick's basis (none at the round's first step)
template <int KM, int MC>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_opt_solve(const float *__restrict__ pts, const float *__restrict__ nrm, int N,
            const int32_t *__restrict__ valid_poses, const int32_t *__restrict__ n_valid_poses,
            const int32_t *__restrict__ palm_pt, int D, int k, int m, double mu, double rho, int max_pivots,
            LpConst cs, int n_inner, int i, const int32_t *__restrict__ cands, const int32_t *__restrict__ set_pt,
            OptSplit os)
{
    __shared__ LpLds<KM> L;
    __shared__ int wb[7][256];
    const int tid = threadIdx.x;
    int64_t next, end;
    lp_share(blockIdx.x, gridDim.x, (int64_t)(*n_valid_poses) * D * n_inner, next, end);
    auto fetch = [&](int64_t g, Lp<KM, MC> &P) {
        const int64_t t = (uint32_t)g / (uint32_t)n_inner;  // candidate ids are below 2^31
        const int j = (int)(g - t * n_inner);
        const int cand = cands[(t * k + i) * n_inner + j];
        if (cand < 0) {  // not a drawn set (k_opt_project)
            os.cJ[g] = INFINITY;
            return false;
        }
        const uint32_t q = (uint32_t)t / (uint32_t)D;
        const int64_t pg = valid_poses[q], sid = pg * D + ((uint32_t)t - q * (uint32_t)D);
        const int pc = palm_pt ? palm_pt[pg] : -1;
        for (int c = 0; c < k; ++c) lp_load(L, tid, c, pts, nrm, N, c == i ? cand : set_pt[sid * k + c]);
        if (pc >= 0) lp_load(L, tid, k, pts, nrm, N, pc);
#pragma unroll
        for (int r = 0; r < 7; ++r) wb[r][tid] = i == 0 ? -1 : os.sB[t * 7 + r];
        P.k = pc >= 0 ? k + 1 : k;
        P.n = P.k * m;
        return true;
    };
    lp_wave<KM, MC, true>(
        L, next, end, m, mu, rho, max_pivots, cs, fetch, [&](int64_t, int r) { return wb[r][tid]; },
        [&](int64_t g, double ts, int status, const Lp<KM, MC> &P) {
            os.cJ[g] = status == 0 ? ts : INFINITY;
#pragma unroll
            for (int r = 0; r < 7; ++r) os.cB[g * 7 + r] = P.basis[r];
        });
}

// Each set's pick at contact step i: the lowest candidate within kOptTau of
// the best t* (the first candidate when none is finite), its point into the
// set, its basis the warm start of the next step when its t* is finite.
__global__ void k_opt_pick(const int32_t *__restrict__ valid_poses, const int32_t *__restrict__ n_valid_poses,
                           const uint32_t *__restrict__ dom_count, const int32_t *__restrict__ palm_pt, int N, int F,
                           int D, int k, int n_inner, int i, bool last, double eps, uint32_t seed_lo,
                           uint32_t seed_hi, uint32_t request_id, int64_t pose_offset,
                           const int32_t *__restrict__ cands, int32_t *__restrict__ set_pt,
                           uint8_t *__restrict__ verdict, double *__restrict__ tstar, OptSplit os)
{
    const int64_t n_work = (int64_t)(*n_valid_poses) * D;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < n_work;
         t += (int64_t)gridDim.x * blockDim.x) {
        int64_t sid;
        int pc;
        if (!opt_set(t, valid_poses, dom_count, palm_pt, set_pt, N, F, D, k, seed_lo, seed_hi, request_id,
                     pose_offset, sid, pc)) {
            verdict[sid] = 0;  // not a drawn set: no criterion
            tstar[sid] = __builtin_nan("");
            continue;
        }
        const double *cj = os.cJ + t * n_inner;
        double mn = INFINITY;
        for (int j = 0; j < n_inner; ++j) mn = fmin(mn, cj[j]);
        int js = -1;
        for (int j = n_inner - 1; j >= 0; --j)
            if (cj[j] <= mn + kOptTau) js = j;
        const int pick = js >= 0 ? cands[(t * k + i) * n_inner + js] : -1;
        double J = i == 0 ? INFINITY : os.sJ[t];
        if (i == 0) os.sB[t * 7] = -1;
        if (pick >= 0) {
            J = cj[js];
            set_pt[sid * k + i] = pick;
            if (!isinf(J)) {
#pragma unroll
                for (int r = 0; r < 7; ++r) os.sB[t * 7 + r] = os.cB[(t * n_inner + js) * 7 + r];
            }
        }
        os.sJ[t] = J;
        if (i == k - 1) {
            tstar[sid] = isinf(J) ? __builtin_nan("") : J;
            if (last) verdict[sid] = J <= eps ? 1 : 0;
        }
    }
}

// links of the (moved) contacts of every set of a pose with non-empty domains,
// picked with the set's draw words exactly as k_draw does
__global__ void k_relink(DevHand H, const float *__restrict__ pts,
                         const float *__restrict__ nrm, int N, const float *__restrict__ poses,
                         const int32_t *__restrict__ valid_poses, const int32_t *__restrict__ n_valid_poses,
                         const uint32_t *__restrict__ dom_count, int D, int k, uint32_t seed_lo, uint32_t seed_hi,
                         uint32_t request_id, int64_t pose_offset, const int32_t *__restrict__ set_pt,
                         int8_t *__restrict__ set_link)
{
    __shared__ float4 cb4[kMaxBins];
    for (int i = threadIdx.x; i < H.B; i += blockDim.x)
        cb4[i] = make_float4(H.bin_c[3 * i], H.bin_c[3 * i + 1], H.bin_c[3 * i + 2], 0.0f);
    __syncthreads();
    const int64_t n_work = (int64_t)(*n_valid_poses) * D;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < n_work;
         t += (int64_t)gridDim.x * blockDim.x) {
        const int64_t g = valid_poses[t / D];
        const int d = (int)(t % D);
        uint32_t w[16];
        for (int blk = 0; blk * 4 < 2 * k; ++blk)
            philox4x32_10((uint32_t)(pose_offset + g), (uint32_t)(4 * d + blk), kPurposeDraw, request_id, seed_lo,
                          seed_hi, w + 4 * blk);
        const int32_t *sp = set_pt + (g * D + d) * k;
        int8_t *sl = set_link + (g * D + d) * k;
        uint32_t fm = choose_fingers(eligible_fingers(dom_count, g, H.F), k, (uint32_t)(pose_offset + g), d,
                                     request_id, seed_lo, seed_hi);
        for (int i = 0; i < k; ++i) {
            const int f = __ffs(fm) - 1;
            fm &= fm - 1u;
            const int idx = sp[i];
            sl[i] = (int8_t)((f >= 0 && idx >= 0 && idx < N)
                                 ? pick_link(H, cb4, window_map(H, poses + 12 * g, f), pts, nrm, N, poses + 12 * g,
                                             f, idx, w[k + i])
                                 : -1);
        }
    }
}

// ---- second contact round (Sec. 5.3, additional search phase; Sec. 5.6) -------
// Finger of link l (its joint's finger).
__device__ inline int link_finger(const DevHand &H, int l)
{
    for (int f = 0; f < H.F; ++f)
        if (l >= H.finger_first[f] && l < H.finger_first[f] + H.finger_dof[f]) return f;
    return -1;
}

// One workgroup per pose.  A round-1 set (k1 contacts) is extended when it is
// listed (list: sorted set ids, list_ok[i] != 0 if given) or, without a list,
// when its draw is whole and its verdict 0; its contacts must all have a
// point and a link.  It gets k_add contacts on unused fingers with non-empty
// domains: the fingers by choose_fingers over them (Philox purpose 19), the
// points as the floor(w * count / 2^32)-th domain bit and the links by the
// reverse lookup (purpose 21: word i and k_add + i for the i-th new finger).
// The extended set lists its k1 + k_add contacts in increasing finger order.
// Sets not extended get set_pt -1, verdict 0, t* NaN; pose_valid[g] = some
// set of the pose was extended (its verdicts are computed next).
__global__ void __launch_bounds__(kDrawThreads)
k_extend(DevHand H, const float *__restrict__ pts, const float *__restrict__ nrm,
         int N, int g0, const float *__restrict__ poses, const uint32_t *__restrict__ dom_bits,
         const uint32_t *__restrict__ dom_count, int D, int k1, int k_add, const int32_t *__restrict__ set_pt1,
         const int8_t *__restrict__ set_link1, const uint8_t *__restrict__ verdict1, const int32_t *__restrict__ list,
         const int32_t *__restrict__ list_n, const uint8_t *__restrict__ list_ok, uint32_t seed_lo, uint32_t seed_hi,
         uint32_t request_id, int64_t pose_offset, int32_t *__restrict__ set_pt2, int8_t *__restrict__ set_link2,
         uint8_t *__restrict__ pose_valid, uint8_t *__restrict__ verdict2, double *__restrict__ tstar2)
{
    extern __shared__ uint32_t prefix[];  // [F][nsb + 1]
    __shared__ LinkLds L;
    __shared__ uint32_t counts[kMaxFingers];
    __shared__ int32_t range[2];
    __shared__ uint32_t any;
    const int g = g0 + (int)blockIdx.x, F = H.F, k2 = k1 + k_add;
    const int NW = (N + 31) >> 5, nsb = (NW + kSuper - 1) / kSuper;
    const uint32_t *dom = dom_bits + (int64_t)g * F * NW;
    const float *pose = poses + 12 * (int64_t)g;
    link_lds(L, H, pose);
    if ((int)threadIdx.x < F) counts[threadIdx.x] = dom_count[(int64_t)g * F + threadIdx.x];
    if (threadIdx.x == 0) {
        any = 0;
        range[0] = range[1] = 0;
        if (list) {  // this pose's entries: ids in [g D, (g + 1) D) of the sorted list
            const int n = *list_n;
            int lo = 0, hi = n;
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if ((int64_t)list[mid] < (int64_t)g * D) lo = mid + 1; else hi = mid;
            }
            range[0] = lo;
            hi = n;
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if ((int64_t)list[mid] < (int64_t)(g + 1) * D) lo = mid + 1; else hi = mid;
            }
            range[1] = lo;
        }
    }
    build_prefix(prefix, dom, F, NW, nsb);
    __syncthreads();
    const uint32_t gg = (uint32_t)(pose_offset + g);
    for (int64_t dd = threadIdx.x; dd < D; dd += blockDim.x) {
        const int d = (int)dd;
        const int64_t sid = (int64_t)g * D + d;
        const int32_t *sp1 = set_pt1 + sid * k1;
        const int8_t *sl1 = set_link1 + sid * k1;
        int32_t *sp2 = set_pt2 + sid * k2;
        int8_t *sl2 = set_link2 + sid * k2;
        bool take;
        if (list) {
            int lo = range[0], hi = range[1];
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if ((int64_t)list[mid] < sid) lo = mid + 1; else hi = mid;
            }
            take = lo < range[1] && (int64_t)list[lo] == sid && (!list_ok || list_ok[lo] != 0);
        } else {
            take = verdict1[sid] == 0;
        }
        uint32_t used = 0;
        int fin1[8];
        for (int i = 0; i < k1 && take; ++i) {
            const int l = sl1[i];
            const int f = (l >= 0 && sp1[i] >= 0 && sp1[i] < N) ? link_finger(H, l) : -1;
            if (f < 0) take = false; else { fin1[i] = f; used |= 1u << f; }
        }
        uint32_t fm = 0;
        if (take) {
            uint32_t elig = 0;
            for (int f = 0; f < F; ++f) elig |= (counts[f] > 0 && !((used >> f) & 1u) ? 1u : 0u) << f;
            fm = choose_fingers(elig, k_add, gg, d, request_id, seed_lo, seed_hi, kPurposeExtFingers);
            take = fm != 0u;
        }
        if (!take) {
            for (int i = 0; i < k2; ++i) {
                sp2[i] = -1;
                sl2[i] = -1;
            }
            verdict2[sid] = 0;
            tstar2[sid] = __builtin_nan("");
            continue;
        }
        any = 1u;  // benign race: every writer stores 1
        uint32_t w[16];
        for (int blk = 0; blk * 4 < 2 * k_add; ++blk)
            philox4x32_10(gg, (uint32_t)(4 * d + blk), kPurposeExtDraw, request_id, seed_lo, seed_hi, w + 4 * blk);
        int np[8], nl[8], nf[8];
        for (int i = 0; i < k_add; ++i) {
            const int f = __ffs(fm) - 1;  // the i-th smallest new finger
            fm &= fm - 1u;
            const int idx = select_domain(prefix + f * (nsb + 1), nsb, dom + (int64_t)f * NW, NW,
                                          __umulhi(w[i], counts[f]));
            nf[i] = f;
            np[i] = idx;
            nl[i] = idx >= 0 ? pick_link(H, L.cb4, L.aff[H.lat ? 0 : f], pts, nrm, N, pose, f, idx, w[k_add + i]) : -1;
        }
        // union in increasing finger order (both groups sorted)
        int a = 0, b = 0;
        for (int o = 0; o < k2; ++o) {
            if (b >= k_add || (a < k1 && fin1[a] < nf[b])) {
                sp2[o] = sp1[a];
                sl2[o] = sl1[a];
                ++a;
            } else {
                sp2[o] = np[b];
                sl2[o] = (int8_t)nl[b];
                ++b;
            }
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) pose_valid[g] = any ? 1 : 0;
}

// flag[s] = set s has every point and link and verdict 0 (an unstable set)
__global__ void k_flag_unstable(const int32_t *__restrict__ set_pt, const int8_t *__restrict__ set_link,
                                const uint8_t *__restrict__ verdict, int64_t n_sets, int k, uint8_t *__restrict__ flag)
{
    const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= n_sets) return;
    bool ok = verdict[s] == 0;
    for (int i = 0; i < k; ++i) ok &= set_pt[s * k + i] >= 0 && set_link[s * k + i] >= 0;
    flag[s] = ok ? 1 : 0;
}

// ---- compaction ------------------------------------------------------------
// Flags are bytes of value 0 or 1.  The 16 flags from i on (i a multiple of 16),
// those at n and beyond 0: one load where the array allows it (al: its alignment,
// 16, 4 or 1).
__device__ inline uint4 flags16(const uint8_t *__restrict__ flag, int64_t i, int64_t n, int al)
{
    uint4 v = make_uint4(0u, 0u, 0u, 0u);
    if (i + 16 <= n && al >= 4) {
        if (al == 16) return *reinterpret_cast<const uint4 *>(flag + i);
        const uint32_t *w = reinterpret_cast<const uint32_t *>(flag + i);
        return make_uint4(w[0], w[1], w[2], w[3]);
    }
    uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int q = 0; q < 16; ++q)
        if (i + q < n) w[q >> 2] |= (uint32_t)flag[i + q] << (8 * (q & 3));
    v = make_uint4(w[0], w[1], w[2], w[3]);
    return v;
}
__device__ inline int flag_alignment(const uint8_t *flag)
{
    const uintptr_t a = reinterpret_cast<uintptr_t>(flag);
    return a % 16 == 0 ? 16 : a % 4 == 0 ? 4 : 1;
}
__device__ inline uint32_t flags_count(const uint4 &v) { return __popc(v.x) + __popc(v.y) + __popc(v.z) + __popc(v.w); }
// the indices of the set flags of v (flags i.. of the array) from list[pos] on
__device__ inline void flags_write(const uint4 &v, int64_t i, int32_t *__restrict__ list, uint32_t &pos)
{
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int q = 0; q < 4; ++q)
        for (uint32_t x = w[q]; x; x &= x - 1u) list[pos++] = (int32_t)(i + 4 * q + ((__ffs(x) - 1) >> 3));
}

// Up to kCompactOneMax flags: one block of 1,024 threads, a run of flags each (a
// multiple of 16), counts scanned over lanes and waves, then each thread writes
// its run's indices.  A few thousand flags take 3-4 us in one launch (18 us in the
// three of count, scan and scatter) on an idle chip; among other streams' work the
// block waits for a CU with 16 free waves (20 us on average under a busy server).
// Beyond the limit one CU's reads and writes cost more than they save (65,536 flags
// 21 us, 262,144 47 us; two launches 10 us).
constexpr int kCompactOneThreads = 1024;
constexpr int64_t kCompactOneMax = 32768;
constexpr int64_t kSelfScanMax = 2048;  // chunks whose counts every scatter block adds up itself (4 us less)

__device__ __forceinline__ void compact_one_block(uint32_t *wsum, const uint8_t *__restrict__ flag, int64_t n,
                                                  int32_t *__restrict__ list, int32_t *__restrict__ total)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, al = flag_alignment(flag);
    const int64_t per = ((n + kCompactOneThreads - 1) / kCompactOneThreads + 15) & ~(int64_t)15;
    const int64_t beg = min(n, tid * per), end = min(n, beg + per);
    uint32_t c = 0;
#pragma unroll 4
    for (int64_t i = beg; i < end; i += 16) c += flags_count(flags16(flag, i, n, al));
    const uint32_t incl = wave_scan_incl(c);
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    uint32_t pos = incl - c, all = 0;
    for (int w = 0; w < kCompactOneThreads / 64; ++w) {
        pos += w < wave ? wsum[w] : 0u;
        all += wsum[w];
    }
    if (tid == 0) *total = (int32_t)all;
    if (c)
        for (int64_t i = beg; i < end; i += 16) flags_write(flags16(flag, i, n, al), i, list, pos);
}

__global__ void __launch_bounds__(kCompactOneThreads)
k_compact_one(const uint8_t *__restrict__ flag, int64_t n, int32_t *__restrict__ list, int32_t *__restrict__ total)
{
    __shared__ uint32_t wsum[kCompactOneThreads / 64];
    compact_one_block(wsum, flag, n, list, total);
}

// block bid: the number of set flags in its kChunk flags
__device__ __forceinline__ void chunk_count_block(uint32_t *part, int64_t bid, const uint8_t *__restrict__ flag,
                                                  int64_t n, uint32_t *__restrict__ chunk_count)
{
    const int64_t base = bid * kChunk + (int64_t)threadIdx.x * kChunkPerThread;
    const int al = flag_alignment(flag);
    uint32_t c = 0;
#pragma unroll
    for (int i = 0; i < kChunkPerThread; i += 16) c += flags_count(flags16(flag, base + i, n, al));
    for (int off = 32; off > 0; off >>= 1) c += __shfl_down(c, off, 64);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t s = 0;
        for (int w = 0; w < kCompactThreads / 64; ++w) s += part[w];
        chunk_count[bid] = s;
    }
}

// one block: exclusive scan of chunk counts, total into n_acc
__device__ __forceinline__ void chunk_scan_block(uint32_t *tot, const uint32_t *__restrict__ chunk_count,
                                                 int64_t n_chunks, uint32_t *__restrict__ chunk_off,
                                                 int32_t *__restrict__ n_acc)
{
    const int64_t per = (n_chunks + kCompactThreads - 1) / kCompactThreads;
    const int64_t b0 = threadIdx.x * per;
    uint32_t s = 0;
    for (int64_t i = b0; i < min(n_chunks, b0 + per); ++i) s += chunk_count[i];
    tot[threadIdx.x] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t run = 0;
        for (int t = 0; t < kCompactThreads; ++t) {
            const uint32_t v = tot[t];
            tot[t] = run;
            run += v;
        }
        *n_acc = (int32_t)run;
    }
    __syncthreads();
    uint32_t run = tot[threadIdx.x];
    for (int64_t i = b0; i < min(n_chunks, b0 + per); ++i) {
        chunk_off[i] = run;
        run += chunk_count[i];
    }
}

// Block bid: the indices of its set flags, in order.  off: the chunks' offsets
// (of chunk_scan_block), or, for at most kSelfScanMax chunks (self), their counts:
// the block adds up those before it, and the last one writes the total.
__device__ __forceinline__ void chunk_scatter_block(uint32_t *wsum, int64_t bid, const uint8_t *__restrict__ flag,
                                                    int64_t n, const uint32_t *__restrict__ off, bool self,
                                                    int32_t *__restrict__ list, int32_t *__restrict__ total)
{
    const int64_t base = bid * kChunk + (int64_t)threadIdx.x * kChunkPerThread;
    const int al = flag_alignment(flag), wave = threadIdx.x >> 6;
    uint32_t before = 0;
    if (self) {
        for (int64_t i = threadIdx.x; i < bid; i += kCompactThreads) before += off[i];
        for (int o = 32; o > 0; o >>= 1) before += __shfl_xor(before, o, 64);
        if ((threadIdx.x & 63) == 0) wsum[kCompactThreads / 64 + wave] = before;
    }
    uint4 v[kChunkPerThread / 16];
    uint32_t c = 0;
#pragma unroll
    for (int i = 0; i < kChunkPerThread / 16; ++i) {
        v[i] = flags16(flag, base + 16 * i, n, al);
        c += flags_count(v[i]);
    }
    const uint32_t incl = wave_scan_incl(c);
    if ((threadIdx.x & 63) == 63) wsum[wave] = incl;
    __syncthreads();
    uint32_t pos = incl - c;
    if (self) {
        for (int w = 0; w < kCompactThreads / 64; ++w) pos += wsum[kCompactThreads / 64 + w];
    } else {
        pos += off[bid];
    }
    for (int w = 0; w < wave; ++w) pos += wsum[w];
    if (self && (bid + 1) * kChunk >= n && threadIdx.x == kCompactThreads - 1) *total = (int32_t)(pos + c);
#pragma unroll
    for (int i = 0; i < kChunkPerThread / 16; ++i) flags_write(v[i], base + 16 * i, list, pos);
}

__global__ void __launch_bounds__(kCompactThreads)
k_chunk_count(const uint8_t *__restrict__ verdict, int64_t n, uint32_t *__restrict__ chunk_count)
{
    __shared__ uint32_t part[kCompactThreads / 64];
    chunk_count_block(part, blockIdx.x, verdict, n, chunk_count);
}

__global__ void __launch_bounds__(kCompactThreads)
k_chunk_scan(const uint32_t *__restrict__ chunk_count, int64_t n_chunks, uint32_t *__restrict__ chunk_off,
             int32_t *__restrict__ n_acc)
{
    __shared__ uint32_t tot[kCompactThreads];
    chunk_scan_block(tot, chunk_count, n_chunks, chunk_off, n_acc);
}

__global__ void __launch_bounds__(kCompactThreads)
k_chunk_scatter(const uint8_t *__restrict__ verdict, int64_t n, const uint32_t *__restrict__ off, bool self,
                int32_t *__restrict__ acc_list, int32_t *__restrict__ n_acc)
{
    __shared__ uint32_t wsum[2 * kCompactThreads / 64];
    chunk_scatter_block(wsum, blockIdx.x, verdict, n, off, self, acc_list, n_acc);
}

// Batched compaction: POSES = the chunk's poses with a usable draw (the
// verdict launch's work list), else its accepted sets.
struct CompactView {
    const uint8_t *flag;
    int64_t n;
    uint32_t *count, *off;
    int32_t *total, *list;
};

template <bool POSES>
__device__ __forceinline__ CompactView compact_view(const ChunkDesc &c)
{
    if (POSES) return {c.pose_valid, (int64_t)c.P, c.pchunk_count, c.pchunk_off, c.n_valid_poses, c.valid_poses};
    return {c.verdict, (int64_t)c.P * c.D, c.chunk_count, c.chunk_off, c.n_acc, c.acc};
}

// every member in one block of its own
template <bool POSES>
__global__ void __launch_bounds__(kCompactOneThreads)
k_compact_batch(const ChunkDesc *__restrict__ d, const uint16_t *__restrict__ idx, const uint32_t *__restrict__ first,
                int n)
{
    __shared__ uint32_t wsum[kCompactOneThreads / 64];
    const CompactView v = compact_view<POSES>(d[idx[batch_member(first, n, blockIdx.x)]]);
    compact_one_block(wsum, v.flag, v.n, v.list, v.total);
}

template <bool POSES>
__global__ void __launch_bounds__(kCompactThreads)
k_count_batch(const ChunkDesc *__restrict__ d, const uint16_t *__restrict__ idx, const uint32_t *__restrict__ first,
              int n)
{
    __shared__ uint32_t part[kCompactThreads / 64];
    const int j = batch_member(first, n, blockIdx.x);
    const CompactView v = compact_view<POSES>(d[idx[j]]);
    chunk_count_block(part, blockIdx.x - first[j], v.flag, v.n, v.count);
}

template <bool POSES>
__global__ void __launch_bounds__(kCompactThreads)
k_scan_batch(const ChunkDesc *__restrict__ d, const uint16_t *__restrict__ idx, const uint32_t *__restrict__ first,
             int n)
{
    __shared__ uint32_t tot[kCompactThreads];
    const int j = batch_member(first, n, blockIdx.x);
    const CompactView v = compact_view<POSES>(d[idx[j]]);
    chunk_scan_block(tot, v.count, (v.n + kChunk - 1) / kChunk, v.off, v.total);
}

template <bool POSES>
__global__ void __launch_bounds__(kCompactThreads)
k_scatter_batch(const ChunkDesc *__restrict__ d, const uint16_t *__restrict__ idx, const uint32_t *__restrict__ first,
                int n, bool self)
{
    __shared__ uint32_t wsum[2 * kCompactThreads / 64];
    const int j = batch_member(first, n, blockIdx.x);
    const CompactView v = compact_view<POSES>(d[idx[j]]);
    chunk_scatter_block(wsum, blockIdx.x - first[j], v.flag, v.n, self ? v.count : v.off, self, v.list, v.total);
}

}  // namespace lg

using namespace lg;

// list = the increasing indices of the n flags that are set, *total their number;
// count, off: a word per kChunk flags (beyond kCompactOneMax)
static lg_status compact(const uint8_t *flag, int64_t n, uint32_t *count, uint32_t *off, int32_t *list, int32_t *total,
                         hipStream_t s)
{
    if (n <= kCompactOneMax) {
        hipLaunchKernelGGL(k_compact_one, dim3(1), dim3(kCompactOneThreads), 0, s, flag, n, list, total);
    } else {
        const int64_t nc = (n + kChunk - 1) / kChunk;
        hipLaunchKernelGGL(k_chunk_count, dim3((unsigned)nc), dim3(kCompactThreads), 0, s, flag, n, count);
        const bool self = nc <= kSelfScanMax;
        if (!self) hipLaunchKernelGGL(k_chunk_scan, dim3(1), dim3(kCompactThreads), 0, s, count, nc, off, total);
        hipLaunchKernelGGL(k_chunk_scatter, dim3((unsigned)nc), dim3(kCompactThreads), 0, s, flag, n,
                           self ? count : off, self, list, total);
    }
    LG_HIP(hipGetLastError());
    return LG_OK;
}

extern "C" {

// workspace: [set chunks: count, offset] [pose chunks: count, offset]
//            [valid pose list P] [n_valid_poses] [pose_valid P bytes]
//            and, for the contact-point optimisation, [grid params]
//            [cell counts/cursor (kGridMax+1)^3] [cell starts +1] [cell points N: xyz + index]
//            [a round's candidates P D k n_inner]
struct SearchWs {
    uint32_t *chunk_count, *chunk_off, *pchunk_count, *pchunk_off;
    int32_t *valid_poses, *n_valid_poses;
    uint8_t *pose_valid;
    GridDev *grid;
    uint32_t *cell_count, *cell_start;
    float4 *cell_pts;
    int32_t *cands;
    OptSplit split;   // per-candidate arrays of the criteria (null when not laid out)
    size_t bytes;
};

static SearchWs search_ws(void *base, int64_t n_points, int64_t n_poses, int64_t draws, bool opt, int64_t k = 0,
                          int64_t n_inner = 0, bool split = false)
{
    const int64_t n_sets = n_poses * draws;
    const int64_t nc = (n_sets + kChunk - 1) / kChunk, npc = (n_poses + kChunk - 1) / kChunk;
    SearchWs w;
    uint32_t *u = static_cast<uint32_t *>(base);
    w.chunk_count = u;
    w.chunk_off = u + nc;
    w.pchunk_count = u + 2 * nc;
    w.pchunk_off = u + 2 * nc + npc;
    w.valid_poses = reinterpret_cast<int32_t *>(u + 2 * nc + 2 * npc);
    w.n_valid_poses = w.valid_poses + n_poses;
    w.pose_valid = reinterpret_cast<uint8_t *>(w.n_valid_poses + 1);
    size_t off = ((size_t)(2 * nc + 2 * npc + n_poses + 1) * 4 + (size_t)n_poses + 255) & ~(size_t)255;
    w.grid = nullptr;
    w.cell_count = w.cell_start = nullptr;
    w.cell_pts = nullptr;
    w.cands = nullptr;
    w.split = OptSplit{};
    if (opt) {
        const int64_t ncell = kGridCells;
        char *b = static_cast<char *>(base);
        w.grid = reinterpret_cast<GridDev *>(b + off);
        off += 256;
        w.cell_count = reinterpret_cast<uint32_t *>(b + off);
        off += (size_t)ncell * 4;
        w.cell_start = reinterpret_cast<uint32_t *>(b + off);
        off += (size_t)(ncell + 1) * 4;
        off = (off + 255) & ~(size_t)255;
        w.cell_pts = reinterpret_cast<float4 *>(b + off);
        off += ((size_t)n_points * 16 + 255) & ~(size_t)255;
        w.cands = reinterpret_cast<int32_t *>(b + off);
        off += (size_t)n_sets * k * n_inner * 4;
        if (split) {
            const size_t nc_ = (size_t)n_sets * n_inner;
            auto take = [&](size_t bytes) {
                off = (off + 255) & ~(size_t)255;
                char *q = b + off;
                off += bytes;
                return q;
            };
            w.split.sJ = reinterpret_cast<double *>(take((size_t)n_sets * 8));
            w.split.sB = reinterpret_cast<int32_t *>(take((size_t)n_sets * 28));
            w.split.cJ = reinterpret_cast<double *>(take(nc_ * 8));
            w.split.cB = reinterpret_cast<int32_t *>(take(nc_ * 28));
        }
    }
    w.bytes = off + 256;
    return w;
}

// Alg. 2 criteria with per-candidate results need candidate ids below 2^31.
static bool split_fits(int64_t n_poses, int64_t draws, const lg_search_params *p)
{
    return p->opt_outer > 0 && n_poses * draws * p->opt_inner < 0x7fffffffLL;
}

// Workspace of the search: with split, the per-candidate arrays of the
// criteria too (what lg_search_workspace_bytes asks for); without, the least
// a search runs in (Alg. 2 then runs its criteria in one launch per round).
static size_t search_ws_bytes(int32_t n_points, int32_t n_poses, const lg_search_params *p, bool split)
{
    if (!p || n_poses <= 0 || p->draws <= 0) return 256;
    return search_ws(nullptr, std::max(n_points, 0), n_poses, p->draws, p->opt_outer > 0, p->k,
                     p->opt_outer > 0 ? p->opt_inner : 0, split && split_fits(n_poses, p->draws, p)).bytes;
}

size_t lg_search_workspace_bytes(int32_t n_points, int32_t n_poses, const lg_search_params *p)
{
    return search_ws_bytes(n_points, n_poses, p, true);
}

// One round of Alg. 2 criteria with per-candidate results: per contact step
// the LPs of every candidate, then the picks.
static lg_status opt_split_round(const float *pts, const float *nrm, int n_points, const SearchWs &ws,
                                 const uint32_t *dom_count, const int32_t *palm, int F, const lg_search_params *p,
                                 int kk, bool m8, const LpConst &cs, dim3 sgrid, dim3 cgrid, bool last,
                                 int32_t *set_pt, uint8_t *verdict, double *tstar, hipStream_t s)
{
    const uint32_t slo = (uint32_t)p->seed, shi = (uint32_t)(p->seed >> 32);
    const double mu = p->mu, rho = p->moment_scale;
    for (int i = 0; i < p->k; ++i) {
#define LG_SPLIT_M(KM, MC)                                                                                       \
    hipLaunchKernelGGL((k_opt_solve<KM, MC>), cgrid, dim3(256), 0, s, pts, nrm, n_points, ws.valid_poses,       \
                       ws.n_valid_poses, palm, p->draws, p->k, p->m_edges, mu, rho, p->max_pivots, cs,           \
                       p->opt_inner, i, ws.cands, set_pt, ws.split)
#define LG_SPLIT(KM) if (m8) LG_SPLIT_M(KM, 8); else LG_SPLIT_M(KM, 0)
        if (kk <= 3) { LG_SPLIT(3); } else if (kk <= 4) { LG_SPLIT(4); } else if (kk <= 5) { LG_SPLIT(5); }
        else if (kk <= 6) { LG_SPLIT(6); } else { LG_SPLIT(8); }
#undef LG_SPLIT
#undef LG_SPLIT_M
        hipLaunchKernelGGL(k_opt_pick, sgrid, dim3(256), 0, s, ws.valid_poses, ws.n_valid_poses, dom_count, palm,
                           n_points, F, p->draws, p->k, p->opt_inner, i, last, (double)p->eps, slo, shi,
                           p->request_id, p->pose_offset, ws.cands, set_pt, verdict, tstar, ws.split);
    }
    LG_HIP(hipGetLastError());
    return LG_OK;
}

}  // extern "C"

LpConst lg::lp_const(int m)
{
    LpConst cs;
    for (int e = 0; e < 16; ++e) {
        const double th = 2.0 * M_PI * e / m;
        cs.ce[e] = e < m ? cos(th) : 0.0;
        cs.se[e] = e < m ? sin(th) : 0.0;
    }
    return cs;
}

// Blocks of an LP launch: no more than are resident at once (two per CU: two
// waves per SIMD), so that each lane takes several LPs; a small launch spreads
// over every SIMD, down to a few LPs per wave (its time is that of its slowest
// LP, and a wave waits for the slowest of its own): 4,096 sets 55 us with 16
// sets per block, 75 us with 64; 1.2 M LPs 0.67 ms with two blocks per CU, 0.68
// with four.
uint32_t lg::verdict_blocks(int64_t n_sets, int n_cu)
{
    return (uint32_t)std::max<int64_t>(1, std::min<int64_t>((n_sets + 15) / 16, (int64_t)n_cu * 2));
}

void lg::chunk_workspace(void *ws, int64_t n_points, int64_t n_poses, int64_t draws, ChunkDesc &c)
{
    const SearchWs w = search_ws(ws, n_points, n_poses, draws, false);
    c.pose_valid = w.pose_valid;
    c.pchunk_count = w.pchunk_count;
    c.pchunk_off = w.pchunk_off;
    c.valid_poses = w.valid_poses;
    c.n_valid_poses = w.n_valid_poses;
    c.chunk_count = w.chunk_count;
    c.chunk_off = w.chunk_off;
}

// the whole search on a given workspace (the caller's, or the static scratch
// array of lg_search_noalloc); allocates nothing
static lg_status search_impl(const lg_field *field, const float *pts, const float *nrm, int32_t n_points,
                             const float *poses, int32_t n_poses, const uint32_t *dom_bits, const uint32_t *dom_count,
                             const lg_search_params *p, int32_t *set_pt, int8_t *set_link, uint8_t *verdict,
                             double *tstar, int32_t *acc_list, int32_t *n_acc, void *workspace,
                             size_t workspace_bytes, void *stream)
{
    if (!field || !p) return fail(LG_EINVAL, "null field or params");
    const DevHand &H = field->dh;
    if (n_points <= 0 || n_poses < 0) return fail(LG_EINVAL, "n_points must be > 0 and n_poses >= 0");
    if (p->k < 1 || p->k > H.F) return fail(LG_EINVAL, "need 1 <= k <= number of fingers (one contact per finger)");
    const int32_t *palm = p->palm_pt;
    const int kk = p->k + (palm ? 1 : 0);  // contacts of the largest set (with a palm contact)
    if (p->draws <= 0 || p->m_edges < 3 || p->m_edges > 16 || kk > 8)
        return fail(LG_EINVAL, "need draws > 0, 3 <= m_edges <= 16, k <= 8 (k <= 7 with palm contacts)");
    if (!(p->mu >= 0.0f) || !(p->moment_scale > 0.0f) || p->max_pivots < 0)
        return fail(LG_EINVAL, "need mu >= 0, moment_scale > 0, max_pivots >= 0");
    if ((int64_t)n_poses * p->draws > 0x7fffffffLL) return fail(LG_EINVAL, "P * D must be < 2^31");
    if (n_poses == 0) return LG_OK;
    if (!pts || !nrm || !poses || !dom_bits || !dom_count || !set_pt || !set_link || !verdict || !tstar ||
        !acc_list || !n_acc || !workspace)
        return fail(LG_EINVAL, "null device buffer");
    if (p->opt_outer < 0 || p->opt_outer > 64 || (p->opt_outer > 0 && (p->opt_inner < 1 || p->opt_inner > 16)) ||
        !(p->opt_sigma >= 0.0f) || (int64_t)p->opt_outer * p->k * p->opt_inner >= (1 << 24))
        return fail(LG_EINVAL, "need 0 <= opt_outer <= 64, 1 <= opt_inner <= 16, opt_sigma >= 0");
    if (workspace_bytes < search_ws_bytes(n_points, n_poses, p, false)) return fail(LG_EINVAL, "workspace too small");
    const int NW = (n_points + 31) / 32, nsb = (NW + kSuper - 1) / kSuper;
    const size_t lds = (size_t)H.F * (nsb + 1) * sizeof(uint32_t);
    if (lds > 48 * 1024) return fail(LG_EUNSUPPORTED, "too many points for the draw rank structure");
    hipStream_t s = as_stream(stream);
    const bool opt = p->opt_outer > 0;
    // Alg. 2 criteria with per-candidate results when the workspace holds their arrays
    const bool split = opt && split_fits(n_poses, p->draws, p) &&
                       workspace_bytes >= search_ws_bytes(n_points, n_poses, p, true);
    const SearchWs ws = search_ws(workspace, n_points, n_poses, p->draws, opt, p->k, opt ? p->opt_inner : 0, split);
    const int64_t row = (int64_t)H.F * NW;
    for (int64_t g0 = 0; g0 < n_poses; g0 += kMaxGridPoses) {
        const int64_t s0 = g0 * p->draws;
        hipLaunchKernelGGL(k_draw, dim3((unsigned)std::min<int64_t>(n_poses - g0, kMaxGridPoses)), dim3(kDrawThreads),
                           lds, s, H, pts, nrm, n_points, poses + 12 * g0, dom_bits + row * g0, dom_count + H.F * g0,
                           palm ? palm + g0 : nullptr, p->draws, p->k, (uint32_t)p->seed, (uint32_t)(p->seed >> 32),
                           p->request_id, p->pose_offset + g0, set_pt + s0 * p->k, set_link + s0 * p->k,
                           ws.pose_valid + g0, verdict + s0, tstar + s0);
    }
    LG_HIP(hipGetLastError());
    // list of poses with at least k non-empty domains (ordered)
    lg_status st = compact(ws.pose_valid, n_poses, ws.pchunk_count, ws.pchunk_off, ws.valid_poses, ws.n_valid_poses, s);
    if (st != LG_OK) return st;
    const int64_t n_sets = (int64_t)n_poses * p->draws;
    const LpConst cs = lp_const(p->m_edges);
    // grid-stride LP launch sized to the device (the valid count is on the device)
    int dev = 0, n_cu = 0;
    LG_HIP(hipGetDevice(&dev));
    LG_HIP(hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev));
    const dim3 lgrid(verdict_blocks(n_sets, n_cu));
    // the common 8-edge cone gets kernels that price a contact's best edge in closed form
    const bool m8 = p->m_edges == 8;
#define LG_VERDICT_M(KM, MC)                                                                                    \
    hipLaunchKernelGGL((k_verdict_lane<KM, MC>), lgrid, dim3(256), 0, s, pts, nrm, n_points, set_pt, palm,       \
                       ws.valid_poses,                                                                          \
                       ws.n_valid_poses, p->draws, p->k, p->m_edges, (double)p->mu, (double)p->moment_scale,     \
                       (double)p->eps, p->max_pivots, cs, verdict, tstar)
#define LG_VERDICT(KM) if (m8) LG_VERDICT_M(KM, 8); else LG_VERDICT_M(KM, 0)
    if (!opt) {
        if (kk <= 3) { LG_VERDICT(3); } else if (kk <= 4) { LG_VERDICT(4); } else if (kk <= 5) { LG_VERDICT(5); }
        else if (kk <= 6) { LG_VERDICT(6); } else { LG_VERDICT(8); }
    } else {
        // cell grid of the object, then Alg. 2 on the drawn sets, then the links of the moved contacts
        const int64_t ncell = kGridCells;
        hipLaunchKernelGGL(k_grid_setup, dim3(1), dim3(1024), 0, s, pts, n_points, p->opt_sigma, ws.grid);
        // zeroed by a kernel, not a memset node (callers may capture the stream in a graph)
        hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)((ncell + 255) / 256)), dim3(256), 0, s, ws.cell_count,
                           ncell, 0u);
        const unsigned pb = (unsigned)((n_points + 255) / 256);
        hipLaunchKernelGGL(k_grid_count, dim3(pb), dim3(256), 0, s, pts, n_points, ws.grid, ws.cell_count);
        hipLaunchKernelGGL(k_grid_rows, dim3(256), dim3(256), 0, s, ws.cell_count, ws.grid, ws.cell_start);
        hipLaunchKernelGGL(k_grid_scatter, dim3(pb), dim3(256), 0, s, pts, n_points, ws.grid, ws.cell_count,
                           ws.cell_pts);
        const int gs = p->opt_inner <= 1 ? 1 : p->opt_inner <= 2 ? 2 : p->opt_inner <= 4 ? 4 : p->opt_inner <= 8 ? 8 : 16;
        const dim3 ogrid((unsigned)std::max<int64_t>(
            1, std::min<int64_t>((n_sets * gs + 255) / 256, (int64_t)n_cu * 8)));
        // projections: kProjSets sets per wave, or waves that fill the chip (seven per SIMD) as far as there
        // are 8 candidates for each
        const int fill = n_cu * 28;
        const int64_t whole = (n_sets + 4 * kProjSets - 1) / (4 * kProjSets);
        const int64_t split8 = (n_sets * ((p->k * p->opt_inner + 7) / 8) + 3) / 4;
        const dim3 pgrid((unsigned)std::max<int64_t>(
            1, std::min<int64_t>(std::max(whole, std::min<int64_t>(split8, fill / 4)), (int64_t)n_cu * 64)));
        // grids of the per-candidate criteria (candidates; sets)
        const dim3 cgrid(verdict_blocks(n_sets * p->opt_inner, n_cu));
        const dim3 sgrid((unsigned)std::max<int64_t>(1, std::min<int64_t>((n_sets + 255) / 256, (int64_t)n_cu * 8)));
#define LG_OPT_M(KM, GS, MC)                                                                                     \
    hipLaunchKernelGGL((k_optimize<KM, GS, MC>), ogrid, dim3(256), 0, s, pts, nrm, n_points, ws.valid_poses,       \
                       ws.n_valid_poses, dom_count, palm, H.F, p->draws, p->k, p->m_edges, (double)p->mu,         \
                       (double)p->moment_scale, (double)p->eps, p->max_pivots, cs, p->opt_inner,                  \
                       r == p->opt_outer - 1, (uint32_t)p->seed, (uint32_t)(p->seed >> 32), p->request_id,        \
                       p->pose_offset, ws.cands, set_pt, verdict, tstar)
#define LG_OPT(KM, GS) LG_OPT_M(KM, GS, 0)
#define LG_OPT_K(GS)                                                                                             \
    if (kk <= 3) LG_OPT(3, GS); else if (kk <= 4) LG_OPT(4, GS); else if (kk <= 5) LG_OPT(5, GS);              \
    else if (kk <= 6) LG_OPT(6, GS); else LG_OPT(8, GS)
#define LG_OPT_K8                                                                                                \
    if (kk <= 3) LG_OPT_M(3, 8, 8); else if (kk <= 4) LG_OPT_M(4, 8, 8); else if (kk <= 5) LG_OPT_M(5, 8, 8);  \
    else if (kk <= 6) LG_OPT_M(6, 8, 8); else LG_OPT_M(8, 8, 8)
        for (int r = 0; r < p->opt_outer; ++r) {
            hipLaunchKernelGGL(k_opt_project, pgrid, dim3(256), 0, s, pts, nrm, n_points, ws.valid_poses,
                               ws.n_valid_poses, dom_bits, dom_count, palm, H.F, p->draws, p->k, r, p->opt_inner,
                               (double)p->opt_sigma, (uint32_t)p->seed, (uint32_t)(p->seed >> 32), p->request_id,
                               p->pose_offset, ws.grid, ws.cell_start, ws.cell_pts, set_pt, fill, ws.cands);
            if (split) {
                const lg_status so = opt_split_round(pts, nrm, n_points, ws, dom_count, palm, H.F, p, kk, m8, cs,
                                                     sgrid, cgrid, r == p->opt_outer - 1, set_pt, verdict, tstar, s);
                if (so != LG_OK) return so;
                continue;
            }
            if (gs == 1) { LG_OPT_K(1); } else if (gs == 2) { LG_OPT_K(2); } else if (gs == 4) { LG_OPT_K(4); }
            else if (gs == 8 && m8) { LG_OPT_K8; } else if (gs == 8) { LG_OPT_K(8); } else { LG_OPT_K(16); }
        }
#undef LG_OPT_K8
#undef LG_OPT_K
#undef LG_OPT
#undef LG_OPT_M
        LG_HIP(hipGetLastError());
        hipLaunchKernelGGL(k_relink, sgrid, dim3(256), 0, s, H, pts, nrm, n_points, poses,
                           ws.valid_poses, ws.n_valid_poses, dom_count, p->draws, p->k, (uint32_t)p->seed,
                           (uint32_t)(p->seed >> 32), p->request_id, p->pose_offset, set_pt, set_link);
    }
#undef LG_VERDICT
#undef LG_VERDICT_M
    LG_HIP(hipGetLastError());
    return compact(verdict, n_sets, ws.chunk_count, ws.chunk_off, acc_list, n_acc, s);
}

// Bytes of device workspace of lg_compact_unstable: set flags, chunk counts and offsets.
static size_t unstable_ws_bytes(int64_t n_sets)
{
    const int64_t nc = (n_sets + kChunk - 1) / kChunk;
    return (((size_t)n_sets + 255) & ~(size_t)255) + (size_t)(2 * nc) * 4 + 256;
}

extern "C" {

size_t lg_compact_unstable_workspace_bytes(int32_t n_poses, int32_t draws)
{
    if (n_poses <= 0 || draws <= 0) return 256;
    return unstable_ws_bytes((int64_t)n_poses * draws);
}

lg_status lg_compact_unstable(const int32_t *set_pt, const int8_t *set_link, const uint8_t *verdict, int32_t n_poses,
                              int32_t draws, int32_t k, int32_t *list, int32_t *n_list, void *workspace,
                              size_t workspace_bytes, void *stream)
{
    if (n_poses < 0 || draws <= 0 || k < 1 || k > 8) return fail(LG_EINVAL, "need n_poses >= 0, draws > 0, 1 <= k <= 8");
    if ((int64_t)n_poses * draws > 0x7fffffffLL) return fail(LG_EINVAL, "P * D must be < 2^31");
    if (!n_list) return fail(LG_EINVAL, "null n_list");
    hipStream_t s = as_stream(stream);
    const int64_t n_sets = (int64_t)n_poses * draws;
    if (n_sets == 0) {  // a count of 0 (a kernel, not a memset node, for callers that capture the stream)
        hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(64), 0, s, reinterpret_cast<uint32_t *>(n_list), (int64_t)1, 0u);
        LG_HIP(hipGetLastError());
        return LG_OK;
    }
    if (!set_pt || !set_link || !verdict || !list || !workspace) return fail(LG_EINVAL, "null device buffer");
    if (workspace_bytes < unstable_ws_bytes(n_sets)) return fail(LG_EINVAL, "workspace too small");
    uint8_t *flag = static_cast<uint8_t *>(workspace);
    uint32_t *cc = reinterpret_cast<uint32_t *>(flag + (((size_t)n_sets + 255) & ~(size_t)255));
    const int64_t nc = (n_sets + kChunk - 1) / kChunk;
    hipLaunchKernelGGL(k_flag_unstable, dim3((unsigned)((n_sets + 255) / 256)), dim3(256), 0, s, set_pt, set_link,
                       verdict, n_sets, k, flag);
    LG_HIP(hipGetLastError());
    return compact(flag, n_sets, cc, cc + nc, list, n_list, s);
}

lg_status lg_search_extend(const lg_field *field, const float *pts, const float *nrm, int32_t n_points,
                           const float *poses, int32_t n_poses, const uint32_t *dom_bits, const uint32_t *dom_count,
                           const lg_search_params *p, const int32_t *set_pt1, const int8_t *set_link1,
                           const uint8_t *verdict1, const lg_extend_params *ep, int32_t *set_pt2, int8_t *set_link2,
                           uint8_t *verdict2, double *tstar2, int32_t *acc_list2, int32_t *n_acc2, void *workspace,
                           size_t workspace_bytes, void *stream)
{
    if (!field || !p || !ep) return fail(LG_EINVAL, "null field or params");
    const DevHand &H = field->dh;
    if (n_points <= 0 || n_poses < 0) return fail(LG_EINVAL, "n_points must be > 0 and n_poses >= 0");
    const int k1 = p->k, k2 = p->k + ep->k_add;
    if (k1 < 1 || ep->k_add < 1 || k2 > H.F || k2 > 8)
        return fail(LG_EINVAL, "need k >= 1, k_add >= 1 and k + k_add <= number of fingers (and <= 8)");
    if (p->palm_pt) return fail(LG_EUNSUPPORTED, "the second contact round takes no palm contacts");
    if (p->draws <= 0 || p->m_edges < 3 || p->m_edges > 16 || !(p->mu >= 0.0f) || !(p->moment_scale > 0.0f) ||
        p->max_pivots < 0)
        return fail(LG_EINVAL, "need draws > 0, 3 <= m_edges <= 16, mu >= 0, moment_scale > 0, max_pivots >= 0");
    if ((int64_t)n_poses * p->draws > 0x7fffffffLL) return fail(LG_EINVAL, "P * D must be < 2^31");
    if (n_poses == 0) return LG_OK;
    if (!pts || !nrm || !poses || !dom_bits || !dom_count || !set_pt1 || !set_link1 || !verdict1 || !set_pt2 ||
        !set_link2 || !verdict2 || !tstar2 || !acc_list2 || !n_acc2 || !workspace)
        return fail(LG_EINVAL, "null device buffer");
    if (ep->list && !ep->list_n) return fail(LG_EINVAL, "a set list needs its device count");
    lg_search_params p2 = *p;
    p2.k = k2;
    p2.opt_outer = 0;
    if (workspace_bytes < lg_search_workspace_bytes(n_points, n_poses, &p2)) return fail(LG_EINVAL, "workspace too small");
    const int NW = (n_points + 31) / 32, nsb = (NW + kSuper - 1) / kSuper;
    const size_t lds = (size_t)H.F * (nsb + 1) * sizeof(uint32_t);
    if (lds > 48 * 1024) return fail(LG_EUNSUPPORTED, "too many points for the draw rank structure");
    hipStream_t s = as_stream(stream);
    const SearchWs ws = search_ws(workspace, n_points, n_poses, p->draws, false);
    for (int64_t g0 = 0; g0 < n_poses; g0 += kMaxGridPoses)
        hipLaunchKernelGGL(k_extend, dim3((unsigned)std::min<int64_t>(n_poses - g0, kMaxGridPoses)), dim3(kDrawThreads),
                           lds, s, H, pts, nrm, n_points, (int)g0, poses, dom_bits, dom_count, p->draws, k1, ep->k_add,
                           set_pt1, set_link1, verdict1, ep->list, ep->list_n, ep->list_ok, (uint32_t)p->seed,
                           (uint32_t)(p->seed >> 32), ep->request_id, p->pose_offset, set_pt2, set_link2,
                           ws.pose_valid, verdict2, tstar2);
    LG_HIP(hipGetLastError());
    const lg_status st =
        compact(ws.pose_valid, n_poses, ws.pchunk_count, ws.pchunk_off, ws.valid_poses, ws.n_valid_poses, s);
    if (st != LG_OK) return st;
    const int64_t n_sets = (int64_t)n_poses * p->draws;
    LpConst cs;
    for (int e = 0; e < 16; ++e) {
        const double th = 2.0 * M_PI * e / p->m_edges;
        cs.ce[e] = e < p->m_edges ? cos(th) : 0.0;
        cs.se[e] = e < p->m_edges ? sin(th) : 0.0;
    }
    int dev = 0, n_cu = 0;
    LG_HIP(hipGetDevice(&dev));
    LG_HIP(hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev));
    const dim3 lgrid(verdict_blocks(n_sets, n_cu));
    const bool m8 = p->m_edges == 8;
#define LG_VERDICT2_M(KM, MC)                                                                                   \
    hipLaunchKernelGGL((k_verdict_lane<KM, MC>), lgrid, dim3(256), 0, s, pts, nrm, n_points, set_pt2, nullptr,    \
                       ws.valid_poses, ws.n_valid_poses, p->draws, k2, p->m_edges, (double)p->mu,                \
                       (double)p->moment_scale, (double)p->eps, p->max_pivots, cs, verdict2, tstar2)
#define LG_VERDICT2(KM) if (m8) LG_VERDICT2_M(KM, 8); else LG_VERDICT2_M(KM, 0)
    if (k2 <= 3) { LG_VERDICT2(3); } else if (k2 <= 4) { LG_VERDICT2(4); } else if (k2 <= 5) { LG_VERDICT2(5); }
    else if (k2 <= 6) { LG_VERDICT2(6); } else { LG_VERDICT2(8); }
#undef LG_VERDICT2
#undef LG_VERDICT2_M
    LG_HIP(hipGetLastError());
    return compact(verdict2, n_sets, ws.chunk_count, ws.chunk_off, acc_list2, n_acc2, s);
}

}  // extern "C"

// Scratch of lg_search_noalloc: one array per device, held until the process
// ends.  Host code never passes the array's name to a kernel (on the host it
// is only a stand-in symbol); it uses the device address that
// hipGetSymbolAddress returns, looked up once per device.
constexpr size_t kStaticScratchBytes = (size_t)8 << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

static lg_status scratch_address(void **out)
{
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static void *addr[kMaxDevices] = {};
    int dev = 0;
    LG_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return fail(LG_EUNSUPPORTED, "device index beyond the scratch table");
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[dev]) {
        void *ptr = nullptr;
        LG_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
        if (!ptr) return fail(LG_EDEVICE, "no device address for the static scratch array");
        addr[dev] = ptr;
    }
    *out = addr[dev];
    return LG_OK;
}

extern "C" {

size_t lg_search_noalloc_max_bytes(void) { return kStaticScratchBytes; }

lg_status lg_search(const lg_field *field, const float *pts, const float *nrm, int32_t n_points, const float *poses,
                    int32_t n_poses, const uint32_t *dom_bits, const uint32_t *dom_count,
                    const lg_search_params *p, int32_t *set_pt, int8_t *set_link, uint8_t *verdict, double *tstar,
                    int32_t *acc_list, int32_t *n_acc, void *workspace, size_t workspace_bytes, void *stream)
{
    return search_impl(field, pts, nrm, n_points, poses, n_poses, dom_bits, dom_count, p, set_pt, set_link, verdict,
                       tstar, acc_list, n_acc, workspace, workspace_bytes, stream);
}

lg_status lg_search_noalloc(const lg_field *field, const float *pts, const float *nrm, int32_t n_points,
                            const float *poses, int32_t n_poses, const uint32_t *dom_bits, const uint32_t *dom_count,
                            const lg_search_params *p, int32_t *set_pt, int8_t *set_link, uint8_t *verdict,
                            double *tstar, int32_t *acc_list, int32_t *n_acc, void *stream)
{
    if (!p) return fail(LG_EINVAL, "null params");
    const size_t need = search_ws_bytes(n_points, n_poses, p, false);  // the least a search runs in
    if (need > kStaticScratchBytes)
        return fail(LG_EINVAL, "search needs " + std::to_string(need) + " bytes of workspace, above the " +
                                   std::to_string(kStaticScratchBytes) + "-byte static scratch");
    void *ws = nullptr;
    const lg_status st = scratch_address(&ws);
    if (st != LG_OK) return st;
    return search_impl(field, pts, nrm, n_points, poses, n_poses, dom_bits, dom_count, p, set_pt, set_link, verdict,
                       tstar, acc_list, n_acc, ws, kStaticScratchBytes, stream);
}

}  // extern "C"

// ---- batched launches over the chunks of several requests -------------------
size_t lg::draw_lds_bytes(int F, int N)
{
    const int NW = (N + 31) / 32, nsb = (NW + kSuper - 1) / kSuper;
    return (size_t)F * (nsb + 1) * sizeof(uint32_t);
}

uint32_t lg::compact_blocks(int64_t n) { return (uint32_t)((n + kChunk - 1) / kChunk); }

lg_status lg::draw_batch(const BatchLaunch &b, size_t lds, hipStream_t s)
{
    if (b.n <= 0 || b.blocks == 0) return LG_OK;
    if (lds > 48 * 1024) return fail(LG_EUNSUPPORTED, "too many points for the draw rank structure");
    hipLaunchKernelGGL(k_draw_batch, dim3(b.blocks), dim3(kDrawThreads), lds, s, b.d, b.idx, b.first, b.n);
    LG_HIP(hipGetLastError());
    return LG_OK;
}

int lg::compact_form(int64_t n)
{
    return n <= kCompactOneMax ? 0 : (n + kChunk - 1) / kChunk <= kSelfScanMax ? 1 : 2;
}

lg_status lg::compact_batch(const BatchLaunch &chunks, const BatchLaunch &ones, int form, bool poses, hipStream_t s)
{
    if (ones.n <= 0 || ones.blocks == 0) return LG_OK;
#define LG_COMPACT(K, B, T, ...)                                                                                 \
    do {                                                                                                         \
        if (poses)                                                                                               \
            hipLaunchKernelGGL(K<true>, dim3(B.blocks), dim3(T), 0, s, B.d, B.idx, B.first, B.n __VA_ARGS__);   \
        else                                                                                                     \
            hipLaunchKernelGGL(K<false>, dim3(B.blocks), dim3(T), 0, s, B.d, B.idx, B.first, B.n __VA_ARGS__);  \
    } while (0)
    if (form == 0) {
        LG_COMPACT(k_compact_batch, ones, kCompactOneThreads);
    } else {
        LG_COMPACT(k_count_batch, chunks, kCompactThreads);
        if (form == 2) LG_COMPACT(k_scan_batch, ones, kCompactThreads);
        LG_COMPACT(k_scatter_batch, chunks, kCompactThreads, , form == 1);
    }
#undef LG_COMPACT
    LG_HIP(hipGetLastError());
    return LG_OK;
}

lg_status lg::verdict_batch(const BatchLaunch &b, int km, bool m8, hipStream_t s)
{
    if (b.n <= 0 || b.blocks == 0) return LG_OK;
#define LG_VB_M(KM, MC)                                                                                          \
    hipLaunchKernelGGL((k_verdict_batch<KM, MC>), dim3(b.blocks), dim3(256), 0, s, b.d, b.idx, b.first, b.n)
#define LG_VB(KM) if (m8) LG_VB_M(KM, 8); else LG_VB_M(KM, 0)
    if (km <= 3) { LG_VB(3); } else if (km <= 4) { LG_VB(4); } else if (km <= 5) { LG_VB(5); }
    else if (km <= 6) { LG_VB(6); } else { LG_VB(8); }
#undef LG_VB
#undef LG_VB_M
    LG_HIP(hipGetLastError());
    return LG_OK;
}
