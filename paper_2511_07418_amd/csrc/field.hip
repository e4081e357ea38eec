// Contact-field construction (Sec. 4.3, Alg. 1; fine-grained per-patch
// fields of Sec. 4.4) and the field object's life cycle.
//
// Alg. 1 organises sampled contact vectors in a box cover of width w and a
// BVH, with the normals of each box stored in its leaf.  On gfx950 the cover
// is a dense G^3 window per finger (O(1) addressing, no BVH traversal) and a
// leaf's normal list is a B-bit mask over a spherical Fibonacci lattice (the
// quantised normals of Sec. 4.4), so one 4- or 8-byte word answers a query.
// All links of a finger share the finger's window, so the finger-level OR of
// the link tables (the merged domain of a dependency group, Sec. 5.3) is a
// table of its own and the query reads one word per finger.
#include <math.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <cmath>
#include <mutex>

#include "lg_internal.h"

namespace lg {

static thread_local std::string g_last_error;

lg_status fail(lg_status s, const std::string &msg)
{
    g_last_error = msg;
    return s;
}

lg_status hip_fail(hipError_t e, const char *what)
{
    g_last_error = std::string(what) + ": " + hipGetErrorString(e);
    return e == hipErrorOutOfMemory ? LG_ENOMEM : LG_EDEVICE;
}

lg_status validate_hand(const lg_hand_desc *hand, const lg_field_params *p)
{
    if (!hand || !p) return fail(LG_EINVAL, "null hand or params");
    const int F = hand->n_fingers, J = hand->n_joints;
    if (F < 1 || F > kMaxFingers) return fail(LG_EINVAL, "n_fingers must be 1..8");
    if (J < F || J > kMaxJoints) return fail(LG_EINVAL, "n_joints must be F..64");
    if (!hand->joint_finger || !hand->joint_parent || !hand->joint_origin || !hand->joint_axis ||
        !hand->capsule || !hand->limits || !hand->surf)
        return fail(LG_EINVAL, "null hand array");
    if (hand->n_surf < 1 || hand->n_surf > 65536) return fail(LG_EINVAL, "n_surf must be 1..65536");
    int prev_f = -1, dof = 0;
    for (int j = 0; j < J; ++j) {
        const int f = hand->joint_finger[j];
        if (f < 0 || f >= F) return fail(LG_EINVAL, "joint_finger out of range");
        if (f != prev_f) {
            if (f != prev_f + 1) return fail(LG_EINVAL, "fingers must be stored contiguously in order");
            if (hand->joint_parent[j] != -1) return fail(LG_EINVAL, "first joint of a finger must have parent -1");
            dof = 0;
            prev_f = f;
        } else if (hand->joint_parent[j] != j - 1) {
            return fail(LG_EINVAL, "a finger must be a serial chain (parent = j - 1)");
        }
        if (++dof > kMaxDof) return fail(LG_EINVAL, "at most 8 joints per finger");
        if (!(hand->limits[2 * j] <= hand->limits[2 * j + 1])) return fail(LG_EINVAL, "limits lo > hi");
    }
    if (prev_f != F - 1) return fail(LG_EINVAL, "every finger needs at least one joint");
    if (hand->n_palm_surf < 0 || hand->n_palm_caps < 0 || (hand->n_palm_surf > 0 && !hand->palm_surf) ||
        (hand->n_palm_caps > 0 && !hand->palm_caps) || hand->n_palm_surf > (1 << 20) || hand->n_palm_caps > 1024)
        return fail(LG_EINVAL, "palm: need 0 <= n_palm_surf <= 2^20, 0 <= n_palm_caps <= 1024 and their arrays");
    for (int c = 0; c < hand->n_palm_caps; ++c)
        if (!(hand->palm_caps[7 * c + 6] >= 0.0f)) return fail(LG_EINVAL, "palm capsule radius must be >= 0");
    if (p->bins != 32 && p->bins != 64) return fail(LG_EINVAL, "bins must be 32 or 64");
    if (p->grid < 4 || p->grid > 128 || p->grid % 4 != 0) return fail(LG_EINVAL, "grid must be a multiple of 4 in 4..128");
    if (!(p->h > 0.0f)) return fail(LG_EINVAL, "h must be > 0");
    if (p->samples < 1 || p->samples > 0x7fffffffLL) return fail(LG_EINVAL, "samples must be 1..2^31-1");
    if (!p->grid_frame) return fail(LG_EINVAL, "null grid_frame");
    return LG_OK;
}

void free_field(lg_field *f)
{
    if (!f) return;
    int cur = 0;
    (void)hipGetDevice(&cur);
    (void)hipSetDevice(f->device);
    (void)hipFree(f->d_params);
    (void)hipFree(f->d_axis_samples);
    (void)hipFree(f->d_bits);
    (void)hipFree(f->d_merged);
    (void)hipFree(f->d_wit);
    (void)hipFree(f->d_cull);
    (void)hipFree(f->d_mask);
    (void)hipSetDevice(cur);
    delete f;
}

__global__ void k_fill_i32(int32_t *__restrict__ p, int64_t n, int32_t v)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = v;
}

// Candidate table of the normal bins over a cube map of directions, in the
// GPU's own cube-map convention (the v_cube* instructions the query uses): a
// direction d goes to face f = 0..5 (+x, -x, +y, -y, +z, -z; on ties z before
// y before x) and face coordinates (s, t) in [-1, 1]^2, s = sc / |d_major|,
// t = tc / |d_major|, with
//   +x: d ~ (1, -t, -s)   -x: d ~ (-1, -t, s)   +y: d ~ (s, 1, t)
//   -y: d ~ (s, -1, -t)   +z: d ~ (s, -t, 1)    -z: d ~ (-s, -t, -1),
// and to cell (is, it) of a kLutRes x kLutRes grid over (s, t).  A cell lists,
// in increasing order, every bin that can be the best anywhere in the closed cell:
// at some point of a dense sub-grid of the cell its dot product is within reach of the
// best bin's a there, that is within |c_b - c_a| times the distance to the farthest
// direction the point stands for (the dot products' difference changes by no more; a
// cube's points are at least as far apart as their directions), plus a margin for
// float products and a direction on a cell or face boundary.  So the argmax over the
// candidates equals the argmax over all bins.  With the pair's own reach instead of
// twice the sub-grid's step 5 % of the cells hold more than two bins (16 %).  Their
// entries have the top bit set, cells with more than four candidates are marked for
// the full search (0xffffffff).
__device__ inline void cube_direction(int face, double s, double t, double *d)
{
    switch (face) {
    case 0: d[0] = 1.0; d[1] = -t; d[2] = -s; break;
    case 1: d[0] = -1.0; d[1] = -t; d[2] = s; break;
    case 2: d[0] = s; d[1] = 1.0; d[2] = t; break;
    case 3: d[0] = s; d[1] = -1.0; d[2] = -t; break;
    case 4: d[0] = s; d[1] = -t; d[2] = 1.0; break;
    default: d[0] = -s; d[1] = -t; d[2] = -1.0; break;
    }
}

constexpr int kLutSub = 9;  // sub-grid points per cell edge, both edges included

// One wave per cell, lanes over its sub-grid points; a lane marks the bins near
// the best at its points, the marks are joined by shuffles: 90 us, 30 ms on one
// CPU thread.
__global__ void __launch_bounds__(64) k_bin_lut(const float *__restrict__ bc, int B, uint32_t *__restrict__ lut)
{
    const int R = kLutRes, cell = blockIdx.x, lane = threadIdx.x;
    const int is = cell % R, it = cell / R % R, face = cell / (R * R);
    const double sub_step = 2.0 / R / (kLutSub - 1);   // in face coordinates
    const double reach = 0.5 * sqrt(2.0) * sub_step;    // to the farthest direction of a sub-grid point
    unsigned long long cand = 0;
    for (int q = lane; q < kLutSub * kLutSub; q += 64) {
        const double sv = -1.0 + 2.0 * (is + (double)(q % kLutSub) / (kLutSub - 1)) / R;
        const double tv = -1.0 + 2.0 * (it + (double)(q / kLutSub) / (kLutSub - 1)) / R;
        double d[3];
        cube_direction(face, sv, tv, d);
        const double rn = 1.0 / sqrt(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]);
        double best = -2.0;
        int a = 0;
        for (int b = 0; b < B; ++b) {
            const double v = (bc[3 * b] * d[0] + bc[3 * b + 1] * d[1] + bc[3 * b + 2] * d[2]) * rn;
            if (v > best) {
                best = v;
                a = b;
            }
        }
        for (int b = 0; b < B; ++b) {
            const double v = (bc[3 * b] * d[0] + bc[3 * b + 1] * d[1] + bc[3 * b + 2] * d[2]) * rn;
            const double ex = (double)bc[3 * b] - bc[3 * a], ey = (double)bc[3 * b + 1] - bc[3 * a + 1],
                         ez = (double)bc[3 * b + 2] - bc[3 * a + 2];
            if (v >= best - reach * sqrt(ex * ex + ey * ey + ez * ez) - 1e-4) cand |= 1ull << b;
        }
    }
    for (int off = 32; off > 0; off >>= 1) cand |= __shfl_xor(cand, off, 64);
    if (lane != 0) return;
    uint32_t e = 0xffffffffu;
    if (__popcll(cand) <= 4) {
        // absent slots repeat the first candidate
        const int first = __ffsll((long long)cand) - 1;
        e = __popcll(cand) > 2 ? 0x80000000u : 0u;
        for (int i = 0; i < 4; ++i) {
            const int b = cand ? __ffsll((long long)cand) - 1 : first;
            cand &= cand - 1;
            e |= (uint32_t)b << (8 * i);
        }
    }
    lut[cell] = e;
}

// Lattice form of the windows (see DevHand::lat): every frame has finger 0's
// rotation (same floats), G is a power of two, and each origin is a whole
// number of 4-voxel bricks from finger 0's, within 1e-4 voxel (a few float
// ulps of the origins; the window faces move by far less than the 1e-6 m
// bands in which the oracle flags voxel decisions).  Otherwise lat = 0 and
// every kernel maps each finger's window on its own.
static void set_lattice(DevHand &H, const float *gf)
{
    H.lat = 0;
    const int F = H.F, G = H.G;
    if (G < 4 || (G & (G - 1)) != 0) return;
    for (int f = 1; f < F; ++f)
        for (int r = 0; r < 3; ++r)
            for (int c = 0; c < 3; ++c)
                if (gf[12 * f + 4 * r + c] != gf[4 * r + c]) return;
    long k[kMaxFingers][3];
    long lo[3] = {0, 0, 0}, hi[3] = {0, 0, 0};
    for (int f = 0; f < F; ++f) {
        const double d[3] = {(double)gf[12 * f + 3] - gf[3], (double)gf[12 * f + 7] - gf[7],
                             (double)gf[12 * f + 11] - gf[11]};
        for (int a = 0; a < 3; ++a) {
            // a-th coordinate in finger 0's frame: column a of its rotation
            const double u = (gf[a] * d[0] + gf[4 + a] * d[1] + gf[8 + a] * d[2]) / (double)H.h;
            const double r = 4.0 * std::nearbyint(u / 4.0);
            if (!(std::fabs(u - r) <= 1e-4) || std::fabs(r) > 4096.0) return;
            k[f][a] = (long)r;
            lo[a] = std::min(lo[a], k[f][a]);
            hi[a] = std::max(hi[a], k[f][a]);
        }
    }
    for (int a = 0; a < 3; ++a)
        if (hi[a] - lo[a] + 3L * G > 1024L) return;
    const uint32_t GB = (uint32_t)(G / 4), m = (uint32_t)(G - 1);
    for (int f = 0; f < F; ++f) {
        for (int a = 0; a < 3; ++a) H.lat_o[f][a] = (int)(k[f][a] - lo[a] + G);
        H.lat_pk[f] = (uint32_t)H.lat_o[f][0] | (uint32_t)H.lat_o[f][1] << 10 | (uint32_t)H.lat_o[f][2] << 20;
        H.lat_idx[f] = brick_word((uint32_t)H.lat_o[f][0], (uint32_t)H.lat_o[f][1], (uint32_t)H.lat_o[f][2], GB);
    }
    H.lat_hi = ~(m | m << 10 | m << 20);
    H.lat = 1;
}

// Copy the hand, compute bin centres and axis sample counts on the host,
// upload them and allocate the (zeroed) tables.
lg_status make_field_shell(const lg_hand_desc *hand, const lg_field_params *p, lg_field **out)
{
    lg_status st = validate_hand(hand, p);
    if (st != LG_OK) return st;
    if (!out) return fail(LG_EINVAL, "null out");
    lg_field *f = new lg_field();
    const int F = hand->n_fingers, J = hand->n_joints, G = p->grid, B = p->bins, S = hand->n_surf;
    (void)hipGetDevice(&f->device);
    f->joint_finger.assign(hand->joint_finger, hand->joint_finger + J);
    f->joint_parent.assign(hand->joint_parent, hand->joint_parent + J);
    f->origin.assign(hand->joint_origin, hand->joint_origin + 12 * J);
    f->axis.assign(hand->joint_axis, hand->joint_axis + 3 * J);
    f->capsule.assign(hand->capsule, hand->capsule + 7 * J);
    f->limits.assign(hand->limits, hand->limits + 2 * J);
    f->surf.assign(hand->surf, hand->surf + (size_t)6 * J * S);
    f->grid_frame.assign(p->grid_frame, p->grid_frame + 12 * F);
    const int PS = hand->n_palm_surf, PC = hand->n_palm_caps;
    if (PS > 0) f->palm_surf.assign(hand->palm_surf, hand->palm_surf + (size_t)6 * PS);
    if (PC > 0) f->palm_caps.assign(hand->palm_caps, hand->palm_caps + (size_t)7 * PC);
    // spherical Fibonacci lattice, evaluated in double and rounded once
    f->bin_c.resize(3 * B);
    const double golden = M_PI * (3.0 - sqrt(5.0));
    for (int b = 0; b < B; ++b) {
        const double z = 1.0 - (2.0 * b + 1.0) / B, r = sqrt(1.0 - z * z), ph = b * golden;
        f->bin_c[3 * b] = (float)(r * cos(ph));
        f->bin_c[3 * b + 1] = (float)(r * sin(ph));
        f->bin_c[3 * b + 2] = (float)z;
    }
    // capsule axis samples for the penetration test: one per mm, ends included
    // (links, then the palm's capsules, which take at least their two ends)
    f->axis_samples.resize(J + PC);
    for (int j = 0; j < J + PC; ++j) {
        const float *c = j < J ? hand->capsule + 7 * j : hand->palm_caps + 7 * (j - J);
        const double dx = (double)c[3] - c[0], dy = (double)c[4] - c[1], dz = (double)c[5] - c[2];
        const double L = sqrt((dx * dx + dy * dy) + dz * dz);
        f->axis_samples[j] = std::max((int32_t)ceil(L / 1e-3) + 1, j < J ? 1 : 2);
    }
    DevHand &H = f->dh;
    memset(&H, 0, sizeof H);
    H.F = F;
    H.J = J;
    H.G = G;
    H.B = B;
    H.W = B / 32;
    H.nsurf = S;
    H.h = p->h;
    H.inv_h = 1.0f / p->h;
    H.seed_lo = (uint32_t)p->seed;
    H.seed_hi = (uint32_t)(p->seed >> 32);
    H.samples = p->samples;
    int maxd = 0;
    for (int fi = 0; fi < F; ++fi) {
        int first = -1, d = 0;
        for (int j = 0; j < J; ++j)
            if (hand->joint_finger[j] == fi) {
                if (first < 0) first = j;
                ++d;
            }
        H.finger_first[fi] = first;
        H.finger_dof[fi] = d;
        maxd = std::max(maxd, d);
    }
    f->max_dof = maxd;
    set_lattice(H, p->grid_frame);
    // packed float parameters
    const size_t n_origin = f->origin.size(), n_axis = f->axis.size(), n_cap = f->capsule.size(),
                 n_lim = f->limits.size(), n_surf = f->surf.size(), n_gf = f->grid_frame.size(),
                 n_bc = f->bin_c.size(), n_ps = f->palm_surf.size(), n_pc = f->palm_caps.size();
    const size_t n_lut = 6 * kLutRes * kLutRes;  // filled on the device
    const size_t n_all = n_origin + n_axis + n_cap + n_lim + n_surf + n_gf + n_bc + n_ps + n_pc + n_lut;
    std::vector<float> packed;
    packed.reserve(n_all);
    for (auto *v : {&f->origin, &f->axis, &f->capsule, &f->limits, &f->surf, &f->grid_frame, &f->bin_c,
                    &f->palm_surf, &f->palm_caps})
        packed.insert(packed.end(), v->begin(), v->end());
    packed.resize(n_all);
    const int64_t G3 = (int64_t)G * G * G;
    hipError_t e = hipMalloc(&f->d_params, n_all * sizeof(float));
    if (e == hipSuccess) e = hipMemcpy(f->d_params, packed.data(), n_all * sizeof(float), hipMemcpyHostToDevice);
    if (e == hipSuccess) {
        hipLaunchKernelGGL(k_bin_lut, dim3((unsigned)n_lut), dim3(64), 0, nullptr,
                           f->d_params + (n_all - n_lut - n_pc - n_ps - n_bc), B,
                           reinterpret_cast<uint32_t *>(f->d_params + (n_all - n_lut)));
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipMalloc(&f->d_axis_samples, (J + PC) * sizeof(int32_t));
    if (e == hipSuccess)
        e = hipMemcpy(f->d_axis_samples, f->axis_samples.data(), (J + PC) * sizeof(int32_t), hipMemcpyHostToDevice);
    const size_t bits_bytes = (size_t)J * G3 * H.W * 4, merged_bytes = (size_t)F * G3 * H.W * 4;
    if (e == hipSuccess) e = hipMalloc(&f->d_bits, bits_bytes);
    if (e == hipSuccess) e = hipMalloc(&f->d_merged, merged_bytes);
    if (e == hipSuccess) e = hipMemset(f->d_bits, 0, bits_bytes);
    if (e == hipSuccess) e = hipMemset(f->d_merged, 0, merged_bytes);
    H.cull_row = (G + 31) / 32;
    const size_t cull_bytes = (size_t)(kCullLevels + 1) * F * G * G * H.cull_row * 4;
    if (e == hipSuccess) e = hipMalloc(&f->d_cull, cull_bytes);
    const size_t mask_bytes = (size_t)F * G3 * B;
    if (e == hipSuccess) e = hipMalloc(&f->d_mask, mask_bytes);
    size_t wit_bytes = 0;
    if (e == hipSuccess && p->keep_witness) {
        wit_bytes = (size_t)J * G3 * B * 4;
        e = hipMalloc(&f->d_wit, wit_bytes);
        if (e == hipSuccess) {
            hipLaunchKernelGGL(k_fill_i32, dim3(2048), dim3(256), 0, nullptr, f->d_wit, (int64_t)J * G3 * B, kNoWitness);
            e = hipGetLastError();
        }
        f->has_witness = true;
    }
    // the fills ran on the null stream; the caller's stream may not wait for it
    if (e == hipSuccess) e = hipDeviceSynchronize();
    if (e != hipSuccess) {
        st = hip_fail(e, "field allocation");
        free_field(f);
        return st;
    }
    f->device_bytes = n_all * 4 + (J + PC) * 4 + bits_bytes + merged_bytes + wit_bytes + cull_bytes + mask_bytes;
    float *base = f->d_params;
    H.origin = base;
    base += n_origin;
    H.axis = base;
    base += n_axis;
    H.capsule = base;
    base += n_cap;
    H.limits = base;
    base += n_lim;
    H.surf = base;
    base += n_surf;
    H.grid_frame = base;
    base += n_gf;
    H.bin_c = base;
    base += n_bc;
    H.palm_surf = n_ps ? base : nullptr;
    base += n_ps;
    H.palm_caps = n_pc ? base : nullptr;
    base += n_pc;
    H.bin_lut = reinterpret_cast<const uint32_t *>(base);
    H.axis_samples = f->d_axis_samples;
    H.cull = f->d_cull;
    H.link_mask = f->d_mask;
    H.n_palm_surf = PS;
    H.n_palm_caps = PC;
    *out = f;
    return LG_OK;
}

// ---------------------------------------------------------------------------
// kernels
// ---------------------------------------------------------------------------
constexpr int kBuildThreads = 256;
constexpr int64_t kBuildMaxParts = 16;
constexpr int64_t kBuildRound = 4096;  // samples of the first round; each further round doubles the total

// *out += the sum of c over the block of kBuildThreads threads: one atomic per
// block (all go to one address, some 10 ns each)
__device__ inline void block_add(unsigned int c, unsigned long long *__restrict__ out)
{
    __shared__ unsigned int part[kBuildThreads / 64];
    for (int off = 32; off > 0; off >>= 1) c += __shfl_down(c, off, 64);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long s = 0;
        for (int w = 0; w < kBuildThreads / 64; ++w) s += part[w];
        if (s) atomicAdd(out, s);
    }
}

// Thread per (link, joint sample, part of the link's surface) of a round: sample
// q, walk the chain to the link, and bin the part's surface samples (blockIdx.z
// of gridDim.z; a short round has several parts, or its threads' serial walk over
// 256 samples would leave the chip idle: 4,096 samples 0.55 ms with one).  done: the table as it was
// before this round (null: nothing yet, or no memory for it).  A vector whose bit is
// set there has a witness of an earlier, smaller sample, so it changes nothing and
// ends at one plain 4-byte read; only the others go on to the live table (whose reads
// pass by the caches) and to the 32 times larger witness table.  The check-before-atomic is safe because table bits only ever go
// 0 -> 1 and witnesses only decrease: a stale read can only cause a redundant
// atomic, never a lost update.
// What bounds it: the random reads.  All vectors against the witness table (1.4
// GiB at 22 links of 64^3 voxels x 64 bins, read from HBM a line per vector), with
// the bins by a scan of all 64 centres, took 41.9 ms for 262,144 samples; with the
// rounds (under 1 % of the vectors are the first of their cell), a link at a time (its
// 2 MiB of bits stay in L2) and the bins by the candidate table it takes 7.2 ms;
// without witnesses 36.9 ms with every vector against the live table, 6.0 ms so.
__global__ void __launch_bounds__(kBuildThreads)
k_field_build(DevHand H, int64_t s0, int64_t s1, const uint32_t *__restrict__ done, uint32_t *__restrict__ bits,
              int32_t *__restrict__ wit, unsigned long long *__restrict__ dropped)
{
    __shared__ float4 cb4[kMaxBins];
    __shared__ uint32_t lut[6 * kLutRes * kLutRes];
    for (int i = threadIdx.x; i < H.B; i += kBuildThreads)
        cb4[i] = make_float4(H.bin_c[3 * i], H.bin_c[3 * i + 1], H.bin_c[3 * i + 2], 0.0f);
    for (int i = threadIdx.x; i < 6 * kLutRes * kLutRes; i += kBuildThreads) lut[i] = H.bin_lut[i];
    __syncthreads();
    const int j = blockIdx.y;
    int f = 0;
    while (j >= H.finger_first[f] + H.finger_dof[f]) ++f;
    const int64_t s = s0 + (int64_t)blockIdx.x * kBuildThreads + threadIdx.x;
    const bool active = s < s1;
    const int first = H.finger_first[f];
    const int G = H.G, W = H.W, B = H.B;
    const int64_t G3 = (int64_t)G * G * G;
    const float *gf = H.grid_frame + 12 * f;
    unsigned int n_drop = 0;
    Tf T;
    for (int t = 0; first + t <= j; ++t) {
        const float q = active ? joint_sample(H, f, (uint32_t)s, t) : 0.0f;
        T = joint_frame(H, T, t > 0, first + t, q);
    }
    // composite link -> window map: u = R_f^T (T x - o_f) / h + G (biased, see window_voxel)
    Affine a;
    {
        const float dx = T.m[3] - gf[3], dy = T.m[7] - gf[7], dz = T.m[11] - gf[11];
#pragma unroll
        for (int r = 0; r < 3; ++r) {
#pragma unroll
            for (int c = 0; c < 3; ++c)
                a.m[4 * r + c] = fmaf(gf[r], T.m[c], fmaf(gf[4 + r], T.m[4 + c], gf[8 + r] * T.m[8 + c])) * H.inv_h;
            a.m[4 * r + 3] = fmaf(fmaf(gf[r], dx, fmaf(gf[4 + r], dy, gf[8 + r] * dz)), H.inv_h, (float)G);
        }
    }
    if (active) {
        const float *sp = H.surf + (size_t)j * H.nsurf * 6;
        const uint32_t *dtab = done ? done + (size_t)j * G3 * W : nullptr;
        uint32_t *tab = bits + (size_t)j * G3 * W;
        int32_t *wtab = wit ? wit + (size_t)j * G3 * B : nullptr;
        const int i1 = (int)((int64_t)H.nsurf * (blockIdx.z + 1) / gridDim.z);
        for (int i = (int)((int64_t)H.nsurf * blockIdx.z / gridDim.z); i < i1; ++i) {
            const float px = sp[6 * i], py = sp[6 * i + 1], pz = sp[6 * i + 2];
            const int v = window_voxel(a, G, px, py, pz);
            if (v < 0) {
                ++n_drop;
                continue;
            }
            float nx, ny, nz;
            tf_dir(T, sp[6 * i + 3], sp[6 * i + 4], sp[6 * i + 5], nx, ny, nz);
            const int b = nearest_bin_any(lut, cb4, B, nx, ny, nz);
            const uint32_t at = (uint32_t)v * W + (uint32_t)(b >> 5), m = 1u << (b & 31);
            if (dtab && (dtab[at] & m)) continue;
            if (!(__atomic_load_n(tab + at, __ATOMIC_RELAXED) & m)) atomicOr(tab + at, m);
            if (wtab) {
                int32_t *ww = wtab + (size_t)v * B + b;
                if (__atomic_load_n(ww, __ATOMIC_RELAXED) > (int32_t)s) atomicMin(ww, (int32_t)s);
            }
        }
    }
    block_add(n_drop, dropped);
}

__global__ void k_copy_u32(const uint4 *__restrict__ src, uint4 *__restrict__ dst, int64_t n4)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n4; i += (int64_t)gridDim.x * blockDim.x)
        dst[i] = src[i];
}

// The rounds of a build (see k_field_build): samples [0, 4096), then up to twice
// as many each time; done holds the table of the rounds before.  Without memory for
// it everything is one round against the live table.
static hipError_t build_rounds(lg_field *f, uint32_t *done, unsigned long long *d_drop, hipStream_t s)
{
    const DevHand &H = f->dh;
    const int64_t n4 = (int64_t)H.J * H.G * H.G * H.G * H.W / 4;  // G is a multiple of 4
    for (int64_t s0 = 0; s0 < H.samples;) {
        const int64_t s1 = done ? std::min(H.samples, std::max(kBuildRound, 2 * s0)) : H.samples;
        if (s0 > 0)
            hipLaunchKernelGGL(k_copy_u32, dim3((unsigned)std::min<int64_t>((n4 + 255) / 256, 4096)), dim3(256), 0, s,
                               reinterpret_cast<const uint4 *>(f->d_bits), reinterpret_cast<uint4 *>(done), n4);
        // parts: enough blocks for eight waves per SIMD
        const int64_t blocks = (s1 - s0 + kBuildThreads - 1) / kBuildThreads;
        const int64_t parts = std::max<int64_t>(1, std::min<int64_t>(kBuildMaxParts, 2048 / (blocks * H.J)));
        hipLaunchKernelGGL(k_field_build, dim3((unsigned)blocks, H.J, (unsigned)parts), dim3(kBuildThreads), 0, s, H,
                           s0, s1, s0 > 0 ? done : nullptr, f->d_bits, f->d_wit, d_drop);
        s0 = s1;
    }
    return hipGetLastError();
}

// Merged finger tables: OR over the links of finger f of their words, laid
// out as merged[f][w][brick_word(v)] (one plane per 32-bin word w, 4x4x4
// voxel bricks), from the canonical per-link tables bits[l][v][w]; and the links
// that hold each (voxel, bin) as a byte (a finger has at most 8 links), so that a
// reverse lookup is one read instead of one per link, each in a table of its own.
__global__ void k_field_merge(DevHand H, const uint32_t *__restrict__ bits, uint32_t *__restrict__ merged,
                              uint4 *__restrict__ masks)
{
    const int G = H.G, W = H.W;
    const int64_t G3 = (int64_t)G * G * G, G3W = G3 * W;
    const int f = blockIdx.y;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < G3W; i += (int64_t)gridDim.x * blockDim.x) {
        uint32_t acc = 0, m[8] = {0, 0, 0, 0, 0, 0, 0, 0};  // m: a byte per bin
        const int first = H.finger_first[f], d = H.finger_dof[f];
        for (int t = 0; t < d; ++t) {
            const uint32_t w = bits[(int64_t)(first + t) * G3W + i];
            acc |= w;
            // four bits to the low bits of four bytes: (x * 0x204081) puts bit b at bit 8 b
#pragma unroll
            for (int q = 0; q < 8; ++q) m[q] |= ((((w >> (4 * q)) & 15u) * 0x204081u) & 0x01010101u) << t;
        }
        const int64_t v = i / W;
        const int w = (int)(i - v * W);
        const uint32_t ix = (uint32_t)(v % G), iy = (uint32_t)((v / G) % G), iz = (uint32_t)(v / ((int64_t)G * G));
        merged[((int64_t)f * W + w) * G3 + brick_word(ix, iy, iz, (uint32_t)(G / 4))] = acc;
        uint4 *o = masks + (f * G3W + i) * 2;
        o[0] = make_uint4(m[0], m[1], m[2], m[3]);
        o[1] = make_uint4(m[4], m[5], m[6], m[7]);
    }
}

// Occupied voxels of the merged tables, one bit per voxel: thread per 32 voxels of a row.
__global__ void k_occupancy(DevHand H, const uint32_t *__restrict__ merged, uint32_t *__restrict__ occ)
{
    const int G = H.G, row = H.cull_row;
    const int64_t G3 = (int64_t)G * G * G, n = (int64_t)G * G * row;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int f = blockIdx.y, w = (int)(i % row);
    const uint32_t iy = (uint32_t)(i / row % G), iz = (uint32_t)(i / row / G);
    uint32_t bits = 0;
    for (uint32_t b = 0; b < 32u && 32u * w + b < (uint32_t)G; ++b) {
        const uint32_t v = brick_word(32u * w + b, iy, iz, (uint32_t)(G / 4));
        uint32_t any = 0;
        for (int q = 0; q < H.W; ++q) any |= merged[((int64_t)f * H.W + q) * G3 + v];
        bits |= (any != 0u ? 1u : 0u) << b;
    }
    occ[f * n + i] = bits;
}

// src dilated by d <= 4 voxels along each axis (box dilations compose, so each
// level comes from the one before): OR of (2d + 1)^2 rows, then along the row.
__global__ void k_dilate(int F, int G, int row, int d, const uint32_t *__restrict__ src, uint32_t *__restrict__ dst)
{
    const int64_t n = (int64_t)G * G * row;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int f = blockIdx.y, w = (int)(i % row), iy = (int)(i / row % G), iz = (int)(i / row / G);
    const uint32_t *s = src + f * n;
    uint32_t a = 0, lo = 0, hi = 0;  // the word, its lower and its upper neighbour
    for (int z = max(0, iz - d); z <= min(G - 1, iz + d); ++z)
        for (int y = max(0, iy - d); y <= min(G - 1, iy + d); ++y) {
            const uint32_t *r = s + ((int64_t)z * G + y) * row;
            a |= r[w];
            if (w > 0) lo |= r[w - 1];
            if (w + 1 < row) hi |= r[w + 1];
        }
    uint32_t o = a;
    for (int k = 1; k <= d; ++k) o |= (a << k) | (lo >> (32 - k)) | (a >> k) | (hi << (32 - k));
    dst[f * n + i] = o;
}

// set bits of n4 groups of four words (16-byte aligned)
__global__ void k_popcount(const uint4 *__restrict__ w, int64_t n4, unsigned long long *__restrict__ out)
{
    unsigned int c = 0;
#pragma unroll 4
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n4; i += (int64_t)gridDim.x * blockDim.x) {
        const uint4 v = w[i];
        c += __popc(v.x) + __popc(v.y) + __popc(v.z) + __popc(v.w);
    }
    block_add(c, out);
}

static lg_status merge_and_count(lg_field *f, hipStream_t st)
{
    const DevHand &H = f->dh;
    const int64_t G3W = (int64_t)H.G * H.G * H.G * H.W;
    dim3 grid((unsigned)std::min<int64_t>((G3W + 255) / 256, 4096), H.F);
    hipLaunchKernelGGL(k_field_merge, grid, dim3(256), 0, st, H, f->d_bits, f->d_merged,
                       reinterpret_cast<uint4 *>(f->d_mask));
    LG_HIP(hipGetLastError());
    // the voxels' occupancy and its dilations, for the query's culling
    const int64_t n_row = (int64_t)H.G * H.G * H.cull_row;
    const dim3 cgrid((unsigned)((n_row + 255) / 256), H.F);
    uint32_t *src = f->d_cull + (int64_t)kCullLevels * H.F * n_row;
    hipLaunchKernelGGL(k_occupancy, cgrid, dim3(256), 0, st, H, f->d_merged, src);
    for (int l = 0; l < kCullLevels; ++l) {
        uint32_t *dst = f->d_cull + (int64_t)l * H.F * n_row;
        hipLaunchKernelGGL(k_dilate, cgrid, dim3(256), 0, st, H.F, H.G, H.cull_row,
                           cull_reach(l) - (l ? cull_reach(l - 1) : 0), src, dst);
        src = dst;
    }
    LG_HIP(hipGetLastError());
    unsigned long long *d_cnt = nullptr;
    LG_HIP(hipMalloc(&d_cnt, sizeof(unsigned long long)));
    (void)hipMemsetAsync(d_cnt, 0, sizeof(unsigned long long), st);
    hipLaunchKernelGGL(k_popcount, dim3(1024), dim3(kBuildThreads), 0, st, reinterpret_cast<const uint4 *>(f->d_bits),
                       (int64_t)H.J * G3W / 4, d_cnt);  // G is a multiple of 4
    unsigned long long cnt = 0;
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = hipMemcpyAsync(&cnt, d_cnt, sizeof cnt, hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    (void)hipFree(d_cnt);
    if (e != hipSuccess) return hip_fail(e, "field merge");
    f->bits_set = cnt;
    return LG_OK;
}

}  // namespace lg

using namespace lg;

extern "C" {

const char *lg_status_str(lg_status s)
{
    switch (s) {
    case LG_OK: return "LG_OK";
    case LG_EINVAL: return "LG_EINVAL";
    case LG_ENOMEM: return "LG_ENOMEM";
    case LG_EDEVICE: return "LG_EDEVICE";
    case LG_EUNSUPPORTED: return "LG_EUNSUPPORTED";
    case LG_EINTERNAL: return "LG_EINTERNAL";
    default: return "LG_UNKNOWN";
    }
}

const char *lg_last_error(void) { return g_last_error.c_str(); }

const char *lg_version(void) { return "lg-gfx950 0.1.0"; }

lg_status lg_build_field(const lg_hand_desc *hand, const lg_field_params *params, void *stream, lg_field **out)
{
    lg_field *f = nullptr;
    lg_status st = make_field_shell(hand, params, &f);
    if (st != LG_OK) return st;
    hipStream_t s = as_stream(stream);
    const DevHand &H = f->dh;
    // scratch: the dropped count and, for more than one round, the table of the rounds before
    unsigned long long *d_drop = nullptr;
    uint32_t *done = nullptr;
    hipError_t e = hipMalloc(&d_drop, sizeof(unsigned long long));
    if (e == hipSuccess) e = hipMemsetAsync(d_drop, 0, sizeof(unsigned long long), s);
    if (e == hipSuccess && H.samples > kBuildRound &&
        hipMalloc(&done, (size_t)H.J * H.G * H.G * H.G * H.W * 4) != hipSuccess) {
        done = nullptr;
        (void)hipGetLastError();
    }
    if (e != hipSuccess) {
        (void)hipFree(d_drop);
        free_field(f);
        return hip_fail(e, "build scratch");
    }
    // the build kernel's own duration (events on the build stream), reported by lg_field_info
    hipEvent_t ev[2] = {nullptr, nullptr};
    if (e == hipSuccess) e = hipEventCreate(&ev[0]);
    if (e == hipSuccess) e = hipEventCreate(&ev[1]);
    if (e == hipSuccess) e = hipEventRecord(ev[0], s);
    if (e == hipSuccess) e = build_rounds(f, done, d_drop, s);
    if (e == hipSuccess) e = hipEventRecord(ev[1], s);
    unsigned long long drop = 0;
    if (e == hipSuccess) e = hipMemcpyAsync(&drop, d_drop, sizeof drop, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    float build_ms = 0.0f;
    if (e == hipSuccess) e = hipEventElapsedTime(&build_ms, ev[0], ev[1]);
    f->build_kernel_ms = build_ms;
    for (hipEvent_t x : ev)
        if (x) (void)hipEventDestroy(x);
    (void)hipFree(d_drop);
    (void)hipFree(done);
    if (e != hipSuccess) {
        free_field(f);
        return hip_fail(e, "k_field_build");
    }
    // dropped counts every (sample, surface point) outside the window
    f->dropped = (int64_t)drop;
    f->vectors = H.samples * (int64_t)H.J * H.nsurf;
    st = merge_and_count(f, s);
    if (st != LG_OK) {
        free_field(f);
        return st;
    }
    *out = f;
    return LG_OK;
}

lg_status lg_field_import(const lg_hand_desc *hand, const lg_field_params *params, const uint32_t *bits_host,
                          const int32_t *witness_host, lg_field **out)
{
    if (!bits_host) return fail(LG_EINVAL, "null bits_host");
    lg_field_params p = *params;
    p.keep_witness = witness_host != nullptr;
    lg_field *f = nullptr;
    lg_status st = make_field_shell(hand, &p, &f);
    if (st != LG_OK) return st;
    const DevHand &H = f->dh;
    const int64_t G3 = (int64_t)H.G * H.G * H.G;
    hipError_t e = hipMemcpy(f->d_bits, bits_host, (size_t)H.J * G3 * H.W * 4, hipMemcpyHostToDevice);
    if (e == hipSuccess && witness_host) {
        const size_t n = (size_t)H.J * G3 * H.B;
        std::vector<int32_t> w(witness_host, witness_host + n);
        for (auto &x : w)
            if (x < 0) x = kNoWitness;
        e = hipMemcpy(f->d_wit, w.data(), n * 4, hipMemcpyHostToDevice);
    }
    if (e != hipSuccess) {
        free_field(f);
        return hip_fail(e, "field import");
    }
    f->vectors = 0;
    f->dropped = 0;
    st = merge_and_count(f, nullptr);
    if (st != LG_OK) {
        free_field(f);
        return st;
    }
    *out = f;
    return LG_OK;
}

lg_status lg_field_export(const lg_field *f, uint32_t *bits_host, int32_t *witness_host)
{
    if (!f || !bits_host) return fail(LG_EINVAL, "null field or bits_host");
    const DevHand &H = f->dh;
    const int64_t G3 = (int64_t)H.G * H.G * H.G;
    LG_HIP(hipDeviceSynchronize());
    LG_HIP(hipMemcpy(bits_host, f->d_bits, (size_t)H.J * G3 * H.W * 4, hipMemcpyDeviceToHost));
    if (witness_host) {
        const size_t n = (size_t)H.J * G3 * H.B;
        if (!f->d_wit) {
            memset(witness_host, 0xff, n * 4);
        } else {
            LG_HIP(hipMemcpy(witness_host, f->d_wit, n * 4, hipMemcpyDeviceToHost));
            for (size_t i = 0; i < n; ++i)
                if (witness_host[i] < 0 || witness_host[i] >= (int32_t)H.samples) witness_host[i] = -1;
        }
    }
    return LG_OK;
}

lg_status lg_field_info(const lg_field *f, lg_field_info_t *info)
{
    if (!f || !info) return fail(LG_EINVAL, "null field or info");
    info->n_fingers = f->dh.F;
    info->n_joints = f->dh.J;
    info->grid = f->dh.G;
    info->bins = f->dh.B;
    info->samples = f->dh.samples;
    info->device_bytes = f->device_bytes;
    info->bits_set = f->bits_set;
    info->vectors = f->vectors;
    info->dropped = f->dropped;
    info->has_witness = f->has_witness ? 1 : 0;
    info->lattice = f->dh.lat;
    info->build_kernel_ms = f->build_kernel_ms;
    return LG_OK;
}

lg_status lg_field_release(lg_field *f)
{
    free_field(f);
    return LG_OK;
}

}  // extern "C"
