// Object contact query (Sec. 4.2-4.3, Def. 4.3) with the per-dependency-group
// merge of Sec. 5.3.
//
// One workgroup per pose; each wave sweeps 64 consecutive object points
// (structure-of-arrays).  Per point: the query normal -R n and its bin, the
// point's voxel in each finger window, one 4-byte gather per finger from the
// plane of its merged table that holds the bin, and a wave ballot that yields
// the 64 domain bits of the finger for the chunk.  Counts are popcounts of
// the ballots.
//
// Windows in lattice form (a shared rotation, origins a whole number of
// 4-voxel bricks apart) take one affine map per point instead of one per
// finger: the point's lattice cell is packed as x | y << 10 | z << 20, and
// finger f's in-window test is one subtraction of its packed offset and one
// mask (a field that went negative or reached G sets a bit of lat_hi).  The
// bricked table word is linear in the cell, so one per-point byte offset
// serves every finger, each finger's offset folded into its scalar base.
//
// With chunk bounds (a bounding sphere per 64 consecutive points, a one-level
// bounding-volume hierarchy over the object; tight when the points are in
// Morton order), a (chunk, finger) pair whose sphere misses the finger's
// window, or every occupied voxel of it, is skipped: its 64 domain bits are
// zero without a lookup, and a chunk that no finger keeps is not loaded at all.
//
// What bounds it: VALU issue, with the L1's line rate close behind (65,536 poses x
// 65,536 points, 22 joints: 6.0 G wave instructions and 3.8 G line accesses in 9.1 ms,
// the latter two thirds of one per CU and cycle; 7 waves per SIMD are 2 % slower than 8,
// and forms with a few more instructions per kept chunk 1 to 2 %).  8.3 G instructions
// in 13.0 ms before the culling by voxels, the bin index in float arithmetic, the
// in-brick word by three multiply-adds, the scalar chunk bookkeeping and two
// candidate bins instead of four; the last 0.5 ms were registers kept in scratch
// memory across the units (up to five fingers none; the kernel for eight spills 5).
// About 105 instructions per kept chunk: 9 for the direction, 40 for its bin, 30 for
// the cell and word, 9 per kept finger.
#include <math.h>

#include <algorithm>
#include <type_traits>
#include <utility>
#include <vector>

#include "lg_internal.h"

namespace lg {

constexpr int kQueryThreads = 256;
constexpr int kQueryWaves = kQueryThreads / 64;
constexpr int kQueryMaxThreads = 1024;
constexpr float kCullMargin = 1e-3f;  // voxels added to a chunk's radius (float rounding is ~1e-4)

// the LLVM writelane intrinsic: lane `lane` (uniform) of v replaced by the uniform x
extern "C" __device__ int lg_writelane(int x, int lane, int v) __asm("llvm.amdgcn.writelane");
__device__ inline uint32_t write_lane(uint32_t v, uint32_t x, int lane)
{
    return (uint32_t)lg_writelane((int)x, lane, (int)v);
}

// Chunks a wave takes at a time: 32 (full 256-byte stores) when that gives each
// wave of the block two or more units, else fewer, so that no wave is idle (2,048
// points are one unit of 32: three of four waves had no work).
__host__ __device__ inline int query_unit(int N, int waves)
{
    const int nchunks = (N + 63) >> 6;
    int uc = 32;
    while (uc > 4 && nchunks < 2 * uc * waves) uc >>= 1;
    return uc;
}

// Bounding sphere (centre of the box, largest distance) of each chunk of 64
// consecutive points; one wave per chunk, radius padded for rounding.
__global__ void __launch_bounds__(256)
k_chunk_bounds(const float *__restrict__ pts, int N, float4 *__restrict__ bounds)
{
    const int nchunks = (N + 63) >> 6;
    const int chunk = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (chunk >= nchunks) return;  // uniform per wave
    const int i = min(chunk * 64 + lane, N - 1);  // lanes past N repeat the last point
    const float x = pts[i], y = pts[N + i], z = pts[2 * N + i];
    float lo[3] = {x, y, z}, hi[3] = {x, y, z};
    for (int off = 32; off > 0; off >>= 1)
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            lo[a] = fminf(lo[a], __shfl_xor(lo[a], off, 64));
            hi[a] = fmaxf(hi[a], __shfl_xor(hi[a], off, 64));
        }
    const float cx = 0.5f * (lo[0] + hi[0]), cy = 0.5f * (lo[1] + hi[1]), cz = 0.5f * (lo[2] + hi[2]);
    const float dx = x - cx, dy = y - cy, dz = z - cz;
    float r = sqrtf(fmaf(dx, dx, fmaf(dy, dy, dz * dz)));
    for (int off = 32; off > 0; off >>= 1) r = fmaxf(r, __shfl_xor(r, off, 64));
    if (lane == 0) bounds[chunk] = make_float4(cx, cy, cz, fmaf(r, 1e-5f, r + 1e-7f));
}

// Largest stretch of an affine map (an upper bound of its 2-norm, equal to it
// for a scaled rotation): a sphere of radius r maps into one of r * map_stretch.
__device__ inline float map_stretch(const Affine &a)
{
    float s = 0.f;
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        float t = 0.f;
#pragma unroll
        for (int c = 0; c < 3; ++c)
            t += fabsf(fmaf(a.m[4 * r], a.m[4 * c], fmaf(a.m[4 * r + 1], a.m[4 * c + 1], a.m[4 * r + 2] * a.m[4 * c + 2])));
        s = fmaxf(s, t);
    }
    return sqrtf(s);
}

// keep[f] bit j: chunk c0 + j (j < 8, below c_end) may hold a domain point of
// finger f; returns the union.  Without bounds every chunk may.  Lane l tests
// chunk c0 + l % 8 against finger l / 8: the distance from the sphere's centre
// (voxel coordinates of map aff[LAT ? 0 : f]) to the finger's window box
// [lo, lo + G]^3 against its radius (win[f] = lo and the map's stretch; lo = G for
// a finger's own, biased, map, lat_o[f] in lattice coordinates), then the window's occupied voxels: with the
// centre moved into the window, every voxel a point of the chunk can fall in is
// within ceil(radius) of the centre's per axis, so the bit of a dilation that
// reaches as far decides.  Of the (chunk, finger) pairs whose sphere meets the
// window, 40-70 % meet no occupied voxel (65,536 points, 22 joints: 58 % of all
// pairs meet a window, 23 % an occupied voxel, 10 % hold a domain point).
template <int FM, bool LAT>
__device__ inline uint32_t group_keep(const float4 *__restrict__ bounds, const Affine *aff, const float4 *win,
                                      const DevHand &H, int c0, int c_end, int lane, uint32_t (&keep)[FM])
{
    const int F = H.F, G = H.G;
    const int f = lane >> 3, ch = c0 + (lane & 7);
    bool in = f < F && ch < c_end;
    if (bounds && in) {
        const float4 sb = bounds[ch];
        const Affine &a = aff[LAT ? 0 : f];
        const float4 o = win[f];
        // window coordinates
        const float ux = fmaf(a.m[0], sb.x, fmaf(a.m[1], sb.y, fmaf(a.m[2], sb.z, a.m[3]))) - o.x;
        const float uy = fmaf(a.m[4], sb.x, fmaf(a.m[5], sb.y, fmaf(a.m[6], sb.z, a.m[7]))) - o.y;
        const float uz = fmaf(a.m[8], sb.x, fmaf(a.m[9], sb.y, fmaf(a.m[10], sb.z, a.m[11]))) - o.z;
        const float dx = fmaxf(fmaxf(-ux, ux - G), 0.f);
        const float dy = fmaxf(fmaxf(-uy, uy - G), 0.f);
        const float dz = fmaxf(fmaxf(-uz, uz - G), 0.f);
        const float rv = fmaf(sb.w, o.w, kCullMargin);
        in = !(fmaf(dx, dx, fmaf(dy, dy, dz * dz)) > rv * rv);
        if (in && rv <= (float)cull_reach(kCullLevels - 1)) {
            // the first level that reaches rv
            const int l = rv <= 4.f ? max((int)ceilf(rv), 1) - 1 : rv <= 6.f ? 4 : rv <= 8.f ? 5 : rv <= 12.f ? 6 : 7;
            const int ix = min(max((int)ux, 0), G - 1), iy = min(max((int)uy, 0), G - 1), iz = min(max((int)uz, 0), G - 1);
            const uint32_t w = H.cull[(uint32_t)((((l * F + f) * G + iz) * G + iy) * H.cull_row + (ix >> 5))];
            in = (w >> (ix & 31)) & 1u;
        }
    }
    const unsigned long long m = __ballot(in);
    uint32_t any = 0u;
#pragma unroll
    for (int q = 0; q < FM; ++q) {
        keep[q] = (uint32_t)(m >> (8 * q)) & 0xffu;  // fingers past F were not tested: 0
        any |= keep[q];
    }
    return any;
}

// LDS of one query block
template <int FM, bool LAT>
struct QueryLds {
    float4 cb4[kMaxBins];
    uint32_t lut[6 * kLutRes * kLutRes];
    Affine aff[LAT ? 1 : FM];
    float4 win[FM];  // see group_keep
};

// The domains of pose g (one block of any number of waves up to 16).  CULL: chunks and
// fingers may be skipped (bounds).  Without bounds, on lattice windows, the kernel has
// no such test at all (16,384 points, 4 fingers, 4,096 poses: 245 us with it, 235
// without); for windows with maps of their own the tested form is the faster one also
// then (303 us, 344 without).
template <int W, int FM, bool LAT, bool CULL>
__device__ __forceinline__ void query_pose(QueryLds<FM, LAT> &L, const DevHand &H, const uint32_t *__restrict__ merged,
                                           const float *__restrict__ pts, const float *__restrict__ nrm, int N,
                                           const float *__restrict__ poses, const float4 *__restrict__ bounds,
                                           uint32_t *__restrict__ dom_bits, uint32_t *__restrict__ dom_count, int uc,
                                           int g)
{
    float4 *cb4 = L.cb4;
    uint32_t *lut = L.lut;
    Affine *aff = L.aff;
    const float *pose = poses + 12 * (int64_t)g;
    for (int i = threadIdx.x; i < H.B; i += blockDim.x)
        cb4[i] = make_float4(H.bin_c[3 * i], H.bin_c[3 * i + 1], H.bin_c[3 * i + 2], 0.0f);
    for (int i = threadIdx.x; i < 6 * kLutRes * kLutRes; i += blockDim.x) lut[i] = H.bin_lut[i];
    if (threadIdx.x < H.F) {
        const int f = threadIdx.x;
        const Affine a = LAT ? lattice_affine(H, pose) : finger_affine(H, pose, f);
        if (!LAT || f == 0) aff[LAT ? 0 : f] = a;
        if (CULL && bounds) {  // only group_keep's culling reads win
            const float sc = map_stretch(a);
            L.win[f] = LAT ? make_float4((float)H.lat_o[f][0], (float)H.lat_o[f][1], (float)H.lat_o[f][2], sc)
                           : make_float4((float)H.G, (float)H.G, (float)H.G, sc);
        }
    }
    __syncthreads();
    // the wave index is uniform: in a scalar register, the block and chunk
    // bookkeeping (and the skip tests) stay on the scalar unit
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int F = H.F, G = H.G, B = H.B;
    const uint32_t GB = (uint32_t)(G >> 2), G3 = (uint32_t)G * G * G;
    // Byte offset of finger f's table less (lattice form) the word of its
    // window origin, or (general form) of the +G bias of each coordinate, so
    // that it plus 4 * (word of the point's cell) addresses the finger's word.
    // The sum is taken in 32 bits: it wraps to the right offset for every
    // lane inside the window (the tables are far below 4 GiB).
    const char *mbase = reinterpret_cast<const char *>(merged);
    uint32_t koff[FM];
#pragma unroll
    for (int f = 0; f < FM; ++f)
        koff[f] = 4u * ((uint32_t)f * W * G3 - (LAT ? H.lat_idx[f < F ? f : 0] : brick_word(G, G, G, GB)));
    const int NW = (N + 31) >> 5, nchunks = (N + 63) >> 6;
    float P[12];
#pragma unroll
    for (int i = 0; i < 12; ++i) P[i] = pose[i];
    uint32_t c[FM];
#pragma unroll
    for (int f = 0; f < FM; ++f) c[f] = 0;
    // Waves take units of uc consecutive chunks (a compact patch of the
    // Morton-ordered object) in turn.  The ballot words of a unit stay in
    // registers, lane 2j / 2j+1 holding chunk j's halves, and leave as one
    // coalesced store per finger.
    const int waves = blockDim.x >> 6, nunit = (nchunks + uc - 1) / uc;
    for (int unit = wave; unit < nunit; unit += waves) {
        uint32_t acc[FM];
#pragma unroll
        for (int f = 0; f < FM; ++f) {
            acc[f] = 0;
            asm volatile("" : "+v"(acc[f]));  // made here, not kept (in scratch memory) from before the loop
        }
        const int u0 = unit * uc, c_end = min(nchunks, u0 + uc);
        for (int c0 = u0; c0 < c_end; c0 += 8) {
          uint32_t keep[FM], todo;
          if constexpr (CULL)
              todo = group_keep<FM, LAT>(bounds, aff, L.win, H, c0, c_end, lane, keep);
          else
              todo = (1u << min(8, c_end - c0)) - 1u;
          for (; todo; todo &= todo - 1u) {
            const uint32_t cbit = todo & (0u - todo);
            const int chunk = c0 + __builtin_ctz(todo);
            // re-read the maps from LDS every chunk instead of pinning their
            // registers for the whole sweep
            asm volatile("" ::: "memory");
            const int i = chunk * 64 + lane;
            const bool valid = i < N;
            // lanes past N read the last point (in bounds, no branch); they
            // are outside every window through `valid`
            const uint32_t il = (uint32_t)min(i, N - 1);
            const char *pb = reinterpret_cast<const char *>(pts), *nb = reinterpret_cast<const char *>(nrm);
            const uint32_t o0 = il << 2, o1 = o0 + ((uint32_t)N << 2), o2 = o1 + ((uint32_t)N << 2);
            const float px = *reinterpret_cast<const float *>(pb + o0);
            const float py = *reinterpret_cast<const float *>(pb + o1);
            const float pz = *reinterpret_cast<const float *>(pb + o2);
            const float nx = *reinterpret_cast<const float *>(nb + o0);
            const float ny = *reinterpret_cast<const float *>(nb + o1);
            const float nz = *reinterpret_cast<const float *>(nb + o2);
            float qx, qy, qz;
            query_dir(P, nx, ny, nz, qx, qy, qz);
            const int b = nearest_bin_lut4(lut, cb4, B, qx, qy, qz);
            const uint32_t plane = W == 2 ? __umul24((uint32_t)(b >> 5), 4u * G3) : 0u;  // byte offset
            uint32_t word[FM];  // 0 outside the window
            uint32_t voff = 0, ip = 0;
            if (LAT) {
                int Ix, Iy, Iz;
                lattice_cell(aff[0], px, py, pz, Ix, Iy, Iz);
                Ix = min(max(Ix, 0), 1023);
                Iy = min(max(Iy, 0), 1023);
                Iz = min(max(Iz, 0), 1023);
                ip = (uint32_t)Ix | (uint32_t)Iy << 10 | (uint32_t)Iz << 20;
                // 4 * (brick word + plane): each coordinate's in-brick part goes with
                // stride 1, 4, 16, its brick part (v & ~3, times a constant) on top
                voff = (uint32_t)Ix << 2;
                voff = mad_u24((uint32_t)Ix & 1020u, 60u, voff) + plane;
                voff += (uint32_t)Iy << 4;
                voff = mad_u24((uint32_t)Iy & 1020u, 64u * GB - 16u, voff);
                voff += (uint32_t)Iz << 6;
                voff = mad_u24((uint32_t)Iz & 1020u, 64u * GB * GB - 64u, voff);
                asm volatile("" : "+v"(voff));  // one add per finger below, not a re-associated pair
            }
            // all finger gathers are issued before any is consumed
#pragma unroll
            for (int f = 0; f < FM; ++f) {
                word[f] = 0u;
                if (CULL ? (keep[f] & cbit) != 0u : f < F) {  // 0 for fingers past F
                    uint32_t off;
                    bool in;
                    if (LAT) {
                        in = ((int)valid & (int)(((ip - H.lat_pk[f]) & H.lat_hi) == 0u)) != 0;
                        off = voff;
                    } else {
                        // biased window coordinates (see window_voxel): inside iff all in [G, 2G)
                        const Affine &a = aff[f];
                        const float ux = fmaf(a.m[0], px, fmaf(a.m[1], py, fmaf(a.m[2], pz, a.m[3])));
                        const float uy = fmaf(a.m[4], px, fmaf(a.m[5], py, fmaf(a.m[6], pz, a.m[7])));
                        const float uz = fmaf(a.m[8], px, fmaf(a.m[9], py, fmaf(a.m[10], pz, a.m[11])));
                        const int Ix = (int)ux, Iy = (int)uy, Iz = (int)uz;
                        in = ((int)valid & (int)(min(Ix, min(Iy, Iz)) >= G) & (int)(max(Ix, max(Iy, Iz)) < 2 * G)) != 0;
                        off = (brick_word_u24((uint32_t)Ix, (uint32_t)Iy, (uint32_t)Iz, GB) << 2) + plane;
                    }
                    if (in) word[f] = *reinterpret_cast<const uint32_t *>(mbase + (off + koff[f]));
                }
            }
            const int j2 = 2 * (chunk - u0);
            uint32_t cb2 = cbit;  // tested again: FM lane masks kept from above take 2 FM scalar registers
            asm volatile("" : "+s"(cb2));
#pragma unroll
            for (int f = 0; f < FM; ++f) {
                if (!(CULL ? (keep[f] & cb2) != 0u : f < F)) continue;  // the ballot would be 0
                const bool hit = (int)(word[f] << (~b & 31)) < 0;  // bit b % 32
                const unsigned long long m = __ballot(hit);
                // the chunk's two ballot halves into lanes j2, j2 + 1 (j2 is uniform)
                acc[f] = write_lane(acc[f], (uint32_t)m, j2);
                acc[f] = write_lane(acc[f], (uint32_t)(m >> 32), j2 + 1);
            }
          }
        }
        const int wi = u0 * 2 + lane;
        int row = g;
        asm volatile("" : "+s"(row));  // likewise the addresses
        if (lane < 2 * uc && wi < NW) {
#pragma unroll
            for (int f = 0; f < FM; ++f)
                if (f < F) dom_bits[((int64_t)row * F + f) * NW + wi] = acc[f];
        }
        // counts per lane from the block's words (bits past N are 0)
#pragma unroll
        for (int f = 0; f < FM; ++f) c[f] += (uint32_t)__popc(acc[f]);
    }
#pragma unroll
    for (int f = 0; f < FM; ++f)
        for (int off = 32; off > 0; off >>= 1) c[f] += __shfl_xor(c[f], off, 64);
    __syncthreads();  // every wave is done with the bin table: its LDS holds the counts [wave][FM]
    uint32_t *cnt = L.lut;
    if (lane == 0) {
#pragma unroll
        for (int f = 0; f < FM; ++f)
            if (f < F) cnt[wave * FM + f] = c[f];
    }
    __syncthreads();
    if (threadIdx.x < F) {
        uint32_t s = 0;
        for (int w = 0; w < waves; ++w) s += cnt[w * FM + threadIdx.x];
        dom_count[(int64_t)g * F + threadIdx.x] = s;
    }
}

template <int W, int FM, bool LAT, bool CULL>
__global__ void __launch_bounds__(kQueryMaxThreads) __attribute__((amdgpu_waves_per_eu(8, 8)))
k_query(DevHand H, const uint32_t *__restrict__ merged, const float *__restrict__ pts,
        const float *__restrict__ nrm, int N, const float *__restrict__ poses, const float4 *__restrict__ bounds,
        uint32_t *__restrict__ dom_bits, uint32_t *__restrict__ dom_count, int uc)
{
    __shared__ QueryLds<FM, LAT> L;
    query_pose<W, FM, LAT, CULL>(L, H, merged, pts, nrm, N, poses, bounds, dom_bits, dom_count, uc, blockIdx.x);
}

// The same over the poses of several chunks (one block per pose).
template <int W, int FM, bool LAT>
__global__ void __launch_bounds__(kQueryThreads) __attribute__((amdgpu_waves_per_eu(8, 8)))
k_query_batch(const ChunkDesc *__restrict__ d, const uint16_t *__restrict__ idx, const uint32_t *__restrict__ first,
              int n)
{
    __shared__ QueryLds<FM, LAT> L;
    const int j = batch_member(first, n, blockIdx.x);
    const ChunkDesc &c = d[idx[j]];
    query_pose<W, FM, LAT, true>(L, c.H, c.merged, c.pts, c.nrm, c.N, c.poses, c.bounds, c.dom_bits, c.dom_count,
                           query_unit(c.N, kQueryWaves), (int)(blockIdx.x - first[j]));
}

// Cone query (Sec. 4.3's theta_hit test): a query (x, -R n) hits finger f if
// a bin b set in the finger's merged word(s) at voxel(x) has c_b . q >= cos_hit.
// Same sweep and block stores as k_query.  Per point the cone is built once as
// a bin mask over the bins of its polar band that some finger's entry holds;
// each finger's test is then one AND with its entry.  What bounds it: VALU issue;
// with 32 bins the masks are 32 bits wide (16,384 poses x 37,176 points without
// bounds 2.25 ms, 2.44 with 64-bit ones); with 64 bins and bounds 8,191 poses x
// 30,011 points take 1.6 ms (2.1 before the culling by voxels).  A pose has 256
// threads also where there are few (more were not tried here).
template <int W, int FM>
__global__ void __launch_bounds__(kQueryThreads)
k_query_cone(DevHand H, const uint32_t *__restrict__ merged, const float *__restrict__ pts,
             const float *__restrict__ nrm, int N, const float *__restrict__ poses, const float4 *__restrict__ bounds,
             float cos_hit, uint32_t *__restrict__ dom_bits, uint32_t *__restrict__ dom_count, int uc)
{
    using mask_t = typename std::conditional<W == 1, uint32_t, unsigned long long>::type;  // a bit per bin
    __shared__ float cb[3 * kMaxBins];  // rows of 3 floats: fewer bank conflicts than of 4
    __shared__ Affine aff[FM];
    __shared__ float4 win[FM];
    __shared__ uint32_t cnt[FM][kQueryWaves];
    const int g = blockIdx.x;
    const float *pose = poses + 12 * (int64_t)g;
    for (int i = threadIdx.x; i < 3 * H.B; i += blockDim.x) cb[i] = H.bin_c[i];
    if (threadIdx.x < H.F) {
        aff[threadIdx.x] = finger_affine(H, pose, threadIdx.x);
        if (bounds)  // only group_keep's culling reads win
            win[threadIdx.x] = make_float4((float)H.G, (float)H.G, (float)H.G, map_stretch(aff[threadIdx.x]));
    }
    __syncthreads();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int F = H.F, G = H.G, B = H.B;
    const float sin_hit = sqrtf(fmaxf(0.f, fmaf(-cos_hit, cos_hit, 1.f)));
    const uint32_t GB = (uint32_t)(G >> 2), G3 = (uint32_t)G * G * G;
    const int NW = (N + 31) >> 5, nchunks = (N + 63) >> 6;
    float P[12];
#pragma unroll
    for (int i = 0; i < 12; ++i) P[i] = pose[i];
    uint32_t c[FM];
#pragma unroll
    for (int f = 0; f < FM; ++f) c[f] = 0;
    const int nunit = (nchunks + uc - 1) / uc;
    for (int unit = wave; unit < nunit; unit += kQueryWaves) {
        uint32_t acc[FM];
#pragma unroll
        for (int f = 0; f < FM; ++f) acc[f] = 0;
        const int u0 = unit * uc, c_end = min(nchunks, u0 + uc);
        for (int c0 = u0; c0 < c_end; c0 += 8) {
          uint32_t keep[FM];
          for (uint32_t todo = group_keep<FM, false>(bounds, aff, win, H, c0, c_end, lane, keep); todo; todo &= todo - 1u) {
            const uint32_t cbit = todo & (0u - todo);
            const int chunk = c0 + __builtin_ctz(todo);
            asm volatile("" ::: "memory");
            const int i = chunk * 64 + lane;
            const bool valid = i < N;
            float px = 0.f, py = 0.f, pz = 0.f, nx = 0.f, ny = 0.f, nz = 1.f;
            if (valid) {
                px = pts[i];
                py = pts[N + i];
                pz = pts[2 * N + i];
                nx = nrm[i];
                ny = nrm[N + i];
                nz = nrm[2 * N + i];
            }
            float qx, qy, qz;
            query_dir(P, nx, ny, nz, qx, qy, qz);
            // bins that can lie within the cone: the polar band |phi_b - phi_q| <=
            // theta_hit, a contiguous index range of the Fibonacci lattice (z_b =
            // 1 - (2b + 1) / B decreases with b), widened by one bin for rounding
            const float sq = sqrtf(fmaxf(0.f, fmaf(-qz, qz, 1.f)));
            const float zhi = qz >= cos_hit ? 1.f : fmaf(qz, cos_hit, sq * sin_hit);
            const float zlo = qz <= -cos_hit ? -1.f : fmaf(qz, cos_hit, -sq * sin_hit);
            const int blo = max(0, (int)floorf(0.5f * fmaf((float)B, 1.f - zhi, -1.f)) - 1);
            const int bhi = min(B - 1, (int)ceilf(0.5f * fmaf((float)B, 1.f - zlo, -1.f)) + 1);
            constexpr int kBits = 8 * (int)sizeof(mask_t);
            const mask_t band = blo > bhi ? (mask_t)0
                                          : (mask_t)((bhi - blo == kBits - 1 ? ~(mask_t)0
                                                                             : (((mask_t)1 << (bhi - blo + 1)) - (mask_t)1))
                                                     << blo);
            mask_t ent[FM];
#pragma unroll
            for (int f = 0; f < FM; ++f) {
                ent[f] = 0;
                if (keep[f] & cbit) {  // 0 for fingers past F
                    // biased window coordinates (see window_voxel): inside iff all in [G, 2G)
                    const Affine &a = aff[f];
                    const float ux = fmaf(a.m[0], px, fmaf(a.m[1], py, fmaf(a.m[2], pz, a.m[3])));
                    const float uy = fmaf(a.m[4], px, fmaf(a.m[5], py, fmaf(a.m[6], pz, a.m[7])));
                    const float uz = fmaf(a.m[8], px, fmaf(a.m[9], py, fmaf(a.m[10], pz, a.m[11])));
                    const unsigned ix = (unsigned)((int)ux - G), iy = (unsigned)((int)uy - G),
                                   iz = (unsigned)((int)uz - G);
                    if (valid && max(ix, max(iy, iz)) < (unsigned)G) {
                        const uint32_t *tab = merged + (int64_t)f * W * G3;
                        const uint32_t wv = brick_word(ix, iy, iz, GB);
                        ent[f] = tab[wv];
                        if constexpr (W == 2) ent[f] |= (mask_t)tab[G3 + wv] << 32;
                    }
                }
            }
            const int j2 = 2 * (chunk - u0);
            // the point's cone as a bin mask over the band's bins that some
            // finger's entry holds (the per-finger test is then one AND)
            mask_t cone = 0;
            {
                mask_t u = 0;
#pragma unroll
                for (int f = 0; f < FM; ++f) u |= ent[f];
                mask_t m = u & band;
                while (m) {
                    const int b = W == 1 ? __ffs((int)m) - 1 : __ffsll((long long)m) - 1;
                    m &= m - (mask_t)1;
                    if (fmaf(cb[3 * b], qx, fmaf(cb[3 * b + 1], qy, cb[3 * b + 2] * qz)) >= cos_hit) cone |= (mask_t)1 << b;
                }
            }
#pragma unroll
            for (int f = 0; f < FM; ++f) {
                if (!(keep[f] & cbit)) continue;  // the ballot would be 0
                const bool hit = (ent[f] & cone) != 0;
                const unsigned long long bm = __ballot(hit);
                acc[f] = write_lane(acc[f], (uint32_t)bm, j2);
                acc[f] = write_lane(acc[f], (uint32_t)(bm >> 32), j2 + 1);
            }
          }
        }
        const int wi = u0 * 2 + lane;
        if (lane < 2 * uc && wi < NW) {
#pragma unroll
            for (int f = 0; f < FM; ++f)
                if (f < F) dom_bits[((int64_t)g * F + f) * NW + wi] = acc[f];
        }
#pragma unroll
        for (int f = 0; f < FM; ++f) c[f] += (uint32_t)__popc(acc[f]);
    }
#pragma unroll
    for (int f = 0; f < FM; ++f)
        for (int off = 32; off > 0; off >>= 1) c[f] += __shfl_xor(c[f], off, 64);
    if (lane == 0) {
#pragma unroll
        for (int f = 0; f < FM; ++f)
            if (f < F) cnt[f][wave] = c[f];
    }
    __syncthreads();
    if (threadIdx.x < F) {
        uint32_t s = 0;
        for (int w = 0; w < kQueryWaves; ++w) s += cnt[threadIdx.x][w];
        dom_count[(int64_t)g * F + threadIdx.x] = s;
    }
}

}  // namespace lg

using namespace lg;

// Threads of a pose's block.  2,048 blocks of 256 threads fill the chip; fewer poses
// get more waves each (16,384 points, 4 fingers: 700 poses 87 us with 256 threads, 57
// with 512; 1,024 poses 95 and 70).
static int query_threads(int n_poses) { return n_poses <= 256 ? 1024 : n_poses <= 1024 ? 512 : kQueryThreads; }

static lg_status query_domains(const lg_field *field, const float *pts, const float *nrm, int32_t n_points,
                               const float *poses, int32_t n_poses, const float4 *bounds, uint32_t *dom_bits,
                               uint32_t *dom_count, void *stream)
{
    if (!field) return fail(LG_EINVAL, "null field");
    if (n_points < 0 || n_poses < 0) return fail(LG_EINVAL, "negative size");
    if (n_poses == 0) return LG_OK;
    if (!poses || !dom_count || (n_points > 0 && (!pts || !nrm || !dom_bits)))
        return fail(LG_EINVAL, "null device buffer");
    if ((int64_t)n_points * 12 > 0xffffffffLL)
        return fail(LG_EUNSUPPORTED, "n_points above 357,913,941 (32-bit byte offsets into the point rows)");
    hipStream_t s = as_stream(stream);
    const DevHand &H = field->dh;
    // A pose is one block.  Few poses leave the chip short of waves, so they
    // get larger blocks (up to 16 waves).
    const int tb = query_threads(n_poses), uc = query_unit(n_points, tb / 64);
    const int64_t row = (int64_t)H.F * ((n_points + 31) / 32);
    for (int64_t g0 = 0; g0 < n_poses; g0 += kMaxGridPoses) {
        const dim3 grid((unsigned)std::min<int64_t>(n_poses - g0, kMaxGridPoses));
        const float *po = poses + 12 * g0;
        uint32_t *db = dom_bits + row * g0, *dc = dom_count + H.F * g0;
#define LG_QUERY_C(W, FM, LAT, CULL)                                                                              \
    hipLaunchKernelGGL((k_query<W, FM, LAT, CULL>), grid, dim3(tb), 0, s, H, field->d_merged, pts, nrm, n_points, \
                       po, bounds, db, dc, uc)
#define LG_QUERY(W, FM, LAT)                                                                                 \
    do { if (bounds || !LAT) LG_QUERY_C(W, FM, LAT, true); else LG_QUERY_C(W, FM, LAT, !LAT); } while (0)
#define LG_QUERY_F(W, LAT)                                                                                   \
    if (H.F <= 3) LG_QUERY(W, 3, LAT); else if (H.F <= 4) LG_QUERY(W, 4, LAT);                               \
    else if (H.F <= 5) LG_QUERY(W, 5, LAT); else LG_QUERY(W, 8, LAT)
        if (H.lat) {
            if (H.W == 1) { LG_QUERY_F(1, true); } else { LG_QUERY_F(2, true); }
        } else {
            if (H.W == 1) { LG_QUERY_F(1, false); } else { LG_QUERY_F(2, false); }
        }
#undef LG_QUERY_F
#undef LG_QUERY
#undef LG_QUERY_C
    }
    LG_HIP(hipGetLastError());
    return LG_OK;
}

extern "C" lg_status lg_query_domains(const lg_field *field, const float *pts, const float *nrm, int32_t n_points,
                                      const float *poses, int32_t n_poses, uint32_t *dom_bits, uint32_t *dom_count,
                                      void *stream)
{
    return query_domains(field, pts, nrm, n_points, poses, n_poses, nullptr, dom_bits, dom_count, stream);
}

extern "C" lg_status lg_query_domains_bounded(const lg_field *field, const float *pts, const float *nrm,
                                              int32_t n_points, const float *poses, int32_t n_poses,
                                              const float *bounds, uint32_t *dom_bits, uint32_t *dom_count,
                                              void *stream)
{
    if (n_points > 0 && n_poses > 0 && !bounds) return fail(LG_EINVAL, "null chunk bounds");
    if (reinterpret_cast<uintptr_t>(bounds) % 16 != 0) return fail(LG_EINVAL, "chunk bounds must be 16-byte aligned");
    return query_domains(field, pts, nrm, n_points, poses, n_poses, reinterpret_cast<const float4 *>(bounds),
                         dom_bits, dom_count, stream);
}

lg_status lg::query_batch(const BatchLaunch &b, int W, int F, bool lat, hipStream_t s)
{
    if (b.n <= 0 || b.blocks == 0) return LG_OK;
#define LG_QUERY(W_, FM, LAT)                                                                                \
    hipLaunchKernelGGL((k_query_batch<W_, FM, LAT>), dim3(b.blocks), dim3(kQueryThreads), 0, s, b.d, b.idx,  \
                       b.first, b.n)
#define LG_QUERY_F(W_, LAT)                                                                                  \
    if (F <= 3) LG_QUERY(W_, 3, LAT); else if (F <= 4) LG_QUERY(W_, 4, LAT);                                 \
    else if (F <= 5) LG_QUERY(W_, 5, LAT); else LG_QUERY(W_, 8, LAT)
    if (lat) {
        if (W == 1) { LG_QUERY_F(1, true); } else { LG_QUERY_F(2, true); }
    } else {
        if (W == 1) { LG_QUERY_F(1, false); } else { LG_QUERY_F(2, false); }
    }
#undef LG_QUERY_F
#undef LG_QUERY
    LG_HIP(hipGetLastError());
    return LG_OK;
}

extern "C" lg_status lg_chunk_bounds(const float *pts, int32_t n_points, float *bounds, void *stream)
{
    if (n_points < 0) return fail(LG_EINVAL, "negative size");
    if (n_points == 0) return LG_OK;
    if (!pts || !bounds) return fail(LG_EINVAL, "null device buffer");
    if (reinterpret_cast<uintptr_t>(bounds) % 16 != 0) return fail(LG_EINVAL, "chunk bounds must be 16-byte aligned");
    const int nchunks = (n_points + 63) / 64;
    hipLaunchKernelGGL(k_chunk_bounds, dim3((unsigned)((nchunks + 3) / 4)), dim3(256), 0, as_stream(stream), pts,
                       n_points, reinterpret_cast<float4 *>(bounds));
    LG_HIP(hipGetLastError());
    return LG_OK;
}

// Morton (Z-order) permutation of host points: 10 bits per axis over the
// points' bounding cube, bits interleaved x, y, z from the lowest; ties keep
// the input order.
extern "C" lg_status lg_morton_order(const float *pts_host, int32_t n_points, int32_t *perm_host)
{
    if (n_points < 0) return fail(LG_EINVAL, "negative size");
    if (n_points == 0) return LG_OK;
    if (!pts_host || !perm_host) return fail(LG_EINVAL, "null host buffer");
    double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (int i = 0; i < n_points; ++i)
        for (int a = 0; a < 3; ++a) {
            const double v = pts_host[3 * i + a];
            if (!std::isfinite(v)) return fail(LG_EINVAL, "non-finite point");
            lo[a] = std::min(lo[a], v);
            hi[a] = std::max(hi[a], v);
        }
    const double ext = std::max(std::max(hi[0] - lo[0], hi[1] - lo[1]), std::max(hi[2] - lo[2], 1e-30));
    std::vector<std::pair<uint32_t, int32_t>> key((size_t)n_points);
    for (int i = 0; i < n_points; ++i) {
        uint32_t code = 0;
        for (int a = 0; a < 3; ++a) {
            const uint32_t q = (uint32_t)std::min(1023.0, std::max(0.0, (pts_host[3 * i + a] - lo[a]) / ext * 1023.0));
            for (int b = 0; b < 10; ++b) code |= ((q >> b) & 1u) << (3 * b + a);
        }
        key[(size_t)i] = {code, i};
    }
    std::stable_sort(key.begin(), key.end(),
                     [](const std::pair<uint32_t, int32_t> &x, const std::pair<uint32_t, int32_t> &y) {
                         return x.first < y.first;
                     });
    for (int i = 0; i < n_points; ++i) perm_host[i] = key[(size_t)i].second;
    return LG_OK;
}

extern "C" lg_status lg_query_domains_cone(const lg_field *field, const float *pts, const float *nrm, int32_t n_points,
                                           const float *poses, int32_t n_poses, const float *bounds, float cos_hit,
                                           uint32_t *dom_bits, uint32_t *dom_count, void *stream)
{
    if (!field) return fail(LG_EINVAL, "null field");
    if (reinterpret_cast<uintptr_t>(bounds) % 16 != 0) return fail(LG_EINVAL, "chunk bounds must be 16-byte aligned");
    if (n_points < 0 || n_poses < 0) return fail(LG_EINVAL, "negative size");
    if (!(cos_hit >= -1.0f && cos_hit <= 1.0f)) return fail(LG_EINVAL, "cos_hit outside [-1, 1]");
    if (n_poses == 0) return LG_OK;
    if (!poses || !dom_count || (n_points > 0 && (!pts || !nrm || !dom_bits)))
        return fail(LG_EINVAL, "null device buffer");
    hipStream_t s = as_stream(stream);
    const DevHand &H = field->dh;
    const int64_t row = (int64_t)H.F * ((n_points + 31) / 32);
    for (int64_t g0 = 0; g0 < n_poses; g0 += kMaxGridPoses) {
        const dim3 grid((unsigned)std::min<int64_t>(n_poses - g0, kMaxGridPoses));
#define LG_QCONE(W, FM)                                                                                          \
    hipLaunchKernelGGL((k_query_cone<W, FM>), grid, dim3(kQueryThreads), 0, s, H, field->d_merged, pts, nrm,     \
                       n_points, poses + 12 * g0, reinterpret_cast<const float4 *>(bounds), cos_hit,             \
                       dom_bits + row * g0, dom_count + H.F * g0, query_unit(n_points, kQueryWaves))
        if (H.W == 1) {
            if (H.F <= 3) LG_QCONE(1, 3); else if (H.F <= 4) LG_QCONE(1, 4); else if (H.F <= 5) LG_QCONE(1, 5); else LG_QCONE(1, 8);
        } else {
            if (H.F <= 3) LG_QCONE(2, 3); else if (H.F <= 4) LG_QCONE(2, 4); else if (H.F <= 5) LG_QCONE(2, 5); else LG_QCONE(2, 8);
        }
#undef LG_QCONE
    }
    LG_HIP(hipGetLastError());
    return LG_OK;
}
