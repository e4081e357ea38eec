// Learned palm-pose proposer on gfx950: a PointNet-style encoder and a
// mixture-density head evaluated with BF16 MFMA (FP32 accumulation), its
// training step (mixture NLL, backward, Adam on FP32 master weights) and a
// Philox sampler of palm poses with a uniform fallback.
//
// The paper names data-driven search as a way to skip unproductive regions
// (Sec. 5.7) and leaves it unimplemented.  This network is the project's own
// configuration: a shared per-point MLP 6 -> 128 -> 256 (ReLU) and a max-pool
// over the points (PointNet, Qi et al. 2017); a head 256 -> 256 -> 256 (ReLU)
// -> 152 = 8 components x (logit, 9 means, 9 log-sigmas) of a diagonal
// Gaussian mixture over y = (first two columns of R, t / 0.1 m), mapped back to
// SO(3) by Gram-Schmidt (the 6-D representation of Zhou et al. 2019).
//
// Work decomposition:
//  * k_encode: 2048 points of one object per workgroup of 8 waves; W2 (BF16,
//    68 KiB) is staged in LDS once, then every wave runs its own 64-point
//    steps without a barrier.  Layer 1 is computed transposed (one 32x32x16
//    MFMA per 32 channels, K = 6 padded to 16, the bias as the accumulator),
//    so a lane holds 4-channel groups of one point; a lane-half swap
//    (v_permlane32_swap) turns them into layer 2's A operand in registers.
//    Layer 2 is 8 x 8 MFMAs per 32 points; the max-pool keeps, per lane and
//    channel, the largest pre-activation and its lowest point (a max tree,
//    then a first-match scan); the pairs are merged across the lane halves,
//    the waves (LDS) and the workgroups (64-bit atomicMax of ordered value
//    bits above the inverted point index); bias and ReLU are applied to the
//    pooled maximum.
//  * the head's layers and their input gradients are chains of small products
//    (rows = objects): a workgroup of 8 waves takes 32 objects through a whole
//    chain (k_head, k_head_bwd), a wave per 32 columns, activations in LDS;
//  * every weight gradient, the biases, the loss and the encoder's backward are
//    independent once the chain is done and run in one launch (k_grads).  The
//    encoder's is sparse: the max-pool routes each channel's gradient to one
//    point, so only B x 256 point rows are revisited (FP32).

#include "lg_internal.h"

namespace lg {
namespace prop {

constexpr int kIn = 6, kInPad = 16, kH1 = 128, kH2 = 256, kHH = 256, kM = 8, kY = 9;
constexpr int kOut = kM * (1 + 2 * kY);  // 152
constexpr float kInvSP = 10.0f;          // 1 / 0.1 m: input point scale
constexpr float kST = 0.1f;              // m: translation scale of y
constexpr float kLsMin = -5.0f, kLsMax = 2.0f;
constexpr uint32_t kPurposeSample = 7u;  // third Philox counter word of the sampler
constexpr uint32_t kPurposeInit = 9u;    // ... of the weight initialisation

// flat FP32 parameter layout: per layer W [in][out] row-major, then b [out]
constexpr int64_t kW1 = 0, kB1 = kW1 + kIn * kH1;
constexpr int64_t kW2 = kB1 + kH1, kB2 = kW2 + kH1 * kH2;
constexpr int64_t kWa = kB2 + kH2, kBa = kWa + kH2 * kHH;
constexpr int64_t kWb = kBa + kHH, kBb = kWb + kHH * kHH;
constexpr int64_t kWc = kBb + kHH, kBc = kWc + kHH * kOut;
constexpr int64_t kNParams = kBc + kOut;
// BF16 weight copies.  Encoder layers: transposed to [out][in_pad], so that an MFMA
// operand (8 consecutive inputs of one output) is one 16-byte load.  Head layers:
// in operand order, twice, so that a wave's load of an operand is 1 KiB in one
// piece (rows of the transposed copy are 32 pieces; a block's weight reads then
// took 12 us instead of 4): for the products with W, tiles of 32 outputs, k = inputs
// (kTa, kTb, kTc); for those with W^T, tiles of 32 inputs, k = outputs (kUa, kUb,
// kUc).  [tile][k / 16][lane][8]; outputs are padded to 160 in the last layer.
constexpr int kOutPad = (kOut + 31) / 32 * 32;
constexpr int64_t kT1 = 0, kT2 = kT1 + kH1 * kInPad, kTa = kT2 + kH2 * kH1, kTb = kTa + kHH * kH2;
constexpr int64_t kTc = kTb + kHH * kHH, kUa = kTc + kHH * kOutPad, kUb = kUa + kHH * kH2;
constexpr int64_t kUc = kUb + kHH * kHH, kNT = kUc + kHH * kOutPad;

struct LayerDesc {
    int in, out, in_pad;  // in_pad: encoder layers only
    int64_t w, b, t, u;
    float init_gain;
};
__host__ __device__ inline LayerDesc layer(int l)
{
    switch (l) {
    case 0: return {kIn, kH1, kInPad, kW1, kB1, kT1, 0, 1.0f};
    case 1: return {kH1, kH2, kH1, kW2, kB2, kT2, 0, 1.0f};
    case 2: return {kH2, kHH, 0, kWa, kBa, kTa, kUa, 1.0f};
    case 3: return {kHH, kHH, 0, kWb, kBb, kTb, kUb, 1.0f};
    default: return {kHH, kOut, 0, kWc, kBc, kTc, kUc, 0.1f};
    }
}
// place of element (k, c) of an operand array: column (or row) c of the tiles, kpad values of k
__host__ __device__ inline int64_t operand_at(int k, int c, int kpad)
{
    return (((int64_t)(c >> 5) * (kpad / 16) + (k >> 4)) * 64 + ((k >> 3) & 1) * 32 + (c & 31)) * 8 + (k & 7);
}

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef unsigned short u16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));

// float -> bfloat16 bits, round to nearest even (inputs are finite)
__device__ inline uint16_t bf16_bits(float f)
{
    const uint32_t u = __float_as_uint(f);
    return (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}
__device__ inline uint16_t bf16_bits(uint16_t h) { return h; }
__device__ inline float bf16_val(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

__device__ inline f32x16_t mfma(const u16x8_t &a, const u16x8_t &b, const f32x16_t &c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a),
                                                   __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}
// 32x32 accumulator layout: register i of lane l holds row c_row(i, l), column l % 32
__device__ inline int c_row(int i, int lane) { return 8 * (i >> 2) + 4 * (lane >> 5) + (i & 3); }

// ---- parameters --------------------------------------------------------------
__global__ void k_init(float *__restrict__ P, uint32_t s_lo, uint32_t s_hi)
{
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= kNParams) return;
    for (int l = 0; l < 5; ++l) {
        const LayerDesc L = layer(l);
        if (idx >= L.w && idx < L.b) {
            uint32_t w[4];
            philox4x32_10((uint32_t)idx, 0u, kPurposeInit, 0u, s_lo, s_hi, w);
            const float a = L.init_gain * sqrtf(6.0f / (float)L.in);  // He-uniform
            P[idx] = (2.0f * u01f(w[0]) - 1.0f) * a;
            return;
        }
        if (idx >= L.b && idx < L.b + L.out) {
            P[idx] = 0.0f;
            return;
        }
    }
}

// the BF16 copies of parameter i (value w); biases have none
__device__ inline void store_bf16(uint16_t *__restrict__ T, int64_t i, float w)
{
    for (int l = 0; l < 5; ++l) {
        const LayerDesc L = layer(l);
        if (i < L.w || i >= L.b) continue;
        const int r = (int)(i - L.w) / L.out, o = (int)(i - L.w) - r * L.out;
        const uint16_t h = bf16_bits(w);
        if (l < 2) {
            T[L.t + (int64_t)o * L.in_pad + r] = h;
        } else {
            T[L.t + operand_at(r, o, kHH)] = h;
            T[L.u + operand_at(o, r, l == 4 ? kOutPad : kHH)] = h;
        }
    }
}

// every copy from the parameters (the padding stays as it was filled: 0)
__global__ void k_refresh_bf16(const float *__restrict__ P, uint16_t *__restrict__ T)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < kNParams) store_bf16(T, i, P[i]);
}

// One step of Adam; the BF16 copies of a weight are written with it.
__global__ void k_adam(float *__restrict__ P, const float *__restrict__ G, float *__restrict__ Mo,
                       float *__restrict__ Vo, uint16_t *__restrict__ T, float lr_t, float b1, float b2, float eps)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= kNParams) return;
    const float g = G[i];
    const float m = b1 * Mo[i] + (1.0f - b1) * g;
    const float v = b2 * Vo[i] + (1.0f - b2) * g * g;
    Mo[i] = m;
    Vo[i] = v;
    const float w = P[i] - lr_t * m / (sqrtf(v) + eps);
    P[i] = w;
    store_bf16(T, i, w);
}

__global__ void k_fill_u64(unsigned long long *__restrict__ p, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0ull;
}

// ---- encoder -----------------------------------------------------------------
constexpr int kEncWaves = 8;
constexpr int kEncThreads = 64 * kEncWaves;
constexpr int kEncPair = 64;                         // points a wave takes per step: two 32-row blocks
constexpr int kEncStep = kEncPair * kEncWaves;       // points a workgroup takes per step
constexpr int kEncMaxSteps = 4;
constexpr int kLd = kH1 + 8;                                   // padded LDS row of W2^T (BF16 elements)
static_assert(kEncThreads >= kH2, "the pooled-key merge takes one thread per channel");
static_assert(kEncWaves * kH2 * 8 <= kH2 * kLd * 2, "the pooled-key merge reuses the W2 buffer");

typedef short s16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

__device__ inline u16x8_t input_row(const float *__restrict__ xp)
{
    u16x8_t a = {0, 0, 0, 0, 0, 0, 0, 0};
    a[0] = bf16_bits(xp[0] * kInvSP);
    a[1] = bf16_bits(xp[1] * kInvSP);
    a[2] = bf16_bits(xp[2] * kInvSP);
    a[3] = bf16_bits(xp[3]);
    a[4] = bf16_bits(xp[4]);
    a[5] = bf16_bits(xp[5]);
    return a;
}

// (bf16(relu(a)), bf16(relu(b))) packed low/high.  Round to nearest even, then
// a signed 16-bit max with 0: a negative BF16 (and -0) has its sign bit set.
__device__ inline uint32_t relu_pk_bf16(float a, float b)
{
    const f32x2_t v = {a, b};
    const s16x2_t h = __builtin_bit_cast(s16x2_t, __builtin_convertvector(v, bf16x2_t));
    const s16x2_t z = {0, 0};
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(h, z));
}

// FP32 -> unsigned with the same order (sign-magnitude flipped); 0 never
// comes out of a finite value, so a zero key means "no point"
__device__ inline uint32_t ord_bits(float v)
{
    const uint32_t u = __float_as_uint(v);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ inline float ord_val(uint32_t o) { return __uint_as_float((o & 0x80000000u) ? (o & 0x7FFFFFFFu) : ~o); }

// Fold one 32-row block of a layer-2 column block into the lane's running
// (max, point) pair: rows ascend with the register index, so the first
// register equal to the maximum is the lowest point.
__device__ inline void fold_rows(f32x16_t a, int row0, int end, int half, float &best, int &bidx)
{
    if (row0 + 32 > end) {  // wave-uniform: the object's last rows
#pragma unroll
        for (int i = 0; i < 16; ++i)
            if (row0 + 8 * (i >> 2) + 4 * half + (i & 3) >= end) a[i] = -INFINITY;
    }
    float m = a[0];
#pragma unroll
    for (int i = 1; i < 16; ++i) m = fmaxf(m, a[i]);
    int ii = 8 * 3 + 3;
#pragma unroll
    for (int i = 14; i >= 0; --i) ii = a[i] == m ? 8 * (i >> 2) + (i & 3) : ii;
    if (m > best) {
        best = m;
        bidx = row0 + 4 * half + ii;
    }
}

// grid (ceil(Np / (kEncStep * steps)), B), kEncThreads threads.  Each wave runs its
// own 64-point steps with no barrier: layer 1 is computed transposed
// (channels x points), so a lane ends up holding 4-channel groups of one
// point; one lane-half swap per dword turns them into the layer-2 A operand
// (8 consecutive channels of one point) without going through LDS.
// Registers, not LDS, set the occupancy: the H1 of two row blocks, two
// accumulators and the running pairs take 158 VGPRs, three waves per SIMD, so a
// CU holds one workgroup of 8 waves.
__global__ __launch_bounds__(kEncThreads) __attribute__((amdgpu_waves_per_eu(2))) void
k_encode(const float *__restrict__ x, int Np, int steps, const uint16_t *__restrict__ T, const float *__restrict__ P,
         unsigned long long *__restrict__ keys)
{
    __shared__ __attribute__((aligned(16))) uint16_t sW2[kH2 * kLd];
    __shared__ __attribute__((aligned(16))) float sB1[kH1];
    const int b = blockIdx.y, tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 31, half = lane >> 5;
    for (int i = tid; i < kH2 * (kH1 / 8); i += kEncThreads) {
        const int n = i / (kH1 / 8), k8 = i % (kH1 / 8);
        *(u16x8_t *)&sW2[n * kLd + 8 * k8] = *(const u16x8_t *)&T[kT2 + (int64_t)n * kH1 + 8 * k8];
    }
    for (int i = tid; i < kH1; i += kEncThreads) sB1[i] = P[kB1 + i];
    __syncthreads();

    float best[kH2 / 32];
    int bidx[kH2 / 32];
#pragma unroll
    for (int c = 0; c < kH2 / 32; ++c) {
        best[c] = -INFINITY;
        bidx[c] = 0;
    }
    const int c0 = blockIdx.x * kEncStep * steps, c1 = min(Np, c0 + kEncStep * steps);
    for (int p0 = c0 + wave * kEncPair; p0 < c1; p0 += kEncWaves * kEncPair) {
        u16x8_t h[2][kH1 / 16];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int pt = p0 + 32 * j + r;
            u16x8_t xb = {0, 0, 0, 0, 0, 0, 0, 0};
            if (half == 0 && pt < c1) xb = input_row(x + ((int64_t)b * Np + pt) * kIn);
#pragma unroll
            for (int cb = 0; cb < kH1 / 32; ++cb) {
                // D[channel][point] = b1 + W1^T x: the bias enters as the accumulator
                f32x16_t acc;
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const f32x4_t bb = *(const f32x4_t *)&sB1[32 * cb + 8 * g + 4 * half];
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[4 * g + e] = bb[e];
                }
                const u16x8_t wa = *(const u16x8_t *)&T[kT1 + (32 * cb + r) * kInPad + 8 * half];
                acc = mfma(wa, xb, acc);
                // group g holds channels 32 cb + 8 g + 4 half + (0..3) of point r
                uint32_t pk[4][2];
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    pk[g][0] = relu_pk_bf16(acc[4 * g], acc[4 * g + 1]);
                    pk[g][1] = relu_pk_bf16(acc[4 * g + 2], acc[4 * g + 3]);
                }
                // K-step kk = 2 cb + gg covers groups 2 gg (half 0 needs both halves' copy)
                // and 2 gg + 1 (half 1 likewise): swap the upper lanes of the first
                // with the lower lanes of the second
#pragma unroll
                for (int gg = 0; gg < 2; ++gg) {
                    uint32_t v1[2] = {pk[2 * gg][0], pk[2 * gg][1]};
                    uint32_t v2[2] = {pk[2 * gg + 1][0], pk[2 * gg + 1][1]};
#pragma unroll
                    for (int d = 0; d < 2; ++d) {
                        const auto sw = __builtin_amdgcn_permlane32_swap(v1[d], v2[d], false, false);
                        v1[d] = sw[0];
                        v2[d] = sw[1];
                    }
                    const u32x4_t q = {v1[0], v1[1], v2[0], v2[1]};
                    h[j][2 * cb + gg] = __builtin_bit_cast(u16x8_t, q);
                }
            }
        }
#pragma unroll
        for (int cb2 = 0; cb2 < kH2 / 32; ++cb2) {
            f32x16_t a0 = {}, a1 = {};
#pragma unroll
            for (int kk = 0; kk < kH1 / 16; ++kk) {
                const u16x8_t bv = *(const u16x8_t *)&sW2[(32 * cb2 + r) * kLd + 16 * kk + 8 * half];
                a0 = mfma(h[0][kk], bv, a0);
                a1 = mfma(h[1][kk], bv, a1);
            }
            fold_rows(a0, p0, c1, half, best[cb2], bidx[cb2]);
            fold_rows(a1, p0 + 32, c1, half, best[cb2], bidx[cb2]);
            __builtin_amdgcn_sched_barrier(0);  // keep the next block's LDS reads after this fold
        }
    }

    // merge: the two lane halves, then the waves (through LDS), then the
    // workgroups (64-bit atomicMax of (ordered value, inverted point))
    __syncthreads();  // every wave is done with W2
    unsigned long long *sKey = reinterpret_cast<unsigned long long *>(sW2);
#pragma unroll
    for (int c = 0; c < kH2 / 32; ++c) {
        const unsigned long long key =
            best[c] == -INFINITY ? 0ull
                                 : ((unsigned long long)ord_bits(best[c]) << 32) | (0xFFFFFFFFu - (uint32_t)bidx[c]);
        const uint32_t lo = __shfl_xor((uint32_t)key, 32, 64), hi = __shfl_xor((uint32_t)(key >> 32), 32, 64);
        const unsigned long long other = ((unsigned long long)hi << 32) | lo;
        if (half == 0) sKey[wave * kH2 + 32 * c + r] = key > other ? key : other;
    }
    __syncthreads();
    if (tid < kH2) {
        unsigned long long k = sKey[tid];
#pragma unroll
        for (int w = 1; w < kEncWaves; ++w) {
            const unsigned long long o = sKey[w * kH2 + tid];
            k = o > k ? o : k;
        }
        if (k) atomicMax(&keys[(int64_t)b * kH2 + tid], k);
    }
}

// ---- head ---------------------------------------------------------------------
constexpr int kHeadWaves = kHH / 32;
constexpr int kHeadThreads = 64 * kHeadWaves;
constexpr int kActLd = kHH + 8;  // padded LDS row of 32 objects' BF16 activations

// Pooling and the three layers for 32 objects (block) of B.  feat = relu(max
// pre-activation + b2); arg = its point, or 0 where the channel is cut to zero
// (every point then ties at 0 and the lowest wins).  Each key is reset to 0 once
// read, ready for the next pass.  A wave computes 32 columns of a layer from the
// block's activations in LDS; its 16 weight operands of a layer are all loaded
// before the layer below is done.  What bounds it: latency (a chain of three
// products of 16 steps in one block per 32 objects): 13 us for 512 objects,
// where pooling and three launches took 5 + 17 us and three copies.  out2, feat2, arg2: the caller's copies, or null.
__global__ __launch_bounds__(kHeadThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void
k_head(unsigned long long *__restrict__ keys, int B, const float *__restrict__ P, const uint16_t *__restrict__ T,
       float *__restrict__ feat, int32_t *__restrict__ arg, float *__restrict__ ua, float *__restrict__ ub,
       float *__restrict__ out, float *__restrict__ feat2, int32_t *__restrict__ arg2, float *__restrict__ out2)
{
    __shared__ __attribute__((aligned(16))) uint16_t act[2][32 * kActLd];
    const int tid = threadIdx.x, lane = tid & 63, r = lane & 31, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), m0 = blockIdx.x * 32, n = 32 * wave + r;
    u16x8_t w[kHH / 16];
    auto weights = [&](int64_t t, int tile) {
#pragma unroll
        for (int k = 0; k < kHH / 16; ++k) w[k] = *(const u16x8_t *)&T[t + ((tile * (kHH / 16) + k) * 64 + lane) * 8];
    };
    auto product = [&](const uint16_t *A) {
        f32x16_t acc = {};
#pragma unroll
        for (int k = 0; k < kHH / 16; ++k) acc = mfma(*(const u16x8_t *)&A[r * kActLd + 16 * k + 8 * half], w[k], acc);
        return acc;
    };
    weights(kTa, wave);
    // thread: one channel of every other object; all its keys are loaded before the first is used
    const int c = tid % kH2, r0 = tid / kH2;
    constexpr int kRows = 32 * kH2 / kHeadThreads, kRowStep = kHeadThreads / kH2;
    unsigned long long key[kRows];
#pragma unroll
    for (int q = 0; q < kRows; ++q) {
        const int row = m0 + r0 + kRowStep * q;
        key[q] = row < B ? keys[(int64_t)row * kH2 + c] : 0ull;
    }
    const float b2 = P[kB2 + c];
#pragma unroll
    for (int q = 0; q < kRows; ++q) {
        const int row = r0 + kRowStep * q;
        float f = 0.0f;
        if (m0 + row < B) {
            const int64_t id = (int64_t)(m0 + row) * kH2 + c;
            keys[id] = 0ull;
            int32_t a = 0;
            if (key[q]) {
                const float t = ord_val((uint32_t)(key[q] >> 32)) + b2;
                if (t > 0.0f) {
                    f = t;
                    a = (int32_t)(0xFFFFFFFFu - (uint32_t)key[q]);
                }
            }
            feat[id] = f;
            arg[id] = a;
            if (feat2) feat2[id] = f;
            if (arg2) arg2[id] = a;
        }
        act[0][row * kActLd + c] = bf16_bits(f);
    }
    __syncthreads();
#pragma unroll
    for (int l = 0; l < 2; ++l) {
        f32x16_t acc = product(act[l]);
        weights(l == 0 ? kTb : kTc, l == 0 ? wave : min(wave, kOutPad / 32 - 1));  // the next layer's
        const float bias = P[(l == 0 ? kBa : kBb) + n];
        float *u = l == 0 ? ua : ub;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int row = c_row(i, lane);
            const float v = fmaxf(acc[i] + bias, 0.0f);
            if (m0 + row < B) u[(int64_t)(m0 + row) * kHH + n] = v;
            act[1 - l][row * kActLd + n] = bf16_bits(v);
        }
        __syncthreads();
    }
    if (32 * wave < kOut) {
        const f32x16_t acc = product(act[0]);
        if (n < kOut) {
            const float bias = P[kBc + n];
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int row = m0 + c_row(i, lane);
                if (row >= B) continue;
                out[(int64_t)row * kOut + n] = acc[i] + bias;
                if (out2) out2[(int64_t)row * kOut + n] = acc[i] + bias;
            }
        }
    }
}

// Input gradients of the head for 32 objects (block): dub = (dO Wc^T) [ub > 0],
// dua = (dub Wb^T) [ua > 0], dfeat = dua Wa^T.  Each is computed transposed
// (rows = inputs, columns = objects); a wave takes 32 inputs.  As separate
// products with the copies for W, 2-byte loads a row apart took 27-40 us each at
// 32 objects; the chain takes 13 us.
__global__ __launch_bounds__(kHeadThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void
k_head_bwd(int B, const uint16_t *__restrict__ T, const float *__restrict__ dO, const float *__restrict__ ua,
           const float *__restrict__ ub, float *__restrict__ dub, float *__restrict__ dua, float *__restrict__ dfeat)
{
    __shared__ __attribute__((aligned(16))) uint16_t act[2][32 * kActLd];
    const int tid = threadIdx.x, lane = tid & 63, r = lane & 31, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), m0 = blockIdx.x * 32, i0 = 32 * wave;
    constexpr int kSteps = kHH / 16;
    const int row = m0 + r;  // this lane's object in the products' columns
    // a layer's weight operands, all loaded before the layer below is done
    u16x8_t w[kSteps];
    auto weights = [&](int64_t u, int steps) {
#pragma unroll
        for (int k = 0; k < kSteps; ++k)
            if (k < steps) w[k] = *(const u16x8_t *)&T[u + ((wave * steps + k) * 64 + lane) * 8];
    };
    weights(kUc, kOutPad / 16);
    for (int i = tid; i < 32 * kOutPad; i += kHeadThreads) {
        const int q = i / kOutPad, j = i % kOutPad;
        act[0][q * kActLd + j] = m0 + q < B && j < kOut ? bf16_bits(dO[(int64_t)(m0 + q) * kOut + j]) : (uint16_t)0;
    }
    __syncthreads();
#pragma unroll
    for (int l = 0; l < 3; ++l) {
        const uint16_t *A = act[l & 1];
        f32x16_t acc = {};
#pragma unroll
        for (int k = 0; k < (l == 0 ? kOutPad / 16 : kSteps); ++k) {
            acc = mfma(w[k], *(const u16x8_t *)&A[r * kActLd + 16 * k + 8 * half], acc);
        }
        if (l < 2) weights(l == 0 ? kUb : kUa, kSteps);
        const float *mask = l == 0 ? ub : ua;
        float *d = l == 0 ? dub : l == 1 ? dua : dfeat;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int in = i0 + 8 * g + 4 * half;  // four consecutive inputs of this lane's object
            float4 v = make_float4(acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]);
            if (row < B) {
                if (l < 2) {
                    const float4 m = *(const float4 *)&mask[(int64_t)row * kHH + in];
                    v = make_float4(m.x > 0.0f ? v.x : 0.0f, m.y > 0.0f ? v.y : 0.0f, m.z > 0.0f ? v.z : 0.0f,
                                    m.w > 0.0f ? v.w : 0.0f);
                }
                *(float4 *)&d[(int64_t)row * kHH + in] = v;
            }
            uint16_t *q = &act[1 - (l & 1)][r * kActLd + in];
            q[0] = bf16_bits(v.x);
            q[1] = bf16_bits(v.y);
            q[2] = bf16_bits(v.z);
            q[3] = bf16_bits(v.w);
        }
        __syncthreads();
    }
}

// ---- mixture NLL -------------------------------------------------------------
__device__ inline void log_softmax8(const float *o, float lp[kM])
{
    float mx = o[0];
#pragma unroll
    for (int m = 1; m < kM; ++m) mx = fmaxf(mx, o[m]);
    float s = 0.0f;
#pragma unroll
    for (int m = 0; m < kM; ++m) s += expf(o[m] - mx);
    const float l = mx + logf(s);
#pragma unroll
    for (int m = 0; m < kM; ++m) lp[m] = o[m] - l;
}

__device__ inline float clamp_ls(float v) { return fminf(fmaxf(v, kLsMin), kLsMax); }

constexpr int kNllTile = 64;  // targets of an object held in LDS at a time
constexpr int kNllThreads = 256;

// Workgroup per object: NLL and responsibilities of its targets, and from them
// the gradient of the batch-mean NLL at its outputs (thread per output, targets
// in order).  The first and last objects also score any targets before and
// after the offsets' range (their NLL counts in the loss).  A thread per target
// and then one per (object, output) over global memory took 8 + 27 us at 32
// objects of 64 targets.
__global__ __launch_bounds__(kNllThreads) void k_nll(const float *__restrict__ out, const float *__restrict__ tg,
                                                     const int32_t *__restrict__ off, int B, int T, float inv_T,
                                                     float *__restrict__ nll, float *__restrict__ dO)
{
    __shared__ float o[kOut], inv_s[kM * kY], lps[kM], comp[kNllTile][kM], resp[kNllTile][kM], y[kNllTile][kY];
    const int b = blockIdx.x, tid = threadIdx.x;
    if (tid < kOut) o[tid] = out[(int64_t)b * kOut + tid];
    __syncthreads();
    if (tid < kM * kY) inv_s[tid] = expf(-clamp_ls(o[kM + kM * kY + tid]));
    if (tid == 0) {
        float lp[kM];
        log_softmax8(o, lp);
#pragma unroll
        for (int m = 0; m < kM; ++m) lps[m] = lp[m];
    }
    __syncthreads();
    const int t0 = max(off[b], 0), t1 = min(off[b + 1], T);
    const int s0 = b == 0 ? 0 : t0, s1 = b == B - 1 ? T : t1;
    const float half_log_2pi = 0.91893853320467274f;
    const int j = tid, m = j < kM ? j : ((j - kM) % (kM * kY)) / kY, d = j < kM ? 0 : (j - kM) % kY;
    const float raw = j < kOut ? o[j] : 0.0f, mu = j < kM || j >= kOut ? 0.0f : o[kM + m * kY + d];
    const float pi = j < kM ? expf(lps[m]) : 0.0f;
    float g = 0.0f;
    for (int base = s0; base < s1; base += kNllTile) {
        const int nt = min(kNllTile, s1 - base);
        for (int i = tid; i < nt * kY; i += kNllThreads) (&y[0][0])[i] = tg[(int64_t)base * kY + i];
        __syncthreads();
        for (int i = tid; i < nt * kM; i += kNllThreads) {
            const int t = i / kM, mm = i % kM;
            float c = lps[mm];
            for (int q = 0; q < kY; ++q) {
                const float ls = clamp_ls(o[kM + kM * kY + mm * kY + q]);
                const float z = (y[t][q] - o[kM + mm * kY + q]) * inv_s[mm * kY + q];
                c += -0.5f * z * z - ls - half_log_2pi;
            }
            comp[t][mm] = c;
        }
        __syncthreads();
        for (int t = tid; t < nt; t += kNllThreads) {
            float mx = -INFINITY, s = 0.0f;
#pragma unroll
            for (int mm = 0; mm < kM; ++mm) mx = fmaxf(mx, comp[t][mm]);
#pragma unroll
            for (int mm = 0; mm < kM; ++mm) s += expf(comp[t][mm] - mx);
            nll[base + t] = -(mx + logf(s));
#pragma unroll
            for (int mm = 0; mm < kM; ++mm) resp[t][mm] = expf(comp[t][mm] - mx) / s;
        }
        __syncthreads();
        if (j < kOut) {
            const int e0 = max(t0 - base, 0), e1 = min(nt, t1 - base);
            if (j < kM) {
                for (int t = e0; t < e1; ++t) g += pi - resp[t][m];
            } else if (j < kM + kM * kY) {
                const float is = inv_s[j - kM];
                for (int t = e0; t < e1; ++t) g -= resp[t][m] * ((y[t][d] - mu) * is) * is;
            } else if (raw > kLsMin && raw < kLsMax) {
                const float is = inv_s[j - kM - kM * kY];
                for (int t = e0; t < e1; ++t) {
                    const float z = (y[t][d] - mu) * is;
                    g += resp[t][m] * (1.0f - z * z);
                }
            }
        }
        __syncthreads();
    }
    if (j < kOut) dO[(int64_t)b * kOut + j] = g * inv_T;
}

// ---- weight gradients -----------------------------------------------------------
constexpr int kGradThreads = 256;
constexpr int kGradTile = 64;  // objects of one channel held in LDS at a time
// tiles of 32 x 32 of the three head weights (rows = inputs): Wc, Wb, Wa
constexpr int kTilesC = (kHH / 32) * ((kOut + 31) / 32), kTilesH = (kHH / 32) * (kHH / 32);
constexpr int kGradTileBlocks = (kTilesC + 2 * kTilesH + 3) / 4;            // a wave per tile
constexpr int kGradBiasBlocks = (kOut + 2 * kHH + kGradThreads - 1) / kGradThreads;
constexpr int kGradEncBlocks = kH2 / 2;                                     // two channels per block
constexpr int kGradBlocks = kGradTileBlocks + kGradBiasBlocks + 1 + kGradEncBlocks;

struct GradArgs {
    const float *x, *feat, *ua, *ub, *dO, *dub, *dua, *dfeat, *nll, *P;
    const uint16_t *T;
    const int32_t *arg;
    float *G, *G2, *loss, *loss2, *part;  // G2, loss2: the caller's copies, or null
    int B, Np, n_targets;
};

// Everything that depends only on the chain's activations and gradients, by
// block: the head's weight gradients A^T D (K = objects) as MFMA tiles; the bias
// gradients (sums over the objects in order); the loss (fixed-order sum of the
// per-target NLL); and the encoder's backward, per (channel c, hidden k): h1 of
// the channel's argmax points is recomputed from their inputs (six multiply-adds
// each, instead of a [B][256][128] array written by one kernel and read by two),
// dW2[k][c] and db2[c] summed over the objects in order, and this channel's part
// of dW1 and db1, [128][7][256], summed over the channels by k_w1.  What bounds
// it: latency (a hundred-odd short blocks): 14 us at 32 objects, 130 us as ten
// launches.
__global__ __launch_bounds__(kGradThreads) void k_grads(GradArgs a)
{
    __shared__ float sh[kGradTile * 2][2 * kIn + 1];
    const int tid = threadIdx.x, lane = tid & 63;
    int blk = blockIdx.x;
    auto put = [&](int64_t i, float v) {
        a.G[i] = v;
        if (a.G2) a.G2[i] = v;
    };
    if (blk < kGradTileBlocks) {
        int tile = blk * 4 + __builtin_amdgcn_readfirstlane(tid >> 6);
        if (tile >= kTilesC + 2 * kTilesH) return;
        const float *A, *D;
        int nc = kHH;
        int64_t w;
        if (tile < kTilesC) {
            A = a.ub;
            D = a.dO;
            nc = kOut;
            w = kWc;
        } else if ((tile -= kTilesC) < kTilesH) {
            A = a.ua;
            D = a.dub;
            w = kWb;
        } else {
            tile -= kTilesH;
            A = a.feat;
            D = a.dua;
            w = kWa;
        }
        const int m0 = 32 * (tile % (kHH / 32)), n0 = 32 * (tile / (kHH / 32));
        const int r = lane & 31, half = lane >> 5, m = m0 + r, n = n0 + r;
        f32x16_t acc = {};
        for (int k0 = 0; k0 < a.B; k0 += 16) {
            u16x8_t av, bv;
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int k = k0 + 8 * half + q;
                av[q] = k < a.B ? bf16_bits(A[(int64_t)k * kHH + m]) : (uint16_t)0;
                bv[q] = k < a.B && n < nc ? bf16_bits(D[(int64_t)k * nc + n]) : (uint16_t)0;
            }
            acc = mfma(av, bv, acc);
        }
        if (n < nc)
#pragma unroll
            for (int i = 0; i < 16; ++i) put(w + (int64_t)(m0 + c_row(i, lane)) * nc + n, acc[i]);
        return;
    }
    blk -= kGradTileBlocks;
    if (blk < kGradBiasBlocks) {
        int i = blk * kGradThreads + tid;
        const float *D = a.dO;
        int nc = kOut;
        int64_t b = kBc;
        if (i >= kOut) {
            i -= kOut;
            nc = kHH;
            D = i < kHH ? a.dub : a.dua;
            b = i < kHH ? kBb : kBa;
            if (i >= kHH) i -= kHH;
            if (i >= kHH) return;
        }
        float s = 0.0f;
#pragma unroll 8
        for (int k = 0; k < a.B; ++k) s += D[(int64_t)k * nc + i];
        put(b + i, s);
        return;
    }
    blk -= kGradBiasBlocks;
    if (blk == 0) {
        float *s = &sh[0][0];
        float v = 0.0f;
        for (int t = tid; t < a.n_targets; t += kGradThreads) v += a.nll[t];
        s[tid] = v;
        __syncthreads();
        for (int w = kGradThreads / 2; w > 0; w >>= 1) {
            if (tid < w) s[tid] += s[tid + w];
            __syncthreads();
        }
        if (tid == 0) {
            a.loss[0] = s[0] / (float)a.n_targets;
            if (a.loss2) a.loss2[0] = s[0] / (float)a.n_targets;
        }
        return;
    }
    // encoder: threads 0-127 channel c0, 128-255 channel c0 + 1; k = hidden unit
    const int c0 = 2 * (blk - 1), half = tid >> 7, c = c0 + half, k = tid & (kH1 - 1);
    float w1[kIn];
#pragma unroll
    for (int i = 0; i < kIn; ++i) w1[i] = bf16_val(a.T[kT1 + k * kInPad + i]);
    const float b1 = a.P[kB1 + k], w2 = bf16_val(a.T[kT2 + (int64_t)c * kH1 + k]);
    float s = 0.0f, sb = 0.0f, p[kIn + 1] = {0, 0, 0, 0, 0, 0, 0};
    for (int b0 = 0; b0 < a.B; b0 += kGradTile) {
        const int nb = min(kGradTile, a.B - b0);
        __syncthreads();
        // per (object, channel): the point as read and as BF16, and the channel's gradient
        for (int i = tid; i < 2 * nb; i += kGradThreads) {
            const int b = b0 + (i >> 1), cc = c0 + (i & 1);
            const int64_t id = (int64_t)b * kH2 + cc;
            const float *xp = a.x + ((int64_t)b * a.Np + a.arg[id]) * kIn;
            const u16x8_t xr = input_row(xp);
#pragma unroll
            for (int q = 0; q < kIn; ++q) {
                sh[i][q] = bf16_val(xr[q]);
                sh[i][kIn + q] = q < 3 ? xp[q] * kInvSP : xp[q];
            }
            sh[i][2 * kIn] = a.feat[id] > 0.0f ? a.dfeat[id] : 0.0f;
        }
        __syncthreads();
        for (int b = 0; b < nb; ++b) {
            const float *v = sh[2 * b + half];
            float z = 0.0f;
#pragma unroll
            for (int i = 0; i < kIn; ++i) z = fmaf(v[i], w1[i], z);
            const float h = bf16_val(bf16_bits(fmaxf(z + b1, 0.0f))), g = v[2 * kIn];
            s = fmaf(h, g, s);
            sb += g;
            const float d = h <= 0.0f ? 0.0f : w2 * g;
            if (d != 0.0f) {  // also keeps an infinite input of a cut unit out of the sum
#pragma unroll
                for (int i = 0; i < kIn; ++i) p[i] = fmaf(v[kIn + i], d, p[i]);
                p[kIn] += d;
            }
        }
    }
    put(kW2 + (int64_t)k * kH2 + c, s);
    if (k == 0) put(kB2 + c, sb);
#pragma unroll
    for (int i = 0; i <= kIn; ++i) a.part[((int64_t)k * (kIn + 1) + i) * kH2 + c] = p[i];
}

// dW1[0..5][k] and db1[k]: workgroup per hidden unit k, a thread per channel's part
__global__ __launch_bounds__(kH2) void k_w1(const float *__restrict__ part, float *__restrict__ G,
                                            float *__restrict__ G2)
{
    __shared__ float s[kIn + 1][kH2 / 64];
    const int k = blockIdx.x, tid = threadIdx.x;
#pragma unroll
    for (int i = 0; i <= kIn; ++i) {
        float v = part[((int64_t)k * (kIn + 1) + i) * kH2 + tid];
        for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
        if ((tid & 63) == 0) s[i][tid >> 6] = v;
    }
    __syncthreads();
    if (tid <= kIn) {
        const float v = (s[tid][0] + s[tid][1]) + (s[tid][2] + s[tid][3]);
        const int64_t at = tid < kIn ? kW1 + (int64_t)tid * kH1 + k : kB1 + k;
        G[at] = v;
        if (G2) G2[at] = v;
    }
}

// ---- sampler -----------------------------------------------------------------
__device__ inline float u01_open(uint32_t w) { return (float)((w >> 8) + 1u) * (1.0f / 16777216.0f); }

__global__ void k_sample(const float *__restrict__ o, int n, uint32_t s_lo, uint32_t s_hi, float ufrac, float d_lo,
                         float d_hi, float *__restrict__ poses)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    uint32_t w[12];
    philox4x32_10((uint32_t)i, 0u, kPurposeSample, 0u, s_lo, s_hi, w);
    philox4x32_10((uint32_t)i, 1u, kPurposeSample, 0u, s_lo, s_hi, w + 4);
    philox4x32_10((uint32_t)i, 2u, kPurposeSample, 0u, s_lo, s_hi, w + 8);
    float R[3][3], t[3];
    if (u01f(w[0]) < ufrac) {
        // uniform fallback: Shoemake rotation, direction on the +z hemisphere, distance U[d_lo, d_hi]
        const float u1 = u01f(w[1]);
        const float a = sqrtf(1.0f - u1), bq = sqrtf(u1);
        float s2, c2, s3, c3;
        sincospif(2.0f * u01f(w[2]), &s2, &c2);
        sincospif(2.0f * u01f(w[3]), &s3, &c3);
        const float qx = a * s2, qy = a * c2, qz = bq * s3, qw = bq * c3;
        R[0][0] = 1 - 2 * (qy * qy + qz * qz); R[0][1] = 2 * (qx * qy - qz * qw); R[0][2] = 2 * (qx * qz + qy * qw);
        R[1][0] = 2 * (qx * qy + qz * qw); R[1][1] = 1 - 2 * (qx * qx + qz * qz); R[1][2] = 2 * (qy * qz - qx * qw);
        R[2][0] = 2 * (qx * qz - qy * qw); R[2][1] = 2 * (qy * qz + qx * qw); R[2][2] = 1 - 2 * (qx * qx + qy * qy);
        const float cz = u01f(w[4]);
        float sp, cp;
        sincospif(2.0f * u01f(w[5]), &sp, &cp);
        const float d = d_lo + (d_hi - d_lo) * u01f(w[6]);
        const float sz = sqrtf(fmaxf(0.0f, 1.0f - cz * cz));
        t[0] = d * sz * cp;
        t[1] = d * sz * sp;
        t[2] = d * cz;
    } else {
        float lp[kM];
        log_softmax8(o, lp);
        const float uc = u01f(w[1]);
        float cum = 0.0f;
        int m = kM - 1;
        for (int c = 0; c < kM; ++c) {
            cum += expf(lp[c]);
            if (uc < cum) {
                m = c;
                break;
            }
        }
        float z[10];
#pragma unroll
        for (int j = 0; j < 5; ++j) {
            const float rr = sqrtf(-2.0f * logf(u01_open(w[2 + 2 * j])));
            float sn, cs;
            sincospif(2.0f * u01f(w[3 + 2 * j]), &sn, &cs);
            z[2 * j] = rr * cs;
            z[2 * j + 1] = rr * sn;
        }
        float y[kY];
#pragma unroll
        for (int d = 0; d < kY; ++d)
            y[d] = o[kM + m * kY + d] + expf(clamp_ls(o[kM + kM * kY + m * kY + d])) * z[d];
        // Gram-Schmidt of (y0..2, y3..5): columns b1, b2, b1 x b2
        const float n1 = fmaxf(sqrtf(y[0] * y[0] + y[1] * y[1] + y[2] * y[2]), 1e-8f);
        const float b1[3] = {y[0] / n1, y[1] / n1, y[2] / n1};
        const float dp = b1[0] * y[3] + b1[1] * y[4] + b1[2] * y[5];
        float v[3] = {y[3] - dp * b1[0], y[4] - dp * b1[1], y[5] - dp * b1[2]};
        const float n2 = fmaxf(sqrtf(v[0] * v[0] + v[1] * v[1] + v[2] * v[2]), 1e-8f);
        const float b2[3] = {v[0] / n2, v[1] / n2, v[2] / n2};
        const float b3[3] = {b1[1] * b2[2] - b1[2] * b2[1], b1[2] * b2[0] - b1[0] * b2[2],
                             b1[0] * b2[1] - b1[1] * b2[0]};
        for (int r = 0; r < 3; ++r) {
            R[r][0] = b1[r];
            R[r][1] = b2[r];
            R[r][2] = b3[r];
            t[r] = y[6 + r] * kST;
        }
    }
    float *q = poses + (int64_t)i * 12;
    for (int r = 0; r < 3; ++r) {
        q[4 * r + 0] = R[r][0];
        q[4 * r + 1] = R[r][1];
        q[4 * r + 2] = R[r][2];
        q[4 * r + 3] = t[r];
    }
}

inline unsigned blocks(int64_t n, int t) { return (unsigned)((n + t - 1) / t); }

}  // namespace prop
}  // namespace lg

using namespace lg;
using namespace lg::prop;

struct lg_prop {
    int device = 0;
    int max_batch = 0, max_points = 0, max_targets = 0;
    int64_t step = 0;
    void *slab = nullptr;
    float *P, *G, *Mo, *Vo;       // [kNParams]
    uint16_t *T;                  // [kNT]
    unsigned long long *keys;     // [maxB][256], all 0 between forward passes
    bool keys_dirty = false;      // a forward pass stopped between k_encode and k_head
    float *feat, *ua, *ub, *out;  // [maxB][256] x3, [maxB][152]
    float *dO, *dub, *dua, *dfeat;
    int32_t *arg;                 // [maxB][256]
    float *nll;                   // [maxT]
    float *part;                  // [128][7][256], see k_grads
    float *loss;                  // [1]
};

namespace {

hipStream_t st(void *s) { return reinterpret_cast<hipStream_t>(s); }

lg_status check_batch(const lg_prop *p, const float *x, int B, int Np)
{
    if (!p) return fail(LG_EINVAL, "null proposer");
    if (!x) return fail(LG_EINVAL, "null input points");
    if (B < 1 || B > p->max_batch) return fail(LG_EINVAL, "batch outside [1, max_batch]");
    if (Np < 1 || Np > p->max_points) return fail(LG_EINVAL, "point count outside [1, max_points]");
    return LG_OK;
}

// out2, feat2, arg2: the caller's copies of the outputs, or null
lg_status forward(lg_prop *p, const float *x, int B, int Np, hipStream_t s, float *out2 = nullptr,
                  float *feat2 = nullptr, int32_t *arg2 = nullptr)
{
    // k_head leaves the keys it read at 0, so the next pass needs no fill
    if (p->keys_dirty)
        hipLaunchKernelGGL(k_fill_u64, dim3(blocks((int64_t)p->max_batch * kH2, 256)), dim3(256), 0, s, p->keys,
                           (int64_t)p->max_batch * kH2);
    p->keys_dirty = true;
    // Steps per wave: as many as leave 512 workgroups, two rounds of the 256 CUs; each
    // stages W2 again, so no more than that (32 objects of 2,048 points: 4 steps 34 us,
    // 1 step 14 us).  With the line at 256, where the last round may be nearly empty,
    // 192 and 384 objects take 48 and 77 us instead of 43 and 66 (128 and 256 objects 4 %
    // less); at 1,024, 256 and 512 objects take 6 and 4 % more.
    int steps = kEncMaxSteps;
    while (steps > 1 && (int64_t)B * blocks(Np, kEncStep * steps) < 512) steps >>= 1;
    hipLaunchKernelGGL(k_encode, dim3(blocks(Np, kEncStep * steps), B), dim3(kEncThreads), 0, s, x, Np, steps, p->T,
                       p->P, p->keys);
    hipLaunchKernelGGL(k_head, dim3(blocks(B, 32)), dim3(kHeadThreads), 0, s, p->keys, B, p->P, p->T, p->feat, p->arg,
                       p->ua, p->ub, p->out, feat2, arg2, out2);
    if (hipPeekAtLastError() == hipSuccess) p->keys_dirty = false;
    LG_HIP(hipGetLastError());
    return LG_OK;
}

// loss2, grad2: the caller's copies, or null
lg_status backward(lg_prop *p, const float *x, int B, int Np, const float *tg, const int32_t *off, int T, float *loss2,
                   float *grad2, hipStream_t s)
{
    lg_status e = forward(p, x, B, Np, s);
    if (e != LG_OK) return e;
    hipLaunchKernelGGL(k_nll, dim3(B), dim3(kNllThreads), 0, s, p->out, tg, off, B, T, 1.0f / (float)T, p->nll, p->dO);
    hipLaunchKernelGGL(k_head_bwd, dim3(blocks(B, 32)), dim3(kHeadThreads), 0, s, B, p->T, p->dO, p->ua, p->ub, p->dub,
                       p->dua, p->dfeat);
    const GradArgs a{x,     p->feat, p->ua, p->ub, p->dO, p->dub, p->dua,  p->dfeat, p->nll,  p->P, p->T,
                     p->arg, p->G,   grad2, p->loss, loss2, p->part, B, Np, T};
    hipLaunchKernelGGL(k_grads, dim3(kGradBlocks), dim3(kGradThreads), 0, s, a);
    hipLaunchKernelGGL(k_w1, dim3(kH1), dim3(kH2), 0, s, p->part, p->G, grad2);
    LG_HIP(hipGetLastError());
    return LG_OK;
}

}  // namespace

extern "C" {

int64_t lg_prop_num_params(void) { return kNParams; }

lg_status lg_prop_create(const lg_prop_params *params, void *stream, lg_prop **out)
{
    if (!params || !out) return fail(LG_EINVAL, "null params or output handle");
    *out = nullptr;
    const int B = params->max_batch, N = params->max_points, T = params->max_targets;
    if (B < 1 || B > 4096 || N < 1 || N > (1 << 24) || T < 1 || T > (1 << 26))
        return fail(LG_EINVAL, "max_batch in [1, 4096], max_points in [1, 2^24], max_targets in [1, 2^26]");
    lg_prop *p = new lg_prop();
    p->max_batch = B;
    p->max_points = N;
    p->max_targets = T;
    LG_HIP(hipGetDevice(&p->device));
    // one slab: every piece 256-byte aligned
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t o = off;
        off += (bytes + 255) & ~(size_t)255;
        return o;
    };
    const size_t oP = take(kNParams * 4), oG = take(kNParams * 4), oM = take(kNParams * 4), oV = take(kNParams * 4);
    const size_t oT = take(kNT * 2), oK = take((size_t)B * kH2 * 8);
    const size_t oF = take((size_t)B * kH2 * 4), oUa = take((size_t)B * kHH * 4), oUb = take((size_t)B * kHH * 4);
    const size_t oO = take((size_t)B * kOut * 4), oDO = take((size_t)B * kOut * 4);
    const size_t oDub = take((size_t)B * kHH * 4), oDua = take((size_t)B * kHH * 4), oDf = take((size_t)B * kH2 * 4);
    const size_t oA = take((size_t)B * kH2 * 4), oN = take((size_t)T * 4);
    const size_t oPt = take((size_t)kH1 * (kIn + 1) * kH2 * 4), oL = take(4);
    hipError_t e = hipMalloc(&p->slab, off);
    if (e != hipSuccess) {
        delete p;
        return hip_fail(e, "hipMalloc(proposer)");
    }
    char *base = static_cast<char *>(p->slab);
    p->P = (float *)(base + oP);
    p->G = (float *)(base + oG);
    p->Mo = (float *)(base + oM);
    p->Vo = (float *)(base + oV);
    p->T = (uint16_t *)(base + oT);
    p->keys = (unsigned long long *)(base + oK);
    p->feat = (float *)(base + oF);
    p->ua = (float *)(base + oUa);
    p->ub = (float *)(base + oUb);
    p->out = (float *)(base + oO);
    p->dO = (float *)(base + oDO);
    p->dub = (float *)(base + oDub);
    p->dua = (float *)(base + oDua);
    p->dfeat = (float *)(base + oDf);
    p->arg = (int32_t *)(base + oA);
    p->nll = (float *)(base + oN);
    p->part = (float *)(base + oPt);
    p->loss = (float *)(base + oL);
    hipStream_t s = st(stream);
    hipLaunchKernelGGL(k_init, dim3(blocks(kNParams, 256)), dim3(256), 0, s, p->P,
                       (uint32_t)params->seed, (uint32_t)(params->seed >> 32));
    static_assert(kNT % 4 == 0, "the copies are filled 8 bytes at a time");
    hipLaunchKernelGGL(k_fill_u64, dim3(blocks(kNT / 4, 256)), dim3(256), 0, s,
                       reinterpret_cast<unsigned long long *>(p->T), kNT / 4);
    hipLaunchKernelGGL(k_refresh_bf16, dim3(blocks(kNParams, 256)), dim3(256), 0, s, p->P, p->T);
    hipLaunchKernelGGL(k_fill_u64, dim3(blocks((int64_t)B * kH2, 256)), dim3(256), 0, s, p->keys, (int64_t)B * kH2);
    e = hipMemsetAsync(p->Mo, 0, kNParams * 4, s);
    if (e == hipSuccess) e = hipMemsetAsync(p->Vo, 0, kNParams * 4, s);
    if (e == hipSuccess) e = hipMemsetAsync(p->G, 0, kNParams * 4, s);
    if (e == hipSuccess) e = hipGetLastError();
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) {
        (void)hipFree(p->slab);
        delete p;
        return hip_fail(e, "proposer initialisation");
    }
    *out = p;
    return LG_OK;
}

lg_status lg_prop_release(lg_prop *p)
{
    if (!p) return LG_OK;
    (void)hipDeviceSynchronize();
    hipError_t e = hipFree(p->slab);
    delete p;
    return e == hipSuccess ? LG_OK : hip_fail(e, "hipFree(proposer)");
}

lg_status lg_prop_get_params(const lg_prop *p, float *host_out)
{
    if (!p || !host_out) return fail(LG_EINVAL, "null proposer or output");
    LG_HIP(hipDeviceSynchronize());
    LG_HIP(hipMemcpy(host_out, p->P, kNParams * 4, hipMemcpyDeviceToHost));
    return LG_OK;
}

lg_status lg_prop_set_params(lg_prop *p, const float *host_in)
{
    if (!p || !host_in) return fail(LG_EINVAL, "null proposer or input");
    LG_HIP(hipDeviceSynchronize());
    LG_HIP(hipMemcpy(p->P, host_in, kNParams * 4, hipMemcpyHostToDevice));
    LG_HIP(hipMemset(p->Mo, 0, kNParams * 4));
    LG_HIP(hipMemset(p->Vo, 0, kNParams * 4));
    hipLaunchKernelGGL(k_refresh_bf16, dim3(blocks(kNParams, 256)), dim3(256), 0, 0, p->P, p->T);
    LG_HIP(hipGetLastError());
    LG_HIP(hipDeviceSynchronize());
    p->step = 0;
    return LG_OK;
}

lg_status lg_prop_forward(lg_prop *p, const float *x, int32_t B, int32_t Np, float *out, float *feat, int32_t *arg,
                          void *stream)
{
    lg_status e = check_batch(p, x, B, Np);
    if (e != LG_OK) return e;
    hipStream_t s = st(stream);
    return forward(p, x, B, Np, s, out, feat, arg);
}

lg_status lg_prop_backward(lg_prop *p, const float *x, int32_t B, int32_t Np, const float *targets,
                           const int32_t *offsets, int32_t T, float *loss, float *grad, void *stream)
{
    lg_status e = check_batch(p, x, B, Np);
    if (e != LG_OK) return e;
    if (!targets || !offsets) return fail(LG_EINVAL, "null targets or offsets");
    if (T < 1 || T > p->max_targets) return fail(LG_EINVAL, "target count outside [1, max_targets]");
    hipStream_t s = st(stream);
    return backward(p, x, B, Np, targets, offsets, T, loss, grad, s);
}

lg_status lg_prop_adam(lg_prop *p, float lr, float beta1, float beta2, float eps, void *stream)
{
    if (!p) return fail(LG_EINVAL, "null proposer");
    if (!(lr >= 0.0f) || !(beta1 >= 0.0f && beta1 < 1.0f) || !(beta2 >= 0.0f && beta2 < 1.0f) || !(eps > 0.0f))
        return fail(LG_EINVAL, "lr >= 0, beta1 and beta2 in [0, 1), eps > 0");
    hipStream_t s = st(stream);
    p->step += 1;
    const double bc1 = 1.0 - pow((double)beta1, (double)p->step), bc2 = 1.0 - pow((double)beta2, (double)p->step);
    const float lr_t = (float)(lr * sqrt(bc2) / bc1);
    hipLaunchKernelGGL(k_adam, dim3(blocks(kNParams, 256)), dim3(256), 0, s, p->P, p->G, p->Mo, p->Vo, p->T, lr_t,
                       beta1, beta2, eps);
    LG_HIP(hipGetLastError());
    return LG_OK;
}

lg_status lg_prop_train_step(lg_prop *p, const float *x, int32_t B, int32_t Np, const float *targets,
                             const int32_t *offsets, int32_t T, float lr, float *loss, void *stream)
{
    lg_status e = lg_prop_backward(p, x, B, Np, targets, offsets, T, loss, nullptr, stream);
    if (e != LG_OK) return e;
    return lg_prop_adam(p, lr, 0.9f, 0.999f, 1e-8f, stream);
}

lg_status lg_prop_sample_mixture(const float *mix, int32_t n_poses, uint64_t seed, float uniform_frac, float d_lo,
                                 float d_hi, float *poses, void *stream)
{
    if (n_poses < 0) return fail(LG_EINVAL, "negative pose count");
    if (n_poses == 0) return LG_OK;
    if (!mix || !poses) return fail(LG_EINVAL, "null mixture or poses");
    if (!(uniform_frac >= 0.0f && uniform_frac <= 1.0f)) return fail(LG_EINVAL, "uniform_frac outside [0, 1]");
    if (!(d_lo >= 0.0f && d_lo <= d_hi)) return fail(LG_EINVAL, "need 0 <= d_lo <= d_hi");
    hipLaunchKernelGGL(k_sample, dim3(blocks(n_poses, 256)), dim3(256), 0, st(stream), mix, n_poses, (uint32_t)seed,
                       (uint32_t)(seed >> 32), uniform_frac, d_lo, d_hi, poses);
    LG_HIP(hipGetLastError());
    return LG_OK;
}

lg_status lg_prop_sample(lg_prop *p, const float *x, int32_t Np, int32_t n_poses, uint64_t seed, float uniform_frac,
                         float d_lo, float d_hi, float *poses, void *stream)
{
    lg_status e = check_batch(p, x, 1, Np);
    if (e != LG_OK) return e;
    if (n_poses < 0) return fail(LG_EINVAL, "negative pose count");
    if (n_poses == 0) return LG_OK;
    if (!poses) return fail(LG_EINVAL, "null poses");
    if (!(uniform_frac >= 0.0f && uniform_frac <= 1.0f)) return fail(LG_EINVAL, "uniform_frac outside [0, 1]");
    if (!(d_lo >= 0.0f && d_lo <= d_hi)) return fail(LG_EINVAL, "need 0 <= d_lo <= d_hi");
    hipStream_t s = st(stream);
    e = forward(p, x, 1, Np, s);
    if (e != LG_OK) return e;
    return lg_prop_sample_mixture(p->out, n_poses, seed, uniform_frac, d_lo, d_hi, poses, stream);
}

}  // extern "C"
