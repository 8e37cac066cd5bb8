// Learned pre-alignment filter: per-pair features and a 16-128-128-1 MLP
// with bf16 weights and activations, fp32 accumulation on MFMA (not part of
// the paper: it predicts whether a candidate pair will pass the identity /
// coverage cut of Section IV-F, so that predicted failures skip alignment).
//
// Features of a pair (a = the shorter sequence): shared-k-mer count; seed-1
// diagonal (pos_b - pos_a) / Lb; |diag2 - diag1| / Lb; ln La; ln Lb; La / Lb;
// and |comp_a - comp_b| over 10 residue groups {AG}{ST}{DE}{NQ}{KRH}{IV}{LM}
// {FYW}{C}{P}.  They are z-scored with training statistics and cast to bf16.
//
// Layout.  A wave handles 16 pairs and computes each layer transposed,
// H^T = W X^T, with v_mfma_f32_16x16x16bf16: the 16x16 accumulator of an
// output-feature tile (lane l: features 4*(l/16)..+3 of pair l%16) is exactly
// the B operand of the next layer's K tile, so layers chain in registers.
// Training stores activations and gradients by tile of 16 pairs, feature by
// feature inside a tile ([pair / 16][feature][pair % 16], bf16): a wave's
// stores of one array share one address with immediate offsets, and both
// operands of the weight-gradient GEMMs (reductions over the batch) load 4
// consecutive pairs of a feature per lane, 512 contiguous bytes per wave.
#include <algorithm>
#include <cmath>

#include "internal.hpp"
#include "mlp.hpp"
#include "prim.hpp"

namespace pastis {
namespace {

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kIn = kMlpIn, kH = kMlpHidden;

__device__ __forceinline__ uint16_t to_bf16(float f) {
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);  // round to nearest, ties to even
    return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float from_bf16(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

__device__ __forceinline__ f32x4 mfma(bf16x4 a, bf16x4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ bf16x4 load4(const uint16_t *p) {
    const uint2 v = *(const uint2 *)p;  // 4 bf16, 8-byte aligned
    bf16x4 r;
    r[0] = (short)(v.x & 0xFFFF);
    r[1] = (short)(v.x >> 16);
    r[2] = (short)(v.y & 0xFFFF);
    r[3] = (short)(v.y >> 16);
    return r;
}

// two non-negative floats to bf16, rounded to nearest even (one instruction)
__device__ __forceinline__ uint32_t to_bf16x2(float a, float b) {
    typedef float float2_t __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
    const float2_t v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}

// group of residue code c (0..23), or 15: four bits per code
__device__ __forceinline__ int group_of(int c) {
    // A R N D C Q E G H I L K M F P S, then T W Y V B Z X *
    constexpr uint64_t lo = 0x1976465402382340ull;
    constexpr uint32_t hi = 0xFFFF5771u;
    return c < 16 ? (int)(lo >> (4 * c) & 15u) : (int)(hi >> (4 * (c - 16)) & 15u);
}

// Compositions, one wave per sequence: 64 residues at a time, counted by ten
// ballots.  (One thread per sequence read single bytes at the stride of a
// sequence: 479 us for 10,000 sequences of 350 residues, one wave 15 us.)
// Rows of comp hold kMlpComp floats, ten of them in use.
constexpr int kGroups = 10;
__global__ __launch_bounds__(256) void comp_kernel(const uint8_t *__restrict__ codes,
                                                   const int64_t *__restrict__ offsets, int64_t n,
                                                   float *__restrict__ comp) {
    const int lane = threadIdx.x & 63;
    for (int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); i < n; i += (int64_t)gridDim.x * 4) {
        int cnt[kGroups] = {};
        const int64_t b = offsets[i], e = offsets[i + 1];
        for (int64_t x = b + lane; x - lane < e; x += 64) {
            const int g = x < e ? group_of(codes[x]) : 15;
#pragma unroll
            for (int k = 0; k < kGroups; ++k) cnt[k] += __popcll(__ballot(g == k));
        }
        const float L = (float)((e - b) > 0 ? (e - b) : 1);
        int mine = 0;
#pragma unroll
        for (int k = 0; k < kGroups; ++k) mine = lane == k ? cnt[k] : mine;
        if (lane < kMlpComp) comp[i * kMlpComp + lane] = (float)mine / L;
    }
}

// One thread per pair; the 64-byte rows of F leave through LDS, 1 KB of
// consecutive bytes per store (bound by the 64 bytes written per pair; stored
// from their threads, a float at a time, 149 us for the 3.67 million candidates
// of 10,000 sequences, so 125).
__global__ __launch_bounds__(256) void features_kernel(
    const uint32_t *__restrict__ lo, const uint32_t *__restrict__ hi, const uint32_t *__restrict__ count,
    const uint32_t *__restrict__ s1, const uint32_t *__restrict__ s2, int64_t n, const int64_t *__restrict__ offsets,
    const float *__restrict__ comp, float *__restrict__ F, int wide) {
    __shared__ float4 rows[4][64][kIn / 4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int64_t q0 = ((int64_t)blockIdx.x * 4 + wave) * 64; q0 < n; q0 += (int64_t)gridDim.x * 256) {
        const int64_t q = min(q0 + lane, n - 1);
        const uint32_t i = lo[q], j = hi[q];
        const int64_t Li = offsets[i + 1] - offsets[i], Lj = offsets[j + 1] - offsets[j];
        const bool swap = !(Li < Lj || (Li == Lj && i < j));
        const float La = (float)(swap ? Lj : Li), Lb = (float)(swap ? Li : Lj);
        const uint32_t ia = swap ? j : i, ib = swap ? i : j;
        float f[kIn], c[kMlpComp];
        const float4 *ca = (const float4 *)(comp + (int64_t)ia * kMlpComp);
        const float4 *cb = (const float4 *)(comp + (int64_t)ib * kMlpComp);
#pragma unroll
        for (int x = 0; x < kMlpComp / 4; ++x) {
            const float4 u = ca[x], v = cb[x];
            c[4 * x] = fabsf(u.x - v.x);
            c[4 * x + 1] = fabsf(u.y - v.y);
            c[4 * x + 2] = fabsf(u.z - v.z);
            c[4 * x + 3] = fabsf(u.w - v.w);
        }
        f[0] = (float)count[q];
        const uint32_t k1 = s1[q], k2 = s2[q];
        auto diag = [&](uint32_t key) {
            const int p_lo = (int)(key >> 16), p_hi = (int)(key & 0xFFFF);
            const int pa = swap ? p_hi : p_lo, pb = swap ? p_lo : p_hi;
            return (float)(pb - pa);
        };
        const float d1 = k1 != kNoSeed ? diag(k1) : 0.f;
        const float d2 = k2 != kNoSeed ? diag(k2) : 0.f;
        f[1] = k1 != kNoSeed ? d1 / Lb : 0.f;
        f[2] = (k1 != kNoSeed && k2 != kNoSeed) ? fabsf(d2 - d1) / Lb : 0.f;
        f[3] = logf(La);
        f[4] = logf(Lb);
        f[5] = La / Lb;
#pragma unroll
        for (int g = 0; g < kGroups; ++g) f[6 + g] = c[g];
        // (slots swapped by row, so that neither side's accesses share banks)
#pragma unroll
        for (int x = 0; x < kIn / 4; ++x)
            rows[wave][lane][x ^ (lane & 3)] = make_float4(f[4 * x], f[4 * x + 1], f[4 * x + 2], f[4 * x + 3]);
        __builtin_amdgcn_wave_barrier();
        const int live = (int)min((int64_t)64, n - q0);
#pragma unroll
        for (int x = 0; x < kIn / 4; ++x) {
            const int row = 16 * x + (lane >> 2), part = lane & 3;
            const float4 v = rows[wave][row][part ^ (row & 3)];
            if (row >= live) continue;
            float *o = F + (q0 + row) * kIn + 4 * part;
            if (wide) {
                *(float4 *)o = v;
            } else {  // a caller's buffer off the 16-byte grid
                o[0] = v.x;
                o[1] = v.y;
                o[2] = v.z;
                o[3] = v.w;
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
}

struct Net {
    const uint16_t *W1b, *W2b, *W2Tb, *w3b;  // bf16 copies
    const float *b1, *b2, *b3;
    const float *mean, *stdv;
};

// B operand of layer 1 for this lane: features 4*kg..+3 of pair p, normalised
// (of a pair of the table where it is not valid: every load is issued at once)
__device__ __forceinline__ bf16x4 input_operand(const float *X, int64_t p, bool valid, int kg, const Net &N) {
    bf16x4 z;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int f = 4 * kg + i;
        const uint16_t h = to_bf16((X[p * kIn + f] - N.mean[f]) / N.stdv[f]);
        z[i] = valid ? (short)h : (short)0;
    }
    return z;
}

// The network on n pairs.  A block keeps the weights in LDS (38 KB, so four
// blocks and 16 waves on a CU) and each wave takes 32 pairs at a time, two B
// operands for every A operand read, with the next pairs' inputs under way: an
// iteration reads 36 KB of LDS for 32 pairs where 16 pairs used to take as much
// through the vector cache.  3.67 million pairs took 616 us that way, 361 with
// W2 in registers (two waves fit on a SIMD and leave half of its issue slots
// empty), 232 so.  The four layer-2 accumulators of a half and pair tile
// advance side by side, each over its K tiles in order, as in
// training, so the logits are the same bits (the K = 32 instruction sums in another order).
// Bound by instruction issue: some 290 vector instructions per 16 pairs for
// inputs, bias and activation beside the 72 matrix ones.
constexpr int kFwdTiles = 2;  // tiles of 16 pairs per wave and iteration
__global__ __launch_bounds__(256, 4) void forward_kernel(const float *__restrict__ X, int64_t n, Net N,
                                                         float *__restrict__ logits, int wide) {
    __shared__ __align__(16) float sb1[kH], sb2[kH], sw3[kH];
    __shared__ __align__(16) uint2 sw1[kH * kIn / 4];
    __shared__ __align__(16) uint2 sw2[8][4][64][2];  // [t2][t / 2][lane][t % 2]
    const int lane = threadIdx.x & 63, col = lane & 15, kg = lane >> 4;
    if (threadIdx.x < kH) {
        sb1[threadIdx.x] = N.b1[threadIdx.x];
        sb2[threadIdx.x] = N.b2[threadIdx.x];
        sw3[threadIdx.x] = from_bf16(N.w3b[threadIdx.x]);
    }
    for (int x = threadIdx.x; x < kH * kIn / 4; x += 256) sw1[x] = ((const uint2 *)N.W1b)[x];
    for (int x = threadIdx.x >> 6; x < 64; x += 4)  // tile (t2, t) of W2
        sw2[x >> 3][(x & 7) >> 1][lane][x & 1] =
            *(const uint2 *)(N.W2b + (16 * (x >> 3) + col) * kH + 16 * (x & 7) + 4 * kg);
    __syncthreads();
    const float b3 = N.b3[0];
    float mean[4], stdv[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        mean[i] = N.mean[4 * kg + i];
        stdv[i] = N.stdv[4 * kg + i];
    }
    const int64_t groups = (n + 16 * kFwdTiles - 1) / (16 * kFwdTiles);
    // inputs of a group, fetched one group ahead (lanes past the last pair take
    // the last pair's)
    float4 next[kFwdTiles];
    auto fetch = [&](int64_t grp) {
#pragma unroll
        for (int x = 0; x < kFwdTiles; ++x) {
            const float *src = X + min(grp * (16 * kFwdTiles) + 16 * x + col, n - 1) * kIn + 4 * kg;
            if (wide)
                next[x] = *(const float4 *)src;
            else  // a caller's buffer off the 16-byte grid
                next[x] = make_float4(src[0], src[1], src[2], src[3]);
        }
    };
    int64_t grp = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (grp < groups) fetch(grp);
    for (; grp < groups; grp += (int64_t)gridDim.x * 4) {
        const int64_t p0 = grp * (16 * kFwdTiles) + col;
        float in[kFwdTiles][4];
#pragma unroll
        for (int x = 0; x < kFwdTiles; ++x)
            in[x][0] = next[x].x, in[x][1] = next[x].y, in[x][2] = next[x].z, in[x][3] = next[x].w;
        if (grp + (int64_t)gridDim.x * 4 < groups) fetch(grp + (int64_t)gridDim.x * 4);
        bf16x4 h1[kFwdTiles][8];
#pragma unroll
        for (int x = 0; x < kFwdTiles; ++x) {
            bf16x4 z;
#pragma unroll
            for (int i = 0; i < 4; ++i) z[i] = (short)to_bf16((in[x][i] - mean[i]) / stdv[i]);
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const f32x4 a = mfma(__builtin_bit_cast(bf16x4, sw1[(16 * t + col) * (kIn / 4) + kg]), z,
                                     f32x4{0.f, 0.f, 0.f, 0.f});
                const float4 b = *(const float4 *)(sb1 + 16 * t + 4 * kg);
                const float q0 = a[0] + b.x, q1 = a[1] + b.y, q2 = a[2] + b.z, q3 = a[3] + b.w;
                const uint2 v = make_uint2(to_bf16x2(q0 > 0.f ? q0 : 0.f, q1 > 0.f ? q1 : 0.f),
                                           to_bf16x2(q2 > 0.f ? q2 : 0.f, q3 > 0.f ? q3 : 0.f));
                h1[x][t] = __builtin_bit_cast(bf16x4, v);
                if (t % 4 == 3) __builtin_amdgcn_sched_barrier(0);
            }
        }
        float part[kFwdTiles] = {};
#pragma unroll 1
        for (int half = 0; half < 2; ++half) {
            f32x4 acc[kFwdTiles][4];
#pragma unroll
            for (int x = 0; x < kFwdTiles; ++x)
#pragma unroll
                for (int u = 0; u < 4; ++u) acc[x][u] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int tp = 0; tp < 4; ++tp) {
                // (the scheduler would lift every read of the weights to the top
                // and spill them)
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const uint4 w = *(const uint4 *)&sw2[4 * half + u][tp][lane][0];
                    const bf16x4 lo = __builtin_bit_cast(bf16x4, make_uint2(w.x, w.y));
                    const bf16x4 hi = __builtin_bit_cast(bf16x4, make_uint2(w.z, w.w));
#pragma unroll
                    for (int x = 0; x < kFwdTiles; ++x) acc[x][u] = mfma(lo, h1[x][2 * tp], acc[x][u]);
#pragma unroll
                    for (int x = 0; x < kFwdTiles; ++x) acc[x][u] = mfma(hi, h1[x][2 * tp + 1], acc[x][u]);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int f = 16 * (4 * half + u) + 4 * kg;
                const float4 b = *(const float4 *)(sb2 + f), w = *(const float4 *)(sw3 + f);
#pragma unroll
                for (int x = 0; x < kFwdTiles; ++x) {
                    const f32x4 a = acc[x][u];
                    const float q0 = a[0] + b.x, q1 = a[1] + b.y, q2 = a[2] + b.z, q3 = a[3] + b.w;
                    const uint32_t v0 = to_bf16x2(q0 > 0.f ? q0 : 0.f, q1 > 0.f ? q1 : 0.f);
                    const uint32_t v1 = to_bf16x2(q2 > 0.f ? q2 : 0.f, q3 > 0.f ? q3 : 0.f);
                    part[x] += w.x * __uint_as_float(v0 << 16);
                    part[x] += w.y * __uint_as_float(v0 & 0xFFFF0000u);
                    part[x] += w.z * __uint_as_float(v1 << 16);
                    part[x] += w.w * __uint_as_float(v1 & 0xFFFF0000u);
                }
            }
        }
#pragma unroll
        for (int x = 0; x < kFwdTiles; ++x) {
            float y = part[x];
            y += __shfl_xor(y, 16, 64);
            y += __shfl_xor(y, 32, 64);
            if (lane < 16 && p0 + 16 * x < n) logits[p0 + 16 * x] = y + b3;
        }
    }
}

// One Adam step of parameter x (Kingma & Ba, bias-corrected moments) when
// A.update, then its bf16 copies from the fp32 master.
struct AdamArgs {
    float *theta, *m, *v;
    uint16_t *W1b, *W2b, *W2Tb, *w3b;
    float lr, b1, b2, eps, c1, c2;
    int update;
};

__device__ __forceinline__ void adam_one(const AdamArgs &A, int x, float g) {
    float w = A.theta[x];
    if (A.update) {
        const float mm = A.b1 * A.m[x] + (1.f - A.b1) * g;
        const float vv = A.b2 * A.v[x] + (1.f - A.b2) * g * g;
        A.m[x] = mm;
        A.v[x] = vv;
        w -= A.lr * (mm / A.c1) / (sqrtf(vv / A.c2) + A.eps);
        A.theta[x] = w;
    }
    const uint16_t h = to_bf16(w);
    if (x < kMlpOffB1) {
        A.W1b[x] = h;
    } else if (x >= kMlpOffW2 && x < kMlpOffB2) {
        const int r = (x - kMlpOffW2) / kH, c = (x - kMlpOffW2) % kH;
        A.W2b[r * kH + c] = h;
        A.W2Tb[c * kH + r] = h;
    } else if (x >= kMlpOffW3 && x < kMlpOffB3) {
        A.w3b[x - kMlpOffW3] = h;
    }
}

// Forward + backward of 16 pairs per wave for one minibatch.  Pairs of the
// batch are examples order[off + p]; p >= count are padding (zero input and
// gradient).  Writes ZT, H1, DH2 and DH1 (bf16, [B / 16][feature][16]) and,
// per tile, the sums of the loss and of the bias /
// w3 gradients over its pairs into part[tile][kMlpPartN] (slot 0 the loss,
// then b1, b2, w3, b3), in a fixed order: no atomics, so a minibatch's
// gradient is the same on every run.
struct Train {
    const float *X;
    const uint8_t *labels;
    const int32_t *order;
    int64_t off, count;  // batch = examples order[off .. off + count)
    int B;               // padded batch size (multiple of 16)
    float pos_weight, inv_n;
    uint16_t *ZT, *H1, *DH2, *DH1;
    float *part;
};

// Part slots: the gradient of parameter x >= kMlpOffB2 (b2, w3, b3 are
// contiguous there) sits in slot kPartB2 + x - kMlpOffB2.
constexpr int kPartB1 = 1, kPartB2 = 1 + kH, kPartW3 = 1 + 2 * kH, kPartB3 = 1 + 3 * kH;

// Sums v[0..N) of every lane over the 16 lanes of its lane group (same
// lane >> 4), reduce-scatter style: after the four exchange steps lane col
// holds the group's totals of v[N/16 * col .. + N/16) in v[0 .. N/16).  Each
// step hands half of the remaining values to the partner lane, so the wave
// does N - N/16 exchanges instead of 4N.
template <int N>
__device__ __forceinline__ void group_reduce_scatter(float (&v)[N], int col) {
#pragma unroll
    for (int m = 8, half = N / 2; m >= 1; m >>= 1, half >>= 1) {
        const bool up = (col & m) != 0;
#pragma unroll
        for (int q = 0; q < half; ++q) {
            const float lo = v[q], hi = v[half + q];  // values, so the selects below are not on addresses
            const float keep = up ? hi : lo, give = up ? lo : hi;
            v[q] = keep + __shfl_xor(give, m, 64);
        }
    }
}

// One block per tile of 16 pairs, its four waves splitting the feature tiles of
// layer 2 and of both backward products (two of eight each); layer 1, the loss
// and the output gradient are cheap and every wave has them for itself.  The
// batch of a step is small (8,192 pairs are 512 tiles for 1,024 SIMDs), so a
// step takes as long as one wave's instructions: 38.6 us with a wave per tile,
// 21.7 so.  The waves exchange layer 2's pre-activations through LDS, and every
// sum runs in the order of one wave, so the gradients are the same bits.
__global__ __launch_bounds__(64 * kMlpTrainWaves) void train_tile_kernel(Net N, Train T) {
    constexpr int W = kMlpTrainWaves, kOwn = 8 / W;  // feature tiles per wave
    __shared__ float4 pre2[8][64];                    // [t2][lane]: features 16 t2 + 4 kg .. + 3 of pair col
    const int lane = threadIdx.x & 63, col = lane & 15, kg = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int tile = blockIdx.x, own = kOwn * w;
    const int pb = tile * 16 + col;  // pair index within the batch
    const bool valid = pb < T.count;
    const int64_t ex = valid ? (int64_t)T.order[T.off + pb] : 0;
    // every weight the wave needs is under way before the first is used
    bf16x4 w1[8], w3[8], w2[kOwn][8], w2t[kOwn][8];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        w1[t] = load4(N.W1b + (16 * t + col) * kIn + 4 * kg);
        w3[t] = load4(N.w3b + 16 * t + 4 * kg);
    }
#pragma unroll
    for (int x = 0; x < kOwn; ++x)
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            w2[x][t] = load4(N.W2b + (16 * (own + x) + col) * kH + 16 * t + 4 * kg);
            w2t[x][t] = load4(N.W2Tb + (16 * (own + x) + col) * kH + 16 * t + 4 * kg);
        }
    const uint8_t label = T.labels[ex];
    __builtin_amdgcn_sched_barrier(0);
    const bf16x4 z = input_operand(T.X, ex, valid, kg, N);
    const size_t at = (size_t)tile * kH * 16 + col;
    if (w == 0) {
        uint16_t *const zt = T.ZT + (size_t)tile * kIn * 16 + col;
#pragma unroll
        for (int i = 0; i < 4; ++i) zt[(4 * kg + i) * 16] = (uint16_t)z[i];
    }
    // forward (K tiles in order)
    bf16x4 h1[8];
    float own1[kOwn][4];  // layer-1 pre-activations of the wave's own tiles
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        const f32x4 a = mfma(w1[t], z, f32x4{0.f, 0.f, 0.f, 0.f});
        const float4 b = *(const float4 *)(N.b1 + 16 * t + 4 * kg);
        const float p[4] = {a[0] + b.x, a[1] + b.y, a[2] + b.z, a[3] + b.w};
#pragma unroll
        for (int x = 0; x < kOwn; ++x)
            if (own + x == t) {
#pragma unroll
                for (int i = 0; i < 4; ++i) own1[x][i] = p[i];
            }
        const uint2 v = make_uint2(to_bf16x2(p[0] > 0.f ? p[0] : 0.f, p[1] > 0.f ? p[1] : 0.f),
                                   to_bf16x2(p[2] > 0.f ? p[2] : 0.f, p[3] > 0.f ? p[3] : 0.f));
        h1[t] = __builtin_bit_cast(bf16x4, v);
        if (t >= own && t < own + kOwn) {
#pragma unroll
            for (int i = 0; i < 4; ++i) T.H1[at + (16 * t + 4 * kg + i) * 16] = (uint16_t)h1[t][i];
        }
    }
    float own2[kOwn][4];
#pragma unroll
    for (int x = 0; x < kOwn; ++x) {
        const int t2 = own + x;
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < 8; ++t) acc = mfma(w2[x][t], h1[t], acc);
        const float4 b = *(const float4 *)(N.b2 + 16 * t2 + 4 * kg);
        own2[x][0] = acc[0] + b.x;
        own2[x][1] = acc[1] + b.y;
        own2[x][2] = acc[2] + b.z;
        own2[x][3] = acc[3] + b.w;
        pre2[t2][lane] = make_float4(own2[x][0], own2[x][1], own2[x][2], own2[x][3]);
    }
    __syncthreads();
    float part = 0.f;
#pragma unroll
    for (int t2 = 0; t2 < 8; ++t2) {
        const float4 q = pre2[t2][lane];
        const float p[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float h = from_bf16(to_bf16(p[i] > 0.f ? p[i] : 0.f));
            part += from_bf16((uint16_t)w3[t2][i]) * h;
        }
    }
    part += __shfl_xor(part, 16, 64);
    part += __shfl_xor(part, 32, 64);
    const float y = part + N.b3[0];
    const float t = valid ? (float)label : 0.f;
    const float s = 1.f / (1.f + expf(-y));
    const float dy = valid ? (T.pos_weight * t * (s - 1.f) + (1.f - t) * s) * T.inv_n : 0.f;
    // layer 3 / layer 2 backward, in the accumulator layout
    bf16x4 dh2op[8];
#pragma unroll
    for (int t2 = 0; t2 < 8; ++t2) {
        const float4 q = pre2[t2][lane];
        const float p[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (int i = 0; i < 4; ++i)
            dh2op[t2][i] = (short)to_bf16(p[i] > 0.f ? dy * from_bf16((uint16_t)w3[t2][i]) : 0.f);
    }
    // the wave's own gradients of w3, b2 and b1, [4 x + i]: feature 16 (own + x) + 4 kg + i
    float g[32] = {};
#pragma unroll
    for (int x = 0; x < kOwn; ++x) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int f = 16 * (own + x) + 4 * kg + i;
            const float p = own2[x][i];
            g[4 * x + i] = dy * from_bf16(to_bf16(p > 0.f ? p : 0.f));
            const float d = p > 0.f ? dy * from_bf16(N.w3b[f]) : 0.f;
            g[8 + 4 * x + i] = d;
            T.DH2[at + f * 16] = to_bf16(d);
        }
    }
    // dH1 = W2^T dH2 (transposed weights as the A operand)
#pragma unroll
    for (int x = 0; x < kOwn; ++x) {
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t2 = 0; t2 < 8; ++t2)
            acc = mfma(w2t[x][t2], dh2op[t2], acc);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int f = 16 * (own + x) + 4 * kg + i;
            const float d = own1[x][i] > 0.f ? acc[i] : 0.f;
            g[16 + 4 * x + i] = d;
            T.DH1[at + f * 16] = to_bf16(d);
        }
    }
    group_reduce_scatter(g, col);
    // lane col now holds entries 2 col and 2 col + 1
    float *const out = T.part + (size_t)tile * kMlpPartN;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int e = 2 * col + q, f = 16 * (own + (e >> 2 & 1)) + 4 * kg + (e & 3);
        if (e < 24) out[(e < 8 ? kPartW3 : e < 16 ? kPartB2 : kPartB1) + f] = 0.f + g[q];
    }
    if (w != 0) return;
    // loss: softplus(-y) for positives, softplus(y) for negatives, computed stably
    const float sp = log1pf(expf(-fabsf(y)));
    float lo = valid ? (T.pos_weight * t * (fmaxf(-y, 0.f) + sp) + (1.f - t) * (fmaxf(y, 0.f) + sp)) * T.inv_n : 0.f;
    float sdy = dy;
#pragma unroll
    for (int m = 1; m < 16; m <<= 1) {
        lo += __shfl_xor(lo, m, 64);
        sdy += __shfl_xor(sdy, m, 64);
    }
    if (lane == 0) {
        out[0] = 0.f + lo;
        out[kPartB3] = 0.f + sdy;
    }
}

// Weight gradients over one minibatch, split over the pairs: dW2 = DH2 H1^T
// (64 tiles of 16x16) and dW1 = DH1 Z^T (8 tiles), each over chunks of
// kMlpSplitK pairs.  One wave per (tile, chunk); chunk c's partial products
// go to wp2 + c * 128 * 128 and wp1 + c * 128 * 16 ([row][col] as the
// parameters), to be summed in chunk order.
__global__ __launch_bounds__(256) void wgrad_kernel(const uint16_t *__restrict__ DH2, const uint16_t *__restrict__ H1,
                                                    const uint16_t *__restrict__ DH1,
                                                    const uint16_t *__restrict__ ZT, int B, int chunks,
                                                    float *__restrict__ wp2, float *__restrict__ wp1) {
    constexpr int kTiles2 = (kH / 16) * (kH / 16), kTiles = kTiles2 + kH / 16;
    const int lane = threadIdx.x & 63, col = lane & 15, kg = lane >> 4;
    const int wave = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (wave >= kTiles * chunks) return;
    const int tile = wave % kTiles, c = wave / kTiles;
    const uint16_t *A, *Bm;
    float *C;
    int Nn, mt, nt;
    if (tile < kTiles2) {
        A = DH2, Bm = H1, Nn = kH, mt = tile / (kH / 16), nt = tile % (kH / 16), C = wp2 + (size_t)c * kH * kH;
    } else {
        A = DH1, Bm = ZT, Nn = kIn, mt = tile - kTiles2, nt = 0, C = wp1 + (size_t)c * kH * kIn;
    }
    // pair tiles [t0, t1) of this chunk; a tile of A holds kH features, of Bm Nn
    const int t0 = c * (kMlpSplitK / 16), t1 = min(B / 16, t0 + kMlpSplitK / 16);
    const uint16_t *ap = A + (size_t)t0 * kH * 16 + (16 * mt + col) * 16 + 4 * kg;
    const uint16_t *bp = Bm + (size_t)t0 * Nn * 16 + (16 * nt + col) * 16 + 4 * kg;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
    for (int t = t0; t < t1; ++t, ap += kH * 16, bp += Nn * 16) acc = mfma(load4(ap), load4(bp), acc);
#pragma unroll
    for (int i = 0; i < 4; ++i) C[(size_t)(16 * mt + 4 * kg + i) * Nn + 16 * nt + col] = acc[i];
}

// The minibatch gradient from the partials, summed in a fixed order, then
// (A.update) the Adam step of every parameter.  Threads [0, nW) take one
// weight of W1 or W2 each (sum over the chunks); then one wave per part slot
// sums the tiles' values (by four, lane-strided, then a fixed shuffle tree) into the
// bias / w3 gradient, and slot 0 adds the batch loss to *loss.  The gradient
// is written to grad either way.
__global__ __launch_bounds__(256) void grad_reduce_kernel(const float *__restrict__ part, int tiles,
                                                          const float *__restrict__ wp2,
                                                          const float *__restrict__ wp1, int chunks,
                                                          float *__restrict__ grad, float *__restrict__ loss,
                                                          AdamArgs A) {
    constexpr int nW1 = kH * kIn, nW2 = kH * kH, nW = nW1 + nW2;
    const int x = blockIdx.x * blockDim.x + threadIdx.x;
    if (x < nW) {
        const bool w1 = x < nW1;
        const float *src = w1 ? wp1 + x : wp2 + (x - nW1);
        const size_t stride = w1 ? nW1 : nW2;
        float a = 0.f;
#pragma unroll 8
        for (int c = 0; c < chunks; ++c) a += src[(size_t)c * stride];
        const int px = w1 ? kMlpOffW1 + x : kMlpOffW2 + x - nW1;
        grad[px] = a;
        if (A.update) adam_one(A, px, a);
        return;
    }
    const int wbase = (nW + 255) / 256 * 4;  // first wave of the slot sums
    const int slot = blockIdx.x * 4 + (threadIdx.x >> 6) - wbase, lane = threadIdx.x & 63;
    if (slot < 0 || slot >= kMlpPartN) return;
    float a = 0.f;
    for (int b = 4 * lane; b < tiles; b += 256) {
        const float *p = part + (size_t)b * kMlpPartN + slot;
        float four = p[0];
#pragma unroll
        for (int q = 1; q < 4; ++q) four += b + q < tiles ? p[q * kMlpPartN] : 0.f;
        a += four;
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) a += __shfl_xor(a, m, 64);
    if (lane != 0) return;
    if (slot == 0) {
        *loss += a;
        return;
    }
    const int px = slot < kPartB2 ? kMlpOffB1 + slot - kPartB1 : kMlpOffB2 + slot - kPartB2;
    grad[px] = a;
    if (A.update) adam_one(A, px, a);
}

// bf16 copies of the fp32 masters (no update).
__global__ void refresh_kernel(AdamArgs A) {
    for (int x = blockIdx.x * blockDim.x + threadIdx.x; x < kMlpParams; x += gridDim.x * blockDim.x)
        adam_one(A, x, 0.f);
}

// mean / std (population) of each feature column, fp64 accumulation
__global__ void moments_kernel(const float *__restrict__ X, int64_t n, double *__restrict__ acc) {
    __shared__ double s[2 * kIn];
    if (threadIdx.x < 2 * kIn) s[threadIdx.x] = 0.0;
    __syncthreads();
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < n * kIn; q += (int64_t)gridDim.x * blockDim.x) {
        const int f = (int)(q % kIn);
        const double x = X[q];
        atomicAdd(&s[f], x);
        atomicAdd(&s[kIn + f], x * x);
    }
    __syncthreads();
    if (threadIdx.x < 2 * kIn) atomicAdd(&acc[threadIdx.x], s[threadIdx.x]);
}

__global__ void moments_finish_kernel(const double *__restrict__ acc, int64_t n, float *__restrict__ mean,
                                      float *__restrict__ stdv) {
    const int f = threadIdx.x;
    if (f < kIn) {
        const double mu = acc[f] / (double)n;
        const double var = acc[kIn + f] / (double)n - mu * mu;
        mean[f] = (float)mu;
        stdv[f] = (float)(var > 1e-12 ? sqrt(var) : 1.0);
    }
}

__global__ void keep_kernel(const float *__restrict__ logits, int64_t n, float tau, uint8_t *__restrict__ keep) {
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < n; q += (int64_t)gridDim.x * blockDim.x)
        keep[q] = logits[q] >= tau ? 1 : 0;
}

__global__ void compact_kernel(const uint8_t *__restrict__ keep, const uint32_t *__restrict__ pos, int64_t n,
                               const uint32_t *__restrict__ in0, const uint32_t *__restrict__ in1,
                               const uint32_t *__restrict__ in2, const uint32_t *__restrict__ in3,
                               const uint32_t *__restrict__ in4, uint32_t *__restrict__ out0,
                               uint32_t *__restrict__ out1, uint32_t *__restrict__ out2, uint32_t *__restrict__ out3,
                               uint32_t *__restrict__ out4) {
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < n; q += (int64_t)gridDim.x * blockDim.x) {
        if (!keep[q]) continue;
        const uint32_t p = pos[q];
        out0[p] = in0[q];
        out1[p] = in1[q];
        out2[p] = in2[q];
        out3[p] = in3[q];
        out4[p] = in4[q];
    }
}

// flag[0] = min position of an index outside [0, limit) (stays ~0 if none)
__global__ void check_order_kernel(const int32_t *__restrict__ order, int64_t n, int64_t limit,
                                   unsigned long long *__restrict__ flag) {
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < n; q += (int64_t)gridDim.x * blockDim.x) {
        const int32_t v = order[q];
        if (v < 0 || (int64_t)v >= limit) atomicMin(flag, (unsigned long long)q);
    }
}

inline unsigned grid_for(int64_t n) {
    int64_t b = (n + 255) / 256;
    if (b > 16384) b = 16384;
    return (unsigned)(b < 1 ? 1 : b);
}

Net net_of(const MlpState &S) {
    Net N;
    N.W1b = S.W1b;
    N.W2b = S.W2b;
    N.W2Tb = S.W2Tb;
    N.w3b = S.w3b;
    N.b1 = S.theta + kMlpOffB1;
    N.b2 = S.theta + kMlpOffB2;
    N.b3 = S.theta + kMlpOffB3;
    N.mean = S.mean;
    N.stdv = S.stdv;
    return N;
}

AdamArgs adam_args(const MlpState &S, float lr, int step) {
    AdamArgs A;
    A.theta = S.theta;
    A.m = S.m;
    A.v = S.v;
    A.W1b = S.W1b;
    A.W2b = S.W2b;
    A.W2Tb = S.W2Tb;
    A.w3b = S.w3b;
    A.b1 = 0.9f;
    A.b2 = 0.999f;
    A.eps = 1e-8f;
    A.lr = lr;
    A.update = step > 0;
    A.c1 = step > 0 ? 1.f - powf(A.b1, (float)step) : 1.f;
    A.c2 = step > 0 ? 1.f - powf(A.b2, (float)step) : 1.f;
    return A;
}

}  // namespace

hipError_t mlp_refresh(const MlpState &S, hipStream_t s) {
    refresh_kernel<<<grid_for(kMlpParams), 256, 0, s>>>(adam_args(S, 0.f, 0));
    return hipGetLastError();
}

hipError_t mlp_features(const uint8_t *codes, const int64_t *offsets, int64_t n, const uint32_t *lo,
                        const uint32_t *hi, const uint32_t *count, const uint32_t *s1, const uint32_t *s2,
                        int64_t npairs, float *comp, float *F, hipStream_t s) {
    if (n > 0) {
        comp_kernel<<<(unsigned)std::min<int64_t>((n + 3) / 4, 16384), 256, 0, s>>>(codes, offsets, n, comp);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (npairs <= 0) return hipSuccess;
    features_kernel<<<grid_for(npairs), 256, 0, s>>>(lo, hi, count, s1, s2, npairs, offsets, comp, F,
                                                      ((uintptr_t)F & 15u) == 0 ? 1 : 0);
    return hipGetLastError();
}

hipError_t mlp_forward(const MlpState &S, const float *X, int64_t n, float *logits, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const int64_t groups = (n + 16 * kFwdTiles - 1) / (16 * kFwdTiles);
    int64_t blocks = (groups + 3) / 4;
    if (blocks > 1024) blocks = 1024;  // what fits on the device: the weights are fetched once a block
    forward_kernel<<<(unsigned)blocks, 256, 0, s>>>(X, n, net_of(S), logits, ((uintptr_t)X & 15u) == 0 ? 1 : 0);
    return hipGetLastError();
}

hipError_t mlp_moments(const float *X, int64_t n, double *acc, float *mean, float *stdv, hipStream_t s) {
    hipError_t e = fill<uint64_t>((uint64_t *)acc, 2 * kIn, 0ull, s);
    if (e != hipSuccess) return e;
    if (n > 0) {
        moments_kernel<<<grid_for(n * kIn / 8 + 1), 256, 0, s>>>(X, n, acc);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    moments_finish_kernel<<<1, 64, 0, s>>>(acc, n > 0 ? n : 1, mean, stdv);
    return hipGetLastError();
}

hipError_t mlp_batch_grad(const MlpState &S, const float *X, const uint8_t *labels, const int32_t *order, int64_t off,
                          int64_t count, int B, float pos_weight, float *loss, float lr, int step, hipStream_t s) {
    if (B <= 0 || B % 16 || B > S.batch_cap || count > B) return hipErrorInvalidValue;
    Train T;
    T.X = X;
    T.labels = labels;
    T.order = order;
    T.off = off;
    T.count = count;
    T.B = B;
    T.pos_weight = pos_weight;
    T.inv_n = 1.f / (float)(count > 0 ? count : 1);
    T.ZT = S.ZT;
    T.H1 = S.H1;
    T.DH2 = S.DH2;
    T.DH1 = S.DH1;
    T.part = S.part;
    const int tiles = B / 16;  // rows of part
    train_tile_kernel<<<tiles, 64 * kMlpTrainWaves, 0, s>>>(net_of(S), T);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int chunks = (B + kMlpSplitK - 1) / kMlpSplitK;  // <= batch_cap / kMlpSplitK
    float *wp2 = S.wpart, *wp1 = S.wpart + (size_t)chunks * kH * kH;
    const int waves = (kH / 16 * kH / 16 + kH / 16) * chunks;
    wgrad_kernel<<<(waves + 3) / 4, 256, 0, s>>>(S.DH2, S.H1, S.DH1, S.ZT, B, chunks, wp2, wp1);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    const int nW = kH * kIn + kH * kH;
    const int rblocks = (nW + 255) / 256 + (kMlpPartN + 3) / 4;
    grad_reduce_kernel<<<rblocks, 256, 0, s>>>(S.part, tiles, wp2, wp1, chunks, S.grad, loss,
                                                adam_args(S, lr, step));
    return hipGetLastError();
}


hipError_t mlp_keep(const float *logits, int64_t n, float tau, uint8_t *keep, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    keep_kernel<<<grid_for(n), 256, 0, s>>>(logits, n, tau, keep);
    return hipGetLastError();
}

hipError_t mlp_check_order(const int32_t *order, int64_t n, int64_t limit, unsigned long long *flag, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    check_order_kernel<<<grid_for(n), 256, 0, s>>>(order, n, limit, flag);
    return hipGetLastError();
}

hipError_t compact5(const uint8_t *keep, const uint32_t *pos, int64_t n, const uint32_t *const in[5],
                    uint32_t *const out[5], hipStream_t s) {
    if (n <= 0) return hipSuccess;
    compact_kernel<<<grid_for(n), 256, 0, s>>>(keep, pos, n, in[0], in[1], in[2], in[3], in[4], out[0], out[1],
                                                out[2], out[3], out[4]);
    return hipGetLastError();
}

}  // namespace pastis
