// Device helpers, arguments and bin shapes shared by the Smith-Waterman kernels (32-bit
// lanes, start bound and statistics in sw.hip; 16-bit lanes in sw16.hip).
#pragma once

#include <type_traits>
#include <utility>

#include "internal.hpp"

namespace pastis {

// What a group kernel runs on: the oriented pairs, the pass's item list with
// its bin bounds, and the buffers of the pass.
struct SwArgs {
    const uint8_t *codes;
    const PairDesc *pairs;
    const int *idx;      // pair indices by bin
    const int *starts;   // bin b: items [starts[b], starts[b + 1])
    const int *bounds;   // 16-bit kernels: rows class c of bin b: [bounds[2 b + c], bounds[2 b + c + 1])
    const int *win;      // 16-bit kernels: windows of class c: win[bounds[c] .. + nwin[c]), their first items
    const int *nwin;
    const int8_t *blosum;
    int go_ge, ge;
    SwPass1Out *p1;
    pastis_pair_record *rec;
    int *scratch;  // per-wave boundary rows of the multi-strip bins
    int64_t scratch_per_wave;
    int *queue;                // work-queue counters of the launch
    unsigned long long *span;  // per bin: two words (span_add)
    unsigned long long *flag;  // intra-pair mode: a wait ran out
    int cov_pct, id_pct;
    // traced statistics pass: direction words of each wave of the grid for
    // one-strip pairs, and of the waves of the multi-strip blocks
    uint32_t *dirs, *dirs_multi;
    int64_t dirs_per_wave, dirs_per_multi;
};

// Pairs whose statistics come from the traceback: 16-bit pass-1 bins whose
// longer sequence fits the direction buffers.
struct TraceRule {
    uint32_t bins;              // pass-1 bins in 16-bit lanes (0: no traceback)
    int max_cols, max_cols_multi;  // longest b of one-strip and of multi-strip pairs
};

namespace {

constexpr int kWave = 64;
constexpr int kNeg = -(1 << 28);
// waves per block of the 32-bit kernels: one int8 profile of 25 x 64 x R
// bytes per wave, blocks of at most ~51 KB of LDS (three per CU)
__host__ __device__ constexpr int wpb32(int R) { return R <= 8 ? 4 : 2; }
constexpr int kProfCodes = kAlpha + 1;  // 24 residues + the pad code
constexpr int kMaxR = 16;               // rows per lane
constexpr int kSingleBins = kMaxR;      // bins 0..15: one strip of 64 * (bin + 1) rows
constexpr int kMultiBin = kSingleBins;  // bins 16..23: several strips of 64 * R rows, R = bin - 7
constexpr int kMultiMinR = kMaxR / 2 + 1;
// bins 24..31: as 16..23 for sequences a of at most kMax16Rows rows, whose
// scores (at most 11 per row with BLOSUM62) stay below 2^15
constexpr int kMulti16Bin = kMultiBin + kMaxR - kMultiMinR + 1;
constexpr int kNumBins = kMulti16Bin + kMaxR - kMultiMinR + 1;
constexpr int kMax16Rows = 32767 / 11;
constexpr int kBoundMaxScore = 30000;  // scores the backward start bound holds in 16 bits
constexpr int kSplitBins = 8;   // one-strip bins 0..7 (up to 8 rows per lane) have two rows classes
// longest b of a pair whose direction bits the traceback keeps, one strip and
// several (up to 1 KB per column and strip, only while its wave works on it);
// pairs of a longer b go to the statistics kernels
constexpr int kTraceCols = 2048, kTraceColsMulti = 4096;
constexpr int kTraceStrips = 3;  // strips of a pair of kMax16Rows rows
static_assert(kTraceStrips * kMaxR * kWave >= kMax16Rows, "strips of the tallest traced pair");
static_assert(kNumBins <= 32, "bin tables hold 32 entries");

__host__ __device__ constexpr int rows_of_bin(int bin) {
    return bin >= kMulti16Bin ? bin - kMulti16Bin + kMultiMinR : bin >= kMultiBin ? bin - kMultiBin + kMultiMinR
                                                                                   : bin + 1;
}
constexpr int kDppWaveShr1 = 0x138;
// work-queue counters of a call, and the window counts of pass 1 and traceback
constexpr int kSwQueues = 11 * kNumBins, kWindows1 = 7 * kNumBins, kWindowsTrace = 9 * kNumBins;

// lane l receives lane l-1's value; lane 0 receives `lane0`
__device__ __forceinline__ int shr1(int lane0, int v) {
    return __builtin_amdgcn_update_dpp(lane0, v, kDppWaveShr1, 0xF, 0xF, false);
}

// lane l receives lane l-1's value; lane 0 receives 0 (the move's bound
// control zero-fills, so no separate write of lane 0's value is needed)
__device__ __forceinline__ int shr1z(int v) { return __builtin_amdgcn_update_dpp(0, v, kDppWaveShr1, 0xF, 0xF, true); }

// R int8 scores per lane and residue code, in ceil(R / 4) words
template <int R>
using ProfWord = typename std::conditional<
    (R <= 4), uint32_t,
    typename std::conditional<(R <= 8), uint2, typename std::conditional<(R <= 12), uint3, uint4>::type>::type>::type;

template <int R>
__device__ __forceinline__ uint32_t word_of(const ProfWord<R> &w, int k) {
    if constexpr (R <= 4) {
        return w;
    } else if constexpr (R <= 8) {
        return k == 0 ? w.x : w.y;
    } else if constexpr (R <= 12) {
        return k == 0 ? w.x : k == 1 ? w.y : w.z;
    } else {
        return k == 0 ? w.x : k == 1 ? w.y : k == 2 ? w.z : w.w;
    }
}

template <int R>
__device__ __forceinline__ ProfWord<R> make_word(const uint32_t (&w)[4]) {
    if constexpr (R <= 4) {
        return w[0];
    } else if constexpr (R <= 8) {
        return make_uint2(w[0], w[1]);
    } else if constexpr (R <= 12) {
        return make_uint3(w[0], w[1], w[2]);
    } else {
        return make_uint4(w[0], w[1], w[2], w[3]);
    }
}

template <int R>
__device__ __forceinline__ int sigma_at(const ProfWord<R> &w, int r) {
    return (int)(int8_t)(word_of<R>(w, r >> 2) >> (8 * (r & 3)));
}

template <int R>
__device__ __forceinline__ void build_profile(ProfWord<R> (*prof)[kWave], const int8_t *sblosum, const uint8_t *a,
                                              int la, int base, int lane) {
    int ar[R];
#pragma unroll
    for (int r = 0; r < R; ++r) ar[r] = (base + r >= 0 && base + r < la) ? a[base + r] : kPadCode;
    for (int c = 0; c < kProfCodes; ++c) {
        uint32_t w[4] = {0, 0, 0, 0};
#pragma unroll
        for (int r = 0; r < R; ++r) w[r >> 2] |= (uint32_t)(uint8_t)sblosum[ar[r] * kProfCodes + c] << (8 * (r & 3));
        prof[c][lane] = make_word<R>(w);
    }
}

__device__ __forceinline__ unsigned long long wave_max_u64(unsigned long long v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        unsigned lo = (unsigned)v, hi = (unsigned)(v >> 32);
        unsigned olo = __shfl_xor(lo, off, kWave), ohi = __shfl_xor(hi, off, kWave);
        unsigned long long o = ((unsigned long long)ohi << 32) | olo;
        v = o > v ? o : v;
    }
    return v;
}

__device__ __forceinline__ void load_blosum(int8_t *sblosum, const int8_t *blosum) {
    for (int t = threadIdx.x; t < kProfCodes * kProfCodes; t += blockDim.x) sblosum[t] = blosum[t];
    __syncthreads();
}

// A load the compiler must issue per lane through the vector memory path (the
// data was written by another lane of the same wave earlier in the kernel).
template <typename T>
__device__ __forceinline__ T vload(const T *p) {
    return __builtin_nontemporal_load(p);
}

// A wave's next window of `count` consecutive items of its bin: lane 0 claims
// it from the bin's queue counter (zeroed before the launch), so that a
// resident grid stays busy until the bin is empty, waves that finish early
// taking more work.  The counter is claimed by a vector atomic.
__device__ __forceinline__ int64_t take(int *queue, const int *starts, int bin, int count) {
    int v = 0;
    if ((threadIdx.x & (kWave - 1)) == 0) v = atomicAdd(queue + bin, count);
    return starts[bin] + (int64_t)__builtin_amdgcn_readfirstlane(v);
}

// the same from a counter of its own over items [begin, ...)
__device__ __forceinline__ int64_t take_from(int *counter, int begin, int count) {
    int v = 0;
    if ((threadIdx.x & (kWave - 1)) == 0) v = atomicAdd(counter, count);
    return begin + (int64_t)__builtin_amdgcn_readfirstlane(v);
}

// max(x - y, 0) for x >= 0, y >= 0 (one clamped subtract)
__device__ __forceinline__ int subs(int x, int y) {
    return (int)__builtin_elementwise_sub_sat((unsigned)x, (unsigned)y);
}

// Rows up to 64 * kMaxR take one strip of 64 * R rows with the smallest R;
// longer ones take the fewest strips of at most 64 * kMaxR rows, with R as
// small as that strip count allows (padding under one row per lane and strip).
__device__ __forceinline__ int rows_bin(int rows) {
    if (rows <= 0) return 0;
    const int r = (rows + kWave - 1) / kWave;
    if (r <= kSingleBins) return r - 1;
    const int strips = (rows + kWave * kSingleBins - 1) / (kWave * kSingleBins);
    const int rm = (rows + kWave * strips - 1) / (kWave * strips);  // in [kMultiMinR, kMaxR]
    return (rows <= kMax16Rows ? kMulti16Bin : kMultiBin) + rm - kMultiMinR;
}

// bin_of between the passes: the bin of the statistics kernels, or
constexpr int8_t kFinal = -1;    // the record is final
constexpr int8_t kToTrace = -2;  // listed for the traceback
constexpr int8_t kToBound = -3;  // listed for the start bound

__device__ __forceinline__ bool can_trace(const TraceRule &T, const PairDesc &pd) {
    const int bin = rows_bin(pd.la);
    return ((T.bins >> bin) & 1u) && pd.lb <= (bin < kSingleBins ? T.max_cols : T.max_cols_multi);
}

// the final record of a pair that takes no statistics pass
__device__ __forceinline__ void sw_final_record(const PairDesc &pd, const SwPass1Out &r1, int64_t q,
                                                pastis_pair_record *__restrict__ out, int8_t *__restrict__ bin_of) {
    bin_of[q] = kFinal;
    pastis_pair_record rec;
    rec.score = r1.score;
    rec.beg_a = rec.beg_b = -1;
    rec.end_a = r1.end_a;
    rec.end_b = max(r1.end_b, -1);  // (a 16-bit pair's end column is a hint until a later pass finds it)
    rec.matches = rec.columns = 0;
    rec.seed_used = -1;
    rec.passed = 0;
    rec.swapped = pd.swapped;
    rec.cells = (int64_t)pd.la * pd.lb;
    out[q] = rec;
}

// SwPass1Out::end_b while the end column is unknown: -2 - (first possible column)
__device__ __forceinline__ int hint_code(int chunk, int pos) { return -2 - max(16 * chunk - pos, 0); }
__device__ __forceinline__ int first_col(int end_b) { return end_b >= 0 ? end_b : max(-2 - end_b, 0); }

// Hand-offs between the waves of a block: monotone counters in LDS, released
// and acquired at workgroup scope.  Every wait is bounded.
constexpr int kSpinLimit = 1 << 24;
__device__ __forceinline__ int lds_acquire(int *p) {
    return __hip_atomic_load(p, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void lds_release(int *p, int v) {
    __hip_atomic_store(p, v, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
}
// wait until *p >= need; false when the bound runs out
__device__ __forceinline__ bool lds_wait(int *p, int need) {
    for (int spin = 0; spin < kSpinLimit; ++spin) {
        if (__builtin_amdgcn_readfirstlane(lds_acquire(p)) >= need) return true;
        __builtin_amdgcn_s_sleep(1);
    }
    return false;
}

// First claim and last finish of a bin's pass-1 windows, in ticks of the
// device's wall clock: span[0] holds the complement of the earliest begin,
// span[1] the latest end (both raised with atomicMax from the counters' zero).
__device__ __forceinline__ unsigned long long span_now() { return __builtin_amdgcn_s_memrealtime(); }
__device__ __forceinline__ void span_add(unsigned long long *span, unsigned long long t0) {
    if ((threadIdx.x & (kWave - 1)) != 0) return;
    atomicMax(span, ~t0);
    atomicMax(span + 1, span_now());
}

}  // namespace
}  // namespace pastis
