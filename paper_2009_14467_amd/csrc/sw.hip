// Smith-Waterman alignment of candidate pairs (Section IV-E): one 64-lane
// wavefront per pair, 32-bit DP words, pairs binned by the length of the
// shorter sequence.
//
// Layout.  The rows of the shorter sequence a are split into strips of 64*R
// rows; lane l owns rows [l*R, l*R + R) of a strip and sweeps the columns of b
// one column behind lane l-1 (lane l is at column t - l in step t).  All DP
// state stays in registers; the bottom row of a lane's block moves to the next
// lane once per step with a DPP wavefront shift, and the column residue moves
// with it (lane 0 takes it from a register chunk of b via readlane).  Pairs
// whose shorter side needs more than one strip pass the strip's bottom row
// through a per-wave global buffer.  R is chosen per pair (one-strip bins
// R = 1..16; multi-strip bins R = 9..16 with the fewest strips of at most
// 1024 rows), so few lanes hold padding rows.
//
// Scores.  A per-lane profile in LDS holds, for every column residue code, the
// R int8 scores of the lane's rows; one LDS load per step serves R cells and
// the byte selects fold into the adds (SDWA).
//
// Pass 1 computes the score and the canonical end: the smallest row, then the
// smallest column, holding the maximum.  Each row keeps max((h << 16) |
// (0xFFFF - column)), which orders by score and then by the earlier column.
//
// Pass 2 recomputes the rectangle [0, end_a] x [0, end_b] carrying, for every
// cell and state (H, E, F), the start cell, identical pairs and diagonal
// columns of the canonical path ending there.  Each cell takes the predecessor
// a traceback would take (diagonal before horizontal before vertical gap,
// extension before opening; a zero diagonal predecessor starts a new path), so
// by induction the end cell holds the traceback's statistics.  The strip rows
// are padded at the top so the end cell is always row R-1 of lane 63.

#include <algorithm>
#include <atomic>

#include "sw_common.hpp"
#include "prim.hpp"
#include "sw16.hpp"
#include "sw_long.hpp"

namespace pastis {

hipError_t launch_bins(const int8_t *bin_of, int64_t n, int nbins, int *counts, int *starts, int *cursor, int *idx,
                       hipStream_t s);

namespace {

// ---------------------------------------------------------------- pass 1, 32-bit lanes

// Pass 1, 32-bit lanes.  The gap states are kept floored at zero, E' =
// max(E, 0) and F' = max(F, 0) (max(E' - e, 0) = max(E - e, 0) for e >= 0,
// one clamped subtract); max(d, E', F') then already holds the local
// alignment's zero.  The strip boundary carries F'.
// One bin's work; the group kernels below run the bodies of several bins.
template <int R, bool MULTI>
__device__ __forceinline__ bool pass1_body(const SwArgs &A, int bin, char *lds, size_t wave_bytes,
                                           const int8_t *sblosum) {
    constexpr int WPB = wpb32(R);
    const uint8_t *__restrict__ codes = A.codes;
    const PairDesc *__restrict__ pairs = A.pairs;
    const int *__restrict__ idx = A.idx, *__restrict__ starts = A.starts;
    const int go_ge = A.go_ge, ge = A.ge;
    SwPass1Out *__restrict__ out = A.p1;
    int *queue = A.queue;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    // waves of a block may be in bins of different profile sizes: each has a
    // fixed share of the block's LDS
    ProfWord<R>(*prof)[kWave] = (ProfWord<R>(*)[kWave])(lds + (size_t)wave * wave_bytes);
    const int64_t gwave = (int64_t)blockIdx.x * WPB + wave;
    int *bnd_h = A.scratch + gwave * A.scratch_per_wave;  // bottom row H / F of the strip above
    int *bnd_f = bnd_h + A.scratch_per_wave / 2;
    const int item_end = starts[bin + 1];
    constexpr int RS = kWave * R;

    bool any = false;  // this wave had work in the bin

    for (int64_t w = take(queue, starts, bin, 1); w < item_end; w = take(queue, starts, bin, 1)) {
        any = true;
        const int q = idx[w];
        const PairDesc pd = pairs[q];
        const uint8_t *a = codes + pd.a_off;
        const uint8_t *b = codes + pd.b_off;
        const int la = pd.la, lb = pd.lb;
        unsigned long long best = 0;  // (score << 32) | ~(row << 16 | col)
        const int nstrips = (la > 0 && lb > 0) ? (MULTI ? (la + RS - 1) / RS : 1) : 0;
        for (int s = 0; s < nstrips; ++s) {
            const int base = s * RS + lane * R;
            build_profile<R>(prof, sblosum, a, la, base, lane);
            const bool from_above = s > 0;
            const bool to_below = s + 1 < nstrips;
            int H[R], G[R], E[R];
            unsigned key[R];  // single strip: (h << 16) | (0xFFFF - col)
            int rmax[R], rcol[R];  // multi strip: scores may exceed 16 bits
#pragma unroll
            for (int r = 0; r < R; ++r) {
                H[r] = 0;
                G[r] = -go_ge;
                E[r] = 0;
                key[r] = 0;
                rmax[r] = 0;
                rcol[r] = 0;
            }
            int hlast = 0, flast = 0, hprev = 0, cres = kPadCode;
            // column residues and the strip boundary row arrive in coalesced
            // chunks of 64 columns, fetched one chunk ahead; lane 0 reads its
            // value for step t with readlane
            int chunk = kPadCode, ch_h = 0, ch_f = 0;
            int nx = (lane < lb) ? (int)b[lane] : kPadCode;
            int nx_h = 0, nx_f = 0;
            if (MULTI && from_above && lane < lb) {
                nx_h = vload(bnd_h + lane);
                nx_f = vload(bnd_f + lane);
            }
            // one DP step; in the tail (t >= lb) lanes past the last column
            // must not touch their running maxima
            auto step = [&](const int t, auto tail_tag) {
                constexpr bool kTail = decltype(tail_tag)::value;
                if ((t & (kWave - 1)) == 0) {
                    chunk = nx;
                    const int c = t + kWave + lane;
                    nx = (c < lb) ? (int)b[c] : kPadCode;
                    if (MULTI && from_above) {
                        ch_h = nx_h;
                        ch_f = nx_f;
                        if (c < lb) {
                            nx_h = vload(bnd_h + c);
                            nx_f = vload(bnd_f + c);
                        }
                    }
                }
                const int bt = __builtin_amdgcn_readlane(chunk, t & (kWave - 1));
                int in_h = 0, in_f = 0;
                if (MULTI && !kTail && from_above) {
                    in_h = __builtin_amdgcn_readlane(ch_h, t & (kWave - 1));
                    in_f = __builtin_amdgcn_readlane(ch_f, t & (kWave - 1));
                }
                const int rh = shr1(in_h, hlast);
                const int rf = shr1(in_f, flast);
                cres = shr1(bt, cres);
                const int j = t - lane;
                const bool valid = j < lb;
                const ProfWord<R> pw = prof[cres][lane];
                const unsigned jinv = (unsigned)(0xFFFF - j) & 0xFFFFu;
                int hd = hprev, gu = rh - go_ge, fu = rf;
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const int e = max(subs(E[r], ge), G[r]);
                    const int f = max(subs(fu, ge), gu);
                    const int d = hd + sigma_at<R>(pw, r);
                    const int h = max(d, max(e, f));
                    hd = H[r];
                    H[r] = h;
                    E[r] = e;
                    const int g = h - go_ge;
                    G[r] = g;
                    gu = g;
                    fu = f;
                    if constexpr (MULTI) {
                        if ((!kTail || valid) && h > rmax[r]) {
                            rmax[r] = h;
                            rcol[r] = j;
                        }
                    } else {
                        const unsigned k = ((unsigned)h << 16) | jinv;
                        const unsigned m = k > key[r] ? k : key[r];
                        key[r] = (!kTail || valid) ? m : key[r];
                    }
                }
                hlast = H[R - 1];
                flast = fu;
                hprev = rh;
                if (MULTI && to_below && lane == kWave - 1 && j >= 0 && j < lb) {
                    bnd_h[j] = hlast;
                    bnd_f[j] = flast;
                }
            };
            for (int t = 0; t < lb; ++t) step(t, std::false_type{});
            for (int t = lb; t < lb + kWave - 1; ++t) step(t, std::true_type{});
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int row = base + r;
                int sc, col;
                if constexpr (MULTI) {
                    sc = rmax[r];
                    col = rcol[r];
                } else {
                    sc = (int)(key[r] >> 16);
                    col = 0xFFFF - (int)(key[r] & 0xFFFFu);
                }
                if (row < la && sc > 0) {
                    const unsigned pos = ((unsigned)row << 16) | (unsigned)col;
                    const unsigned long long k = ((unsigned long long)(unsigned)sc << 32) | (unsigned)(~pos);
                    best = k > best ? k : best;
                }
            }
            if (MULTI) __threadfence_block();  // lane 0 of the next strip reads lane 63's row
        }
        best = wave_max_u64(best);
        if (lane == 0) {
            SwPass1Out o;
            o.score = (int32_t)(best >> 32);
            const unsigned pos = ~(unsigned)best;
            o.end_a = o.score > 0 ? (int32_t)(pos >> 16) : -1;
            o.end_b = o.score > 0 ? (int32_t)(pos & 0xFFFF) : -1;
            o.pad = 0;
            out[q] = o;
        }
    }
    return any;
}

// ---------------------------------------------------------------- pass 1, one workgroup per long pair

// Intra-pair mode for long sequences a: the W waves of a block work on one
// pair.  Wave w takes strips w, w + W, ... (strips of 64 R rows in 32-bit
// lanes, as in the multi-strip kernel above), so W strips run at once, each
// a little behind the one above.  The bottom row of strip s (H and F' of
// every column) reaches strip s + 1 through a full-length row buffer of slot
// s mod W in global memory.  Two monotone LDS counters per slot order the
// hand-off, in columns over all strips that used the slot for this pair:
// prod (written) and cons (loaded by the reader).  The reader of strip s + 1
// waits for prod (strip s); the writer of strip s + W waits until strip
// s + 1 has loaded the columns it overwrites.  Every wait is for an earlier
// strip, so the earliest unfinished strip never waits and the pipeline
// drains; each wait is also bounded, and a wait that runs out sets *flag and
// gives up (the call then fails) instead of spinning on.  The counters are
// released and acquired at workgroup scope, which orders the row buffer's
// global stores and loads between the waves of the block.
constexpr int kIntraWaves = 4;

struct IntraLds {
    int prod[kIntraWaves], cons[kIntraWaves];
    unsigned long long best[kIntraWaves];
    int take;
};

template <int R>
__device__ __forceinline__ bool intra_body(const SwArgs &A, int bin, char *lds, size_t wave_bytes,
                                           const int8_t *sblosum, IntraLds &L) {
    constexpr int W = kIntraWaves;
    const uint8_t *__restrict__ codes = A.codes;
    const PairDesc *__restrict__ pairs = A.pairs;
    const int *__restrict__ idx = A.idx, *__restrict__ starts = A.starts;
    const int go_ge = A.go_ge, ge = A.ge;
    SwPass1Out *__restrict__ out = A.p1;
    int *scratch = A.scratch;
    const int64_t scratch_per_wave = A.scratch_per_wave;
    int *queue = A.queue;
    unsigned long long *flag = A.flag;
    int *const prod = L.prod, *const cons = L.cons;
    unsigned long long *const s_best = L.best;
    int &s_take = L.take;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    ProfWord<R>(*prof)[kWave] = (ProfWord<R>(*)[kWave])(lds + (size_t)wave * wave_bytes);
    const int item_end = starts[bin + 1];
    constexpr int RS = kWave * R;
    const int in_slot = (wave + W - 1) % W;  // the slot this wave's strips read
    // slot k's row buffer: H at row[k], F' at row[k] + scratch_per_wave / 2
    int *const out_h = scratch + ((int64_t)blockIdx.x * W + wave) * scratch_per_wave;
    int *const out_f = out_h + scratch_per_wave / 2;
    const int *const in_h = scratch + ((int64_t)blockIdx.x * W + in_slot) * scratch_per_wave;
    const int *const in_f = in_h + scratch_per_wave / 2;

    bool any = false;

    for (;;) {
        // every wave is past the last pair (the barrier at its end), so the
        // block's counters and window may be reset
        if (threadIdx.x == 0) s_take = atomicAdd(queue + bin, 1);
        if (threadIdx.x < W) {
            prod[threadIdx.x] = 0;
            cons[threadIdx.x] = 0;
        }
        __syncthreads();
        const int64_t w = starts[bin] + s_take;
        if (w >= item_end) break;
        any = true;
        const int q = idx[w];
        const PairDesc pd = pairs[q];
        const uint8_t *a = codes + pd.a_off;
        const uint8_t *b = codes + pd.b_off;
        const int la = pd.la, lb = pd.lb;
        unsigned long long best = 0;  // (score << 32) | ~(row << 16 | col)
        bool ok = true;
        const int nstrips = (la > 0 && lb > 0) ? (la + RS - 1) / RS : 0;
        for (int s = wave; ok && s < nstrips; s += W) {
            const int base = s * RS + lane * R;
            build_profile<R>(prof, sblosum, a, la, base, lane);
            const bool from_above = s > 0;
            const bool to_below = s + 1 < nstrips;
            // first absolute column of the slot uses this strip reads / writes
            const int in0 = (s > 0 ? (s - 1) / W : 0) * lb, out0 = (s / W) * lb;
            int H[R], G[R], E[R], rmax[R], rcol[R];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                H[r] = 0;
                G[r] = -go_ge;
                E[r] = 0;
                rmax[r] = 0;
                rcol[r] = 0;
            }
            int hlast = 0, flast = 0, hprev = 0, cres = kPadCode;
            int chunk = kPadCode, nx = (lane < lb) ? (int)b[lane] : kPadCode;
            // the row above arrives in chunks of 64 columns, one chunk ahead
            int ch_h = 0, ch_f = 0, nx_h = 0, nx_f = 0;
            auto fetch_above = [&](int c0) {  // columns c0 .. c0 + 63 into nx
                const int hi = min(c0 + kWave, lb);
                if (ok && !lds_wait(&prod[in_slot], in0 + hi)) ok = false;
                nx_h = c0 + lane < lb ? in_h[c0 + lane] : 0;
                nx_f = c0 + lane < lb ? in_f[c0 + lane] : 0;
                if (lane == 0) lds_release(&cons[in_slot], in0 + hi);
            };
            if (from_above) fetch_above(0);
            auto step = [&](const int t, auto tail_tag) {
                constexpr bool kTail = decltype(tail_tag)::value;
                if ((t & (kWave - 1)) == 0) {
                    chunk = nx;
                    const int c = t + kWave + lane;
                    nx = (c < lb) ? (int)b[c] : kPadCode;
                    if (!kTail && from_above) {
                        ch_h = nx_h;
                        ch_f = nx_f;
                        if (t + kWave < lb) fetch_above(t + kWave);
                    }
                }
                const int bt = __builtin_amdgcn_readlane(chunk, t & (kWave - 1));
                int in_hv = 0, in_fv = 0;
                if (!kTail && from_above) {
                    in_hv = __builtin_amdgcn_readlane(ch_h, t & (kWave - 1));
                    in_fv = __builtin_amdgcn_readlane(ch_f, t & (kWave - 1));
                }
                const int rh = shr1(in_hv, hlast);
                const int rf = shr1(in_fv, flast);
                cres = shr1(bt, cres);
                const int j = t - lane;
                const bool valid = j < lb;
                const ProfWord<R> pw = prof[cres][lane];
                int hd = hprev, gu = rh - go_ge, fu = rf;
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const int e = max(subs(E[r], ge), G[r]);
                    const int f = max(subs(fu, ge), gu);
                    const int d = hd + sigma_at<R>(pw, r);
                    const int h = max(d, max(e, f));
                    hd = H[r];
                    H[r] = h;
                    E[r] = e;
                    const int g = h - go_ge;
                    G[r] = g;
                    gu = g;
                    fu = f;
                    if ((!kTail || valid) && h > rmax[r]) {
                        rmax[r] = h;
                        rcol[r] = j;
                    }
                }
                hlast = H[R - 1];
                flast = fu;
                hprev = rh;
                // lane 63 leaves column jw = t - 63 for the strip below
                const int jw = t - (kWave - 1);
                if (to_below && jw >= 0 && jw < lb) {
                    // the reader of the slot's previous use (strip s + 1 - W)
                    // must have loaded columns jw .. jw + 63 first
                    if ((jw & (kWave - 1)) == 0 && out0 > 0 && ok &&
                        !lds_wait(&cons[wave], out0 - lb + min(jw + kWave, lb)))
                        ok = false;
                    if (lane == kWave - 1) {
                        out_h[jw] = hlast;
                        out_f[jw] = flast;
                        if ((jw & (kWave - 1)) == kWave - 1 || jw == lb - 1) lds_release(&prod[wave], out0 + jw + 1);
                    }
                }
            };
            for (int t = 0; t < lb; ++t) step(t, std::false_type{});
            for (int t = lb; t < lb + kWave - 1; ++t) step(t, std::true_type{});
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int row = base + r;
                if (row < la && rmax[r] > 0) {
                    const unsigned pos = ((unsigned)row << 16) | (unsigned)rcol[r];
                    const unsigned long long k = ((unsigned long long)(unsigned)rmax[r] << 32) | (unsigned)(~pos);
                    best = k > best ? k : best;
                }
            }
        }
        if (!ok && lane == 0) atomicOr(flag, 1ull);
        best = wave_max_u64(best);
        if (lane == 0) s_best[wave] = best;
        __syncthreads();
        if (threadIdx.x == 0) {
            unsigned long long m = 0;
            for (int k = 0; k < W; ++k) m = s_best[k] > m ? s_best[k] : m;
            SwPass1Out o;
            o.score = (int32_t)(m >> 32);
            const unsigned pos = ~(unsigned)m;
            o.end_a = o.score > 0 ? (int32_t)(pos >> 16) : -1;
            o.end_b = o.score > 0 ? (int32_t)(pos & 0xFFFF) : -1;
            o.pad = 0;
            out[q] = o;
        }
        __syncthreads();
    }
    return any;
}

// sort keys of the pairing: bin, then the rows class (strip bins of up to
// 8 rows per lane: sequences a of more than 64 R - 32 rows in class 1, which
// the strip kernel runs with one row per lane more than class 0), then
// sequence a (low 24 bits of its index; the kernel checks equality itself),
// then the longer b first
constexpr int kPairKeyBits = 48;
__global__ void sw_pair_keys_kernel(const PairDesc *__restrict__ pairs, const int8_t *__restrict__ bin_of,
                                    int64_t npairs, uint64_t *__restrict__ keys, uint32_t *__restrict__ vals) {
    int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= npairs) return;
    const PairDesc pd = pairs[q];
    const int bin = (uint8_t)bin_of[q];
    const int tall = bin < kSplitBins && pd.la > kWave * (bin + 1) - kWave / 2;
    keys[q] = ((uint64_t)(2 * bin + tall) << 40) | ((uint64_t)((uint32_t)pd.a_seq & 0xFFFFFFu) << 16) |
              (uint64_t)(0xFFFF - pd.lb);
    vals[q] = (uint32_t)q;
}

// Bounds of the sorted items: class c of bin b holds [bounds[2 b + c],
// bounds[2 b + c + 1]) (lower bounds over the keys), and starts[b] =
// bounds[2 b] for the kernels that take a bin's items whole.
__global__ void sw_bounds_kernel(const uint64_t *__restrict__ keys, int npairs, int *__restrict__ bounds,
                                 int *__restrict__ starts) {
    const int k = threadIdx.x;
    if (k > 2 * kNumBins) return;
    int lo = 0, hi = npairs;
    const uint64_t key = (uint64_t)k << 40;
    while (lo < hi) {
        const int mid = lo + (hi - lo) / 2;
        if (keys[mid] < key)
            lo = mid + 1;
        else
            hi = mid;
    }
    bounds[k] = lo;
    if ((k & 1) == 0) starts[k / 2] = lo;
}

// ---------------------------------------------------------------- between the passes

// Bins by rows per lane; counters[0] += DP cells of the pairs, and
// counters[kCounterBinCells + bin] / [kCounterBinPairs + bin] += the cells and
// pairs of each bin (the host plans the launches from the latter).
__global__ void sw_bin1_kernel(const PairDesc *__restrict__ pairs, int64_t npairs, int8_t *__restrict__ bin_of,
                               unsigned long long *__restrict__ counters, int *__restrict__ queue) {
    // the work queues of this call's launches
    if (blockIdx.x == 0)
        for (int x = threadIdx.x; x < kSwQueues; x += blockDim.x) queue[x] = 0;
    __shared__ unsigned long long cells[kNumBins];
    __shared__ unsigned count[kNumBins], long_b;
    if (threadIdx.x == 0) long_b = 0;
    if (threadIdx.x < kNumBins) {
        cells[threadIdx.x] = 0;
        count[threadIdx.x] = 0;
    }
    __syncthreads();
    int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q < npairs) {
        const PairDesc pd = pairs[q];
        const int bin = rows_bin(pd.la);
        bin_of[q] = (int8_t)bin;
        atomicAdd(&cells[bin], (unsigned long long)pd.la * (unsigned long long)pd.lb);
        atomicAdd(&count[bin], 1u);
        if (bin >= kMulti16Bin && pd.lb > kTraceColsMulti) atomicAdd(&long_b, 1u);
    }
    __syncthreads();
    if (threadIdx.x == 0 && long_b) atomicAdd(&counters[kCounterLongB], (unsigned long long)long_b);
    if (threadIdx.x < kNumBins && count[threadIdx.x]) {
        atomicAdd(&counters[0], cells[threadIdx.x]);
        atomicAdd(&counters[kCounterBinCells + threadIdx.x], cells[threadIdx.x]);
        atomicAdd(&counters[kCounterBinPairs + threadIdx.x], (unsigned long long)count[threadIdx.x]);
    }
}

// Pair and cell counts are summed per block in LDS and added to counters[]
// once per block (one atomic per pair would serialise on a few addresses).
__device__ __forceinline__ void flush_counts(unsigned long long (&acc)[4], unsigned long long *counters) {
    __syncthreads();
    if (threadIdx.x < 4 && acc[threadIdx.x]) atomicAdd(&counters[1 + threadIdx.x], acc[threadIdx.x]);
}

// Records of pairs that need no statistics pass are final here; the others
// are listed for the start bound (its list and count) or go on to the
// statistics.  stats_mode: 0 = only pairs whose coverage cut can hold, 1 =
// every aligned pair, 2 = none (the normalised-score weight needs no
// traceback).  forward: the start bound is the forward one (bins by the height
// of the end rectangle; see sw_bound_kernel), and the last binning counts the
// pairs left.  counters[3], [4]: pairs and cells of the start bound, [1], [2]
// of the statistics.
__global__ __launch_bounds__(256) void sw_bin2_kernel(const PairDesc *__restrict__ pairs,
                                                      SwPass1Out *__restrict__ p1, int64_t npairs, int cov_pct,
                                                      int stats_mode, int direct_pct, int forward, TraceRule T,
                                                      pastis_pair_record *__restrict__ out,
                                                      int8_t *__restrict__ bin_of, int *__restrict__ list,
                                                      int *__restrict__ list_count,
                                                      unsigned long long *__restrict__ counters) {
    __shared__ unsigned long long acc[4];  // counters[1..4]
    __shared__ int s_n, s_base;
    if (threadIdx.x < 4) acc[threadIdx.x] = 0;
    if (threadIdx.x == 0) s_n = 0;
    __syncthreads();
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int slot = -1;
    if (q < npairs) {
        const PairDesc pd = pairs[q];
        const SwPass1Out r1 = p1[q];
        // coverage needs span_a >= cov% of la, and span_a <= end_a + 1
        const bool need = r1.score > 0 && stats_mode != 2 &&
                          (stats_mode == 1 || 100LL * (r1.end_a + 1) >= (long long)cov_pct * pd.la);
        if (need) {
            const int cols = r1.end_b >= 0 ? r1.end_b + 1 : pd.lb;
            bool direct = stats_mode == 1 || 100LL * r1.score >= (long long)direct_pct * pd.la;
            // the backward bound holds scores below 2^15
            if (!forward) direct = direct || r1.score > kBoundMaxScore;
            const int8_t bin = (int8_t)rows_bin(r1.end_a + 1);
            if (direct || forward) {
                bin_of[q] = direct && can_trace(T, pd) ? kToTrace : bin;
                if (forward) p1[q].pad = direct ? -1 : 0;  // (-1: no start bound)
            } else {
                bin_of[q] = kToBound;
                slot = atomicAdd(&s_n, 1);
            }
            const int at = direct ? 0 : 2;
            if (!(direct && forward && stats_mode == 0)) {
                atomicAdd(&acc[at], 1ull);
                atomicAdd(&acc[at + 1], (unsigned long long)(r1.end_a + 1) * (unsigned long long)cols);
            }
        } else {
            sw_final_record(pd, r1, q, out, bin_of);
        }
    }
    flush_counts(acc, counters);
    if (threadIdx.x == 0 && s_n > 0) s_base = atomicAdd(list_count, s_n);
    __syncthreads();
    if (slot >= 0) list[s_base + slot] = (int)q;
}

// ---------------------------------------------------------------- start bound

// Scores of the packed recomputation must fit 15 bits; a local alignment
// gains at most 11 per row, so rectangles up to this many rows qualify.
constexpr int kBoundMaxRows = 32000 / 11;
constexpr int kBoundMaxRowsCoarse = (1 << 19) / 11;

// The forward start bound, for records that leave the library: which pairs
// carry statistics then depends on the exact bound alone, and it finds the end
// column of the pairs it rejects, which 16-bit records then carry.
// For a pair that still needs the statistics pass, recompute its end
// rectangle [0, end_a] x [0, end_b] with every DP value packed as
// score * 65536 + (65535 - start row).  Each max then keeps the higher score
// and, between equal scores, the smaller start row, so by induction a cell
// holds the smallest start row over all optimal local alignments ending in
// it (an empty alignment ending at row i starts the next path at row i + 1).
// The canonical alignment is one of those ending at the end cell, so its
// coverage of a is at most end_a - bound + 1.  The bound goes to p1[q].pad.
// Scores must fit the high bits: rectangles of up to kBoundMaxRows rows (a
// local alignment gains at most 11 per row) use 16 low bits; up to
// kBoundMaxRowsCoarse rows pack score * 4096 + (4095 - start row / 16), a
// bound rounded down to a multiple of 16 rows (still a valid bound); taller
// ones keep bound 0 (no pruning).
template <int R, bool MULTI>
__device__ __forceinline__ void bound_body(const SwArgs &A, int bin, char *lds, size_t wave_bytes,
                                           const int8_t *sblosum) {
    constexpr int WPB = wpb32(R);
    const uint8_t *__restrict__ codes = A.codes;
    const PairDesc *__restrict__ pairs = A.pairs;
    const int *__restrict__ idx = A.idx, *__restrict__ starts = A.starts;
    const int go_ge = A.go_ge, ge = A.ge;
    SwPass1Out *__restrict__ p1 = A.p1;
    int *queue = A.queue;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    ProfWord<R>(*prof)[kWave] = (ProfWord<R>(*)[kWave])(lds + (size_t)wave * wave_bytes);
    const int64_t gwave = (int64_t)blockIdx.x * WPB + wave;
    int *bnd_h = A.scratch + gwave * A.scratch_per_wave;
    int *bnd_f = bnd_h + A.scratch_per_wave / 2;
    const int item_end = starts[bin + 1];
    constexpr int RS = kWave * R;
    constexpr int kNegP = -(1 << 30);
    const int GO16 = go_ge * 65536, GE16 = ge * 65536;

    // windows of two pairs per claim
    for (int64_t w0 = take(queue, starts, bin, 2); w0 < item_end; w0 = take(queue, starts, bin, 2))
    for (int64_t w = w0; w < min(w0 + 2, (int64_t)item_end); ++w) {
        const int q = idx[w];
        const PairDesc pd = pairs[q];
        const SwPass1Out r1 = p1[q];
        if (r1.pad < 0) continue;  // sent straight to the statistics pass
        // end_b < 0: unknown (16-bit pass 1); the end column is then the first
        // one where row end_a reaches the score
        const bool search = r1.end_b < 0;
        const int la = r1.end_a + 1, lb = search ? pd.lb : r1.end_b + 1;
        if (la > kBoundMaxRowsCoarse) {
            if (lane == 0) p1[q].pad = 0;
            continue;
        }
        // packing: sb low bits hold (mask - start row >> shift)
        const int sb = la > kBoundMaxRows ? 12 : 16, shift = 16 - sb;
        const int mask = (1 << sb) - 1, unit = 1 << sb;
        const int kZero = mask;  // score 0, start row 0
        const int GO = sb == 16 ? GO16 : go_ge * unit, GE = sb == 16 ? GE16 : ge * unit;
        const uint8_t *a = codes + pd.a_off;
        const uint8_t *b = codes + pd.b_off;
        const int nstrips = MULTI ? (la + RS - 1) / RS : 1;
        const int top = nstrips * RS - la;  // padding rows above row 0
        int fin = 0, fend = -1;  // lane 63: the end cell's value and (search) its column
        // profile entries are addressed by byte offset: lane base + code * stride
        const char *prof_lane = (const char *)&prof[0][lane];
        constexpr int kStride = (int)(sizeof(ProfWord<R>) * kWave);
        for (int s = 0; s < nstrips; ++s) {
            const int base = s * RS - top + lane * R;
            build_profile<R>(prof, sblosum, a, la, base, lane);
            const bool from_above = s > 0;
            const bool to_below = s + 1 < nstrips;
            const bool last = s + 1 == nstrips;
            int H[R], G[R], E[R], Z[R];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                Z[r] = mask - (max(base + r + 1, 0) >> shift);  // empty alignment ending in row base + r
                H[r] = Z[r];                           // column -1
                G[r] = Z[r] - GO;
                E[r] = kNegP;
            }
            int hlast = kZero, flast = kNegP, hprev = kZero, cres = kPadCode * kStride, chunk = kPadCode * kStride;
            int nx = ((lane < lb) ? (int)b[lane] : kPadCode) * kStride;
            int ch_h = kZero, ch_f = kNegP, nx_h = kZero, nx_f = kNegP;
            if (MULTI && from_above && lane < lb) {
                nx_h = vload(bnd_h + lane);
                nx_f = vload(bnd_f + lane);
            }
            const int steps = __builtin_amdgcn_readfirstlane(lb + kWave - 1);
            auto step = [&](const int t) {
                if ((t & (kWave - 1)) == 0) {
                    chunk = nx;
                    const int c = t + kWave + lane;
                    nx = ((c < lb) ? (int)b[c] : kPadCode) * kStride;
                    if (MULTI && from_above) {
                        ch_h = nx_h;
                        ch_f = nx_f;
                        if (c < lb) {
                            nx_h = vload(bnd_h + c);
                            nx_f = vload(bnd_f + c);
                        }
                    }
                }
                const int bt = __builtin_amdgcn_readlane(chunk, t & (kWave - 1));
                int in_h = kZero, in_f = kNegP;
                if (MULTI && from_above && t < lb) {
                    in_h = __builtin_amdgcn_readlane(ch_h, t & (kWave - 1));
                    in_f = __builtin_amdgcn_readlane(ch_f, t & (kWave - 1));
                }
                const int rh = shr1(in_h, hlast);
                const int rf = shr1(in_f, flast);
                cres = shr1(bt, cres);
                const ProfWord<R> pw = *(const ProfWord<R> *)(prof_lane + cres);
                int hd = hprev, gu = rh - GO, fu = rf;
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    // E' = max(E, Z): the row's empty-alignment floor rides
                    // along the row (max(E' - e, Z) = max(E - e, Z), since Z
                    // - e < Z), so h is one three-way max
                    const int e = max(max(E[r] - GE, G[r]), Z[r]);
                    const int f = max(fu - GE, gu);
                    const int d = hd + sigma_at<R>(pw, r) * unit;
                    const int h = max(max(d, e), f);
                    hd = H[r];
                    H[r] = h;
                    E[r] = e;
                    const int g = h - GO;
                    G[r] = g;
                    gu = g;
                    fu = f;
                }
                hlast = H[R - 1];
                flast = fu;
                hprev = rh;
                if (MULTI && to_below) {
                    const int j = t - (kWave - 1);
                    if (lane == kWave - 1 && j >= 0 && j < lb) {
                        bnd_h[j] = hlast;
                        bnd_f[j] = flast;
                    }
                }
            };
            int t = 0;
            if (!(search && last)) {
                // two steps per iteration; lane 63's last value is the end cell's
                for (; t + 1 < steps; t += 2) {
                    step(t);
                    step(t + 1);
                }
                if (t < steps) step(t);
                if (last) fin = hlast;
            } else {
                // the end column is the first where lane 63 (row end_a) reaches
                // the score; no cell exceeds it, so reaching is h >= score * unit
                const int thr = r1.score * unit;
                for (; t < kWave - 1; ++t) step(t);  // lane 63 is still left of column 0
                for (; t + 1 < steps; t += 2) {
                    step(t);
                    const int h1 = hlast;
                    step(t + 1);
                    if (__builtin_amdgcn_readlane(h1, kWave - 1) >= thr) {
                        fin = h1;
                        fend = t - (kWave - 1);
                        break;
                    }
                    if (__builtin_amdgcn_readlane(hlast, kWave - 1) >= thr) {
                        fin = hlast;
                        fend = t + 1 - (kWave - 1);
                        break;
                    }
                }
                if (fend < 0 && t < steps) {
                    step(t);
                    if (__builtin_amdgcn_readlane(hlast, kWave - 1) >= thr) {
                        fin = hlast;
                        fend = t - (kWave - 1);
                    }
                }
            }
            if (MULTI) __threadfence_block();
        }
        if (lane == kWave - 1) {
            p1[q].pad = (mask - (fin & mask)) << shift;
            if (search) p1[q].end_b = fend;
        }
    }
}

// Pairs binned for the statistics pass whose coverage bound already fails
// get their final record here; the rest are listed for the traceback or keep
// their bin.  counters[1] and [2] count the pairs and cells left.
__global__ __launch_bounds__(256) void sw_bin3_kernel(const PairDesc *__restrict__ pairs,
                                                      const SwPass1Out *__restrict__ p1, int64_t npairs,
                                                      int cov_pct, TraceRule T, pastis_pair_record *__restrict__ out,
                                                      int8_t *__restrict__ bin_of,
                                                      unsigned long long *__restrict__ counters) {
    __shared__ unsigned long long acc[4];  // counters[1..4]; [1] and [2] here
    if (threadIdx.x < 4) acc[threadIdx.x] = 0;
    __syncthreads();
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q < npairs && bin_of[q] != -1) {
        const PairDesc pd = pairs[q];
        const SwPass1Out r1 = p1[q];
        // pad < 0: sent straight here (bound 0 in effect: the coverage test of
        // the first binning already holds)
        if (r1.pad < 0 || 100LL * (r1.end_a - r1.pad + 1) >= (long long)cov_pct * pd.la) {
            const int cols = r1.end_b >= 0 ? r1.end_b + 1 : pd.lb;
            if (can_trace(T, pd)) bin_of[q] = kToTrace;
            atomicAdd(&acc[0], 1ull);
            atomicAdd(&acc[1], (unsigned long long)(r1.end_a + 1) * (unsigned long long)cols);
        } else {
            sw_final_record(pd, r1, q, out, bin_of);
        }
    }
    flush_counts(acc, counters);
}

// The traceback's list, in the order of pass 1's sorted items (so that pairs
// of one sequence a stay together): flags by sorted position, then (after an
// exclusive scan of them) the kept items and their class bounds.
__global__ void trace_flags_kernel(const int *__restrict__ idx, const int8_t *__restrict__ bin_of, int npairs,
                                   uint8_t *__restrict__ flag) {
    const int x = blockIdx.x * blockDim.x + threadIdx.x;
    if (x < npairs) flag[x] = bin_of[idx[x]] == kToTrace ? 1 : 0;
}

__global__ void trace_list_kernel(const int *__restrict__ idx, const uint8_t *__restrict__ flag,
                                  const uint32_t *__restrict__ pos, int npairs, const int *__restrict__ bounds,
                                  int *__restrict__ list, int *__restrict__ list_bounds) {
    const int x = blockIdx.x * blockDim.x + threadIdx.x;
    if (x < npairs && flag[x]) list[pos[x]] = idx[x];
    if (x <= 2 * kNumBins) list_bounds[x] = (int)pos[min(bounds[x], npairs)];  // pos[npairs]: the total
}

// ---------------------------------------------------------------- pass 2

// No per-wave profile: a row's score against the column residue is read from
// the 625-entry table, so LDS does not limit the waves per SIMD (occupancy
// matters here: the statistics selects are long dependent chains).  Entries
// are 32-bit; the statistics increment of each code pair (0x10001 for
// identical codes, else 1) follows the scores, so a cell reads it at its
// score's address plus a constant.  Column residues travel as byte offsets
// (code * 4) into a row of the table.
constexpr int kTab = kProfCodes * kProfCodes;

template <int R, bool MULTI>
__device__ __forceinline__ void stats_body(const SwArgs &A, int bin, const int *stab) {
    constexpr int WPB = wpb32(R);
    const uint8_t *__restrict__ codes = A.codes;
    const PairDesc *__restrict__ pairs = A.pairs;
    const int *__restrict__ idx = A.idx, *__restrict__ starts = A.starts;
    const int go_ge = A.go_ge, ge = A.ge, cov_pct = A.cov_pct, id_pct = A.id_pct;
    const SwPass1Out *__restrict__ p1 = A.p1;
    pastis_pair_record *__restrict__ out = A.rec;
    int *queue = A.queue;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    const int64_t gwave = (int64_t)blockIdx.x * WPB + wave;
    // strip bottom row per column: H, F, H.beg, H.md, F.beg, F.md
    int *bnd = A.scratch + gwave * A.scratch_per_wave;
    const int64_t plane = A.scratch_per_wave / 6;
    const int item_end = starts[bin + 1];
    constexpr int RS = kWave * R;

    for (int64_t w = take(queue, starts, bin, 1); w < item_end; w = take(queue, starts, bin, 1)) {
        const int q = idx[w];
        const PairDesc pd = pairs[q];
        const SwPass1Out r1 = p1[q];
        const uint8_t *a = codes + pd.a_off;
        const uint8_t *b = codes + pd.b_off;
        // the rectangle ending at the end cell; with the end column unknown
        // (16-bit pass 1), the full width until row end_a first reaches the score
        const bool search = r1.end_b < 0;
        const int la = r1.end_a + 1, lb = search ? pd.lb : r1.end_b + 1;
        const int nstrips = MULTI ? (la + RS - 1) / RS : 1;
        const int top = nstrips * RS - la;  // padding rows above row 0
        unsigned fin_beg = 0, fin_md = 0;
        int fend = -1;
        for (int s = 0; s < nstrips; ++s) {
            const int base = s * RS - top + lane * R;
            const char *srow[R];  // the row's table entries, at byte offset code * 4
            unsigned rowpart[R];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int ar = (base + r >= 0 && base + r < la) ? (int)a[base + r] : kPadCode;
                srow[r] = (const char *)(stab + ar * kProfCodes);
                rowpart[r] = (unsigned)(base + r) << 16;
            }
            const bool from_above = s > 0;
            const bool to_below = s + 1 < nstrips;
            const bool last = s + 1 == nstrips;
            int H[R], G[R], E[R];
            unsigned sHb[R], sHm[R], sEb[R], sEm[R];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                H[r] = 0;
                G[r] = -go_ge;
                E[r] = kNeg;
                sHb[r] = sHm[r] = sEb[r] = sEm[r] = 0u;
            }
            int hlast = 0, flast = kNeg, hprev = 0, cres = 4 * kPadCode, chunk = 4 * kPadCode;
            unsigned hb_last = 0, hm_last = 0, fb_last = 0, fm_last = 0, db_prev = 0, dm_prev = 0;
            // chunked, one-ahead prefetch of residues and boundary planes (see pass 1)
            int nx = 4 * ((lane < lb) ? (int)b[lane] : kPadCode);
            int cb[6] = {0, kNeg, 0, 0, 0, 0}, nb[6] = {0, kNeg, 0, 0, 0, 0};
            if (MULTI && from_above && lane < lb) {
#pragma unroll
                for (int p = 0; p < 6; ++p) nb[p] = vload(bnd + p * plane + lane);
            }
            const int steps = __builtin_amdgcn_readfirstlane(lb + kWave - 1);
            // one column step; true once the search has found the end column
            auto step = [&](const int t) -> bool {
                if ((t & (kWave - 1)) == 0) {
                    chunk = nx;
                    const int c = t + kWave + lane;
                    nx = 4 * ((c < lb) ? (int)b[c] : kPadCode);
                    if (MULTI && from_above) {
#pragma unroll
                        for (int p = 0; p < 6; ++p) cb[p] = nb[p];
                        if (c < lb) {
#pragma unroll
                            for (int p = 0; p < 6; ++p) nb[p] = vload(bnd + p * plane + c);
                        }
                    }
                }
                const int bt = __builtin_amdgcn_readlane(chunk, t & (kWave - 1));
                int rh, rf;
                unsigned rhb, rhm, rfb, rfm;
                if (MULTI) {
                    int in_h = 0, in_f = kNeg;
                    unsigned in_hb = 0, in_hm = 0, in_fb = 0, in_fm = 0;
                    if (from_above && t < lb) {
                        const int tt = t & (kWave - 1);
                        in_h = __builtin_amdgcn_readlane(cb[0], tt);
                        in_f = __builtin_amdgcn_readlane(cb[1], tt);
                        in_hb = (unsigned)__builtin_amdgcn_readlane(cb[2], tt);
                        in_hm = (unsigned)__builtin_amdgcn_readlane(cb[3], tt);
                        in_fb = (unsigned)__builtin_amdgcn_readlane(cb[4], tt);
                        in_fm = (unsigned)__builtin_amdgcn_readlane(cb[5], tt);
                    }
                    rh = shr1(in_h, hlast);
                    rf = shr1(in_f, flast);
                    rhb = (unsigned)shr1((int)in_hb, (int)hb_last);
                    rhm = (unsigned)shr1((int)in_hm, (int)hm_last);
                    rfb = (unsigned)shr1((int)in_fb, (int)fb_last);
                    rfm = (unsigned)shr1((int)in_fm, (int)fm_last);
                } else {
                    // row -1 above a single strip: H = 0 with empty
                    // statistics, F closed; the zero-filling shift writes
                    // lane 0's zeros itself
                    rh = shr1z(hlast);
                    rf = shr1(kNeg, flast);
                    rhb = (unsigned)shr1z((int)hb_last);
                    rhm = (unsigned)shr1z((int)hm_last);
                    rfb = (unsigned)shr1z((int)fb_last);
                    rfm = (unsigned)shr1z((int)fm_last);
                }
                cres = shr1(bt, cres);
                const int j = t - lane;
                const unsigned colpart = (unsigned)j & 0xFFFFu;
                int hd = hprev, gu = rh - go_ge, fu = rf;
                unsigned db = db_prev, dm = dm_prev, ub = rhb, um = rhm, fb = rfb, fm = rfm;
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    // horizontal gap: extend when at least as good as opening
                    const int e_ext = E[r] - ge;
                    const bool ee = e_ext >= G[r];
                    const int e = ee ? e_ext : G[r];
                    const unsigned eb = ee ? sEb[r] : sHb[r];
                    const unsigned em = ee ? sEm[r] : sHm[r];
                    // vertical gap
                    const int f_ext = fu - ge;
                    const bool fe = f_ext >= gu;
                    const int f = fe ? f_ext : gu;
                    const unsigned nfb = fe ? fb : ub;
                    const unsigned nfm = fe ? fm : um;
                    // diagonal; a zero predecessor starts a new path at this cell
                    const int d = hd + *(const int *)(srow[r] + cres);
                    const int h = max(max(d, 0), max(e, f));
                    const bool start = hd == 0;
                    const unsigned xb = start ? (rowpart[r] | colpart) : db;
                    const unsigned xm = (start ? 0u : dm) + *(const unsigned *)(srow[r] + 4 * kTab + cres);
                    const bool is_d = h == d, is_e = h == e;
                    const unsigned hb = is_d ? xb : (is_e ? eb : nfb);
                    const unsigned hm = is_d ? xm : (is_e ? em : nfm);
                    hd = H[r];
                    db = sHb[r];
                    dm = sHm[r];
                    H[r] = h;
                    E[r] = e;
                    const int g = h - go_ge;
                    G[r] = g;
                    sHb[r] = hb;
                    sHm[r] = hm;
                    sEb[r] = eb;
                    sEm[r] = em;
                    gu = g;
                    fu = f;
                    ub = hb;
                    um = hm;
                    fb = nfb;
                    fm = nfm;
                }
                hlast = H[R - 1];
                flast = fu;
                hb_last = ub;
                hm_last = um;
                fb_last = fb;
                fm_last = fm;
                hprev = rh;
                db_prev = rhb;
                dm_prev = rhm;
                if (last && lane == kWave - 1 && j >= 0 && j < lb &&
                    (search ? (fend < 0 && hlast == r1.score) : j == lb - 1)) {
                    fin_beg = hb_last;
                    fin_md = hm_last;
                    fend = j;
                }
                if (MULTI && to_below && lane == kWave - 1 && j >= 0 && j < lb) {
                    bnd[j] = hlast;
                    bnd[plane + j] = flast;
                    bnd[2 * plane + j] = (int)hb_last;
                    bnd[3 * plane + j] = (int)hm_last;
                    bnd[4 * plane + j] = (int)fb_last;
                    bnd[5 * plane + j] = (int)fm_last;
                }
                return search && last && __builtin_amdgcn_readlane(fend, kWave - 1) >= 0;
            };
            if constexpr (MULTI && R >= 14) {
                // the boundary planes leave no registers for a second step
                for (int t = 0; t < steps; ++t)
                    if (step(t)) break;
            } else {
                // two steps per iteration, so the rows' registers need no rotation
                int t = 0;
                bool done = false;
                for (; t + 1 < steps; t += 2) {
                    if (step(t) || step(t + 1)) {
                        done = true;
                        break;
                    }
                }
                if (!done && t < steps) step(t);
            }
            if (MULTI) __threadfence_block();
        }
        if (lane == kWave - 1) {
            pastis_pair_record rec;
            rec.score = r1.score;
            rec.end_a = r1.end_a;
            rec.end_b = fend;
            rec.beg_a = (int32_t)(fin_beg >> 16);
            rec.beg_b = (int32_t)(fin_beg & 0xFFFF);
            rec.matches = (int32_t)(fin_md >> 16);
            const int32_t diag = (int32_t)(fin_md & 0xFFFF);
            rec.columns = (rec.end_a - rec.beg_a + 1) + (rec.end_b - rec.beg_b + 1) - diag;
            rec.seed_used = -1;
            const long long span = (long long)rec.end_a - rec.beg_a + 1;
            rec.passed = (100LL * rec.matches >= (long long)id_pct * rec.columns) &&
                         (100LL * span >= (long long)cov_pct * pd.la);
            rec.swapped = pd.swapped;
            rec.cells = (int64_t)pd.la * pd.lb;
            out[q] = rec;
        }
    }
}

// ---------------------------------------------------------------- group launches

// One launch runs the bins of a group (a range of rows per lane), the tallest
// first: a wave that finds a bin's queue empty goes on to the next bin, so a
// call has one launch tail per group instead of one per bin.  A bin's tail is
// as long as its longest pair (0.3 to 5 ms), whatever its pair count, so
// launching bin after bin cost a set of 10,000 sequences 27 ms of pass 1 for
// 3 ms of work.  The groups keep the occupancy of their bins: one profile size
// and about one register count each.
template <int R, bool MULTI>
constexpr int bin_of_rows(int half) {
    return !MULTI ? R - 1 : (half ? kMulti16Bin : kMultiBin) + R - kMultiMinR;
}

template <int R>
__host__ __device__ constexpr size_t prof_bytes() {
    return sizeof(ProfWord<R>) * kProfCodes * kWave;
}

// Calls f(integral R, bin) for the group's non-empty bins of the mask, tallest first.
template <int R, bool MULTI, typename F>
__device__ __forceinline__ void for_rows(const int *starts, uint32_t bins, F &f) {
#pragma unroll 1
    for (int half = 0; half < (MULTI ? 2 : 1); ++half) {
        const int bin = bin_of_rows<R, MULTI>(half);
        if (((bins >> bin) & 1u) && starts[bin] < starts[bin + 1]) f(std::integral_constant<int, R>{}, bin);
    }
}

template <int HI, bool MULTI, typename F, int... I>
__device__ __forceinline__ void for_bins_of(const int *starts, uint32_t bins, F &f, std::integer_sequence<int, I...>) {
    (for_rows<HI - I, MULTI>(starts, bins, f), ...);
}

template <int LO, int HI, bool MULTI, typename F>
__device__ __forceinline__ void for_bins(const int *starts, uint32_t bins, F &&f) {
    for_bins_of<HI, MULTI>(starts, bins, f, std::make_integer_sequence<int, HI - LO + 1>{});
}

template <int LO, int HI, bool MULTI>
__global__ __launch_bounds__(64 * wpb32(HI)) void sw_pass1_kernel(SwArgs A, uint32_t bins) {
    static_assert(wpb32(LO) == wpb32(HI), "one block size per group");
    __shared__ __align__(16) char lds[wpb32(HI) * prof_bytes<HI>()];
    __shared__ int8_t sblosum[kProfCodes * kProfCodes];
    load_blosum(sblosum, A.blosum);
    for_bins<LO, HI, MULTI>(A.starts, bins, [&](auto r_tag, int bin) {
        const unsigned long long t0 = span_now();
        if (pass1_body<decltype(r_tag)::value, MULTI>(A, bin, lds, prof_bytes<HI>(), sblosum))
            span_add(A.span + 2 * bin, t0);
    });
}

template <int LO, int HI>
__global__ __launch_bounds__(64 * kIntraWaves) void sw_intra_pass1_kernel(SwArgs A, uint32_t bins) {
    __shared__ __align__(16) char lds[kIntraWaves * prof_bytes<HI>()];
    __shared__ int8_t sblosum[kProfCodes * kProfCodes];
    __shared__ IntraLds L;
    load_blosum(sblosum, A.blosum);
    for_bins<LO, HI, true>(A.starts, bins, [&](auto r_tag, int bin) {
        const unsigned long long t0 = span_now();
        if (intra_body<decltype(r_tag)::value>(A, bin, lds, prof_bytes<HI>(), sblosum, L))
            span_add(A.span + 2 * bin, t0);
        __syncthreads();  // every wave has read the last window before the next bin's first claim
    });
}

template <int LO, int HI, bool MULTI>
__global__ __launch_bounds__(64 * wpb32(HI)) void sw_bound_kernel(SwArgs A, uint32_t bins) {
    static_assert(wpb32(LO) == wpb32(HI), "one block size per group");
    __shared__ __align__(16) char lds[wpb32(HI) * prof_bytes<HI>()];
    __shared__ int8_t sblosum[kProfCodes * kProfCodes];
    load_blosum(sblosum, A.blosum);
    for_bins<LO, HI, MULTI>(A.starts, bins, [&](auto r_tag, int bin) {
        bound_body<decltype(r_tag)::value, MULTI>(A, bin, lds, prof_bytes<HI>(), sblosum);
    });
}

// waves per SIMD the statistics groups ask for: those their bins reached
// alone (the selects' dependent chains need them)
constexpr int stats_waves(int HI) { return HI <= 4 ? 4 : HI <= 12 ? 2 : 1; }

template <int LO, int HI, bool MULTI>
__global__ __launch_bounds__(64 * wpb32(HI), stats_waves(HI)) void sw_pass2_kernel(SwArgs A, uint32_t bins) {
    static_assert(wpb32(LO) == wpb32(HI), "one block size per group");
    __shared__ int stab[2 * kTab];
    for (int t = threadIdx.x; t < kTab; t += blockDim.x) {
        stab[t] = A.blosum[t];
        stab[kTab + t] = t / kProfCodes == t % kProfCodes ? 0x10001 : 1;
    }
    __syncthreads();
    for_bins<LO, HI, MULTI>(A.starts, bins,
                            [&](auto r_tag, int bin) { stats_body<decltype(r_tag)::value, MULTI>(A, bin, stab); });
}

// The groups: one-strip bins of 1-4, 5-8, 9-12 and 13-16 rows per lane, and
// the multi-strip bins (all of a group's kernels take the same mask of bins).
constexpr int kGroups = 5, kMultiGroup = 4;
constexpr int kLongGroup = 5;                 // the pairs of the multi-strip bins that take a block each
constexpr uint32_t kOverBins = 0x00FF0000u;  // multi-strip bins of over kMax16Rows rows
static_assert(kOverBins == (1u << kMulti16Bin) - (1u << kMultiBin), "bins of the tallest sequences");
constexpr uint32_t kGroupBins[kGroups] = {0x000Fu, 0x00F0u, 0x0F00u, 0xF000u, 0xFFFF0000u};

typedef void (*SwKernel)(SwArgs, uint32_t);
const SwKernel kPass1[kGroups] = {sw_pass1_kernel<1, 4, false>, sw_pass1_kernel<5, 8, false>,
                                  sw_pass1_kernel<9, 12, false>, sw_pass1_kernel<13, 16, false>,
                                  sw_pass1_kernel<9, 16, true>};
const SwKernel kBound[kGroups] = {sw_bound_kernel<1, 4, false>, sw_bound_kernel<5, 8, false>,
                                  sw_bound_kernel<9, 12, false>, sw_bound_kernel<13, 16, false>,
                                  sw_bound_kernel<9, 16, true>};
const SwKernel kStats[kGroups] = {sw_pass2_kernel<1, 4, false>, sw_pass2_kernel<5, 8, false>,
                                  sw_pass2_kernel<9, 12, false>, sw_pass2_kernel<13, 16, false>,
                                  sw_pass2_kernel<9, 16, true>};
constexpr int kGroupWpb[kGroups] = {4, 4, 2, 2, 2};
// blocks that fit on the device at once: the LDS footprint of the profiles
// (26, 52, 39 and 52 KB per block) on 256 CUs
constexpr int kGroupBlocks[kGroups] = {256 * 6, 256 * 3, 256 * 4, 256 * 3, 256 * 3};
// intra-pair pass 1: one block of four waves per pair, one block per CU (the
// four strip profiles take up to 100 KB of LDS); the row buffers of the
// block's slots are four of the per-wave boundary buffers
constexpr int kIntraBlocks = 256;

// 16-bit kernels: the blocks resident at once, those that also take the
// multi-strip bins in the traceback, and the call size up to which the bins of
// up to 8 rows per lane run across all 64 lanes.  With that many pairs two to
// a wave, every SIMD has about four waves (3,164 pairs of up to 600 rows: pass
// 1 in 0.37 ms across 64 lanes, 0.57 in strips of 16 and 32).  Full records of n
// pairs of families of 350 residues: 2.3 ms across 64 lanes and 2.45 in strips at
// 4,096, 2.4 and 3.1 at 8,192, 2.5 and 3.05 at 12,288, 3.3 and 3.65 at 16,384: the
// line is where the chip is full, and pairs that share their sequence less than
// these do not lose at it.
constexpr int kBlocks16 = 256 * 6, kTraceMultiBlocks = 256;
constexpr int64_t kWidePairs = 8192;

// Pairs of the 32-bit multi-strip bins, and pairs that may need the multi-strip
// statistics, up to this many take one block of eight waves each (sw_long.hip);
// beyond, the waves that work strip after strip keep the chip as busy.  Where only
// those of at most kMax16Rows rows are too many, the others still take blocks if a
// single wave would take longer for the longest pair than the chip for all of them
// (a wave takes 0.39 ns for a cell of 25,000 rows' pairs, the chip 0.42 ps: a factor
// of about kWaveShare).
// Pass 1 + statistics, blocks against waves: n pairs of 3,000 to 4,000 rows 8.4 +
// 15.2 ms against 11.4 + 20.8 (n = 1,024), 16.6 + 30.0 against 14.2 + 34.6 (2,048),
// 32.8 + 59.6 against 24.6 + 67.1 (4,096); of 8,000 to 9,000 rows 80 + 110 against
// 78 + 197 (2,048); of 3,000 to 25,000 rows, where single waves are as long as the
// longest pair, 281 + 288 against 439 + 1,094 (2,048); of 1,030 to 1,500 rows 2.6 +
// 5.4 against 1.8 + 3.0 (1,024), 5.2 + 10.5 against 2.1 + 4.8 (2,048).  A block's
// scratch grows with the longest sequence (20 MB for 25,000 residues); blocks are
// dropped beyond kLongBytes.
constexpr int64_t kLongPairs = 2048, kWaveShare = 1024;
constexpr int kLongBlocks = 256;

// Resident blocks per CU of the one-strip statistics kernels: they keep no
// profile in LDS, so registers set their occupancy, which the runtime reports
// for the compiled code; a grid of that many blocks per CU drains each group.
std::atomic<int> stats_blocks_per_cu[kGroups];

}  // namespace

void sw_init_occupancy() {
    if (stats_blocks_per_cu[kGroups - 1].load(std::memory_order_acquire) != 0) return;
    for (int g = 0; g < kGroups; ++g) {
        int nb = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, kStats[g], 64 * kGroupWpb[g], 0) != hipSuccess || nb < 1) {
            (void)hipGetLastError();
            nb = 2;
        }
        stats_blocks_per_cu[g].store(nb, std::memory_order_release);
    }
}

int sw_num_bins() { return kNumBins; }

void sw_bin_shape(int bin, int32_t *rows_per_lane, int32_t *multi) {
    *multi = bin >= kMultiBin;
    *rows_per_lane = rows_of_bin(bin);
}

// Only the multi-strip bins use the boundary buffers (one per wave of the
// grid).
int sw_one_strip_max_rows() { return kWave * kSingleBins; }

int64_t sw_scratch_waves() {
    return std::max<int64_t>((int64_t)kGroupBlocks[kMultiGroup] * kGroupWpb[kMultiGroup],
                             (int64_t)kIntraBlocks * kIntraWaves);
}
bool sw_bins_multi(uint32_t bins) { return (bins & kGroupBins[kMultiGroup]) != 0; }

// The 16-bit profile holds each biased score s + o + e in one byte, with
// s <= 11 in BLOSUM62; other gap costs run in 32-bit lanes.
bool sw16_supported(const Scoring &sc) {
    const int oe = sc.gap_open + sc.gap_extend;
    return oe >= 4 && oe + 11 <= 255;
}

bool sw_bin_is16(int bin, int max16) {
    return (bin < kSingleBins || bin >= kMulti16Bin) && rows_of_bin(bin) <= max16;
}

hipError_t launch_sw_bins(const PairDesc *pairs, int64_t npairs, const SwWork &wk, hipStream_t s) {
    if (npairs <= 0) return hipSuccess;
    sw_bin1_kernel<<<(unsigned)((npairs + 255) / 256), 256, 0, s>>>(pairs, npairs, wk.bin_of, wk.counters, wk.queue);
    return hipGetLastError();
}

// direction words of a wave's one-strip and multi-strip pairs
static int64_t dirs_of_wave(int max_len) { return (int64_t)(std::min(max_len, kTraceCols) + kWave) * sw16_step_words(); }
static int64_t dirs_of_multi(int max_len) {
    return (int64_t)kTraceStrips * (std::min(max_len, kTraceColsMulti) + kWave) * sw16_step_words();
}

size_t sw_dirs_most(int max_len) {
    return sizeof(uint32_t) * (size_t)sw16_waves() *
           (size_t)(kBlocks16 * dirs_of_wave(max_len) + kTraceMultiBlocks * dirs_of_multi(max_len));
}

// The launches of a call, from its pairs per bin.
SwPlan sw_plan(const unsigned long long *bin_pairs, const unsigned long long *bin_cells, int64_t long_b, int max16,
               int max_len, bool trace, bool slots, const pastis_tuning &tune) {
    SwPlan p;
    p.max16 = max16;
    p.intra = tune.sw_intra_pair;
    // multi-strip launches: at most long_blocks blocks per CU (they run beside
    // the one-strip bins on another stream; fewer resident waves leave the
    // one-strip kernels more room).  Fewer blocks than the default never
    // exceed the boundary buffers, which are sized for the default grids.
    auto fit = [&](int g, int blocks, int64_t pairs) {
        const int scale = g == kMultiGroup ? 1 : g < 2 ? tune.sw_grid_scale : tune.sw_grid_scale_wide;
        const int64_t b = g == kMultiGroup ? std::min(blocks, 256 * tune.sw_long_blocks) : (int64_t)blocks * scale;
        // no launch needs more blocks than its pairs could fill
        return (int)std::min<int64_t>(b, (pairs + kGroupWpb[g] - 1) / kGroupWpb[g]);
    };
    // every group from the tallest non-empty one down may hold pairs of the
    // later passes, whose end rectangles are no taller than the pairs; a
    // multi-strip pair may end in any bin
    int64_t later = 0, n16 = 0, wide16 = 0, strips16 = 0, multi16 = 0;
    bool any32 = false;
    for (int g = kMultiGroup; g >= 0; --g) {
        int64_t n32 = 0;
        for (int b = 0; b < kNumBins; ++b) {
            if (!((kGroupBins[g] >> b) & 1u) || bin_pairs[b] == 0) continue;
            const int64_t n = (int64_t)bin_pairs[b];
            later += n;
            if (sw_bin_is16(b, max16)) {
                n16 += n;
                (b < kSplitBins ? strips16 : wide16) += n;
                if (b >= kMulti16Bin) multi16 += n;
                p.p16.bins |= 1u << b;
            } else {
                n32 += n;
                p.bins32[g] |= 1u << b;
            }
        }
        any32 = any32 || n32 > 0;
        p.blocks32[g] = n32 ? fit(g, kGroupBlocks[g], n32) : 0;
        p.blocks_bound[g] = later ? fit(g, kGroupBlocks[g], later) : 0;
        const int per_cu = g == kMultiGroup ? 3 : std::max(1, stats_blocks_per_cu[g].load(std::memory_order_acquire));
        p.blocks_stats[g] = later ? fit(g, 256 * per_cu, later) : 0;
    }
    // pairs of the multi-strip bins of over kMax16Rows rows, and of fewer: those of
    // pass 1 in 32-bit lanes, and those that may come to the multi-strip statistics
    int64_t over = 0, low1 = 0, low2 = n16 > 0 && trace ? long_b : 0, cells = 0;
    int64_t over_cells = 0, cells16 = 0;
    for (int b = 0; b < kNumBins; ++b)
        if (sw_bin_is16(b, max16)) cells16 += (int64_t)bin_cells[b];
    for (int b = kMultiBin; b < kNumBins; ++b) {
        const bool is16 = sw_bin_is16(b, max16);
        cells += (int64_t)bin_cells[b];
        if (b < kMulti16Bin) {
            over += (int64_t)bin_pairs[b];
            over_cells += (int64_t)bin_cells[b];
        }
        if (b >= kMulti16Bin && !is16) low1 += (int64_t)bin_pairs[b];
        if (b >= kMulti16Bin && !(is16 && trace)) low2 += (int64_t)bin_pairs[b];
    }
    if (slots) {
        const int64_t slot = sw_long_slot_words(max_len);
        const int64_t room = std::max<int64_t>(8, (int64_t)kLongBytes / (int64_t)(slot * sizeof(int)));
        const bool apart = cells < kWaveShare * max_len * max_len;
        auto take = [&](int64_t low, uint32_t &bins, int &blocks) {
            bins = over + low <= kLongPairs ? kGroupBins[kMultiGroup] : over <= kLongPairs && apart ? kOverBins : 0u;
            const int64_t pairs = bins == 0 ? 0 : bins == kOverBins ? over : over + low;
            blocks = (int)std::min<int64_t>({kLongBlocks, room, pairs});
            if (blocks == 0) bins = 0;
        };
        take(low1, p.long_bins1, p.long_blocks1);
        take(low2, p.long_bins2, p.long_blocks2);
        if (p.long_blocks1 > 0 || p.long_blocks2 > 0) p.long_slot = slot;
        p.long_bins1 &= p.bins32[kMultiGroup];
        p.bins32[kMultiGroup] &= ~p.long_bins1;
        if (p.bins32[kMultiGroup] == 0)
            p.blocks32[kMultiGroup] = 0;
        else if (p.long_bins1 != 0)
            p.blocks32[kMultiGroup] = fit(kMultiGroup, kGroupBlocks[kMultiGroup], low1);
        if (p.long_bins2 == kGroupBins[kMultiGroup]) p.blocks_stats[kMultiGroup] = 0;
        // few long pairs, none of them long to do: the traceback comes after them.
        // Beside them its first blocks, which take the multi-strip pairs, crowd on the
        // CUs that the long pairs leave free (a search of 250,000 sequences with the
        // learned filter: 5 ms of long pairs, then 107 of traceback; 118 side by side)
        p.trace_after_long = p.long_blocks2 > 0 && 16 * over_cells < cells16 &&
                             4 * kWaveShare * max_len * max_len < cells16;
    }
    if (n16 == 0) return p;
    Sw16Launch &k = p.p16;
    k.narrow = tune.sw16_narrow_rows;
    k.wide = n16 <= kWidePairs ? 1 : 0;
    k.lean = n16 <= kWidePairs / 2 ? 1 : 0;  // two pairs per wave: two waves per SIMD take them all
    // a block takes up to four pairs of the full-wave bins, eight or sixteen in
    // strips, of one sequence a; half as many where sequences have few partners
    const int64_t windows = (wide16 + 1) / 2 + (strips16 + (k.wide ? 1 : 3)) / (k.wide ? 2 : 4);
    const int scale = std::max(tune.sw_grid_scale, tune.sw_grid_scale_wide);
    k.blocks = (int)std::min<int64_t>((int64_t)kBlocks16 * (multi16 ? 1 : scale), std::max<int64_t>(windows, 1));
    k.multi_blocks = std::min(k.blocks, kBlocks16 * tune.sw_long_blocks / 4);
    p.t16 = k;
    // the traceback's list is thinner than pass 1's (large: 9 pairs of a family
    // share a sequence a where 43 candidates do), so windows of eight pairs
    // fill worse: strips of 32 lanes took 128 ms where those of 16 took 139
    p.t16.narrow = 0;
    p.t16.blocks = std::min(k.blocks, kBlocks16);
    p.t16.multi_blocks = multi16 ? std::min(p.t16.blocks, kTraceMultiBlocks) : 0;
    p.dirs_per_wave = dirs_of_wave(max_len);
    p.dirs_per_multi = dirs_of_multi(max_len);
    p.dirs_words =
        sw16_waves() * (p.t16.blocks * p.dirs_per_wave + p.t16.multi_blocks * p.dirs_per_multi);
    p.stats_after_trace = any32 || max_len > kTraceCols;
    return p;
}

hipError_t launch_sw(pastis_ctx *ctx, const uint8_t *codes, const PairDesc *pairs, int64_t npairs,
                     const int8_t *blosum, const Scoring &sc, SwPass1Out *p1, pastis_pair_record *out,
                     const SwWork &wk, int stats_mode, const SwPlan &plan, bool timed, hipStream_t s) {
    // timed = false (graph capture): no stage events
    const bool use16 = plan.max16 > 0;
    auto begin = [&](int st) { return timed ? stage_begin(ctx, st, s) : hipSuccess; };
    auto end = [&](int st) { return timed ? stage_end(ctx, st, s) : hipSuccess; };
    if (npairs <= 0) return hipSuccess;
    // The launches of a pass run beside one another: the multi-strip pairs on lane
    // 0 (those of single waves on lane 2 where others take blocks), the 16-bit kernel
    // (own, called as group -1) on lane 1, both off the call's stream, whose hardware
    // queue may be that of any lane; the one-strip groups on lane 2, the call's stream
    // and (1-8 rows per lane) where room is.  Those come before the 16-bit kernel on
    // its lane: its resident grid leaves later launches no room (statistics of
    // 250,000 sequences: the groups of 1-8 rows, 3 ms of work, lasted as long as the
    // traceback beside them, and both 150 ms; 137 with the groups first).  The long
    // pairs' blocks (kLongGroup) begin before all, as they need most of a CU's LDS
    // each: the others wait for an event of their lane, a few microseconds after
    // their launch.  Beside many multi-strip pairs in single waves it is the 16-bit
    // kernel that begins: either grid fills the chip, and pass 1 of 52,650 such pairs
    // and 5.5 million others takes 9.7 s with the 16-bit kernel first, up to 10.6
    // with the other.
    // run(phase, own, busy, f) calls f(group, stream) for every busy group and
    // orders its work after the call's stream's and before what follows on it.
    auto run = [&](int phase, bool own, auto &&busy, auto &&f) -> hipError_t {
        const bool blocks = busy(kLongGroup), waves = !blocks && own && busy(kMultiGroup);
        int job[kLongGroup + 2], n = 0;
        if (waves) job[n++] = -1;
        for (int g = kLongGroup; g >= 0; --g)
            if (busy(g)) job[n++] = g;
        if (own && !waves) job[n++] = -1;
        if (n == 0) return hipSuccess;
        if (n == 1) return f(job[0], s);  // alone: no fork
        hipError_t e = fork_acquire(ctx);
        if (e != hipSuccess || (e = hipEventRecord(ctx->fork_ev[phase], s)) != hipSuccess) return e;
        constexpr int kCall = kLanes;  // the call's stream
        const bool multi = blocks || busy(kMultiGroup);
        // (not in a capture, where the order of branches is the graph's: a wait for a
        // lane's event makes the waiting stream that lane's branch, and two passes led
        // by different lanes would make each lane a branch of the other, which ending
        // the capture follows without end)
        const bool lead = timed && (blocks || waves);
        const int first = waves ? 1 : 0;  // the leader's lane
        // lanes by group + 1.  In pass 1, where every group may be large, the groups of
        // 9-16 rows per lane share a lane (a search in 32-bit lanes 119 ms, 123 with a
        // lane each); later the groups of few rows make room for the traceback.
        const int lane_of[2][kLongGroup + 2] = {{1, own ? kCall : 1, kCall, 2, 2, blocks ? 2 : 0, 0},
                                                {1, waves ? kCall : 1, waves ? 2 : multi ? 1 : 0, kCall, 2, blocks ? 2 : 0, 0}};
        bool used[kLanes + 1] = {};
        // (a failed pass does not leave the lanes at work on the caller's inputs)
        auto fail = [&](hipError_t x) {
            for (int l = 0; l < kLanes; ++l)
                if (used[l]) (void)hipStreamSynchronize(ctx->lane[l]);
            return x;
        };
        for (int k = 0; k < n; ++k) {
            const int l = lane_of[phase > 0][job[k] + 1];
            hipStream_t st = l == kCall ? s : ctx->lane[l];
            const bool behind = lead && l != first;
            if (!used[l] && (behind || l != kCall) &&
                (e = hipStreamWaitEvent(st, behind ? ctx->lead_ev[phase] : ctx->fork_ev[phase], 0)) != hipSuccess)
                return fail(e);
            used[l] = true;
            if (job[k] < 0 && blocks && phase == 2 && plan.trace_after_long &&
                ((e = hipEventRecord(ctx->join_ev[phase][0], ctx->lane[0])) != hipSuccess ||
                 (e = hipStreamWaitEvent(st, ctx->join_ev[phase][0], 0)) != hipSuccess))
                return fail(e);
            if (lead && k == 0 && (e = hipEventRecord(ctx->lead_ev[phase], st)) != hipSuccess) return fail(e);
            if ((e = f(job[k], st)) != hipSuccess) return fail(e);
        }
        for (int l = 0; l < kLanes; ++l)
            if (used[l] && ((e = hipEventRecord(ctx->join_ev[phase][l], ctx->lane[l])) != hipSuccess ||
                            (e = hipStreamWaitEvent(s, ctx->join_ev[phase][l], 0)) != hipSuccess))
                return fail(e);
        return hipSuccess;
    };
    const int nb = (int)((npairs + 255) / 256);
    SwArgs A{};
    A.codes = codes;
    A.pairs = pairs;
    A.blosum = blosum;
    A.go_ge = sc.gap_open + sc.gap_extend;
    A.ge = sc.gap_extend;
    A.p1 = p1;
    A.rec = out;
    A.scratch = wk.scratch;
    A.scratch_per_wave = wk.scratch_per_wave;
    A.cov_pct = sc.cov_pct;
    A.id_pct = sc.id_pct;
    A.span = wk.counters + kCounterSpan;
    A.flag = wk.counters + kCounterIntraFlag;
    A.bounds = wk.bounds;
    hipError_t e = begin(kStSched);
    if (e != hipSuccess) return e;
    A.idx = wk.idx;
    A.starts = wk.starts;
    int *win = nullptr;
    if (use16) {
        // pair up pairs of one sequence a with similar column counts; the sort
        // by (bin, rows class, a) also bins the pairs
        sw_pair_keys_kernel<<<nb, 256, 0, s>>>(pairs, wk.bin_of, npairs, wk.sort_keys, (uint32_t *)wk.idx);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        bool alt = false;
        if ((e = radix_sort(wk.sort_keys, (uint32_t *)wk.idx, wk.sort_keys_alt, wk.sort_vals_alt, npairs,
                            kPairKeyBits, wk.sort_temp, s, &alt)) != hipSuccess)
            return e;
        if (alt) A.idx = (const int *)wk.sort_vals_alt;
        sw_bounds_kernel<<<1, 128, 0, s>>>(alt ? wk.sort_keys_alt : wk.sort_keys, (int)npairs, wk.bounds, wk.starts);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        win = alt ? wk.idx : (int *)wk.sort_vals_alt;  // the sort's other buffer
        A.win = win;
        A.nwin = wk.queue + kWindows1;
        if ((e = launch_sw16_windows(npairs, plan.p16, A, win, wk.queue + kWindows1, s)) != hipSuccess) return e;
    } else if ((e = launch_bins(wk.bin_of, npairs, kNumBins, wk.counts, wk.starts, wk.cursor, wk.idx, s)) !=
               hipSuccess) {
        return e;
    }
    if ((e = end(kStSched)) != hipSuccess || (e = begin(kStAlign1)) != hipSuccess) return e;
    // the 16-bit kernel runs beside the 32-bit groups
    e = run(0, plan.p16.blocks > 0,
            [&](int g) { return g == kLongGroup ? plan.long_blocks1 > 0 : plan.blocks32[g] > 0; },
            [&](int g, hipStream_t st) -> hipError_t {
                if (g < 0) {
                    SwArgs B = A;
                    B.queue = wk.queue;
                    B.scratch = wk.scratch16;
                    B.scratch_per_wave = wk.scratch16_per_wave;
                    return launch_sw16(false, plan.p16, B, st);
                }
                A.queue = wk.queue + 2 * kNumBins;
                if (g == kLongGroup) {
                    SwArgs B = A;
                    B.scratch = wk.long_scratch;
                    B.scratch_per_wave = plan.long_slot;
                    return launch_sw_long(false, plan.long_blocks1, plan.long_bins1, B, st);
                }
                if (g == kMultiGroup && plan.intra)
                    sw_intra_pass1_kernel<9, 16><<<kIntraBlocks, 64 * kIntraWaves, 0, st>>>(A, plan.bins32[g]);
                else
                    kPass1[g]<<<plan.blocks32[g], 64 * kGroupWpb[g], 0, st>>>(A, plan.bins32[g]);
                return hipGetLastError();
            });
    if (e != hipSuccess || (e = end(kStAlign1)) != hipSuccess || (e = begin(kStAlign2)) != hipSuccess) return e;
    const bool trace = wk.dirs != nullptr;
    const TraceRule T{trace ? plan.p16.bins : 0u, kTraceCols, kTraceColsMulti};
    const int *const idx1 = A.idx;  // pass 1's sorted items
    const bool forward = plan.forward_bound != 0;
    int *const bound_queue = wk.queue + 3 * kNumBins;  // claims, then the list's length
    // without a pair that the traceback refuses, only the forward bound uses bins
    const bool stats = !trace || plan.stats_after_trace;
    // a call of few pairs traces them all: the bound is as long as its longest
    // pair there (0.20 ms of 2.2 for 3,164 pairs, 63 of them bounded), and the
    // traceback no longer for a few pairs more
    const bool bound = stats_mode == 0 && (forward || stats || !plan.p16.wide);
    sw_bin2_kernel<<<nb, 256, 0, s>>>(pairs, p1, npairs, sc.cov_pct, stats_mode, bound ? sc.direct_pct : 0,
                                      forward ? 1 : 0, T, out, wk.bin_of, wk.idx2, bound_queue + 1, wk.counters);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (stats_mode == 2) return end(kStAlign2);  // every record is final
    A.idx = wk.idx2;
    A.starts = wk.starts2;
    A.queue = bound_queue;
    if (bound && forward) {
        // start bound, then only the pairs whose coverage can still hold
        if ((e = launch_bins(wk.bin_of, npairs, kNumBins, wk.counts, wk.starts2, wk.cursor, wk.idx2, s)) !=
            hipSuccess)
            return e;
        e = run(1, false, [&](int g) { return g < kGroups && plan.blocks_bound[g] > 0; },
                [&](int g, hipStream_t st) {
                    kBound[g]<<<plan.blocks_bound[g], 64 * kGroupWpb[g], 0, st>>>(A, kGroupBins[g]);
                    return hipGetLastError();
                });
        if (e != hipSuccess) return e;
        sw_bin3_kernel<<<nb, 256, 0, s>>>(pairs, p1, npairs, sc.cov_pct, T, out, wk.bin_of, wk.counters);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    } else if (bound) {
        if ((e = launch_sw16_bound(npairs, A, T, wk.bin_of, wk.counters, s)) != hipSuccess) return e;
    }
    if (stats && (e = launch_bins(wk.bin_of, npairs, kNumBins, wk.counts, wk.starts2, wk.cursor, wk.idx2, s)) !=
                     hipSuccess)
        return e;
    SwArgs B = A;  // the traceback's launches
    if (trace) {
        // the sort's keys are spent: their buffers hold the flags and the list,
        // and the scan
        uint8_t *flag = (uint8_t *)wk.sort_keys;
        int *list = (int *)(wk.sort_keys + (npairs + 1) / 2);
        uint32_t *pos = (uint32_t *)wk.sort_keys_alt;
        trace_flags_kernel<<<nb, 256, 0, s>>>(idx1, wk.bin_of, (int)npairs, flag);
        if ((e = exclusive_scan<uint8_t, uint32_t>(flag, npairs, pos, pos + npairs, wk.sort_temp, s)) != hipSuccess)
            return e;
        trace_list_kernel<<<nb, 256, 0, s>>>(idx1, flag, pos, (int)npairs, wk.bounds, list, wk.trace_bounds);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        B.idx = list;
        B.scratch = wk.scratch16;
        B.scratch_per_wave = wk.scratch16_per_wave;
        B.bounds = wk.trace_bounds;
        B.queue = wk.queue + 5 * kNumBins;
        B.nwin = wk.queue + kWindowsTrace;
        if ((e = launch_sw16_windows(npairs, plan.t16, B, win, wk.queue + kWindowsTrace, s)) != hipSuccess) return e;
        B.dirs_per_wave = plan.dirs_per_wave;
        B.dirs_per_multi = plan.dirs_per_multi;
        B.dirs = wk.dirs;
        B.dirs_multi = wk.dirs + sw16_waves() * plan.t16.blocks * plan.dirs_per_wave;
    }
    A.queue = wk.queue + 4 * kNumBins;
    e = run(2, trace,
            [&](int g) {
                return stats && (g == kLongGroup ? plan.long_blocks2 > 0 : plan.blocks_stats[g] > 0);
            },
            [&](int g, hipStream_t st) -> hipError_t {
                if (g < 0) return launch_sw16(true, plan.t16, B, st);
                if (g == kLongGroup) {
                    SwArgs C = A;
                    C.scratch = wk.long_scratch;
                    C.scratch_per_wave = plan.long_slot;
                    return launch_sw_long(true, plan.long_blocks2, plan.long_bins2, C, st);
                }
                kStats[g]<<<plan.blocks_stats[g], 64 * kGroupWpb[g], 0, st>>>(A, kGroupBins[g] & ~plan.long_bins2);
                return hipGetLastError();
            });
    if (e != hipSuccess) return e;
    return end(kStAlign2);
}

}  // namespace pastis
