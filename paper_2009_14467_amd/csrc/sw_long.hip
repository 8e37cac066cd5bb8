// Smith-Waterman of long pairs in 32-bit lanes, one workgroup per pair: pass 1
// and the statistics by checkpointed traceback.
#include <algorithm>

#include "sw_long.hpp"

namespace pastis {
namespace {

// A few pairs of tens of thousands of rows are as long as the slowest of them
// takes: in one wave, strip after strip, 25,000 x 25,000 cells took 245 ms in
// pass 1 and 442 with the statistics carried along.  Here the eight waves of a
// block work on one pair.  Wave w takes strips w, w + 8, ... of 512 rows (8 per
// lane: 102 KB of profiles per block, one block and two waves per SIMD on a CU),
// so eight strips run at once, each a little behind the one above.  Every strip
// leaves its bottom row (H and F' of every column) in a row buffer of its own in
// global memory; prog[s] counts the columns that strip s has written, and strip
// s + 1 waits for it 64 columns at a time.  Every wait is for an earlier strip,
// so the earliest unfinished strip never waits and the pipeline drains; each
// wait is also bounded, and one that runs out sets *flag and gives up (the call
// then fails).
//
// Statistics.  The forward sweep over the end rectangle also leaves, every
// kLongTile steps, the state of every lane (H, E of its rows and the two words
// on their way down).  The walk back from the end cell then needs direction
// bits along its path only: wave 0 repeats one tile of a strip at a time, from
// the state at the tile's begin and the row above, files the four bits of
// every cell (as the traceback in 16-bit lanes does) and walks until it leaves
// the tile.  A path visits about two tiles per strip, so the statistics cost
// little more than a second pass 1 where carrying them along costs 2.5.
//
// 1,225 pairs of 3,000 to 25,000 rows take 149 ms in pass 1 and 118 with
// statistics.  Bound by the instructions of two waves per SIMD (the profiles'
// LDS) and, in the statistics of few pairs, by the longest pair.
constexpr int kLongR = 8, kLongWaves = 8, kLongRows = kWave * kLongR;
constexpr int kLongTile = 512;  // steps
constexpr int kLongStrips = (65536 + kLongRows - 1) / kLongRows;
constexpr int kLongState = 2 * kLongR + 2;  // words of a lane's state

struct LongLds {
    int8_t sblosum[kProfCodes * kProfCodes];
    int prog[kLongStrips];
    unsigned long long best[kLongWaves];
    int take, end_b;
};

// One pair's work and its place in the block's slot of scratch memory.
struct LongPair {
    const uint8_t *a, *b;
    int rows, cols;   // the rectangle
    int end_a, score; // find: the end column is sought where row end_a holds the score
    bool find;
    int snaps;        // states per strip
    int *slot;
    __device__ int *row_h(int s) const { return slot + (int64_t)s * 2 * cols; }
    __device__ int *state(int s, int k) const {
        const int64_t strips = (rows + kLongRows - 1) / kLongRows;
        return slot + strips * 2 * cols + ((int64_t)s * snaps + k) * (kWave * kLongState);
    }
    __device__ int *tile() const { return state((rows + kLongRows - 1) / kLongRows, 0); }
};

enum LongMode { kPass1, kForward, kTile };

// Steps [t0, t1) of strip s by the calling wave.  kPass1: best gets the
// maximum, (score << 32) | ~(row << 16 | column); kForward: states and (find)
// the end column; kTile: direction words of the steps, one per lane, from t0 (a
// multiple of kLongTile) and the state filed there.
template <LongMode MODE>
__device__ __forceinline__ void long_strip(const LongPair &P, int s, int t0, int t1, ProfWord<kLongR> (*prof)[kWave],
                                           LongLds &L, int go_ge, int ge, bool &ok, unsigned long long &best) {
    constexpr int R = kLongR;
    const int lane = threadIdx.x & (kWave - 1);
    const int base = s * kLongRows + lane * R;
    const bool from_above = s > 0, to_below = MODE != kTile && (s + 1) * kLongRows < P.rows;
    const int cols = P.cols;
    build_profile<R>(prof, L.sblosum, P.a, P.rows, base, lane);
    __builtin_amdgcn_wave_barrier();
    int *const out_h = P.row_h(s), *const out_f = out_h + cols;
    const int *const in_h = P.row_h(max(s - 1, 0)), *const in_f = in_h + cols;
    int H[R], G[R], E[R], rmax[MODE == kPass1 ? R : 1], rcol[MODE == kPass1 ? R : 1];
    int flast = 0, hprev = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        H[r] = 0;
        E[r] = 0;
        if constexpr (MODE == kPass1) rmax[r] = rcol[r] = 0;
    }
    if (MODE == kTile && t0 > 0) {
        const int *st = P.state(s, t0 / kLongTile) + lane;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            H[r] = vload(st + (2 * r) * kWave);
            E[r] = vload(st + (2 * r + 1) * kWave);
        }
        flast = vload(st + (2 * R) * kWave);
        hprev = vload(st + (2 * R + 1) * kWave);
    }
#pragma unroll
    for (int r = 0; r < R; ++r) G[r] = H[r] - go_ge;
    int hlast = H[R - 1];
    auto col = [&](int c) { return c >= 0 && c < cols ? (int)P.b[c] : kPadCode; };
    int cres = col(t0 - 1 - lane), chunk = 0, nx = col(t0 + lane);
    int ch_h = 0, ch_f = 0;
    // the row that holds the end cell, if this lane does
    const int re = P.end_a - base;
    bool need = MODE == kForward && P.find && re >= 0 && re < R;
    for (int t = t0; t < t1; ++t) {
        if ((t & (kWave - 1)) == 0) {
            chunk = nx;
            nx = col(t + kWave + lane);
            if (from_above && t < cols) {
                if (MODE != kTile && ok && !lds_wait(&L.prog[s - 1], min(t + kWave, cols))) ok = false;
                const int c = t + lane;
                ch_h = c < cols ? vload(in_h + c) : 0;
                ch_f = c < cols ? vload(in_f + c) : 0;
            } else {
                ch_h = ch_f = 0;
            }
            if (MODE == kForward && t > 0 && t % kLongTile == 0) {
                int *st = P.state(s, t / kLongTile) + lane;
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    st[(2 * r) * kWave] = H[r];
                    st[(2 * r + 1) * kWave] = E[r];
                }
                st[(2 * R) * kWave] = flast;
                st[(2 * R + 1) * kWave] = hprev;
            }
        }
        const int x = t & (kWave - 1);
        const int rh = shr1(__builtin_amdgcn_readlane(ch_h, x), hlast);
        const int rf = shr1(__builtin_amdgcn_readlane(ch_f, x), flast);
        cres = shr1(__builtin_amdgcn_readlane(chunk, x), cres);
        const ProfWord<R> pw = prof[cres][lane];
        const int j = t - lane;
        int hd = hprev, gu = rh - go_ge, fu = rf;
        uint32_t bits = 0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int ex = subs(E[r], ge), fx = subs(fu, ge);
            const int e = max(ex, G[r]), f = max(fx, gu);
            const int d = hd + sigma_at<R>(pw, r);
            const int m = max(e, f), h = max(d, m);
            if constexpr (MODE == kTile) {
                bits |= (d < m ? 1u : 0u) << r;           // not the diagonal
                bits |= (e < f ? 0x100u : 0u) << r;       // the vertical gap
                bits |= (ex < G[r] ? 0x10000u : 0u) << r; // e was opened
                bits |= (fx < gu ? 0x1000000u : 0u) << r; // f was opened
            }
            hd = H[r];
            H[r] = h;
            E[r] = e;
            G[r] = h - go_ge;
            gu = G[r];
            fu = f;
            if constexpr (MODE == kPass1) {
                if (h > rmax[r] && j < cols) {
                    rmax[r] = h;
                    rcol[r] = j;
                }
            }
        }
        hlast = H[R - 1];
        flast = fu;
        hprev = rh;
        if constexpr (MODE == kTile) P.tile()[(t - t0) * kWave + lane] = (int)bits;
        if constexpr (MODE == kForward) {
            if (need && j >= 0) {
                int h = H[0];
#pragma unroll
                for (int r = 1; r < R; ++r) h = re == r ? H[r] : h;
                if (h == P.score) {
                    L.end_b = j;
                    need = false;
                }
            }
        }
        const int jw = t - (kWave - 1);  // lane 63's column
        if (to_below && jw >= 0 && jw < cols && lane == kWave - 1) {
            out_h[jw] = hlast;
            out_f[jw] = flast;
            if ((jw & (kWave - 1)) == kWave - 1 || jw == cols - 1) lds_release(&L.prog[s], jw + 1);
        }
    }
    if constexpr (MODE == kPass1) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int row = base + r;
            if (row < P.rows && rmax[r] > 0) {
                const unsigned pos = ((unsigned)row << 16) | (unsigned)rcol[r];
                const unsigned long long k = ((unsigned long long)(unsigned)rmax[r] << 32) | (unsigned)(~pos);
                best = k > best ? k : best;
            }
        }
    }
}

// Walks back from cell (i, j) of value h, repeating the tiles on the way (one
// wave; see walk_back of the 16-bit lanes for the run of diagonal steps).
__device__ __forceinline__ void long_walk(const LongPair &P, int &i, int &j, int h, int &matches, int &diag,
                                          ProfWord<kLongR> (*prof)[kWave], LongLds &L, int go_ge, int ge) {
    constexpr int R = kLongR;
    const int lane = threadIdx.x & (kWave - 1);
    int state = 0;  // 0: H, 1: horizontal gap, 2: vertical gap
    bool done = i < 0 || j < 0;
    while (!done) {
        const int s = i / kLongRows, base = s * kLongRows;
        const int t = j + (i - base) / R, t0 = t / kLongTile * kLongTile;
        bool ok = true;
        unsigned long long none = 0;
        long_strip<kTile>(P, s, t0, t + 1, prof, L, go_ge, ge, ok, none);
        __threadfence_block();
        const int *tile = P.tile();
        // the direction word of a cell of the tile, shifted to its row's bits
        auto step_of = [&](int x, int y) { return y + (x - base) / R; };
        auto bits_at = [&](int x, int y) {
            return (uint32_t)vload(tile + (step_of(x, y) - t0) * kWave + (x - base) / R) >> ((x - base) % R);
        };
        while (!done && i >= base && step_of(i, j) >= t0) {
            if (state == 0) {
                const int x = i - lane, y = j - lane;
                bool stop = true, match = false;
                int sum = 0;
                const bool in = x >= base && y >= 0 && step_of(x, y) >= t0;
                if (in) {
                    stop = (bits_at(x, y) & 1u) != 0;
                    const int ca = P.a[x], cb = P.b[y];
                    match = ca == cb;
                    sum = L.sblosum[ca * kProfCodes + cb];
                }
                const unsigned long long stops = __ballot(stop), inside = __ballot(in);
                const int run = stops ? __ffsll((long long)stops) - 1 : kWave;
#pragma unroll
                for (int d = 1; d < kWave; d <<= 1) {
                    const int o = __shfl_up(sum, d, kWave);
                    sum += lane >= d ? o : 0;
                }
                const unsigned long long zero = __ballot(lane < run && h == sum);
                const int n = zero ? __ffsll((long long)zero) : run;  // diagonal cells taken
                const unsigned long long taken = n >= 64 ? ~0ull : (1ull << n) - 1ull;
                diag += n;
                matches += __popcll(__ballot(match) & taken);
                if (zero) {  // the path starts at the last of them
                    i -= n - 1;
                    j -= n - 1;
                    done = true;
                    break;
                }
                h -= n > 0 ? __shfl(sum, max(n - 1, 0), kWave) : 0;
                i -= n;
                j -= n;
                // the run ended at the tile's edge, or at a cell that is not diagonal
                if (n == kWave || !((inside >> n) & 1ull)) {
                    done = i < 0 || j < 0;
                    continue;
                }
                state = (bits_at(i, j) & 0x100u) ? 2 : 1;
            }
            const bool opened = (bits_at(i, j) & (state == 1 ? 0x10000u : 0x1000000u)) != 0;
            h += opened ? go_ge : ge;
            if (state == 1)
                --j;
            else
                --i;
            if (opened) state = 0;
            done = i < 0 || j < 0;
        }
        i = __builtin_amdgcn_readfirstlane(i);
        j = __builtin_amdgcn_readfirstlane(j);
    }
}

template <bool STATS>
__global__ __launch_bounds__(kWave *kLongWaves, 2) void sw_long_kernel(SwArgs A, uint32_t bins) {
    __shared__ __align__(16) char lds[kLongWaves * kProfCodes * kWave * sizeof(ProfWord<kLongR>)];
    __shared__ LongLds L;
    load_blosum(L.sblosum, A.blosum);
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    auto *prof = (ProfWord<kLongR>(*)[kWave])(lds + (size_t)wave * (kProfCodes * kWave * sizeof(ProfWord<kLongR>)));
    for (int bin = kNumBins - 1; bin >= 0; --bin) {
        if (!((bins >> bin) & 1u)) continue;
        const unsigned long long t_begin = span_now();
        bool any = false;
        for (;;) {
            if (threadIdx.x == 0) L.take = atomicAdd(A.queue + bin, 1);
            __syncthreads();
            const int64_t w = A.starts[bin] + (int64_t)__builtin_amdgcn_readfirstlane(L.take);
            __syncthreads();  // every wave has read it before the next claim
            if (w >= A.starts[bin + 1]) break;
            any = true;
            const int q = A.idx[w];
            const PairDesc pd = A.pairs[q];
            SwPass1Out r1{};
            if constexpr (STATS) r1 = A.p1[q];
            LongPair P;
            P.a = A.codes + pd.a_off;
            P.b = A.codes + pd.b_off;
            P.find = STATS && r1.end_b < 0;
            P.rows = STATS ? r1.end_a + 1 : pd.la;
            P.cols = STATS && r1.end_b >= 0 ? r1.end_b + 1 : pd.lb;
            P.end_a = r1.end_a;
            P.score = r1.score;
            P.snaps = (P.cols + kWave) / kLongTile + 1;
            P.slot = A.scratch + (int64_t)blockIdx.x * A.scratch_per_wave;
            const int strips = P.cols > 0 ? (P.rows + kLongRows - 1) / kLongRows : 0;
            for (int x = threadIdx.x; x < strips; x += blockDim.x) L.prog[x] = 0;
            if (threadIdx.x == 0) L.end_b = r1.end_b;
            __syncthreads();
            unsigned long long best = 0;
            bool ok = true;
            for (int s = wave; s < strips; s += kLongWaves)
                long_strip<STATS ? kForward : kPass1>(P, s, 0, P.cols + kWave - 1, prof, L, A.go_ge, A.ge, ok, best);
            if (!ok && lane == 0) atomicOr(A.flag, 1ull);
            if constexpr (!STATS) {
                best = wave_max_u64(best);
                if (lane == 0) L.best[wave] = best;
            }
            __threadfence_block();
            __syncthreads();
            if constexpr (STATS) {
                if (wave == 0) {
                    const int end_b = __builtin_amdgcn_readfirstlane(L.end_b);
                    int i = r1.end_a, j = end_b, matches = 0, diag = 0;
                    long_walk(P, i, j, r1.score, matches, diag, prof, L, A.go_ge, A.ge);
                    if (lane == 0) {
                        pastis_pair_record rec;
                        rec.score = r1.score;
                        rec.end_a = r1.end_a;
                        rec.end_b = end_b;
                        rec.beg_a = i;
                        rec.beg_b = j;
                        rec.matches = matches;
                        rec.columns = (r1.end_a - i + 1) + (end_b - j + 1) - diag;
                        rec.seed_used = -1;
                        const long long span = (long long)r1.end_a - i + 1;
                        rec.passed = (100LL * rec.matches >= (long long)A.id_pct * rec.columns) &&
                                     (100LL * span >= (long long)A.cov_pct * pd.la);
                        rec.swapped = pd.swapped;
                        rec.cells = (int64_t)pd.la * pd.lb;
                        A.rec[q] = rec;
                    }
                }
            } else if (threadIdx.x == 0) {
                unsigned long long m = 0;
                for (int k = 0; k < kLongWaves; ++k) m = L.best[k] > m ? L.best[k] : m;
                SwPass1Out o;
                o.score = (int32_t)(m >> 32);
                const unsigned pos = ~(unsigned)m;
                o.end_a = o.score > 0 ? (int32_t)(pos >> 16) : -1;
                o.end_b = o.score > 0 ? (int32_t)(pos & 0xFFFF) : -1;
                o.pad = 0;
                A.p1[q] = o;
            }
            __syncthreads();
        }
        if (!STATS && any) span_add(A.span + 2 * bin, t_begin);
    }
}

}  // namespace

int64_t sw_long_slot_words(int max_len) {
    const int64_t n = std::max(max_len, 1), strips = (n + kLongRows - 1) / kLongRows;
    const int64_t snaps = (n + kWave) / kLongTile + 1;
    return strips * 2 * n + strips * snaps * (kWave * kLongState) + kLongTile * kWave;
}

hipError_t launch_sw_long(bool stats, int blocks, uint32_t bins, const SwArgs &A, hipStream_t s) {
    if (stats)
        sw_long_kernel<true><<<blocks, kWave * kLongWaves, 0, s>>>(A, bins);
    else
        sw_long_kernel<false><<<blocks, kWave * kLongWaves, 0, s>>>(A, bins);
    return hipGetLastError();
}

}  // namespace pastis
