// Smith-Waterman in 16-bit lanes: two pairs in the halves of every DP word.
#include <algorithm>
#include <climits>

#include "sw16.hpp"
#include "walk_reach.hpp"

namespace pastis {
namespace {

// Two pairs per wave in the 16-bit halves of every DP word (pair P low, Q
// high), same lane layout as the 32-bit pass, in strips of up to 16 rows per lane
// (one strip, or up to three for sequences a of 1,025 to 2,978 rows).  The two
// pairs share their shorter sequence a (pairs are sorted by bin, then a, then
// the longer b first), so one int8 profile serves both (see the windows below;
// items that share the sort key's 24 bits of a but differ in a run one after
// the other).  Only G = H - (o + e) is
// kept per row: the diagonal term H(i-1, j-1) + s becomes G(i-1, j-1) +
// (s + o + e), with the biased scores s + o + e >= 0 in the profile (each
// row's two bytes are spread into the halves by one byte permute).  Padding
// residues score -(o + e).  Each row keeps only its maximum: cells outside a
// pair (padding rows and columns, columns before the first) score strictly
// below its best real cell, so the score and the first row holding it are
// exact; the end column is found later, for the pairs that need it (end_b
// holds a hint here, see hint_code).  A row gains at most 11, so scores stay within
// 11 * 2,978 = 32,758, nine below the 16-bit limit.
// The gap states are kept floored at zero, E' = max(E, 0) and F' = max(F, 0):
// their recurrences stay closed (max(E' - e, 0) = max(E - e, 0) for e >= 0,
// one saturating subtract), and max(d, E', F') then already holds the local
// alignment's zero, so a cell takes 10 packed ops instead of 11.
constexpr int kMax16R = kMaxR;
// (also the limit of the differences whose signs are the traceback's bits: their
// terms are at least -(o + e), and a gap's value is o + e below some cell's)
static_assert(11 * kMax16Rows <= 32767, "scores of 16-bit pairs stay below 2^15");

typedef short short2_t __attribute__((ext_vector_type(2)));
typedef unsigned short ushort2_t __attribute__((ext_vector_type(2)));

__device__ __forceinline__ short2_t s2(uint32_t x) { return __builtin_bit_cast(short2_t, x); }
// max(x - y, 0) per half, for 0 <= x < 2^15
__device__ __forceinline__ short2_t psubs(short2_t x, uint32_t y) {
    return __builtin_bit_cast(short2_t, __builtin_elementwise_sub_sat(__builtin_bit_cast(ushort2_t, x),
                                                                      __builtin_bit_cast(ushort2_t, y)));
}
__device__ __forceinline__ uint32_t u2(short2_t x) { return __builtin_bit_cast(uint32_t, x); }
__device__ __forceinline__ short2_t pmax(short2_t a, short2_t b) { return __builtin_elementwise_max(a, b); }
__device__ __forceinline__ int shr1u(uint32_t lane0, uint32_t v) { return shr1((int)lane0, (int)v); }

// 16-bit profile: entry [c][p] holds the biased scores s + o + e >= 0 (pad
// rows: 0) of rows p * RP .. p * RP + RP - 1 of a against code c, one byte
// each.  The calling thread writes the codes c = group (mod NG) for position
// pos; NG groups of threads together cover all codes.
template <int RP, int W, int NG>
__device__ __forceinline__ void build_profile16(ProfWord<RP> (*prof)[W], const int8_t *sblosum, const uint8_t *a,
                                                int la, int pos, int group, int oe) {
    int ar[RP];
#pragma unroll
    for (int r = 0; r < RP; ++r) ar[r] = (pos * RP + r < la) ? a[pos * RP + r] : kPadCode;
    for (int c = group; c < kProfCodes; c += NG) {
        uint32_t w[4] = {0, 0, 0, 0};
#pragma unroll
        for (int r = 0; r < RP; ++r) {
            const int sc = max((int)sblosum[ar[r] * kProfCodes + c], -oe) + oe;
            w[r >> 2] |= (uint32_t)sc << (8 * (r & 3));
        }
        prof[c][pos] = make_word<RP>(w);
    }
}

template <int R>
__device__ __forceinline__ uint32_t prof_word(const ProfWord<R> &w, int r) {
    return word_of<R>(w, r >> 2);
}

__device__ __forceinline__ unsigned wave_max_u32(unsigned v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = max(v, (unsigned)__shfl_xor((int)v, off, kWave));
    return v;
}


__device__ __forceinline__ int wave_min_i32(int v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = min(v, __shfl_xor(v, off, kWave));
    return v;
}

__device__ __forceinline__ int wave_max_i32(int v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = max(v, __shfl_xor(v, off, kWave));
    return v;
}

// ---------------------------------------------------------------- traceback
//
// The statistics of a pair that can still pass the cut (begin, matches,
// columns of the canonical alignment) come from a traceback.  The forward
// sweep is pass 1's, with four direction bits per cell in place of the row
// maxima:
//   A  h != d          (else the diagonal, which wins ties)
//   B  f > e           (else the horizontal gap, which wins over the vertical)
//   C  e was opened    (else extended, which wins ties)
//   D  f was opened
// On the path every state's value is positive, where the floored recurrences
// compare exactly as the unfloored ones.  The differences d - (e or f), e - f,
// ... carry the bits in their signs; a byte permute spreads two differences'
// signs (both pairs) to bytes of ones or zeros and a bit-select by a constant
// files them under the row, eight ops for the four bits of two cells.  A cell
// costs 8.5 ops where carrying the statistics along costs 27, and the bits of
// a step leave as 4, 8, 12 or 16 contiguous bytes per lane (half a byte per
// cell).  The walk then goes back from the end cell: a group of S / 2 lanes per
// pair fetches the bits of at least 16 rows (9 in the wider bins) over at
// least 16 columns at a time, so a pair waits for memory once per fetch instead of once per
// cell, and knows its value h at every cell, which is how it finds the begin
// (the diagonal predecessor's h is 0).
//
// Word k of a lane's step holds its rows 4 k .. 4 k + 3 in bits 0..3 of each
// byte and their C / D bits in bits 4..7: bytes 0 and 1 are pair P's (A | C,
// B | D), bytes 2 and 3 pair Q's.
template <int RP>
constexpr int dir_words() {
    return (RP + 3) / 4;
}

template <int NW>
__device__ __forceinline__ void store_dirs(uint32_t *p, const uint32_t (&w)[NW]) {
    if constexpr (NW == 1) {
        *p = w[0];
    } else if constexpr (NW == 2) {
        *(uint2 *)p = make_uint2(w[0], w[1]);
    } else if constexpr (NW == 3) {
        *(uint3 *)p = make_uint3(w[0], w[1], w[2]);
    } else {
        *(uint4 *)p = make_uint4(w[0], w[1], w[2], w[3]);
    }
}

// files the direction bits of row r (d, e, f: the row's candidates; x, y: the
// extended gaps; g, gu: the opened ones)
template <int NW>
__device__ __forceinline__ void file_dirs(uint32_t (&w)[NW], int r, short2_t d, short2_t m, short2_t e, short2_t f,
                                          short2_t x, short2_t g, short2_t y, short2_t gu) {
    // selectors 8 / 9 and 10 / 11 spread the sign bits of the second and the
    // first operand's halves
    const uint32_t ab = __builtin_amdgcn_perm(u2(d - m), u2(e - f), 0x090B080Au);
    const uint32_t cd = __builtin_amdgcn_perm(u2(x - g), u2(y - gu), 0x090B080Au);
    const uint32_t k1 = 0x01010101u << (r & 3), k2 = 0x10101010u << (r & 3);
    uint32_t v = w[r >> 2];
    v = (ab & k1) | (v & ~k1);
    v = (cd & k2) | (v & ~k2);
    w[r >> 2] = v;
}

// A walk's fetch: the bits of kSlots lanes' rows (at least 16 rows where a
// strip has one piece) over kCols columns.
template <int S, int RP, bool MULTI>
struct WalkShape {
    static constexpr int W = S / 2;  // lanes of the group
    static constexpr int kSlots = walk_slots(RP, MULTI);
    static constexpr int kCols = walk_cols(W);
    static constexpr int kRows = kSlots * RP;
    static constexpr int NW = dir_words<RP>();
    struct Lds {
        uint32_t dir[kCols][kSlots * NW];
        uint8_t b[kCols];
        uint8_t a[(kRows + 3) / 4 * 4];
    };
};

struct Walk {
    int i, j;        // the end cell, then the begin cell
    int h;           // the end cell's score
    int matches = 0, diag = 0;
};

// Walks one pair back from its end cell.  The calling lanes are a group of W =
// S / 2 (lane `sub` of it) that share the pair and the LDS area; slot0 is the
// wave lane of the pair's row block 0, half its half of the words, dirs the
// wave's direction words and strip_words the distance between strips.  A run of
// diagonal steps is taken at once: lane k looks at the k-th cell up the
// diagonal, a ballot ends the run at the first cell that is not diagonal, and a
// prefix sum of the scores finds the begin (h falls to 0); gap cells go one by
// one.
template <int S, int RP, bool MULTI>
__device__ __forceinline__ void walk_back(Walk &P, bool act, const uint32_t *dirs, int64_t strip_words,
                                          const uint8_t *__restrict__ a, int la, const uint8_t *__restrict__ b,
                                          int slot0, int half, int sub,
                                          typename WalkShape<S, RP, MULTI>::Lds &L, const int8_t *sblosum, int go_ge,
                                          int ge) {
    using T = WalkShape<S, RP, MULTI>;
    constexpr int W = T::W, NW = T::NW;
    const int g0 = (int)(threadIdx.x & (kWave - 1)) - sub;  // the group's first lane
    const unsigned long long gmask = W == 64 ? ~0ull : (1ull << W) - 1ull;
    int i = P.i, j = P.j, h = P.h, state = 0;  // 0: H, 1: horizontal gap, 2: vertical gap
    bool done = !act || i < 0 || j < 0;
    while (!done) {
        const int blk = i / RP, j0 = j;
        const int p = MULTI ? blk % kWave : blk;
        const int pb = p - (T::kSlots - 1);               // first slot fetched (may be negative)
        const int r0 = walk_first_row(blk, RP, T::kSlots);  // its first row (so may this)
        const uint32_t *src = dirs + (MULTI ? (blk / kWave) * strip_words : 0);
#pragma unroll
        for (int m = 0; m < T::kCols / W; ++m) {
            const int c = m * W + sub, col = j0 - c;
            if (col < 0) continue;
#pragma unroll
            for (int k = 0; k < T::kSlots; ++k) {
                if (pb + k < 0) continue;
                const uint32_t *w = src + (int64_t)(col + pb + k) * (kWave * NW) + (slot0 + pb + k) * NW;
#pragma unroll
                for (int x = 0; x < NW; ++x) L.dir[c][k * NW + x] = vload(w + x);
            }
            L.b[c] = b[col];
        }
        for (int r = sub; r < T::kRows; r += W)
            if (walk_holds_row(r0, r, la)) L.a[r] = a[r0 + r];
        __builtin_amdgcn_wave_barrier();
        int r = i - r0, c = 0;
        const int cend = min(T::kCols, j0 + 1);
        auto bits_at = [&](int rr, int cc) {
            const int s = rr / RP, x = rr % RP;
            return L.dir[cc][s * NW + (x >> 2)] >> ((x & 3) + 16 * half);
        };
        while (r >= 0 && c < cend && !done) {
            if (state == 0) {
                const int rr = r - sub, cc = c + sub;
                bool stop = true, match = false;
                int sum = 0;
                if (walk_reads(r0, rr, cc, cend)) {
                    stop = (bits_at(rr, cc) & 1u) != 0;
                    const int ca = L.a[rr], cb = L.b[cc];
                    match = ca == cb;
                    sum = sblosum[ca * kProfCodes + cb];
                }
                const unsigned long long stops = (__ballot(stop) >> g0) & gmask;
                const int run = stops ? __ffsll((long long)stops) - 1 : W;
#pragma unroll
                for (int d = 1; d < W; d <<= 1) {
                    const int o = __shfl_up(sum, d, W);
                    sum += sub >= d ? o : 0;
                }
                const unsigned long long zero = (__ballot(sub < run && h == sum) >> g0) & gmask;
                const int n = zero ? __ffsll((long long)zero) : run;  // diagonal cells taken
                const unsigned long long taken = n >= 64 ? ~0ull : (1ull << n) - 1ull;
                P.diag += n;
                P.matches += __popcll((__ballot(match) >> g0) & taken);
                if (zero) {  // the path starts at the last of them
                    r -= n - 1;
                    c += n - 1;
                    done = true;
                    break;
                }
                const int back = __shfl(sum, max(n - 1, 0), W);
                h -= n > 0 ? back : 0;
                r -= n;
                c += n;
                // the run ended inside the fetch: at a cell that is not diagonal
                if (n == W || r < 0 || c >= cend) continue;
                state = (bits_at(r, c) & 0x100u) ? 2 : 1;
            }
            const bool opened = (bits_at(r, c) & (state == 1 ? 0x10u : 0x1000u)) != 0;
            h += opened ? go_ge : ge;
            if (state == 1)
                ++c;
            else
                --r;
            if (opened) state = 0;
        }
        i = r0 + r;
        j = j0 - c;
        done = done || i < 0 || j < 0;
        __builtin_amdgcn_wave_barrier();
    }
    P.i = i;
    P.j = j;
}

// the record of a walked pair (its descriptor is read again rather than kept
// in registers through the sweep)
__device__ __forceinline__ void walk_record(const SwArgs &A, const Walk &P, int score, int end_a, int end_b, int q) {
    const PairDesc pd = A.pairs[q];
    pastis_pair_record rec;
    rec.score = score;
    rec.end_a = end_a;
    rec.end_b = end_b;
    rec.beg_a = P.i;
    rec.beg_b = P.j;
    rec.matches = P.matches;
    rec.columns = (end_a - P.i + 1) + (end_b - P.j + 1) - P.diag;
    rec.seed_used = -1;
    const long long span = (long long)end_a - P.i + 1;
    rec.passed = (100LL * rec.matches >= (long long)A.id_pct * rec.columns) &&
                 (100LL * span >= (long long)A.cov_pct * pd.la);
    rec.swapped = pd.swapped;
    rec.cells = (int64_t)pd.la * pd.lb;
    A.rec[q] = rec;
}

// Pass 1's hint at a pair's end column: the first column the end row can
// reach its maximum in.  Every 16 steps a lane compares the maximum over its
// rows with the one 16 steps before; the last change marks the 16 steps in
// which the lane first reached its final maximum, which no later column can
// precede.  Kept per half (pair), in units of 16 steps.
template <int RP>
__device__ __forceinline__ void note_rise(const uint32_t (&M)[RP], uint32_t &seen, uint32_t &when, int chunk) {
    uint32_t m = M[0];
#pragma unroll
    for (int r = 1; r < RP; ++r) m = u2(pmax(s2(m), s2(M[r])));
    const uint32_t diff = m ^ seen;
    seen = m;
    const uint32_t mask = ((diff & 0xFFFFu) ? 0xFFFFu : 0u) | ((diff >> 16) ? 0xFFFF0000u : 0u);
    when = (when & ~mask) | (((uint32_t)chunk * 0x10001u) & mask);
}

// Full-wave layout for the wider bins.  A block takes 2 * WPB consecutive
// pairs (two per wave) and its waves share one profile, built once per
// distinct sequence a among them (pairs are sorted by a), so the LDS of a
// block does not grow with its wave count.  MULTI: sequences a of more than
// 1024 rows (and at most kMax16Rows, so that scores stay below 2^15) run in
// strips of 64 R rows, one after the other; lane 63 leaves the G and F' words
// of the strip's bottom row for every column in a per-wave buffer, and lane 0
// reads them back as the top boundary of the next strip.
template <int WPB>
struct WaveLds {
    // first unfinished pair of each wave, double-buffered by round parity so
    // that a round's writes never meet the previous round's reads
    int next[2][WPB];
    int take;  // the block's window, claimed from the bin's queue
};

// Windows.  What a block or wave takes at once shares sequence a: a sequence's
// pairs (neighbours in the sorted list) are cut into windows of `width` pairs,
// so that none straddles two sequences.  (Windows at multiples of the width
// did, and ran their sequences one after the other: with ten partners per
// sequence pass 1 of 10,000 sequences took 5.8 ms, its last tall window 5.2 of
// them, and takes 4.6 so; with 43, 534 ms of 250,000 sequences are 511.)  The order of a class's windows is that of the list up to blocks of 1,024
// items.  Sequences count as one if they agree in the 24 bits that the list is
// sorted by; the kernels check a_seq itself.
constexpr int kClasses = 2 * kNumBins, kWindowBlock = 1024;
__device__ __forceinline__ bool same_seq24(int x, int y) { return ((x ^ y) & 0xFFFFFF) == 0; }

__global__ __launch_bounds__(kWindowBlock) void sw16_windows_kernel(const PairDesc *__restrict__ pairs,
                                                                    const int *__restrict__ idx,
                                                                    const int *__restrict__ bounds, Sw16Launch P,
                                                                    int *__restrict__ win, int *__restrict__ nwin) {
    __shared__ int sb[kClasses + 1], count[kClasses], base[kClasses], seq[kWindowBlock];
    const int tid = threadIdx.x, i0 = blockIdx.x * kWindowBlock, i = i0 + tid;
    const int n = bounds[kClasses];
    if (i0 >= n) return;
    if (tid <= kClasses) sb[tid] = bounds[tid];
    if (tid < kClasses) count[tid] = 0;
    const int a = i < n ? pairs[idx[i]].a_seq : 0;
    seq[tid] = a;
    __syncthreads();
    int cls = 0, rank = -1;
    if (i < n) {
        int hi = kClasses;  // the last class that begins at or before i
        while (cls < hi) {
            const int mid = (cls + hi + 1) / 2;
            if (sb[mid] <= i)
                cls = mid;
            else
                hi = mid - 1;
        }
        auto same = [&](int x) { return same_seq24(x >= i0 ? seq[x - i0] : pairs[idx[x]].a_seq, a); };
        // head: the first item of the sequence in the class; out: one before it
        int head = i, step = 1;
        while (head - step >= sb[cls] && same(head - step)) {
            head -= step;
            step *= 2;
        }
        int out = max(head - step, sb[cls] - 1);
        while (head - out > 1) {
            const int mid = out + (head - out) / 2;
            if (same(mid))
                head = mid;
            else
                out = mid;
        }
        const int bin = cls / 2;
        const int width = !P.wide && bin < 4 && bin < P.narrow ? 8 : 4;
        if ((i - head) % width == 0) rank = atomicAdd(&count[cls], 1);
    }
    __syncthreads();
    if (tid < kClasses && count[tid] > 0) base[tid] = atomicAdd(nwin + tid, count[tid]);
    __syncthreads();
    if (rank >= 0) win[sb[cls] + base[cls] + rank] = i;
}

// pairs of the window at item w that share its sequence (at most `width`)
template <int WIDTH>
__device__ __forceinline__ int window_size(const SwArgs &A, int w, int end) {
    const int a = A.pairs[A.idx[w]].a_seq;
    int n = 1;
    while (n < WIDTH && w + n < end && same_seq24(A.pairs[A.idx[w + n]].a_seq, a)) ++n;
    return n;
}

// TRACE: the statistics pass of the pairs listed (see the traceback above), in
// the same layout.
template <int R, int WPB, bool MULTI, bool TRACE>
__device__ __forceinline__ bool wave16_body(const SwArgs &A, int bin, char *lds, const int8_t *sblosum,
                                            WaveLds<WPB> &L) {
    static_assert(R <= kMax16R, "at most 1024 rows per strip");
    constexpr int NI = 2 * WPB;  // pairs per block
    constexpr int RS = kWave * R;  // rows per strip
    const uint8_t *__restrict__ codes = A.codes;
    const PairDesc *__restrict__ pairs = A.pairs;
    const int *__restrict__ idx = A.idx;
    const int go_ge = A.go_ge, ge = A.ge;
    SwPass1Out *__restrict__ out = A.p1;
    ProfWord<R>(*prof)[kWave] = (ProfWord<R>(*)[kWave])lds;
    auto &s_next = L.next;
    int &s_take = L.take;
    // a bin's two rows classes (bins of up to 8 rows per lane) count as one here
    const int tall = A.nwin[2 * bin + 1], windows = tall + A.nwin[2 * bin];
    constexpr int NW = dir_words<R>();
    const int64_t gwave = (int64_t)blockIdx.x * WPB + __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    uint32_t *const dirs =
        !TRACE ? nullptr : MULTI ? A.dirs_multi + gwave * A.dirs_per_multi : A.dirs + gwave * A.dirs_per_wave;
    const int64_t strip_words = A.dirs_per_multi / kTraceStrips;
    bool any = false;
    const int lane = threadIdx.x & (kWave - 1);
    // wave-uniform values are made so for the compiler, which keeps them (and
    // the loops they bound) out of the vector registers
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    const uint32_t OE2 = (uint32_t)go_ge * 0x10001u, GE2 = (uint32_t)ge * 0x10001u;
    const uint32_t G0 = ((uint32_t)(-go_ge) & 0xFFFFu) * 0x10001u;  // G of an H = 0 cell
    uint32_t *bnd_g = nullptr, *bnd_f = nullptr;
    if constexpr (MULTI) {
        bnd_g = (uint32_t *)A.scratch + gwave * A.scratch_per_wave;
        bnd_f = bnd_g + A.scratch_per_wave / 2;
    }
    int par = 0;

    for (;;) {
        // every thread has read the last window before the round loop's
        // first barrier, so thread 0 may claim the next one
        if (threadIdx.x == 0) s_take = atomicAdd(A.queue + 2 * bin, 1);
        __syncthreads();
        const int k = __builtin_amdgcn_readfirstlane(s_take);
        if (k >= windows) break;
        any = true;
        const int cls = 2 * bin + (k < tall ? 1 : 0);
        const int w = __builtin_amdgcn_readfirstlane(A.win[A.bounds[cls] + (k < tall ? k : k - tall)]);
        const int nit = __builtin_amdgcn_readfirstlane(window_size<NI>(A, w, A.bounds[cls + 1]));
        const int iP = 2 * wave, iQ = iP + 1;
        const int qP = iP < nit ? idx[w + iP] : -1;
        const int qQ = iQ < nit ? idx[w + iQ] : -1;
        const int q0 = idx[w];
        const PairDesc dP = pairs[qP < 0 ? q0 : qP], dQ = pairs[qQ < 0 ? q0 : qQ];
        bool doneP = qP < 0, doneQ = qQ < 0;
        for (;;) {
            // this round's sequence a: that of the block's first unfinished pair
            if (lane == 0) s_next[par][wave] = !doneP ? iP : !doneQ ? iQ : NI;
            __syncthreads();
            int first = NI;
#pragma unroll
            for (int k = 0; k < WPB; ++k) first = min(first, s_next[par][k]);
            first = __builtin_amdgcn_readfirstlane(first);
            par ^= 1;
            if (first >= NI) break;
            const PairDesc dA = pairs[idx[w + first]];
            const bool actP = !doneP && dP.a_seq == dA.a_seq;
            const bool actQ = !doneQ && dQ.a_seq == dA.a_seq;
            const int laA = dA.la, lbP = actP ? dP.lb : 0, lbQ = actQ ? dQ.lb : 0;
            const uint8_t *bP = codes + dP.b_off, *bQ = codes + dQ.b_off;
            const int lb = max(lbP, lbQ);
            const int steps = lb > 0 ? lb + kWave - 1 : 0;
            const int nstrips = MULTI ? (laA + RS - 1) / RS : 1;
            // best row of each pair: (score << 16) | (0xFFFF - row), maximised,
            // and the lane's hint at its end column
            unsigned kp = 0u, kq = 0u;
            int hintP = 0, hintQ = 0;
            // TRACE: each pair's end row, first possible end column and score, and
            // the last strip that holds an end cell
            int rowP = -1, rowQ = -1, fcP = 0, fcQ = 0, scP = 0, scQ = 0;
            int endP = -1, endQ = -1, last_strip = 0;
            if constexpr (TRACE) {
                if (actP) {
                    const SwPass1Out r1 = A.p1[qP];
                    rowP = r1.end_a, fcP = first_col(r1.end_b), scP = r1.score;
                }
                if (actQ) {
                    const SwPass1Out r1 = A.p1[qQ];
                    rowQ = r1.end_a, fcQ = first_col(r1.end_b), scQ = r1.score;
                }
                if constexpr (MULTI) last_strip = __builtin_amdgcn_readfirstlane(max(max(rowP, rowQ), 0) / RS);
            }
            for (int sidx = 0; sidx < nstrips; ++sidx) {
                const int base = sidx * RS;
                if (sidx > 0) __syncthreads();  // every wave is done with the last strip's profile
                build_profile16<R, kWave, WPB>(prof, sblosum, codes + dA.a_off + base, laA - base, lane, wave,
                                               go_ge);
                __syncthreads();
                const bool from_above = MULTI && sidx > 0;
                const bool to_below = MULTI && sidx + 1 < nstrips;
                if (TRACE && sidx > last_strip) continue;  // nothing below this wave's end cells
                uint32_t G[R], E[R], M[TRACE ? 1 : R];
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    G[r] = G0;
                    E[r] = 0u;
                    if constexpr (!TRACE) M[r] = 0u;
                }
                uint32_t seen = 0u, when = 0u;
                int noted = 0;  // step of the last note_rise
                // TRACE: does this lane hold an end cell of this strip still to be
                // found, and the first step one can be found in (tn, wave-uniform)
                const int eP = rowP - base, eQ = rowQ - base;
                bool needP = TRACE && eP >= 0 && eP < RS && eP / R == lane;
                bool needQ = TRACE && eQ >= 0 && eQ < RS && eQ / R == lane;
                const int reP = eP % R, reQ = eQ % R;
                auto first_step = [&]() {
                    return __builtin_amdgcn_readfirstlane(
                        wave_min_i32(min(needP ? fcP + lane : INT_MAX, needQ ? fcQ + lane : INT_MAX)));
                };
                int tn = TRACE ? first_step() : INT_MAX;
                uint32_t glast = G0, flast = 0u, gprev = G0;
                // column residues travel as byte offsets into the profile, P's
                // in the low half and Q's in the high half (at most 24 * 1024)
                constexpr uint32_t kStride = (uint32_t)(sizeof(ProfWord<R>) * kWave);
                const char *plane = (const char *)&prof[0][lane];
                int cres = (int)((kPadCode * kStride) * 0x10001u);
                auto col = [&](int c) {
                    const uint32_t x = c < lbP ? (uint32_t)bP[c] : (uint32_t)kPadCode;
                    const uint32_t y = c < lbQ ? (uint32_t)bQ[c] : (uint32_t)kPadCode;
                    return (int)((x * kStride) | ((y * kStride) << 16));
                };
                int chunk = col(lane);  // columns 0..63; nx holds the next 64
                int nx = col(kWave + lane);
                // top boundary words of columns 0..63 and 64..127 (columns past
                // lb: an H = 0 row above)
                uint32_t ch_g = G0, ch_f = 0u, nx_g = G0, nx_f = 0u;
                if (from_above) {
                    if (lane < lb) {
                        ch_g = vload(bnd_g + lane);
                        ch_f = vload(bnd_f + lane);
                    }
                    if (kWave + lane < lb) {
                        nx_g = vload(bnd_g + kWave + lane);
                        nx_f = vload(bnd_f + kWave + lane);
                    }
                }
                // kTop: lane 0 takes its top boundary from the buffer (t < lb)
                auto step = [&](const int t, auto top_tag) {
                    constexpr bool kTop = decltype(top_tag)::value;
                    if ((t & (kWave - 1)) == 0 && t > 0) {
                        chunk = nx;
                        nx = col(t + kWave + lane);
                        if constexpr (kTop) {
                            ch_g = nx_g;
                            ch_f = nx_f;
                            const int c = t + kWave + lane;
                            nx_g = c < lb ? vload(bnd_g + c) : G0;
                            nx_f = c < lb ? vload(bnd_f + c) : 0u;
                        }
                    }
                    const int bt = __builtin_amdgcn_readlane(chunk, t & (kWave - 1));
                    uint32_t rg, rf;
                    if constexpr (kTop) {
                        rg = (uint32_t)shr1u((uint32_t)__builtin_amdgcn_readlane((int)ch_g, t & (kWave - 1)), glast);
                        rf = (uint32_t)shr1u((uint32_t)__builtin_amdgcn_readlane((int)ch_f, t & (kWave - 1)), flast);
                    } else {
                        rg = (uint32_t)shr1u(G0, glast);
                        rf = (uint32_t)shr1z((int)flast);
                    }
                    cres = shr1(bt, cres);
                    const ProfWord<R> cP = *(const ProfWord<R> *)(plane + ((uint32_t)cres & 0xFFFFu));
                    const ProfWord<R> cQ = *(const ProfWord<R> *)(plane + ((uint32_t)cres >> 16));
                    short2_t gd = s2(gprev), gu = s2(rg), fu = s2(rf);
                    uint32_t dw[NW] = {};
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        // byte r of P's and Q's words into the two halves
                        const uint32_t sel =
                            (uint32_t)(r & 3) | 0x0C00u | ((uint32_t)(4 + (r & 3)) << 16) | 0x0C000000u;
                        const short2_t sig =
                            s2(__builtin_amdgcn_perm(prof_word<R>(cQ, r), prof_word<R>(cP, r), sel));
                        const short2_t ex = psubs(s2(E[r]), GE2), fx = psubs(fu, GE2);
                        const short2_t e = pmax(ex, s2(G[r]));
                        const short2_t f = pmax(fx, gu);
                        const short2_t d = gd + sig;
                        const short2_t m = pmax(e, f);
                        const short2_t h = pmax(d, m);
                        if constexpr (TRACE) file_dirs(dw, r, d, m, e, f, ex, s2(G[r]), fx, gu);
                        gd = s2(G[r]);
                        const short2_t g = h - s2(OE2);
                        G[r] = u2(g);
                        E[r] = u2(e);
                        if constexpr (!TRACE) M[r] = u2(pmax(s2(M[r]), h));
                        gu = g;
                        fu = f;
                    }
                    glast = G[R - 1];
                    flast = u2(fu);
                    gprev = rg;
                    if constexpr (TRACE)
                        store_dirs(dirs + (MULTI ? sidx * strip_words : 0) + (int64_t)t * (kWave * NW) + lane * NW, dw);
                    if (to_below) {
                        const int j = t - (kWave - 1);
                        if (lane == kWave - 1 && j >= 0 && j < lb) {
                            bnd_g[j] = glast;
                            bnd_f[j] = flast;
                        }
                    }
                };
                // one step, and in TRACE the test for the end cells it can hold:
                // the end column is the first where row end_a reaches the score
                auto advance = [&](const int t, auto top_tag) {
                    step(t, top_tag);
                    if constexpr (TRACE) {
                        if (t < tn) return;
                        // (the empty statement keeps the row tests here: hoisted out
                        // of the loop they would hold two masks per row)
                        int rp = reP, rq = reQ;
                        asm volatile("" : "+v"(rp), "+v"(rq));
                        uint32_t gP = G[0], gQ = G[0];
#pragma unroll
                        for (int r = 1; r < R; ++r) {
                            gP = rp == r ? G[r] : gP;
                            gQ = rq == r ? G[r] : gQ;
                        }
                        const int c = t - lane;
                        const bool hitP = needP && c >= 0 && (int)(int16_t)(gP & 0xFFFFu) + go_ge == scP;
                        const bool hitQ = needQ && c >= 0 && ((int)gQ >> 16) + go_ge == scQ;
                        if (hitP) endP = c;
                        if (hitQ) endQ = c;
                        needP = needP && !hitP;
                        needQ = needQ && !hitQ;
                        if (__ballot(hitP || hitQ)) tn = first_step();
                    }
                };
                // (TRACE) every end cell of the wave is found
                auto found = [&]() { return TRACE && tn == INT_MAX && sidx == last_strip; };
                // two steps per iteration, so the old and new G registers can
                // swap roles instead of being copied back every step
                int t = 0;
                if (from_above) {
                    for (; t + 1 < lb && !found(); t += 2) {
                        if constexpr (!TRACE)
                            if ((t & 15) == 0) note_rise(M, seen, when, (noted = t, (t >> 4) - 1));
                        advance(t, std::true_type{});
                        advance(t + 1, std::true_type{});
                    }
                    if (t < lb && !found()) advance(t++, std::true_type{});
                }
                for (; t + 1 < steps && !found(); t += 2) {
                    if constexpr (!TRACE)
                        if ((t & 15) <= 1) note_rise(M, seen, when, (noted = t, (t >> 4) - 1));
                    advance(t, std::false_type{});
                    advance(t + 1, std::false_type{});
                }
                if (t < steps && !found()) advance(t, std::false_type{});
                if constexpr (!TRACE) {
                    note_rise(M, seen, when, noted >> 4);  // the steps since the last note
                    unsigned sp = 0u, sq = 0u;
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        const int row = base + lane * R + r;
                        const unsigned rk = 0xFFFFu - (unsigned)row;
                        if (row < laA) {
                            sp = max(sp, ((M[r] & 0xFFFFu) << 16) | rk);
                            sq = max(sq, (M[r] & 0xFFFF0000u) | rk);
                        }
                    }
                    if (sp > kp) {
                        kp = sp;
                        hintP = hint_code((int)(when & 0xFFFFu), lane);
                    }
                    if (sq > kq) {
                        kq = sq;
                        hintQ = hint_code((int)(when >> 16), lane);
                    }
                }
                if (to_below) __threadfence_block();  // lane 0 of the next strip reads lane 63's row
            }
            if constexpr (TRACE) {
                __syncthreads();  // every wave is done with the profile: its LDS serves the walks
                __threadfence_block();
                const int half = lane / 32, sub = lane % 32;
                const bool act = half ? actQ : actP;
                const int q = half ? qQ : qP;
                const int colP = __shfl(endP, max(rowP, 0) % RS / R, kWave);
                const int colQ = __shfl(endQ, max(rowQ, 0) % RS / R, kWave);
                const int end_a = half ? rowQ : rowP, end_b = half ? colQ : colP, score = half ? scQ : scP;
                Walk P;
                P.i = end_a;
                P.j = end_b;
                P.h = score;
                auto *wl = (typename WalkShape<kWave, R, MULTI>::Lds *)lds + 2 * wave + half;
                walk_back<kWave, R, MULTI>(P, act, dirs, strip_words, codes + dA.a_off, laA, half ? bQ : bP, 0, half,
                                           sub, *wl, sblosum, go_ge, ge);
                if (act && sub == 0) walk_record(A, P, score, end_a, end_b, q);
                doneP = doneP || actP;
                doneQ = doneQ || actQ;
                continue;
            }
            const unsigned lp = kp, lq = kq;  // the lane's own
            kp = wave_max_u32(kp);
            kq = wave_max_u32(kq);
            // the winning lane's hint (its key holds its row, so it is alone)
            const int hp = __shfl(hintP, __ffsll((long long)__ballot(lp == kp)) - 1, kWave);
            const int hq = __shfl(hintQ, __ffsll((long long)__ballot(lq == kq)) - 1, kWave);
            if (lane == 0) {
                SwPass1Out o;
                o.pad = 0;
                if (actP) {
                    o.score = (int32_t)(kp >> 16);
                    o.end_a = o.score > 0 ? (int32_t)(0xFFFFu - (kp & 0xFFFFu)) : -1;
                    o.end_b = o.score > 0 ? hp : -1;
                    out[qP] = o;
                }
                if (actQ) {
                    o.score = (int32_t)(kq >> 16);
                    o.end_a = o.score > 0 ? (int32_t)(0xFFFFu - (kq & 0xFFFFu)) : -1;
                    o.end_b = o.score > 0 ? hq : -1;
                    out[qQ] = o;
                }
            }
            doneP = doneP || actP;
            doneQ = doneQ || actQ;
        }
    }
    return any;
}

// ---------------------------------------------------------------- pass 1, 16-bit lanes, strips of S lanes

// For short sequences a the wave splits into 64 / S independent strips of S
// lanes (S = 16 or 32).  Each strip runs two pairs of the wave's sequence a in
// the halves of its words, with the same recurrence as above; lane p of a
// strip owns rows [p * RP, p * RP + RP), so a bin of 64 R rows takes RP =
// 64 R / S rows per lane.  A pair then pays S - 1 steps of wavefront fill and
// drain instead of 63, and the fixed work of a step (lane shifts, residue and
// profile fetches) serves 64 / S times more cells.  All strips read one
// profile of 25 codes x S lanes.  Column residues enter at a strip's first
// lane from a chunk of 16 columns held across the strip's first 16 lanes,
// rotated by one lane per step.
constexpr int kDppRowShr1 = 0x111;
constexpr int kDppRowRor15 = 0x12F;
constexpr int kDppRowRor8 = 0x128, kDppRowRor4 = 0x124, kDppRowRor2 = 0x122, kDppRowRor1 = 0x121;

// lane p of a strip receives lane p - 1's value; the strip's first lane
// receives `first`
template <int S>
__device__ __forceinline__ uint32_t strip_shr(uint32_t first, uint32_t v, int lane) {
    if constexpr (S == 16) {
        return (uint32_t)__builtin_amdgcn_update_dpp((int)first, (int)v, kDppRowShr1, 0xF, 0xF, false);
    } else {
        // a zero-filled shift writes every lane (no prior value of the result
        // is needed); the strips' first lanes, 0 and 32, then take `first`
        const uint32_t t = (uint32_t)__builtin_amdgcn_mov_dpp((int)v, kDppWaveShr1, 0xF, 0xF, true);
        return (lane & (S - 1)) == 0 ? first : t;
    }
}

// as strip_shr with first = 0 (zero-filled by the move's bound control)
template <int S>
__device__ __forceinline__ uint32_t strip_shrz(uint32_t v, int lane) {
    if constexpr (S == 16) {
        return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kDppRowShr1, 0xF, 0xF, true);
    } else {
        const uint32_t t = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kDppWaveShr1, 0xF, 0xF, true);
        return lane == kWave / 2 ? 0u : t;
    }
}

template <int S>
__device__ __forceinline__ unsigned strip_max_u32(unsigned v) {
#pragma unroll
    for (int off = S / 2; off > 0; off >>= 1) v = max(v, (unsigned)__shfl_xor((int)v, off, kWave));
    return v;
}

// One rows class of a bin's pairs (sorted by rows class first): class c holds
// the items [bounds[2 bin + c], bounds[2 bin + c + 1]) and has its own queue.
template <int S, int RP, bool TRACE>
__device__ __forceinline__ bool strip16_body(const SwArgs &A, int cls, char *lds, size_t wave_bytes,
                                             const int8_t *sblosum) {
    static_assert((S == 16 || S == 32) && RP <= kMax16R, "strip shape");
    constexpr int NI = 2 * kWave / S;  // pairs per wave: two per strip
    const uint8_t *__restrict__ codes = A.codes;
    const PairDesc *__restrict__ pairs = A.pairs;
    const int *__restrict__ idx = A.idx;
    const int go_ge = A.go_ge, ge = A.ge;
    SwPass1Out *__restrict__ out = A.p1;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    const int pos = lane % S, strip = lane / S, cl = lane & 15;
    // waves of a block may be in bins of different profile sizes: each has a
    // fixed share of the block's LDS
    ProfWord<RP>(*prof)[S] = (ProfWord<RP>(*)[S])(lds + (size_t)wave * wave_bytes);
    const int item_begin = A.bounds[cls], item_end = A.bounds[cls + 1], windows = A.nwin[cls];
    int *const counter = A.queue + cls;
    constexpr int NW = dir_words<RP>();
    uint32_t *const dirs =
        TRACE ? A.dirs + ((int64_t)blockIdx.x * (blockDim.x / kWave) + wave) * A.dirs_per_wave : nullptr;
    bool any = false;
    const uint32_t OE2 = (uint32_t)go_ge * 0x10001u, GE2 = (uint32_t)ge * 0x10001u;
    const uint32_t G0 = ((uint32_t)(-go_ge) & 0xFFFFu) * 0x10001u;  // G of an H = 0 cell

    for (int64_t k = take_from(counter, 0, 1); k < windows; k = take_from(counter, 0, 1)) {
        any = true;
        const int w = __builtin_amdgcn_readfirstlane(A.win[item_begin + k]);
        const int nit = __builtin_amdgcn_readfirstlane(window_size<NI>(A, w, item_end));
        const int iP = 2 * strip, iQ = iP + 1;
        const int qP = iP < nit ? idx[w + iP] : -1;
        const int qQ = iQ < nit ? idx[w + iQ] : -1;
        const int q0 = idx[w];
        const PairDesc dP = pairs[qP < 0 ? q0 : qP], dQ = pairs[qQ < 0 ? q0 : qQ];
        bool doneP = qP < 0, doneQ = qQ < 0;
        // one round per distinct sequence a among the wave's pairs (pairs are
        // sorted by a, so nearly always one)
        for (;;) {
            const int mine = !doneP ? iP : !doneQ ? iQ : NI;
            const int first = __builtin_amdgcn_readfirstlane(wave_min_i32(mine));
            if (first >= NI) break;
            const int src = (first >> 1) * S;
            const bool fq = (first & 1) != 0;
            const int a_seq = __builtin_amdgcn_readlane(fq ? dQ.a_seq : dP.a_seq, src);
            const int la = __builtin_amdgcn_readlane(fq ? dQ.la : dP.la, src);
            const int64_t a_off_v = fq ? dQ.a_off : dP.a_off;
            const uint32_t off_lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)a_off_v, src);
            const uint32_t off_hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(a_off_v >> 32), src);
            const int64_t a_off = (int64_t)(((uint64_t)off_hi << 32) | off_lo);
            const bool actP = !doneP && dP.a_seq == a_seq;
            const bool actQ = !doneQ && dQ.a_seq == a_seq;
            const int lbP = actP ? dP.lb : 0, lbQ = actQ ? dQ.lb : 0;
            const uint8_t *bP = codes + dP.b_off, *bQ = codes + dQ.b_off;
            build_profile16<RP, S, kWave / S>(prof, sblosum, codes + a_off, la, pos, strip, go_ge);
            // lanes read entries written by other lanes of the wave (LDS
            // operations of one wave complete in order)
            __builtin_amdgcn_wave_barrier();
            const int lbmax = wave_max_i32(max(lbP, lbQ));
            const int steps = __builtin_amdgcn_readfirstlane(lbmax > 0 ? lbmax + S - 1 : 0);
            uint32_t G[RP], E[RP], M[TRACE ? 1 : RP];
#pragma unroll
            for (int r = 0; r < RP; ++r) {
                G[r] = G0;
                E[r] = 0u;
                if constexpr (!TRACE) M[r] = 0u;
            }
            uint32_t seen = 0u, when = 0u;
                int noted = 0;  // step of the last note_rise
            // TRACE: each pair's end cell, whether this lane holds one still to
            // be found, and the first step one can be found in (tn, wave-uniform)
            int rowP = -1, rowQ = -1, fcP = 0, fcQ = 0, scP = 0, scQ = 0;
            if constexpr (TRACE) {
                if (actP) {
                    const SwPass1Out r1 = A.p1[qP];
                    rowP = r1.end_a, fcP = first_col(r1.end_b), scP = r1.score;
                }
                if (actQ) {
                    const SwPass1Out r1 = A.p1[qQ];
                    rowQ = r1.end_a, fcQ = first_col(r1.end_b), scQ = r1.score;
                }
            }
            int endP = -1, endQ = -1;
            bool needP = TRACE && rowP >= 0 && rowP / RP == pos, needQ = TRACE && rowQ >= 0 && rowQ / RP == pos;
            const int reP = rowP % RP, reQ = rowQ % RP;
            auto first_step = [&]() {
                return __builtin_amdgcn_readfirstlane(
                    wave_min_i32(min(needP ? fcP + pos : INT_MAX, needQ ? fcQ + pos : INT_MAX)));
            };
            int tn = TRACE ? first_step() : INT_MAX;
            uint32_t glast = G0, flast = 0u, gprev = G0;
            // column residues travel as byte offsets into the profile, P's in
            // the low half and Q's in the high half (at most 24 * 512 bytes)
            constexpr uint32_t kStride = (uint32_t)(sizeof(ProfWord<RP>) * S);
            const char *plane = (const char *)&prof[0][pos];
            uint32_t cres = (kPadCode * kStride) * 0x10001u;
            auto col = [&](int c) -> uint32_t {
                const uint32_t x = c < lbP ? (uint32_t)bP[c] : (uint32_t)kPadCode;
                const uint32_t y = c < lbQ ? (uint32_t)bQ[c] : (uint32_t)kPadCode;
                return (x * kStride) | ((y * kStride) << 16);
            };
            auto at = [&](uint32_t off) { return *(const ProfWord<RP> *)(plane + off); };
            uint32_t chunk = col(cl);  // columns 0..15; nx holds the next 16
            uint32_t nx = col(16 + cl);
            // the residues of step tn enter at each strip's first lane
            auto feed = [&](const int tn) {
                if ((tn & 15) == 0 && tn > 0) {
                    chunk = nx;
                    nx = col(tn + 16 + cl);
                }
                cres = strip_shr<S>(chunk, cres, lane);
                chunk = (uint32_t)__builtin_amdgcn_mov_dpp((int)chunk, kDppRowRor15, 0xF, 0xF, false);
            };
            // as in the full-wave kernel: with few rows per lane the profile
            // words of step t + 1 are loaded during step t
            constexpr bool kAhead = RP <= 8;
            ProfWord<RP> wP = prof[kPadCode][pos], wQ = wP;
            auto step = [&](const int t) {
                const uint32_t rg = strip_shr<S>(G0, glast, lane);
                const uint32_t rf = strip_shrz<S>(flast, lane);
                ProfWord<RP> cP, cQ;
                if constexpr (kAhead) {
                    feed(t + 1);
                    cP = wP;
                    cQ = wQ;
                    wP = at(cres & 0xFFFFu);
                    wQ = at(cres >> 16);
                } else {
                    feed(t);
                    cP = at(cres & 0xFFFFu);
                    cQ = at(cres >> 16);
                }
                short2_t gd = s2(gprev), gu = s2(rg), fu = s2(rf);
                uint32_t dw[NW] = {};
#pragma unroll
                for (int r = 0; r < RP; ++r) {
                    const uint32_t sel =
                        (uint32_t)(r & 3) | 0x0C00u | ((uint32_t)(4 + (r & 3)) << 16) | 0x0C000000u;
                    const short2_t sig = s2(__builtin_amdgcn_perm(prof_word<RP>(cQ, r), prof_word<RP>(cP, r), sel));
                    const short2_t ex = psubs(s2(E[r]), GE2), fx = psubs(fu, GE2);
                    const short2_t e = pmax(ex, s2(G[r]));
                    const short2_t f = pmax(fx, gu);
                    const short2_t d = gd + sig;
                    const short2_t m = pmax(e, f);
                    const short2_t h = pmax(d, m);
                    if constexpr (TRACE) file_dirs(dw, r, d, m, e, f, ex, s2(G[r]), fx, gu);
                    gd = s2(G[r]);
                    const short2_t g = h - s2(OE2);
                    G[r] = u2(g);
                    E[r] = u2(e);
                    if constexpr (!TRACE) M[r] = u2(pmax(s2(M[r]), h));
                    gu = g;
                    fu = f;
                }
                glast = G[RP - 1];
                flast = u2(fu);
                gprev = rg;
                if constexpr (TRACE) {
                    store_dirs(dirs + (int64_t)t * (kWave * NW) + lane * NW, dw);
                    if (t < tn) return;
                    // the end column is the first where row end_a reaches the score
                    // (the empty statement keeps the row tests here: hoisted out
                    // of the loop they would hold two masks per row)
                    int rp = reP, rq = reQ;
                    asm volatile("" : "+v"(rp), "+v"(rq));
                    uint32_t gP = G[0], gQ = G[0];
#pragma unroll
                    for (int r = 1; r < RP; ++r) {
                        gP = rp == r ? G[r] : gP;
                        gQ = rq == r ? G[r] : gQ;
                    }
                    const int c = t - pos;
                    const bool hitP = needP && c >= 0 && (int)(int16_t)(gP & 0xFFFFu) + go_ge == scP;
                    const bool hitQ = needQ && c >= 0 && ((int)gQ >> 16) + go_ge == scQ;
                    if (hitP) endP = c;
                    if (hitQ) endQ = c;
                    needP = needP && !hitP;
                    needQ = needQ && !hitQ;
                    if (__ballot(hitP || hitQ)) tn = first_step();
                }
            };
            // (TRACE) every end cell of the wave is found
            auto found = [&]() { return TRACE && tn == INT_MAX; };
            if constexpr (kAhead) {
                feed(0);
                wP = at(cres & 0xFFFFu);
                wQ = at(cres >> 16);
            }
            int t = 0;
            for (; t + 1 < steps && !found(); t += 2) {
                if constexpr (!TRACE)
                    if ((t & 15) == 0) note_rise(M, seen, when, (noted = t, (t >> 4) - 1));
                step(t);
                step(t + 1);
            }
            if (t < steps && !found()) step(t);
            if constexpr (TRACE) {
                // the wave's own profile is done with: its LDS serves the walks
                __threadfence_block();
                const int half = pos / (S / 2), sub = pos % (S / 2);
                const bool act = half ? actQ : actP;
                const int q = half ? qQ : qP;
                const int colP = __shfl(endP, strip * S + max(rowP, 0) / RP, kWave);
                const int colQ = __shfl(endQ, strip * S + max(rowQ, 0) / RP, kWave);
                const int end_a = half ? rowQ : rowP, end_b = half ? colQ : colP, score = half ? scQ : scP;
                Walk P;
                P.i = end_a;
                P.j = end_b;
                P.h = score;
                auto *wl = (typename WalkShape<S, RP, false>::Lds *)(lds + (size_t)wave * wave_bytes) + 2 * strip + half;
                walk_back<S, RP, false>(P, act, dirs, 0, codes + a_off, la, half ? bQ : bP, strip * S, half, sub, *wl,
                                        sblosum, go_ge, ge);
                if (act && sub == 0) walk_record(A, P, score, end_a, end_b, q);
                doneP = doneP || actP;
                doneQ = doneQ || actQ;
                continue;
            }
            unsigned kp = 0u, kq = 0u;
            if constexpr (!TRACE) {
                note_rise(M, seen, when, noted >> 4);  // the steps since the last note
#pragma unroll
                for (int r = 0; r < RP; ++r) {
                    const int row = pos * RP + r;
                    const unsigned rk = 0xFFFFu - (unsigned)row;
                    if (row < la) {
                        kp = max(kp, ((M[r] & 0xFFFFu) << 16) | rk);
                        kq = max(kq, (M[r] & 0xFFFF0000u) | rk);
                    }
                }
            }
            kp = strip_max_u32<S>(kp);
            kq = strip_max_u32<S>(kq);
            // the end rows' lanes and their hints at the end columns
            const int posP = (int)(0xFFFFu - (kp & 0xFFFFu)) / RP % S, posQ = (int)(0xFFFFu - (kq & 0xFFFFu)) / RP % S;
            const uint32_t whenP = (uint32_t)__shfl((int)when, strip * S + posP, kWave);
            const uint32_t whenQ = (uint32_t)__shfl((int)when, strip * S + posQ, kWave);
            if (pos == 0) {
                SwPass1Out o;
                o.pad = 0;
                if (actP) {
                    o.score = (int32_t)(kp >> 16);
                    o.end_a = o.score > 0 ? (int32_t)(0xFFFFu - (kp & 0xFFFFu)) : -1;
                    o.end_b = o.score > 0 ? hint_code((int)(whenP & 0xFFFFu), posP) : -1;
                    out[qP] = o;
                }
                if (actQ) {
                    o.score = (int32_t)(kq >> 16);
                    o.end_a = o.score > 0 ? (int32_t)(0xFFFFu - (kq & 0xFFFFu)) : -1;
                    o.end_b = o.score > 0 ? hint_code((int)(whenQ >> 16), posQ) : -1;
                    out[qQ] = o;
                }
            }
            doneP = doneP || actP;
            doneQ = doneQ || actQ;
        }
    }
    return any;
}

// ---------------------------------------------------------------- start bound
//
// Before the statistics: pairs whose score does not already promise a long
// alignment are checked against the coverage cut.  The DP is run backwards
// from the end row, upwards and to the left, from every column of pass 1's
// window at the end column: the value of a cell is then the best score of an
// alignment from it to the end row, and the cells that reach the pair's score
// are the starts of optimal alignments, so the highest of their rows bounds the
// canonical alignment's coverage.  (The window begins at or before the first
// column that holds the score in the end row, so it contains that column if any
// cell reaches the score; where none does, another row of pass 1's lane held
// the maximum first, and the pair goes on to the statistics.)  No value
// exceeds the score (the largest of the matrix), and every proper suffix of an
// optimal alignment scores above 0, so the sweep ends when no value is above 0:
// after some 120 columns for unrelated pairs, against the whole width for a
// forward sweep, and over the 256 rows above the end row whatever the
// sequences' length.  An alignment that is still alive in the topmost of them
// cannot be bounded here and goes on to the statistics, where it fails the cut
// like any other; a pair that has ended (by either test, or at its first column)
// is dead in every cell from then on, since a value of 0 or less could rise again
// and its pair's answer would depend on how long the wave's other pairs keep the
// sweep going.  Only the
// edges of a search use this bound (138,000 of 3.07 million
// at 250,000 sequences, 14 ms of traceback).  There the forward kernel, which
// sweeps the end rectangle in 32-bit lanes, took 132 ms, this one 36; where
// sequences reach 25,000 residues 115 against 1.3.
//
// Two pairs per strip of 16 lanes and 16 rows per lane, eight pairs per wave,
// in 16-bit lanes as in pass 1, but with saturating adds and dead cells at
// -2^15 (a dead path gains at most 11 per row and never gets near 0).  The
// pairs share nothing, so scores come from the 25 x 25 table in LDS, one read
// per row and pair, which costs as much as the vector instructions beside it.
constexpr int kBoundLanes = 16, kBoundRP = 16, kBoundRows = kBoundLanes * kBoundRP;
constexpr int kBoundWaves = 4;
constexpr int kBoundWindow = 18;  // columns a hint can stand for: 16 steps, and the last note's odd ones

__device__ __forceinline__ short2_t adds(short2_t a, short2_t b) { return __builtin_elementwise_add_sat(a, b); }
__device__ __forceinline__ short2_t subss(short2_t a, short2_t b) { return __builtin_elementwise_sub_sat(a, b); }

__global__ __launch_bounds__(64 * kBoundWaves, 4) void sw16_bound_kernel(SwArgs A, TraceRule T,
                                                                         int8_t *__restrict__ bin_of,
                                                                         unsigned long long *__restrict__ counters) {
    constexpr int S = kBoundLanes, RP = kBoundRP, NI = 2 * kWave / S;
    __shared__ uint32_t stab[kProfCodes * kProfCodes];  // score + o + e, in the low half
    for (int t = threadIdx.x; t < kProfCodes * kProfCodes; t += blockDim.x)
        stab[t] = (uint32_t)(A.blosum[t] + A.go_ge) & 0xFFFFu;
    __syncthreads();
    const uint8_t *__restrict__ codes = A.codes;
    const int lane = threadIdx.x & (kWave - 1), pos = lane % S, strip = lane / S;
    const int go_ge = A.go_ge;
    const uint32_t OE2 = (uint32_t)go_ge * 0x10001u, GE2 = (uint32_t)A.ge * 0x10001u;
    const uint32_t kDead = 0x80008000u;
    const uint32_t G0 = ((uint32_t)(-go_ge) & 0xFFFFu) * 0x10001u;  // G of an H = 0 cell
    const int n = A.queue[1];  // listed pairs
    for (int64_t w = take_from(A.queue, 0, NI); w < n; w = take_from(A.queue, 0, NI)) {
        int q[2], la[2], score[2], end_a[2], hi[2], win[2];
        const uint8_t *pa[2], *pb[2];
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            const int64_t at = w + 2 * strip + x;
            q[x] = at < n ? A.idx[at] : -1;
            la[x] = score[x] = 0;
            end_a[x] = hi[x] = -1;
            win[x] = 0;
            pa[x] = pb[x] = codes;
            if (q[x] >= 0) {
                const PairDesc pd = A.pairs[q[x]];
                const SwPass1Out r1 = A.p1[q[x]];
                const int lo = first_col(r1.end_b);
                la[x] = pd.la;
                score[x] = r1.score;
                end_a[x] = r1.end_a;
                hi[x] = r1.end_b >= 0 ? lo : min(lo + kBoundWindow, pd.lb) - 1;
                win[x] = hi[x] - lo + 1;
                pa[x] = codes + pd.a_off;
                pb[x] = codes + pd.b_off;
            }
        }
        // byte offsets into the table, P's in the low half and Q's in the high
        // half: rows (code * 100, at most 2,400) and columns (code * 4)
        uint32_t row[RP];
#pragma unroll
        for (int r = 0; r < RP; ++r) {
            const int iP = end_a[0] - (pos * RP + r), iQ = end_a[1] - (pos * RP + r);
            const uint32_t x = iP >= 0 ? (uint32_t)pa[0][iP] : (uint32_t)kPadCode;
            const uint32_t y = iQ >= 0 ? (uint32_t)pa[1][iQ] : (uint32_t)kPadCode;
            row[r] = (x | y << 16) * (4u * kProfCodes);
        }
        auto col = [&](int v) -> uint32_t {
            const int jP = hi[0] - v, jQ = hi[1] - v;
            const uint32_t x = jP >= 0 ? (uint32_t)pb[0][jP] : (uint32_t)kPadCode;
            const uint32_t y = jQ >= 0 ? (uint32_t)pb[1][jQ] : (uint32_t)kPadCode;
            return (x * 4u) | (y * 4u << 16);
        };
        // (whole chunks of 16 steps: a pair's sweep ends at the same step in any wave)
        const int steps = (__builtin_amdgcn_readfirstlane(wave_max_i32(max(hi[0], hi[1]))) + S + 15) & ~15;
        uint32_t G[RP], E[RP], M[RP];
#pragma unroll
        for (int r = 0; r < RP; ++r) {
            G[r] = kDead;
            E[r] = kDead;
            M[r] = 0u;
        }
        // the row below the end row: H = 0 left of every window column (an
        // alignment ends in a diagonal step), else dead
        uint32_t gprev = pos == 0 ? G0 : kDead, glast = kDead, flast = kDead, out = kDead;
        uint32_t cres = (kPadCode * 4u) * 0x10001u, chunk = col(pos), nx = col(16 + pos);
        for (int t = 0; t < steps; ++t) {
            if ((t & 15) == 0 && t > 0) {
                chunk = nx;
                nx = col(t + 16 + pos);
                if (t >= kBoundWindow) {
                    // values above 0 anywhere: the rows', or on their way down
                    uint32_t g = u2(pmax(s2(gprev), s2(glast))), e = flast;
#pragma unroll
                    for (int r = 0; r < RP; ++r) {
                        g = u2(pmax(s2(g), s2(G[r])));
                        e = u2(pmax(s2(e), s2(E[r])));
                    }
                    // (over the strip, whose lanes are a row of the wave's)
                    uint32_t m = u2(pmax(adds(s2(g), s2(OE2)), s2(e)));
                    m = u2(pmax(s2(m), s2((uint32_t)__builtin_amdgcn_mov_dpp((int)m, kDppRowRor8, 0xF, 0xF, false))));
                    m = u2(pmax(s2(m), s2((uint32_t)__builtin_amdgcn_mov_dpp((int)m, kDppRowRor4, 0xF, 0xF, false))));
                    m = u2(pmax(s2(m), s2((uint32_t)__builtin_amdgcn_mov_dpp((int)m, kDppRowRor2, 0xF, 0xF, false))));
                    m = u2(pmax(s2(m), s2((uint32_t)__builtin_amdgcn_mov_dpp((int)m, kDppRowRor1, 0xF, 0xF, false))));
                    const uint32_t o = (uint32_t)__shfl((int)out, strip * S + S - 1, kWave);  // G in the top row
                    const bool overP = end_a[0] >= kBoundRows && (int)(int16_t)(o & 0xFFFFu) + go_ge > 0;
                    const bool overQ = end_a[1] >= kBoundRows && ((int)o >> 16) + go_ge > 0;
                    const bool onP = (int)(int16_t)(m & 0xFFFFu) > 0 && !overP && t - S < hi[0];
                    const bool onQ = ((int)m >> 16) > 0 && !overQ && t - S < hi[1];
                    const uint32_t settled = (onP ? 0u : 0xFFFFu) | (onQ ? 0u : 0xFFFF0000u);
                    if (__ballot(settled != ~0u) == 0ull) break;
                    if (__ballot(settled != 0u)) {
                        auto kill = [&](uint32_t x) { return (kDead & settled) | (x & ~settled); };
                        gprev = kill(gprev), glast = kill(glast), flast = kill(flast);
#pragma unroll
                        for (int r = 0; r < RP; ++r) G[r] = kill(G[r]), E[r] = kill(E[r]);
                    }
                }
            }
            uint32_t first = kDead;
            if (t < kBoundWindow)
                first = ((t + 1 < win[0] ? G0 : kDead) & 0xFFFFu) | ((t + 1 < win[1] ? G0 : kDead) & 0xFFFF0000u);
            const uint32_t rg = strip_shr<S>(first, glast, lane), rf = strip_shr<S>(kDead, flast, lane);
            cres = strip_shr<S>(chunk, cres, lane);
            chunk = (uint32_t)__builtin_amdgcn_mov_dpp((int)chunk, kDppRowRor15, 0xF, 0xF, false);
            short2_t gd = s2(gprev), gu = s2(rg), fu = s2(rf);
#pragma unroll
            for (int r = 0; r < RP; ++r) {
                const uint32_t at = row[r] + cres;
                const uint32_t sp = *(const uint32_t *)((const char *)stab + (at & 0xFFFFu));
                const uint32_t sq = *(const uint32_t *)((const char *)stab + (at >> 16));
                const short2_t e = pmax(subss(s2(E[r]), s2(GE2)), s2(G[r]));
                const short2_t f = pmax(subss(fu, s2(GE2)), gu);
                const short2_t d = adds(gd, s2(sp | (sq << 16)));
                const short2_t h = pmax(d, pmax(e, f));
                gd = s2(G[r]);
                const short2_t g = subss(h, s2(OE2));
                G[r] = u2(g);
                E[r] = u2(e);
                M[r] = u2(pmax(s2(M[r]), h));
                gu = g;
                fu = f;
            }
            glast = G[RP - 1];
            flast = u2(fu);
            gprev = rg;
            out = u2(pmax(s2(out), s2(glast)));
        }
        // the highest row with the pair's score, counted from the end row
        int up = -1, uq = -1;
#pragma unroll
        for (int r = 0; r < RP; ++r) {
            up = (int)(M[r] & 0xFFFFu) == score[0] ? pos * RP + r : up;
            uq = (int)(M[r] >> 16) == score[1] ? pos * RP + r : uq;
        }
#pragma unroll
        for (int off = S / 2; off > 0; off >>= 1) {
            up = max(up, __shfl_xor(up, off, kWave));
            uq = max(uq, __shfl_xor(uq, off, kWave));
        }
        const uint32_t o = (uint32_t)__shfl((int)out, strip * S + S - 1, kWave);
        const bool over[2] = {end_a[0] >= kBoundRows && (int)(int16_t)(o & 0xFFFFu) + go_ge > 0,
                              end_a[1] >= kBoundRows && ((int)o >> 16) + go_ge > 0};
        const int top[2] = {up, uq};
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            if (pos != x || q[x] < 0) continue;
            const PairDesc pd = A.pairs[q[x]];
            const SwPass1Out r1 = A.p1[q[x]];
            // (a pair whose score was met in no row is not bounded)
            if (!over[x] && top[x] >= 0 && 100LL * (top[x] + 1) < (long long)A.cov_pct * la[x]) {
                sw_final_record(pd, r1, q[x], A.rec, bin_of);
                continue;
            }
            bin_of[q[x]] = can_trace(T, pd) ? kToTrace : (int8_t)rows_bin(end_a[x] + 1);
            const int cols = r1.end_b >= 0 ? r1.end_b + 1 : pd.lb;
            atomicAdd(&counters[1], 1ull);
            atomicAdd(&counters[2], (unsigned long long)(end_a[x] + 1) * (unsigned long long)cols);
        }
    }
}

// ---------------------------------------------------------------- kernel

// f(integral HI), f(integral HI - 1), ... down to 1 + HI - count
template <int HI, typename F, int... I>
__device__ __forceinline__ void descending(F &f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, HI - I>{}), ...);
}

// One launch for every bin in 16-bit lanes, the tallest first: waves take a
// bin's windows until its queue is empty, then go on to the next bin, so the
// launch has one tail, made of the shortest windows (see the 32-bit groups for
// what a tail per bin cost).  Blocks of two waves: a pair of more than 512 rows
// shares its profile between the block's waves, and a window of four pairs
// keeps the rounds per distinct sequence a few where sequences have few
// partners; 26 KB of LDS and at most 168 registers keep six blocks (three
// waves per SIMD) on a CU.  Pass 1 of 250,000 sequences issues vector instructions
// in 0.96 of the slots (2.98e11 in 503 ms), their traceback in 0.87 (7.0e10 in 131).
//
// Bins of up to 8 rows per lane run in strips of 16 lanes (R <= narrow: 4 R
// rows per lane, eight pairs per wave) or 32 lanes (2 R rows, four pairs), the
// taller rows class first.  A call of few pairs (wide) runs them across all 64
// lanes, two pairs per wave: a lone wave issues one instruction every 10 to 12
// cycles whatever its mix, so the fewest rows per lane finish first while the
// chip has waves to spare.
constexpr int kBlockWaves = 2;
constexpr size_t kBlockLds = kProfCodes * kWave * 16;  // a full-wave profile of 16 rows per lane

//
// WAVES: waves per SIMD to make room for.  The traceback's bodies spill at three
// (118 spills by the compiler's count, 120 bytes per lane; nearly all of them
// outside the loops over steps, but every window pays them) and not at two.  Two
// are what a call of up to 4,096 pairs fills (3,164 pairs: a search of 1.79 ms
// against 1.65; full records of 4,096 family pairs 2.24 against 2.32).  Across 64
// lanes two stay ahead of three beyond that (8,192 pairs 2.32 against 2.44, 16,384
// 3.2 against 3.3), in strips they do not (250,001: 9.6 ms against 10.9 in the
// pass).
template <bool TRACE, int WAVES>
__global__ __launch_bounds__(64 * kBlockWaves, WAVES) void sw16_kernel(SwArgs A, Sw16Launch P) {
    __shared__ __align__(16) char lds[kBlockLds];
    __shared__ int8_t sblosum[kProfCodes * kProfCodes];
    __shared__ WaveLds<kBlockWaves> L;
    load_blosum(sblosum, A.blosum);
    auto full = [&](auto r_tag, auto multi_tag, int bin) {
        if (!((P.bins >> bin) & 1u) || A.bounds[2 * bin] >= A.bounds[2 * bin + 2]) return;
        const unsigned long long t0 = span_now();
        if (wave16_body<decltype(r_tag)::value, kBlockWaves, decltype(multi_tag)::value, TRACE>(A, bin, lds, sblosum,
                                                                                               L) &&
            !TRACE)
            span_add(A.span + 2 * bin, t0);
        __syncthreads();  // every wave has read the last window before the next bin's first claim
    };
    auto multi = [&](auto r_tag) {
        full(r_tag, std::true_type{}, kMulti16Bin + decltype(r_tag)::value - kMultiMinR);
    };
    auto one = [&](auto r_tag) { full(r_tag, std::false_type{}, decltype(r_tag)::value - 1); };
    if (blockIdx.x < (unsigned)P.multi_blocks) descending<kMaxR>(multi, std::make_integer_sequence<int, kMaxR - kMultiMinR + 1>{});
    descending<kMaxR>(one, std::make_integer_sequence<int, kMaxR - kSplitBins>{});
    if (WAVES == 2 || P.wide) {  // (the kernel for two waves per SIMD runs calls of few pairs only)
        descending<kSplitBins>(one, std::make_integer_sequence<int, kSplitBins>{});
        return;
    }
    if constexpr (WAVES > 2) {
        auto cls = [&](auto s_tag, auto rp_tag, int c) {
            if (A.bounds[c] >= A.bounds[c + 1]) return;
            const unsigned long long t0 = span_now();
            if (strip16_body<decltype(s_tag)::value, decltype(rp_tag)::value, TRACE>(A, c, lds, kBlockLds / kBlockWaves,
                                                                                     sblosum) &&
                !TRACE)
                span_add(A.span + (c & ~1), t0);
        };
        auto strips = [&](auto r_tag) {
            constexpr int R = decltype(r_tag)::value;
            constexpr int bin = R - 1;
            if (!((P.bins >> bin) & 1u)) return;
            std::integral_constant<int, 16> s16;
            std::integral_constant<int, 32> s32;
            if constexpr (R <= 4 && !TRACE) {  // (the traceback's launches have narrow = 0)
                if (R <= P.narrow) {
                    cls(s16, std::integral_constant<int, 4 * R>{}, 2 * bin + 1);
                    cls(s16, std::integral_constant<int, 4 * R - 2>{}, 2 * bin);
                    return;
                }
            }
            cls(s32, std::integral_constant<int, 2 * R>{}, 2 * bin + 1);
            cls(s32, std::integral_constant<int, 2 * R - 1>{}, 2 * bin);
        };
        descending<kSplitBins>(strips, std::make_integer_sequence<int, kSplitBins>{});
    }
}

}  // namespace

int sw16_waves() { return kBlockWaves; }
int sw16_step_words() { return kWave * dir_words<kMaxR>(); }

hipError_t launch_sw16_bound(int64_t npairs, const SwArgs &A, const TraceRule &T, int8_t *bin_of,
                             unsigned long long *counters, hipStream_t s) {
    // a resident grid (four blocks per CU: 128 registers) draining the list
    const int64_t per_block = 2 * kWave / kBoundLanes * kBoundWaves;
    const int blocks = (int)std::min<int64_t>(256 * 4, (npairs + per_block - 1) / per_block);
    sw16_bound_kernel<<<blocks, 64 * kBoundWaves, 0, s>>>(A, T, bin_of, counters);
    return hipGetLastError();
}

hipError_t launch_sw16_windows(int64_t npairs, const Sw16Launch &P, const SwArgs &A, int *win, int *nwin,
                               hipStream_t s) {
    sw16_windows_kernel<<<(unsigned)((npairs + kWindowBlock - 1) / kWindowBlock), kWindowBlock, 0, s>>>(
        A.pairs, A.idx, A.bounds, P, win, nwin);
    return hipGetLastError();
}

hipError_t launch_sw16(bool trace, const Sw16Launch &P, const SwArgs &A, hipStream_t s) {
    if (trace && P.lean)
        sw16_kernel<true, 2><<<P.blocks, 64 * kBlockWaves, 0, s>>>(A, P);
    else if (trace)
        sw16_kernel<true, 3><<<P.blocks, 64 * kBlockWaves, 0, s>>>(A, P);
    else
        sw16_kernel<false, 3><<<P.blocks, 64 * kBlockWaves, 0, s>>>(A, P);
    return hipGetLastError();
}

}  // namespace pastis
