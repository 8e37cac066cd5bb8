// Smith-Waterman in 16-bit lanes: two pairs in the halves of every DP word.
#include <algorithm>

#include "sw16.hpp"

namespace pastis {
namespace {

// Two pairs per wave in the 16-bit halves of every DP word (pair P low, Q
// high), same lane layout as the 32-bit pass, one strip (R <= 16).  The two
// pairs share their shorter sequence a (pairs are sorted by bin, then a, then
// the longer b first), so one int8 profile serves both; a wave whose two
// items differ in a runs them one after the other.  Only G = H - (o + e) is
// kept per row: the diagonal term H(i-1, j-1) + s becomes G(i-1, j-1) +
// (s + o + e), with the biased scores s + o + e >= 0 in the profile (each
// row's two bytes are spread into the halves by one byte permute).  Padding
// residues score -(o + e).  Each row keeps only its maximum: cells outside a
// pair (padding rows and columns, columns before the first) score strictly
// below its best real cell, so the score and the first row holding it are
// exact; the end column is found later, for the pairs that need it (end_b =
// -1 here).  Scores stay below 11 * 1024, far from the 16-bit limit.
// The gap states are kept floored at zero, E' = max(E, 0) and F' = max(F, 0):
// their recurrences stay closed (max(E' - e, 0) = max(E - e, 0) for e >= 0,
// one saturating subtract), and max(d, E', F') then already holds the local
// alignment's zero, so a cell takes 10 packed ops instead of 11.
constexpr int kMax16R = kMaxR;

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

template <int R, int WPB, bool MULTI>
__device__ __forceinline__ bool wave16_body(const SwArgs &A, int bin, char *lds, const int8_t *sblosum,
                                            WaveLds<WPB> &L) {
    static_assert(R > 8 && R <= kMax16R, "more than 512 rows per strip");
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
    const int item_begin = A.bounds[2 * bin];
    bool any = false;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    const int item_end = A.bounds[2 * bin + 2];
    const uint32_t OE2 = (uint32_t)go_ge * 0x10001u, GE2 = (uint32_t)ge * 0x10001u;
    const uint32_t G0 = ((uint32_t)(-go_ge) & 0xFFFFu) * 0x10001u;  // G of an H = 0 cell
    uint32_t *bnd_g = nullptr, *bnd_f = nullptr;
    if constexpr (MULTI) {
        bnd_g = (uint32_t *)A.scratch + ((int64_t)blockIdx.x * WPB + wave) * A.scratch_per_wave;
        bnd_f = bnd_g + A.scratch_per_wave / 2;
    }
    int par = 0;

    for (;;) {
        // every thread has read the last window before the round loop's
        // first barrier, so thread 0 may claim the next one
        if (threadIdx.x == 0) s_take = atomicAdd(A.queue + 2 * bin, NI);
        __syncthreads();
        const int64_t w = item_begin + (int64_t)s_take;
        if (w >= item_end) break;
        any = true;
        const int nit = (int)min((int64_t)NI, item_end - w);
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
            // best row of each pair: (score << 16) | (0xFFFF - row), maximised
            unsigned kp = 0u, kq = 0u;
            for (int sidx = 0; sidx < nstrips; ++sidx) {
                const int base = sidx * RS;
                if (sidx > 0) __syncthreads();  // every wave is done with the last strip's profile
                build_profile16<R, kWave, WPB>(prof, sblosum, codes + dA.a_off + base, laA - base, lane, wave,
                                               go_ge);
                __syncthreads();
                const bool from_above = MULTI && sidx > 0;
                const bool to_below = MULTI && sidx + 1 < nstrips;
                uint32_t G[R], E[R], M[R];
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    G[r] = G0;
                    E[r] = 0u;
                    M[r] = 0u;
                }
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
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        // byte r of P's and Q's words into the two halves
                        const uint32_t sel =
                            (uint32_t)(r & 3) | 0x0C00u | ((uint32_t)(4 + (r & 3)) << 16) | 0x0C000000u;
                        const short2_t sig =
                            s2(__builtin_amdgcn_perm(prof_word<R>(cQ, r), prof_word<R>(cP, r), sel));
                        const short2_t e = pmax(psubs(s2(E[r]), GE2), s2(G[r]));
                        const short2_t f = pmax(psubs(fu, GE2), gu);
                        const short2_t d = gd + sig;
                        const short2_t h = pmax(d, pmax(e, f));
                        gd = s2(G[r]);
                        const short2_t g = h - s2(OE2);
                        G[r] = u2(g);
                        E[r] = u2(e);
                        M[r] = u2(pmax(s2(M[r]), h));
                        gu = g;
                        fu = f;
                    }
                    glast = G[R - 1];
                    flast = u2(fu);
                    gprev = rg;
                    if (to_below) {
                        const int j = t - (kWave - 1);
                        if (lane == kWave - 1 && j >= 0 && j < lb) {
                            bnd_g[j] = glast;
                            bnd_f[j] = flast;
                        }
                    }
                };
                // two steps per iteration, so the old and new G registers can
                // swap roles instead of being copied back every step
                int t = 0;
                if (from_above) {
                    for (; t + 1 < lb; t += 2) {
                        step(t, std::true_type{});
                        step(t + 1, std::true_type{});
                    }
                    if (t < lb) step(t++, std::true_type{});
                }
                for (; t + 1 < steps; t += 2) {
                    step(t, std::false_type{});
                    step(t + 1, std::false_type{});
                }
                if (t < steps) step(t, std::false_type{});
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const int row = base + lane * R + r;
                    const unsigned rk = 0xFFFFu - (unsigned)row;
                    if (row < laA) {
                        kp = max(kp, ((M[r] & 0xFFFFu) << 16) | rk);
                        kq = max(kq, (M[r] & 0xFFFF0000u) | rk);
                    }
                }
                if (to_below) __threadfence_block();  // lane 0 of the next strip reads lane 63's row
            }
            kp = wave_max_u32(kp);
            kq = wave_max_u32(kq);
            if (lane == 0) {
                SwPass1Out o;
                o.end_b = -1;
                o.pad = 0;
                if (actP) {
                    o.score = (int32_t)(kp >> 16);
                    o.end_a = o.score > 0 ? (int32_t)(0xFFFFu - (kp & 0xFFFFu)) : -1;
                    out[qP] = o;
                }
                if (actQ) {
                    o.score = (int32_t)(kq >> 16);
                    o.end_a = o.score > 0 ? (int32_t)(0xFFFFu - (kq & 0xFFFFu)) : -1;
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


// One rows class of a bin's pairs (sorted by rows class first): class c holds
// the items [bounds[2 bin + c], bounds[2 bin + c + 1]) and has its own queue.
template <int S, int RP>
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
    const int item_begin = A.bounds[cls], item_end = A.bounds[cls + 1];
    int *const counter = A.queue + cls;
    bool any = false;
    const uint32_t OE2 = (uint32_t)go_ge * 0x10001u, GE2 = (uint32_t)ge * 0x10001u;
    const uint32_t G0 = ((uint32_t)(-go_ge) & 0xFFFFu) * 0x10001u;  // G of an H = 0 cell

    for (int64_t w = take_from(counter, item_begin, NI); w < item_end; w = take_from(counter, item_begin, NI)) {
        any = true;
        const int nit = (int)min((int64_t)NI, item_end - w);
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
            uint32_t G[RP], E[RP], M[RP];
#pragma unroll
            for (int r = 0; r < RP; ++r) {
                G[r] = G0;
                E[r] = 0u;
                M[r] = 0u;
            }
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
#pragma unroll
                for (int r = 0; r < RP; ++r) {
                    const uint32_t sel =
                        (uint32_t)(r & 3) | 0x0C00u | ((uint32_t)(4 + (r & 3)) << 16) | 0x0C000000u;
                    const short2_t sig = s2(__builtin_amdgcn_perm(prof_word<RP>(cQ, r), prof_word<RP>(cP, r), sel));
                    const short2_t e = pmax(psubs(s2(E[r]), GE2), s2(G[r]));
                    const short2_t f = pmax(psubs(fu, GE2), gu);
                    const short2_t d = gd + sig;
                    const short2_t h = pmax(d, pmax(e, f));
                    gd = s2(G[r]);
                    const short2_t g = h - s2(OE2);
                    G[r] = u2(g);
                    E[r] = u2(e);
                    M[r] = u2(pmax(s2(M[r]), h));
                    gu = g;
                    fu = f;
                }
                glast = G[RP - 1];
                flast = u2(fu);
                gprev = rg;
            };
            if constexpr (kAhead) {
                feed(0);
                wP = at(cres & 0xFFFFu);
                wQ = at(cres >> 16);
            }
            int t = 0;
            for (; t + 1 < steps; t += 2) {
                step(t);
                step(t + 1);
            }
            if (t < steps) step(t);
            unsigned kp = 0u, kq = 0u;
#pragma unroll
            for (int r = 0; r < RP; ++r) {
                const int row = pos * RP + r;
                const unsigned rk = 0xFFFFu - (unsigned)row;
                if (row < la) {
                    kp = max(kp, ((M[r] & 0xFFFFu) << 16) | rk);
                    kq = max(kq, (M[r] & 0xFFFF0000u) | rk);
                }
            }
            kp = strip_max_u32<S>(kp);
            kq = strip_max_u32<S>(kq);
            if (pos == 0) {
                SwPass1Out o;
                o.end_b = -1;
                o.pad = 0;
                if (actP) {
                    o.score = (int32_t)(kp >> 16);
                    o.end_a = o.score > 0 ? (int32_t)(0xFFFFu - (kp & 0xFFFFu)) : -1;
                    out[qP] = o;
                }
                if (actQ) {
                    o.score = (int32_t)(kq >> 16);
                    o.end_a = o.score > 0 ? (int32_t)(0xFFFFu - (kq & 0xFFFFu)) : -1;
                    out[qQ] = o;
                }
            }
            doneP = doneP || actP;
            doneQ = doneQ || actQ;
        }
    }
    return any;
}

// ---------------------------------------------------------------- group kernels

// f(integral HI), f(integral HI - 1), ...
template <int HI, typename F, int... I>
__device__ __forceinline__ void descending(F &f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, HI - I>{}), ...);
}

// The bins of a group, tallest first, in one launch (see the group launches
// of the 32-bit kernels); a bin of up to 8 rows per lane runs its taller rows
// class first.
template <int HI, int... I>
__device__ __forceinline__ void strip_bins(const SwArgs &A, uint32_t bins, int narrow, char *lds, size_t wave_bytes,
                                           const int8_t *sblosum, std::integer_sequence<int, I...>) {
    auto cls = [&](auto s_tag, auto rp_tag, int c) {
        if (A.bounds[c] >= A.bounds[c + 1]) return;
        const unsigned long long t0 = span_now();
        if (strip16_body<decltype(s_tag)::value, decltype(rp_tag)::value>(A, c, lds, wave_bytes, sblosum))
            span_add(A.span + (c & ~1), t0);
    };
    auto one = [&](auto r_tag) {
        constexpr int R = decltype(r_tag)::value;
        constexpr int bin = R - 1;
        if (!((bins >> bin) & 1u)) return;
        std::integral_constant<int, 16> s16;
        std::integral_constant<int, 32> s32;
        if constexpr (R <= 4) {
            // strips of 16 lanes with 4 R rows per lane (eight pairs per
            // wave), or, when not narrow, of 32 lanes with 2 R rows (four
            // pairs per wave: fewer pairs that must share their sequence a)
            if (R <= narrow) {
                cls(s16, std::integral_constant<int, 4 * R>{}, 2 * bin + 1);
                cls(s16, std::integral_constant<int, 4 * R - 2>{}, 2 * bin);
                return;
            }
        }
        cls(s32, std::integral_constant<int, 2 * R>{}, 2 * bin + 1);
        cls(s32, std::integral_constant<int, 2 * R - 1>{}, 2 * bin);
    };
    descending<HI>(one, std::integer_sequence<int, I...>{});
}

constexpr int kStripWaves = 4;

template <int LO, int HI>
__global__ __launch_bounds__(64 * kStripWaves) void sw16s_pass1_kernel(SwArgs A, uint32_t bins, int narrow) {
    // strips of 16 lanes with 4 R rows each take no more than those of 32
    // lanes with 2 R rows: sixteen bytes per code and lane at most
    constexpr size_t kWaveBytes = kProfCodes * (HI <= 4 ? 16 * 16 : 32 * 16);
    __shared__ __align__(16) char lds[kStripWaves * kWaveBytes];
    __shared__ int8_t sblosum[kProfCodes * kProfCodes];
    load_blosum(sblosum, A.blosum);
    strip_bins<HI>(A, bins, narrow, lds, kWaveBytes, sblosum, std::make_integer_sequence<int, HI - LO + 1>{});
}

template <int LO, int HI, int WPB, bool MULTI>
__global__ __launch_bounds__(64 * WPB) void sw16_pass1_kernel(SwArgs A, uint32_t bins, int) {
    __shared__ __align__(16) char lds[kProfCodes * kWave * sizeof(ProfWord<HI>)];
    __shared__ int8_t sblosum[kProfCodes * kProfCodes];
    __shared__ WaveLds<WPB> L;
    load_blosum(sblosum, A.blosum);
    auto one = [&](auto r_tag) {
        constexpr int R = decltype(r_tag)::value;
        constexpr int bin = MULTI ? kMulti16Bin + R - kMultiMinR : R - 1;
        if (!((bins >> bin) & 1u) || A.bounds[2 * bin] >= A.bounds[2 * bin + 2]) return;
        const unsigned long long t0 = span_now();
        if (wave16_body<R, WPB, MULTI>(A, bin, lds, sblosum, L)) span_add(A.span + 2 * bin, t0);
        __syncthreads();  // every wave has read the last window before the next bin's first claim
    };
    descending<HI>(one, std::make_integer_sequence<int, HI - LO + 1>{});
}

// one-strip bins of more than 512 rows share a profile between the waves of a
// block, and a block runs one round per distinct sequence a of its window:
// two waves (four pairs) per block keep those rounds few where sequences have
// few partners, and eight (six) such blocks per CU keep four (three) waves
// per SIMD within LDS
constexpr int kWpbShared = 2;
constexpr int kWpbMulti = 4;

}  // namespace

int sw16_waves(int group) { return group < 2 ? kStripWaves : group < 4 ? kWpbShared : kWpbMulti; }

hipError_t launch_sw16(int group, int blocks, int narrow, const SwArgs &A, uint32_t bins, hipStream_t s) {
    typedef void (*Kernel)(SwArgs, uint32_t, int);
    static const Kernel kernels[5] = {sw16s_pass1_kernel<1, 4>, sw16s_pass1_kernel<5, 8>,
                                      sw16_pass1_kernel<9, 12, kWpbShared, false>,
                                      sw16_pass1_kernel<13, 16, kWpbShared, false>,
                                      sw16_pass1_kernel<9, 16, kWpbMulti, true>};
    kernels[group]<<<blocks, 64 * sw16_waves(group), 0, s>>>(A, bins, narrow);
    return hipGetLastError();
}

}  // namespace pastis
