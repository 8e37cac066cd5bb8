// Device primitives: fill, exclusive scan, and a stable LSD radix sort of
// 64-bit keys with 32-bit payloads.  All are enqueued on a stream with no host
// round trip; temporary storage comes from the caller.
#include "internal.hpp"
#include "prim.hpp"

namespace pastis {
namespace {

constexpr int kWave = 64;
constexpr int kScanThreads = 256;
constexpr int kScanItems = 16;
constexpr int kScanTile = kScanThreads * kScanItems;

template <typename T>
__global__ void fill_kernel(T *p, int64_t n, T v) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

// inclusive prefix over the 256 threads of a block
__device__ __forceinline__ uint64_t block_inclusive(uint64_t v, uint64_t *smem_waves) {
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const uint64_t o = __shfl_up(v, d, kWave);
        if (lane >= d) v += o;
    }
    if (lane == kWave - 1) smem_waves[wave] = v;
    __syncthreads();
    uint64_t add = 0;
    for (int w = 0; w < wave; ++w) add += smem_waves[w];
    __syncthreads();
    return v + add;
}

template <typename TIn>
__global__ __launch_bounds__(kScanThreads) void scan_partials_kernel(const TIn *__restrict__ in, int64_t n,
                                                                     uint64_t *__restrict__ partial) {
    __shared__ uint64_t sw[kScanThreads / kWave];
    const int64_t base = (int64_t)blockIdx.x * kScanTile;
    uint64_t s = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        const int64_t i = base + (int64_t)k * kScanThreads + threadIdx.x;
        if (i < n) s += (uint64_t)in[i];
    }
    const uint64_t inc = block_inclusive(s, sw);
    if (threadIdx.x == kScanThreads - 1) partial[blockIdx.x] = inc;
}

template <typename TIn, typename TOut>
__global__ __launch_bounds__(kScanThreads) void scan_tiles_kernel(const TIn *__restrict__ in, int64_t n,
                                                                  const uint64_t *__restrict__ offs,
                                                                  TOut *__restrict__ out, TOut *__restrict__ total) {
    __shared__ uint64_t sw[kScanThreads / kWave];
    const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
    uint64_t v[kScanItems];
    uint64_t s = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        const int64_t i = base + k;
        v[k] = (i < n) ? (uint64_t)in[i] : 0;
        s += v[k];
    }
    const uint64_t inc = block_inclusive(s, sw);
    uint64_t run = inc - s + (offs ? offs[blockIdx.x] : 0);
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        const int64_t i = base + k;
        if (i < n) out[i] = (TOut)run;
        run += v[k];
    }
    if (total && blockIdx.x == gridDim.x - 1 && threadIdx.x == kScanThreads - 1) *total = (TOut)run;
}

// ---- radix sort (8-bit digits, stable) ----
constexpr int kSortThreads = 256;
constexpr int kSortItems = 16;  // per thread per pass over a tile
constexpr int kSortTile = kSortThreads * kSortItems;
constexpr int kWavesPerSortBlock = kSortThreads / kWave;
// Middle sizes, up to kMidMax keys: tiles of half the size, so that the chip
// has more of them, and a histogram of one row per tile, which every scatter
// block sums for itself (a row is 1 KB, at most kMidMax / kMidTile of them,
// from L2).  A pass is then two launches instead of five: 33 us with the scan
// for 250,000 keys, 17 without.  A call of five passes (cluster scores) takes 136
// us instead of 202 for 2^16 keys and 168 instead of 271 for 2^18.  The line bounds
// the rows to sum, which grow as the square of the keys; it is on the safe side
// (332 us instead of 402 for 2^20).
constexpr int kMidItems = 8;
constexpr int kMidTile = kSortThreads * kMidItems;
constexpr int64_t kMidMax = 1 << 18;

// FUSED: hist rows by tile, else by digit
template <int ITEMS, bool FUSED>
__global__ __launch_bounds__(kSortThreads) void radix_hist_kernel(const uint64_t *__restrict__ keys, int64_t n,
                                                                  int shift, int nblocks, uint32_t *__restrict__ hist) {
    __shared__ uint32_t h[256];
    h[threadIdx.x] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * (kSortThreads * ITEMS);
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const int64_t i = base + (int64_t)k * kSortThreads + threadIdx.x;
        if (i < n) atomicAdd(&h[(keys[i] >> shift) & 0xFF], 1u);
    }
    __syncthreads();
    hist[FUSED ? (int64_t)blockIdx.x * 256 + threadIdx.x : (int64_t)threadIdx.x * nblocks + blockIdx.x] =
        h[threadIdx.x];
}

// exclusive scan of 256 counts in LDS (one wave, four per lane)
__device__ __forceinline__ void wave_scan256(uint32_t *c, int lane) {
    uint32_t c4[4], sum = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        c4[j] = c[4 * lane + j];
        sum += c4[j];
    }
    uint32_t inc = sum;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const uint32_t o = (uint32_t)__shfl_up((int)inc, off, kWave);
        if (lane >= off) inc += o;
    }
    uint32_t run = inc - sum;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        c[4 * lane + j] = run;
        run += c4[j];
    }
}

// the lanes of the wave (of those with ok) that hold digit d
__device__ __forceinline__ uint64_t digit_peers(bool ok, int d) {
    uint64_t peers = __ballot(ok);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        const uint64_t bal = __ballot((d >> b) & 1);
        peers &= ((d >> b) & 1) ? bal : ~bal;
    }
    return peers;
}

// One tile per block.  The tile is ranked stably by digit in LDS (each wave
// ranks its contiguous quarter 64 elements at a time with ballots), then
// written out in digit order, so a digit's run of the tile goes to
// consecutive addresses from consecutive threads.
template <int ITEMS, bool FUSED>
__global__ __launch_bounds__(kSortThreads) void radix_scatter_kernel(
    const uint64_t *__restrict__ keys, const uint32_t *__restrict__ vals, int64_t n, int shift, int nblocks,
    const uint64_t *__restrict__ offs, const uint32_t *__restrict__ hist, uint64_t *__restrict__ okeys,
    uint32_t *__restrict__ ovals) {
    constexpr int kTile = kSortThreads * ITEMS;
    constexpr int kWaveTile = kTile / kWavesPerSortBlock;  // consecutive elements per wave
    constexpr int kWaveChunks = kWaveTile / kWave;
    __shared__ __align__(16) uint64_t skey[kTile];
    __shared__ uint32_t sval[kTile];
    __shared__ uint32_t whist[kWavesPerSortBlock][256];  // then each wave's next local slot per digit
    __shared__ uint32_t dstart[256];                     // the digit's first slot in the tile
    __shared__ uint64_t gbase[256];                      // the digit's first output address of this tile
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    for (int d = threadIdx.x; d < kWavesPerSortBlock * 256; d += kSortThreads) (&whist[0][0])[d] = 0;
    __syncthreads();
    const int64_t tstart = (int64_t)blockIdx.x * kTile;
    const int64_t wstart = tstart + (int64_t)wave * kWaveTile;
    uint64_t k[kWaveChunks];
    uint32_t v[kWaveChunks];
#pragma unroll
    for (int c = 0; c < kWaveChunks; ++c) {
        const int64_t i = wstart + c * kWave + lane;
        const bool ok = i < n;
        k[c] = ok ? keys[i] : 0;
        v[c] = ok ? vals[i] : 0;
        if (ok) atomicAdd(&whist[wave][(k[c] >> shift) & 0xFF], 1u);
    }
    __syncthreads();
    {
        const int d = threadIdx.x;  // 256 threads, one digit each
        if constexpr (!FUSED) gbase[d] = offs[(int64_t)d * nblocks + blockIdx.x];
        uint32_t tot = 0;
        for (int w = 0; w < kWavesPerSortBlock; ++w) tot += whist[w][d];
        dstart[d] = tot;  // the digit's count, scanned below
    }
    __syncthreads();
    if (wave == 0) wave_scan256(dstart, lane);
    if constexpr (FUSED) {
        // each wave sums a quarter of the rows, four digits per lane: all of
        // them, and those of the tiles before this one
        uint32_t(*const stot)[256] = (uint32_t(*)[256])skey;  // (the tile's keys come later)
        uint32_t(*const sbef)[256] = stot + kWavesPerSortBlock;
        static_assert(2 * kWavesPerSortBlock * 256 * sizeof(uint32_t) <= sizeof(skey), "row sums fit");
        uint4 all = make_uint4(0, 0, 0, 0), bef = all;
#pragma unroll 8
        for (int b = wave; b < nblocks; b += kWavesPerSortBlock) {
            const uint4 r = ((const uint4 *)hist)[b * 64 + lane];
            const bool earlier = b < (int)blockIdx.x;
            all.x += r.x, all.y += r.y, all.z += r.z, all.w += r.w;
            bef.x += earlier ? r.x : 0u, bef.y += earlier ? r.y : 0u;
            bef.z += earlier ? r.z : 0u, bef.w += earlier ? r.w : 0u;
        }
        ((uint4 *)stot[wave])[lane] = all;
        ((uint4 *)sbef[wave])[lane] = bef;
        __syncthreads();
        const int d = threadIdx.x;
        uint32_t tot = 0, before = 0;
#pragma unroll
        for (int w = 0; w < kWavesPerSortBlock; ++w) {
            tot += stot[w][d];
            before += sbef[w][d];
        }
        __syncthreads();
        stot[0][d] = tot;
        __syncthreads();
        if (wave == 0) wave_scan256(stot[0], lane);
        __syncthreads();
        gbase[d] = stot[0][d] + before;
    }
    __syncthreads();
    {
        const int d = threadIdx.x;
        uint32_t run = dstart[d];
        for (int w = 0; w < kWavesPerSortBlock; ++w) {
            const uint32_t c = whist[w][d];
            whist[w][d] = run;
            run += c;
        }
    }
    __syncthreads();
    const uint64_t lt = (1ull << lane) - 1ull;
#pragma unroll
    for (int c = 0; c < kWaveChunks; ++c) {
        const int64_t i = wstart + c * kWave + lane;
        const bool ok = i < n;
        const int d = (int)((k[c] >> shift) & 0xFF);
        const uint64_t peers = digit_peers(ok, d);
        const int before = __popcll(peers & lt);
        uint32_t slot = 0;
        if (ok) slot = whist[wave][d] + (uint32_t)before;
        __builtin_amdgcn_wave_barrier();
        if (ok && before == 0) whist[wave][d] += (uint32_t)__popcll(peers);
        __builtin_amdgcn_wave_barrier();
        if (ok) {
            skey[slot] = k[c];
            sval[slot] = v[c];
        }
    }
    __syncthreads();
    const int count = (int)((n - tstart) < (int64_t)kTile ? (n - tstart) : (int64_t)kTile);
    for (int p = threadIdx.x; p < count; p += kSortThreads) {
        const uint64_t key = skey[p];
        const int d = (int)((key >> shift) & 0xFF);
        const uint64_t pos = gbase[d] + (uint64_t)(p - (int)dstart[d]);
        okeys[pos] = key;
        ovals[pos] = sval[p];
    }
}

// Small sizes: one block of 16 waves keeps the keys in LDS through every pass
// (a wave's contiguous 256 in its registers), in place.  A call's pairing sort
// of 3,000 keys took 18 launches and 200 us, mostly launches of a few us each;
// one launch takes 19.  Cluster scores of 1,024 keys take 65 us and 85 with the
// middle path, of 4,096 77 and 106; the size is what the keys' LDS allows.
constexpr int kOneWaves = 16, kOneChunks = 4;
constexpr int kOneMax = kOneWaves * kOneChunks * kWave;
__global__ __launch_bounds__(kOneWaves *kWave) void radix_one_kernel(uint64_t *__restrict__ keys,
                                                                     uint32_t *__restrict__ vals, int n, int bits) {
    __shared__ uint64_t skey[kOneMax];
    __shared__ uint32_t sval[kOneMax];
    __shared__ uint16_t whist[kOneWaves][256];  // counts, then each wave's next slot per digit
    __shared__ uint32_t dstart[256];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const int wstart = wave * kOneChunks * kWave;
    const uint64_t lt = (1ull << lane) - 1ull;
    uint64_t k[kOneChunks];
    uint32_t v[kOneChunks];
#pragma unroll
    for (int c = 0; c < kOneChunks; ++c) {
        const int i = wstart + c * kWave + lane;
        k[c] = i < n ? keys[i] : 0;
        v[c] = i < n ? vals[i] : 0;
    }
    for (int shift = 0; shift < bits; shift += 8) {
        for (int d = lane; d < 256; d += kWave) whist[wave][d] = 0;
        __builtin_amdgcn_wave_barrier();
        uint32_t rank[kOneChunks];  // among the wave's keys of the digit
#pragma unroll
        for (int c = 0; c < kOneChunks; ++c) {
            const bool ok = wstart + c * kWave + lane < n;
            const int d = (int)((k[c] >> shift) & 0xFF);
            const uint64_t peers = digit_peers(ok, d);
            const int before = __popcll(peers & lt);
            rank[c] = ok ? whist[wave][d] + (uint32_t)before : 0u;
            __builtin_amdgcn_wave_barrier();
            if (ok && before == 0) whist[wave][d] = (uint16_t)(rank[c] + (uint32_t)__popcll(peers));
            __builtin_amdgcn_wave_barrier();
        }
        __syncthreads();
        if (threadIdx.x < 256) {
            const int d = threadIdx.x;
            uint32_t run = 0;
#pragma unroll
            for (int w = 0; w < kOneWaves; ++w) {
                const uint32_t c = whist[w][d];
                whist[w][d] = (uint16_t)run;
                run += c;
            }
            dstart[d] = run;
        }
        __syncthreads();
        if (wave == 0) wave_scan256(dstart, lane);
        __syncthreads();
#pragma unroll
        for (int c = 0; c < kOneChunks; ++c) {
            if (wstart + c * kWave + lane >= n) continue;
            const int d = (int)((k[c] >> shift) & 0xFF);
            const uint32_t slot = dstart[d] + whist[wave][d] + rank[c];
            skey[slot] = k[c];
            sval[slot] = v[c];
        }
        __syncthreads();
#pragma unroll
        for (int c = 0; c < kOneChunks; ++c) {
            const int i = wstart + c * kWave + lane;
            k[c] = i < n ? skey[i] : 0;
            v[c] = i < n ? sval[i] : 0;
        }
    }
#pragma unroll
    for (int c = 0; c < kOneChunks; ++c) {
        const int i = wstart + c * kWave + lane;
        if (i >= n) continue;
        keys[i] = k[c];
        vals[i] = v[c];
    }
}

__global__ void iota_kernel(uint32_t *p, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = (uint32_t)i;
}

inline unsigned grid_for(int64_t n, int threads) {
    int64_t b = (n + threads - 1) / threads;
    if (b > 16384) b = 16384;
    return (unsigned)(b < 1 ? 1 : b);
}

}  // namespace

template <typename T>
hipError_t fill(T *p, int64_t n, T v, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    fill_kernel<T><<<grid_for(n, 256), 256, 0, s>>>(p, n, v);
    return hipGetLastError();
}
template hipError_t fill<int>(int *, int64_t, int, hipStream_t);
template hipError_t fill<uint32_t>(uint32_t *, int64_t, uint32_t, hipStream_t);
template hipError_t fill<int64_t>(int64_t *, int64_t, int64_t, hipStream_t);
template hipError_t fill<uint64_t>(uint64_t *, int64_t, uint64_t, hipStream_t);
template hipError_t fill<unsigned long long>(unsigned long long *, int64_t, unsigned long long, hipStream_t);

hipError_t iota(uint32_t *p, int64_t n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    iota_kernel<<<grid_for(n, 256), 256, 0, s>>>(p, n);
    return hipGetLastError();
}

size_t scan_temp_bytes(int64_t n) {
    size_t total = 0;
    int64_t m = n;
    while (m > 1) {
        m = (m + kScanTile - 1) / kScanTile;
        total += sizeof(uint64_t) * (size_t)(2 * m + 2);
    }
    return total + 256;
}

template <typename TIn, typename TOut>
hipError_t exclusive_scan(const TIn *in, int64_t n, TOut *out, TOut *total, void *temp, hipStream_t s) {
    if (n <= 0) {
        if (total) return fill<TOut>(total, 1, (TOut)0, s);
        return hipSuccess;
    }
    const int64_t nb = (n + kScanTile - 1) / kScanTile;
    if (nb == 1) {
        scan_tiles_kernel<TIn, TOut><<<1, kScanThreads, 0, s>>>(in, n, nullptr, out, total);
        return hipGetLastError();
    }
    uint64_t *partial = (uint64_t *)temp;
    uint64_t *poffs = partial + nb + 1;
    void *rest = poffs + nb + 1;
    scan_partials_kernel<TIn><<<(unsigned)nb, kScanThreads, 0, s>>>(in, n, partial);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    e = exclusive_scan<uint64_t, uint64_t>(partial, nb, poffs, (uint64_t *)nullptr, rest, s);
    if (e != hipSuccess) return e;
    scan_tiles_kernel<TIn, TOut><<<(unsigned)nb, kScanThreads, 0, s>>>(in, n, poffs, out, total);
    return hipGetLastError();
}
template hipError_t exclusive_scan<uint32_t, uint64_t>(const uint32_t *, int64_t, uint64_t *, uint64_t *, void *,
                                                       hipStream_t);
template hipError_t exclusive_scan<uint32_t, uint32_t>(const uint32_t *, int64_t, uint32_t *, uint32_t *, void *,
                                                       hipStream_t);
template hipError_t exclusive_scan<uint64_t, uint64_t>(const uint64_t *, int64_t, uint64_t *, uint64_t *, void *,
                                                       hipStream_t);
template hipError_t exclusive_scan<int, int64_t>(const int *, int64_t, int64_t *, int64_t *, void *, hipStream_t);
template hipError_t exclusive_scan<uint8_t, uint32_t>(const uint8_t *, int64_t, uint32_t *, uint32_t *, void *,
                                                      hipStream_t);

size_t radix_temp_bytes(int64_t n) {
    const int64_t nb = (n + kSortTile - 1) / kSortTile;
    const int64_t h = 256 * (nb > 0 ? nb : 1);
    return sizeof(uint32_t) * (size_t)h + sizeof(uint64_t) * (size_t)h + scan_temp_bytes(h) + 256;
}

hipError_t radix_sort(uint64_t *keys, uint32_t *vals, uint64_t *keys_alt, uint32_t *vals_alt, int64_t n, int bits,
                      void *temp, hipStream_t s, bool *result_in_alt) {
    *result_in_alt = false;
    if (n <= 1) return hipSuccess;
    if (n <= kOneMax) {
        radix_one_kernel<<<1, kOneWaves * kWave, 0, s>>>(keys, vals, (int)n, bits);
        return hipGetLastError();
    }
    const bool mid = n <= kMidMax;
    const int64_t nb = mid ? (n + kMidTile - 1) / kMidTile : (n + kSortTile - 1) / kSortTile;
    // (middle sizes use the histogram alone, 4 bytes of 256 entries for tiles of
    // half the size: within the 12 bytes that radix_temp_bytes counts)
    uint32_t *hist = (uint32_t *)temp;
    uint64_t *offs = (uint64_t *)(hist + 256 * nb);
    void *stemp = offs + 256 * nb;
    uint64_t *k0 = keys, *k1 = keys_alt;
    uint32_t *v0 = vals, *v1 = vals_alt;
    for (int shift = 0; shift < bits; shift += 8) {
        hipError_t e;
        if (mid) {
            radix_hist_kernel<kMidItems, true><<<(unsigned)nb, kSortThreads, 0, s>>>(k0, n, shift, (int)nb, hist);
            if ((e = hipGetLastError()) != hipSuccess) return e;
            radix_scatter_kernel<kMidItems, true><<<(unsigned)nb, kSortThreads, 0, s>>>(
                k0, v0, n, shift, (int)nb, nullptr, hist, k1, v1);
        } else {
            radix_hist_kernel<kSortItems, false><<<(unsigned)nb, kSortThreads, 0, s>>>(k0, n, shift, (int)nb, hist);
            if ((e = hipGetLastError()) != hipSuccess) return e;
            e = exclusive_scan<uint32_t, uint64_t>(hist, 256 * nb, offs, (uint64_t *)nullptr, stemp, s);
            if (e != hipSuccess) return e;
            radix_scatter_kernel<kSortItems, false><<<(unsigned)nb, kSortThreads, 0, s>>>(
                k0, v0, n, shift, (int)nb, offs, nullptr, k1, v1);
        }
        if ((e = hipGetLastError()) != hipSuccess) return e;
        uint64_t *tk = k0;
        k0 = k1;
        k1 = tk;
        uint32_t *tv = v0;
        v0 = v1;
        v1 = tv;
        *result_in_alt = !*result_in_alt;
    }
    return hipSuccess;
}

}  // namespace pastis
