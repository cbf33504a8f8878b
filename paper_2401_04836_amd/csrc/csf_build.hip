// GPU construction of a CSF tree from coordinate lists (Sec. 2.1, "CSF representation").
//
// Steps, all on the device:
//   1. pack each coordinate tuple, permuted into level order, into one 64-bit key (outermost
//      level in the most significant bits) and check ranges; tuples that need 65 to 128 bits get a
//      second, more significant word holding the outer levels (no level straddles the two words);
//   2. stable radix sort of (key, value) -- lexicographic order in mode_order (own LSD sort, see
//      below; its first pass does step 1); with two-word keys of (key, original position);
//   3. per tile, count for every level the positions where the key prefix of that level
//      changes ("head" of a node); a duplicate coordinate is a position whose full key
//      equals its predecessor's;
//   4. scan the tile counts; the host reads the node totals and allocates the level arrays;
//   5. per tile, rank the heads (block scan) and emit idx[l], ptr[l] and the permuted values.
// The result is the canonical array layout documented in include/conststn.h.
#include <algorithm>
#include <cstring>
#include <type_traits>

#include "plan.hpp"

namespace cst {

constexpr int kTileThreads = 256;
constexpr int kItems = 8;
constexpr int kTile = kTileThreads * kItems;

struct Levels {
    int order;
    int word[CONSTSTN_MAX_ORDER];           // 0: the level's field lies in the low key word, 1: in the high one
    int shift[CONSTSTN_MAX_ORDER];          // bit offset of the level's field inside its word
    uint64_t mask[CONSTSTN_MAX_ORDER];      // field mask (after shifting)
    int64_t dim[CONSTSTN_MAX_ORDER];        // extent of the mode at this level
    const int32_t *coord[CONSTSTN_MAX_ORDER];
};

struct LevelOut {
    int32_t *idx[CONSTSTN_MAX_ORDER];
    int64_t *ptr[CONSTSTN_MAX_ORDER];
};

__device__ __forceinline__ uint64_t prefix_of(uint64_t key, int shift) {
    return shift >= 64 ? 0 : (key >> shift);
}

// keys_hi = nullptr for keys of one word
__global__ void __launch_bounds__(256)
pack_keys_kernel(int64_t nnz, Levels lv, uint64_t *keys, uint64_t *keys_hi, uint32_t *payload, int *flags) {
    int64_t n = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    const int64_t stride = int64_t(gridDim.x) * blockDim.x;
    bool bad = false;
    for (; n < nnz; n += stride) {
        uint64_t key = 0, hi = 0;
        for (int l = 0; l < lv.order; ++l) {
            int32_t c = lv.coord[l][n];
            if (c < 0 || int64_t(c) >= lv.dim[l]) { bad = true; c = 0; }
            if (lv.shift[l] < 64) {
                if (lv.word[l]) hi |= uint64_t(uint32_t(c)) << lv.shift[l];
                else key |= uint64_t(uint32_t(c)) << lv.shift[l];
            }
        }
        keys[n] = key;
        if (keys_hi) keys_hi[n] = hi;
        payload[n] = uint32_t(n);
    }
    if (bad) atomicOr(&flags[0], 1);
}

// out[i] = in[index[i]]
__global__ void __launch_bounds__(256)
gather_u64_kernel(int64_t n, const uint64_t *__restrict__ in, const uint32_t *__restrict__ index, uint64_t *__restrict__ out) {
    const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (i < n) out[i] = in[index[i]];
}

// A two-word key (hi = 0 throughout for keys of one word).  The prefix of level l is every bit from the
// level's field upwards: inside the high word for a level stored there, the whole high word plus the
// upper part of the low word otherwise.
struct Key2 { uint64_t hi, lo; };
template <bool WIDE>
__device__ __forceinline__ Key2 load_key(const uint64_t *keys, const uint64_t *keys_hi, int64_t n) {
    return Key2{WIDE ? keys_hi[n] : 0, keys[n]};
}
template <bool WIDE>
__device__ __forceinline__ bool same_prefix(const Levels &lv, int l, Key2 a, Key2 b) {
    if (WIDE && lv.word[l]) return prefix_of(a.hi, lv.shift[l]) == prefix_of(b.hi, lv.shift[l]);
    return (!WIDE || a.hi == b.hi) && prefix_of(a.lo, lv.shift[l]) == prefix_of(b.lo, lv.shift[l]);
}

// For every level the number of node heads inside each tile; leaf-level non-heads are duplicates.
template <bool WIDE>
__global__ void __launch_bounds__(kTileThreads)
count_heads_kernel(int64_t nnz, Levels lv, const uint64_t *__restrict__ keys, const uint64_t *__restrict__ keys_hi,
                   unsigned *__restrict__ tile_counts, int64_t ntiles, int *flags) {
    __shared__ unsigned wsum[CONSTSTN_MAX_ORDER][kTileThreads / 64];
    const int64_t tile = blockIdx.x;
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
    unsigned cnt[CONSTSTN_MAX_ORDER];                 // the same in every lane of a wavefront
#pragma unroll
    for (int l = 0; l < CONSTSTN_MAX_ORDER; ++l) cnt[l] = 0;
    bool dup = false;
    Key2 k[kItems], prev[kItems];
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
        const int64_t n = tile * kTile + i * kTileThreads + int(threadIdx.x), at = n < nnz ? n : nnz - 1;
        k[i] = load_key<WIDE>(keys, keys_hi, at);
        prev[i] = load_key<WIDE>(keys, keys_hi, at > 0 ? at - 1 : 0);
    }
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
        const int64_t n = tile * kTile + i * kTileThreads + int(threadIdx.x);
        const bool live = n < nnz;
#pragma unroll
        for (int l = 0; l < CONSTSTN_MAX_ORDER; ++l) {
            if (l < lv.order) {
                const bool head = live && (n == 0 || !same_prefix<WIDE>(lv, l, k[i], prev[i]));
                cnt[l] += unsigned(__popcll(__builtin_amdgcn_ballot_w64(head)));
                if (l == lv.order - 1 && live && !head) dup = true;
            }
        }
    }
    if (dup) atomicOr(&flags[1], 1);
    if (lane == 0) {
#pragma unroll
        for (int l = 0; l < CONSTSTN_MAX_ORDER; ++l) wsum[l][wave] = cnt[l];
    }
    __syncthreads();
    if (threadIdx.x < lv.order) {
        unsigned s = 0;
        for (int w = 0; w < kTileThreads / 64; ++w) s += wsum[threadIdx.x][w];
        tile_counts[int64_t(threadIdx.x) * ntiles + tile] = s;
    }
}

// Exclusive scan of the tile counts of every level (one block per level); totals[l] = node count.
// The block walks its row in chunks of 4096 counts, four adjacent ones per thread, and carries the
// running total from chunk to chunk.
template <typename OFF>
__global__ void __launch_bounds__(1024)
scan_tiles_kernel(const unsigned *__restrict__ tile_counts, OFF *__restrict__ tile_offsets,
                  int64_t ntiles, int64_t *totals) {
    __shared__ int64_t wtot[16];
    const int l = blockIdx.x;
    const unsigned *in = tile_counts + int64_t(l) * ntiles;
    OFF *out = tile_offsets + int64_t(l) * ntiles;
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    int64_t carry = 0;
    for (int64_t t0 = 0; t0 < ntiles; t0 += 4096) {
        const int64_t t = t0 + int64_t(threadIdx.x) * 4;
        unsigned v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = t + k < ntiles ? in[t + k] : 0u;
        const int64_t mine = int64_t(v[0]) + v[1] + v[2] + v[3];
        int64_t inc = mine;
        for (int off = 1; off < 64; off <<= 1) {
            const int64_t up = __shfl_up(inc, off, 64);
            if (lane >= off) inc += up;
        }
        if (lane == 63) wtot[wave] = inc;
        __syncthreads();
        int64_t before = 0, total = 0;
#pragma unroll
        for (int w = 0; w < 16; ++w) {
            const int64_t x = wtot[w];
            before += w < wave ? x : 0;
            total += x;
        }
        int64_t run = carry + before + inc - mine;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (t + k < ntiles) out[t + k] = OFF(run);
            run += v[k];
        }
        carry += total;
        __syncthreads();
    }
    if (threadIdx.x == 0) totals[l] = carry;
}

// ---- stable LSD radix sort of (key, payload) pairs, 8 or 9 bits per pass ---------------------
//
// A workgroup of eight wavefronts owns a tile of kSortTile consecutive pairs, wavefront w the w-th
// eighth of it.  Per pass: (1) every workgroup counts the digits of its tile; (2) scan_tiles_kernel
// (one block per digit value) turns the counts into the tile's starting offset inside each digit's
// bucket; (3) every workgroup re-reads its tile, ranks each pair among the pairs of the tile with the
// same digit that come before it (in a wavefront: 64 pairs at a time, one ballot per bit narrows the set
// of peers; across wavefronts: their digit counts), lays the keys out by digit in LDS and writes them
// from there, so that neighbouring threads write neighbouring addresses of a bucket, and then the
// payload through the same LDS.  Tiles are visited in index order inside a bucket and pairs in order
// inside a tile, so the sort is stable, which the CSF needs: equal keys (duplicates) must keep input
// order.
// The first pass of a CSF build reads the coordinates and packs the keys itself (COORDS), and the payload
// is the value: 8 bytes more per pair and pass than the position, but the values are then not read at random
// afterwards, a cache line each (emission at 76 M nonzeros: 1.75 -> 0.45 ms, a scatter 0.44 -> 0.55).
// Bound: memory; a pass moves 40 bytes per pair (32 with positions), and the writes more than their bytes: a run of a
// bucket that begins and ends inside a line.  So the tiles are as large as two workgroups of a compute unit with four
// wavefronts per SIMD allow: 12 pairs a lane instead of 16 (118 registers instead of 151), 8 wavefronts, counts of
// 2 bytes; runs of 12 (9 bits) or 24 pairs on average.  76 M pairs, whole build: 4 wavefronts of 16 pairs, 4096 a tile,
// 4.57 ms; of 12 pairs 4.75; 8 of 10 pairs 4.25, of 12 4.16, of 14 4.31; 12 of 16 pairs (one workgroup) 4.30.
// Neighbouring tiles write neighbouring runs and neighbouring counts: consecutive tiles are given to one
// XCD, whose L2 puts the parts of a cache line together (in launch order a build takes 1.1 ms longer).
// The counts of a tile are kept in kCountCopies copies, one for every eighth lane: lanes of skewed data that meet at one
// address wait for each other (the build takes 4.23 ms with one copy, 4.17 with four, 4.16 with eight).
// Build of 76 M nonzeros, 43 key bits: 7.2 ms with a packing pass, six passes of 8 bits and positions, 4.55 with
// tiles of 4096 -> 4.15 ms (per pass: counts 0.147, their scan 0.022, scatter 0.50: 4.8 TB/s of the 32 bytes it moves).
// Work space 33 bytes per pair, 25 with positions: a build that runs out of memory is tried again with those.
constexpr int kSortItems = 12;
constexpr int kSortWave = kSortItems * 64;            // pairs of one wavefront
constexpr int kSortWaves = 8;
constexpr int kSortThreads = 64 * kSortWaves;
constexpr int kSortTile = kSortWaves * kSortWave;
constexpr int kCountCopies = 8;                       // of a digit's count

// key[i] = keys (one word) of the nonzeros min(first + i * step, n - 1), i < COUNT; of fields that begin below bit
// `below` only.  The level is the outer loop: a lane's loads of one level are in flight together.
// ALL: every level's coordinates are read and tested, also of a level that holds no bit of the key (extent 1 above
// fields that fill 64 bits: its shift is 64); the result says whether one was out of range.
template <bool ALL, int COUNT, typename KEY>
__device__ __forceinline__ bool keys_of(const Levels &lv, int64_t first, int step, int64_t n, int below, KEY (&key)[COUNT]) {
    bool bad = false;
#pragma unroll
    for (int i = 0; i < COUNT; ++i) key[i] = 0;
    for (int l = 0; l < lv.order; ++l) {
        const int shift = lv.shift[l];
        if (!ALL && shift >= below) continue;
        const int32_t *coord = lv.coord[l];
        int32_t c[COUNT];
#pragma unroll
        for (int i = 0; i < COUNT; ++i) {
            const int64_t e = first + int64_t(i) * step;
            c[i] = coord[e < n ? e : n - 1];
        }
#pragma unroll
        for (int i = 0; i < COUNT; ++i) {
            const bool out = c[i] < 0 || int64_t(c[i]) >= lv.dim[l];
            bad = bad || out;
            if (shift < below) key[i] |= KEY(uint32_t(out ? 0 : c[i])) << shift;
        }
    }
    return bad;
}

template <int BITS, bool COORDS>
__global__ void __launch_bounds__(kSortThreads)
radix_count_kernel(int64_t n, const uint64_t *__restrict__ keys, Levels lv, int shift, unsigned *__restrict__ tile_counts,
                   int64_t ntiles) {
    constexpr int kBins = 1 << BITS;
    __shared__ unsigned hist[kBins * kCountCopies];
    unsigned *mine = hist + threadIdx.x % kCountCopies;
    // each XCD takes a contiguous range of tiles, as in the scatter: its L2 puts their counts together
    const int64_t per_xcd = (ntiles + 7) / 8, tile = int64_t(blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
    if (tile >= ntiles) return;
    for (int d = threadIdx.x; d < kBins * kCountCopies; d += kSortThreads) hist[d] = 0;
    __syncthreads();
    const int64_t base = tile * kSortTile;
    const int live = int(n - base < kSortTile ? n - base : int64_t(kSortTile));
    if (COORDS) {
        uint32_t key[kSortItems];                     // (what is out of range is reported by the scatter)
        keys_of<false>(lv, base + int(threadIdx.x), kSortThreads, n, BITS, key);
#pragma unroll
        for (int i = 0; i < kSortItems; ++i)
            if (i * kSortThreads + int(threadIdx.x) < live) atomicAdd(&mine[(key[i] & (kBins - 1)) * kCountCopies], 1u);
    } else {
        // two keys per load (tiles begin at multiples of 48 KB of a buffer that is aligned to 16 bytes)
        const ulonglong2 *pairs = reinterpret_cast<const ulonglong2 *>(keys + base);
        ulonglong2 k[kSortItems / 2];
#pragma unroll
        for (int i = 0; i < kSortItems / 2; ++i) {
            const int m = i * kSortThreads + int(threadIdx.x);
            k[i] = pairs[2 * m < live ? m : 0];       // (an odd last key: the buffers' allocations end on 256 bytes)
        }
#pragma unroll
        for (int i = 0; i < kSortItems / 2; ++i) {
            const int m = 2 * (i * kSortThreads + int(threadIdx.x));
            if (m < live) atomicAdd(&mine[(unsigned(k[i].x >> shift) & (kBins - 1)) * kCountCopies], 1u);
            if (m + 1 < live) atomicAdd(&mine[(unsigned(k[i].y >> shift) & (kBins - 1)) * kCountCopies], 1u);
        }
    }
    __syncthreads();
    for (int d = threadIdx.x; d < kBins; d += kSortThreads) {
        unsigned sum = 0;
#pragma unroll
        for (int c = 0; c < kCountCopies; ++c) sum += hist[d * kCountCopies + c];
        tile_counts[int64_t(d) * ntiles + tile] = sum;
    }
}

template <int BITS, bool COORDS, typename PAY>
__global__ void __launch_bounds__(kSortThreads) __attribute__((amdgpu_waves_per_eu(4)))
radix_scatter_kernel(int64_t n, const uint64_t *__restrict__ keys_in, const PAY *__restrict__ pay_in, Levels lv, int *flags,
                     uint64_t *__restrict__ keys_out, PAY *__restrict__ pay_out, int shift,
                     const uint32_t *__restrict__ tile_offsets, const int64_t *__restrict__ totals, int64_t ntiles) {
    constexpr int kBins = 1 << BITS, kPer = (kBins + kSortThreads - 1) / kSortThreads;      // digits of a thread
    __shared__ uint64_t lkey[kSortTile];                      // the tile's keys by digit, then its positions
    __shared__ uint16_t run[kSortWaves][kBins];                        // per wavefront: pairs of each digit seen so far, then the place of the next
    __shared__ uint32_t gbase[kBins];                         // address of the tile's place p holding digit d: gbase[d] + p (mod 2^32)
    __shared__ unsigned wsum[2][kSortWaves];
    const int wv = threadIdx.x / 64, lane = threadIdx.x % 64;
    // workgroup b runs on XCD b % 8: each XCD takes a contiguous range of tiles
    const int64_t per_xcd = (ntiles + 7) / 8, tile = int64_t(blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
    if (tile >= ntiles) return;
    const int64_t base = tile * kSortTile + int64_t(wv) * kSortWave;
    for (int d = threadIdx.x; d < kSortWaves * kBins; d += kSortThreads) (&run[0][0])[d] = 0;
    __syncthreads();
    const unsigned long long lt = (1ull << lane) - 1ull;
    uint64_t key[kSortItems];
    PAY pay[kSortItems];
    unsigned rank[kSortItems];                                // among the wavefront's earlier pairs of the same digit
    // pairs past the end sort last: all-ones keys, and they are the last pairs of the last tile
    if (COORDS) {
        const bool bad = keys_of<true>(lv, base + lane, 64, n, 64, key);
        if (bad) atomicOr(&flags[0], 1);
    }
#pragma unroll
    for (int i = 0; i < kSortItems; ++i) {
        const int64_t e = base + int64_t(i) * 64 + lane, at = e < n ? e : n - 1;
        if (!COORDS) key[i] = keys_in[at];
        pay[i] = pay_in[at];
    }
#pragma unroll
    for (int i = 0; i < kSortItems; ++i)
        if (base + int64_t(i) * 64 + lane >= n) key[i] = ~uint64_t(0);
#pragma unroll
    for (int i = 0; i < kSortItems; ++i) {
        const unsigned digit = unsigned(key[i] >> shift) & (kBins - 1);
        unsigned long long peers = ~0ull;
#pragma unroll
        for (int b = 0; b < BITS; ++b) {
            const bool bit = (digit >> b) & 1u;
            const unsigned long long m = __builtin_amdgcn_ballot_w64(bit);
            peers &= bit ? m : ~m;
        }
        const unsigned before = unsigned(__popcll(peers & lt));
        rank[i] = run[wv][digit] + before;
        __builtin_amdgcn_wave_barrier();
        if (before == 0) run[wv][digit] += uint16_t(__popcll(peers));      // the lowest peer advances the digit's count
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    {
        // a thread's digits: where they begin in the buckets' array and in the tile's layout, and inside that
        // where each wavefront's share begins
        const int d0 = int(threadIdx.x) * kPer;
        unsigned mine = 0, all = 0;
        for (int x = 0; x < kPer && d0 + x < kBins; ++x) {
            for (int w = 0; w < kSortWaves; ++w) mine += run[w][d0 + x];
            all += unsigned(totals[d0 + x]);
        }
        unsigned inc = mine, inc_all = all;
        for (int off = 1; off < 64; off <<= 1) {
            const unsigned up = __shfl_up(inc, off, 64), up_all = __shfl_up(inc_all, off, 64);
            if (lane >= off) { inc += up; inc_all += up_all; }
        }
        if (lane == 63) { wsum[0][wv] = inc; wsum[1][wv] = inc_all; }
        __syncthreads();
        unsigned first = inc - mine, bucket = inc_all - all;
        for (int w = 0; w < wv; ++w) { first += wsum[0][w]; bucket += wsum[1][w]; }
        for (int x = 0; x < kPer && d0 + x < kBins; ++x) {
            const int d = d0 + x;
            gbase[d] = bucket + tile_offsets[int64_t(d) * ntiles + tile] - first;
            bucket += unsigned(totals[d]);
            for (int w = 0; w < kSortWaves; ++w) {
                const unsigned c = run[w][d];
                run[w][d] = uint16_t(first);
                first += c;
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kSortItems; ++i) {
        rank[i] += run[wv][unsigned(key[i] >> shift) & (kBins - 1)];       // place in the tile's layout
        lkey[rank[i]] = key[i];
    }
    __syncthreads();
    const int64_t rest = n - tile * kSortTile;
    const int live_pairs = rest < kSortTile ? int(rest) : kSortTile;
    uint32_t pos[kSortItems];
#pragma unroll
    for (int i = 0; i < kSortItems; ++i) {
        const int p = i * kSortThreads + int(threadIdx.x);
        const uint64_t k = lkey[p];
        pos[i] = gbase[unsigned(k >> shift) & (kBins - 1)] + unsigned(p);
        if (p < live_pairs) keys_out[pos[i]] = k;
    }
    __syncthreads();
    PAY *lpay = reinterpret_cast<PAY *>(lkey);
#pragma unroll
    for (int i = 0; i < kSortItems; ++i) lpay[rank[i]] = pay[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kSortItems; ++i) {
        const int p = i * kSortThreads + int(threadIdx.x);
        if (p < live_pairs) pay_out[pos[i]] = lpay[p];
    }
}

static size_t up256(size_t bytes) { return (bytes + 255) / 256 * 256; }

constexpr int kSortBins = 512;                        // the pass tables hold digits of up to 9 bits

// bytes of pass tables a sort of n pairs needs (handed in by callers that keep one allocation for all their
// temporaries; every device allocation and release costs a fraction of a millisecond)
size_t radix_sort_scratch_bytes(int64_t n) {
    const size_t stiles = size_t(div_up(std::max<int64_t>(n, 1), kSortTile));
    return 2 * up256(stiles * kSortBins * sizeof(unsigned)) + up256(kSortBins * sizeof(int64_t));
}

// Queues the passes on `stream` without waiting.  lv: not null for a first pass that packs the keys (of one word)
// from the coordinates and takes the payload from pay_first; keys_a and pay_a are then only work space.
template <typename PAY>
static conststn_status radix_passes(uint64_t *keys_a, uint64_t *keys_b, PAY *pay_a, PAY *pay_b, int64_t n, int bits,
                                    hipStream_t stream, const uint64_t **keys_sorted, const PAY **pay_sorted, void *scratch,
                                    const Levels *lv, const PAY *pay_first, int *flags) {
    const int64_t stiles = div_up(n, kSortTile);
    char *at = static_cast<char *>(scratch);
    unsigned *counts = reinterpret_cast<unsigned *>(at);
    at += up256(size_t(stiles) * kSortBins * sizeof(unsigned));
    uint32_t *offsets = reinterpret_cast<uint32_t *>(at);
    at += up256(size_t(stiles) * kSortBins * sizeof(unsigned));
    int64_t *totals = reinterpret_cast<int64_t *>(at);
    uint64_t *kin = keys_a, *kout = keys_b;
    PAY *pin = pay_a, *pout = pay_b;
    const dim3 grid{unsigned(div_up(stiles, 8) * 8)}, block(kSortThreads);
    const Levels none{};
    // 9 bits where that saves a pass: 5 instead of 6 at 43 bits, 4.16 against 4.62 ms at 76 M pairs (a pass of 9 bits costs
    // more than one of 8, so where the number is the same 8 are taken)
    const bool nine = (bits + 8) / 9 < (bits + 7) / 8;
    auto pass = [&](auto digit_bits, auto coords, int shift) {
        constexpr int B = decltype(digit_bits)::value;
        constexpr bool C = decltype(coords)::value;
        radix_count_kernel<B, C><<<grid, block, 0, stream>>>(n, kin, C ? *lv : none, shift, counts, stiles);
        scan_tiles_kernel<uint32_t><<<dim3(1u << B), dim3(1024), 0, stream>>>(counts, offsets, stiles, totals);
        radix_scatter_kernel<B, C><<<grid, block, 0, stream>>>(n, kin, C ? pay_first : pin, C ? *lv : none, flags, kout, pout, shift, offsets, totals, stiles);
    };
    using std::integral_constant;
    for (int shift = 0; shift < bits; shift += nine ? 9 : 8) {
        const bool coords = lv && shift == 0;
        if constexpr (sizeof(PAY) == 8) {                     // (only the CSF build sorts values)
            if (nine && coords) pass(integral_constant<int, 9>{}, std::true_type{}, shift);
            if (!nine && coords) pass(integral_constant<int, 8>{}, std::true_type{}, shift);
        }
        if (nine && !coords) pass(integral_constant<int, 9>{}, std::false_type{}, shift);
        if (!nine && !coords) pass(integral_constant<int, 8>{}, std::false_type{}, shift);
        CST_HIP(hipGetLastError());
        std::swap(kin, kout);
        std::swap(pin, pout);
    }
    *keys_sorted = kin;
    *pay_sorted = pin;
    return CONSTSTN_OK;
}

// Sorts n (key, payload) pairs by the low `bits` bits of the key, stably; a and b are two buffers of n
// entries each (keys aligned to 16 bytes), the input is in a, the result in whichever *keys_sorted / *pay_sorted
// name.  Waits for the stream before it returns where the pass tables are its own (they are released then).
conststn_status radix_sort_pairs_u64(uint64_t *keys_a, uint64_t *keys_b, uint32_t *pay_a, uint32_t *pay_b, int64_t n,
                                     int bits, hipStream_t stream, const uint64_t **keys_sorted,
                                     const uint32_t **pay_sorted, void *scratch) {
    *keys_sorted = keys_a;
    *pay_sorted = pay_a;
    if (bits <= 0 || n <= 1) return CONSTSTN_OK;
    DevBuf<char> own;
    const bool lent = scratch != nullptr;
    if (!lent) {
        CST_TRY(own.alloc(radix_sort_scratch_bytes(n)));
        scratch = own.p;
    }
    CST_TRY(radix_passes(keys_a, keys_b, pay_a, pay_b, n, bits, stream, keys_sorted, pay_sorted, scratch, nullptr, static_cast<const uint32_t *>(nullptr), nullptr));
    if (!lent) CST_HIP(hipStreamSynchronize(stream));
    return CONSTSTN_OK;
}

// Rank heads and write the level arrays.  A head at level l is also a head at every deeper
// level, so its child pointer is simply its own rank one level down.  Thread t of a tile takes the
// pairs t, t + 256, ...: every read and write of a wavefront is to neighbouring addresses, the tile's
// keys go through LDS so that each pair sees the one before it, and the values are requested before
// anything else is done.  A pair's
// rank among the heads of a level is its rank in its wavefront's ballot plus the heads of the
// wavefronts and chunks of 256 before it in the tile.
// VALS: the values come in key order (vals_in), otherwise through the sorted positions.
template <bool WIDE, bool VALS>
__global__ void __launch_bounds__(kTileThreads)
emit_levels_kernel(int64_t nnz, Levels lv, const uint64_t *__restrict__ keys, const uint64_t *__restrict__ keys_hi,
                   const uint32_t *__restrict__ payload, const double *__restrict__ vals_in,
                   const int64_t *__restrict__ tile_offsets, int64_t ntiles, LevelOut out,
                   double *__restrict__ vals_out, int has_dups) {
    static_assert(CONSTSTN_MAX_ORDER * kItems * (kTileThreads / 64) == kTileThreads, "one thread per (level, chunk, wavefront)");
    constexpr int kWaves = kTileThreads / 64, kSlots = kItems * kWaves;
    __shared__ uint64_t lkey[kTile + 1];                       // [0]: the last key of the tile before
    __shared__ uint64_t lkey_hi[WIDE ? kTile + 1 : 1];
    __shared__ unsigned heads[CONSTSTN_MAX_ORDER][kSlots];     // heads of (chunk, wavefront), then those before it in the tile
    const int64_t tile = blockIdx.x, base = tile * kTile;
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    Key2 k[kItems];
    double v[kItems];
    uint32_t from[kItems];
#pragma unroll
    for (int i = 0; i < kItems; ++i) {               // (clamped, so that no load waits for a test)
        const int64_t n = base + i * kTileThreads + int(threadIdx.x), at = n < nnz ? n : nnz - 1;
        if (!VALS) from[i] = payload[at];
        else v[i] = vals_in[at];
        k[i] = load_key<WIDE>(keys, keys_hi, at);
    }
    if (!VALS) {
#pragma unroll
        for (int i = 0; i < kItems; ++i) v[i] = vals_in[from[i]];
    }
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
        const int m = i * kTileThreads + int(threadIdx.x);
        lkey[1 + m] = k[i].lo;
        if (WIDE) lkey_hi[1 + m] = k[i].hi;
    }
    if (threadIdx.x == 0) {
        lkey[0] = base > 0 ? keys[base - 1] : 0;
        if (WIDE) lkey_hi[0] = base > 0 ? keys_hi[base - 1] : 0;
    }
    __syncthreads();
    unsigned headbits[kItems];                       // bit l set: head at level l
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
        const int m = i * kTileThreads + int(threadIdx.x);
        const int64_t n = base + m;
        headbits[i] = 0;
        if (n < nnz) {
            const Key2 prev{WIDE ? lkey_hi[m] : 0, lkey[m]};
            for (int l = 0; l < lv.order; ++l)
                if (n == 0 || !same_prefix<WIDE>(lv, l, k[i], prev)) headbits[i] |= 1u << l;
        }
#pragma unroll
        for (int l = 0; l < CONSTSTN_MAX_ORDER; ++l) {
            const unsigned long long mask = __builtin_amdgcn_ballot_w64((headbits[i] >> l) & 1u);
            if (lane == 0) heads[l][i * kWaves + wave] = unsigned(__popcll(mask));
        }
    }
    __syncthreads();
    {
        // thread (l, slot): exclusive scan over the 32 (chunk, wavefront) slots of level l, in tile order
        const int l = int(threadIdx.x) / kSlots, slot = int(threadIdx.x) % kSlots;
        const unsigned mine = heads[l][slot];
        unsigned inc = mine;
        for (int off = 1; off < kSlots; off <<= 1) {
            const unsigned up = __shfl_up(inc, off, kSlots);
            if (slot >= off) inc += up;
        }
        heads[l][slot] = inc - mine;
    }
    __syncthreads();
    const unsigned long long lt = (1ull << lane) - 1ull;
    const int last = lv.order - 1;
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
        const int64_t n = base + i * kTileThreads + int(threadIdx.x);
        int64_t pos[CONSTSTN_MAX_ORDER];
#pragma unroll
        for (int l = 0; l < CONSTSTN_MAX_ORDER; ++l) {
            const unsigned long long mask = __builtin_amdgcn_ballot_w64((headbits[i] >> l) & 1u);
            pos[l] = l < lv.order ? tile_offsets[int64_t(l) * ntiles + tile] + heads[l][i * kWaves + wave] + __popcll(mask & lt) : 0;
        }
#pragma unroll
        for (int l = 0; l < CONSTSTN_MAX_ORDER; ++l) {
            if (l < lv.order && (headbits[i] & (1u << l))) {
                const uint64_t w = (WIDE && lv.word[l]) ? k[i].hi : k[i].lo;
                out.idx[l][pos[l]] = int32_t((lv.shift[l] >= 64 ? 0 : (w >> lv.shift[l])) & lv.mask[l]);
                if (l < last) out.ptr[l][pos[l]] = pos[l + 1 < CONSTSTN_MAX_ORDER ? l + 1 : l];
                if (l == last) {
                    // leaf head: its value is the sum of the run of equal keys, in input order
                    // (the sort is stable); without duplicates the run has length one
                    double sum = v[i];
                    if (has_dups)
                        for (int64_t m = n + 1; m < nnz && keys[m] == k[i].lo && (!WIDE || keys_hi[m] == k[i].hi); ++m) sum += vals_in[VALS ? m : int64_t(payload[m])];
                    vals_out[pos[l]] = sum;
                }
            }
        }
    }
}

__global__ void close_ptrs_kernel(LevelOut out, int order, const int64_t *totals) {
    const int l = threadIdx.x;
    if (l < order - 1) out.ptr[l][totals[l]] = totals[l + 1];
}

static conststn_status build_levels(int order, const int64_t *dims, int64_t nnz,
                                    const int32_t *const *coords, const double *vals,
                                    const int *mode_order, unsigned flags, hipStream_t stream,
                                    conststn_csf_s *csf) {
    Levels lv{};
    lv.order = order;
    int total_bits = 0;
    int bits[CONSTSTN_MAX_ORDER];
    for (int l = 0; l < order; ++l) {
        const int m = mode_order[l];
        bits[l] = ceil_log2_u64(uint64_t(dims[m]));
        total_bits += bits[l];
        lv.dim[l] = dims[m];
        lv.coord[l] = coords[m];
    }
    // The innermost levels fill the low word as far as whole fields fit, the others the high word.
    int sh = 0, lo_bits = 0, hi_bits = 0;
    bool in_hi = false;
    for (int l = order - 1; l >= 0; --l) {
        if (!in_hi && sh + bits[l] > 64) { in_hi = true; lo_bits = sh; sh = 0; }
        lv.word[l] = in_hi ? 1 : 0;
        lv.shift[l] = sh;
        lv.mask[l] = bits[l] >= 64 ? ~uint64_t(0) : ((uint64_t(1) << bits[l]) - 1);
        sh += bits[l];
    }
    if (in_hi) hi_bits = sh; else lo_bits = sh;
    const bool wide = in_hi;
    if (hi_bits > 64) {
        set_error("packed coordinate key needs %d bits in fields that do not fit two 64-bit words", total_bits);
        return CONSTSTN_EUNSUPPORTED;
    }

    csf->order = order;
    csf->nnz = nnz;
    for (int l = 0; l < order; ++l) {
        csf->dims[l] = dims[l];
        csf->mode_order[l] = mode_order[l];
    }
    CST_HIP(hipGetDevice(&csf->device));

    LevelOut lo{};
    if (nnz == 0) {
        for (int l = 0; l < order; ++l) {
            csf->nodes[l] = 0;
            CST_TRY(csf->idx[l].alloc(0));
            if (l < order - 1) {
                CST_TRY(csf->ptr[l].alloc(1));
                CST_HIP(hipMemsetAsync(csf->ptr[l].p, 0, sizeof(int64_t), stream));
            }
        }
        CST_TRY(csf->vals.alloc(0));
        CST_HIP(hipStreamSynchronize(stream));
        return CONSTSTN_OK;
    }

    // every temporary of the build in one allocation
    const int64_t ntiles = div_up(nnz, kTile);
    // the sort packs the keys and carries the values; or, with a third less work space, it carries positions
    const bool fused = !wide && total_bits > 0 && nnz > 1 && !(flags & CONSTSTN_LEAN_BUILD);
    const size_t pay_bytes = size_t(nnz) * (fused ? 8 : 4);
    const size_t sort_bytes = radix_sort_scratch_bytes(nnz);
    const size_t arena_bytes = 2 * up256(size_t(nnz) * 8) + 2 * up256(pay_bytes) + up256(2 * sizeof(int)) +
                               (wide ? 2 * up256(size_t(nnz) * 8) : 0) + sort_bytes +
                               up256(size_t(ntiles) * order * sizeof(unsigned)) + up256(size_t(ntiles) * order * sizeof(int64_t)) +
                               up256(CONSTSTN_MAX_ORDER * sizeof(int64_t));
    DevBuf<char> arena;
    CST_TRY(arena.alloc(arena_bytes));
    size_t arena_at = 0;
    auto take = [&](size_t bytes) { char *q = arena.p + arena_at; arena_at += up256(bytes); return q; };
    struct { uint64_t *p; } keys_a{reinterpret_cast<uint64_t *>(take(size_t(nnz) * 8))}, keys_b{reinterpret_cast<uint64_t *>(take(size_t(nnz) * 8))};
    struct { uint32_t *p; } pay_a{reinterpret_cast<uint32_t *>(take(pay_bytes))}, pay_b{reinterpret_cast<uint32_t *>(take(pay_bytes))};
    struct { int *p; } dflags{reinterpret_cast<int *>(take(2 * sizeof(int)))};
    CST_HIP(hipMemsetAsync(dflags.p, 0, 2 * sizeof(int), stream));
    struct { uint64_t *p; } lo_orig{nullptr}, hi_orig{nullptr};      // two-word keys only: the words in input order
    if (wide) {
        lo_orig.p = reinterpret_cast<uint64_t *>(take(size_t(nnz) * 8));
        hi_orig.p = reinterpret_cast<uint64_t *>(take(size_t(nnz) * 8));
    }
    void *sort_scratch = take(sort_bytes);
    const uint64_t *skeys = keys_a.p, *skeys_hi = nullptr;
    const uint32_t *spay = pay_a.p;
    const uint64_t *svals = nullptr;                                   // the values in key order, where the sort carried them
    if (!fused) {
        const int64_t blocks = std::min<int64_t>(div_up(nnz, 256), 65536);
        pack_keys_kernel<<<dim3(unsigned(blocks)), dim3(256), 0, stream>>>(nnz, lv, wide ? lo_orig.p : keys_a.p,
                                                                          wide ? hi_orig.p : nullptr, pay_a.p, dflags.p);
        CST_HIP(hipGetLastError());
    }
    if (!wide) {
        if (!fused)
            CST_TRY(radix_sort_pairs_u64(keys_a.p, keys_b.p, pay_a.p, pay_b.p, nnz, total_bits, stream, &skeys, &spay, sort_scratch));
        else
            CST_TRY(radix_passes(keys_a.p, keys_b.p, reinterpret_cast<uint64_t *>(pay_a.p), reinterpret_cast<uint64_t *>(pay_b.p), nnz,
                                 total_bits, stream, &skeys, &svals, sort_scratch, &lv, reinterpret_cast<const uint64_t *>(vals), dflags.p));
    } else {
        // least significant word first: sort (low word, position), bring the high words into that order, sort
        // again by the high word (stable), then fetch the low words in the final order
        const unsigned gb = unsigned(div_up(nnz, 256));
        CST_HIP(hipMemcpyAsync(keys_a.p, lo_orig.p, size_t(nnz) * sizeof(uint64_t), hipMemcpyDeviceToDevice, stream));
        CST_TRY(radix_sort_pairs_u64(keys_a.p, keys_b.p, pay_a.p, pay_b.p, nnz, lo_bits, stream, &skeys, &spay, sort_scratch));
        uint64_t *k_free = skeys == keys_a.p ? keys_b.p : keys_a.p, *k_used = skeys == keys_a.p ? keys_a.p : keys_b.p;
        uint32_t *p_used = spay == pay_a.p ? pay_a.p : pay_b.p, *p_free = spay == pay_a.p ? pay_b.p : pay_a.p;
        gather_u64_kernel<<<dim3(gb), dim3(256), 0, stream>>>(nnz, hi_orig.p, p_used, k_free);
        CST_HIP(hipGetLastError());
        const uint64_t *shi = nullptr;
        CST_TRY(radix_sort_pairs_u64(k_free, k_used, p_used, p_free, nnz, hi_bits, stream, &shi, &spay, sort_scratch));
        uint64_t *lo_sorted = shi == k_free ? k_used : k_free;
        gather_u64_kernel<<<dim3(gb), dim3(256), 0, stream>>>(nnz, lo_orig.p, spay, lo_sorted);
        CST_HIP(hipGetLastError());
        skeys = lo_sorted;
        skeys_hi = shi;
    }

    struct { unsigned *p; } tile_counts{reinterpret_cast<unsigned *>(take(size_t(ntiles) * order * sizeof(unsigned)))};
    struct { int64_t *p; } tile_offsets{reinterpret_cast<int64_t *>(take(size_t(ntiles) * order * sizeof(int64_t)))},
        totals{reinterpret_cast<int64_t *>(take(CONSTSTN_MAX_ORDER * sizeof(int64_t)))};
    if (wide)
        count_heads_kernel<true><<<dim3(unsigned(ntiles)), dim3(kTileThreads), 0, stream>>>(
            nnz, lv, skeys, skeys_hi, tile_counts.p, ntiles, dflags.p);
    else
        count_heads_kernel<false><<<dim3(unsigned(ntiles)), dim3(kTileThreads), 0, stream>>>(
            nnz, lv, skeys, nullptr, tile_counts.p, ntiles, dflags.p);
    CST_HIP(hipGetLastError());
    scan_tiles_kernel<int64_t><<<dim3(unsigned(order)), dim3(1024), 0, stream>>>(tile_counts.p, tile_offsets.p,
                                                                               ntiles, totals.p);
    CST_HIP(hipGetLastError());

    int hflags[2] = {0, 0};
    int64_t htotals[CONSTSTN_MAX_ORDER] = {0};
    CST_HIP(hipMemcpyAsync(hflags, dflags.p, sizeof(hflags), hipMemcpyDeviceToHost, stream));
    CST_HIP(hipMemcpyAsync(htotals, totals.p, sizeof(int64_t) * order, hipMemcpyDeviceToHost, stream));
    CST_HIP(hipStreamSynchronize(stream));
    if (hflags[0]) {
        set_error("a coordinate is negative or not below its mode extent");
        return CONSTSTN_ERANGE;
    }
    if (hflags[1] && !(flags & CONSTSTN_COALESCE_DUPS)) {
        set_error("duplicate coordinate in the input (the nonzero structure must be a set)");
        return CONSTSTN_EDUP;
    }

    for (int l = 0; l < order; ++l) {
        csf->nodes[l] = htotals[l];
        CST_TRY(csf->idx[l].alloc(size_t(htotals[l])));
        lo.idx[l] = csf->idx[l].p;
        if (l < order - 1) {
            CST_TRY(csf->ptr[l].alloc(size_t(htotals[l]) + 1));
            lo.ptr[l] = csf->ptr[l].p;
        }
    }
    CST_TRY(csf->vals.alloc(size_t(htotals[order - 1])));
    csf->nnz = htotals[order - 1];

    const dim3 egrid{unsigned(ntiles)}, eblock(kTileThreads);
    if (wide)
        emit_levels_kernel<true, false><<<egrid, eblock, 0, stream>>>(
            nnz, lv, skeys, skeys_hi, spay, vals, tile_offsets.p, ntiles, lo, csf->vals.p, hflags[1]);
    else if (svals)
        emit_levels_kernel<false, true><<<egrid, eblock, 0, stream>>>(
            nnz, lv, skeys, nullptr, nullptr, reinterpret_cast<const double *>(svals), tile_offsets.p, ntiles, lo, csf->vals.p, hflags[1]);
    else
        emit_levels_kernel<false, false><<<egrid, eblock, 0, stream>>>(
            nnz, lv, skeys, nullptr, spay, vals, tile_offsets.p, ntiles, lo, csf->vals.p, hflags[1]);
    CST_HIP(hipGetLastError());
    close_ptrs_kernel<<<dim3(1), dim3(64), 0, stream>>>(lo, order, totals.p);
    CST_HIP(hipGetLastError());
    CST_HIP(hipStreamSynchronize(stream));
    return CONSTSTN_OK;
}

conststn_status build_csf_device(int order, const int64_t *dims, int64_t nnz,
                                 const int32_t *const *coords, const double *vals,
                                 const int *mode_order, unsigned flags, hipStream_t stream,
                                 conststn_csf_s *csf) {
    conststn_status st = build_levels(order, dims, nnz, coords, vals, mode_order, flags, stream, csf);
    if (st != CONSTSTN_ENOMEM || (flags & CONSTSTN_LEAN_BUILD)) return st;
    // once more with the smaller work space, and with what is kept for reuse given back
    for (int l = 0; l < order; ++l) {
        csf->idx[l].release();
        csf->ptr[l].release();
    }
    csf->vals.release();
    release_idle_memory();
    clear_error();
    return build_levels(order, dims, nnz, coords, vals, mode_order, flags | CONSTSTN_LEAN_BUILD, stream, csf);
}

// ---- a second layout of a tensor that is already a CSF ------------------------------------------
//
// The level order fixes the loop order (Sec. 3.2), and a result indexed by a level other than the root
// would have to be added into from everywhere.  For the order-3 MTTKRP / TTMc of such a mode the plan
// therefore keeps a copy of the tensor with that level at the root: the coordinates are read back
// out of the level arrays (a leaf's ancestors by binary search in the pointer arrays) and sorted again.
__global__ void expand_csf3_kernel(int64_t nnz, int64_t n0, int64_t n1, const int64_t *__restrict__ ptr0,
                                   const int64_t *__restrict__ ptr1, const int32_t *__restrict__ idx0,
                                   const int32_t *__restrict__ idx1, const int32_t *__restrict__ idx2,
                                   int32_t *c0, int32_t *c1, int32_t *c2) {
    const int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (e >= nnz) return;
    const int64_t f = parent_of(ptr1, n1, e);
    const int64_t s = parent_of(ptr0, n0, f);
    c0[e] = idx0[s];
    c1[e] = idx1[f];
    c2[e] = idx2[e];
}

conststn_status reroot_csf3(const conststn_csf_s *src, const int new_levels[3], conststn_csf_s *dst) {
    if (src->order != 3) { set_error("only order-3 tensors are re-sorted"); return CONSTSTN_EUNSUPPORTED; }
    const int64_t nnz = src->nnz;
    DevBuf<int32_t> c[3];
    for (int l = 0; l < 3; ++l) CST_TRY(c[l].alloc(size_t(nnz)));
    if (nnz > 0) {
        expand_csf3_kernel<<<dim3(unsigned(div_up(nnz, 256))), dim3(256)>>>(
            nnz, src->nodes[0], src->nodes[1], src->ptr[0].p, src->ptr[1].p, src->idx[0].p, src->idx[1].p,
            src->idx[2].p, c[0].p, c[1].p, c[2].p);
        CST_HIP(hipGetLastError());
    }
    // coordinates by tensor mode, and the new level order in tensor modes
    const int32_t *by_mode[3] = {nullptr, nullptr, nullptr};
    int mode_order[3];
    for (int l = 0; l < 3; ++l) by_mode[src->mode_order[l]] = c[l].p;
    for (int l = 0; l < 3; ++l) mode_order[l] = src->mode_order[new_levels[l]];
    CST_TRY(build_csf_device(3, src->dims, nnz, by_mode, src->vals.p, mode_order, 0, hipStream_t(0), dst));
    CST_HIP(hipDeviceSynchronize());
    return CONSTSTN_OK;
}

}  // namespace cst
