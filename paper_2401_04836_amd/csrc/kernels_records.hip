// MTTKRP of order 3 and 4 as a walk over one stream of records (Sec. 5.2, 5.3):
//     M[i,r] = sum_{j,k} X[i,j,k] B[j,r] C[k,r]       and       M[i,r] = sum X[i,j,k,l] B[j,r] C[k,r] D[l,r]
// fused on the whole sparse prefix, so that every intermediate is one length-R vector (Fig. 3b).
//
// The plan turns the tree into a flat stream in which every record reads exactly ONE factor row:
//     leaf             t   += v * F_leaf[index]
//     end of a fiber   acc += t * F_1[index], t = 0         (order 4: u += t * F_2[index], t = 0)
//     end of a node    acc += u * F_1[index], u = 0         (order 4 only)
//     nothing          an end whose vector the chunks before it have used up; reads a row of zeros
// and the last record of a slice is marked.  The stream is cut into chunks of q records; LPR lanes own a chunk
// and hold NV pairs of rank entries each.  The four (eight) lane groups of a wavefront walk their chunks in
// lock step, one record per step: a step is NV gathers in which every group takes part, whatever its record is.
// With the rows of ended fibers read beside the leaf rows, as a stream of leaves needs it, half the gathers serve
// 1.4 of 4 groups.  The bound is the L1 pipeline, which takes 16 cycles for such a gather (64 bytes a cycle) and
// more where it misses: busy in 96 % of the cycles at 76 M nonzeros, rank 32, 89 M records (its address unit 95 %,
// 72 % of its requests hit the L2), 91 % at 20 M and rank 50, 93 % at order 4 (L2 hits 55 and 67 %).  Neither fewer
// instructions per record (groups of 4 or 8 lanes with 4 or 2 pairs each: 1.54, 1.28 against 1.23 ms), nor
// selects in place of branches (1.25), nor twice the rows in flight (1.20), nor the most named rows in LDS (1.20)
// change it by more than that.
//   - a block of LPR records is read with one load per lane, two blocks ahead; each lane forms the address of
//     its record's row and the group takes address and value round with row broadcasts;
//   - which groups meet an end in a step is known per wavefront (a ballot per block), so the two kinds of step
//     differ by lane masks made in scalar registers;
//   - a slice that ends in the chunk it began in is stored; its parts in other chunks go to partial rows,
//     two per chunk, which records_fixup_kernel adds in chunk order.  No atomics: the sums are reproducible.
// Ranks that do not fill the lanes: a lane past the row's end takes the row's last two entries and stores
// nothing; with an odd rank one lane repeats an entry of its neighbour.
#include <algorithm>
#include <utility>

#include "plan.hpp"

namespace cst {

namespace {

constexpr uint32_t kRecFiberEnd = 1u << 30, kRecNodeEnd = 2u << 30, kRecNothing = 3u << 30, kRecSliceEnd = 1u << 29,
                   kRecIndex = (1u << 28) - 1;
constexpr uint32_t kChunkInside = 1u << 31;           // the chunk begins inside its first slice
// Chunks of up to so many records take the SHORT instances (the plan gives small tensors chunks of 32): with the fix-up's
// 16-byte descriptors 14.6 -> 13.7 us at 33 K nonzeros, rank 50; 29.5 -> 27.6 at 384 K, rank 64.  At 512 records the wait at
// the end is one of 512 steps, and the registers that hold the rows cost a wavefront per SIMD at some ranks.
constexpr int kRecShort = 64;

typedef double v2f64_u __attribute__((ext_vector_type(2), aligned(8)));
typedef double v2f64 __attribute__((ext_vector_type(2)));
typedef int v2i32 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(1))) const v2f64_u global_v2f64_u;     // an address put together from integers

struct RecordArgs {
    int64_t n_chunks;
    int q, R;
    int32_t slices;
    const uint32_t *code;
    const double *vals;
    const uint32_t *chunk_slice;
    const int32_t *open1, *open2;                      // rows of the fiber / node left open at a chunk's end, or -1
    const int32_t *row_of_slice;
    const double *f0, *f1, *f2;                        // factors of the leaves, of the fibers, of the nodes above them
    const double *zeros;                               // R zeros, the row of a record that adds nothing
    double *out, *partial;
};

// entry T of every LPR lanes, to all of them
template <int LPR, int T>
__device__ __forceinline__ int group_bcast(int x) {
    if (LPR == 16) return __builtin_amdgcn_mov_dpp(x, 0x150 + T, 0xf, 0xf, false);
    const int lo = __builtin_amdgcn_update_dpp(0, x, 0x150 + T, 0xf, 0x3, false);
    return __builtin_amdgcn_update_dpp(lo, x, 0x150 + 8 + T % 8, 0xf, 0xc, false);
}

template <int... I, class F>
__device__ __forceinline__ void each(std::integer_sequence<int, I...>, F &&f) {
    (f(std::integral_constant<int, I>{}), ...);
}

// SHORT: chunks of few records, whose time is the chain of loads from the first to the last: the rows that the chunk leaves
// open are fetched at its start.
template <int LPR, int NV, int LEVELS, bool SHORT>
__global__ void __launch_bounds__(256)
records_kernel(RecordArgs a) {
    constexpr int U = NV == 1 ? 8 : 4;                 // rows in flight per lane group
    constexpr uint64_t kOne = LPR == 16 ? 0x0001000100010001ull : 0x0101010101010101ull;
    const int gl = threadIdx.x % LPR;
    int64_t c = int64_t(blockIdx.x) * (256 / LPR) + threadIdx.x / LPR;
    const bool live = c < a.n_chunks;
    if (!live) c = a.n_chunks - 1;                     // walks along and stores nothing
    const int R = a.R;
    int col[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) col[v] = min(2 * (LPR * v + gl), R - 2);
    const uint32_t row_bytes = uint32_t(R) * 8u;
    const uint32_t *code = a.code + c * a.q;
    const double *vals = a.vals + c * a.q;
    const uint32_t head = a.chunk_slice[c];
    int32_t s = int32_t(head & ~kChunkInside);
    bool whole = !(head & kChunkInside);               // the slice being summed began in this chunk
    bool first = true;                                 // and is the chunk's first
    int32_t row = a.row_of_slice[s];

    double t[NV][2], u[NV][2], acc[NV][2];
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
        for (int e = 0; e < 2; ++e) t[v][e] = u[v][e] = acc[v][e] = 0.0;

    auto put = [&](double *dst) {
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const int mine = 2 * (LPR * v + gl);
            if (mine + 1 < R) *reinterpret_cast<v2f64_u *>(dst + mine) = v2f64_u{acc[v][0], acc[v][1]};
            else if (mine < R) dst[mine] = acc[v][1];  // odd rank: this lane holds entries R-2 and R-1
        }
    };
    auto emit = [&](bool ends) {
        double *dst = (ends && whole) ? a.out + int64_t(row) * R : a.partial + (2 * c + (first ? 0 : 1)) * R;
        if (live) put(dst);
#pragma unroll
        for (int v = 0; v < NV; ++v) acc[v][0] = acc[v][1] = 0.0;
        whole = true;
        first = false;
        ++s;
        row = a.row_of_slice[min(s, a.slices - 1)];
    };

    // what the chunk leaves open behind it, and the rows of that
    int32_t o1, o2 = -1;
    v2f64 r1[NV], r2[NV];
    auto fetch_open = [&]() {
        o1 = a.open1[c];
        if (LEVELS == 3) o2 = a.open2[c];
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            r1[v] = *reinterpret_cast<const v2f64_u *>(a.f1 + int64_t(max(o1, 0)) * R + col[v]);
            if (LEVELS == 3) r2[v] = *reinterpret_cast<const v2f64_u *>(a.f2 + int64_t(max(o2, 0)) * R + col[v]);
        }
    };
    if (SHORT) fetch_open();

    const int blocks = a.q / LPR;
    uint32_t code_cur = code[gl], code_nxt = code[(blocks > 1 ? LPR : 0) + gl];
    double val_cur = vals[gl], val_nxt = vals[(blocks > 1 ? LPR : 0) + gl];
    for (int b = 0; b < blocks; ++b) {
        const int ahead = min(b + 2, blocks - 1) * LPR + gl;
        const uint32_t code_n2 = code[ahead];
        const double val_n2 = vals[ahead];
        const uint32_t kind = code_cur >> 30;
        const double *base = a.f0;
        if (kind == 1) base = a.f1;
        if (LEVELS == 3 && kind == 2) base = a.f2;
        if (kind == 3) base = a.zeros;
        const uint64_t addr = reinterpret_cast<uint64_t>(base) + uint64_t(code_cur & kRecIndex) * row_bytes;
        const int addr_lo = int(uint32_t(addr)), addr_hi = int(uint32_t(addr >> 32));
        const int val_lo = __double2loint(val_cur), val_hi = __double2hiint(val_cur);
        const uint64_t ends1 = __builtin_amdgcn_ballot_w64(kind == 1);
        const uint64_t ends2 = LEVELS == 3 ? __builtin_amdgcn_ballot_w64(kind == 2) : 0;
        const uint64_t last = __builtin_amdgcn_ballot_w64((code_cur & kRecSliceEnd) != 0);
        // lanes of the groups whose step-T record is marked in m
        auto groups = [&](uint64_t m, int T) -> uint64_t {
            const uint64_t x = (m >> T) & kOne;
            return (x << LPR) - x;
        };
        auto batch = [&](auto T0c) {
            constexpr int T0 = decltype(T0c)::value * U;
            v2f64 x[U][NV];
            each(std::make_integer_sequence<int, U>{}, [&](auto Uc) {
                constexpr int k = decltype(Uc)::value, T = T0 + k;
                const v2i32 at{group_bcast<LPR, T>(addr_lo), group_bcast<LPR, T>(addr_hi)};
                const uint64_t p = __builtin_bit_cast(uint64_t, at);
#pragma unroll
                for (int v = 0; v < NV; ++v) x[k][v] = *reinterpret_cast<global_v2f64_u *>(p + uint64_t(uint32_t(col[v] * 8)));
            });
            each(std::make_integer_sequence<int, U>{}, [&](auto Uc) {
                constexpr int k = decltype(Uc)::value, T = T0 + k;
                const v2f64 *row_x = x[k];
                const bool e1 = __builtin_amdgcn_inverse_ballot_w64(groups(ends1, T));
                const double value = __hiloint2double(group_bcast<LPR, T>(val_hi), group_bcast<LPR, T>(val_lo));
                if (e1) {
#pragma unroll
                    for (int v = 0; v < NV; ++v)
#pragma unroll
                        for (int e = 0; e < 2; ++e) {
                            if (LEVELS == 3) u[v][e] = fma(t[v][e], row_x[v][e], u[v][e]);
                            else acc[v][e] = fma(t[v][e], row_x[v][e], acc[v][e]);
                            t[v][e] = 0.0;
                        }
                } else if (LEVELS == 2 || !__builtin_amdgcn_inverse_ballot_w64(groups(ends2, T))) {
#pragma unroll
                    for (int v = 0; v < NV; ++v)
#pragma unroll
                        for (int e = 0; e < 2; ++e) t[v][e] = fma(value, row_x[v][e], t[v][e]);
                } else {
#pragma unroll
                    for (int v = 0; v < NV; ++v)
#pragma unroll
                        for (int e = 0; e < 2; ++e) {
                            acc[v][e] = fma(u[v][e], row_x[v][e], acc[v][e]);
                            u[v][e] = 0.0;
                        }
                }
                if (last & (kOne << T)) {
                    if (__builtin_amdgcn_inverse_ballot_w64(groups(last, T))) emit(true);
                }
            });
        };
        each(std::make_integer_sequence<int, LPR / U>{}, batch);
        code_cur = code_nxt;
        val_cur = val_nxt;
        code_nxt = code_n2;
        val_nxt = val_n2;
    }
    // the chunk may end inside a fiber, a node and a slice: their sums so far count with the rows still to come
    if (!SHORT) fetch_open();
    if (o1 >= 0) {
#pragma unroll
        for (int v = 0; v < NV; ++v)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                if (LEVELS == 3) u[v][e] = fma(t[v][e], r1[v][e], u[v][e]);
                else acc[v][e] = fma(t[v][e], r1[v][e], acc[v][e]);
            }
    }
    if (LEVELS == 3 && o2 >= 0) {
#pragma unroll
        for (int v = 0; v < NV; ++v)
#pragma unroll
            for (int e = 0; e < 2; ++e) acc[v][e] = fma(u[v][e], r2[v][e], acc[v][e]);
    }
    if (s < a.slices) emit(false);
}

// ---- rows of slices that several chunks share ---------------------------------------------------------
//
// One launch: first the slices of many chunks (kRecLight and more; a workgroup, or kRecSegments of them, per
// slice), then those of a few (W threads each), then the rows of empty slices, which are zero.
constexpr int kRecOneBlock = 1024, kRecSegments = 32;

struct RecordFixArgs {
    int R, segments;
    int64_t n_heavy, n_light, n_empty, heavy_blocks, light_blocks;
    const RecordShare *heavy, *light;
    const int32_t *empty;
    const double *partial;
    double *heavy_partial, *out;
};

// Partial rows of a slice: `first` in its first chunk (the second one there where the slice begins inside the chunk), the
// first one of every chunk behind that.
template <int W, int THREADS>
__global__ void __launch_bounds__(THREADS)
records_fixup_kernel(RecordFixArgs a) {
    constexpr int G = THREADS / W;
    __shared__ double red[THREADS];
    const int g = threadIdx.x / W, col = threadIdx.x % W, R = a.R;
    const bool mine = col < R;
    int64_t b = blockIdx.x;
    if (b < a.heavy_blocks) {
        const int64_t h = b / a.segments, seg = b % a.segments;
        const RecordShare s = a.heavy[h];
        const int64_t n = s.count, c0 = n * seg / a.segments, c1 = n * (seg + 1) / a.segments;
        double sum = 0.0;
        if (mine) {
            // (one address that moves on: the choice of the first chunk's row inside the loop cost 0.5 us of 16 over 900 chunks)
            int64_t c = c0 + g;
            const int64_t step = 2 * int64_t(G) * R;
            const double *p = a.partial + (s.first & ~int64_t(1)) * R + col + 2 * c * R;
            int64_t begins = c == 0 ? (s.first & 1) * R : 0;
            for (; c + 7 * G < c1; c += 8 * G, p += 8 * step) {
                double x[8];
                x[0] = p[begins];
                begins = 0;
#pragma unroll
                for (int k = 1; k < 8; ++k) x[k] = p[k * step];
#pragma unroll
                for (int k = 0; k < 8; ++k) sum += x[k];
            }
            for (; c < c1; c += G, p += step) {
                sum += p[begins];
                begins = 0;
            }
        }
        red[threadIdx.x] = sum;
        __syncthreads();
        if (g == 0 && mine) {
            for (int gg = 1; gg < G; ++gg) sum += red[gg * W + col];
            if (a.segments == 1) a.out[int64_t(s.row) * R + col] = sum;
            else a.heavy_partial[(h * a.segments + seg) * R + col] = sum;
        }
        return;
    }
    b -= a.heavy_blocks;
    if (b < a.light_blocks) {
        const int64_t k = b * G + g;
        if (k >= a.n_light || !mine) return;
        const RecordShare s = a.light[k];
        double sum = a.partial[s.first * R + col];
        const double *x0 = a.partial + (s.first & ~int64_t(1)) * R + col;
        int64_t c = 1;
        for (; c + 4 <= s.count; c += 4) {
            double x[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = x0[2 * (c + e) * R];
#pragma unroll
            for (int e = 0; e < 4; ++e) sum += x[e];
        }
        for (; c < s.count; ++c) sum += x0[2 * c * R];
        a.out[int64_t(s.row) * R + col] = sum;
        return;
    }
    b -= a.light_blocks;
    const int64_t k = b * G + g;
    if (k < a.n_empty && mine) a.out[int64_t(a.empty[k]) * R + col] = 0.0;
}

__global__ void __launch_bounds__(128)
records_final_kernel(RecordFixArgs a) {
    const int64_t h = blockIdx.x;
    const int col = threadIdx.x;
    if (col >= a.R) return;
    double sum = 0.0;
#pragma unroll 8
    for (int seg = 0; seg < kRecSegments; ++seg) sum += a.heavy_partial[(h * kRecSegments + seg) * a.R + col];
    a.out[int64_t(a.heavy[h].row) * a.R + col] = sum;
}

// ---- the plan's side ------------------------------------------------------------------------------------

// parent[e] = the node one level up that child e hangs below.  A workgroup takes 2048 children: it finds the
// parent of the first by binary search and marks where the others begin.
constexpr int kExpandTile = 2048;
__global__ void __launch_bounds__(256)
expand_parents_kernel(int64_t children, int64_t parents, const int64_t *__restrict__ ptr, int32_t *__restrict__ parent) {
    __shared__ uint8_t begins[kExpandTile];
    __shared__ int64_t p0_shared;
    __shared__ int wtot[4];
    const int64_t base = int64_t(blockIdx.x) * kExpandTile;
    const int64_t end = base + kExpandTile < children ? base + kExpandTile : children;
    reinterpret_cast<uint64_t *>(begins)[threadIdx.x] = 0;
    if (threadIdx.x == 0) p0_shared = parent_of(ptr, parents, base);
    __syncthreads();
    const int64_t p0 = p0_shared;
    for (int64_t p = p0 + 1 + threadIdx.x; p < parents; p += 256) {
        const int64_t at = ptr[p];
        if (at >= end) break;
        begins[at - base] = 1;
    }
    __syncthreads();
    const uint64_t mine = reinterpret_cast<const uint64_t *>(begins)[threadIdx.x];
    const int cnt = __popcll(mine);                                  // bytes are 0 or 1
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    int inc = cnt;
    for (int off = 1; off < 64; off <<= 1) {
        const int up = __shfl_up(inc, off, 64);
        if (lane >= off) inc += up;
    }
    if (lane == 63) wtot[wave] = inc;
    __syncthreads();
    int run = inc - cnt;
    for (int w = 0; w < wave; ++w) run += wtot[w];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        run += int((mine >> (8 * k)) & 1u);
        const int64_t e = base + threadIdx.x * 8 + k;
        if (e < end) parent[e] = int32_t(p0 + run);
    }
}

struct RecordFill {
    int64_t leaves, fibers, nodes, slices, n_rec, total;             // nodes: order 4 only (0 otherwise)
    const int64_t *ptr_slice, *ptr_node, *ptr_fiber;                  // slices -> level 1, nodes -> fibers, fibers -> leaves
    const int32_t *idx_slice, *idx_node, *idx_fiber, *idx_leaf;
    const double *vals;
    const int32_t *fiber_of, *node_of;
    uint32_t *code;
    double *out_vals;
    int64_t *slice_rec;
};

__global__ void __launch_bounds__(256)
record_leaves_kernel(RecordFill a) {
    const int64_t e = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (e >= a.leaves) {
        // records past the end name the last leaf's row with the value 0
        const int64_t pad = a.n_rec + (e - a.leaves);
        if (pad < a.total) { a.code[pad] = uint32_t(a.idx_leaf[a.leaves - 1]); a.out_vals[pad] = 0.0; }
        return;
    }
    const int32_t f = a.fiber_of[e];
    const int64_t at = e + f + (a.nodes ? a.node_of[f] : 0);
    a.code[at] = uint32_t(a.idx_leaf[e]);
    a.out_vals[at] = a.vals[e];
}

__device__ __forceinline__ int64_t fiber_end_record(const RecordFill &a, int64_t f) {
    return a.ptr_fiber[f + 1] + f + (a.nodes ? a.node_of[f] : 0);
}
__device__ __forceinline__ int64_t node_end_record(const RecordFill &a, int64_t n) {
    const int64_t f = a.ptr_node[n + 1];
    return a.ptr_fiber[f] + f + n;
}

__global__ void __launch_bounds__(256)
record_ends_kernel(RecordFill a) {
    const int64_t x = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (x < a.fibers) {
        const int64_t at = fiber_end_record(a, x);
        a.code[at] = kRecFiberEnd | uint32_t(a.idx_fiber[x]);
        a.out_vals[at] = 0.0;
    }
    if (x < a.nodes) {
        const int64_t at = node_end_record(a, x);
        a.code[at] = kRecNodeEnd | uint32_t(a.idx_node[x]);
        a.out_vals[at] = 0.0;
    }
    if (x <= a.slices) {
        int64_t f = x, n = 0;
        if (a.nodes) { n = a.ptr_slice[x]; f = a.ptr_node[n]; }
        else f = a.ptr_slice[x];
        a.slice_rec[x] = a.ptr_fiber[f] + f + n;
    }
}

__global__ void __launch_bounds__(256)
record_slices_kernel(RecordFill a) {
    const int64_t s = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (s < a.slices) a.code[a.slice_rec[s + 1] - 1] |= kRecSliceEnd;
}

// smallest x in [0, n) with end(x) >= at
template <class F>
__device__ __forceinline__ int64_t first_end(int64_t n, int64_t at, F &&end) {
    int64_t lo = 0, hi = n - 1;
    while (lo < hi) {
        const int64_t mid = (lo + hi) / 2;
        if (end(mid) >= at) hi = mid; else lo = mid + 1;
    }
    return lo;
}

__global__ void __launch_bounds__(256)
record_chunks_kernel(RecordFill a, int64_t n_chunks, int64_t q, uint32_t *chunk_slice, int32_t *open1, int32_t *open2) {
    const int64_t c = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (c >= n_chunks) return;
    const int64_t r0 = c * q, r1 = (c + 1) * q < a.n_rec ? (c + 1) * q : a.n_rec;
    const int64_t s = parent_of(a.slice_rec, a.slices, r0);
    chunk_slice[c] = uint32_t(s) | (a.slice_rec[s] == r0 ? 0u : kChunkInside);
    const uint32_t kind = a.code[r1 - 1] >> 30;
    int32_t o1 = -1, o2 = -1;                          // (nothing is open behind the last record)
    if (kind == 0) o1 = a.idx_fiber[first_end(a.fibers, r1, [&](int64_t f) { return fiber_end_record(a, f); })];
    if (a.nodes && kind != 2 && r1 < a.n_rec) o2 = a.idx_node[first_end(a.nodes, r1, [&](int64_t n) { return node_end_record(a, n); })];
    open1[c] = o1;
    if (open2) open2[c] = o2;
}

// A chunk that begins with the end of a fiber or of a node (or, at order 4, of both) has added nothing to that vector,
// and the chunk before has taken it with the row: 0 times the row would make NaN of an infinite one.
__global__ void __launch_bounds__(256)
record_spent_ends_kernel(int64_t n_chunks, int64_t q, int64_t n_rec, uint32_t *code) {
    const int64_t c = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (c >= n_chunks) return;
    for (int64_t r = c * q; r < c * q + 2 && r < n_rec; ++r) {
        if (code[r] >> 30 == 0) break;
        code[r] = kRecNothing | (code[r] & kRecSliceEnd);
    }
}

__global__ void __launch_bounds__(256)
record_shared_kernel(int64_t slices, const int64_t *__restrict__ slice_rec, int64_t q, int kind, int64_t *flag, int *widest) {
    const int64_t s = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (s >= slices) return;
    flag[s] = share_of(slice_rec, s, q) == kind;
    if (kind == 2 && flag[s]) {
        const int64_t span = (slice_rec[s + 1] - 1) / q - slice_rec[s] / q + 1;
        atomicMax(widest, int(span < 0x7fffffff ? span : 0x7fffffff));
    }
}
__global__ void __launch_bounds__(256)
list_flagged_kernel(int64_t n, const int64_t *__restrict__ flag, const int64_t *__restrict__ pos, int32_t *list) {
    const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (i < n && flag[i]) list[pos[i]] = int32_t(i);
}
// what the fix-up launch needs of the listed slices, in one 16-byte read
__global__ void __launch_bounds__(256)
record_shares_kernel(int64_t n, const int32_t *__restrict__ list, const int64_t *__restrict__ slice_rec, const int32_t *__restrict__ row_of_slice,
                     int64_t q, RecordShare *share) {
    const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (i >= n) return;
    share[i] = record_share(slice_rec, list[i], q, row_of_slice[list[i]]);
}
__global__ void __launch_bounds__(256)
empty_rows_kernel(int64_t rows, int64_t slices, const int32_t *__restrict__ idx0, int64_t *flag) {
    const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (i >= rows) return;
    int64_t lo = 0, hi = slices;                                      // root indices ascend
    while (lo < hi) {
        const int64_t mid = (lo + hi) / 2;
        if (idx0[mid] < i) lo = mid + 1; else hi = mid;
    }
    flag[i] = lo == slices || idx0[lo] != i;
}
__global__ void __launch_bounds__(256)
rows_of_slices_kernel(int64_t slices, const int32_t *__restrict__ idx0, int compact, int32_t *row) {
    const int64_t s = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (s < slices) row[s] = compact ? int32_t(s) : idx0[s];
}

dim3 blocks_for(int64_t n) { return dim3(unsigned(div_up(std::max<int64_t>(n, 1), 256))); }

conststn_status list_of_flags(DevBuf<int64_t> &flag, int64_t n, DevBuf<int32_t> &list, int64_t *count) {
    DevBuf<int64_t> pos;
    CST_TRY(pos.alloc(size_t(n)));
    CST_TRY(exscan(flag.p, pos.p, n, count));
    CST_TRY(list.alloc(size_t(*count)));
    if (*count > 0) {
        list_flagged_kernel<<<blocks_for(n), dim3(256)>>>(n, flag.p, pos.p, list.p);
        CST_HIP(hipGetLastError());
        CST_HIP(hipDeviceSynchronize());
    }
    return CONSTSTN_OK;
}

// Every record and its value recomputed from the level arrays, every chunk's slice and open rows, the row of every
// slice, and what the fix-up launch works through (the shares of its slices and the empty rows) against what it must be.
struct RecordCheck {
    RecordFill a;
    int64_t q, n_chunks, out_rows, n_light, n_heavy, n_empty;
    const uint32_t *chunk_slice;
    const int32_t *open1, *open2, *row_of_slice, *empty, *idx0;
    const RecordShare *light, *heavy;
    int compact;
    unsigned bad_code, bad_chunk, bad_list;
};

// whether x is in the ascending list
__device__ __forceinline__ bool listed(const int32_t *list, int64_t n, int64_t x) {
    int64_t lo = 0, hi = n;
    while (lo < hi) {
        const int64_t mid = (lo + hi) / 2;
        if (list[mid] < x) lo = mid + 1; else hi = mid;
    }
    return lo < n && list[lo] == x;
}

__global__ void __launch_bounds__(256)
check_records_kernel(RecordCheck c, int64_t threads, unsigned *flags) {
    const RecordFill &a = c.a;
    const int64_t q = c.q;
    unsigned bad = 0;
    for (int64_t t = int64_t(blockIdx.x) * 256 + threadIdx.x; t < threads; t += int64_t(gridDim.x) * 256) {
        if (t < a.n_rec) {
            uint32_t want;
            double value = 0.0;
            int64_t n = 0, n_end = -1;
            if (a.nodes) {
                n = first_end(a.nodes, t, [&](int64_t x) { return node_end_record(a, x); });
                n_end = node_end_record(a, n);
            }
            if (t == n_end) want = kRecNodeEnd | uint32_t(a.idx_node[n]);
            else {
                // records before t that belong to fibers: t minus the node ends before it
                auto end_of = [&](int64_t f) { return a.ptr_fiber[f + 1] + f + (a.nodes ? parent_of(a.ptr_node, a.nodes, f) : 0); };
                const int64_t f = first_end(a.fibers, t, end_of);
                const int64_t nf = a.nodes ? parent_of(a.ptr_node, a.nodes, f) : 0;
                if (t == end_of(f)) want = kRecFiberEnd | uint32_t(a.idx_fiber[f]);
                else {
                    want = uint32_t(a.idx_leaf[t - f - nf]);
                    value = a.vals[t - f - nf];
                }
            }
            // the ends that open a chunk (two of them at order 4: the record before is in the chunk and an end, too)
            const int64_t in_chunk = t % q;
            if (want >> 30 != 0 && (in_chunk == 0 || (in_chunk == 1 && a.code[t - 1] >> 30 == 3))) want = kRecNothing;
            const int64_t s = parent_of(a.slice_rec, a.slices, t);
            if (a.slice_rec[s + 1] == t + 1) want |= kRecSliceEnd;
            if (a.code[t] != want || __double_as_longlong(a.out_vals[t]) != __double_as_longlong(value)) bad |= c.bad_code;
        } else if (t < a.total && (a.code[t] >> 29 != 0 || a.code[t] != uint32_t(a.idx_leaf[a.leaves - 1]) || a.out_vals[t] != 0.0)) bad |= c.bad_code;
        if (a.slices && t <= a.slices) {
            if (t == a.slices ? a.slice_rec[t] != a.n_rec : (a.slice_rec[t] < 0 || a.slice_rec[t + 1] <= a.slice_rec[t])) bad |= c.bad_chunk;
            else if (t < a.slices) {
                if (c.row_of_slice[t] != (c.compact ? int32_t(t) : c.idx0[t]) || c.row_of_slice[t] >= c.out_rows) bad |= c.bad_chunk;
                const int kind = share_of(a.slice_rec, t, q);
                if (kind && !share_listed(kind == 1 ? c.light : c.heavy, kind == 1 ? c.n_light : c.n_heavy,
                                          record_share(a.slice_rec, t, q, c.row_of_slice[t])))
                    bad |= c.bad_list;
            }
        }
        if (t < c.n_chunks) {
            const int64_t s = c.chunk_slice[t] & ~kChunkInside;
            if (s >= a.slices || a.slice_rec[s] > t * q || a.slice_rec[s + 1] <= t * q ||
                (a.slice_rec[s] != t * q) != ((c.chunk_slice[t] & kChunkInside) != 0))
                bad |= c.bad_chunk;
            // what is open behind the chunk: the fiber and the node of the next record, unless the chunk ends them
            const int64_t r1 = (t + 1) * q;
            int32_t o1 = -1, o2 = -1;
            if (r1 < a.n_rec) {
                if (a.code[r1 - 1] >> 30 == 0) o1 = a.idx_fiber[first_end(a.fibers, r1, [&](int64_t f) { return a.ptr_fiber[f + 1] + f + (a.nodes ? parent_of(a.ptr_node, a.nodes, f) : 0); })];
                if (a.nodes && a.code[r1 - 1] >> 30 != 2) o2 = a.idx_node[first_end(a.nodes, r1, [&](int64_t n) { return node_end_record(a, n); })];
            }
            if (c.open1[t] != o1 || (c.open2 && c.open2[t] != o2)) bad |= c.bad_chunk;
        }
        // the lists ascend (so that the searches above find what is there) and hold nothing else
        if (t < c.n_light && !share_entry_right(c.light, t, 1, a.slice_rec, a.slices, a.n_rec, q, c.row_of_slice)) bad |= c.bad_list;
        if (t < c.n_heavy && !share_entry_right(c.heavy, t, 2, a.slice_rec, a.slices, a.n_rec, q, c.row_of_slice)) bad |= c.bad_list;
        if (t < c.n_empty && (c.empty[t] < 0 || c.empty[t] >= c.out_rows || (t > 0 && c.empty[t - 1] >= c.empty[t]) ||
                              listed(c.idx0, a.slices, c.empty[t])))
            bad |= c.bad_list;
    }
    if (bad) atomicOr(flags, bad);
}

RecordFill view_of_stream(const conststn_csf_s *X, const RecordStream &rs) {
    const int n = X->order;
    RecordFill a{};
    a.leaves = X->nnz;
    a.fibers = X->nodes[n - 2];
    a.nodes = n == 4 ? X->nodes[1] : 0;
    a.slices = X->nodes[0];
    a.n_rec = a.leaves + a.fibers + a.nodes;
    a.total = rs.n_chunks * rs.q;
    a.ptr_slice = X->ptr[0].p;
    a.ptr_node = n == 4 ? X->ptr[1].p : nullptr;
    a.ptr_fiber = X->ptr[n - 2].p;
    a.idx_slice = X->idx[0].p;
    a.idx_node = n == 4 ? X->idx[1].p : nullptr;
    a.idx_fiber = X->idx[n - 2].p;
    a.idx_leaf = X->idx[n - 1].p;
    a.vals = X->vals.p;
    a.code = rs.code.p;
    a.out_vals = rs.vals.p;
    a.slice_rec = rs.slice_rec.p;
    return a;
}

}  // namespace

conststn_status check_record_stream(const conststn_plan_s *plan, unsigned bad_code, unsigned bad_chunk, unsigned bad_list,
                                    unsigned *flags) {
    const conststn_csf_s *X = plan->X;
    const RecordStream &rs = plan->records;
    RecordCheck c{};
    c.a = view_of_stream(X, rs);
    if (!plan->compact && !rs.zero_all && rs.n_empty != plan->out_rows - c.a.slices) {
        set_error("plan tables: %lld rows to clear where %lld are empty", (long long)rs.n_empty, (long long)(plan->out_rows - c.a.slices));
        return CONSTSTN_EINVAL;
    }
    c.q = rs.q;
    c.n_chunks = rs.n_chunks;
    c.out_rows = plan->out_rows;
    c.n_light = rs.n_light;
    c.n_heavy = rs.n_heavy;
    c.n_empty = rs.n_empty;
    c.chunk_slice = rs.chunk_slice.p;
    c.open1 = rs.open1.p;
    c.open2 = rs.open2.p;
    c.row_of_slice = rs.row_of_slice.p;
    c.light = rs.light_share.p;
    c.heavy = rs.heavy_share.p;
    c.empty = rs.empty.p;
    c.idx0 = X->idx[0].p;
    c.compact = plan->compact ? 1 : 0;
    c.bad_code = bad_code;
    c.bad_chunk = bad_chunk;
    c.bad_list = bad_list;
    const int64_t threads = std::max({c.a.total, c.a.slices + 1, rs.n_chunks, rs.n_empty});
    const dim3 grid{unsigned(std::min<int64_t>(div_up(threads, 256), int64_t(1) << 20))};
    check_records_kernel<<<grid, dim3(256)>>>(c, threads, flags);
    CST_HIP(hipGetLastError());
    return CONSTSTN_OK;
}

bool record_stream_fits(const conststn_csf_s *X, int R) {
    if ((X->order != 3 && X->order != 4) || R < 2 || R > 128) return false;
    for (int l = 1; l < X->order; ++l)
        if (X->dims[X->mode_order[l]] > int64_t(kRecIndex) + 1) return false;
    return X->nodes[X->order - 2] < (int64_t(1) << 31);
}

conststn_status build_record_stream(conststn_plan_s *plan) {
    const conststn_csf_s *X = plan->X;
    RecordStream &rs = plan->records;
    const int n = X->order, R = plan->rank_of_level[1];
    rs.levels = n - 1;
    RecordFill a = view_of_stream(X, rs);
    rs.slices = a.slices;
    rs.n_rec = a.n_rec;
    rs.n_chunks = rs.n_heavy = rs.n_light = rs.n_empty = 0;
    // Chunks: short enough that every SIMD has several wavefronts even for a small tensor, long enough that
    // their partial rows (two per chunk) and the loads at their start stay a small part.
    const int lanes = R <= 16 ? 8 : 16;
    int64_t q = plan->opt("mttkrp_chunk", 0);
    if (q <= 0) q = std::max<int64_t>(32, std::min<int64_t>(a.n_rec / (int64_t(plan->n_cus) * 4 * 12 * (64 / lanes)), 512));
    q = div_up(std::min<int64_t>(q, std::max<int64_t>(a.n_rec, 1)), 16) * 16;      // (the last chunk is filled up)
    rs.q = q;
    if (!plan->compact && a.slices < plan->out_rows) {
        // up to 2^24 empty rows the fix-up launch clears them (128 threads each at most, and a launch takes fewer
        // than 2^32; more are cut off without an error)
        rs.zero_all = plan->out_rows - a.slices > (int64_t(1) << 24);
        if (!rs.zero_all) {
            DevBuf<int64_t> flag;
            CST_TRY(flag.alloc(size_t(plan->out_rows)));
            empty_rows_kernel<<<blocks_for(plan->out_rows), dim3(256)>>>(plan->out_rows, a.slices, X->idx[0].p, flag.p);
            CST_HIP(hipGetLastError());
            CST_TRY(list_of_flags(flag, plan->out_rows, rs.empty, &rs.n_empty));
        }
    }
    if (a.leaves == 0) return CONSTSTN_OK;
    rs.n_chunks = div_up(a.n_rec, q);
    a.total = rs.n_chunks * q;
    DevBuf<int32_t> fiber_of, node_of;
    CST_TRY(fiber_of.alloc(size_t(a.leaves)));
    expand_parents_kernel<<<dim3(unsigned(div_up(a.leaves, kExpandTile))), dim3(256)>>>(a.leaves, a.fibers, a.ptr_fiber, fiber_of.p);
    CST_HIP(hipGetLastError());
    if (n == 4) {
        CST_TRY(node_of.alloc(size_t(a.fibers)));
        expand_parents_kernel<<<dim3(unsigned(div_up(a.fibers, kExpandTile))), dim3(256)>>>(a.fibers, a.nodes, a.ptr_node, node_of.p);
        CST_HIP(hipGetLastError());
    }
    CST_TRY(rs.code.alloc(size_t(a.total)));
    CST_TRY(rs.vals.alloc(size_t(a.total)));
    CST_TRY(rs.slice_rec.alloc(size_t(a.slices) + 1));
    CST_TRY(rs.row_of_slice.alloc(size_t(a.slices)));
    CST_TRY(rs.chunk_slice.alloc(size_t(rs.n_chunks)));
    CST_TRY(rs.open1.alloc(size_t(rs.n_chunks)));
    if (n == 4) CST_TRY(rs.open2.alloc(size_t(rs.n_chunks)));
    CST_TRY(rs.partial.alloc(size_t(rs.n_chunks) * 2 * size_t(R)));
    a.fiber_of = fiber_of.p;
    a.node_of = node_of.p;
    a.code = rs.code.p;
    a.out_vals = rs.vals.p;
    a.slice_rec = rs.slice_rec.p;
    record_leaves_kernel<<<blocks_for(a.leaves + a.total - a.n_rec), dim3(256)>>>(a);
    CST_HIP(hipGetLastError());
    record_ends_kernel<<<blocks_for(std::max(std::max(a.fibers, a.nodes), a.slices + 1)), dim3(256)>>>(a);
    CST_HIP(hipGetLastError());
    record_slices_kernel<<<blocks_for(a.slices), dim3(256)>>>(a);
    CST_HIP(hipGetLastError());
    record_chunks_kernel<<<blocks_for(rs.n_chunks), dim3(256)>>>(a, rs.n_chunks, q, rs.chunk_slice.p, rs.open1.p,
                                                                  n == 4 ? rs.open2.p : nullptr);
    CST_HIP(hipGetLastError());
    record_spent_ends_kernel<<<blocks_for(rs.n_chunks), dim3(256)>>>(rs.n_chunks, q, a.n_rec, rs.code.p);
    CST_HIP(hipGetLastError());
    CST_TRY(rs.zeros.alloc(size_t(R)));
    CST_TRY(zero_fill(rs.zeros.p, R, hipStream_t(0)));
    rows_of_slices_kernel<<<blocks_for(a.slices), dim3(256)>>>(a.slices, X->idx[0].p, plan->compact ? 1 : 0, rs.row_of_slice.p);
    CST_HIP(hipGetLastError());
    DevBuf<int64_t> flag;
    DevBuf<int> widest;
    DevBuf<int32_t> light, heavy;                                     // the slices themselves
    CST_TRY(flag.alloc(size_t(a.slices)));
    CST_TRY(widest.alloc(1));
    CST_HIP(hipMemset(widest.p, 0, sizeof(int)));
    record_shared_kernel<<<blocks_for(a.slices), dim3(256)>>>(a.slices, rs.slice_rec.p, q, 1, flag.p, widest.p);
    CST_HIP(hipGetLastError());
    CST_TRY(list_of_flags(flag, a.slices, light, &rs.n_light));
    record_shared_kernel<<<blocks_for(a.slices), dim3(256)>>>(a.slices, rs.slice_rec.p, q, 2, flag.p, widest.p);
    CST_HIP(hipGetLastError());
    CST_TRY(list_of_flags(flag, a.slices, heavy, &rs.n_heavy));
    CST_TRY(rs.heavy_share.alloc(size_t(rs.n_heavy)));
    CST_TRY(rs.light_share.alloc(size_t(rs.n_light)));
    record_shares_kernel<<<blocks_for(rs.n_heavy), dim3(256)>>>(rs.n_heavy, heavy.p, rs.slice_rec.p, rs.row_of_slice.p, q, rs.heavy_share.p);
    record_shares_kernel<<<blocks_for(rs.n_light), dim3(256)>>>(rs.n_light, light.p, rs.slice_rec.p, rs.row_of_slice.p, q, rs.light_share.p);
    CST_HIP(hipGetLastError());
    int span = 0;
    CST_HIP(hipMemcpy(&span, widest.p, sizeof(int), hipMemcpyDeviceToHost));
    rs.segments = span > kRecOneBlock ? kRecSegments : 1;
    if (rs.segments > 1) CST_TRY(rs.heavy_partial.alloc(size_t(rs.n_heavy) * kRecSegments * size_t(R)));
    CST_HIP(hipDeviceSynchronize());
    return CONSTSTN_OK;
}

template <int LEVELS, bool SHORT>
static void launch_records_kernel(const RecordArgs &a, hipStream_t stream) {
    const int lanes = a.R <= 16 ? 8 : 16;
    const dim3 grid(unsigned(div_up(a.n_chunks, 256 / lanes))), block(256);
    if (a.R <= 16) records_kernel<8, 1, LEVELS, SHORT><<<grid, block, 0, stream>>>(a);
    else if (a.R <= 32) records_kernel<16, 1, LEVELS, SHORT><<<grid, block, 0, stream>>>(a);
    else if (a.R <= 64) records_kernel<16, 2, LEVELS, SHORT><<<grid, block, 0, stream>>>(a);
    else if (a.R <= 96) records_kernel<16, 3, LEVELS, SHORT><<<grid, block, 0, stream>>>(a);
    else records_kernel<16, 4, LEVELS, SHORT><<<grid, block, 0, stream>>>(a);
}

conststn_status launch_record_stream(const conststn_plan_s *plan, const double *const *dense, double *out, hipStream_t stream) {
    const RecordStream &rs = plan->records;
    const int n = plan->X->order;
    RecordArgs a{};
    a.n_chunks = rs.n_chunks;
    a.q = int(rs.q);
    a.R = plan->rank_of_level[1];
    a.slices = int32_t(rs.slices);
    a.code = rs.code.p;
    a.vals = rs.vals.p;
    a.chunk_slice = rs.chunk_slice.p;
    a.open1 = rs.open1.p;
    a.open2 = rs.open2.p;
    a.row_of_slice = rs.row_of_slice.p;
    a.zeros = rs.zeros.p;
    a.f0 = dense[plan->factor_of_level[n - 1]];
    a.f1 = dense[plan->factor_of_level[n - 2]];
    a.f2 = n == 4 ? dense[plan->factor_of_level[1]] : nullptr;
    a.out = out;
    a.partial = rs.partial.p;
    if (rs.zero_all) CST_TRY(zero_fill(out, plan->out_rows * plan->row_elems, stream));
    if (rs.n_chunks > 0) {
        ProfScope prof(plan, stream);
        const bool small = rs.q <= kRecShort;
        if (rs.levels == 3) {
            if (small) launch_records_kernel<3, true>(a, stream);
            else launch_records_kernel<3, false>(a, stream);
        } else {
            if (small) launch_records_kernel<2, true>(a, stream);
            else launch_records_kernel<2, false>(a, stream);
        }
        CST_HIP(hipGetLastError());
    }
    RecordFixArgs f{};
    f.R = a.R;
    f.segments = rs.segments;
    f.n_heavy = rs.n_heavy;
    f.n_light = rs.n_light;
    f.n_empty = rs.n_empty;
    f.heavy = rs.heavy_share.p;
    f.light = rs.light_share.p;
    f.empty = rs.empty.p;
    f.partial = rs.partial.p;
    f.heavy_partial = rs.heavy_partial.p;
    f.out = out;
    const int W = a.R <= 16 ? 16 : (a.R <= 32 ? 32 : (a.R <= 64 ? 64 : 128));
    // A heavy slice's sum is a chain of loads as long as its chunks divided by the lane groups of a workgroup: large
    // workgroups where one does it alone (150 K nonzeros: 16.5 -> 13.7 us for the whole pass), small ones where several
    // share it and there are many slices (37 us at 76 M nonzeros against 116).
    const int threads = rs.segments == 1 ? 1024 : 256;
    f.heavy_blocks = rs.n_heavy * rs.segments;
    f.light_blocks = div_up(rs.n_light, threads / W);
    const int64_t blocks = f.heavy_blocks + f.light_blocks + div_up(rs.n_empty, threads / W);
    if (blocks == 0) return CONSTSTN_OK;
    const dim3 grid{unsigned(blocks)}, block{unsigned(threads)};
    auto run = [&](auto Wc) {
        constexpr int kW = decltype(Wc)::value;
        if (threads == 1024) records_fixup_kernel<kW, 1024><<<grid, block, 0, stream>>>(f);
        else records_fixup_kernel<kW, 256><<<grid, block, 0, stream>>>(f);
    };
    if (W == 16) run(std::integral_constant<int, 16>{});
    else if (W == 32) run(std::integral_constant<int, 32>{});
    else if (W == 64) run(std::integral_constant<int, 64>{});
    else run(std::integral_constant<int, 128>{});
    CST_HIP(hipGetLastError());
    if (rs.segments > 1 && rs.n_heavy > 0) {
        records_final_kernel<<<dim3(unsigned(rs.n_heavy)), dim3(128), 0, stream>>>(f);
        CST_HIP(hipGetLastError());
    }
    return CONSTSTN_OK;
}

}  // namespace cst
