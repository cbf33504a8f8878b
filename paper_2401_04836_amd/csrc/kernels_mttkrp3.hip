// Fused order-3 MTTKRP over a CSF tensor (Sec. 5.2):  M[i,r] = sum_{j,k} X[i,j,k] B[j,r] C[k,r].
//
// The schedule is the two-statement tree  T[i,j,r] = X[i,j,k] C[k,r] ; M[i,r] = T[i,j,r] B[j,r]
// fused on the loops i and j, so the intermediate shrinks to one length-R vector per (i,j)
// fiber (the reduced-order dense workspace of Fig. 3b); r is a batch index.
//
// Most MTTKRPs run on the record stream (kernels_records.hip); build_mttkrp3_tables chooses.  This file holds
//   - the form for rank 32 on large power-law tensors: the leaves whose factor row is among the most referenced
//     ("hot") ones and the others as two sub-tensors, walked side by side by two teams of wavefronts;
//   - the form that walks the CSF itself, for what the records cannot name: rank 1 (a lane takes a pair of
//     entries there) and extents above 2^28.
//
// The leaf array is cut into equal chunks (partition.hip).  A group of lanes owns one chunk and walks it leaf by
// leaf; each lane keeps two rank entries of the fiber vector T and of the slice accumulator in registers.  At a
// fiber end the group folds T * B[j,:] into the accumulator; at a slice end it puts the row into the result (slice
// wholly inside the chunk) or stores a partial row (slice shared with neighbouring chunks).  A second kernel adds
// the partial rows of shared slices in chunk order, so results are bit-reproducible.
#include <algorithm>

#include "plan.hpp"

namespace cst {

struct MttkrpArgs {
    int64_t nnz, q, n_chunks, slices;
    int R;
    const int64_t *ptr0, *ptr1;                // on the CSF itself only, as idx2 and compact
    const int32_t *idx0, *idx1, *idx2;         // result row of every slice; level-1 index of every fiber; leaves
    int compact;                               // 1: the result row is the slice's number
    int add;                                   // 1: rows are added to what the result holds (the two sub-tensors)
    const double *vals;
    const int64_t *chunk_fiber;
    const int32_t *chunk_slice;
    const int64_t *slice_leaf;
    const double *B, *C;
    double *out, *partial;
    const int32_t *heavy_slices;
    double *heavy_partial;
    int n_heavy;
};

typedef double v2f64_u __attribute__((ext_vector_type(2), aligned(8)));       // a pair of row entries at any double

// ---- on the CSF itself ------------------------------------------------------------------------
//
// Groups of LPR lanes, the smallest power of two with 2 LPR >= R.  PAIRS: an even rank, whose rows are read and
// written two entries at a time.  Slower than the stream wherever that applies (rank 50, 20 M nonzeros: 1.51 ms
// against 0.91): the loads of a step depend on the pointer arrays.
template <bool PAIRS>
__device__ __forceinline__ void load2(const double *__restrict__ row, int r0, int R, double &x, double &y) {
    if (PAIRS) {
        const v2f64_u v = *reinterpret_cast<const v2f64_u *>(row + r0);
        x = v[0];
        y = v[1];
    } else {
        x = r0 < R ? row[r0] : 0.0;
        y = r0 + 1 < R ? row[r0 + 1] : 0.0;
    }
}

template <bool PAIRS>
__device__ __forceinline__ void store2(double *__restrict__ row, int r0, int R, double x, double y) {
    if (PAIRS) {
        *reinterpret_cast<v2f64_u *>(row + r0) = v2f64_u{x, y};
    } else {
        if (r0 < R) row[r0] = x;
        if (r0 + 1 < R) row[r0 + 1] = y;
    }
}

template <int LPR, bool PAIRS>
__global__ void __launch_bounds__(256)
mttkrp3_csf_kernel(MttkrpArgs a) {
    const int64_t gid = (int64_t(blockIdx.x) * 256 + threadIdx.x) / LPR;
    const int gl = threadIdx.x % LPR;
    if (gid >= a.n_chunks) return;
    const int r0 = 2 * gl;
    const int R = a.R;
    if (PAIRS && r0 >= R) return;
    const int64_t n0 = gid * a.q;
    const int64_t n1 = n0 + a.q < a.nnz ? n0 + a.q : a.nnz;
    int64_t f = a.chunk_fiber[gid];
    int32_t s = a.chunk_slice[gid];
    const int32_t s_first = s;
    int64_t fiber_end = a.ptr1[f + 1];
    if (fiber_end > n1) fiber_end = n1;
    int64_t slice_fend = a.ptr0[s + 1];
    int32_t j = a.idx1[f];
    double t0 = 0.0, t1 = 0.0, acc0 = 0.0, acc1 = 0.0;

    auto emit = [&](int32_t sl, double x, double y) {
        const int64_t lo = a.slice_leaf[sl], hi = a.slice_leaf[sl + 1];
        if (lo >= n0 && hi <= n1) {
            const int64_t row = a.compact ? int64_t(sl) : int64_t(a.idx0[sl]);
            store2<PAIRS>(a.out + row * R, r0, R, x, y);
        } else {
            const int64_t slot = 2 * gid + (sl == s_first ? 0 : 1);
            store2<PAIRS>(a.partial + slot * R, r0, R, x, y);
        }
    };
    auto fiber_done = [&](int64_t n) {          // n = position after the fiber's last leaf in this chunk
        double b0, b1;
        load2<PAIRS>(a.B + int64_t(j) * R, r0, R, b0, b1);
        acc0 = fma(b0, t0, acc0);
        acc1 = fma(b1, t1, acc1);
        t0 = 0.0;
        t1 = 0.0;
        if (n < n1) {
            ++f;
            if (f == slice_fend) {
                emit(s, acc0, acc1);
                acc0 = 0.0;
                acc1 = 0.0;
                ++s;
                slice_fend = a.ptr0[s + 1];
            }
            j = a.idx1[f];
            fiber_end = a.ptr1[f + 1];
            if (fiber_end > n1) fiber_end = n1;
        }
    };

    constexpr int U = 4;
    int64_t n = n0;
    while (n + U <= n1) {
        int32_t kk[U];
        double vv[U], c0[U], c1[U];
#pragma unroll
        for (int u = 0; u < U; ++u) { kk[u] = a.idx2[n + u]; vv[u] = a.vals[n + u]; }
#pragma unroll
        for (int u = 0; u < U; ++u) load2<PAIRS>(a.C + int64_t(kk[u]) * R, r0, R, c0[u], c1[u]);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            t0 = fma(vv[u], c0[u], t0);
            t1 = fma(vv[u], c1[u], t1);
            ++n;
            if (n == fiber_end) fiber_done(n);
        }
    }
    for (; n < n1;) {
        const int32_t k = a.idx2[n];
        const double v = a.vals[n];
        double c0, c1;
        load2<PAIRS>(a.C + int64_t(k) * R, r0, R, c0, c1);
        t0 = fma(v, c0, t0);
        t1 = fma(v, c1, t1);
        ++n;
        if (n == fiber_end) fiber_done(n);
    }
    emit(s, acc0, acc1);
}

// ---- rank-32 path ---------------------------------------------------------------------------
//
// R = 32: a factor row is 256 B = 16 lanes x 16 B.  Built around the rate of vector-memory instructions per
// compute unit:
//   * the leaf stream is read 16 entries at a time, one entry per lane of the 16-lane group,
//     and handed round with DPP row broadcasts instead of one broadcast load per leaf;
//   * the stream is the plan's re-encoded copy of a sub-tensor: leaf indices, or LDS slots of the hot rows that
//     every workgroup stages once;
//   * end-of-fiber / end-of-slice marks travel in the stream, so the child-pointer arrays
//     are not read at all;
//   * workgroups are persistent and loop over chunks, so the staging cost is paid once.
constexpr uint32_t kFiberEnd = 0x40000000u, kSliceEnd = 0x20000000u,
                   kRowMask = 0x0fffffffu;

struct MttkrpR32Args {
    MttkrpArgs base;
    const uint32_t *code;
    const int32_t *hot_rows;
    int n_hot;
};

struct lds_pair { double x, y; };
typedef __attribute__((address_space(3))) lds_pair lds_double2;

template <int T>
__device__ __forceinline__ uint32_t row_bcast(uint32_t x) {
    return uint32_t(__builtin_amdgcn_mov_dpp(int(x), 0x150 + T, 0xf, 0xf, false));
}
template <int T>
__device__ __forceinline__ double row_bcast(double x) {
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(x), 0x150 + T, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(x), 0x150 + T, 0xf, 0xf, false);
    return __hiloint2double(hi, lo);
}

// Exclusive count, inside each 16-lane row, of the lanes below this one whose flag is set.
__device__ __forceinline__ int row_rank_of_flag(bool flag, int gl, int &row_total) {
    const unsigned long long m = __builtin_amdgcn_ballot_w64(flag);
    const int shift = (threadIdx.x & 48);                 // first lane of this row inside the wave
    const unsigned row = unsigned(m >> shift) & 0xffffu;
    row_total = __popc(row);
    return __popc(row & ((1u << gl) - 1u));
}

// HOT: every leaf's row is in LDS, and no gather for leaf rows goes to the vector-memory path; otherwise none is,
// and every one is fully populated.  The traversal is for NT threads (tid = 0 .. NT-1, whole wavefronts) that are
// the `part`-th of `parts` such teams: the teams share the chunks round-robin.  `hot` = the staged hot rows.
template <int NT, bool HOT>
__device__ __forceinline__ void mttkrp3_r32_body(const MttkrpR32Args &aa, int tid, int64_t part, int64_t parts,
                                                 const double2 *hot) {
    const MttkrpArgs &a = aa.base;
    const int gl = tid & 15;
    const lds_double2 *hot_lds = (const lds_double2 *)hot;
    const v2f64_u *Cv = reinterpret_cast<const v2f64_u *>(a.C);
    const v2f64_u *Bv = reinterpret_cast<const v2f64_u *>(a.B);
    const int64_t groups = parts * (NT / 16);
    // every lane group of a wave runs the same number of rounds so that the wave-wide ballot
    // and the row broadcasts below always execute with all rows present
    const int64_t rounds = (a.n_chunks + groups - 1) / groups;
    for (int64_t rnd = 0; rnd < rounds; ++rnd) {
        const int64_t c = rnd * groups + part * (NT / 16) + tid / 16;
        const bool live = c < a.n_chunks;
        const int64_t n0 = live ? c * a.q : 0;
        const int64_t n1 = live ? (n0 + a.q < a.nnz ? n0 + a.q : a.nnz) : 0;
        int64_t f = live ? a.chunk_fiber[c] : 0;          // first fiber not yet closed
        int32_t s = live ? a.chunk_slice[c] : 0;
        const int32_t s_first = s;
        double t0 = 0.0, t1 = 0.0, acc0 = 0.0, acc1 = 0.0;
        uint32_t last = kFiberEnd | kSliceEnd;            // marks of the last leaf consumed

        auto emit = [&]() {
            const int64_t lo = a.slice_leaf[s], hi = a.slice_leaf[s + 1];
            v2f64_u *dst;
            if (lo >= n0 && hi <= n1) {
                const int64_t row = a.idx0[s];
                dst = reinterpret_cast<v2f64_u *>(a.out + row * 32);
            } else {
                dst = reinterpret_cast<v2f64_u *>(a.partial + (2 * c + (s == s_first ? 0 : 1)) * 32);
            }
            if (lo >= n0 && hi <= n1) {
                const v2f64_u old = dst[gl];
                acc0 += old[0];
                acc1 += old[1];
            }
            dst[gl] = v2f64_u{acc0, acc1};
            acc0 = 0.0;
            acc1 = 0.0;
        };
        auto pair_of = [](v2f64_u x) -> double2 { return make_double2(x[0], x[1]); };
        // the factor row of a leaf; the LDS read goes through an explicitly LDS-qualified pointer
        auto fetch = [&](uint32_t cd) -> double2 {
            if (!HOT) return pair_of(Cv[(cd & kRowMask) * 16u + uint32_t(gl)]);
            const lds_double2 *src = hot_lds + ((cd & kRowMask) * 16 + gl);
            return make_double2(src->x, src->y);
        };
        // B row of the fiber that ends at this leaf (no load when the leaf ends no fiber)
        auto fetch_b = [&](uint32_t cd, int32_t j) -> double2 {
            double2 r = make_double2(0.0, 0.0);        // only used where the condition holds
            if (cd & kFiberEnd) r = pair_of(Bv[uint32_t(j) * 16u + uint32_t(gl)]);
            return r;
        };
        auto consume = [&](uint32_t cd, double v, double2 cv, double2 bv) {
            t0 = fma(v, cv.x, t0);
            t1 = fma(v, cv.y, t1);
            last = cd;
            if (cd & kFiberEnd) {
                acc0 = fma(bv.x, t0, acc0);
                acc1 = fma(bv.y, t1, acc1);
                t0 = 0.0;
                t1 = 0.0;
                if (cd & kSliceEnd) { emit(); ++s; }
            }
        };

        // Software pipeline over blocks of 16 leaves.  While block b is consumed, the leaf
        // entries of block b+2 and the level-1 indices (j) of the fibers ending in block b+1
        // are already in flight, and every load a block needs is issued before the first wait,
        // so no step waits on a dependent load.
        const int64_t nblocks = (n1 - n0 + 15) / 16;
        auto load_block = [&](int64_t blk, uint32_t &cd, double &vl) {
            cd = 0;
            vl = 0.0;
            const int64_t pos = n0 + blk * 16 + gl;
            if (blk < nblocks && pos < n1) { cd = aa.code[pos]; vl = a.vals[pos]; }
        };
        // j of the fiber closed by this lane's leaf, given the first fiber open at block start
        auto load_j = [&](uint32_t cd, int64_t fbase, int &ends) -> int32_t {
            const bool is_end = (cd & kFiberEnd) != 0;
            const int rank = row_rank_of_flag(is_end, gl, ends);
            int32_t j = 0;
            if (is_end) j = a.idx1[fbase + rank];
            return j;
        };
        uint32_t code_cur, code_nxt, code_n2 = 0;
        double val_cur, val_nxt, val_n2 = 0.0;
        load_block(0, code_cur, val_cur);
        load_block(1, code_nxt, val_nxt);
        int ends_cur = 0, ends_nxt = 0;
        int32_t j_cur = load_j(code_cur, f, ends_cur), j_nxt = 0;
        for (int64_t b = 0; b < nblocks; ++b) {
            const int64_t base = n0 + b * 16;
            load_block(b + 2, code_n2, val_n2);
            j_nxt = load_j(code_nxt, f + ends_cur, ends_nxt);
            if (base + 16 <= n1) {
                // Eight leaves at a time: what a step waits for is the B rows of the fibers that end in it (and the C
                // rows of cold leaves), a trip to L2 each time, so twice as many in flight halve the waits per block.
#define CST_GROUP8(T0)                                                                        \
                {                                                                             \
                    const uint32_t c0 = row_bcast<T0 + 0>(code_cur), c1 = row_bcast<T0 + 1>(code_cur), \
                                   c2 = row_bcast<T0 + 2>(code_cur), c3 = row_bcast<T0 + 3>(code_cur), \
                                   c4 = row_bcast<T0 + 4>(code_cur), c5 = row_bcast<T0 + 5>(code_cur), \
                                   c6 = row_bcast<T0 + 6>(code_cur), c7 = row_bcast<T0 + 7>(code_cur); \
                    const double2 b0 = fetch_b(c0, int32_t(row_bcast<T0 + 0>(uint32_t(j_cur)))), \
                                  b1 = fetch_b(c1, int32_t(row_bcast<T0 + 1>(uint32_t(j_cur)))), \
                                  b2 = fetch_b(c2, int32_t(row_bcast<T0 + 2>(uint32_t(j_cur)))), \
                                  b3 = fetch_b(c3, int32_t(row_bcast<T0 + 3>(uint32_t(j_cur)))), \
                                  b4 = fetch_b(c4, int32_t(row_bcast<T0 + 4>(uint32_t(j_cur)))), \
                                  b5 = fetch_b(c5, int32_t(row_bcast<T0 + 5>(uint32_t(j_cur)))), \
                                  b6 = fetch_b(c6, int32_t(row_bcast<T0 + 6>(uint32_t(j_cur)))), \
                                  b7 = fetch_b(c7, int32_t(row_bcast<T0 + 7>(uint32_t(j_cur)))); \
                    double2 g0, g1, g2, g3, g4, g5, g6, g7;                                   \
                    if (!HOT) {                                                               \
                        g0 = fetch(c0); g1 = fetch(c1); g2 = fetch(c2); g3 = fetch(c3);       \
                        g4 = fetch(c4); g5 = fetch(c5); g6 = fetch(c6); g7 = fetch(c7);       \
                    }                                                                         \
                    if (HOT) { g0 = fetch(c0); g1 = fetch(c1); g2 = fetch(c2); g3 = fetch(c3); } \
                    consume(c0, row_bcast<T0 + 0>(val_cur), g0, b0);                        \
                    consume(c1, row_bcast<T0 + 1>(val_cur), g1, b1);                        \
                    consume(c2, row_bcast<T0 + 2>(val_cur), g2, b2);                        \
                    consume(c3, row_bcast<T0 + 3>(val_cur), g3, b3);                        \
                    if (HOT) { g4 = fetch(c4); g5 = fetch(c5); g6 = fetch(c6); g7 = fetch(c7); } \
                    consume(c4, row_bcast<T0 + 4>(val_cur), g4, b4);                        \
                    consume(c5, row_bcast<T0 + 5>(val_cur), g5, b5);                        \
                    consume(c6, row_bcast<T0 + 6>(val_cur), g6, b6);                        \
                    consume(c7, row_bcast<T0 + 7>(val_cur), g7, b7);                        \
                }
                CST_GROUP8(0)
                CST_GROUP8(8)
#undef CST_GROUP8
            } else {
                // ragged tail of the last chunk: same steps, one leaf at a time, bounds-checked
                const int left = int(n1 - base);
#define CST_ONE(T)                                                                            \
                {                                                                             \
                    const uint32_t cd = row_bcast<T>(code_cur);                               \
                    const double v = row_bcast<T>(val_cur);                                   \
                    const int32_t jj = int32_t(row_bcast<T>(uint32_t(j_cur)));                \
                    if (T < left) consume(cd, v, fetch(cd), fetch_b(cd, jj)); \
                }
                CST_ONE(0) CST_ONE(1) CST_ONE(2) CST_ONE(3) CST_ONE(4) CST_ONE(5) CST_ONE(6) CST_ONE(7)
                CST_ONE(8) CST_ONE(9) CST_ONE(10) CST_ONE(11) CST_ONE(12) CST_ONE(13) CST_ONE(14) CST_ONE(15)
#undef CST_ONE
            }
            f += ends_cur;
            code_cur = code_nxt;
            val_cur = val_nxt;
            code_nxt = code_n2;
            val_nxt = val_n2;
            j_cur = j_nxt;
            ends_cur = ends_nxt;
        }
        if (!(last & kFiberEnd)) {                         // the chunk ends inside fiber f
            const double2 bv = pair_of(Bv[int64_t(a.idx1[f]) * 16 + gl]);
            acc0 = fma(bv.x, t0, acc0);
            acc1 = fma(bv.y, t1, acc1);
        }
        if (!(last & kSliceEnd)) emit();
    }
}

// Hot and cold sub-tensor in ONE launch: the first NH wavefronts of every workgroup walk chunks of the
// hot sub-tensor (rows from LDS: vector issue slots and LDS bandwidth), the other NC chunks of the cold
// one (rows from L2 / memory: the vector-memory path), so that the two passes load different units of
// a CU at the same time instead of one after the other.  The two write different buffers (the cold team
// `cold.base.out`), added afterwards: both may own the same output row.
struct MttkrpDualArgs { MttkrpR32Args hot, cold; };

template <int NH, int NC>
__global__ void __launch_bounds__(64 * (NH + NC), 4)
mttkrp3_r32_dual_kernel(MttkrpDualArgs d) {
    extern __shared__ double2 hot[];                       // n_hot rows x 16 pairs
    for (int e = threadIdx.x; e < d.hot.n_hot * 16; e += 64 * (NH + NC))
    {
        const v2f64_u x = reinterpret_cast<const v2f64_u *>(d.hot.base.C + int64_t(d.hot.hot_rows[e >> 4]) * 32)[e & 15];
        hot[e] = make_double2(x[0], x[1]);
    }
    __syncthreads();
    if (threadIdx.x < 64 * NH) mttkrp3_r32_body<64 * NH, true>(d.hot, int(threadIdx.x), int64_t(blockIdx.x), int64_t(gridDim.x), hot);
    else mttkrp3_r32_body<64 * NC, false>(d.cold, int(threadIdx.x) - 64 * NH, int64_t(blockIdx.x), int64_t(gridDim.x), hot);
}

__global__ void __launch_bounds__(256)
mttkrp3_add_kernel(v2f64_u *__restrict__ out, const v2f64_u *__restrict__ add, int64_t n) {
    for (int64_t e = int64_t(blockIdx.x) * 256 + threadIdx.x; e < n; e += int64_t(gridDim.x) * 256) out[e] += add[e];
}

// Rows of slices shared by several chunks: add the partial rows in chunk order.
// One block per slice; G lane groups stride over the chunks, then a fixed-order LDS reduction.
template <int LPR>
__device__ __forceinline__ void mttkrp3_fixup_body(const MttkrpArgs &a, int64_t s, double *red) {
    constexpr int G = 256 / LPR;
    const int64_t lo = a.slice_leaf[s], hi = a.slice_leaf[s + 1];
    const int64_t ca = lo / a.q, cb = (hi - 1) / a.q;
    if (ca == cb) return;                           // stored directly by the main kernel
    if (cb - ca >= kHeavySpan) return;              // left to the two-stage kernels below
    const int g = threadIdx.x / LPR, gl = threadIdx.x % LPR;
    const int r0 = 2 * gl, R = a.R;
    double x = 0.0, y = 0.0;
    for (int64_t c = ca + g; c <= cb; c += G) {
        const int64_t slot = 2 * c + ((c == ca && lo != ca * a.q) ? 1 : 0);
        const double *row = a.partial + slot * R;
        if (r0 < R) x += row[r0];
        if (r0 + 1 < R) y += row[r0 + 1];
    }
    red[threadIdx.x * 2] = x;
    red[threadIdx.x * 2 + 1] = y;
    __syncthreads();
    if (g == 0) {
        for (int gg = 1; gg < G; ++gg) {
            x += red[(gg * LPR + gl) * 2];
            y += red[(gg * LPR + gl) * 2 + 1];
        }
        const int64_t row = a.compact ? s : int64_t(a.idx0[s]);
        if (a.add) {
            if (r0 < R) x += a.out[row * R + r0];
            if (r0 + 1 < R) y += a.out[row * R + r0 + 1];
        }
        if (r0 < R) a.out[row * R + r0] = x;
        if (r0 + 1 < R) a.out[row * R + r0 + 1] = y;
    }
}
// Heavy slices (shared by at least kHeavySpan chunks): stage 1 reduces kHeavySegments equal
// segments of the slice's chunk range in parallel, stage 2 adds the segment sums in order.
template <int LPR>
__device__ __forceinline__ void mttkrp3_fixup_heavy_body(const MttkrpArgs &a, int64_t h, int seg, double *red) {
    constexpr int G = 256 / LPR;
    const int64_t s = a.heavy_slices[h];
    const int64_t lo = a.slice_leaf[s], hi = a.slice_leaf[s + 1];
    const int64_t ca = lo / a.q, cb = (hi - 1) / a.q;
    const int64_t n = cb - ca + 1;
    const int64_t c0 = ca + n * seg / kHeavySegments, c1 = ca + n * (seg + 1) / kHeavySegments;
    const int g = threadIdx.x / LPR, gl = threadIdx.x % LPR;
    const int r0 = 2 * gl, R = a.R;
    double x = 0.0, y = 0.0;
    for (int64_t c = c0 + g; c < c1; c += G) {
        const int64_t slot = 2 * c + ((c == ca && lo != ca * a.q) ? 1 : 0);
        const double *row = a.partial + slot * R;
        if (r0 < R) x += row[r0];
        if (r0 + 1 < R) y += row[r0 + 1];
    }
    red[threadIdx.x * 2] = x;
    red[threadIdx.x * 2 + 1] = y;
    __syncthreads();
    if (g == 0) {
        for (int gg = 1; gg < G; ++gg) {
            x += red[(gg * LPR + gl) * 2];
            y += red[(gg * LPR + gl) * 2 + 1];
        }
        double *dst = a.heavy_partial + (h * kHeavySegments + seg) * R;
        if (r0 < R) dst[r0] = x;
        if (r0 + 1 < R) dst[r0 + 1] = y;
    }
}
__device__ __forceinline__ void mttkrp3_fixup_final_body(const MttkrpArgs &a, int64_t h) {
    const int64_t s = a.heavy_slices[h];
    const int r = threadIdx.x;
    if (r >= a.R) return;
    double x = 0.0;
    for (int seg = 0; seg < kHeavySegments; ++seg)
        x += a.heavy_partial[(h * kHeavySegments + seg) * a.R + r];
    const int64_t row = a.compact ? s : int64_t(a.idx0[s]);
    if (a.add) x += a.out[row * a.R + r];
    a.out[row * a.R + r] = x;
}
// The three passes for the two sub-tensors, which write different outputs, in one launch each: the
// first blocks take the first sub-tensor's slices (heavy slices), the others the second's.
// A launch takes fewer than 2^32 threads (more are cut off without an error), so the slices from s0 on go 2^23 at a time
// (a loop over slices in the kernel costs 20 % of the whole at rank 1 over a million short slices).
struct MttkrpPairArgs { MttkrpArgs first, second; };
constexpr int64_t kFixupBlocks = int64_t(1) << 23;
template <int LPR>
__global__ void __launch_bounds__(256)
mttkrp3_fixup_pair_kernel(MttkrpPairArgs p, int64_t s0) {
    __shared__ double red[256 * 2];
    const int64_t s = s0 + blockIdx.x;
    if (s < p.first.slices) mttkrp3_fixup_body<LPR>(p.first, s, red);
    else mttkrp3_fixup_body<LPR>(p.second, s - p.first.slices, red);
}
template <int LPR>
__global__ void __launch_bounds__(256)
mttkrp3_fixup_heavy_pair_kernel(MttkrpPairArgs p) {
    __shared__ double red[256 * 2];
    if (int(blockIdx.x) < p.first.n_heavy) mttkrp3_fixup_heavy_body<LPR>(p.first, blockIdx.x, int(blockIdx.y), red);
    else mttkrp3_fixup_heavy_body<LPR>(p.second, int64_t(blockIdx.x) - p.first.n_heavy, int(blockIdx.y), red);
}
__global__ void __launch_bounds__(128)
mttkrp3_fixup_final_pair_kernel(MttkrpPairArgs p) {
    if (int(blockIdx.x) < p.first.n_heavy) mttkrp3_fixup_final_body(p.first, blockIdx.x);
    else mttkrp3_fixup_final_body(p.second, int64_t(blockIdx.x) - p.first.n_heavy);
}

template <int LPR>
static conststn_status launch_fixup_pair(const MttkrpArgs &a0, const MttkrpArgs &a1, hipStream_t stream) {
    const MttkrpPairArgs p{a0, a1};
    for (int64_t s0 = 0, n = a0.slices + a1.slices; s0 < n; s0 += kFixupBlocks) {
        mttkrp3_fixup_pair_kernel<LPR><<<dim3(unsigned(std::min(n - s0, kFixupBlocks))), dim3(256), 0, stream>>>(p, s0);
        CST_HIP(hipGetLastError());
    }
    const int nh = a0.n_heavy + a1.n_heavy;
    if (nh > 0) {
        mttkrp3_fixup_heavy_pair_kernel<LPR><<<dim3(unsigned(nh), kHeavySegments), dim3(256), 0, stream>>>(p);
        CST_HIP(hipGetLastError());
        mttkrp3_fixup_final_pair_kernel<<<dim3(unsigned(nh)), dim3(128), 0, stream>>>(p);
        CST_HIP(hipGetLastError());
    }
    return CONSTSTN_OK;
}

// The hot rows lie in dynamic LDS (256 B per row): its limit is raised when the plan is built.
conststn_status prepare_mttkrp3_launch(conststn_plan_s *plan) {
    const void *dual = nullptr;
    switch (plan->mttkrp_dual) {
        case 35: dual = reinterpret_cast<const void *>(&mttkrp3_r32_dual_kernel<3, 5>); break;
        case 53: dual = reinterpret_cast<const void *>(&mttkrp3_r32_dual_kernel<5, 3>); break;
        case 88: dual = reinterpret_cast<const void *>(&mttkrp3_r32_dual_kernel<8, 8>); break;
        default: dual = reinterpret_cast<const void *>(&mttkrp3_r32_dual_kernel<4, 4>); break;
    }
    CST_HIP(hipFuncSetAttribute(dual, hipFuncAttributeMaxDynamicSharedMemorySize, plan->n_hot * 256));
    return CONSTSTN_OK;
}

conststn_status launch_mttkrp3(const conststn_plan_s *plan, const double *const *dense, double *out,
                               hipStream_t stream) {
    // X = X_hot + X_cold: the hot sub-tensor writes the output, the cold team its own buffer, added afterwards
    const int64_t n = plan->out_rows * plan->row_elems;
    CST_TRY(zero_fill(out, n, stream));
    CST_TRY(zero_fill(plan->mttkrp_out2.p, n, stream));
    MttkrpR32Args pa[2];
    for (int part = 0; part < 2; ++part) {
        const MttkrpPart &P = plan->part[part];
        MttkrpR32Args &aa = pa[part];
        aa = MttkrpR32Args{};
        aa.base.nnz = P.nnz;
        aa.base.q = P.chunk_q;
        aa.base.n_chunks = P.n_chunks;
        aa.base.slices = P.slices;
        aa.base.R = plan->rank_of_level[1];
        aa.base.idx0 = P.row_of_slice.p;
        aa.base.idx1 = P.idx1.p;
        aa.base.add = 1;
        aa.base.vals = P.vals.p;
        aa.base.chunk_fiber = P.chunk_fiber.p;
        aa.base.chunk_slice = P.chunk_slice.p;
        aa.base.slice_leaf = P.slice_leaf.p;
        aa.base.B = dense[plan->factor_of_level[1]];
        aa.base.C = dense[plan->factor_of_level[2]];
        aa.base.out = part == 0 ? out : plan->mttkrp_out2.p;
        aa.base.partial = P.partial.p;
        aa.base.heavy_slices = P.heavy_slices.p;
        aa.base.heavy_partial = P.heavy_partial.p;
        aa.base.n_heavy = P.n_heavy;
        aa.code = P.code.p;
        aa.hot_rows = plan->hot_rows.p;
        aa.n_hot = plan->n_hot;
    }
    const MttkrpDualArgs d{pa[0], pa[1]};
    // wavefronts per workgroup, and as many workgroups per CU as its LDS and its registers (96 per
    // lane: five wavefronts per SIMD) hold
    const size_t lds = size_t(plan->n_hot) * 256;
    const int waves = plan->mttkrp_dual / 10 + plan->mttkrp_dual % 10;
    const int per_cu = std::max(1, std::min(int(160 * 1024 / lds), 20 / waves));
    const dim3 grid(unsigned(plan->n_cus * per_cu)), block(unsigned(64 * waves));
    {
        ProfScope prof(plan, stream);
        switch (plan->mttkrp_dual) {
            case 35: mttkrp3_r32_dual_kernel<3, 5><<<grid, block, lds, stream>>>(d); break;
            case 53: mttkrp3_r32_dual_kernel<5, 3><<<grid, block, lds, stream>>>(d); break;
            case 88: mttkrp3_r32_dual_kernel<8, 8><<<grid, block, lds, stream>>>(d); break;
            default: mttkrp3_r32_dual_kernel<4, 4><<<grid, block, lds, stream>>>(d); break;
        }
        CST_HIP(hipGetLastError());
    }
    CST_TRY(launch_fixup_pair<16>(pa[0].base, pa[1].base, stream));
    mttkrp3_add_kernel<<<dim3(unsigned(std::min(div_up(n / 2, 256), kFixupBlocks))), dim3(256), 0, stream>>>(
        reinterpret_cast<v2f64_u *>(out), reinterpret_cast<const v2f64_u *>(plan->mttkrp_out2.p), n / 2);
    CST_HIP(hipGetLastError());
    return CONSTSTN_OK;
}

// A tensor by itself.  (With 1.3 M slices of 1.6 leaves the passes are most of the time, and the pair's kernels, which read
// twice the arguments and a branch more per slice, cost 10 % of the whole.)
template <int LPR>
__global__ void __launch_bounds__(256)
mttkrp3_fixup_kernel(MttkrpArgs a, int64_t s0) {
    __shared__ double red[256 * 2];
    mttkrp3_fixup_body<LPR>(a, s0 + blockIdx.x, red);
}
template <int LPR>
__global__ void __launch_bounds__(256)
mttkrp3_fixup_heavy_kernel(MttkrpArgs a) {
    __shared__ double red[256 * 2];
    mttkrp3_fixup_heavy_body<LPR>(a, blockIdx.x, int(blockIdx.y), red);
}
__global__ void __launch_bounds__(128)
mttkrp3_fixup_final_kernel(MttkrpArgs a) {
    mttkrp3_fixup_final_body(a, blockIdx.x);
}

template <int LPR>
static conststn_status launch_csf(const conststn_plan_s *plan, const MttkrpArgs &a, hipStream_t stream) {
    const dim3 grid(unsigned(div_up(a.n_chunks, 256 / LPR))), block(256);
    {
        ProfScope prof(plan, stream);
        if (a.R % 2 == 0) mttkrp3_csf_kernel<LPR, true><<<grid, block, 0, stream>>>(a);
        else mttkrp3_csf_kernel<LPR, false><<<grid, block, 0, stream>>>(a);
    }
    CST_HIP(hipGetLastError());
    for (int64_t s0 = 0; s0 < a.slices; s0 += kFixupBlocks) {
        mttkrp3_fixup_kernel<LPR><<<dim3(unsigned(std::min(a.slices - s0, kFixupBlocks))), block, 0, stream>>>(a, s0);
        CST_HIP(hipGetLastError());
    }
    if (a.n_heavy > 0) {
        mttkrp3_fixup_heavy_kernel<LPR><<<dim3(unsigned(a.n_heavy), kHeavySegments), block, 0, stream>>>(a);
        CST_HIP(hipGetLastError());
        mttkrp3_fixup_final_kernel<<<dim3(unsigned(a.n_heavy)), dim3(128), 0, stream>>>(a);
        CST_HIP(hipGetLastError());
    }
    return CONSTSTN_OK;
}

conststn_status launch_mttkrp3_csf(const conststn_plan_s *plan, const double *const *dense, double *out, hipStream_t stream) {
    const conststn_csf_s *X = plan->X;
    const MttkrpPart &P = plan->part[0];                    // chunk tables over X itself
    MttkrpArgs a{};
    a.nnz = X->nnz;
    a.q = P.chunk_q;
    a.n_chunks = P.n_chunks;
    a.slices = X->nodes[0];
    a.R = plan->rank_of_level[1];
    a.ptr0 = X->ptr[0].p;
    a.ptr1 = X->ptr[1].p;
    a.idx0 = X->idx[0].p;
    a.idx1 = X->idx[1].p;
    a.idx2 = X->idx[2].p;
    a.compact = plan->compact ? 1 : 0;
    a.vals = X->vals.p;
    a.chunk_fiber = P.chunk_fiber.p;
    a.chunk_slice = P.chunk_slice.p;
    a.slice_leaf = P.slice_leaf.p;
    a.B = dense[plan->factor_of_level[1]];
    a.C = dense[plan->factor_of_level[2]];
    a.out = out;
    a.partial = P.partial.p;
    a.heavy_slices = P.heavy_slices.p;
    a.heavy_partial = P.heavy_partial.p;
    a.n_heavy = P.n_heavy;
    if (!plan->compact && a.slices < plan->out_rows)        // rows of empty slices are zero
        CST_TRY(zero_fill(out, plan->out_rows * plan->row_elems, stream));
    if (a.nnz == 0) return CONSTSTN_OK;
    int lpr = 1;
    while (2 * lpr < a.R) lpr *= 2;
    switch (lpr) {
        case 1: return launch_csf<1>(plan, a, stream);
        case 2: return launch_csf<2>(plan, a, stream);
        case 4: return launch_csf<4>(plan, a, stream);
        case 8: return launch_csf<8>(plan, a, stream);
        case 16: return launch_csf<16>(plan, a, stream);
        case 32: return launch_csf<32>(plan, a, stream);
        default: return launch_csf<64>(plan, a, stream);
    }
}

}  // namespace cst
