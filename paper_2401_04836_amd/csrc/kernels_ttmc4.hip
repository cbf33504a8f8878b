// Fused order-4 TTMc over a CSF tensor (order-4 form of Sec. 5.3):
//     Y[i,r1,r2,r3] = sum_{j,k,l} X[i,j,k,l] U1[j,r1] U2[k,r2] U3[l,r3]
// as the three-statement tree
//     T1[i,j,k,r3] = X U3 ;  T2[i,j,r2,r3] = T1 U2 ;  Y[i,r1,r2,r3] = T2 U1
// fused on (i,j,k) and (i,j): T1 shrinks to a length-R3 vector per (i,j,k) node and T2 to an
// R2 x R3 matrix per (i,j) fiber -- the largest intermediate is order 2 (the l = 2 solution
// of Sec. 3).
//
// General kernel, ranks up to 16: one wavefront per work item (a range of (i,j) fibers of one
// slice).  Lane = (q, r3) with q = lane/16: the four lane rows split the leaves of a node for
// T1 (then an xor-shuffle sum), and row q holds T2[r2, r3] for r2 = q, q+4, q+8, q+12 and the
// matching 16 x 4 part of Y_i in registers.
#include <type_traits>

#include "plan.hpp"

namespace cst {

struct Ttmc4Args {
    int64_t n_items;
    int R1, R2, R3;
    const int64_t *ptr1, *ptr2;
    const int32_t *idx0, *idx1, *idx2, *idx3;
    const double *vals;
    const SliceItem *items;
    const double *U1, *U2, *U3;
    double *out, *partial;
    int compact;
};

__device__ __forceinline__ int64_t uni64(int64_t v) {
    const int lo = __builtin_amdgcn_readfirstlane(int(v & 0xffffffffll));
    const int hi = __builtin_amdgcn_readfirstlane(int(v >> 32));
    return (int64_t(hi) << 32) | int64_t(uint32_t(lo));
}

__global__ void __launch_bounds__(256)
ttmc4_kernel(Ttmc4Args a) {
    const int lane = threadIdx.x % 64;
    const int64_t w = uni64(int64_t(blockIdx.x) * 4 + threadIdx.x / 64);
    if (w >= a.n_items) return;
    const SliceItem it = a.items[w];
    const int32_t s = __builtin_amdgcn_readfirstlane(it.slice);
    const int64_t fa = uni64(it.begin), fb = uni64(it.end), dest = uni64(it.dest);
    const int R1 = a.R1, R2 = a.R2, R3 = a.R3;
    const int q = lane / 16, c3 = lane % 16;
    const bool col_ok = c3 < R3;
    const int col = col_ok ? c3 : 0;

    double y[16][4];
#pragma unroll
    for (int r = 0; r < 16; ++r)
#pragma unroll
        for (int t = 0; t < 4; ++t) y[r][t] = 0.0;

    for (int64_t f = fa; f < fb; ++f) {
        const int32_t j = __builtin_amdgcn_readfirstlane(a.idx1[f]);
        const int64_t ga = uni64(a.ptr1[f]), gb = uni64(a.ptr1[f + 1]);
        double t2[4] = {0.0, 0.0, 0.0, 0.0};
        for (int64_t g = ga; g < gb; ++g) {
            const int32_t k = __builtin_amdgcn_readfirstlane(a.idx2[g]);
            const int64_t la = uni64(a.ptr2[g]), lb = uni64(a.ptr2[g + 1]);
            double t1 = 0.0;
            for (int64_t n = la; n < lb; n += 4) {
                const int64_t m = n + q;
                if (m < lb) {
                    const int32_t l = a.idx3[m];
                    t1 = fma(a.vals[m], a.U3[int64_t(l) * R3 + col], t1);
                }
            }
            t1 += __shfl_xor(t1, 16, 64);
            t1 += __shfl_xor(t1, 32, 64);
            const double *u2 = a.U2 + int64_t(k) * R2;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int r2 = q + 4 * t;
                if (r2 < R2) t2[t] = fma(u2[r2], t1, t2[t]);
            }
        }
        const double *u1 = a.U1 + int64_t(j) * R1;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            if (r < R1) {
                const double u = u1[r];
#pragma unroll
                for (int t = 0; t < 4; ++t) y[r][t] = fma(u, t2[t], y[r][t]);
            }
        }
    }
    const int64_t RR = int64_t(R1) * R2 * R3;
    double *base = dest < 0 ? a.out + (a.compact ? int64_t(s) : int64_t(a.idx0[s])) * RR
                            : a.partial + dest * RR;
    if (col_ok) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            if (r < R1) {
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const int r2 = q + 4 * t;
                    if (r2 < R2) base[(int64_t(r) * R2 + r2) * R3 + c3] = y[r][t];
                }
            }
        }
    }
}

// ---- MFMA kernel (any ranks up to 16) ---------------------------------------------------------
//
// Both dense stages run on the fp64 matrix cores:
//   mid level   T2_f (R2 x R3)     = sum over the fiber's pieces  U2[k,:]^T . T1   K = four pieces
//   slice level Y_i  (R1 x R2 R3) += U1[J,:]^T . T2                                K = four fibers
// A piece is at most two leaves of one (i,j,k) node.  The plan stores the pieces of a fiber four
// at a time in "groups" (the last group of a fiber padded with empty records) and the fibers of
// a slice four at a time in "K-steps"; a long node or fiber simply gives several pieces or
// groups, which is legal by distributivity, so the kernel walks ONE flat stream of groups whatever
// the skew of the tensor.  Per group: lane (s,c) takes record s -- level-2 index, two leaf indices,
// two leaf values, 32 bytes -- builds T1_s[r3 = c] and supplies U2[k_s, r2 = c]; one 16x16x4
// instruction adds the group to the fiber's T2 (accumulator layout: register v of lane
// (s,c) = T2[r2 = s+4v][r3 = c]).  When a group ends its fiber the tile goes to the wave-private
// LDS buffer, flat over (r2,r3); when it ends its K-step, slot s reads back the tile of fiber s.
// The structure (ends a fiber / ends a K-step / starts a K-step, and the four j of a K-step) travels
// in the records, so nothing but the stream itself is read.
// All ranks 16: sixteen 16x16x4 instructions per K-step, A = U1[j_s, c], B = row r2 of the four tiles.
// Ranks below 16: the slice level runs on the 4x4x4 instruction with four blocks (7 ns of a SIMD
// against 27), whose blocks take sixteen flat elements (r2,r3) as rows and the same four r1, held by
// every block, as columns: only the products that hold results are issued, ceil(R1/4) per sixteen flat
// elements.  Which flat element is which row is free, as the operand comes out of LDS: lane (s, 4 b + x)
// reads elements 32 u + 2 (4 x + b) and the next in one 16-byte read.  Operand lanes beyond a rank
// repeat its last column; what they produce stays in rows and columns that are not stored.
// (With all ranks 16 the 4x4x4 form issues 64 instructions for 16 and measured slower: 3.9 ms against
// 3.07 at 40 M nonzeros.)
// Records are fetched three groups ahead and the factor rows one group ahead (register rings,
// loop unrolled four times), so a group waits for no load issued in its own iteration.
// Ranks below 16 against the general kernel: 8 x 8 x 8, 5.3 M nonzeros, 2.26 -> 0.60 ms;
// 10 x 12 x 7, 5.4 M, 2.96 -> 0.34 ms and 63 K, 345 -> 33 us.
typedef double v4d __attribute__((ext_vector_type(4)));
typedef double v2d __attribute__((ext_vector_type(2)));
typedef double v2d_u __attribute__((ext_vector_type(2), aligned(8)));     // a pair at any element

struct Ttmc4RowArgs {
    int64_t n_items;
    int R1, R2, R3;
    const int64_t *kstep_group;
    const PieceDesc *rec;
    const int32_t *idx0;
    const SliceItem *items;                 // ranges of K-steps inside one slice
    const double *U1, *U2, *U3;
    double *out, *partial;
    int compact;
};

// One wavefront per workgroup: items differ in length, and a wavefront slot shared with three
// others stays idle until the longest of them is done.
// MU: 32-element parts of a T2 tile the instance has room for; FULL: all ranks 16.
template <int MU, bool FULL>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2, 8)))
ttmc4_mfma_kernel(Ttmc4RowArgs a) {
    constexpr int kStride = MU * 32 + 16;    // doubles per tile in LDS (+16: bank skew)
    __shared__ __align__(16) double lds[4 * kStride];
    const int lane = threadIdx.x;
    const int slot = lane >> 4, c = lane & 15;
    const int R1 = FULL ? 16 : a.R1, R2 = FULL ? 16 : a.R2, R3 = FULL ? 16 : a.R3;
    const int R23 = R2 * R3;
    const int nu = (R23 + 31) / 32, nq = (R1 + 3) / 4;
    const int c2 = FULL ? c : min(c, R2 - 1), c3 = FULL ? c : min(c, R3 - 1);
    // all ranks 16: tiles of absent fibers are multiplied by a zero A operand, so whatever they hold must be finite
    if (FULL)
        for (int e = lane; e < 4 * kStride; e += 64) lds[e] = 0.0;
    const int64_t w = int64_t(blockIdx.x);
    const SliceItem it = a.items[w];
    const int32_t s = __builtin_amdgcn_readfirstlane(it.slice);
    const int64_t dest = uni64(it.dest);
    const int64_t ga = uni64(a.kstep_group[it.begin]), gb = uni64(a.kstep_group[it.end]);

    v4d y[FULL ? 16 : 1];                    // all ranks 16: y[t][v] = Y[r1 = slot + 4v][r2 = t][r3 = c]
    double acc[FULL ? 1 : 2 * MU][4];        // below: acc[2 u + e][q] = Y[r1 = 4 q + c % 4][flat = 32 u + 2 (4 slot + c / 4) + e]
#pragma unroll
    for (int t = 0; t < (FULL ? 16 : 1); ++t) y[t] = v4d{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int t = 0; t < (FULL ? 1 : 2 * MU); ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[t][q] = 0.0;
    v4d t2 = v4d{0.0, 0.0, 0.0, 0.0};
    double uq[FULL ? 1 : 4];                 // U1[j_s, c], or U1[j_s, 4 q + c % 4], of the current K-step
#pragma unroll
    for (int q = 0; q < (FULL ? 1 : 4); ++q) uq[q] = 0.0;
    bool here = true;                        // the current K-step has a fiber s
    int ft = 0;                              // fibers of the current K-step already parked in LDS

    // A group's four records are 128 bytes.  Lane (s, c) fetches dword c mod 8 of record s -- one
    // 4-byte load per lane for the whole group instead of two 16-byte ones -- and the eight
    // dwords of a record are handed round inside the 16-lane row when they are needed.
    constexpr int kRec = 4, kRow = 2;        // record and row rings: fetched kRec - 1 and kRow - 1 groups ahead
    uint32_t raw[kRec];
    double gu2[kRow], gx0[kRow], gx1[kRow];
    const uint32_t *words = reinterpret_cast<const uint32_t *>(a.rec);
    auto load_rec = [&](int64_t g) -> uint32_t {
        return words[((g < gb ? g : gb - 1) * 4 + slot) * 8 + (c & 7)];
    };
    auto field = [&](uint32_t x, auto which) -> int32_t {
        return __builtin_amdgcn_mov_dpp(int(x), 0x150 + decltype(which)::value, 0xf, 0xf, false);
    };
    auto field64 = [&](uint32_t x, auto lo, auto hi) -> double {
        return __hiloint2double(field(x, hi), field(x, lo));
    };
    using W0 = std::integral_constant<int, 0>;
    using W1 = std::integral_constant<int, 1>;
    using W2 = std::integral_constant<int, 2>;
    using W3 = std::integral_constant<int, 3>;
    using W4 = std::integral_constant<int, 4>;
    using W5 = std::integral_constant<int, 5>;
    using W6 = std::integral_constant<int, 6>;
    using W7 = std::integral_constant<int, 7>;
    const char *U1b = reinterpret_cast<const char *>(a.U1), *U2b = reinterpret_cast<const char *>(a.U2),
               *U3b = reinterpret_cast<const char *>(a.U3);
    auto load_rows = [&](uint32_t x, double &u2, double &x0, double &x1) {
        const int32_t kf = field(x, W0{}), l0 = field(x, W1{}), l1 = field(x, W2{});
        const int32_t k = int32_t(uint32_t(kf) & kGrpIndexMask);
        // 32-bit byte offsets against the scalar bases of the factors (their extents stay below 2^25 on
        // this path): one vector instruction per address
        u2 = *reinterpret_cast<const double *>(U2b + (uint32_t(k * R2 + c2) << 3));
        x0 = *reinterpret_cast<const double *>(U3b + (uint32_t(l0 * R3 + c3) << 3));
        x1 = *reinterpret_cast<const double *>(U3b + (uint32_t(l1 * R3 + c3) << 3));
    };
    auto consume = [&](uint32_t x, double u2, double x0, double x1) {
        const int32_t kf = field(x, W0{});
        const uint32_t flags = uint32_t(__builtin_amdgcn_readfirstlane(kf));            // same on the four records
        if (flags & kGrpStartsKstep) {
            const int32_t j = field(x, W3{});                                           // -1: no such fiber
            if constexpr (FULL) {
                uq[0] = j >= 0 ? *reinterpret_cast<const double *>(U1b + (uint32_t(j * 16 + c) << 3)) : 0.0;
            } else {
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    uq[q] = *reinterpret_cast<const double *>(U1b + (uint32_t(max(j, 0) * R1 + min(4 * q + (c & 3), R1 - 1)) << 3));
                here = j >= 0;
            }
        }
        double t1;
        if (FULL) {
            t1 = fma(field64(x, W6{}, W7{}), x1, field64(x, W4{}, W5{}) * x0);         // what is absent carries value 0
        } else {
            // absent leaves name a row with value 0: left out, so that a row that is not finite reaches no other result
            t1 = field64(x, W4{}, W5{}) * x0;
            t1 = uint32_t(kf) & kRecOneLeaf ? t1 : fma(field64(x, W6{}, W7{}), x1, t1);
            t1 = uint32_t(kf) & kRecEmpty ? 0.0 : t1;
            u2 = uint32_t(kf) & kRecEmpty ? 0.0 : u2;
        }
        t2 = __builtin_amdgcn_mfma_f64_16x16x4f64(u2, t1, t2, 0, 0, 0);
        if (flags & kGrpEndsFiber) {
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (FULL || (slot + 4 * v < R2 && c < R3)) lds[ft * kStride + (slot + 4 * v) * R3 + c] = t2[v];
            t2 = v4d{0.0, 0.0, 0.0, 0.0};
            ++ft;
            if (flags & kGrpEndsKstep) {
                if constexpr (FULL) {        // slot s supplies fiber s; fibers the K-step lacks are multiplied by 0
                    const double a_op = slot < ft ? uq[0] : 0.0;
#pragma unroll
                    for (int t = 0; t < 16; ++t)
                        y[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a_op, lds[slot * kStride + t * 16 + c], y[t], 0, 0, 0);
                } else {
                    if (ft < 4) {            // fibers the K-step lacks: both operands are made 0
                        for (int e = ft * kStride + lane; e < 4 * kStride; e += 64) lds[e] = 0.0;
#pragma unroll
                        for (int q = 0; q < 4; ++q) uq[q] = here ? uq[q] : 0.0;
                    }
                    const double *tile = lds + slot * kStride + 2 * (4 * (c & 3) + (c >> 2));
#pragma unroll
                    for (int u = 0; u < MU; ++u) {
                        if (u < nu) {
                            const v2d b = *reinterpret_cast<const v2d *>(tile + 32 * u);
#pragma unroll
                            for (int q = 0; q < 4; ++q) {
                                if (q < nq) {
                                    acc[2 * u][q] = __builtin_amdgcn_mfma_f64_4x4x4f64(b.x, uq[q], acc[2 * u][q], 0, 0, 0);
                                    acc[2 * u + 1][q] = __builtin_amdgcn_mfma_f64_4x4x4f64(b.y, uq[q], acc[2 * u + 1][q], 0, 0, 0);
                                }
                            }
                        }
                    }
                }
                ft = 0;
            }
        }
    };
#pragma unroll
    for (int u = 0; u < kRec - 1; ++u) raw[u] = load_rec(ga + u);
#pragma unroll
    for (int u = 0; u < kRow - 1; ++u) load_rows(raw[u], gu2[u], gx0[u], gx1[u]);
    for (int64_t g0 = ga; g0 < gb; g0 += kRec) {
#pragma unroll
        for (int u = 0; u < kRec; ++u) {
            const int64_t g = g0 + u;
            raw[(u + kRec - 1) % kRec] = load_rec(g + kRec - 1);
            load_rows(raw[(u + kRow - 1) % kRec], gu2[(u + kRow - 1) % kRow], gx0[(u + kRow - 1) % kRow], gx1[(u + kRow - 1) % kRow]);
            if (g < gb) consume(raw[u], gu2[u % kRow], gx0[u % kRow], gx1[u % kRow]);
        }
    }
    const int64_t RR = int64_t(R1) * R23;
    double *base = dest < 0 ? a.out + (a.compact ? int64_t(s) : int64_t(a.idx0[s])) * RR
                            : a.partial + dest * RR;
    if constexpr (FULL) {
#pragma unroll
        for (int t = 0; t < 16; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) base[((slot + 4 * v) * 16 + t) * 16 + c] = y[t][v];
    } else {
#pragma unroll
        for (int u = 0; u < MU; ++u)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int flat = 32 * u + 2 * (4 * slot + (c >> 2)), r1 = 4 * q + (c & 3);
                if (r1 < R1) {
                    double *at = base + r1 * R23 + flat;
                    if (flat + 1 < R23) *reinterpret_cast<v2d_u *>(at) = v2d_u{acc[2 * u][q], acc[2 * u + 1][q]};
                    else if (flat < R23) *at = acc[2 * u][q];
                }
            }
    }
}

conststn_status launch_ttmc4(const conststn_plan_s *plan, const double *const *dense, double *out,
                             hipStream_t stream) {
    const conststn_csf_s *X = plan->X;
    Ttmc4Args a{};
    a.n_items = plan->n_items;
    a.R1 = plan->rank_of_level[1];
    a.R2 = plan->rank_of_level[2];
    a.R3 = plan->rank_of_level[3];
    a.ptr1 = X->ptr[1].p;
    a.ptr2 = X->ptr[2].p;
    a.idx0 = X->idx[0].p;
    a.idx1 = X->idx[1].p;
    a.idx2 = X->idx[2].p;
    a.idx3 = X->idx[3].p;
    a.vals = X->vals.p;
    a.items = plan->items.p;
    a.U1 = dense[plan->factor_of_level[1]];
    a.U2 = dense[plan->factor_of_level[2]];
    a.U3 = dense[plan->factor_of_level[3]];
    a.out = out;
    a.partial = plan->partial.p;
    a.compact = plan->compact ? 1 : 0;
    if (a.R1 > 16 || a.R2 > 16 || a.R3 > 16) {
        set_error("order-4 TTMc ranks above 16 are not implemented");
        return CONSTSTN_EUNSUPPORTED;
    }
    if (!plan->compact && X->nodes[0] < plan->out_rows)
        CST_TRY(zero_fill(out, plan->out_rows * plan->row_elems, stream));
    if (a.n_items == 0) return CONSTSTN_OK;
    {
        ProfScope prof(plan, stream);
        if (plan->use_rows) {
            Ttmc4RowArgs ra{};
            ra.n_items = plan->n_items;
            ra.R1 = a.R1;
            ra.R2 = a.R2;
            ra.R3 = a.R3;
            ra.kstep_group = plan->kstep_group.p;
            ra.rec = plan->pieces.p;
            ra.idx0 = a.idx0;
            ra.items = a.items;
            ra.U1 = a.U1;
            ra.U2 = a.U2;
            ra.U3 = a.U3;
            ra.out = out;
            ra.partial = a.partial;
            ra.compact = a.compact;
            const int parts = (a.R2 * a.R3 + 31) / 32;
            CST_TRY(in_item_ranges(ra, [&](const Ttmc4RowArgs &r) -> conststn_status {
                const dim3 grid{unsigned(r.n_items)}, block(64);
                if (r.R1 == 16 && r.R2 == 16 && r.R3 == 16) ttmc4_mfma_kernel<8, true><<<grid, block, 0, stream>>>(r);
                else if (parts > 4) ttmc4_mfma_kernel<8, false><<<grid, block, 0, stream>>>(r);
                else if (parts > 2) ttmc4_mfma_kernel<4, false><<<grid, block, 0, stream>>>(r);
                else ttmc4_mfma_kernel<2, false><<<grid, block, 0, stream>>>(r);
                return CONSTSTN_OK;
            }));
        } else
            CST_TRY(in_item_ranges(a, [&](const Ttmc4Args &r) -> conststn_status {
                ttmc4_kernel<<<dim3(unsigned(div_up(r.n_items, 4))), dim3(256), 0, stream>>>(r);
                return CONSTSTN_OK;
            }));
    }
    CST_HIP(hipGetLastError());
    return launch_ttmc_fixup(plan, out, stream);
}

}  // namespace cst
