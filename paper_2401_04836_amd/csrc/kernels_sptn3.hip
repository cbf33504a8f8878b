// Fused three-tensor network of Sec. 1:  Z[i,m] = sum_{j,k,l} U[i,j,k] V[j,l] W[k,l,m]
// evaluated as the tree (U.V).W:
//     T[i,k,l] = U[i,k,j] V[j,l]   loops i,k,j,l      (U stored i>k>j)
//     Z[i,m]   = T[i,k,l] W[k,l,m] loops i,k,l,m      (W stored k>l>m)
// fused on the loops i and k, so T shrinks to one length-L vector per (i,k) fiber of U and no
// full intermediate is formed.
//
// Baseline kernel: one workgroup per root slice i of U.  For each (i,k) fiber the threads
// build T[0..L) in LDS (thread = l, coalesced rows of V), then the wavefronts walk the (k,l)
// fibers of W below root k: lanes take the m leaves and add T[l]*W into a per-wavefront copy
// of Z_i in LDS (no atomics: leaves of one fiber have distinct m).  The copies are added in
// fixed order at the end, so results are bit-reproducible.
#include <algorithm>
#include <type_traits>
#include <utility>

#include "plan.hpp"

namespace cst {

struct Sptn3Args {
    int64_t slices;
    int64_t L, M;
    const int64_t *uptr0, *uptr1;
    const int32_t *uidx0, *uidx1, *uidx2;
    const double *uvals;
    const int64_t *wptr0, *wptr1;
    const int32_t *widx1, *widx2;
    const double *wvals;
    const int64_t *w_root_of_k;
    const double *V;
    double *out;
    int compact;
};

__global__ void __launch_bounds__(256)
sptn3_kernel(Sptn3Args a) {
    extern __shared__ double lds[];
    double *T = lds;                         // L
    double *Zw = lds + a.L;                  // 4 x M
    const int64_t s = blockIdx.x;
    const int tid = threadIdx.x, wave = tid / 64, lane = tid % 64;
    const int64_t L = a.L, M = a.M;
    for (int64_t e = tid; e < 4 * M; e += 256) Zw[e] = 0.0;
    const int64_t fa = a.uptr0[s], fb = a.uptr0[s + 1];
    for (int64_t f = fa; f < fb; ++f) {
        const int32_t k = a.uidx1[f];
        const int64_t root = a.w_root_of_k[k];
        if (root < 0) continue;                                   // W has nothing at this k
        const int64_t na = a.uptr1[f], nb = a.uptr1[f + 1];
        __syncthreads();                                          // T free for reuse
        for (int64_t l = tid; l < L; l += 256) {
            double t = 0.0;
            for (int64_t n = na; n < nb; ++n)
                t = fma(a.uvals[n], a.V[int64_t(a.uidx2[n]) * L + l], t);
            T[l] = t;
        }
        __syncthreads();
        const int64_t ga = a.wptr0[root], gb = a.wptr0[root + 1];
        double *Z = Zw + int64_t(wave) * M;
        for (int64_t g = ga + wave; g < gb; g += 4) {
            const double tl = T[a.widx1[g]];
            const int64_t ea = a.wptr1[g], eb = a.wptr1[g + 1];
            for (int64_t e = ea + lane; e < eb; e += 64) {
                const int32_t m = a.widx2[e];
                Z[m] = fma(tl, a.wvals[e], Z[m]);
            }
        }
    }
    __syncthreads();
    const int64_t row = a.compact ? s : int64_t(a.uidx0[s]);
    for (int64_t m = tid; m < M; m += 256)
        a.out[row * M + m] = ((Zw[m] + Zw[M + m]) + Zw[2 * M + m]) + Zw[3 * M + m];
}

// ---- tiled kernel: both stages on the fp64 matrix cores --------------------------------------
//
// Sixteen root slices of U are taken together (a "group"); a workgroup owns one group and one
// chunk of the k range and walks the k values present in any of its slices (a 16-way merge of
// the slices' level-1 lists).  For one k:
//   1. the j indices of the up to sixteen (i,k) fibers are merged through a bit mask in LDS into
//      their sorted union; the fibers are scattered into a dense LDS tile Uc[union rank][i]
//      (zero where a slice has no such j) -- at most kCap union rows per pass, more passes if
//      the union is longer (each pass is a unit of its own: the consumer is linear in T);
//   2. producer, per tile of 16 l values:  T^t[l, i] = sum_j V[j, l] Uc[j, i]  as 16x16x4 matrix
//      instructions, A = V[j_s, l0 + c] (row segments of 128 B from L2), B = Uc[j_s, c];
//   3. consumer: the accumulator registers of T^t are exactly the B operand layout, so
//      Z^t[m, i] += sum_l W[l, m] T^t[l, i]  follows without any data movement, A = the dense
//      16 x 16 tiles of W that the plan prepared (only tiles that hold a nonzero).
// A wavefront owns every fourth l tile and accumulates its own Z^t (all m tiles) in registers
// while it works on one k; after each k the four wavefronts add theirs, one after the other, to
// the group's Z^t in LDS, and the partial results of the k chunks are added by a fix-up kernel in
// chunk order, so results are bit-reproducible.  One wavefront per SIMD: latency is hidden by a
// software pipeline (kRing batches of four K-steps in flight) that runs across l tile boundaries;
// every load in it is unconditional (clamped addresses), and the W tiles of the current l tile
// are parked in a per-lane LDS area (indexable at run time, which registers are not).
// The zero entries of Uc and of the W tiles multiply real factor values, so V must be finite.

typedef double v4d __attribute__((ext_vector_type(4)));
typedef double v2d __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) v2d lds_v2d;

constexpr int kCap = 320;             // union rows of Uc per pass (40 KB)
constexpr int kStage = 6;             // W tiles parked in LDS per l tile and wavefront
constexpr int kBatch = 4;             // K-steps per pipeline batch
constexpr int kHeld = 16;             // leaves per lane kept in registers between mask and scatter
constexpr int kRing = 3;              // batches in flight (loads issued kRing - 1 batches ahead)

struct Sptn3TileArgs {
    int64_t slices, L, M, LT;
    int MT, nwords, n_groups, n_kc;        // n_kc: partial results of a row
    int l_parts;                           // of every chunk of the k range (two wavefronts per SIMD)
    int64_t k_per;
    const int64_t *uptr0, *uptr1;
    const int32_t *uidx0, *uidx1, *uidx2;
    const double *uvals;
    const int64_t *w_root_of_k;
    const uint32_t *wmask, *wfirst;
    const int32_t *wcell_ptr;              // cells of a root of W, see SpCell
    const SpCell *wcells;
    const double *wtiles;
    uint32_t zero_tile;
    const double *V;
    double *out, *partial;
    int compact, xcd_ranges;
    const int64_t *chunk_fiber;            // [(k chunks + 1) x slices] first fiber of a slice in a k chunk
    const int32_t *chunk_k;                // ... and the k there
    const int32_t *work;                   // pairs of the workgroups with two wavefronts per SIMD (-1: none), from the launch's first on
    const int32_t *wg_order;               // workgroup -> (k chunk, group) pair, heaviest pairs first (or null)
};

__device__ inline int64_t lower_bound_i32(const int32_t *__restrict__ a, int64_t lo, int64_t hi, int64_t key) {
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (int64_t(a[mid]) < key) lo = mid + 1; else hi = mid;
    }
    return lo;
}

struct SpPipe {
    double Vr[kRing][kBatch], Ur[kRing][kBatch];
    int32_t Jr[kRing][kBatch];
    v2d Wr[kRing][2];
};

__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1)))
sptn3_tiled_kernel(Sptn3TileArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    double *Uc = reinterpret_cast<double *>(smem);                        // kCap x 16
    double *Wb = Uc + kCap * 16;                                          // 4 x kStage x 256
    double *Zs = Wb + 4 * kStage * 256;                                   // MT x 16 x 16: Z^t[m][i]
    int32_t *jl = reinterpret_cast<int32_t *>(Zs + a.MT * 256);           // kCap: row offset j*L
    uint32_t *mask = reinterpret_cast<uint32_t *>(jl + kCap);             // nwords
    int32_t *wpre = reinterpret_cast<int32_t *>(mask + a.nwords);         // nwords
    int32_t *scan = wpre + a.nwords;                                      // 8

    const int tid = threadIdx.x, lane = tid & 63, slot = lane >> 4, c = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);          // uniform, and known to be
    // Workgroups are dealt to the 8 XCDs round-robin.  Optionally each XCD gets a contiguous range
    // of (k chunk, group) pairs instead, so that the workgroups sharing one L2 walk the same k
    // values over neighbouring groups (same W tiles, largely the same rows of V).
    const int n_wg = a.n_groups * a.n_kc, per_xcd = (n_wg + 7) / 8;
    if (int(blockIdx.x) >= n_wg && !a.xcd_ranges) return;
    const int logical = a.xcd_ranges ? (int(blockIdx.x) % 8) * per_xcd + int(blockIdx.x) / 8
                                     : (a.wg_order ? a.wg_order[blockIdx.x] : int(blockIdx.x));
    if (logical >= n_wg) return;
    const int group = logical % a.n_groups, kc = logical / a.n_groups;
    const int64_t s0 = int64_t(group) * kSpGroup;
    const int64_t k_lo = int64_t(kc) * a.k_per, k_hi = k_lo + a.k_per;
    const int64_t L = a.L;
    const int L32 = int(a.L);
    const char *Vbytes = reinterpret_cast<const char *>(a.V);
    const uint32_t lane16 = uint32_t(lane) * 16u;
    const int nwords = a.nwords;
    double *Wbw = Wb + wave * (kStage * 256);
    // the same area through an LDS-typed pointer, so that reads of it stay LDS instructions
    const lds_v2d *Wpark = (const lds_v2d *)(Wbw);

    // lane c (in each of the four lane rows) holds the cursor of slice s0 + c
    int64_t cur = 0, end = 0;
    if (s0 + c < a.slices) {
        const int64_t na = a.uptr0[s0 + c], nb = a.uptr0[s0 + c + 1];
        cur = lower_bound_i32(a.uidx1, na, nb, k_lo);
        end = lower_bound_i32(a.uidx1, cur, nb, k_hi);
    }
    for (int x = tid; x < a.MT * 256; x += 256) Zs[x] = 0.0;

    const int NTw = a.LT > wave ? int((a.LT - wave + 3) >> 2) : 0;       // l tiles of this wavefront

    for (;;) {
        const int32_t kk = cur < end ? a.uidx1[cur] : INT32_MAX;
        int32_t kmin = kk;
        kmin = min(kmin, __shfl_xor(kmin, 8, 16));
        kmin = min(kmin, __shfl_xor(kmin, 4, 16));
        kmin = min(kmin, __shfl_xor(kmin, 2, 16));
        kmin = min(kmin, __shfl_xor(kmin, 1, 16));
        kmin = __builtin_amdgcn_readfirstlane(kmin);
        if (kmin == INT32_MAX) break;
        const bool has = kk == kmin;
        const int64_t f = cur;
        cur += has ? 1 : 0;
        const int64_t root = a.w_root_of_k[kmin];                         // same address in every lane
        if (root < 0) continue;                                           // W has nothing at this k
        int64_t la = 0, lb = 0;
        if (has) { la = a.uptr1[f]; lb = a.uptr1[f + 1]; }
        // this lane row scatters the fiber of slice 4*wave + slot
        const int irow = 4 * wave + slot;
        const int64_t ea = __shfl(la, irow), eb = __shfl(lb, irow);

        __syncthreads();                                                  // LDS of the previous k is free
        for (int w = tid; w < nwords; w += 256) mask[w] = 0u;
        __syncthreads();
        // the first kHeld leaves per lane stay in registers for the scatter below: all their loads
        // are in flight together instead of one memory round trip per loop iteration
        int32_t jheld[kHeld];
        double vheld[kHeld];
#pragma unroll
        for (int h = 0; h < kHeld; ++h) {
            const int64_t e = ea + c + 16 * h;
            jheld[h] = e < eb ? a.uidx2[e] : -1;
            vheld[h] = e < eb ? a.uvals[e] : 0.0;
        }
#pragma unroll
        for (int h = 0; h < kHeld; ++h)
            if (jheld[h] >= 0) atomicOr(&mask[jheld[h] >> 5], 1u << (jheld[h] & 31));
        for (int64_t e = ea + c + 16 * kHeld; e < eb; e += 16) {
            const int32_t j = a.uidx2[e];
            atomicOr(&mask[j >> 5], 1u << (j & 31));
        }
        __syncthreads();
        {   // exclusive prefix of the set-bit counts of the mask words (thread t: words 4t .. 4t+3)
            int cnt[4], mine = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int w = 4 * tid + q;
                cnt[q] = w < nwords ? __popc(mask[w]) : 0;
                mine += cnt[q];
            }
            int incl = mine;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const int up = __shfl_up(incl, d);
                if (lane >= d) incl += up;
            }
            if (lane == 63) scan[wave] = incl;
            __syncthreads();
            int base = 0;
            for (int w = 0; w < wave; ++w) base += scan[w];
            int run = base + incl - mine;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int w = 4 * tid + q;
                if (w < nwords) wpre[w] = run;
                run += cnt[q];
            }
        }
        const int n_union = __builtin_amdgcn_readfirstlane(scan[0] + scan[1] + scan[2] + scan[3]);
        __syncthreads();

        // Prepare one pass: union rows [p0, p0 + np) -> Uc rows and j offsets.  The first pass takes
        // the leaves held in registers (they are dead before the matrix stages start); later passes
        // re-read the fibers.
        auto prepare = [&](int p0, int np, int npad, auto first) {
            for (int x = tid; x < npad * 16; x += 256) Uc[x] = 0.0;
            if (tid < npad - np) jl[np + tid] = 0;
            for (int w = tid; w < nwords; w += 256) {
                uint32_t m = mask[w];
                int r = wpre[w] - p0;
                while (m) {
                    const int b = __builtin_ctz(m);
                    m &= m - 1u;
                    if (r >= 0 && r < np) jl[r] = int32_t(int64_t(w * 32 + b) * L);
                    ++r;
                }
            }
            __syncthreads();
            auto place = [&](int32_t j, double v) {
                const int r = wpre[j >> 5] + __popc(mask[j >> 5] & ((1u << (j & 31)) - 1u)) - p0;
                if (r >= 0 && r < np) Uc[r * 16 + irow] = v;
            };
            if (decltype(first)::value) {
#pragma unroll
                for (int h = 0; h < kHeld; ++h)
                    if (jheld[h] >= 0) place(jheld[h], vheld[h]);
            }
            for (int64_t e = ea + c + (decltype(first)::value ? 16 * kHeld : 0); e < eb; e += 16)
                place(a.uidx2[e], a.uvals[e]);
            __syncthreads();
        };
        int p0 = 0;
        int np = min(kCap, n_union);
        int npad = (np + 4 * kBatch - 1) & ~(4 * kBatch - 1);                 // whole batches
        if (n_union > 0) prepare(0, np, npad, std::true_type{});
        while (p0 < n_union) {
            // ---- the two matrix stages over this wavefront's l tiles, 64 tiles per round ----
            v4d accZ[kSpMaxMTiles];
#pragma unroll
            for (int mt = 0; mt < kSpMaxMTiles; ++mt) accZ[mt] = v4d{0.0, 0.0, 0.0, 0.0};
            const int nBt = npad / (4 * kBatch);                          // batches per l tile
            for (int tr = 0; tr < NTw; tr += 64) {
                const int NT = min(64, NTw - tr);
                // lane t holds mask and first tile of its t-th l tile of this round
                uint32_t mreg = 0u, freg = a.zero_tile;
                if (lane < NT) {
                    const int64_t cell = root * a.LT + (wave + 4 * (tr + lane));
                    mreg = a.wmask[cell];
                    freg = mreg ? a.wfirst[cell] : a.zero_tile;
                }
                const int TB = NT * nBt;
                SpPipe P;
                v4d accT0 = v4d{0.0, 0.0, 0.0, 0.0}, accT1 = accT0;
                // stream positions: (t, q) = (l tile of the round, batch inside it)
                int t0 = 0, q0 = 0;                                       // batch being consumed
                int t2 = 0, q2 = 0;                                       // batch whose V/U/W loads are issued
                int q3 = 0;                                               // batch whose j offsets are read

                auto read_j = [&](int32_t (&J)[kBatch]) {
#pragma unroll
                    for (int ks = 0; ks < kBatch; ++ks) J[ks] = jl[q3 * (4 * kBatch) + ks * 4 + slot];
                    q3 = q3 + 1 == nBt ? 0 : q3 + 1;
                };
                auto issue = [&](const int32_t (&J)[kBatch], double (&Vv)[kBatch], double (&Uu)[kBatch], v2d (&Ww)[2]) {
                    const int tt = min(t2, NT - 1);
                    const int col = min(16 * (wave + 4 * (tr + tt)) + c, L32 - 1);
                    // 32-bit element offsets against the scalar base of V (J L < 2^29, checked by the plan):
                    // one vector instruction per address
#pragma unroll
                    for (int ks = 0; ks < kBatch; ++ks) {
                        Vv[ks] = *reinterpret_cast<const double *>(Vbytes + (uint32_t(J[ks] + col) << 3));
                        Uu[ks] = Uc[q2 * (64 * kBatch) + ks * 64 + lane];
                    }
                    const uint32_t m2 = __builtin_amdgcn_readlane(mreg, tt);
                    const uint32_t f2 = __builtin_amdgcn_readlane(freg, tt);
                    const int last = max(__popc(m2) - 1, 0);
                    const int tq = min(min(q2, kStage - 1), last);            // all scalar
                    const char *tb = reinterpret_cast<const char *>(a.wtiles + (int64_t(f2) + tq) * 256);
                    Ww[0] = *reinterpret_cast<const v2d *>(tb + lane16);
                    Ww[1] = *reinterpret_cast<const v2d *>(tb + lane16 + 1024);
                    if (q2 + 1 == nBt) { q2 = 0; ++t2; } else ++q2;
                };
                auto consume = [&](int b, const double (&Vv)[kBatch], const double (&Uu)[kBatch], const v2d (&Ww)[2]) {
                    // park the W tile that came with this batch
                    double *wp = Wbw + min(q0, kStage - 1) * 256 + lane * 2;
                    *reinterpret_cast<v2d *>(wp) = Ww[0];
                    *reinterpret_cast<v2d *>(wp + 128) = Ww[1];
                    if (b < TB) {
                        accT0 = __builtin_amdgcn_mfma_f64_16x16x4f64(Vv[0], Uu[0], accT0, 0, 0, 0);
                        accT1 = __builtin_amdgcn_mfma_f64_16x16x4f64(Vv[1], Uu[1], accT1, 0, 0, 0);
                        accT0 = __builtin_amdgcn_mfma_f64_16x16x4f64(Vv[2], Uu[2], accT0, 0, 0, 0);
                        accT1 = __builtin_amdgcn_mfma_f64_16x16x4f64(Vv[3], Uu[3], accT1, 0, 0, 0);
                        if (q0 + 1 == nBt) {
                            // consumer: Z^t += W^t . T^t for the m tiles present below this l tile
                            const v4d T = accT0 + accT1;
                            const uint32_t m0 = __builtin_amdgcn_readlane(mreg, t0);
                            const uint32_t f0 = __builtin_amdgcn_readlane(freg, t0);
                            const int have = __popc(m0);
                            int staged = min(nBt, kStage);                // tiles parked so far
                            int first_p = 0;                              // tile held by slot 0
                            for (;;) {
                                int p = 0;
#pragma unroll
                                for (int mt = 0; mt < kSpMaxMTiles; ++mt) {
                                    if ((m0 >> mt) & 1u) {
                                        if (p >= first_p && p < first_p + staged) {
                                            const lds_v2d *rp = Wpark + ((p - first_p) * 128 + lane);
                                            const v2d w0 = rp[0], w1 = rp[64];
                                            v4d z = accZ[mt];
                                            z = __builtin_amdgcn_mfma_f64_16x16x4f64(w0.x, T.x, z, 0, 0, 0);
                                            z = __builtin_amdgcn_mfma_f64_16x16x4f64(w0.y, T.y, z, 0, 0, 0);
                                            z = __builtin_amdgcn_mfma_f64_16x16x4f64(w1.x, T.z, z, 0, 0, 0);
                                            z = __builtin_amdgcn_mfma_f64_16x16x4f64(w1.y, T.w, z, 0, 0, 0);
                                            accZ[mt] = z;
                                        }
                                        ++p;
                                    }
                                }
                                first_p += staged;
                                if (first_p >= have) break;               // the usual case: one round
                                // more tiles below this l tile than were parked (rare): fetch the
                                // next ones and park them, then go round again
                                staged = min(kStage, have - first_p);
                                for (int sl = 0; sl < staged; ++sl) {
                                    const double *tp = a.wtiles + (int64_t(f0) + first_p + sl) * 256 + lane * 2;
                                    const v2d w0 = *reinterpret_cast<const v2d *>(tp);
                                    const v2d w1 = *reinterpret_cast<const v2d *>(tp + 128);
                                    double *wp = Wbw + sl * 256 + lane * 2;
                                    *reinterpret_cast<v2d *>(wp) = w0;
                                    *reinterpret_cast<v2d *>(wp + 128) = w1;
                                }
                            }
                            accT0 = v4d{0.0, 0.0, 0.0, 0.0};
                            accT1 = accT0;
                            q0 = 0;
                            ++t0;
                        } else {
                            ++q0;
                        }
                    }
                };

                if (TB > 0) {
#pragma unroll
                    for (int u = 0; u < kRing; ++u) read_j(P.Jr[u]);
#pragma unroll
                    for (int u = 0; u < kRing - 1; ++u) issue(P.Jr[u], P.Vr[u], P.Ur[u], P.Wr[u]);
                    for (int b = 0; b < TB; b += kRing) {
#pragma unroll
                        for (int u = 0; u < kRing; ++u) {
                            const int su = (u + kRing - 1) % kRing;
                            issue(P.Jr[su], P.Vr[su], P.Ur[su], P.Wr[su]);
                            read_j(P.Jr[u]);
                            consume(b + u, P.Vr[u], P.Ur[u], P.Wr[u]);
                        }
                    }
                }
            }
            // add this k's contribution to the group's Z^t, wavefront after wavefront
            for (int w = 0; w < 4; ++w) {
                if (wave == w) {
#pragma unroll
                    for (int mt = 0; mt < kSpMaxMTiles; ++mt) {
                        if (mt < a.MT) {
#pragma unroll
                            for (int v = 0; v < 4; ++v) Zs[(16 * mt + slot + 4 * v) * 16 + c] += accZ[mt][v];
                        }
                    }
                }
                __syncthreads();
            }
            p0 += kCap;
            if (p0 < n_union) {
                np = min(kCap, n_union - p0);
                npad = (np + 4 * kBatch - 1) & ~(4 * kBatch - 1);
                prepare(p0, np, npad, std::false_type{});
            }
        }
    }

    // ---- store the group's rows ----------------------------------------------------------------
    __syncthreads();
    const int64_t M = a.M;
    for (int64_t x = tid; x < 16 * M; x += 256) {
        const int64_t i = x / M, m = x - i * M;
        const int64_t s = s0 + i;
        if (s >= a.slices) break;
        const double z = Zs[m * 16 + i];
        if (a.n_kc == 1) {
            const int64_t row = a.compact ? s : int64_t(a.uidx0[s]);
            a.out[row * M + m] = z;
        } else {
            a.partial[(int64_t(kc) * a.slices + s) * M + m] = z;
        }
    }
}

// ---- tiled kernel with two wavefronts per SIMD ------------------------------------------------
// The kernel above reads one operand from memory and one from LDS for every matrix instruction, and its 200
// accumulator registers leave room for one wavefront per SIMD.  Here a workgroup of eight wavefronts takes 32 slices
// (two *halves* of sixteen; H = 1: one) and only the blocks of sixteen l below which W holds anything under the k at hand (a
// list made with the plan; T is read nowhere else).  Sixteen blocks make a *round*:
//   producer: wavefront w computes T^t of the blocks w and w + 8 for both halves, so that four operands (two
//     8-byte pieces of V's rows, one 16-byte read of Uc) feed four matrix instructions.  The union rows stand in the
//     order (first half only, both, second half only): a batch of eight rows that a half does not hold costs that
//     half nothing, so 32 slices never take more matrix instructions than twice 16 would.
//   consumer: split by m.  Wavefront w owns half w % 2 and the m tiles x = (w / 2) mod 4, + 4, + 8, ... (seven
//     accumulator tiles, kept in registers across all k of the workgroup); with one half the tiles w mod 8, + 8, ... (four).
//     The two wavefronts of a SIMD own tiles of one parity: a block of W spans two or three neighbouring tiles, which so
//     spread over the SIMDs.  The T^t of a round go through LDS; W's tiles come straight from memory, eight ahead, the first
//     four of them before the producer starts.  A wavefront finds its tiles of a round by a prefix sum over the blocks' masks.
// Two barriers a round, around the writes of T^t: a wavefront with few tiles goes on to the next round's producer.
// V's loads run three batches ahead across rounds; a round is padded to whole groups of four batches, whose empty
// batches load and do nothing.
// 2000 x 2000 x 400 in blocks of 100 x 100 x 20 (356 M matrix instructions, 9.7 ms at the 28 ns one takes): 23.4 -> 15.4 ms.
// The form before took 16 slices at a time: one 8-byte piece of V and one of Uc for every instruction, 363 M of them.
// Of a workgroup's time (taken at 15.8 ms, before the kernel did without lists of pairs) the producer has 40 %, the consumer
// 26 %, waiting at the two barriers 18 %, finding W's tiles 4 %, everything between two k 12 % (16 us of latencies).  With all
// of W's tiles read from one place (a switched-off copy) it takes 14.6 ms: their way from past the L2 costs 0.8; V's rows
// read from one cache line change nothing.
// H = 1 is for networks that leave compute units with a pair or less: half the matrix instructions of a pair follow one
// another, and two lane rows fetch a slice's leaves.  Where the line lies stands with the plan's choice (choose_cut).
constexpr int kOwnWaves = 8;
constexpr int64_t kOwnLaunch = int64_t(1) << 22;                        // workgroups of a launch
constexpr int kOwnCap = kSpUnionRows;                                   // union rows of Uc per pass (78 KB)
constexpr int kOwnHeld = 24;                                            // leaves per lane and half kept between mask and scatter
constexpr int kOwnRows = 8;                                             // union rows of a batch (two K-steps)
constexpr int kOwnRing = 4;                                             // batches of a group = stages of V's ring
constexpr int kOwnBlocks = 2 * kOwnWaves;                               // blocks of l in a round
constexpr int kOwnChunk = 8;                                            // rounds whose blocks a wavefront holds (128 blocks)
// with H halves: m tile mod 8 / H -> H wavefronts, and accumulator tiles per wavefront
constexpr int own_classes(int h) { return kOwnWaves / h; }
constexpr int own_z(int h) { return (kSpMaxMTiles + own_classes(h) - 1) / own_classes(h); }
constexpr int kOwnNoZ = 7;                                              // the accumulator of a place behind a list: none
constexpr int kOwnList = 128;                                           // places for a wavefront's W tiles of a round
constexpr int kOwnOffsets = (kOwnCap + kOwnRows * kOwnRing - 1) / (kOwnRows * kOwnRing) * (kOwnRows * kOwnRing);
constexpr int kOwnWRing = 8;                                            // W tiles in flight in the consumer ...
constexpr int kOwnWAhead = 4;                                           // ... and beside the producer
static_assert(kOwnBlocks * own_z(2) + 2 * kOwnWRing <= kOwnList && kOwnList == 2 * 64, "a wavefront's list of W tiles lies in two registers");
static_assert(kSpGroupWide == 32 && own_z(2) == 7 && own_z(1) == 4, "slices of a workgroup; accumulators that the consumer tests for");

// LDS: Uc, T^t, ranks of the mask words, offsets of V's rows (read 16 bytes at a time), masks, lists, scan
__host__ __device__ constexpr size_t sptn3_owned_offsets_at(int nwords, int h) {
    return size_t(kOwnCap * 16 + kOwnBlocks * 256) * size_t(h) * 8 + size_t((nwords + 1) & ~1) * 8;
}
__host__ __device__ constexpr size_t sptn3_owned_lds(int nwords, int h) {
    return sptn3_owned_offsets_at(nwords, h) + size_t(kOwnOffsets) * 4 + size_t((nwords + 1) & ~1) * 4 * size_t(h) +
           size_t(kOwnWaves * kOwnList) * 2 + 256;
}
static_assert(sptn3_owned_offsets_at(1, 1) % 16 == 0 && sptn3_owned_offsets_at(2, 1) % 16 == 0 && sptn3_owned_offsets_at(1, 2) % 16 == 0 &&
              sptn3_owned_offsets_at(2, 2) % 16 == 0 && sptn3_owned_lds(1, 1) % 8 == 0 && sptn3_owned_lds(1, 2) % 8 == 0,
              "16-byte reads of the offsets, 8-byte ones of the scan");
static_assert(sptn3_owned_lds(29696 / 32, 2) <= 160 * 1024, "J up to 29 696");

// orders LDS between the wavefronts of a workgroup without waiting for loads from memory in flight
__device__ __forceinline__ void sp_lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

template <int... I, typename F>
__device__ __forceinline__ void sp_each(std::integer_sequence<int, I...>, F &&f) {
    (f(std::integral_constant<int, I>{}), ...);
}

__device__ inline uint64_t shfl_up_u64(uint64_t x, int d) {
    const uint32_t lo = __shfl_up(uint32_t(x), d), hi = __shfl_up(uint32_t(x >> 32), d);
    return uint64_t(hi) << 32 | lo;
}

template <int H>
__global__ void __launch_bounds__(64 * kOwnWaves) __attribute__((amdgpu_waves_per_eu(2, 2)))
sptn3_owned_kernel(Sptn3TileArgs a) {
    constexpr int kClasses = own_classes(H), kZ = own_z(H), kSlices = 16 * H;
    constexpr int kLeafLanes = 64 * kOwnWaves / kSlices;                  // lanes of a slice between two k: one lane row, or two
    using Col = typename std::conditional<H == 2, v2d, double>::type;     // what one row of Uc holds under a column
    using lds_col = __attribute__((address_space(3))) Col;
    extern __shared__ __align__(16) unsigned char smem[];
    double *Uc = reinterpret_cast<double *>(smem);                        // kOwnCap x 16 columns x H halves
    double *Tx = Uc + kOwnCap * 16 * H;                                   // kOwnBlocks x H halves x 256
    uint64_t *wpre = reinterpret_cast<uint64_t *>(Tx + kOwnBlocks * H * 256);  // nwords: ranks, 21 bits a category
    uint32_t *jl = reinterpret_cast<uint32_t *>(smem + sptn3_owned_offsets_at(a.nwords, H));  // kOwnOffsets: byte offsets of V's rows
    uint32_t *mask = jl + kOwnOffsets;                                    // H x nwords
    uint16_t *lists = reinterpret_cast<uint16_t *>(mask + H * ((a.nwords + 1) & ~1));  // kOwnWaves x kOwnList
    uint64_t *scan = reinterpret_cast<uint64_t *>(smem + sptn3_owned_lds(a.nwords, H) - 64);  // kOwnWaves

    const int tid = threadIdx.x, lane = tid & 63, slot = lane >> 4, c = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t L = a.L;
    const int L32 = int(a.L);
    const char *Vbytes = reinterpret_cast<const char *>(a.V);
    const uint32_t lane16 = uint32_t(lane) * 16u;
    const int nwords = a.nwords;
    const lds_col *UcV = (const lds_col *)(Uc);
    const lds_v2d *TxV = (const lds_v2d *)(Tx);
    const int my_half = wave & (H - 1), my_class = wave / H;
    uint32_t own = 0u;                                                    // m tiles of this wavefront
#pragma unroll
    for (int x = 0; x < kZ; ++x) own |= my_class + kClasses * x < 32 ? 1u << (my_class + kClasses * x) : 0u;
    uint16_t *list = lists + wave * kOwnList;

    // A workgroup per (k chunk, part of l, group) triple
    const int logical = __builtin_amdgcn_readfirstlane(a.work[blockIdx.x]);
    if (logical < 0) return;
    const int group = logical % a.n_groups, kc = logical / a.n_groups, chunk = kc / a.l_parts, part = kc % a.l_parts;
    const int64_t s0 = int64_t(group) * kSlices;
    // lane sl (and sl + 32) holds the cursor of slice s0 + sl, its place in the k chunk, and the k there
    int64_t cur = 0, end = 0;
    int32_t kk = INT32_MAX;
    if ((lane & 31) < kSlices && s0 + (lane & 31) < a.slices) {
        const int64_t at = int64_t(chunk) * a.slices + s0 + (lane & 31);
        cur = a.chunk_fiber[at];
        end = a.chunk_fiber[at + a.slices];
        kk = a.chunk_k[at];
    }
    v4d accZ[kZ] = {};                                                    // (indexed by constants only, see the end)

    // Walk over the k that any of the slices holds.  What a k needs from the tables is fetched while the one before it
    // is prepared: its fibers' leaves, its root in W, and (kk) the k that follows in every slice.
    int64_t la = 0, lb = 0, root = -1;
    auto next_k = [&]() -> int {
        int32_t kmin = kk;
#pragma unroll
        for (int d = 16; d; d >>= 1) kmin = min(kmin, __shfl_xor(kmin, d, 32));
        kmin = __builtin_amdgcn_readfirstlane(kmin);
        la = lb = 0;
        if (kmin != INT32_MAX) {
            root = a.w_root_of_k[kmin];                                   // same address in every lane
            if (kk == kmin) {
                la = a.uptr1[cur];
                lb = a.uptr1[cur + 1];
                ++cur;
                kk = cur < end ? a.uidx1[cur] : INT32_MAX;
            }
        }
        return kmin;
    };
    for (int kmin = next_k(); kmin != INT32_MAX;) {
        const bool known = root >= 0;                                     // W has something at this k
        // the blocks of l below which it has, this pair's share of them
        const int64_t cell_row = known ? root : 0;
        const int cell_all = __builtin_amdgcn_readfirstlane(a.wcell_ptr[cell_row]);
        const int n_all = __builtin_amdgcn_readfirstlane(a.wcell_ptr[cell_row + 1]) - cell_all;
        const int cell0 = cell_all + n_all * part / a.l_parts;
        const int cells = cell_all + n_all * (part + 1) / a.l_parts - cell0;
        // one lane row per slice: slice 4*wave + slot, of half wave / 4; with one half two, 16 leaves in turn
        const int irow = (4 * wave + slot) & (kSlices - 1);
        const int64_t ea = __shfl(la, irow), eb = known ? __shfl(lb, irow) : ea;
        const int64_t e0 = ea + c + (H == 1 ? 16 * (wave >> 2) : 0);
        uint32_t *my_mask = mask + (H == 2 ? wave >> 2 : 0) * nwords;
        double *my_col = Uc + (irow & 15) * H + (H == 2 ? wave >> 2 : 0);
        // the first leaves of a lane stay in registers for the scatter below
        constexpr int kHeld = kOwnHeld * H / 2;
        int32_t jheld[kHeld];
        double vheld[kHeld];
#pragma unroll
        for (int h = 0; h < kHeld; ++h) {
            const int64_t e = e0 + kLeafLanes * h;
            jheld[h] = e < eb ? a.uidx2[e] : -1;
            vheld[h] = e < eb ? a.uvals[e] : 0.0;
        }
        sp_lds_barrier();                                                 // LDS of the previous k is free
        for (int w = tid; w < H * nwords; w += 64 * kOwnWaves) mask[w] = 0u;
        for (int x = tid; x < min(kOwnCap, 32 * nwords) * 8 * H; x += 64 * kOwnWaves) reinterpret_cast<v2d *>(Uc)[x] = v2d{0.0, 0.0};
        for (int x = tid; x < kOwnOffsets; x += 64 * kOwnWaves) jl[x] = 0u;
        sp_lds_barrier();
        // (neighbouring leaves tend to share a word, on which the lanes' atomics would queue: the bits of the lanes of a
        // row with the word of its first lane are joined first)
#pragma unroll
        for (int h = 0; h < kHeld; ++h) {
            const int word = jheld[h] >> 5;                               // (-1: no leaf)
            const uint32_t bit = jheld[h] >= 0 ? 1u << (jheld[h] & 31) : 0u;
            const int word0 = row_first(word);
            const uint32_t joined = row_or(word == word0 ? bit : 0u);
            if (bit && (c == 0 || word != word0)) atomicOr(&my_mask[word], c == 0 ? joined : bit);
        }
        for (int64_t e = e0 + kLeafLanes * kHeld; e < eb; e += kLeafLanes) {
            const int32_t j = a.uidx2[e];
            atomicOr(&my_mask[j >> 5], 1u << (j & 31));
        }
        kmin = next_k();
        sp_lds_barrier();
        // Ranks of the union rows: exclusive prefix of the set bits of every category (first half only, both, second
        // only; thread t: words 2t, 2t+1), the categories one behind the other.  At most 32768 a category.
        uint64_t cnt[2], mine = 0;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int w = 2 * tid + q;
            cnt[q] = 0;
            if (w < nwords) {
                const uint32_t m0 = mask[w], m1 = H == 2 ? mask[nwords + w] : 0u;
                cnt[q] = uint64_t(__popc(m0 & ~m1)) | uint64_t(__popc(m0 & m1)) << 21 | uint64_t(__popc(m1 & ~m0)) << 42;
            }
            mine += cnt[q];
        }
        uint64_t incl = mine;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const uint64_t up = shfl_up_u64(incl, d);
            if (lane >= d) incl += up;
        }
        if (lane == 63) scan[wave] = incl;
        sp_lds_barrier();
        uint64_t base = 0, total = 0;
#pragma unroll
        for (int w = 0; w < kOwnWaves; ++w) {
            const uint64_t s = scan[w];
            base += w < wave ? s : 0;
            total += s;
        }
        const int n_one = __builtin_amdgcn_readfirstlane(int(total & 0x1fffff));
        const int n_both = __builtin_amdgcn_readfirstlane(int(total >> 21 & 0x1fffff));
        const int end0 = n_one + n_both;                                  // rows [0, end0) hold the first half,
        const int n_union = end0 + __builtin_amdgcn_readfirstlane(int(total >> 42));   // [n_one, n_union) the second
        uint64_t run = base + incl - mine + (uint64_t(n_one) << 21 | uint64_t(end0) << 42);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int w = 2 * tid + q;
            if (w < nwords) wpre[w] = run;
            run += cnt[q];
        }

        // Prepare one pass: union rows [p0, p0 + np) -> Uc rows and V offsets (row r of batch r / 8, K-step
        // (r / 4) % 2, lane row r % 4).  The first pass takes the leaves held in registers and finds both cleared.
        auto prepare = [&](int p0, int np, auto first) {
            if (!decltype(first)::value) {
                for (int x = tid; x < kOwnCap * 8 * H; x += 64 * kOwnWaves) reinterpret_cast<v2d *>(Uc)[x] = v2d{0.0, 0.0};
                for (int x = tid; x < kOwnOffsets; x += 64 * kOwnWaves) jl[x] = 0u;
                sp_lds_barrier();
            }
            // the place of j in the pass, for one that is in the union
            auto place_of = [&](uint32_t bit, uint32_t m0, uint32_t m1, uint64_t pre) {
                const uint32_t in0 = m0 & bit ? ~0u : 0u, in1 = m1 & bit ? ~0u : 0u;
                const uint32_t same = ~(m0 ^ in0) & ~(m1 ^ in1);           // the rows of j's category
                return int(pre >> (in1 ? in0 ? 21 : 42 : 0) & 0x1fffff) + __popc(same & (bit - 1u)) - p0;
            };
            for (int x = tid; x < 8 * nwords; x += 64 * kOwnWaves) {      // four bits of a mask word each
                const int w = x >> 3;
                const uint32_t m0 = mask[w], m1 = H == 2 ? mask[nwords + w] : 0u;
                const uint64_t pre = wpre[w];
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    const int j = 4 * x + b;
                    const uint32_t bit = 1u << (j & 31);
                    const int r = place_of(bit, m0, m1, pre);
                    if (((m0 | m1) & bit) && r >= 0 && r < np)
                        jl[(r & ~31) + (r & 3) * 8 + ((r >> 2) & 7)] = uint32_t(j) * uint32_t(L) << 3;
                }
            }
            auto place = [&](int32_t j, double v) {
                const int r = place_of(1u << (j & 31), mask[j >> 5], H == 2 ? mask[nwords + (j >> 5)] : 0u, wpre[j >> 5]);
                if (r >= 0 && r < np) my_col[r * kSlices] = v;
            };
            if (decltype(first)::value) {
#pragma unroll
                for (int h = 0; h < kHeld; ++h)
                    if (jheld[h] >= 0) place(jheld[h], vheld[h]);
            }
            for (int64_t e = e0 + (decltype(first)::value ? kLeafLanes * kHeld : 0); e < eb; e += kLeafLanes)
                place(a.uidx2[e], a.uvals[e]);
            sp_lds_barrier();
        };
        sp_lds_barrier();
        int p0 = 0;
        if (n_union > 0) prepare(0, min(kOwnCap, n_union), std::true_type{});
        while (p0 < n_union) {
            const int np = min(kOwnCap, n_union - p0);
            const int n_groups = (np + kOwnRows * kOwnRing - 1) / (kOwnRows * kOwnRing);
            const int row_end0 = min(end0 - p0, np), row_one = n_one - p0;
            for (int c0 = 0; c0 < cells; c0 += kOwnChunk * kOwnBlocks) {
                const int here = min(kOwnChunk * kOwnBlocks, cells - c0);
                const int rounds = (here + kOwnBlocks - 1) / kOwnBlocks;
                // lane x holds the blocks x and x + 64 of the chunk (absent ones: no tile, any l)
                uint32_t mreg[2], freg[2];
                int lreg[2];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const SpCell cell = a.wcells[cell0 + c0 + min(64 * h + lane, here - 1)];
                    mreg[h] = 64 * h + lane < here ? cell.mask : 0u;
                    freg[h] = cell.first;
                    lreg[h] = cell.l_tile;
                }
                // byte offset of this lane's column of V in the wavefront's blocks of a round
                auto columns = [&](int r, uint32_t (&col)[2]) {
#pragma unroll
                    for (int d = 0; d < 2; ++d) {
                        const int x = (r & 3) * kOwnBlocks + d * kOwnWaves + wave;
                        const int lt = r < 4 ? __builtin_amdgcn_readlane(lreg[0], x) : __builtin_amdgcn_readlane(lreg[1], x);
                        col[d] = uint32_t(min(16 * lt + c, L32 - 1)) << 3;
                    }
                };
                double V[kOwnRing][2][2];                                 // [batch of the group][K-step][block]
                Col U[2][2];                                              // [parity of the batch][K-step] halves
                auto half = [](const Col &u, int h) -> double {
                    if constexpr (H == 2) return u[h];
                    else return u;
                };
                uint4 J[2];                                               // V offsets of the group's eight K-steps
                auto offset = [&](int i) -> uint32_t {
                    const uint4 &q = J[i >> 2];
                    return (i & 3) == 0 ? q.x : (i & 3) == 1 ? q.y : (i & 3) == 2 ? q.z : q.w;
                };
                auto read_j = [&](int g) {
                    const uint4 *p = reinterpret_cast<const uint4 *>(jl + g * 32 + slot * 8);
                    J[0] = p[0];
                    J[1] = p[1];
                };
                auto issue = [&](double (&v)[2][2], int u, const uint32_t (&col)[2]) {
#pragma unroll
                    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                        for (int d = 0; d < 2; ++d)
                            v[ks][d] = *reinterpret_cast<const double *>(Vbytes + (offset(2 * u + ks) + col[d]));
                };
                auto read_u = [&](Col (&u)[2], int b) {                   // (batches behind the last row read T^t: unused)
                    u[0] = UcV[b * 128 + lane];
                    u[1] = UcV[b * 128 + 64 + lane];
                };
                uint32_t col[2], col_next[2];
                columns(0, col);
                read_j(0);
#pragma unroll
                for (int u = 0; u < kOwnRing - 1; ++u) issue(V[u], u, col);
                read_u(U[0], 0);

                for (int r = 0; r < rounds; ++r) {
                    columns(min(r + 1, rounds - 1), col_next);
                    // ---- this wavefront's W tiles of the round: a list (tile - first, block, accumulator) ----
                    const int src = (r & 3) * kOwnBlocks + c;
                    const uint32_t bm = __shfl(r < 4 ? mreg[0] : mreg[1], src);
                    const uint32_t bf = __shfl(r < 4 ? freg[0] : freg[1], src);
                    const uint32_t first = __builtin_amdgcn_readfirstlane(bf);
                    uint32_t todo = lane < kOwnBlocks ? bm & own : 0u;
                    int upto = __popc(todo);
#pragma unroll
                    for (int d = 1; d < 16; d <<= 1) {
                        const int up = __shfl_up(upto, d, 16);
                        if (c >= d) upto += up;
                    }
                    // (nothing to do where the half holds no slice with this k)
                    const bool idle = H == 2 && (my_half ? n_union == n_one : end0 == 0);
                    const int n_tiles = idle ? 0 : __builtin_amdgcn_readlane(upto, kOwnBlocks - 1);
                    int at = upto - __popc(todo);
                    while (todo) {
                        const int b = __builtin_ctz(todo);
                        todo &= todo - 1u;
                        list[at++] = uint16_t((bf - first + __popc(bm & ((1u << b) - 1u))) | uint32_t(c) << 9 |
                                              uint32_t(b / kClasses) << 13);
                    }
                    // (behind the list's end: the round's first tile, added to nothing)
                    if (lane < 2 * kOwnWRing) list[n_tiles + lane] = uint16_t(kOwnNoZ << 13);
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                    const uint32_t code0 = list[lane], code1 = list[64 + lane];
                    const char *round_tiles = reinterpret_cast<const char *>(a.wtiles + int64_t(first) * 256);
                    v2d W[kOwnWRing][2];
                    uint32_t code[kOwnWRing];
                    auto fetch = [&](int u, uint32_t codes, int e) {      // codes: the half of the list that holds e
                        code[u] = __builtin_amdgcn_readlane(codes, e & 63);
                        const uint32_t at = lane16 + ((code[u] & 511u) << 11);
                        W[u][0] = *reinterpret_cast<const v2d *>(round_tiles + at);
                        W[u][1] = *reinterpret_cast<const v2d *>(round_tiles + at + 1024);
                    };
#pragma unroll
                    for (int u = 0; u < kOwnWAhead; ++u) fetch(u, code0, u);

                    // ---- producer ----
                    v4d T[2][H];                                          // [block][half]
#pragma unroll
                    for (int d = 0; d < 2; ++d)
#pragma unroll
                        for (int h = 0; h < H; ++h) T[d][h] = v4d{0.0, 0.0, 0.0, 0.0};
                    // (simple tests without alternatives: an if / else around matrix instructions makes the compiler copy
                    // the accumulators where the paths meet)
                    const bool two = here - r * kOwnBlocks > kOwnWaves + wave, some = here - r * kOwnBlocks > wave;
                    const int stop0[2] = {some ? row_end0 : 0, two ? row_end0 : 0};
                    const int stop1[2] = {some ? np : 0, two ? np : 0};
                    auto group = [&](int g) {
                        const bool last = g + 1 == n_groups;
                        const uint32_t coln[2] = {last ? col_next[0] : col[0], last ? col_next[1] : col[1]};
#pragma unroll
                        for (int u = 0; u < kOwnRing; ++u) {
                            if (u == 0) {
                                issue(V[kOwnRing - 1], kOwnRing - 1, col);
                                read_j(last ? 0 : g + 1);
                            } else {
                                issue(V[u - 1], u - 1, coln);
                            }
                            const int b = g * kOwnRing + u, row = b * kOwnRows;
                            read_u(U[(u + 1) & 1], u + 1 == kOwnRing && last ? 0 : b + 1);
                            const int row1 = row + kOwnRows > row_one ? row : INT32_MAX;
#pragma unroll
                            for (int d = 0; d < 2; ++d) {
                                if (row < stop0[d]) {
                                    T[d][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(V[u][0][d], half(U[u & 1][0], 0), T[d][0], 0, 0, 0);
                                    T[d][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(V[u][1][d], half(U[u & 1][1], 0), T[d][0], 0, 0, 0);
                                }
                                if constexpr (H == 2) {
                                    if (row1 < stop1[d]) {
                                        T[d][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(V[u][0][d], half(U[u & 1][0], 1), T[d][1], 0, 0, 0);
                                        T[d][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(V[u][1][d], half(U[u & 1][1], 1), T[d][1], 0, 0, 0);
                                    }
                                }
                            }
                        }
                    };
                    // the groups whose rows both halves hold, then those with tests
                    int g = 0;
                    if (H == 1 || n_one <= p0) {
                        const int whole = min(min(row_end0, np) / (kOwnRows * kOwnRing), n_groups - 1);
                        for (; g < whole; ++g) {
#pragma unroll
                            for (int u = 0; u < kOwnRing; ++u) {
                                if (u == 0) {
                                    issue(V[kOwnRing - 1], kOwnRing - 1, col);
                                    read_j(g + 1);
                                } else {
                                    issue(V[u - 1], u - 1, col);
                                }
                                read_u(U[(u + 1) & 1], g * kOwnRing + u + 1);
                                __builtin_amdgcn_sched_barrier(0);        // (the loads stay this far ahead)
#pragma unroll
                                for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                                    for (int d = 0; d < 2; ++d) {
                                        T[d][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(V[u][ks][d], half(U[u & 1][ks], 0), T[d][0], 0, 0, 0);
                                        if constexpr (H == 2)
                                            T[d][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(V[u][ks][d], half(U[u & 1][ks], 1), T[d][1], 0, 0, 0);
                                    }
                            }
                        }
                    }
                    for (; g < n_groups; ++g) group(g);
                    col[0] = col_next[0];
                    col[1] = col_next[1];

                    // ---- exchange ----
                    sp_lds_barrier();                                     // T^t of the round before has been read
#pragma unroll
                    for (int d = 0; d < 2; ++d)
#pragma unroll
                        for (int h = 0; h < H; ++h) {
                            double *tp = Tx + ((d * kOwnWaves + wave) * H + h) * 256 + lane * 2;
                            *reinterpret_cast<v2d *>(tp) = v2d{T[d][h].x, T[d][h].y};
                            *reinterpret_cast<v2d *>(tp + 128) = v2d{T[d][h].z, T[d][h].w};
                        }
                    // (into the registers that T^t has left)
#pragma unroll
                    for (int u = kOwnWAhead; u < kOwnWRing; ++u) fetch(u, code0, u);
                    sp_lds_barrier();

                    // ---- consumer: T^t of the next tile is read while a tile is multiplied ----
                    v2d Tr[2][2];
                    auto read_t = [&](v2d (&t)[2], uint32_t code) {
                        const lds_v2d *tp = TxV + ((code >> 9 & 15u) * H + my_half) * 128 + lane;
                        t[0] = tp[0];
                        t[1] = tp[64];
                    };
                    read_t(Tr[0], code[0]);
                    for (int e0 = 0; e0 < n_tiles; e0 += kOwnWRing) {
                        const uint32_t codes = e0 + kOwnWRing < 64 ? code0 : code1;
#pragma unroll
                        for (int u = 0; u < kOwnWRing; ++u) {
                            read_t(Tr[(u + 1) & 1], code[(u + 1) % kOwnWRing]);
                            // one bit per accumulator, its origin hidden: tests that the compiler can see to exclude one
                            // another become a switch, and accumulators are copied where its cases meet
                            uint32_t hot = 1u << (code[u] >> 13);
                            asm("" : "+s"(hot));
                            auto add = [&](v4d &z) {
                                z = __builtin_amdgcn_mfma_f64_16x16x4f64(W[u][0].x, Tr[u & 1][0].x, z, 0, 0, 0);
                                z = __builtin_amdgcn_mfma_f64_16x16x4f64(W[u][0].y, Tr[u & 1][0].y, z, 0, 0, 0);
                                z = __builtin_amdgcn_mfma_f64_16x16x4f64(W[u][1].x, Tr[u & 1][1].x, z, 0, 0, 0);
                                z = __builtin_amdgcn_mfma_f64_16x16x4f64(W[u][1].y, Tr[u & 1][1].y, z, 0, 0, 0);
                            };
                            if (H == 1 || hot & 0x0fu) {
                                if (hot & 0x01u) add(accZ[0]);
                                if (hot & 0x02u) add(accZ[1]);
                                if (hot & 0x04u) add(accZ[2]);
                                if (hot & 0x08u) add(accZ[3]);
                            }
                            if constexpr (H == 2) {
                                if (hot & 0x70u) {
                                    if (hot & 0x10u) add(accZ[4]);
                                    if (hot & 0x20u) add(accZ[5]);
                                    if (hot & 0x40u) add(accZ[6]);
                                }
                            }
                            fetch(u, codes, e0 + u + kOwnWRing);
                        }
                    }
                }
            }
            p0 += kOwnCap;
            if (p0 < n_union) {
                sp_lds_barrier();                                         // Uc and the offsets have been read
                prepare(p0, min(kOwnCap, n_union - p0), std::false_type{});
            }
        }
    }

    // ---- store the group's rows: lane holds Z^t[m = 16 mt + slot + 4 v][i = c] ----------------------
    const int64_t M = a.M;
    const int64_t s = s0 + 16 * my_half + c;
    if (s < a.slices) {
        const int64_t row = a.compact ? s : int64_t(a.uidx0[s]);
        double *dst = a.n_kc == 1 ? a.out + row * M : a.partial + (int64_t(kc) * a.slices + s) * M;
        // (a loop over the tiles, though unrolled later, makes the compiler hold four of them as one vector of 32 registers,
        // which it copies whole at every test of the consumer)
        sp_each(std::make_integer_sequence<int, kZ>{}, [&](auto X) {
            constexpr int x = decltype(X)::value;
            const int mt = my_class + kClasses * x;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int m = 16 * mt + slot + 4 * v;
                if (mt < a.MT && m < M) dst[m] = accZ[x][v];
            }
        });
    }
}

// Sums the partial results of the k chunks in chunk order; of those marked `present` where the others were not written.
// Sixteen loads in flight: a chain of single ones took 12 us over 44 chunks, this 4.
// Row r of the result is that of slice r, or of slice_of_row[r] (-1: none, zeros).  The launch takes the elements from `first`
// on: a result of 2^32 of them and more needs several launches, each of which has fewer threads than that.
constexpr int64_t kSpFixupLaunch = int64_t(1) << 31;
__global__ void sptn3_fixup_kernel(int64_t first, int64_t rows, int64_t slices, int64_t M, int n_kc,
                                   const int32_t *__restrict__ slice_of_row, const double *__restrict__ partial,
                                   const uint8_t *__restrict__ present, int n_groups, int group_shift, double *out) {
    const int64_t x = first + int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (x >= rows * M) return;
    const int64_t row = x / M, m = x - row * M, s = slice_of_row ? slice_of_row[row] : row;
    if (s < 0) {
        out[x] = 0.0;
        return;
    }
    double z = 0.0;
    for (int kc = 0; kc < n_kc; kc += 16) {
        double v[16];
        bool has[16];
#pragma unroll
        for (int u = 0; u < 16; ++u)
            has[u] = kc + u < n_kc && (!present || present[int64_t(min(kc + u, n_kc - 1)) * n_groups + (s >> group_shift)]);
#pragma unroll
        for (int u = 0; u < 16; ++u) v[u] = partial[(int64_t(min(kc + u, n_kc - 1)) * slices + s) * M + m];
#pragma unroll
        for (int u = 0; u < 16; ++u) z += has[u] ? v[u] : 0.0;
    }
    out[x] = z;
}

bool sptn3_two_waves_fit(int nwords) { return sptn3_owned_lds(nwords, 2) <= 160 * 1024; }

static conststn_status launch_sptn3_tiled(const conststn_plan_s *plan, const double *const *dense, double *out,
                                          hipStream_t stream) {
    const conststn_csf_s *U = plan->X, *W = plan->W;
    const bool owned = plan->sp_two_waves;
    Sptn3TileArgs a{};
    a.slices = U->nodes[0];
    a.L = W->dims[W->mode_order[1]];
    a.M = W->dims[W->mode_order[2]];
    a.LT = (a.L + 15) / 16;
    a.MT = int((a.M + 15) / 16);
    const int64_t J = U->dims[U->mode_order[2]];
    a.nwords = int((J + 31) / 32);
    a.n_groups = int((a.slices + plan->sp_group() - 1) / plan->sp_group());
    a.n_kc = plan->sp_kc * plan->sp_l_parts;
    a.l_parts = plan->sp_l_parts;
    a.k_per = plan->sp_k_per;
    a.uptr0 = U->ptr[0].p;
    a.uptr1 = U->ptr[1].p;
    a.uidx0 = U->idx[0].p;
    a.uidx1 = U->idx[1].p;
    a.uidx2 = U->idx[2].p;
    a.uvals = U->vals.p;
    a.w_root_of_k = plan->w_root_of_k.p;
    a.wmask = plan->w_tile_mask.p;
    a.wfirst = plan->w_tile_first.p;
    a.wcell_ptr = plan->w_cell_ptr.p;
    a.wcells = plan->w_cells.p;
    a.wtiles = plan->w_tiles.p;
    a.zero_tile = uint32_t(plan->n_w_tiles);
    a.V = dense[0];
    a.out = out;
    a.partial = plan->partial.p;
    a.compact = plan->compact ? 1 : 0;
    a.chunk_fiber = plan->sp_chunk_fiber.p;
    a.chunk_k = plan->sp_chunk_k.p;
    const int64_t n_work = owned ? int64_t(plan->sp_work.n) : 0;
    a.wg_order = plan->sp_xcd_ranges ? nullptr : plan->sp_wg_order.p;
    a.xcd_ranges = plan->sp_xcd_ranges ? 1 : 0;      // measured: halves the HBM fetch, 4 % slower
    const size_t lds_bytes = size_t(kCap) * 16 * 8 + size_t(4 * kStage) * 256 * 8 + size_t(a.MT) * 256 * 8 +
                             size_t(kCap) * 4 + size_t(a.nwords) * 8 + 64;
    // (with partial results the rows of absent slices are cleared by the pass that adds those up)
    if (!plan->compact && a.slices < plan->out_rows && (a.n_kc == 1 || a.slices == 0))
        CST_TRY(zero_fill(out, plan->out_rows * plan->row_elems, stream));
    if (a.slices == 0) return CONSTSTN_OK;
    // two wavefronts per SIMD (m tiles owned by wavefronts) when the plan chose it, else one (l tiles owned)
    const size_t lds_owned = sptn3_owned_lds(a.nwords, plan->sp_halves);
    {
        ProfScope prof(plan, stream);
        const unsigned n_wg = unsigned(a.n_groups) * unsigned(a.n_kc);
        // (a launch has fewer than 2^32 threads)
        for (int64_t first = 0; first < n_work; first += kOwnLaunch) {
            const dim3 grid(unsigned(std::min(n_work - first, kOwnLaunch))), block(64 * kOwnWaves);
            a.work = plan->sp_work.p + first;
            if (plan->sp_halves == 1) sptn3_owned_kernel<1><<<grid, block, lds_owned, stream>>>(a);
            else sptn3_owned_kernel<2><<<grid, block, lds_owned, stream>>>(a);
        }
        if (!owned) sptn3_tiled_kernel<<<dim3((n_wg + 7) / 8 * 8), dim3(256), lds_bytes, stream>>>(a);
    }
    CST_HIP(hipGetLastError());
    if (a.n_kc > 1) {
        const bool all = plan->compact || a.slices == plan->out_rows;
        const int64_t rows = plan->compact ? a.slices : plan->out_rows;
        for (int64_t first = 0; first < rows * a.M; first += kSpFixupLaunch) {
            const int64_t here = std::min(rows * a.M - first, kSpFixupLaunch);
            sptn3_fixup_kernel<<<dim3(unsigned((here + 255) / 256)), dim3(256), 0, stream>>>(
                first, rows, a.slices, a.M, a.n_kc, all ? nullptr : plan->sp_slice_of_row.p, a.partial,
                owned ? plan->sp_present.p : nullptr, a.n_groups, plan->sp_group() == kSpGroupWide ? 5 : 4, out);
            CST_HIP(hipGetLastError());
        }
    }
    return CONSTSTN_OK;
}

// Both tiled kernels take up to the whole 160 KB of a CU's LDS: the limit is raised when the plan is built.
conststn_status prepare_sptn3_launch(conststn_plan_s *plan) {
    plan->sp_xcd_ranges = plan->opt("sptn3_xcd", 0) == 1;
    CST_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(sptn3_tiled_kernel),
                                hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024));
    CST_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(sptn3_owned_kernel<1>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024));
    CST_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(sptn3_owned_kernel<2>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024));
    return CONSTSTN_OK;
}

conststn_status launch_sptn3(const conststn_plan_s *plan, const double *const *dense, double *out,
                             hipStream_t stream) {
    if (plan->w_tiled) return launch_sptn3_tiled(plan, dense, out, stream);
    const conststn_csf_s *U = plan->X, *W = plan->W;
    Sptn3Args a{};
    a.slices = U->nodes[0];
    a.L = W->dims[W->mode_order[1]];
    a.M = W->dims[W->mode_order[2]];
    a.uptr0 = U->ptr[0].p;
    a.uptr1 = U->ptr[1].p;
    a.uidx0 = U->idx[0].p;
    a.uidx1 = U->idx[1].p;
    a.uidx2 = U->idx[2].p;
    a.uvals = U->vals.p;
    a.wptr0 = W->ptr[0].p;
    a.wptr1 = W->ptr[1].p;
    a.widx1 = W->idx[1].p;
    a.widx2 = W->idx[2].p;
    a.wvals = W->vals.p;
    a.w_root_of_k = plan->w_root_of_k.p;
    a.V = dense[0];
    a.out = out;
    a.compact = plan->compact ? 1 : 0;
    const size_t lds_bytes = size_t(a.L + 4 * a.M) * sizeof(double);
    if (lds_bytes > 64 * 1024) {
        set_error("three-tensor kernel needs %zu bytes of LDS (L=%lld, M=%lld); at most 65536 implemented",
                  lds_bytes, (long long)a.L, (long long)a.M);
        return CONSTSTN_EUNSUPPORTED;
    }
    if (!plan->compact && a.slices < plan->out_rows)
        CST_TRY(zero_fill(out, plan->out_rows * plan->row_elems, stream));
    if (a.slices == 0) return CONSTSTN_OK;
    {
        ProfScope prof(plan, stream);
        sptn3_kernel<<<dim3(unsigned(a.slices)), dim3(256), lds_bytes, stream>>>(a);
    }
    CST_HIP(hipGetLastError());
    return CONSTSTN_OK;
}

}  // namespace cst
