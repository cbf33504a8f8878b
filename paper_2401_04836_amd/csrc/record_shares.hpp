// Slices of the MTTKRP record stream that several chunks share: what the fix-up launch reads of them, how it is made, and
// what the plan check holds it against.  Plain C++, so that the check itself is tested on the host.
#pragma once

#include <cstdint>

#ifdef __HIPCC__
#define CST_BOTH __host__ __device__ __forceinline__
#else
#define CST_BOTH inline
#endif

namespace cst {

constexpr int kRecLight = 32;              // chunks of a slice from which on it counts as one of many

struct alignas(16) RecordShare {
    int64_t first;                         // 2 x its first chunk, + 1 where it begins inside that
    int32_t count, row;                    // number of its chunks; row of the result
};

// 0: inside one chunk; 1: shared by a few chunks; 2: by many
CST_BOTH int share_of(const int64_t *slice_rec, int64_t s, int64_t q) {
    const int64_t span = (slice_rec[s + 1] - 1) / q - slice_rec[s] / q;
    return span == 0 ? 0 : (span < kRecLight ? 1 : 2);
}

CST_BOTH RecordShare record_share(const int64_t *slice_rec, int64_t s, int64_t q, int32_t row) {
    const int64_t lo = slice_rec[s], hi = slice_rec[s + 1], first = lo / q;
    return RecordShare{2 * first + (lo != first * q ? 1 : 0), int32_t((hi - 1) / q - first + 1), row};
}

CST_BOTH bool same_share(const RecordShare &a, const RecordShare &b) {
    return a.first == b.first && a.count == b.count && a.row == b.row;
}

// Whether the list (ascending: a slice that shares a chunk with the next begins in an earlier one) holds the share.
CST_BOTH bool share_listed(const RecordShare *list, int64_t n, const RecordShare &share) {
    int64_t lo = 0, hi = n;
    while (lo < hi) {
        const int64_t mid = (lo + hi) / 2;
        if (list[mid].first < share.first) lo = mid + 1; else hi = mid;
    }
    return lo < n && same_share(list[lo], share);
}

// Whether entry e of the list of slices of one kind is that of such a slice, and stands behind the entry before.  The slice
// is the one that goes on behind its first chunk.
CST_BOTH bool share_entry_right(const RecordShare *list, int64_t e, int kind, const int64_t *slice_rec, int64_t slices,
                                int64_t n_rec, int64_t q, const int32_t *row_of_slice) {
    if (e > 0 && list[e - 1].first >= list[e].first) return false;
    const int64_t chunk = list[e].first >> 1;
    if (chunk < 0 || chunk >= n_rec / q || (chunk + 1) * q >= n_rec) return false;
    int64_t lo = 0, hi = slices;                                      // the slice of that record
    while (hi - lo > 1) {
        const int64_t mid = (lo + hi) / 2;
        if (slice_rec[mid] <= (chunk + 1) * q) lo = mid; else hi = mid;
    }
    return share_of(slice_rec, lo, q) == kind && same_share(list[e], record_share(slice_rec, lo, q, row_of_slice[lo]));
}

}  // namespace cst
