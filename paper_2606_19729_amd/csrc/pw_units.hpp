// pw_units.hpp -- the work units of the grouped widening step's likelihood
// stage: which rows of which group a wave evaluates.  Plain index arithmetic,
// for the kernels and for the host.
//
// A unit is `rows` consecutive successors of one group (the group's last unit
// may be shorter).  Groups that do not overlap have at most T / 32 + M units
// between them, and these are listed, one record each, before the likelihood
// runs.  Offsets come from device memory and may be anything: when they fall
// and rise again, groups can share successors and have far more units than
// that.  Such offsets are not listed; the likelihood then walks every group's
// kPwMaxGroup / rows possible units instead, most of them empty.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace voila {

constexpr int kPwMaxGroup = 8192;  // successors per group (one workgroup normalises and resamples a group)

// Successors first .. end - 1 belong to group `group` (the unit's are the first
// `rows` of them; none if first = end).
struct PwUnit {
    int group, first, end;
};

// Group m's successors [lo, lo + n) if its own two offsets are in order within
// [0, T] and it fits one workgroup; otherwise none.
__host__ __device__ inline bool pw_rows(const int32_t* seg, int m, int T, int& lo, int& n) {
    const int a = seg[m], b = seg[m + 1];
    const bool ok = a >= 0 && b >= a && b <= T && b - a <= kPwMaxGroup;
    lo = ok ? a : 0;
    n = ok ? b - a : 0;
    return ok;
}
__host__ __device__ inline int pw_unit_count(int n, int rows) { return (n + rows - 1) / rows; }
// Records there is room for.
__host__ __device__ inline long pw_unit_capacity(int T, int M) { return (long)T / 32 + M; }
// What the prefix sums' last entry holds: the number of records, or -1 where
// `total` units are too many to list.
__host__ __device__ inline int pw_listed(long total, int T, int M) {
    return total <= pw_unit_capacity(T, M) ? (int)total : -1;
}
// Unit q of group m, whose successors are [lo, lo + n).
__host__ __device__ inline PwUnit pw_unit(int m, int lo, int n, int q, int rows) {
    const int at = q * rows;
    return PwUnit{m, lo + (at < n ? at : n), lo + n};
}
// Units of offsets that are not listed, and unit u of them.
__host__ __device__ inline long pw_unlisted_units(int M, int rows) { return (long)M * (kPwMaxGroup / rows); }
__host__ __device__ inline PwUnit pw_unlisted_unit(const int32_t* seg, int T, long u, int rows) {
    const int m = (int)(u / (kPwMaxGroup / rows)), q = (int)(u % (kPwMaxGroup / rows));
    int lo, n;
    pw_rows(seg, m, T, lo, n);
    return pw_unit(m, lo, n, q, rows);
}

}  // namespace voila
