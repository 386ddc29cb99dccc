// Device helpers shared by the library's kernels.
#pragma once

#include "kvr_internal.h"

namespace kvr {

__device__ __forceinline__ void flag_domain(int *status)
{
    __hip_atomic_store(status, kStatusDomain, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

struct Sample {
    double w, T;
};

// Read sample j of a resample (row offset row_off into idx), replacing bad
// values by safe ones and flagging the status word.
__device__ __forceinline__ Sample fetch_sample(const SampleSrc &s, int64_t row_off, int64_t j,
                                               int *status)
{
    int64_t i = j;
    if (s.idx) {
        int32_t ii = s.idx[row_off + j];
        if (ii < 0 || (int64_t)ii >= s.n) {
            flag_domain(status);
            ii = 0;
        }
        i = ii;
    }
    double w = s.w[i];
    int32_t t = s.T[i];
    // finite and >= 0 (or -0.0), tested on the bits so that no floating-point
    // mode or NaN assumption can remove the check
    const uint64_t bits = (uint64_t)__double_as_longlong(w);
    if (!(bits < 0x7ff0000000000000ull || bits == 0x8000000000000000ull)) {
        flag_domain(status);
        w = 0.0;
    }
    if (t < 1) {
        flag_domain(status);
        t = 1;
    }
    Sample out;
    out.w = w + 0.0;  // -0.0 -> +0.0
    out.T = (double)t;
    return out;
}

template <typename V>
__device__ __forceinline__ V wave_sum(V v)
{
    for (int off = kWave / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
    return v;
}

// Total order used by every selection: smaller cost first, then larger f.
__device__ __forceinline__ void argmin_merge(double &bc, int32_t &bf, double oc, int32_t of)
{
    const bool take = (oc < bc) | ((oc == bc) & (of > bf));
    bc = take ? oc : bc;
    bf = take ? of : bf;
}

__device__ __forceinline__ void wave_argmin(double &bc, int32_t &bf)
{
    for (int off = kWave / 2; off > 0; off >>= 1) {
        double oc = __shfl_xor(bc, off, kWave);
        int32_t of = __shfl_xor(bf, off, kWave);
        argmin_merge(bc, bf, oc, of);
    }
}

// Hardware hands work-groups to the 8 XCDs round-robin; remap so that each
// XCD walks a contiguous range of logical blocks (same resample rows, same
// L2).
__device__ __forceinline__ int64_t xcd_logical_block(int64_t hw, int64_t nblocks)
{
    const int64_t nx = 8;
    int64_t x = hw % nx, q = nblocks / nx, rem = nblocks % nx;
    return x * q + (x < rem ? x : rem) + hw / nx;
}

// Values v0 + v[q] strictly below x, for ascending v[0..K).
__device__ __forceinline__ int rank_below(const double *v, int K, double v0, double x)
{
    int lo = 0, hi = K;   // first q with v0 + v[q] >= x
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (v0 + v[mid] < x) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// Grid deadlines fl(t1[a] + t2[k]) strictly below x and equal to x, added to
// below and equal: one search along each row (column when K1 > K2, whichever
// are fewer; rounding is monotone, so both are non-decreasing) first,
// first + step, ...
__device__ __forceinline__ void deadlines_rank(const double *t1v, int K1, const double *t2v, int K2,
                                               double x, int first, int step, int &below,
                                               int &equal)
{
    const bool rows = K1 <= K2;
    const int lines = rows ? K1 : K2, len = rows ? K2 : K1;
    const double *line0 = rows ? t1v : t2v, *v = rows ? t2v : t1v;
    for (int q = first; q < lines; q += step) {
        const double v0 = line0[q];
        const int lo = rank_below(v, len, v0, x);
        below += lo;
        int run = lo, hi = len;   // values equal to x: [lo, run)
        if (lo < len && v0 + v[lo] == x) {
            while (run < hi) {
                const int mid = (run + hi) >> 1;
                if (v0 + v[mid] <= x) run = mid + 1;
                else hi = mid;
            }
        }
        equal += run - lo;
    }
}

// The closed form of policy f for every load, from the tokens (N) and
// tokens x waits (S) of the waits <= t1 and <= e; loads l0, l0 + lstep, ... are
// written.
__device__ __forceinline__ void closed_form_values(int64_t tot, int64_t n1, int64_t ne, double s1,
                                                   double se, int64_t n, const Tables &tb,
                                                   const PriceDev &pr, int64_t f, double t1,
                                                   double e, int l0, int lstep,
                                                   double *__restrict__ cost)
{
    const int64_t P = (int64_t)tb.K1 * tb.K2;
    const double hbm = s1 + t1 * (double)(tot - n1);
    double hold = (se - s1) - t1 * (double)(ne - n1);
    if (!isinf(e)) hold += (e - t1) * (double)(tot - ne);
    const double fixed = pr.a1 * hbm + pr.b2 * (double)(ne - n1) + pr.b3 * (double)(tot - ne);
    const double nd = (double)n;
    for (int l = l0; l < tb.L; l += lstep) cost[(int64_t)l * P + f] = (fixed + tb.a2[l] * hold) / nd;
}

}  // namespace kvr
