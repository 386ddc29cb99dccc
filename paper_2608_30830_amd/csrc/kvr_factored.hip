// Bootstrap selection by the multiplicity-count closed form, a second method
// beside the brute-force grid (Eq. 1 and Eq. 3 integrated over sorted waits,
// as in the SORTED path, with bootstrap multiplicities as weights).
//
// With the base waits sorted once and, for one resample, c_i the number of
// times it draws base sample i, let N(x) = sum_{w_i <= x} c_i T_i and
// S(x) = sum_{w_i <= x} c_i T_i w_i, Ttot = N(inf).  Then for policy
// (t1, t2, lambda), e = t1 + t2:
//   m*C = a1*[S(t1) + t1*(Ttot - N(t1))]
//       + a2*[(S(e) - S(t1)) - t1*(N(e) - N(t1)) + (e - t1)*(Ttot - N(e))]
//       + b2*(N(e) - N(t1)) + b3*(Ttot - N(e)),
// dropping (e - t1)*(Ttot - N(e)) when e = +inf.  Per resample the work is a
// weighted histogram of its m draws over sorted positions, one prefix scan of
// length n, and O(1) per (policy, load): O(m + n + P*L) instead of the brute
// force's O(m*P*L).  N is exact (unsigned 64-bit); S, and so the costs, round
// differently from the brute force's per-sample sums, so the two methods
// agree within rounding and their selections up to rounding-level ties.
//
// Once per call: the base waits are radix-sorted; each t1 and each deadline
// gets its count of waits at or below it (a sorted position, a query), and
// the distinct query positions are numbered in order (slots).  (The queries
// need no order within a bin of the deadlines, but the sums' roundings follow
// it, and where a resample holds no wait between two deadlines the selection
// between them hangs on those roundings.)  Per batch of
// resamples: factored_prefix_kernel (one block per resample, four per CU: the
// draws' multiplicities per base sample in LDS, then, from LDS, a fixed-order
// scan of the weights c_k T_k (exact) and c_k T_k w_k over the positions that
// records N and S only at the query positions; up to 65,536 base samples
// factored_prefix_small_kernel, the same sums in the same order in fewer
// instructions), factored_policy_kernel (one block per (resample, tile of 32 or
// 16 loads): every policy from its two slots, fused arg-min on the numerators m*C).
#include "kvr_device.h"
#include "kvr_dpp.h"
#include "kvr_factored.h"

#include <type_traits>

namespace kvr {

constexpr int kFThreads = 1024;
constexpr int kFPThreads = 256;         // prefix kernel: four blocks (resamples) per CU
constexpr int kFLdsWords = 8192;        // 32 KiB of LDS counters per block
constexpr int kFBits = 4;               // bits of a narrow multiplicity counter
constexpr int kFPerWord = 32 / kFBits;  // narrow counters per LDS word
constexpr uint32_t kFMask = (1u << kFBits) - 1u;
constexpr int kFScanPer = 8;            // consecutive positions per thread in the scan
constexpr int kFUnroll = 8;             // draws per thread and step, fetched together
constexpr int kFLoads = 32;             // loads per policy-kernel block (16 when L <= 16)
constexpr int kFPolThreads = 256;
// Draws per resample up to which every N sum (m times a context size below
// 2^31) is an integer below 2^53, exact in double.
constexpr int64_t kFExactDoubleDraws = int64_t(1) << 22;

// Number of sorted waits <= x.
__device__ __forceinline__ int32_t count_le(const uint64_t *__restrict__ skeys, int64_t n, double x)
{
    int64_t lo = 0, hi = n;
    while (lo < hi) {
        const int64_t mid = lo + (hi - lo) / 2;
        if (__longlong_as_double((long long)skeys[mid]) <= x) lo = mid + 1;
        else hi = mid;
    }
    return (int32_t)lo;
}

// Items 0..n-1, per sorted position k: the sorted wait and the context size
// there (below 1 counts as 1; the sort has flagged it) and, per base sample, its
// sorted position; with cpos the place of the sample's counter in
// factored_prefix_small_kernel.  Items n..n+K1-1:
// u1[a] = #(w <= t1[a]); then P items: ue[f] = #(w <= e_f).  Both are
// marked in the position bitmask.
__global__ void __launch_bounds__(256) factored_rank_kernel(
    const uint64_t *__restrict__ skeys, const int32_t *__restrict__ perm,
    const int32_t *__restrict__ T, int64_t n, Tables tb, double *__restrict__ sw,
    int32_t *__restrict__ Ts, int32_t *__restrict__ rank, uint32_t *__restrict__ cpos,
    int32_t *__restrict__ u1, int32_t *__restrict__ ue,
    uint32_t *__restrict__ qbits)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t P = (int64_t)tb.K1 * tb.K2;
    if (k < n) {
        const int32_t i = perm[k];
        sw[k] = __longlong_as_double((long long)skeys[k]);
        const int32_t t = T[i];
        Ts[k] = t < 1 ? 1 : t;
        rank[i] = (int32_t)k;
        if (cpos != nullptr) {   // uniform: n <= 65,536
            const uint32_t ui = (uint32_t)i;
            cpos[k] = ((ui >> 1) & 0x7ffcu) | ((ui & 7u) << 18);
        }
        return;
    }
    const int64_t g = k - n;
    if (g >= tb.K1 + P) return;
    double x;
    if (g < tb.K1) {
        x = tb.t1[g];
    } else {
        const int64_t f = g - tb.K1;
        const int a = (int)(f / tb.K2), c = (int)(f % tb.K2);
        x = tb.t1[a] + tb.t2[c];
    }
    const int32_t q = count_le(skeys, n, x);
    if (g < tb.K1) u1[g] = q;
    else ue[g - tb.K1] = q;
    atomicOr(&qbits[q >> 5], 1u << (q & 31));
}

__global__ void __launch_bounds__(256) factored_fill_kernel(uint32_t *__restrict__ qbits,
                                                            int64_t nwords)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < nwords) qbits[i] = 0u;
}

// One block: qbase[w] = the marked positions in words 0 .. w-1 (an exclusive
// scan of the words' bit counts; each thread a run of consecutive words, the
// runs across the block in order).
__global__ void __launch_bounds__(kFThreads) factored_slot_kernel(const uint32_t *__restrict__ qbits,
                                                                  int32_t *__restrict__ qbase,
                                                                  int64_t nwords)
{
    constexpr int nw = kFThreads / kWave;
    __shared__ int32_t wsum[nw];
    const int lane = threadIdx.x % kWave, wv = threadIdx.x / kWave;
    const int64_t per = (nwords + kFThreads - 1) / kFThreads;
    const int64_t w0 = (int64_t)threadIdx.x * per;
    const int64_t w1 = (w0 + per < nwords) ? w0 + per : nwords;
    int32_t cnt = 0;
    for (int64_t w = w0; w < w1; ++w) cnt += __popc(qbits[w]);
    int32_t x = cnt;   // inclusive scan of the run totals within the wave
    for (int off = 1; off < kWave; off <<= 1) {
        const int32_t y = __shfl_up(x, off, kWave);
        if (lane >= off) x += y;
    }
    if (lane == kWave - 1) wsum[wv] = x;
    __syncthreads();
    int32_t next = x - cnt;
    for (int q = 0; q < wv; ++q) next += wsum[q];
    for (int64_t w = w0; w < w1; ++w) {
        qbase[w] = next;
        next += __popc(qbits[w]);
    }
}

// Slot of a marked position k: the marks below it.
__device__ __forceinline__ int32_t slot_of(const uint32_t *__restrict__ qbits,
                                           const int32_t *__restrict__ qbase, int64_t k)
{
    const uint32_t below = (1u << (k & 31)) - 1u;
    return qbase[k >> 5] + __popc(qbits[k >> 5] & below);
}

// Items 0..K1-1 and K1..K1+P-1: u1[a] and ue[f] from sorted positions to
// slots; items K1+P .. K1+P+last (for factored_prefix_kernel): the slot of each
// sorted position 0..last, -1 if it is no query position.
__global__ void __launch_bounds__(256) factored_remap_kernel(int32_t *__restrict__ u1,
                                                             int32_t *__restrict__ ue, int32_t K1,
                                                             int64_t P, int64_t last,
                                                             const uint32_t *__restrict__ qbits,
                                                             const int32_t *__restrict__ qbase,
                                                             int32_t *__restrict__ qslot)
{
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g < K1) {
        u1[g] = slot_of(qbits, qbase, u1[g]);
    } else if (g - K1 < P) {
        ue[g - K1] = slot_of(qbits, qbase, ue[g - K1]);
    } else if (g - K1 - P <= last) {
        const int64_t k = g - K1 - P;
        qslot[k] = ((qbits[k >> 5] >> (k & 31)) & 1u) ? slot_of(qbits, qbase, k) : -1;
    }
}

// One block per resample of the batch.  Per pass over a range of sorted
// positions: the number of the resample's draws of each position, counted in
// LDS, then a scan over the range in a fixed order (each thread its
// kFScanPer consecutive positions, the thread totals across the block: the
// lanes of a wave in wave_incl_scan's tree, the waves in order, then the
// earlier passes), which records
// at every query position k N(k) = sum_{j < k} c_j T_j (exact, then rounded
// to double as the closed form uses it) and S(k) = sum_{j < k} c_j T_j w_j
// (reproducible) in the query row, one 16-byte record per slot so that a
// policy's two lookups are two loads.  Position n (every wait) closes the
// row; tot[rb] = N(n).
//
// Counters: kFBits-bit fields of 32-bit LDS words, kFLdsWords * kFPerWord
// positions per pass (32 KiB, so that four blocks share a CU and one's
// barriers and loads overlap the others').  When that covers every position
// the draws are counted by base sample instead (no rank gather per draw) and
// the scan reads each position's count through the sort order.  A field that
// passes its maximum carries into (or out of) its word, and that only ever
// lowers the decoded total (a carry turns 2^kFBits counts into 1), so
// comparing the decoded total with the number of draws in the range (counted
// exactly) detects it; the resample then restarts with 32-bit counters by
// sorted position, kFLdsWords positions per pass.  A bootstrap row's
// multiplicities are Poisson(1)-like, so 4-bit fields almost never wrap.
// NT carries the N sums: double when every sum is an integer below 2^53 (the
// host picks it for m <= 2^22, a context size being below 2^31), where it is
// exact in any order and costs fewer instructions than 64-bit integers;
// unsigned 64-bit otherwise.
template <typename NT>
__global__ void __launch_bounds__(kFPThreads) factored_prefix_kernel(
    const int32_t *__restrict__ idx, int64_t n, int64_t m, int64_t r0,
    const int32_t *__restrict__ rank, const int32_t *__restrict__ perm,
    const int32_t *__restrict__ Ts,
    const double *__restrict__ sw, const int32_t *__restrict__ qslot, int64_t nqs,
    double2 *__restrict__ TQ, unsigned long long *__restrict__ tot, int *status)
{
    constexpr int nw = kFPThreads / kWave;
    constexpr int kTile = kFPThreads * kFScanPer;
    __shared__ uint32_t lh[kFLdsWords];
    __shared__ NT wn[nw];
    __shared__ double wsd[nw];
    __shared__ long long wchk[nw];
    const int64_t rb = blockIdx.x;
    const int64_t r = r0 + rb;
    double2 *qrow = TQ + rb * nqs;
    const int lane = threadIdx.x % kWave, wv = threadIdx.x / kWave;
    const int64_t B = blockDim.x;
    NT carry_n = 0;   // totals of the earlier positions (same in every thread)
    double carry_s = 0.0;
    for (int wide = 0; wide < 2; ++wide) {
        const int64_t PP = wide ? kFLdsWords : kFPerWord * (int64_t)kFLdsWords;   // positions per pass
        bool overflow = false;
        carry_n = 0;
        carry_s = 0.0;
        for (int64_t k0 = 0; k0 < n && !overflow; k0 += PP) {
            const int64_t nk = (n - k0 < PP) ? n - k0 : PP;
            const int64_t nwords = wide ? nk : (nk + kFPerWord - 1) / kFPerWord;
            // narrow counters over every position at once (n <= PP): count by
            // base sample instead of sorted position, so a draw needs no rank
            // gather; the scan then finds each position's count through perm
            const bool byidx = !wide && nk == n;
            for (int64_t x = threadIdx.x; x < nwords; x += B) lh[x] = 0u;
            __syncthreads();
            long long inr = 0;                              // draws counted in this range
            for (int64_t j = threadIdx.x; j < m; j += kFUnroll * B) {
                // the kFUnroll draws are loaded unconditionally (a position past
                // the row re-reads its last draw and is dropped) and checked with
                // selects and one branch for all, so the index loads, and then
                // the rank gathers, are in flight together
                int32_t ii[kFUnroll];
                bool live[kFUnroll];
#pragma unroll
                for (int u = 0; u < kFUnroll; ++u) {
                    live[u] = j + u * B < m;
                    ii[u] = idx[r * m + (live[u] ? j + u * B : m - 1)];
                }
                bool bad = false;
#pragma unroll
                for (int u = 0; u < kFUnroll; ++u) {
                    const bool out = ii[u] < 0 || (int64_t)ii[u] >= n;
                    bad = bad || (live[u] && out);
                    ii[u] = out ? 0 : ii[u];                // a bad draw counts as sample 0
                }
                if (bad) flag_domain(status);
                int64_t kk[kFUnroll];
#pragma unroll
                for (int u = 0; u < kFUnroll; ++u) {
                    kk[u] = byidx ? (int64_t)ii[u] : (int64_t)rank[ii[u]] - k0;
                    if (!live[u]) kk[u] = -1;                // past the row: no draw
                }
#pragma unroll
                for (int u = 0; u < kFUnroll; ++u) {
                    if (kk[u] >= 0 && kk[u] < nk) {
                        ++inr;
                        if (wide) atomicAdd(&lh[kk[u]], 1u);
                        else atomicAdd(&lh[kk[u] / kFPerWord], 1u << (kFBits * (int)(kk[u] % kFPerWord)));
                    }
                }
            }
            __syncthreads();
            if (!wide) {
                // decoded total minus the draws counted, over the whole block
                long long d = -inr;
                for (int64_t x = threadIdx.x; x < nwords; x += B) {
                    const uint32_t v = lh[x];
#pragma unroll
                    for (int h = 0; h < kFPerWord; ++h) d += (long long)((v >> (kFBits * h)) & kFMask);
                }
                d = wave_sum(d);
                if (lane == 0) wchk[wv] = d;
                __syncthreads();
                long long all = 0;
                for (int q = 0; q < nw; ++q) all += wchk[q];
                overflow = all != 0;                        // the same in every thread
                __syncthreads();
                if (overflow) break;
            }
            for (int64_t base = 0; base < nk; base += kTile) {
                const int64_t kl = base + (int64_t)threadIdx.x * kFScanPer;   // position in the pass
                NT cw[kFScanPer];
                double sv[kFScanPer];
                int32_t qs[kFScanPer];
                NT tn = 0;
                double ts = 0.0;
                // a full run of kFScanPer positions starts on a multiple of
                // kFScanPer (pass starts are multiples of 2^14): 16-byte loads
                // of Ts, qslot and perm (4 positions) and of sw (2) instead of
                // an element each
                int32_t tv[kFScanPer], qv[kFScanPer], pv[kFScanPer];
                double wv4[kFScanPer];
                if (kl + kFScanPer <= nk) {
                    static_assert(kFScanPer % 4 == 0, "the vector loads below read 4 positions");
#pragma unroll
                    for (int h = 0; h < kFScanPer; h += 4) {
                        const int4 t4 = *reinterpret_cast<const int4 *>(Ts + k0 + kl + h);
                        const int4 q4 = *reinterpret_cast<const int4 *>(qslot + k0 + kl + h);
                        const double2 w0 = reinterpret_cast<const double2 *>(sw + k0 + kl + h)[0];
                        const double2 w1 = reinterpret_cast<const double2 *>(sw + k0 + kl + h)[1];
                        tv[h] = t4.x; tv[h + 1] = t4.y; tv[h + 2] = t4.z; tv[h + 3] = t4.w;
                        qv[h] = q4.x; qv[h + 1] = q4.y; qv[h + 2] = q4.z; qv[h + 3] = q4.w;
                        wv4[h] = w0.x; wv4[h + 1] = w0.y; wv4[h + 2] = w1.x; wv4[h + 3] = w1.y;
                        if (byidx) {
                            const int4 p4 = *reinterpret_cast<const int4 *>(perm + k0 + kl + h);
                            pv[h] = p4.x; pv[h + 1] = p4.y; pv[h + 2] = p4.z; pv[h + 3] = p4.w;
                        }
                    }
                } else {
#pragma unroll
                    for (int q = 0; q < kFScanPer; ++q) {
                        const int64_t k = kl + q;
                        tv[q] = (k < nk) ? Ts[k0 + k] : 0;
                        qv[q] = (k < nk) ? qslot[k0 + k] : -1;
                        wv4[q] = (k < nk) ? sw[k0 + k] : 0.0;
                        if (byidx) pv[q] = (k < nk) ? perm[k0 + k] : 0;
                    }
                }
#pragma unroll
                for (int q = 0; q < kFScanPer; ++q) {
                    const int64_t k = kl + q;
                    const bool in = k < nk;
                    uint32_t c = 0u;
                    // the counter of position k, or of the base sample there
                    const int64_t ck = byidx ? (int64_t)((uint32_t)pv[q] < (uint32_t)n ? pv[q] : 0) : k;
                    if (in) c = wide ? lh[k] : (lh[ck / kFPerWord] >> (kFBits * (int)(ck % kFPerWord))) & kFMask;
                    const NT cwq = in ? (NT)c * (NT)tv[q] : (NT)0;   // exact
                    cw[q] = cwq;
                    sv[q] = (double)cwq * wv4[q];
                    qs[q] = in ? qv[q] : -1;
                    tn += cwq;
                    ts += sv[q];
                }
                // scan of the thread totals in the wave (DPP moves, a fixed tree)
                const NT xn = wave_incl_scan(tn), en = wave_lane_back(xn);
                const double xs = wave_incl_scan(ts), es = wave_lane_back(xs);
                if (lane == kWave - 1) {
                    wn[wv] = xn;
                    wsd[wv] = xs;
                }
                __syncthreads();
                NT pn = carry_n;
                double ps = carry_s;
                for (int q = 0; q < wv; ++q) {
                    pn += wn[q];
                    ps += wsd[q];
                }
                pn += en;
                ps += es;
                for (int q = 0; q < nw; ++q) {
                    carry_n += wn[q];
                    carry_s += wsd[q];
                }
#pragma unroll
                for (int q = 0; q < kFScanPer; ++q) {
                    if (qs[q] >= 0 && qs[q] < nqs) qrow[qs[q]] = make_double2((double)pn, ps);
                    pn += cw[q];
                    ps += sv[q];
                }
                __syncthreads();   // wn and wsd are rewritten by the next tile
            }
        }
        if (!overflow) break;
    }
    if (threadIdx.x == 0) {
        const int32_t q = qslot[n];
        if (q >= 0 && q < nqs) qrow[q] = make_double2((double)carry_n, carry_s);
        tot[rb] = (unsigned long long)carry_n;
    }
}

// The same rows for base samples of at most 65,536 (every 4-bit counter of a
// resample in LDS at once) and double N sums, with what the scan reads per
// position made ready: cpos[k] = byte address of the counter word of the base
// sample at sorted position k | its bit << 16.  A draw is five VALU operations
// and an LDS add, a position a 4-bit extract, two conversions and six fp64
// operations, everything in 32-bit indices; the rows are read 16
// bytes a lane from the first aligned draw on.  A wave's query slots are
// consecutive, so their records are gathered in LDS and stored as one run
// (up to kFStage of them, else one by one): scattered 16-byte stores took 200 of
// 660 us on the two-tier call (4,096 rows of 65,536 draws).  The draws alone
// take 189 us; the scan is bound by its VALU operations and the chain of each
// tile (reads, wave scans, barrier).  Two-tier: 786 us in
// factored_prefix_kernel, 580 us here.  Two resamples per block that share the
// reads measured the same, and the next tile's reads in flight 3 % less there but
// with a block less per CU (141 VGPRs) 5 % more at 1,024 rows.
//
// A wrapped counter is found as above (the decoded total differs from m); the
// resample is then counted again by sorted position with 32-bit counters,
// kFLdsWords positions per pass.  At m = 4 n and n = 65,536 about a quarter of the
// rows wrap, from m = 8 n practically all.  The recount is bound by the latency, and
// with four blocks to a CU by the rate, of its gathers of the ranks, 4 or 16 of them
// in flight per thread: 256 rows of 4 n, 8 n and 16 n draws 1.49, 4.32 and 8.45 ms per
// call (factored_prefix_kernel 2.44, 5.61 and 11.05; one draw at a time 3.44,
// 9.31 and 18.47).
constexpr int kFStage = 108;   // records per wave: four blocks of 39.5 KiB per CU

__global__ void __launch_bounds__(kFPThreads) factored_prefix_small_kernel(
    const int32_t *__restrict__ idx, int n, int m, int64_t r0, const int32_t *__restrict__ rank,
    const uint32_t *__restrict__ cpos, const int32_t *__restrict__ Ts,
    const double *__restrict__ sw, const uint32_t *__restrict__ qbits,
    const int32_t *__restrict__ qbase, int nqs, double2 *__restrict__ TQ,
    unsigned long long *__restrict__ tot, int *status)
{
    constexpr int nw = kFPThreads / kWave;
    constexpr int kTile = kFPThreads * kFScanPer;
    __shared__ uint32_t lh[kFLdsWords];
    __shared__ double2 wtot[2][nw];
    __shared__ double2 stage[nw][kFStage];
    __shared__ int wchk[nw];
    const int64_t rb = blockIdx.x;
    const int32_t *row = idx + (r0 + rb) * m;
    double2 *qrow = TQ + rb * nqs;
    const int t = threadIdx.x, lane = t % kWave, wv = t / kWave;
    double carry_n = 0.0, carry_s = 0.0;   // totals of the earlier positions (same in every thread)
    int parity = 0;

    // past one position, rounded as factored_prefix_kernel rounds (the product,
    // then the sum)
    auto advance = [](double &pn, double &ps, double cw, double w) {
#pragma clang fp contract(off)
        const double s = cw * w;
        pn = pn + cw;
        ps = ps + s;
    };
    // scan of positions [p0, p1), count(k, packed) the multiplicity at position k
    auto scan = [&](int p0, int p1, auto count) {
        for (int base = p0; base < p1; base += kTile) {
            const int k0 = base + t * kFScanPer;
            double w[kFScanPer], cw[kFScanPer];
            int32_t Ti[kFScanPer];
            uint32_t cp[kFScanPer];
            // marks of the 8 positions (k0 is a multiple of 8) and the slot of the first
            const int kw = (k0 < p1 ? k0 : p1 - 1) >> 5;
            const uint32_t word = qbits[kw];
            const int32_t wbase = qbase[kw];
            if (k0 + kFScanPer <= p1) {   // k0 is a multiple of 8: 16-byte loads
#pragma unroll
                for (int h = 0; h < kFScanPer; h += 4) {
                    const uint4 c4 = *reinterpret_cast<const uint4 *>(cpos + k0 + h);
                    const int4 t4 = *reinterpret_cast<const int4 *>(Ts + k0 + h);
                    cp[h] = c4.x; cp[h + 1] = c4.y; cp[h + 2] = c4.z; cp[h + 3] = c4.w;
                    Ti[h] = t4.x; Ti[h + 1] = t4.y; Ti[h + 2] = t4.z; Ti[h + 3] = t4.w;
                }
#pragma unroll
                for (int h = 0; h < kFScanPer; h += 2) {
                    const double2 w2 = *reinterpret_cast<const double2 *>(sw + k0 + h);
                    w[h] = w2.x; w[h + 1] = w2.y;
                }
            } else {
#pragma unroll
                for (int q = 0; q < kFScanPer; ++q) {
                    const bool in = k0 + q < p1;
                    const int k = in ? k0 + q : p1 - 1;
                    cp[q] = cpos[k];
                    Ti[q] = in ? Ts[k] : 0;
                    w[q] = in ? sw[k] : 0.0;
                }
            }
            double tn = 0.0, ts = 0.0;
#pragma unroll
            for (int q = 0; q < kFScanPer; ++q) {
                const int k = k0 + q < p1 ? k0 + q : p1 - 1;
                cw[q] = (double)count(k, cp[q]) * (double)Ti[q];   // exact, and so are their
                tn += cw[q];                                       // sums: integers below 2^53
                ts = fma(cw[q], w[q], ts);
            }
            const double xn = wave_incl_scan(tn), en = wave_lane_back(xn);
            const double xs = wave_incl_scan(ts), es = wave_lane_back(xs);
            if (lane == kWave - 1) wtot[parity][wv] = make_double2(xn, xs);
            __syncthreads();   // the next tile uses the other set of wave totals
            double pn = carry_n, ps = carry_s;
#pragma unroll
            for (int q = 0; q < nw; ++q) {
                const double2 v = wtot[parity][q];
                if (q < wv) {   // uniform per wave
                    pn += v.x;
                    ps += v.y;
                }
                carry_n += v.x;
                carry_s += v.y;
            }
            parity ^= 1;
            pn += en;
            ps += es;
            // marked positions of this lane, below p1, and the wave's slots
            const int shift = k0 & 31;
            uint32_t marks = (word >> shift) & 0xffu;
            if (k0 + kFScanPer > p1) marks &= k0 < p1 ? (1u << (p1 - k0)) - 1u : 0u;
            const int32_t slot0 = wbase + __popc(word & ((1u << shift) - 1u));
            const int32_t first = __builtin_amdgcn_readfirstlane(slot0);
            const int cnt = __popc(marks);
            const int upto = wave_incl_scan(cnt);   // marks are numbered in position order
            const int total = __builtin_amdgcn_readlane(upto, kWave - 1);
            int at = upto - cnt;
            if (total <= kFStage) {   // uniform per wave
#pragma unroll
                for (int q = 0; q < kFScanPer; ++q) {
                    if ((marks >> q) & 1u) stage[wv][at++] = make_double2(pn, ps);
                    advance(pn, ps, cw[q], w[q]);
                }
                __builtin_amdgcn_wave_barrier();
                for (int x = lane; x < total; x += kWave)
                    if (first + x < nqs) qrow[first + x] = stage[wv][x];
                __builtin_amdgcn_wave_barrier();
            } else {
#pragma unroll
                for (int q = 0; q < kFScanPer; ++q) {
                    if ((marks >> q) & 1u) {
                        if (first + at < nqs) qrow[first + at] = make_double2(pn, ps);
                        ++at;
                    }
                    advance(pn, ps, cw[q], w[q]);
                }
            }
        }
    };

    for (int x = t; x < kFLdsWords; x += kFPThreads) lh[x] = 0u;
    __syncthreads();
    // every draw of the row, read 16 bytes a lane from the first aligned one on, kQ
    // reads in flight: take(d) gets an array of 1, 4 or 4 kQ of them
    const int head_all = (int)((16u - ((uint32_t)(uintptr_t)row & 15u)) & 15u) / 4;   // to 16-byte alignment
    const int head = head_all < m ? head_all : m;
    const int quads = (m - head) / 4;
    auto each_draw = [&](auto take) {
        constexpr int kQ = 4;
        const int4 *v = reinterpret_cast<const int4 *>(row + head);
        auto one = [&](int j) {
            const int32_t d[1] = {row[j]};
            take(d);
        };
        if (t < head) one(t);
        int q = t;
        for (; q + (kQ - 1) * kFPThreads < quads; q += kQ * kFPThreads) {
            int4 x[kQ];
            int32_t d[4 * kQ];
#pragma unroll
            for (int u = 0; u < kQ; ++u) x[u] = v[q + u * kFPThreads];
#pragma unroll
            for (int u = 0; u < kQ; ++u) {
                d[4 * u] = x[u].x;
                d[4 * u + 1] = x[u].y;
                d[4 * u + 2] = x[u].z;
                d[4 * u + 3] = x[u].w;
            }
            take(d);
        }
        for (; q < quads; q += kFPThreads) {
            const int4 x = v[q];
            const int32_t d[4] = {x.x, x.y, x.z, x.w};
            take(d);
        }
        for (int j = head + 4 * quads + t; j < m; j += kFPThreads) one(j);
    };
    uint32_t most = 0;   // the largest index met, as unsigned
    each_draw([&](const auto &d) {
#pragma unroll
        for (int u = 0; u < (int)(sizeof(d) / sizeof(d[0])); ++u) {
            const uint32_t i = (uint32_t)d[u];
            most = most > i ? most : i;
            // a bad index counts somewhere in the table
            uint32_t *word = reinterpret_cast<uint32_t *>(reinterpret_cast<char *>(lh) + ((i >> 1) & 0x7ffcu));
            atomicAdd(word, 1u << ((i << 2) & 31u));
        }
    });
    if (most >= (uint32_t)n) flag_domain(status);
    __syncthreads();
    int decoded = 0;
    for (int x = t; x < kFLdsWords; x += kFPThreads) {
        uint32_t v = lh[x];
        v = (v & 0x0f0f0f0fu) + ((v >> 4) & 0x0f0f0f0fu);   // eight counts: four bytes up to 30
        decoded += (int)((v * 0x01010101u) >> 24);
    }
    decoded = wave_sum(decoded);
    if (lane == 0) wchk[wv] = decoded;
    __syncthreads();
    decoded = 0;
    for (int q = 0; q < nw; ++q) decoded += wchk[q];
    if (decoded == m) {   // the same in every thread
        scan(0, n, [&](int, uint32_t packed) {
            const uint32_t v = *reinterpret_cast<const uint32_t *>(
                reinterpret_cast<const char *>(lh) + (packed & 0xffffu));
            return (v >> (packed >> 16)) & kFMask;
        });
    } else {
        for (int p0 = 0; p0 < n; p0 += kFLdsWords) {
            const int p1 = n - p0 < kFLdsWords ? n : p0 + kFLdsWords;
            __syncthreads();
            for (int x = t; x < kFLdsWords; x += kFPThreads) lh[x] = 0u;
            __syncthreads();
            each_draw([&](const auto &d) {
                constexpr int nd = (int)(sizeof(d) / sizeof(d[0]));
                int32_t k[nd];
#pragma unroll
                for (int u = 0; u < nd; ++u)   // the ranks in flight together
                    k[u] = rank[(uint32_t)d[u] < (uint32_t)n ? d[u] : 0] - p0;
#pragma unroll
                for (int u = 0; u < nd; ++u)
                    if ((uint32_t)k[u] < (uint32_t)(p1 - p0)) atomicAdd(&lh[k[u]], 1u);
            });
            __syncthreads();
            scan(p0, p1, [&](int k, uint32_t) { return lh[k - p0]; });
        }
    }
    if (t == 0) {
        if ((qbits[n >> 5] >> (n & 31)) & 1u) {
            const int32_t q = qbase[n >> 5] + __popc(qbits[n >> 5] & ((1u << (n & 31)) - 1u));
            if (q < nqs) qrow[q] = make_double2(carry_n, carry_s);
        }
        tot[rb] = (unsigned long long)carry_n;
    }
}

// What the policies of one t1 row share: t1, (N, S) at t1 and a1 times the HBM
// term.
struct PolicyRow {
    double t1, n1, s1, hbm;
};

__device__ __forceinline__ PolicyRow policy_row(double2 q1, double t1, const PriceDev &pr,
                                                double tot)
{
    return PolicyRow{t1, q1.x, q1.y, pr.a1 * fma(t1, tot - q1.x, q1.y)};
}

// The load-independent part of a policy's total m*C and the factor of a2, from
// its row and (N, S) at its deadline.  Every multiply-add is spelled out, so two
// evaluations give the same bits.  No token is left past an infinite deadline
// (tot equals its N), so any finite holding time stands for it there.
__device__ __forceinline__ double2 policy_line(const PolicyRow &row, double2 qe, double t2,
                                               const PriceDev &pr, double tot)
{
#pragma clang fp contract(off)
    const double held = fmin((row.t1 + t2) - row.t1, 1.7976931348623157e308);
    const double host = qe.x - row.n1, past = tot - qe.x;
    const double after = fma(-row.t1, host, qe.y - row.s1);
    const double fixed = fma(pr.b3, past, fma(pr.b2, host, row.hbm));
    const double waiting = held * past;   // rounded by itself
    return make_double2(fixed, after + waiting);
}

// Arg-min over the 64 lanes of kPolLoads values each, by halves: at each step a
// lane hands one half of its values to the lane `off` away and keeps the
// other, so 15 merges replace 16 times six; then two steps for the last value.
// Lane 4 q ends with load q's result in c[0], f[0].
constexpr int kPolLoads = 16;           // loads per thread of the policy kernel
__device__ __forceinline__ void wave_argmin_halves(double (&c)[kPolLoads], int32_t (&f)[kPolLoads])
{
    const int lane = threadIdx.x % kWave;
#pragma unroll
    for (int half = kPolLoads / 2, off = kWave / 2; half > 0; half >>= 1, off >>= 1) {
        const bool up = (lane & off) != 0;   // keeps the upper half
#pragma unroll
        for (int l = 0; l < kPolLoads / 2; ++l) {
            if (l >= half) break;
            double c0 = c[l], c1 = c[l + half];
            int32_t f0 = f[l], f1 = f[l + half];
            // opaque copies: as elements of the arrays they are selected by a
            // run-time index, and the arrays leave the registers' names
            asm("" : "+v"(c0), "+v"(c1), "+v"(f0), "+v"(f1));
            const double oc = __shfl_xor(up ? c0 : c1, off, kWave);
            const int32_t of = __shfl_xor(up ? f0 : f1, off, kWave);
            c[l] = up ? c1 : c0;
            f[l] = up ? f1 : f0;
            argmin_merge(c[l], f[l], oc, of);
        }
    }
#pragma unroll
    for (int off = 2; off > 0; off >>= 1)
        argmin_merge(c[0], f[0], __shfl_xor(c[0], off, kWave), __shfl_xor(f[0], off, kWave));
}

// One block per (resample of the batch, tile of FL loads): every policy's
// closed-form total m*C for the tile's loads, the optional cost output, and
// the arg-min per load under the library's total order (smaller first, then
// larger flat index).  Dividing by m is monotone, so the arg-min compares the
// totals and only the selected one is divided.
//
// A thread evaluates groups of U host timers of one t1 row at 16 loads (a tile
// of 32 is shared by two halves of the block).  With U = 4 it takes the smallest
// of the four before it compares with its best so far and notes only the
// group: four FMAs, four mins, a compare and a select per four policies and
// load, 2.5 operations each in place of 4; which of the four it was (the largest
// index among equals) is found once per load at the end, from the same lines.
// Groups are numbered in the order of their policies and a thread meets its own
// in that order, so ties go to the larger index as the total order asks.
//
// The lines (policy_line) pass through LDS in chunks of 256 groups, two buffers
// deep: the query records of the next chunk are in flight while the current
// one is evaluated, and their slots, the same for every resample, are read a
// chunk earlier still.  A chunk is 256 / 2^lcp t1 rows by 2^lcp groups of a row, so its
// records lie near each other in the query row (deadlines of neighbouring t2)
// and leave L2 once: the kernel is bound by the latency of those gathers and by
// its FMAs and mins.  Two-tier (16,448
// policies, 32 loads) 384 us, with one record per policy looked up straight from
// the row by each thread 504 us; without the evaluation the gathers alone take
// 309 us (67 million 16-byte records), and records fetched two chunks ahead
// change nothing.
//
// COST (kernels of their own: the store's registers would cost the others a wave per
// SIMD, 986 -> 1,094 us for the two-tier call): the chunks run in the flat order of
// the policies, whose costs are stored from the lines in LDS, 64 consecutive ones a
// wave.  Stored as the lines are formed, from the windows of rows above, in runs
// of as few as 16 policies, most cache lines were written in two parts: 64 x 257
// policies, 16 loads and 512 rows (1.08 GB) took 757 us per call and 414 now (one thread a
// policy in flat order, the form before the lines, 416), 37 rows with 32 loads 377
// and 250 (320), 1,024 rows of 16 x 100 policies with 32 loads 188 and 141 (161).
// With chunks that meet in the middle of a line the first took 449.
template <int FL, int U, bool COST>
__global__ void __launch_bounds__(kFPolThreads *FL / kPolLoads) factored_policy_kernel(
    const double2 *__restrict__ TQ, int64_t nqs,
    const unsigned long long *__restrict__ totN, int64_t m, int64_t r0, int ntl, Tables tb,
    PriceDev pr, const int32_t *__restrict__ u1, const int32_t *__restrict__ ue, int lcp,
    int32_t *__restrict__ best, double *__restrict__ best_cost, double *__restrict__ cost_out)
{
    constexpr int kHalves = FL / kPolLoads, kThreads = kFPolThreads * kHalves;
    constexpr int kChunkP = kFPolThreads * U;            // policies per chunk
    constexpr int kPer = kChunkP / kThreads > 0 ? kChunkP / kThreads : 1;
    constexpr int nw = kFPolThreads / kWave;
    // line of policy U g + u of the chunk at [u][g]; a row is one record longer
    // than it needs, so that neighbouring policies' stores fall in other banks
    __shared__ double2 lines[2][U][kFPolThreads + 1];
    __shared__ PolicyRow rows_of[kFPolThreads];          // the chunk's t1 rows
    __shared__ double rc[nw][FL];
    __shared__ int32_t rf[nw][FL];
    __shared__ double la2[COST ? FL : 1];                // the tile's loads
    const int64_t rb = blockIdx.x / ntl;
    const int tile = (int)(blockIdx.x % ntl);
    const int64_t r = r0 + rb;
    const double2 *qrow = TQ + rb * nqs;   // (N, S) at the query slots
    const int64_t P = (int64_t)tb.K1 * tb.K2;
    const int l0 = tile * FL;
    const int nl = (tb.L - l0 < FL) ? tb.L - l0 : FL;
    const double tot = (double)totN[rb];
    const double md = (double)m;
    const int t = threadIdx.x;
    const int g = t % kFPolThreads;
    // uniform per wave: the half of the tile's loads this thread evaluates
    const int h0 = __builtin_amdgcn_readfirstlane(t / kFPolThreads) * kPolLoads;
    double a2[kPolLoads], bc[kPolLoads];
    int32_t bf[kPolLoads];   // group (policy for U = 1)
#pragma unroll
    for (int l = 0; l < kPolLoads; ++l) {
        a2[l] = tb.a2[l0 + h0 + l];   // zero-padded to whole tiles
        bc[l] = INFINITY;
        bf[l] = -1;
    }
    const int gpr = (tb.K2 + U - 1) / U;                   // groups of a row
    const int cp = 1 << lcp;                               // groups of a row per chunk
    // t1 rows per chunk (COST: at most)
    const int rp = COST ? min(kFPolThreads, (kFPolThreads - 1) / gpr + 2) : kFPolThreads >> lcp;
    // COST: a chunk begins again with the last groups (15 policies or more) of the one
    // before, whose costs up to the next multiple of 16 that one stores
    constexpr int kNext = kFPolThreads - (U > 1 ? 8 : 16);
    const int nchunk = COST ? (max(tb.K1 * gpr - kFPolThreads, 0) + kNext - 1) / kNext + 1
                            : ((gpr + cp - 1) >> lcp) * ((tb.K1 + rp - 1) / rp);
    // row (from the chunk's first) and group in it of group x of a chunk that begins
    // at group kg0 of a row
    const float per_gpr = 1.0f / (float)gpr, per_row = 1.0f / (float)tb.K2;
    auto place = [&](int kg0, int x) {
        if (!COST) return make_int2(x >> lcp, kg0 + (x & (cp - 1)));
        const int y = kg0 + x;   // below gpr + 256: at most one row on, or a quotient below 512
        const int row = gpr > kFPolThreads ? (y >= gpr ? 1 : 0) : (int)(((float)y + 0.5f) * per_gpr);
        return make_int2(row, y - row * gpr);
    };
    // the kPer policies of a chunk whose lines this thread forms: policy
    // p = x kThreads + t of the chunk is number p % U of group p / U
    const bool forms = kPer > 1 || t < kChunkP;            // uniform per wave
    const uint32_t last = (uint32_t)nqs - 1u;
    int32_t slot[kPer];
    double t2[kPer];
    double2 qe[kPer];
    auto group_of = [&](int x) { return (x * kThreads + t) / U; };
    // slots of the chunk whose first row and group of the row are a0 and kg0;
    // positions past a row's end or past the last row repeat the last one and
    // are never the smallest below
    auto slots = [&](int a0, int kg0) {
#pragma unroll
        for (int x = 0; x < kPer; ++x) {
            const int2 at = place(kg0, group_of(x));
            const int a = min(a0 + at.x, tb.K1 - 1);
            const int k = min(at.y * U + t % U, tb.K2 - 1);
            slot[x] = (int32_t)min((uint32_t)ue[a * tb.K2 + k], last);   // P < 2^24
            t2[x] = tb.t2[k];
        }
    };
    auto rows = [&](int a0) {
        if (t < rp) {
            const int a = min(a0 + t, tb.K1 - 1);
            rows_of[t] = policy_row(qrow[u1[a]], tb.t1[a], pr, tot);
        }
    };
    auto form = [&](int a0, int kg0, int buf) {
#pragma unroll
        for (int x = 0; x < kPer; ++x) {
            const int gx = group_of(x);
            const int2 at = place(kg0, gx);
            const int a = a0 + at.x, k = at.y * U + t % U;
            double2 ln = policy_line(rows_of[at.x], qe[x], t2[x], pr, tot);
            if (a >= tb.K1 || k >= tb.K2) ln = make_double2(INFINITY, 0.0);
            lines[buf][t % U][gx] = ln;
        }
    };
    // COST: a chunk's policies are consecutive; they are stored from a multiple of 16 to
    // the next chunk's, 64 a wave: whole cache lines where the rows of costs are aligned
    auto store_costs = [&](int a0, int kg0, int a1, int kg1, bool more, int buf) {
        const int row0 = a0 * tb.K2, f0 = (row0 + kg0 * U + 15) & ~15;
        const int f1 = more ? (a1 * tb.K2 + kg1 * U + 15) & ~15 : (int)P;
        for (int f = f0 + t; f < f1; f += kThreads) {
            // below K2 + 1,024: at most one row on, or a quotient below 2,048
            const int y = f - row0;
            const int row = tb.K2 > kChunkP ? (y >= tb.K2 ? 1 : 0) : (int)(((float)y + 0.5f) * per_row);
            const int k = y - row * tb.K2;
            const double2 ln = lines[buf][k % U][row * gpr + k / U - kg0];
            double *out = cost_out + (r * tb.L + l0) * P + f;
#pragma unroll 4
            for (int l = 0; l < nl; ++l) out[l * P] = fma(la2[l], ln.y, ln.x) / md;
        }
    };
    static_assert(kThreads % U == 0, "a thread's policies have one place in their groups");
    if (COST && t < FL) la2[t] = tb.a2[l0 + t];
    rows(0);
    if (forms) {
        slots(0, 0);
#pragma unroll
        for (int x = 0; x < kPer; ++x) qe[x] = qrow[slot[x]];
    }
    // the chunks run along the groups of a row, then to the next rows
    int a0 = 0, kg0 = 0;                        // chunk evaluated
    auto step = [&](int &a, int &kg) {
        if (COST) {
            kg += kNext;
            a += kg / gpr;
            kg %= gpr;
            return;
        }
        kg += cp;
        if (kg >= gpr) {
            kg = 0;
            a += rp;
        }
    };
    int a1 = 0, kg1 = 0;                        // the next one
    step(a1, kg1);
    int a2n = a1, kg2 = kg1;                    // the one after it
    step(a2n, kg2);
    __syncthreads();
    if (forms) {
        form(0, 0, 0);
        if (nchunk > 1) slots(a1, kg1);
    }
    __syncthreads();
    for (int c = 0, cur = 0; c < nchunk; ++c, cur ^= 1) {
        const bool more = c + 1 < nchunk;   // uniform
        if (more && forms) {
#pragma unroll
            for (int x = 0; x < kPer; ++x) qe[x] = qrow[slot[x]];
        }
        const int2 mine = place(kg0, g);                   // the group evaluated
        const int a = a0 + mine.x, kg = mine.y;
        if (a < tb.K1 && kg < gpr) {
            double2 ln[U];
#pragma unroll
            for (int u = 0; u < U; ++u) ln[u] = lines[cur][u][g];
            const int32_t id = a * gpr + kg;
            // a2 is zero-padded past L (never stored); groups come in
            // increasing order, so "not larger" keeps the larger index
#pragma unroll
            for (int l = 0; l < kPolLoads; ++l) {
                double v = fma(a2[l], ln[0].y, ln[0].x);
#pragma unroll
                for (int u = 1; u < U; ++u) v = fmin(v, fma(a2[l], ln[u].y, ln[u].x));
                const bool take = v <= bc[l];
                bc[l] = fmin(bc[l], v);
                bf[l] = take ? id : bf[l];
            }
        }
        if (COST) store_costs(a0, kg0, a1, kg1, more, cur);
        if (more) {
            if (COST || kg1 == 0) {   // the next chunk begins other t1 rows
                rows(a1);
                __syncthreads();
            }
            if (forms) {
                form(a1, kg1, cur ^ 1);
                if (c + 2 < nchunk) slots(a2n, kg2);
            }
        }
        a0 = a1;
        kg0 = kg1;
        a1 = a2n;
        kg1 = kg2;
        step(a2n, kg2);
        __syncthreads();
    }
    wave_argmin_halves(bc, bf);
    if (t % 4 == 0) {
        const int l = h0 + (t % kWave) / 4;
        rc[g / kWave][l] = bc[0];
        rf[g / kWave][l] = bf[0];
    }
    __syncthreads();
    if (t < nl) {
        const int l = t;
        double c = rc[0][l];
        int32_t id = rf[0][l];
        for (int q = 1; q < nw; ++q) argmin_merge(c, id, rc[q][l], rf[q][l]);
        int32_t f = id;
        if (id >= 0) {   // the policy of the group: the same lines, the same FMA
            const int a = id / gpr, k0 = (id - a * gpr) * U;
            f = a * tb.K2 + k0;
            const PolicyRow row = policy_row(qrow[u1[a]], tb.t1[a], pr, tot);
            double low = INFINITY;
            for (int k = k0; U > 1 && k < k0 + U && k < tb.K2; ++k) {
                const double2 ln = policy_line(row, qrow[ue[a * tb.K2 + k]], tb.t2[k], pr, tot);
                const double v = fma(tb.a2[l0 + l], ln.y, ln.x);
                if (v <= low) {
                    low = v;
                    f = a * tb.K2 + k;
                }
            }
        }
        best[r * tb.L + l0 + l] = f;
        best_cost[r * tb.L + l0 + l] = c / md;
    }
}

// Every 4-bit counter of a resample fits one block's LDS, and the N sums are
// exact in double.
bool factored_small(int64_t n, int64_t m)
{
    return n <= (int64_t)kFPerWord * kFLdsWords && m <= kFExactDoubleDraws;
}

int64_t factored_query_slots(int64_t n, int64_t K1, int64_t P)
{
    // distinct query positions: at most one per t1 and deadline, at most n + 1
    return (K1 + P < n + 1) ? K1 + P : n + 1;
}

int64_t factored_batch(int64_t nqs, int64_t R)
{
    // at most 2 GiB of query rows per batch, and batches of equal size (a
    // short last batch would leave most of the chip idle)
    const int64_t per = nqs * 16 + 8;
    int64_t rb = ((int64_t)1 << 31) / per;
    if (rb < 1) rb = 1;
    if (rb >= R) return R;
    const int64_t nb = (R + rb - 1) / rb;
    return (R + nb - 1) / nb;
}

// Logarithm of the groups of a row per chunk of the policy kernel: the fewest
// chunks, and among those the most rows (the narrowest span of deadlines).
static int policy_columns(int64_t K1, int64_t groups)
{
    int best = 0;
    int64_t least = INT64_MAX;
    for (int lcp = 0; (1 << lcp) <= kFPolThreads; ++lcp) {
        const int64_t rp = kFPolThreads >> lcp, cp = 1 << lcp;
        const int64_t chunks = ((K1 + rp - 1) / rp) * ((groups + cp - 1) / cp);
        if (chunks < least) {
            least = chunks;
            best = lcp;
        }
    }
    return best;
}

hipError_t launch_factored(const SampleSrc &src, int64_t R, const Tables &tb, const PriceDev &pr,
                           FactoredWs &ws, int32_t *best, double *best_cost, double *cost_out,
                           int *status, hipStream_t stream)
{
    const int64_t n = src.n, m = src.m;
    const int64_t P = (int64_t)tb.K1 * tb.K2;
    const int64_t nwords = (n + 1 + 31) / 32;
    int cur = 0;
    hipError_t err = launch_sort_keys(src.w, src.T, n, ws.sort, &cur, status, stream);
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(factored_fill_kernel, dim3((unsigned)((nwords + 255) / 256)), dim3(256), 0,
                       stream, ws.qbits, nwords);
    const dim3 gr((unsigned)((n + tb.K1 + P + 255) / 256));
    hipLaunchKernelGGL(factored_rank_kernel, gr, dim3(256), 0, stream, ws.sort.keys[cur],
                       ws.sort.vals[cur], src.T, n, tb, ws.sw, ws.Ts, ws.rank, ws.cpos, ws.u1,
                       ws.ue, ws.qbits);
    hipLaunchKernelGGL(factored_slot_kernel, dim3(1), dim3(kFThreads), 0, stream, ws.qbits, ws.qbase,
                       nwords);
    // the small prefix kernel reads the slots from qbits and qbase itself
    const int64_t last = ws.qslot != nullptr ? n : -1;
    hipLaunchKernelGGL(factored_remap_kernel, dim3((unsigned)((tb.K1 + P + last + 1 + 255) / 256)),
                       dim3(256), 0, stream, ws.u1, ws.ue, tb.K1, P, last, ws.qbits, ws.qbase,
                       ws.qslot);
    if ((err = hipGetLastError()) != hipSuccess) return err;
    // Groups of four host timers from where they fill a chunk on; fewer policies
    // keep a thread each (calls of 1,024 rows x 9,000 draws by U = 1 and 4: 1 x 257
    // policies 122.6 and 125.5 us, 4 x 257 127.1 and 131.1, 128 x 8 133.6 and 133.0,
    // 64 x 16 equal, 256 x 16 160.9 and 152.2, 512 x 8 166.1 and 157.4).
    const int U = tb.K2 >= 8 && P >= 4 * kFPolThreads ? 4 : 1;
    // Loads per policy block: up to 16 take half a tile, except where costs are wanted of
    // no more rows than CUs; there a block of 512 threads stores them faster (1, 64, 256
    // and 300 rows of 64 x 257 policies and 16 loads 250, 256, 297 and 352 us; with 256
    // threads 269, 274, 307 and 350).
    const bool few = cost_out != nullptr && R <= 256 && U == 4;
    const int FL = tb.L <= 16 && !few ? 16 : kFLoads;
    const int ntl = (tb.L + FL - 1) / FL;
    const int lcp = policy_columns(tb.K1, (tb.K2 + U - 1) / U);
    for (int64_t r0 = 0; r0 < R; r0 += ws.Rb) {
        const int64_t rb = (R - r0 < ws.Rb) ? R - r0 : ws.Rb;
        if (ws.cpos != nullptr)
            hipLaunchKernelGGL(factored_prefix_small_kernel, dim3((unsigned)rb), dim3(kFPThreads), 0,
                               stream, src.idx, (int)n, (int)m, r0, ws.rank, ws.cpos, ws.Ts, ws.sw,
                               ws.qbits, ws.qbase, (int)ws.nqs, ws.TQ, ws.tot, status);
        else if (m <= kFExactDoubleDraws)
            hipLaunchKernelGGL(factored_prefix_kernel<double>, dim3((unsigned)rb),
                               dim3(kFPThreads), 0, stream, src.idx, n, m, r0, ws.rank,
                               ws.sort.vals[cur], ws.Ts, ws.sw, ws.qslot, ws.nqs, ws.TQ, ws.tot,
                               status);
        else
            hipLaunchKernelGGL(factored_prefix_kernel<unsigned long long>, dim3((unsigned)rb),
                               dim3(kFPThreads), 0, stream, src.idx, n, m, r0, ws.rank,
                               ws.sort.vals[cur], ws.Ts, ws.sw, ws.qslot, ws.nqs, ws.TQ, ws.tot,
                               status);
        const dim3 gp((unsigned)(rb * ntl)), bp((unsigned)(kFPolThreads * FL / kPolLoads));
        auto pick = [&](auto cost) {
            constexpr bool C = decltype(cost)::value;
            return FL == 16 ? (U == 4 ? factored_policy_kernel<16, 4, C> : factored_policy_kernel<16, 1, C>)
                            : (U == 4 ? factored_policy_kernel<kFLoads, 4, C>
                                      : factored_policy_kernel<kFLoads, 1, C>);
        };
        auto policy = cost_out != nullptr ? pick(std::true_type()) : pick(std::false_type());
        hipLaunchKernelGGL(policy, gp, bp, 0, stream, ws.TQ, ws.nqs, ws.tot, m, r0, ntl, tb, pr,
                           ws.u1, ws.ue, lcp, best, best_cost, cost_out);
        if ((err = hipGetLastError()) != hipSuccess) return err;
    }
    return hipSuccess;
}

}  // namespace kvr
