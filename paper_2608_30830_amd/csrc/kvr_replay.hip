// Finite-capacity admission replay for gfx950 (Appendix D; the evaluation
// behind Table 6).
//
// Every request is offloaded to host DRAM at suspension.  The host tier has C2
// slots: a request that arrives while a slot is free is admitted, one that
// finds the tier full recomputes at resume, residents are never displaced.
// Under a host timer t2 an admitted request whose wait exceeds t2 leaves at
// arrival + t2 (discarded, recompute at resume); otherwise it leaves at
// arrival + wait (restored from host).  Departures at or before an arrival free
// their slots first.  A replay reports the tokens restored from host; the mean
// cost per request is (b2*R + b3*(Ttot - R)) / n.
//
// GPU formulation (no heap, no sort): a departure only matters through the
// arrival that finds its slot free, so request i is reduced to one integer per
// timer, its release: the first arrival j > i with a_j >= its departure instant
// (n when there is none).  Releases depend neither on each other nor on the
// admissions, so replay_release_kernel computes all of them in parallel;
// requests released at one arrival are interchangeable, so nothing has to be
// ordered.  What remains serial is a counter: at arrival j the slots of the
// admitted requests with release j are freed, then j is admitted if a slot is
// free.  replay_admit_kernel walks that recurrence 64 arrivals at a time, one
// wave per (timer, sequence).
//
// Measured on MI355X, 8,192 sequences x 4,000 requests x 5 timers: 0.65 ms per call, traced
// 0.31 ms for the releases and 0.37 ms for the walk.  The first form of this replay
// (a bitonic sort of the resume instants, 1.08 ms, two binary searches per
// request and timer, 0.36 ms, and one lane per (timer, sequence) stepping
// through every arrival, 0.95 ms) took 2.31 ms per call; with 100 sequences x
// 2 timers its walk, a chain of 4,000 steps per lane, took 0.84 ms against
// 0.047 ms now.
#include "kvr_device.h"
#include "kvr_dpp.h"

#include <math.h>

namespace kvr {

constexpr int kReplayMaxN = 8192;
constexpr int kReplayIlp = 4;                    // requests a thread searches together
constexpr unsigned kReplayMaxBlocks = 1u << 20;  // rows or pairs beyond this many loop
constexpr uint32_t kStaysBit = 0x8000u;

// Threads and time buckets of the release kernel for rows of up to MAXN
// requests: blocks of eight waves, three to a CU (41 KiB of LDS each), at
// 4,096; half as many buckets as arrivals at 8,192, so that two blocks fit.
constexpr int replay_threads(int maxn) { return maxn / 8 < 512 ? maxn / 8 : 512; }
constexpr int replay_buckets(int maxn) { return maxn < 4096 ? maxn : 4096; }

__device__ __forceinline__ bool valid_time(double x)
{
    const uint64_t b = (uint64_t)__double_as_longlong(x);   // finite and >= 0, or -0.0
    return b < 0x7ff0000000000000ull || b == 0x8000000000000000ull;
}

// Bucket of instant x among nb equal parts of the row's arrivals: a monotone
// function of x (each step rounds monotonically), clamped to 0 .. nb - 1 before
// it becomes an integer.  No NaN: a0 is finite, so x - a0 is none for a departure
// that overflowed to infinity, and the scale is positive.
__device__ __forceinline__ int time_bucket(double x, double a0, double scale, int nb)
{
    const double t = fmin((x - a0) * scale, (double)(nb - 1));
    return (int)fmax(t, 0.0);
}

// For every request j of a row (n <= MAXN) and timer k the packed word
//   release | [w_j <= t2_k] << 15
// laid out [timer][reps][n] for the kc timers t2s[0..kc): release = the first
// arrival after j at or after fl(a_j + w_j) when w_j <= t2_k, else at or after
// fl(a_j + t2_k); n when no arrival is.  One block per row (blocks stride over
// the rows).
//
// The searches go through a table of the first arrival of each of many equal
// time buckets (two bytes each, beside the row's arrivals in LDS): the bucket
// function being monotone, the answer lies between the first arrivals of the
// instant's own bucket and of the next one, about one arrival apart for a
// Poisson row, so a lane takes about three dependent LDS reads where a search
// over the row takes twelve; any other row (bursts, one instant repeated) is
// still searched exactly, at worst over the whole row.  A thread's searches
// advance kReplayIlp together, so their reads overlap.  The kernel is bound by
// its VALU instructions (one fp64 bucket per search) and by LDS latency, not by
// HBM (16 B read per request, 2 B written per request and timer).
//
// With counts given (the controller), the row's waits <= t_star and its tokens
// are added to them in the same pass (integers: the order cannot matter).
template <int MAXN>
__global__ void __launch_bounds__(replay_threads(MAXN))
__attribute__((amdgpu_waves_per_eu(MAXN <= 4096 ? 6 : 4))) replay_release_kernel(
    const double *__restrict__ arrival, const double *__restrict__ wait,
    const int32_t *__restrict__ ctx, int64_t reps, int n, const double *__restrict__ t2s, int kc,
    uint16_t *__restrict__ rel, double t_star, unsigned long long *counts, int *status)
{
    constexpr int kThreads = replay_threads(MAXN), kPer = MAXN / kThreads;
    constexpr int kBuckets = replay_buckets(MAXN);
    __shared__ double A[MAXN];
    __shared__ uint16_t first[kBuckets + 1];   // first arrival of each bucket's instants or later
    __shared__ int64_t part[2][kThreads / kWave];
    const int t = threadIdx.x;
    for (int64_t row = blockIdx.x; row < reps; row += gridDim.x) {
        bool bad = false;
        {
            double a[kPer];
#pragma unroll
            for (int q = 0; q < kPer; ++q) {
                const int j = t + q * kThreads;
                a[q] = j < n ? arrival[row * n + j] : 0.0;
            }
#pragma unroll
            for (int q = 0; q < kPer; ++q) {
                const int j = t + q * kThreads;
                if (!valid_time(a[q])) {
                    bad = true;
                    a[q] = 0.0;
                }
                if (j < n) A[j] = a[q];
            }
        }
        __syncthreads();
        const double a0 = A[0], span = A[n - 1] - a0;
        double scale = (double)kBuckets / span;
        // no span, or one so small that its scale overflows: every arrival in bucket 0
        // (a scale of 0 would make an infinite departure inf * 0)
        if (!(span > 0.0) || !(scale <= 1.7976931348623157e308)) scale = 2.2250738585072014e-308;
        for (int j = t; j < n; j += kThreads) {
            const double aj = A[j], before = j > 0 ? A[j - 1] : aj;
            if (!(before <= aj)) bad = true;   // arrivals must not decrease
            // the buckets after the previous arrival's, up to this one's,
            // start here; the last arrival also closes the table
            const int b = time_bucket(aj, a0, scale, kBuckets);
            const int b0 = j > 0 ? time_bucket(before, a0, scale, kBuckets) + 1 : 0;
            for (int x = b0; x <= b; ++x) first[x] = (uint16_t)j;
            if (j == n - 1)
                for (int x = b + 1; x <= kBuckets; ++x) first[x] = (uint16_t)n;
        }
        __syncthreads();

        int n_short = 0;
        int64_t tokens = 0;
        for (int j0 = t; j0 < n; j0 += kReplayIlp * kThreads) {
            double a[kReplayIlp], w[kReplayIlp];
            int lo[kReplayIlp], hi[kReplayIlp], resume[kReplayIlp];
#pragma unroll
            for (int q = 0; q < kReplayIlp; ++q) {
                const int j = j0 + q * kThreads;
                w[q] = j < n ? wait[row * n + j] : 0.0;
                a[q] = j < n ? A[j] : 0.0;
            }
            if (ctx != nullptr) {   // uniform
#pragma unroll
                for (int q = 0; q < kReplayIlp; ++q) {
                    const int j = j0 + q * kThreads;
                    const int32_t T = j < n ? ctx[row * n + j] : 1;
                    bad |= T < 1;
                    tokens += j < n ? T : 0;
                }
            }
#pragma unroll
            for (int q = 0; q < kReplayIlp; ++q) {
                if (!valid_time(w[q])) {
                    bad = true;
                    w[q] = 0.0;
                }
                n_short += j0 + q * kThreads < n && w[q] <= t_star ? 1 : 0;
            }
            // [lo, hi] holds the first arrival after j at or after instant d
            auto open_range = [&](int q, double d) {
                const int j = j0 + q * kThreads;
                const int b = time_bucket(d, a0, scale, kBuckets);
                const int f = first[b];
                lo[q] = f > j + 1 ? f : j + 1;
                hi[q] = first[b + 1];
            };
            // narrows every lo[q] to the first arrival of its range at or
            // after a[q] + add(q)
            auto search = [&](auto add) {
                bool more = false;
#pragma unroll
                for (int q = 0; q < kReplayIlp; ++q) more |= lo[q] < hi[q];
                while (__any(more)) {   // each open range at least halves
                    more = false;
#pragma unroll
                    for (int q = 0; q < kReplayIlp; ++q) {
                        const bool open = lo[q] < hi[q];
                        const int mid = open ? (lo[q] + hi[q]) >> 1 : 0;
                        const bool less = A[mid] < a[q] + add(q);
                        lo[q] = open && less ? mid + 1 : lo[q];
                        hi[q] = open && !less ? mid : hi[q];
                        more |= lo[q] < hi[q];
                    }
                }
            };
#pragma unroll
            for (int q = 0; q < kReplayIlp; ++q) {
                lo[q] = hi[q] = 0;
                if (j0 + q * kThreads < n) open_range(q, a[q] + w[q]);
            }
            search([&](int q) { return w[q]; });
#pragma unroll
            for (int q = 0; q < kReplayIlp; ++q) resume[q] = lo[q];
            for (int k = 0; k < kc; ++k) {
                const double t2 = t2s[k];
                uint16_t *out = rel + ((int64_t)k * reps + row) * n;
#pragma unroll
                for (int q = 0; q < kReplayIlp; ++q) {
                    lo[q] = hi[q] = resume[q];
                    if (j0 + q * kThreads < n && !(w[q] <= t2)) open_range(q, a[q] + t2);
                }
                search([&](int) { return t2; });
#pragma unroll
                for (int q = 0; q < kReplayIlp; ++q) {
                    const int j = j0 + q * kThreads;
                    if (j < n) out[j] = (uint16_t)((uint32_t)lo[q] | (w[q] <= t2 ? kStaysBit : 0u));
                }
            }
        }
        if (bad) flag_domain(status);
        if (counts != nullptr) {   // uniform
            const int64_t shorts = wave_sum((int64_t)n_short);
            tokens = wave_sum(tokens);
            if (t % kWave == 0) {
                part[0][t / kWave] = shorts;
                part[1][t / kWave] = tokens;
            }
            __syncthreads();
            if (t < 2) {
                int64_t s = 0;
                for (int x = 0; x < kThreads / kWave; ++x) s += part[t][x];
                if (t == 1 && ctx == nullptr) s = n;   // one token per request
                atomicAdd(&counts[t], (unsigned long long)s);
            }
        }
        __syncthreads();   // the next row rewrites the arrivals and the table
    }
}

// One wave per (timer k0 + k, sequence) pair, k < kc, the pairs numbered
// timer-major; blocks stride over the pairs.  freed[j] counts the admitted
// requests with release j in 16 bits (at most n <= 8,192), two to a word.
//
// The wave takes 64 arrivals at a time, one per lane.  With the slots freed at
// each of them known, the occupancy is x_j = min(x_{j-1} - freed_j + 1, cap): a
// sum reflected at cap.  So with S_j the running sum of 1 - freed_j,
// M_j = max(0, max_{i <= j} (x + S_i - cap)) counts the refusals so far, and j
// is admitted exactly when M_j = M_{j-1}: two scans by DPP moves in place of 64
// dependent steps (one when the 64 fit below cap in any case).  Only requests
// released within their own 64 arrivals make freed_j depend on the decisions
// being made: they start out counted as admitted, and the scans are repeated
// with the corrected counts until no such decision changes.  A decision depends
// on earlier lanes only, so each round settles at least one more lane: at most
// 65 rounds.  How many depends on the chains of requests that free a slot for the
// next one within 64 arrivals, so on C2: for Poisson arrivals at one to three times
// the critical load 1.0-2.8 on average at C2 = 425, 4-7 at 8, 9-14 at 2 (regular
// patterns of arrivals and waits reach 33 at 2 to 4).  8,192 sequences x 4,000
// requests x 5 timers take 0.58-0.63 ms per call at C2 = 425, 0.97-1.07 at 8 and
// 1.78-1.85 at 2.
//
// ONE: with a single slot the admitted requests are a chain, each the arrival that
// releases the one before, and everything between is refused; so the wave follows
// the releases, a run of admissions of neighbouring arrivals at a time, without
// counts.  At 0.1, 1 and 3 times the critical load that call takes 0.62, 1.12 and
// 1.12 ms, by rounds (5 to 20 per 64 arrivals) 1.11, 2.67 and 2.68.
//
// Bound by the wave's instruction stream (about 100 VALU instructions and four
// LDS accesses per 64 arrivals and round), 19 waves per CU by LDS at n = 4,000; the
// packed words are read four steps ahead.
template <bool CTX, bool ONE>
__global__ void __launch_bounds__(kWave) replay_admit_kernel(
    const int32_t *__restrict__ ctx, int64_t reps, int n, int64_t c2,
    const uint16_t *__restrict__ rel, double b2, double b3, double *__restrict__ cost,
    int64_t *__restrict__ restored_out, int64_t *__restrict__ admitted_out, int k0, int kn, int K)
{
    extern __shared__ uint32_t freed[];   // [64 * ceil(n / 64) / 2], none with ONE
    const int lane = threadIdx.x;
    const int steps = (n + kWave - 1) / kWave;
    const int words = ONE ? 0 : steps * (kWave / 2);
    const int64_t pairs = reps * kn;
    // occupancy is at most n, so C2 above n is the same as n + 1
    const int cap = (c2 > (int64_t)n) ? n + 1 : (int)c2;
    for (int64_t F = blockIdx.x; F < pairs; F += gridDim.x) {
        const int k = (int)(F / reps);
        const int64_t row = F % reps;
        const uint16_t *R = rel + F * n;
        const int32_t *C = CTX ? ctx + row * n : nullptr;
        for (int q = lane; q < words; q += kWave) freed[q] = 0u;
        __syncthreads();

        int occ = 0, admitted = 0;      // uniform
        int next = 0;                   // ONE: the next arrival that finds the slot free
        int64_t restored = 0, total = 0;
        auto count = [&](bool adm, bool in, bool stays, int32_t T) {
            admitted += __popcll(__ballot(adm));
            if (CTX) {
                T = T < 1 ? 1 : T;
                total += in ? T : 0;
                restored += adm && stays ? T : 0;
            } else {
                restored += __popcll(__ballot(adm && stays));
            }
        };
        auto follow = [&](uint32_t x, int32_t T, int j0) {
            const int end = j0 + kWave < n ? j0 + kWave : n, last = end - j0 - 1;
            const int release = (int)(x & (kStaysBit - 1));   // later than its request
            // where a run of admissions ends: the slot is not free again at the next arrival
            const uint64_t stops = __ballot(release != j0 + lane + 1) | 1ull << last;
            uint64_t chain = 0;
            while (next < end) {
                const int p = next - j0, q = p + __builtin_ctzll(stops >> p);   // q <= last
                chain |= (~0ull >> (kWave - 1 - q)) & (~0ull << p);
                const int f = __builtin_amdgcn_readlane(release, q);
                next = f > j0 + q ? f : j0 + q + 1;
            }
            count(((chain >> lane) & 1u) != 0u, j0 + lane < n, (x & kStaysBit) != 0u, T);
        };
        auto step = [&](uint32_t x, int32_t T, int j0) {
            const int j = j0 + lane;
            const bool in = j < n;
            const int f = in ? (int)(x & (kStaysBit - 1)) : n;
            const bool stays = (x & kStaysBit) != 0u;
            const bool inner = f < n && f < j0 + kWave;    // released within these 64
            uint32_t *word = &freed[f < n ? f >> 1 : 0];
            const uint32_t one = 1u << ((f & 1) * 16);
            const uint64_t inners = __ballot(inner);       // uniform
            if (inner) atomicAdd(word, one);
            __syncthreads();
            bool adm = in;
            const bool fits = occ + kWave <= cap;          // uniform
            int s, m;
            for (bool guess = true;;) {
                const uint32_t pairw = freed[j >> 1];
                const int free_j = (int)((pairw >> ((j & 1) * 16)) & 0xffffu);
                s = wave_incl_scan(in ? 1 - free_j : 0);
                m = 0;
                if (fits) break;
                m = wave_incl_max(occ + s - cap);
                m = m > 0 ? m : 0;
                adm = in && m == wave_lane_back(m);
                const bool changed = inner && adm != guess;
                if (inners == 0 || __ballot(changed) == 0) break;
                __syncthreads();
                if (changed) atomicAdd(word, adm ? one : 0u - one);
                guess = adm;
                __syncthreads();
            }
            occ += __builtin_amdgcn_readlane(s, kWave - 1) - __builtin_amdgcn_readlane(m, kWave - 1);
            count(adm, in, stays, T);
            if (adm && !inner && f < n) atomicAdd(word, one);
            __syncthreads();
        };
        constexpr int kAhead = 4;
        uint32_t x[kAhead];
        int32_t T[kAhead];
        auto fetch = [&](int u, int j0) {   // positions past the row re-read its last word
            const int j = j0 + lane < n ? j0 + lane : n - 1;
            x[u] = R[j];
            T[u] = CTX ? C[j] : 1;
        };
#pragma unroll
        for (int u = 0; u < kAhead; ++u) fetch(u, u * kWave);
        for (int jb = 0; jb < n; jb += kAhead * kWave) {
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                const int j0 = jb + u * kWave;
                if (j0 < n) {   // uniform
                    const uint32_t xu = x[u];
                    const int32_t Tu = T[u];
                    fetch(u, j0 + kAhead * kWave);
                    if constexpr (ONE) follow(xu, Tu, j0);
                    else step(xu, Tu, j0);
                }
            }
        }
        if (CTX) {
            restored = wave_sum(restored);
            total = wave_sum(total);
        } else {
            total = n;
        }
        if (lane == 0) {
            const int64_t sim = row * K + k0 + k;
            cost[sim] = (b2 * (double)restored + b3 * (double)(total - restored)) / (double)n;
            if (restored_out) restored_out[sim] = restored;
            if (admitted_out) admitted_out[sim] = admitted;
        }
        __syncthreads();   // the next pair clears the counts
    }
}

// Timers per pass of the two kernels: at most 1 GiB of release words.
static int replay_timer_chunk(int64_t reps, int64_t n, int K)
{
    int64_t kc = ((int64_t)1 << 30) / (2 * reps * n);
    if (kc < 1) kc = 1;
    return (int)(kc < K ? kc : K);
}

size_t replay_ws_bytes(int64_t reps, int64_t n, int K)
{
    auto a256 = [](size_t x) { return (x + 255) & ~(size_t)255; };
    const int kc = replay_timer_chunk(reps, n, K);
    return a256(sizeof(uint16_t) * kc * reps * n) + a256(sizeof(double) * K);
}

template <int MAXN>
static void launch_release(const double *arrival, const double *wait, const int32_t *ctx,
                           int64_t reps, int n, const double *t2, int kc, uint16_t *rel,
                           double t_star, unsigned long long *counts, int *status,
                           hipStream_t stream)
{
    const unsigned blocks = reps < kReplayMaxBlocks ? (unsigned)reps : kReplayMaxBlocks;
    hipLaunchKernelGGL(replay_release_kernel<MAXN>, dim3(blocks), dim3(replay_threads(MAXN)), 0,
                       stream, arrival, wait, ctx, reps, n, t2, kc, rel, t_star, counts, status);
}

hipError_t launch_replay(const double *arrival, const double *wait, const int32_t *ctx,
                         int64_t reps, int64_t n, const double *h_t2, int K, int64_t c2, double b2,
                         double b3, void *ws, double *cost, int64_t *restored,
                         int64_t *admitted, double t_star, void *counts, int *status,
                         hipStream_t stream)
{
    auto a256 = [](size_t x) { return (x + 255) & ~(size_t)255; };
    const int kc = replay_timer_chunk(reps, n, K);
    char *p = static_cast<char *>(ws);
    uint16_t *rel = reinterpret_cast<uint16_t *>(p);
    p += a256(sizeof(uint16_t) * kc * reps * n);
    double *t2 = reinterpret_cast<double *>(p);
    double *const dst[3] = {t2, nullptr, nullptr};
    const double *const src[3] = {h_t2, nullptr, nullptr};
    const int64_t cnt[3] = {K, 0, 0};
    hipError_t err = launch_stage(status, dst, src, cnt, static_cast<unsigned *>(counts), 4, stream);
    const int ni = (int)n;
    for (int k0 = 0; k0 < K && err == hipSuccess; k0 += kc) {
        const int kn = (K - k0 < kc) ? K - k0 : kc;
        // the counts are taken once, with the first timers
        unsigned long long *c = k0 == 0 ? static_cast<unsigned long long *>(counts) : nullptr;
        if (n <= 1024)
            launch_release<1024>(arrival, wait, ctx, reps, ni, t2 + k0, kn, rel, t_star, c, status, stream);
        else if (n <= 4096)
            launch_release<4096>(arrival, wait, ctx, reps, ni, t2 + k0, kn, rel, t_star, c, status, stream);
        else
            launch_release<kReplayMaxN>(arrival, wait, ctx, reps, ni, t2 + k0, kn, rel, t_star, c, status, stream);
        if ((err = hipGetLastError()) != hipSuccess) break;
        const int64_t pairs = reps * kn;
        const unsigned blocks = pairs < kReplayMaxBlocks ? (unsigned)pairs : kReplayMaxBlocks;
        // one slot is followed, more are counted (the kernel's comment has both measured)
        const size_t lds = c2 == 1 ? 0 : sizeof(uint16_t) * kWave * (size_t)((n + kWave - 1) / kWave);
        auto admit = c2 == 1 ? (ctx != nullptr ? replay_admit_kernel<true, true>
                                               : replay_admit_kernel<false, true>)
                             : (ctx != nullptr ? replay_admit_kernel<true, false>
                                               : replay_admit_kernel<false, false>);
        hipLaunchKernelGGL(admit, dim3(blocks), dim3(kWave), lds, stream, ctx, reps, ni, c2, rel,
                           b2, b3, cost, restored, admitted, k0, kn, K);
        err = hipGetLastError();
    }
    return err;
}

}  // namespace kvr
