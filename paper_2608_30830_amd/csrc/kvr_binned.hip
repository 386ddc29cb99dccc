// SORTED cost grid of one sample when no order is requested: N and S by
// deadline bins instead of a sort.
//
// The closed form (kvr_device.h, closed_form_values) needs N(x) = sum T [w <= x]
// and S(x) = sum T w [w <= x] only at the grid's own thresholds x: the K1
// timers t1 and the K1*K2 deadlines fl(t1 + t2).  With the thresholds in order,
// thr[0] <= thr[1] <= ..., and bin(x) = the number of thresholds strictly below
// x, w <= x holds exactly when bin(w) <= bin(x); so N and S at a threshold are
// inclusive prefix sums over its bin of per-bin sums, and the sample is read
// once (12 B per wait) instead of passing eight times through a radix sort
// (about 226 B per wait).
//
// The per-bin sums are exact integers, so neither the order of the atomics nor
// the split of the sample over blocks can change a result.  Within bin b the
// waits lie in (lower edge, upper edge], so T*w = T*edge + T*(w - edge), and
// w - edge is kept as a 64-bit fraction of the power of two above the bin's
// width; T times it (95 bits) is added in two 48-bit limbs.  So that this
// fraction is at least as fine as the binary64 product T*w for any grid and any
// wait, the powers 2^(10 q) over the whole range of finite numbers (and the
// largest one) are thresholds too: no bin is wider than 2^10 times its lower
// edge, and every wait has an upper edge.
//
// Measured on MI355X, the whole call against the sort: 2^24 waits and 66
// thresholds 68 us against 1,092 (the sums 56 us, 3.6 TB/s); 100,003 waits and
// 510 thresholds 31 us against 104 (28 launches of 3-5 us each, four now).
#include "kvr_device.h"
#include "kvr_dpp.h"

#include <math.h>

namespace kvr {

constexpr int kBinThreads = 1024;
constexpr int kBinIlp = 4;                 // waits per thread in flight
constexpr int kBinRange = 4095;            // bins of one range: 128 KiB of LDS with their edges
constexpr int64_t kBinChunk = 65536;       // waits per block at most: 48-bit limbs, 64-bit sums
constexpr int64_t kBinBlocks = 512;        // chunks that fill the chip (two blocks to a CU)
constexpr int kBinFused = 4096;            // bins that the closed form's own blocks scan
constexpr int kBinWords = 4;               // per bin: sum of T, then three 47-bit limbs of S
constexpr uint64_t kLimb = (uint64_t(1) << 47) - 1;
constexpr int kBinCopies = 8;              // of every bin, while a block scans them all itself
constexpr int kFixedEdges = 211;           // 2^-1070, 2^-1060, ..., 2^1020, the largest finite
constexpr int kBuckets = 512;              // search table: 16 buckets per binade, 32 binades
constexpr int kBinTiles = 64;              // tiles of kBinThreads bins, of 2 * 16,384 + 212 at most
constexpr int kBinLdsTable = 4096;         // timer-table entries staged in LDS
constexpr int kItemLanes = 8;              // lanes per threshold
constexpr int kFormPolicies = 64;          // policies of one closed-form block

static inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }
static inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// Waits per chunk, never more than kBinChunk.  B chunks cost n / B waits of work
// each (0.6 us per 1,024) and B * bins global adds of three words (about 32 a
// nanosecond on MI355X), least together at B = sqrt(6.25 n / bins); at most two
// blocks per CU.  (2^20 waits and 1,026 thresholds: 256 chunks
// 55 us, the 72 of this rule 23.)
static int64_t bin_chunk(int64_t n, int64_t bins)
{
    int64_t b = (int64_t)sqrt(6.25 * (double)n / (double)bins);
    b = b < 1 ? 1 : b < kBinBlocks ? b : kBinBlocks;
    const int64_t c = cdiv(cdiv(n, b), kBinThreads) * kBinThreads;
    return c < kBinChunk ? c : kBinChunk;
}

// Whether the costs come from the bins: up to 16,384 policies (nine ranges of bins
// at most, each of which reads the sample once).  With an order requested the scans
// that the bins replace (with the last scatter's keys) are cheap until their gather
// of the context sizes through the order leaves the caches, and the bins cost more
// the more thresholds there are.  By the scans and by the bins, us: 2^20 waits and 65
// policies 178 and 167, 544 policies 178 and 176, 1,025 policies 185 and 188; 2^21 waits
// and 1,025 policies 245 and 228, 15,120 policies 257 and 313; 16.4M waits and 65
// policies 1,612 and 1,104, 15,120 policies 1,639 and 1,584.
//
// A sample that one block sorts (kvr_sorted.hip) costs less in order than the search of
// the thresholds' own ranks along more than 48 rows of deadlines (columns, whichever are
// fewer).  By the sort and by the bins, us: 100 waits and 64 x 64 policies 25.2 and 26.3,
// 56 x 56 25.3 and 28.1, 128 x 128 29.5 and 37.4; 2,048 waits 29.1 and 29.5, 29.4 and
// 31.1, 33.8 and 40.9; with 48 x 48 25.1 and 23.6, 28.8 and 25.6, with 16 x 1,024 33.6 and
// 32.1, 38.3 and 34.4.
constexpr int64_t kOrderBinsFrom = int64_t(1) << 20;
constexpr int64_t kFewLines = 48;

bool bins_apply(int64_t n, int64_t K1, int64_t K2, bool order)
{
    const int64_t P = K1 * K2;
    if (n <= kOneBlockSort && (K1 < K2 ? K1 : K2) > kFewLines) return false;
    return P <= 16384 && (!order || (n >= kOrderBinsFrom && P <= n / 2048));
}

// Global copies of each bin, block q of the sums adding into copy q % copies:
// with one copy the atomics of 512 blocks on the same few addresses took 28 us
// of a 2^24-wait call with 66 thresholds (90 us; 68 with eight copies).  Reading
// eight copies costs the closed form's blocks 5 us at 723 bins, more than the
// adds of 98 blocks do; grids of more bins spread the adds by themselves.
static int bin_copies(int64_t n, int64_t bins)
{
    return bins <= kBinFused && cdiv(n, bin_chunk(n, bins)) > 128 ? kBinCopies : 1;
}

size_t bin_ws_bytes(int64_t n, int64_t K1, int64_t P)
{
    const int64_t M = K1 + P + kFixedEdges;
    return align256(sizeof(double) * (M + 1)) + align256(sizeof(int32_t) * (K1 + P)) +
           align256(sizeof(uint64_t) * kBinWords * bin_copies(n, M + 1) * (M + 1)) +
           2 * align256(sizeof(double) * (M + 1 + kBinTiles));
}

void bin_ws_carve(void *base, int64_t n, int64_t K1, int64_t P, double largest, BinWs &ws)
{
    char *p = static_cast<char *>(base);
    auto take = [&](size_t bytes) {
        char *q = p;
        p += align256(bytes);
        return q;
    };
    ws.M = (int)(K1 + P) + kFixedEdges;
    ws.chunk = bin_chunk(n, ws.M + 1);
    uint64_t bits;
    __builtin_memcpy(&bits, &largest, 8);
    const int top = (int)(bits >> 48);   // largest >= 0
    ws.bucket0 = top > kBuckets - 1 ? top - (kBuckets - 1) : 0;
    ws.nblocks = (int)cdiv(n, ws.chunk);
    ws.thr = (double *)take(sizeof(double) * (ws.M + 1));
    ws.at = (int32_t *)take(sizeof(int32_t) * (K1 + P));
    ws.copies = bin_copies(n, ws.M + 1);
    ws.bins = (unsigned long long *)take(sizeof(uint64_t) * kBinWords * ws.copies * (ws.M + 1));
    ws.cumN = (int64_t *)take(sizeof(int64_t) * (ws.M + 1 + kBinTiles));
    ws.cumS = (double *)take(sizeof(double) * (ws.M + 1 + kBinTiles));
}

__device__ __forceinline__ double fixed_edge(int q)
{
    if (q == kFixedEdges - 1) return 1.7976931348623157e308;
    const int ex = 10 * q - 1070;
    const uint64_t bits = ex >= -1022 ? (uint64_t)(ex + 1023) << 52 : 1ull << (ex + 1074);
    return __longlong_as_double((long long)bits);
}

// Biased exponent of a bin's width, whose sums count units of 2^(it - 1022 - 64).  From
// 12 down that unit is 2^-1074, of which every binary64 number is a multiple.
__device__ __forceinline__ int bin_scale(double width)
{
    const int e = (int)((uint64_t)__double_as_longlong(width) >> 52);
    return e > 12 ? e : 12;
}

// Item i < K1 is timer t1[i], item K1 + f policy f's deadline, the rest the
// fixed edges.  The bin of a timer or a deadline (the thresholds strictly
// below it) goes to at[i]; the thresholds in order to
// thr[0..M) (an item equal to others fills their whole run, and is left out
// when its neighbour on the searched axis is equal, so a run has at most
// min(K1, K2) + 2 writers, all of one value), thr[M] = inf.  The bins are
// cleared.  kItemLanes lanes share an item's searches.
__global__ void __launch_bounds__(256) bin_thresholds_kernel(Tables tb, BinWs ws)
{
    __shared__ double lt[kBinLdsTable];
    const double *t1v = tb.t1, *t2v = tb.t2;
    if (tb.K1 + tb.K2 <= kBinLdsTable) {   // uniform
        for (int q = threadIdx.x; q < tb.K1 + tb.K2; q += blockDim.x)
            lt[q] = q < tb.K1 ? tb.t1[q] : tb.t2[q - tb.K1];
        __syncthreads();
        t1v = lt;
        t2v = lt + tb.K1;
    }
    const int lane = (int)threadIdx.x % kItemLanes;
    const int i = (int)(blockIdx.x * (blockDim.x / kItemLanes) + threadIdx.x / kItemLanes);
    if (i > ws.M) return;   // whole groups of lanes
    for (int q = lane; q < kBinWords * ws.copies; q += kItemLanes)
        ws.bins[(int64_t)i * kBinWords * ws.copies + q] = 0ull;
    if (i == ws.M) {
        if (lane == 0) ws.thr[i] = INFINITY;
        return;
    }
    double x;
    bool fill = true;
    const int items = ws.M - kFixedEdges;
    if (i < tb.K1) {
        x = t1v[i];
    } else if (i >= items) {
        x = fixed_edge(i - items);
    } else {
        const int f = i - tb.K1, a = f / tb.K2, k = f % tb.K2;
        x = t1v[a] + t2v[k];
        if (tb.K1 <= tb.K2) fill = k == 0 || t1v[a] + t2v[k - 1] != x;
        else fill = a == 0 || t1v[a - 1] + t2v[k] != x;
    }
    int below = 0, equal = 0;   // this lane's rows (or columns), then all of them
    deadlines_rank(t1v, tb.K1, t2v, tb.K2, x, lane, kItemLanes, below, equal);
    if (lane == 0) {            // the timers are distinct: at most one equals x
        const int q = rank_below(t1v, tb.K1, 0.0, x);
        below += q;
        if (q < tb.K1 && t1v[q] == x) ++equal;
    }
    if (lane == 1) {
        int lo = 0, hi = kFixedEdges;   // first fixed edge >= x
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (fixed_edge(mid) < x) lo = mid + 1;
            else hi = mid;
        }
        below += lo;
        if (lo < kFixedEdges && fixed_edge(lo) == x) ++equal;
    }
    for (int off = kItemLanes / 2; off > 0; off >>= 1) {
        below += __shfl_xor(below, off, kItemLanes);
        equal += __shfl_xor(equal, off, kItemLanes);
    }
    if (lane == 0 && i < items) ws.at[i] = below;
    if (fill)
        for (int q = below + lane; q < below + equal; q += kItemLanes) ws.thr[q] = x;
}

// Block (range, chunk): the chunk's waits whose bin lies in the range
// [b0, b0 + nb) are added to the range's bins in LDS, then to the global ones.
// RP is the power of two above the number of bins (kBinRange + 1 at most): edge[0]
// is the range's lower edge, edge[1 + i] the upper edge of bin b0 + i, and
// from edge[1 + nb] on infinity.
//
// A wait's bin is searched between the edges of its bucket, the upper 16 bits
// of its binary64 word (16 buckets a binade, the top one holding the grid's
// largest timer; waits below or above take the end buckets): zero to three
// dependent LDS reads for grids of 64 to 1,024 log-spaced timers in place of
// log2(RP) (2^24 waits, nine steps: 87 -> 79 us).
template <int RP>
__global__ void __launch_bounds__(kBinThreads) bin_sums_kernel(const double *__restrict__ w,
                                                               const int32_t *__restrict__ T,
                                                               int64_t n, BinWs ws, int nranges,
                                                               int *status)
{
    __shared__ double edge[RP + 1];
    __shared__ unsigned long long sumT[RP], lo48[RP], hi48[RP];
    __shared__ uint16_t first[kBuckets + 1];
    const int range = (int)(blockIdx.x % nranges);
    const int64_t chunk = blockIdx.x / nranges;
    const int b0 = range * kBinRange;
    const int total = ws.M + 1;                       // bins 0..M
    const int nb = total - b0 < kBinRange ? total - b0 : kBinRange;
    const int64_t j0 = chunk * ws.chunk;
    const int64_t j1 = j0 + ws.chunk < n ? j0 + ws.chunk : n;
    double x[kBinIlp];
    int32_t t[kBinIlp];
    auto fetch = [&](int64_t jb) {   // positions past the chunk re-read its last wait
#pragma unroll
        for (int u = 0; u < kBinIlp; ++u) {
            const int64_t j = jb + u * kBinThreads;
            const int64_t jc = j < j1 ? j : j1 - 1;
            x[u] = w[jc];
            t[u] = T[jc];
        }
    };
    fetch(j0 + threadIdx.x);   // in flight while the tables are set up
    for (int q = threadIdx.x; q < RP; q += kBinThreads) {
        edge[q + 1] = q < nb ? ws.thr[b0 + q] : INFINITY;
        sumT[q] = lo48[q] = hi48[q] = 0ull;
    }
    // below the first range lies nothing: waits are >= 0, so an edge of -1
    // keeps w = 0 inside bin 0, whose offsets are taken from 0
    if (threadIdx.x == 0) edge[0] = b0 > 0 ? ws.thr[b0 - 1] : -1.0;
    __syncthreads();
    const double lower = edge[0], upper = edge[nb];   // of the whole range
    // first[b] = edges of the range (from edge[1] on) below every value of bucket b
    const int base0 = ws.bucket0;
    if ((int)threadIdx.x <= kBuckets) {
        const int b = threadIdx.x;
        const double v = __longlong_as_double((long long)((uint64_t)(base0 + b) << 48));
        int pos = 0;
        for (int step = RP / 2; step > 0; step >>= 1)   // pos + step < RP
            if (edge[pos + step] < v) pos += step;
        first[b] = (uint16_t)(b == 0 ? 0 : b == kBuckets || pos > nb - 1 ? nb - 1 : pos);
    }
    __syncthreads();
    bool bad = false;
    for (int64_t jb = j0 + threadIdx.x; jb < j1; jb += kBinIlp * kBinThreads) {
        if (jb != j0 + threadIdx.x) fetch(jb);
        int pos[kBinIlp], hi[kBinIlp];
        bool in[kBinIlp], more = false;
#pragma unroll
        for (int u = 0; u < kBinIlp; ++u) {
            const uint64_t bits = (uint64_t)__double_as_longlong(x[u]);
            if (!(bits < 0x7ff0000000000000ull || bits == 0x8000000000000000ull)) {
                bad = true;
                x[u] = 0.0;
            }
            if (t[u] < 1) {
                bad = true;
                t[u] = 1;
            }
            x[u] += 0.0;                                   // -0.0 -> +0.0
            in[u] = jb + u * kBinThreads < j1 && x[u] > lower && x[u] <= upper;
            const int b = (int)((uint64_t)__double_as_longlong(x[u]) >> 48) - base0;
            const int bc = b < 0 ? 0 : b < kBuckets ? b : kBuckets - 1;
            pos[u] = first[bc];
            hi[u] = in[u] ? (int)first[bc + 1] : pos[u];
            more |= pos[u] < hi[u];
        }
        while (__any(more)) {   // the number of edges below x lies in [pos, hi]
            more = false;
#pragma unroll
            for (int u = 0; u < kBinIlp; ++u) {
                const int mid = (pos[u] + hi[u]) >> 1;
                const bool open = pos[u] < hi[u], below = edge[mid + 1] < x[u];
                pos[u] = open && below ? mid + 1 : pos[u];
                hi[u] = open && !below ? mid : hi[u];
                more |= pos[u] < hi[u];
            }
        }
#pragma unroll
        for (int u = 0; u < kBinIlp; ++u) {
            if (!in[u]) continue;
            const double top = edge[pos[u] + 1];
            atomicAdd(&sumT[pos[u]], (unsigned long long)t[u]);
            double base = edge[pos[u]];
            base = base > 0.0 ? base : 0.0;
            // width < 2^(e - 1022): (w - base) * 2^(32 - (e - 1022)) < 2^32, by an
            // exponent add (the power itself overflows for widths below 2^-991)
            const int es = bin_scale(top - base);
            const double d = ldexp(x[u] - base, 1054 - es);
            const uint32_t dh = (uint32_t)d;
            const uint32_t dl = (uint32_t)((d - (double)dh) * 4294967296.0);
            const uint64_t p0 = (uint64_t)(uint32_t)t[u] * dl;
            const uint64_t p1 = (uint64_t)(uint32_t)t[u] * dh + (p0 >> 32);
            atomicAdd(&lo48[pos[u]], (unsigned long long)(((p1 & 0xffffu) << 32) | (uint32_t)p0));
            atomicAdd(&hi48[pos[u]], (unsigned long long)(p1 >> 16));
        }
    }
    if (bad) flag_domain(status);
    __syncthreads();
    for (int q = threadIdx.x; q < nb; q += kBinThreads) {
        if (sumT[q] == 0ull) continue;
        unsigned long long *out =
            ws.bins + ((int64_t)(b0 + q) * ws.copies + blockIdx.x % ws.copies) * kBinWords;
        atomicAdd(out, sumT[q]);
        // hi48 * 2^48 + lo48 (below 2^113) as limbs of 47, 47 and 19 bits: the
        // last is zero below 2^30 tokens a block
        const uint64_t lo = lo48[q], hi = hi48[q] + (lo >> 48);
        const uint64_t l0 = lo & kLimb, l1 = ((lo >> 47) & 1u) | ((hi << 1) & kLimb);
        if (l0 | l1) {
            atomicAdd(out + 1, l0);
            atomicAdd(out + 2, l1);
        }
        if (hi >> 46) atomicAdd(out + 3, hi >> 46);
    }
}

// One block of kBinThreads: the inclusive prefix sums of T and T*w over the bins
// [first, end), each thread a run of consecutive bins, in a fixed order
// (cumN and cumS are indexed from first).  An empty
// bin's S is that of the last bin before it that is not empty, bit for bit, so
// policies that no wait separates get equal costs.
template <typename NOut, typename SOut>
__device__ __forceinline__ void bin_prefix(const BinWs &ws, int first, int end, NOut *cumN,
                                           SOut *cumS)
{
    __shared__ int64_t wn[kBinThreads / kWave];
    __shared__ double wsum[kBinThreads / kWave];
    __shared__ int wl[kBinThreads / kWave];
    const int t = threadIdx.x, lane = t % kWave, wave = t / kWave;
    const int total = end - first;
    const int per = (total + kBinThreads - 1) / kBinThreads;
    const int q0 = t * per, q1 = q0 + per < total ? q0 + per : total;
    auto bin_of = [&](int b, int64_t &N, double &S) {
        const unsigned long long *from = ws.bins + (int64_t)b * kBinWords * ws.copies;
        unsigned long long in[kBinWords] = {0ull, 0ull, 0ull, 0ull};
        for (int c = 0; c < ws.copies; ++c)
#pragma unroll
            for (int q = 0; q < kBinWords; ++q) in[q] += from[c * kBinWords + q];
        N = (int64_t)in[0];
        const double base = b > 0 ? ws.thr[b - 1] : 0.0, top = ws.thr[b];
        if (isinf(top)) {   // no finite wait lies beyond the last fixed edge
            S = 0.0;
            return;
        }
        const int es = bin_scale(top - base);
        // the limbs count units of 2^(es - 1022 - 64)
        const double frac = (double)in[1] + ldexp((double)in[2] + ldexp((double)in[3], 47), 47);
        S = fma(base, (double)N, ldexp(frac, es - 1022 - 64));
    };
#pragma unroll 4
    for (int b = t; b < total; b += kBinThreads) {   // coalesced, read back below
        int64_t N;
        double S;
        bin_of(first + b, N, S);
        cumN[b] = N;
        cumS[b] = S;
    }
    __syncthreads();
    int64_t sn = 0;
    double ss = 0.0;
    int last = -1;
#pragma unroll 4
    for (int b = q0; b < q1; ++b) {
        const int64_t N = cumN[b];
        sn += N;
        ss += cumS[b];
        if (N != 0) last = b;
    }
    const int64_t xn = wave_incl_scan(sn);
    const double xs = wave_incl_scan(ss);
    const int xl = wave_incl_max(last);
    if (lane == kWave - 1) {
        wn[wave] = xn;
        wsum[wave] = xs;
        wl[wave] = xl;
    }
    __syncthreads();
    int64_t pn = 0;
    double ps = 0.0;
    int pl = -1;
    for (int q = 0; q < wave; ++q) {
        pn += wn[q];
        ps += wsum[q];
        pl = wl[q] > pl ? wl[q] : pl;
    }
    pn += wave_lane_back(xn);
    ps += wave_lane_back(xs);
    const int back = __shfl_up(xl, 1, kWave);   // every lane takes part
    if (lane > 0 && back > pl) pl = back;
    for (int b = q0; b < q1; ++b) {
        const int64_t N = cumN[b];
        pn += N;
        ps += cumS[b];
        cumN[b] = pn;
        if (N != 0) cumS[b] = ps;
    }
    __syncthreads();
    for (int b = q0; b < q1; ++b) {   // the empty bins
        const bool full = cumN[b] != (b > 0 ? cumN[b - 1] : 0);
        if (full) pl = b;
        else cumS[b] = pl >= 0 ? cumS[pl] : 0.0;
    }
    __syncthreads();
}

// Tile q of kBinThreads bins: the prefix sums within it, and its totals after the
// bins' own entries.  A tile's total is the sum at its last bin, so the sum before
// a tile is, bit for bit, the one at the last bin before it that is not empty.
__global__ void __launch_bounds__(kBinThreads) bin_prefix_kernel(BinWs ws)
{
    const int first = blockIdx.x * kBinThreads;
    const int end = first + kBinThreads < ws.M + 1 ? first + kBinThreads : ws.M + 1;
    bin_prefix(ws, first, end, ws.cumN + first, ws.cumS + first);
    if (threadIdx.x == 0) {
        ws.cumN[ws.M + 1 + blockIdx.x] = ws.cumN[end - 1];
        ws.cumS[ws.M + 1 + blockIdx.x] = ws.cumS[end - 1];
    }
}

// kFormPolicies policies per block, the block's other threads sharing their
// loads.  FUSED: the block forms the prefix sums itself, in LDS; else they come
// in tiles, whose totals every block adds up.
template <bool FUSED>
__global__ void __launch_bounds__(kBinThreads) bin_form_kernel(BinWs ws, int64_t n, Tables tb,
                                                               PriceDev pr,
                                                               double *__restrict__ cost)
{
    __shared__ int64_t lN[FUSED ? kBinFused : kBinTiles];
    __shared__ double lS[FUSED ? kBinFused : kBinTiles];
    if (FUSED) {
        bin_prefix(ws, 0, ws.M + 1, lN, lS);
    } else {
        const int tiles = (ws.M + kBinThreads) / kBinThreads;   // of M + 1 bins
        if ((int)threadIdx.x < tiles) {   // the sums before tile threadIdx.x
            int64_t N = 0;
            double S = 0.0;
            for (int q = 0; q < (int)threadIdx.x; ++q) {
                N += ws.cumN[ws.M + 1 + q];
                S += ws.cumS[ws.M + 1 + q];
            }
            lN[threadIdx.x] = N;
            lS[threadIdx.x] = S;
        }
        __syncthreads();
    }
    auto at = [&](int b, int64_t &N, double &S) {
        if (FUSED) {
            N = lN[b];
            S = lS[b];
        } else {
            N = lN[b / kBinThreads] + ws.cumN[b];
            S = lS[b / kBinThreads] + ws.cumS[b];
        }
    };
    const int64_t P = (int64_t)tb.K1 * tb.K2;
    const int64_t f = (int64_t)blockIdx.x * kFormPolicies + threadIdx.x % kFormPolicies;
    if (f >= P) return;
    const int a = (int)(f / tb.K2), k = (int)(f % tb.K2);
    const double t1 = tb.t1[a];
    int64_t tot, n1, ne;
    double sall, s1, se;
    at(ws.M, tot, sall);
    at(ws.at[a], n1, s1);
    at(ws.at[tb.K1 + f], ne, se);
    closed_form_values(tot, n1, ne, s1, se, n, tb, pr, f, t1, t1 + tb.t2[k],
                       (int)threadIdx.x / kFormPolicies, kBinThreads / kFormPolicies, cost);
}

hipError_t launch_binned(const double *w, const int32_t *T, int64_t n, const Tables &tb,
                         const PriceDev &pr, const BinWs &ws, double *cost_out, int *status,
                         hipStream_t stream)
{
    const int64_t P = (int64_t)tb.K1 * tb.K2;
    const int total = ws.M + 1;
    const int nranges = (int)cdiv(total, kBinRange);
    hipLaunchKernelGGL(bin_thresholds_kernel, dim3((unsigned)cdiv(total, 256 / kItemLanes)),
                       dim3(256), 0, stream, tb, ws);
    const dim3 grid((unsigned)(ws.nblocks * nranges)), block(kBinThreads);
    if (total < 512)
        hipLaunchKernelGGL(bin_sums_kernel<512>, grid, block, 0, stream, w, T, n, ws, nranges, status);
    else if (total < 2048)
        hipLaunchKernelGGL(bin_sums_kernel<2048>, grid, block, 0, stream, w, T, n, ws, nranges, status);
    else
        hipLaunchKernelGGL(bin_sums_kernel<kBinRange + 1>, grid, block, 0, stream, w, T, n, ws,
                           nranges, status);
    const dim3 form((unsigned)cdiv(P, kFormPolicies));
    if (total <= kBinFused) {
        hipLaunchKernelGGL(bin_form_kernel<true>, form, block, 0, stream, ws, n, tb, pr, cost_out);
    } else {
        const int tiles = (int)cdiv(total, kBinThreads);
        if (tiles > kBinTiles) return hipErrorInvalidValue;
        hipLaunchKernelGGL(bin_prefix_kernel, dim3((unsigned)tiles), block, 0, stream, ws);
        hipLaunchKernelGGL(bin_form_kernel<false>, form, block, 0, stream, ws, n, tb, pr, cost_out);
    }
    return hipGetLastError();
}

}  // namespace kvr
