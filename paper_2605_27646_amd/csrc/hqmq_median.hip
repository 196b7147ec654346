// Med3x outlier extraction, first half: the exact per-head median of the squared chunk norms
// (paper Sec. 3 "Median-multiplier outlier extraction", Alg. 1 "Outlier extraction").
//
// The median is the lower median (element (n-1)/2 of the sorted norms) of all B*T*ceil(D/4) chunks
// of a head.  Non-negative IEEE doubles order like their bit patterns read as unsigned integers,
// and nothing is sorted and no float arithmetic is involved after r^2 itself, so the result is the exact order
// statistic.  Each sweep recomputes r^2 in registers from the fp16 tensor (8 B per chunk).
//
// A sample predicts a narrow range of keys around the median (its ranks within four standard deviations of the middle
// one).  One sweep then counts the keys below the range and keeps those in it, in 16 lists by where in the range
// they lie, and the wanted rank is located in the one list that holds it by histograms over ever narrower ranges
// (select_rank).  The prediction decides which keys are kept, never the result.
//   heads of at most 1024 rows   one workgroup selects from its registers (k_select_head)
//   longer heads                 k_select_predict (one to eight workgroups per head), k_select_count (the sweep), k_select_digit (the
//                                selection), k_select_finish (only where the prediction missed)
// For a head whose prediction missed, or whose list overflowed, k_select_digit makes a histogram of 8192 equal parts of the
// predicted range, or of a first digit of all keys, and k_select_finish collects the keys of the bin that holds the median;
// every other head's workgroups leave at once.  The first digit is made of the exponent and 6 mantissa bits (the squares of
// fp16 data span 83 binades, which at 64 bins each fit the 8192 bins of a workgroup's LDS).
// The sequence-sharded median further down is a plain most-significant-digit radix select on the 63 value bits.
#include <algorithm>

#include "hqmq_tables.h"

namespace hqmq {

namespace {

constexpr unsigned long long kKeyMask = 0x7fffffffffffffffull;
constexpr int kPickScratch = kSelectThreads / 64 + 4;

// Exclusive scan position of `rank` in a histogram: returns the bin holding the rank-th key
// (0-based) and how many keys lie in earlier bins.  Called by every thread of the block with the
// same arguments; `hist` may be global memory.  kBins is a multiple of the block size.
template <int kBins, int kBlock>
__device__ __forceinline__ void pick_bin(const uint32_t *hist, uint32_t rank, uint32_t *scratch /* LDS, kBlock / 64 + 2 */,
                                         uint32_t &bin_out, uint32_t &before_out)
{
    constexpr int kPer = kBins / kBlock;
    static_assert(kBins % kBlock == 0 && kBlock % 64 == 0, "bins must tile the block");
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    uint32_t local[kPer];
    uint32_t sum = 0;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        local[i] = hist[tid * kPer + i];
        sum += local[i];
    }
    // inclusive scan over the block: inside each wave, then wave totals through LDS
    const uint32_t inc = wave_scan(sum);
    if (lane == 63)
        scratch[wv] = inc;
    __syncthreads();
    uint32_t wave_before = 0;
    for (int k = 0; k < kBlock / 64; ++k)
        if (k < wv)
            wave_before += scratch[k];
    uint32_t before = wave_before + inc - sum;
    if (rank >= before && rank < before + sum) {
        bool found = false;
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            if (!found && rank < before + local[i]) {
                scratch[kBlock / 64] = tid * kPer + i;
                scratch[kBlock / 64 + 1] = before;
                found = true;
            }
            if (!found)
                before += local[i];
        }
    }
    __syncthreads();
    bin_out = scratch[kBlock / 64];
    before_out = scratch[kBlock / 64 + 1];
    __syncthreads();
}

// pick_bin for two ranks of one histogram, which ranks(n, a, b) sets from the number of keys in it.
template <int kBins, int kBlock, typename Ranks>
__device__ __forceinline__ void pick_two(const uint32_t *hist, Ranks ranks, uint32_t *scratch /* LDS, kBlock / 64 + 4 */, uint32_t &bin_a,
                                         uint32_t &before_a, uint32_t &bin_b, uint32_t &before_b)
{
    constexpr int kPer = kBins / kBlock, kW = kBlock / 64;
    static_assert(kBins % kBlock == 0, "bins must tile the block");
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    uint32_t local[kPer], sum = 0;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        local[i] = hist[tid * kPer + i];
        sum += local[i];
    }
    const uint32_t inc = wave_scan(sum);
    if (lane == 63)
        scratch[wv] = inc;
    __syncthreads();
    uint32_t before = inc - sum, n = 0, rank_a, rank_b;
#pragma unroll
    for (int k = 0; k < kW; ++k) {
        const uint32_t total = scratch[k];
        before += k < wv ? total : 0u;
        n += total;
    }
    ranks(n, rank_a, rank_b);
    if (rank_a - before < sum || rank_b - before < sum) {
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            if (rank_a - before < local[i]) {
                scratch[kW] = tid * kPer + i;
                scratch[kW + 1] = before;
            }
            if (rank_b - before < local[i]) {
                scratch[kW + 2] = tid * kPer + i;
                scratch[kW + 3] = before;
            }
            before += local[i];
        }
    }
    __syncthreads();
    bin_a = scratch[kW];
    before_a = scratch[kW + 1];
    bin_b = scratch[kW + 2];
    before_b = scratch[kW + 3];
    __syncthreads();
}

constexpr int kRankBits = 12, kRankBins = 1 << kRankBits;
constexpr int kFew = 64;  // keys that one wave ranks by counting
struct RankScratch {      // LDS
    unsigned long long few[kFew], result;
    uint32_t n_few, pick[kPickScratch];
};

// The key of the given rank (0-based) among those in [lo, hi] that each(f) passes to f, every thread its share; there are
// more than `rank` of them.  A histogram of 4096 equal parts of the range, then of the part that holds the rank, until few
// enough keys are left in it (keys spread evenly over the range: at once) or it is a single value.  Called by the whole
// workgroup; bins: LDS, kRankBins.
template <typename Each>
__device__ __forceinline__ unsigned long long select_rank(Each each, unsigned long long lo, unsigned long long hi, uint32_t rank,
                                                          uint32_t *bins, RankScratch &sc)
{
    const int tid = threadIdx.x;
    for (;;) {  // at most 6 rounds: each fixes 12 bits of the 63
        if (lo >= hi)
            return lo;
        const int width = 64 - __clzll((long long)(hi - lo));
        const int shift = width > kRankBits ? width - kRankBits : 0;
        for (int i = tid; i < kRankBins; i += kSelectThreads)
            bins[i] = 0;
        if (tid == 0)
            sc.n_few = 0;
        __syncthreads();
        each([&](unsigned long long key) {
            if (key - lo <= hi - lo)
                atomicAdd(&bins[(uint32_t)((key - lo) >> shift)], 1u);
        });
        __syncthreads();
        uint32_t bin, before;
        pick_bin<kRankBins, kSelectThreads>(bins, rank, sc.pick, bin, before);
        const uint32_t count = bins[bin];
        rank -= before;
        lo += (unsigned long long)bin << shift;
        const unsigned long long top = lo + ((1ull << shift) - 1ull);
        hi = top < hi ? top : hi;
        if (count <= (uint32_t)kFew && lo < hi) {
            each([&](unsigned long long key) {
                if (key - lo <= hi - lo)
                    sc.few[atomicAdd(&sc.n_few, 1u)] = key;
            });
            __syncthreads();
            if ((uint32_t)tid < count) {  // one wave
                const unsigned long long mine = sc.few[tid];
                uint32_t less = 0;
                for (uint32_t j = 0; j < count; ++j) {
                    const unsigned long long other = sc.few[j];
                    less += other < mine || (other == mine && j < (uint32_t)tid) ? 1u : 0u;
                }
                if (less == rank)
                    sc.result = mine;
            }
            __syncthreads();
            return sc.result;
        }
        __syncthreads();  // every thread has read its count
    }
}

}  // namespace

// First digit: exponent and 6 mantissa bits of r^2, offset so that the squares
// that fp16 data can produce (0, and 2^-48 up to below 2^35) fill bins 0 and 1..5312.  Monotone; bins
// 1..kBins0-2 each hold exactly the keys of one 17-bit prefix bin + kFineBase; bin 0 holds the keys
// below 2^-48 (for fp16 data: zero only), the last bin everything from 2^(kBins0-2)/64 binades up
// (never reached by finite fp16 data).
__device__ __forceinline__ uint32_t fine_bin(unsigned long long key)
{
    const uint32_t p = (uint32_t)(key >> kFineShift);
    const uint32_t d = p > kFineBase ? p - kFineBase : 0u;
    return min(d, (uint32_t)kBins0 - 1u);
}
__device__ __forceinline__ bool fine_bin_is_prefix(uint32_t bin) { return bin >= 1u && bin <= (uint32_t)kBins0 - 2u; }

// ---------------------------------------------------------------------------------------
// reset of the per-call state of head h: what the search's index counts in, or the operands of its matrix screen, and the
// caller's counters
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ void reset_head(const Geometry &g, const Workspace &ws, const EncodeTensor &tn, int h, int tid, int threads)
{
    const EncodedPtrs &enc = tn.enc;
    if (g.cell_n == 0)
        build_operands(g, ws, tn.sec, h, tid, threads);
    else
        for (int i = tid; i < 1 + g.cell_words; i += threads)
            cell_index_of(g, ws, h).n_groups[i] = 0;  // and the bits behind it
    if (tid == 0) {
        enc.n_outliers[h] = 0;
        if (h == 0) {
            enc.n_outliers[g.H] = 0;
            enc.status[0] = 0;
        }
    }
}

// Without a select: thresholds from the caller, or +infinity (nothing is flagged).  grid = (H, 1, tensors).
__global__ __launch_bounds__(kSelectThreads) void k_init(Geometry g, WorkspaceOffsets wo, EncodeBatch batch)
{
    const EncodeTensor &tn = batch.t[blockIdx.z];
    const Workspace ws = carve_workspace(tn.ws, wo);
    const int h = blockIdx.x;
    reset_head(g, ws, tn, h, threadIdx.x, kSelectThreads);
    if (threadIdx.x == 0)
        ws.thr[h] = tn.thr_given ? tn.thr_given[h] : __longlong_as_double(0x7ff0000000000000LL);
}

// Rows r, r + step, r + 2 step, ... of a head, those of all batch entries one after the other: where row r lies and how far it is
// from each to the next.  A step is so many whole entries and rows, and one entry more when the rows run over its end: the
// time of a step does not depend on T.  (One entry at a time, [1024, 8, 1, 128] took 49 us more.)
struct RowWalk {
    int64_t first, step, wrap;
    uint32_t t, rows;
    __device__ __forceinline__ RowWalk(const Geometry &g, uint32_t r, uint32_t by)
    {
        t = r;
        rows = by;
        first = (int64_t)r * g.st;
        step = (int64_t)by * g.st;
        wrap = 0;
        if (g.B > 1) {  // uniform
            const uint32_t T = (uint32_t)g.T, b = r / T, entries = by / T;
            t = r - b * T;
            rows = by - entries * T;
            wrap = g.sb - (int64_t)T * g.st;
            first += (int64_t)b * wrap;
            step += (int64_t)entries * wrap;
        }
    }
    __device__ __forceinline__ int64_t over_end(const Geometry &g)  // after each step, where there are entries
    {
        asm volatile("" : "+v"(t));  // a branch, not 16 more instructions per step for a call without entries (0.8 us of 15)
        t += rows;
        const bool over = t >= (uint32_t)g.T;
        t -= over ? (uint32_t)g.T : 0u;
        return over ? wrap : 0;
    }
};

// threshold on squares: fl(fl(C*C) * median), C widened from fp32
__device__ __forceinline__ double threshold_of(unsigned long long median_bits, float C)
{
    const double c = (double)C;
    const double c2 = c * c;
    return c2 * __longlong_as_double((long long)median_bits);
}

// ---------------------------------------------------------------------------------------
// A head of at most 1024 rows (of all batch entries one after the other) in one workgroup, its chunks in registers: a lane
// per chunk and 32 rows per step, all requested before the first is used.  A histogram of the squared norms in fp32 (exact
// squares, three rounded additions: within 3 * 2^-24 of the fp64 sum), exponent and 9 mantissa bits; the fp64 median lies in
// the bin that holds the rank, or within that error of its ends, and what is below the bin by more than twice the error is
// below the median: only the chunks in and 8 units around the bin (some 25 of 32768 smooth ones) get an fp64 norm, and a
// thread for each ranks them by counting.  More than 256 (values that repeat or lie close together): all norms in fp64, in
// registers, and select_rank between the least and the most of them.  Select of 8 tensors with 8 such heads of 1024 rows, in us,
// all norms in fp64 / fp32 and select_rank over the bin with norms taken again in each round / so: multiples of 1 48 / 59 / 39, of
// 1/4 25 / 33 / 26, constant 154 / 162 / 51, chunks of one norm 33 / 54 / 43.
// Bound by that compute unit's loads and latency: 10.6 us for 1024 rows of 128 elements, which a lane loads 16 bytes at a time
// (12.3 with 8), 6.2 for 256 and fewer; with every norm in fp64, a second histogram, addresses multiplied out per step and scans
// through LDS 17 and 8.7.
// grid = (H, 1, tensors), 1024 threads.
// ---------------------------------------------------------------------------------------
constexpr int kHeadBits = 9, kHeadShift = 23 - kHeadBits;
// fp32 exponents 79 (2^-48) to 162; bin 0: zero, the last: not finite.  Even, so that the bins on either side of a power of two,
// which hold all norms of unit chunks, are counted in two words.
constexpr uint32_t kHeadBase = (79u << kHeadBits) - 2u;
constexpr int kHeadBins = 84 << kHeadBits, kHeadWords = kHeadBins / 2;
constexpr int kHeadFew = 256;        // keys that are ranked by counting
constexpr uint32_t kHeadSlack = 8u;  // twice the error of a norm in fp32, in units of the last place
static_assert(kHeadRows * kChunksPerRow < 1 << 16, "two counters share a word");

template <int kSteps, bool kFull>
__global__ __launch_bounds__(kSelectThreads) void k_select_head(Geometry g, WorkspaceOffsets wo, EncodeBatch batch, float C)
{
    const EncodeTensor &tn = batch.t[blockIdx.z];
    const Workspace ws = carve_workspace(tn.ws, wo);
    const int h = blockIdx.x, tid = threadIdx.x, c = tid & 31, lane = tid & 63, wv = tid >> 6;
    constexpr int kPer = kHeadWords / kSelectThreads, kW = kSelectThreads / 64;
    static_assert(kHeadWords % kSelectThreads == 0 && kRankBins <= kHeadWords, "bins tile the block; the histograms share memory");
    __shared__ __align__(16) uint32_t hist[kHeadWords];
    __shared__ RankScratch sc;
    __shared__ unsigned long long few[kHeadFew];
    const uint32_t R = (uint32_t)g.B * (uint32_t)g.T;
    const bool active = kFull || c < g.n_c;
    half4_t v[kSteps];
    // kFull: two chunks of a row per load, 16 lanes to a row and 64 rows to two steps
    constexpr int kWide = kFull ? 2 : 1, kLanes = kChunksPerRow / kWide, kStepRows = kSelectThreads / kLanes;
    const uint32_t first_row = (uint32_t)tid / kLanes;
    {
        uint32_t r = first_row;
        const _Float16 *row = tn.x + (int64_t)h * g.sh;
        RowWalk walk(g, r, kStepRows);
        row += walk.first;
#pragma unroll
        for (int u = 0; u < kSteps; u += kWide) {
            v[u] = half4_t{0, 0, 0, 0};
            if (kFull) {
                v[u + kWide - 1] = v[u];
                if (r < R) {
                    typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
                    const half8_t two = *reinterpret_cast<const half8_t *>(row + 8 * (tid % kLanes));
                    v[u] = half4_t{two[0], two[1], two[2], two[3]};
                    v[u + kWide - 1] = half4_t{two[4], two[5], two[6], two[7]};
                }
            } else if (active && r < R) {
                v[u] = load_row_chunk<false>(row, c, g);
            }
            r += kStepRows;
            row += walk.step;
            if (g.B > 1)
                row += walk.over_end(g);
        }
    }
    for (int i = tid; i < kHeadWords / 4; i += kSelectThreads)
        reinterpret_cast<uint4 *>(hist)[i] = make_uint4(0u, 0u, 0u, 0u);
    if (tid == 0)
        sc.n_few = sc.result = 0;
    reset_head(g, ws, tn, h, tid, kSelectThreads);
    __syncthreads();
    uint32_t key[kSteps];
#pragma unroll
    for (int u = 0; u < kSteps; ++u) {
        const bool in = active && first_row + (uint32_t)(kStepRows * (u / kWide)) < R;
        const float x0 = (float)v[u][0], x1 = (float)v[u][1], x2 = (float)v[u][2], x3 = (float)v[u][3];
        key[u] = in ? __float_as_uint(fmaf(x3, x3, fmaf(x2, x2, fmaf(x1, x1, x0 * x0)))) & 0x7fffffffu : ~0u;
        if (in) {
            const uint32_t bin = min(max(key[u] >> kHeadShift, kHeadBase) - kHeadBase, (uint32_t)kHeadBins - 1u);
            atomicAdd(&hist[bin >> 1], 1u << (16u * (bin & 1u)));
        }
    }
    __syncthreads();
    const uint32_t rank = (R * (uint32_t)g.n_c - 1u) / 2u;
    uint32_t bin, below_bin;
    {
        uint32_t sum = 0;
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const uint32_t two = hist[tid * kPer + i];
            sum += (two & 0xffffu) + (two >> 16);
        }
        uint32_t before = wave_scan(sum);
        if (lane == 63)
            sc.pick[wv] = before;
        __syncthreads();
        before -= sum;
#pragma unroll
        for (int k = 0; k < kW; ++k)
            before += k < wv ? sc.pick[k] : 0u;
        if (rank - before < sum) {
            sc.pick[kW] = tid;
            sc.pick[kW + 1] = before;
        }
        __syncthreads();
        // every wave: a lane per bin of the thread whose bins hold the rank
        static_assert(2 * kPer <= 64, "a lane per bin");
        const int owner = (int)sc.pick[kW];
        const uint32_t two = hist[owner * kPer + min(lane >> 1, kPer - 1)];
        const uint32_t n = lane < 2 * kPer ? two >> (16 * (lane & 1)) & 0xffffu : 0u;
        const uint32_t first = sc.pick[kW + 1] + wave_scan(n) - n;
        const int at = __ffsll((unsigned long long)ballot(rank - first < n)) - 1;
        bin = (uint32_t)(2 * owner * kPer + at);
        below_bin = (uint32_t)__builtin_amdgcn_readlane((int)first, at);
    }
    unsigned long long median = bin == 0u ? 0ull : 0x7ff0000000000000ull;  // zeros; not finite
    if (bin != 0u && bin != (uint32_t)kHeadBins - 1u) {
        const uint32_t first = (bin + kHeadBase) << kHeadShift, f_lo = first - kHeadSlack;
        const uint32_t f_span = (1u << kHeadShift) - 1u + 2u * kHeadSlack;
#pragma unroll
        for (int u = 0; u < kSteps; ++u) {
            const bool near = key[u] - f_lo <= f_span;
            const unsigned long long mask = ballot(near);
            if (mask != 0ull) {  // one count per wave: a value may repeat in every chunk
                const uint32_t n = (uint32_t)__popcll(mask) | (uint32_t)__popcll(ballot(near && key[u] < first)) << 16;
                uint32_t at = 0;
                if (lane == 0)
                    at = atomicAdd(&sc.n_few, n);
                at = (__builtin_amdgcn_readfirstlane((int)at) & 0xffffu) +
                     __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
                if (near && at < (uint32_t)kHeadFew)
                    few[at] = key_of(chunk_norm2(v[u]));
            }
        }
        __syncthreads();
        const uint32_t count = sc.n_few & 0xffffu, left = rank - (below_bin - (sc.n_few >> 16));
        if (count <= (uint32_t)kHeadFew) {
            if ((uint32_t)tid < count) {
                const unsigned long long mine = few[tid];
                uint32_t less = 0;
#pragma unroll 4
                for (uint32_t j = 0; j < count; ++j) {
                    const unsigned long long other = few[j];
                    less += other < mine || (other == mine && j < (uint32_t)tid) ? 1u : 0u;
                }
                if (less == left)
                    sc.result = mine;
            }
            __syncthreads();
            median = sc.result;
        } else {
            // values that repeat: between the ends of what is there, a single value at once
            unsigned long long wide[kSteps], least_inverse = 0ull, most = 0ull;
#pragma unroll
            for (int u = 0; u < kSteps; ++u) {
                const bool near = key[u] - f_lo <= f_span;
                const unsigned long long k = key_of(chunk_norm2(v[u]));
                wide[u] = near ? k : ~0ull;  // outside every range of keys
                least_inverse = umax64(least_inverse, ~wide[u]);
                most = umax64(most, near ? k : 0ull);
            }
            least_inverse = wave_umax64(least_inverse);
            most = wave_umax64(most);
            __syncthreads();  // every thread has read the count, which select_rank clears
            if (lane == 0) {
                few[2 * wv] = least_inverse;
                few[2 * wv + 1] = most;
            }
            __syncthreads();
#pragma unroll
            for (int k = 0; k < kW; ++k) {
                least_inverse = umax64(least_inverse, few[2 * k]);
                most = umax64(most, few[2 * k + 1]);
            }
            median = select_rank(
                [&](auto f) {
#pragma unroll
                    for (int u = 0; u < kSteps; ++u)
                        f(wide[u]);
                },
                ~least_inverse, most, left, hist, sc);
        }
    }
    if (tid == 0)
        ws.thr[h] = threshold_of(median, C);
}

// ---------------------------------------------------------------------------------------
// Longer heads, prediction (and reset): one workgroup per head, beyond 2^18 chunks four and beyond 2^19 eight, bound by their
// compute unit's instructions and latency (8 us with 8 chunks per thread, 18 with 32: hence several).  The narrower range of
// more parts leaves the end of the candidate list to the box index.
// A workgroup's sample: pieces of 8 chunks (64 bytes) of 128 rows per step, so that chunks of one row, which are alike
// where the rows differ in scale, are few among it; every row's piece follows the one before, turned once more per round,
// at an odd stride of rows, so that structures of a power-of-two period in either direction do not alias with the sample.
// The parts of a head take the sampled rows in turn, and the turn goes round (each part once first, with one more step per
// round): a part that took every eighth would see two of a period's 16 rows only, and its ends, 1/8 of the average, moved the
// range past the median of heads with one row of 16 ten times smaller (select of two tensors with 8 such heads of 32768 rows 140
// us, 60 so).
// The range ends at the sample's ranks four standard deviations of a binomial count (sqrt(n) / 2 each) below and above its
// middle one, for n chunks of all parts, whose ends are averaged: the whole head's median falls outside it about once in
// 16000 heads of independent chunks.
// In fp32, which only a prediction may be: exponent and 8 mantissa bits (a bin holds about 0.2% of smooth data), the range
// widened by the rounding of the sum; 10 bits more where those two bins hold more than 1/64 of the sample.
// A head in one part keeps 4.7% of smooth data, in four 2.6%, in eight 1.85%; the lists hold at least 9.7, 4.8 and 2.4%.
// grid = (H, parts, tensors).
// ---------------------------------------------------------------------------------------
constexpr int kPredictBits = 8, kPredictShift = 23 - kPredictBits;
constexpr uint32_t kPredictBase = (79u << kPredictBits) - 1u;  // fp32 exponents 79 (2^-48) to 162; bin 0: zero
constexpr int kPredictBins = 84 << kPredictBits;
constexpr int kBuckets = 16;
constexpr int kBucketPitch = kBins1 / kBuckets;  // words between the counters: atomics to one line wait for each other
constexpr int kMaxParts = 8;
constexpr uint32_t kDenseBit = 1u << 31;  // sign of a part's lower end: the range holds a large share of the sample
__host__ __device__ __forceinline__ int predict_parts(const Geometry &g)
{
    const uint64_t n_h = (uint64_t)g.B * g.T * g.n_c;
    return n_h <= 1u << 18 ? 1 : n_h <= 1u << 19 ? 4 : kMaxParts;
}
__device__ __forceinline__ uint32_t *bucket_counts(const Workspace &ws, int h) { return ws.hist1 + (size_t)h * kBins1; }
__device__ __forceinline__ float2 *predicted_ends(const Workspace &ws, int h)  // between the first two counters
{
    return reinterpret_cast<float2 *>(ws.hist1 + (size_t)h * kBins1 + kBucketPitch / 2);
}

template <bool kFull>
__global__ __launch_bounds__(kSelectThreads) void k_select_predict(Geometry g, WorkspaceOffsets wo, EncodeBatch batch)
{
    const EncodeTensor &tn = batch.t[blockIdx.z];
    const Workspace ws = carve_workspace(tn.ws, wo);
    const int h = blockIdx.x, tid = threadIdx.x;
    __shared__ __align__(16) uint32_t hist[kPredictBins];
    __shared__ uint32_t pick[kPickScratch];
    constexpr int kSteps = 8, kPieceChunks = 8, kPieceRows = kSelectThreads / kPieceChunks;
    const uint32_t R = (uint32_t)g.B * (uint32_t)g.T;
    half4_t v[kSteps];
    uint32_t loaded = 0;  // a bit per step
    const uint32_t parts = gridDim.y, part = blockIdx.y;
    {
        const uint32_t samples = kPieceRows * kSteps * parts, stride = (R + samples - 1) / samples | 1u;
        const uint32_t pieces = (uint32_t)(g.n_c + kPieceChunks - 1) / kPieceChunks;
        const uint32_t inverse = ((1u << 20) + pieces - 1u) / pieces;  // i / pieces = i * inverse >> 20 for i below 2^12
        static_assert(kPieceRows * kSteps * 2 + kMaxParts < 1 << 12, "j + part + j / pieces");
        static_assert(kPieceRows % (kMaxParts * kMaxParts) == 0, "the turn of a thread's rows is the same in every step");
        uint32_t j = tid / kPieceChunks;
        const uint32_t turn = (part + j + (j >> (__ffs((int)parts) - 1))) & (parts - 1u);
        uint32_t r = (j * parts + turn) * stride;
        const uint32_t more = kPieceRows * parts * stride;
        const _Float16 *row = tn.x + (int64_t)h * g.sh;
        RowWalk walk(g, r, more);
        row += walk.first;
#pragma unroll
        for (int u = 0; u < kSteps; ++u) {
            const uint32_t i = j + part + (j * inverse >> 20);
            const uint32_t c = (i - (i * inverse >> 20) * pieces) * kPieceChunks + tid % kPieceChunks;
            v[u] = half4_t{0, 0, 0, 0};
            if (r < R && c < (uint32_t)g.n_c) {
                v[u] = load_row_chunk<kFull>(row, (int)c, g);
                loaded |= 1u << u;
            }
            j += kPieceRows;
            r += more;
            row += walk.step;
            if (g.B > 1)
                row += walk.over_end(g);
        }
    }
    if (part == 0) {
        reset_head(g, ws, tn, h, tid, kSelectThreads);
        for (int i = tid; i < kBins0; i += kSelectThreads)
            ws.hist0[(size_t)h * kBins0 + i] = 0;
        if (tid < kBuckets)
            bucket_counts(ws, h)[tid * kBucketPitch] = 0;
        if (tid == 0)
            ws.plan[h] = SelectPlan{0u, 0u, 0u, 0u, ~0ull, 0ull};
    }
    for (int i = tid; i < kPredictBins / 4; i += kSelectThreads)
        reinterpret_cast<uint4 *>(hist)[i] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    uint32_t key[kSteps];
    auto bin_of = [&](uint32_t k) { return min(max(k >> kPredictShift, kPredictBase) - kPredictBase, (uint32_t)kPredictBins - 1u); };
#pragma unroll
    for (int u = 0; u < kSteps; ++u) {
        const float x0 = (float)v[u][0], x1 = (float)v[u][1], x2 = (float)v[u][2], x3 = (float)v[u][3];
        key[u] = __float_as_uint(fmaf(x3, x3, fmaf(x2, x2, fmaf(x1, x1, x0 * x0)))) & 0x7fffffffu;
        if ((loaded >> u) & 1u)
            atomicAdd(&hist[bin_of(key[u])], 1u);
    }
    __syncthreads();
    uint32_t rank_lo, rank_hi, n, bin_lo, bin_hi, before_lo, before_hi;
    pick_two<kPredictBins, kSelectThreads>(
        hist,
        [&](uint32_t total, uint32_t &a, uint32_t &b) {
            const uint32_t mid = (total - 1) / 2, margin = (uint32_t)(2.0f * sqrtf((float)total / (float)parts)) + 2u;
            n = total;
            a = rank_lo = mid > margin ? mid - margin : 0u;
            b = rank_hi = min(total - 1, mid + margin);
        },
        pick, bin_lo, before_lo, bin_hi, before_hi);
    uint32_t f_lo = bin_lo == 0u ? 0u : (bin_lo + kPredictBase) << kPredictShift;
    uint32_t f_hi = bin_hi == 0u ? 0u : ((bin_hi + kPredictBase) << kPredictShift) | ((1u << kPredictShift) - 1u);
    const uint32_t n_lo = hist[bin_lo];
    bool dense = false;
    if (n_lo + hist[bin_hi] > n / 64u) {  // uniform: concentrated or coarse data
        __syncthreads();
        for (int i = tid; i < 2 * kBins1; i += kSelectThreads)
            hist[i] = 0;
        __syncthreads();
        constexpr int kSubShift = kPredictShift - kBits1;
#pragma unroll
        for (int u = 0; u < kSteps; ++u) {
            if ((loaded >> u) & 1u) {
                const uint32_t bin = bin_of(key[u]), digit = (key[u] >> kSubShift) & (kBins1 - 1);
                if (bin == bin_lo)
                    atomicAdd(&hist[digit], 1u);
                if (bin == bin_hi)
                    atomicAdd(&hist[kBins1 + digit], 1u);
            }
        }
        __syncthreads();
        uint32_t sub_lo, sub_hi, before;
        pick_two<2 * kBins1, kSelectThreads>(
            hist,
            [&](uint32_t, uint32_t &a, uint32_t &b) {
                a = rank_lo - before_lo;
                b = n_lo + rank_hi - before_hi;
            },
            pick, sub_lo, before, sub_hi, before);
        // a range holds no more than a few per cent of the sample besides what shares the parts at its ends
        dense = 8u * (hist[sub_lo] + hist[sub_hi]) > 3u * n;
        if (bin_lo != 0u)
            f_lo |= sub_lo << kSubShift;
        if (bin_hi != 0u)
            f_hi = f_hi >> kPredictShift << kPredictShift | (sub_hi & (kBins1 - 1)) << kSubShift | ((1u << kSubShift) - 1u);
        // a sample that holds one value between the two ranks: that value alone (a constant or coarsely quantised tensor,
        // whose squares are exact in fp32: its keys need no list)
        uint32_t least = 0xffffffffu, most = 0u;
#pragma unroll
        for (int u = 0; u < kSteps; ++u) {
            if (((loaded >> u) & 1u) && key[u] >= f_lo && key[u] <= f_hi) {
                least = min(least, key[u]);
                most = max(most, key[u]);
            }
        }
        if (tid == 0) {
            pick[0] = 0xffffffffu;
            pick[1] = 0u;
        }
        __syncthreads();
        if (least <= most) {
            atomicMin(&pick[0], least);
            atomicMax(&pick[1], most);
        }
        __syncthreads();
        if (pick[0] == pick[1])
            f_lo = f_hi = pick[0];
    }
    if (tid == 0) {
        if (f_lo != f_hi) {  // three roundings of 2^-24 each: 4 units of the last place on either side
            f_lo = f_lo <= 4u ? 0u : f_lo - 4u;
            f_hi += 4u;
        }
        predicted_ends(ws, h)[part] = make_float2(__uint_as_float(f_lo | (dense ? kDenseBit : 0u)), __uint_as_float(f_hi));
    }
}

// The kept keys' lists: 16 equal parts of the range of values (of bit patterns, the parts above a power of two would hold
// twice what those below it do).
__device__ __forceinline__ uint32_t bucket_capacity(const Geometry &g) { return (uint32_t)g.cand_room / kBuckets; }
struct Buckets {
    unsigned long long lo, span;  // keys
    float scale, first, last;     // their values
    bool dense;                   // wanted by many of the chunks
    __device__ __forceinline__ Buckets(const Geometry &g, const Workspace &ws, int h)
    {
        // sums over the parts in pairs, so that equal ends sum up exactly
        const int n = predict_parts(g), lane = threadIdx.x & 63;
        const float2 own = lane < n ? predicted_ends(ws, h)[lane] : make_float2(0.0f, 0.0f);
        dense = ballot((__float_as_uint(own.x) & kDenseBit) != 0u) != 0ull;
        auto sum8 = [](float v) {  // of the first eight lanes
            v += dpp_move<0xb1>(v);   // neighbours
            v += dpp_move<0x4e>(v);   // pairs
            v += dpp_move<0x141>(v);  // fours: the half row mirrored
            return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
        };
        static_assert(kMaxParts == 8, "a part per lane of the sum");
        // exact, if the parts agree on a single value; else their ends are 4 units of the last place wide
        first = sum8(fabsf(own.x)) * (1.0f / (float)n);
        last = sum8(own.y) * (1.0f / (float)n);
        lo = key_of((double)first);
        span = key_of((double)last) - lo;
        scale = (float)kBuckets / (last - first);  // not used for a single value
    }
    __device__ __forceinline__ bool holds(unsigned long long key) const { return key - lo <= span; }
    __device__ __forceinline__ uint32_t of(unsigned long long key) const  // monotone in key
    {
        const double past = __longlong_as_double((long long)key) - __longlong_as_double((long long)lo);
        return min((uint32_t)((float)past * scale), (uint32_t)kBuckets - 1u);
    }
};

// What the sweep counted for a head, a list per lane: requested together with the range, not after it.
struct KeptCounts {
    uint32_t below, mine;
    __device__ __forceinline__ KeptCounts(const Workspace &ws, int h)
        : below(ws.plan[h].below), mine((threadIdx.x & 63) < kBuckets ? bucket_counts(ws, h)[(threadIdx.x & 63) * kBucketPitch] : 0u)
    {
    }
};

// Where the key of the given rank is among the kept ones: its list and its rank there.  False: not at all, because it lies
// outside the predicted range, or inside but its list overflowed (a range of one value needs none).
__device__ __forceinline__ bool find_kept(const Geometry &g, const KeptCounts &kept, const Buckets &range, uint32_t rank,
                                          uint32_t &bucket, uint32_t &rank_in, uint32_t &n, bool &inside)
{
    const uint32_t below = kept.below, mine = kept.mine;
    const int lane = threadIdx.x & 63;  // every wave for itself
    const uint32_t inc = wave_scan(mine);
    const unsigned long long past = ballot(lane < kBuckets && rank >= below && rank - below < inc);
    inside = past != 0ull;
    if (!inside)
        return false;
    bucket = (uint32_t)__ffsll((long long)past) - 1u;
    n = (uint32_t)__builtin_amdgcn_readlane((int)mine, (int)bucket);
    rank_in = rank - below - ((uint32_t)__builtin_amdgcn_readlane((int)inc, (int)bucket) - n);
    return n <= bucket_capacity(g) || range.span == 0ull;
}

// What the histogram of a head whose kept keys do not answer is made of: equal parts of the predicted range's bit patterns
// where the wanted key lies in it, else, and where the range starts at zero (whose pattern is far from all others), the
// first digit of every key.
struct SecondLook {
    unsigned long long lo, span;
    int shift;
    bool linear;
    __device__ __forceinline__ SecondLook(const Buckets &range, bool inside)
        : lo(range.lo), span(range.span), linear(inside && range.lo != 0ull)
    {
        const int width = 64 - __clzll((long long)(span | 1ull));
        shift = width > kBits0 ? width - kBits0 : 0;
    }
    __device__ __forceinline__ bool counts(unsigned long long key) const { return !linear || key - lo <= span; }
    __device__ __forceinline__ uint32_t bin_of(unsigned long long key) const
    {
        return linear ? (uint32_t)((key - lo) >> shift) : fine_bin(key);
    }
    __device__ __forceinline__ uint32_t rank_of(uint32_t rank, uint32_t below) const { return linear ? rank - below : rank; }
    // Whether the bin's keys have to be looked at; else the key is `known`.
    __device__ __forceinline__ bool bounds(uint32_t bin, unsigned long long &first, unsigned long long &last,
                                           unsigned long long &known) const
    {
        if (linear) {
            first = lo + ((unsigned long long)bin << shift);
            last = first + ((1ull << shift) - 1ull);
            return true;
        }
        known = bin == 0u ? 0ull : 0x7ff0000000000000ull;  // zeros; beyond finite fp16 data (not reached)
        first = (unsigned long long)(bin + kFineBase) << kFineShift;
        last = first | ((1ull << kFineShift) - 1ull);
        return fine_bin_is_prefix(bin);
    }
};

// The sweep: keys below the predicted range are counted, those in it kept, staged in LDS so that a workgroup updates each
// list's counter once.  Norms in fp32 tell nearly all chunks apart; what may be in the range waits in a queue of the wave for its
// key in fp64.  Two [1, 8, 32768, 128] tensors with the smallest index beside it in 29 us, 4.6 TB/s, one of 131072 rows in 47, 5.7
// (all keys in fp64: 31 and 53; with no arithmetic but the norms 24 and 42).
// Where most chunks are wanted the queue only adds to the work.  Two values of norms and nothing else / half zeros / two close
// values in 40 of 100 chunks, all queued up and all not, us: those two tensors 63, 56 / 60, 55 / 44, 36; two [1, 8, 16384, 96]
// 32, 28 / 31, 28 / 24, 25; the long one 121, 99 / 110, 97 / 94, 105; in 25 of 100 chunks 34, 34 / 20, 25 / 66, 92.
// A thread has eight loads of 16 bytes (rows of 128 elements) or of a chunk in flight, next to one another over the rows.
// kCells: workgroups in between build the search's box index, which needs the secondaries only, while the others wait for
// their rows; a quarter of the sweep's alternates with them, eight by eight (one for each XCD), the rest follows (half, three
// quarters, all: within 1 %).  The two launches one after the other / together / together with the norms in fp32, in us:
// 16 heads of 32768 rows, S = 256, 51 / 43 / 37; 8 heads of 131072, 76 / 58 / 50; 64 heads of 8192 rows of 96 elements, S = 192,
// 81 / 74 / 68 (bound by VALU issue); 4 heads of 3074 rows of 100, S = 96, 23 / 14 / 13.
// `rows` of one (b, h) segment per workgroup; grid: cell_blocks() * H * n_tensors, rounded up to 8, and ceil(T / rows) * B * H *
// n_tensors, likewise.
constexpr int kCountThreads = kCellThreads;
constexpr int kCountRows = 512;  // of a workgroup, at most
constexpr int kStageKeys = 144;  // keys a workgroup stages per list
constexpr int kQueue = 256;      // chunks a wave queues up
constexpr int kStageDense = kStageKeys + kCountThreads / 64 * kQueue / kBuckets;  // where no wave has a queue
struct CountStage {              // LDS
    union {
        struct {
            unsigned long long staged[kBuckets][kStageKeys];
            uint2 queue[kCountThreads / 64][kQueue];  // of each wave: chunks whose keys are wanted
        };
        // Two values of norms in 128 rows of 12 elements fill 192 places of two lists: sweep of 8 heads of 20000 such rows 12 us
        // with fewer, 8 with these.
        unsigned long long dense[kBuckets][kStageDense];
    };
    uint32_t n_staged[kBuckets], n_below;            // n_staged: all keys of the list, also those past the stage
    uint32_t n_direct[kBuckets], full[kBuckets];     // those of them that the list's counter has; the list is full
};
template <bool kFull, bool kCells>
__global__ __launch_bounds__(kCountThreads, 6) void k_select_count(Geometry g, WorkspaceOffsets wo, EncodeBatch batch, int rows,
                                                                uint32_t n_tensors)
{
    constexpr size_t kLds = kCells && sizeof(CellBuild) > sizeof(CountStage) ? sizeof(CellBuild) : sizeof(CountStage);
    __shared__ __align__(16) unsigned char lds[kLds];
    uint32_t block = blockIdx.x, tensor;
    if (kCells) {
        const uint32_t per_head = (uint32_t)cell_blocks(g), n_cells = n_tensors * (uint32_t)g.H * per_head;
        const uint32_t cells8 = (n_cells + 7u) / 8u, rows8 = (gridDim.x - 8u * cells8) / 8u;
        const uint32_t beside = rows8 / 4u, mixed = cells8 + beside;  // the sweep's that alternate with the build's
        const uint32_t i = block / 8u;
        const uint32_t rows_before = i < mixed ? (uint32_t)((uint64_t)i * beside / mixed) : i - cells8;
        if (i < mixed && (uint32_t)((uint64_t)(i + 1u) * beside / mixed) == rows_before) {
            block = 8u * (i - rows_before) + (block & 7u);
            if (block >= n_cells)
                return;
            const uint32_t head = block / per_head;
            tensor = head / (uint32_t)g.H;
            const EncodeTensor &tn = batch.t[tensor];
            build_cells(g, carve_workspace(tn.ws, wo), tn.sec, (int)(head - tensor * (uint32_t)g.H), (int)(block - head * per_head),
                        *reinterpret_cast<CellBuild *>(lds));
            return;
        }
        block = 8u * rows_before + (block & 7u);
    }
    const uint32_t per_seg = (uint32_t)(g.T + rows - 1) / (uint32_t)rows, per_tensor = per_seg * (uint32_t)(g.B * g.H);
    tensor = block / per_tensor;
    if (kCells && tensor >= n_tensors)
        return;
    block -= tensor * per_tensor;
    const EncodeTensor &tn = batch.t[tensor];
    const Workspace ws = carve_workspace(tn.ws, wo);
    CountStage &st = *reinterpret_cast<CountStage *>(lds);
    const int seg = (int)(block / per_seg), b = seg / g.H, h = seg % g.H;
    const int t0 = (int)(block - (uint32_t)seg * per_seg) * rows, n_rows = min(rows, g.T - t0);
    const _Float16 *base = tn.x + (int64_t)b * g.sb + (int64_t)h * g.sh + (int64_t)t0 * g.st;
    const Buckets range(g, ws, h);
    const uint32_t cap = bucket_capacity(g);
    unsigned long long *lists = ws.cand + (size_t)h * g.cand_cap;
    uint32_t *count = bucket_counts(ws, h);
    const int tid = threadIdx.x;
    if (tid < kBuckets)
        st.n_staged[tid] = st.n_direct[tid] = st.full[tid] = 0;
    if (tid == 0)
        st.n_below = 0;
    __syncthreads();
    // Keys past the stage go straight to their list: one update of its counter for all of a wave's, and none once the list is
    // full (a tensor that repeats a value a hundred thousand times would queue up at one counter: 28 ns each).
    auto append = [&](uint32_t k, unsigned long long key) {
        const int lane = tid & 63;
        for (unsigned long long left = __ballot(1); left;) {  // uniform over the lanes that are here
            const int leader = __ffsll((long long)left) - 1;
            const uint32_t k0 = (uint32_t)__shfl((int)k, leader, 64);
            const unsigned long long same = __ballot(k == k0);
            left &= ~same;
            const uint32_t n = (uint32_t)__popcll(same);
            uint32_t at = 0;
            if (lane == leader) {
                at = atomicAdd(&count[k0 * kBucketPitch], n);
                atomicAdd(&st.n_direct[k0], n);
                if (at + n > cap)
                    st.full[k0] = 1u;
            }
            at = (uint32_t)__shfl((int)at, leader, 64) + (uint32_t)__popcll(same & ((1ull << lane) - 1ull));
            if (k == k0 && at < cap)
                lists[k * cap + at] = key;
        }
    };
    // A squared norm in fp32 differs from the fp64 one by at most 3 * 2^-24 of it: below the range or above it by more than that it
    // needs no other.  The rest, some 5 in 100 chunks, queue up until a wave has 64, which then get their keys together.
    const float under = range.first * (1.0f - 0x1p-21f), over = range.last * (1.0f + 0x1p-21f);
    const bool single = range.span == 0ull;  // uniform; a range of one value: its keys may be all there are, and only their number counts
    const int lane = tid & 63;
    uint2 *queue = st.queue[tid / 64];
    const bool wide = !kFull && range.dense;  // rows of 128 elements fill any number
    const uint32_t stage = wide ? kStageDense : kStageKeys;
    auto staged = [&](uint32_t k, uint32_t pos) -> unsigned long long & { return wide ? st.dense[k][pos] : st.staged[k][pos]; };
    uint32_t below = 0, equal = 0, queued = 0;  // of the wave
    auto keep = [&](const half4_t v, bool in) {
        const unsigned long long key = key_of(chunk_norm2(v)) & kKeyMask;
        below += (uint32_t)__popcll(ballot(in && key < range.lo));
        if (in && range.holds(key)) {
            const uint32_t k = range.of(key), pos = atomicAdd(&st.n_staged[k], 1u);
            if (pos < stage)
                staged(k, pos) = key;
            else if (!*(volatile uint32_t *)&st.full[k])
                append(k, key);
        }
    };
    auto keep_queued = [&](uint32_t n) {        // the last n, at most 64
        wave_lds_sync();
        queued -= n;
        const bool mine = (uint32_t)lane < n;
        keep(__builtin_bit_cast(half4_t, queue[mine ? queued + lane : 0u]), mine);
        wave_lds_sync();
    };
    // Queues up a wave's chunks whose keys are wanted; false, and nothing done, if they don't fit.  A chunk of infinities (what
    // lanes without one have) is above every range.
    auto take = [&](const half4_t v) {
        const float x0 = (float)v[0], x1 = (float)v[1], x2 = (float)v[2], x3 = (float)v[3];
        const float r2 = fmaf(x3, x3, fmaf(x2, x2, fmaf(x1, x1, x0 * x0)));
        const unsigned long long less = ballot(r2 < under);
        unsigned long long wanted = ballot(r2 <= over) & ~less;
        const bool fits = queued + (uint32_t)__popcll(wanted) <= (uint32_t)kQueue;
        wanted = fits ? wanted : 0ull;
        below += fits ? (uint32_t)__popcll(less) : 0u;
        if (of_mask(wanted))
            queue[queued + __builtin_amdgcn_mbcnt_hi((uint32_t)(wanted >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)wanted, 0u))] =
                __builtin_bit_cast(uint2, v);
        queued += (uint32_t)__popcll(wanted);
        return fits;
    };
    auto take_single = [&](const half4_t v) {
        const unsigned long long key = key_of(chunk_norm2(v)) & kKeyMask;
        below += (uint32_t)__popcll(ballot(key < range.lo));
        equal += (uint32_t)__popcll(ballot(key == range.lo));
    };
    const _Float16 inf = __builtin_bit_cast(_Float16, (uint16_t)0x7c00);
    const half4_t none = {inf, inf, inf, inf};
    // Empties the queue, and keeps what it had no room for, again from memory, four in flight.  (Emptied at each of the places where
    // it may be full, the code of that alone was 25 KB.)
    auto settle = [&](uint32_t left, auto again) {
        while (queued >= 64u)  // uniform, as the next
            keep_queued(64u);
        while (left) {
            half4_t v[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                v[k] = left ? again(__ffs((int)left) - 1) : none;
                left &= left - 1u;  // 0 stays 0
            }
#pragma unroll 1
            for (int k = 0; k < 4; ++k) {
                keep(v[0], true);
                v[0] = v[1], v[1] = v[2], v[2] = v[3];
            }
        }
    };
    // A wave takes the keys of all chunks at once, none of them queued, where the prediction's sample says that three in eight are
    // wanted, or from the step on after one that left three of eight loads over.  A loop for each way: inside one loop the other
    // ways cost the usual one 2 % of the sweep.
    constexpr int kLoads = 8, kMany = 3;
    if (kFull) {
        typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
        constexpr int kPieces = kChunksPerRow / 2, kStep = kCountThreads / kPieces;  // 16-byte pieces of a row, rows per load
        const _Float16 *at = base + (int64_t)(tid / kPieces) * g.st + 8 * (tid % kPieces);
        int r0 = 0;
        auto steps = [&](auto f) {  // until f says no
            for (bool more = true; more && r0 < n_rows; r0 += kLoads * kStep, at += (int64_t)(kLoads * kStep) * g.st) {  // uniform
                half8_t two[kLoads];
                if (r0 + kLoads * kStep <= n_rows) {  // uniform
#pragma unroll
                    for (int u = 0; u < kLoads; ++u)
                        two[u] = *reinterpret_cast<const half8_t *>(at + (int64_t)(kStep * u) * g.st);
                } else {
#pragma unroll
                    for (int u = 0; u < kLoads; ++u) {
                        two[u] = half8_t{inf, inf, inf, inf, inf, inf, inf, inf};
                        if (r0 + tid / kPieces + kStep * u < n_rows)
                            two[u] = *reinterpret_cast<const half8_t *>(at + (int64_t)(kStep * u) * g.st);
                    }
                }
                more = f([&](int i) {
                    const half8_t v = two[i >> 1];
                    return i & 1 ? half4_t{v[4], v[5], v[6], v[7]} : half4_t{v[0], v[1], v[2], v[3]};
                });
            }
        };
        if (single) {
            steps([&](auto chunk) {
#pragma unroll
                for (int i = 0; i < 2 * kLoads; ++i)
                    take_single(chunk(i));
                return true;
            });
        } else {
            if (!range.dense)
                steps([&](auto chunk) {
                    uint32_t left = 0;
#pragma unroll
                    for (int i = 0; i < 2 * kLoads; ++i)
                        left |= take(chunk(i)) ? 0u : 1u << i;
                    settle(left, [&](int i) {
                        const int r = kStep * (i >> 1);
                        return r0 + tid / kPieces + r < n_rows ? load_chunk(at + (int64_t)r * g.st + 4 * (i & 1)) : none;
                    });
                    return __popc(left) < 2 * kMany;
                });
            steps([&](auto chunk) {
#pragma unroll
                for (int i = 0; i < 2 * kLoads; ++i)
                    keep(chunk(i), true);
                return true;
            });
        }
    } else {
        const int n_chunks = n_rows * g.n_c;
        auto load = [&](int q) {
            if (q >= n_chunks)
                return none;
            const int r = row_of_chunk(q, g);
            return load_row_chunk<false>(base + (int64_t)r * g.st, q - r * g.n_c, g);
        };
        int q0 = 0;
        auto steps = [&](auto f) {  // as above
            for (bool more = true; more && q0 < n_chunks; q0 += kLoads * kCountThreads) {  // uniform
                half4_t v[kLoads];
#pragma unroll
                for (int u = 0; u < kLoads; ++u)
                    v[u] = load(q0 + u * kCountThreads + tid);
                more = f([&](int u) { return v[u]; });
            }
        };
        if (single) {
            steps([&](auto chunk) {
#pragma unroll
                for (int u = 0; u < kLoads; ++u)
                    take_single(chunk(u));
                return true;
            });
        } else {
            if (!range.dense)
                steps([&](auto chunk) {
                    uint32_t left = 0;
#pragma unroll
                    for (int u = 0; u < kLoads; ++u)
                        left |= take(chunk(u)) ? 0u : 1u << u;
                    settle(left, [&](int i) { return load(q0 + i * kCountThreads + tid); });
                    return __popc(left) < kMany;
                });
            steps([&](auto chunk) {
#pragma unroll
                for (int u = 0; u < kLoads; ++u)
                    keep(chunk(u), true);
                return true;
            });
        }
    }
    if (queued)
        keep_queued(queued);
    if (lane == 0) {
        atomicAdd(&st.n_below, below);
        if (equal)
            atomicAdd(&st.n_staged[0], equal);
    }
    __syncthreads();
    if (range.span == 0ull) {
        if (tid == 0 && st.n_staged[0])
            atomicAdd(&count[0], st.n_staged[0]);
    } else {
        // a thread per list takes the places (with those that a full list made nobody append), a wave at a time fills them
        if (tid < kBuckets && st.n_staged[tid])
            st.full[tid] = atomicAdd(&count[tid * kBucketPitch], st.n_staged[tid] - st.n_direct[tid]);
        __syncthreads();
        for (int k = tid / 64; k < kBuckets; k += kCountThreads / 64) {
            const uint32_t n = min(st.n_staged[k], stage), at = st.full[k];
            for (uint32_t i = tid & 63; i < n; i += 64)
                if (at + i < cap)
                    lists[k * cap + at + i] = staged(k, i);
        }
    }
    if (tid == 0 && st.n_below)
        atomicAdd(&ws.plan[h].below, st.n_below);
}

// ---------------------------------------------------------------------------------------
// Workgroups that share the rows of a head whose kept keys do not answer (of all batch entries one after the other).  Every other
// head's return at once, but for the first in k_select_digit, which selects; but their launch takes time too: 512 workgroups in
// all, at least 4 for a long head and at most one per 256 rows.  (16 per head: the two launches took 42 us instead of 14 for 512
// heads of 1400 rows, and 287 instead of 77 where 8 heads of 131072 were missed, on half the chip.)
// ---------------------------------------------------------------------------------------
static int missed_parts(const Geometry &g, unsigned n_tensors)
{
    const uint64_t heads = (uint64_t)g.H * n_tensors, rows = (uint64_t)g.B * g.T;
    uint64_t parts = (512 + heads - 1) / heads;
    if (rows >= 8192 && parts < 4)
        parts = 4;
    const uint64_t most = rows / 256 < 64 ? rows / 256 : 64;  // 4 and more: these heads have over 1024 rows
    return (int)(parts < most ? parts : most);
}
// f of the key of every chunk of the rows [first, last) of head h, a lane per chunk, 128 rows per step in flight; after each
// step, then() by the whole workgroup.
constexpr int kStepRows = 128;
template <bool kFull, typename F, typename Then>
__device__ __forceinline__ void each_key(const Geometry &g, const _Float16 *x, int h, uint32_t first, uint32_t last, F f, Then then)
{
    const int c = threadIdx.x & 31;
    for (uint32_t at = first; at < last; at += kStepRows) {  // uniform
        const uint32_t r0 = at + (threadIdx.x >> 5);
        half4_t v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t r = r0 + 32u * u, b = r / (uint32_t)g.T, t = r - b * (uint32_t)g.T;
            v[u] = half4_t{0, 0, 0, 0};
            if (r < last)
                v[u] = load_row_chunk<kFull>(x + (int64_t)b * g.sb + (int64_t)h * g.sh + (int64_t)t * g.st, c, g);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if ((kFull || c < g.n_c) && r0 + 32u * u < last)
                f(key_of(chunk_norm2(v[u])) & kKeyMask);
        then();
    }
}
template <bool kFull, typename F>
__device__ __forceinline__ void each_key(const Geometry &g, const _Float16 *x, int h, uint32_t first, uint32_t last, F f)
{
    each_key<kFull>(g, x, h, first, last, f, [] {});
}
// The head of a workgroup.  Workgroups go to the eight XCDs in turn and there to the 32 compute units in turn: the next head
// for the next part, and one more after every 256 workgroups, so that neither the first parts of all heads nor the parts of
// one head share an XCD or a compute unit (64 parts of one head: 187 us for the call's select on half the compute units, 140).
__device__ __forceinline__ int missed_head(const Geometry &g, uint32_t part)
{
    return (int)((blockIdx.x + part + gridDim.x * gridDim.y * part / 256u) % (uint32_t)g.H);
}
__device__ __forceinline__ void part_of_rows(const Geometry &g, uint32_t part, uint32_t parts, uint32_t &first, uint32_t &last)
{
    const uint64_t R = (uint64_t)g.B * g.T;
    first = (uint32_t)(R * part / parts);
    last = (uint32_t)(R * (part + 1) / parts);
}

// The key of the given rank of a list of n kept keys, by one workgroup; bins: LDS, kRankBins.
__device__ __forceinline__ unsigned long long select_kept(const unsigned long long *list, uint32_t n, uint32_t rank, const Buckets &range,
                                                          uint32_t *bins, RankScratch &sc)
{
    const int tid = threadIdx.x;
    constexpr int kHeld = 8;  // keys per thread that stay in registers
    if (range.span == 0ull)
        return range.lo;
    if (n <= kHeld * kSelectThreads) {
        unsigned long long key[kHeld];
#pragma unroll
        for (int u = 0; u < kHeld; ++u)
            key[u] = u * kSelectThreads + tid < n ? list[u * kSelectThreads + tid] : ~0ull;  // outside every range of keys
        return select_rank(
            [&](auto f) {
#pragma unroll
                for (int u = 0; u < kHeld; ++u)
                    if (u * kSelectThreads < n)  // uniform
                        f(key[u]);
            },
            range.lo, range.lo + range.span, rank, bins, sc);
    }
    return select_rank(
        [&](auto f) {
            for (uint32_t i = tid; i < n; i += kSelectThreads)
                f(list[i]);
        },
        range.lo, range.lo + range.span, rank, bins, sc);
}

// For a head whose kept keys hold the wanted rank, the first workgroup selects from their list; for any other, all of them make
// the histogram.  The box index that was built beside the sweep is finished in the same launch (finish_parts workgroups of every
// head; 0 without an index), beside the selection: with that in k_select_finish, which now has nothing left to do for such a
// head, the encode of two [1, 8, 32768, 128] tensors took 178.6 us instead of 176.2, of one [2, 4, 1537, 100] 43.5 instead of 40.3.
// kFinishFirst: these come first, where all workgroups lie beside one another, two per compute unit (that last tensor's encode 40.7,
// 41.0 with them last); else last, so that those of missed heads keep their places (the launch in us, 16 missed heads of 32768
// rows alike within a row: 24.4 with them first, 17.0 so; half zero rows 41, 40).
// Two per compute unit take at most 96 scalar registers per wave, hence the launch bound (100 left it one: 32 instead of 26 for
// 16 heads in steps of 1/8, 92 instead of 73 for 8 heads of 131072 rows, half of them zero).
// Writes thr[h] = fl(fl(C*C) * median).  grid = (H, tensors, missed_parts() + finish_parts).
template <bool kFull, bool kFinishFirst>
__global__ __launch_bounds__(kSelectThreads, 8) void k_select_digit(Geometry g, WorkspaceOffsets wo, EncodeBatch batch,
                                                                    uint32_t finish_parts, float C)
{
    const EncodeTensor &tn = batch.t[blockIdx.y];
    const Workspace ws = carve_workspace(tn.ws, wo);
    __shared__ uint32_t hist[kBins0];
    __shared__ RankScratch sc;
    static_assert(kRankBins <= kBins0, "the histograms share their memory");
    static_assert(kFinishThreads == kSelectThreads && kFinishWords <= kBins0, "the same workgroup and memory");
    const uint32_t parts = gridDim.z - finish_parts, part = blockIdx.z - (kFinishFirst ? finish_parts : 0u);
    if (kFinishFirst ? blockIdx.z < finish_parts : part >= parts) {  // uniform
        const int h = blockIdx.x;
        const CellIndex ix = cell_index_of(g, ws, h);
        finish_cells<true>(g, ws, reinterpret_cast<const float4_t *>(tn.sec) + (size_t)h * g.S, h, (int)(kFinishFirst ? blockIdx.z : part - parts), (int)finish_parts,
                                   CellPlaces{ix.list, reinterpret_cast<uint2 *>(ix.head), ix.id, ix.function}, hist);
        return;
    }
    const int h = missed_head(g, part);
    uint32_t bucket, rank_in, n, first, last;
    bool inside;
    const KeptCounts kept(ws, h);
    const Buckets range(g, ws, h);
    if (find_kept(g, kept, range, (uint32_t)(((uint64_t)g.B * g.T * g.n_c - 1) / 2), bucket, rank_in, n, inside)) {  // uniform
        if (part != 0)
            return;
        const unsigned long long median =
            select_kept(ws.cand + (size_t)h * g.cand_cap + bucket * bucket_capacity(g), n, rank_in, range, hist, sc);
        if (threadIdx.x == 0) {
            ws.thr[h] = threshold_of(median, C);
            ws.plan[h].selected = 1u;
        }
        return;
    }
    const SecondLook look(range, inside);
    for (int i = threadIdx.x; i < kBins0; i += kSelectThreads)
        hist[i] = 0;
    __syncthreads();
    part_of_rows(g, part, parts, first, last);
    each_key<kFull>(g, tn.x, h, first, last, [&](unsigned long long key) {
        if (look.counts(key))
            atomicAdd(&hist[look.bin_of(key)], 1u);
    });
    __syncthreads();
    for (int i = threadIdx.x; i < kBins0; i += kSelectThreads)
        if (hist[i])
            atomicAdd(&ws.hist0[(size_t)h * kBins0 + i], hist[i]);
}

// ---------------------------------------------------------------------------------------
// finish, for a head without a list that holds the wanted rank: all of its workgroups collect the keys of the histogram's bin that
// holds it, and the last of them to end selects among these.  If they were too many, the bin mostly holds a single value (a
// coarsely quantised tensor), which is the median; else the last workgroup selects among the head's raw rows: slow, exact, and
// only for such inputs.
// A call with heads that were missed (16 heads of 2^20 chunks, 8 of 2^22): 30 and 60 us more, with a list that overflowed 75 and
// 120, with half the keys of one value 165 and 290.
// Writes thr[h] = fl(fl(C*C) * median).  grid = (H, tensors, missed_parts()).
// ---------------------------------------------------------------------------------------
constexpr int kVmcnt0 = 0x0f70;  // s_waitcnt vmcnt(0), the other counters at their largest
template <bool kFull>
__global__ __launch_bounds__(kSelectThreads) void k_select_finish(Geometry g, WorkspaceOffsets wo, EncodeBatch batch,
                                                                  float C)
{
    const EncodeTensor &tn = batch.t[blockIdx.y];
    const Workspace ws = carve_workspace(tn.ws, wo);
    // the keys staged for the candidate list, which takes them when there are more than kStaged after a step
    constexpr int kStaged = 4096;
    __shared__ unsigned long long staged[kStaged + kStepRows * kChunksPerRow];
    uint32_t *const bins = reinterpret_cast<uint32_t *>(staged);
    static_assert(kRankBins * sizeof(uint32_t) <= sizeof(staged), "the histograms share their memory");
    __shared__ RankScratch sc;
    __shared__ unsigned long long least, most;
    __shared__ uint32_t n_staged, list_at, arrived;
    const int h = missed_head(g, blockIdx.z), tid = threadIdx.x;
    uint32_t rank = (uint32_t)(((uint64_t)g.B * g.T * g.n_c - 1) / 2);
    unsigned long long *cand = ws.cand + (size_t)h * g.cand_cap;
    const bool selects = blockIdx.z == 0;  // the workgroups that start first
    // done by k_select_digit: one scalar load, not all that find_kept looks at (0.9 us of those 40.3)
    if (*(const __attribute__((address_space(4))) uint32_t *)(uintptr_t)&ws.plan[h].selected)
        return;
    unsigned long long median;
    const KeptCounts kept(ws, h);
    const Buckets range(g, ws, h);
    uint32_t bucket, rank_in, n;
    bool inside;
    (void)find_kept(g, kept, range, rank, bucket, rank_in, n, inside);
    SelectPlan &plan = ws.plan[h];
    const SecondLook look(range, inside);
    uint32_t bin, before;
    unsigned long long lo, hi;
    rank = look.rank_of(rank, plan.below);
    pick_bin<kBins0, kSelectThreads>(ws.hist0 + (size_t)h * kBins0, rank, sc.pick, bin, before);
    rank -= before;
    if (!look.bounds(bin, lo, hi, median)) {
        if (!selects)
            return;
    } else {
        if (tid == 0) {
            least = ~0ull;
            most = 0ull;
            n_staged = 0u;
        }
        __syncthreads();
        uint32_t first, last;
        part_of_rows(g, blockIdx.z, gridDim.z, first, last);
        unsigned long long my_least = ~0ull, my_most = 0ull;
        auto flush = [&] {  // by the whole workgroup
            __syncthreads();
            if (tid == 0)
                list_at = atomicAdd(&plan.n_cand, n_staged);
            __syncthreads();
            for (uint32_t i = tid; i < n_staged; i += kSelectThreads)
                if (list_at + i < (uint32_t)g.cand_room)
                    cand[list_at + i] = staged[i];
            __syncthreads();
            if (tid == 0)
                n_staged = 0u;
            __syncthreads();
        };
        each_key<kFull>(
            g, tn.x, h, first, last,
            [&](unsigned long long key) {
                if (look.counts(key) && look.bin_of(key) == bin) {
                    my_least = key < my_least ? key : my_least;
                    my_most = key > my_most ? key : my_most;
                    staged[atomicAdd(&n_staged, 1u)] = key;
                }
            },
            [&] {
                __syncthreads();
                if (n_staged > (uint32_t)kStaged)  // uniform: nobody adds before flush's barrier or the next
                    flush();
                else
                    __syncthreads();
            });
        flush();
        if (my_least <= my_most) {
            atomicMin(&least, my_least);
            atomicMax(&most, my_most);
        }
        __syncthreads();
        if (tid == 0 && least <= most) {
            atomicMin(&plan.least, least);
            atomicMax(&plan.most, most);
        }
        // The list and its ends before the arrival: every wave waits for its own stores, then one thread makes the whole
        // workgroup's visible (a fence by each of the 16 waves writes the L2 back 16 times: 200 us for 512 workgroups).
        __builtin_amdgcn_s_waitcnt(kVmcnt0);
        __syncthreads();
        if (tid == 0) {
            __threadfence();
            arrived = atomicAdd(&plan.n_done, 1u);
        }
        __syncthreads();
        if (arrived != gridDim.z - 1u)
            return;
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        n = __hip_atomic_load(&plan.n_cand, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        lo = __hip_atomic_load(&plan.least, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        hi = __hip_atomic_load(&plan.most, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (n <= (uint32_t)g.cand_room)
            median = select_rank(
                [&](auto f) {
                    for (uint32_t i = tid; i < n; i += kSelectThreads)
                        f(cand[i]);
                },
                lo, hi, rank, bins, sc);
        else  // at once where lo == hi
            median = select_rank([&](auto f) { each_key<kFull>(g, tn.x, h, 0u, (uint32_t)g.B * (uint32_t)g.T, f); }, lo, hi, rank,
                                 bins, sc);
    }
    if (tid == 0)
        ws.thr[h] = threshold_of(median, C);
}

// ---------------------------------------------------------------------------------------
// outlier bookkeeping after the search kernel has written the flag words, the per-row offsets local to its workgroup (of
// search_rows rows) and the workgroup totals:
//   k_gather  adds the totals of the workgroups before a row's to its offset and copies the flagged chunks into the outlier
//             list in ascending linear chunk order; per-head totals, grand total and status on the way
//   k_scan    before it where workgroups are many: exclusive scan of the totals (linear row order), per-head totals, status
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(1024) void k_scan(Geometry g, WorkspaceOffsets wo, EncodeBatch batch,
                                               uint32_t n_blocks, uint64_t n_rows)
{
    const EncodeTensor &tn = batch.t[blockIdx.z];
    const Workspace ws = carve_workspace(tn.ws, wo);
    const EncodedPtrs enc = tn.enc;
    const uint64_t outlier_capacity = tn.outlier_capacity;
    __shared__ uint32_t wave_tot[16];
    __shared__ uint32_t carry_s;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const uint32_t blocks_per_seg = g.n_search_blocks_per_seg;
    if (threadIdx.x == 0)
        carry_s = 0;
    __syncthreads();
    for (uint32_t start = 0; start < n_blocks; start += 1024) {
        const uint32_t i = start + threadIdx.x;
        const uint32_t v = (i < n_blocks) ? ws.block_sum[i] : 0;
        uint32_t inc = v;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            uint32_t o = __shfl_up(inc, d, 64);
            if (lane >= d)
                inc += o;
        }
        if (lane == 63)
            wave_tot[wv] = inc;
        __syncthreads();
        uint32_t wave_before = 0, all = 0;
        for (int k = 0; k < 16; ++k) {
            const uint32_t wt = wave_tot[k];
            if (k < wv)
                wave_before += wt;
            all += wt;
        }
        const uint32_t carry = carry_s;
        if (i < n_blocks)
            ws.block_pre[i] = carry + wave_before + inc - v;
        __syncthreads();
        if (threadIdx.x == 0)
            carry_s = carry + all;
        __syncthreads();
    }
    const uint32_t total = carry_s;
    // per-head totals from the prefix array: a head's workgroups are contiguous inside each batch
    // entry's segment (the block's own global writes are visible to it after the barriers above)
    for (uint32_t h = threadIdx.x; h < (uint32_t)g.H; h += 1024) {
        uint32_t sum = 0;
        for (uint32_t b = 0; b < (uint32_t)g.B; ++b) {
            const uint32_t first = (b * (uint32_t)g.H + h) * blocks_per_seg, last = first + blocks_per_seg;
            const uint32_t hi = (last < n_blocks) ? ws.block_pre[last] : total;
            sum += hi - ws.block_pre[first];
        }
        enc.n_outliers[h] = sum;
    }
    if (threadIdx.x == 0) {
        enc.n_outliers[g.H] = total;
        enc.row_off[n_rows] = total;
        if ((uint64_t)total > outlier_capacity)
            atomicOr(enc.status, HQMQ_STATUS_OUTLIER_OVERFLOW);  // next to what the search may have reported
    }
}

// kOwnPrefix: no k_scan before it; every workgroup sums the totals of the search workgroups before its rows itself, and the
// first of a head, and the last of all, write what else k_scan would.  Taken up to kOwnPrefixBlocks, eight loads per thread,
// and while all workgroups together sum at most kOwnPrefixSums totals: own prefix / scan in us, 8 heads each: 16 tensors of
// 32768 rows (2^23) 112 / 123, 2 of 256 batch entries of 32 rows (2^23) 11 / 34, 32 of 32768 rows of 4 elements (2^25) 43 / 29.
// 256 rows per workgroup, a thread per row, four of its outliers in flight.  Bound by the latency of its loads: 7.5 us for
// two [1, 8, 32768, 128] tensors (11.5 with k_scan before it and one outlier at a time), 29 instead of 39 at 5% outliers.
// grid = (ceil(T / 256), B*H, tensors).
constexpr uint32_t kOwnPrefixBlocks = 2048;
constexpr uint64_t kOwnPrefixSums = 1ull << 24;
// This thread's share of the sum of the n totals v[at(0)], v[at(1)], ..., four requested before the first is used.
template <typename At>
__device__ __forceinline__ uint32_t sum_of(const uint32_t *v, uint32_t n, At at)
{
    uint32_t sum = 0;
    for (uint32_t i0 = threadIdx.x; i0 < n; i0 += 4 * kThreads) {
        uint32_t part[4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            part[u] = i0 + u * kThreads < n ? v[at(i0 + u * kThreads)] : 0u;
        sum += part[0] + part[1] + part[2] + part[3];
    }
    return sum;
}
template <bool kFull, bool kOwnPrefix>
__global__ __launch_bounds__(kThreads) void k_gather(Geometry g, WorkspaceOffsets wo, EncodeBatch batch, uint32_t n_blocks)
{
    const EncodeTensor &tn = batch.t[blockIdx.z];
    const Workspace ws = carve_workspace(tn.ws, wo);
    const EncodedPtrs enc = tn.enc;
    const uint64_t outlier_capacity = tn.outlier_capacity;
    __shared__ uint32_t sums[2], starts[64];
    const int tid = threadIdx.x, lane = tid & 63;
    const int seg = blockIdx.y, b = seg / g.H, h = seg % g.H;
    const int t = blockIdx.x * kThreads + tid;
    const int64_t R = (int64_t)seg * g.T + t;
    const bool in = t < g.T;
    uint32_t word = in ? enc.flags[R] : 0u;
    uint32_t off = in ? enc.row_off[R] : 0u;
    const uint32_t per_seg = g.n_search_blocks_per_seg;
    const uint32_t block = (uint32_t)seg * per_seg + (uint32_t)min(t, g.T - 1) / g.search_rows;
    if (kOwnPrefix) {
        // everything that is read is requested before the first use
        const uint32_t first = (uint32_t)seg * per_seg + blockIdx.x * (uint32_t)kThreads / g.search_rows;
        const bool last = blockIdx.x == gridDim.x - 1 && blockIdx.y == gridDim.y - 1;
        // the totals of the search workgroups of these rows: one of 256 rows and more, up to 32 of 8
        const uint32_t n_own = g.search_rows >= kThreads ? 1u : (uint32_t)kThreads / g.search_rows;
        const uint32_t own = (uint32_t)tid < n_own && first + tid < n_blocks ? ws.block_sum[first + tid] : 0u;
        uint32_t before = sum_of(ws.block_sum, first, [](uint32_t i) { return i; });
        uint32_t of_head = 0;
        const bool counts = blockIdx.x == 0 && b == 0;  // uniform
        if (counts)  // of all batch entries: H per_seg apart
            of_head = sum_of(ws.block_sum, (uint32_t)g.B * per_seg, [&](uint32_t i) {
                const uint32_t bb = i / per_seg;
                return (bb * ((uint32_t)g.H - 1u) + (uint32_t)h) * per_seg + i;
            });
        if (tid == 0)
            sums[0] = sums[1] = 0;
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) {
            before += __shfl_xor(before, d, 64);
            of_head += __shfl_xor(of_head, d, 64);
        }
        if (tid < 64)  // one wave: where each search workgroup's outliers start behind those before `first`; own is 0 past n_own
            starts[tid] = wave_scan(own);
        __syncthreads();
        if (lane == 0) {
            atomicAdd(&sums[0], before);
            atomicAdd(&sums[1], of_head);
        }
        __syncthreads();
        off += sums[0] + (block > first ? starts[block - first - 1] : 0u);
        if (tid == 0) {
            if (counts)
                enc.n_outliers[h] = sums[1];
            if (last) {
                const uint32_t total = sums[0] + starts[63];
                enc.n_outliers[g.H] = total;
                enc.row_off[R - t + g.T] = total;
                if ((uint64_t)total > outlier_capacity)
                    atomicOr(enc.status, HQMQ_STATUS_OUTLIER_OVERFLOW);  // next to what the search may have reported
            }
        }
    } else {
        off += ws.block_pre[block];
    }
    if (in)
        enc.row_off[R] = off;
    const _Float16 *row = tn.x + (int64_t)b * g.sb + (int64_t)h * g.sh + (int64_t)t * g.st;
    uint64_t pos = off;
    while (word) {
        half4_t v[4];
        const int n = min(__popc(word), 4);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (u < n)
                v[u] = load_row_chunk<kFull>(row, __ffs((int)word) - 1, g);
            word &= word - 1;  // 0 stays 0
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (u < n && pos + u < outlier_capacity)
                *reinterpret_cast<uint2 *>(enc.outliers + 4 * (pos + u)) = __builtin_bit_cast(uint2, v[u]);
        pos += n;
    }
}

// The outlier list of a small tensor whose search ran in its fused form (no kernel before it): one
// workgroup per tensor does what k_scan and k_gather do, and what k_init would have done for them:
//   scan    exclusive scan of the search workgroups' totals (at most kSmallListBlocks of them, one per
//           thread), per-head totals, grand total, status word (overflow; non-finite input, which the search
//           workgroups report in bit 31 of their totals)
//   gather  every row adds its workgroup's prefix to its offset and copies its flagged chunks
// grid = (1, 1, tensors), 1024 threads.
template <bool kFull>
__global__ __launch_bounds__(1024) void k_list_small(Geometry g, WorkspaceOffsets wo, EncodeBatch batch)
{
    const EncodeTensor &tn = batch.t[blockIdx.z];
    const Workspace ws = carve_workspace(tn.ws, wo);
    const EncodedPtrs enc = tn.enc;
    const uint64_t outlier_capacity = tn.outlier_capacity;
    const _Float16 *__restrict__ x = tn.x;
    __shared__ uint32_t pre[kSmallListBlocks + 1];  // exclusive prefix of the workgroup totals, then the grand total
    __shared__ uint32_t wave_tot[16];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const uint32_t blocks_per_seg = g.n_search_blocks_per_seg;
    const uint32_t n_blocks = (uint32_t)g.B * g.H * blocks_per_seg;  // <= kSmallListBlocks (checked by the host)
    const uint32_t n_rows = (uint32_t)g.B * g.H * g.T;
    // the first round of rows: flag word and local offset requested together with the workgroup totals
    uint32_t word0 = 0, off0 = 0;
    if ((uint32_t)tid < n_rows) {
        word0 = enc.flags[tid];
        off0 = enc.row_off[tid];
    }
    const uint32_t raw = (uint32_t)tid < n_blocks ? ws.block_sum[tid] : 0u;
    const uint32_t v = raw & 0x7fffffffu;
    const int bad = __syncthreads_or((int)(raw >> 31));
    uint32_t inc = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        uint32_t o = __shfl_up(inc, d, 64);
        if (lane >= d)
            inc += o;
    }
    if (lane == 63)
        wave_tot[wv] = inc;
    __syncthreads();
    uint32_t wave_before = 0, total = 0;
    for (int k = 0; k < 16; ++k) {
        const uint32_t wt = wave_tot[k];
        if (k < wv)
            wave_before += wt;
        total += wt;
    }
    if ((uint32_t)tid < n_blocks)
        pre[tid] = wave_before + inc - v;
    if (tid == 0)
        pre[n_blocks] = total;
    __syncthreads();
    for (uint32_t h = tid; h < (uint32_t)g.H; h += 1024) {
        uint32_t sum = 0;
        for (uint32_t b = 0; b < (uint32_t)g.B; ++b) {
            const uint32_t first = (b * (uint32_t)g.H + h) * blocks_per_seg;
            sum += pre[first + blocks_per_seg] - pre[first];
        }
        enc.n_outliers[h] = sum;
    }
    if (tid == 0) {
        enc.n_outliers[g.H] = total;
        enc.row_off[n_rows] = total;
        enc.status[0] = ((uint64_t)total > outlier_capacity ? HQMQ_STATUS_OUTLIER_OVERFLOW : 0u) |
                        (bad ? HQMQ_STATUS_NONFINITE : 0u);
    }
    for (uint32_t R = tid; R < n_rows; R += 1024) {
        const uint32_t seg = R / (uint32_t)g.T, t = R - seg * (uint32_t)g.T;
        const uint32_t b = seg / (uint32_t)g.H, h = seg - b * (uint32_t)g.H;
        uint32_t word = R == (uint32_t)tid ? word0 : enc.flags[R];
        const uint32_t off = (R == (uint32_t)tid ? off0 : enc.row_off[R]) +
                             pre[seg * blocks_per_seg + t / (uint32_t)g.search_rows];
        enc.row_off[R] = off;
        const _Float16 *row = x + (int64_t)b * g.sb + (int64_t)h * g.sh + (int64_t)t * g.st;
        uint64_t pos = off;
        while (word) {
            const int c = __ffs((int)word) - 1;
            word &= word - 1;
            if (pos < outlier_capacity)
                *reinterpret_cast<uint2 *>(enc.outliers + 4 * pos) =
                    __builtin_bit_cast(uint2, load_row_chunk<kFull>(row, c, g));
            ++pos;
        }
    }
}

// ---------------------------------------------------------------------------------------
// The median of a head whose token axis is split over several shards (a context-parallel cache: every
// shard holds a slice of T; paper Sec. 3 takes the median per (layer, head, role) over the whole
// batch).  Plain most-significant-digit radix select with histograms only, so that the one thing the
// shards have to exchange is a histogram: pass 0 counts bits 62..50 of every key, passes 1..5 the
// next 10 bits of the keys under the prefix fixed so far; the caller sums the pass's histogram over
// the shards before the next call, and every shard then takes the same decisions.
//   k_shard_pick   one workgroup per head: (pass > 0) locates the wanted rank in the summed histogram
//                  of the previous pass and extends the prefix; clears the histogram of this pass;
//                  (finish) writes the threshold fl(fl(C C) median)
//   k_shard_hist   sweep of this shard's rows
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ int shard_digit_bits(int pass) { return pass == 0 ? kBits0 : kBits1; }
__device__ __forceinline__ int shard_digit_shift(int pass) { return pass == 0 ? kShift0 : kShift1 - 10 * (pass - 1); }

// pass: the pass about to run (0..5), or 6 = finish.
__global__ __launch_bounds__(kSelectThreads) void k_shard_pick(Geometry g, WorkspaceOffsets wo, EncodeBatch batch,
                                                               int pass, unsigned long long total_per_head, float C)
{
    const EncodeTensor &tn = batch.t[blockIdx.z];
    const Workspace ws = carve_workspace(tn.ws, wo);
    __shared__ uint32_t scratch[kPickScratch];
    const int h = blockIdx.x;
    unsigned long long prefix = 0;
    uint32_t rank = (uint32_t)((total_per_head - 1) / 2);
    if (pass > 0) {
        prefix = ws.state[h].prefix;
        rank = ws.state[h].rank;
        uint32_t bin, before;
        if (pass == 1)
            pick_bin<kBins0, kSelectThreads>(ws.hist0 + (size_t)h * kBins0, rank, scratch, bin, before);
        else
            pick_bin<kBins1, kSelectThreads>(ws.hist1 + (size_t)h * kBins1, rank, scratch, bin, before);
        prefix = (prefix << shard_digit_bits(pass - 1)) | bin;
        rank -= before;
    }
    if (pass < 6) {
        uint32_t *hist = pass == 0 ? ws.hist0 + (size_t)h * kBins0 : ws.hist1 + (size_t)h * kBins1;
        const int bins = pass == 0 ? kBins0 : kBins1;
        for (int i = threadIdx.x; i < bins; i += kSelectThreads)
            hist[i] = 0;  // after pick_bin's barriers: every thread has read the previous counts
    }
    if (threadIdx.x == 0) {
        ws.state[h].prefix = prefix;
        ws.state[h].rank = rank;
        if (pass == 6) {
            ws.thr[h] = threshold_of(prefix, C);  // all 63 bits fixed: the median itself
        }
    }
}

template <bool kFull>
__global__ __launch_bounds__(kSelectThreads) void k_shard_hist(Geometry g, WorkspaceOffsets wo, EncodeBatch batch, int pass)
{
    const EncodeTensor &tn = batch.t[blockIdx.z];
    const Workspace ws = carve_workspace(tn.ws, wo);
    const _Float16 *__restrict__ x = tn.x;
    __shared__ uint32_t lh[kBins0];
    const int seg = blockIdx.y, b = seg / g.H, h = seg % g.H;
    const int bins = pass == 0 ? kBins0 : kBins1;
    const int shift = shard_digit_shift(pass), nbits = shard_digit_bits(pass);
    const unsigned long long prefix = ws.state[h].prefix;  // pass 0: zero, and every key matches
    for (int i = threadIdx.x; i < bins; i += kSelectThreads)
        lh[i] = 0;
    __syncthreads();
    const int c = threadIdx.x & 31, sub = threadIdx.x >> 5;
    const int t0 = blockIdx.x * kSelectRows;
    const int t1 = min(g.T, t0 + kSelectRows);
    const _Float16 *base = x + (int64_t)b * g.sb + (int64_t)h * g.sh;
    if (kFull || c < g.n_c) {
        for (int t = t0 + sub; t < t1; t += kSelectThreads / 32) {
            const unsigned long long key =
                key_of(chunk_norm2(load_row_chunk<kFull>(base + (int64_t)t * g.st, c, g))) & kKeyMask;
            // (key >> 63) == 0 == prefix in pass 0; a shift by shift + nbits <= 63 is always defined
            if ((key >> (shift + nbits)) == prefix)
                atomicAdd(&lh[(uint32_t)(key >> shift) & (uint32_t)(bins - 1)], 1u);
        }
    }
    __syncthreads();
    uint32_t *gh = pass == 0 ? ws.hist0 + (size_t)h * kBins0 : ws.hist1 + (size_t)h * kBins1;
    for (int i = threadIdx.x; i < bins; i += kSelectThreads) {
        const uint32_t n = lh[i];
        if (n)
            atomicAdd(&gh[i], n);
    }
}

hipError_t launch_shard_median_pass(const Geometry &g, const WorkspaceOffsets &wo, const EncodeBatch &batch, int pass,
                                    unsigned long long total_per_head, float C, hipStream_t stream)
{
    hipLaunchKernelGGL(k_shard_pick, dim3(g.H, 1, 1), dim3(kSelectThreads), 0, stream, g, wo, batch, pass,
                       total_per_head, C);
    if (pass < 6) {
        dim3 grid((g.T + kSelectRows - 1) / kSelectRows, g.B * g.H, 1);
        if (g.D == 4 * kChunksPerRow)
            hipLaunchKernelGGL(k_shard_hist<true>, grid, dim3(kSelectThreads), 0, stream, g, wo, batch, pass);
        else
            hipLaunchKernelGGL(k_shard_hist<false>, grid, dim3(kSelectThreads), 0, stream, g, wo, batch, pass);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// host-side launch sequences
// ---------------------------------------------------------------------------------------
template <bool kFull>
static void launch_select_for(const Geometry &g, const WorkspaceOffsets &wo, const EncodeBatch &batch, unsigned n, float C,
                              hipStream_t stream)
{
    const dim3 heads(g.H, 1, n), samples(g.H, predict_parts(g), n), block(kSelectThreads);
    const uint64_t head_rows = (uint64_t)g.B * g.T;
    if (head_rows <= 256) {
        hipLaunchKernelGGL((k_select_head<8, kFull>), heads, block, 0, stream, g, wo, batch, C);
        return;
    }
    if (head_rows <= (uint64_t)kHeadRows) {
        hipLaunchKernelGGL((k_select_head<32, kFull>), heads, block, 0, stream, g, wo, batch, C);
        return;
    }
    const dim3 parts(g.H, n, missed_parts(g, n));
    hipLaunchKernelGGL(k_select_predict<kFull>, samples, block, 0, stream, g, wo, batch);
    int rows = kCountRows;  // down to the 128 of one step while four workgroups per compute unit are not there
    while (rows > 128 && (uint64_t)((g.T + rows - 1) / rows) * g.B * g.H * n < 1024)
        rows /= 2;
    // Its workgroups lie along one axis, whose threads have to stay below 2^32: that leaves room for 130,000 heads with an index of
    // 125 workgroups each, fewer than 32 tensors may have (one tensor's always fit: at most 65535 heads, 2^27 rows).
    const uint32_t cells = g.cell_n > 0 ? (uint32_t)(cell_blocks(g) * g.H) : 0u;                    // of a tensor
    const uint32_t sweep = (uint32_t)((g.T + rows - 1) / rows) * (uint32_t)(g.B * g.H);
    const unsigned most = (0xffffffffu / (unsigned)kCountThreads - 16u) / (cells + sweep);
    EncodeBatch rest = batch;
    for (unsigned first = 0; first < n; first += most) {
        const unsigned m = n - first < most ? n - first : most;
        if (first > 0)
            std::copy(batch.t + first, batch.t + first + m, rest.t);
        if (g.cell_n > 0)
            hipLaunchKernelGGL((k_select_count<kFull, true>), dim3((cells * m + 7) / 8 * 8 + (sweep * m + 7) / 8 * 8), dim3(kCountThreads),
                               0, stream, g, wo, rest, rows, m);
        else
            hipLaunchKernelGGL((k_select_count<kFull, false>), dim3(sweep * m), dim3(kCountThreads), 0, stream, g, wo, rest, rows, m);
    }
    // Workgroups that finish a head's index: a step of theirs is 1024 of its 24 S codewords and of up to 5120 list groups, and
    // all heads' lie beside one another, two per compute unit.  The launch in us by 1 / 2 / 4 / 8 of them, heads of 4100 rows: S = 256:
    // 8 heads 8.4 / 5.7 / 5.2 / 5.3, 64 heads 10.6 / 7.8 / 7.3 / 7.2, 128 heads 11.0 / 10.0 / 9.0 / 10.2, 256 heads 15.2 / 14.2 / 15.5 /
    // 18.0; S = 64: 16 heads 6.4 / 5.8 / 5.7 / 5.8, 256 heads 9.9 / 10.2 / 11.6 / 14.5; S = 16: 16 heads 5.4 / 5.9 / 5.3 / 5.7, 128
    // heads 6.0 / 6.0 / 7.1 / 8.5.
    const uint32_t heads_all = n * (uint32_t)g.H;
    const uint32_t finish_parts = g.cell_n == 0 ? 0u : std::max(1u, std::min({(uint32_t)(g.S + 31) / 32u, 512u / heads_all, kFinishParts}));
    const dim3 all(g.H, n, parts.z + finish_parts);
    if (heads_all * all.z <= 512u)
        hipLaunchKernelGGL((k_select_digit<kFull, true>), all, block, 0, stream, g, wo, batch, finish_parts, C);
    else
        hipLaunchKernelGGL((k_select_digit<kFull, false>), all, block, 0, stream, g, wo, batch, finish_parts, C);
    hipLaunchKernelGGL(k_select_finish<kFull>, parts, block, 0, stream, g, wo, batch, C);
}

hipError_t launch_select_median(const Geometry &g, const WorkspaceOffsets &wo, const EncodeBatch &batch, int n_tensors,
                                float C, bool skip_select, hipStream_t stream)
{
    const unsigned n = (unsigned)n_tensors;
    if (skip_select)
        hipLaunchKernelGGL(k_init, dim3(g.H, 1, n), dim3(kSelectThreads), 0, stream, g, wo, batch);
    else if (g.D == 4 * kChunksPerRow)
        launch_select_for<true>(g, wo, batch, n, C, stream);
    else
        launch_select_for<false>(g, wo, batch, n, C, stream);
    return hipGetLastError();
}

hipError_t launch_outlier_list_small(const Geometry &g, const WorkspaceOffsets &wo, const EncodeBatch &batch,
                                     int n_tensors, hipStream_t stream)
{
    const dim3 grid(1, 1, (unsigned)n_tensors);
    if (g.D == 4 * kChunksPerRow)
        hipLaunchKernelGGL(k_list_small<true>, grid, dim3(1024), 0, stream, g, wo, batch);
    else
        hipLaunchKernelGGL(k_list_small<false>, grid, dim3(1024), 0, stream, g, wo, batch);
    return hipGetLastError();
}

hipError_t launch_outlier_list(const Geometry &g, const WorkspaceOffsets &wo, const EncodeBatch &batch, int n_tensors,
                               hipStream_t stream)
{
    const unsigned n = (unsigned)n_tensors;
    const uint32_t n_blocks = (uint32_t)g.B * g.H * g.n_search_blocks_per_seg;
    const uint64_t n_rows = (uint64_t)g.B * g.H * g.T;
    const bool full = g.D == 4 * kChunksPerRow;
    const dim3 grid((g.T + kThreads - 1) / kThreads, g.B * g.H, n);
    if (n_blocks <= kOwnPrefixBlocks && (uint64_t)n * grid.x * grid.y * n_blocks <= kOwnPrefixSums) {
        if (full)
            hipLaunchKernelGGL((k_gather<true, true>), grid, dim3(kThreads), 0, stream, g, wo, batch, n_blocks);
        else
            hipLaunchKernelGGL((k_gather<false, true>), grid, dim3(kThreads), 0, stream, g, wo, batch, n_blocks);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_scan, dim3(1, 1, n), dim3(1024), 0, stream, g, wo, batch, n_blocks, n_rows);
    if (full)
        hipLaunchKernelGGL((k_gather<true, false>), grid, dim3(kThreads), 0, stream, g, wo, batch, n_blocks);
    else
        hipLaunchKernelGGL((k_gather<false, false>), grid, dim3(kThreads), 0, stream, g, wo, batch, n_blocks);
    return hipGetLastError();
}

}  // namespace hqmq
