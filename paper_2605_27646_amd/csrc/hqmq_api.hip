// C ABI of the HQMQ library (declared in include/hqmq.h): argument validation, workspace
// carve-up and the stream-ordered kernel sequences.  No allocation, no synchronisation.
#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstring>
#include <mutex>

#include "hqmq_device.h"

namespace hqmq {

static thread_local int32_t g_last_hip_error = 0;

}  // namespace hqmq

// Workspace of hqmq_encode_static, for callers that cannot allocate: every GPU the library runs on holds
// its own copy of this array, at its own address, until the process ends.  Host code never uses the
// array's name as an address: the per-device set-up below asks the runtime for it.
static __device__ __align__(256) unsigned char scratch[HQMQ_STATIC_SCRATCH_BYTES];

namespace hqmq {

// Per-device set-up, done once: the search kernels' LDS limit and the device address of `scratch`.  The flag
// of a device is set only after its set-up succeeded, so a failed attempt is retried by the next call;
// devices beyond the table are set up on every call.
constexpr int kMaxDevices = 64;
static std::atomic<bool> g_device_ready[kMaxDevices];
static void *g_scratch_ptr[kMaxDevices];  // written before the device's flag is set, read after it is seen
static std::mutex g_setup_mutex;

// scratch_out: null, or receives the current device's address of the static scratch array.
static hipError_t ensure_device_setup(void **scratch_out = nullptr)
{
    int device = 0;
    hipError_t err = hipGetDevice(&device);
    if (err != hipSuccess)
        return err;
    const bool tracked = device >= 0 && device < kMaxDevices;
    if (!(tracked && g_device_ready[device].load(std::memory_order_acquire))) {
        std::lock_guard<std::mutex> lock(g_setup_mutex);
        if (!(tracked && g_device_ready[device].load(std::memory_order_relaxed))) {
            err = prepare_search_kernels();
            if (err == hipSuccess)
                err = prepare_attend_kernels();
            if (err != hipSuccess)
                return err;
            void *ptr = nullptr;
            err = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
            if (err != hipSuccess)
                return err;
            if (!ptr)
                return hipErrorInvalidSymbol;
            if (!tracked) {  // nowhere to keep it: hand it out and set up again next time
                if (scratch_out)
                    *scratch_out = ptr;
                return hipSuccess;
            }
            g_scratch_ptr[device] = ptr;
            g_device_ready[device].store(true, std::memory_order_release);
        }
    }
    if (scratch_out)
        *scratch_out = g_scratch_ptr[device];
    return hipSuccess;
}

static inline uint64_t align_up(uint64_t v, uint64_t a) { return (v + a - 1) / a * a; }

static int index_bits(int S)
{
    int j = 0;
    while ((1ll << j) < 24ll * S)
        ++j;
    return j;
}

// Largest S the search kernel's LDS tables are sized for (paper sweeps S up to 192).
constexpr int kMaxS = HQMQ_MAX_S;

static int32_t check_params(const hqmq_params *p)
{
    if (!p)
        return HQMQ_ERR_INVALID_ARG;
    if (p->B <= 0 || p->H <= 0 || p->T <= 0 || p->D <= 0)
        return HQMQ_ERR_INVALID_ARG;
    if (p->D > 4 * kChunksPerRow)
        return HQMQ_ERR_UNSUPPORTED;
    if (p->S < 1 || p->S > kMaxS || p->b_r < 1 || p->b_r > 8)
        return HQMQ_ERR_UNSUPPORTED;
    if (!(p->flags & HQMQ_FLAG_NO_OUTLIERS) && !(std::isfinite(p->C) && p->C > 0.f))
        return HQMQ_ERR_UNSUPPORTED;
    if (p->stride_b < 0 || p->stride_h < 0 || p->stride_t < p->D)
        return HQMQ_ERR_INVALID_ARG;
    // D = 128 runs the kernels written for full rows: 16-byte accesses, every row aligned to them
    if (p->D == 4 * kChunksPerRow && ((p->stride_b % 8) || (p->stride_h % 8) || (p->stride_t % 8)))
        return HQMQ_ERR_INVALID_ARG;
    if ((int64_t)p->B * p->H > 65535)
        return HQMQ_ERR_UNSUPPORTED;  // grid.y
    const uint64_t n_rows = (uint64_t)p->B * p->H * p->T;
    if (n_rows * kChunksPerRow >= (1ull << 32))
        return HQMQ_ERR_UNSUPPORTED;  // 32-bit outlier offsets and ranks
    return HQMQ_OK;
}

static Geometry make_geometry(const hqmq_params *p)
{
    Geometry g;
    g.B = p->B;
    g.H = p->H;
    g.T = p->T;
    g.D = p->D;
    g.n_c = (p->D + 3) / 4;
    g.n_c_magic = g.n_c >= 2 ? (uint32_t)((1ull << 32) / (uint64_t)g.n_c + 1ull) : 0u;
    g.vec_ok = (p->D % 4 == 0 && p->stride_b % 4 == 0 && p->stride_h % 4 == 0 && p->stride_t % 4 == 0) ? 1 : 0;
    g.S = p->S;
    g.S16 = (p->S + 15) / 16;
    g.A16 = p->S <= kScreenMaxS ? g.S16 : 0;
    g.b_r = p->b_r;
    g.w_idx = index_bits(p->S);
    g.w = g.w_idx + p->b_r;
    g.row_words = (g.n_c * g.w + 31) / 32;
    g.sb = p->stride_b;
    g.sh = p->stride_h;
    g.st = p->stride_t;
    g.inv_S = (1.0f / (float)p->S) * (1.0f + 0x1.0p-18f);
    g.inv_L = 1.0f / (float)((1 << p->b_r) - 1);
    g.log2_S = -1;
    for (int j = 0; j < 16; ++j)
        if ((1 << j) == p->S)
            g.log2_S = j;
    g.check_finite = (p->flags & HQMQ_FLAG_CHECK_FINITE) ? 1 : 0;
    g.fused_by_head = 0;
    {
        // the select of a long head keeps the keys of a narrow range around the median: 4.7 % of a head's chunks up to 2^18
        // of them, 2.6 % up to 2^19, 1.85 % beyond; with the box index behind them there is room for twice, 1.9 and 1.3
        // times as many at least
        const uint64_t n_h = (uint64_t)p->B * p->T * g.n_c;
        const uint64_t want = (n_h / 32 + 1023) / 1024 * 1024;
        g.cand_cap = (int32_t)(want > (uint64_t)kCandCap ? want : (uint64_t)kCandCap);
        g.cand_room = g.cand_cap;
    }
    g.cell_n = g.cell_groups = g.cell_used = g.cell_words = 0;
    g.search_rows = search_rows_for(p->T, g.S16, g.A16, g.D, g.row_words);
    g.n_search_blocks_per_seg = (uint32_t)((p->T + g.search_rows - 1) / g.search_rows);
    return g;
}

// The search of the general path: the box index (built beside the select's sweep, or where a head has at most 1024 rows in a
// launch of its own, of 12 to 25 us; then a search that hardly depends on S) from chunks per head x (S + 32) = 6.3 million on, the
// matrix screen below.  Whole encodes with heads of 128 elements, screen / index in us.  4 tensors of 8 heads: S = 256: 55 / 60 at
// T = 512, 70 / 64 at 683, 85 / 65 at 1024, 262 / 89 at 4096; S = 64: 58 / 57 at 1100, 62 / 58 at 1536, 75 / 61 at 2048, 119 / 74 at
// 4096; S = 16: 46 / 46 at 1100, 57 / 50 at 2048, 72 / 59 at 3072, 84 / 64 at 4096.  Of 64 heads the two meet earlier (S = 256: 83 / 86
// at 512; S = 16: 66 / 60 at 1100), of fewer later: 8 heads S = 256: 37 / 43 at 1024, 50 / 46 at 1100; S = 64: 38 / 38 at 2048; S = 16:
// 42 / 40 at 4096; 2 heads S = 256: 27 / 41 at 1024, 45 / 42 at 4096; S = 16: 34 / 36 at 8192.
// A workgroup copies the whole index for rows of one (batch entry, head) only, so their chunks x (S + 32) have to reach 2^17: two
// tensors with 8 heads and many batch entries: S = 256: 400 / 384 at B = 1024, T = 4, 245 / 201 at 512 x 8, 362 / 214 at 512 x 16; S =
// 64: 360 / 394 at 1024 x 8, 433 / 410 at 1024 x 16, 289 / 217 at 512 x 32, 217 / 117 at 256 x 64; S = 16: 102 / 96 at 256 x 32, 90 /
// 73 at 128 x 64, 84 / 61 at 64 x 128.  With known thresholds, where each of the search's workgroups finishes the index for itself:
// 186 / 209 at S = 256, 512 x 8, 304 / 224 at 512 x 16; 230 / 208 at S = 64, 512 x 32; 62 / 51 at S = 16, 64 x 128; 4 tensors of 8 heads
// 45 / 49 at S = 64, T = 1536, 51 / 50 at S = 16, 3072.
// (Both lines were laid when every call did that: behind a select they now lie up to 20 % too high for 4 tensors and more.)
static bool use_cells(const Geometry &g)
{
    const uint64_t work = (uint64_t)g.T * g.n_c * (uint64_t)(g.S + 32);
    return g.A16 > 0 && work >= (1ull << 17) && g.B * work >= (3ull << 21);
}

// Rows per workgroup of the matrix screen: 64, or 256 where rows are short and workgroups plenty, so that copying the
// operands does not outweigh a workgroup's few chunks.  Search of n tensors with 8 heads, 256 / 64 rows in us: D = 4,
// S = 16, T = 32768: 19 / 29 (n = 1), 191 / 499 (n = 32); D = 16, T = 32759: 28 / 34 (n = 1); D = 32, T = 16375: 513 / 568
// (n = 32); but D = 16, S = 64, T = 16375 (512 workgroups): 30 / 28; D = 96, S = 16, T = 4096 (n = 1): 96 / 66, T = 2100
// (n = 32, 2304 workgroups): 219 / 193; D = 128, T = 4087 (n = 32, 4096 workgroups): 472 / 472.
static int screen_rows(const Geometry &g, int n)
{
    const int64_t blocks = (int64_t)n * g.B * g.H * ((g.T + kSearchRowsLarge - 1) / kSearchRowsLarge);
    const int64_t enough = 192 * g.n_c > 512 ? 192 * g.n_c : 512;
    const bool large = g.n_c < kChunksPerRow && g.search_rows == kSearchRowsLarge && blocks >= enough &&
                       4 * search_lds_bytes(g.S16, g.A16, g.D, g.row_words, kSearchWaves, kSearchRowsLarge) <= kLdsPerCu;
    if (large)
        return kSearchRowsLarge;
    // Few workgroups: down to 8 rows each, while a launch then has at most 2048, two waves still get a pass of 64 chunks, and by
    // this estimate the search gains: the passes of a workgroup's busiest wave, for every round of workgroups and, as those of a
    // compute unit share its SIMDs, for every one of them.  In ns with operands to copy, and then times the rows that there is room
    // for, as a nearly empty last workgroup takes a good part of a full one's time; in passes beyond 512 secondaries.  Fitted to
    // whole encodes of 2000 shapes (S = 1 to 512, D = 4 to 128) with 64, 32, 16 and 8 rows.  Of 1500 others 3 are more than 8 %
    // slower than with 64 rows, where by the counts alone 64 were (up to 62 %: they copy 70 KB of operands for 8 rows, in several
    // rounds, and split 10 rows in two); of 300 with more than 512 secondaries 3, were 14.  64 / 32 / 16 / 8 rows in us (by the
    // counts, so): 8 heads of 128 elements, S = 16, T = 1024 38 / 31 / 28 / 28 (8, 8); S = 256, T = 256 64 / 42 / 31 / 25 (8, 8);
    // 512 heads of 64, S = 384, T = 35 51 / 75 / 66 / 86 (16, 64); 256 of 96, S = 512, T = 10 31 / 31 / 30 / 42 (8, 16); 128 of 90,
    // S = 512, T = 127 89 / 73 / 90 / 97 (8, 32).
    const auto estimate = [&](int rows) {
        const int64_t per_seg = (g.T + rows - 1) / rows, wgs = (int64_t)n * g.B * g.H * per_seg;
        const int chunks = (g.T < rows ? g.T : rows) * g.n_c;
        const double passes = (chunks + 64 * kSearchWaves - 1) / (64 * kSearchWaves);
        const size_t lds_fit = kLdsPerCu / search_lds_bytes(g.S16, g.A16, g.D, g.row_words, kSearchWaves, rows);
        const double fit = (double)std::min<size_t>(lds_fit, g.A16 > 0 ? 4 : 8), per_cu = (double)((wgs + 255) / 256);
        if (g.A16 == 0)
            return passes * (std::ceil(per_cu / fit) + 0.25 * per_cu);
        const double ns = std::max(1.0, per_cu / fit) * passes * (1460 + 8.9 * g.S) + per_cu * (240 + 5.4 * passes * g.S);
        return per_seg > 1 ? ns * (double)(per_seg * rows) / g.T : ns;
    };
    int rows = kSearchRowsSmall;
    double least = estimate(rows);
    int64_t least_wgs = (int64_t)n * g.B * g.H * ((g.T + rows - 1) / rows);
    for (int half = rows / 2; half >= 2 * kSearchWaves; half /= 2) {
        const int64_t wgs = (int64_t)n * g.B * g.H * ((g.T + half - 1) / half);
        if (wgs > 2048 || half * g.n_c < 128)
            break;
        const double ns = estimate(half);
        if (ns < least || wgs == least_wgs) {  // more workgroups for less time only
            rows = half;
            least = ns;
            least_wgs = wgs;
        }
    }
    return rows;
}

// The fused search of short segments takes the rows of a head in all batch entries on one workgroup, which then builds the head's
// tables once, while these fill no more than one pass of its waves (rows of 128 elements).
static bool fused_takes_heads(const Geometry &g)
{
    return g.B > 1 && (int64_t)g.B * g.T <= 2 * kSearchWaves && g.D == 4 * kChunksPerRow;
}

// Rows of a generation step with thresholds known beforehand: one launch for up to 64 tensors (k_append), or two for up to 32
// (the fused search and its list).  k_append's workgroups, of a segment each or of a head in all batch entries, read the chunks of
// the whole tensor and score two rows at a time: it loses where segments are many (and dimensions no multiples of 4), or rows per
// workgroup; it saves a launch and the operand tables.  Which, by the time in ns that each takes: a first round of workgroups,
// and what every further one adds.  The terms are fitted to the three forms of 6500 shapes (1 to 64 tensors and rows, S = 1 to
// 512, D = 1 to 128; 6 to 150 us), two launches within 3.4 % rms, k_append 8: of these, 10 are 5 to 10 % slower than by two
// launches, none more (by k_append for all of them 205 are, up to 70 %).  In us, two launches / k_append by segment / by
// head, S = 256 unless said: 64 tensors of 8 heads x 1 row 26 / 8.4, of 4 rows 35 / 18, of 8 batch entries 36 / 48 / 28, 32 of
// these 18 / 27 / 20; 32 of 64 heads x 1 row, D = 127, S = 16 17 / 29; 24 of 8 x 8 segments, S = 8 10 / 17 / 13; 64 of 4 x 4
// segments x 4 rows, D = 40 34 / 29 / 39; one of 8 heads x 1 row 12.3 / 7.6.
constexpr int kNoAppend = 0, kAppendSegments = 1, kAppendHeads = 2;
static double append_ns(const Geometry &g, int n, bool heads)
{
    const bool whole_chunks = g.D % 4 == 0;
    const int passes = ((heads ? g.B * g.T : g.T) + 1) / 2;
    const double chunks = (double)g.B * g.H * g.T * g.n_c, more = (n * g.H * (heads ? 1 : g.B) + 255) / 256 - 1;
    return 4000 + passes * (1830 + 8.8 * g.S) + chunks * (whole_chunks ? 0.32 : 1.5) +
           more * (370 + passes * (290 + 3.7 * g.S) + chunks * (whole_chunks ? 0.63 : 0.97));
}
static double fused_ns(const Geometry &g, int n_tensors)
{
    const bool full = g.D == 4 * kChunksPerRow, heads = fused_takes_heads(g);
    const bool coop = full && (heads ? g.B * g.T : g.T) <= 2;  // the waves share a pass's secondaries
    const size_t lds = search_lds_bytes(g.S16, g.A16, g.D, g.row_words, kSearchWaves, g.search_rows) + (full ? 3072 : 0);
    const size_t most = full ? 3 : 4, per_cu = kLdsPerCu / lds < most ? kLdsPerCu / lds : most;
    double ns = 0;
    for (int left = n_tensors; left > 0; left -= kMaxEncodeBatch) {
        const int workgroups = (left < kMaxEncodeBatch ? left : kMaxEncodeBatch) * g.H * (heads ? 1 : g.B);
        const double rounds = (double)((workgroups + 256 * per_cu - 1) / (256 * per_cu));
        ns += 8600 + g.S * (coop ? 16 : 27) + 8.0 * g.T * g.n_c + (rounds - 1) * (2700 + g.S * (coop ? 14 : 21)) +
              workgroups * (1.3 + 0.0067 * g.S) + (g.D % 4 == 0 ? 0.0 : 1070 * rounds);
    }
    return ns;
}
static int append_route(const Geometry &g, int n_tensors)
{
    if (g.A16 == 0 || g.T > 4 || (int64_t)g.B * g.H * g.T > kAppendRows)
        return kNoAppend;
    const int n = n_tensors < kMaxAppendBatch ? n_tensors : kMaxAppendBatch;
    const double segments = append_ns(g, n, false), heads = append_ns(g, n, true);
    // a head per workgroup where these fill most of the chip: of fewer with many passes each the fit is not sure
    const bool by_head = g.B > 1 && n * g.H >= 200 && heads < segments;
    if ((by_head ? heads : segments) > fused_ns(g, n))
        return kNoAppend;
    return by_head ? kAppendHeads : kAppendSegments;
}

struct WorkspaceLayout {
    uint64_t state, thr, hist0, hist1, plan, cand, block_sum, block_pre, aop, total;
};

static WorkspaceLayout workspace_layout(const Geometry &g)
{
    WorkspaceLayout l;
    uint64_t off = 0;
    const uint64_t n_blocks = (uint64_t)g.B * g.H * g.n_search_blocks_per_seg;
    auto take = [&](uint64_t bytes) {
        const uint64_t at = off;
        off = align_up(off + bytes, 256);
        return at;
    };
    l.state = take((uint64_t)g.H * sizeof(SelectState));
    l.thr = take((uint64_t)g.H * sizeof(double));
    l.hist0 = take((uint64_t)g.H * kBins0 * sizeof(uint32_t));
    l.hist1 = take((uint64_t)g.H * kBins1 * sizeof(uint32_t));
    l.plan = take((uint64_t)g.H * sizeof(SelectPlan));
    l.cand = take((uint64_t)g.H * g.cand_cap * sizeof(unsigned long long));
    l.block_sum = take(n_blocks * sizeof(uint32_t));
    l.block_pre = take(n_blocks * sizeof(uint32_t));
    l.aop = take((uint64_t)g.H * g.A16 * kATiles * 64 * 16);
    l.total = off;
    return l;
}

static bool misaligned(const void *p, uintptr_t a) { return (reinterpret_cast<uintptr_t>(p) % a) != 0; }

static int32_t check_encoded(const hqmq_encoded *e, bool need_counts, uint64_t outlier_capacity)
{
    if (!e || !e->codes || !e->sigma || !e->flags || !e->row_off)
        return HQMQ_ERR_INVALID_ARG;
    if (outlier_capacity > 0 && !e->outliers)
        return HQMQ_ERR_INVALID_ARG;  // an empty list needs no storage
    if (need_counts && (!e->n_outliers || !e->status))
        return HQMQ_ERR_INVALID_ARG;
    if (misaligned(e->codes, 4) || misaligned(e->sigma, 2) || misaligned(e->flags, 4) ||
        misaligned(e->row_off, 4) || misaligned(e->outliers, 8))
        return HQMQ_ERR_INVALID_ARG;
    if (need_counts && (misaligned(e->n_outliers, 4) || misaligned(e->status, 4)))
        return HQMQ_ERR_INVALID_ARG;
    return HQMQ_OK;
}

static EncodedPtrs to_ptrs(const hqmq_encoded *e)
{
    EncodedPtrs p;
    p.codes = e->codes;
    p.sigma = e->sigma;
    p.flags = e->flags;
    p.row_off = e->row_off;
    p.outliers = e->outliers;
    p.n_outliers = e->n_outliers;
    p.status = e->status;
    return p;
}

static int32_t hip_failed(hipError_t err)
{
    g_last_hip_error = (int32_t)err;
    return HQMQ_ERR_HIP;
}

}  // namespace hqmq

using namespace hqmq;

extern "C" int32_t hqmq_last_hip_error(void) { return g_last_hip_error; }

extern "C" int32_t hqmq_init(void)
{
    const hipError_t err = ensure_device_setup();
    return err == hipSuccess ? HQMQ_OK : hip_failed(err);
}

extern "C" int32_t hqmq_sizes(const hqmq_params *params, hqmq_size_info *out)
{
    if (!out)
        return HQMQ_ERR_INVALID_ARG;
    int32_t rc = check_params(params);
    if (rc != HQMQ_OK)
        return rc;
    const Geometry g = make_geometry(params);
    std::memset(out, 0, sizeof(*out));
    const uint64_t n_rows = (uint64_t)g.B * g.H * g.T;
    out->n_rows = n_rows;
    out->index_bits = (uint32_t)g.w_idx;
    out->code_bits = (uint32_t)g.w;
    out->code_words_per_row = (uint32_t)g.row_words;
    out->chunks_per_row = (uint32_t)g.n_c;
    out->code_bytes = n_rows * (uint64_t)g.row_words * 4;
    out->sigma_bytes = n_rows * 2;
    out->flag_bytes = n_rows * 4;
    out->row_off_bytes = (n_rows + 1) * 4;
    out->n_outliers_bytes = ((uint64_t)g.H + 1) * 4;
    out->status_bytes = 4;
    // A chunk is flagged when r^2 > C^2 * median.  For C >= 1 that needs r^2 above the lower
    // median of its head, which at most floor(n_h / 2) chunks are; for C < 1 any chunk may be.
    const uint64_t n_h = (uint64_t)g.B * g.T * g.n_c;
    uint64_t cap = (uint64_t)g.H * n_h;
    if (params->flags & HQMQ_FLAG_NO_OUTLIERS)
        cap = 0;
    else if (params->C >= 1.0f)
        cap = (uint64_t)g.H * (n_h / 2);
    out->outlier_capacity_max = cap;
    out->outlier_bytes_max = cap * 8;
    out->workspace_bytes = workspace_layout(g).total;
    return HQMQ_OK;
}

static WorkspaceOffsets workspace_offsets(const WorkspaceLayout &l)
{
    WorkspaceOffsets o;
    o.state = (uint32_t)l.state;
    o.thr = (uint32_t)l.thr;
    o.hist0 = (uint32_t)l.hist0;
    o.hist1 = (uint32_t)l.hist1;
    o.plan = (uint32_t)l.plan;
    o.cand = (uint32_t)l.cand;
    o.block_sum = (uint32_t)l.block_sum;
    o.block_pre = (uint32_t)l.block_pre;
    o.aop = (uint32_t)l.aop;
    return o;
}

// Encode n_tensors tensors of one shape: up to kMaxEncodeBatch of them share each kernel launch
// (select -> search -> outlier list per group); a group's tensor i uses slice i of the workspace.
static int32_t encode_impl(const hqmq_params *params, int32_t n_tensors, const void *const *x_dev,
                           const float *const *sec_dev, const hqmq_encoded *enc,
                           const uint64_t *outlier_capacity, void *workspace_dev, uint64_t workspace_bytes,
                           void *stream, void *const *phase_events, const double *const *thr_given = nullptr,
                           bool static_scratch = false)
{
    int32_t rc = check_params(params);
    if (rc != HQMQ_OK)
        return rc;
    if (n_tensors <= 0 || !x_dev || !sec_dev || !enc || !outlier_capacity)
        return HQMQ_ERR_INVALID_ARG;
    if (static_scratch)  // the library's own array stands in for the caller's workspace
        workspace_bytes = HQMQ_STATIC_SCRATCH_BYTES;
    else if (!workspace_dev || misaligned(workspace_dev, 256))
        return HQMQ_ERR_INVALID_ARG;
    for (int32_t i = 0; i < n_tensors; ++i) {
        if (!x_dev[i] || !sec_dev[i] || misaligned(x_dev[i], 16) || misaligned(sec_dev[i], 16))
            return HQMQ_ERR_INVALID_ARG;
        rc = check_encoded(&enc[i], true, outlier_capacity[i]);
        if (rc != HQMQ_OK)
            return rc;
    }
    const Geometry g = make_geometry(params);
    const WorkspaceLayout l = workspace_layout(g);
    const int group = n_tensors < kMaxEncodeBatch ? n_tensors : kMaxEncodeBatch;
    if (workspace_bytes < l.total * (uint64_t)group)
        return HQMQ_ERR_BUFFER_TOO_SMALL;
    if (l.total >= (1ull << 32))
        return HQMQ_ERR_UNSUPPORTED;  // 32-bit offsets inside a slice
    const WorkspaceOffsets wo = workspace_offsets(l);
    hipStream_t st = static_cast<hipStream_t>(stream);
    const bool no_outliers = (params->flags & HQMQ_FLAG_NO_OUTLIERS) != 0;
    if (thr_given) {
        if (no_outliers)
            return HQMQ_ERR_INVALID_ARG;
        for (int32_t i = 0; i < n_tensors; ++i)
            if (!thr_given[i] || misaligned(thr_given[i], 8))
                return HQMQ_ERR_INVALID_ARG;
    }
    {
        void *own = nullptr;
        const hipError_t ready = ensure_device_setup(&own);
        if (ready != hipSuccess)
            return hip_failed(ready);
        if (static_scratch)
            workspace_dev = own;
    }
    auto mark = [&](int i) -> hipError_t {
        if (phase_events && phase_events[i])
            return hipEventRecord(static_cast<hipEvent_t>(phase_events[i]), st);
        return hipSuccess;
    };
    // the pointers of tensor i, as the launch of a generation step's rows takes them: 48 bits each
    auto append_parts = [&](int32_t i, uint64_t (&at)[kAppParts]) {
        const void *const parts[kAppParts] = {x_dev[i],     sec_dev[i],       thr_given ? thr_given[i] : nullptr, enc[i].codes,
                                              enc[i].sigma, enc[i].flags,     enc[i].row_off,
                                              enc[i].outliers, enc[i].n_outliers, enc[i].status};
        uint64_t all = 0;
        for (int p = 0; p < kAppParts; ++p)
            all |= at[p] = reinterpret_cast<uintptr_t>(parts[p]);
        return all >> 48 == 0;
    };
    const int route = no_outliers || thr_given != nullptr ? append_route(g, n_tensors) : kNoAppend;
    bool append = route != kNoAppend;
    for (int32_t i = 0; i < n_tensors && append; ++i) {
        uint64_t at[kAppParts];
        append = append_parts(i, at);
    }
    if (append) {
        AppendShape shape = {g.B, g.H, g.T, g.D, g.n_c, g.n_c_magic, g.row_words, g.vec_ok, g.S, g.b_r, g.w_idx, g.w, g.check_finite,
                             0, route == kAppendHeads, g.sb, g.sh, g.st, static_cast<char *>(workspace_dev) + l.thr, l.total};
        hipError_t err = mark(0);
        if (err == hipSuccess)
            err = mark(1);
        for (int32_t first = 0; first < n_tensors && err == hipSuccess; first += kMaxAppendBatch) {
            shape.n_tensors = n_tensors - first < kMaxAppendBatch ? n_tensors - first : kMaxAppendBatch;
            AppendBatch batch;
            for (int i = 0; i < shape.n_tensors; ++i) {
                uint64_t at[kAppParts];
                append_parts(first + i, at);
                for (int p = 0; p < kAppParts; ++p) {
                    batch.low[p][i] = (uint32_t)at[p];
                    batch.high[p][i] = (uint16_t)(at[p] >> 32);
                }
                batch.capacity[i] = (uint16_t)(outlier_capacity[first + i] < (uint64_t)kAppendChunks ? outlier_capacity[first + i] : kAppendChunks);
            }
            err = launch_append(shape, batch, st);
        }
        if (err == hipSuccess)
            err = mark(2);
        if (err == hipSuccess)
            err = mark(3);
        return err == hipSuccess ? HQMQ_OK : hip_failed(err);
    }
    for (int32_t first = 0; first < n_tensors; first += kMaxEncodeBatch) {
        const int n = (n_tensors - first < kMaxEncodeBatch) ? n_tensors - first : kMaxEncodeBatch;
        EncodeBatch batch;
        std::memset(&batch, 0, sizeof(batch));
        for (int i = 0; i < n; ++i) {
            EncodeTensor &t = batch.t[i];
            t.x = static_cast<const _Float16 *>(x_dev[first + i]);
            t.sec = sec_dev[first + i];
            t.enc = to_ptrs(&enc[first + i]);
            t.ws = static_cast<char *>(workspace_dev) + l.total * (uint64_t)i;
            t.outlier_capacity = outlier_capacity[first + i];
            t.thr_given = thr_given ? thr_given[first + i] : nullptr;
        }
        hipError_t err = first == 0 ? mark(0) : hipSuccess;
        if (err != hipSuccess)
            return hip_failed(err);
        // A tensor of a few rows whose thresholds are known beforehand (appended tokens, extraction off)
        // takes two launches: the fused search, then one workgroup per tensor for the outlier list.
        const uint64_t n_rows_t = (uint64_t)g.B * g.H * g.T;
        const uint64_t n_blocks_t = (uint64_t)g.B * g.H * g.n_search_blocks_per_seg;
        const bool fused = (no_outliers || thr_given != nullptr) && n_rows_t <= (uint64_t)kSmallListRows &&
                           n_blocks_t <= (uint64_t)kSmallListBlocks && search_fused_available(g);
        if (fused) {
            Geometry gf = g;
            gf.fused_by_head = fused_takes_heads(g) ? 1 : 0;
            err = mark(1);
            if (err == hipSuccess)
                err = launch_search_fused(gf, wo, batch, n, st);
            if (err == hipSuccess)
                err = mark(2);
            if (err == hipSuccess)
                err = launch_outlier_list_small(g, wo, batch, n, st);
            if (err == hipSuccess)
                err = mark(3);
            if (err != hipSuccess)
                return hip_failed(err);
            continue;
        }
        Geometry gs = g;
        WorkspaceOffsets wos = wo;
        if (use_cells(g)) {
            const CellShape c = cell_shape_for(g.S);
            gs.cell_n = c.n;
            gs.cell_groups = c.groups;
            gs.cell_used = c.used;
            gs.cell_words = (24 * g.S + 31) / 32;
            gs.cand_room = g.cand_cap - cell_index_keys(c, g.H, g.S16, gs.cell_words);
            // the most rows per workgroup (its copy of the index is made once) that leave 512 workgroups
            const auto blocks = [&](int rows) { return (int64_t)n * g.B * g.H * ((g.T + rows - 1) / rows); };
            gs.search_rows = blocks(kSearchRowsHuge) >= 512 ? kSearchRowsHuge : blocks(kSearchRowsLarge) >= 512 ? kSearchRowsLarge : kSearchRowsSmall;
        } else {
            gs.search_rows = screen_rows(g, n);
        }
        gs.n_search_blocks_per_seg = (uint32_t)((g.T + gs.search_rows - 1) / gs.search_rows);
        if (gs.search_rows < g.search_rows) {
            // more workgroups than the arrays of their totals were sized for (256 or 512 rows each): the totals take the
            // histograms' memory, which the select is done with (8 bytes per workgroup, 32 KiB per head).  They fit: fewer
            // rows are taken only while a launch has under 512 workgroups of 256 rows (index; screen of rows of one chunk),
            // or under 3 << 21 chunks per head times S + 32 (screen of others: such workspaces start at 2048 rows, and the
            // rows of one segment then reach the index rule's 2^17), or at most 2048 workgroups (screen of under 64 rows).
            const uint64_t bytes = align_up((uint64_t)g.B * g.H * gs.n_search_blocks_per_seg * 4, 256);
            if (2 * bytes > (uint64_t)g.H * kBins0 * sizeof(uint32_t))
                return HQMQ_ERR_UNSUPPORTED;
            wos.block_sum = wo.hist0;
            wos.block_pre = wo.hist0 + (uint32_t)bytes;
        }
        const bool skip_select = no_outliers || thr_given != nullptr;
        err = launch_select_median(gs, wo, batch, n, params->C, skip_select, st);
        if (err == hipSuccess)
            err = mark(1);
        if (err != hipSuccess)
            return hip_failed(err);
        err = launch_search(gs, wos, batch, n, cells_beside_select(gs, skip_select), st);
        if (err == hipSuccess)
            err = mark(2);
        if (err != hipSuccess)
            return hip_failed(err);
        err = launch_outlier_list(gs, wos, batch, n, st);
        if (err == hipSuccess)
            err = mark(3);
        if (err != hipSuccess)
            return hip_failed(err);
    }
    return HQMQ_OK;
}

extern "C" int32_t hqmq_encode(const hqmq_params *params, const void *x_dev, const float *sec_dev,
                               const hqmq_encoded *enc, uint64_t outlier_capacity,
                               void *workspace_dev, uint64_t workspace_bytes, void *stream)
{
    return encode_impl(params, 1, &x_dev, &sec_dev, enc, &outlier_capacity, workspace_dev, workspace_bytes,
                       stream, nullptr);
}

extern "C" int32_t hqmq_encode_static(const hqmq_params *params, const void *x_dev, const float *sec_dev,
                                      const hqmq_encoded *enc, uint64_t outlier_capacity, void *stream)
{
    return encode_impl(params, 1, &x_dev, &sec_dev, enc, &outlier_capacity, nullptr, 0, stream, nullptr, nullptr,
                       true);
}

extern "C" int32_t hqmq_encode_timed(const hqmq_params *params, const void *x_dev,
                                     const float *sec_dev, const hqmq_encoded *enc,
                                     uint64_t outlier_capacity, void *workspace_dev,
                                     uint64_t workspace_bytes, void *stream, void *const *phase_events)
{
    return encode_impl(params, 1, &x_dev, &sec_dev, enc, &outlier_capacity, workspace_dev, workspace_bytes,
                       stream, phase_events);
}

// the multiplier is not used when the thresholds are final
static int32_t params_for_given_thresholds(const hqmq_params *params, hqmq_params *out)
{
    if (!params)
        return HQMQ_ERR_INVALID_ARG;
    *out = *params;
    if (!(out->flags & HQMQ_FLAG_NO_OUTLIERS))
        out->C = 1.0f;
    return HQMQ_OK;
}

extern "C" int32_t hqmq_encode_given_thresholds(const hqmq_params *params, const void *x_dev,
                                                const float *sec_dev, const double *thr_dev,
                                                const hqmq_encoded *enc, uint64_t outlier_capacity,
                                                void *workspace_dev, uint64_t workspace_bytes, void *stream)
{
    hqmq_params p;
    int32_t rc = params_for_given_thresholds(params, &p);
    if (rc != HQMQ_OK)
        return rc;
    if (!thr_dev)
        return HQMQ_ERR_INVALID_ARG;
    return encode_impl(&p, 1, &x_dev, &sec_dev, enc, &outlier_capacity, workspace_dev, workspace_bytes, stream,
                       nullptr, &thr_dev);
}

extern "C" int32_t hqmq_encode_batch_given_thresholds(const hqmq_params *params, int32_t n_tensors,
                                                      const void *const *x_dev, const float *const *sec_dev,
                                                      const double *const *thr_dev, const hqmq_encoded *enc,
                                                      const uint64_t *outlier_capacity, void *workspace_dev,
                                                      uint64_t workspace_bytes, void *stream)
{
    hqmq_params p;
    int32_t rc = params_for_given_thresholds(params, &p);
    if (rc != HQMQ_OK)
        return rc;
    if (!thr_dev)
        return HQMQ_ERR_INVALID_ARG;
    return encode_impl(&p, n_tensors, x_dev, sec_dev, enc, outlier_capacity, workspace_dev, workspace_bytes,
                       stream, nullptr, thr_dev);
}

extern "C" int32_t hqmq_thresholds(const hqmq_params *params, const void *workspace_dev, uint64_t workspace_bytes,
                                   int32_t slice, double *thr_out_dev, void *stream)
{
    int32_t rc = check_params(params);
    if (rc != HQMQ_OK)
        return rc;
    if (!workspace_dev || !thr_out_dev || slice < 0 || slice >= kMaxEncodeBatch ||
        misaligned(workspace_dev, 256) || misaligned(thr_out_dev, 8))
        return HQMQ_ERR_INVALID_ARG;
    const WorkspaceLayout l = workspace_layout(make_geometry(params));
    if (workspace_bytes < l.total * ((uint64_t)slice + 1))
        return HQMQ_ERR_BUFFER_TOO_SMALL;  // the slice lies (partly) outside the caller's workspace
    const char *src = static_cast<const char *>(workspace_dev) + l.total * (uint64_t)slice + l.thr;
    hipError_t err = hipMemcpyAsync(thr_out_dev, src, (size_t)params->H * sizeof(double), hipMemcpyDeviceToDevice,
                                    static_cast<hipStream_t>(stream));
    if (err != hipSuccess)
        return hip_failed(err);
    return HQMQ_OK;
}

extern "C" int32_t hqmq_shard_median_region(const hqmq_params *params, int32_t pass, uint64_t *offset_bytes,
                                            uint64_t *n_counters)
{
    int32_t rc = check_params(params);
    if (rc != HQMQ_OK)
        return rc;
    if (pass < 0 || pass > 5 || !offset_bytes || !n_counters)
        return HQMQ_ERR_INVALID_ARG;
    const WorkspaceLayout l = workspace_layout(make_geometry(params));
    *offset_bytes = pass == 0 ? l.hist0 : l.hist1;
    *n_counters = (uint64_t)params->H * (pass == 0 ? kBins0 : kBins1);
    return HQMQ_OK;
}

extern "C" int32_t hqmq_shard_median_pass(const hqmq_params *params, uint64_t total_chunks_per_head, int32_t pass,
                                          const void *x_dev, void *workspace_dev, uint64_t workspace_bytes,
                                          void *stream)
{
    int32_t rc = check_params(params);
    if (rc != HQMQ_OK)
        return rc;
    if (pass < 0 || pass > 6 || !workspace_dev || misaligned(workspace_dev, 256))
        return HQMQ_ERR_INVALID_ARG;
    if (pass < 6 && (!x_dev || misaligned(x_dev, 16)))  // the finish reads no rows
        return HQMQ_ERR_INVALID_ARG;
    if (params->flags & HQMQ_FLAG_NO_OUTLIERS)
        return HQMQ_ERR_INVALID_ARG;
    const Geometry g = make_geometry(params);
    const uint64_t own = (uint64_t)g.B * g.T * g.n_c;
    if (total_chunks_per_head < own)
        return HQMQ_ERR_INVALID_ARG;
    if (total_chunks_per_head >= (1ull << 32))
        return HQMQ_ERR_UNSUPPORTED;  // 32-bit ranks and counters
    const WorkspaceLayout l = workspace_layout(g);
    if (workspace_bytes < l.total)
        return HQMQ_ERR_BUFFER_TOO_SMALL;
    EncodeBatch batch;
    std::memset(&batch, 0, sizeof(batch));
    batch.t[0].x = static_cast<const _Float16 *>(x_dev);
    batch.t[0].ws = static_cast<char *>(workspace_dev);
    hipError_t err = launch_shard_median_pass(g, workspace_offsets(l), batch, pass, total_chunks_per_head, params->C,
                                              static_cast<hipStream_t>(stream));
    if (err != hipSuccess)
        return hip_failed(err);
    return HQMQ_OK;
}

extern "C" int32_t hqmq_encode_batch(const hqmq_params *params, int32_t n_tensors, const void *const *x_dev,
                                     const float *const *sec_dev, const hqmq_encoded *enc,
                                     const uint64_t *outlier_capacity, void *workspace_dev,
                                     uint64_t workspace_bytes, void *stream, void *const *phase_events)
{
    return encode_impl(params, n_tensors, x_dev, sec_dev, enc, outlier_capacity, workspace_dev, workspace_bytes,
                       stream, phase_events);
}

static int32_t decode_impl(const hqmq_params *params, int32_t n_tensors, const hqmq_encoded *enc,
                           const uint64_t *outlier_capacity, const float *const *sec_dev,
                           void *const *out_dev, void *stream)
{
    int32_t rc = check_params(params);
    if (rc != HQMQ_OK)
        return rc;
    if (n_tensors <= 0 || !enc || !outlier_capacity || !sec_dev || !out_dev)
        return HQMQ_ERR_INVALID_ARG;
    for (int32_t i = 0; i < n_tensors; ++i) {
        if (!sec_dev[i] || !out_dev[i] || misaligned(out_dev[i], 16) || misaligned(sec_dev[i], 16))
            return HQMQ_ERR_INVALID_ARG;
        rc = check_encoded(&enc[i], false, outlier_capacity[i]);
        if (rc != HQMQ_OK)
            return rc;
    }
    const Geometry g = make_geometry(params);
    for (int32_t first = 0; first < n_tensors; first += kMaxDecodeBatch) {
        const int n = (n_tensors - first < kMaxDecodeBatch) ? n_tensors - first : kMaxDecodeBatch;
        DecodeBatch batch;
        std::memset(&batch, 0, sizeof(batch));
        for (int i = 0; i < n; ++i) {
            const hqmq_encoded &e = enc[first + i];
            DecodeTensor &t = batch.t[i];
            t.codes = e.codes;
            t.sigma = e.sigma;
            t.flags = e.flags;
            t.row_off = e.row_off;
            t.outliers = e.outliers;
            t.sec = sec_dev[first + i];
            t.out = static_cast<_Float16 *>(out_dev[first + i]);
            t.outlier_capacity = outlier_capacity[first + i];
        }
        hipError_t err = launch_decode(g, batch, n, static_cast<hipStream_t>(stream));
        if (err != hipSuccess)
            return hip_failed(err);
    }
    return HQMQ_OK;
}

extern "C" int32_t hqmq_decode(const hqmq_params *params, const hqmq_encoded *enc,
                               uint64_t outlier_capacity, const float *sec_dev, void *out_dev,
                               void *stream)
{
    return decode_impl(params, 1, enc, &outlier_capacity, &sec_dev, &out_dev, stream);
}

extern "C" int32_t hqmq_decode_batch(const hqmq_params *params, int32_t n_tensors,
                                     const hqmq_encoded *enc, const uint64_t *outlier_capacity,
                                     const float *const *sec_dev, void *const *out_dev, void *stream)
{
    return decode_impl(params, n_tensors, enc, outlier_capacity, sec_dev, out_dev, stream);
}

static int32_t check_attend(const hqmq_params *params, int32_t n_q_heads)
{
    int32_t rc = check_params(params);
    if (rc != HQMQ_OK)
        return rc;
    if (n_q_heads <= 0 || n_q_heads % params->H)
        return HQMQ_ERR_INVALID_ARG;
    if (params->D != 128 && params->D != 96 && params->D != 64)
        return HQMQ_ERR_UNSUPPORTED;  // the attention kernel takes the head dimensions of the paper's models
    if (n_q_heads / params->H > kMaxGroup)
        return HQMQ_ERR_UNSUPPORTED;
    return HQMQ_OK;
}

extern "C" uint64_t hqmq_attend_workspace_bytes(const hqmq_params *params, int32_t n_q_heads)
{
    if (check_attend(params, n_q_heads) != HQMQ_OK)
        return 0;
    return plan_attend(make_geometry(params), n_q_heads / params->H, (params->flags & HQMQ_FLAG_ATTEND_TABLES) != 0)
        .total_bytes;
}

static int32_t attend_impl(const hqmq_params *params, int32_t n_q_heads, const void *q_dev,
                           float scale, const hqmq_encoded *enc_k, uint64_t cap_k,
                           const float *sec_k_dev, const hqmq_encoded *enc_v, uint64_t cap_v,
                           const float *sec_v_dev, void *out_dev, float *lse_dev, const int32_t *visible_dev,
                           void *workspace_dev, uint64_t workspace_bytes, void *stream)
{
    int32_t rc = check_attend(params, n_q_heads);
    if (rc != HQMQ_OK)
        return rc;
    if (!q_dev || !out_dev || !sec_k_dev || !sec_v_dev || !workspace_dev || !std::isfinite(scale))
        return HQMQ_ERR_INVALID_ARG;
    if (misaligned(q_dev, 16) || misaligned(out_dev, 16) || misaligned(sec_k_dev, 16) ||
        misaligned(sec_v_dev, 16) || misaligned(workspace_dev, 256))
        return HQMQ_ERR_INVALID_ARG;
    rc = check_encoded(enc_k, false, cap_k);
    if (rc == HQMQ_OK)
        rc = check_encoded(enc_v, false, cap_v);
    if (rc != HQMQ_OK)
        return rc;
    const Geometry g = make_geometry(params);
    const int G = n_q_heads / params->H;
    const AttendPlan plan = plan_attend(g, G, (params->flags & HQMQ_FLAG_ATTEND_TABLES) != 0);
    if (workspace_bytes < plan.total_bytes)
        return HQMQ_ERR_BUFFER_TOO_SMALL;
    {  // the kernels may ask for more LDS than a launch gets by default (large S)
        const hipError_t ready = ensure_device_setup();
        if (ready != hipSuccess)
            return hip_failed(ready);
    }

    auto side = [](const hqmq_encoded *e, const float *sec, uint64_t cap) {
        AttendSide s;
        s.codes = e->codes;
        s.sigma = e->sigma;
        s.flags = e->flags;
        s.row_off = e->row_off;
        s.outliers = e->outliers;
        s.sec = sec;
        s.outlier_capacity = cap;
        return s;
    };
    AttendArgs a;
    a.k = side(enc_k, sec_k_dev, cap_k);
    a.v = side(enc_v, sec_v_dev, cap_v);
    a.q = static_cast<const _Float16 *>(q_dev);
    a.out = static_cast<_Float16 *>(out_dev);
    a.lse = lse_dev;
    a.visible = visible_dev;
    a.part_ml = reinterpret_cast<float *>(workspace_dev);
    a.part_acc = reinterpret_cast<float *>(static_cast<char *>(workspace_dev) + plan.ml_bytes);
    a.qscale = scale * 1.44269504088896340736f;
    a.G = G;
    a.D = params->D;
    a.n_splits = plan.n_splits;
    a.rows_per_split = plan.rows_per_split;
    a.joint = plan.joint;
    hipError_t err = launch_attend(g, a, static_cast<hipStream_t>(stream));
    if (err != hipSuccess)
        return hip_failed(err);
    return HQMQ_OK;
}

extern "C" int32_t hqmq_attend(const hqmq_params *params, int32_t n_q_heads, const void *q_dev,
                               float scale, const hqmq_encoded *enc_k, uint64_t cap_k,
                               const float *sec_k_dev, const hqmq_encoded *enc_v, uint64_t cap_v,
                               const float *sec_v_dev, void *out_dev, void *workspace_dev,
                               uint64_t workspace_bytes, void *stream)
{
    return attend_impl(params, n_q_heads, q_dev, scale, enc_k, cap_k, sec_k_dev, enc_v, cap_v, sec_v_dev, out_dev,
                       nullptr, nullptr, workspace_dev, workspace_bytes, stream);
}

extern "C" int32_t hqmq_attend_lse(const hqmq_params *params, int32_t n_q_heads, const void *q_dev,
                                   float scale, const hqmq_encoded *enc_k, uint64_t cap_k,
                                   const float *sec_k_dev, const hqmq_encoded *enc_v, uint64_t cap_v,
                                   const float *sec_v_dev, void *out_dev, float *lse_dev, void *workspace_dev,
                                   uint64_t workspace_bytes, void *stream)
{
    if (!lse_dev || misaligned(lse_dev, 4))
        return HQMQ_ERR_INVALID_ARG;
    return attend_impl(params, n_q_heads, q_dev, scale, enc_k, cap_k, sec_k_dev, enc_v, cap_v, sec_v_dev, out_dev,
                       lse_dev, nullptr, workspace_dev, workspace_bytes, stream);
}

extern "C" int32_t hqmq_attend_masked(const hqmq_params *params, int32_t n_q_heads, const void *q_dev,
                                      float scale, const hqmq_encoded *enc_k, uint64_t cap_k,
                                      const float *sec_k_dev, const hqmq_encoded *enc_v, uint64_t cap_v,
                                      const float *sec_v_dev, const int32_t *visible_dev, void *out_dev,
                                      float *lse_dev, void *workspace_dev, uint64_t workspace_bytes, void *stream)
{
    if (!visible_dev || misaligned(visible_dev, 4) || misaligned(lse_dev, 4))
        return HQMQ_ERR_INVALID_ARG;
    return attend_impl(params, n_q_heads, q_dev, scale, enc_k, cap_k, sec_k_dev, enc_v, cap_v, sec_v_dev, out_dev,
                       lse_dev, visible_dev, workspace_dev, workspace_bytes, stream);
}
