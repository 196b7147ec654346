// The tables of the search that are built before it (what they are: hqmq_search.hip): the operands of the matrix screen, by the
// call's first kernel, and the box index over the codewords, beside the sweep of the median select or in a launch of its own.
#pragma once

#include "hqmq_device.h"

namespace hqmq {

namespace {

template <int kCtrl>
__device__ __forceinline__ unsigned long long dpp_move64(unsigned long long v)
{
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, kCtrl, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(v >> 32), kCtrl, 0xf, 0xf, true);
    return ((unsigned long long)(uint32_t)hi << 32) | (uint32_t)lo;
}

__device__ __forceinline__ unsigned long long umax64(unsigned long long a, unsigned long long b)
{
    return a > b ? a : b;
}

template <int kCtrl>
__device__ __forceinline__ float dpp_move(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), kCtrl, 0xf, 0xf, true));
}
template <int kCtrl>
__device__ __forceinline__ int dpp_move(int v)
{
    return __builtin_amdgcn_update_dpp(0, v, kCtrl, 0xf, 0xf, true);
}

// Inclusive sums over the wave.
__device__ __forceinline__ uint32_t wave_scan(uint32_t v)
{
    v += (uint32_t)dpp_move<0x111>((int)v);                                          // row_shr 1, 2, 4, 8: zeros come in
    v += (uint32_t)dpp_move<0x112>((int)v);
    v += (uint32_t)dpp_move<0x114>((int)v);
    v += (uint32_t)dpp_move<0x118>((int)v);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);   // row_bcast15 into rows 1 and 3
    return v + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);  // row_bcast31 into rows 2 and 3
}

// Nearest 24-cell vertex to v in the order of the primary table: p = 0..7 are +1, -1, +i, -i,
// +j, -j, +k, -k, p = 8 + 8 b0 + 4 b1 + 2 b2 + b3 is ((-1)^b0, (-1)^b1, (-1)^b2, (-1)^b3)/2.
// Exact ties go to the lowest p.
__device__ __forceinline__ int nearest_primary(float v0, float v1, float v2, float v3, float &score)
{
    float a0 = fabsf(v0), a1 = fabsf(v1), a2 = fabsf(v2), a3 = fabsf(v3);
    float ax = a0;
    int pi = (v0 < 0.f) ? 1 : 0;
    if (a1 > ax) { ax = a1; pi = 2 + ((v1 < 0.f) ? 1 : 0); }
    if (a2 > ax) { ax = a2; pi = 4 + ((v2 < 0.f) ? 1 : 0); }
    if (a3 > ax) { ax = a3; pi = 6 + ((v3 < 0.f) ? 1 : 0); }
    float hs = 0.5f * (((a0 + a1) + a2) + a3);
    int ph = 8 + ((v0 < 0.f) ? 8 : 0) + ((v1 < 0.f) ? 4 : 0) + ((v2 < 0.f) ? 2 : 0) + ((v3 < 0.f) ? 1 : 0);
    if (ax >= hs) {
        score = ax;
        return pi;
    }
    score = hs;
    return ph;
}


// v = u conj(q) in fp32 and its closed-form score max_p <v, P_p>
__device__ __forceinline__ float score_secondary(const float *q, float u0, float u1, float u2, float u3, float &v0,
                                                 float &v1, float &v2, float &v3)
{
    const float a = q[0], bq = q[1], cq = q[2], d = q[3];
    v0 = fmaf(d, u3, fmaf(cq, u2, fmaf(bq, u1, a * u0)));
    v1 = fmaf(cq, u3, fmaf(-d, u2, fmaf(a, u1, -bq * u0)));
    v2 = fmaf(-bq, u3, fmaf(a, u2, fmaf(d, u1, -cq * u0)));
    v3 = fmaf(a, u3, fmaf(bq, u2, fmaf(-cq, u1, -d * u0)));
    const float a0 = fabsf(v0), a1 = fabsf(v1), a2 = fabsf(v2), a3 = fabsf(v3);
    return fmaxf(fmaxf(fmaxf(fmaxf(a0, a1), a2), a3), 0.5f * (((a0 + a1) + a2) + a3));  // two v_max3
}

// Maximum of a 64-bit key over the wave (every lane gets it).
__device__ __forceinline__ unsigned long long wave_umax64(unsigned long long k)
{
    k = umax64(k, dpp_move64<0xB1>(k));   // quad_perm [1, 0, 3, 2]
    k = umax64(k, dpp_move64<0x4E>(k));   // quad_perm [2, 3, 0, 1]
    k = umax64(k, dpp_move64<0x141>(k));  // row_half_mirror
    k = umax64(k, dpp_move64<0x140>(k));  // row_mirror
    k = umax64(k, (unsigned long long)__shfl_xor((long long)k, 16, 64));
    k = umax64(k, (unsigned long long)__shfl_xor((long long)k, 32, 64));
    return k;
}

typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
constexpr float kOperandScale = 1024.f;

__device__ __forceinline__ uint32_t pack2(_Float16 lo, _Float16 hi)
{
    typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
    const half2_t v = {lo, hi};
    return __builtin_bit_cast(uint32_t, v);
}

// x = h + l to 24 bits (|x - h - l| <= 2^-24 |x|), each part an fp16
struct Parts2 {
    _Float16 h, l;
};
// Hides how an fp32 value was computed.  split2 needs it: left to itself the compiler folds the
// multiplication that produced x into one of the two conversions (v_fma_mixlo_f16 rounds the exact product
// once) and converts the rounded x for the other (rounded twice); where x sits on the midpoint between two
// fp16 values the two disagree by one fp16 step and h + l misses x by 2^-11 |x|.  Seen once in 786,432
// chunks; harmless only when the product is exact (a scaling by a power of two).
__device__ __forceinline__ float opaque(float x)
{
    asm volatile("" : "+v"(x));
    return x;
}
// x: a value that went through opaque(), or an exact scaling of one.
__device__ __forceinline__ Parts2 split2(float x)
{
    Parts2 p;
    p.h = (_Float16)x;
    p.l = (_Float16)(x - (float)p.h);
    return p;
}

// The search's MFMA A operands (how they are used: hqmq_search.hip).
// Entry idx of a head's operand table: tile idx / 64 of 8 secondaries, lane l = idx % 64 holding row
// l % 32 = 4 (secondary in tile) + i and the factors k = 2 (l / 32), 2 (l / 32) + 1 of that row, each in the
// slots [h h l l].
__device__ __forceinline__ uint4 operand_entry(const float *sec_h, int S, int idx)
{
    const int tile = idx >> 6, l = idx & 63;
    const int row = l & 31, kh = l >> 5;
    const int i = row & 3;
    const int sidx = 8 * tile + (row >> 2);
    float a = 0.f, bq = 0.f, c = 0.f, d = 0.f;  // zero rows pad S up to a multiple of 16
    if (sidx < S) {
        const float *q = sec_h + 4 * sidx;
        a = q[0], bq = q[1], c = q[2], d = q[3];
    }
    // v = u (x) conj(q):  v0 =  a u0 + b u1 + c u2 + d u3
    //                     v1 = -b u0 + a u1 - d u2 + c u3
    //                     v2 = -c u0 + d u1 + a u2 - b u3
    //                     v3 = -d u0 - c u1 + b u2 + a u3
    auto entry = [&](int k) -> float {  // A[i][k]
        if (i == 0)
            return (k == 0) ? a : (k == 1) ? bq : (k == 2) ? c : d;
        if (i == 1)
            return (k == 0) ? -bq : (k == 1) ? a : (k == 2) ? -d : c;
        if (i == 2)
            return (k == 0) ? -c : (k == 1) ? d : (k == 2) ? a : -bq;
        return (k == 0) ? -d : (k == 1) ? -c : (k == 2) ? bq : a;
    };
    const float va = entry(2 * kh), vb = entry(2 * kh + 1);
    const Parts2 pa = split2(opaque(va) * kOperandScale), pb = split2(opaque(vb) * kOperandScale);
    return make_uint4(pack2(pa.h, pa.h), pack2(pa.l, pa.l), pack2(pb.h, pb.h), pack2(pb.l, pb.l));
}

// Head h's operands into the workspace, once per call: the workgroups of the search then only copy them into LDS.  Done by
// the call's first kernel, a workgroup per head (a launch of their own took 4 us).
__device__ __forceinline__ void build_operands(const Geometry &g, const Workspace &ws, const float *sec, int h, int tid, int threads)
{
    const int n = g.A16 * kATiles * 64;
    for (int idx = tid; idx < n; idx += threads)
        ws.aop[(size_t)h * n + idx] = operand_entry(sec + (size_t)h * g.S * 4, g.S, idx);
}

constexpr int kCellThreads = 256;      // workgroup of the index build: 4 lanes per box
constexpr int kCoarseCap = 1024;       // codewords of a block of 4^3 boxes
constexpr int kMidCap = 384;           // codewords of a sub-block of 2^3 boxes
constexpr float kListEps = 1.0e-5f;    // lists keep what comes within this fraction of the centre's best score: more than
                                       // kCellBand times the ratio of two scores of a box plus the rounding of the test
constexpr uint32_t kCellPad = 0x7fffu; // list entry without a codeword; bit 15 marks the last group of a list


// Component i of primary p.
__device__ __forceinline__ float primary_component(int p, int i)
{
    if (p < 8)
        return (p >> 1) == i ? ((p & 1) ? -1.f : 1.f) : 0.f;
    return (((p - 8) >> (3 - i)) & 1) ? -0.5f : 0.5f;
}

// P_p q as (c_1, c_2, c_3, c_0): the linear function of a box point.
__device__ __forceinline__ float4_t codeword_function(int p, const float4_t q)
{
    const float a = primary_component(p, 0), b = primary_component(p, 1), c = primary_component(p, 2),
                d = primary_component(p, 3);
    float4_t f;
    f[3] = fmaf(-d, q[3], fmaf(-c, q[2], fmaf(-b, q[1], a * q[0])));
    f[0] = fmaf(-d, q[2], fmaf(c, q[3], fmaf(b, q[0], a * q[1])));
    f[1] = fmaf(d, q[1], fmaf(c, q[0], fmaf(-b, q[3], a * q[2])));
    f[2] = fmaf(d, q[0], fmaf(-c, q[1], fmaf(b, q[2], a * q[3])));
    return f;
}

__device__ __forceinline__ float value_at(const float4_t f, float m1, float m2, float m3)
{
    return fmaf(f[0], m1, fmaf(f[1], m2, fmaf(f[2], m3, f[3])));
}

// b (value vb at the centre) ahead of c (value vc) by more than eps all over the box of half width h
__device__ __forceinline__ bool ahead_in_box(const float4_t b, float vb, const float4_t c, float vc, float h, float eps)
{
    const float spread = (fabsf(b[0] - c[0]) + fabsf(b[1] - c[1])) + fabsf(b[2] - c[2]);
    return vb - vc > fmaf(h, spread, eps);
}

// Box of half width h around m meets the octahedron (with room for the rounding of y).
__device__ __forceinline__ bool meets_octahedron(float m1, float m2, float m3, float h)
{
    return (fmaxf(fabsf(m1) - h, 0.f) + fmaxf(fabsf(m2) - h, 0.f)) + fmaxf(fabsf(m3) - h, 0.f) <= 1.0001f;
}

struct CellIndex {        // parts of one head's index in the workspace; finish_cells turns lists and boxes into LDS addresses
    uint2 *list;          // [cell_groups] groups of four 16-bit entries k = p S + s; group 0 belongs to no list
    uint16_t *head;       // [n^3] first group of the box's list; 0 = no list; behind the lists, as in LDS
    uint32_t *n_groups;   // groups handed out beyond group 0
    uint32_t *used;       // [cell_words] bit k: codeword k is in some list
    uint32_t *id;         // [cell_used] p << 16 | s of the codewords in use, ascending
    float4_t *function;   // [cell_used + 1] their functions
};
__device__ __forceinline__ CellIndex cell_index_of(const Geometry &g, const Workspace &ws, int h)
{
    CellIndex ix;
    char *base = reinterpret_cast<char *>(ws.cand + (size_t)h * g.cand_cap + g.cand_room);
    ix.list = reinterpret_cast<uint2 *>(base);
    ix.head = reinterpret_cast<uint16_t *>(ix.list + g.cell_groups);
    const CellOffsets at = cell_offsets(g.H, g.cell_words, g.cell_used);
    ix.n_groups = reinterpret_cast<uint32_t *>(ws.cell_state) + (size_t)h * (1 + g.cell_words);
    ix.used = ix.n_groups + 1;
    ix.id = reinterpret_cast<uint32_t *>(ws.cell_state + at.id) + (size_t)h * g.cell_used;
    ix.function = cell_functions_behind_lists(g.H, g.S16, at)
                      ? reinterpret_cast<float4_t *>(reinterpret_cast<char *>(ix.head) + cell_head_bytes(g.cell_n))
                      : reinterpret_cast<float4_t *>(ws.cell_state + at.function) + (size_t)h * (g.cell_used + 1);
    return ix;
}

// LDS image of a head's index during the search, at the start of the workgroup's LDS (address 0: the kernel has no static LDS,
// checked by the host).  List entries and box heads are LDS addresses, so that neither takes arithmetic (the first two arrays
// end below 2^16, checked by the host).
struct CellTables {
    uint32_t base;    // address of the codeword functions (c_1, c_2, c_3, c_0) [cell_used + 1]; the last never wins
    uint32_t list;    // [cell_groups] groups of four addresses of functions, the first two ascending in the last group of a list
    uint32_t head;    // [n^3] u16 address of the box's first group
    uint32_t id;      // [cell_used] p' << 16 | s of the codeword
    uint32_t mul;     // [kFolds][32] u8: FoldTable
    uint32_t sec;     // [S][4] the head's secondaries
    uint32_t end;
};
constexpr int kFolds = 33;
__host__ __device__ inline CellTables cell_tables(const Geometry &g)
{
    CellTables t;
    t.base = 0;
    t.list = t.base + ((uint32_t)g.cell_used + 1u) * 16u;
    t.head = t.list + (uint32_t)g.cell_groups * 8u;
    t.id = t.head + (uint32_t)cell_head_bytes(g.cell_n);
    t.mul = t.id + (uint32_t)g.cell_used * 4u;
    t.sec = t.mul + (uint32_t)kFolds * 32u;
    t.end = t.sec + (uint32_t)g.S * 16u;
    return t;
}

}  // namespace

// Index build: a workgroup of kCellThreads does the 4^3 boxes of one block of the grid.
//   1  the best codeword at the block's centre, and the codewords that it is not ahead of all over the block
//   2  the same for its 2^3 sub-blocks of 2^3 boxes against that list (32 lanes each)
//   3  the same for every box against its sub-block's list (4 lanes each, a bit per entry), then the survivors against eight
//      strong ones, the best two of each lane's share (every pair: 2 % fewer entries for three times the work)
//   4  the lists, four entries to a group, in space handed out by one counter per head
// For S = 256 about 136, 28, 7 and 5.5 codewords are left after steps 1, 2 and 3.
// A box whose list does not fit any of the arrays gets none; its chunks take the search over all S secondaries.
// Its space is zeroed beforehand (reset_head: the counter and the bits).
// Bound by VALU issue where heads are many (1640 instructions a wave) and by the latency of its steps where they are few: 52 us
// for 64 heads (S = 192), 22 for 16 (S = 256), 18 for 8 (68, 27 and 19 with the survivors of step 1 made into functions where
// they are found, and step 3's survivors listed by votes).
struct CellBuild {  // LDS
    float4_t cf[kCoarseCap];
    float4_t wave_q[kCellThreads / 64];
    unsigned long long wave_key[kCellThreads / 64];
    uint16_t ck[kCoarseCap];
    uint32_t cused[kCoarseCap / 32];
    uint16_t mid[8][kMidCap];
    uint32_t first_group[64];
    uint32_t n_coarse, list_base;
};
__host__ __device__ inline int cell_blocks(const Geometry &g)  // of a head
{
    return (g.cell_n / 4) * (g.cell_n / 4) * (g.cell_n / 4);
}
__device__ __forceinline__ void build_cells(const Geometry &g, const Workspace &ws, const float *sec, int h, int block, CellBuild &lds)
{
    const int S = g.S, n = g.cell_n, nb = n / 4;
    const float4_t *sec_h = reinterpret_cast<const float4_t *>(sec + (size_t)h * S * 4);
    const CellIndex ix = cell_index_of(g, ws, h);

    const int tid = threadIdx.x, lane = tid & 63;
    const int b0 = block / (nb * nb), b1 = (block / nb) % nb, b2 = block % nb;
    // box of this lane's quad: sub-block tid / 32, box of it (tid / 4) % 8
    const int cell = tid >> 2, sub = tid & 3, sb = tid >> 5;
    const int s0 = sb >> 2, s1 = (sb >> 1) & 1, s2 = sb & 1;
    const int i0 = 4 * b0 + 2 * s0 + ((cell >> 2) & 1), i1 = 4 * b1 + 2 * s1 + ((cell >> 1) & 1), i2 = 4 * b2 + 2 * s2 + (cell & 1);
    const int cell_id = (i0 * n + i1) * n + i2;
    const float hf = 1.0f / (float)n;
    const float margin = 1.2e-5f;  // y and the box number are rounded (7e-7), the latter shrunk by 4e-6 as well
    const float m1 = (float)(8 * b0 + 4) * hf - 1.f, m2 = (float)(8 * b1 + 4) * hf - 1.f, m3 = (float)(8 * b2 + 4) * hf - 1.f;
    if (block == 0 && tid == 0)
        ix.list[0] = make_uint2(kCellPad | 0x8000u | (kCellPad << 16), kCellPad | (kCellPad << 16));
    if (!meets_octahedron(m1, m2, m3, 4.f * hf)) {  // uniform
        if (sub == 0)
            ix.head[cell_id] = 0;
        return;
    }

    // ---- 1: the block ------------------------------------------------------------------------------------------------
    constexpr int kOwn = kScreenMaxS / kCellThreads;  // secondaries of a thread
    float4_t q[kOwn];
    {
        unsigned long long key = 0ull;
        float4_t q_key = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int u = 0; u < kOwn; ++u) {
            const int s = tid + u * kCellThreads;
            q[u] = float4_t{0.f, 0.f, 0.f, 0.f};
            if (s < S) {
                q[u] = sec_h[s];
                const float qs[4] = {q[u][0], q[u][1], q[u][2], q[u][3]};
                float v0, v1, v2, v3;
                const float sc = score_secondary(qs, 1.f, m1, m2, m3, v0, v1, v2, v3);
                const unsigned long long k = ((unsigned long long)__float_as_uint(sc) << 32) | (0xffffffffu - (uint32_t)s);
                if (k > key) {
                    key = k;
                    q_key = q[u];
                }
            }
        }
        if (tid == 0)
            lds.n_coarse = 0;
        if (tid < kCoarseCap / 32)
            lds.cused[tid] = 0;
        const unsigned long long top = wave_umax64(key);
        if (key == top) {  // one lane, or all of a wave without secondaries
            lds.wave_key[tid >> 6] = key;
            lds.wave_q[tid >> 6] = q_key;
        }
    }
    __syncthreads();
    float4_t best;
    float v_best;
    {
        unsigned long long key = lds.wave_key[0];
        int w_best = 0;
#pragma unroll
        for (int w = 1; w < kCellThreads / 64; ++w) {
            const unsigned long long k = lds.wave_key[w];
            w_best = k > key ? w : w_best;
            key = umax64(key, k);
        }
        const float4_t qb = lds.wave_q[w_best];
        const float qs[4] = {qb[0], qb[1], qb[2], qb[3]};
        float v0, v1, v2, v3, sc;
        (void)score_secondary(qs, 1.f, m1, m2, m3, v0, v1, v2, v3);
        best = codeword_function(nearest_primary(v0, v1, v2, v3, sc), qb);
        v_best = value_at(best, m1, m2, m3);
    }
    {
        const float hb = 4.f * hf + margin, eps = kListEps * fabsf(v_best);
#pragma unroll
        for (int u = 0; u < kOwn; ++u) {
            if (u * kCellThreads >= S)  // uniform
                break;
            const int s = tid + u * kCellThreads;
            // c: P_p q as (c_1, c_2, c_3, c_0), v its value at the centre; its negative is tested along with it
            uint32_t left = 0;
            auto test = [&](const float4_t c, float v, int p, int p_neg) {
                left |= ahead_in_box(best, v_best, c, v, hb, eps) ? 0u : 1u << p;
                left |= ahead_in_box(best, v_best, -c, -v, hb, eps) ? 0u : 1u << p_neg;
            };
            const float4_t e0 = {q[u][1], q[u][2], q[u][3], q[u][0]}, e1 = {q[u][0], -q[u][3], q[u][2], -q[u][1]};  // q, i q
            const float4_t e2 = {q[u][3], q[u][0], -q[u][1], -q[u][2]}, e3 = {-q[u][2], q[u][1], q[u][0], -q[u][3]};  // j q, k q
            const float v0 = value_at(e0, m1, m2, m3), v1 = value_at(e1, m1, m2, m3);
            const float v2 = value_at(e2, m1, m2, m3), v3 = value_at(e3, m1, m2, m3);
            test(e0, v0, 0, 1);
            test(e1, v1, 2, 3);
            test(e2, v2, 4, 5);
            test(e3, v3, 6, 7);
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                const float4_t ea = a ? e0 - e1 : e0 + e1;
                const float va = a ? v0 - v1 : v0 + v1;
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    const float4_t eb = (b & 2 ? -e2 : e2) + (b & 1 ? -e3 : e3);
                    const float vb = (b & 2 ? -v2 : v2) + (b & 1 ? -v3 : v3);
                    const int p = 8 + 4 * a + b;
                    test(0.5f * (ea + eb), 0.5f * (va + vb), p, 31 - p);
                }
            }
            if (s >= S)
                left = 0;
            // the wave's survivors take consecutive places
            const uint32_t count = __popc(left), inc = wave_scan(count);
            uint32_t base = 0;
            if (lane == 63)
                base = atomicAdd(&lds.n_coarse, inc);
            uint32_t at = (uint32_t)__builtin_amdgcn_readlane((int)base, 63) + inc - count;
            for (; left; left &= left - 1u, ++at)
                if (at < (uint32_t)kCoarseCap)
                    lds.ck[at] = (uint16_t)((__ffs((int)left) - 1) * S + s);
        }
    }
    __syncthreads();
    const int nc = lds.n_coarse <= (uint32_t)kCoarseCap ? (int)lds.n_coarse : 0;  // 0: no lists in this block
    for (int i = tid; i < nc; i += kCellThreads) {
        const uint32_t k = lds.ck[i], p = (uint32_t)((float)k * g.inv_S);
        lds.cf[i] = codeword_function((int)p, sec_h[k - p * (uint32_t)S]);
    }
    __syncthreads();

    // ---- 2: the sub-block ----------------------------------------------------------------------------------------------
    int nm = 0;
    if (nc > 0) {
        const float z1 = (float)(8 * b0 + 4 * s0 + 2) * hf - 1.f, z2 = (float)(8 * b1 + 4 * s1 + 2) * hf - 1.f,
                    z3 = (float)(8 * b2 + 4 * s2 + 2) * hf - 1.f;
        if (meets_octahedron(z1, z2, z3, 2.f * hf)) {
            const int l = tid & 31;
            float v = -3.4e38f;
            int j_best = 0;
            for (int j = l; j < nc; j += 32) {
                const float w = value_at(lds.cf[j], z1, z2, z3);
                j_best = w > v ? j : j_best;
                v = fmaxf(v, w);
            }
            float vb = fmaxf(v, dpp_move<0xB1>(v));  // as in a row maximum: quad_perm twice, row_half_mirror, row_mirror
            vb = fmaxf(vb, dpp_move<0x4E>(vb));
            vb = fmaxf(vb, dpp_move<0x141>(vb));
            vb = fmaxf(vb, dpp_move<0x140>(vb));
            vb = fmaxf(vb, __shfl_xor(vb, 16, 64));
            const uint32_t holds = (uint32_t)(__ballot(v == vb) >> (lane & 32));
            const float4_t bf = lds.cf[__shfl(j_best, (lane & 32) + __ffs((int)holds) - 1, 64)];
            const float eps = kListEps * fabsf(vb), hm = 2.f * hf + margin;
            for (int j0 = 0; j0 < nc; j0 += 32) {  // uniform over the half-wave
                const int j = j0 + l;
                const float4_t c = lds.cf[min(j, nc - 1)];
                const bool stays = j < nc && !ahead_in_box(bf, vb, c, value_at(c, z1, z2, z3), hm, eps);
                const uint32_t votes = (uint32_t)(__ballot(stays) >> (lane & 32));
                const int at = nm + __popc(votes & ((1u << l) - 1u));
                if (stays && at < kMidCap)
                    lds.mid[sb][at] = (uint16_t)j;
                nm += __popc(votes);
            }
        }
    }
    wave_lds_sync();  // the lanes of a sub-block, and of a box, belong to one wave
    if (nm > kMidCap)
        nm = 0;

    // ---- 3: the box ------------------------------------------------------------------------------------------------------
    constexpr int kMask = (kMidCap + 127) / 128;
    uint32_t keep[kMask] = {};  // bit i of word k: entry 128 k + 4 i + sub of the sub-block's list
    const uint16_t *list = lds.mid[sb];
    {
        const float y1 = (float)(2 * i0 + 1) * hf - 1.f, y2 = (float)(2 * i1 + 1) * hf - 1.f, y3 = (float)(2 * i2 + 1) * hf - 1.f;
        if (nm > 0 && meets_octahedron(y1, y2, y3, hf)) {
            const float hc = hf + margin;
            float vb = -3.4e38f;
            int jb = 0;
            for (int j = sub; j < nm; j += 4) {
                const int i = list[j];
                const float w = value_at(lds.cf[i], y1, y2, y3);
                jb = w > vb ? i : jb;
                vb = fmaxf(vb, w);
            }
            auto quad_max = [&](float vo, int jo) {
                const bool take = vo > vb || (vo == vb && jo < jb);
                vb = take ? vo : vb;
                jb = take ? jo : jb;
            };
            quad_max(dpp_move<0xB1>(vb), dpp_move<0xB1>(jb));
            quad_max(dpp_move<0x4E>(vb), dpp_move<0x4E>(jb));
            const float4_t bf = lds.cf[jb];
            const float eps = kListEps * fabsf(vb);
            float v_own[2] = {-3.4e38f, -3.4e38f};  // the two strongest survivors of this lane's share
            int j_own[2] = {jb, jb};
#pragma unroll
            for (int k = 0; k < kMask; ++k) {
                for (int j = 128 * k + sub, bit = 0; j < min(nm, 128 * (k + 1)); j += 4, ++bit) {
                    const int i = list[j];
                    const float4_t c = lds.cf[i];
                    const float v = value_at(c, y1, y2, y3);
                    if (!ahead_in_box(bf, vb, c, v, hc, eps)) {
                        keep[k] |= 1u << bit;
                        j_own[1] = v > v_own[0] ? j_own[0] : v > v_own[1] ? i : j_own[1];
                        v_own[1] = __builtin_amdgcn_fmed3f(v, v_own[0], v_own[1]);
                        j_own[0] = v > v_own[0] ? i : j_own[0];
                        v_own[0] = fmaxf(v_own[0], v);
                    }
                }
            }
            const int at[8] = {dpp_move<0x00>(j_own[0]), dpp_move<0x00>(j_own[1]), dpp_move<0x55>(j_own[0]), dpp_move<0x55>(j_own[1]),
                               dpp_move<0xAA>(j_own[0]), dpp_move<0xAA>(j_own[1]), dpp_move<0xFF>(j_own[0]), dpp_move<0xFF>(j_own[1])};
            float4_t strong[8];
            float v_strong[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                strong[k] = lds.cf[at[k]];
                v_strong[k] = value_at(strong[k], y1, y2, y3);
            }
#pragma unroll
            for (int k = 0; k < kMask; ++k) {
                for (uint32_t left = keep[k]; left; left &= left - 1u) {
                    const uint32_t bit = left & (0u - left);
                    const float4_t c = lds.cf[list[128 * k + 4 * (__ffs((int)left) - 1) + sub]];
                    const float v = value_at(c, y1, y2, y3);
                    bool out = false;
#pragma unroll
                    for (int i = 0; i < 8; ++i)
                        out |= ahead_in_box(strong[i], v_strong[i], c, v, hc, eps);
                    keep[k] &= out ? ~bit : ~0u;
                }
            }
        }
    }
    // ---- 4: space for the lists, entries -----------------------------------------------------------------------------------
    int mine = 0;
#pragma unroll
    for (int k = 0; k < kMask; ++k)
        mine += __popc(keep[k]);
    // entries of the quad's lanes in front of this one, and of all four
    const int of[4] = {dpp_move<0x00>(mine), dpp_move<0x55>(mine), dpp_move<0xAA>(mine), dpp_move<0xFF>(mine)};
    const uint32_t before = (uint32_t)((sub > 0 ? of[0] : 0) + (sub > 1 ? of[1] : 0) + (sub > 2 ? of[2] : 0));
    const uint32_t total = (uint32_t)(of[0] + of[1] + of[2] + of[3]);
    const uint32_t groups = (total + 3) >> 2;
    if (sub == 0)
        lds.first_group[cell] = groups;
    __syncthreads();
    if (tid < 64) {
        const uint32_t v = lds.first_group[tid], inc = wave_scan(v);
        if (tid == 63)
            lds.list_base = 1u + (inc ? atomicAdd(ix.n_groups, inc) : 0u);
        lds.first_group[tid] = inc - v;
    }
    __syncthreads();
    const uint32_t first = lds.list_base + lds.first_group[cell];
    const bool fits = groups > 0 && first + groups <= (uint32_t)g.cell_groups;
    if (sub == 0)
        ix.head[cell_id] = fits ? (uint16_t)first : (uint16_t)0;
    if (fits) {
        uint16_t *dst = reinterpret_cast<uint16_t *>(ix.list + first);
        uint32_t at = before;
#pragma unroll
        for (int k = 0; k < kMask; ++k) {
            for (uint32_t left = keep[k]; left; left &= left - 1u) {
                const int j = list[128 * k + 4 * (__ffs((int)left) - 1) + sub];
                atomicOr(&lds.cused[j >> 5], 1u << (j & 31));
                dst[at] = (uint16_t)(lds.ck[j] | (at == 4 * (groups - 1) ? 0x8000u : 0u));
                ++at;
            }
        }
        if (sub == 3)  // the last lane's entries end the list
            for (at = total; at < 4 * groups; ++at)
                dst[at] = (uint16_t)kCellPad;
    }
    __syncthreads();
    for (int j = tid; j < nc; j += kCellThreads)
        if ((lds.cused[j >> 5] >> (j & 31)) & 1u)
            atomicOr(&ix.used[lds.ck[j] >> 5], 1u << (lds.ck[j] & 31));
}

// The built index in the form that the search reads from LDS: entries k become addresses, and the functions of the codewords that
// lists name are tabulated.  Where the select follows the build, its launches have room for that (up to kFinishParts workgroups of
// 1024 threads per head, in place): done by each of the search's workgroups for itself it was 500 of a wave's 4500 instructions for 512
// rows, and more than the search for 64.  A launch of its own for it takes what it saves (32 tensors of 8 heads of 1024 rows, S =
// 256, known thresholds: 262 us, 246 without), so without a select each workgroup does it into its LDS.
// bits: LDS, scratch.
constexpr int kFinishThreads = 1024;
constexpr uint32_t kFinishParts = 8;
constexpr int kFinishWords = 2 * (24 * kScreenMaxS / 32) + 1;  // of LDS
struct CellPlaces {
    uint2 *list;
    uint2 *head;
    uint32_t *id;
    float4_t *function;
};
template <bool kShared>  // by `parts` workgroups, or else by one
__device__ __forceinline__ void finish_cells(const Geometry &g, const Workspace &ws, const float4_t *sec_h, int h, int part, int parts,
                                             const CellPlaces to, uint32_t *bits)
{
    const int tid = threadIdx.x, lane = tid & 63;
    const CellIndex ix = cell_index_of(g, ws, h);
    const CellTables ct = cell_tables(g);
    const int nw = g.cell_words, used_cap = g.cell_used;
    uint32_t *pre = bits + nw;  // [nw], then the number of codewords in use
    if (tid < 64) {  // exclusive prefix of the used bits, nw <= 6 * 64 words
        uint32_t w[6], sum = 0;
#pragma unroll
        for (int j = 0; j < 6; ++j) {
            const int i = 6 * lane + j;
            w[j] = i < nw ? ix.used[i] : 0u;
            sum += __popc(w[j]);
        }
        const uint32_t inc = wave_scan(sum);
        uint32_t run = inc - sum;
#pragma unroll
        for (int j = 0; j < 6; ++j) {
            const int i = 6 * lane + j;
            if (i < nw) {
                bits[i] = w[j];
                pre[i] = run;
            }
            run += __popc(w[j]);
        }
        if (lane == 63)
            pre[nw] = inc;
    }
    const int first = part * kFinishThreads + tid;
    const int step = kShared ? parts * kFinishThreads : kFinishThreads;
    __syncthreads();
    const int n_used = (int)pre[nw];
    const bool whole = n_used <= used_cap;  // else no box gets a list
    {
        const uint2 *head = reinterpret_cast<const uint2 *>(ix.head);
        const int words = g.cell_n * g.cell_n * g.cell_n / 4;  // n is a multiple of 4
        auto address = [&](uint32_t group) { return ct.list + 8u * (whole ? min(group, (uint32_t)g.cell_groups - 1u) : 0u); };
        for (int i = first; i < words; i += step) {
            const uint2 v = head[i];
            to.head[i] = make_uint2(address(v.x & 0xffffu) | (address(v.x >> 16) << 16), address(v.y & 0xffffu) | (address(v.y >> 16) << 16));
        }
    }
    const uint32_t S = (uint32_t)g.S, n_code = 24u * S;
    auto place_of = [&](uint32_t k) { return pre[k >> 5] + (uint32_t)__popc(bits[k >> 5] & ((1u << (k & 31u)) - 1u)); };
    const int n_groups = min((int)*ix.n_groups + 1, g.cell_groups);
    const uint32_t pad = ct.base + 16u * (uint32_t)used_cap;
    auto address_of = [&](uint32_t k) {  // a pad, or a group that belongs to no list: the function that never wins
        return k < n_code ? min(ct.base + 16u * place_of(k), pad) : pad;
    };
    for (int i = first; i < n_groups; i += step) {
        const uint2 raw = ix.list[i];
        const uint32_t a = address_of(raw.x & 0x7fffu), b = address_of(raw.x >> 16);
        const uint32_t low = min(a, b), high = max(a, b);  // equal: pads
        to.list[i] = make_uint2(raw.x & 0x8000u ? low | (high << 16) : high | (low << 16),
                                address_of(raw.y & 0xffffu) | (address_of(raw.y >> 16) << 16));
    }
    const int n_functions = min(n_used, used_cap);
    if (kShared) {
        for (uint32_t k = (uint32_t)first; k < n_code; k += step) {
            if ((bits[k >> 5] >> (k & 31u)) & 1u) {
                const uint32_t at = place_of(k), p = (uint32_t)((float)k * g.inv_S), s = k - p * S;  // k / S
                if (at < (uint32_t)used_cap) {
                    to.id[at] = (p << 16) | s;
                    to.function[at] = codeword_function((int)p, sec_h[s]);
                }
            }
        }
    } else {  // a tenth of the codewords is in use: one step for their functions where a thread per codeword would take six
        for (int i = tid; i < nw; i += kFinishThreads) {
            uint32_t left = bits[i], at = pre[i];
            for (; left; left &= left - 1u, ++at) {
                const uint32_t k = 32u * (uint32_t)i + (uint32_t)__ffs((int)left) - 1u, p = (uint32_t)((float)k * g.inv_S);
                if (at < (uint32_t)used_cap && k < n_code)
                    to.id[at] = (p << 16) | (k - p * S);
            }
        }
        __syncthreads();
        for (int i = tid; i < n_functions; i += kFinishThreads)
            to.function[i] = codeword_function((int)(to.id[i] >> 16), sec_h[to.id[i] & 0xffffu]);
    }
    for (int i = n_functions + first; i <= used_cap; i += step)
        to.function[i] = float4_t{0.f, 0.f, 0.f, -1.0e30f};
    if (n_used == 0 && first == 0)
        to.id[0] = 0;  // what a chunk without a list reads before the fp32 search
}

}  // namespace hqmq
