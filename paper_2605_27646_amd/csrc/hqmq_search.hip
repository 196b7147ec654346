// HQMQ encode, second half: outlier flags, per-row scale, nearest-codeword search, radius code and
// bit packing (paper Alg. 1 "Encode", App. D "Encode").
//
// Search formulation.  The score of codeword (p, s) is <u, P_p q_s>.  Right multiplication by
// conj(q_s) is an isometry of R^4 up to the common factor |q_s|^2, so
//     <u, P_p q_s> = <u conj(q_s), P_p>,
// and for a fixed s the best primary is the 24-cell vertex nearest to v = u conj(q_s):
//     max_p <v, P_p> = max( max_i |v_i| , (|v_0|+|v_1|+|v_2|+|v_3|)/2 )
// (first term: the 8 axis elements +-1, +-i, +-j, +-k; second: the 16 half-integer elements).
// The map u -> v is linear, v = A(q_s) u with a 4x4 matrix per secondary, so all S products of
// 32 chunks are one [4S x 4] x [4 x 32] contraction with K = 4 on the matrix cores (how it is fed
// to them is described at the kernel).  One MFMA gives every lane the four components of v for
// four (chunk, secondary) pairs; the closed form and the running argmax over s are a handful of
// VALU instructions per pair.  The search stays exhaustive over all S secondaries and, through
// the closed form, over all 24 primaries.
//
// The kernel is bound by VALU issue: with four waves on a SIMD the matrix products run behind the other
// waves' vector work (counters: the VALU is busy for the whole kernel, the MFMA pipe for a quarter of it),
// so the VALU count per (chunk, secondary) pair is what is minimised: the running argmax
// is kept per group of 16 secondaries (8 per lane) with v_max3 chains, one compare-and-select per
// group, and the winner inside the winning group is found afterwards by re-scoring its candidates.
//
// The matrix pass is a screen, not the decision.  It runs on v_mfma_f32_32x32x16_f16 with every fp32
// factor split into two fp16 parts (24 bits), i.e. four products per term, half of what a
// three-part split costs on the matrix cores and a quarter of the fp32 shape's time.  A screened score is
// within 7e-7 of the true one.  Next to its best group every lane keeps the runner-up score; a chunk whose
// winning group is not ahead of every other group by 6e-6 of its score is searched again over all S secondaries with
// plain fp32 arithmetic.  Either way the choice between secondaries is made on fp32 closed-form scores.
//
// Work split: a workgroup of 4 waves owns 64 rows of one (b, h) segment (down to 8 where workgroups are
// few, 256 where rows are short and many), so the A matrices of the head sit in LDS once per workgroup.
// A wave takes 64 chunks, one per lane, at a time and runs them as two 32-chunk MFMA column groups: two whole rows of 128 elements in
// k_search, 64 consecutive chunks of the workgroup's flattened rows in k_search_flat (any other
// head dimension).  The per-chunk steps (scale, radius code, direction search) are shared.
//
// That is the search of short tensors.  Long ones locate a chunk's direction in a box index over the codewords
// (k_cells, k_search_cells below), which replaces the scan over all S secondaries.
#include <algorithm>

#include "hqmq_tables.h"

namespace hqmq {

namespace {

__device__ __forceinline__ uint16_t double_to_half_rne_sat(double v)
{
    // v >= 0 and finite.  Round to nearest even from the full 53-bit significand (no double
    // rounding through fp32), saturate at 65504.
    if (!(v < 65504.0))
        return 0x7bff;
    unsigned long long bits = (unsigned long long)__double_as_longlong(v);
    int e = (int)(bits >> 52) - 1023;
    if (e < -40)
        return 0;  // far below half of the smallest subnormal 2^-24
    unsigned long long m = (bits & 0x000fffffffffffffull) | 0x0010000000000000ull;
    int E = e < -14 ? -14 : e;
    int sh = 42 + (E - e);  // 42 .. 68
    if (sh > 63)
        return 0;
    unsigned long long q = m >> sh;
    unsigned long long rem = m & ((1ull << sh) - 1ull);
    unsigned long long half = 1ull << (sh - 1);
    if (rem > half || (rem == half && (q & 1ull)))
        ++q;
    uint32_t out = ((uint32_t)(E + 14) << 10) + (uint32_t)q;
    return out > 0x7bff ? (uint16_t)0x7bff : (uint16_t)out;
}

template <int kCtrl>
__device__ __forceinline__ double dpp_move_f64(double v)
{
    return __longlong_as_double((long long)dpp_move64<kCtrl>((unsigned long long)__double_as_longlong(v)));
}

template <int kCtrl>
__device__ __forceinline__ double dpp_move(double v)
{
    return dpp_move_f64<kCtrl>(v);
}

// Maximum with the lane 16 away (lane ^ 16).
__device__ __forceinline__ float max_across_16(float v)
{
    const auto pair = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(pair[0]), __uint_as_float(pair[1]));
}
__device__ __forceinline__ double max_across_16(double v) { return fmax(v, __shfl_xor(v, 16, 64)); }

__device__ __forceinline__ double half_bits_to_double(uint16_t h)
{
    return (double)(float)__builtin_bit_cast(_Float16, h);
}

// sigma = fp16(sqrt(rmax)), round to nearest even, saturating.  The fp32 square root is within
// 2 ulp(fp32) of the exact one, so it rounds to the same fp16 value unless it lies within a few
// fp32 ulp of a rounding boundary (the 13 dropped bits close to 0x1000) or the result is
// subnormal; only then is the fp64 recipe run.
__device__ __forceinline__ uint16_t sigma_of_row_max(double rmax)
{
    const float sf = __builtin_amdgcn_sqrtf((float)rmax);  // 1 ulp; a flushed subnormal takes the fp64 recipe below
    const uint32_t sb = __float_as_uint(sf);
    const int dist = (int)(sb & 0x1fffu) - 0x1000;
    const bool slow = rmax != 0.0 && sf < 65504.f && (sf < 0x1.0p-14f || (dist >= -8 && dist <= 8));
    uint16_t sigma16 = sf >= 65504.f ? (uint16_t)0x7bff : __builtin_bit_cast(uint16_t, (_Float16)sf);
    if (__any(slow)) {
        if (slow)
            sigma16 = double_to_half_rne_sat(sqrt(rmax));
    }
    return sigma16;
}

// Whether sigma_of_row_max has to take the fp64 recipe: sf the fp32 square root, at most 65504.  It is within 4 units of the
// last place: 1 of the instruction, 3 / 2 roundings of 2^-24 of an fp32 argument.
__device__ __forceinline__ bool scale_unsure(float sf)
{
    const uint32_t bits = __float_as_uint(sf);
    return ((bits - (0x1000u - 8u)) & 0x1fffu) <= 16u || bits - 1u < 0x387fffffu;  // next to a midpoint; below 2^-14, not zero
}

__device__ __forceinline__ int radius_code_exact(double r2, uint16_t sigma16, double Lq)
{
    const double sigma = half_bits_to_double(sigma16);
    double q = rint((sqrt(r2) * Lq) / sigma);
    q = q < 0.0 ? 0.0 : (q > Lq ? Lq : q);
    return (int)q;
}

// Radius code r_q = clamp(rint(sqrt(r2) * L / sigma), 0, L), defined in fp64.  An fp32
// evaluation with the hardware's 1-ulp square root (r_f) and reciprocal is off by at most
// 6e-7 * L (five roundings of <= 1.2e-7 each); it rounds the same way unless it lands within
// that distance of a rounding boundary, and only then is the fp64 recipe run (about one wave
// in two hundred at L = 63).
__device__ __forceinline__ int radius_code(double r2, float r_f, uint16_t sigma16, double Lq)
{
    int rq = 0;
    const float sigma_f = (float)__builtin_bit_cast(_Float16, sigma16);
    bool exact_needed = false;
    if (sigma16 != 0 && r2 != 0.0) {
        const float qf = fminf(r_f * (float)Lq * __builtin_amdgcn_rcpf(sigma_f), (float)Lq);
        const float fr = qf - floorf(qf);
        exact_needed = fabsf(fr - 0.5f) < 6e-7f * (float)Lq + 1e-6f;
        rq = (int)rintf(qf);
    }
    if (__any(exact_needed)) {
        if (exact_needed)
            rq = radius_code_exact(r2, sigma16, Lq);
    }
    return rq;
}

// Direction of a chunk in fp32: kOperandScale times the unit vector (zeros for a zero chunk).
struct Direction {
    float u0, u1, u2, u3;
};
__device__ __forceinline__ Direction unit_direction(const half4_t xv, double r2, float r_f)
{
    // times kOperandScale, the factor the matrix operands carry: a power of two, so every comparison
    // between scores comes out as for the unit vector itself
    const float inv = r2 != 0.0 ? __builtin_amdgcn_rcpf(r_f) * kOperandScale : 0.f;
    Direction d;
    d.u0 = (float)xv[0] * inv;
    d.u1 = (float)xv[1] * inv;
    d.u2 = (float)xv[2] * inv;
    d.u3 = (float)xv[3] * inv;
    return d;
}

typedef float float16_t __attribute__((ext_vector_type(16)));

// Two groups of secondaries whose screened maxima lie closer than this fraction of the larger one are
// not told apart by the screen.  Its error is below 7e-7 |q_s| per score (operands carried to 2^-24 each,
// fp32 accumulation, three fp32 additions; 2.9e-7 measured), the best score is at least |q_s| / sqrt(2),
// so the band is at least three times that bound on the error of the two scores compared (seven times
// the measured value), whatever the common scale
// (the scores of the matrix pass carry a factor kOperandScale^2 = 2^20).
constexpr float kScreenBand = 6.0e-6f;

// Exhaustive nearest-codeword search for the wave's 64 chunks (one per lane, direction u as
// unit_direction returns it): returns
// the chunk's code word (rq << w_idx) | k with k = p S + s of the best joint codeword; 0 for a
// flagged chunk (also to be passed for a lane without a chunk) and for a zero chunk (r2 == 0).
// Called by all 64 lanes.  amat / secl: the head's A operands and secondaries in LDS.
//
// Three steps.  Screen: all S secondaries on the matrix cores with operands split in two fp16
// parts; lane (col = l % 32, half = l / 32) sees, for the chunks col and 32 + col, the secondaries
// 16 grp + 2 t + half (t = 0..7) of every group grp, and keeps per chunk slot the best group, its
// score and the runner-up score.  Decide: the two lanes of a chunk exchange their results; a clear
// winner (ahead of every other lane-group by more than the band) names 8 candidate secondaries, which
// are scored again in fp32.  Otherwise (a few chunks in a thousand) the wave scores all S secondaries
// of that chunk in fp32, 64 at a time.  The decision between secondaries is therefore always taken
// on fp32 closed-form scores, the lowest s winning exact ties.
//
// kCoop (a workgroup whose rows fill a single pass): all waves of the workgroup hold the same 64
// chunks, each screens its share of the groups, the per-chunk results (best lane-group, its score, the
// runner-up) meet in `merge` [kSearchWaves][64][3], and wave 0 alone decides and returns the code words (the other
// waves return 0).  The merged triple is what one wave screening every group would have found, except when two
// waves tie for the best score exactly; the runner-up then equals the best and the chunk takes the fp32 search,
// as any tie between groups does.
template <bool kCoop = false, bool kScreen = true>
__device__ __forceinline__ uint32_t search_codeword(const Geometry &g, int lane, const Direction u, bool flagged,
                                                    double r2, int rq, const uint4 *amat, const float *secl,
                                                    int wv = 0, float *merge = nullptr)
{
    const float u0 = opaque(u.u0), u1 = opaque(u.u1), u2 = opaque(u.u2), u3 = opaque(u.u3);
    const int half = lane >> 5;
    // B operands: lane (col, half) supplies components 2 half, 2 half + 1 of chunk 32 j + col in the
    // slots [h l h l | h l h l]; chunk 32 half + col is its own, the other one its partner's (lane ^ 32)
    half8_t bop[2];
    {
        const Parts2 p0 = split2(u0), p1 = split2(u1), p2 = split2(u2), p3 = split2(u3);
        const uint32_t k0 = pack2(p0.h, p0.l), k1 = pack2(p1.h, p1.l), k2 = pack2(p2.h, p2.l), k3 = pack2(p3.h, p3.l);
        const uint32_t own_a = half ? k2 : k0, own_b = half ? k3 : k1;
        const uint32_t snd_a = half ? k0 : k2, snd_b = half ? k1 : k3;
        const uint32_t rcv_a = (uint32_t)__shfl_xor((int)snd_a, 32, 64), rcv_b = (uint32_t)__shfl_xor((int)snd_b, 32, 64);
        const uint32_t j0a = half ? rcv_a : own_a, j0b = half ? rcv_b : own_b;
        const uint32_t j1a = half ? own_a : rcv_a, j1b = half ? own_b : rcv_b;
        bop[0] = __builtin_bit_cast(half8_t, make_uint4(j0a, j0a, j0b, j0b));
        bop[1] = __builtin_bit_cast(half8_t, make_uint4(j1a, j1a, j1b, j1b));
    }

    // ---- screen ----------------------------------------------------------------------------------------
    float best[2] = {-1.f, -1.f}, second[2] = {-1.f, -1.f};
    int bkey[2] = {0, 0};
    float16_t zero16;
#pragma unroll
    for (int e = 0; e < 16; ++e)
        zero16[e] = 0.f;
    // groups this wave screens: those held as matrix operands (none beyond kScreenMaxS secondaries: the
    // screen is then skipped and every chunk takes the fp32 search below)
    const int n_grp = kScreen ? g.S16 : 0;
    const int per_wave = kCoop ? (n_grp + kSearchWaves - 1) / kSearchWaves : n_grp;
    const int grp_begin = kCoop ? min(wv * per_wave, n_grp) : 0;
    const int grp_end = kCoop ? min(grp_begin + per_wave, n_grp) : n_grp;
    const uint4 *arow = amat + lane;
    half8_t a0 = __builtin_bit_cast(half8_t, make_uint4(0u, 0u, 0u, 0u)), a1 = a0;
    float16_t ahead = zero16;
    if (kScreen) {
        a0 = __builtin_bit_cast(half8_t, arow[2 * min(grp_begin, n_grp - 1) * 64]);
        a1 = __builtin_bit_cast(half8_t, arow[2 * min(grp_begin, n_grp - 1) * 64 + 64]);
        // the product of (tile 0, chunk slot 0) of the next group is issued before the arithmetic on the last
        // product of this one: a VALU instruction right behind the MFMA it depends on idles for the depth of
        // the matrix pipeline
        ahead = __builtin_amdgcn_mfma_f32_32x32x16_f16(a0, bop[0], zero16, 0, 0, 0);
    }
    for (int grp = grp_begin; grp < grp_end; ++grp) {
        // the next group's operands replace this group's as soon as their last product is issued (the
        // last group re-reads itself; that product is dropped)
        const uint4 *anext = arow + 2 * min(grp + 1, n_grp - 1) * 64;
        // over the group's 8 secondaries on this lane: GA = largest |v_i| (best axis element), GH = largest
        // |v_0|+|v_1|+|v_2|+|v_3| (twice the best half-integer element)
        float GA[2], GH[2];
#pragma unroll
        for (int k = 0; k < 4; ++k) {  // (tile k / 2, chunk slot k % 2)
            const int j = k & 1;
            const float16_t c = ahead;
            if (k == 0) {
                ahead = __builtin_amdgcn_mfma_f32_32x32x16_f16(a0, bop[1], zero16, 0, 0, 0);
                a0 = __builtin_bit_cast(half8_t, anext[0]);
            } else if (k == 1) {
                ahead = __builtin_amdgcn_mfma_f32_32x32x16_f16(a1, bop[0], zero16, 0, 0, 0);
            } else if (k == 2) {
                ahead = __builtin_amdgcn_mfma_f32_32x32x16_f16(a1, bop[1], zero16, 0, 0, 0);
                a1 = __builtin_bit_cast(half8_t, anext[64]);
            } else {
                ahead = __builtin_amdgcn_mfma_f32_32x32x16_f16(a0, bop[0], zero16, 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
            float t[16], h[4];
#pragma unroll
            for (int e = 0; e < 16; ++e)
                t[e] = fabsf(c[e]);
#pragma unroll
            for (int i = 0; i < 4; ++i)  // secondary i of the tile's four
                h[i] = ((t[4 * i] + t[4 * i + 1]) + t[4 * i + 2]) + t[4 * i + 3];
            // v_max3 chains; the group's first tile starts them from its own values (|v| >= 0: no zero needed)
            float ga, gh;
            if (k < 2) {
                ga = fmaxf(fmaxf(t[0], t[1]), t[2]);
#pragma unroll
                for (int e = 3; e < 15; e += 2)
                    ga = fmaxf(fmaxf(ga, t[e]), t[e + 1]);
                ga = fmaxf(ga, t[15]);
                gh = fmaxf(fmaxf(fmaxf(h[0], h[1]), h[2]), h[3]);
            } else {
                ga = GA[j];
#pragma unroll
                for (int e = 0; e < 16; e += 2)
                    ga = fmaxf(fmaxf(ga, t[e]), t[e + 1]);
                gh = fmaxf(fmaxf(fmaxf(fmaxf(GH[j], h[0]), h[1]), h[2]), h[3]);
            }
            GA[j] = ga;
            GH[j] = gh;
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const float M = fmaxf(GA[j], 0.5f * GH[j]);
            second[j] = __builtin_amdgcn_fmed3f(M, best[j], second[j]);  // second <= best on entry
            if (M > best[j]) {
                best[j] = M;
                bkey[j] = 16 * grp;
            }
        }
    }

    // ---- decide: chunk 32 j + col was screened by lanes col and 32 + col (slot j of each) and is
    // owned by lane 32 j + col, i.e. slot `half` of the owner and of its partner ------------------------
    const float my_b = half ? best[1] : best[0], my_s = half ? second[1] : second[0];
    const int my_k = half ? bkey[1] : bkey[0];
    const float ot_b = __shfl_xor(half ? best[0] : best[1], 32, 64);
    const float ot_s = __shfl_xor(half ? second[0] : second[1], 32, 64);
    const int ot_k = __shfl_xor(half ? bkey[0] : bkey[1], 32, 64);
    const bool other = ot_b > my_b;
    float top = other ? ot_b : my_b;
    float runner = fmaxf(fmaxf(fminf(my_b, ot_b), my_s), ot_s);
    int first = (other ? ot_k : my_k) + (other ? 1 - half : half);  // candidates first + 2 t
    if (kCoop) {
        float *mine = merge + (wv * 64 + lane) * 3;
        mine[0] = top;
        mine[1] = runner;
        mine[2] = __int_as_float(first);
        __syncthreads();
        if (wv != 0)
            return 0u;
#pragma unroll
        for (int k = 1; k < kSearchWaves; ++k) {  // a wave without groups left its initial -1: never the best
            const float *theirs = merge + (k * 64 + lane) * 3;
            const float tb = theirs[0], tr = theirs[1];
            const int tf = __float_as_int(theirs[2]);
            const bool better = tb > top;
            runner = fmaxf(fmaxf(fminf(top, tb), runner), tr);
            first = better ? tf : first;
            top = better ? tb : top;
        }
    }
    const bool live = !flagged && r2 != 0.0;
    const bool unclear = live && (!kScreen || !(top - runner >= kScreenBand * top));

    // The 8 candidates first + 2 t in ascending order, strict comparison: the lowest s wins a tie.  Padding
    // secondaries (zeros, s >= S) score 0 and every real one scores at least |q_s| / sqrt(2) > 0 for a
    // non-zero chunk, so a group that won the screen never yields a padding index; the bound below only
    // keeps the index inside the codebook should the input break the contract (non-finite values).
    int bs = first;
    if (live && kScreen) {
        const float *cq = secl + 4 * first;  // < 16 S16 entries: inside the padded table
        float bsc = -1.f;
        int bt = 0;
#pragma unroll
        for (int tt = 0; tt < 8; ++tt) {
            float v0, v1, v2, v3;
            const float sc = score_secondary(cq + 8 * tt, u0, u1, u2, u3, v0, v1, v2, v3);
            const bool take = sc > bsc;
            bsc = take ? sc : bsc;
            bt = take ? tt : bt;
        }
        bs = min(first + 2 * bt, g.S - 1);
    }
    // the unclear chunks, one at a time: every lane scores the secondaries lane, lane + 64, ...; the key
    // orders by score, then by descending s (scores are positive, so their bit patterns order like them).
    // Without a screen they are all of them, two steps of 64 secondaries at a time (the last one over again past the end): with
    // a bound per lane it was bound by latency, and the same instructions have taken 3 to 9 % longer at another place in the code.
    // In us, before / now: 40 tensors of 16 x 3 rows of 64, S = 600 138 / 120, S = 2730 456 / 382; two of 8 x 2000 rows of 96, S =
    // 1024 791 / 766.
    unsigned long long todo = __ballot(unclear);
    while (todo) {  // wave-uniform
        const int src = __ffsll((long long)todo) - 1;
        todo &= todo - 1ull;
        const float e0 = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(u0), src));
        const float e1 = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(u1), src));
        const float e2 = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(u2), src));
        const float e3 = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(u3), src));
        unsigned long long key = 0ull;
        const auto score = [&](int s) {
            float v0, v1, v2, v3;
            const float sc = score_secondary(secl + 4 * s, e0, e1, e2, e3, v0, v1, v2, v3);
            key = umax64(key, ((unsigned long long)__float_as_uint(sc) << 32) | (0xffffffffu - (uint32_t)s));
        };
        if (kScreen) {
            for (int s = lane; s < g.S; s += 64)
                score(s);
        } else {
#pragma unroll 2
            for (int s0 = 0; s0 < g.S; s0 += 64)
                score(min(s0 + lane, g.S - 1));
        }
        key = wave_umax64(key);
        if (lane == src)
            bs = (int)min(0xffffffffu - (uint32_t)key, (uint32_t)g.S - 1u);
    }

    uint32_t code = 0;
    if (live) {
        float w0, w1, w2, w3, sc;
        (void)score_secondary(secl + 4 * bs, u0, u1, u2, u3, w0, w1, w2, w3);
        const int p = nearest_primary(w0, w1, w2, w3, sc);
        code = ((uint32_t)rq << g.w_idx) | (uint32_t)(p * g.S + bs);
    }
    return code;
}

// Outlier offsets local to the workgroup of kRows rows from t0 on, and its total; the global prefix is added by the
// scan / gather kernels that follow.  Called by one wave.
template <int kRows>
__device__ __forceinline__ void write_row_offsets(const Geometry &g, const Workspace &ws, const EncodedPtrs &enc, int lane,
                                                  int seg, int t0, const uint2 *state)
{
    uint32_t carry = 0;
#pragma unroll
    for (int part = 0; part < kRows / 64; ++part) {
        const int r = 64 * part + lane;
        const uint32_t cnt = t0 + r < g.T ? __popc(state[r].x) : 0u, inc = wave_scan(cnt);
        if (t0 + r < g.T)
            enc.row_off[(int64_t)seg * g.T + t0 + r] = carry + inc - cnt;
        carry += (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
    }
    if (lane == 0)
        ws.block_sum[(size_t)seg * g.n_search_blocks_per_seg + blockIdx.x] = carry;
}

}  // namespace

// The K = 4 contraction v = A(q_s) u on v_mfma_f32_32x32x16_f16: a product covers 8 secondaries (32 rows =
// 8 x 4 components of v) and 32 chunks (columns); its K = 16 are the 4 terms of the contraction times the
// 4 products of a two-part split (both operands are scaled by 2^10 first so that the low parts stay
// normal).  Lane l of an operand holds row (column) l % 32 and the terms 2 (l / 32), 2 (l / 32) + 1, each in
// four fp16 slots: A as [h h l l], B as [h l h l].  The four fp16 x fp16 products are exact in fp32 and
// add up inside the matrix core.  Lane l of the result holds, for column l % 32, the rows
// 8 i + 4 (l / 32) + c (i, c = 0..3): all four components of v for the secondaries 2 i + l / 32 of the tile.
// The scores come out scaled by 2^20, which no comparison notices.
//
// Dynamic LDS layout:
//   amat  [2*S16][64] x 16 B   MFMA A operands, one 64-lane tile per 8 secondaries
//                              (copied from the table that the call's first kernel built for the head)
//   secl  [16*S16][4] f32      the head's secondaries (zero padded to a multiple of 16)
//   pack  [kSearchWaves][2][32] u32 row code words being assembled
//   rcnt  [search_rows] u32    outliers per row of the workgroup
// This kernel is for rows of 128 elements (32 chunks: two rows per wave); k_search_flat below takes
// every other head dimension.
// kFused: the form for tensors of a few rows whose thresholds are known beforehand (appended tokens with
// supplied thresholds, extraction switched off): no kernel runs before this one, so it takes its thresholds
// from the caller's array (+infinity without one), builds the head's operand table itself, and reports a
// non-finite input through bit 31 of its workgroup total, which the list kernel turns into the status word.
template <bool kFused = false, bool kScreen = true>
__global__ __launch_bounds__(64 * kSearchWaves, kFused ? 1 : 4) void k_search(Geometry g, WorkspaceOffsets wo, EncodeBatch batch)
{
    constexpr int kThreadsS = 64 * kSearchWaves;
    const EncodeTensor &tn = batch.t[blockIdx.z];
    const Workspace ws = carve_workspace(tn.ws, wo);
    const EncodedPtrs enc = tn.enc;
    const _Float16 *__restrict__ x = tn.x;
    const float *__restrict__ sec = tn.sec;
    extern __shared__ float smem[];
    uint4 *amat = reinterpret_cast<uint4 *>(smem);
    float *secl = reinterpret_cast<float *>(amat + (size_t)(kScreen ? g.S16 : 0) * kATiles * 64);
    uint32_t *pack = reinterpret_cast<uint32_t *>(secl + (size_t)g.S16 * 16 * 4);
    uint32_t *rcnt = pack + kSearchWaves * 2 * 32;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform, and known to be
    // by_head (kFused, several batch entries of a few rows each): one workgroup per head takes the rows of all
    // batch entries, so that the head's tables are built once; its rows are the pairs (b, t), b-major
    const bool by_head = kFused && g.fused_by_head != 0;
    const int seg = blockIdx.y, b = by_head ? 0 : seg / g.H, h = by_head ? seg : seg % g.H;
    const int rows = g.search_rows;  // of a workgroup: 2 kSearchWaves to 64
    const int t0 = blockIdx.x * rows;
    const int n_here = by_head ? g.B * g.T : g.T;  // rows this workgroup column addresses
    const float *sec_h = sec + (size_t)h * g.S * 4;
    // row v of the column: its batch entry and token, the address of its chunk c, its linear row index
    struct RowAt {
        const _Float16 *chunk;
        int64_t R;
    };
    auto row_at = [&](int v, int c) {
        const int bb = by_head ? v / g.T : b;
        const int tt = by_head ? v - bb * g.T : v;
        RowAt r;
        r.chunk = x + (int64_t)bb * g.sb + (int64_t)h * g.sh + (int64_t)tt * g.st + 4 * c;
        r.R = ((int64_t)bb * g.H + h) * g.T + tt;
        return r;
    };
    // kFused (a launch of a few rows, bound by latency): a workgroup with one or two rows (one appended token)
    // runs its single pass on all its waves together (search_codeword's cooperative form), and the first
    // chunk is requested before the tables
    const bool coop = kFused && n_here - t0 <= 2;  // uniform over the workgroup
    __shared__ float merge[kFused ? kSearchWaves * 64 * 3 : 1];
    half4_t first_chunk = {0, 0, 0, 0};
    if (kFused) {
        const int v = t0 + (coop ? 0 : wv * 2) + (lane >> 5);
        if (v < n_here)
            first_chunk = load_chunk(row_at(v, lane & 31).chunk);
    }

    // ---- setup: secondaries and A operands into LDS ---------------------------------------
    for (int s = tid; s < g.S16 * 16; s += kThreadsS) {
        float4_t q = {0.f, 0.f, 0.f, 0.f};
        if (s < g.S)
            q = *reinterpret_cast<const float4_t *>(sec_h + 4 * s);
        *reinterpret_cast<float4_t *>(secl + 4 * s) = q;
    }
    if (kFused) {
        for (int idx = tid; idx < (kScreen ? g.S16 : 0) * kATiles * 64; idx += kThreadsS)
            amat[idx] = operand_entry(sec_h, g.S, idx);
        if (coop)  // the one pass writes the counters of rows 0 and 1 only
            for (int r = tid; r < rows; r += kThreadsS)
                rcnt[r] = 0;
    } else {
        const uint4 *src = ws.aop + (size_t)h * (kScreen ? g.S16 : 0) * kATiles * 64;
        for (int idx = tid; idx < (kScreen ? g.S16 : 0) * kATiles * 64; idx += kThreadsS)
            amat[idx] = src[idx];
    }

    __syncthreads();

    const double thr = !kFused ? ws.thr[h] : tn.thr_given ? tn.thr_given[h] : __longlong_as_double(0x7ff0000000000000LL);
    if (kFused && blockIdx.x == 0 && b == 0 && tid == 0)
        ws.thr[h] = thr;  // what hqmq_thresholds reads back
    uint32_t bad_seen = 0;  // kFused: this lane saw a ballot with a non-finite chunk in it
    const double Lq = (double)((1 << g.b_r) - 1);
    const int c = lane & 31, half_id = lane >> 5;
    uint32_t *my_pack = pack + wv * 64;

    const int n_it = coop ? 1 : rows / (2 * kSearchWaves);
    for (int it = 0; it < n_it; ++it) {
        const int r_in_block = coop ? half_id : it * 2 * kSearchWaves + wv * 2 + half_id;
        const int t = t0 + r_in_block;
        const bool valid = t < n_here;
        if (!coop && t0 + it * 2 * kSearchWaves + wv * 2 >= n_here) {  // wave-uniform: both rows of this iteration lie past the end
            if (c == 0)
                rcnt[r_in_block] = 0;
            continue;
        }

        // ---- chunk, norm, flag, row scale --------------------------------------------------
        const RowAt here = row_at(valid ? t : t0, c);
        half4_t xv = (kFused && it == 0) ? first_chunk : valid ? load_chunk(here.chunk) : half4_t{0, 0, 0, 0};
        const double r2 = chunk_norm2(xv);
        const bool flagged = valid && (r2 > thr);
        const unsigned long long ballot = __ballot(flagged);
        const uint32_t word = half_id ? (uint32_t)(ballot >> 32) : (uint32_t)ballot;
        if (g.check_finite) {  // uniform
            const bool bad = valid && chunk_nonfinite(xv);
            if (__ballot(bad) != 0ull) {
                if (kFused)
                    bad_seen = 1u;
                else if (lane == 0)
                    atomicOr(enc.status, HQMQ_STATUS_NONFINITE);
            }
        }

        // max over the 32 lanes of the row: four DPP steps inside each 16-lane row (after each step the
        // running maxima are uniform over a block twice as large, so the mirror patterns pair the right
        // blocks), one swap across rows
        double rmax = flagged ? 0.0 : r2;
        rmax = fmax(rmax, dpp_move_f64<0xB1>(rmax));   // quad_perm [1, 0, 3, 2]
        rmax = fmax(rmax, dpp_move_f64<0x4E>(rmax));   // quad_perm [2, 3, 0, 1]
        rmax = fmax(rmax, dpp_move_f64<0x141>(rmax));  // row_half_mirror
        rmax = fmax(rmax, dpp_move_f64<0x140>(rmax));  // row_mirror
        rmax = fmax(rmax, __shfl_xor(rmax, 16, 64));
        const uint16_t sigma16 = sigma_of_row_max(rmax);
        const float r_f = __builtin_amdgcn_sqrtf((float)r2);
        const int rq = radius_code(r2, r_f, sigma16, Lq);
        const Direction u = unit_direction(xv, r2, r_f);
        my_pack[lane] = 0;  // after the previous iteration's reads of it: LDS serves a wave in order
        uint32_t code;
        if (coop) {
            code = search_codeword<true>(g, lane, u, flagged, r2, rq, amat, secl, wv, merge);
            if (wv != 0)
                continue;  // wave 0 holds the result and writes the two rows
        } else {
            code = search_codeword<false, kScreen>(g, lane, u, flagged, r2, rq, amat, secl);
        }

        // ---- pack the row: chunk c at bits [c*w, (c+1)*w) -----------------------------------------
        {
            uint32_t bitpos = (uint32_t)c * g.w;
            uint32_t d0 = bitpos >> 5, sh = bitpos & 31;
            uint32_t *rowp = my_pack + half_id * 32;
            if (code) {
                atomicOr(&rowp[d0], code << sh);
                if (sh + g.w > 32)
                    atomicOr(&rowp[d0 + 1], code >> (32 - sh));
            }
        }
        wave_lds_sync();
        if (valid) {
            const int64_t R = here.R;
            if (c < g.w)
                enc.codes[R * g.w + c] = my_pack[half_id * 32 + c];
            if (c == 0) {
                enc.sigma[R] = sigma16;
                enc.flags[R] = word;
            }
        }
        if (c == 0)
            rcnt[r_in_block] = valid ? __popc(word) : 0;
    }

    // ---- outlier offsets local to the workgroup and its total; the global prefix is added by the
    // scan / gather kernels that follow --------------------------------------------------------------
    const uint32_t bad_any = kFused ? (uint32_t)__syncthreads_or((int)bad_seen) : (__syncthreads(), 0u);
    if (wv == 0) {
        const int r = lane;  // a lane per row
        const uint32_t cnt = r < rows ? rcnt[r] : 0u, inc = wave_scan(cnt);
        if (by_head) {
            // every batch entry's rows are a run of their own in the list's order: offsets restart at each run, and each run
            // reports its total as a workgroup would
            const int run = r / g.T, start = run * g.T;
            const uint32_t before_run = __shfl(inc - cnt, min(start, 63), 64);
            if (r < n_here) {
                enc.row_off[row_at(r, 0).R] = inc - cnt - before_run;
                if (r - start == g.T - 1)
                    ws.block_sum[(size_t)run * g.H + h] = (inc - before_run) | (bad_any ? 0x80000000u : 0u);
            }
        } else if (r < rows && t0 + r < g.T) {
            enc.row_off[row_at(t0 + r, 0).R] = inc - cnt;
        }
        const uint32_t carry = (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
        if (lane == 0 && !by_head)  // a workgroup holds at most 512 x 32 outliers: bit 31 is free for the flag
            ws.block_sum[(size_t)seg * g.n_search_blocks_per_seg + blockIdx.x] = carry | (bad_any ? 0x80000000u : 0u);
    }
}


// The same search for any head dimension: rows of n_c = ceil(D / 4) <= 32 chunks.  A workgroup owns
// 8 to 64, or 256, rows of one (b, h) segment and treats their chunks as one flat list, 64 consecutive
// chunks per wave and iteration, so that every lane of every matrix product carries a chunk whatever
// n_c is.  Rows then straddle waves, so what the row-per-half-wave kernel does with cross-lane
// operations goes through LDS here:
//   pass 1  every chunk's squared norm once: flagged chunks set their bit in the row's flag word,
//           the others take part in the row's maximum (atomics on LDS); one lane per row then turns
//           the maximum into the fp16 scale and writes scale and flag word out;
//   pass 2  the chunks again (second read from L2): radius code against the row's scale, direction
//           search, code word OR-ed into the row's slot of the packing area;
//   end     the packing area goes out as one contiguous block, then the outlier offsets as above.
// Dynamic LDS: amat | secl as in k_search, then rowmax u64 [kRows] | fword u32 [kRows] |
// sig u32 [kRows] | rcnt u32 [kRows] | pack u32 [kRows * row_words].
// kFused: as in k_search.
template <bool kFused = false, bool kScreen = true>
__global__ __launch_bounds__(64 * kSearchWaves) void k_search_flat(Geometry g, WorkspaceOffsets wo, EncodeBatch batch)
{
    constexpr int kThreadsS = 64 * kSearchWaves;
    const EncodeTensor &tn = batch.t[blockIdx.z];
    const Workspace ws = carve_workspace(tn.ws, wo);
    const EncodedPtrs enc = tn.enc;
    const _Float16 *__restrict__ x = tn.x;
    const int rows_wg = g.search_rows;  // of a workgroup: 8 to 64, or 256 on 4 waves; a thread per row in the scale pass
    extern __shared__ float smem[];
    uint4 *amat = reinterpret_cast<uint4 *>(smem);
    float *secl = reinterpret_cast<float *>(amat + (size_t)(kScreen ? g.S16 : 0) * kATiles * 64);
    unsigned long long *rowmax = reinterpret_cast<unsigned long long *>(secl + (size_t)g.S16 * 16 * 4);
    uint32_t *fword = reinterpret_cast<uint32_t *>(rowmax + rows_wg);
    uint32_t *sig = fword + rows_wg;
    uint32_t *rcnt = sig + rows_wg;
    uint32_t *pack = rcnt + rows_wg;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int seg = blockIdx.y, b = seg / g.H, h = seg % g.H;
    const int t0 = blockIdx.x * rows_wg;
    const int nrows = min(rows_wg, g.T - t0);       // >= 1 by the grid's size
    const int nchunks = nrows * g.n_c;
    const int row_words = g.row_words;
    const int64_t row0 = (int64_t)seg * g.T + t0;  // linear index of the workgroup's first row
    const float *sec_h = tn.sec + (size_t)h * g.S * 4;

    // ---- setup: tables into LDS, per-row state cleared ------------------------------------------
    for (int s = tid; s < g.S16 * 16; s += kThreadsS) {
        float4_t q = {0.f, 0.f, 0.f, 0.f};
        if (s < g.S)
            q = *reinterpret_cast<const float4_t *>(sec_h + 4 * s);
        *reinterpret_cast<float4_t *>(secl + 4 * s) = q;
    }
    if (kFused) {
        for (int idx = tid; idx < (kScreen ? g.S16 : 0) * kATiles * 64; idx += kThreadsS)
            amat[idx] = operand_entry(sec_h, g.S, idx);
    } else {
        const uint4 *src = ws.aop + (size_t)h * (kScreen ? g.S16 : 0) * kATiles * 64;
        for (int idx = tid; idx < (kScreen ? g.S16 : 0) * kATiles * 64; idx += kThreadsS)
            amat[idx] = src[idx];
    }
    for (int i = tid; i < rows_wg; i += kThreadsS) {
        rowmax[i] = 0ull;
        fword[i] = 0u;
    }
    for (int i = tid; i < rows_wg * row_words; i += kThreadsS)
        pack[i] = 0u;
    __syncthreads();

    const double thr = !kFused ? ws.thr[h] : tn.thr_given ? tn.thr_given[h] : __longlong_as_double(0x7ff0000000000000LL);
    if (kFused && blockIdx.x == 0 && b == 0 && tid == 0)
        ws.thr[h] = thr;  // what hqmq_thresholds reads back
    uint32_t bad_seen = 0;
    const double Lq = (double)((1 << g.b_r) - 1);
    const _Float16 *base = x + (int64_t)b * g.sb + (int64_t)h * g.sh + (int64_t)t0 * g.st;

    // ---- pass 1: flags and row maxima ---------------------------------------------------------------
    for (int q = tid; q < nchunks; q += kThreadsS) {
        const int r = row_of_chunk(q, g), c = q - r * g.n_c;
        const half4_t xv = load_row_chunk<false>(base + (int64_t)r * g.st, c, g);
        const double r2 = chunk_norm2(xv);
        if (g.check_finite && chunk_nonfinite(xv)) {
            if (kFused)
                bad_seen = 1u;
            else
                atomicOr(enc.status, HQMQ_STATUS_NONFINITE);
        }
        if (r2 > thr)
            atomicOr(&fword[r], 1u << c);
        else
            atomicMax(&rowmax[r], key_of(r2));  // non-negative doubles order like their bit patterns
    }
    const uint32_t bad_any = kFused ? (uint32_t)__syncthreads_or((int)bad_seen) : (__syncthreads(), 0u);
    if (tid < rows_wg) {
        uint32_t word = 0;
        if (tid < nrows) {
            word = fword[tid];
            const uint16_t sigma16 = sigma_of_row_max(__longlong_as_double((long long)rowmax[tid]));
            sig[tid] = sigma16;
            enc.sigma[row0 + tid] = sigma16;
            enc.flags[row0 + tid] = word;
        }
        rcnt[tid] = __popc(word);
    }
    __syncthreads();

    // ---- pass 2: radius codes and the direction search ----------------------------------------------
    for (int q0 = wv * 64; q0 < nchunks; q0 += kThreadsS) {  // wave-uniform trip count
        const int q = q0 + lane;
        const bool valid = q < nchunks;
        const int r = valid ? row_of_chunk(q, g) : 0, c = valid ? q - r * g.n_c : 0;
        const half4_t xv = valid ? load_row_chunk<false>(base + (int64_t)r * g.st, c, g) : half4_t{0, 0, 0, 0};
        const double r2 = chunk_norm2(xv);
        const bool flagged = valid && (r2 > thr);
        const uint16_t sigma16 = (uint16_t)sig[r];
        const float r_f = __builtin_amdgcn_sqrtf((float)r2);
        const int rq = radius_code(r2, r_f, sigma16, Lq);
        const Direction u = unit_direction(xv, r2, r_f);
        const uint32_t code = search_codeword<false, kScreen>(g, lane, u, flagged || !valid, r2, rq, amat, secl);
        if (code) {
            const uint32_t bitpos = (uint32_t)c * g.w;
            const uint32_t d0 = bitpos >> 5, sh = bitpos & 31;
            uint32_t *rowp = pack + r * row_words;
            atomicOr(&rowp[d0], code << sh);
            if (sh + g.w > 32)
                atomicOr(&rowp[d0 + 1], code >> (32 - sh));
        }
    }
    __syncthreads();

    // ---- the workgroup's code words: one contiguous block ------------------------------------------
    {
        uint32_t *dst = enc.codes + row0 * row_words;
        for (int i = tid; i < nrows * row_words; i += kThreadsS)
            dst[i] = pack[i];
    }
    // ---- outlier offsets local to the workgroup and its total ---------------------------------------
    if (wv == 0) {
        uint32_t carry = 0;
        for (int r0 = 0; r0 < rows_wg; r0 += 64) {
            const int r = r0 + lane;
            const uint32_t cnt = r < rows_wg ? rcnt[r] : 0u, inc = wave_scan(cnt);
            if (r < nrows)
                enc.row_off[row0 + r] = carry + inc - cnt;
            carry += (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
        }
        if (lane == 0)
            ws.block_sum[(size_t)seg * g.n_search_blocks_per_seg + blockIdx.x] = carry | (bad_any ? 0x80000000u : 0u);
    }
}

// ---------------------------------------------------------------------------------------------------------------
// The rows that a generation step appends, thresholds known beforehand (or none): everything in one launch.
// Workgroup (segment, tensor) encodes the T rows of one (batch entry, head), or of a head in all batch entries, two at a time: all waves hold the same 64 chunks
// (a single row: its 32 chunks twice) and score a share of the secondaries each in fp32, which for so few rows is less work
// than the operand tables of a matrix screen (3840 vector instructions a row at S = 256, one operand table: 1920 and the
// screen).  The best of the shares, the lowest secondary on exact ties, is what the other searches find.
// The outlier list needs the outliers of the rows before a workgroup's, of other heads and batch entries: every workgroup
// counts those of the whole tensor itself (at most kAppendChunks chunks, four loads a thread in flight), so that no
// second launch and no order among workgroups is needed.
// Measured with 64 tensors of 8 heads, S = 256, in us, four launches (operand tables, screen and a list kernel for 32 tensors
// each) / now: one row per head 27 / 9, four rows 36 / 19, four batch entries 35 / 19, eight 38 / 31; two tensors 14.7 / 8.4.
// Bound by VALU issue from some thousand rows on and by the call's latency below.
// grid = (B * H, or H by head, tensors), block = 512.
// ---------------------------------------------------------------------------------------------------------------
constexpr int kAppendWaves = 8, kAppendThreads = 64 * kAppendWaves;
template <bool kFull>
__global__ __launch_bounds__(kAppendThreads) void k_append(AppendShape g, AppendBatch batch)
{
    const int tensor = blockIdx.y;
    auto part = [&](AppendPart p) { return ((uintptr_t)batch.high[p][tensor] << 32) | batch.low[p][tensor]; };
    const _Float16 *x = reinterpret_cast<const _Float16 *>(part(kAppX));
    const double *thr_given = reinterpret_cast<const double *>(part(kAppThr));
    const double never = __longlong_as_double(0x7ff0000000000000LL);

    __shared__ float4_t secl[kScreenMaxS];
    __shared__ uint32_t count[kAppendRows], any_bad;
    __shared__ float best_of[kAppendWaves][64];
    __shared__ int s_of[kAppendWaves][64];
    __shared__ uint32_t pack[64];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int b = g.by_head ? 0 : blockIdx.x / g.H, h = blockIdx.x - b * g.H;
    const int n_here = g.by_head ? g.B * g.T : g.T;  // rows of this workgroup: of all batch entries, or of one
    const int c = lane & 31, half = lane >> 5;
    const int n_rows = g.B * g.H * g.T, n_chunks = n_rows * g.n_c;
    const bool in_row = kFull || c < g.n_c;
    auto load_own = [&](int v, int &R) {  // chunk c of the workgroup's row v, and its linear row
        const int bb = g.by_head ? v / g.T : b, t = g.by_head ? v - bb * g.T : v;
        R = (bb * g.H + h) * g.T + t;
        half4_t xv = {0, 0, 0, 0};
        if (in_row)
            xv = load_row_chunk<kFull>(x + (int64_t)bb * g.sb + (int64_t)h * g.sh + (int64_t)t * g.st, c, g);
        return xv;
    };

    // ---- requested first: the first rows, the secondaries, the tensor's chunks for the count ---------------------------
    int R;
    half4_t xv = load_own(min(half, n_here - 1), R);
    float4_t q_own = {0.f, 0.f, 0.f, 0.f};
    if (tid < g.S)
        q_own = reinterpret_cast<const float4_t *>(part(kAppSec))[(size_t)h * g.S + tid];
    const double thr = thr_given ? thr_given[h] : never;
    const bool counts = thr_given != nullptr || g.check_finite != 0;  // uniform
    constexpr int kLoads = kAppendChunks / kAppendThreads;
    half4_t v[kLoads];
    double thr_of[kLoads];
    int row_of[kLoads];
    if (counts) {
#pragma unroll
        for (int u = 0; u < kLoads; ++u) {
            const int q = tid + u * kAppendThreads;
            v[u] = half4_t{0, 0, 0, 0};
            thr_of[u] = never;
            row_of[u] = 0;
            if (u * kAppendThreads < n_chunks && q < n_chunks) {
                const int r = row_of_chunk(q, g), sg = r / g.T, bb = sg / g.H, hh = sg - bb * g.H;
                row_of[u] = r;
                v[u] = load_row_chunk<kFull>(x + (int64_t)bb * g.sb + (int64_t)hh * g.sh + (int64_t)(r - sg * g.T) * g.st,
                                             q - r * g.n_c, g);
                if (thr_given)
                    thr_of[u] = thr_given[hh];
            }
        }
    }
    if (tid < kAppendRows)
        count[tid] = 0;
    if (tid == 0)
        any_bad = 0;
    if (tid < g.S)
        secl[tid] = q_own;
    __syncthreads();
    if (counts) {
#pragma unroll
        for (int u = 0; u < kLoads; ++u) {
            if (u * kAppendThreads < n_chunks) {  // uniform; past the end: zeros that nothing flags
                if (chunk_norm2(v[u]) > thr_of[u])
                    atomicAdd(&count[row_of[u]], 1u);
                if (g.check_finite && chunk_nonfinite(v[u]))
                    any_bad = 1u;
            }
        }
    }
    __syncthreads();
    // ---- wave 0: where each row's outliers start in the list, over the counts; totals -------------------------------------
    if (wv == 0) {
        static_assert(kAppendRows == 64, "a lane per row");
        const uint32_t mine = count[lane], inc = wave_scan(mine), total = (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
        uint32_t *n_outliers = reinterpret_cast<uint32_t *>(part(kAppCounts));
        if (b == 0) {
            uint32_t of_head = 0;
            for (int i = lane; i < g.B * g.T; i += 64) {
                const int bb = i / g.T;
                of_head += count[(bb * g.H + h) * g.T + i - bb * g.T];
            }
            of_head = (uint32_t)__builtin_amdgcn_readlane((int)wave_scan(of_head), 63);
            if (lane == 0) {
                n_outliers[h] = of_head;
                if (tensor + kMaxEncodeBatch >= g.n_tensors)
                    reinterpret_cast<double *>(g.thr_out + (uint64_t)(tensor % kMaxEncodeBatch) * g.thr_stride)[h] = thr;
            }
        }
        if (blockIdx.x == 0 && lane == 0) {
            n_outliers[g.H] = total;
            reinterpret_cast<uint32_t *>(part(kAppRowOff))[n_rows] = total;
            *reinterpret_cast<uint32_t *>(part(kAppStatus)) = (total > (uint32_t)batch.capacity[tensor] ? HQMQ_STATUS_OUTLIER_OVERFLOW : 0u) |
                                                              (any_bad ? HQMQ_STATUS_NONFINITE : 0u);
        }
        wave_lds_sync();
        count[lane] = inc - mine;
        wave_lds_sync();
    }

    const double Lq = (double)((1 << g.b_r) - 1);
    for (int v0 = 0; v0 < n_here; v0 += 2) {
        const bool single = v0 + 1 == n_here;  // uniform: both halves hold the same row
        if (v0 > 0)
            xv = load_own(min(v0 + half, n_here - 1), R);
        const double r2 = chunk_norm2(xv);
        const float r_f = __builtin_amdgcn_sqrtf((float)r2);
        const Direction u = unit_direction(xv, r2, r_f);
        const float u0 = opaque(u.u0), u1 = opaque(u.u1), u2 = opaque(u.u2), u3 = opaque(u.u3);
        // this lane's share of the secondaries
        const int share = single ? 2 * wv + half : wv, shares = single ? 2 * kAppendWaves : kAppendWaves;
        const int per = (g.S + shares - 1) / shares, s0 = share * per;
        float best = -1.f;
        int s_best = 0;
#pragma unroll 4
        for (int j = 0; j < per; ++j) {
            const int s = min(s0 + j, g.S - 1);
            float v0, v1, v2, v3;
            const float sc = score_secondary(reinterpret_cast<const float *>(secl + s), u0, u1, u2, u3, v0, v1, v2, v3);
            s_best = sc > best ? s : s_best;
            best = fmaxf(best, sc);
        }
        if (v0 > 0)
            __syncthreads();  // wave 0 has read the shares of the rows before
        best_of[wv][lane] = best;
        s_of[wv][lane] = s_best;
        __syncthreads();
        if (wv != 0)
            continue;
        // ---- wave 0: the best of the shares (ascending secondaries), and all that is written ------------------------------
        best = -1.f;
#pragma unroll
        for (int k = 0; k < kAppendWaves; ++k) {
            const int l = single ? c : lane;
            float sc = best_of[k][l];
            int s = s_of[k][l];
            s_best = sc > best ? s : s_best;
            best = fmaxf(best, sc);
            if (single) {
                sc = best_of[k][32 + c];
                s = s_of[k][32 + c];
                s_best = sc > best ? s : s_best;
                best = fmaxf(best, sc);
            }
        }
        const bool valid = in_row && (!single || half == 0);
        const bool flagged = valid && r2 > thr;
        const unsigned long long flags = ballot(flagged);
        const uint32_t word = half ? (uint32_t)(flags >> 32) : (uint32_t)flags;
        double rmax = flagged ? 0.0 : r2;
        rmax = fmax(rmax, dpp_move_f64<0xB1>(rmax));   // quad_perm [1, 0, 3, 2]
        rmax = fmax(rmax, dpp_move_f64<0x4E>(rmax));   // quad_perm [2, 3, 0, 1]
        rmax = fmax(rmax, dpp_move_f64<0x141>(rmax));  // row_half_mirror
        rmax = fmax(rmax, dpp_move_f64<0x140>(rmax));  // row_mirror
        rmax = fmax(rmax, __shfl_xor(rmax, 16, 64));
        const uint16_t sigma16 = sigma_of_row_max(rmax);
        const int rq = radius_code(r2, r_f, sigma16, Lq);
        uint32_t code = 0;
        if (valid && !flagged && r2 != 0.0) {
            float v0, v1, v2, v3, sc;
            const int s = min(s_best, g.S - 1);
            (void)score_secondary(reinterpret_cast<const float *>(secl + s), u0, u1, u2, u3, v0, v1, v2, v3);
            code = ((uint32_t)rq << g.w_idx) | (uint32_t)(nearest_primary(v0, v1, v2, v3, sc) * g.S + s);
        }
        pack[lane] = 0;
        wave_lds_sync();
        if (code) {
            const uint32_t bitpos = (uint32_t)c * g.w, sh = bitpos & 31;
            uint32_t *d0 = pack + 32 * half + (bitpos >> 5);
            atomicOr(d0, code << sh);
            if (sh + g.w > 32)
                atomicOr(d0 + 1, code >> (32 - sh));
        }
        wave_lds_sync();
        const uint32_t off = count[R];
        if (!single || half == 0) {
            if (c < g.row_words)
                reinterpret_cast<uint32_t *>(part(kAppCodes))[R * g.row_words + c] = pack[lane];
            if (c == 0) {
                reinterpret_cast<uint16_t *>(part(kAppSigma))[R] = sigma16;
                reinterpret_cast<uint32_t *>(part(kAppFlags))[R] = word;
                reinterpret_cast<uint32_t *>(part(kAppRowOff))[R] = off;
            }
            const uint32_t pos = off + (uint32_t)__popc(word & ((1u << c) - 1u));
            if (flagged && pos < (uint32_t)batch.capacity[tensor])
                reinterpret_cast<uint2 *>(part(kAppOutliers))[pos] = __builtin_bit_cast(uint2, xv);
        }
    }
}

hipError_t launch_append(const AppendShape &g, const AppendBatch &batch, hipStream_t stream)
{
    const dim3 grid((unsigned)(g.by_head ? g.H : g.B * g.H), (unsigned)g.n_tensors);
    if (g.D == 4 * kChunksPerRow)
        hipLaunchKernelGGL(k_append<true>, grid, dim3(kAppendThreads), 0, stream, g, batch);
    else
        hipLaunchKernelGGL(k_append<false>, grid, dim3(kAppendThreads), 0, stream, g, batch);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------------------------
// The search of long tensors: point location instead of a scan over the secondaries.
//
// Folding.  The score of codeword P_p q_s is <u, P_p q_s> = <conj(P_0) u, P_p' q_s> with P_p = P_0 P_p' for any P_0 of
// 2T.  With P_0 the element nearest to u, w = conj(P_0) u lies in the cell of 1: w_0 >= |w_i| and
// w_0 >= (w_0 + |w_1| + |w_2| + |w_3|) / 2, that is, y = (w_1, w_2, w_3) / w_0 lies in the octahedron
// |y_1| + |y_2| + |y_3| <= 1 (24-cell: its cells are octahedra).  Scores divided by w_0 > 0 are
// c_0 + c_1 y_1 + c_2 y_2 + c_3 y_3: linear in y.
// Cells.  The cube [-1, 1]^3 is cut into n^3 boxes; a box has the list of the codewords that are the best, or within
// kListEps of the best, somewhere in it.  Codeword c is left out when another one b is ahead of it all over the box:
// <b - c, (1, m)> > h sum_i |b_i - c_i| + eps at the centre m with half width h: exact for linear functions, whatever
// the norms of the secondaries.  About 6 of the 24 S codewords stay (S = 256, n = 20).
// A chunk then costs the fold, a look-up of its box and 3 FMA and 5 more operations per listed codeword instead of
// 5.5 S operations; best and runner-up decide as in the screen above: a chunk whose two best lie within kCellBand
// is searched again over all S secondaries in fp32.  Either way the codeword is the best one, or the fp32 search's choice
// between codewords whose scores differ by no more than its own rounding.
// Measured, two [1, 8, 32768, 128] tensors in a call, S = 256: 1017 us (matrix screen), 114 by the index (and 7 beside the
// select's sweep).  Bound by VALU issue: 258 instructions per 64 chunks, 113 of them in the list loop (the longest of 64 lists has
// 3.3 groups of four on average), 1.01 per SIMD and four cycles.  A third of them, additions, multiplications and moves, issue in
// 2.4 cycles, the others in 4.2: the VALUs are busy for some nine tenths of the time, LDS for 65 % (list entries read one
// by one, without the instructions that take them apart: 139 us).  118 us and 262 with the rows of one pass at a time, 129 and 282
// with the index finished by every workgroup (finish_cells), 145 and 327 with fp64 norms of every chunk, ballots of integers, the fold by all sixteen products
// and the rows' state stored row by row.
// What a codebook costs whose lists do not fit (secondaries close together or equal) stands at the fall-back in cell_codeword.
// ---------------------------------------------------------------------------------------------------------------

namespace {

// Two codewords whose scores lie closer than this fraction of the best are not told apart by the lists' arithmetic: more
// than its largest possible error, so that a clear winner has the best score in exact arithmetic too.  In units of 2^-24,
// for two unit codewords a and b that tie near the best (both within 45 degrees of the chunk: |a - b| <= sqrt(2)):
//   y          11.2 |a - b|: a common factor of 5 (three additions in w_0, the reciprocal), 3 sqrt(3) + 1 across it
//   functions  3 each: three additions of 1/2 per component, times 1 + |y_1| + |y_2| + |y_3| <= 2
//   values     3 each: three FMA of at most sqrt(2)
// 27.9 in all, of a best that is at least 1/sqrt(2): 2.35e-6 (3.4e-7 measured on 800,000 chunks).  Secondaries of other
// norms scale both sides by the largest.
constexpr float kCellBand = 2.5e-6f;
static_assert(2.0f * kCellBand < kListEps, "a list holds the runner-up of every chunk in the band");
constexpr float kCellShrink = 1.0f - 4.0e-6f;  // keeps the box numbers of y = -1 and 1, which rounding can move past the
                                               // cube by 5.4e-7 (fold 3.6e-7, reciprocal and product 1.8e-7), in 0 .. n - 1
// The search numbers the element P_0 that it folds with by 4 f + 16 for f = p_0 / 4 + p_1 / 2 + p_2 + 2 p_3 in twice its
// components: odd from 1 to 31 for the half-integer elements, even for the axis elements.  It needs the index of P_0 P_p' in
// the order of the primaries: [fold][p'], rows of 32 bytes.
struct FoldTable {
    alignas(16) uint8_t at[kFolds * 32];
};
constexpr FoldTable make_fold_table()
{
    FoldTable t{};
    int el[24][4] = {};  // twice the components
    for (int p = 0; p < 24; ++p)
        for (int i = 0; i < 4; ++i)
            el[p][i] = p < 8 ? ((p >> 1) == i ? ((p & 1) ? -2 : 2) : 0) : ((((p - 8) >> (3 - i)) & 1) ? -1 : 1);
    for (int a = 0; a < 24; ++a)
        for (int b = 0; b < 24; ++b) {
            const int *x = el[a], *y = el[b], fold = x[0] + 2 * x[1] + 4 * x[2] + 8 * x[3] + 16;
            const int c[4] = {x[0] * y[0] - x[1] * y[1] - x[2] * y[2] - x[3] * y[3],
                              x[0] * y[1] + x[1] * y[0] + x[2] * y[3] - x[3] * y[2],
                              x[0] * y[2] - x[1] * y[3] + x[2] * y[0] + x[3] * y[1],
                              x[0] * y[3] + x[1] * y[2] - x[2] * y[1] + x[3] * y[0]};
            for (int p = 0; p < 24; ++p)
                if (c[0] == 2 * el[p][0] && c[1] == 2 * el[p][1] && c[2] == 2 * el[p][2] && c[3] == 2 * el[p][3])
                    t.at[32 * fold + b] = (uint8_t)p;
        }
    return t;
}
__constant__ const FoldTable kFoldTable = make_fold_table();

}  // namespace

// The index build as a launch of its own, where no sweep over the rows goes before the search.
// grid = (cell_blocks(), H, tensors).
__global__ __launch_bounds__(kCellThreads) void k_cells(Geometry g, WorkspaceOffsets wo, EncodeBatch batch)
{
    __shared__ CellBuild lds;
    const EncodeTensor &tn = batch.t[blockIdx.z];
    build_cells(g, carve_workspace(tn.ws, wo), tn.sec, blockIdx.y, blockIdx.x, lds);
}
namespace {

template <typename T>
__device__ __forceinline__ T lds_at(uint32_t address)
{
    return *(__attribute__((address_space(3))) const T *)(uintptr_t)address;
}
template <typename T>
__device__ __forceinline__ T *lds_ptr(uint32_t address)
{
    return (T *)(__attribute__((address_space(3))) T *)(uintptr_t)address;
}

typedef uint32_t uint2v __attribute__((ext_vector_type(2)));

// Code word of the lane's chunk x, as search_codeword returns it (called by all 64 lanes);
// live: the wave's chunks that are neither flagged nor zero nor past the end.
struct Chunk4 {
    float x0, x1, x2, x3;
};
__device__ __forceinline__ double chunk_norm2(const Chunk4 &x)  // as of the fp16 values
{
    // opaque: rare branches use it, and what they have in common would be kept in registers for all of them
    const double x0 = (double)opaque(x.x0), x1 = (double)opaque(x.x1), x2 = (double)opaque(x.x2), x3 = (double)opaque(x.x3);
    return fma(x3, x3, fma(x2, x2, fma(x1, x1, x0 * x0)));
}
__device__ __forceinline__ bool chunk_nonfinite(const Chunk4 &x)
{
    auto field = [](float v) { return __float_as_uint(v) & 0x7f800000u; };
    return max(max(field(x.x0), field(x.x1)), max(field(x.x2), field(x.x3))) == 0x7f800000u;
}
__device__ __forceinline__ uint32_t cell_codeword(const Geometry &g, const CellTables &ct, int lane, const Chunk4 x,
                                                  unsigned long long live, int rq)
{
    // ---- fold: P_0 nearest to x, in twice its components.  An axis element when twice the largest |x_i| exceeds the sum
    // (never for two at once); either way w_0 is the larger of the two ------------------------------------------------------
    const float a0 = fabsf(x.x0), a1 = fabsf(x.x1), a2 = fabsf(x.x2), a3 = fabsf(x.x3);
    const float big = fmaxf(fmaxf(fmaxf(a0, a1), a2), a3), sum = ((a0 + a1) + a2) + a3;
    const bool axis = big + big > sum;
    const float bound = axis ? big : 0.f, mag = axis ? 2.f : 1.f;
    auto component = [&](float v) { return fabsf(v) >= bound ? copysignf(mag, v) : 0.f; };
    const float p0 = component(x.x0), p1 = component(x.x1), p2 = component(x.x2), p3 = component(x.x3);
    const float inv = __builtin_amdgcn_rcpf(fmaxf(big + big, sum));
    const float w1 = fmaf(p3, x.x2, fmaf(-p2, x.x3, fmaf(-p1, x.x0, p0 * x.x1)));
    const float w2 = fmaf(-p3, x.x1, fmaf(-p2, x.x0, fmaf(p1, x.x3, p0 * x.x2)));
    const float w3 = fmaf(-p3, x.x0, fmaf(p2, x.x1, fmaf(-p1, x.x2, p0 * x.x3)));
    const float y1 = w1 * inv, y2 = w2 * inv, y3 = w3 * inv;
    const float f = fmaf(p3, 2.f, fmaf(p1, 0.5f, p2) + 0.25f * p0);  // exact
    const uint32_t fold_row = (uint32_t)fmaf(f, 128.f, (float)(512u + ct.mul));
    // ---- the box.  Shrunk about the centre, y stays inside the cube at either end; the last bound is for inputs that break
    // the contract (a zero chunk's 0 / 0 becomes 0, a corner box without a list) ----------------------------------------------
    const uint32_t n = (uint32_t)g.cell_n;
    const float middle = 0.5f * (float)n, hn = middle * kCellShrink;
    const uint32_t i0 = (uint32_t)fmaf(y1, hn, middle), i1 = (uint32_t)fmaf(y2, hn, middle), i2 = (uint32_t)fmaf(y3, hn, middle);
    const uint32_t box = min(__umul24(i0, n * n) + __umul24(i1, n) + i2, n * n * n - 1u);
    uint32_t group = lds_at<uint16_t>(ct.head + 2u * box);
    // ---- best and runner-up of the list ----------------------------------------------------------------------------------
    float best = 0.f, second = 0.f;
    uint32_t at = ct.base;
    for (bool last = false; !last; group += 8u) {
        const uint2v e = lds_at<uint2v>(group);
        const uint32_t o[4] = {e.x & 0xffffu, e.x >> 16, e.y & 0xffffu, e.y >> 16};
        last = o[0] <= o[1];
        float4_t fn[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
            fn[i] = lds_at<float4_t>(o[i]);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float v = value_at(fn[i], y1, y2, y3);
            second = __builtin_amdgcn_fmed3f(v, best, second);  // second <= best
            if (v > best)
                at = o[i];
            best = fmaxf(best, v);
        }
    }
    unsigned long long todo = live & ballot(!(best * (1.f - kCellBand) > second));  // true without a list
    const uint32_t id = lds_at<uint32_t>((at >> 2) + (ct.id - (ct.base >> 2)));
    uint32_t p = lds_at<uint8_t>(fold_row + (id >> 16));
    uint32_t s = id & 0xffffu;
    // ---- the others over all secondaries in fp32 (as in search_codeword), one at a time (75 + 0.42 S instructions each) or,
    // where they are many (secondaries that repeat, lists that do not fit), every lane its own (26 S): two tensors with 8 heads
    // of 16384 rows in us, one at a time / every lane / matrix screen of short tensors: 16 secondaries twice 8 1033 / 154 / 117,
    // 64 within a cap of 0.05 712 / 343 / 205, 256 803 / 883 / 521, 256 twice 128 2312 / 1180 / 2666, 512 within 0.3 2440 / 1540
    // / 877 (a screen in this place, or behind it for what it leaves over, costs every other call 1 to 5 % or 4 us) ------------
    if (todo) {
        const bool unclear = of_mask(todo);
        const float *secl = lds_ptr<float>(ct.sec);
        // as unit_direction, from the fp64 norm: ties fall the same way in every search
        const float scale = __builtin_amdgcn_rcpf(__builtin_amdgcn_sqrtf((float)chunk_norm2(x))) * kOperandScale;
        const float u0 = opaque(x.x0 * scale), u1 = opaque(x.x1 * scale), u2 = opaque(x.x2 * scale), u3 = opaque(x.x3 * scale);
        if (__builtin_expect_with_probability(__popcll(todo) > min(4 + g.S / 10, 30), false, 0.9999)) {
            todo = 0ull;
            float most = -1.f;
            uint32_t first = 0;
#pragma unroll 1
            for (int j = 0; j < g.S; ++j) {
                float v0, v1, v2, v3;
                const float sc = score_secondary(secl + 4 * j, u0, u1, u2, u3, v0, v1, v2, v3);
                first = sc > most ? (uint32_t)j : first;
                most = fmaxf(most, sc);
            }
            s = unclear ? first : s;
        }
        while (todo) {  // wave-uniform
            const int src = __ffsll((long long)todo) - 1;
            todo &= todo - 1ull;
            const float e0 = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(u0), src));
            const float e1 = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(u1), src));
            const float e2 = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(u2), src));
            const float e3 = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(u3), src));
            unsigned long long key = 0ull;
            for (int j = lane; j < g.S; j += 64) {
                float v0, v1, v2, v3;
                const float sc = score_secondary(secl + 4 * j, e0, e1, e2, e3, v0, v1, v2, v3);
                key = umax64(key, ((unsigned long long)__float_as_uint(sc) << 32) | (0xffffffffu - (uint32_t)j));
            }
            key = wave_umax64(key);
            if (lane == src)
                s = min(0xffffffffu - (uint32_t)key, (uint32_t)g.S - 1u);
        }
        float v0, v1, v2, v3, sc;
        (void)score_secondary(secl + 4 * min(s, (uint32_t)g.S - 1u), u0, u1, u2, u3, v0, v1, v2, v3);
        const uint32_t pu = (uint32_t)nearest_primary(v0, v1, v2, v3, sc);
        p = unclear ? pu : p;
    }
    return of_mask(live) ? ((uint32_t)rq << g.w_idx) | (__umul24(p, (uint32_t)g.S) + s) : 0u;
}

// A head's index from the workspace into LDS, with the folds and the secondaries.  A finished one 16 bytes at a time, all
// requested before the first is written; else it is finished on the way (bits: scratch).  Ends with a barrier.
template <int kThreadsS>
__device__ __forceinline__ void load_cells(const Geometry &g, const Workspace &ws, int h, const float *sec_h, const CellTables &ct,
                                           bool finished, uint32_t *bits)
{
    static_assert(kThreadsS == kFinishThreads, "finish_cells");
    const int tid = threadIdx.x;
    if (!finished) {  // uniform
        if (tid < kFolds * 2)
            lds_ptr<uint4>(ct.mul)[tid] = reinterpret_cast<const uint4 *>(kFoldTable.at)[tid];
        if (tid < g.S)
            lds_ptr<uint4>(ct.sec)[tid] = reinterpret_cast<const uint4 *>(sec_h)[tid];
        // its first barrier comes before it looks at the secondaries
        finish_cells<false>(g, ws, lds_ptr<float4_t>(ct.sec), h, 0, 1,
                        CellPlaces{lds_ptr<uint2>(ct.list), lds_ptr<uint2>(ct.head), lds_ptr<uint32_t>(ct.id), lds_ptr<float4_t>(ct.base)}, bits);
        __syncthreads();
        return;
    }
    const CellIndex ix = cell_index_of(g, ws, h);
    constexpr int kMax = 5120 * 8 + 20 * 20 * 20 * 2;  // bytes of the largest lists and boxes
    constexpr int kLists = (kMax / 16 + kThreadsS - 1) / kThreadsS, kFunctions = 2;
    static_assert((13 * kScreenMaxS / 5 + 99) / 4 * 4 + 1 <= kFunctions * kThreadsS && kScreenMaxS <= kThreadsS, "loads of a thread");
    const int n_lists = (int)(ct.id - ct.list) / 16, n_functions = g.cell_used + 1, n_ids = g.cell_used / 4, n_folds = kFolds * 2;
    uint4 lists[kLists], functions[kFunctions], ids = {}, folds = {}, secondaries = {};
#pragma unroll
    for (int u = 0; u < kLists; ++u)
        lists[u] = reinterpret_cast<const uint4 *>(ix.list)[min(tid + u * kThreadsS, n_lists - 1)];
#pragma unroll
    for (int u = 0; u < kFunctions; ++u)
        functions[u] = reinterpret_cast<const uint4 *>(ix.function)[min(tid + u * kThreadsS, n_functions - 1)];
    if (tid < n_ids)
        ids = reinterpret_cast<const uint4 *>(ix.id)[tid];
    if (tid < n_folds)
        folds = reinterpret_cast<const uint4 *>(kFoldTable.at)[tid];
    if (tid < g.S)
        secondaries = reinterpret_cast<const uint4 *>(sec_h)[tid];
#pragma unroll
    for (int u = 0; u < kLists; ++u)
        if (tid + u * kThreadsS < n_lists)
            lds_ptr<uint4>(ct.list)[tid + u * kThreadsS] = lists[u];
#pragma unroll
    for (int u = 0; u < kFunctions; ++u)
        if (tid + u * kThreadsS < n_functions)
            lds_ptr<uint4>(ct.base)[tid + u * kThreadsS] = functions[u];
    if (tid < n_ids)
        lds_ptr<uint4>(ct.id)[tid] = ids;
    if (tid < n_folds)
        lds_ptr<uint4>(ct.mul)[tid] = folds;
    if (tid < g.S)
        lds_ptr<uint4>(ct.sec)[tid] = secondaries;
    __syncthreads();
}

}  // namespace

// A value that all lanes have, in a scalar register.
__device__ __forceinline__ float scalar(float v) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v))); }

constexpr int kCellWaves = 16;  // of a workgroup
constexpr int cell_passes(int rows, int slot) { return slot > 0 && rows * slot >= kCellWaves * 64 * 2 ? 2 : 1; }

// Dynamic LDS of a workgroup: the index, then the rows' state and the waves' words, in whose place it is finished.
inline size_t cell_lds_bytes(const Geometry &g)
{
    const size_t rows = kCellWaves * 64 * 4 + (size_t)g.search_rows * 8, scratch = (size_t)g.cell_words * 8 + 4;
    return cell_tables(g).end + std::max(rows, scratch);
}

// 16 waves and kRows rows per workgroup; a wave takes several whole rows at a time, one lane per chunk: kSlot = 32 or 16
// lanes per row, the lanes past the row's chunks idle (row maxima are then DPP steps), or kSlot = 0 for rows that would
// leave many idle: 64 / n_c rows next to one another.
// kFull: rows of 128 elements.
// Dynamic LDS: cell_lds_bytes().
template <int kRows, int kSlot, bool kFull, int kPasses = cell_passes(kRows, kSlot)>
__global__ __launch_bounds__(1024, 8) void k_search_cells(Geometry g, WorkspaceOffsets wo, EncodeBatch batch, int cells_finished)
{
    constexpr int kWaves = kCellWaves;
    const EncodeTensor &tn = batch.t[blockIdx.z];
    const Workspace ws = carve_workspace(tn.ws, wo);
    const EncodedPtrs enc = tn.enc;
    const CellTables ct = cell_tables(g);
    uint2 *state = lds_ptr<uint2>(ct.end);                           // of a row: flag word, scale
    uint32_t *pack = reinterpret_cast<uint32_t *>(state + kRows);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int seg = blockIdx.y, b = seg / g.H, h = seg % g.H;
    const int t0 = blockIdx.x * kRows;
    load_cells<64 * kWaves>(g, ws, h, tn.sec + (size_t)h * g.S * 4, ct, cells_finished != 0, reinterpret_cast<uint32_t *>(state));  // scratch

    const double thr = ws.thr[h];
    // a squared norm in fp32 differs from the fp64 one by at most 3 * 2^-24 of it: outside these it decides
    const float thr_sure = scalar((float)thr * (1.f + 0x1p-21f)), thr_perhaps = scalar((float)thr * (1.f - 0x1p-21f));
    const int n_c = kFull ? kChunksPerRow : g.n_c, row_words = kFull ? g.w : g.row_words;
    const int slot = kSlot ? kSlot : n_c;
    const int rows_pass = 64 / slot;
    const int rl = lane / slot, c = lane - rl * slot;  // the lane's row of a pass and chunk of the row
    const int n_rows = min(kRows, g.T - t0);         // >= 1 by the grid's size
    uint32_t *my_pack = pack + wv * 64;              // rows_pass * row_words <= 64 words: w <= 22 as S <= kScreenMaxS
    // Two passes at a time where a workgroup has rows enough for all waves (launch_search): the steps that every lane of a row
    // takes alike (scale, its reciprocal, what is kept of a row) are then taken once, the even lanes for the first pass and the odd
    // for the second.
    const bool second = kPasses == 2 && of_mask(0xaaaaaaaaaaaaaaaaull);
    const _Float16 *rows = tn.x + (int64_t)b * g.sb + (int64_t)h * g.sh + (int64_t)(t0 + wv * kPasses * rows_pass) * g.st;
    const int64_t row_step = (int64_t)(kWaves * kPasses * rows_pass) * g.st;
    // Lanes without a chunk, and rows past the end, load another once more: they are masked where it matters.
    const bool mine = kFull || (rl < rows_pass && c < n_c);
    const unsigned long long in_slot = kFull ? ~0ull : ballot(mine);
    const uint32_t first_chunk = mine ? 8u * (uint32_t)c : 0u;
    const uint32_t own_chunk = (mine ? 2u * (uint32_t)rl * (uint32_t)g.st : 0u) + first_chunk;  // kSlot: bytes, below 2^32 (launch_search)
    const int64_t row0 = (int64_t)seg * g.T + t0;
    auto *pass_codes = (__attribute__((address_space(1))) uint32_t *)(enc.codes + (row0 + wv * kPasses * rows_pass) * row_words);
    const uint32_t code_step = (uint32_t)(kWaves * kPasses * rows_pass * row_words);
    const float Lf = scalar((float)((1 << g.b_r) - 1)), surely = scalar(0.5f - (6e-7f * Lf + 1e-6f));
    // where the lane's code goes in a pass's words: the word's LDS address and, below it, the bit in the word
    const uint32_t bit = (uint32_t)(rl * row_words * 32 + c * g.w);
    uint32_t place = ((uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint32_t *)(my_pack + (bit >> 5)) << 5) | (bit & 31u);
    // The largest of a row's values, in every lane of the row; of both passes' in their lanes.
    auto row_max = [&](auto first, auto other) {
        if (kSlot) {  // after each step the running maxima are uniform over a block twice as large
            first = fmax(first, dpp_move<0xB1>(first));  // quad_perm [1, 0, 3, 2]
            if (kPasses == 2) {
                other = fmax(other, dpp_move<0xB1>(other));
                first = second ? other : first;
            }
            first = fmax(first, dpp_move<0x4E>(first));   // quad_perm [2, 3, 0, 1]
            first = fmax(first, dpp_move<0x124>(first));  // row_ror 4
            first = fmax(first, dpp_move<0x128>(first));  // row_ror 8
            return kSlot == 32 ? max_across_16(first) : first;
        }
        for (int d = 1; d < n_c; d <<= 1) {
            const auto o = __shfl(first, lane + d, 64);
            first = c + d < n_c ? fmax(first, o) : first;
        }
        return __shfl(first, lane - c, 64);
    };
    // a value of the row in all its lanes
    auto of_pass = [&](auto v, int p) { return kPasses == 1 ? v : p ? dpp_move<0xF5>(v) : dpp_move<0xA0>(v); };  // quad_perm [1, 1, 3, 3], [0, 0, 2, 2]
    for (int r0 = wv * kPasses * rows_pass; r0 < n_rows; r0 += kWaves * kPasses * rows_pass, rows += row_step, pass_codes += code_step) {  // wave-uniform
        Chunk4 x[kPasses];
        float r2f[kPasses];
        unsigned long long flags[kPasses];
        half4_t xv[kPasses];
#pragma unroll
        for (int p = 0; p < kPasses; ++p) {
            const int first = r0 + p * rows_pass;  // of the pass's rows
            const _Float16 *at = first < n_rows ? rows + (int64_t)(p * rows_pass) * g.st : rows;
            const bool in = kFull ? first + 1 < n_rows : rl < n_rows - first;
            const _Float16 *own = kSlot ? reinterpret_cast<const _Float16 *>(reinterpret_cast<const char *>(at) + (in ? own_chunk : first_chunk))
                                        : at + (in && mine ? (int64_t)rl * g.st : 0) + first_chunk / 2;
            if (kFull || g.vec_ok) {
                xv[p] = load_chunk(own);
            } else {
                xv[p] = half4_t{0, 0, 0, 0};
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (first_chunk / 2 + e < (uint32_t)g.D)
                        xv[p][e] = own[e];
            }
        }
#pragma unroll
        for (int p = 0; p < kPasses; ++p) {
            x[p] = Chunk4{opaque((float)xv[p][0]), opaque((float)xv[p][1]), opaque((float)xv[p][2]), opaque((float)xv[p][3])};
            r2f[p] = fmaf(x[p].x3, x[p].x3, fmaf(x[p].x2, x[p].x2, fmaf(x[p].x1, x[p].x1, x[p].x0 * x[p].x0)));  // squares are exact: three roundings
            // Predicates of the whole wave are kept as masks: combined on the scalar unit, they cost no vector instruction.
            flags[p] = ballot(r2f[p] > thr_sure);
            if (flags[p] != ballot(r2f[p] > thr_perhaps))  // a ten-millionth of the chunks
                flags[p] = ballot(chunk_norm2(x[p]) > thr);
            flags[p] &= in_slot;
            if (g.check_finite) {  // uniform
                if (ballot(chunk_nonfinite(x[p])) != 0ull && lane == 0)
                    atomicOr(enc.status, HQMQ_STATUS_NONFINITE);
            }
        }
        constexpr int kLast = kPasses - 1;
        auto counts = [&](int p) { return of_mask(in_slot & ~flags[p]); };  // for the scale
        // The row's scale, sigma_of_row_max of the largest r^2: the fp32 maximum is within 3 * 2^-24 of the fp64 one and decides
        // unless its square root lies next to a rounding boundary; then the fp64 maximum is taken as well.
        // r^2 is 0 or at least 2^-48: the fp32 value is zero for a zero chunk only.
        const float sf = fminf(__builtin_amdgcn_sqrtf(row_max(counts(0) ? r2f[0] : 0.f, counts(kLast) ? r2f[kLast] : 0.f)), 65504.f);  // 1 ulp
        uint16_t sigma16 = __builtin_bit_cast(uint16_t, (_Float16)sf);
        const bool unsure_scale = scale_unsure(sf);
        if (ballot(unsure_scale)) {
            const double exact = row_max(counts(0) ? chunk_norm2(x[0]) : 0.0, counts(kLast) ? chunk_norm2(x[kLast]) : 0.0);
            if (unsure_scale)
                sigma16 = double_to_half_rne_sat(sqrt(exact));
        }
        // radius codes per unit of norm; a scale of zero gives the code 0
        const float per_norm = sigma16 != 0 ? Lf * __builtin_amdgcn_rcpf((float)__builtin_bit_cast(_Float16, sigma16)) : 0.f;
        // what is kept of the rows: lane 0 of a row for the first pass, lane 1 for the second
        {
            const int r = r0 + (second ? rows_pass : 0) + rl;
            uint32_t word = 0;
            if (kFull) {
                const uint32_t low = second ? (uint32_t)flags[kLast] : (uint32_t)flags[0];
                const uint32_t high = second ? (uint32_t)(flags[kLast] >> 32) : (uint32_t)(flags[0] >> 32);
                word = lane >= 32 ? high : low;
            } else {
                const unsigned long long both = second ? flags[kLast] : flags[0];
                word = (uint32_t)(both >> ((unsigned)(rl * slot) & 63u)) & (uint32_t)((1ull << n_c) - 1ull);
            }
            if (c < kPasses && (kFull || rl < rows_pass) && r < n_rows)
                state[r] = make_uint2(word, sigma16);
        }
#pragma unroll
        for (int p = 0; p < kPasses; ++p) {
            const int first = r0 + p * rows_pass;
            if (p > 0 && first >= n_rows)  // uniform
                break;
            const unsigned long long live = in_slot & ballot(r2f[p] != 0.f) & ~flags[p];
            // radius_code
            int rq;
            {
                const float q = fminf(__builtin_amdgcn_sqrtf(r2f[p]) * of_pass(per_norm, p), Lf), whole = rintf(q);
                rq = (int)whole;
                const unsigned long long unsure = live & ballot(fabsf(q - whole) > surely);
                if (unsure) {
                    const uint16_t own = (uint16_t)of_pass((int)sigma16, p);
                    if (of_mask(unsure))
                        rq = radius_code_exact(chunk_norm2(x[p]), own, (double)opaque(Lf));  // not kept in 64 bits for all passes
                }
            }
            asm volatile("" : "+v"(place));  // one register for all passes, not one for its word's address as well
            my_pack[lane] = 0;  // after the previous pass's reads of it: LDS serves a wave in order
            const uint32_t code = cell_codeword(g, ct, lane, x[p], live, rq);
            wave_lds_sync();
            if (code) {
                const uint64_t shifted = (uint64_t)code << (place & 63u);
                uint32_t *d0 = lds_ptr<uint32_t>(place >> 5);
                atomicOr(d0, (uint32_t)shifted);
                if (shifted >> 32)
                    atomicOr(d0 + 1, (uint32_t)(shifted >> 32));
            }
            wave_lds_sync();
            // the pass's rows are neighbours, and so are their code words
            auto *codes = pass_codes + (uint32_t)(p * rows_pass * row_words);
            asm volatile("" : "+s"(codes));  // a lane's offset to a scalar base, not an address per lane
            if (lane < min(rows_pass, n_rows - first) * row_words)
                codes[(uint32_t)lane] = my_pack[lane];
        }
    }
    __syncthreads();
    for (int r = tid; r < n_rows; r += 64 * kWaves) {
        const uint2 of = state[r];
        enc.flags[row0 + r] = of.x;
        enc.sigma[row0 + r] = (uint16_t)of.y;
    }
    if (wv == 0)
        write_row_offsets<kRows>(g, ws, enc, lane, seg, t0, state);
}

// The search kernels' dynamic LDS may exceed the 64 KiB a kernel gets by default: raises the limit
// of every variant on the current device.  Stateless; the caller (the library's per-device set-up) runs it
// once per device, before any launch and outside any stream capture.
hipError_t prepare_search_kernels()
{
    // the fused forms also hold static LDS (the workgroup-wide OR, the merge buffer of the cooperative pass: up to
    // 6 KiB), which counts against the same 160 KiB
    const void *fused[] = {reinterpret_cast<const void *>(k_search<true>), reinterpret_cast<const void *>(k_search_flat<true>)};
    const void *variants[] = {reinterpret_cast<const void *>(k_search<>),
                              reinterpret_cast<const void *>(k_search_flat<>),
                              reinterpret_cast<const void *>(k_search<false, false>),
                              reinterpret_cast<const void *>(k_search_flat<false, false>)};
    const void *cells[] = {reinterpret_cast<const void *>(k_search_cells<kSearchRowsSmall, 32, true, 1>),
                           reinterpret_cast<const void *>(k_search_cells<kSearchRowsSmall, 32, false, 1>),
                           reinterpret_cast<const void *>(k_search_cells<kSearchRowsSmall, 32, true>),
                           reinterpret_cast<const void *>(k_search_cells<kSearchRowsSmall, 32, false>),
                           reinterpret_cast<const void *>(k_search_cells<kSearchRowsSmall, 16, false>),
                           reinterpret_cast<const void *>(k_search_cells<kSearchRowsSmall, 0, false>),
                           reinterpret_cast<const void *>(k_search_cells<kSearchRowsLarge, 32, true>),
                           reinterpret_cast<const void *>(k_search_cells<kSearchRowsLarge, 32, false>),
                           reinterpret_cast<const void *>(k_search_cells<kSearchRowsLarge, 16, false>),
                           reinterpret_cast<const void *>(k_search_cells<kSearchRowsLarge, 0, false>),
                           reinterpret_cast<const void *>(k_search_cells<kSearchRowsHuge, 32, true>),
                           reinterpret_cast<const void *>(k_search_cells<kSearchRowsHuge, 32, false>),
                           reinterpret_cast<const void *>(k_search_cells<kSearchRowsHuge, 16, false>),
                           reinterpret_cast<const void *>(k_search_cells<kSearchRowsHuge, 0, false>)};
    hipError_t err = hipSuccess;
    for (const void *f : fused)
        if (err == hipSuccess)
            err = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsPerCu - 8192);
    for (const void *f : variants)
        if (err == hipSuccess)
            err = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsPerCu);
    for (const void *f : cells) {
        hipFuncAttributes own;
        if (err == hipSuccess)
            err = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsPerCu);
        if (err == hipSuccess)
            err = hipFuncGetAttributes(&own, f);
        if (err == hipSuccess && own.sharedSizeBytes != 0)  // the index in the workspace holds LDS addresses from 0 on
            err = hipErrorInvalidConfiguration;
    }
    return err;
}

// The fused form exists for the workgroups that short segments get, of 64 rows, and codebooks that are screened.
bool search_fused_available(const Geometry &g) { return g.A16 > 0 && g.search_rows == kSearchRowsSmall; }

hipError_t launch_search_fused(const Geometry &g, const WorkspaceOffsets &wo, const EncodeBatch &batch, int n_tensors,
                               hipStream_t stream)
{
    dim3 grid((g.T + g.search_rows - 1) / g.search_rows, g.fused_by_head ? g.H : g.B * g.H, (unsigned)n_tensors);
    const size_t lds = search_lds_bytes(g.S16, g.A16, g.D, g.row_words, kSearchWaves, g.search_rows);
    if (g.D == 4 * kChunksPerRow)
        hipLaunchKernelGGL(k_search<true>, grid, dim3(64 * kSearchWaves), lds, stream, g, wo, batch);
    else
        hipLaunchKernelGGL(k_search_flat<true>, grid, dim3(64 * kSearchWaves), lds, stream, g, wo, batch);
    return hipGetLastError();
}

// cells_built: the select's launches have built and finished the box index.
hipError_t launch_search(const Geometry &g, const WorkspaceOffsets &wo, const EncodeBatch &batch, int n_tensors,
                         bool cells_built, hipStream_t stream)
{
    dim3 grid((g.T + g.search_rows - 1) / g.search_rows, g.B * g.H, (unsigned)n_tensors);
    const bool full = g.D == 4 * kChunksPerRow;
    if (g.cell_n > 0) {
        const bool narrow = g.st < (1ll << 29), full_rows = full && narrow;  // 32-bit offsets inside a pass
        if (!cells_built)
            hipLaunchKernelGGL(k_cells, dim3(cell_blocks(g), g.H, (unsigned)n_tensors), dim3(kCellThreads), 0, stream, g, wo, batch);
        const size_t lds_cells = cell_lds_bytes(g);
#define HQMQ_LAUNCH_CELLS(...) \
    hipLaunchKernelGGL((k_search_cells<__VA_ARGS__>), grid, dim3(64 * kCellWaves), lds_cells, stream, g, wo, batch, cells_built)
#define HQMQ_LAUNCH_CELLS_OF(R, ...)                                                                                 \
    do {                                                                                                             \
        if (full_rows)                                                                                               \
            HQMQ_LAUNCH_CELLS(R, 32, true, ##__VA_ARGS__);                                                           \
        else if (narrow && g.n_c > 21)                                                                               \
            HQMQ_LAUNCH_CELLS(R, 32, false, ##__VA_ARGS__);                                                          \
        else if (narrow && g.n_c <= 16 && g.n_c > 12)                                                                \
            HQMQ_LAUNCH_CELLS(R, 16, false, ##__VA_ARGS__);                                                          \
        else                                                                                                         \
            HQMQ_LAUNCH_CELLS(R, 0, false, ##__VA_ARGS__);                                                           \
    } while (0)
        // The form for the rows that a workgroup has, not for those that it may have: up to two per wave in single passes, for which
        // pairs would leave half of the waves without any (eight for 16 rows, four so); and the forms for more rows hold
        // more in scalar registers than there are.  Known thresholds, 8 heads of two tensors, S = 256, the form for 512 rows / this
        // one, call in us: 512 batch entries of 16 rows of 128 elements 243 / 230, 256 of 32 122 / 117, 128 of 64 87 / 83, 341 of 24
        // rows of 96 184 / 169, 256 of 32 rows of 64 114 / 99, 113 of 72 rows of 128 89 / 88.
        const int most = std::min(g.T, g.search_rows);
        if (most > kSearchRowsLarge)
            HQMQ_LAUNCH_CELLS_OF(kSearchRowsHuge);
        else if (most > kSearchRowsSmall)
            HQMQ_LAUNCH_CELLS_OF(kSearchRowsLarge);
        else if (most > kCellWaves * 2)
            HQMQ_LAUNCH_CELLS_OF(kSearchRowsSmall);
        else
            HQMQ_LAUNCH_CELLS_OF(kSearchRowsSmall, 1);
#undef HQMQ_LAUNCH_CELLS_OF
#undef HQMQ_LAUNCH_CELLS
        return hipGetLastError();
    }
    const size_t lds = search_lds_bytes(g.S16, g.A16, g.D, g.row_words, kSearchWaves, g.search_rows);
    // rows per workgroup that the kernels take: two per wave and up to 64, or 256 for the flat form
    const int rows = g.search_rows;
    if (full ? rows > kSearchRowsSmall || rows % (2 * kSearchWaves) : rows > kSearchRowsSmall && rows != kSearchRowsLarge)
        return hipErrorInvalidConfiguration;
#define HQMQ_LAUNCH(...) hipLaunchKernelGGL((__VA_ARGS__), grid, dim3(64 * kSearchWaves), lds, stream, g, wo, batch)
    if (g.A16 == 0) {  // more secondaries than the matrix-core screen holds: every chunk scored in fp32
        if (full)
            HQMQ_LAUNCH(k_search<false, false>);
        else
            HQMQ_LAUNCH(k_search_flat<false, false>);
    } else if (full) {
        HQMQ_LAUNCH(k_search<>);
    } else {
        HQMQ_LAUNCH(k_search_flat<>);
    }
#undef HQMQ_LAUNCH
    return hipGetLastError();
}

}  // namespace hqmq
