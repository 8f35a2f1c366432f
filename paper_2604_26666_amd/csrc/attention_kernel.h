// Fused multi-head attention forward for gfx950: O = softmax(scale * Q K^T + causal mask) V per
// (batch entry, query head), grouped-query aware (a query head reads key/value head
// h / (Hq / Hkv); nothing is expanded in memory).  The paper's first block pattern (Section 5.2.4
// pattern p1; Section 5.2.5 pattern p1 for the grouped form) replaces this sub-graph with one
// kernel that tiles over keys and never writes the score matrix to HBM (Section 2.1); this is
// that kernel for 64-lane wavefronts and MFMA 32x32x16, written from the definition.
//
// Shape of the computation
//   A work-group owns BQ = NW * 32 consecutive queries of one (batch, query head), a wave 32 of
//   them.  Keys and values are walked in blocks of BKV (64 or 32), staged in LDS (double-buffered, global->LDS
//   direct loads) and shared by the waves.  With KG key groups each 32 queries have KG waves, which take the blocks of a
//   step (KG of them) one each and add their sums up at the end: a shorter chain where a launch has few work-groups
//   (the rule and its figures stand at the launch).  Everything is computed TRANSPOSED so that a lane owns
//   pieces of ONE query:
//     S^T (keys x queries) = K_block (A operand, rows = keys) x Q^T (B operand, columns = queries)
//     O^T (d    x queries) = V_block^T (A operand, rows = d)  x P^T (B operand, columns = queries)
//   MFMA 32x32x16 result layout: lane (r32 = lane % 32, h = lane / 32), register r holds
//   D[8 (r / 4) + 4 h + r % 4][r32]: rows come from the A operand, the column is the lane's query.
//   Hence
//   * the running maximum of a query needs its 32 in-lane values per key block and one exchange
//     with the other lane that holds the same query (lane ^ 32); its sum likewise, at the very end;
//   * P^T in registers already IS the B operand of the second MFMA: a B operand lane holds 8
//     K-values (here: keys) of one column (query).  The 8 keys a lane holds of a 16-key group u are
//     {16u + 4h + 0..3} and {16u + 8 + 4h + 0..3}, not 8 consecutive ones, so the A operand
//     (V^T) is fetched with the same permutation - the transposing LDS read takes one address per
//     4-key group anyway.
//   What it spends its cycles on: vector ALU and matrix pipe, mostly in turn.  A score costs an fma, an exponential (two issue slots), half a
//   conversion and half an addition: 135 vector instructions per wave and key block, 580 cycles,
//   next to 16 MFMAs (512 cycles) at head_dim 64 and 32 (1024) at 128, of which each takes about
//   10 issue cycles from its SIMD.  A wave does the two in turn, so what matters is that another wave
//   of the SIMD is at the other: 32 queries per wave leave room for three waves per SIMD at
//   head_dim 64 and two at 128, and a work-group's first loads and last stores are covered the
//   same way.  (Blocks of 32 keys need 110 registers at head_dim 64: four waves.)  Against 64 queries per wave, one wave per SIMD and scores of one block computed
//   between the exponentials of another (which this kernel replaces at every size): 16 x 500 tokens,
//   12 heads of 64: 33 -> 19.8 us; 8 x 1024 causal 31 -> 23; 4 x 1999 causal, 32 / 8 heads of 128:
//   156 -> 144; 1 x 2048 61 -> 44; 1 x 8192 563 -> 507 (1085 TFLOP/s); 4 x 4096, 16 heads of 64, full,
//   338 -> 288.  Counters of the last: vector ALU issuing 61 % of the cycles, matrix pipe busy 49 %.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fact {
namespace attn {

#define FACT_ATTN_LDS_PTR(p) ((__attribute__((address_space(3))) void *)(p))

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef u32x4_t u32x4_by8 __attribute__((aligned(8)));       // rows of O start at any multiple of 8 bytes

struct AttnArgs {
    const __bf16 *Q, *K, *V;
    __bf16 *O;
    // element strides: batch entry, token, head (the head_dim elements of a row are contiguous)
    int64_t q_sb, k_sb, v_sb, o_sb, q_sh, k_sh, v_sh, o_sh;
    int q_st, k_st, v_st, o_st;
    int B, T, Hq, Hkv;
    int causal;
    float scale_log2;       // softmax scale * log2(e)
    float lowest;           // scores below it are masked keys' (see the reference exponent)
    int q_blocks;           // ceil(T / BQ)
    int total;              // q_blocks * Hq * B work-groups
    int grid_x;             // work-groups in a row of the grid, a multiple of 8 where there is more than one row
    int fold;               // positions of the work-group order (of an XCD's part of it) from here on run backwards
    int group;              // (batch, query head) pairs per group of the work-group order; divides the pairs of an XCD
};

constexpr uint32_t kBufFlags = 0x00020000u;      // raw buffer descriptor word 3 (32-bit data format)

__device__ __forceinline__ const char *uniform_ptr(const char *ptr)
{
    const uint64_t v = (uint64_t)ptr;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return (const char *)(((uint64_t)hi << 32) | lo);
}

// (Device-only builtins live in __device__ helpers: used directly in a __global__ template they
// make the host pass drop the kernel's launch stub without a diagnostic.)
__device__ __forceinline__ float exp2_fast(float x) { return __builtin_amdgcn_exp2f(x); }
// max over lane and lane ^ 32, in both, without LDS: v_permlane32_swap exchanges the upper half of its
// first operand with the lower half of its second; applied to two copies of x, the two results hold x
// and its partner's x in every lane.
__device__ __forceinline__ float max_with_lane_xor32(float x)
{
    const uint32_t w = __builtin_bit_cast(uint32_t, x);
    auto b = __builtin_amdgcn_permlane32_swap(w, w, false, false);
    return fmaxf(__builtin_bit_cast(float, (uint32_t)b[0]), __builtin_bit_cast(float, (uint32_t)b[1]));
}
__device__ __forceinline__ float sum_with_lane_xor32(float x)
{
    const uint32_t w = __builtin_bit_cast(uint32_t, x);
    auto b = __builtin_amdgcn_permlane32_swap(w, w, false, false);
    return __builtin_bit_cast(float, (uint32_t)b[0]) + __builtin_bit_cast(float, (uint32_t)b[1]);
}
// 16 bytes per lane from global memory straight into LDS at lds + 16 * lane (lds uniform over the wave)
__device__ __forceinline__ void load_to_lds_16(__amdgpu_buffer_rsrc_t rsrc, char *lds, uint32_t voffset, uint32_t soffset)
{
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, FACT_ATTN_LDS_PTR(lds), 16, voffset, soffset, 0, 0);
}
// 64-bit transposing LDS read (see the V^T fragment addresses)
__device__ __forceinline__ s16x4_t read_transposed(const char *lds)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t *)lds);
#else
    return s16x4_t{};
#endif
}

// LDS layout of a step's keys or values: [rows = keys of all key groups][D] bf16, the 16-byte chunk c of row r stored at
// chunk position c ^ swz(r).
//  K (read as MFMA A operand: 32 consecutive rows x 2 consecutive chunks per instruction): the
//    XOR puts 16 consecutive rows into the 16 chunks of the 256 bytes that the banks span: with the row number
//    where a row has 16 chunks, with half of it where two rows of 8 share them (the row number there
//    cost a third of the LDS cycles in conflicts: 16 x 500 tokens, 12 heads of 64, 21.3 -> 20.3 us).
//  V (read with the transposing 64-bit read: per 32 lanes, 4 rows x 64 bytes at the same column):
//    the XOR moves the 4 rows to different 64-byte windows of 256 bytes.
template <int D> __device__ __forceinline__ int swz_keys(int row)
{
    if constexpr (D == 128) return row & 15;
    else return (row >> 1) & 7;
}
template <int D> __device__ __forceinline__ int swz_vals(int row)
{
    if constexpr (D == 128) return (row & 3) << 2;
    else return ((row >> 1) & 1) << 2;
}

// LDS of a work-group: two stages of the groups' K and V blocks, afterwards the sums that the key groups exchange
constexpr int lds_bytes(int d, int nw, int kg, int bkv)
{
    const int stages = 2 * 2 * kg * bkv * d * 2, sums = d / 32 * (kg - 1) * nw * 4096 + nw * kg * 512;
    return kg > 1 && sums > stages ? sums : stages;
}

template <int D, int NW, int KG, int BKV>
__global__ void __launch_bounds__(NW * KG * 64, D == 64 && KG == 1 ? 3 : 2)
attn_fwd_kernel(const AttnArgs p)
{
#if defined(__HIP_DEVICE_COMPILE__)      // the host pass only needs the kernel's symbol
    static_assert(D == 64 || D == 128, "head_dim");
    constexpr int QW = 32, BQ = NW * QW, NT = NW * KG;         // queries per wave and per work-group, waves
    constexpr int KT = BKV / 32, UB = BKV / 16, ROWS = KG * BKV;       // a wave's key block: row tiles, 16-key groups; keys of a step
    constexpr int KS = D / 16, DT = D / 32;                    // 16-wide groups / 32-row tiles of head_dim
    constexpr int CPR = D / 8, ROWB = D * 2;                   // chunks and bytes per LDS row
    constexpr int TILE_BYTES = ROWS * ROWB, STAGE_BYTES = 2 * TILE_BYTES;
    constexpr int RPL = 1024 / ROWB;                           // rows per wave-wide load
    constexpr int L = TILE_BYTES / 1024 / NT;                  // wave-wide loads per tile and wave
    static_assert(L >= 1 && L * NT * 1024 == TILE_BYTES, "tile split over the waves");
    static_assert(NT * RPL % 16 == 0 && BKV % 16 == 0, "a wave's pieces, and the groups' blocks, are whole swizzle periods apart");

    extern __shared__ __attribute__((aligned(1024))) char smem[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int qw = KG > 1 ? wave % NW : wave, kg = KG > 1 ? wave / NW : 0;      // the wave's queries, its key group
    const int r32 = lane & 31, h = lane >> 5;

    // Work-group -> (batch, key/value head, query head, query block).  Consecutive work-group ids go
    // to different XCDs (each with its own L2): id % 8 picks the XCD, and every XCD gets its own
    // eighth of the (batch, head) pairs, the query heads that read the same K/V next to each other.
    // Within an XCD the pairs come in groups of p.group: a group's work-groups are ordered by query
    // block, the heaviest (last) first, all pairs of the group before the next lighter block.  So
    // runs of p.group consecutive work-groups carry the same amount of work, and the K/V of one
    // group (sized by the host to fit the L2) is what the XCD reads at any one time.
    // (The hardware hands consecutive work-groups of an XCD to its shader engines in turn and in
    // order; with a heavy .. light pattern whose period matched that turn, one engine got all the
    // heavy work-groups and the others idled between theirs - measured 30% of the time.)
    // Where all work-groups of a causal launch are resident at once, the last one that each compute unit
    // gets comes from the other end (p.fold): the light ones join the heaviest.
    const int G = p.Hq / p.Hkv;
    const int pairs = p.total / p.q_blocks;                    // batch * query heads
    int qb, pair;
    {
        const int v = (int)(blockIdx.y * (uint32_t)p.grid_x + blockIdx.x);
        if (v >= p.total) return;                              // (the whole work-group)
        const bool split = (pairs & 7) == 0;                   // else: one sequence over all pairs
        int pos = split ? v >> 3 : v;
        if (pos >= p.fold) pos = p.fold + (split ? p.total >> 3 : p.total) - 1 - pos;
        const int first = split ? (v & 7) * (pairs >> 3) : 0;
        const int per_group = p.group * p.q_blocks;
        const int gi = pos / per_group, within = pos - gi * per_group;
        qb = p.q_blocks - 1 - within / p.group;
        pair = first + gi * p.group + within % p.group;
    }
    const int kv = pair / G;
    const int b = kv / p.Hkv, hk = kv - b * p.Hkv;
    const int hq = hk * G + (pair - kv * G);
    const int q0 = qb * BQ, q0w = q0 + qw * QW;
    const int T = p.T;

    // steps this work-group walks, and the keys this wave's queries see
    const int kend = p.causal ? (q0 + BQ < T ? q0 + BQ : T) : T;
    const int nb = (kend + ROWS - 1) / ROWS;
    int kend_w = p.causal && q0w + QW < T ? q0w + QW : T;
    if (q0w >= T) kend_w = 0;
    const int nbw = (kend_w + BKV - 1) / BKV;                // without key groups: the steps this wave needs

    auto make_rsrc = [&](const __bf16 *base, int64_t st) {
        return __builtin_amdgcn_make_buffer_rsrc((void *)uniform_ptr((const char *)base), 0,
                                                 __builtin_amdgcn_readfirstlane((uint32_t)((((int64_t)T - 1) * st + D) * 2)), kBufFlags);
    };
    const __amdgpu_buffer_rsrc_t rsrc_q = make_rsrc(p.Q + (int64_t)b * p.q_sb + (int64_t)hq * p.q_sh, p.q_st);
    const __amdgpu_buffer_rsrc_t rsrc_k = make_rsrc(p.K + (int64_t)b * p.k_sb + (int64_t)hk * p.k_sh, p.k_st);
    const __amdgpu_buffer_rsrc_t rsrc_v = make_rsrc(p.V + (int64_t)b * p.v_sb + (int64_t)hk * p.v_sh, p.v_st);

    // ---- K / V block loads: wave w fills the 1 KB pieces w, w + NT, ... of each tile -------------
    // Lane l of a wave-wide load writes 16 bytes at piece + 16 l, i.e. row l / CPR of the piece,
    // chunk position l % CPR: it fetches the chunk that belongs there under the swizzle.  Rows at
    // or beyond T lie outside the descriptor's range and arrive as zeros.  One per-lane offset serves
    // all of a wave's loads; the piece and the key block go into the scalar offset.
    // LDS: two stages of a K tile and a V tile; block j uses stage j % 2.
    uint32_t k_off, v_off;
    {
        const int row = wave * RPL + lane / CPR, pos = lane % CPR;
        k_off = (uint32_t)(row * p.k_st * 2 + ((pos ^ swz_keys<D>(row)) << 4));
        v_off = (uint32_t)(row * p.v_st * 2 + ((pos ^ swz_vals<D>(row)) << 4));
    }
    const uint32_t k_blk = (uint32_t)(ROWS * p.k_st * 2), v_blk = (uint32_t)(ROWS * p.v_st * 2);
    const uint32_t k_piece = (uint32_t)(NT * RPL * p.k_st * 2), v_piece = (uint32_t)(NT * RPL * p.v_st * 2);
    auto load_block = [&](int j, int stage) __attribute__((always_inline)) {
        char *const dst = smem + stage * STAGE_BYTES + wave * 1024;
#pragma unroll
        for (int t = 0; t < L; ++t) load_to_lds_16(rsrc_k, dst + t * NT * 1024, k_off, j * k_blk + t * k_piece);
#pragma unroll
        for (int t = 0; t < L; ++t) load_to_lds_16(rsrc_v, dst + TILE_BYTES + t * NT * 1024, v_off, j * v_blk + t * v_piece);
    };
    load_block(0, 0);

    // ---- Q^T fragments: query r32 of the wave, d = 16 ks + 8 h .. + 7 ----------------------------
    bf16x8_t qf[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
        qf[ks] = __builtin_bit_cast(bf16x8_t, __builtin_amdgcn_raw_buffer_load_b128(rsrc_q, (uint32_t)(((q0w + r32) * p.q_st + 16 * ks + 8 * h) * 2), 0, 0));

    // ---- LDS fragment addresses (relative to the tile) -------------------------------------------
    // K tile kt, group ks: row 32 kt + r32, chunk (2 ks + h) ^ swizzle(r32): ks sits in address bits 5
    // and up, which the XOR leaves to it, so group ks is the group-0 address ^ (ks << 5).
    const uint32_t k_addr = (uint32_t)(r32 * ROWB + ((h ^ swz_keys<D>(r32)) << 4));
    // V^T tile dt, 16-key group u, half: a transposing read hands lane i of a 16-lane group column
    // (= d) i of the 4 rows (= keys) whose addresses lanes 4 jj + cc supply for columns 4 cc .. 4 cc + 3.
    // Keys 16 u + 8 half + 4 h + jj: the permutation P^T comes in.  Tile dt is the tile-0 address ^ (dt << 6).
    const int jj = (lane >> 2) & 3, cc = lane & 3, g1 = (lane >> 4) & 1;
    const uint32_t v_addr = (uint32_t)((4 * h + jj) * ROWB + (((2 * g1 + (cc >> 1)) ^ swz_vals<D>(4 * h + jj)) << 4) + (cc & 1) * 8);

    f32x16_t o[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[dt][r] = 0.f;
    // m is the REFERENCE exponent of the query's running sums, not its running maximum: it is the first
    // block's largest score, and is raised (and the sums rescaled) only when the probabilities that a
    // lane has computed with it add up to more than kMaxSum (or to no number).  None of them is above
    // kMaxSum then, harmless in bf16 and fp32, and most key blocks need neither a maximum nor a rescaling:
    // 26 of 150 vector instructions of a block.  The branch is uniform over the wave.
    // It is never below p.lowest = -2^31 / c, where m * c is rounded by more than the exponential can hold.  Callers mask keys through
    // scores of minus infinity or of a type's lowest value, and all keys of a block, or of a key group, may be such: with a reference
    // among them their probabilities would be infinite or no numbers, and so would the sums that they are added to, even with weight
    // zero.  Like this they are zero.
    constexpr float kMaxSum = 256.0f;
    const float c = p.scale_log2;
    float m = p.lowest, l = 0.f;

    // One key block.  `stage` is a constant after inlining.
    auto step = [&](int j, int stage) __attribute__((always_inline)) {
        // block j has landed, for every wave, and every wave is done with block j - 1, whose stage the
        // next loads overwrite
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        const int k0 = j * ROWS + kg * BKV;                      // the wave's key block
        if (KG > 1 ? k0 >= kend_w : j >= nbw) {                  // nothing (more) this wave's queries may see
            if (j + 1 < nb) load_block(j + 1, stage ^ 1);
            return;
        }
        const char *const kt_lds = smem + stage * STAGE_BYTES + kg * BKV * ROWB, *const vt_lds = kt_lds + TILE_BYTES;
        f32x16_t S[KT];
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
#pragma unroll
            for (int r = 0; r < 16; ++r) S[kt][r] = 0.f;
        // Priority while the score MFMAs are issued: two waves that reach them together would share the pipe, finish
        // together and then compete for the vector ALU; like this one of them goes ahead and the other's
        // MFMAs run under its softmax (2 x 4096 tokens, 32 / 8 heads of 128, full: 498 -> 478 us).
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_setprio(1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int kt = 0; kt < KT; ++kt)
                S[kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*(const bf16x8_t *)(kt_lds + (k_addr ^ (ks << 5)) + kt * 32 * ROWB), qf[ks], S[kt], 0, 0, 0);

        // The V^T fragments go to registers here, before the next block's loads: the compiler waits for every
        // outstanding load into LDS before a transposing read.
        s16x4_t vf[UB][DT][2];
#pragma unroll
        for (int u = 0; u < UB; ++u)
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                for (int half = 0; half < 2; ++half)
                    vf[u][dt][half] = read_transposed(vt_lds + ((v_addr ^ (dt << 6)) + (16 * u + 8 * half) * ROWB));
        // all of it in one order: a few K fragments, then LDS reads between the MFMAs (296 -> 290 us at 4 x 4096 tokens, 16 heads of 64)
        __builtin_amdgcn_sched_group_barrier(0x100, 6, 0);
#pragma unroll
        for (int i = 0; i < KS * KT; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (j + 1 < nb) load_block(j + 1, stage ^ 1);
        __builtin_amdgcn_s_setprio(0);
        __builtin_amdgcn_sched_barrier(0);

        if (p.causal ? (k0 + BKV - 1 > q0w) : (k0 + BKV > T)) {
            const int last = (p.causal ? q0w + r32 : T - 1) - k0 - 4 * h;       // last key this query sees
#pragma unroll
            for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (32 * kt + 8 * (r / 4) + r % 4 > last) S[kt][r] = -__builtin_inff();
        }
        // the probabilities, and the lane's sum of them as rounded (the numerator uses the same), in fp32
        u32x4_t pf[UB];
        float lb = 0.f;
        auto probabilities = [&]() __attribute__((always_inline)) {
            const float mc = m * c;
            const bf16x2_t ones = __builtin_bit_cast(bf16x2_t, 0x3F803F80u);
            lb = 0.f;
#pragma unroll
            for (int u = 0; u < UB; ++u)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int r = 8 * (u & 1) + 2 * i;
                    const f32x2_t pr = {exp2_fast(__builtin_fmaf(S[u / 2][r], c, -mc)), exp2_fast(__builtin_fmaf(S[u / 2][r + 1], c, -mc))};
                    const bf16x2_t pb = __builtin_convertvector(pr, bf16x2_t);
                    lb = __builtin_amdgcn_fdot2_f32_bf16(pb, ones, lb, false);
                    pf[u][i] = __builtin_bit_cast(uint32_t, pb);
                }
        };
        bool raise = j == 0;
        if (!raise) {
            probabilities();
            raise = __builtin_amdgcn_ballot_w64(!(lb <= kMaxSum)) != 0;
        }
        if (raise) {
            float mx = fmaxf(S[0][0], S[0][1]);
#pragma unroll
            for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                for (int r = 0; r < 16; r += 2) mx = fmaxf(fmaxf(mx, S[kt][r]), S[kt][r + 1]);
            mx = max_with_lane_xor32(mx);
            const float m_new = fmaxf(m, mx);
            const float alpha = exp2_fast((m - m_new) * c);
            m = m_new;
            l *= alpha;
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                for (int r = 0; r < 16; ++r) o[dt][r] *= alpha;
            probabilities();
        }
        l += lb;
#pragma unroll
        for (int u = 0; u < UB; ++u)
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
                o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, __builtin_shufflevector(vf[u][dt][0], vf[u][dt][1], 0, 1, 2, 3, 4, 5, 6, 7)),
                                                                __builtin_bit_cast(bf16x8_t, pf[u]), o[dt], 0, 0, 0);
    };
    for (int j = 0; j < nb; j += 2) {
        step(j, 0);
        if (j + 1 < nb) step(j + 1, 1);
    }

    // ---- the key groups' sums: group g finishes the d tiles g, g + KG, ... of its queries and gets the other groups' sums of them
    // through LDS, with their reference exponents.  Added in ascending group order: the result is bit-reproducible.
    if constexpr (KG > 1) {
        typedef float f32x4_t __attribute__((ext_vector_type(4)));
        f32x4_t *const tiles = (f32x4_t *)smem;                                    // [d tile][sender's rank][query group][quarter][lane]
        f32x2_t *const refs = (f32x2_t *)(smem + DT * (KG - 1) * NW * 4096);       // [group][query group][lane]
        static_assert(DT * (KG - 1) * NW * 4096 + NT * 512 <= lds_bytes(D, NW, KG, BKV), "LDS");
        __syncthreads();                                                           // every wave is done with the key blocks
        refs[(kg * NW + qw) * 64 + lane] = f32x2_t{m, l};
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
            if (dt % KG != kg) {
                f32x4_t *const to = tiles + ((dt * (KG - 1) + (kg + KG - dt % KG) % KG - 1) * NW + qw) * 256 + lane;
#pragma unroll
                for (int i = 0; i < 4; ++i) to[i * 64] = f32x4_t{o[dt][4 * i], o[dt][4 * i + 1], o[dt][4 * i + 2], o[dt][4 * i + 3]};
            }
        __syncthreads();
        f32x2_t of[KG];
        float m_all = m;
#pragma unroll
        for (int g = 0; g < KG; ++g) { of[g] = refs[(g * NW + qw) * 64 + lane]; m_all = fmaxf(m_all, of[g].x); }
        l = 0.f;
#pragma unroll
        for (int g = 0; g < KG; ++g) { of[g].x = exp2_fast((of[g].x - m_all) * c); l += of[g].x * of[g].y; }
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
            if (dt % KG == kg) {
                f32x16_t sum;
#pragma unroll
                for (int r = 0; r < 16; ++r) sum[r] = 0.f;
#pragma unroll
                for (int g = 0; g < KG; ++g) {
                    const f32x4_t *const from = tiles + ((dt * (KG - 1) + (g + KG - dt % KG) % KG - 1) * NW + qw) * 256 + lane;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const f32x4_t other = g == kg ? f32x4_t{o[dt][4 * i], o[dt][4 * i + 1], o[dt][4 * i + 2], o[dt][4 * i + 3]} : from[i * 64];
#pragma unroll
                        for (int e = 0; e < 4; ++e) sum[4 * i + e] += of[g].x * other[e];
                    }
                }
                o[dt] = sum;
            }
    }
    if (KG > 1 ? q0w >= T : nbw == 0) return;

    // ---- normalise and store: lane holds d = 32 dt + 8 g + 4 h + 0..3 (g = 0..3) of query q0w + r32; the two
    // lanes of a query trade halves, after which a lane holds 8 consecutive d -----------------------
    const float inv = 1.0f / sum_with_lane_xor32(l);
    const int query = q0w + r32;
    __bf16 *row = p.O + (int64_t)b * p.o_sb + (int64_t)hq * p.o_sh + (int64_t)query * p.o_st + 8 * h;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
        if (KG > 1 && dt % KG != kg) continue;
#pragma unroll
        for (int g = 0; g < 4; g += 2) {
            uint32_t w[2][2];
#pragma unroll
            for (int e = 0; e < 2; ++e)
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const int r = 4 * (g + e) + 2 * i;
                    const f32x2_t v = {o[dt][r] * inv, o[dt][r + 1] * inv};
                    w[e][i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
                }
            const auto lo = __builtin_amdgcn_permlane32_swap(w[0][0], w[1][0], false, false);
            const auto hi = __builtin_amdgcn_permlane32_swap(w[0][1], w[1][1], false, false);
            if (query < T) *(u32x4_by8 *)(row + 32 * dt + 8 * g) = u32x4_t{(uint32_t)lo[0], (uint32_t)hi[0], (uint32_t)lo[1], (uint32_t)hi[1]};
        }
    }
#else
    (void)p;
#endif
}

}  // namespace attn
}  // namespace fact
