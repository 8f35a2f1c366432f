// GEMM with little to do for each work-group: few rows against weights as a linear layer stores them (B as [N][K]; decode
// steps, a handful of tokens), and small outputs of either layout of B.
// A call of few rows reads N x K weights once and does next to nothing with them, so it is bound by how many bytes the
// whole chip has in flight.  The main kernel's tiles give it too few work-groups (64 of 64 x 64 for 4096 columns) that
// each walk all of K through a ring of LDS stages with a barrier per step.  Here a work-group owns 16 NT columns and
// its NW waves split K between them, 64 values at a time in turn.  Each wave has a ring of S stages in LDS to itself,
// filled by direct global -> LDS loads of 8 rows x 128 bytes (whole lines), S - 1 stages ahead, so there is no barrier
// until the waves' sums meet at the end.  (Loads into registers, in the matrix instruction's own layout of 16 rows x
// 64 bytes or as whole lines with the halves exchanged between lanes, stay at 23 and 33 GB/s per compute unit however
// many are in flight: 16 x 4096 x 14336 took 38 and 33 us, this form 25.6 us.)
#include "launch.h"
#include "lds_limit.h"
#include "shift_down.h"

namespace fact {

template <bool F16>
__device__ __forceinline__ f32x4_t mfma_skinny(u32x4_t a, u32x4_t b, f32x4_t c)
{
    typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));
    if constexpr (F16) return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8_t, a), __builtin_bit_cast(f16x8_t, b), c, 0, 0, 0);
    else return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}

// LDS layout of a block of a [K][N] operand: 64 K-rows of 16 NT columns as in memory, the 16-byte piece c of K-row k at
// position c ^ swz_cols(k).  A transposing read takes 4 K-rows x 32 bytes per 16 lanes: rows of 128 bytes (NT = 4) would put
// the four into the same banks, so they are spread over the four 32-byte slots of a row; shorter rows are apart as they are.
template <int NT> __device__ __forceinline__ int swz_cols(int k) { return NT == 4 ? (k & 3) << 1 : 0; }
// The fragments of such a block: [column tile][32 K-values], lane (r16, q) gets K-values 8q .. 8q + 7 of column r16.  Reads
// and wait in one statement: the compiler does not track what inline assembly loads.  (Through the builtin it would wait for
// all loads into LDS before each read.)
template <int NT>
__device__ __forceinline__ void columns_of(uint32_t block, int lane, u32x4_t (&f)[NT][2])
{
    const int q = lane >> 4, jj = (lane >> 2) & 3, c = lane & 3;
    const uint32_t row = block + (8 * q + jj) * (NT * 32) + (c & 1) * 8;
    u32x2_t lo[NT][2], hi[NT][2];
    uint32_t at[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) at[j] = row + (((2 * j + (c >> 1)) ^ swz_cols<NT>(jj)) << 4);
    constexpr int ROW4 = 4 * NT * 32, ROW32 = 32 * NT * 32;      // 4 K-rows on: the lane's upper half; 32: the second sub-step
    if constexpr (NT == 1) {
        asm volatile("ds_read_b64_tr_b16 %0, %4\n\tds_read_b64_tr_b16 %1, %4 offset:%5\n\tds_read_b64_tr_b16 %2, %4 offset:%6\n\t"
                     "ds_read_b64_tr_b16 %3, %4 offset:%7\n\ts_waitcnt lgkmcnt(0)"
                     : "=&v"(lo[0][0]), "=&v"(hi[0][0]), "=&v"(lo[0][1]), "=&v"(hi[0][1])
                     : "v"(at[0]), "n"(ROW4), "n"(ROW32), "n"(ROW32 + ROW4) : "memory");
    } else {
#pragma unroll
        for (int j = 0; j < NT; j += 2)
            asm volatile("ds_read_b64_tr_b16 %0, %8\n\tds_read_b64_tr_b16 %1, %8 offset:%10\n\tds_read_b64_tr_b16 %2, %8 offset:%11\n\t"
                         "ds_read_b64_tr_b16 %3, %8 offset:%12\n\tds_read_b64_tr_b16 %4, %9\n\tds_read_b64_tr_b16 %5, %9 offset:%10\n\t"
                         "ds_read_b64_tr_b16 %6, %9 offset:%11\n\tds_read_b64_tr_b16 %7, %9 offset:%12\n\ts_waitcnt lgkmcnt(0)"
                         : "=&v"(lo[j][0]), "=&v"(hi[j][0]), "=&v"(lo[j][1]), "=&v"(hi[j][1]),
                           "=&v"(lo[j + 1][0]), "=&v"(hi[j + 1][0]), "=&v"(lo[j + 1][1]), "=&v"(hi[j + 1][1])
                         : "v"(at[j]), "v"(at[j + 1]), "n"(ROW4), "n"(ROW32), "n"(ROW32 + ROW4) : "memory");
    }
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) f[j][kk] = u32x4_t{lo[j][kk].x, lo[j][kk].y, hi[j][kk].x, hi[j][kk].y};
}

// The waves' sums, added in ascending wave order (a fixed order: the result is bit-reproducible), the epilogue, the store.  A wave
// finishes at most one tile; its bias and residual are asked for before the sums meet, in one trip to memory (one after the other
// behind the sums, and element by element where 4 columns cross the last one: 7 x 2731 x 1284 4.6 us, like this 4.2, 5 x 207 x 205
// [K][N] 4.5 and 3.9).  Calls of few rows are a chain of latencies, in which 0.1 us of branches count: a gate only where one can be asked
// for (GATE), bias and residual behind one uniform branch and no test for rows that the grid guarantees (24 x 664 x 248 2.94 -> 2.76 us,
// 52 x 2176 x 120 3.48 -> 3.28).
template <int MT, int NT, int NW, bool GATE, bool F16>
__device__ __forceinline__ void finish(const GemmArgs &p, const f32x4_t (&acc)[MT][NT], f32x4_t *sums, int wave, int lane, int m0, int n0, int64_t z)
{
    static_assert(MT * NT <= NW, "a tile per wave");
    const int r16 = lane & 15, q = lane >> 4;
    const bool gated = GATE && p.act == ACT_SILU_GATE;
    const int nout = gated ? p.N >> 1 : p.N;
    const int OT = gated ? NT / 2 : NT;                      // output column tiles
    const uint16_t *res = p.res ? (const uint16_t *)(p.res + z * p.stride_r) : nullptr;
    const uint16_t *bias = (const uint16_t *)p.bias;
    const int t = wave / OT, j = wave - t * OT;
    const int m = m0 + 16 * t + r16, n = n0 + 16 * j + 4 * q;             // the lane's four columns
    const bool live = t < MT && m < p.M && n < nout, full = n + 4 <= nout;
    auto load4 = [&](const uint16_t *from) __attribute__((always_inline)) {
        if (full) return *(const u32x2_any *)from;
        const int left = nout - n;
        const uint32_t x0 = from[0], x1 = from[left > 1 ? 1 : 0], x2 = from[left > 2 ? 2 : 0];
        return u32x2_t{x0 | (x1 << 16), x2};
    };
    u32x2_t wb = {0u, 0u}, wr = {0u, 0u};
    if (bias || res) {
        if (live && bias) wb = load4(bias + n);
        if (live && res) wr = load4(res + (int64_t)m * p.ldr + n);
    }
    __syncthreads();                                         // every wave is done with its blocks
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int k = 0; k < NT; ++k) sums[((i * NT + k) * NW + wave) * 64 + lane] = acc[i][k];
    __syncthreads();
    if (live) {
        auto total = [&](int tile) __attribute__((always_inline)) {
            f32x4_t v = sums[tile * NW * 64 + lane];
#pragma unroll
            for (int w = 1; w < NW; ++w) v += sums[(tile * NW + w) * 64 + lane];
            return v;
        };
        f32x4_t v = total(t * NT + j);
        if (gated) {
            const f32x4_t u = total(t * NT + NT / 2 + j);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = silu(v[e]) * u[e];
        }
        if (bias) {
            v[0] += in16<F16>(wb.x & 0xFFFFu); v[1] += in16<F16>(wb.x >> 16); v[2] += in16<F16>(wb.y & 0xFFFFu); v[3] += in16<F16>(wb.y >> 16);
        }
        if (p.act == ACT_GELU_TANH) {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = gelu_tanh(v[e]);
        }
        if (res) {
            v[0] += in16<F16>(wr.x & 0xFFFFu); v[1] += in16<F16>(wr.x >> 16); v[2] += in16<F16>(wr.y & 0xFFFFu); v[3] += in16<F16>(wr.y >> 16);
        }
        if (p.c_f32) {
            float *c = (float *)p.C + z * p.stride_c + (int64_t)m * p.ldc + n;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (n + e < nout) c[e] = v[e];
        } else {
            uint16_t *c = (uint16_t *)(p.C + z * p.stride_c) + (int64_t)m * p.ldc + n;
            if (full) {
                *(u32x2_any *)c = u32x2_t{pack2<F16>(pk_f32_t{v[0], v[1]}), pack2<F16>(pk_f32_t{v[2], v[3]})};
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (n + e < nout) c[e] = (uint16_t)out16<F16>(v[e]);
            }
        }
    }
}

// MT x NT tiles of 16 x 16; gated: the first NT / 2 column tiles are gate columns, the others the same up columns.
// STREAM: B is asked for as non-temporal data, which leaves no copy of it in the memory-side cache (see kStreamBytes).
template <int MT, int NT, int NW, int S, bool TRANS_B, bool STREAM, bool F16>
__global__ void __launch_bounds__(64 * NW)
skinny_kernel(const GemmArgs p)
{
#if defined(__HIP_DEVICE_COMPILE__)      // the host pass only needs the kernel's symbol
    constexpr int STAGE = (MT + NT) * 2048, L = (MT + NT) * 2;       // bytes and loads of a stage
    static_assert((S - 1) * L <= 63, "vmcnt range");
    constexpr int kPolicyB = STREAM ? 2 : 0;                         // cache-policy bit nt
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    f32x4_t *const sums = (f32x4_t *)smem;                           // [tile][wave][lane], once the rings are done with
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int r16 = lane & 15, q = lane >> 4;
    constexpr bool GATE = TRANS_B && NT == 2;                // the tiles that gated calls take
    const bool gated = GATE && p.act == ACT_SILU_GATE;
    const int nout = gated ? p.N >> 1 : p.N;
    const int OT = gated ? NT / 2 : NT;                      // output column tiles
    const int n0 = blockIdx.x * 16 * OT, m0 = blockIdx.y * 16 * MT;
    const int64_t z = blockIdx.z;

    // Loads: lane l writes 16 bytes at stage + 1024 load + 16 l, row l / 8 of the load, and fetches the piece that belongs
    // there under the swizzle.  Rows past the matrix are beyond the descriptor's range and pieces past K are pushed
    // there by an offset bit: both arrive as zeros.
    auto rsrc_of = [&](const __bf16 *base, int64_t row0, int rows_left, int64_t ld, int rows_max) __attribute__((always_inline)) {
        const int rows = rows_left < rows_max ? rows_left : rows_max;        // (at least 1: the grid ends with the matrix; ld <= 2^21: the range fits 31 bits)
        return __builtin_amdgcn_make_buffer_rsrc((void *)wave_uniform((const char *)(base + row0 * ld)), 0,
                                                 wave_uniform((uint32_t)(((int64_t)(rows - 1) * ld + p.K) * 2)), kBufferFlags);
    };
    const int chunk = (lane & 7) ^ (lane >> 3);
    const __amdgpu_buffer_rsrc_t rsrc_a = rsrc_of(p.A + z * p.stride_a, m0, p.M - m0, p.lda, 16 * MT);
    __amdgpu_buffer_rsrc_t rsrc_b, rsrc_u;
    uint32_t va[2 * MT], vb[2 * NT];
#pragma unroll
    for (int i = 0; i < 2 * MT; ++i) va[i] = (uint32_t)(((8 * i + (lane >> 3)) * p.lda + chunk * 8) * 2);
    // B as [K][N]: a block's 64 K-rows of 16 NT columns, RPL rows to a load; the descriptor moves with the block, so that its
    // range ends with the last K-row, and pieces past the last column are pushed beyond it (N is a multiple of 8).
    constexpr int CPR = 2 * NT, RPL = 64 / CPR;              // 16-byte pieces of a K-row, K-rows of a load
    const char *slab = nullptr;
    int64_t slab_bytes = 0;
    if constexpr (TRANS_B) {
        rsrc_b = rsrc_of(p.B + z * p.stride_b, n0, nout - n0, p.ldb, 16 * OT);
        rsrc_u = rsrc_of((gated ? p.B_up : p.B) + z * p.stride_b, n0, nout - n0, p.ldb, 16 * OT);
#pragma unroll
        for (int j = 0; j < 2 * NT; ++j) vb[j] = (uint32_t)(((8 * (gated && j >= NT ? j - NT : j) + (lane >> 3)) * p.ldb + chunk * 8) * 2);
    } else {
        slab = (const char *)(p.B + z * p.stride_b + (int64_t)wave * 64 * p.ldb + n0);
        slab_bytes = (int64_t)NW * 64 * p.ldb * 2;
        const int nc = (lane % CPR) ^ swz_cols<NT>(lane / CPR);
        const uint32_t past = n0 + nc * 8 < p.N ? 0u : kOobOffset;
#pragma unroll
        for (int j = 0; j < 2 * NT; ++j) vb[j] = (uint32_t)(((j * RPL + lane / CPR) * p.ldb + nc * 8) * 2) | past;
    }
    const int blocks = (p.K + 63) >> 6;
    const int mine = blocks > wave ? (blocks - wave + NW - 1) / NW : 0;
    char *const ring = smem + wave * S * STAGE;
    auto load = [&](int i, int slot) __attribute__((always_inline)) {        // (a block past the last reads nothing)
        const int k = (wave + i * NW) * 64;
        const uint32_t beyond = i >= mine || k + chunk * 8 >= p.K ? kOobOffset : 0u;
        const int soff = i < mine ? k * 2 : 0;
        char *dst = ring + slot * STAGE;
        if constexpr (!TRANS_B) {
            const int rows = i < mine ? (p.K - k < 64 ? p.K - k : 64) : 0;
            rsrc_b = __builtin_amdgcn_make_buffer_rsrc((void *)wave_uniform(slab + i * slab_bytes), 0,
                                                       wave_uniform((uint32_t)(rows > 0 ? ((int64_t)(rows - 1) * p.ldb + (p.N - n0)) * 2 : 0)), kBufferFlags);
#pragma unroll
            for (int j = 0; j < 2 * NT; ++j) __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_b, FACT_LDS_PTR(dst + (2 * MT + j) * 1024), 16, vb[j], 0, 0, kPolicyB);
        } else
#pragma unroll
        for (int j = 0; j < 2 * NT; ++j) {
            if (gated && j >= NT) __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_u, FACT_LDS_PTR(dst + (2 * MT + j) * 1024), 16, vb[j] | beyond, soff, 0, kPolicyB);
            else __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_b, FACT_LDS_PTR(dst + (2 * MT + j) * 1024), 16, vb[j] | beyond, soff, 0, kPolicyB);
        }
#pragma unroll
        for (int t = 0; t < 2 * MT; ++t) __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_a, FACT_LDS_PTR(dst + t * 1024), 16, va[t] | beyond, soff, 0, 0);
    };
    f32x4_t acc[MT][NT];
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[t][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int d = 0; d < S - 1; ++d) load(d, d);
    int slot = 0, fill = S - 1;
    for (int i = 0; i < mine; ++i) {
        // block i has landed; the previous block's fragments are in registers, so its slot may be filled again
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((S - 2) * L) : "memory");
        load(i + S - 1, fill);
        const char *s = ring + slot * STAGE;
        u32x4_t bt[TRANS_B ? 1 : NT][2];
        if constexpr (!TRANS_B) columns_of<NT>((uint32_t)(size_t)FACT_LDS_PTR(s + MT * 2048), lane, bt);
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            const int at = r16 * 128 + (((4 * kk + q) ^ (r16 & 7)) << 4);
            u32x4_t a[MT], b[NT];
#pragma unroll
            for (int t = 0; t < MT; ++t) a[t] = *(const u32x4_t *)(s + t * 2048 + at);
#pragma unroll
            for (int j = 0; j < NT; ++j) {
                if constexpr (TRANS_B) b[j] = *(const u32x4_t *)(s + (MT + j) * 2048 + at);
                else b[j] = bt[j][kk];
            }
#pragma unroll
            for (int t = 0; t < MT; ++t)
#pragma unroll
                for (int j = 0; j < NT; ++j) acc[t][j] = mfma_skinny<F16>(b[j], a[t], acc[t][j]);
        }
        fill = slot;
        slot = slot + 1 == S ? 0 : slot + 1;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // loads past the last block still write LDS
    finish<MT, NT, NW, GATE, F16>(p, acc, sums, wave, lane, m0, n0, z);
#else
    (void)p;
#endif
}

// The same for rows that start at any 2-byte address and any M, N, K of at least a piece (not gated): the pieces pass through
// registers, D blocks of 64 K-values ahead, into an LDS block of the wave's own, still without a barrier until the sums meet.  A
// piece that would cross the end of a row, or the last column of a [K][N] operand, is loaded so that it ends there and
// moved down; K-values past K are zeros, so that every wave may run whole rounds of D blocks.
template <int MT, int NT, int NW, int D, bool TRANS_B, bool F16>
__global__ void __launch_bounds__(64 * NW)
skinny_any_kernel(const GemmArgs p)
{
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int STAGE = (MT + NT) * 2048, CPR = 2 * NT, RPL = 64 / CPR;
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int r16 = lane & 15, q = lane >> 4, K = p.K;
    const int n0 = blockIdx.x * 16 * NT, m0 = blockIdx.y * 16 * MT;
    const int64_t z = blockIdx.z;
    // lane -> piece lane % 8 of rows lane / 8 + 8 i (K-contiguous), piece lane % CPR of K-rows lane / CPR + RPL j ([K][N]); rows past
    // the edge repeat the last one: their results are not stored
    const int kc = lane & 7;
    const uint16_t *pa[2 * MT], *pb[TRANS_B ? 2 * NT : 1];
#pragma unroll
    for (int i = 0; i < 2 * MT; ++i) {
        const int m = m0 + 8 * i + (lane >> 3);
        pa[i] = (const uint16_t *)(p.A + z * p.stride_a) + (int64_t)(m < p.M ? m : p.M - 1) * p.lda;
    }
    int shift_n = 0;
    if constexpr (TRANS_B) {
#pragma unroll
        for (int j = 0; j < 2 * NT; ++j) {
            const int n = n0 + 8 * j + (lane >> 3);
            pb[j] = (const uint16_t *)(p.B + z * p.stride_b) + (int64_t)(n < p.N ? n : p.N - 1) * p.ldb;
        }
    } else {
        int n = n0 + (lane % CPR) * 8;
        if (n > p.N - 8) { shift_n = n - (p.N - 8); n = p.N - 8; }
        pb[0] = (const uint16_t *)(p.B + z * p.stride_b) + n;
    }
    const bool ragged_n = !TRANS_B && n0 + 16 * NT > p.N;
    struct Block { u32x4_t a[2 * MT], b[2 * NT]; } r[D];
    auto fetch = [&](Block &t, int i) __attribute__((always_inline)) {
        const int k = (wave + i * NW) * 64, c = k + kc * 8, at = c < K - 8 ? c : K - 8;
#pragma unroll
        for (int j = 0; j < 2 * NT; ++j) {
            if constexpr (TRANS_B) t.b[j] = *(const u32x4_any *)(pb[j] + at);
            else {
                const int row = k + j * RPL + lane / CPR;
                t.b[j] = *(const u32x4_any *)(pb[0] + (int64_t)(row < K ? row : K - 1) * p.ldb);
            }
        }
#pragma unroll
        for (int x = 0; x < 2 * MT; ++x) t.a[x] = *(const u32x4_any *)(pa[x] + at);
    };
    char *const s = smem + wave * STAGE;
    auto put = [&](Block &t, int i) __attribute__((always_inline)) {
        const int k = (wave + i * NW) * 64;
        if (k + 64 > K) {
            const int c = k + kc * 8, by = c < K - 8 ? 0 : c - (K - 8);
#pragma unroll
            for (int x = 0; x < 2 * MT; ++x) t.a[x] = shift_down(t.a[x], by);
#pragma unroll
            for (int j = 0; j < 2 * NT; ++j) {
                if constexpr (TRANS_B) t.b[j] = shift_down(t.b[j], by);
                else if (k + j * RPL + lane / CPR >= K) t.b[j] = u32x4_t{0u, 0u, 0u, 0u};
            }
        }
        if (ragged_n) {
#pragma unroll
            for (int j = 0; j < 2 * NT; ++j) t.b[j] = shift_down(t.b[j], shift_n);
        }
        const int at = (lane >> 3) * 128 + ((kc ^ (lane >> 3)) << 4);        // (rows 8 apart: the same swizzle)
#pragma unroll
        for (int x = 0; x < 2 * MT; ++x) *(u32x4_t *)(s + x * 1024 + at) = t.a[x];
#pragma unroll
        for (int j = 0; j < 2 * NT; ++j) {
            if constexpr (TRANS_B) *(u32x4_t *)(s + (2 * MT + j) * 1024 + at) = t.b[j];
            else {
                const int row = j * RPL + lane / CPR;
                *(u32x4_t *)(s + MT * 2048 + row * (NT * 32) + (((lane % CPR) ^ swz_cols<NT>(row)) << 4)) = t.b[j];
            }
        }
    };
    f32x4_t acc[MT][NT];
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[t][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    const int blocks = (K + 63) >> 6;
    const int mine = blocks > wave ? (blocks - wave + NW - 1) / NW : 0;
    auto multiply = [&]() __attribute__((always_inline)) {
        u32x4_t bt[TRANS_B ? 1 : NT][2];
        if constexpr (!TRANS_B) columns_of<NT>((uint32_t)(size_t)FACT_LDS_PTR(s + MT * 2048), lane, bt);
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            const int at = r16 * 128 + (((4 * kk + q) ^ (r16 & 7)) << 4);
            u32x4_t a[MT], b[NT];
#pragma unroll
            for (int t = 0; t < MT; ++t) a[t] = *(const u32x4_t *)(s + t * 2048 + at);
#pragma unroll
            for (int j = 0; j < NT; ++j) {
                if constexpr (TRANS_B) b[j] = *(const u32x4_t *)(s + (MT + j) * 2048 + at);
                else b[j] = bt[j][kk];
            }
#pragma unroll
            for (int t = 0; t < MT; ++t)
#pragma unroll
                for (int j = 0; j < NT; ++j) acc[t][j] = mfma_skinny<F16>(b[j], a[t], acc[t][j]);
        }
    };
    // The lanes read what other lanes of the wave have stored.  The hardware keeps a wave's LDS accesses in order; this keeps the
    // compiler, which reasons per lane, from moving one over another that only a different lane's address makes depend on it.
    auto in_order = []() __attribute__((always_inline)) { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); __builtin_amdgcn_wave_barrier(); };
    if (mine > D) {
#pragma unroll
        for (int d = 0; d < D; ++d) fetch(r[d], d);
        for (int i = 0; i < mine; i += D) {
#pragma unroll
            for (int d = 0; d < D; ++d) {
                put(r[d], i + d);
                in_order();
                fetch(r[d], i + d + D);
                multiply();
                in_order();
            }
        }
    } else {
        // No more blocks than are loaded ahead: none past the last one, which count where they are half of them (1 x 3001 x 201 [K][N]
        // 3.7 -> 3.1 us, 129 x 513 x 201 5.5 -> 3.7, 129 x 513 x 511 5.9 -> 4.9; with the loop's last round without loads as well, K of 2000 and
        // 4000 is up to 7 % slower).
        static_assert(D == 2, "one block or both");
        if (mine == 2) {
            fetch(r[0], 0);
            fetch(r[1], 1);
            put(r[0], 0);
            in_order();
            multiply();
            in_order();
            put(r[1], 1);
            in_order();
            multiply();
        } else if (mine == 1) {
            fetch(r[0], 0);
            put(r[0], 0);
            in_order();
            multiply();
        }
    }
    finish<MT, NT, NW, false, F16>(p, acc, (f32x4_t *)smem, wave, lane, m0, n0, z);
#else
    (void)p;
#endif
}

template <int MT, int NT, int NW, int D, bool TRANS_B, bool F16>
static hipError_t launch_any_as(const GemmArgs &a, int grid_z, hipStream_t stream)
{
    const dim3 grid((unsigned)((a.N + (int64_t)16 * NT - 1) / (16 * NT)), (unsigned)((a.M + 16 * MT - 1) / (16 * MT)), (unsigned)grid_z);
    constexpr int lds = NW * (MT + NT) * 2048;
    static_assert(lds <= 64 * 1024 && MT * NT * 1024 <= (MT + NT) * 2048, "LDS: the waves' blocks, then their sums");
    hipLaunchKernelGGL((skinny_any_kernel<MT, NT, NW, D, TRANS_B, F16>), grid, dim3(64 * NW), lds, stream, a);
    return hipGetLastError();
}

template <int MT, int NT, int NW, int S, bool TRANS_B, bool STREAM, bool F16>
static hipError_t launch_skinny_as(const GemmArgs &a, int grid_z, hipStream_t stream)
{
    const bool gated = a.act == ACT_SILU_GATE;
    const int nout = gated ? a.N / 2 : a.N, cols = 16 * (gated ? NT / 2 : NT);
    const dim3 grid((unsigned)((nout + (int64_t)cols - 1) / cols), (unsigned)((a.M + 16 * MT - 1) / (16 * MT)), (unsigned)grid_z);
    auto kern = skinny_kernel<MT, NT, NW, S, TRANS_B, STREAM, F16>;
    constexpr int lds = NW * S * (MT + NT) * 2048;
    static_assert(lds <= 160 * 1024 && MT * NT * 1024 <= S * (MT + NT) * 2048, "LDS: rings, then the waves' sums");
    if constexpr (lds > 64 * 1024) {
        static LdsLimit limit;
        const hipError_t e = raise_lds_limit(limit, lds, {(const void *)kern});
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kern, grid, dim3(64 * NW), lds, stream, a);
    return hipGetLastError();
}

// B larger than this is asked for as non-temporal data, which leaves no copy of it in the memory-side cache (us per
// feed-forward block of 16 rows, three sets of weights in turn, cached -> non-temporal; megabytes of the products' weights: 4096 x
// 14336, 352 MB: 73.3 -> 70.7; 2048 x 5632, 69 MB: 17.7 -> 23.0; 1024 x 4096, 17 MB: 10.4 -> 12.0; 768 x 3072: 8.8 -> 10.4).  A fourth of the
// memory-side cache: several such matrices are found there again, larger ones push each other out.  Where a program has so many that
// none is (the caches filled with other data before every call), ordinary loads cost next to nothing up to 23 MB and a few
// per cent above, and where they are they gain up to a third (GEMM of 16 rows, us, ordinary / non-temporal, cold; the same warm):
//    N x K  768 x 3072  6.6 / 6.6; 4.9 / 6.2      2048 x 5632 (23 MB)  9.9 / 9.9; 6.9 / 9.8     4096 x 4096 (34 MB)  9.1 / 9.0; 8.4 / 8.9
//          6144 x 4096 (50 MB) 14.0 / 13.8; 11.0 / 13.3    7168 x 4096 (59 MB) 14.7 / 14.3; 11.5 / 13.6    4096 x 7168 13.5 / 13.0; 11.1 / 12.5
//    (the worst cold: 4096 x 7168 of 1 row 12.3 / 11.5).
constexpr int64_t kStreamBytes = (int64_t)64 << 20;
static bool streams(const GemmArgs &a, int64_t batch) { return (int64_t)a.N * a.K * 2 * batch > kStreamBytes; }

template <int MT, int NT, int NW, int S, bool TRANS_B, bool STREAM>
static hipError_t launch_tile(const GemmArgs &a, int grid_z, hipStream_t stream)
{
    return a.f16 ? launch_skinny_as<MT, NT, NW, S, TRANS_B, STREAM, true>(a, grid_z, stream) : launch_skinny_as<MT, NT, NW, S, TRANS_B, STREAM, false>(a, grid_z, stream);
}

struct Tile { int mt, nt, waves, stages; };
static constexpr Tile kTiles[] = {{1, 1, 4, 4}, {2, 1, 4, 3}, {2, 2, 4, 2}, {1, 2, 4, 4}, {1, 4, 4, 3}, {4, 1, 8, 2}, {2, 2, 4, 4}, {1, 2, 4, 3}, {2, 2, 4, 3}};
static int64_t groups_of(const Tile &t, const GemmArgs &a, int64_t batch)
{
    const bool gated = a.act == ACT_SILU_GATE;
    const int64_t cols = 16 * (gated ? t.nt / 2 : t.nt), nout = gated ? a.N / 2 : a.N;
    return (nout + cols - 1) / cols * (((int64_t)a.M + 16 * t.mt - 1) / (16 * t.mt)) * batch;
}
static int resident(const Tile &t) { return 160 * 1024 / (t.waves * t.stages * (t.mt + t.nt) * 2048); }       // work-groups of a compute unit

// At most 64 rows (32 gated) of [N][K] weights, whatever their size: one 16-column tile per work-group (two for gated calls, one of
// each half, and for many columns of 17-32 rows: half the reads of A); four waves and three or four stages, so that two or
// three work-groups share a compute unit.  Up to 64 rows eight waves and all of the LDS.
static int row_tile(const GemmArgs &a)
{
    if (a.act == ACT_SILU_GATE) return a.M <= 16 ? 7 : 6;
    if (a.M <= 16) return 0;
    if (a.M <= 32) return a.N > 6144 ? 6 : 1;
    return 5;
}

// (a grid's threads are counted in 32 bits: 32 for each column here)
bool skinny_takes(const GemmArgs &a, bool trans_b) { return trans_b && a.M <= (a.act == ACT_SILU_GATE ? 32 : 64) && a.N < 1 << 27; }

// Estimated microseconds: a work-group's K steps one after the other, each at least a load's latency and at most 60 GB/s per
// compute unit, in as many rounds as the work-groups need; a start and an end per round, which nothing covers where
// only one work-group fits a compute unit; never faster than HBM delivers the weights, and A to each XCD.  Rows of weights that
// are no whole 128-byte lines cost more: each 128-byte piece lies on two lines (16 x 4096 x 14336 24.0 us, K = 14344 32.6).
double skinny_us(const GemmArgs &a, int64_t batch, bool whole_lines)
{
    const Tile &t = kTiles[row_tile(a)];
    const bool gated = a.act == ACT_SILU_GATE;
    const int nout = gated ? a.N / 2 : a.N, cols = 16 * (gated ? t.nt / 2 : t.nt);
    const double wx = (double)((nout + (int64_t)cols - 1) / cols), wgs = (double)groups_of(t, a, batch);
    const int fit = resident(t), blocks = (int)(((int64_t)a.K + 63) / 64);
    const double rounds = wgs > 256.0 * fit ? wgs / (256.0 * fit) : 1.0;
    const double sharing = wgs < 256.0 ? 1.0 : wgs / 256.0 < fit ? wgs / 256.0 : fit;
    const double rows_a = 0.5 * (16 * t.mt + (a.M < 16 * t.mt ? a.M : 16 * t.mt));       // (rows past M are not fetched, but their zeros are written)
    const double bytes = 128.0 * (blocks < t.waves ? blocks : t.waves) * (rows_a + 16 * t.nt), step = sharing * bytes / (whole_lines ? 60e3 : 50e3);
    const double chain = 1.4 + 0.004 * wgs + rounds * (0.8 + (blocks + t.waves - 1) / t.waves * (step > 0.2 ? step : 0.2)) + (fit == 1 ? 2.0 * (rounds - 1.0) : 0.0);
    const double memory = 1.4 + (double)batch * a.K * 2.0 * (a.N + (wx < 8.0 ? wx : 8.0) * a.M) / (whole_lines ? 5.4e6 : 4.7e6);
    return chain > memory ? chain : memory;
}

// Small outputs of any number of rows and either layout of B, B from the caches: the tile with the least estimated microseconds,
// among those whose work-groups are all resident at once.  Against the tile kernel, which such a call reaches with a fraction of
// the compute units, a work-group here has a quarter of K per wave, no barrier in the loop, a start and an end 2 us shorter, and
// there are more of them.  The estimate: 3 us, the K steps one after the other at 84 (B as [K][N]) or 108 GB/s per compute unit;
// never faster than the 8.2 or 11.2 TB/s at which the L2s deliver what the work-groups ask for together, nor than B arrives
// once in each XCD that asks for a piece of its lines (as [K][N], a work-group's 16 NT columns are a part of 128-byte lines).
// Fitted to 900 calls of 1 to 1536 rows, 32 to 8192 columns, K of 64 to 8192 (profiles/gemm_small_calls.csv; mean error 9 and 12 %).
struct SmallRates { double start, group, rate, memory_start, memory, pull; };
// B as [K][N], as [N][K], and the latter of many rows: fitted, with plan_one_round, to 1050 calls of up to 8192 rows whose operands lie in the memory-side cache (mean
// error 10 %, the second's there 13: 111 x 2048 x 5632 takes 11.9 us, priced at 15.9 and 19.5)
static constexpr SmallRates kSmallRates[3] = {{3.07, 0.002, 83.6e3, 3.0, 5.38e6, 8.2e6}, {3.07, 0.0015, 107.7e3, 3.0, 4.42e6, 11.2e6}, {3.15, 0.002, 95.1e3, 3.15, 5.27e6, 13.8e6}};
// most: 0, or the most work-groups of a launch in the place of one that plan_one_round priced.
double small_us(const GemmArgs &a, bool trans_b, int64_t batch, int most, int *tile)
{
    const SmallRates &r = kSmallRates[!trans_b ? 0 : most ? 2 : 1];
    double best = 0.0;
    *tile = -1;
    if (a.act == ACT_SILU_GATE || a.N > 8192 || streams(a, batch)) return best;
    if (!trans_b && (int64_t)a.N * a.K >= 1 << 24) return best;      // (from 32 MB of [K][N] on both are bound by memory: 4 x 3928 x 7208 25.9 / 22.7, 3 x 7856 x 4152 17.8 / 18.7)
    const int64_t blocks = ((int64_t)a.K + 63) / 64;
    for (int i = 0; i < 5; ++i) {
        const Tile &t = kTiles[i];
        if (trans_b ? t.nt > t.mt : i == 1) continue;
        // (32 columns for at most 32 rows of weights as [N][K] only where 16 give more work-groups than compute units: up to there the estimates of
        // the two are level, and half of the chip fetches what all of it could: 27 x 3248 x 1864 cold 9.4 and 7.2 us, warm 7.1 and 5.6,
        // 30 x 3800 x 880 6.3 and 5.3, 24 x 3504 x 328 4.5 and 3.8; but 26 x 4856 x 2336, 304 work-groups of 16 columns, 9.8 and 11.9)
        if (trans_b && i == 2 && a.M <= 32 && groups_of(kTiles[1], a, batch) <= 256) continue;
        const int64_t wgs = groups_of(t, a, batch);
        const int fit = resident(t);
        if (wgs > (most && trans_b ? most : 256 * fit) || ((int64_t)a.M + 16 * t.mt - 1) / (16 * t.mt) > 65535) continue;
        const double sharing = wgs > 256 ? wgs / 256.0 : 1.0;
        const double rows_a = 0.5 * (16 * t.mt + (a.M < 16 * t.mt ? a.M : 16 * t.mt));
        const double cols = 16 * t.nt * (trans_b ? 1.0 : t.nt == 1 ? 1.48 : t.nt == 2 ? 1.25 : 1.0);       // (a line's lookups for less than a line)
        double step = sharing * 128.0 * (blocks < t.waves ? blocks : t.waves) * (rows_a + cols) / r.rate;
        if (!trans_b && step < 0.2) step = 0.2;
        const double chain = r.start + r.group * wgs + (blocks + t.waves - 1) / t.waves * step;
        const int64_t wx = ((int64_t)a.N + 16 * t.nt - 1) / (16 * t.nt);
        const double memory = r.memory_start + (double)batch * a.K * 2.0 * (a.N * (trans_b ? 1.0 : 4.0 / t.nt) + (wx < 8 ? wx : 8) * (double)a.M) / r.memory;
        const double pull = r.memory_start + (double)wgs * blocks * 128.0 * (rows_a + cols) / r.pull;
        double us = chain > memory ? chain : memory;
        if (pull > us) us = pull;
        if (*tile < 0 || us < best) { best = us; *tile = i; }
    }
    return best;
}

// The index in kTiles of what runs; tile: small_us's choice, or -1 for the tile of few rows (skinny_us).
int skinny_form(const GemmArgs &a, bool trans_b, int64_t batch, int tile)
{
    if (tile < 0) return row_tile(a);
    // Where the work-groups have a compute unit each, two blocks ahead instead of one, from 2048 K-values on (us; one -> two; 256 x 512 x 8192
    // 16.0 -> 13.3, 96 x 1536 x 4096 10.0 -> 8.5, 64 x 2048 x 2048 6.8 -> 6.2, 300 x 600 x 2048 7.8 -> 7.4; but 256 x 512 x 1024 4.2 -> 4.8, 128 x 1024 x 1024
    // 4.1 -> 4.8; three: as two.  B as [K][N] has nothing of it: 256 x 512 x 8192 19.6 -> 20.0)
    return trans_b && tile == 2 && a.K >= 2048 && groups_of(kTiles[2], a, batch) <= 256 ? 8 : tile;
}

hipError_t launch_skinny_gemm(const GemmArgs &a, bool trans_b, int form, int grid_z, hipStream_t stream)
{
    const bool nt = streams(a, grid_z);
    if (!trans_b) {
        switch (form) {
        case 0: return launch_tile<1, 1, 4, 4, false, false>(a, grid_z, stream);
        case 2: return launch_tile<2, 2, 4, 2, false, false>(a, grid_z, stream);
        case 3: return launch_tile<1, 2, 4, 4, false, false>(a, grid_z, stream);
        case 4: return launch_tile<1, 4, 4, 3, false, false>(a, grid_z, stream);
        default: return hipErrorInvalidConfiguration;
        }
    }
    switch (form) {
    case 0: return nt ? launch_tile<1, 1, 4, 4, true, true>(a, grid_z, stream) : launch_tile<1, 1, 4, 4, true, false>(a, grid_z, stream);
    case 1: return nt ? launch_tile<2, 1, 4, 3, true, true>(a, grid_z, stream) : launch_tile<2, 1, 4, 3, true, false>(a, grid_z, stream);
    case 2: return launch_tile<2, 2, 4, 2, true, false>(a, grid_z, stream);
    case 8: return launch_tile<2, 2, 4, 3, true, false>(a, grid_z, stream);
    case 5: return nt ? launch_tile<4, 1, 8, 2, true, true>(a, grid_z, stream) : launch_tile<4, 1, 8, 2, true, false>(a, grid_z, stream);
    case 6: return nt ? launch_tile<2, 2, 4, 4, true, true>(a, grid_z, stream) : launch_tile<2, 2, 4, 4, true, false>(a, grid_z, stream);
    case 7: return nt ? launch_tile<1, 2, 4, 3, true, true>(a, grid_z, stream) : launch_tile<1, 2, 4, 3, true, false>(a, grid_z, stream);
    default: return hipErrorInvalidConfiguration;
    }
}

// Operands of any alignment: the estimate of small_us with what loads at odd addresses reach (16 bytes per lane from half a
// word run at 36 GB/s per compute unit, from whole words at 99), for a tile of 16 x 16 and one of 32 x 32; fitted to 420 calls of 1 to 3000
// rows, 16 to 4096 columns, K of 16 to 4096 (profiles/gemm_small_odd_calls.csv; mean error 6-9 %).
struct AnyTile { int mt, nt; double start[2], group[2], latency[2], rate[2], pull[2]; };       // [B as [K][N], as [N][K]]
static constexpr AnyTile kAnyTiles[2] = {{1, 1, {3.38, 3.25}, {0.0006, 0.0007}, {0.255, 0.196}, {42.6e3, 78.3e3}, {6.26e6, 10.5e6}},
                                         {2, 2, {4.33, 3.87}, {0.0009, 0.0014}, {0.025, 0.012}, {59.1e3, 75.0e3}, {6.76e6, 9.6e6}}};
double small_any_us(const GemmArgs &a, bool trans_b, int64_t batch, int *tile)
{
    double best = 0.0;
    *tile = -1;
    if (a.act == ACT_SILU_GATE) return best;
    const int64_t blocks = ((int64_t)a.K + 63) / 64;
    for (int i = 0; i < 2; ++i) {
        const AnyTile &t = kAnyTiles[i];
        const int64_t wgs = ((int64_t)a.N + 16 * t.nt - 1) / (16 * t.nt) * (((int64_t)a.M + 16 * t.mt - 1) / (16 * t.mt)) * batch;
        if (wgs > 8192) continue;
        const double rows = 128.0 * 16 * (t.mt + t.nt), sharing = wgs > 256 ? wgs / 256.0 : 1.0;
        const double load = sharing * rows * (blocks < 4 ? blocks : 4) / t.rate[trans_b], step = load > t.latency[trans_b] ? load : t.latency[trans_b];
        const double chain = t.start[trans_b] + t.group[trans_b] * wgs + (blocks + 3) / 4 * step, pull = t.start[trans_b] + (double)wgs * blocks * rows / t.pull[trans_b];
        const double us = chain > pull ? chain : pull;
        if (*tile < 0 || us < best) { best = us; *tile = i; }
    }
    return best;
}

hipError_t launch_small_any(const GemmArgs &a, bool trans_b, int tile, int grid_z, hipStream_t stream)
{
    auto pick = [&](auto tb, auto half) {
        constexpr bool T = decltype(tb)::value, F16 = decltype(half)::value;
        return tile == 0 ? launch_any_as<1, 1, 4, 2, T, F16>(a, grid_z, stream) : launch_any_as<2, 2, 4, 2, T, F16>(a, grid_z, stream);
    };
    if (a.f16) return trans_b ? pick(std::true_type{}, std::true_type{}) : pick(std::false_type{}, std::true_type{});
    return trans_b ? pick(std::true_type{}, std::false_type{}) : pick(std::false_type{}, std::false_type{});
}

}  // namespace fact
