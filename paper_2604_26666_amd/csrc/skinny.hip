// GEMM of few rows against weights as a linear layer stores them (B as [N][K]): decode steps, a handful of tokens.
// Such a call reads N x K weights once and does next to nothing with them, so it is bound by how many bytes the
// whole chip has in flight.  The main kernel's tiles give it too few work-groups (64 of 64 x 64 for 4096 columns) that
// each walk all of K through a ring of LDS stages with a barrier per step.  Here a work-group owns 16 NT columns and
// its NW waves split K between them, 64 values at a time in turn.  Each wave has a ring of S stages in LDS to itself,
// filled by direct global -> LDS loads of 8 rows x 128 bytes (whole lines), S - 1 stages ahead, so there is no barrier
// until the waves' sums meet at the end.  (Loads into registers, in the matrix instruction's own layout of 16 rows x
// 64 bytes or as whole lines with the halves exchanged between lanes, stay at 23 and 33 GB/s per compute unit however
// many are in flight: 16 x 4096 x 14336 took 38 and 33 us, this form 25.6 us.)
#include "launch.h"
#include "lds_limit.h"

namespace fact {

template <bool F16>
__device__ __forceinline__ f32x4_t mfma_skinny(u32x4_t a, u32x4_t b, f32x4_t c)
{
    typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));
    if constexpr (F16) return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8_t, a), __builtin_bit_cast(f16x8_t, b), c, 0, 0, 0);
    else return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}

// MT x NT tiles of 16 x 16; gated: the first NT / 2 column tiles are gate columns, the others the same up columns.
template <int MT, int NT, int NW, int S, bool F16>
__global__ void __launch_bounds__(64 * NW)
skinny_kernel(const GemmArgs p)
{
#if defined(__HIP_DEVICE_COMPILE__)      // the host pass only needs the kernel's symbol
    constexpr int STAGE = (MT + NT) * 2048, L = (MT + NT) * 2;       // bytes and loads of a stage
    static_assert((S - 1) * L <= 63, "vmcnt range");
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    f32x4_t *const sums = (f32x4_t *)smem;                           // [tile][wave][lane], once the rings are done with
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int r16 = lane & 15, q = lane >> 4;
    const bool gated = p.act == ACT_SILU_GATE;
    const int nout = gated ? p.N >> 1 : p.N;
    const int OT = gated ? NT / 2 : NT;                      // output column tiles
    const int n0 = blockIdx.x * 16 * OT, m0 = blockIdx.y * 16 * MT;
    const int64_t z = blockIdx.z;

    // Loads: lane l writes 16 bytes at stage + 1024 load + 16 l, row l / 8 of the load, and fetches the piece that belongs
    // there under the swizzle.  Rows past the matrix are beyond the descriptor's range and pieces past K are pushed
    // there by an offset bit: both arrive as zeros.
    auto rsrc_of = [&](const __bf16 *base, int64_t row0, int rows_left, int64_t ld, int rows_max) __attribute__((always_inline)) {
        const int rows = rows_left < rows_max ? rows_left : rows_max;        // (ld <= 2^21: the range fits 31 bits)
        return __builtin_amdgcn_make_buffer_rsrc((void *)wave_uniform((const char *)(base + row0 * ld)), 0,
                                                 wave_uniform((uint32_t)(rows > 0 ? ((int64_t)(rows - 1) * ld + p.K) * 2 : 0)), kBufferFlags);
    };
    const int chunk = (lane & 7) ^ (lane >> 3);
    const __amdgpu_buffer_rsrc_t rsrc_a = rsrc_of(p.A + z * p.stride_a, m0, p.M - m0, p.lda, 16 * MT);
    const __amdgpu_buffer_rsrc_t rsrc_b = rsrc_of(p.B + z * p.stride_b, n0, nout - n0, p.ldb, 16 * OT);
    const __amdgpu_buffer_rsrc_t rsrc_u = rsrc_of((gated ? p.B_up : p.B) + z * p.stride_b, n0, nout - n0, p.ldb, 16 * OT);
    uint32_t va[2 * MT], vb[2 * NT];
#pragma unroll
    for (int i = 0; i < 2 * MT; ++i) va[i] = (uint32_t)(((8 * i + (lane >> 3)) * p.lda + chunk * 8) * 2);
#pragma unroll
    for (int j = 0; j < 2 * NT; ++j) vb[j] = (uint32_t)(((8 * (gated && j >= NT ? j - NT : j) + (lane >> 3)) * p.ldb + chunk * 8) * 2);
    const int blocks = (p.K + 63) >> 6;
    const int mine = blocks > wave ? (blocks - wave + NW - 1) / NW : 0;
    char *const ring = smem + wave * S * STAGE;
    auto load = [&](int i, int slot) __attribute__((always_inline)) {        // (a block past the last reads nothing)
        const int k = (wave + i * NW) * 64;
        const uint32_t beyond = i >= mine || k + chunk * 8 >= p.K ? kOobOffset : 0u;
        const int soff = i < mine ? k * 2 : 0;
        char *dst = ring + slot * STAGE;
#pragma unroll
        for (int j = 0; j < 2 * NT; ++j) {
            if (gated && j >= NT) __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_u, FACT_LDS_PTR(dst + (2 * MT + j) * 1024), 16, vb[j] | beyond, soff, 0, 2);
            else __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_b, FACT_LDS_PTR(dst + (2 * MT + j) * 1024), 16, vb[j] | beyond, soff, 0, 2);
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
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            const int at = r16 * 128 + (((4 * kk + q) ^ (r16 & 7)) << 4);
            u32x4_t a[MT], b[NT];
#pragma unroll
            for (int t = 0; t < MT; ++t) a[t] = *(const u32x4_t *)(s + t * 2048 + at);
#pragma unroll
            for (int j = 0; j < NT; ++j) b[j] = *(const u32x4_t *)(s + (MT + j) * 2048 + at);
#pragma unroll
            for (int t = 0; t < MT; ++t)
#pragma unroll
                for (int j = 0; j < NT; ++j) acc[t][j] = mfma_skinny<F16>(b[j], a[t], acc[t][j]);
        }
        fill = slot;
        slot = slot + 1 == S ? 0 : slot + 1;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // loads past the last block still write LDS
    __syncthreads();

    // the waves' sums, added in ascending wave order (a fixed order: the result is bit-reproducible)
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int j = 0; j < NT; ++j) sums[((t * NT + j) * NW + wave) * 64 + lane] = acc[t][j];
    __syncthreads();
    const uint16_t *res = p.res ? (const uint16_t *)(p.res + z * p.stride_r) : nullptr;
    const uint16_t *bias = (const uint16_t *)p.bias;
    for (int o = wave; o < MT * OT; o += NW) {
        const int t = o / OT, j = o - t * OT;
        const int m = m0 + 16 * t + r16, n = n0 + 16 * j + 4 * q;         // the lane's four columns
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
        if (m >= p.M || n >= nout) continue;
        const bool full = n + 4 <= nout;
        if (full) {
            if (bias) {
                const u32x2_t w = *(const u32x2_any *)(bias + n);
                v[0] += in16<F16>(w.x & 0xFFFFu); v[1] += in16<F16>(w.x >> 16); v[2] += in16<F16>(w.y & 0xFFFFu); v[3] += in16<F16>(w.y >> 16);
            }
            if (p.act == ACT_GELU_TANH) {
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = gelu_tanh(v[e]);
            }
            if (res) {
                const u32x2_t w = *(const u32x2_any *)(res + (int64_t)m * p.ldr + n);
                v[0] += in16<F16>(w.x & 0xFFFFu); v[1] += in16<F16>(w.x >> 16); v[2] += in16<F16>(w.y & 0xFFFFu); v[3] += in16<F16>(w.y >> 16);
            }
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (n + e >= nout) continue;
                if (bias) v[e] += in16<F16>(bias[n + e]);
                if (p.act == ACT_GELU_TANH) v[e] = gelu_tanh(v[e]);
                if (res) v[e] += in16<F16>(res[(int64_t)m * p.ldr + n + e]);
            }
        }
        if (p.c_f32) {
            float *c = (float *)p.C + z * p.stride_c + (int64_t)m * p.ldc + n;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (n + e < nout) c[e] = v[e];
        } else {
            uint16_t *c = (uint16_t *)(p.C + z * p.stride_c) + (int64_t)m * p.ldc + n;
            if (full) {
                *(u32x2_any *)c = u32x2_t{out16<F16>(v[0]) | (out16<F16>(v[1]) << 16), out16<F16>(v[2]) | (out16<F16>(v[3]) << 16)};
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (n + e < nout) c[e] = (uint16_t)out16<F16>(v[e]);
            }
        }
    }
#else
    (void)p;
#endif
}

template <int MT, int NT, int NW, int S, bool F16>
static hipError_t launch_skinny_as(const GemmArgs &a, int grid_z, hipStream_t stream)
{
    const bool gated = a.act == ACT_SILU_GATE;
    const int nout = gated ? a.N / 2 : a.N, cols = 16 * (gated ? NT / 2 : NT);
    const dim3 grid((unsigned)((nout + (int64_t)cols - 1) / cols), (unsigned)((a.M + 16 * MT - 1) / (16 * MT)), (unsigned)grid_z);
    auto kern = skinny_kernel<MT, NT, NW, S, F16>;
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

template <int MT, int NT, int NW, int S>
static hipError_t launch_tile(const GemmArgs &a, int grid_z, hipStream_t stream)
{
    return a.f16 ? launch_skinny_as<MT, NT, NW, S, true>(a, grid_z, stream) : launch_skinny_as<MT, NT, NW, S, false>(a, grid_z, stream);
}

// One 16-column tile per work-group (two for gated calls, one of each half, and for many columns of 17-32 rows: half the
// reads of A); four waves and three or four stages, so that two or three work-groups share a compute unit.  Up to 64 rows
// eight waves and all of the LDS.
struct Tile { int mt, nt, waves, stages; };
static Tile tile_of(const GemmArgs &a)
{
    if (a.act == ACT_SILU_GATE) return a.M <= 16 ? Tile{1, 2, 4, 3} : Tile{2, 2, 4, 4};
    if (a.M <= 16) return {1, 1, 4, 4};
    if (a.M <= 32) return a.N > 6144 ? Tile{2, 2, 4, 4} : Tile{2, 1, 4, 3};
    return {4, 1, 8, 2};
}

// (a grid's threads are counted in 32 bits: 32 for each column here)
bool skinny_takes(const GemmArgs &a, bool trans_b) { return trans_b && a.M <= (a.act == ACT_SILU_GATE ? 32 : 64) && a.N < 1 << 27; }

// Estimated microseconds: a work-group's K steps one after the other, each at least a load's latency and at most 60 GB/s per
// compute unit, in as many rounds as the work-groups need; a start and an end per round, which nothing covers where
// only one work-group fits a compute unit; never faster than HBM delivers the weights, and A to each XCD.  Rows of weights that
// are no whole 128-byte lines cost more: each 128-byte piece lies on two lines (16 x 4096 x 14336 24.0 us, K = 14344 32.6).
double skinny_us(const GemmArgs &a, int64_t batch, bool whole_lines)
{
    const Tile t = tile_of(a);
    const bool gated = a.act == ACT_SILU_GATE;
    const int nout = gated ? a.N / 2 : a.N, cols = 16 * (gated ? t.nt / 2 : t.nt);
    const double wx = (double)((nout + (int64_t)cols - 1) / cols), wgs = wx * ((a.M + 16 * t.mt - 1) / (16 * t.mt)) * (double)batch;
    const int fit = 160 * 1024 / (t.waves * t.stages * (t.mt + t.nt) * 2048), blocks = (int)(((int64_t)a.K + 63) / 64);
    const double rounds = wgs > 256.0 * fit ? wgs / (256.0 * fit) : 1.0;
    const double sharing = wgs < 256.0 ? 1.0 : wgs / 256.0 < fit ? wgs / 256.0 : fit;
    const double rows_a = 0.5 * (16 * t.mt + (a.M < 16 * t.mt ? a.M : 16 * t.mt));       // (rows past M are not fetched, but their zeros are written)
    const double bytes = 128.0 * (blocks < t.waves ? blocks : t.waves) * (rows_a + 16 * t.nt), step = sharing * bytes / (whole_lines ? 60e3 : 50e3);
    const double chain = 1.4 + 0.004 * wgs + rounds * (0.8 + (blocks + t.waves - 1) / t.waves * (step > 0.2 ? step : 0.2)) + (fit == 1 ? 2.0 * (rounds - 1.0) : 0.0);
    const double memory = 1.4 + (double)batch * a.K * 2.0 * (a.N + (wx < 8.0 ? wx : 8.0) * a.M) / (whole_lines ? 5.4e6 : 4.7e6);
    return chain > memory ? chain : memory;
}

hipError_t launch_skinny_gemm(const GemmArgs &a, int grid_z, hipStream_t stream)
{
    const Tile t = tile_of(a);
    if (t.mt == 4) return launch_tile<4, 1, 8, 2>(a, grid_z, stream);
    if (t.mt == 2) return t.nt == 2 ? launch_tile<2, 2, 4, 4>(a, grid_z, stream) : launch_tile<2, 1, 4, 3>(a, grid_z, stream);
    return t.nt == 2 ? launch_tile<1, 2, 4, 3>(a, grid_z, stream) : launch_tile<1, 1, 4, 4>(a, grid_z, stream);
}

}  // namespace fact
