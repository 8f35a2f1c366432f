// Split-K reduction pass with the fused epilogue, and the guarded fallback GEMM for
// shapes neither the main kernel nor the ragged one takes.
#include "launch.h"

namespace fact {

// 16-bit pattern <-> fp32 in the launch's format (these kernels are bound by memory traffic: a run-time choice)
__device__ __forceinline__ float in16_rt(int f16, uint32_t bits) { return f16 ? f16_bits_to_f32(bits) : bf16_bits_to_f32(bits); }
__device__ __forceinline__ uint32_t out16_rt(int f16, float x) { return f16 ? f32_to_f16_bits(x) : f32_to_bf16_bits(x); }
__device__ __forceinline__ uint32_t pack2_rt(int f16, float a, float b) { return f16 ? pack2<true>(pk_f32_t{a, b}) : pack2<false>(pk_f32_t{a, b}); }

// ---- split-K reduction -----------------------------------------------------------------
// P holds `splits` fp32 partial products [M][N].  A lane owns 4 consecutive output columns of
// one row; the W waves of a work-group own the same 64 such column groups and a W-th of the K
// ranges each (consecutive ranges, added in ascending order); the W sums are then added in
// ascending order by the first wave, which applies the epilogue and rounds once.  W depends on
// the problem's M, N and number of ranges only (reduce_waves below), so the order of additions is
// fixed for a given problem and the result is bit-reproducible.  Many ranges of a small output want W = 8 (one wave
// per column group adding all ranges in turn was bound by its trips to memory: 8.5 us for the
// 17 MB of 64 ranges of a 256 x 256 output, whatever the number of loads in flight per wave);
// few ranges of a large output want W = 1 (with W = 8 six of the eight waves idled and every
// 64 column groups paid two barriers: 61 us for 2 ranges of a 256 x 8192 output).  The paper's
// counterpart is the fix-up step of its Stream-K schedule (Section 5.2.3).
template <int kReduceWaves>
__global__ void __launch_bounds__(64 * kReduceWaves) splitk_reduce_kernel(const GemmArgs p)
{
    __shared__ float part[kReduceWaves > 1 ? kReduceWaves - 1 : 1][2][4][64];        // sums of waves 1..: [wave-1][gate|up][column][lane]
    const bool gated = p.act == ACT_SILU_GATE;
    const int nout = gated ? (p.N >> 1) : p.N;
    const int groups = (nout + 3) >> 2;
    const int64_t total = (int64_t)p.M * groups;
    const int64_t plane = (int64_t)p.M * p.N;
    const bool vec_p = (p.N & 3) == 0 && (!gated || (nout & 3) == 0);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int per = (p.splits + kReduceWaves - 1) / kReduceWaves;      // K ranges per wave
    const int s_begin = wave * per < p.splits ? wave * per : p.splits;
    const int s_end = s_begin + per < p.splits ? s_begin + per : p.splits;
    for (int64_t t0 = (int64_t)blockIdx.x * 64; t0 < total; t0 += (int64_t)gridDim.x * 64) {
        const int64_t t = t0 + lane;
        const bool live = t < total;
        int m = 0, n = 0;
        if (live) {
            if (total <= 0x7FFFFFFF) { m = (int)((uint32_t)t / (uint32_t)groups); n = (int)((uint32_t)t - (uint32_t)m * (uint32_t)groups) * 4; }
            else { m = (int)(t / groups); n = (int)(t % groups) * 4; }
        }
        float v[4] = {0.f, 0.f, 0.f, 0.f}, u[4] = {0.f, 0.f, 0.f, 0.f};
        const float *src = p.P + (int64_t)m * p.N + n + (int64_t)s_begin * plane;
        const bool full = n + 3 < nout, vec_e = full && p.vec_store;
        const int cnt = live ? s_end - s_begin : 0;
        // the first wave's bias and residual travel with the partials
        u32x2_t bias4 = {0u, 0u}, res4 = {0u, 0u};
        if (wave == 0 && live && vec_e) {
            if (p.bias) bias4 = *(const u32x2_t *)((const uint16_t *)p.bias + n);
            if (p.res) res4 = *(const u32x2_t *)((const uint16_t *)p.res + (int64_t)m * p.ldr + n);
        }
        if (full && vec_p) {
            // Batches of 8, 4, 2 and 1 ranges, in each every load issued before the first add: a wave is bound by its trips to
            // memory, and with a trip per range past the last 8, and one each for bias and residual after the sums, 4 ranges of
            // 208 x 4096 took 11.4 us, like this 7.7 (GEMM and reduction: 192 x 64 x 10112 11.1 -> 9.7, 384 x 256 x 69120 38.9 -> 36.4).
            int s0 = 0;
            auto batch = [&](auto nb_) __attribute__((always_inline)) {
                constexpr int NB = decltype(nb_)::value;
                f32x4_t a[NB], b[NB];
#pragma unroll
                for (int j = 0; j < NB; ++j) a[j] = *(const f32x4_t *)(src + (s0 + j) * plane);
                if (gated) {
#pragma unroll
                    for (int j = 0; j < NB; ++j) b[j] = *(const f32x4_t *)(src + (s0 + j) * plane + nout);
                }
#pragma unroll
                for (int j = 0; j < NB; ++j) { v[0] += a[j].x; v[1] += a[j].y; v[2] += a[j].z; v[3] += a[j].w; }
                if (gated) {
#pragma unroll
                    for (int j = 0; j < NB; ++j) { u[0] += b[j].x; u[1] += b[j].y; u[2] += b[j].z; u[3] += b[j].w; }
                }
                s0 += NB;
            };
            while (s0 + 8 <= cnt) batch(std::integral_constant<int, 8>{});
            if (s0 + 4 <= cnt) batch(std::integral_constant<int, 4>{});
            if (s0 + 2 <= cnt) batch(std::integral_constant<int, 2>{});
            if (s0 < cnt) batch(std::integral_constant<int, 1>{});
        } else {
            for (int s0 = 0; s0 < cnt; ++s0)
                for (int e = 0; e < 4; ++e)
                    if (n + e < nout) {
                        v[e] += src[s0 * plane + e];
                        if (gated) u[e] += src[s0 * plane + nout + e];
                    }
        }
        if (kReduceWaves > 1) {
            if (wave > 0) {
#pragma unroll
                for (int e = 0; e < 4; ++e) { part[wave - 1][0][e][lane] = v[e]; part[wave - 1][1][e][lane] = u[e]; }
            }
            __syncthreads();
        }
        if (wave == 0 && live) {
#pragma unroll
            for (int w = 0; w < kReduceWaves - 1; ++w)
#pragma unroll
                for (int e = 0; e < 4; ++e) { v[e] += part[w][0][e][lane]; u[e] += part[w][1][e][lane]; }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (n + e >= nout) continue;
                float zv = v[e];
                if (gated) zv = silu(zv) * u[e];
                if (p.bias) zv += in16_rt(p.f16, vec_e ? (bias4[e / 2] >> (16 * (e & 1))) & 0xFFFFu : ((const uint16_t *)p.bias)[n + e]);
                if (p.act == ACT_GELU_TANH) zv = gelu_tanh(zv);
                if (p.res) zv += in16_rt(p.f16, vec_e ? (res4[e / 2] >> (16 * (e & 1))) & 0xFFFFu : ((const uint16_t *)p.res)[(int64_t)m * p.ldr + n + e]);
                v[e] = zv;
            }
            if (p.out_f32) {                                   // fp32 output: no rounding at all
                float *cf = (float *)p.C + (int64_t)m * p.ldc + n;
                if (vec_e) {
                    *(f32x4_t *)cf = f32x4_t{v[0], v[1], v[2], v[3]};
                } else {
                    for (int e = 0; e < 4; ++e)
                        if (n + e < nout) cf[e] = v[e];
                }
            } else {
                __bf16 *cp = p.C + (int64_t)m * p.ldc + n;
                if (vec_e) {
                    *(u32x2_t *)cp = u32x2_t{pack2_rt(p.f16, v[0], v[1]), pack2_rt(p.f16, v[2], v[3])};
                } else {
                    uint16_t *cs = (uint16_t *)cp;
                    for (int e = 0; e < 4; ++e)
                        if (n + e < nout) cs[e] = (uint16_t)out16_rt(p.f16, v[e]);
                }
            }
        }
        if (kReduceWaves > 1) __syncthreads();                 // the waves' sums are read before the next round overwrites them
    }
}

// Waves that share a column group's K ranges: as many (1, 2, 4 or 8) as it takes to have some 2048 waves
// at work, each with at least four ranges.  A function of the problem alone (M, N, split factor).
static int reduce_waves(int splits, int64_t blocks)
{
    int w = 1;
    while (w < 8 && blocks * w < 2048 && splits >= 8 * w) w *= 2;
    return w;
}

hipError_t launch_splitk_reduce(const GemmArgs &args, hipStream_t stream)
{
    const int nout = args.act == ACT_SILU_GATE ? args.N / 2 : args.N;
    const int64_t total = (int64_t)args.M * ((nout + 3) / 4);
    // 64 column groups per work-group: even a 256 x 256 output spreads over all CUs
    int64_t blocks = (total + 63) / 64;
    if (blocks > 256 * 256) blocks = 256 * 256;
    switch (reduce_waves(args.splits, (total + 63) / 64)) {
    case 8: hipLaunchKernelGGL(splitk_reduce_kernel<8>, dim3((unsigned)blocks), dim3(512), 0, stream, args); break;
    case 4: hipLaunchKernelGGL(splitk_reduce_kernel<4>, dim3((unsigned)blocks), dim3(256), 0, stream, args); break;
    case 2: hipLaunchKernelGGL(splitk_reduce_kernel<2>, dim3((unsigned)blocks), dim3(128), 0, stream, args); break;
    default: hipLaunchKernelGGL(splitk_reduce_kernel<1>, dim3((unsigned)blocks), dim3(64), 0, stream, args); break;
    }
    return hipGetLastError();
}

// ---- guarded fallback ---------------------------------------------------------------------
// One thread per output element, ascending-k fp32 FMA.  No alignment or divisibility
// requirement; every access is bounds-guarded.  Slow by design: it serves rows shorter than
// one 16-byte piece (the ragged kernel takes the rest) and is the reference result of the on-device sweep.
template <bool TRANS_B>
__global__ void __launch_bounds__(256) fallback_gemm_kernel(const GemmArgs p)
{
    const bool gated = p.act == ACT_SILU_GATE;
    const int nout = gated ? (p.N >> 1) : p.N;
    const uint32_t tiles_n = ((uint32_t)nout + 15u) >> 4;
    int64_t row = blockIdx.x / tiles_n, column = blockIdx.x % tiles_n;
    if (gridDim.y > 1) {                                     // large outputs: further rows of the grid
        const int64_t block = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
        row = block / tiles_n; column = block % tiles_n;
    }
    if (row * 16 + (threadIdx.x >> 4) >= p.M || column * 16 + (threadIdx.x & 15) >= nout) return;
    const int n = (int)column * 16 + (threadIdx.x & 15), m = (int)row * 16 + (threadIdx.x >> 4);
    const int z = blockIdx.z;
    const uint16_t *A = (const uint16_t *)(p.A + z * p.stride_a) + (int64_t)m * p.lda;
    const uint16_t *B = (const uint16_t *)(p.B + z * p.stride_b);
    float acc = 0.f, acc_up = 0.f;
    if (TRANS_B) {
        const uint16_t *w = B + (int64_t)n * p.ldb;
        const uint16_t *wu = gated ? (const uint16_t *)(p.B_up + z * p.stride_b) + (int64_t)n * p.ldb : nullptr;
        for (int k = 0; k < p.K; ++k) {
            const float a = in16_rt(p.f16, A[k]);
            acc = __builtin_fmaf(a, in16_rt(p.f16, w[k]), acc);
            if (gated) acc_up = __builtin_fmaf(a, in16_rt(p.f16, wu[k]), acc_up);
        }
    } else {
        for (int k = 0; k < p.K; ++k)
            acc = __builtin_fmaf(in16_rt(p.f16, A[k]), in16_rt(p.f16, B[(int64_t)k * p.ldb + n]), acc);
    }
    float zv = acc;
    if (gated) zv = silu(zv) * acc_up;
    if (p.bias) zv += in16_rt(p.f16, ((const uint16_t *)p.bias)[n]);
    if (p.act == ACT_GELU_TANH) zv = gelu_tanh(zv);
    if (p.res) zv += in16_rt(p.f16, ((const uint16_t *)(p.res + z * p.stride_r))[(int64_t)m * p.ldr + n]);
    ((uint16_t *)(p.C + z * p.stride_c))[(int64_t)m * p.ldc + n] = (uint16_t)out16_rt(p.f16, zv);
}

hipError_t launch_fallback_gemm(const GemmArgs &args, bool trans_b, int grid_z, hipStream_t stream)
{
    const int nout = args.act == ACT_SILU_GATE ? args.N / 2 : args.N;
    const int64_t blocks = ((int64_t)nout + 15) / 16 * (((int64_t)args.M + 15) / 16);
    const int64_t gx = blocks > 1 << 20 ? 1 << 20 : blocks, gy = (blocks + gx - 1) / gx;       // (a grid's threads are counted in 32 bits)
    if (gy > 65535) return hipErrorInvalidConfiguration;
    dim3 grid((unsigned)gx, (unsigned)gy, (unsigned)grid_z);
    if (trans_b)
        hipLaunchKernelGGL(fallback_gemm_kernel<true>, grid, dim3(256), 0, stream, args);
    else
        hipLaunchKernelGGL(fallback_gemm_kernel<false>, grid, dim3(256), 0, stream, args);
    return hipGetLastError();
}

}  // namespace fact
