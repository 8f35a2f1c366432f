// The pieces of a transformer block around attention and the feed-forward network - LayerNorm /
// RMSNorm and the rotary embedding, two small memory-bound kernels - and the composition of the
// whole block from this library's entry points.  The paper composes its patterns into one module
// that keeps the sub-graph's interface (Section 4.3) and evaluates two blocks (Section 5.1: a
// GPT-style block with LayerNorm and GELU, a Llama-3-8B decoder block with RMSNorm, grouped-query
// attention and SwiGLU); fact_block_forward is that composition with every stage on the GPU.
#include "../../include/fact.h"

#include "launch.h"
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <cmath>

namespace fact {

int record_hip_failure(hipError_t e, const char *what);      // fact_api.hip

namespace blockk {

typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float lo16(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float hi16(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
// two values rounded to nearest even, low half first: one instruction.  Rounding in integer arithmetic took about ten for a pair, a third of all
// that a norm issues, and that work is not hidden: every wave of a launch loads, then sums, then rounds at about the same time (us, before ->
// now, operands from the memory-side cache: norms of 8192 x 768 7.9 -> 6.7, 2048 x 4096 8.0 -> 7.2, 16 x 4096 2.56 -> 2.37, 65536 x 64
// 17.4 -> 13.0; rotary embedding of 2048 tokens of 40 heads of 128 9.0 -> 7.5, 16 tokens 3.5 -> 3.1; above 100 MB, bound by HBM,
// within 2 %: norms of 65536 x 2040 100.3 -> 98.6, 262144 x 1152 204 -> 209).
__device__ __forceinline__ uint32_t pack2(float a, float b) { return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_t{a, b}, bf16x2_t)); }
// sum over the wave, the same in every lane: rotations inside each 16-lane row, then exchanges of rows and halves, all on
// the vector ALU (through LDS permutes the six dependent steps of a sum took 0.35 us)
template <int CTRL>
__device__ __forceinline__ float add_rotated(float v)
{
    return v + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, false));
}
__device__ __forceinline__ float wave_sum(float v)
{
    v = add_rotated<0x128>(v);       // row_ror:8
    v = add_rotated<0x124>(v);
    v = add_rotated<0x122>(v);
    v = add_rotated<0x121>(v);
    const uint32_t u = __builtin_bit_cast(uint32_t, v);
    const auto s = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    v = __builtin_bit_cast(float, (uint32_t)s[0]) + __builtin_bit_cast(float, (uint32_t)s[1]);
    const uint32_t w = __builtin_bit_cast(uint32_t, v);
    const auto h = __builtin_amdgcn_permlane32_swap(w, w, false, false);
    return __builtin_bit_cast(float, (uint32_t)h[0]) + __builtin_bit_cast(float, (uint32_t)h[1]);
}

// A row is read once (16 bytes per lane and piece), kept in registers in fp32, reduced, normalised and written once;
// d <= 8192, a multiple of 8.  Bound by memory traffic where there are many rows and by one row's chain of latencies
// where there are few, so gamma and beta are asked for before the sums need them, and a wide row is shared by the four
// waves of a work-group (their sums meet in LDS; the launch says which rows).  Operands
// from HBM: 2048 x 4096 7.6 us (4.4 TB/s; 12.4 with a wave per row that asked for gamma and beta after its sums), 32768 x 4096 89 us
// (6.0 TB/s; 113), 8192 x 768 7.8 us (9.9).
// Narrower rows take a wave each, in pieces of 8 columns a lane also where half of the last one is idle (768 = 1.5 pieces): with pieces of 4
// columns 8192 x 768 took 8.2 us, 65536 x 768 39.6 (35.8), 16384 x 1280 18.7 (16.9): more, smaller requests cost what the idle lanes did.
// The number of 512-element pieces per wave is a template parameter.
constexpr int kMaxWidth = 8192;
template <bool RMS, int WPR, int PIECES>
__global__ void __launch_bounds__(256)
norm_kernel(const uint16_t *X, int64_t ldx, const uint16_t *gamma, const uint16_t *beta, float eps,
            uint16_t *Y, int64_t ldy, int T, int d)
{
    __shared__ float part[2][4];
    const int wave = threadIdx.x >> 6;
    const int64_t wg = (int64_t)blockIdx.y * gridDim.x + blockIdx.x, row = WPR == 1 ? wg * 4 + wave : wg;
    if (row >= T) return;                                    // (the whole work-group where it shares a row)
    const int c0 = (WPR == 1 ? (int)threadIdx.x & 63 : (int)threadIdx.x) * 8;        // the lane's first column; pieces are WPR * 512 apart
    auto over_row = [&](float v, int which) __attribute__((always_inline)) {
        v = wave_sum(v);
        if constexpr (WPR > 1) {
            if ((threadIdx.x & 63) == 0) part[which][wave] = v;
            __syncthreads();
            v = (part[which][0] + part[which][1]) + (part[which][2] + part[which][3]);
        }
        return v;
    };
    const uint16_t *x = X + row * ldx;
    u32x4_t w[PIECES], g[PIECES], b[PIECES];
#pragma unroll
    for (int p = 0; p < PIECES; ++p) {
        const int c = p * WPR * 512 + c0;
        w[p] = c < d ? *(const u32x4_t *)(x + c) : u32x4_t{0u, 0u, 0u, 0u};
    }
#pragma unroll
    for (int p = 0; p < PIECES; ++p) {
        const int c = p * WPR * 512 + c0;
        g[p] = c < d ? *(const u32x4_t *)(gamma + c) : u32x4_t{0u, 0u, 0u, 0u};
        b[p] = !RMS && beta && c < d ? *(const u32x4_t *)(beta + c) : u32x4_t{0u, 0u, 0u, 0u};
    }
    float v[PIECES][8], s = 0.f, q = 0.f, mean = 0.f;
#pragma unroll
    for (int p = 0; p < PIECES; ++p)
#pragma unroll
        for (int e = 0; e < 4; ++e) { v[p][2 * e] = lo16(w[p][e]); v[p][2 * e + 1] = hi16(w[p][e]); }
    if constexpr (!RMS) {
#pragma unroll
        for (int p = 0; p < PIECES; ++p)
#pragma unroll
            for (int e = 0; e < 8; ++e) s += v[p][e];
        mean = over_row(s, 0) / (float)d;
    }
#pragma unroll
    for (int p = 0; p < PIECES; ++p)
        if (p * WPR * 512 + c0 < d) {
#pragma unroll
            for (int e = 0; e < 8; ++e) { const float t = v[p][e] - mean; q += t * t; }
        }
    const float rstd = 1.0f / sqrtf(over_row(q, 1) / (float)d + eps);
    uint16_t *y = Y + row * ldy;
#pragma unroll
    for (int p = 0; p < PIECES; ++p) {
        const int c = p * WPR * 512 + c0;
        if (c < d) {
            u32x4_t o;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                o[e] = pack2((v[p][2 * e] - mean) * rstd * lo16(g[p][e]) + lo16(b[p][e]),
                             (v[p][2 * e + 1] - mean) * rstd * hi16(g[p][e]) + hi16(b[p][e]));
            *(u32x4_t *)(y + c) = o;
        }
    }
}

// Rotary embedding in place, "rotate-half" pairing.  A work-group takes a few tokens and up to 256 of their angles
// (blockIdx.y: further angles of a wider head); each thread computes one sine and cosine, once per token, into
// LDS - the precise functions cost more than the traffic - and then walks 16-byte pieces of its heads: the piece at i
// and the one at i + D/2.  Many heads of few tokens are shared by several work-groups (4096 heads of 128, one token: 100 -> 3.7 us).
// 2048 tokens of 40 heads of 128, from HBM: 8.6 us (4.9 TB/s), 16 tokens 3.1 us (15.1 and 6.3 with a thread that computed eight angles and
// walked eight heads).
template <bool GROUPS>
__global__ void __launch_bounds__(256)
rope_kernel(uint16_t *X, int64_t sb, int64_t st, int64_t sh, int64_t tokens, int T, int H, int D, int per_wg, int per_group, float log2_base)
{
    __shared__ float2 turn[256];
    const int first = blockIdx.y * 256;                      // first angle of this work-group
    // blockIdx.z: the group of heads, or (all heads in one work-group) further rows of the grid
    const int h0 = GROUPS ? (int)blockIdx.z * per_group : 0, heads = GROUPS && H - h0 > per_group ? per_group : H - h0;
    const int angles = D / 2 - first < 256 ? D / 2 - first : 256, pieces = angles >> 3;
    const int64_t bt0 = (GROUPS ? (int64_t)blockIdx.x : (int64_t)blockIdx.z * gridDim.x + blockIdx.x) * per_wg;
    if (bt0 >= tokens || (GROUPS && heads <= 0)) return;     // (the whole work-group)
    const int mine = tokens - bt0 < per_wg ? (int)(tokens - bt0) : per_wg;
    {
        const int k = threadIdx.x / angles, i = threadIdx.x - k * angles;        // token of the work-group, angle
        if (k < mine) {
            const float inv_freq = exp2f(-2.0f * (float)(first + i) / (float)D * log2_base);
            float sn, cs;
            sincosf((float)(int)((bt0 + k) % T) * inv_freq, &sn, &cs);
            turn[threadIdx.x] = make_float2(cs, sn);
        }
    }
    __syncthreads();
    const int per_token = heads * pieces;
    for (int j = threadIdx.x; j < mine * per_token; j += 256) {
        const int k = j / per_token, r = j - k * per_token, h = r / pieces, piece = r - h * pieces;
        const int64_t bt = bt0 + k;
        uint16_t *p = X + bt / T * sb + bt % T * st + (int64_t)(h0 + h) * sh + first + piece * 8;
        const float2 *cs = turn + k * angles + piece * 8;
        const u32x4_t lo = *(const u32x4_t *)p, hi = *(const u32x4_t *)(p + D / 2);
        u32x4_t olo, ohi;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float2 t0 = cs[2 * e], t1 = cs[2 * e + 1];
            const float a0 = lo16(lo[e]), a1 = hi16(lo[e]), c0 = lo16(hi[e]), c1 = hi16(hi[e]);
            olo[e] = pack2(a0 * t0.x - c0 * t0.y, a1 * t1.x - c1 * t1.y);
            ohi[e] = pack2(c0 * t0.x + a0 * t0.y, c1 * t1.x + a1 * t1.y);
        }
        *(u32x4_t *)p = olo;
        *(u32x4_t *)(p + D / 2) = ohi;
    }
}

// The same for few heads: a thread takes 8 angles of one token - the 16-byte piece at i and the one at i + D/2 - and walks the
// heads, so nothing passes through LDS and no thread idles while others read (us, the kernel above -> this one; tokens x heads x
// D): 65536 x 1 x 128 21.8 -> 12.2, 65536 x 2 x 128 22.5 -> 15.8, 65536 x 4 x 128 28.0 -> 22.9, 16384 x 1 x 1024 39 -> 20.
__global__ void __launch_bounds__(256)
rope_few_heads_kernel(uint16_t *X, int64_t sb, int64_t st, int64_t sh, int64_t tokens, int T, int H, int D, float log2_base)
{
    const int per_token = D / 16;
    const int64_t id = ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * 256 + threadIdx.x, bt = id / per_token;
    if (bt >= tokens) return;
    const int i0 = (int)(id - bt * per_token) * 8, t = (int)(bt % T);
    float sn[8], cs[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const float inv_freq = exp2f(-2.0f * (float)(i0 + e) / (float)D * log2_base);
        sincosf((float)t * inv_freq, &sn[e], &cs[e]);
    }
    uint16_t *p = X + bt / T * sb + t * st + i0;
    for (int h = 0; h < H; ++h, p += sh) {
        const u32x4_t lo = *(const u32x4_t *)p, hi = *(const u32x4_t *)(p + D / 2);
        u32x4_t olo, ohi;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float a0 = lo16(lo[e]), a1 = hi16(lo[e]), c0 = lo16(hi[e]), c1 = hi16(hi[e]);
            olo[e] = pack2(a0 * cs[2 * e] - c0 * sn[2 * e], a1 * cs[2 * e + 1] - c1 * sn[2 * e + 1]);
            ohi[e] = pack2(c0 * cs[2 * e] + a0 * sn[2 * e], c1 * cs[2 * e + 1] + a1 * sn[2 * e + 1]);
        }
        *(u32x4_t *)p = olo;
        *(u32x4_t *)(p + D / 2) = ohi;
    }
}

static bool aligned16(const void *p) { return ((uintptr_t)p & 15u) == 0; }
static size_t up256(size_t v) { return (v + 255) & ~(size_t)255; }

struct Layout {
    size_t n1, qkv, a, x1, n2, h, ws, ws_bytes, least, total;
};

static int plan(const fact_block *b, Layout &L)
{
    if (!b) return FACT_ERR_NULL;
    if (b->batch <= 0 || b->tokens <= 0 || b->d_model <= 0 || b->n_q_heads <= 0 || b->n_kv_heads <= 0 || b->d_ff <= 0) return FACT_ERR_DIM;
    if (b->n_q_heads % b->n_kv_heads) return FACT_ERR_DIM;
    if (b->head_dim != 64 && b->head_dim != 128) return FACT_ERR_UNSUPPORTED;
    if (b->d_model % 8 || b->d_model > 8192 || b->d_ff % 8) return FACT_ERR_UNSUPPORTED;
    if (b->act != FACT_ACT_GELU_TANH && b->act != FACT_ACT_SILU_GATE && b->act != FACT_ACT_NONE) return FACT_ERR_EPILOGUE;
    if (!b->norm1_g || !b->norm2_g || !b->Wqkv || !b->Wo || !b->W1 || !b->W2) return FACT_ERR_NULL;
    if (b->act == FACT_ACT_SILU_GATE && (!b->W1u || b->b1)) return FACT_ERR_EPILOGUE;
    if (b->act != FACT_ACT_SILU_GATE && b->W1u) return FACT_ERR_EPILOGUE;
    const int64_t T = b->batch * b->tokens, d = b->d_model, nq = b->n_q_heads * b->head_dim;
    const int64_t nqkv = (b->n_q_heads + 2 * b->n_kv_heads) * b->head_dim;
    // what the later stages would refuse is refused here, before anything is launched: the attention
    // kernel's 32-bit row offsets inside a batch entry of the packed projection and its grid limit,
    // the norm kernels' 16-byte access to their parameters
    if ((b->tokens + 512) * nqkv * 2 >= (int64_t)1 << 31 || b->tokens > 0x7FFFFFFF - 1024) return FACT_ERR_UNSUPPORTED;
    if (b->batch * b->n_q_heads * ((b->tokens + 127) / 128) > 0x7FFFFFFF || T > 0x7FFFFFFF) return FACT_ERR_UNSUPPORTED;
    if (!aligned16(b->norm1_g) || !aligned16(b->norm2_g) || (!b->norm_rms && ((b->norm1_b && !aligned16(b->norm1_b)) || (b->norm2_b && !aligned16(b->norm2_b)))))
        return FACT_ERR_ALIGN;
    if (b->norm_rms != 0 && b->norm_rms != 1) return FACT_ERR_LAYOUT;
    size_t off = 0;
    L.n1 = off; off += up256((size_t)T * d * 2);
    L.qkv = off; off += up256((size_t)T * nqkv * 2);
    L.a = off; off += up256((size_t)T * nq * 2);
    L.x1 = off; off += up256((size_t)T * d * 2);
    L.n2 = off; off += up256((size_t)T * d * 2);
    L.h = off; off += up256((size_t)T * b->d_ff * 2);
    const Workspace parts[3] = {splitk_workspace(T, nqkv, d), splitk_workspace(T, d, nq), mlp_workspace(T, d, b->d_ff, b->act)};
    size_t least = 0, full = 0;
    for (const Workspace &w : parts) {
        if (w.least > least) least = w.least;
        if (w.full > full) full = w.full;
    }
    L.ws = off; L.ws_bytes = full;
    L.least = off + up256(least);       // (a scratch buffer of that size serves as well)
    L.total = off + up256(full);
    return FACT_OK;
}

}  // namespace blockk
}  // namespace fact

extern "C" {

int fact_norm(int64_t T, int64_t d, const void *X, int64_t ldx, const void *gamma, const void *beta, float eps, int rms,
              void *Y, int64_t ldy, void *stream)
{
    using namespace fact::blockk;
    if (!X || !gamma || !Y) return FACT_ERR_NULL;
    if (T <= 0 || d <= 0 || ldx < d || ldy < d || T > 0x7FFFFFFF) return FACT_ERR_DIM;
    if (rms != 0 && rms != 1) return FACT_ERR_LAYOUT;
    if (rms && beta) return FACT_ERR_EPILOGUE;
    if (d % 8 || d > kMaxWidth) return FACT_ERR_UNSUPPORTED;
    if (!aligned16(X) || !aligned16(Y) || !aligned16(gamma) || (beta && !aligned16(beta)) || (ldx & 7) || (ldy & 7)) return FACT_ERR_ALIGN;
    if (!(eps >= 0.f)) return FACT_ERR_DIM;
    // Four waves per row from 2048 elements on, and from 1032 on where there are few rows; with many a wave takes up to 2040 elements
    // by itself, since four waves leave lanes idle (us, four waves -> one; LayerNorm: 262144 x 1152 340 -> 210, 16384 x 1536
    // 23.8 -> 21.1, 4096 x 1032 8.7 -> 7.1, 4096 x 1792 9.4 -> 9.3, 65536 x 2040 100 -> 101; RMSNorm: 65536 x 2048 86 -> 91;
    // 1024 x 1544 3.9 -> 4.3, 16 x 1544 2.2 -> 3.1).
    const bool wide = d > 1024 && (d >= 2048 || T < 2048);
    // (at most 2^20 work-groups along x: a grid's threads are counted in 32 bits)
    const int64_t wgs = wide ? T : (T + 3) / 4, gx = wgs > 1 << 20 ? 1 << 20 : wgs;
    const dim3 grid((unsigned)gx, (unsigned)((wgs + gx - 1) / gx));
    hipStream_t s = (hipStream_t)stream;
    const int pieces = (int)((d + (wide ? 2047 : 511)) / (wide ? 2048 : 512));
#define FACT_NORM_LAUNCH(R, W, P) hipLaunchKernelGGL((norm_kernel<R, W, P>), grid, dim3(256), 0, s, (const uint16_t *)X, ldx, \
        (const uint16_t *)gamma, (const uint16_t *)(R ? nullptr : beta), eps, (uint16_t *)Y, ldy, (int)T, (int)d)
#define FACT_NORM_PICK(R) do { if (!wide && pieces == 1) FACT_NORM_LAUNCH(R, 1, 1); else if (!wide && pieces == 2) FACT_NORM_LAUNCH(R, 1, 2); \
        else if (!wide && pieces == 3) FACT_NORM_LAUNCH(R, 1, 3); else if (!wide) FACT_NORM_LAUNCH(R, 1, 4); \
        else if (pieces == 1) FACT_NORM_LAUNCH(R, 4, 1); else if (pieces == 2) FACT_NORM_LAUNCH(R, 4, 2); else FACT_NORM_LAUNCH(R, 4, 4); } while (0)
    if (rms) FACT_NORM_PICK(true); else FACT_NORM_PICK(false);
#undef FACT_NORM_PICK
#undef FACT_NORM_LAUNCH
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? FACT_OK : fact::record_hip_failure(e, "norm launch");
}

int fact_rope(int64_t batch, int64_t T, int64_t n_heads, int64_t head_dim, void *X, const int64_t *strides, float base, void *stream)
{
    using namespace fact::blockk;
    if (!X || !strides) return FACT_ERR_NULL;
    if (batch <= 0 || T <= 0 || n_heads <= 0 || strides[1] < head_dim || strides[0] < 0 || strides[2] < 0) return FACT_ERR_DIM;
    if (head_dim <= 0 || head_dim % 16) return FACT_ERR_UNSUPPORTED;
    if (!aligned16(X) || (strides[0] & 7) || (strides[1] & 7) || (strides[2] & 7)) return FACT_ERR_ALIGN;
    if (!(base > 1.0f)) return FACT_ERR_DIM;
    const int64_t tokens = batch * T;
    if (batch > 0x7FFFFFFF || T > 0x7FFFFFFF || n_heads > 524280 || (tokens * (head_dim / 16) + 255) / 256 > 0x7FFFFFFF) return FACT_ERR_UNSUPPORTED;
    const int64_t chunks = (head_dim / 2 + 255) / 256;
    if (head_dim > 0x7FFFFFFF || chunks > 65535) return FACT_ERR_UNSUPPORTED;
    // Few heads: with up to four, from 50000 pieces of 8 angles per head on the kernel without LDS is the faster one (us, rope_kernel / it;
    // tokens x heads x D: 4000 x 2 x 512 7.6 / 6.4, 16384 x 4 x 256 17.6 / 16.0, 65536 x 2 x 64 13.4 / 10.5; 16384 x 2 x 64 4.9 / 5.0,
    // 16384 x 4 x 64 6.5 / 7.0, 65536 x 8 x 64 22.8 / 23.4), with one also for a few thousand tokens (4000 x 1 x 64 4.4 / 3.5, 1000 x 1 x 64 3.0 / 3.5).
    const int64_t threads = tokens * (head_dim / 16);
    if (n_heads <= 4 && (threads >= 50000 * n_heads || (n_heads == 1 && tokens >= 2048 && tokens < 8192))) {
        const int64_t wgs = (threads + 255) / 256, gx = wgs > 1 << 20 ? 1 << 20 : wgs;          // (a grid's threads are counted in 32 bits)
        hipLaunchKernelGGL(rope_few_heads_kernel, dim3((unsigned)gx, (unsigned)((wgs + gx - 1) / gx)), dim3(256), 0, (hipStream_t)stream, (uint16_t *)X,
                           strides[0], strides[1], strides[2], tokens, (int)T, (int)n_heads, (int)head_dim, std::log2(base));
        const hipError_t e = hipGetLastError();
        return e == hipSuccess ? FACT_OK : fact::record_hip_failure(e, "rope launch");
    }
    // as many tokens per work-group as have their angles fit its 256 threads, fewer where that leaves less than 1024 work-groups
    // (16384 tokens of a head of 16: 9.3 -> 4.0 us with 8 in place of 2), one where there are few tokens
    const int fit = head_dim >= 512 ? 1 : (int)(512 / head_dim);
    int per_wg = tokens >= 512 && fit > 1 ? 2 : 1;
    while (2 * per_wg <= fit && tokens >= 4096 * (int64_t)per_wg) per_wg *= 2;
    if (tokens >= 1024 * (int64_t)fit) per_wg = fit;
    const int64_t wgs = (tokens + per_wg - 1) / per_wg, gx = wgs > 1 << 20 ? 1 << 20 : wgs;
    if ((wgs + gx - 1) / gx > 65535) return FACT_ERR_UNSUPPORTED;
    // heads are shared where they give every thread more than two pieces and the chip has room
    const int64_t pieces = (head_dim < 512 ? head_dim : 512) / 16;
    int64_t groups = n_heads * pieces * per_wg / 512;
    if (groups > 1024 / (wgs * chunks)) groups = 1024 / (wgs * chunks);
    if (groups > 1)
        hipLaunchKernelGGL(rope_kernel<true>, dim3((unsigned)wgs, (unsigned)chunks, (unsigned)groups), dim3(256), 0, (hipStream_t)stream, (uint16_t *)X,
                           strides[0], strides[1], strides[2], tokens, (int)T, (int)n_heads, (int)head_dim, per_wg, (int)((n_heads + groups - 1) / groups), std::log2(base));
    else
        hipLaunchKernelGGL(rope_kernel<false>, dim3((unsigned)gx, (unsigned)chunks, (unsigned)((wgs + gx - 1) / gx)), dim3(256), 0, (hipStream_t)stream, (uint16_t *)X,
                           strides[0], strides[1], strides[2], tokens, (int)T, (int)n_heads, (int)head_dim, per_wg, (int)n_heads, std::log2(base));
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? FACT_OK : fact::record_hip_failure(e, "rope launch");
}

size_t fact_block_scratch_bytes(const fact_block *blk)
{
    fact::blockk::Layout L;
    return fact::blockk::plan(blk, L) == FACT_OK ? L.total : 0;
}

int fact_block_scratch_offsets(const fact_block *blk, size_t *offsets)
{
    fact::blockk::Layout L;
    const int rc = fact::blockk::plan(blk, L);
    if (rc != FACT_OK) return rc;
    if (!offsets) return FACT_ERR_NULL;
    offsets[0] = L.n1; offsets[1] = L.qkv; offsets[2] = L.a; offsets[3] = L.x1; offsets[4] = L.n2; offsets[5] = L.h; offsets[6] = L.ws;
    return FACT_OK;
}

int fact_block_forward(const fact_block *blk, const void *X, void *Y, void *scratch, size_t scratch_bytes, void *stream)
{
    using namespace fact::blockk;
    Layout L;
    int rc = plan(blk, L);
    if (rc != FACT_OK) return rc;
    if (!X || !Y || !scratch) return FACT_ERR_NULL;
    if (scratch_bytes < L.least) return FACT_ERR_WORKSPACE;
    if (scratch_bytes < L.total) L.ws_bytes = scratch_bytes - L.ws;
    if (!aligned16(X) || !aligned16(Y) || ((uintptr_t)scratch & 255u)) return FACT_ERR_ALIGN;
    const fact_block &b = *blk;
    const int64_t T = b.batch * b.tokens, d = b.d_model, D = b.head_dim, nq = b.n_q_heads * D;
    const int64_t nqkv = (b.n_q_heads + 2 * b.n_kv_heads) * D;
    char *s = (char *)scratch;
    void *N1 = s + L.n1, *QKV = s + L.qkv, *A = s + L.a, *X1 = s + L.x1, *N2 = s + L.n2, *H = s + L.h, *ws = s + L.ws;
    const float eps = b.eps > 0.f ? b.eps : 1e-5f;

    rc = fact_norm(T, d, X, d, b.norm1_g, b.norm_rms ? nullptr : b.norm1_b, eps, b.norm_rms, N1, d, stream);
    if (rc != FACT_OK) return rc;
    fact_epilogue e1 = {b.bqkv, nullptr, 0, 0, FACT_ACT_NONE};
    rc = fact_gemm_splitk(T, nqkv, d, N1, d, b.Wqkv, d, 1, QKV, nqkv, &e1, 0, ws, L.ws_bytes, stream);
    if (rc != FACT_OK) return rc;
    const int64_t st[3] = {b.tokens * nqkv, nqkv, D};
    if (b.rope) {
        rc = fact_rope(b.batch, b.tokens, b.n_q_heads + b.n_kv_heads, D, QKV, st, b.rope_base > 1.f ? b.rope_base : 500000.f, stream);
        if (rc != FACT_OK) return rc;
    }
    const int64_t so[3] = {b.tokens * nq, nq, D};
    rc = fact_attention(b.batch, b.tokens, b.n_q_heads, b.n_kv_heads, D, QKV, st, (char *)QKV + 2 * nq, st,
                        (char *)QKV + 2 * (nq + b.n_kv_heads * D), st, A, so, 1, 0.f, stream);
    if (rc != FACT_OK) return rc;
    fact_epilogue e2 = {b.bo, X, d, 0, FACT_ACT_NONE};
    rc = fact_gemm_splitk(T, d, nq, A, nq, b.Wo, nq, 1, X1, d, &e2, 0, ws, L.ws_bytes, stream);
    if (rc != FACT_OK) return rc;
    rc = fact_norm(T, d, X1, d, b.norm2_g, b.norm_rms ? nullptr : b.norm2_b, eps, b.norm_rms, N2, d, stream);
    if (rc != FACT_OK) return rc;
    return fact_block_mlp(T, d, b.d_ff, N2, b.W1, b.W1u, b.b1, b.act, b.W2, b.b2, X1, H, Y, ws, L.ws_bytes, stream);
}

}  // extern "C"
