// fact_attention: argument validation and launch of the fused attention kernel.  Host code only;
// the computation runs in attention_kernel.h.
#include "../../include/fact.h"
#include "attention_kernel.h"
#include "lds_limit.h"

#include <cfloat>
#include <cmath>
#include <cstdlib>

namespace fact {

int record_hip_failure(hipError_t e, const char *what);      // fact_api.hip: text for fact_last_error()

namespace attn {

template <int D, int NW, int KG, int BKV>
static hipError_t launch(AttnArgs a, hipStream_t stream)
{
    auto kern = attn_fwd_kernel<D, NW, KG, BKV>;
    constexpr int lds = lds_bytes(D, NW, KG, BKV);
    static LdsLimit limit;
    const hipError_t e = raise_lds_limit(limit, lds, {(const void *)kern});
    if (e != hipSuccess) return e;
    constexpr int BQ = NW * 32;
    a.q_blocks = (a.T + BQ - 1) / BQ;
    a.total = a.q_blocks * a.Hq * a.B;
    // Pairs per group of the work-group order (see the kernel): a multiple of 4, so that each of an
    // XCD's shader engines gets the same mix of heavy and light work-groups; as large as the K/V of
    // the group's heads still fits an XCD's L2 (4 MB), which also starts the heavy work-groups early.
    {
        const int pairs = a.Hq * a.B, per = (pairs & 7) == 0 ? pairs >> 3 : pairs, G = a.Hq / a.Hkv;
        int best = 0, smallest = 0;
        for (int r = 4; r <= per; r += 4) {
            if (per % r) continue;
            if (!smallest) smallest = r;
            const int64_t kv_heads = r >= G ? (r + G - 1) / G : 1;
            if (kv_heads * a.T * D * 4 <= (int64_t)4 << 20) best = r;
        }
        a.group = best ? best : smallest ? smallest : per;
    }
    // Work-groups of one residency round (see attn_fwd_kernel's launch bounds: 3 and 2 per compute unit) reach the
    // compute units in layers of 32 per XCD; the last layer is folded back (1 x 2048 tokens, 32 heads of 128:
    // 47.0 -> 44.4 us).
    {
        const bool split = (a.Hq * a.B & 7) == 0;
        const int n = split ? a.total >> 3 : a.total, layer = split ? 32 : 256, layers = (n + layer - 1) / layer;
        a.fold = a.causal && layers >= 2 && layers <= (KG > 1 ? 1 : D == 64 ? 3 : 2) ? (layers - 1) * layer : n;
    }
    // (a grid's threads are counted in 32 bits: more than 2^20 work-groups go into further rows of the grid)
    a.grid_x = a.total > 1 << 20 ? 1 << 20 : a.total;
    hipLaunchKernelGGL(kern, dim3((unsigned)a.grid_x, (unsigned)(((int64_t)a.total + a.grid_x - 1) / a.grid_x)), dim3(NW * KG * 64), lds, stream, a);
    return hipGetLastError();
}

// Which shape of work-group: query groups of 32, key groups, keys of a block.  With few work-groups, above all causal ones of
// which the last walks all the keys, a launch lasts as long as its longest work-group, at one wave per SIMD: key groups shorten
// that chain and put more waves on a compute unit, fewer queries per work-group make more of them; each costs more K and V from
// the L2 per query.  Key blocks of 32 leave four waves per SIMD at head_dim 64 in place of three.  us, 4 x 1 x 64 -> the choice
// (batch x tokens, query heads): head_dim 64 causal 1 x 616, 12 10.6 -> 6.8 (1 x 4 x 32), 7 x 2049, 2 26.7 -> 18.2 (2 x 2 x 64), 36 x 208, 12 14.7 -> 11.8
// (4 x 1 x 32), full 1 x 509, 16 9.2 -> 6.5 (1 x 4 x 32); head_dim 128 causal 1 x 1172, 16 24.1 -> 19.1, 1 x 393, 32 10.9 -> 9.5 (2 x 2 x 32).
// The estimate in us: a start, then the longer of one chain (`chain` per step of the longest work-group) and the chip's throughput
// (`step` and `group` per step and work-group, over 256 compute units); with one key group, where work-groups of all lengths
// share a compute unit, the two overlap badly (the fourth root of the fourth powers' sum).  Fitted to 262 calls of head_dim 64 and 202 of
// 128 (profiles/attention_shape_calls.csv), mean error 6-8 %; a shape other than 4 x 1 x 64 is taken where it is 3 % below: over those calls 5.2 %
// and 1.6 % faster, the best shape of each 7.2 % and 2.3 %, the worst choice 7 % slower.  `resident`: work-groups of the chip at once
// (LDS); beyond that shapes with key groups do not serve.
struct Shape { int nw, kg, bkv, resident; double start, chain, step, group; };
static constexpr Shape kShapes64[4] = {{4, 1, 64, 0, 3.52, 0.775, 0.56, 1.36}, {4, 1, 32, 0, 3.46, 0.45, 0.289, 1.12},
                                       {2, 2, 64, 512, 3.63, 0.932, 0.592, 1.734}, {1, 4, 32, 512, 3.4, 0.86, 0.404, 1.511}};
static constexpr Shape kShapes128[3] = {{4, 1, 64, 0, 3.96, 1.07, 0.97, 1.91}, {2, 2, 32, 512, 4.29, 0.823, 0.55, 2.11},
                                        {1, 4, 32, 256, 3.54, 1.61, 1.04, 3.4}};
template <int N>
static int choose(const AttnArgs &a, const Shape (&shapes)[N])
{
    if (a.T <= 64) return 0;                                 // (one key block: nothing to share)
    const double pairs = (double)a.B * a.Hq;
    int best = 0;
    double least = 0.0;
    for (int i = 0; i < N; ++i) {
        const Shape &s = shapes[i];
        const int bq = s.nw * 32, rows = s.kg * s.bkv;
        const double blocks = (a.T + bq - 1) / bq, longest = (a.T + rows - 1) / rows;
        if (s.resident && blocks * pairs > s.resident) continue;
        // steps of all query blocks of a head: the first ends at key bq, the last at T
        const double steps = a.causal ? blocks * (bq > rows ? (double)bq / rows + longest : 1.0 + longest) / 2.0 : blocks * longest;
        const double x = longest * s.chain, y = pairs * (steps * s.step + blocks * s.group) / 256.0;
        const double us = s.start + (s.kg > 1 ? (x > y ? x : y) : std::sqrt(std::sqrt(x * x * x * x + y * y * y * y)));
        if (i == 0) least = 0.97 * us;
        else if (us < least) { least = us; best = i; }
    }
    return best;
}

}  // namespace attn
}  // namespace fact

extern "C" int fact_test_attention_shape(int64_t batch, int64_t T, int64_t n_q_heads, int64_t head_dim, int causal, int *query_groups, int *key_groups, int *keys)
{
    using namespace fact::attn;
    if (batch <= 0 || T <= 0 || n_q_heads <= 0 || batch > 0x7FFFFFFF || T > 0x7FFFFFFF - 1024 || n_q_heads > 0x7FFFFFFF) return FACT_ERR_DIM;
    if (head_dim != 64 && head_dim != 128) return FACT_ERR_UNSUPPORTED;
    AttnArgs a;
    a.B = (int)batch; a.T = (int)T; a.Hq = (int)n_q_heads; a.causal = causal;
    const Shape &s = head_dim == 128 ? kShapes128[choose(a, kShapes128)] : kShapes64[choose(a, kShapes64)];
    if (query_groups) *query_groups = s.nw;
    if (key_groups) *key_groups = s.kg;
    if (keys) *keys = s.bkv;
    return FACT_OK;
}

extern "C" int fact_attention(int64_t batch, int64_t T, int64_t n_q_heads, int64_t n_kv_heads, int64_t head_dim,
                              const void *Q, const int64_t *q_strides, const void *K, const int64_t *k_strides,
                              const void *V, const int64_t *v_strides, void *O, const int64_t *o_strides,
                              int causal, float scale, void *stream)
{
    using namespace fact::attn;
    if (!Q || !K || !V || !O || !q_strides || !k_strides || !v_strides || !o_strides) return FACT_ERR_NULL;
    if (batch <= 0 || T <= 0 || n_q_heads <= 0 || n_kv_heads <= 0) return FACT_ERR_DIM;
    if (n_q_heads % n_kv_heads) return FACT_ERR_DIM;
    if (head_dim != 64 && head_dim != 128) return FACT_ERR_UNSUPPORTED;
    if (causal != 0 && causal != 1) return FACT_ERR_LAYOUT;
    if (!(scale == scale) || std::isinf(scale)) return FACT_ERR_DIM;
    // a row's head_dim elements are contiguous; the kernel addresses rows with 32-bit byte offsets
    // inside one (batch entry, head) and moves 16 bytes (inputs) or 8 bytes (output) at a time
    const int64_t *in[3] = {q_strides, k_strides, v_strides};
    const void *ptr[3] = {Q, K, V};
    for (int i = 0; i < 3; ++i) {
        const int64_t sb = in[i][0], st = in[i][1], sh = in[i][2];
        if (st < head_dim || sb < 0 || sh < 0) return FACT_ERR_DIM;
        if ((T + 512) * st * 2 >= (int64_t)1 << 31) return FACT_ERR_UNSUPPORTED;
        if (((uintptr_t)ptr[i] & 15u) || (sb & 7) || (st & 7) || (sh & 7)) return FACT_ERR_ALIGN;
    }
    if (o_strides[1] < head_dim || o_strides[0] < 0 || o_strides[2] < 0) return FACT_ERR_DIM;
    if (o_strides[1] > 0x7FFFFFFF) return FACT_ERR_UNSUPPORTED;
    if (((uintptr_t)O & 7u) || (o_strides[0] & 3) || (o_strides[1] & 3) || (o_strides[2] & 3)) return FACT_ERR_ALIGN;
    if (batch * n_q_heads * ((T + 127) / 128) > 0x7FFFFFFF || T > 0x7FFFFFFF - 1024) return FACT_ERR_UNSUPPORTED;

    AttnArgs a;
    a.Q = (const __bf16 *)Q; a.K = (const __bf16 *)K; a.V = (const __bf16 *)V; a.O = (__bf16 *)O;
    a.q_sb = q_strides[0]; a.q_st = (int)q_strides[1]; a.q_sh = q_strides[2];
    a.k_sb = k_strides[0]; a.k_st = (int)k_strides[1]; a.k_sh = k_strides[2];
    a.v_sb = v_strides[0]; a.v_st = (int)v_strides[1]; a.v_sh = v_strides[2];
    a.o_sb = o_strides[0]; a.o_st = (int)o_strides[1]; a.o_sh = o_strides[2];
    a.B = (int)batch; a.T = (int)T; a.Hq = (int)n_q_heads; a.Hkv = (int)n_kv_heads;
    a.causal = causal;
    const float sc = scale > 0.f ? scale : 1.0f / std::sqrt((float)head_dim);
    a.scale_log2 = sc * 1.4426950408889634f;
    a.lowest = std::fmax(-0x1p31f / a.scale_log2, -FLT_MAX);
    a.q_blocks = 0; a.total = 0; a.grid_x = 0; a.group = 1; a.fold = 0;

    hipStream_t s = (hipStream_t)stream;
    hipError_t e;
    if (head_dim == 128) {
        switch (choose(a, kShapes128)) {
        case 0: e = launch<128, 4, 1, 64>(a, s); break;
        case 1: e = launch<128, 2, 2, 32>(a, s); break;
        default: e = launch<128, 1, 4, 32>(a, s); break;
        }
    } else {
        switch (choose(a, kShapes64)) {
        case 0: e = launch<64, 4, 1, 64>(a, s); break;
        case 1: e = launch<64, 4, 1, 32>(a, s); break;
        case 2: e = launch<64, 2, 2, 64>(a, s); break;
        default: e = launch<64, 1, 4, 32>(a, s); break;
        }
    }
    return e == hipSuccess ? FACT_OK : fact::record_hip_failure(e, "attention launch");
}
