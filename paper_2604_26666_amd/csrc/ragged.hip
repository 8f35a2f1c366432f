// GEMM for operands the main kernel cannot take: rows that start at any 2-byte address, and any M, N, K
// (odd leading dimensions, K or N no multiple of 8, unaligned pointers).  The main kernel moves operands
// straight from global memory into LDS, which needs 16-byte aligned rows; here they pass through registers,
// where a 16-byte global load may start at any 2-byte address (the unaligned-access mode that the compiler
// targets on this architecture), and go to LDS in the same swizzled layouts.  Measured: 2000 x 1999 x 1777 33.6 us = 423 TFLOP/s (when it was
// 35, rows that all begin at whole words took 29 and all at half words 36-40); the main kernel on 2000 x 2000 x 1784 24.4.  Two steps of loads in flight,
// with the order of loads and matrix products fixed, were slower (37.4), so the loop's order is the compiler's.
#include "launch.h"
#include "lds_limit.h"
#include "shift_down.h"

namespace fact {

template <bool F16>
__device__ __forceinline__ f32x4_t mfma_any(bf16x8_t a, bf16x8_t b, f32x4_t c)
{
    typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));
    if constexpr (F16) return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8_t, a), __builtin_bit_cast(f16x8_t, b), c, 0, 0, 0);
    else return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ s16x4_t read_tr16(const char *lds)
{
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t *)(lds));
}

// A work-group owns a BM x BN tile; its 4 KW waves form KW groups of WGM x WGN waves, and group g takes the 64-deep
// K steps g, g + KW, ...  Each group keeps two LDS stages and two further steps of operands in registers on their
// way there (the K loop is bound by the loads' latency: with one step in flight and one group per compute unit
// 2000 x 1999 x 1777 took 45 us, as it stands 33.6; the one-thread-per-element kernel 3416 us).  A 16-byte piece that would cross the end of a row (K-contiguous operand) or of the
// matrix's columns (B as [K][N]) is loaded so that it ends there and shifted into place, so nothing outside the
// matrices is ever read; a step past the end of K brings zeros.
template <int BM, int BN, int WGM, int WGN, int KW, bool TRANS_B, bool F16>
__global__ void __launch_bounds__(256 * KW, KW == 1 ? 2 : 1)
ragged_kernel(const GemmArgs p)
{
    static_assert(WGM * WGN == 4, "four waves per group");
    constexpr int WTM = BM / WGM, WTN = BN / WGN, MT = WTM / 16, NT = WTN / 16, HT = NT / 2;
    static_assert(NT % 2 == 0, "a gated wave tile pairs gate and up tiles");
    constexpr int A_BYTES = BM * 128, STAGE = (BM + BN) * 128;
    constexpr int A_LD = BM / 32, B_LD = BN / 32;            // 16-byte pieces per thread and step
    constexpr int NCH = BN / 8;                              // pieces per K-row of a [K][N] operand
    extern __shared__ __attribute__((aligned(1024))) char smem[];

    const int tid = threadIdx.x & 255, lane = tid & 63;
    const int wave_all = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), group = wave_all >> 2, wave = wave_all & 3;
    const int wm = wave / WGN, wn = wave % WGN, r16 = lane & 15, q = lane >> 4;
    const bool gated = p.act == ACT_SILU_GATE;
    const int nout = gated ? p.N >> 1 : p.N;
    int tm, tn;
    tile_coords(p, blockIdx.x, p.tiles_m * p.tiles_n, tm, tn);
    const int m0 = tm * BM, n0 = tn * (gated ? BN / 2 : BN);
    const int64_t z = blockIdx.z;
    const int K = p.K;

    // ---- global addresses: thread -> piece tid % 8 of rows tid / 8 + 32 i (K-contiguous), piece tid % NCH of K-rows
    // tid / NCH + i * 256 / NCH ([K][N]).  Rows past the edge repeat the last one: their results are not stored.
    const int kc = tid & 7;
    const uint16_t *pa[A_LD], *pb[TRANS_B ? B_LD : 1];
#pragma unroll
    for (int i = 0; i < A_LD; ++i) {
        const int m = m0 + (tid >> 3) + 32 * i;
        pa[i] = (const uint16_t *)(p.A + z * p.stride_a) + (int64_t)(m < p.M ? m : p.M - 1) * p.lda;
    }
    constexpr int KR = 256 / NCH;                            // K-rows a round of loads covers
    const int nc = tid % NCH, kr = tid / NCH;
    int shift_n = 0;                                         // [K][N]: this thread's pieces end at column N and move down
    if constexpr (TRANS_B) {
#pragma unroll
        for (int i = 0; i < B_LD; ++i) {
            const int r = (tid >> 3) + 32 * i;               // LDS row; gated: 16 gate columns, the same 16 up columns, and so on
            const int n = n0 + (gated ? (r >> 5) * 16 + (r & 15) : r);
            const __bf16 *base = gated && (r & 16) ? p.B_up : p.B;
            pb[i] = (const uint16_t *)(base + z * p.stride_b) + (int64_t)(n < nout ? n : nout - 1) * p.ldb;
        }
    } else {
        int n = n0 + nc * 8;
        if (n > p.N - 8) { shift_n = n - (p.N - 8); n = p.N - 8; }
        pb[0] = (const uint16_t *)(p.B + z * p.stride_b) + n;
    }
    const bool ragged_n = !TRANS_B && n0 + BN > p.N;         // uniform

    // Loads of the group's step i: a piece that would pass K ends at K instead, a K-row past K repeats the last one;
    // to_lds puts such pieces right (uniform branch, taken for the last steps only).
    struct Step { u32x4_t a[A_LD], b[B_LD]; };
    auto load = [&](Step &r, int i) __attribute__((always_inline)) {
        const int k0 = (i * KW + group) * 64;
        const int c = k0 + kc * 8, at = c < K - 8 ? c : K - 8;
#pragma unroll
        for (int x = 0; x < A_LD; ++x) r.a[x] = *(const u32x4_any *)(pa[x] + at);
#pragma unroll
        for (int x = 0; x < B_LD; ++x) {
            if constexpr (TRANS_B) r.b[x] = *(const u32x4_any *)(pb[x] + at);
            else {
                const int k = k0 + kr + x * KR;
                r.b[x] = *(const u32x4_any *)(pb[0] + (int64_t)(k < K ? k : K - 1) * p.ldb);
            }
        }
    };
    char *const ring = smem + group * 2 * STAGE;
    auto to_lds = [&](Step &r, int i) __attribute__((always_inline)) {
        char *s = ring + (i & 1) * STAGE;
        const int k0 = (i * KW + group) * 64;
        if (k0 + 64 > K) {
            const int c = k0 + kc * 8, sh = c < K - 8 ? 0 : c - (K - 8);
#pragma unroll
            for (int x = 0; x < A_LD; ++x) r.a[x] = shift_down(r.a[x], sh);
#pragma unroll
            for (int x = 0; x < B_LD; ++x) {
                if constexpr (TRANS_B) r.b[x] = shift_down(r.b[x], sh);
                else if (k0 + kr + x * KR >= K) r.b[x] = u32x4_t{0u, 0u, 0u, 0u};
            }
        }
        if (ragged_n) {
#pragma unroll
            for (int x = 0; x < B_LD; ++x) r.b[x] = shift_down(r.b[x], shift_n);
        }
#pragma unroll
        for (int x = 0; x < A_LD; ++x) {
            const int row = (tid >> 3) + 32 * x;
            *(u32x4_t *)(s + row * 128 + ((kc ^ swz_k(row)) << 4)) = r.a[x];
        }
#pragma unroll
        for (int x = 0; x < B_LD; ++x) {
            if constexpr (TRANS_B) {
                const int row = (tid >> 3) + 32 * x;
                *(u32x4_t *)(s + A_BYTES + row * 128 + ((kc ^ swz_k(row)) << 4)) = r.b[x];
            } else {
                const int k = kr + x * KR;
                *(u32x4_t *)(s + A_BYTES + k * (BN * 2) + ((nc ^ swz_n<BN>(k)) << 4)) = r.b[x];
            }
        }
    };

    f32x4_t acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    auto compute = [&](int slot) __attribute__((always_inline)) {
        const char *s = ring + slot * STAGE;
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            bf16x8_t a[MT], b[NT];
            const int ch = ((4 * kk + q) ^ swz_k(r16)) << 4;
#pragma unroll
            for (int i = 0; i < MT; ++i) a[i] = *(const bf16x8_t *)(s + (wm * WTM + i * 16 + r16) * 128 + ch);
#pragma unroll
            for (int j = 0; j < NT; ++j) {
                if constexpr (TRANS_B) {
                    b[j] = *(const bf16x8_t *)(s + A_BYTES + (wn * WTN + j * 16 + r16) * 128 + ch);
                } else {
                    // transposing reads (see the main kernel): lane 4 jj + c of a 16-lane group names K-row jj, columns 4c ..
                    const int k = 32 * kk + 8 * q + ((lane >> 2) & 3), n = wn * WTN + j * 16 + 4 * (lane & 3);
                    const char *at = s + A_BYTES + k * (BN * 2) + (((n >> 3) ^ swz_n<BN>(k)) << 4) + (lane & 1) * 8;
                    const s16x4_t lo = read_tr16(at), hi = read_tr16(at + 4 * BN * 2);
                    b[j] = __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
                }
            }
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int j = 0; j < NT; ++j) acc[i][j] = mfma_any<F16>(b[j], a[i], acc[i][j]);
        }
    };

    const int steps = ((K + 63) / 64 + KW - 1) / KW;         // per group, the same for all
    Step r0, r1;
    load(r0, 0);
    if (steps > 1) load(r1, 1);
    to_lds(r0, 0);
    __syncthreads();
    // (The last steps apart, so that nothing past them is loaded: loads are what bounds this kernel, and two steps' worth beyond the
    // end, with the loop left in the middle, made 2000 x 1999 x 1777 35.2 us for 33.6, 1803 x 2101 x 301 12.6 for 12.0, 1207 x 1032 x 31 5.0
    // for 4.3; the same with a condition at each load was slower than either, 36.5.)
    int i = 0;
    for (; i + 3 < steps; i += 2) {
        load(r0, i + 2);
        compute(0);
        to_lds(r1, i + 1);
        __syncthreads();
        load(r1, i + 3);
        compute(1);
        to_lds(r0, i + 2);
        __syncthreads();
    }
    const int rest = steps - i;                              // 1, 2 or 3
    if (rest == 3) load(r0, i + 2);
    compute(0);
    if (rest > 1) {
        to_lds(r1, i + 1);
        __syncthreads();
        compute(1);
        if (rest == 3) {
            to_lds(r0, i + 2);
            __syncthreads();
            compute(0);
        }
    }
    __syncthreads();

    // ---- sums of the K groups, through LDS: unit (i, j) of a wave tile (its tiles 2 j and 2 j + 1 of row i) is finished by
    // group i mod KW, which adds the groups' sums in ascending order
    if constexpr (KW > 1) {
        f32x4_t *const sums = (f32x4_t *)smem;               // [unit][half][group][thread of the group]
#pragma unroll
        for (int u = 0; u < MT * HT; ++u)
            if (u / HT % KW != group) {
                sums[((u * 2 + 0) * KW + group) * 256 + tid] = acc[u / HT][u % HT * 2];
                sums[((u * 2 + 1) * KW + group) * 256 + tid] = acc[u / HT][u % HT * 2 + 1];
            }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < MT * HT; ++u)
            if (u / HT % KW == group) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const f32x4_t own = acc[u / HT][u % HT * 2 + h];
                    f32x4_t v = group == 0 ? own : sums[((u * 2 + h) * KW) * 256 + tid];
#pragma unroll
                    for (int g = 1; g < KW; ++g) v += group == g ? own : sums[((u * 2 + h) * KW + g) * 256 + tid];
                    acc[u / HT][u % HT * 2 + h] = v;
                }
            }
    }

    // ---- epilogue: lane (r16, q) of tile (i, j) holds columns 4q .. 4q + 3 of row r16
    const uint16_t *res = p.res ? (const uint16_t *)(p.res + z * p.stride_r) : nullptr;
    uint16_t *C = (uint16_t *)(p.C + z * p.stride_c);
    const uint16_t *bias = (const uint16_t *)p.bias;
    const int n_wave = n0 + wn * (gated ? WTN / 2 : WTN);
    if (gated) {
#pragma unroll
        for (int u = 0; u < MT * HT; ++u) {
            if (KW > 1 && u / HT % KW != group) continue;
            const int i = u / HT, j = u % HT, n = n_wave + j * 16 + 4 * q, m = m0 + wm * WTM + i * 16 + r16;
            if (m >= p.M || n >= nout) continue;
            const bool full = n + 4 <= nout;
            float v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                v[e] = silu(acc[i][2 * j][e]) * acc[i][2 * j + 1][e];
                if (bias && n + e < nout) v[e] += in16<F16>(bias[n + e]);
            }
            if (res) {
                const uint16_t *rp = res + (int64_t)m * p.ldr + n;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (n + e < nout) v[e] += in16<F16>(rp[e]);
            }
            uint16_t *cp = C + (int64_t)m * p.ldc + n;
            if (full) *(u32x2_any *)cp = u32x2_t{pack2<F16>(pk_f32_t{v[0], v[1]}), pack2<F16>(pk_f32_t{v[2], v[3]})};
            else {
#pragma unroll
                for (int e = 0; e < 3; ++e)
                    if (n + e < nout) cp[e] = (uint16_t)out16<F16>(v[e]);
            }
        }
        return;
    }
    // 8 columns of a row to a lane: two tiles' rows change places between lanes 16 apart; store8_of_row moves them to whole words
    // (before: 4 columns at any 2-byte address, the bias element by element; with a bias 2000 x 1999 x 1777 36.9 -> 35.1 us,
    // 1859 x 1658 x 92 13.1 -> 9.9, 1445 x 3347 x 349 23.7 -> 20.8, 3404 x 2085 x 34 without one 11.7 -> 10.6).
    const int n = n_wave + (q & 1) * 16 + (q >> 1) * 8, next_lane = (((0x0132 >> (q * 4)) & 3) * 16 + r16) * 4;
    const bool odd_rows = ((p.ldc & 1) | ((size_t)C >> 1 & 1)) != 0;
    // 8 elements of which left lie inside the row (single ones at indexes kept inside it: behind a branch each would wait for the last)
    auto load8 = [&](const uint16_t *from, int left) __attribute__((always_inline)) {
        u32x4_t w = {0u, 0u, 0u, 0u};
        if (left >= 8) w = *(const u32x4_any *)from;
        else if (left > 0) {
            uint32_t x[7];
#pragma unroll
            for (int e = 0; e < 7; ++e) x[e] = from[e < left ? e : 0];
#pragma unroll
            for (int e = 0; e < 7; ++e) w[e / 2] |= x[e] << (16 * (e & 1));
        }
        return w;
    };
    u32x4_t bv[HT];
    if (bias) {
#pragma unroll
        for (int jh = 0; jh < HT; ++jh) bv[jh] = load8(bias + n + jh * 32, nout - (n + jh * 32));
    }
#pragma unroll
    for (int i = 0; i < MT; ++i) {
        if (KW > 1 && i % KW != group) continue;
        const int m = m0 + wm * WTM + i * 16 + r16;
        const bool live = m < p.M;
        uint32_t first = 0;
#pragma unroll
        for (int jh = HT - 1; jh >= 0; --jh) {
            const int nj = n + jh * 32, left = nout - nj;
            float v[8];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float a0 = acc[i][2 * jh][e], a1 = acc[i][2 * jh + 1][e];
                const auto sw = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, a0), __builtin_bit_cast(uint32_t, a1), false, false);
                v[e] = __builtin_bit_cast(float, (uint32_t)sw[0]);
                v[4 + e] = __builtin_bit_cast(float, (uint32_t)sw[1]);
            }
            if (bias) {
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] += in16<F16>(bv[jh][e / 2] >> (16 * (e & 1)) & 0xFFFFu);
            }
            if (p.act == ACT_GELU_TANH) {
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] = gelu_tanh(v[e]);
            }
            if (res && live) {
                const u32x4_t w = load8(res + (int64_t)m * p.ldr + nj, left);
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] += in16<F16>(w[e / 2] >> (16 * (e & 1)) & 0xFFFFu);
            }
            u32x4_t o;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = pack2<F16>(pk_f32_t{v[2 * e], v[2 * e + 1]});
            uint16_t *at = C + (int64_t)m * p.ldc + nj;
            if (odd_rows) {
                const uint32_t follow = (uint32_t)__builtin_amdgcn_ds_bpermute(next_lane, (int)(q == 0 ? first : o[0]));
                first = o[0];
                if (live) store8_of_row<true>(at, o, follow, jh == 0 && q == 0, jh == HT - 1 && q == 3, left);
            } else if (live) {
                if (left >= 8) *(u32x4_words *)at = o;
                else store_few(at, o, 0, left);
            }
        }
    }
}

template <int BM, int BN, int WGM, int WGN, int KW, bool TRANS_B, bool F16>
static hipError_t launch_one(const GemmArgs &a, dim3 grid, hipStream_t stream)
{
    auto kern = ragged_kernel<BM, BN, WGM, WGN, KW, TRANS_B, F16>;
    constexpr int lds = KW * 2 * (BM + BN) * 128;
    static_assert(lds <= 160 * 1024 && (BM / WGM / 16) * (BN / WGN / 16) * KW * 4096 <= lds, "LDS: rings, then the groups' sums");
    if constexpr (lds > 64 * 1024) {
        static LdsLimit limit;
        const hipError_t e = raise_lds_limit(limit, lds, {(const void *)kern});
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kern, grid, dim3(256 * KW), lds, stream, a);
    return hipGetLastError();
}

template <int BM, int BN, int WGM, int WGN, int KW>
static hipError_t launch_tile(GemmArgs a, bool trans_b, int grid_z, hipStream_t stream)
{
    const bool gated = a.act == ACT_SILU_GATE;
    const int nout = gated ? a.N / 2 : a.N, bn_out = gated ? BN / 2 : BN;
    const int64_t tm = (a.M + (int64_t)BM - 1) / BM, tn = (nout + (int64_t)bn_out - 1) / bn_out;
    if (tm * tn > 0x7FFFFFFF / 2) return hipErrorInvalidConfiguration;
    a.tiles_m = (int)tm; a.tiles_n = (int)tn; a.group_m = 4;
    const dim3 grid((unsigned)(tm * tn), 1, (unsigned)grid_z);
    if (a.f16) return trans_b ? launch_one<BM, BN, WGM, WGN, KW, true, true>(a, grid, stream) : launch_one<BM, BN, WGM, WGN, KW, false, true>(a, grid, stream);
    return trans_b ? launch_one<BM, BN, WGM, WGN, KW, true, false>(a, grid, stream) : launch_one<BM, BN, WGM, WGN, KW, false, false>(a, grid, stream);
}

// Operands whose rows hold at least one 16-byte piece; shorter ones stay with the guarded kernel.  So do sizes of which the
// edge of a last tile, or K-values past the end, would leave the 32-bit indexes: a last K group's step begins up to 3 x 64 past
// the last block of 64, and a wave of the kernel whose waves split K loads up to 3 turns of 4 waves (12 blocks) past it.  A wrapped
// index is negative, which the clamps take for inside.
// And so does a K of a few elements where the guarded kernel has little to do, or where a tile here is mostly edge (us, guarded
// and this kernel, K = 9 unless said): 8 x 8 2.1 / 2.7, 1 x 1000 2.5 / 3.3, 300 x 300 2.8 / 3.3 (K = 13 3.2 / 3.2, 17 3.7 / 3.3),
// 100000 x 9 8.7 / 17.2 (K = 17 13.5 / 17.3, with [N][K] 20.4 / 16.6), 9 x 100000 12.4 / 13.6 (K = 13 16.0 / 13.7);
// but 1000 x 1000 6.9 / 4.3, 4000 x 300 8.0 / 5.2, 100000 x 33 26.9 / 20.5.
static bool guarded_is_faster(const GemmArgs &a, bool trans_b, int64_t batch)
{
    if (a.K > 24) return false;
    const int nout = a.act == ACT_SILU_GATE ? a.N / 2 : a.N;
    const int64_t blocks = ((int64_t)a.M + 15) / 16 * (((int64_t)nout + 15) / 16) * batch;      // the guarded kernel's work-groups
    if (blocks * a.K <= 4096) return a.K <= 13;
    if (nout <= 16) return a.K <= 13 || (!trans_b && blocks >= 2048);
    return a.M <= 16 && a.K <= 9;
}

bool ragged_serves(const GemmArgs &a, bool trans_b, int64_t batch)
{
    constexpr int kLast = INT32_MAX - 4096;
    return a.K >= 8 && (trans_b || a.N >= 8) && a.M <= kLast && a.N <= kLast && a.K <= kLast && !guarded_is_faster(a, trans_b, batch);
}

// The largest tile that still gives most compute units a work-group, and several K groups per work-group where
// K is long enough to share: what is short here is loads in flight, not matrix cores.  Measured (us, one launch,
// operands in the memory-side cache; tile and K groups):
//   2000 x 1999 x 1777   128/1 41.7   128/2 35.7   64/2 46.7   32x64/4 91.0   guarded kernel 3416
//   1000 x  999 x 1777   128/2 31.4    64/1 17.6   64/2 14.5   32x64/4 24.0
//    300 x  999 x  777    64/1 10.2    64/2  9.6   32x64/1 9.3   32x64/4  9.6
//      7 x 2731 x 1284    64/1  9.9    64/4  9.5   32x64/1 8.5   32x64/4  8.2   guarded kernel  119
//      1 x 4001 x 4001    64/1 26.3    64/4 20.5   32x64/1 23.1  32x64/4 16.5
//   3850 x 1884 x   31   128/1 12.3   128/2 18.8    64/1 12.9
//    858 x  133 x   33   128/1 11.6    64/1  5.4   32x64/1 4.4   32x64/4  6.5
struct RaggedTile { int bm, bn, groups; };
static constexpr RaggedTile kRaggedTiles[6] = {{128, 128, 1}, {128, 128, 2}, {64, 64, 1}, {64, 64, 2}, {32, 64, 1}, {32, 64, 4}};
static int ragged_tile(const GemmArgs &a, int64_t batch)
{
    auto tiles = [&](int64_t bm, int64_t bn) { return (a.M + bm - 1) / bm * ((a.N + bn - 1) / bn) * batch; };
    if (tiles(128, 128) >= 160) return a.K >= 512 && tiles(128, 128) < 512 ? 1 : 0;
    if (tiles(64, 64) >= 160) return a.K >= 256 ? 3 : 2;
    return a.K >= 768 ? 5 : 4;
}

// Its estimated microseconds where there are few work-groups (fitted to the calls of small_any_us, mean error 5 and 8 %).
static double ragged_us(const GemmArgs &a, bool trans_b, int64_t batch)
{
    const RaggedTile t = kRaggedTiles[ragged_tile(a, batch)];
    const double wgs = (double)((a.M + (int64_t)t.bm - 1) / t.bm * ((a.N + (int64_t)t.bn - 1) / t.bn) * batch);
    const int64_t blocks = ((int64_t)a.K + 63) / 64;
    const double load = (wgs > 256 ? wgs / 256.0 : 1.0) * 128.0 * t.groups * (t.bm + t.bn) / (trans_b ? 55.6e3 : 43.7e3);
    const double step = !trans_b && load < 0.376 ? 0.376 : load;
    return (trans_b ? 2.44 : 2.71) + 0.0021 * wgs + (trans_b ? 2.07 : 1.51) * t.bm * t.bn / 4096.0 + (double)((blocks + t.groups - 1) / t.groups) * step;
}

// Small outputs go to the kernel whose waves split K where that is the faster one by its estimate (us, this kernel -> that one; M x N x K: 1 x 34 x 1917
// [N][K] 11.1 -> 4.9, 9 x 83 x 1443 [N][K] 9.0 -> 4.3, 273 x 53 x 3855 [K][N] 21.5 -> 10.7, 45 x 2916 x 3331 [N][K] 18.0 -> 12.8; but 304 x 3477 x 246 [N][K]
// 6.4 -> 9.2, 137 x 3402 x 334 [K][N] 6.2 -> 8.6).  Over the 420 calls of profiles/gemm_small_odd_calls.csv the choice is 1.23 times as fast, the better kernel of every call 1.25.
static constexpr int kSmallForms = 6;                        // the tiles of small_any_us follow those of kRaggedTiles
int ragged_form(const GemmArgs &a, bool trans_b, int64_t batch)
{
    int small = -1;
    const double us = small_any_us(a, trans_b, batch, &small);
    return small >= 0 && us < 0.96 * ragged_us(a, trans_b, batch) ? kSmallForms + small : ragged_tile(a, batch);
}

hipError_t launch_ragged_gemm(const GemmArgs &a, bool trans_b, int form, int grid_z, hipStream_t stream)
{
    switch (form) {
    case 0: return launch_tile<128, 128, 2, 2, 1>(a, trans_b, grid_z, stream);
    case 1: return launch_tile<128, 128, 2, 2, 2>(a, trans_b, grid_z, stream);
    case 2: return launch_tile<64, 64, 2, 2, 1>(a, trans_b, grid_z, stream);
    case 3: return launch_tile<64, 64, 2, 2, 2>(a, trans_b, grid_z, stream);
    case 4: return launch_tile<32, 64, 2, 2, 1>(a, trans_b, grid_z, stream);
    case 5: return launch_tile<32, 64, 2, 2, 4>(a, trans_b, grid_z, stream);
    default: return launch_small_any(a, trans_b, form - kSmallForms, grid_z, stream);
    }
}

}  // namespace fact
