// Routed FP8 / FP4 GEMM for a handful of (token, slot) pairs (see qgemm_small_w4.hip for why these have a kernel of
// their own).  The problem is split by pair (combine epilogue: by token, all of its slots together) and by 16-row
// weight tiles, one wavefront per tile and slot.  Unlike the int4 kernel a wavefront keeps the whole k range of its
// tile: the fp32 sum of these formats runs through one accumulator from k = 0 on, and the matrix core aligns the
// products of a block to the largest of them and to that sum, so only the same chain of 16x16x32 instructions gives
// the streaming kernel's bits.  8 to 16 KiB per wavefront are in flight.  The workgroup quantizes its 16-bit rows itself,
// one wavefront per row, with the row quantizer's arithmetic.
//
// 128 experts, hidden 2048, intermediate 768, top-8, layer of router, gate_up, down + combine: 1 token FP8 81 -> 26 us
// (gate_up 49 -> 10.5, down + combine 29 -> 10), FP4 52 -> 25 us.
#include "route_token.hpp"

namespace qarl {

namespace {

struct SmallFp8Params {
    const uint32_t *codes;   // e4m3 bytes as words [E][N][K/4], or packed e2m1 codes [E][N][K/8]
    const float *scales;     // [E][N]
    const uint16_t *x;       // bf16 rows
    const int32_t *ids;      // [T][topk]
    const float *combine_w;  // [T][topk], combine epilogue
    void *out;
    int E, N, K, out_f32, topk, x_per_token;
    // SILU_MUL: the workgroup routes its token itself and the token's first one writes ids and weights (ids is not read)
    const uint16_t *logits;   // [T][E], or null
    int32_t *ids_out;
    float *w_out;
    int renorm;
    int n_slices;            // workgroups along the weight tiles
};

// EPI: NONE, SILU_MUL (the tiles of a workgroup are gate tiles and their up tiles in turn) or COMBINE (one tile per
// workgroup, a wavefront per slot)
template <int EPI, bool W4>
__global__ __launch_bounds__(EPI == QARL_EPI_COMBINE ? 512 : 256, 2) void qgemm_small_fp8_kernel(SmallFp8Params p)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    constexpr bool kSilu = (EPI == QARL_EPI_SILU_MUL), kComb = (EPI == QARL_EPI_COMBINE);
    constexpr int kWaves = kComb ? 8 : 4;
    constexpr int R = 8, kH = W4 ? 1 : 2;   // 128-k steps in flight; 16-byte loads per lane and step

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, q = lane >> 4;
    const int N = p.N, K = p.K, G = K / kGroup, words_per_row = W4 ? K / 8 : K / 4;
    const int slice = blockIdx.x % p.n_slices, item = blockIdx.x / p.n_slices;   // item: pair, or token (combine)
    const int nslot = kComb ? p.topk : 1;
    const int pair0 = item * nslot;

    unsigned char *xs = smem;                            // [nslot][K] e4m3
    float *s_rsc = (float *)(smem + nslot * K);          // [16] row scales
    float *s_y = s_rsc + 16;                             // [nslot or kWaves][16] results

    int idv = -1;   // expert of every slot, lane i: slot i
    TokenLogits<kMaxPerLane> routed;   // of the workgroup that writes its token's ids and weights
    bool writes = false;
    if (kSilu && p.logits) {
        const int token = item / p.topk, slot = item - token * p.topk;
        TokenLogits<kMaxPerLane> l(p.logits + (int64_t)token * p.E, p.E);
        routed = l;
        writes = slice == 0 && slot == 0 && wave == kWaves - 1;
        idv = l.expert((uint32_t)__builtin_amdgcn_readlane((int)l.select(slot + 1), slot));
    } else if (lane < nslot) idv = p.ids[pair0 + lane];
    // rows to quantize: wave, wave + kWaves, ...; lane L holds the chunks L, L + 64, ... of eight values
    const int n16 = K / 8;
    const bool same_row = kComb && p.x_per_token;
    const int64_t xrow0 = p.x_per_token ? item / (kComb ? 1 : p.topk) : pair0;
    const int n_rows = same_row ? 1 : nslot;             // distinct rows
    auto load_row = [&](int r, u32x4 (&v)[8]) {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int ch = lane + 64 * u;
            v[u] = u32x4{0, 0, 0, 0};
            if (ch < n16) v[u] = *(const u32x4 *)(p.x + (xrow0 + r) * K + ch * 8);
        }
    };
    auto quantize_row = [&](int r, const u32x4 (&v)[8]) {
        float am = 0.f;
#pragma unroll
        for (int u = 0; u < 8; ++u) am = absmax_bf16x8(v[u], am);
        am = wave_max(am);
        const float sxr = am / 448.0f;
        const RowScale rs(sxr);
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int ch = lane + 64 * u;
            if (ch < n16) *(u32x2 *)(xs + r * K + ch * 8) = e4m3_quantize_bf16x8(rs, v[u]);
        }
        if (lane == 0) s_rsc[r] = sxr;
    };
    u32x4 v0[8];
    if (wave < n_rows) load_row(wave, v0);
    if (!kComb) {
        const int e = __builtin_amdgcn_readfirstlane(idv);
        if (e < 0 || e >= p.E) return;   // the row stays unwritten
    }
    idv = (idv < 0 || idv >= p.E) ? -1 : idv;

    // weight rows of tile w of this workgroup
    const int tiles = kComb ? 1 : kWaves;
    auto tile_row0 = [&](int w) -> int {
        if (kSilu) return (w & 1 ? N / 2 : 0) + (slice * (tiles / 2) + (w >> 1)) * 16;
        return (slice * tiles + w) * 16;
    };
    struct Slot {
        u32x4 w[kH];
    };
    Slot ring[R];
    const uint32_t *src = nullptr;
    float sw = 0.f;
    auto fill = [&](Slot &dst, int g) {
#pragma unroll
        for (int i = 0; i < kH; ++i) dst.w[i] = *(const u32x4 *)(src + min(g, G - 1) * (16 * kH) + i * 4);
    };
    const int my_row0 = tile_row0(kComb ? 0 : wave);
    const bool busy = kSilu ? (slice * (tiles / 2) + (wave >> 1)) * 16 < N / 2 : my_row0 < N;
    auto start = [&](int slot) {   // request the first R steps of the tile for this slot's expert
        const int e = max(0, __builtin_amdgcn_readlane(idv, slot));
        const int64_t row = (int64_t)e * N + my_row0 + c;
        src = p.codes + row * words_per_row + q * (4 * kH);
#pragma unroll
        for (int r = 0; r < R; ++r) fill(ring[r], r);
        sw = p.scales[row];
    };
    if (busy && wave < (kComb ? nslot : kWaves)) start(kComb ? wave : 0);
    if (kSilu && writes) {   // under the weights' way
        const int64_t o = (int64_t)(item / p.topk) * p.topk;
        route_token<kMaxPerLane>(routed, p.E, p.topk, p.renorm, p.ids_out + o, p.w_out + o);
    }

    if (wave < n_rows) quantize_row(wave, v0);
    for (int r = wave + kWaves; r < n_rows; r += kWaves) {
        load_row(r, v0);
        quantize_row(r, v0);
    }
    lds_barrier();

    for (int slot = kComb ? wave : 0; slot < (kComb ? nslot : 1) && busy; slot += kWaves) {
        if (kComb && slot != wave) start(slot);
        const int xr = same_row ? 0 : slot;
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        for (int g0 = 0; g0 < G; g0 += R) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int g = g0 + r;
                if (g < G) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        long b;
                        if (W4) {
                            const u32x2 e2 = widen_e2m1_word(ring[r].w[0][j]);
                            b = (long)(((uint64_t)e2[1] << 32) | e2[0]);
                        } else {
                            const u32x4 w = ring[r].w[(j >> 1) % kH];
                            b = (long)(((uint64_t)w[(j & 1) * 2 + 1] << 32) | w[(j & 1) * 2]);
                        }
                        const long a = *(const long *)(xs + xr * K + g * 128 + q * 32 + j * 8);   // sixteen copies of the row
                        acc = __builtin_amdgcn_mfma_f32_16x16x32_fp8_fp8(a, b, acc, 0, 0, 0);
                    }
                    fill(ring[r], g + R);
                }
            }
        }
        // lane (c, q), register i: row 4 q + i of sixteen equal ones, column c
        const float v = acc[0] * (s_rsc[xr] * sw);
        if (q == 0) s_y[(kComb ? slot : wave) * 16 + c] = (kComb && __builtin_amdgcn_readlane(idv, slot) < 0) ? 0.f : v;
    }
    const float wl = kComb && lane < nslot ? p.combine_w[pair0 + lane] : 0.f;
    lds_barrier();
    if (kSilu) {
        const int pr = tid >> 4, col = (slice * (tiles / 2) + pr) * 16 + c;   // gate tile 2 pr, up tile 2 pr + 1
        if (tid < tiles / 2 * 16 && col < N / 2)
            ((uint16_t *)p.out)[(int64_t)pair0 * (N / 2) + col] = f32_to_bf16_hw(silu_mul_f32(s_y[2 * pr * 16 + c], s_y[(2 * pr + 1) * 16 + c]));
    } else if (!kComb) {
        const int col = slice * tiles * 16 + tid;
        if (tid < tiles * 16 && col < N) {
            const int64_t o = (int64_t)pair0 * N + col;
            if (p.out_f32) ((float *)p.out)[o] = s_y[tid];
            else ((uint16_t *)p.out)[o] = f32_to_bf16_hw(s_y[tid]);
        }
    } else if (wave == 0) {
        float y = 0.f;
        for (int s = 0; s < nslot; ++s)
            y = fmaf(__uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(wl), s)), s_y[s * 16 + c], y);
        if (q == 0) {
            const int64_t o = (int64_t)item * N + slice * 16 + c;
            if (p.out_f32) ((float *)p.out)[o] = y;
            else ((uint16_t *)p.out)[o] = (uint16_t)f32_to_bf16_bits(y);
        }
    }
}

// Where the line lies (the shapes of the int4 kernel's comment, layer): 5 tokens = 40 pairs FP8 55 us here against 62 on
// the streaming kernel, FP4 30 against 46; 8 tokens 75 against 66, 43 against 47.  Below that the estimated times decide: the
// combine keeps a wavefront of eight busy per slot, so with few slots it loses early (128 experts, 2048 x 768, top-1 and 64
// tokens: FP8 2.8 times the streaming kernel's time, FP4 4 times), and with few experts both epilogues do.
constexpr int kSmallPairs = 64;

}  // namespace

bool qgemm_small_fp8_supported(int N, int K, int T, int topk, int epilogue)
{
    if ((int64_t)T * topk > kSmallPairs || N % 32 != 0 || K % kGroup != 0 || K > 4096) return false;
    return epilogue != QARL_EPI_COMBINE || topk <= 16;   // row scales and results of 16 slots
}

// See qgemm_small_w4_us; 19 500 calls, as many on the streaming kernel with its ring in LDS: off by 5 to 11 %.  By these estimates 5 % (FP4 2 %) of
// the calls run on the kernel that is slower by more than 5 %, and the mean call takes 0.8 % (0.3 %) more than on the faster of the two; by
// those for the register ring it was 16 % (8 %) and 4.4 % (1.7 %).  Combine: a round of 256 workgroups takes its slots' rows and one tile (a second one beyond 8 slots).
double qgemm_small_fp8_us(int fmt, int N, int K, int T, int topk, int epilogue)
{
    const bool w4 = fmt == QARL_FP4_E2M1_CH;
    const int G = K / kGroup, M = T * topk;
    if (epilogue == QARL_EPI_COMBINE) {
        const int rounds = (T * (N / 16) + 255) / 256, more = topk > 8;
        return w4 ? 2.34 + rounds * (0.49 + 0.183 * topk + 0.069 * G + 0.024 * topk * G + more * (0.82 + 0.122 * G))
                  : 1.38 + rounds * (1.03 + 0.455 * topk + 0.073 * G + 0.052 * topk * G + more * (0.54 + 0.147 * G));
    }
    const double wgs = M * ((N / 16 + 3) / 4) / 512.;
    return w4 ? 3.28 + 0.136 * G + wgs * (1.36 + 0.233 * G) : 3.72 + 0.205 * G + wgs * (3.5 + 0.41 * G);
}

int launch_qgemm_small_fp8(const GemmArgs &a, const float *combine_w, hipStream_t s)
{
    const int epi = combine_w ? (int)QARL_EPI_COMBINE : a.epilogue;
    SmallFp8Params p;
    p.codes = (const uint32_t *)a.codes;
    p.scales = (const float *)a.scales;
    p.x = (const uint16_t *)a.x;
    p.ids = a.ids;
    p.combine_w = combine_w;
    p.out = a.out;
    p.E = a.E;
    p.N = a.N;
    p.K = a.K;
    p.out_f32 = a.out_f32;
    p.topk = a.topk;
    p.x_per_token = a.x_per_token;
    p.logits = (const uint16_t *)a.logits;
    p.ids_out = a.ids_out;
    p.w_out = a.w_out;
    p.renorm = a.renorm;
    const int slots = epi == QARL_EPI_COMBINE ? a.topk : 1;
    p.n_slices = epi == QARL_EPI_COMBINE ? a.N / 16 : (a.N / 16 + 3) / 4;
    const size_t lds = (size_t)slots * a.K + 64 + 16 * 16 * 4;
    const dim3 grid((unsigned)(a.M / slots * p.n_slices)), block(epi == QARL_EPI_COMBINE ? 512 : 256);
    static LdsLimitOnce once[2];
    auto go = [&](auto kern, int i) -> int {
        if (lds > 64 * 1024)   // combine of 16 slots at K = 4096
            if (int rc = raise_lds_limit((const void *)kern, once[i], "hipFuncSetAttribute(small fp8)")) return rc;
        kern<<<grid, block, lds, s>>>(p);
        return check_hip(hipGetLastError(), "qgemm_small_fp8_kernel");
    };
    const bool w4 = a.fmt == QARL_FP4_E2M1_CH;
    if (epi == QARL_EPI_SILU_MUL)
        return w4 ? go(qgemm_small_fp8_kernel<QARL_EPI_SILU_MUL, true>, 0) : go(qgemm_small_fp8_kernel<QARL_EPI_SILU_MUL, false>, 0);
    if (epi == QARL_EPI_COMBINE)
        return w4 ? go(qgemm_small_fp8_kernel<QARL_EPI_COMBINE, true>, 0) : go(qgemm_small_fp8_kernel<QARL_EPI_COMBINE, false>, 1);
    return w4 ? go(qgemm_small_fp8_kernel<QARL_EPI_NONE, true>, 0) : go(qgemm_small_fp8_kernel<QARL_EPI_NONE, false>, 0);
}

}  // namespace qarl
