// Routed W4A16 / W4A8 GEMM for a handful of (token, slot) pairs: the decode step of one or a few sequences, when most
// experts have no row and those that have one have a single one.  Latency is everything there: the weights of eight
// experts are 13 MB, and the streaming kernel (a workgroup per expert and half of its rows, a wavefront per 16 KiB of
// codes) brings them in through 16 of the 256 CUs.
//
// Work layout.  The problem is split by pair (for the combine epilogue by token, all of its slots together) and by
// columns; a workgroup of eight wavefronts reads its pair's expert id itself, so there is no list of rows to build,
// and requests its first 64 KiB of weights right behind it.  The unit of work of a wavefront is a TASK: one 128-k scale
// group of one pair of 16-row weight tiles (2 KiB of codes), so the k range is spread over the wavefronts too.  A task
// leaves its 32 group sums in LDS; one thread per column folds them over the groups in ascending order.  Every value is
// formed by the operations of the streaming kernel in the same order (group sums of x by the same matrix instruction,
// the same 32x32x16 chain per group started at -1.5 * sum x, the same fold), so results equal its results bit for
// bit.  The matrix instruction multiplies 32 copies of the row: its time is hidden behind the loads.
//
// Combine epilogue: the topk slots of a token meet in one workgroup, which weights and adds them in slot order (as
// combine_kernel does) and writes the output row: no staging rows, no second launch.
#include "route_token.hpp"

namespace qarl {

namespace {

constexpr int kThreads = 512;
constexpr int kWaves = 8;

struct SmallParams {
    const uint32_t *codes;   // 1 KiB blocks [E*N/16][K/128][256 words]
    const uint16_t *scales;  // bf16 [E][N][K/128]
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
    int qx;          // W4A8: the rows go through the activation quantizer
    int n_units;     // pairs of 16-row weight tiles per expert
    int units;       // of them per workgroup
    int n_slices;    // workgroups along the units
    uint32_t g_magic;   // t / G == (t * g_magic) >> 16 for every task index
};

__host__ __device__ constexpr int x_stride(int K) { return K * 2 + 16; }

size_t small_lds_bytes(int K, int slots, int units)
{
    const size_t G = K / kGroup;
    return (size_t)slots * x_stride(K) + (slots * G + 16) * 4 + slots * G * units * 32 * 4 + (size_t)slots * units * 32 * 4;
}

template <int EPI>
__global__ __launch_bounds__(kThreads, 4) void qgemm_small_w4_kernel(SmallParams p)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    constexpr bool kSilu = (EPI == QARL_EPI_SILU_MUL), kComb = (EPI == QARL_EPI_COMBINE);
    constexpr int R = 4;   // tasks in flight per wavefront

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, tt = (lane >> 4) & 1, h = lane >> 5, m32 = lane & 31;
    const int N = p.N, K = p.K, G = K / kGroup, stride = x_stride(K);
    const int slice = blockIdx.x % p.n_slices, item = blockIdx.x / p.n_slices;   // item: pair, or token (combine)
    const int nslot = kComb ? p.topk : 1;
    const int pair0 = item * nslot;
    const int u_lo = slice * p.units, n_u = min(p.units, p.n_units - u_lo);

    unsigned char *xs = smem;                                   // [nslot][stride]
    float *sx = (float *)(smem + nslot * stride);               // [nslot][G]  -1.5 * group sums
    float *s_rsc = sx + nslot * G;                              // [16] row scales (W4A8)
    float *s_ag = s_rsc + 16;                                   // [tasks][32] group results
    float *s_y = s_ag + nslot * G * p.units * 32;               // [nslot][units * 32] (combine)

    // expert of every slot: lane i holds slot i's; an id outside [0, E) selects no expert
    int idv = -1;
    TokenLogits<kMaxPerLane> routed;   // of the workgroup that writes its token's ids and weights
    bool writes = false;
    if (kSilu && p.logits) {
        const int token = item / p.topk, slot = item - token * p.topk;
        TokenLogits<kMaxPerLane> l(p.logits + (int64_t)token * p.E, p.E);
        routed = l;
        writes = slice == 0 && slot == 0 && wave == kWaves - 1;
        idv = l.expert((uint32_t)__builtin_amdgcn_readlane((int)l.select(slot + 1), slot));
    } else if (lane < nslot) idv = p.ids[pair0 + lane];
    // token rows, 16-byte chunks: thread -> chunk tid, tid + 512, ... of the nslot rows
    const int n16 = K / 8, chunks = nslot * n16;
    const int64_t xrow0 = p.x_per_token ? item / (kComb ? 1 : p.topk) : pair0;
    const bool same_row = kComb && p.x_per_token;               // every slot reads the token's row
    const u32x4 *xsrc = (const u32x4 *)(p.x + xrow0 * K);
    constexpr int kXRegs = 4;
    u32x4 xv[kXRegs];
#pragma unroll
    for (int i = 0; i < kXRegs; ++i) {
        const int ch = tid + i * kThreads;
        xv[i] = u32x4{0, 0, 0, 0};
        if (ch < chunks) xv[i] = xsrc[same_row ? ch % n16 : ch];
    }
    if (!kComb) {
        const int e = __builtin_amdgcn_readfirstlane(idv);
        if (e < 0 || e >= p.E) return;   // the row stays unwritten
    }
    idv = (idv < 0 || idv >= p.E) ? -1 : idv;

    // ---- tasks of this wavefront: wave, wave + 8, ... in the order (slot, unit, group)
    const int n_tasks = nslot * n_u * G;
    auto tile16 = [&](int u, int t) -> int { return kSilu ? (t ? (N / 2) / 16 : 0) + u : u * 2 + t; };
    auto split = [&](int task, int &slot, int &u, int &g) {
        const int su = (int)(((uint32_t)task * p.g_magic) >> 16);
        g = task - su * G;
        slot = 0;
        u = su;
        if (kComb)
            while (u >= n_u) {
                u -= n_u;
                ++slot;
            }
    };
    struct Slot {
        u32x4 w[2];
    };
    Slot ring[R];
    auto fill = [&](Slot &dst, int task) {   // past the end: the last task again (cached)
        int slot, u, g;
        split(min(task, n_tasks - 1), slot, u, g);
        const int e = max(0, __builtin_amdgcn_readlane(idv, slot));
        const int64_t tile = (int64_t)e * (N / 16) + tile16(u_lo + u, tt);
        const uint32_t *src = p.codes + (tile * G + g) * 256 + h * 64 + c * 4;
        dst.w[0] = *(const u32x4 *)src;
        dst.w[1] = *(const u32x4 *)(src + 128);
    };
#pragma unroll
    for (int r = 0; r < R; ++r) fill(ring[r], wave + r * kWaves);
    // scales of the column this thread folds: thread -> (slot, unit, column)
    const int f_cols = n_u * 32, f_slot = kComb ? tid / f_cols : 0, f_rest = tid - f_slot * f_cols;
    const bool folds = tid < nslot * f_cols;
    uint32_t sc[8];
    const int f_e = __shfl(idv, min(f_slot, nslot - 1), 64);
    {
        const int e = folds ? max(0, f_e) : 0;
        const int fu = f_rest >> 5, col = f_rest & 31;
        const int64_t row = (int64_t)e * N + tile16(u_lo + fu, col >> 4) * 16 + (col & 15);
        const uint32_t *src = (const uint32_t *)p.scales + row * (G / 2);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            sc[i] = 0;
            if (folds && i < G / 2) sc[i] = src[i];
        }
    }

    if (kSilu && writes) {   // under the weights' way
        const int64_t o = (int64_t)(item / p.topk) * p.topk;
        route_token<kMaxPerLane>(routed, p.E, p.topk, p.renorm, p.ids_out + o, p.w_out + o);
    }

    // ---- token rows to LDS
#pragma unroll
    for (int i = 0; i < kXRegs; ++i) {
        const int ch = tid + i * kThreads;
        if (ch < chunks) {
            const int r = ch / n16, b = ch - r * n16;
            *(u32x4 *)(xs + r * stride + b * 16) = xv[i];
        }
    }
    for (int ch = tid + kXRegs * kThreads; ch < chunks; ch += kThreads) {
        const int r = ch / n16, b = ch - r * n16;
        *(u32x4 *)(xs + r * stride + b * 16) = xsrc[same_row ? b : ch];
    }
    lds_barrier();
    if (p.qx) {
        // W4A8: the activation quantizer of eq. (2), one wavefront per row, in place (the streaming kernel's steps)
        for (int r = wave; r < nslot; r += kWaves) {
            u32x4 v[4];
            float am = 0.f;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int ch = lane + 64 * u;
                v[u] = u32x4{0, 0, 0, 0};
                if (ch < n16) v[u] = *(const u32x4 *)(xs + r * stride + ch * 16);
                am = absmax_bf16x8(v[u], am);
            }
            am = wave_max(am);
            const float sxr = am / 448.0f;
            const RowScale rs(sxr);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int ch = lane + 64 * u;
                if (ch < n16) *(u32x4 *)(xs + r * stride + ch * 16) = e4m3_as_bf16x8(e4m3_quantize_bf16x8(rs, v[u]));
            }
            if (lane == 0) s_rsc[r] = sxr;
        }
        lds_barrier();
    }
    {
        // group sums, sx[slot][g] = -1.5 * sum_k x: up to 16 rows times a matrix of ones
        const u32x4 ones4 = {0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};
        const bf16x8 ones = __builtin_bit_cast(bf16x8, ones4);
        const int q = lane >> 4;
        for (int g = wave; g < G; g += kWaves) {
            f32x4 d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const bf16x8 a = *(const bf16x8 *)(xs + min(c, nslot - 1) * stride + (g * 128 + q * 32 + j * 8) * 2);
                d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, ones, d, 0, 0, 0);
            }
            if (c == 0) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (4 * q + i < nslot) sx[(4 * q + i) * G + g] = d[i] * -1.5f;
            }
        }
    }
    lds_barrier();

    for (int i0 = 0; wave + i0 * kWaves < n_tasks; i0 += R) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int task = wave + (i0 + r) * kWaves;
            if (task < n_tasks) {
                int slot, u, g;
                split(task, slot, u, g);
                const float init = sx[slot * G + g];
                f32x16 ag;
#pragma unroll
                for (int i = 0; i < 16; ++i) ag[i] = init;
                const unsigned char *xa = xs + slot * stride + (g * 128 + h * 32) * 2;
#pragma unroll
                for (int L = 0; L < 2; ++L)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const bf16x8 bw = unpack_int4_word(ring[r].w[L][j]);
                        const bf16x8 a = *(const bf16x8 *)(xa + (L * 64 + j * 8) * 2);
                        ag = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, bw, ag, 0, 0, 0);
                    }
                if (h == 0) s_ag[task * 32 + m32] = ag[0];   // every row of the tile is the same row
                fill(ring[r], task + R * kWaves);
            }
        }
    }
    lds_barrier();

    // ---- fold the groups in ascending order
    float acc = 0.f;
    if (folds && f_e >= 0) {   // a slot without an expert adds nothing
        const float *ag = s_ag + ((f_slot * n_u + (f_rest >> 5)) * G) * 32 + (f_rest & 31);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (i < G / 2) {
                acc = fmaf(16.f * __uint_as_float(sc[i] << 16), ag[(2 * i) * 32], acc);
                acc = fmaf(16.f * __uint_as_float(sc[i] & 0xffff0000u), ag[(2 * i + 1) * 32], acc);
            }
        }
        if (p.qx) acc *= s_rsc[f_slot];
    }
    if (kSilu) {
        const float other = __shfl_xor(acc, 16, 64);   // the up value of the same column
        if (folds && !(tid & 16))
            ((uint16_t *)p.out)[(int64_t)pair0 * (N / 2) + (u_lo + (f_rest >> 5)) * 16 + (f_rest & 15)] =
                f32_to_bf16_hw(silu_mul_f32(acc, other));
    } else if (!kComb) {
        if (folds) {
            const int64_t o = (int64_t)pair0 * N + u_lo * 32 + f_rest;
            if (p.out_f32) ((float *)p.out)[o] = acc;
            else ((uint16_t *)p.out)[o] = f32_to_bf16_hw(acc);
        }
    } else {
        if (folds) s_y[f_slot * f_cols + f_rest] = acc;
        const float wl = lane < nslot ? p.combine_w[pair0 + lane] : 0.f;
        lds_barrier();
        float y = 0.f;
        for (int s = 0; s < nslot; ++s) {
            const float v = tid < f_cols ? s_y[s * f_cols + tid] : 0.f;
            const float w = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(wl), s));
            y = fmaf(w, v, y);
        }
        if (tid < f_cols) {
            const int64_t o = (int64_t)item * N + u_lo * 32 + tid;
            if (p.out_f32) ((float *)p.out)[o] = y;
            else ((uint16_t *)p.out)[o] = (uint16_t)f32_to_bf16_bits(y);
        }
    }
}

// Where the line lies.  128 experts, hidden 2048, intermediate 768, top-8; layer of router, gate_up, down + combine: 8
// tokens = 64 pairs 41 us here against 58 on the streaming kernel; 12 tokens 61 against 58: by then a third of the pairs
// share their expert with another one, and every pair reads its weights by itself.  1 token: 26 against 56 us (the host
// issues three calls in 25 us; gate_up 9.5 against 30 us between events, down + combine 9.7 against 22.5).
// With few experts all pairs share them (six experts of 4096 x 2048, combine: 6 pairs 15 us here against 20 streaming, 30
// pairs 38 against 22), so up to 64 pairs the estimated times decide.
constexpr int kSmallPairs = 64;

// The workgroups of a call: pairs of 16-row weight tiles each computes (about two workgroups per CU; a thread folds one
// column of one slot), and their number along the columns.
struct SmallGrid {
    int units, n_slices;
    int64_t items;
};
SmallGrid small_grid(int N, int64_t M, int slots)
{
    SmallGrid g;
    const int n_units = N / 32;   // SILU_MUL: (N / 2) / 16
    g.items = M / slots;
    const int64_t units = (g.items * n_units + 511) / 512;
    const int max_units = kThreads / (32 * slots);
    g.units = (int)(units < 1 ? 1 : units > max_units ? max_units : units);
    g.n_slices = (n_units + g.units - 1) / g.units;
    return g;
}

}  // namespace

// Time of a call in us: start-up, a wavefront's tasks one after the other, and a share per workgroup beyond the chip's first
// 512.  This and the estimates beside it are least squares over 2000 calls per format (1 to 256 experts, N 32 to 4096, every
// K, top-1 to top-16, up to 64 pairs, all epilogues; both kernels timed, launches back to back): off by 8 % here (rms), 6 to
// 10 % for FP8 and FP4, 8 to 15 % for the streaming kernels.  A rule of pairs alone took the kernel that was slower by more
// than 5 % in an eighth of the calls, at worst 14 times slower; the estimates do in 2 %, at worst 1.3 times.
double qgemm_small_w4_us(int fmt, int N, int K, int T, int topk, int epilogue)
{
    const bool comb = epilogue == QARL_EPI_COMBINE, qx = fmt == QARL_W4A8_G128;
    const int slots = comb ? topk : 1, G = K / kGroup;
    const SmallGrid g = small_grid(N, (int64_t)T * topk, slots);
    const double wgs = (double)(g.items * g.n_slices) / 512, per_wave = (double)(slots * g.units * G) / kWaves;
    return qx ? 4.4 + 0.89 * per_wave + wgs * (1.6 + 0.4 * per_wave + 0.055 * slots * G) + (comb ? 0.35 : 0.)
              : 3.3 + 0.79 * per_wave + wgs * (1.55 + 0.49 * per_wave + 0.034 * slots * G) + (comb ? 0.3 : 0.);
}

bool qgemm_small_w4_supported(int N, int K, int T, int topk, int epilogue)
{
    if ((int64_t)T * topk > kSmallPairs || N % 32 != 0 || K % 256 != 0 || K > 2048) return false;
    return epilogue != QARL_EPI_COMBINE || topk <= 16;   // 16 rows of group sums, 512 threads for 32 columns of every slot
}

int launch_qgemm_small_w4(const GemmArgs &a, const float *combine_w, hipStream_t s)
{
    const int epi = combine_w ? (int)QARL_EPI_COMBINE : a.epilogue;
    SmallParams p;
    p.codes = (const uint32_t *)a.codes;
    p.scales = (const uint16_t *)a.scales;
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
    p.qx = a.fmt == QARL_W4A8_G128;
    p.n_units = a.N / 32;
    const int G = a.K / kGroup, slots = epi == QARL_EPI_COMBINE ? a.topk : 1;
    const SmallGrid sg = small_grid(a.N, a.M, slots);
    p.units = sg.units;
    p.n_slices = sg.n_slices;
    p.g_magic = (65536u + G - 1) / G;   // exact for task indices below 65536 / (G - 1); there are at most 16 * 16 * 16
    const size_t lds = small_lds_bytes(a.K, slots, p.units);
    const dim3 grid((unsigned)(sg.items * p.n_slices)), block(kThreads);
    static LdsLimitOnce once[3];
    auto go = [&](auto kern, int i) -> int {
        if (lds > 64 * 1024)
            if (int rc = raise_lds_limit((const void *)kern, once[i], "hipFuncSetAttribute(small w4)")) return rc;
        kern<<<grid, block, lds, s>>>(p);
        return check_hip(hipGetLastError(), "qgemm_small_w4_kernel");
    };
    if (epi == QARL_EPI_SILU_MUL) return go(qgemm_small_w4_kernel<QARL_EPI_SILU_MUL>, 0);
    if (epi == QARL_EPI_COMBINE) return go(qgemm_small_w4_kernel<QARL_EPI_COMBINE>, 1);
    return go(qgemm_small_w4_kernel<QARL_EPI_NONE>, 2);
}

}  // namespace qarl
