// LM head fused with the per-token log-prob: logits z = inv_T * h W^T are formed tile by tile
// in fp32 MFMA accumulators and reduced on the spot to (max, sum of exp(z - max)) per token and
// 256-row block of the vocabulary; a second small kernel merges the blocks and subtracts from the
// target logit, which a third one computes as a plain dot product:
//     logprob = z_target - (m + log sum).
// The [T][V] logits never reach memory.  This is the learner-forward half of the comparison in
// eq. (3).
//
// The big kernel is a dense bf16 contraction, D^T = W_tile (256 vocab rows) x h_tile^T (256 tokens):
// vocabulary rows are the MFMA row operand, so that a lane ends up with 64 logits of ONE token per
// token tile and the max / sum-exp reduction runs down its own registers; only the two 32-lane halves
// and the two wavefronts that share a token meet through a shuffle and LDS.  Both operands reach LDS
// by asynchronous global -> LDS copies (no staging registers), two 64-k stages deep; 16-byte chunks of
// a row are XOR-swizzled with the row index so that the copies (8 rows x 128 bytes per wavefront
// instruction, coalesced) and the operand reads (32 rows, one chunk) are both free of bank conflicts.
// Operand reads run one 16-k slice ahead of the MFMAs, across the stage barrier as well.
#include "common.hpp"
#include <type_traits>

namespace qarl {

constexpr int kLThreads = 512;
constexpr int kLTile = 256;                 // vocabulary rows and tokens per workgroup
constexpr int kLKS = 64;                    // k per stage
constexpr int kLRowB = kLKS * 2;            // bytes per tile row and stage
constexpr int kLTileB = kLTile * kLRowB;    // one operand tile of one stage
constexpr int kLStageB = 2 * kLTileB;       // W tile, then h tile
constexpr int kLLds = 2 * kLStageB;         // two stages
constexpr int kLGroupM = 8;                 // token tiles of the workgroups that run together on an XCD, at most

struct LogprobParams {
    const uint16_t *h;
    const uint16_t *w;
    float *pmax, *psum;  // [n_blocks][T]
    int T, H, V, n_blocks, m_tiles, n_mgroups, group_m, per_xcd;
    float inv_temp;
};

__global__ __launch_bounds__(kLThreads, 2) void lmhead_lse_kernel(LogprobParams p)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 2, wt = wave & 3;   // 128 vocabulary rows x 64 tokens per wavefront
    const int c = lane & 31, h = lane >> 5;

    // Consecutive workgroup ids go round-robin over the 8 XCDs; every XCD takes a contiguous eighth of the tiles, in
    // the order (group of token tiles, vocabulary tile, token tile of the group).  The 32 workgroups that run together on
    // one XCD (one per CU) so cover a block of group_m token tiles x 32 / group_m vocabulary tiles (8 x 4 where there
    // are that many token tiles), and its L2 fetches 12 operand tiles for 32 output tiles.  No workgroup is without
    // a tile (but for the last few): ids go round-robin over the shader engines of an XCD too, whether they have work
    // or not, and a regular pattern of empty ones leaves engines idle (256 tokens on places for 2048, 151936 x 2048:
    // 500 us; so: 210; 2300 tokens, nine tiles on places for sixteen, 1760 us; in groups of five and four: 1160).
    const int tile = (blockIdx.x & 7) * p.per_xcd + (blockIdx.x >> 3);
    if (tile >= p.m_tiles * p.n_blocks) return;
    const int mg = min(tile / (p.group_m * p.n_blocks), p.n_mgroups - 1);
    const int in_group = tile - mg * p.group_m * p.n_blocks;
    const int gm = min(p.group_m, p.m_tiles - mg * p.group_m);   // the last group may be smaller
    const int mt = mg * p.group_m + in_group % gm, nb = in_group / gm;

    const int T = p.T, H = p.H, V = p.V;
    const int v0 = nb * kLTile, t0 = mt * kLTile;

    // ---- copies: a wavefront instruction moves 8 rows x 128 bytes; this wavefront owns rows
    // [32 wave, 32 wave + 32) of both tiles.  Chunk q of row r sits at r * 128 + (q ^ ((r >> 1) & 7)) * 16.
    uint32_t woff[4], hoff[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r = wave * 32 + i * 8 + (lane >> 3);
        const int q = (lane & 7) ^ ((r >> 1) & 7);
        woff[i] = (uint32_t)min(r, V - 1 - v0) * (uint32_t)(H * 2) + q * 16;   // rows past V or T read the last
        hoff[i] = (uint32_t)min(r, T - 1 - t0) * (uint32_t)(H * 2) + q * 16;   // valid row: never used
    }
    const unsigned char *wbase = (const unsigned char *)p.w + (int64_t)v0 * H * 2;
    const unsigned char *hbase = (const unsigned char *)p.h + (int64_t)t0 * H * 2;
    const int stages = H / kLKS;
    // copy i of the wavefront's eight per stage (four W row groups, then four h row groups)
    auto copy_one = [&](int ks, int buf, int i) {
        unsigned char *dst = smem + buf * kLStageB + wave * 32 * kLRowB;
        if (i < 4) copy16_to_lds(wbase + (int64_t)ks * kLRowB + woff[i], dst + i * 8 * kLRowB);
        else copy16_to_lds(hbase + (int64_t)ks * kLRowB + hoff[i - 4], dst + kLTileB + (i - 4) * 8 * kLRowB);
    };
    auto copy_stage = [&](int ks, int buf) {
#pragma unroll
        for (int i = 0; i < 8; ++i) copy_one(ks, buf, i);
    };

    // ---- operand reads: lane (c,h) takes row c of a 32-row tile, k in [16 j + 8 h, +8) = chunk 2j + h
    int aoff[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) aoff[j] = c * kLRowB + (((2 * j + h) ^ ((c >> 1) & 7)) * 16);
    const int a_wave = wm * 128 * kLRowB, b_wave = kLTileB + wt * 64 * kLRowB;
    struct Frags {
        bf16x8 a[4], b[2];
    };
    f32x16 acc[4][2];
#pragma unroll
    for (int ms = 0; ms < 4; ++ms)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[ms][nt][i] = 0.f;
    auto mfma8 = [&](const Frags &f) {
#pragma unroll
        for (int ms = 0; ms < 4; ++ms)
#pragma unroll
            for (int nt = 0; nt < 2; ++nt)
                acc[ms][nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[ms], f.b[nt], acc[ms][nt], 0, 0, 0);
    };
    // Slice j of a stage, in a fixed issue order: the eight MFMAs on `cur`; behind each of the first six, one of the
    // six operand reads of `nxt` (an LDS read every 32 cycles instead of six at once: 3 % faster than all six
    // behind the first MFMA); in slices 0 and 1, behind every second MFMA, one of the next stage's eight copies.
    // Measured at 16384 x 151936 x 2048: all eight at the top of the stage 9.0 ms (a wavefront that waits for room
    // in the memory pipeline is kept from its matrix instructions), two per slice 8.45, three-three-two 8.07,
    // four-four 7.86 (the later a copy goes out, the less of its latency the rest of the stage covers), one behind
    // each MFMA of slice 0 7.99.
    auto slice = [&](const Frags &cur, Frags &nxt, int ks, int j, auto more_t) {
        const int buf = ks & 1;
        const unsigned char *base = smem + buf * kLStageB + aoff[j];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int ms = i >> 1, nt = i & 1;
            acc[ms][nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(cur.a[ms], cur.b[nt], acc[ms][nt], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            if (i < 4) nxt.a[i] = *(const bf16x8 *)(base + a_wave + i * 32 * kLRowB);
            else if (i < 6) nxt.b[i - 4] = *(const bf16x8 *)(base + b_wave + (i - 4) * 32 * kLRowB);
            if (decltype(more_t)::value && j < 2 && (i & 1)) copy_one(ks + 1, buf ^ 1, 4 * j + (i >> 1));
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    auto stage_barrier = [&]() {
        // own copies landed, own operand reads done; then everybody's
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    };

    // Rotated loop: the MFMAs of a stage's last slice run in the next trip, behind the stage barrier and
    // under the first operand reads of the next stage, so no operand read is outstanding at the back edge
    // and every wait inside the trip counts exactly the reads it needs.
    Frags last, f0, f1, f2, f3;
#pragma unroll
    for (int i = 0; i < 4; ++i) last.a[i] = bf16x8{0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < 2; ++i) last.b[i] = bf16x8{0, 0, 0, 0, 0, 0, 0, 0};
    copy_stage(0, 0);
    stage_barrier();
    // One stage; the last has no copies to issue, so the loop's last trip is peeled.
    auto stage = [&](int ks, auto more_t) {
        slice(last, f0, ks, 0, more_t);
        slice(f0, f1, ks, 1, more_t);
        slice(f1, f2, ks, 2, more_t);
        slice(f2, f3, ks, 3, more_t);
        stage_barrier();
        last = f3;
    };
    for (int ks = 0; ks + 1 < stages; ++ks) stage(ks, std::true_type{});
    stage(stages - 1, std::false_type{});
    mfma8(last);

    // ---- per token: max and sum of exp over this wavefront's 128 vocabulary rows.
    // lane (c,h), register i of acc[ms][nt] -> vocabulary row v0 + 128 wm + 32 ms + 8 (i/4) + 4 h + i%4,
    // token t0 + 64 wt + 32 nt + c.  exp(inv_T (a - m)) = exp2(k a - k m), k = inv_T log2 e > 0.
    float *s_m = (float *)smem, *s_s = s_m + 2 * kLTile;   // [wm][token] (the tiles are dead by now)
    const float k2 = p.inv_temp * 1.44269504088896340736f;
    const int vrow_lane = v0 + wm * 128 + 4 * h;
    const bool ragged = v0 + kLTile > V;
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) {
        if (ragged) {
#pragma unroll
            for (int ms = 0; ms < 4; ++ms)
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    if (vrow_lane + ms * 32 + 8 * (i >> 2) + (i & 3) >= V) acc[ms][nt][i] = -INFINITY;
        }
        float m = -INFINITY;
#pragma unroll
        for (int ms = 0; ms < 4; ++ms)
#pragma unroll
            for (int i = 0; i < 16; ++i) m = fmaxf(m, acc[ms][nt][i]);
        m = fmaxf(m, __shfl_xor(m, 32, 64));   // the other 64 rows of this token
        float s = 0.f;
        if (m > -INFINITY) {
            const float mk = m * k2;
#pragma unroll
            for (int ms = 0; ms < 4; ++ms)
#pragma unroll
                for (int i = 0; i < 16; ++i) s += __builtin_amdgcn_exp2f(fmaf(acc[ms][nt][i], k2, -mk));
        }
        s += __shfl_xor(s, 32, 64);
        if (h == 0) {
            s_m[wm * kLTile + wt * 64 + nt * 32 + c] = m;
            s_s[wm * kLTile + wt * 64 + nt * 32 + c] = s;
        }
    }
    lds_barrier();
    if (tid < kLTile && t0 + tid < T) {
        const float m0 = s_m[tid], m1 = s_m[kLTile + tid];
        const float m = fmaxf(m0, m1);
        float s = 0.f;
        if (m0 > -INFINITY) s += s_s[tid] * __builtin_amdgcn_exp2f((m0 - m) * k2);
        if (m1 > -INFINITY) s += s_s[kLTile + tid] * __builtin_amdgcn_exp2f((m1 - m) * k2);
        p.pmax[(int64_t)nb * T + t0 + tid] = m * p.inv_temp;
        p.psum[(int64_t)nb * T + t0 + tid] = s;
    }
}

// <a, b> over K bf16 elements in fp32 by one wavefront (K % 8 == 0).
__device__ __forceinline__ float row_dot(const uint16_t *a, const uint16_t *b, int K, int lane)
{
    const u32x4 *ar = (const u32x4 *)a, *br = (const u32x4 *)b;
    float s = 0.f;
    for (int q = lane; q < K / 8; q += 64) {
        const u32x4 va = ar[q], vb = br[q];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            s = fmaf(__uint_as_float(va[i] << 16), __uint_as_float(vb[i] << 16), s);
            s = fmaf(__uint_as_float(va[i] & 0xffff0000u), __uint_as_float(vb[i] & 0xffff0000u), s);
        }
    }
    return wave_sum(s);
}

// Target logit of each token: inv_T * <h_t, w_{y_t}> in fp32, one wavefront per token.  A target outside
// [0, V) yields NaN.
__global__ __launch_bounds__(256) void target_logit_kernel(const uint16_t *__restrict__ hmat,
                                                           const uint16_t *__restrict__ w,
                                                           const int32_t *__restrict__ target, int T, int H, int V,
                                                           float inv_temp, float *__restrict__ tgt)
{
    const int t = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (t >= T) return;
    const int y = target[t];
    if (y < 0 || y >= V) {
        if (lane == 0) tgt[t] = __uint_as_float(0x7fc00000u);
        return;
    }
    const float s = row_dot(hmat + (int64_t)t * H, w + (int64_t)y * H, H, lane);
    if (lane == 0) tgt[t] = s * inv_temp;
}

// Merge the per-block partials of one token and emit the log-prob.  16 tokens per workgroup; sixteen
// threads per token each fold every sixteenth block into a running (max, sum) (a chain of n_blocks / 16
// dependent steps: with four threads per token the launch took 88 us at 594 blocks), and the sixteen meet in
// LDS in a fixed order, so the result does not depend on scheduling.
constexpr int kFinTokens = 16, kFinSlices = 16;
__global__ __launch_bounds__(256) void lse_finalize_kernel(const float *__restrict__ pmax,
                                                           const float *__restrict__ psum,
                                                           const float *__restrict__ tgt, int T, int n_blocks,
                                                           float *__restrict__ logprob)
{
    __shared__ float s_m[kFinSlices][kFinTokens], s_s[kFinSlices][kFinTokens];
    const int tl = threadIdx.x % kFinTokens, slice = threadIdx.x / kFinTokens;
    const int t = blockIdx.x * kFinTokens + tl;
    float m = -INFINITY, s = 0.f;
    if (t < T) {
        for (int b = slice; b < n_blocks; b += kFinSlices) {
            const float mb = pmax[(int64_t)b * T + t], sb = psum[(int64_t)b * T + t];
            if (mb > m) {
                s = s * expf(m - mb) + sb;   // exp(-inf) = 0 on the first block
                m = mb;
            } else if (mb > -INFINITY) {
                s += sb * expf(mb - m);
            }
        }
    }
    s_m[slice][tl] = m;
    s_s[slice][tl] = s;
    __syncthreads();
    if (slice == 0 && t < T) {
        float mm = -INFINITY;
#pragma unroll
        for (int q = 0; q < kFinSlices; ++q) mm = fmaxf(mm, s_m[q][tl]);
        double ss = 0.0;
#pragma unroll
        for (int q = 0; q < kFinSlices; ++q)
            if (s_m[q][tl] > -INFINITY) ss += (double)s_s[q][tl] * (double)expf(s_m[q][tl] - mm);
        logprob[t] = tgt[t] - (mm + (float)log(ss));
    }
}

// ---- few tokens (a decode step; at most kSMaxTok): the vocabulary matrix is read once, and that is all the time
// there is.  A workgroup owns a contiguous range of vocabulary rows and walks it in tiles of `rows` <= 256 rows x kTok
// tokens; W rows and h rows reach LDS by the same asynchronous copies and swizzle as above, in a ring of kSBufs 64-k
// stages that runs on across the tiles: two or three stages (50-75 KB of W per CU) are in flight at any time, with
// one barrier per stage and a counted wait for the oldest.  The h rows are re-read from L2 once per tile
// (kTok / rows of the W bytes).  Copies of rows past T are not issued: what the LDS holds there only reaches columns
// that no one reads.  The running (max, sum) of the workgroup's rows stays in LDS over its tiles: one partial per
// token and workgroup, so the merge is one wavefront per token, which computes the target logit as well.
// Operand reads run one slice ahead of the matrix instructions, across the stage barrier: 128 tokens 137-140 -> 131 us,
// 61 tokens of a 32003-row vocabulary 28.9 -> 27.0.
// 151936 x 2048, whole call: 1 token 456 -> 99 us (6.3 TB/s), 61 tokens 484 -> 103 us, 128 tokens 497 -> 130 us (the rows of
// h, once per tile, are two thirds of the W bytes there: 8.4 TB/s of copies).  Beyond that the 256 x 256 tiles, which take
// 206-209 us for 129 to 256 tokens, are as good: two 128-token tiles here took 220-230, tiles of 120 rows x 256 tokens
// 200-219 (32003 rows 49-50 -> 44-47, 65000 x 1024 42-46 -> 46-48).
constexpr int kSWaves = 8, kSMaxTok = 128;

struct LogprobStreamParams {
    const uint16_t *h;
    const uint16_t *w;
    float *pmax, *psum;  // [T][n_ranges]
    int T, H, V;
    int n_ranges;        // ranges of vocabulary rows
    int rows8;           // 8-row units per tile, at most 32
    int passes;          // tiles per range
    float inv_temp;
};

// s_waitcnt vmcnt(n) for a wave-uniform n the compiler does not know (0 for n beyond the table: waits for more)
__device__ __forceinline__ void wait_vmcnt_uniform(int n)
{
    switch (n) {
    case 1: asm volatile("s_waitcnt vmcnt(1)" ::: "memory"); break;
    case 2: asm volatile("s_waitcnt vmcnt(2)" ::: "memory"); break;
    case 3: asm volatile("s_waitcnt vmcnt(3)" ::: "memory"); break;
    case 4: asm volatile("s_waitcnt vmcnt(4)" ::: "memory"); break;
    case 5: asm volatile("s_waitcnt vmcnt(5)" ::: "memory"); break;
    case 6: asm volatile("s_waitcnt vmcnt(6)" ::: "memory"); break;
    case 8: asm volatile("s_waitcnt vmcnt(8)" ::: "memory"); break;
    case 10: asm volatile("s_waitcnt vmcnt(10)" ::: "memory"); break;
    default: asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); break;
    }
}

template <int kTok, int kSBufs>
__global__ __launch_bounds__(64 * kSWaves, 2) void lmhead_stream_kernel(LogprobStreamParams p)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    constexpr int WT = kTok > 64 ? 2 : 1;            // wavefronts along the tokens
    constexpr int WM = kSWaves / WT;                 // and along the rows
    constexpr int MS = WT, NT = kTok / 32 / WT;      // 32-row and 32-token MFMA tiles of a wavefront
    constexpr int kHCopies = kTok > 64 ? kTok / 64 : 1;   // h copies per wavefront and stage (at most)
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WT, wt = wave % WT;
    const int c = lane & 31, h = lane >> 5;
    const int H = p.H, V = p.V, rows = p.rows8 * 8;
    const int stage_b = (rows + kTok) * kLRowB;
    // (max, sum) of each wavefront row group in the current tile, then the workgroup's running pair
    float *s_m = (float *)smem, *s_s = s_m + WM * kTok, *s_run = s_s + WM * kTok;
    unsigned char *ring = smem + (2 * WM + 2) * kTok * 4;

    const int range = blockIdx.x, T = p.T;
    const int64_t first = (int64_t)range * p.passes * rows;
    if (tid < kTok) {
        s_run[tid] = -INFINITY;
        s_run[kTok + tid] = 0.f;
    }
    // tiles of this workgroup that hold rows of the vocabulary
    const int my_rows = (int)max((int64_t)0, min((int64_t)V - first, (int64_t)p.passes * rows));
    const int my_tiles = (my_rows + rows - 1) / rows;
    const int stages = H / kLKS, total = my_tiles * stages;

    // this wavefront's copies of a stage: 8-row units wave, wave + 8, ... of the W tile, then of the h tile
    const int nw = (p.rows8 - wave + kSWaves - 1) / kSWaves;                   // wave-uniform, 0..4
    const int nh = max(0, ((T + 7) / 8 - wave + kSWaves - 1) / kSWaves);       // 0..kHCopies
    const int n_copies = nw + nh;
    uint32_t hoff[kHCopies];
#pragma unroll
    for (int i = 0; i < kHCopies; ++i) {
        const int r = (wave + i * kSWaves) * 8 + (lane >> 3);
        hoff[i] = (uint32_t)min(r, T - 1) * (uint32_t)(H * 2) + (((lane & 7) ^ ((r >> 1) & 7)) * 16);
    }
    const unsigned char *hbase = (const unsigned char *)p.h;
    uint32_t woff[4];
    const unsigned char *wbase = nullptr;
    auto set_tile = [&](int tile) {
        const int64_t v0 = first + (int64_t)tile * rows;
        wbase = (const unsigned char *)p.w + v0 * H * 2;
        const int last = (int)min((int64_t)V - 1 - v0, (int64_t)(rows - 1));   // rows past V read the last one: never used
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int r = (wave + i * kSWaves) * 8 + (lane >> 3);
            woff[i] = (uint32_t)min(r, last) * (uint32_t)(H * 2) + (((lane & 7) ^ ((r >> 1) & 7)) * 16);
        }
    };
    // The next stage to request.  The tiles start their k range at different places: rows lie H * 2 bytes apart, and
    // workgroups that all read the same k of their rows at the same time meet on a fraction of the memory channels
    // (151936 x 2048, 61 tokens: 135 us with one starting point, 104 us with these).
    int c_tile = 0, c_ks = 0, k_at = (range / 8) % stages;
    auto copy_one = [&](int buf, int i) {   // i < 4: W, else h
        unsigned char *dst = ring + buf * stage_b;
        if (i < 4) {
            if (i < nw)   // nontemporal: read once (temporal: 117 us)
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(wbase + k_at * kLRowB + woff[i]),
                                                 (__attribute__((address_space(3))) void *)(dst + (wave + i * kSWaves) * 8 * kLRowB),
                                                 16, 0, 2);
        } else if (i - 4 < nh) {
            copy16_to_lds(hbase + k_at * kLRowB + hoff[i - 4], dst + rows * kLRowB + (wave + (i - 4) * kSWaves) * 8 * kLRowB);
        }
    };
    auto advance = [&]() {
        k_at = k_at + 1 == stages ? 0 : k_at + 1;
        if (++c_ks == stages) {
            c_ks = 0;
            ++c_tile;
        }
    };
    auto copy_stage = [&](int buf) {
        if (c_ks == 0) set_tile(c_tile);
#pragma unroll
        for (int i = 0; i < 4 + kHCopies; ++i) copy_one(buf, i);
        advance();
    };

    const bool busy = wm * MS * 32 < rows;
    int aoff[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) aoff[j] = c * kLRowB + (((2 * j + h) ^ ((c >> 1) & 7)) * 16);
    f32x16 acc[MS][NT];
    auto clear = [&]() {
#pragma unroll
        for (int ms = 0; ms < MS; ++ms)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[ms][nt][i] = 0.f;
    };
    clear();
    const float k2 = p.inv_temp * 1.44269504088896340736f;
#pragma unroll
    for (int b = 0; b < kSBufs - 1; ++b)
        if (b < total) copy_stage(b);
    // Operands of a slice, and of the slice before: reads run one slice ahead of the matrix instructions, across the stage
    // barrier as well (a stage's last slice is multiplied behind the next barrier, under the first reads of that stage).
    struct Frags {
        bf16x8 a[MS], b[NT];
    };
    Frags f[2];
    auto clear_last = [&]() {
#pragma unroll
        for (int ms = 0; ms < MS; ++ms) f[1].a[ms] = bf16x8{0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) f[1].b[nt] = bf16x8{0, 0, 0, 0, 0, 0, 0, 0};
    };
    auto multiply = [&](const Frags &g) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int ms = 0; ms < MS; ++ms)
                acc[ms][nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(g.a[ms], g.b[nt], acc[ms][nt], 0, 0, 0);
    };
    clear_last();
    int ks = 0, tile = 0, buf = 0;
    for (int s = 0; s < total; ++s) {
        // stage s has landed: at most the copies of the kSBufs - 2 stages behind it are still on their way
        wait_vmcnt_uniform(s + kSBufs - 1 <= total ? n_copies * (kSBufs - 2) : 0);
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // everybody's; and stage s - 1 is no longer read
        const bool more = s + kSBufs - 1 < total;
        const int nbuf = buf == 0 ? kSBufs - 1 : buf - 1;
        if (more && c_ks == 0) set_tile(c_tile);
        const unsigned char *abase = ring + buf * stage_b + wm * MS * 32 * kLRowB;
        const unsigned char *bbase = ring + buf * stage_b + (rows + wt * NT * 32) * kLRowB;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (busy) {
                Frags &g = f[j & 1];
#pragma unroll
                for (int ms = 0; ms < MS; ++ms) g.a[ms] = *(const bf16x8 *)(abase + ms * 32 * kLRowB + aoff[j]);
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) g.b[nt] = *(const bf16x8 *)(bbase + nt * 32 * kLRowB + aoff[j]);
                __builtin_amdgcn_sched_barrier(0);
                multiply(f[(j & 1) ^ 1]);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (more) {   // the copies go out between the matrix instructions (128 tokens: 2-3 % faster than all in front)
#pragma unroll
                for (int i = 2 * j; i < 2 * j + 2; ++i)
                    if (i < 4 + kHCopies) copy_one(nbuf, i);
            }
        }
        if (more) advance();
        buf = buf + 1 == kSBufs ? 0 : buf + 1;
        if (++ks == stages) {
            // end of a tile: lane (c, h), register i of acc[ms][nt] -> row 32 (MS wm + ms) + 8 (i / 4) + 4 h + i % 4,
            // token 32 (NT wt + nt) + c
            if (busy) multiply(f[1]);
            clear_last();
            const int valid = (int)min((int64_t)rows, (int64_t)V - (first + (int64_t)tile * rows));
            const int row_lane = wm * MS * 32 + 4 * h;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                float m = -INFINITY;
#pragma unroll
                for (int ms = 0; ms < MS; ++ms)
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        if (row_lane + ms * 32 + 8 * (i >> 2) + (i & 3) >= valid) acc[ms][nt][i] = -INFINITY;
                        m = fmaxf(m, acc[ms][nt][i]);
                    }
                m = fmaxf(m, __shfl_xor(m, 32, 64));
                float sum = 0.f;
                if (m > -INFINITY) {
                    const float mk = m * k2;
#pragma unroll
                    for (int ms = 0; ms < MS; ++ms)
#pragma unroll
                        for (int i = 0; i < 16; ++i) sum += __builtin_amdgcn_exp2f(fmaf(acc[ms][nt][i], k2, -mk));
                }
                sum += __shfl_xor(sum, 32, 64);
                if (h == 0) {
                    s_m[wm * kTok + (wt * NT + nt) * 32 + c] = m;
                    s_s[wm * kTok + (wt * NT + nt) * 32 + c] = sum;
                }
            }
            clear();
            lds_barrier();
            // the next write of s_m / s_s lies behind at least one further stage barrier
            if (tid < kTok) {
                float m = s_run[tid];
                const float m_old = m;
#pragma unroll
                for (int w = 0; w < WM; ++w) m = fmaxf(m, s_m[w * kTok + tid]);
                float sum = m_old > -INFINITY ? s_run[kTok + tid] * __builtin_amdgcn_exp2f((m_old - m) * k2) : 0.f;
#pragma unroll
                for (int w = 0; w < WM; ++w) {
                    const float mw = s_m[w * kTok + tid];
                    if (mw > -INFINITY) sum += s_s[w * kTok + tid] * __builtin_amdgcn_exp2f((mw - m) * k2);
                }
                s_run[tid] = m;
                s_run[kTok + tid] = sum;
            }
            ks = 0;
            ++tile;
        }
    }
    if (tid < T) {   // own thread's entry
        p.pmax[(int64_t)tid * p.n_ranges + range] = s_run[tid] * p.inv_temp;
        p.psum[(int64_t)tid * p.n_ranges + range] = s_run[kTok + tid];
    }
}

// One wavefront per token: the target logit as in target_logit_kernel, then the workgroups' partials, folded by a
// wavefront reduction in a fixed order.
__global__ __launch_bounds__(64) void lse_stream_finalize_kernel(LogprobStreamParams p, const int32_t *__restrict__ target,
                                                                 float *__restrict__ logprob)
{
    const int t = blockIdx.x, lane = threadIdx.x;
    float m = -INFINITY, s = 0.f;
    for (int b = lane; b < p.n_ranges; b += 64) {
        const float mb = p.pmax[(int64_t)t * p.n_ranges + b], sb = p.psum[(int64_t)t * p.n_ranges + b];
        if (mb > m) {
            s = s * expf(m - mb) + sb;
            m = mb;
        } else if (mb > -INFINITY) {
            s += sb * expf(mb - m);
        }
    }
    const float mm = wave_max(m);
    double ss = m > -INFINITY ? (double)s * (double)expf(m - mm) : 0.0;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o, 64);
    const int y = target[t];
    float z = __uint_as_float(0x7fc00000u);
    if (y >= 0 && y < p.V) z = row_dot(p.h + (int64_t)t * p.H, p.w + (int64_t)y * p.H, p.H, lane) * p.inv_temp;
    if (lane == 0) logprob[t] = z - (mm + (float)log(ss));
}

template <int kTok, int kSBufs>
int launch_lmhead_stream(const LogprobStreamParams &p, hipStream_t s)
{
    auto kern = lmhead_stream_kernel<kTok, kSBufs>;
    static LdsLimitOnce once;
    if (int rc = raise_lds_limit((const void *)kern, once, "hipFuncSetAttribute(lmhead stream)")) return rc;
    const size_t lds = (size_t)(2 * (kTok > 64 ? 4 : 8) + 2) * kTok * 4 + (size_t)kSBufs * (p.rows8 * 8 + kTok) * kLRowB;
    kern<<<dim3((unsigned)p.n_ranges), dim3(64 * kSWaves), lds, s>>>(p);
    return check_hip(hipGetLastError(), "lmhead_stream_kernel");
}

// Ranges of the streaming path: one per CU, none below 64 rows.
static int stream_ranges(int V) { return (int)min((int64_t)256, ((int64_t)V + 63) / 64); }

int launch_logprob_stream(LogprobStreamParams p, const int32_t *target, float *logprob, void *ws, size_t ws_bytes, hipStream_t s)
{
    // a workspace of the least size holds a partial per token and tile column: 126 ranges for 32003 rows, which took
    // 31 us for one token (H = 2048) and 27 on 251
    const int64_t units = ((int64_t)p.V + 7) / 8;
    const int tok = p.T <= 32 ? 32 : p.T <= 64 ? 64 : 128;
    p.n_ranges = (int)min((int64_t)stream_ranges(p.V), (int64_t)(ws_bytes / (2 * sizeof(float) * (size_t)p.T)));
    p.passes = (int)((units + (int64_t)p.n_ranges * 32 - 1) / ((int64_t)p.n_ranges * 32));   // at most 32 units per tile
    p.rows8 = (int)((units + (int64_t)p.n_ranges * p.passes - 1) / ((int64_t)p.n_ranges * p.passes));
    p.pmax = (float *)ws;
    p.psum = p.pmax + (size_t)p.n_ranges * p.T;
    int rc;
    if (tok == 32) rc = launch_lmhead_stream<32, 4>(p, s);
    else if (tok == 64 && p.rows8 <= 30) rc = launch_lmhead_stream<64, 4>(p, s);
    else if (tok == 64) rc = launch_lmhead_stream<64, 3>(p, s);
    else rc = launch_lmhead_stream<128, 3>(p, s);
    if (rc) return rc;
    lse_stream_finalize_kernel<<<dim3((unsigned)p.T), dim3(64), 0, s>>>(p, target, logprob);
    return check_hip(hipGetLastError(), "lse_stream_finalize_kernel");
}

size_t logprob_ws_least(int T, int V) { return (2 * ((size_t)(V + kLTile - 1) / kLTile) + 1) * (size_t)T * sizeof(float); }

size_t logprob_ws_bytes(int T, int H, int V)
{
    (void)H;
    const size_t least = logprob_ws_least(T, V);
    return T <= kSMaxTok ? max(least, 2 * (size_t)stream_ranges(V) * T * sizeof(float)) : least;
}

int launch_logprob(const void *h, const void *wlm, const int32_t *target, int T, int H, int V, float inv_temp,
                   float *logprob, void *ws, size_t ws_bytes, hipStream_t s)
{
    LogprobParams p;
    p.h = (const uint16_t *)h;
    p.w = (const uint16_t *)wlm;
    p.T = T;
    p.H = H;
    p.V = V;
    p.n_blocks = (V + kLTile - 1) / kLTile;
    p.m_tiles = (T + kLTile - 1) / kLTile;
    p.n_mgroups = (p.m_tiles + kLGroupM - 1) / kLGroupM;
    p.group_m = (p.m_tiles + p.n_mgroups - 1) / p.n_mgroups;
    p.pmax = (float *)ws;
    p.psum = p.pmax + (size_t)p.n_blocks * T;
    float *tgt = p.psum + (size_t)p.n_blocks * T;
    p.inv_temp = inv_temp;
    if ((int64_t)kLTile * H * 2 >= (1LL << 31)) {
        set_error("logprob: H too large");
        return QARL_ERR_UNSUPPORTED;
    }
    // The streaming path's last kernel writes results while it still reads h, the vocabulary rows and the targets; the tiled
    // one has finished with them by then, so a caller may put logprob on top of any of them.
    const bool in_place = ranges_overlap(logprob, (size_t)T * 4, h, (size_t)T * H * 2) ||
                          ranges_overlap(logprob, (size_t)T * 4, wlm, (size_t)V * H * 2) ||
                          ranges_overlap(logprob, (size_t)T * 4, target, (size_t)T * 4);
    if (T <= kSMaxTok && !in_place) {
        LogprobStreamParams q;
        q.h = p.h;
        q.w = p.w;
        q.T = T;
        q.H = H;
        q.V = V;
        q.inv_temp = inv_temp;
        return launch_logprob_stream(q, target, logprob, ws, ws_bytes, s);
    }
    const int64_t tiles = (int64_t)p.m_tiles * p.n_blocks;
    if (tiles > 0x7ffffff0LL) {
        set_error("logprob: grid too large");
        return QARL_ERR_UNSUPPORTED;
    }
    p.per_xcd = (int)((tiles + 7) / 8);
    static LdsLimitOnce once;
    if (int rc0 = raise_lds_limit((const void *)lmhead_lse_kernel, once, "hipFuncSetAttribute(lmhead)")) return rc0;
    target_logit_kernel<<<dim3((T + 3) / 4), dim3(256), 0, s>>>(p.h, p.w, target, T, H, V, inv_temp, tgt);
    int rc = check_hip(hipGetLastError(), "target_logit_kernel");
    if (rc) return rc;
    lmhead_lse_kernel<<<dim3((unsigned)p.per_xcd * 8), dim3(kLThreads), kLLds, s>>>(p);
    rc = check_hip(hipGetLastError(), "lmhead_lse_kernel");
    if (rc) return rc;
    lse_finalize_kernel<<<dim3((T + kFinTokens - 1) / kFinTokens), dim3(kFinTokens * kFinSlices), 0, s>>>(p.pmax, p.psum, tgt, T, p.n_blocks,
                                                                                                           logprob);
    return check_hip(hipGetLastError(), "lse_finalize_kernel");
}

// ---- the library's own scratch for callers that cannot allocate.  One copy of the array exists on every GPU
// the library's code object is loaded on, at that GPU's own address.  In host code the array's NAME is only a
// handle for the symbol lookup below, never a device address: everything that touches the memory (kernel
// arguments, copies, fills) takes the pointer this function returns.
static __device__ __align__(256) unsigned char scratch[kLogprobScratchBytes];
static std::atomic<void *> g_scratch_ptr[64];   // per device, filled on the first call with that device current

int logprob_static_scratch(void **ptr)
{
    int dev = -1;
    int rc = check_hip(hipGetDevice(&dev), "hipGetDevice");
    if (rc) return rc;
    if (dev < 0 || dev >= 64) {
        set_error("logprob (library scratch): device index %d outside the table of 64", dev);
        return QARL_ERR_UNSUPPORTED;
    }
    void *p = g_scratch_ptr[dev].load(std::memory_order_acquire);
    if (!p) {
        rc = check_hip(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)), "hipGetSymbolAddress(scratch)");
        if (rc) return rc;
        if (!p) {
            set_error("logprob (library scratch): symbol lookup returned a null address");
            return QARL_ERR_HIP;
        }
        g_scratch_ptr[dev].store(p, std::memory_order_release);
    }
    *ptr = p;
    return QARL_OK;
}

}  // namespace qarl
