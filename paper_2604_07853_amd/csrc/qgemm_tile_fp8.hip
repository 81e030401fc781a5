// Grouped quantized GEMM, MFMA-tiled ("prefill" / training-forward) path for the FP8 W8A8 format:
// eq. (2) of section 2.2 with e4m3 activations (one scale per token row) and e4m3 weights (one scale
// per output channel), Y = s_x s_w (X_q W_q^T), on the same codes and scales as the streaming path.
//
// Both operands are MFMA inputs as stored, so the kernel is a plain dense contraction: a workgroup owns
// 128 token rows x 256 weight rows of one expert; its eight wavefronts (2 x 4) own 64 x 64 each as 2 x 2
// v_mfma_f32_32x32x64_f8f6f4 tiles (e4m3 x e4m3, unit block scales).  The weight rows are the MFMA's row
// operand and the tokens its column operand, so a lane ends up with four consecutive output columns of ONE
// token per register quad, and the gate and up value of a column meet in the same lane; results turn through LDS and leave
// as whole row pieces.  Token rows (gathered through row_map) and weight rows reach LDS by
// asynchronous global -> LDS copies; 16-byte chunks of a row are XOR-swizzled with the row index so that the copies
// and the operand reads (32 rows, one chunk) are free of bank conflicts.
//
// Two workgroups share a CU (66 KiB of LDS and at most 128 registers each): copies, operand reads and matrix instructions of ONE
// workgroup add up instead of overlapping, whatever the tile and the depth of its pipeline, and a third of a launch was lookups, first
// stages and epilogues; another workgroup on the same SIMDs fills all of these.  The matrix instructions run at raised wave priority
// (large calls 1-2 % faster) with the copies between them, and the first weight rows are requested before the token
// rows' ids are known (FP8 1-2 %).
//
// What bounds it: the copies (gate_up of 8192 tokens, 2.6 GB out of L2).  A copy instruction is served at the rate of a 128-byte line per two
// cycles, whether it takes the line or half of it: copies of rows of 64 bytes (64-k stages of e4m3) reach 17 TB/s out of L2 and
// copies of 128 bytes 35.  So an e4m3 stage has 128 k.  Two double-buffered stages of that size do not fit half a CU's LDS; instead
// the operands of a phase (half of the stage's weight rows) are read into registers at once, the tokens held over both phases, and the LDS
// they came from is free for the next copies: 64 KiB hold the tokens of one stage and three units of weight rows, and a copy
// has two to three phases to land.  Layers of 128 experts 2048 x 768, top-8, even / Zipf router, us, three 64-k stages -> this: 520 tokens
// 158 / 143 -> 154 / 136, 1024 182 / 179 -> 180 / 167, 3000 302 / 311 -> 279 / 285, 8192 649 / 645 -> 599 / 602, 16384 1205 / 1211 -> 1124 / 1133
// (gate_up of 8192 tokens 269 -> 228, down 235 -> 222); 64 experts 1024 x 512, top-4, 16000 tokens 296 -> 283.  The SiLU results
// through LDS in whole 256-byte pieces instead of 8 bytes per lane are 1 to 4 % of a layer of it (FP4 too).
//
// FP4 weights (W4 = true): the instruction reads e2m1 codes natively in its first
// operand (format select 4), 16 bytes per lane instead of 32.  A weight row then has 64 bytes per stage of 128 k, a workgroup two stages of
// 32 KiB, and no e4m3 copy of the weights is ever written.  (The register-held form above in whole 128-k phases: 520 to 1024 tokens 2-4 % slower,
// 3000 to 16384 level.)  The library packs the eight codes of a word as (element b, element 4 + b) in
// byte b; the instruction pairs nibble n of its first operand with byte n of the second within a group of
// 16 k, so the token bytes of every 8-byte group are put into the order 0 4 1 5 2 6 3 7 after their LDS
// read (two byte permutes per 8 bytes).  Across groups it pairs the 2 x 16 codes of first-operand lane h
// (k-half h of the 64) with bytes [16 h, 16 h + 16) of second-operand lanes 0 and 1: the token lanes
// therefore read the 16-byte chunks h and 2 + h of a half stage instead of 2 h and 2 h + 1.
#include <type_traits>

#include "common.hpp"

namespace qarl {

constexpr int kFThreads = 512;
constexpr int kFTM = 128, kFTN = 256;        // token rows, weight rows per workgroup
constexpr int kFStageK = 128;                // k per stage = bytes of a token row
constexpr int kFUnitB = 16384;               // LDS of a stage's token rows; of a unit of weight rows
constexpr int kFUnits = 3;                   // weight units in LDS (e4m3)
constexpr int kFStageB = (1 + kFUnits) * kFUnitB;
constexpr int kFLds = kFStageB + (3 * kFTM + kFTN) * 4;

struct Tile8Params {
    const unsigned char *codes;   // [E][N][K] e4m3, or [E][N][K/2] packed e2m1
    const float *scales;          // [E][N]
    const unsigned char *x;       // [x_rows][K] e4m3
    const float *x_scales;        // [x_rows]
    const int32_t *row_map;
    const int32_t *out_row_map;
    const int32_t *offsets;
    void *out;
    int E, N, K, out_f32;
    int n_blocks;   // column blocks per expert
};

// v, which the compiler takes for a new value every time: what is made from it inside a loop is made there, and takes no register
// across it.
__device__ __forceinline__ uint32_t fresh_sgpr(uint32_t v)
{
    asm volatile("" : "+s"(v));
    return v;
}

template <int EPI, bool W4>
__global__ __launch_bounds__(kFThreads, 4) void qgemm_tile_fp8_kernel(Tile8Params p)
{
    extern __shared__ __attribute__((aligned(128))) unsigned char smem[];
    constexpr bool kSilu = (EPI == QARL_EPI_SILU_MUL);
    int *s_rows = (int *)(smem + kFStageB), *s_orow = s_rows + kFTM;
    float *s_xs = (float *)(s_orow + kFTM);
    float *s_wn = s_xs + kFTM;   // [kFTN] channel scale of every weight row of the tile

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 2, wn = wave & 3;

    GroupedTile tile;
    if (!find_grouped_tile<kFTM>(p.offsets, p.E, p.n_blocks, tile)) return;
    const int e = tile.e, nb = tile.block;
    const int row0 = tile.row0, mrem = tile.rows;
    // row ids (their loads go out in front of the weight copies below)
    int xrow = 0, orow_g = -1;
    if (tid < kFTM) {
        // rows past the expert's end read the tile's first row (valid data, results never stored)
        const int i = row0 + (tid < mrem ? tid : 0);
        xrow = p.row_map ? p.row_map[i] : i;
        orow_g = tid < mrem ? (p.out_row_map ? p.out_row_map[i] : i) : -1;
    }

    const int N = p.N, K = p.K, stages = K / kFStageK;
    // Row rho (0..255) of the weight tile -> weight row of the expert.  SILU_MUL: every 32-row
    // tile holds 16 gate rows then the 16 matching up rows, so gate j and up j sit 16 lanes apart in the
    // MFMA result.  Tiles past N read the expert's first rows (valid data, results never stored).
    auto weight_row = [&](int rho) -> int {
        int n;
        bool ok;
        if (kSilu) {
            const int j = nb * (kFTN / 2) + (rho >> 5) * 16 + (rho & 15);
            n = ((rho & 16) ? N / 2 : 0) + j;
            ok = j - (rho & 15) + 16 <= N / 2;
        } else {
            n = nb * kFTN + rho;
            ok = n - (rho & 31) + 32 <= N;
        }
        return ok ? n : rho & 15;
    };

    const uint32_t rowb = (uint32_t)(W4 ? K / 2 : K);   // bytes of a weight row; an expert's stay below 2^32 (checked by the launcher)
    const unsigned char *wbase = p.codes + (int64_t)e * N * rowb;
    const float *sbase = p.scales + (int64_t)e * N;
    // A wavefront whose 64 rows lie past the expert's end only copies (layers of 128 experts, even / Zipf router, FP4: 520 tokens 116 / 98 ->
    // 112 / 97 us, 1024 136 / 134 -> 134 / 129, 3000 245 / 253 -> 240 / 244; FP8: 520 153 / 134 -> 154 / 136, 700 160 / 147 -> 165 / 146, 1024
    // 173 / 169 -> 180 / 167, 1200 187 / 182 -> 191 / 179, 1500 201 / 203 -> 198 / 203, 3000 284 / 286 -> 280 / 279, 8192 600 / 608 -> 593 / 596).
    // At every size, although FP8 loses 2 to 4 % from about 45 to 75 rows per expert under an even router: the same sizes gain 1 % under the Zipf
    // router and 2 to 4 % in layers of 64 experts (1024 x 512, top-4, 1024 tokens 50.5 / 55.5 -> 49.7 / 53.5), so no line by size serves both.
    const bool busy = wm * 64 < mrem;
    f32x16 acc[2][2];
#pragma unroll
    for (int ms = 0; ms < 2; ++ms)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[ms][nt][i] = 0.f;
    // e4m3 (or e2m1: format 4) x e4m3, no block scales
    auto mfma1 = [&](const i32x8 &w, const i32x8 &x, f32x16 &d) {
        d = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(w, x, d, W4 ? 4 : 0, 0, 0, 0, 0, 0);
    };
    auto as_operand = [](u32x4 lo, u32x4 hi) -> i32x8 {
        return i32x8{(int)lo[0], (int)lo[1], (int)lo[2], (int)lo[3], (int)hi[0], (int)hi[1], (int)hi[2], (int)hi[3]};
    };
    // the block's 256 channel scales, 4 bytes per lane (wavefronts w and w + 4 copy the same 64)
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(sbase + weight_row((wave & 3) * 64 + lane)),
                                     (__attribute__((address_space(3))) void *)(&s_wn[(wave & 3) * 64]), 4, 0, 0);
    // row ids and scales to LDS, after the first weight rows have been requested: these wait for no row id
    auto rows_to_lds = [&]() {
        if (tid < kFTM) {
            s_rows[tid] = xrow;
            s_orow[tid] = orow_g;
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(p.x_scales + xrow),
                                             (__attribute__((address_space(3))) void *)(&s_xs[wave * 64]), 4, 0, 0);
        }
        lds_barrier();
    };

    // Copies of 1 KiB.  Rows of 128 bytes: 8 per copy, chunk q of row r at r * 128 + (q ^ ((r >> 1) & 7)) * 16; rows of 64 bytes: 16 per copy,
    // chunk q at r * 64 + (q ^ ((r >> 2) & 3)) * 16.
    if constexpr (!W4) {
        // ---- e4m3 weights.  LDS: the tokens of a stage and three units of 128 weight rows (unit u of a stage: rows 64 wn + 32 u .. + 31
        // of the tile for every wn).  This wavefront copies 16 rows of each; rows of one copy are neighbours in memory too: one offset
        // per lane, the rest is the same in all lanes.
        const int sub = lane >> 3, x0 = (lane & 7) ^ (lane >> 4);
        const uint32_t wlane = (uint32_t)sub * rowb + (uint32_t)(x0 << 4);
        uint32_t wrow[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) wrow[u] = (uint32_t)weight_row((wave >> 1) * 64 + u * 32 + (wave & 1) * 16) * rowb;
        // copy i of two of weight unit u of stage ks to the slot at byte `slot`
        auto copy_w = [&](int ks, int u, int i, uint32_t slot) {
            const uint32_t at = wrow[u] + (uint32_t)ks * 128u + (uint32_t)(8 * i) * rowb;
            copy16_to_lds(wbase + ((wlane ^ (i ? fresh_sgpr(64) : 0u)) + fresh_sgpr(at)), smem + kFUnitB + slot + wave * 2048 + i * 1024);
        };
        uint32_t xline[2];   // 128-byte line of the token row (its offset in bytes may pass 2^32)
        const uint32_t xchunk = (uint32_t)x0 << 4;
        auto copy_x = [&](int ks, int i) {
            const uint32_t line = xline[i] + fresh_sgpr((uint32_t)ks), lo = opaque_vgpr((line << 7) | (xchunk ^ (64u * i)));
            copy16_to_lds(p.x + (((uint64_t)(line >> 25) << 32) | lo), smem + wave * 2048 + i * 1024);
        };
#pragma unroll
        for (int v = 0; v < kFUnits; ++v)
            if (v / 2 < stages) {
                copy_w(v / 2, v % 2, 0, v * kFUnitB);
                copy_w(v / 2, v % 2, 1, v * kFUnitB);
            }
        rows_to_lds();
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            xline[i] = (uint32_t)s_rows[wave * 16 + i * 8 + sub] * (uint32_t)(K / 128);
            copy_x(0, i);
        }

        // Operand reads: v_mfma_f32_32x32x64_f8f6f4 takes 32 bytes per lane and operand, lane (c,h) -> row c, bytes [32 h, +32) of the 64-k half t
        // of the stage = chunks 4 t + 2 h + u.  Held: the LDS addresses of half 0; in half 1 bit 2 of the chunk is the other way.
        typedef const __attribute__((address_space(3))) u32x4 *lds_u32x4;
        uint32_t aoff[2], boff[2];
        {
            const int c = lane & 31, h = lane >> 5;
            const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)smem;
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const uint32_t at = lds0 + c * 128 + (((2 * h + u) ^ ((c >> 1) & 7)) << 4);
                aoff[u] = opaque_vgpr(at + wm * 64 * 128);
                boff[u] = opaque_vgpr(at + kFUnitB + wn * 32 * 128);
            }
        }
        auto read8 = [&](const uint32_t (&off)[2], uint32_t flip, uint32_t add) -> i32x8 {
            return as_operand(*(lds_u32x4)(uintptr_t)((off[0] ^ flip) + add), *(lds_u32x4)(uintptr_t)((off[1] ^ flip) + add));
        };
        // Two phases per stage, one per unit: wait for it (and the stage's tokens), read the phase's operands into registers and, once every
        // wavefront has, send the next copies into the places just read, between the phase's matrix instructions: the next stage's
        // tokens, then the unit three ahead.
        auto run = [&](auto busy_t) {
            constexpr bool kBusy = decltype(busy_t)::value;
            i32x8 fa[2][2], fb[2];   // tokens [row tile][half], held over the stage; weights [half]
            uint32_t slot = 0;
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the tokens of stage 0, the last copies issued
#pragma unroll 1
            for (int ks = 0; ks < stages; ++ks) {
                const bool more = ks + 1 < stages;
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    // younger than what this phase needs, two copies each: u = 0: the stage's other unit and the next stage's first; u = 1:
                    // the next stage's two and its tokens
                    if (!more && u == 1) copy_barrier();
                    else if (!more) asm volatile("s_waitcnt vmcnt(2) lgkmcnt(0)\n\ts_barrier" ::: "memory");
                    else if (u == 0) asm volatile("s_waitcnt vmcnt(4) lgkmcnt(0)\n\ts_barrier" ::: "memory");
                    else asm volatile("s_waitcnt vmcnt(6) lgkmcnt(0)\n\ts_barrier" ::: "memory");
                    if constexpr (kBusy) {
#pragma unroll
                        for (int t = 0; t < 2; ++t) {
                            const uint32_t flip = t ? fresh_sgpr(64) : 0u;
                            fb[t] = read8(boff, flip, slot);
                            if (u == 0) {
                                fa[0][t] = read8(aoff, flip, 0);
                                fa[1][t] = read8(aoff, flip, 32 * 128);
                            }
                        }
                        __builtin_amdgcn_sched_barrier(0);
                        __builtin_amdgcn_s_setprio(1);
                        mfma1(fb[0], fa[0][0], acc[0][u]);
                        __builtin_amdgcn_sched_barrier(0);
                        mfma1(fb[0], fa[1][0], acc[1][u]);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // every wavefront has read
                    if (u == 0 && more) {
                        copy_x(ks + 1, 0);
                        copy_x(ks + 1, 1);
                    }
                    if (ks + 1 + u < stages) {
                        copy_w(ks + 1 + u, 1 - u, 0, slot);
                        copy_w(ks + 1 + u, 1 - u, 1, slot);
                    }
                    slot = slot == (kFUnits - 1) * kFUnitB ? 0 : slot + kFUnitB;
                    __builtin_amdgcn_sched_barrier(0);
                    if constexpr (kBusy) {
                        mfma1(fb[1], fa[0][1], acc[0][u]);
                        __builtin_amdgcn_sched_barrier(0);
                        mfma1(fb[1], fa[1][1], acc[1][u]);
                        __builtin_amdgcn_sched_barrier(0);
                        __builtin_amdgcn_s_setprio(0);
                    }
                }
            }
        };
        if (busy) run(std::true_type{});
        else run(std::false_type{});
    } else {
        // ---- e2m1 weights: two stages of 128 k (16 KiB of token rows, 256 weight rows of 64 bytes), a plain loop.  This wavefront copies
        // token rows [16 w, 16 w + 16) and weight rows [32 w, 32 w + 32) of the tile.
        constexpr int kStageB = 2 * kFUnitB;
        const unsigned char *aptr[2];
        uint32_t boff[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int r = wave * 32 + i * 16 + (lane >> 2);
            boff[i] = (uint32_t)weight_row(r) * rowb + (((lane & 3) ^ ((r >> 2) & 3)) << 4);
        }
        // copy j of the wavefront's four of stage ks into buffer buf
        auto copy_one = [&](int ks, int buf, int j) {
            unsigned char *dst = smem + buf * kStageB + (j >> 1) * kFUnitB + wave * 2048 + (j & 1) * 1024;
            if (j < 2) copy16_to_lds(aptr[j] + ks * kFStageK, dst);
            else copy16_to_lds(wbase + (int64_t)ks * 64 + boff[j - 2], dst);
        };
        copy_one(0, 0, 2);
        copy_one(0, 0, 3);
        rows_to_lds();
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int r = wave * 16 + i * 8 + (lane >> 3);
            aptr[i] = p.x + (int64_t)s_rows[r] * K + (((lane & 7) ^ ((r >> 1) & 7)) << 4);
            copy_one(0, 0, i);
        }
        // Operand reads: the e2m1 operand takes 16 bytes per lane, chunk 2 t + h of the row's four in half t of the stage.  The instruction pairs its
        // lane h with bytes [16 h, 16 h + 16) of the token operand's lanes 0 and 1 (measured), so the token lanes take the chunks
        // h and 2 + h of the half stage.
        const int c = lane & 31, h = lane >> 5;
        int foff[4], woff[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
#pragma unroll
            for (int u = 0; u < 2; ++u) foff[t * 2 + u] = wm * 64 * 128 + c * 128 + (((4 * t + h + 2 * u) ^ ((c >> 1) & 7)) << 4);
            woff[t] = kFUnitB + wn * 64 * 64 + c * 64 + (((2 * t + h) ^ ((c >> 2) & 3)) << 4);
        }
        int buf = 0;
        for (int ks = 0; ks < stages; ++ks) {
            copy_barrier();   // stage ks has landed and stage ks - 1 is no longer read
            const bool more = ks + 1 < stages;
            const unsigned char *base = smem + buf * kStageB;
            if (busy) {
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    i32x8 fa[2], fb[2];
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        fa[i] = as_operand(*(const u32x4 *)(base + foff[t * 2] + i * 32 * 128), *(const u32x4 *)(base + foff[t * 2 + 1] + i * 32 * 128));
                        fb[i] = as_operand(*(const u32x4 *)(base + woff[t] + i * 32 * 64), u32x4{0, 0, 0, 0});
                    }
                    // token bytes 0..7 of every 8-byte group -> order 0 4 1 5 2 6 3 7 (nibble n of a packed word
                    // holds element n / 2 + 4 (n % 2))
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int d = 0; d < 8; d += 2) {
                            const uint32_t lo = (uint32_t)fa[i][d], hi = (uint32_t)fa[i][d + 1];
                            fa[i][d] = (int)__builtin_amdgcn_perm(hi, lo, 0x05010400u);
                            fa[i][d + 1] = (int)__builtin_amdgcn_perm(hi, lo, 0x07030602u);
                        }
                    __builtin_amdgcn_s_setprio(1);
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        if (t == 0 && more) copy_one(ks + 1, buf ^ 1, i);
                        mfma1(fb[i & 1], fa[i >> 1], acc[i >> 1][i & 1]);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    __builtin_amdgcn_s_setprio(0);
                }
            } else if (more) {
#pragma unroll
                for (int j = 0; j < 4; ++j) copy_one(ks + 1, buf ^ 1, j);
            }
            buf ^= 1;
        }
    }
    lds_barrier();   // no stage buffer is read any more

    // ---- epilogue: lane (c,h), register i of acc[ms][nt] -> token row 64 wm + 32 ms + c, row 64 wn + 32 nt + 8 (i/4) + 4 h + i%4 of the
    // weight tile: four consecutive rows, i.e. output columns, per register quad.  (The lane is read anew: values of it that
    // only the epilogue needs would be kept through the loop.)
    const int etid = (int)opaque_vgpr(threadIdx.x), el = etid & 63, c = el & 31, h = el >> 5;
    if constexpr (kSilu) {
        // rows 32 nt .. +15 of a wavefront's 64 are gate rows, the next sixteen the matching up rows: registers i and i + 8.  The results turn
        // through LDS ([128 rows][128 columns] bf16, 16-byte chunks XOR-swizzled with the row) and leave as whole 256-byte row pieces.
#pragma unroll
        for (int ms = 0; ms < 2; ++ms) {
            const int trow = wm * 64 + ms * 32 + c;
            const float xs = s_xs[trow];
#pragma unroll
            for (int nt = 0; nt < 2; ++nt) {
                const int rho0 = wn * 64 + nt * 32;
#pragma unroll
                for (int a4 = 0; a4 < 2; ++a4) {
                    const int r = 8 * a4 + 4 * h;
                    const f32x4 sg = *(const f32x4 *)(s_wn + rho0 + r), su = *(const f32x4 *)(s_wn + rho0 + 16 + r);
                    u32x2 o;
#pragma unroll
                    for (int b2 = 0; b2 < 2; ++b2) {
                        uint32_t pk = 0;
#pragma unroll
                        for (int q = 0; q < 2; ++q) {
                            const int i = 2 * b2 + q;
                            const float g = acc[ms][nt][4 * a4 + i] * (xs * sg[i]);
                            const float u = acc[ms][nt][8 + 4 * a4 + i] * (xs * su[i]);
                            pk |= (uint32_t)f32_to_bf16_hw(silu_mul_f32(g, u)) << (16 * q);
                        }
                        o[b2] = pk;
                    }
                    const int chunk = wn * 4 + nt * 2 + a4;
                    *(u32x2 *)(smem + trow * 256 + ((chunk ^ (trow & 15)) << 4) + h * 8) = o;
                }
            }
        }
        lds_barrier();
        const uint32_t rstride = (uint32_t)N;   // bytes per output row
#pragma unroll
        for (int pass = 0; pass < 4; ++pass) {
            const int row = pass * 32 + (etid >> 4), chunk = etid & 15, orow = s_orow[row];
            const int col = nb * (kFTN / 2) + chunk * 8;
            const u32x4 v4 = *(const u32x4 *)(smem + row * 256 + ((chunk ^ (row & 15)) << 4));
            if (orow >= 0 && col + 8 <= N / 2) *(u32x4 *)((unsigned char *)p.out + ((uint64_t)(uint32_t)orow * rstride + (uint32_t)col * 2u)) = v4;
        }
    } else {
        const int esz = p.out_f32 ? 4 : 2;
        const uint32_t rstride = (uint32_t)N * (uint32_t)esz;
#pragma unroll
        for (int ms = 0; ms < 2; ++ms) {
            const float xs = s_xs[wm * 64 + ms * 32 + c];
#pragma unroll
            for (int nt = 0; nt < 2; ++nt) {
                const int rho0 = wn * 64 + nt * 32;
                const int ocol0 = nb * kFTN + rho0;
                const bool tile_ok = ocol0 + 32 <= N;
                // The 32 x 32 tile turns through this wavefront's 4 KiB of the stage buffers and leaves as 16-byte pieces of whole
                // 128-byte row segments.  Chunks are XOR-swizzled with the row.
                unsigned char *ot = smem + wave * 4096;
#pragma unroll
                for (int a4 = 0; a4 < 4; ++a4) {
                    const int r = 8 * a4 + 4 * h;
                    const f32x4 sw = *(const f32x4 *)(s_wn + rho0 + r);
                    f32x4 vv;
#pragma unroll
                    for (int i = 0; i < 4; ++i) vv[i] = acc[ms][nt][4 * a4 + i] * (xs * sw[i]);
                    *(f32x4 *)(ot + c * 128 + (((2 * a4 + h) ^ (c & 7)) << 4)) = vv;
                }
#pragma unroll
                for (int pass = 0; pass < 4; ++pass) {
                    const int row = pass * 8 + (el >> 3);
                    const f32x4 v4 = *(const f32x4 *)(ot + row * 128 + (el & 7) * 16);
                    const int orow_r = s_orow[wm * 64 + ms * 32 + row];
                    const int col = ocol0 + (((el & 7) ^ (row & 7)) << 2);
                    if (orow_r >= 0 && tile_ok) {
                        unsigned char *dstp = (unsigned char *)p.out + (uint64_t)(uint32_t)orow_r * rstride;
                        if (p.out_f32) {
                            __builtin_nontemporal_store(v4, (f32x4 *)(dstp + col * 4));   // fp32 rows for the combine: written once, read once by another kernel
                        } else {
                            u32x2 o;
                            o[0] = (uint32_t)f32_to_bf16_hw(v4[0]) | ((uint32_t)f32_to_bf16_hw(v4[1]) << 16);
                            o[1] = (uint32_t)f32_to_bf16_hw(v4[2]) | ((uint32_t)f32_to_bf16_hw(v4[3]) << 16);
                            *(u32x2 *)(dstp + col * 2) = o;
                        }
                    }
                }
            }
        }
    }
}

template <int EPI, bool W4>
static int launch_fp8_cfg(const GemmArgs &a, hipStream_t s)
{
    if (a.E > 256) {
        set_error("qgemm (prefill path): at most 256 experts (got %d)", a.E);
        return QARL_ERR_UNSUPPORTED;
    }
    if (a.N % 32 != 0 || a.N > (1 << 28) || (int64_t)a.N * a.K >= (1LL << 32)) {
        set_error("qgemm (prefill path): N %% 32 == 0 and N * K < 2^32 required (got N=%d K=%d)", a.N, a.K);
        return QARL_ERR_UNSUPPORTED;
    }
    Tile8Params p;
    p.codes = (const unsigned char *)a.codes;
    p.scales = (const float *)a.scales;
    p.x = (const unsigned char *)a.x;
    p.x_scales = a.x_scales;
    p.row_map = a.row_map;
    p.out_row_map = a.out_row_map;
    p.offsets = a.offsets;
    p.out = a.out;
    p.E = a.E;
    p.N = a.N;
    p.K = a.K;
    p.out_f32 = a.out_f32;
    p.n_blocks = (EPI == QARL_EPI_SILU_MUL) ? (a.N / 2 + kFTN / 2 - 1) / (kFTN / 2) : (a.N + kFTN - 1) / kFTN;
    const int64_t slots = (a.M + kFTM - 1) / kFTM + a.E;
    const int64_t total = ((slots * p.n_blocks + 7) / 8) * 8;
    if (total > 0x7fffffffLL) {
        set_error("qgemm (prefill path): grid too large");
        return QARL_ERR_UNSUPPORTED;
    }
    static LdsLimitOnce once;
    auto kern = qgemm_tile_fp8_kernel<EPI, W4>;
    if (int rc = raise_lds_limit((const void *)kern, once, "hipFuncSetAttribute(tile fp8)")) return rc;
    kern<<<dim3((unsigned)total), dim3(kFThreads), kFLds, s>>>(p);
    return check_hip(hipGetLastError(), "qgemm_tile_fp8_kernel");
}

int launch_qgemm_tile_fp8(const GemmArgs &a, hipStream_t s)
{
    if (a.fmt == QARL_FP4_E2M1_CH)
        return a.epilogue == QARL_EPI_SILU_MUL ? launch_fp8_cfg<QARL_EPI_SILU_MUL, true>(a, s) : launch_fp8_cfg<QARL_EPI_NONE, true>(a, s);
    return a.epilogue == QARL_EPI_SILU_MUL ? launch_fp8_cfg<QARL_EPI_SILU_MUL, false>(a, s) : launch_fp8_cfg<QARL_EPI_NONE, false>(a, s);
}

}  // namespace qarl
