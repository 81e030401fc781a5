// Grouped quantized GEMM, MFMA-tiled ("prefill" / training-forward) path for W4A16: the same
// contraction as the weight-streaming path (eq. (1) of section 2.2), on the same codes and
// scales and with the same exact dequantized weight s*q, for experts that see hundreds to
// thousands of token rows, where the path is a dense contraction.  (FP8: qgemm_tile_fp8.hip.)
//
// A workgroup owns 64 token rows x 256 columns of one expert, its four wavefronts 64 x 64 each (2 x 2 tiles of
// v_mfma_f32_32x32x16_bf16): every operand read, every start value and every expanded word feeds two matrix
// instructions, and no packed weight is read or expanded twice in a workgroup.  Everything a stage (one scale group)
// needs reaches LDS by asynchronous copies one stage ahead: 16 KiB of gathered token rows (16-byte chunks XOR-swizzled
// with the row, so that copies and operand reads are free of bank conflicts), the rows' group sums, copied once for the
// workgroup, and, for each wavefront alone, its four 1 KiB blocks of codes and its columns' scales, where the groups are even in
// number a dword of two groups every second stage (sums and scales per wavefront and stage: 1 % slower at 16384 tokens; with
// none of either in the loop 4 % faster).  Two stages are 66.5 KiB, a wavefront takes at most 256 registers: two workgroups per CU that run out of step, one's lookup, first stage and stores under the other's loop.
// In a slice of 8 k per lane the operand reads and the expansion of the next slice are spread between the four matrix
// instructions of this one.  (Eight wavefronts of 64 x 32 with the codes in registers, operand reads twice as many per
// matrix instruction, ran 2 % slower.)  A workgroup computes up to four neighbouring column blocks one after the other: the
// expert lookup and the row gather are paid once, and the next block's first stage travels during the epilogue.  In
// turn on one box a W4A16 layer of 16384 tokens with popular experts took 1570 us with four blocks, 1585 with two, 1640 with
// one, 1690 with all six / eight (fewer workgroups share a token tile in L2), and 1670 with the wavefronts of 64 x 32; boxes
// differ by several per cent (1570 to 1610 us).  Against those wavefronts a launch of one round or less is up to 1 us longer
// (one wavefront per SIMD where there were two), and launches of two scale groups up to 15 %.
//
// What bounds it: 0.825 TFLOP of gate_up in 0.82-0.93 ms, about 0.95 PFLOP/s, where nothing but the matrix instructions of
// this shape runs at 1.35; next to them a stage issues 6 VALU operations per matrix instruction (expansion 3.5, fold 2).
//
// The group handling is the one described in qgemm_stream_w4.hip: codes become the exact bf16 values (q+24)/16, every
// scale group accumulates in its own fp32 accumulator that starts at -1.5 * sum_k x (the sums come from a small pre-pass
// over the activations, once per call), and is folded in with one FMA by 16*s.
#include <algorithm>
#include <type_traits>

#include "common.hpp"

namespace qarl {

constexpr int kRows = 64, kCols = 256;        // tile of a workgroup
constexpr int kWaves = 4, kThreads = 64 * kWaves;
constexpr int kRowBytes = kGroup * 2;         // bytes of a token row per stage (bf16, no padding: chunks are swizzled)
constexpr int kXBytes = kRows * kRowBytes;    // token rows of a stage
constexpr int kWaveBytes = 4 * 1024;          // a wavefront's codes
constexpr int kStageBytes = kXBytes + kWaves * kWaveBytes + 256;   // and the rows' group sums
constexpr int kScaleBytes = 256;              // a wavefront's scales, a dword (two groups where they are even in number) per column
constexpr int kTileLds = 2 * kStageBytes + 2 * kWaves * kScaleBytes;

struct TileParams {
    const unsigned char *codes;   // 1 KiB blocks [E * N / 16][K / 128]
    const unsigned char *scales;  // bf16 [E][N][K / 128]
    const unsigned char *x;       // bf16 [x_rows][K]
    const float *x_group_sums;    // [x_rows][K / 128]: -1.5 * sum of the group
    const float *x_scales;        // W4A8: scale of each activation row (x then holds e4m3 values as bf16), else null
    const int32_t *row_map;
    const int32_t *out_row_map;
    const int32_t *offsets;
    void *out;
    int E, N, K, out_f32;
    int n_blocks;   // column blocks per expert
    int bpw;        // consecutive column blocks one workgroup computes
    int n_bgroups;  // ceil(n_blocks / bpw)
};

__device__ __forceinline__ void copy4_to_lds(const void *gsrc, void *lds_dst)
{
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)gsrc,
                                     (__attribute__((address_space(3))) void *)lds_dst, 4, 0, 0);
}

template <int EPI>
__global__ __launch_bounds__(kThreads, 2) void qgemm_tile_kernel(TileParams p)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    constexpr bool kSilu = (EPI == QARL_EPI_SILU_MUL);
    __shared__ __attribute__((aligned(16))) int s_rows[kRows];   // activation row of each tile row (clamped to a valid one)
    __shared__ __attribute__((aligned(16))) int s_orow[kRows];   // output row, -1 past the expert's last row
    __shared__ __attribute__((aligned(16))) float s_xsc[kRows];  // row scale s_x

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 31, h = lane >> 5;

    GroupedTile tile;
    if (!find_grouped_tile<kRows>(p.offsets, p.E, p.n_bgroups, tile)) return;
    const int e = tile.e, nb_end = min(p.n_blocks, (tile.block + 1) * p.bpw);
    int nb = tile.block * p.bpw;   // column block
    const int row0 = tile.row0, mrem = tile.rows;
    if (tid < kRows) {
        // rows past the expert's end read the tile's first row (valid data, results never stored)
        const int i = row0 + (tid < mrem ? tid : 0);
        const int xrow = p.row_map ? p.row_map[i] : i;
        s_rows[tid] = xrow;
        s_orow[tid] = tid < mrem ? (p.out_row_map ? p.out_row_map[i] : i) : -1;
        s_xsc[tid] = p.x_scales ? p.x_scales[xrow] : 1.f;
    }
    lds_barrier();

    const int N = p.N, K = p.K, G = K / kGroup;
    // Column tile t (0..7, 32 columns; this wavefront's are 2 wave and 2 wave + 1) -> first weight rows of its two 16-row
    // blocks.  SILU_MUL: 16 gate rows and the matching 16 up rows, so gate j and up j sit 16 lanes apart in the result.
    // Tiles past N read the expert's first rows (valid data, results never stored).
    auto tile_ok = [&](int t) { return kSilu ? nb * (kCols / 2) + t * 16 + 16 <= N / 2 : nb * kCols + t * 32 + 32 <= N; };
    auto block_row = [&](int t, int half) {
        const int n = kSilu ? nb * (kCols / 2) + t * 16 + half * (N / 2) : nb * kCols + t * 32 + half * 16;
        return tile_ok(t) ? n : half * 16;   // N >= 32
    };

    // ---- copies.  Token rows: an instruction moves 4 rows x 256 bytes, chunk q of row r to position q ^ (r & 15).
    const unsigned char *xsrc[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r = wave * 16 + i * 4 + (lane >> 4);
        xsrc[i] = p.x + (int64_t)s_rows[r] * K * 2 + (((lane & 15) ^ (r & 15)) << 4);
    }
    const float *sum_src = p.x_group_sums + (int64_t)s_rows[lane] * G;
    // Codes: whole blocks.  Scales: the aligned dword that holds the column's bf16 scale (lane = column of the wavefront).
    // Byte offsets from the array bases; the launcher checks that the codes stay below 4 GiB.
    uint32_t boff[4], sidx, sidx_c[2];
    auto set_block = [&]() {
#pragma unroll
        for (int i = 0; i < 4; ++i) boff[i] = (uint32_t)((e * (int64_t)N + block_row(2 * wave + (i >> 1), i & 1)) / 16 * G) * 1024u + lane * 16;
        sidx = (uint32_t)((e * (int64_t)N + block_row(2 * wave + (lane >> 5), (lane >> 4) & 1) + (lane & 15)) * G);
        sidx_c[0] = (uint32_t)__shfl((int)sidx, c, 64);
        sidx_c[1] = (uint32_t)__shfl((int)sidx, 32 + c, 64);
    };
    set_block();
    const int sc_sh = 1 - (G & 1);   // the dword of a column's scale serves two groups where there is an even number of them
    auto copy_stage = [&](int g, int buf) {
        unsigned char *xs = smem + buf * kStageBytes, *ws = xs + kXBytes + wave * kWaveBytes;
#pragma unroll
        for (int j = 0; j < 4; ++j) copy16_to_lds(xsrc[j] + g * kRowBytes, xs + (wave * 16 + j * 4) * kRowBytes);
#pragma unroll
        for (int j = 0; j < 4; ++j) copy16_to_lds(p.codes + (boff[j] + (uint32_t)g * 1024u), ws + j * 1024);
        if (wave == (g & 3)) copy4_to_lds(sum_src + g, xs + kXBytes + kWaves * kWaveBytes);
        if (!(g & sc_sh)) copy4_to_lds(p.scales + (((sidx + (uint32_t)g) * 2u) & ~3u), smem + 2 * kStageBytes + (((g >> sc_sh) & 1) * kWaves + wave) * kScaleBytes);
    };

    // ---- operand reads.  Lane (row or column c of the tile, half h) takes k [64 h + 8 j, + 8) of the stage in slice j: chunk
    // 8 h + j of its token row, word j % 4 of piece 2 h + j / 4 of its weight row.
    int xoff[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) xoff[j] = c * kRowBytes + (((8 * h + j) ^ (c & 15)) << 4);
    const int woff = kXBytes + wave * kWaveBytes + (c >> 4) * 1024 + h * 512 + (c & 15) * 16;
    const int soff = kXBytes + kWaves * kWaveBytes;

    f32x16 acc[2][2];   // [row tile][column tile]
    auto stage = [&](int g, auto buf_c) {
        constexpr int buf = decltype(buf_c)::value;
        const unsigned char *st = smem + buf * kStageBytes;
        u32x4 w[2][2];
#pragma unroll
        for (int ns = 0; ns < 2; ++ns)
#pragma unroll
            for (int u = 0; u < 2; ++u) w[ns][u] = *(const u32x4 *)(st + woff + ns * 2048 + u * 256);
        f32x16 init[2];
#pragma unroll
        for (int ms = 0; ms < 2; ++ms)
#pragma unroll
            for (int i4 = 0; i4 < 4; ++i4) {
                const f32x4 v = *(const f32x4 *)(st + soff + (ms * 32 + 8 * i4 + 4 * h) * 4);
#pragma unroll
                for (int i = 0; i < 4; ++i) init[ms][i4 * 4 + i] = v[i];
            }
        float s16[2];
#pragma unroll
        for (int ns = 0; ns < 2; ++ns) {
            const uint32_t d = *(const uint32_t *)(smem + 2 * kStageBytes + (((g >> sc_sh) & 1) * kWaves + wave) * kScaleBytes + (ns * 32 + c) * 4);
            s16[ns] = 16.f * __uint_as_float(((sidx_c[ns] + (uint32_t)g) & 1) ? d & 0xffff0000u : d << 16);
        }
        f32x16 ag[2][2];
        // Slice j: its four MFMAs with the expansion and the operand reads of slice j + 1 spread between them.
        bf16x8 a[2][2], b[2][2];   // [slice parity]
        auto operands = [&](int j) {
#pragma unroll
            for (int ms = 0; ms < 2; ++ms) a[j & 1][ms] = *(const bf16x8 *)(st + xoff[j] + ms * 32 * kRowBytes);
#pragma unroll
            for (int ns = 0; ns < 2; ++ns) b[j & 1][ns] = unpack_int4_word(w[ns][j >> 2][j & 3]);
        };
        operands(0);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            if (j < 7) operands(j + 1);
#pragma unroll
            for (int ns = 0; ns < 2; ++ns)
#pragma unroll
                for (int ms = 0; ms < 2; ++ms)
                    ag[ms][ns] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[j & 1][ms], b[j & 1][ns], j == 0 ? init[ms] : ag[ms][ns], 0, 0, 0);
            if (j < 7) {
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);               // MFMA
                    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // LDS read (two in all)
                    __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);   // VALU
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int ns = 0; ns < 2; ++ns)
#pragma unroll
            for (int ms = 0; ms < 2; ++ms)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[ms][ns][i] = fmaf(s16[ns], ag[ms][ns][i], acc[ms][ns][i]);
    };

    // The copies of a stage travel during the stage before it.
    copy_stage(0, 0);
  for (;;) {   // column blocks (body not indented)
#pragma unroll
    for (int ms = 0; ms < 2; ++ms)
#pragma unroll
        for (int ns = 0; ns < 2; ++ns)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[ms][ns][i] = 0.f;
    copy_barrier();   // also: the last block's epilogue has left the second buffer
    for (int g = 0; g < G; g += 2) {
        if (g + 1 < G) copy_stage(g + 1, 1);
        stage(g, std::integral_constant<int, 0>());
        copy_barrier();
        if (g + 1 >= G) break;
        if (g + 2 < G) copy_stage(g + 2, 0);
        stage(g + 1, std::integral_constant<int, 1>());
        copy_barrier();
    }

    const int nb_done = nb;
    if (++nb < nb_end) {   // the next block's first stage travels during the epilogue, which keeps to the second buffer
        set_block();
        copy_stage(0, 0);
    }

    // ---- epilogue: lane (c, h), register i -> token row 8 (i / 4) + 4 h + i % 4, column c of the tile.  A direct store would
    // move 2 or 4 bytes per lane: the results take a turn through the stage buffers and leave as 16-byte pieces.
    if (kSilu) {
        uint16_t *ot = (uint16_t *)(smem + kStageBytes);   // [64 rows][128 columns] bf16
#pragma unroll
        for (int ns = 0; ns < 2; ++ns)
#pragma unroll
            for (int ms = 0; ms < 2; ++ms)
#pragma unroll
                for (int i4 = 0; i4 < 4; ++i4)
#pragma unroll
                    for (int ip = 0; ip < 2; ++ip) {
                        // Registers i and i+1 trade 16-lane rows: afterwards every lane holds a gate value and the up
                        // value of the same column; lanes c < 16 for row i, lanes c >= 16 for row i+1.
                        const u32x2 sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(acc[ms][ns][i4 * 4 + 2 * ip]),
                                                                          __float_as_uint(acc[ms][ns][i4 * 4 + 2 * ip + 1]), false, false);
                        const int row = ms * 32 + 8 * i4 + 4 * h + 2 * ip + (c >> 4);
                        const float rs = s_xsc[row];
                        const float a = silu_mul_f32(__uint_as_float(sw[0]) * rs, __uint_as_float(sw[1]) * rs);
                        ot[row * (kCols / 2) + (2 * wave + ns) * 16 + (c & 15)] = f32_to_bf16_hw(a);
                    }
        lds_barrier();
        constexpr int kPieces = kRows * (kCols / 2) * 2 / 16;   // 16 pieces per row
        const uint32_t rstride = (uint32_t)(N / 2) * 2u;        // bytes per output row (< 2^31: checked by the launcher)
#pragma unroll
        for (int q0 = 0; q0 < kPieces; q0 += kThreads) {
            const int q = q0 + tid, row = q >> 4, piece = q & 15;
            const int orow = s_orow[row];
            const int oc = nb_done * (kCols / 2) + piece * 8;
            const u32x4 v4 = *(const u32x4 *)(ot + row * (kCols / 2) + piece * 8);
            if (orow >= 0 && oc + 8 <= N / 2)
                *(u32x4 *)((unsigned char *)p.out + ((uint64_t)(uint32_t)orow * rstride + (uint32_t)oc * 2u)) = v4;
        }
    } else {
        // per wavefront [32 rows][64 columns] fp32 in LDS, 16-byte chunks XOR-swizzled with the row; only the wavefront itself
        // touches its region, and the LDS operations of a wavefront execute in order
        float *ot = (float *)(smem + kStageBytes) + wave * (32 * 64);
        const int esz = p.out_f32 ? 4 : 2;
        const uint32_t rstride = (uint32_t)N * (uint32_t)esz;   // bytes per output row (< 2^31: checked by the launcher)
        const int oc = nb_done * kCols + wave * 64 + (lane & 15) * 4;   // first of this lane's four columns
        const bool ok = oc - (lane & 7) * 4 + 32 <= N;
        unsigned char *obase = (unsigned char *)p.out + (int64_t)oc * esz;
#pragma unroll
        for (int ms = 0; ms < 2; ++ms) {
#pragma unroll
            for (int i4 = 0; i4 < 4; ++i4) {
                const f32x4 rs4 = *(const f32x4 *)(s_xsc + ms * 32 + 8 * i4 + 4 * h);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int row = 8 * i4 + 4 * h + i;
#pragma unroll
                    for (int ns = 0; ns < 2; ++ns)
                        ot[row * 64 + ((ns * 32 + c) ^ ((row & 4) << 3))] = acc[ms][ns][i4 * 4 + i] * rs4[i];
                }
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
            for (int pass = 0; pass < 8; ++pass) {
                const int row = pass * 4 + (lane >> 4);
                const f32x4 v4 = *(const f32x4 *)(ot + row * 64 + (((lane & 15) * 4) ^ ((row & 4) << 3)));
                const int orow = s_orow[ms * 32 + row];
                if (orow >= 0 && ok) {
                    unsigned char *dst = obase + (uint64_t)(uint32_t)orow * rstride;
                    if (p.out_f32) {
                        __builtin_nontemporal_store(v4, (f32x4 *)dst);
                    } else {
                        u32x2 o;
                        o[0] = (uint32_t)f32_to_bf16_hw(v4[0]) | ((uint32_t)f32_to_bf16_hw(v4[1]) << 16);
                        o[1] = (uint32_t)f32_to_bf16_hw(v4[2]) | ((uint32_t)f32_to_bf16_hw(v4[3]) << 16);
                        __builtin_nontemporal_store(o, (u32x2 *)dst);
                    }
                }
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        }
    }
    if (nb >= nb_end) break;
  }
}

constexpr int kItems = 2048, kMaxBlocks = 4;   // see the launcher

template <int EPI>
static int launch_cfg(const GemmArgs &a, hipStream_t s)
{
    if (a.E > 256) {
        set_error("qgemm (prefill path): at most 256 experts (got %d)", a.E);
        return QARL_ERR_UNSUPPORTED;
    }
    if (a.N % 32 != 0 || a.N > (1 << 28)) {
        set_error("qgemm (prefill path): N %% 32 == 0 and N <= 2^28 required (got %d)", a.N);
        return QARL_ERR_UNSUPPORTED;
    }
    const int64_t n_w = (int64_t)a.E * a.N * a.K;
    if (n_w / 2 >= (1LL << 32)) {
        set_error("qgemm (prefill path): quantized weights of one call must stay below 4 GiB");
        return QARL_ERR_UNSUPPORTED;
    }
    TileParams p;
    p.codes = (const unsigned char *)a.codes;
    p.scales = (const unsigned char *)a.scales;
    p.x = (const unsigned char *)a.x;
    p.x_group_sums = a.x_group_sums;
    p.x_scales = a.fmt == QARL_W4A8_G128 ? a.x_scales : nullptr;
    p.row_map = a.row_map;
    p.out_row_map = a.out_row_map;
    p.offsets = a.offsets;
    p.out = a.out;
    p.E = a.E;
    p.N = a.N;
    p.K = a.K;
    p.out_f32 = a.out_f32;
    p.n_blocks = (EPI == QARL_EPI_SILU_MUL) ? (a.N / 2 + kCols / 2 - 1) / (kCols / 2) : (a.N + kCols - 1) / kCols;
    const int64_t slots = (a.M + kRows - 1) / kRows + a.E;
    // up to kMaxBlocks column blocks per workgroup, as long as kItems workgroups remain (four rounds of the two a CU
    // holds; with half as many a layer of 3001 tokens takes 398 us instead of 389), in groups of about equal size
    int bpw = (int)std::min<int64_t>(std::max<int64_t>(slots * p.n_blocks / kItems, 1), std::min(kMaxBlocks, p.n_blocks));
    p.n_bgroups = (p.n_blocks + bpw - 1) / bpw;
    p.bpw = (p.n_blocks + p.n_bgroups - 1) / p.n_bgroups;
    p.n_bgroups = (p.n_blocks + p.bpw - 1) / p.bpw;
    const int64_t total = ((slots * p.n_bgroups + 7) / 8) * 8;
    if (total > 0x7fffffffLL) {
        set_error("qgemm (prefill path): grid too large");
        return QARL_ERR_UNSUPPORTED;
    }
    static LdsLimitOnce once;
    auto kern = qgemm_tile_kernel<EPI>;
    if (int rc = raise_lds_limit((const void *)kern, once, "hipFuncSetAttribute(tile)")) return rc;
    kern<<<dim3((unsigned)total), dim3(kThreads), kTileLds, s>>>(p);
    return check_hip(hipGetLastError(), "qgemm_tile_kernel");
}

// sums[row][g] = -1.5 * sum over the 128 k of group g of x[row][k]: the start value of a group's
// accumulator (it cancels the +24/16 offset of the expanded codes).  16 lanes own a group.
__global__ __launch_bounds__(256) void group_sums_kernel(const u32x4 *__restrict__ x, int64_t n_chunks,
                                                         float *__restrict__ sums)
{
    const int64_t c = (int64_t)blockIdx.x * 256 + threadIdx.x;  // 16-byte chunk = 8 elements
    u32x4 v = {0, 0, 0, 0};
    if (c < n_chunks) v = x[c];
    float s = group_chunk_sum(v);
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) s += __shfl_xor(s, o, 64);
    if (c < n_chunks && (c & 15) == 0) sums[c >> 4] = -1.5f * s;
}

int launch_group_sums(const void *x_bf16, int64_t rows, int K, float *sums, hipStream_t s)
{
    const int64_t n_chunks = rows * (int64_t)(K / 8);
    if (n_chunks == 0) return QARL_OK;
    const int64_t blocks = (n_chunks + 255) / 256;
    if (blocks > 0x7fffffffLL) {
        set_error("group sums: grid too large");
        return QARL_ERR_UNSUPPORTED;
    }
    group_sums_kernel<<<dim3((unsigned)blocks), dim3(256), 0, s>>>((const u32x4 *)x_bf16, n_chunks, sums);
    return check_hip(hipGetLastError(), "group_sums_kernel");
}

int launch_qgemm_tile(const GemmArgs &a, hipStream_t s)
{
    if (a.fmt == QARL_W4A16_G128 || a.fmt == QARL_W4A8_G128)
        return a.epilogue == QARL_EPI_SILU_MUL ? launch_cfg<QARL_EPI_SILU_MUL>(a, s) : launch_cfg<QARL_EPI_NONE>(a, s);
    return launch_qgemm_tile_fp8(a, s);
}

}  // namespace qarl
