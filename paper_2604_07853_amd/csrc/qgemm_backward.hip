// Backward of the rollout-aligned W4A16 forward under the straight-through estimator (section 3.1, item 2: the
// forward runs on the low-bit weights; gradients are computed as if Quant were the identity, in the trainer's
// 16-bit precision, and applied to the BF16 masters).  For Y[i] = What_e x[row(i)] (eq. (1), What = s*q):
//     dX[i][k]    = sum_n dY[i][n] * What_e[n][k]                -> qgemm_dx_kernel
//     dW[e][n][k] = sum_{i in expert e} dY[i][n] * x[row(i)][k]  -> grouped_dw_kernel
// Both are dense contractions on v_mfma_f32_32x32x16_bf16 with fp32 accumulation.  In both the contraction index
// is the one the operands do NOT store contiguously (n for dX: the codes are packed along k; the token index for
// dW), while the matrix instruction wants 8 consecutive contraction elements per lane.  The tiles go to LDS as
// they are stored (rows = contraction index, 16-byte pieces) and are read with the transposing LDS read
// ds_read_b64_tr_b16, which hands a lane four consecutive ROWS of one column: within each group of 16 lanes, lane
// 4 a + b receives element b of the 8 bytes addressed by lanes a, a + 4, a + 8 and a + 12 of the group.
//
// dX.  A workgroup owns 128 rows x 128 output columns k, i.e. exactly one scale group g of every weight row, so
// the scale s[n][g] depends on the contraction index alone and is folded into the gradient operand:
// A'[i][n] = bf16(dY[i][n] * s[n][g]), rounded once (the 16-bit backward; a one-hot dY and the exact-integer
// regime stay exact).  The codes go through the same exponent trick as in the forward, (q+24)/16 as an exact
// bf16, written row by row ([n][k]) into LDS; the offset is removed at the end with the row sums of A' (fp32,
// accumulated while A' is staged): dX = 16 * acc - 24 * rowsum.
#include <algorithm>
#include <type_traits>

#include "common.hpp"

namespace qarl {

namespace {

constexpr int kBwThreads = 512;
constexpr int kTM = 128;   // rows (dX) / weight rows n (dW) per workgroup
constexpr int kTK = 128;   // output columns k per workgroup
constexpr int kStageN = 128;   // dX: contraction elements n per stage
constexpr int kStageM = 64;    // dW: contraction elements (token rows) per stage

struct DxParams {
    const uint32_t *codes;    // 1 KiB blocks [E * N / 16][K / 128][256 words]
    const uint16_t *scales;   // bf16 [E][N][K / 128]
    const uint16_t *dy;       // bf16 [M][N], rows grouped by expert
    const int32_t *offsets;
    const int32_t *out_row_map;
    void *out;                // [M][K]
    int E, N, K, out_f32;
};

// 16-byte chunk swizzles of 256-byte LDS rows.  As: rows are gradient rows, read by 32 consecutive rows at once.
// Tiles read by the transposing read: a 32-lane pass touches four consecutive rows (from a multiple of four) and 64
// bytes of each, so the rows go to different quarters of the 256 bytes; the second term spreads the sixteen rows a
// code block is written to.
__device__ __forceinline__ int swz_a(int m) { return m & 15; }
__device__ __forceinline__ int swz_tr(int row) { return ((row & 3) << 2) | ((row >> 2) & 3); }

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// MFMA operand of lane `lane` (row or column l % 32, contraction elements 8 (l / 32) .. + 7) from a tile stored
// [contraction index][128 columns] bf16 in 256-byte rows with swz_tr chunks: columns col0 .. col0 + 31 (col0 a
// multiple of 32), contraction rows 16 st .. 16 st + 15.  The two addresses a lane passes are its base offsets
// (computed once: the swizzle of row 16 st + c does not depend on st) plus 4096 st, an immediate of the read.
struct TrBase {
    int lo, hi;
};
__device__ __forceinline__ TrBase tr_base(int col0, int lane)
{
    const int r16 = lane & 15, g = lane >> 4;
    const int row = 8 * (g >> 1) + (r16 >> 2);                // the row this lane ADDRESSES (second read: + 4)
    const int colq = col0 + 16 * (g & 1) + 4 * (r16 & 3);     // first of the four columns it addresses
    TrBase b;
    b.lo = row * 256 + (((colq >> 3) ^ swz_tr(row)) << 4) + (colq & 4) * 2;
    b.hi = (row + 4) * 256 + (((colq >> 3) ^ swz_tr(row + 4)) << 4) + (colq & 4) * 2;
    return b;
}
template <int ST>
__device__ __forceinline__ bf16x8 read_operand_tr(const unsigned char *tile, const TrBase &b)
{
    struct {
        s16x4 lo, hi;
    } v;
    v.lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(tile + b.lo + ST * 4096));
    v.hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(tile + b.hi + ST * 4096));
    return __builtin_bit_cast(bf16x8, v);
}

// compile-time loop over the 16-element contraction steps of a stage
template <int I, int N, typename F>
__device__ __forceinline__ void static_for(F &&f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>());
        static_for<I + 1, N>(f);
    }
}

__global__ __launch_bounds__(kBwThreads, 4) void qgemm_dx_kernel(DxParams p)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    __shared__ __attribute__((aligned(16))) int s_orow[kTM];
    __shared__ __attribute__((aligned(16))) float s_rs[kTM];
    unsigned char *As = smem;                       // [kTM][kStageN] bf16, 256-byte rows
    unsigned char *Bs = smem + kTM * kStageN * 2;   // [kStageN n][kTK k] bf16 (q+24)/16, 256-byte rows
    float *sc = (float *)(smem + (kTM + kTK) * kStageN * 2);   // [N] scales of group g as fp32

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int N = p.N, K = p.K, G = K / kGroup;

    GroupedTile tile;
    if (!find_grouped_tile<kTM>(p.offsets, p.E, G, tile)) return;
    const int e = tile.e, g = tile.block;   // output column block = scale group
    const int row0 = tile.row0, mrem = tile.rows;
    if (tid < kTM) s_orow[tid] = tid < mrem ? (p.out_row_map ? p.out_row_map[row0 + tid] : row0 + tid) : -1;
    for (int n = tid; n < N; n += kBwThreads) sc[n] = bf16_bits_to_f32(p.scales[((int64_t)e * N + n) * G + g]);

    // gradient staging: chunk id = tid + 512 u -> row id >> 4, 16-byte piece id & 15 of the stage's 128 n
    const int am = tid >> 4, acn = tid & 15;
    float rowsum[4] = {0.f, 0.f, 0.f, 0.f};
    const bf16x2 ones2 = __builtin_bit_cast(bf16x2, 0x3f803f80u);
    // weight staging: this wavefront expands the block of rows n0 + 16 wave .. + 15; lane = (k range q, row c)
    const int bq = lane >> 4, bc = lane & 15;
    // matrix phase: wavefront (wm, wk) owns rows 32 wm .. + 31, columns 64 wk .. + 63
    const int wm = wave >> 1, wk = wave & 1, m32 = lane & 31, h = lane >> 5;
    f32x16 acc[2];
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[kt][i] = 0.f;

    const TrBase tb[2] = {tr_base(wk * 64, lane), tr_base(wk * 64 + 32, lane)};
    // The global loads of a stage are issued one stage ahead, right after the previous stage's operands have
    // been written to LDS, so they travel during that stage's matrix phase.
    u32x4 gv[4], wv;
    const uint16_t *gbase = p.dy + (int64_t)(row0 + am) * N + acn * 8;                      // row am of the tile; row am + 32 u: + 32 u N
    const uint32_t *cbase = p.codes + (((int64_t)e * N / 16 + wave) * G + g) * 256 + lane * 4;   // tile of rows n0 + 16 wave ..: + (n0 / 16) G blocks
    auto load_stage = [&](int n0) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            gv[u] = u32x4{0, 0, 0, 0};
            if (am + 32 * u < mrem) gv[u] = *(const u32x4 *)(gbase + (uint32_t)(32 * u) * (uint32_t)N + n0);
        }
        wv = *(const u32x4 *)(cbase + (uint32_t)(n0 / 16) * (uint32_t)(G * 256));
    };
    load_stage(0);
    for (int n0 = 0; n0 < N; n0 += kStageN) {
        lds_barrier();   // the matrix phase of the previous stage is done (first trip: the scales are written)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int m = am + 32 * u;
            const f32x4 s_lo = *(const f32x4 *)(sc + n0 + acn * 8), s_hi = *(const f32x4 *)(sc + n0 + acn * 8 + 4);
            u32x4 o;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float s0 = i < 2 ? s_lo[2 * i] : s_hi[2 * i - 4], s1 = i < 2 ? s_lo[2 * i + 1] : s_hi[2 * i - 3];
                bf16x2 pr;
                pr[0] = (__bf16)(__uint_as_float(gv[u][i] << 16) * s0);
                pr[1] = (__bf16)(__uint_as_float(gv[u][i] & 0xffff0000u) * s1);
                // row sum of the ROUNDED values: both halves times 1.0, added to the running sum in one operation
                rowsum[u] = __builtin_amdgcn_fdot2_f32_bf16(pr, ones2, rowsum[u], false);
                o[i] = __builtin_bit_cast(uint32_t, pr);
            }
            *(u32x4 *)(As + m * 256 + ((acn ^ swz_a(m)) << 4)) = o;
        }
        {
            const int nl = wave * 16 + bc;   // row of the stage; word j of the lane = columns 32 bq + 8 j .. + 7
#pragma unroll
            for (int j = 0; j < 4; ++j)
                *(u32x4 *)(Bs + nl * 256 + (((bq * 4 + j) ^ swz_tr(nl)) << 4)) = __builtin_bit_cast(u32x4, unpack_int4_word(wv[j]));
        }
        if (n0 + kStageN < N) load_stage(n0 + kStageN);
        lds_barrier();
        static_for<0, kStageN / 16>([&](auto st_c) {
            constexpr int st = decltype(st_c)::value;
            const int ch = 2 * st + h;
            const int m = wm * 32 + m32;
            const bf16x8 a = *(const bf16x8 *)(As + m * 256 + ((ch ^ swz_a(m)) << 4));
#pragma unroll
            for (int kt = 0; kt < 2; ++kt) {
                const bf16x8 b = read_operand_tr<st>(Bs, tb[kt]);
                acc[kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc[kt], 0, 0, 0);
            }
        });
    }
    // row sums of A': the 16 threads of a row sit in 16 consecutive lanes
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        float r = rowsum[u];
#pragma unroll
        for (int o = 1; o < 16; o <<= 1) r += __shfl_xor(r, o, 64);
        if (acn == 0) s_rs[am + 32 * u] = r;
    }
    lds_barrier();
    // lane (column m32 of tile kt, half h), register i -> row 32 wm + 8 (i / 4) + 4 h + i % 4
#pragma unroll
    for (int i4 = 0; i4 < 4; ++i4) {
        const int r0 = wm * 32 + 8 * i4 + 4 * h;
        const i32x4 orow4 = *(const i32x4 *)(s_orow + r0);
        const f32x4 rs4 = *(const f32x4 *)(s_rs + r0);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int64_t orow = orow4[i];
            if (orow < 0) continue;
#pragma unroll
            for (int kt = 0; kt < 2; ++kt) {
                const float val = fmaf(16.f, acc[kt][i4 * 4 + i], -24.f * rs4[i]);
                const int64_t col = g * kTK + wk * 64 + kt * 32 + m32;
                if (p.out_f32) ((float *)p.out)[orow * K + col] = val;
                else ((uint16_t *)p.out)[orow * K + col] = f32_to_bf16_hw(val);
            }
        }
    }
}

// ---- dX on 256 x 256 tiles, i.e. two scale groups.  A stage holds 64 contraction elements n: the gradient rows as they are
// stored, Ds [256 rows][64 n] (asynchronous copies, 128-byte rows, chunk c of row r at position c ^ (r & 7)), and the
// expanded codes Ws [64 n][256 k] (512-byte rows, swz_tr); two of each, and two of the raw codes Cs, each wavefront its own
// 1 KiB block, copied two stages ahead and expanded one stage ahead.  Eight wavefronts of 64 rows x 128 columns, one scale group
// each, so that a wavefront scales exactly the operand it multiplies, in registers: the gradient operand comes from LDS unscaled, and
// the matrix core scales it.  v_mfma_f32_4x4x4 is sixteen products of 4 x 4 matrices, one per four neighbouring lanes; lane j of the
// four holds column j of the second operand and of the result (four elements each) and row j of the first.  With diag(s[n .. n + 3])
// as the first, a lane's four gradients of its row come back as four exact fp32 products: one instruction of 8 cycles for two
// unpackings and a multiplication per element.  Rows that no wavefront has (a wavefront of 64 rows past the expert's end) are not
// multiplied.  Gate_up, 16384 tokens, Zipf router: 1332 -> 1110 us (the 128 x 128 tiles
// above move twice the LDS bytes per matrix instruction and scale through VALU); without copies, scaling and expansion it would take 747, without the
// scaling 1029, without the copies 1018: what is left is matrix instructions, and the rest adds to them.
constexpr int kDxWTile = 256, kDxWStage = 64;
constexpr int kDxWDsB = kDxWTile * kDxWStage * 2, kDxWWs = 2 * kDxWDsB, kDxWWsB = kDxWStage * kDxWTile * 2, kDxWCs = kDxWWs + 2 * kDxWWsB;
constexpr int kDxWCsB = kDxWStage * kDxWTile / 2, kDxWSc = kDxWCs + 2 * kDxWCsB;   // LDS offsets and sizes; then [2][N] scales
__host__ __device__ constexpr size_t dx_wide_lds(int N) { return kDxWSc + (size_t)N * 4; }

__device__ __forceinline__ TrBase tr_base_dx(int col0, int lane)
{
    const int r16 = lane & 15, g = lane >> 4;
    const int row = 8 * (g >> 1) + (r16 >> 2);                // the row this lane ADDRESSES (second read: + 4)
    const int colq = col0 + 16 * (g & 1) + 4 * (r16 & 3);     // first of the four columns it addresses
    TrBase b;
    b.lo = row * 512 + (((colq >> 3) ^ swz_tr(row)) << 4) + (colq & 4) * 2;
    b.hi = (row + 4) * 512 + (((colq >> 3) ^ swz_tr(row + 4)) << 4) + (colq & 4) * 2;
    return b;
}

__global__ __launch_bounds__(kBwThreads, 2) void qgemm_dx_wide_kernel(DxParams p)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    __shared__ __attribute__((aligned(16))) int s_orow[kDxWTile];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave >> 1, wg = wave & 1, m32 = lane & 31, h = lane >> 5;   // rows 64 wr .., scale group wg of the two
    const int N = p.N, K = p.K, G = K / kGroup;

    GroupedTile tile;
    if (!find_grouped_tile<kDxWTile>(p.offsets, p.E, K / kDxWTile, tile)) return;
    const int e = tile.e, kb = tile.block;
    const int row0 = tile.row0, mrem = tile.rows;

    // ---- copies.  Instruction i (0..3) of the wavefront moves the gradient rows 32 w + 8 i .. + 7; lane L fills position L % 8 of
    // row L / 8 of them.  Rows past the expert's end repeat its last one (their results are never stored).
    const unsigned char *ybase = (const unsigned char *)(p.dy + (int64_t)row0 * N);
    uint32_t yoff[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
        yoff[i] = (uint32_t)min(wave * 32 + 8 * i + (lane >> 3), mrem - 1) * (uint32_t)(N * 2) + (uint32_t)(((lane & 7) ^ (lane >> 3)) << 4);
    const unsigned char *cbase = (const unsigned char *)(p.codes + (((int64_t)e * N / 16 + wr) * G + 2 * kb + wg) * 256) + lane * 16;
    auto copy_rows = [&](int s, int i) {
        copy16_to_lds(ybase + yoff[i] + (uint32_t)(s * kDxWStage * 2), smem + (s & 1) * kDxWDsB + (wave * 32 + 8 * i) * (kDxWStage * 2));
    };
    auto copy_codes = [&](int s) {
        copy16_to_lds(cbase + (uint64_t)(uint32_t)s * (uint32_t)(4 * G * 1024), smem + kDxWCs + (s & 1) * kDxWCsB + wave * 1024);
    };
    const int stages = N / kDxWStage;   // at least two
#pragma unroll
    for (int i = 0; i < 4; ++i) copy_rows(0, i);
    copy_codes(0);
    copy_codes(1);
    if (tid < kDxWTile) s_orow[tid] = tid < mrem ? (p.out_row_map ? p.out_row_map[row0 + tid] : row0 + tid) : -1;
    {
        uint16_t *sc = (uint16_t *)(smem + kDxWSc);
        for (int n = tid; n < N; n += kBwThreads) {
            const uint32_t v = *(const uint32_t *)(p.scales + ((int64_t)e * N + n) * G + 2 * kb);
            sc[n] = (uint16_t)v;
            sc[N + n] = (uint16_t)(v >> 16);
        }
    }

    // ---- expansion: lane (k range q = lane / 16, row lane % 16) of this wavefront's block of stage s
    const uint32_t lds0 = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void *)smem;
    const int nl = wr * 16 + (lane & 15);
    const uint32_t wdst = kDxWWs + nl * 512 + (((wg * 16 + (lane >> 4) * 4) ^ swz_tr(nl)) << 4);
    auto read_codes = [&](int s) { return *(const u32x4 *)(smem + kDxWCs + (s & 1) * kDxWCsB + wave * 1024 + lane * 16); };
    // (as asm: in front of an LDS store the compiler can see it drains the copies in flight)
    auto expand_word = [&](int s, uint32_t w, int j) {
        const u32x4 v = __builtin_bit_cast(u32x4, unpack_int4_word(w));
        asm volatile("ds_write_b128 %0, %1" ::"v"((wdst ^ (uint32_t)(j << 4)) + (lds0 + (uint32_t)((s & 1) * kDxWWsB))), "v"(v) : "memory");
    };

    // ---- operands of a slice (16 contraction elements): the gradient rows, the scales of the lane's row of the two diagonals, the codes
    int aoff[4];
#pragma unroll
    for (int st = 0; st < 4; ++st) aoff[st] = (wr * 64 + m32) * (kDxWStage * 2) + (((2 * st + h) ^ (m32 & 7)) << 4);
    const int soff = kDxWSc + (wg * N + 8 * h + (lane & 3)) * 2;
    TrBase tb[4];
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) tb[nt] = tr_base_dx(wg * 128 + nt * 32, lane);
    struct Frags {
        bf16x8 a[2], b[4];   // scaled gradients, codes
    };
    // (asm for the same reason; waited for by hand, with the wait tied to the registers)
    auto read_tr = [&](uint32_t base, const TrBase &t, auto off_c) -> bf16x8 {
        constexpr int off = decltype(off_c)::value;
        struct {
            s16x4 lo, hi;
        } v;
        asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(v.lo) : "v"(base + (uint32_t)t.lo), "n"(off));
        asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(v.hi) : "v"(base + (uint32_t)t.hi), "n"(off));
        return __builtin_bit_cast(bf16x8, v);
    };
    auto wait_frags = [&](Frags &f) {
        asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(f.b[0]), "+v"(f.b[1]), "+v"(f.b[2]), "+v"(f.b[3]));
    };
    const int dsh = (lane & 1) * 16;
    const uint32_t dlo = (lane & 2) ? 0u : 0xffffffffu;
    const bf16x2 ones2 = __builtin_bit_cast(bf16x2, 0x3f803f80u);
    // Row sums in sixteen chains of N / 32 additions and a tree, as in the 128 x 128 tiles: here half a chunk of eight elements each (the
    // lane's half h, slice j, half w).  Two chains of N / 4 put the error of dX up to 1 % above those tiles' (N = 2048: 1.071e-6
    // against 1.063e-6 of the results, now 1.063e-6), and are no faster.
    float rowsum[2][4][2];
#pragma unroll
    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
        for (int i = 0; i < 8; ++i) rowsum[rt][i >> 1][i & 1] = 0.f;
    f32x16 acc[2][4];
#pragma unroll
    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
        for (int nt = 0; nt < 4; ++nt)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[rt][nt][i] = 0.f;
    // gradient rows of one row tile times the two diagonals (eight contraction elements per lane)
    auto scaled = [&](u32x4 g, const u32x2 (&diag)[2], float (&chain)[2]) -> bf16x8 {
        u32x4 o;
#pragma unroll
        for (int w = 0; w < 2; ++w) {
            const u32x2 gw = {g[2 * w], g[2 * w + 1]};
            const f32x4 d = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(__builtin_bit_cast(s16x4, diag[w]), __builtin_bit_cast(s16x4, gw),
                                                                   f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                bf16x2 pr;
                pr[0] = (__bf16)d[2 * i];
                pr[1] = (__bf16)d[2 * i + 1];
                // row sum of the ROUNDED values: both halves times 1.0, added to the running sum in one operation
                chain[w] = __builtin_amdgcn_fdot2_f32_bf16(pr, ones2, chain[w], false);
                o[2 * w + i] = __builtin_bit_cast(uint32_t, pr);
            }
        }
        return __builtin_bit_cast(bf16x8, o);
    };
    // Under the eight MFMAs of `cur`, slice j of stage ks is read (behind the first three) and scaled (from the fifth on) into
    // `nxt`; stage ks + 1 is copied in slice 0, its codes, copied a stage ago, are expanded in slices 1 and 2.
    u32x4 cw = {0, 0, 0, 0};
    auto slice = [&](const Frags &cur, Frags &nxt, int ks, auto j_c, auto more_t) {
        constexpr int j = decltype(j_c)::value;
        constexpr bool more = decltype(more_t)::value;
        const int buf = ks & 1;
        const uint32_t base = lds0 + kDxWWs + buf * kDxWWsB;
        constexpr std::integral_constant<int, j * 16 * 512> off{};
        u32x4 g[2];
        uint32_t sv[2];
        u32x2 diag[2];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int nt = i >> 1, rt = i & 1;
            acc[rt][nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(cur.a[rt], cur.b[nt], acc[rt][nt], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            if (i == 0) {
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    g[r] = *(const u32x4 *)(smem + buf * kDxWDsB + aoff[j] + r * (32 * kDxWStage * 2));
                    sv[r] = *(const uint16_t *)(smem + soff + ks * (kDxWStage * 2) + (16 * j + 4 * r) * 2);
                }
            } else if (i < 3) {
                nxt.b[2 * i - 2] = read_tr(base, tb[2 * i - 2], off);
                nxt.b[2 * i - 1] = read_tr(base, tb[2 * i - 1], off);
            } else if (i == 4) {
                wait_frags(nxt);
#pragma unroll
                for (int w = 0; w < 2; ++w) {
                    const uint32_t v = sv[w] << dsh;
                    diag[w] = u32x2{v & dlo, v & ~dlo};
                }
                nxt.a[0] = scaled(g[0], diag, rowsum[0][j]);
            } else if (i == 5) {
                nxt.a[1] = scaled(g[1], diag, rowsum[1][j]);
            }
            if (more) {
                if (j == 0 && (i & 1)) copy_rows(ks + 1, i >> 1);
                if (j == 1 && i == 0 && ks + 2 < stages) copy_codes(ks + 2);
                if (j == 0 && i == 2) cw = read_codes(ks + 1);
                if ((j == 1 || j == 2) && (i == 3 || i == 7)) expand_word(ks + 1, cw[(j - 1) * 2 + (i >> 2)], (j - 1) * 2 + (i >> 2));
            }
            if (i < 4) __builtin_amdgcn_sched_barrier(0);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    auto stage_barrier = [&]() {   // own copies landed, own LDS operations done; then everybody's
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    };
    Frags last, f0, f1, f2, f3;
#pragma unroll
    for (int i = 0; i < 2; ++i) last.a[i] = bf16x8{0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < 4; ++i) last.b[i] = bf16x8{0, 0, 0, 0, 0, 0, 0, 0};
    stage_barrier();
    cw = read_codes(0);
#pragma unroll
    for (int j = 0; j < 4; ++j) expand_word(0, cw[j], j);
    stage_barrier();
    auto stage = [&](int ks, auto more_t) {
        slice(last, f0, ks, std::integral_constant<int, 0>{}, more_t);
        slice(f0, f1, ks, std::integral_constant<int, 1>{}, more_t);
        slice(f1, f2, ks, std::integral_constant<int, 2>{}, more_t);
        slice(f2, f3, ks, std::integral_constant<int, 3>{}, more_t);
        stage_barrier();
        last = f3;
    };
    if (wr * 64 >= mrem) {   // no row of this wavefront's: its copies and its share of the codes only
        for (int ks = 0; ks < stages; ++ks) {
            if (ks + 1 < stages) {
#pragma unroll
                for (int i = 0; i < 4; ++i) copy_rows(ks + 1, i);
                cw = read_codes(ks + 1);
                if (ks + 2 < stages) copy_codes(ks + 2);
#pragma unroll
                for (int j = 0; j < 4; ++j) expand_word(ks + 1, cw[j], j);
            }
            stage_barrier();
        }
        return;
    }
    for (int ks = 0; ks + 1 < stages; ++ks) stage(ks, std::true_type{});
    stage(stages - 1, std::false_type{});
#pragma unroll
    for (int nt = 0; nt < 4; ++nt)
#pragma unroll
        for (int rt = 0; rt < 2; ++rt) acc[rt][nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(last.a[rt], last.b[nt], acc[rt][nt], 0, 0, 0);

    // ---- epilogue: lane (column m32 of tile nt, half h), register i -> row 32 rt + 8 (i / 4) + 4 h + i % 4.  32 rows x 128 columns
    // turn through this wavefront's own LDS (rows that differ by 4 trade their 32-column halves: no bank conflicts) and
    // leave as whole 512-byte (fp32) or 256-byte (bf16) row segments.
    float *rs = (float *)(smem + kDxWCs) + wave * 64;
    float *ot = (float *)smem + wave * (32 * 128);
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) {
        float r4[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) r4[j] = rowsum[rt][j][0] + rowsum[rt][j][1];
        float r = (r4[0] + r4[1]) + (r4[2] + r4[3]);
        r += __shfl_xor(r, 32, 64);
        if (h == 0) rs[rt * 32 + m32] = r;
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) {
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4) {
            const f32x4 rs4 = *(const f32x4 *)(rs + rt * 32 + 8 * i4 + 4 * h);
#pragma unroll
            for (int nt = 0; nt < 4; ++nt)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int row = 8 * i4 + 4 * h + i;
                    ot[row * 128 + ((nt * 32 + m32) ^ ((row & 4) << 3))] = fmaf(16.f, acc[rt][nt][i4 * 4 + i], -24.f * rs4[i]);
                }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll 4
        for (int pass = 0; pass < 16; ++pass) {
            const int row = pass * 2 + h, col = m32 * 4;
            const int64_t orow = s_orow[wr * 64 + rt * 32 + row];
            const f32x4 v4 = *(const f32x4 *)(ot + row * 128 + (col ^ ((row & 4) << 3)));
            if (orow < 0) continue;
            const int64_t at = orow * K + kb * kDxWTile + wg * 128 + col;
            if (p.out_f32) {
                *(f32x4 *)((float *)p.out + at) = v4;
            } else {
                u32x2 ob;
                ob[0] = (uint32_t)f32_to_bf16_hw(v4[0]) | ((uint32_t)f32_to_bf16_hw(v4[1]) << 16);
                ob[1] = (uint32_t)f32_to_bf16_hw(v4[2]) | ((uint32_t)f32_to_bf16_hw(v4[3]) << 16);
                *(u32x2 *)((uint16_t *)p.out + at) = ob;
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
}

struct DwParams {
    const uint16_t *dy;   // bf16 [M][N], rows grouped by expert
    const uint16_t *x;    // bf16 [x_rows][K]
    const int32_t *row_map;
    const int32_t *offsets;
    void *out;            // [E][N][K]
    int E, N, K, out_f32;
    int chain;            // wide kernel: neighbouring tiles of an expert one workgroup computes
    int heavy_rows;       // wide kernel: an expert with more rows may be heavy; 0: the experts are not looked at
};

__global__ __launch_bounds__(kBwThreads, 4) void grouped_dw_kernel(DwParams p)
{
    __shared__ __attribute__((aligned(16))) unsigned char Ys[kStageM * kTM * 2];   // [64 token rows][128 n] bf16
    __shared__ __attribute__((aligned(16))) unsigned char Xs[kStageM * kTK * 2];   // [64 token rows][128 k] bf16
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int N = p.N, K = p.K;
    const int nbk = K / kTK, nbn = N / kTM;
    const int kb = blockIdx.x % nbk, nb = (blockIdx.x / nbk) % nbn, e = blockIdx.x / (nbk * nbn);
    if (e >= p.E) return;
    const int row0 = p.offsets[e], Me = p.offsets[e + 1] - row0;

    // staging: thread -> token rows tid / 16 and tid / 16 + 32 of the stage, 16-byte piece tid % 16 of their 128
    // columns (16 lanes take 256 contiguous bytes of a row)
    const int sr = tid >> 4, sc = tid & 15;
    const int wn = wave >> 1, wk = wave & 1, m32 = lane & 31, h = lane >> 5;
    f32x16 acc[2];
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[kt][i] = 0.f;

    const TrBase ta = tr_base(wn * 32, lane), tb[2] = {tr_base(wk * 64, lane), tr_base(wk * 64 + 32, lane)};
    // The global loads of a stage (row ids first, then the two tiles) are issued one stage ahead, right after the
    // previous stage's tiles have been written to LDS, so they travel during that stage's matrix phase.
    // (addresses: one pointer per tile and one widening multiply-add per load)
    u32x4 yv[2], xv[2];
    const uint16_t *ybase = p.dy + (int64_t)row0 * N + nb * kTM + sc * 8;
    const uint16_t *xbase = p.x + kb * kTK + sc * 8;
    const int32_t *mbase = p.row_map ? p.row_map + row0 : nullptr;
    auto load_stage = [&](int m0) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int r = m0 + sr + 32 * u;
            yv[u] = u32x4{0, 0, 0, 0};
            xv[u] = u32x4{0, 0, 0, 0};
            if (r < Me) {   // rows past the expert's end contribute zeros
                const uint32_t xrow = mbase ? (uint32_t)mbase[r] : (uint32_t)(row0 + r);
                yv[u] = *(const u32x4 *)(ybase + (uint64_t)(uint32_t)r * (uint32_t)N);
                xv[u] = *(const u32x4 *)(xbase + (uint64_t)xrow * (uint32_t)K);
            }
        }
    };
    load_stage(0);
    for (int m0 = 0; m0 < Me; m0 += kStageM) {
        lds_barrier();   // the matrix phase of the previous stage is done
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int r = sr + 32 * u;
            const int off = r * 256 + ((sc ^ swz_tr(r)) << 4);
            *(u32x4 *)(Ys + off) = yv[u];
            *(u32x4 *)(Xs + off) = xv[u];
        }
        if (m0 + kStageM < Me) load_stage(m0 + kStageM);
        lds_barrier();
        static_for<0, kStageM / 16>([&](auto st_c) {
            constexpr int st = decltype(st_c)::value;
            const bf16x8 a = read_operand_tr<st>(Ys, ta);
#pragma unroll
            for (int kt = 0; kt < 2; ++kt) {
                const bf16x8 b = read_operand_tr<st>(Xs, tb[kt]);
                acc[kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc[kt], 0, 0, 0);
            }
        });
    }
    // lane (column m32 of tile kt, half h), register i -> weight row 32 wn + 8 (i / 4) + 4 h + i % 4
    const int64_t obase = ((int64_t)e * N + nb * kTM + wn * 32 + 4 * h) * K + kb * kTK + wk * 64 + m32;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const uint32_t orow = (uint32_t)(8 * (i >> 2) + (i & 3)) * (uint32_t)K;
#pragma unroll
        for (int kt = 0; kt < 2; ++kt) {
            if (p.out_f32) ((float *)p.out + obase)[orow + kt * 32] = acc[kt][i];
            else ((uint16_t *)p.out + obase)[orow + kt * 32] = f32_to_bf16_hw(acc[kt][i]);
        }
    }
}


// ---- dW on 256 x 256 tiles: the structure of the LM head kernel (logprob.hip) with the token index as the
// contraction.  A stage holds 64 token rows of both operands as they are stored, Ys [64][256 n] and Xs [64][256 k]
// (512-byte rows, 64 KiB per stage, two stages), filled by asynchronous global -> LDS copies: a wavefront instruction
// moves two rows; chunk q (16 bytes) of row r sits at position q ^ ((r & 3) << 2) of the row, so that the four rows
// a transposing read touches at once lie in different quarters of the 256 bytes the LDS serves per clock.  Rows past
// the expert's end are copied from a row of zeros.  Eight wavefronts of 128 n x 64 k (4 x 2 MFMA tiles, 128
// accumulator registers); the twelve transposing reads of a 16-token slice go out one pair behind each of the first
// six MFMAs of the slice before, the eight copies of the next stage one behind every second MFMA of the first two
// slices, the last slice's MFMAs run behind the stage barrier.  The x rows are gathered through row_map; the ids
// are the same for all lanes of a wavefront and are read with scalar loads (vector loads would share the counter
// the copies are waited on with) one stage before they are turned into addresses.
constexpr int kDwWTile = 256;                       // n rows and k columns per workgroup
constexpr int kDwWRowB = kDwWTile * 2;              // bytes of an LDS row
constexpr int kDwWTileB = kStageM * kDwWRowB;       // one operand tile of a stage: 32 KiB
constexpr int kDwWStageB = 2 * kDwWTileB;           // Ys, then Xs
constexpr int kDwRankE = 256;                       // experts that are put in order
__host__ __device__ inline bool dw_wide_by_xcd(int N, int K) { return (N / kDwWTile) % 2 == 0 && (K / kDwWTile) % 4 == 0; }
__device__ __attribute__((aligned(256))) const unsigned char kDwZeroRow[kDwWRowB] = {0};

__device__ __forceinline__ TrBase tr_base_512(int col0, int lane)
{
    const int r16 = lane & 15, g = lane >> 4;
    const int row = 8 * (g >> 1) + (r16 >> 2);                // the row this lane ADDRESSES (second read: + 4)
    const int colq = col0 + 16 * (g & 1) + 4 * (r16 & 3);     // first of the four columns it addresses
    TrBase b;
    b.lo = row * kDwWRowB + (((colq >> 3) ^ ((row & 3) << 2)) << 4) + (colq & 4) * 2;
    b.hi = b.lo + 4 * kDwWRowB;                               // row + 4: same row & 3, same swizzle
    return b;
}

// kOrdered: more than one tile per workgroup or an order of the experts (p.chain > 1 or p.heavy_rows > 0); else tile = workgroup.
template <bool kOrdered>
__global__ __launch_bounds__(kBwThreads, 2) void grouped_dw_wide_kernel(DwParams p, const int32_t *__restrict__ row_map,
                                                                        const int32_t *__restrict__ offsets)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn = wave >> 2, wk = wave & 3;   // 128 n x 64 k per wavefront
    const int h = lane >> 5;
    const int N = p.N, K = p.K;
    const int nbn = N / kDwWTile, nbk = K / kDwWTile;
    // Lists of tiles.  Consecutive workgroup ids go round-robin over the eight XCDs; where the tile grid allows it an XCD
    // has its own list with half of the n blocks and a quarter of the k blocks of every expert, so that a skewed router
    // loads the XCDs alike and an XCD's L2 fetches a fifth of the expert's operand bytes, not all.
    const bool by_xcd = dw_wide_by_xcd(N, K);
    const int xcd = by_xcd ? blockIdx.x % 8 : 0, first = by_xcd ? blockIdx.x / 8 : blockIdx.x;
    const int hn = by_xcd ? nbn / 2 : nbn, per = by_xcd ? nbn * nbk / 8 : nbn * nbk;   // n blocks, tiles per expert of the list
    // Items of the list: one tile of a heavy expert (below), p.chain neighbouring tiles of another.  The workgroups of the
    // list take item `first`, then (heavy experts make more items than workgroups) go back and forth over the rest.
    const int chain0 = kOrdered ? p.chain : 1;
    const int wpe = kOrdered ? (per + chain0 - 1) / chain0 : per;
    const int wgs = by_xcd ? gridDim.x / 8 : gridDim.x;   // E wpe

    // ---- copies: instruction i (0..3) of this wavefront moves rows 8 w + 2 i and 8 w + 2 i + 1 of a tile; lane L
    // fills position L % 32 of row 8 w + 2 i + L / 32 with the chunk that belongs there
    int rrow[4];
    uint32_t chunkb[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        rrow[i] = wave * 8 + 2 * i + h;
        chunkb[i] = (uint32_t)(((lane & 31) ^ ((rrow[i] & 3) << 2)) << 4);
    }
    int row0 = 0, Me = 0, stages = 0;   // of the item's expert
    const unsigned char *ybase = nullptr, *xbase = nullptr;
    const int32_t *mbase = nullptr;
    int32_t ids[8];                       // x rows of the wavefront's eight token rows of the stage addressed next
    const unsigned char *ysrc[4], *xsrc[4];
    auto load_ids = [&](int s) {
        const int m0 = s * kStageM + wave * 8;
        if (mbase) {
#pragma unroll
            for (int r = 0; r < 8; ++r) ids[r] = mbase[min(m0 + r, Me - 1)];
        } else {
#pragma unroll
            for (int r = 0; r < 8; ++r) ids[r] = row0 + m0 + r;
        }
    };
    auto form_addresses = [&](int s) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int m = s * kStageM + rrow[i];
            const bool valid = m < Me;
            const int id = h ? ids[2 * i + 1] : ids[2 * i];
            ysrc[i] = valid ? ybase + (uint64_t)(uint32_t)m * (uint32_t)(N * 2) + chunkb[i] : kDwZeroRow + chunkb[i];
            xsrc[i] = valid ? xbase + (uint64_t)(uint32_t)id * (uint32_t)(K * 2) + chunkb[i] : kDwZeroRow + chunkb[i];
        }
    };
    auto copy_one = [&](int buf, int i) {   // i = 0..3: Ys, 4..7: Xs
        unsigned char *dst = smem + buf * kDwWStageB + (wave * 8 + 2 * (i & 3)) * kDwWRowB;
        if (i < 4) copy16_to_lds(ysrc[i], dst);
        else copy16_to_lds(xsrc[i - 4], dst + kDwWTileB);
    };

    // ---- operands: transposing reads, n columns 128 wn + 32 ms of Ys and k columns 64 wk + 32 nt of Xs
    TrBase ta[4], tb[2];
#pragma unroll
    for (int ms = 0; ms < 4; ++ms) ta[ms] = tr_base_512(wn * 128 + ms * 32, lane);
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) {
        tb[nt] = tr_base_512(wk * 64 + nt * 32, lane);
        tb[nt].lo += kDwWTileB;
        tb[nt].hi += kDwWTileB;
    }
    struct Frags {
        bf16x8 a[4], b[2];
    };
    // The transposing reads are written as asm: in front of a read the compiler can see it drains the asynchronous
    // copies in flight (it cannot tell that they fill the other stage buffer).  The results are therefore waited for
    // by hand: wait_frags() in front of the slice that multiplies them.
    const uint32_t lds0 = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void *)smem;
    auto read_tr = [&](uint32_t base, const TrBase &t, auto off_c) -> bf16x8 {
        constexpr int off = decltype(off_c)::value;
        struct {
            s16x4 lo, hi;
        } v;
        asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(v.lo) : "v"(base + (uint32_t)t.lo), "n"(off));
        asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(v.hi) : "v"(base + (uint32_t)t.hi), "n"(off));
        return __builtin_bit_cast(bf16x8, v);
    };
    auto wait_frags = [&](Frags &f) {
        asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(f.a[0]), "+v"(f.a[1]), "+v"(f.a[2]), "+v"(f.a[3]), "+v"(f.b[0]), "+v"(f.b[1]));
    };
    f32x16 acc[4][2];
    // Slice j (16 token rows) of stage ks: the eight MFMAs on `cur`, behind each of the first six one operand of
    // `nxt` (two transposing reads), in slices 0 and 1 behind every second MFMA one copy of the next stage.
    auto slice = [&](Frags &cur, Frags &nxt, int ks, auto j_c, auto more_t) {
        constexpr int j = decltype(j_c)::value;
        const int buf = ks & 1;
        const uint32_t base = lds0 + buf * kDwWStageB;
        constexpr std::integral_constant<int, j * 16 * kDwWRowB> off{};
        wait_frags(cur);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int ms = i >> 1, nt = i & 1;
            acc[ms][nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(cur.a[ms], cur.b[nt], acc[ms][nt], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            if (i < 4) nxt.a[i] = read_tr(base, ta[i], off);
            else if (i < 6) nxt.b[i - 4] = read_tr(base, tb[i - 4], off);
            if (decltype(more_t)::value && j < 2 && (i & 1)) copy_one(buf ^ 1, 4 * j + (i >> 1));
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    auto stage_barrier = [&]() {   // own copies landed, own operand reads done; then everybody's
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    };

    // Tile t of the expert: blocks and operand bases, and the copies of its first stage into buffer 0
    int nb = 0, kb = 0;
    auto begin_tile = [&](int t) {
        nb = (xcd & 1) * hn + t % hn;
        kb = (xcd >> 1) * (nbk / 4) + t / hn;
        if (stages == 0) return;
        ybase = (const unsigned char *)p.dy + ((int64_t)row0 * N + nb * kDwWTile) * 2;
        xbase = (const unsigned char *)p.x + (int64_t)kb * kDwWTile * 2;
        load_ids(0);
        form_addresses(0);
#pragma unroll
        for (int i = 0; i < 8; ++i) copy_one(0, i);
        load_ids(1);
    };
    int e, t0, t1;
    auto begin_item = [&](int expert, int item, int chain) {   // item: of the expert
        e = expert;
        t0 = item * chain;
        t1 = kOrdered ? min(t0 + chain, per) : t0 + 1;
        row0 = offsets[e];
        Me = offsets[e + 1] - row0;
        stages = (Me + kStageM - 1) / kStageM;
        mbase = row_map ? row_map + row0 : nullptr;
        begin_tile(t0);
    };
    // Heavy experts: more than twice the mean of rows, and more than heavy_rows.  If there are any, the experts are taken in
    // descending order of their rows (ties by id), so that what starts last is short; in the order of their ids a
    // popular expert's tiles (0.5 ms each under a Zipf router of 16384 tokens) may start when the others are done: 1.25 ->
    // 1.02 ms for gate_up.  Without heavy experts the order of the ids stays, and the first item's copies, which are
    // issued before the counts are looked at, are the right ones.
    int cnt[kDwRankE / 64];
#pragma unroll
    for (int q = 0; q < kDwRankE / 64; ++q) {
        const int ex = q * 64 + lane;
        cnt[q] = kOrdered && p.heavy_rows > 0 && ex < p.E ? p.offsets[ex + 1] - p.offsets[ex] : 0;
    }
    __builtin_amdgcn_sched_barrier(0);
    begin_item(first / wpe, first % wpe, chain0);
    bool begun = true;
    int n_heavy = 0;
    if (kOrdered && p.heavy_rows > 0) {
        const int64_t twice = 2 * (int64_t)(offsets[p.E] - offsets[0]);
#pragma unroll
        for (int q = 0; q < kDwRankE / 64; ++q) n_heavy += __popcll(__ballot(cnt[q] > p.heavy_rows && (int64_t)cnt[q] * p.E > twice));
    }
    __shared__ __attribute__((aligned(16))) int s_key[kDwRankE];
    __shared__ int s_rank[kDwRankE], s_order[kDwRankE];
    if (kOrdered && n_heavy > 0) {   // a thread counts the larger keys among a part of the experts for one of them
        const int ep = p.E <= 128 ? 128 : 256, i = tid & (ep - 1), len = ep * ep / kBwThreads, j0 = (tid / ep) * len;
        if (tid < ep) {
            const int rows = tid < p.E ? min(offsets[tid + 1] - offsets[tid], 0x7ffffe) : -1;
            s_key[tid] = rows * 256 + 255 - tid;   // padding: below every expert's key
            s_rank[tid] = 0;
        }
        lds_barrier();
        const int key = s_key[i];
        int larger = 0;
        for (int j = 0; j < len; j += 4) {
            const i32x4 k4 = *(const i32x4 *)(s_key + j0 + j);
#pragma unroll
            for (int q = 0; q < 4; ++q) larger += k4[q] > key;
        }
        atomicAdd(&s_rank[i], larger);
        lds_barrier();
        if (tid < p.E) s_order[s_rank[tid]] = tid;
        stage_barrier();   // also: the copies of the item that is given up have landed
        begun = false;
    }
    const int n_items = n_heavy * per + (p.E - n_heavy) * wpe;
    for (int round = 0; kOrdered ? round * wgs < n_items : round < 1; ++round) {
        if (kOrdered && !begun) {
            const int idx = round * wgs + ((round & 1) ? wgs - 1 - first : first);
            if (idx >= n_items) continue;
            const bool light = idx >= n_heavy * per;
            const int li = light ? idx - n_heavy * per : idx, w = light ? wpe : per;
            const int r = (light ? n_heavy : 0) + li / w;
            if (round > 0) lds_barrier();   // the last item's epilogue has left the buffers
            begin_item(n_heavy > 0 ? __builtin_amdgcn_readfirstlane(s_order[r]) : r, li % w, light ? chain0 : 1);
        }
        begun = false;
        for (int t = t0; kOrdered ? t < t1 : t == t0; ++t) {
            const int64_t obase = ((int64_t)e * N + nb * kDwWTile + wn * 128) * K + kb * kDwWTile + wk * 64;
#pragma unroll
            for (int ms = 0; ms < 4; ++ms)
#pragma unroll
                for (int nt = 0; nt < 2; ++nt)
#pragma unroll
                    for (int i = 0; i < 16; ++i) acc[ms][nt][i] = 0.f;
            if (stages > 0) {
                Frags last, f0, f1, f2, f3;
#pragma unroll
                for (int i = 0; i < 4; ++i) last.a[i] = bf16x8{0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
                for (int i = 0; i < 2; ++i) last.b[i] = bf16x8{0, 0, 0, 0, 0, 0, 0, 0};
                stage_barrier();   // the first stage has landed; the last tile's epilogue has left the second buffer
                auto stage = [&](int ks, auto more_t) {
                    if (decltype(more_t)::value) {
                        form_addresses(ks + 1);   // from the ids loaded during the stage before
                        load_ids(ks + 2);
                    }
                    slice(last, f0, ks, std::integral_constant<int, 0>{}, more_t);
                    slice(f0, f1, ks, std::integral_constant<int, 1>{}, more_t);
                    slice(f1, f2, ks, std::integral_constant<int, 2>{}, more_t);
                    slice(f2, f3, ks, std::integral_constant<int, 3>{}, more_t);
                    stage_barrier();
                    last = f3;
                };
                for (int ks = 0; ks + 1 < stages; ++ks) stage(ks, std::true_type{});
                stage(stages - 1, std::false_type{});
                wait_frags(last);
#pragma unroll
                for (int ms = 0; ms < 4; ++ms)
#pragma unroll
                    for (int nt = 0; nt < 2; ++nt)
                        acc[ms][nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(last.a[ms], last.b[nt], acc[ms][nt], 0, 0, 0);
            }
            if (kOrdered && t + 1 < t1) begin_tile(t + 1);   // travels during the epilogue, which keeps to the second buffer

            // ---- epilogue: lane (k column m32 of tile nt, half h), register i -> weight row 32 ms + 8 (i / 4) + 4 h + i % 4.
            // 32 rows x 64 columns turn through this wavefront's own piece of the second stage buffer (rows that differ by 4
            // trade their halves: no bank conflicts) and leave as whole 256-byte (fp32) or 128-byte (bf16) row segments.
            int el = lane;   // opaque: addresses worked out here, not kept in registers across the k loop
            asm volatile("" : "+v"(el));
            const int ec = el & 31, eh = el >> 5;
            const int esz = p.out_f32 ? 4 : 2;
            unsigned char *dst = (unsigned char *)p.out + (obase + (int64_t)(el >> 4) * K + (el & 15) * 4) * esz;   // row el / 16
            const int64_t step = (int64_t)4 * K * esz;
            float *ot = (float *)(smem + kDwWStageB) + wave * (32 * 64);
#pragma unroll
            for (int ms = 0; ms < 4; ++ms) {
#pragma unroll
                for (int nt = 0; nt < 2; ++nt)
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const int row = 8 * (i >> 2) + 4 * eh + (i & 3);
                        ot[row * 64 + ((nt * 32 + ec) ^ ((row & 4) << 3))] = acc[ms][nt][i];
                    }
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
                for (int pass = 0; pass < 8; ++pass) {
                    const int row = pass * 4 + (el >> 4);
                    const f32x4 v4 = *(const f32x4 *)(ot + row * 64 + (((el & 15) * 4) ^ ((row & 4) << 3)));
                    if (p.out_f32) {
                        *(f32x4 *)dst = v4;
                    } else {
                        u32x2 ob;
                        ob[0] = (uint32_t)f32_to_bf16_hw(v4[0]) | ((uint32_t)f32_to_bf16_hw(v4[1]) << 16);
                        ob[1] = (uint32_t)f32_to_bf16_hw(v4[2]) | ((uint32_t)f32_to_bf16_hw(v4[3]) << 16);
                        *(u32x2 *)dst = ob;
                    }
                    dst += step;
                }
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            }
        }
    }
}

}  // namespace

// The 256 x 256 tiles take 0.8-0.95 of the 128 x 128 ones' time on a full chip, but a tile is four times the work and there is one per CU:
// from 512 rows per expert (a partial tile hurts less) and three rounds of workgroups on (half a tile more per expert than the rows
// fill).  us, 128 x 128 against 256 x 256, 128 experts, even / Zipf router: gate_up (N 1536, K 2048) 2048 tokens
// 204 / 229 against 194 / 255, 4096 343 / 364 against 304 / 373, 8192 640 / 660 against 542 / 565, 16384 (Zipf) 1332 against
// 1110; down (N 2048, K 768) 4096 170 / 185 against 178 / 193, 8192 301 / 322 against 273 / 302; 64 experts (N 1024, K 512), two
// rounds: 61 against 73.
static bool dx_wide(const GemmArgs &a)
{
    return a.K % kDxWTile == 0 && dx_wide_lds(a.N) + 4 * kDxWTile <= (size_t)kMaxLdsBytes && a.M >= (int64_t)a.E * 512 &&
           (a.M / kDxWTile + a.E / 2) * (a.K / kDxWTile) >= 3 * 256;
}

int launch_qgemm_dx(const GemmArgs &a, hipStream_t s)
{
    if (a.E > 256 || a.N % kStageN != 0 || a.K % kTK != 0 || a.N > 8192) {
        set_error("qgemm dx: needs E <= 256, N %% 128 == 0, N <= 8192, K %% 128 == 0 (got E=%d N=%d K=%d)", a.E, a.N, a.K);
        return QARL_ERR_UNSUPPORTED;
    }
    DxParams p;
    p.codes = (const uint32_t *)a.codes;
    p.scales = (const uint16_t *)a.scales;
    p.dy = (const uint16_t *)a.x;
    p.offsets = a.offsets;
    p.out_row_map = a.out_row_map;
    p.out = a.out;
    p.E = a.E;
    p.N = a.N;
    p.K = a.K;
    p.out_f32 = a.out_f32;
    const bool wide = dx_wide(a);
    const int tm = wide ? kDxWTile : kTM, tk = wide ? kDxWTile : kTK;
    const int64_t slots = (a.M + tm - 1) / tm + a.E;
    const int64_t total = ((slots * (a.K / tk) + 7) / 8) * 8;
    if (total > 0x7fffffffLL) {
        set_error("qgemm dx: grid too large");
        return QARL_ERR_UNSUPPORTED;
    }
    if (wide) {
        static LdsLimitOnce once;
        if (int rc = raise_lds_limit((const void *)qgemm_dx_wide_kernel, once, "hipFuncSetAttribute(qgemm dx wide)")) return rc;
        qgemm_dx_wide_kernel<<<dim3((unsigned)total), dim3(kBwThreads), dx_wide_lds(a.N), s>>>(p);
        return check_hip(hipGetLastError(), "qgemm_dx_wide_kernel");
    }
    const size_t lds = (size_t)(kTM + kTK) * kStageN * 2 + (size_t)a.N * 4;
    static LdsLimitOnce once;
    if (int rc = raise_lds_limit((const void *)qgemm_dx_kernel, once, "hipFuncSetAttribute(qgemm dx)")) return rc;
    qgemm_dx_kernel<<<dim3((unsigned)total), dim3(kBwThreads), lds, s>>>(p);
    return check_hip(hipGetLastError(), "qgemm_dx_kernel");
}

int launch_grouped_dw(const void *dy, const void *x, const int32_t *row_map, const int32_t *offsets, int64_t M, int E, int N,
                      int K, void *out, int out_f32, hipStream_t s)
{
    if (N % kTM != 0 || K % kTK != 0) {
        set_error("grouped dw: needs N %% 128 == 0 and K %% 128 == 0 (got N=%d K=%d)", N, K);
        return QARL_ERR_UNSUPPORTED;
    }
    const int64_t grid = (int64_t)E * (N / kTM) * (K / kTK);
    if (grid > 0x7fffffffLL) {
        set_error("grouped dw: grid too large");
        return QARL_ERR_UNSUPPORTED;
    }
    DwParams p;
    p.dy = (const uint16_t *)dy;
    p.x = (const uint16_t *)x;
    p.row_map = row_map;
    p.offsets = offsets;
    p.out = out;
    p.E = E;
    p.N = N;
    p.K = K;
    p.out_f32 = out_f32;
    p.chain = 1;
    p.heavy_rows = 0;
    // 256 x 256 tiles, but not for up to four rounds of workgroups with few rows each: there a tile is mostly start-up and
    // result, of which the two smaller workgroups of a CU hide each other's (64 experts, 512 x 1024 weights: 51 instead of
    // 58 us at 62 rows per expert, popular experts; 57 instead of 56 at 125, even experts; from 1500 tiles on 124 instead of
    // 110 us at 62)
    const int64_t wide_tiles = (int64_t)E * (N / kDwWTile) * (K / kDwWTile);
    const bool few = wide_tiles <= 4 * 256 && M < (int64_t)96 * E;
    if (!few && N % kDwWTile == 0 && K % kDwWTile == 0 && (int64_t)N * 2 < (1LL << 31) && (int64_t)K * 2 < (1LL << 31)) {
        // Tiles of a workgroup: up to three, as long as six rounds of workgroups remain.  Chains and an order of the experts
        // cost a tile 1 us (scalar registers spill, the loops start cold), looking for heavy experts another 0.5 and ranking
        // them 1: worth it where the order of the work matters.  Chained tiles: heavy experts from 4 stages on, if there are
        // rows enough for one (512 tokens, top-4, popular experts, 128 of 1536 x 2048: 201 us in the order of their ids, 226
        // ranked; 1024 tokens: 258, 244).  Single tiles: from four rounds and 128 rows per expert on, heavy from 16 stages on;
        // 1024 tiles, 187 rows per expert: popular experts 157 -> 142 us, 121 -> 122 without.  There not for few experts, whose
        // workgroups all meet the heavy one (8 of 4096 x 4096, 187 rows: 98 us unordered, 107 ordered), and not for more than
        // 128, whose heavy ones have few tiles each (256 of 512 x 1024, 187 rows, even 123 and 140, popular 336 either way).
        const int lists = dw_wide_by_xcd(N, K) ? 8 : 1;
        const int64_t per = wide_tiles / E / lists;
        p.chain = E > kDwRankE ? 1 : (int)std::min<int64_t>(std::min<int64_t>(3, per), std::max<int64_t>(1, wide_tiles / (6 * 256)));
        const bool single = E >= 16 && E <= 128 && M >= (int64_t)128 * E && wide_tiles >= 4 * 256;
        p.heavy_rows = E > kDwRankE ? 0 : p.chain > 1 ? (M >= 3072 ? 3 * kStageM : 0) : single ? 15 * kStageM : 0;
        const int64_t total = lists * E * ((per + p.chain - 1) / p.chain);
        static LdsLimitOnce once[2];
        const bool ordered = p.chain > 1 || p.heavy_rows > 0;
        auto kern = ordered ? grouped_dw_wide_kernel<true> : grouped_dw_wide_kernel<false>;
        if (int rc = raise_lds_limit((const void *)kern, once[ordered], "hipFuncSetAttribute(grouped dw)")) return rc;
        kern<<<dim3((unsigned)total), dim3(kBwThreads), 2 * kDwWStageB, s>>>(p, row_map, offsets);
        return check_hip(hipGetLastError(), "grouped_dw_wide_kernel");
    }
    grouped_dw_kernel<<<dim3((unsigned)grid), dim3(kBwThreads), 0, s>>>(p);
    return check_hip(hipGetLastError(), "grouped_dw_kernel");
}

}  // namespace qarl
