// Grouped quantized GEMM, weight-streaming ("decode") path for the FP8 format: eq. (2) of
// section 2.2 when every expert sees only a few token rows, so the kernel is bound by
// reading each expert's e4m3 weights from HBM exactly once (the regime the paper's
// appendix on quantization schemes calls memory-bound).  The W4A16 format has its own
// kernel (qgemm_stream_w4.hip).  Two sources instantiate the kernel: qgemm_stream_fp8.hip (e4m3 codes; the dispatch of the streaming path
// is there too) and qgemm_stream_fp4.hip (e2m1 codes).
//
// Work layout.  A workgroup of 8 wavefronts owns (expert, slice of its weight rows, block
// of <= 16*MT token rows).  It gathers its e4m3 token rows ONCE into LDS for the whole K;
// after that single barrier every wavefront runs on its own: it walks its pairs of 16-row
// weight tiles and, per pair, K in steps, with the codes of the next R steps always in
// flight in a ring of the wavefront's own.  Codes and token rows meet as stored in
// v_mfma_f32_16x16x32_fp8_fp8; the row scale s_x and the channel scale s_w are applied to
// the fp32 sums in the epilogue.
//
// The ring has two forms.  Routed calls keep it in LDS where it fits beside the token tile
// (below).  Grouped calls, and routed ones whose ring does not fit or that have fewer steps
// than it, keep it in registers: steps of 128 k, two 16-byte loads per lane, tile and step
// (e2m1: one), lane (c, q) reads k in [128 g + 32 q, +32) of row c.
//
// Experts with more than 16*MT rows: the grid carries m_split row blocks per (expert,
// slice), mapped to consecutive workgroups of the same XCD so that their identical weight
// reads meet in that XCD's L2; rows beyond 16*MT*m_split take further passes, or, in the
// routed mode, are dealt to the workgroups without rows and those of the popular experts
// (routed_rows.hpp).
//
// Ring in LDS (routed mode, where it fits beside the token tile).  A load into registers in the layout of the matrix instruction takes 64 bytes of
// each of 16 rows, half lines; an asynchronous copy to LDS can take whole 128-byte lines of 8 rows and be nontemporal (a nontemporal
// half line is fetched twice).  402 MB in tiles of 16 rows, 8 KiB per wavefront in flight: register loads 5.97 TB/s, nontemporal 5.86, copies of
// half lines 5.84, of whole lines 6.00, of whole lines nontemporal 6.80.  A wavefront has a ring of its own (two stages of 4 KiB: 128 bytes of
// k of both tiles), reads a stage into registers as soon as it has landed and refills it at once: nothing in the stream waits for another
// wavefront.  Layer of 128 experts 2048 x 768, top-8, even router, us, registers -> ring: FP8 12 tokens 95 -> 71, 37 114 -> 94, 100 128 -> 109,
// 256 138 -> 119, FP4 63 -> 48, 72 -> 58, 82 -> 69, 90 -> 78; 64 experts 1024 x 512, top-4, 512 tokens FP8 51 -> 42, FP4 42 -> 40; Zipf router 256 tokens
// FP8 119 -> 107, FP4 87 -> 78.  Three stages: 4 % slower in the mean.  Blocks of 64 rows of long K (2048; the line is near 1400 and falls with N) leave no room and keep the registers.
//
// Routed mode (QX): the kernel is driven by the router's ids and by 16-bit activations.  Every
// workgroup lists its expert's (token, slot) pairs itself and quantizes the token rows it
// gathers with the row quantizer's own arithmetic (one wavefront per row: absmax, s_x =
// absmax / 448, e4m3 codes of x / s_x), so a decode step needs neither a grouping pass nor an
// activation-quantizer launch between the router and the two expert GEMMs, and its results
// equal theirs bit for bit.
#pragma once
#include <type_traits>

#include "routed_rows.hpp"

namespace qarl {

namespace stream8 {

constexpr int kSThreads = 512;
constexpr int kSWaves = 8;

struct StreamParams {
    const uint32_t *codes;   // e4m3 bytes viewed as words [E][N][K/4]
    const float *scales;     // [E][N]
    const void *x;           // e4m3 rows
    const float *x_scales;
    const int32_t *row_map;
    const int32_t *out_row_map;
    const int32_t *offsets;
    void *out;
    int E, N, K, out_f32;
    int n_units;     // pairs of 16-row weight tiles per expert
    int n_slices;    // workgroups along the weight rows of one expert
    int m_split;     // row blocks per (expert, slice) in the grid
    int w4;          // weights are packed e2m1 codes [E][N][K/8] words
    // routed mode: x is bf16; row = pair id t * topk + slot of expert ids[row], activation row t (x_per_token)
    // or the pair id, output row = pair id
    const int32_t *ids;
    int n_ids, topk, x_per_token;
    int spread;      // row blocks beyond the grid's are dealt out (spread_item)
};

// LDS bytes per activation row: the row plus 16 bytes, so consecutive rows skew by 4 banks.
__host__ __device__ constexpr int x_stride(int K) { return K + 16; }

// Dynamic LDS of a workgroup: row ids, output rows, row scales, pair counter, token tile.
inline size_t stream_lds_bytes(int K, int MT, bool routed = false)
{
    const size_t rows = (size_t)MT * 16;
    return rows * 12 + 16 + rows * x_stride(K) + (routed ? (size_t)kIdsBytes : 0);
}

// Ring in LDS: stages of a wavefront, and the place behind the token tile and the lists of the routed mode.
constexpr int kLrStages = 2;
__host__ __device__ constexpr int lr_ring_at(int K, int MT) { return (MT * 16 * 12 + 16 + MT * 16 * x_stride(K) + kIdsBytes + 127) & ~127; }

// LDS stores and the draw of a pair the compiler does not see as such: in front of those it sees it waits for every copy in flight.
__device__ __forceinline__ uint32_t lds_addr(const void *p) { return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void *)p; }
__device__ __forceinline__ void lds_store8(void *p, u32x2 v) { asm volatile("ds_write_b64 %0, %1" ::"v"(lds_addr(p)), "v"(v) : "memory"); }
__device__ __forceinline__ void lds_store4(void *p, uint32_t v) { asm volatile("ds_write_b32 %0, %1" ::"v"(lds_addr(p)), "v"(v) : "memory"); }
__device__ __forceinline__ int lds_draw(int *p)
{
    int v;
    asm volatile("ds_add_rtn_u32 %0, %1, %2\n\ts_waitcnt lgkmcnt(0)" : "=&v"(v) : "v"(lds_addr(p)), "v"(1) : "memory");
    return v;
}

// EPI: NONE or SILU_MUL; MT: 16-row token tiles per block; R: ring depth in 128-k steps (must divide K/128);
// W4: the weights are packed e2m1 codes (half a byte per weight) instead of e4m3 bytes; QX: routed mode;
// SPREAD (with QX): the row blocks beyond the grid's are dealt out (spread_item) instead of being further passes.
// TAIL: the shares of popular experts, after the workgroup's own row block; returns whether to go on with them.
// LR: 0 the ring is in registers; 1, 2 in LDS, R stages, 2: nontemporal (no other row block reads the same weights; the shares of popular experts
// do: with temporal copies there the Zipf router's 256 tokens take FP8 107 us per layer instead of 116).
template <int EPI, int MT, int R, bool W4, bool QX, int LR, bool SPREAD, bool TAIL>
__device__ __forceinline__ bool stream_fp8_body(const StreamParams &p, int tid, unsigned bid)
{
    extern __shared__ __attribute__((aligned(128))) unsigned char smem[];
    constexpr int kRowsMax = MT * 16;
    static_assert(LR == 0 || QX, "the ring in LDS belongs to the routed mode");

    const int lane = tid & 63, wave = tid >> 6;
    const int c = lane & 15, q = lane >> 4;
    const int N = p.N, K = p.K, G = K / kGroup;
    const int stride = x_stride(K);

    // workgroup id -> (expert, slice, row block).  Ids go round-robin over the 8 XCDs; the row
    // blocks of one (expert, slice) take consecutive positions on the same XCD.
    const int xcd = (int)(bid & 7), pos = (int)(bid >> 3);
    const int mh = pos % p.m_split;
    const int unit_id = (pos / p.m_split) * 8 + xcd;
    if (unit_id >= p.E * p.n_slices) return false;
    int e = unit_id / p.n_slices;
    const int slice = unit_id % p.n_slices;

    int *s_row = (int *)smem;                              // [kRowsMax] activation row of each tile row
    int *s_orow = (int *)(smem + kRowsMax * 4);            // [kRowsMax] output row, -1 past the expert's last row
    float *s_xs = (float *)(smem + kRowsMax * 8);          // [kRowsMax] activation scale of the row
    int *s_next = (int *)(smem + kRowsMax * 12);           // next undrawn pair
    unsigned char *xs = smem + kRowsMax * 12 + 16;         // [kRowsMax][stride]

    // this workgroup's pairs of weight tiles: units u_lo .. u_hi-1
    const int per_slice = (p.n_units + p.n_slices - 1) / p.n_slices;
    int u_lo = slice * per_slice, n_pairs = max(0, min(p.n_units, u_lo + per_slice) - u_lo);  // pairs of this workgroup; wavefronts draw them from an LDS counter
    const int words_per_row = W4 ? K / 8 : K / 4;
    int64_t ebase = (int64_t)e * N;

    auto tile_row = [&](int pi, int nt) -> int {  // weight row of this lane in tile nt of the slice's pi-th pair
        const int u = u_lo + pi;
        if (EPI == QARL_EPI_SILU_MUL) return (nt ? N / 2 : 0) + u * 16 + c;
        return u * 32 + nt * 16 + c;
    };

    constexpr int kH = W4 ? 1 : 2;   // 16-byte loads per lane, tile and 128-k step: 32 weights of one row
    struct Slot {
        u32x4 w[2][kH];
    };
    Slot ring[LR ? 1 : R];
    // Base pointer of the R-step batch (pair pi, steps g0..) of tile nt for this lane.  Past this
    // wavefront's work the pointer falls back to the start of the expert's codes: the ring is refilled
    // without a branch (a conditional refill turns every slot into a merge of old and new value and
    // doubles the registers the ring takes), and those few loads all hit one cached line.
    auto batch_src = [&](int pi, int g0, int nt) -> const uint32_t * {
        const bool ok = pi < n_pairs;
        const int64_t row = ebase + (ok ? tile_row(pi, nt) : c);
        return p.codes + row * words_per_row + (ok ? g0 * (8 * kH * 2) + q * (4 * kH) : 0);
    };
    // Plain (temporal) loads on purpose: with row-major codes one load instruction takes half of each
    // 128-byte line it touches and the h = 1 load the other half.  A nontemporal load drops the line
    // after the first half and fetches it again for the second (measured: 7 % of the 256-token layer,
    // 16 % at 512 tokens).
    auto fill = [&](Slot &dst, int r, const uint32_t *const (&src)[2]) {
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
#pragma unroll
            for (int h = 0; h < kH; ++h) dst.w[nt][h] = *(const u32x4 *)(src[nt] + r * (16 * kH) + h * 4);
    };
    auto fill_ring = [&](int pi, int g0) {
        const uint32_t *src[2] = {batch_src(pi, g0, 0), batch_src(pi, g0, 1)};
#pragma unroll
        for (int r = 0; r < R; ++r) fill(ring[r], r, src);
    };

    // ---- ring in LDS (LR): a wavefront's own R stages of 4 KiB, 128 bytes of k of both tiles of its pair, in whole 128-byte lines: an
    // instruction copies 8 rows, chunk b (16 bytes) of row r to position b ^ ((r >> 1) & 7) of the row.
    const int n_steps = K / (W4 ? 256 : 128);
    const uint32_t rowb = (uint32_t)words_per_row * 4u;
    unsigned char *lring = smem + lr_ring_at(K, MT) + wave * (R * 4096);
    float *s_sw = (float *)(smem + lr_ring_at(K, MT) + kSWaves * R * 4096);   // [pairs][2][16] channel scales of the slice
    uint32_t voff[2], roff[2];
    if constexpr (LR != 0) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            voff[i] = (uint32_t)(i * 8 + (lane >> 3)) * rowb + (uint32_t)(((lane & 7) ^ ((4 * i + (lane >> 4)) & 7)) << 4);
            // operand reads: 16-byte chunks 2 q + i (e4m3), 4 i + q (e2m1: 128-k half i) of row c
            roff[i] = (uint32_t)(c * 128 + (((W4 ? 4 * i + q : 2 * q + i) ^ ((c >> 1) & 7)) << 4));
        }
    }
    auto copy_step = [&](int pi, int st, int slot) {   // past this wavefront's work: the expert's first rows (cached)
        const bool ok = pi < n_pairs;
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
            const int u = u_lo + pi;
            const int n0 = EPI == QARL_EPI_SILU_MUL ? (nt ? N / 2 : 0) + u * 16 : u * 32 + nt * 16;
            const unsigned char *base = (const unsigned char *)p.codes + (ebase + (ok ? n0 : 0)) * (int64_t)rowb + (ok ? st * 128 : 0);
#pragma unroll
            for (int i = 0; i < 2; ++i)
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(base + voff[i]),
                                                 (__attribute__((address_space(3))) void *)(lring + slot * 4096 + nt * 2048 + i * 1024), 16, 0,
                                                 LR == 2 && !TAIL ? 2 : 0);
        }
    };

    int row0, Me;
    int *tmp_map = (int *)(xs + kRowsMax * stride);   // routed mode: [kIdsRows] activation rows, [kIdsRows] pair ids, [kSWaves] counts
    if (QX) {
        row0 = Me = 0;
        if (!TAIL) Me = list_pairs(p.ids, p.n_ids, e, p.x_per_token, p.topk, tmp_map);
    } else {
        row0 = p.offsets[e];
        Me = p.offsets[e + 1] - row0;
    }
    // one row block, rows m0 .. of the expert's, against the pairs u_lo .. u_lo + n_pairs - 1
    auto run_block = [&](int m0) __attribute__((always_inline)) {
        const int mrem = min(kRowsMax, Me - m0);
        lds_barrier();  // the pair list is complete / the previous pass is done with the LDS tile
        if (tid < kRowsMax) {
            const int i = row0 + m0 + tid;
            if (QX) {
                s_row[tid] = (tid < mrem) ? tmp_map[i] : -1;
                s_orow[tid] = (tid < mrem) ? tmp_map[kIdsRows + i] : -1;
            } else {
                s_row[tid] = (tid < mrem) ? (p.row_map ? p.row_map[i] : i) : -1;
                s_orow[tid] = (tid < mrem) ? (p.out_row_map ? p.out_row_map[i] : i) : -1;
                s_xs[tid] = (tid < mrem) ? p.x_scales[p.row_map ? p.row_map[i] : i] : 0.f;
            }
        }
        if (tid == 0) *s_next = kSWaves;  // pairs 0..7 start on wavefronts 0..7, the rest are drawn
        // LR: the channel scales of the slice go to LDS (a load in the loop would wait for the copies in flight)
        float sw_r[2];
        auto scale_of = [&](int i) -> float {   // i: pair, tile, column
            const int u = u_lo + (i >> 5), nt = (i >> 4) & 1;
            const int n = EPI == QARL_EPI_SILU_MUL ? (nt ? N / 2 : 0) + u * 16 + (i & 15) : u * 32 + (i & 31);
            return p.scales[ebase + n];
        };
        if constexpr (LR != 0) {
#pragma unroll
            for (int i = 0; i < 2; ++i) sw_r[i] = tid + i * kSThreads < n_pairs * 32 ? scale_of(tid + i * kSThreads) : 0.f;
        }
        auto store_scales = [&]() {
#pragma unroll
            for (int i = 0; i < 2; ++i)
                if (tid + i * kSThreads < n_pairs * 32) s_sw[tid + i * kSThreads] = sw_r[i];
            for (int i = tid + 2 * kSThreads; i < n_pairs * 32; i += kSThreads) s_sw[i] = scale_of(i);
        };
        lds_barrier();
        // ---- gather the token rows into LDS (whole K) in 16-byte blocks.  A thread keeps one block
        // column and walks down the rows (at most kBatch of them: the workgroup sweeps >= 2 rows at a
        // time), so the only index arithmetic is an add per block, and all its loads are in flight at
        // once.  Vector loads return in order: the token rows are requested first and the weight
        // stream right behind them, so it flows in while the tile is being built.
        if (QX) {
            // ---- routed mode: 16-bit token rows, quantized on their way into LDS.  One wavefront per row (rows
            // wave, wave + 8, ...): lane L holds the 16-byte chunks L, L + 64, ... of the row, the row's absmax is
            // a wavefront reduction, and the codes are the row quantizer's (same scale, same division, same
            // conversion).  Rows past the expert's end are left alone: a tile row feeds only its own output row,
            // which is never stored.
            const int n16 = K / 8;   // chunks of 8 values per row
            auto gather_q = [&](auto rows_c, auto kch_c, int rbase, bool first, bool last) {
                constexpr int ROWS = decltype(rows_c)::value, KCH = decltype(kch_c)::value;
                u32x4 v[ROWS][KCH];
                int xrow[ROWS];
#pragma unroll
                for (int rr = 0; rr < ROWS; ++rr) {
                    xrow[rr] = __builtin_amdgcn_readfirstlane(s_row[rbase + rr * kSWaves + wave]);
#pragma unroll
                    for (int u = 0; u < KCH; ++u) {
                        const int ch = lane + 64 * u;
                        v[rr][u] = u32x4{0, 0, 0, 0};
                        if (xrow[rr] >= 0 && ch < n16)
                            v[rr][u] = *(const u32x4 *)((const unsigned char *)p.x + ((int64_t)xrow[rr] * K + ch * 8) * 2);
                    }
                }
                if constexpr (LR == 0) {
                    if (first) fill_ring(wave, 0);   // the weight stream is requested right behind the token rows
                } else if (last) {
                    // ... once they are here: with copies in flight the compiler would let every use of a loaded register, and every LDS
                    // store it can see, wait for all of them
#pragma unroll
                    for (int rr = 0; rr < ROWS; ++rr)
#pragma unroll
                        for (int u = 0; u < KCH; ++u) asm volatile("" : "+v"(v[rr][u]));
                    store_scales();
#pragma unroll
                    for (int r = 0; r < R; ++r) copy_step(wave, r, r);
                }
#pragma unroll
                for (int rr = 0; rr < ROWS; ++rr) {
                    if (xrow[rr] < 0) continue;
                    const int r = rbase + rr * kSWaves + wave;
                    float am = 0.f;
#pragma unroll
                    for (int u = 0; u < KCH; ++u) am = absmax_bf16x8(v[rr][u], am);
                    am = wave_max(am);
                    const float sxr = am / 448.0f;
                    const RowScale rs(sxr);
#pragma unroll
                    for (int u = 0; u < KCH; ++u) {
                        const int ch = lane + 64 * u;
                        if (ch < n16) {
                            const u32x2 q8 = e4m3_quantize_bf16x8(rs, v[rr][u]);
                            if constexpr (LR == 0) *(u32x2 *)(xs + r * stride + ch * 8) = q8;
                            else lds_store8(xs + r * stride + ch * 8, q8);
                        }
                    }
                    if (lane == 0) {
                        if constexpr (LR == 0) s_xs[r] = sxr;
                        else lds_store4(s_xs + r, __float_as_uint(sxr));
                    }
                }
            };
            if (n16 <= 4 * 64) {
                // (64 rows: two batches of four rows per wavefront, as many as its registers hold)
#pragma unroll 1
                for (int i = 0; i < (MT + 1) / 2; ++i)
                    gather_q(std::integral_constant<int, MT == 1 ? 2 : 4>(), std::integral_constant<int, 4>(), i * 32, i == 0, i == (MT + 1) / 2 - 1);
            } else {
#pragma unroll 1
                for (int i = 0; i < MT; ++i)
                    gather_q(std::integral_constant<int, 2>(), std::integral_constant<int, 8>(), i * 16, i == 0, i == MT - 1);   // rows 16 i + wave, + 8
            }
        } else {
            const int bpr = K / 16;                      // blocks per row
            const int rpp = kSThreads / bpr;             // rows covered per sweep of the workgroup
            const int rsub = tid / bpr, b = tid - rsub * bpr;
            const bool active = rsub < rpp;
            constexpr int kBatch = 16;
            u32x4 v[kBatch];
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                const int r = rsub + u * rpp;
                v[u] = u32x4{0, 0, 0, 0};
                if (active && r < kRowsMax) {
                    const int xrow = s_row[r];
                    if (xrow >= 0)
                        v[u] = *(const u32x4 *)((const unsigned char *)p.x + (int64_t)xrow * K + b * 16);
                }
            }
            fill_ring(wave, 0);
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                const int r = rsub + u * rpp;
                const u32x4 o4 = v[u];
                if (active && r < kRowsMax) *(u32x4 *)(xs + r * stride + b * 16) = o4;
            }
        }
        lds_barrier();

        if constexpr (LR != 0) {
            // ---- the same stream through the LDS ring.  A wavefront waits for its own oldest stage, reads it into registers, and sends the
            // copies of the stage R ahead into the place just read.  The waits count: behind a stage lie the copies of the R - 1 younger
            // ones and, for the first R stages after an epilogue, its result stores, whose number is fixed (a row past the expert's end is
            // stored out of the buffer's bounds, i.e. nowhere).
            constexpr int kAhead = 4 * (R - 1), kStores = (EPI == QARL_EPI_SILU_MUL ? 1 : 2) * MT * 4;
            const bool half = EPI == QARL_EPI_SILU_MUL || !p.out_f32;
            const uint32_t ostride = (uint32_t)(EPI == QARL_EPI_SILU_MUL ? N / 2 : N) * (half ? 2u : 4u);
            const auto obuf = __builtin_amdgcn_make_buffer_rsrc(p.out, 0, (int)((uint32_t)p.n_ids * ostride), 0x00027000);
            int slot = 0;
            bool stored = false;
            for (int pi = wave; pi < n_pairs;) {
                int npi = 0;
                if (lane == 0) npi = lds_draw(s_next);
                npi = __builtin_amdgcn_readfirstlane(npi);
                f32x4 acc[2][MT];
#pragma unroll
                for (int nt = 0; nt < 2; ++nt)
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) acc[nt][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
                for (int st = 0; st < n_steps; ++st) {
                    if (stored && st < R) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kAhead + kStores) : "memory");
                    else asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kAhead) : "memory");
                    u32x4 w[2][2];
#pragma unroll
                    for (int nt = 0; nt < 2; ++nt)
#pragma unroll
                        for (int i = 0; i < 2; ++i) w[nt][i] = *(const u32x4 *)(lring + slot * 4096 + nt * 2048 + roff[i]);
                    asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(w[0][0]), "+v"(w[0][1]), "+v"(w[1][0]), "+v"(w[1][1])::"memory");
                    const bool same = st + R < n_steps;
                    copy_step(same ? pi : npi, same ? st + R : st + R - n_steps, slot);
                    slot = slot == R - 1 ? 0 : slot + 1;
#pragma unroll
                    for (int t = 0; t < (W4 ? 2 : 1); ++t)
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            long b0, b1;   // the 8 weights k = 8 j .. 8 j + 7 of this lane's row in either tile
                            if (W4) {
                                const u32x2 e0 = widen_e2m1_word(w[0][t][j]), e1 = widen_e2m1_word(w[1][t][j]);
                                b0 = (long)(((uint64_t)e0[1] << 32) | e0[0]);
                                b1 = (long)(((uint64_t)e1[1] << 32) | e1[0]);
                            } else {
                                b0 = (long)(((uint64_t)w[0][j >> 1][(j & 1) * 2 + 1] << 32) | w[0][j >> 1][(j & 1) * 2]);
                                b1 = (long)(((uint64_t)w[1][j >> 1][(j & 1) * 2 + 1] << 32) | w[1][j >> 1][(j & 1) * 2]);
                            }
#pragma unroll
                            for (int mt = 0; mt < MT; ++mt) {
                                const long a = *(const long *)(xs + (mt * 16 + c) * stride + (W4 ? 2 * st + t : st) * 128 + q * 32 + j * 8);
                                acc[0][mt] = __builtin_amdgcn_mfma_f32_16x16x32_fp8_fp8(a, b0, acc[0][mt], 0, 0, 0);
                                acc[1][mt] = __builtin_amdgcn_mfma_f32_16x16x32_fp8_fp8(a, b1, acc[1][mt], 0, 0, 0);
                            }
                        }
                }
                // ---- epilogue of this pair: lane (c,q) holds rows 4q..4q+3 of each token tile, column c
                const int n0 = tile_row(pi, 0), n1 = tile_row(pi, 1);
                const float sw0 = s_sw[pi * 32 + c], sw1 = s_sw[pi * 32 + 16 + c];
                asm volatile("" ::: "memory");
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    const i32x4 orow4 = *(const i32x4 *)(s_orow + mt * 16 + 4 * q);
                    const f32x4 sx4 = *(const f32x4 *)(s_xs + mt * 16 + 4 * q);
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const uint32_t at = orow4[i] >= 0 ? (uint32_t)orow4[i] * ostride : 0xfffffff0u;
                        const float v0 = acc[0][mt][i] * (sx4[i] * sw0), v1 = acc[1][mt][i] * (sx4[i] * sw1);
                        const uint32_t o0 = orow4[i] >= 0 ? at + (uint32_t)n0 * (half ? 2u : 4u) : at, o1 = orow4[i] >= 0 ? at + (uint32_t)n1 * (half ? 2u : 4u) : at;
                        if (EPI == QARL_EPI_SILU_MUL) {
                            __builtin_amdgcn_raw_buffer_store_b16((short)f32_to_bf16_hw(silu_mul_f32(v0, v1)), obuf, o0, 0, 0);
                        } else if (p.out_f32) {
                            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v0), obuf, o0, 0, 0);
                            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v1), obuf, o1, 0, 0);
                        } else {
                            __builtin_amdgcn_raw_buffer_store_b16((short)f32_to_bf16_hw(v0), obuf, o0, 0, 0);
                            __builtin_amdgcn_raw_buffer_store_b16((short)f32_to_bf16_hw(v1), obuf, o1, 0, 0);
                        }
                    }
                }
                stored = true;
                pi = npi;
            }
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // no copy may land after the workgroup has moved on
            return;
        }
        // ---- stream this wavefront's weight tiles
        // Wavefronts draw pairs from the LDS counter one pair ahead, so the two wavefronts that share a
        // SIMD (one of which the arbiter favours) finish together instead of the slower one trailing.
        for (int pi = wave; pi < n_pairs;) {
            int npi = 0;
            if (lane == 0) npi = atomicAdd(s_next, 1);
            npi = __builtin_amdgcn_readfirstlane(npi);
            f32x4 acc[2][MT];
#pragma unroll
            for (int nt = 0; nt < 2; ++nt)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) acc[nt][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
            for (int g0 = 0; g0 < G; g0 += R) {
                // the batch that refills the ring while this one is consumed: same pair or the next one
                const bool same = g0 + R < G;
                const uint32_t *nsrc[2] = {batch_src(same ? pi : npi, same ? g0 + R : 0, 0),
                                           batch_src(same ? pi : npi, same ? g0 + R : 0, 1)};
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const int g = g0 + r;
                    Slot &cur = ring[r];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        long b0, b1;   // the 8 weights k = 8 j .. 8 j + 7 of this lane's row in either tile
                        if (W4) {
                            const u32x2 e0 = widen_e2m1_word(cur.w[0][0][j]), e1 = widen_e2m1_word(cur.w[1][0][j]);
                            b0 = (long)(((uint64_t)e0[1] << 32) | e0[0]);
                            b1 = (long)(((uint64_t)e1[1] << 32) | e1[0]);
                        } else {
                            const u32x4 w0 = cur.w[0][(j >> 1) % kH], w1 = cur.w[1][(j >> 1) % kH];
                            b0 = (long)(((uint64_t)w0[(j & 1) * 2 + 1] << 32) | w0[(j & 1) * 2]);
                            b1 = (long)(((uint64_t)w1[(j & 1) * 2 + 1] << 32) | w1[(j & 1) * 2]);
                        }
#pragma unroll
                        for (int mt = 0; mt < MT; ++mt) {
                            const long a = *(const long *)(xs + (mt * 16 + c) * stride + g * 128 + q * 32 + j * 8);
                            acc[0][mt] = __builtin_amdgcn_mfma_f32_16x16x32_fp8_fp8(a, b0, acc[0][mt], 0, 0, 0);
                            acc[1][mt] = __builtin_amdgcn_mfma_f32_16x16x32_fp8_fp8(a, b1, acc[1][mt], 0, 0, 0);
                        }
                    }
                    // refill this slot with the step R ahead
                    fill(cur, r, nsrc);
                }
            }
            // ---- epilogue of this pair: lane (c,q) holds rows 4q..4q+3 of each token tile, column c
            const int n0 = tile_row(pi, 0), n1 = tile_row(pi, 1);
            const float sw0 = p.scales[ebase + n0], sw1 = p.scales[ebase + n1];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int r = mt * 16 + 4 * q + i;
                    const int64_t orow = s_orow[r];
                    if (orow >= 0) {
                        const float sxr = s_xs[r];
                        const float v0 = acc[0][mt][i] * (sxr * sw0), v1 = acc[1][mt][i] * (sxr * sw1);
                        if (EPI == QARL_EPI_SILU_MUL) {
                            const float a = silu_mul_f32(v0, v1);
                            ((uint16_t *)p.out)[orow * (N / 2) + n0] = f32_to_bf16_hw(a);
                        } else if (p.out_f32) {
                            ((float *)p.out)[orow * N + n0] = v0;
                            ((float *)p.out)[orow * N + n1] = v1;
                        } else {
                            ((uint16_t *)p.out)[orow * N + n0] = f32_to_bf16_hw(v0);
                            ((uint16_t *)p.out)[orow * N + n1] = f32_to_bf16_hw(v1);
                        }
                    }
                }
            }
            pi = npi;
        }
    };
    if constexpr (!SPREAD) {
        for (int m0 = mh * kRowsMax; m0 < Me; m0 += kRowsMax * p.m_split) run_block(m0);
        return false;
    } else if constexpr (!TAIL) {
        if (mh * kRowsMax < Me) run_block(mh * kRowsMax);
        return mh * kRowsMax >= Me || Me > p.m_split * kRowsMax;   // no row of its own, or a popular expert
    } else {
        // shares of the row blocks beyond the grid's: a pair per wavefront each, or a slice
        const int e_own = e, subs = (per_slice + kSWaves - 1) / kSWaves;
        int *s_hist = tmp_map + 2 * kIdsRows + kListWaves;
        count_rows(p.ids, p.n_ids, p.E, s_hist);
        SpreadItem it;
#pragma unroll 1
        for (int k = 0; spread_item(s_hist, p.E, MT == 1 ? 4 : MT == 2 ? 5 : 6, p.m_split, p.n_slices, subs, e_own, mh, slice, k, it); ++k) {
            e = it.e;
            ebase = (int64_t)e * N;
            const int sl = it.sub / subs;
            u_lo = sl * per_slice + (it.sub - sl * subs) * kSWaves;
            n_pairs = max(0, min(min(p.n_units, (sl + 1) * per_slice), u_lo + it.n_sub * kSWaves) - u_lo);
            if (n_pairs == 0) continue;   // the last slice may hold fewer pairs than it has shares for
            lds_barrier();   // the previous block is done with the list
            Me = list_pairs(p.ids, p.n_ids, e, p.x_per_token, p.topk, tmp_map);
            if (it.block * kRowsMax < Me) run_block(it.block * kRowsMax);
        }
        return false;
    }
}

template <int EPI, int MT, int R, bool W4, bool QX, int LR, bool SPREAD>
__global__ __launch_bounds__(kSThreads, 1) void qgemm_stream_fp8_kernel(StreamParams p)
{
    if (!stream_fp8_body<EPI, MT, R, W4, QX, LR, SPREAD, false>(p, threadIdx.x, blockIdx.x)) return;
    if constexpr (SPREAD) {
        const FreshArgs<StreamParams> f;
        stream_fp8_body<EPI, MT, R, W4, QX, LR, SPREAD, true>(f.p, f.tid, f.bid);
    }
}

inline size_t lr_lds_bytes(int K, int MT, int R, int n_units, int n_slices)
{
    const int per_slice = (n_units + n_slices - 1) / n_slices;
    return (size_t)lr_ring_at(K, MT) + (size_t)kSWaves * R * 4096 + (size_t)per_slice * 32 * 4;
}

// Whether a routed launch of this shape keeps its ring in LDS: whole lines of k in stages of 128 bytes, one per stage of the ring at least
inline bool lr_shape_fits(bool w4, int K, int MT, int R, int n_units, int n_slices)
{
    const int k_stage = w4 ? 256 : 128;
    return K % k_stage == 0 && K / k_stage >= R && lr_lds_bytes(K, MT, R, n_units, n_slices) <= 160 * 1024;
}

inline bool lr_fits(const StreamParams &p, int MT, int R)
{
    return p.ids && lr_shape_fits(p.w4, p.K, MT, R, p.n_units, p.n_slices) && (int64_t)p.n_ids * p.N * 4 < 0xfffffff0LL;
}

template <int EPI, int MT, int R, bool W4, bool QX, int LR = 0, bool SPREAD = false>
int launch_cfg_w(const StreamParams &p, hipStream_t s)
{
    if constexpr (QX && !SPREAD)
        if (p.spread) return launch_cfg_w<EPI, MT, R, W4, QX, LR, true>(p, s);
    const size_t lds = LR ? lr_lds_bytes(p.K, MT, R, p.n_units, p.n_slices) : stream_lds_bytes(p.K, MT, QX);
    if (lds > 160 * 1024) {
        set_error("qgemm (decode path): K=%d needs %zu bytes of LDS per workgroup, more than the 160 KiB of a CU", p.K, lds);
        return QARL_ERR_UNSUPPORTED;
    }
    static LdsLimitOnce once;
    auto kern = qgemm_stream_fp8_kernel<EPI, MT, R, W4, QX, LR, SPREAD>;
    if (int rc = raise_lds_limit((const void *)kern, once, "hipFuncSetAttribute(stream fp8)")) return rc;
    const int64_t units = (int64_t)p.E * p.n_slices;
    const int64_t grid = ((units + 7) / 8) * 8 * p.m_split;
    kern<<<dim3((unsigned)grid), dim3(kSThreads), lds, s>>>(p);
    return check_hip(hipGetLastError(), "qgemm_stream_fp8_kernel");
}

template <int EPI, int MT, int R, bool W4>
int launch_lr(const StreamParams &p, hipStream_t s)
{
    return p.m_split == 1 ? launch_cfg_w<EPI, MT, R, W4, true, 2>(p, s) : launch_cfg_w<EPI, MT, R, W4, true, 1>(p, s);
}

template <int EPI, int MT, bool W4>
int launch_ring(const StreamParams &p, hipStream_t s)
{
    const int G = p.K / kGroup;
    if (lr_fits(p, MT, kLrStages)) return launch_lr<EPI, MT, kLrStages, W4>(p, s);
    auto go = [&](auto r_c) -> int {
        constexpr int R = decltype(r_c)::value;
        // (64 rows of e2m1 codes in the routed mode: only K = 256 and odd numbers of groups come here)
        if constexpr (W4 && MT == 4 && R == 4) return launch_cfg_w<EPI, MT, R, W4, false>(p, s);
        else return p.ids ? launch_cfg_w<EPI, MT, R, W4, true>(p, s) : launch_cfg_w<EPI, MT, R, W4, false>(p, s);
    };
    // ring depth (steps in flight per wavefront): 8 KiB per wavefront, i.e. two steps of e4m3 codes (4 KiB each: two
    // tiles, two 1 KiB loads per tile) or four steps of e2m1 codes, already saturate HBM with eight wavefronts per CU;
    // twice that measured 4 % slower on the gate_up launch, and a deeper ring would push the gather into spilling
    if constexpr (W4) {
        if (G % 4 == 0 && !(MT == 4 && p.ids)) return go(std::integral_constant<int, 4>());
        if (G % 3 == 0) return go(std::integral_constant<int, 3>());
    }
    if (G % 2 == 0) return go(std::integral_constant<int, 2>());
    if (!W4 && G % 3 == 0) return go(std::integral_constant<int, 3>());
    return go(std::integral_constant<int, 1>());
}

// The launch of one source: EPI and MT (1, 2, 4) at run time
template <bool W4>
int launch_codes(const StreamParams &p, int epilogue, int MT, hipStream_t s)
{
    if (epilogue == QARL_EPI_SILU_MUL)
        return MT == 1 ? launch_ring<QARL_EPI_SILU_MUL, 1, W4>(p, s) : MT == 2 ? launch_ring<QARL_EPI_SILU_MUL, 2, W4>(p, s) : launch_ring<QARL_EPI_SILU_MUL, 4, W4>(p, s);
    return MT == 1 ? launch_ring<QARL_EPI_NONE, 1, W4>(p, s) : MT == 2 ? launch_ring<QARL_EPI_NONE, 2, W4>(p, s) : launch_ring<QARL_EPI_NONE, 4, W4>(p, s);
}
int launch_fp4(const StreamParams &p, int epilogue, int MT, hipStream_t s);   // qgemm_stream_fp4.hip

}  // namespace stream8

}  // namespace qarl
