// Shared device helpers of the QaRL hot-path kernels (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

#include "../../include/qarl.h"

namespace qarl {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef __attribute__((ext_vector_type(8))) int i32x8;
typedef __attribute__((ext_vector_type(4))) int i32x4;

constexpr int kWave = 64;
constexpr int kGroup = 128;  // k per int4 scale group

__device__ __forceinline__ float bf16_bits_to_f32(uint32_t h) { return __uint_as_float(h << 16); }

// Round-to-nearest-even fp32 -> bf16 bit pattern (NaN kept quiet).
__device__ __forceinline__ uint32_t f32_to_bf16_bits(float f)
{
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (u >> 16) | 0x40u;
    u += 0x7fffu + ((u >> 16) & 1u);
    return u >> 16;
}

// The same conversion by the hardware instruction (round-to-nearest-even).
__device__ __forceinline__ uint16_t f32_to_bf16_hw(float f)
{
    return __builtin_bit_cast(uint16_t, (__bf16)f);
}

// silu(g) * u with g / (1 + e^-g) evaluated as g * rcp(1 + exp2(-g log2 e)): hardware exp2 and rcp,
// each within 1 ulp of fp32, far below the bf16 rounding the result goes through.
__device__ __forceinline__ float silu_mul_f32(float g, float u)
{
    const float t = __builtin_amdgcn_exp2f(g * -1.44269504088896340736f);
    return g * __builtin_amdgcn_rcpf(1.f + t) * u;
}

// Largest value of the wavefront (all lanes active), the same in every lane: row shifts and two row broadcasts bring it to
// lane 63 (six dependent VALU operations; six LDS permutes took the routed quantizers' start-up about 0.3 us).
__device__ __forceinline__ float wave_max(float v)
{
#define QARL_MAX_STEP(CTRL, ROWS) \
    v = fmaxf(v, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, v), __builtin_bit_cast(int, v), CTRL, ROWS, 0xf, false)))
    QARL_MAX_STEP(0x111, 0xf);   // row_shr:1
    QARL_MAX_STEP(0x112, 0xf);   // row_shr:2
    QARL_MAX_STEP(0x114, 0xf);   // row_shr:4
    QARL_MAX_STEP(0x118, 0xf);   // row_shr:8
    QARL_MAX_STEP(0x142, 0xa);   // row_bcast:15 into rows 1 and 3
    QARL_MAX_STEP(0x143, 0xc);   // row_bcast:31 into rows 2 and 3
#undef QARL_MAX_STEP
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}

__device__ __forceinline__ float wave_sum(float v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// ---- FP quantizer of section 2.2 along a row, e4m3 flavour (alpha = 448), shared by the row quantizer and by the
// decode GEMM that quantizes its token rows while it gathers them, so that both produce the same bytes.
// x / s, correctly rounded, without a divide per element: with y = RN(1 / s) (one IEEE divide per row),
// q0 = RN(x y) and the exact remainder r = x - q0 s from one FMA, RN(q0 + r y) is the correctly rounded
// quotient (Markstein's correction step; it needs the correctly rounded reciprocal and no underflow on the
// way, hence the guard on s; below 2^-11 a quotient may differ from the IEEE one, where every value rounds
// to an e4m3 zero; the sign is copied from x, as s > 0).  Checked against the IEEE divide for all 65536 bf16
// values of x and 2^20 scales (the quantizer's own absmax / alpha and random ones): no difference at |x / s| >= 2^-11.
// The scale is the same in all lanes (a wavefront reduction formed it) and is held as such, so that which of the two divisions a row
// takes is one scalar branch per eight elements (a lane mask and a branch per element before: in the routed FP8 gate_up
// launch of 256 tokens, 32 k elements per workgroup, 285 branches).
struct RowScale {
    float s, y;
    bool fast;
    __device__ __forceinline__ explicit RowScale(float s_) : s(__uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(s_)))), y(1.0f / s)
    {
        fast = s >= 0x1p-100f && s < 0x1p100f && (__float_as_uint(s) & 0x7fffffu) != 0x7fffffu;
    }
    // x / s of eight bf16 values held in four dwords
    __device__ __forceinline__ void div8(u32x4 v, float (&t)[8]) const
    {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t w = v[i];
            t[2 * i] = __uint_as_float(w << 16);
            t[2 * i + 1] = __uint_as_float(w & 0xffff0000u);
        }
        if (fast) {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float x = t[i], q0 = x * y;
                t[i] = copysignf(fmaf(fmaf(-q0, s, x), y, q0), x);   // the sign of x also where the steps end in +0 (x = -0)
            }
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) t[i] = t[i] / s;
        }
    }
};

// Sum of eight bf16 values, in the order of the group sums (pairs, then ascending).
__device__ __forceinline__ float group_chunk_sum(u32x4 v)
{
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) s += __uint_as_float(v[i] << 16) + __uint_as_float(v[i] & 0xffff0000u);
    return s;
}

// absmax of eight bf16 values held in four dwords, folded into am
__device__ __forceinline__ float absmax_bf16x8(u32x4 v, float am)
{
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        am = fmaxf(am, fabsf(__uint_as_float(v[i] << 16)));
        am = fmaxf(am, fabsf(__uint_as_float(v[i] & 0xffff0000u)));
    }
    return am;
}

// Eight bf16 values -> eight e4m3 bytes of x / s (zeros for a zero row).  v_cvt_pk_fp8_f32 rounds to nearest even
// into OCP e4m3 (subnormals included) for every finite |t| <= 448 (checked over all 2^32 bit patterns on gfx950
// against a software encoder); the clamp keeps the quotient of the row's absmax, which may exceed 448 by an ulp,
// in that range (and sends a NaN to -448).
__device__ __forceinline__ u32x2 e4m3_quantize_bf16x8(const RowScale &rs, u32x4 v)
{
    u32x2 o = {0, 0};
    if (rs.s != 0.f) {
        float t[8];
        rs.div8(v, t);
#pragma unroll
        for (int i = 0; i < 8; ++i) t[i] = __builtin_amdgcn_fmed3f(t[i], -448.f, 448.f);
        int w0 = __builtin_amdgcn_cvt_pk_fp8_f32(t[0], t[1], 0, false);
        w0 = __builtin_amdgcn_cvt_pk_fp8_f32(t[2], t[3], w0, true);
        int w1 = __builtin_amdgcn_cvt_pk_fp8_f32(t[4], t[5], 0, false);
        w1 = __builtin_amdgcn_cvt_pk_fp8_f32(t[6], t[7], w1, true);
        o[0] = (uint32_t)w0;
        o[1] = (uint32_t)w1;
    }
    return o;
}

// Eight e4m3 bytes -> the bf16 values they stand for (exact: four significant bits).
__device__ __forceinline__ u32x4 e4m3_as_bf16x8(u32x2 q8)
{
    u32x4 o;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const auto lo = __builtin_amdgcn_cvt_pk_f32_fp8((int)q8[i], false);
        const auto hi = __builtin_amdgcn_cvt_pk_f32_fp8((int)q8[i], true);
        o[2 * i] = (__float_as_uint(lo[0]) >> 16) | (__float_as_uint(lo[1]) & 0xffff0000u);
        o[2 * i + 1] = (__float_as_uint(hi[0]) >> 16) | (__float_as_uint(hi[1]) & 0xffff0000u);
    }
    return o;
}

// A constant the optimiser cannot see through, held in a scalar (vector) register.  (a & mask) | c with such operands
// is selected as one v_and_or_b32; with literal operands the compiler emits v_and + v_or (a VOP3 encoding takes no
// literal on this target).  The operation itself must stay an instruction the compiler knows: a matrix instruction
// that reads a register needs wait states after the VALU instruction that wrote it, which the compiler inserts for
// its own instructions and cannot insert for the contents of an inline asm (with v_and_or_b32 written as inline
// asm, a matrix instruction scheduled directly behind it read the register's previous contents now and then).
__device__ __forceinline__ uint32_t opaque_sgpr(uint32_t v)
{
    asm("" : "+s"(v));
    return v;
}
__device__ __forceinline__ uint32_t opaque_vgpr(uint32_t v)
{
    asm("" : "+v"(v));
    return v;
}

// Bit position of the low bit of element e (0..7) of a packed word of int4 codes (stored as u = q+8).
// Elements 2i and 2i+1 (i < 3) sit 16 bits apart at bits 3+4i and 19+4i, i.e. already in the top four
// mantissa bits of the two bf16 halves of a dword after a right shift by 4i; element 6 sits at bits
// 15..18 and element 7 wraps around the word (its low bit at bit 31, the other three at bits 0..2), so
// that a rotation by 12 brings both into place.
__host__ __device__ constexpr int int4_bit_pos(int e) { return e < 6 ? 3 + 4 * (e >> 1) + 16 * (e & 1) : (e == 6 ? 15 : 31); }

// One packed word of eight int4 codes -> eight exact bf16 values (q+24)/16 in element order 0..7: the
// code lands in the top four mantissa bits of bf16 1.0.  Seven VALU operations per word: one and-or for
// the first pair, a shift (or the rotation) and an and-or for each of the other three.
__device__ __forceinline__ bf16x8 unpack_int4_word(uint32_t w)
{
    const uint32_t mask = opaque_sgpr(0x00780078u), one = opaque_vgpr(0x3f803f80u);
    u32x4 d;
    d[0] = (w & mask) | one;
    d[1] = ((w >> 4) & mask) | one;
    d[2] = ((w >> 8) & mask) | one;
    d[3] = (__builtin_rotateright32(w, 12) & mask) | one;
    return __builtin_bit_cast(bf16x8, d);
}

// e2m1 magnitude code (3 bits) -> e4m3 byte of the same value: 0, 0.5, 1, 1.5 | 2, 3, 4, 6.  Every e2m1 value is
// an e4m3 value, so FP4 weights are widened in registers (one byte permute per four codes) and meet the e4m3
// token rows in the same matrix instruction as FP8 weights do.
constexpr uint32_t kE2m1LutLo = 0x3c383000u, kE2m1LutHi = 0x4c484440u;

// A word of eight packed e2m1 codes (byte b: element b in the low nibble, element 4 + b in the high nibble)
// -> the eight e4m3 bytes in element order.
__device__ __forceinline__ u32x2 widen_e2m1_word(uint32_t w)
{
    u32x2 o;
    o[0] = __builtin_amdgcn_perm(kE2m1LutHi, kE2m1LutLo, w & 0x07070707u) | ((w & 0x08080808u) << 4);
    o[1] = __builtin_amdgcn_perm(kE2m1LutHi, kE2m1LutLo, (w >> 4) & 0x07070707u) | (w & 0x80808080u);
    return o;
}

// Workgroup barrier that orders LDS traffic only.  __syncthreads() also drains every outstanding
// global load of the wavefront (the workgroup-scope fence waits on vmcnt), which would stall the
// weight prefetch rings; kernels whose cross-wavefront traffic goes through LDS alone use this.
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Asynchronous global -> LDS copy of one wavefront: active lane L's 16 bytes land at lds_dst + 16 L.
// lds_dst must be the same in all lanes.  Completion is counted by vmcnt, in order with the
// wavefront's other vector loads.
__device__ __forceinline__ void copy16_to_lds(const void *gsrc, void *lds_dst)
{
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)gsrc,
                                     (__attribute__((address_space(3))) void *)lds_dst, 16, 0, 0);
}

// Barrier for LDS buffers filled by copy16_to_lds: every wavefront first waits for its own copies
// (and LDS operations), then for the others.
__device__ __forceinline__ void copy_barrier()
{
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Tiles of a grouped launch: `rows` (expert_offsets) are cut into tiles of kTile rows that never span two experts, and
// every tile has n_blocks work items.  The host only knows an upper bound of the tiles (every expert may end in a
// partial one), so the grid is that bound, rounded up, and the true number comes from the scan every wavefront makes
// here (four experts per lane, E <= 256, no barrier).  Workgroup ids go round-robin over the 8 XCDs; an XCD gets a
// contiguous eighth of the TRUE items (the blocks of one tile share its L2), the surplus workgroups of all XCDs leave.
// (Eighths of the bound left the surplus on the last XCDs: 7 of 8 worked on 3001 tokens and 128 experts.  W4A8 layer of
// 3001 tokens 415 -> 389 us, FP8 of 8192 723 -> 695, W4A16 of 16384 1697 -> 1682.)
// The tile's rows come out of the scan as well: a second look at the offsets was one more dependent load in front of the row
// ids (layers of 128 experts, W4A16 16384 tokens 1596 -> 1586 us, FP8 8192 651 -> 645, W4A8 3001 381 -> 374).
struct GroupedTile {
    int e, block;     // expert, work item of the tile
    int row0, rows;   // first row, rows up to the expert's end (at most kTile)
};
template <int kTile>
__device__ __forceinline__ bool find_grouped_tile(const int32_t *offsets, int E, int n_blocks, GroupedTile &t)
{
    const int lane = threadIdx.x & 63;
    int off[5], cnt[4], sum = 0;
#pragma unroll
    for (int q = 0; q < 5; ++q) off[q] = offsets[min(lane * 4 + q, E)];   // (experts past E: no rows)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        cnt[q] = (off[q + 1] - off[q] + kTile - 1) / kTile;
        sum += cnt[q];
    }
    int incl = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int up = __shfl_up(incl, o, 64);
        if (lane >= o) incl += up;
    }
    const unsigned items = (unsigned)__builtin_amdgcn_readlane(incl, 63) * (unsigned)n_blocks;   // at most the grid: below 2^31
    const unsigned per_xcd = (items + 7) / 8, idx = blockIdx.x / 8, v = (blockIdx.x % 8) * per_xcd + idx;
    if (idx >= per_xcd || v >= items) return false;
    const int slot = (int)(v / (unsigned)n_blocks);
    t.block = (int)(v - (unsigned)slot * (unsigned)n_blocks);
    int base = incl - sum, found = -1, row0 = 0, rows = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        if (slot >= base && slot < base + cnt[q]) {
            found = lane * 4 + q;
            row0 = off[q] + (slot - base) * kTile;
            rows = min(kTile, off[q + 1] - row0);
        }
        base += cnt[q];
    }
    const unsigned long long hit = __ballot(found >= 0);
    if (hit == 0) return false;   // does not happen: slot < number of tiles
    const int src = __ffsll((long long)hit) - 1;
    t.e = __builtin_amdgcn_readlane(found, src);
    t.row0 = __builtin_amdgcn_readlane(row0, src);
    t.rows = __builtin_amdgcn_readlane(rows, src);
    return true;
}

// Whether two byte ranges share memory.
inline bool ranges_overlap(const void *a, size_t na, const void *b, size_t nb)
{
    return (uintptr_t)a < (uintptr_t)b + nb && (uintptr_t)b < (uintptr_t)a + na;
}

// Host-side error plumbing (api.hip).
void set_error(const char *fmt, ...);
int check_hip(hipError_t e, const char *what);

// Kernels that take more than the default 64 KiB of dynamic LDS need their limit raised once per device.
// Every caller raises it to the same value (the 160 KiB of a gfx950 CU less the kernel's static LDS), so concurrent host threads cannot
// undo each other; `done` (one object per kernel instantiation, zero-initialised) remembers the devices served.
constexpr int kMaxLdsBytes = 160 * 1024;
struct LdsLimitOnce {
    std::atomic<unsigned> devices_done[2];   // bit d of word d / 32: device d (devices >= 64 are set every call)
};
int raise_lds_limit(const void *kernel, LdsLimitOnce &done, const char *what);

// Kernel launchers (one per .hip file); all validate nothing: api.hip does.
int launch_quantize_int4(const void *w, int64_t rows, int K, void *codes, void *scales, hipStream_t s);
int launch_quantize_fp8_rows(const void *x, int64_t rows, int K, void *codes, float *scales, hipStream_t s);
int launch_quantize_fp4_rows(const void *x, int64_t rows, int K, void *codes, float *scales, hipStream_t s);
int launch_canonical_codes(int fmt, const void *codes, int64_t rows, int K, void *out, hipStream_t s);
int launch_e4m3_to_bf16(const void *x8, int64_t n, void *x16, float *sums, hipStream_t s);  // e4m3 bytes -> bf16 (exact); sums: as launch_group_sums, or null
int launch_route_only(const void *logits, int T, int E, int topk, int renorm, int32_t *ids, float *w, hipStream_t s);
int launch_route(const void *logits, int T, int E, int topk, int renorm, int32_t *ids, float *w,
                 int32_t *counts, int32_t *offsets, int32_t *pairs, int32_t *tokens, hipStream_t s);

struct GemmArgs {
    int fmt;
    int E, N, K;
    const void *codes;
    const void *scales;
    const void *x;
    const float *x_scales;       // FP8 / FP4: scale of each activation row; W4A8: the same, applied in the epilogue
    const float *x_group_sums;   // W4A16 prefill path: -1.5 * sum of x over each 128-k group, [x_rows][K/128]
    const int32_t *row_map;      // gather of activation rows, or null
    const int32_t *out_row_map;  // scatter of output rows, or null
    const int32_t *offsets;
    int64_t M;
    int64_t x_rows;     // rows of x (bound of row_map values)
    int epilogue;       // NONE or SILU_MUL here; COMBINE is NONE into ws + combine kernel
    void *out;          // [M][N] or [M][N/2]
    int out_f32;
    // routed mode of the decode kernels (ids != null; offsets and row maps unused): row = pair id
    // t * topk + slot of expert ids[row], activation row t (x_per_token) or the pair id, output row = pair id;
    // x is bf16 for every format (the e4m3-activation formats quantize the rows they gather)
    const int32_t *ids = nullptr;
    int topk = 0;
    int x_per_token = 0;
    // few-pair kernels, SILU_MUL: route the tokens themselves (logits bf16 [T][E]) and write ids and weights, which `ids` then is not read for
    const void *logits = nullptr;
    int renorm = 0;
    int32_t *ids_out = nullptr;
    float *w_out = nullptr;
    int spread = 0;     // routed mode: a popular expert's rows may be worked on by any workgroup (out overlaps neither x nor ids)
};
int launch_qgemm_stream(const GemmArgs &a, hipStream_t s);
bool qgemm_stream_supported(int fmt, int N, int K);
bool qgemm_stream_routed_supported(int fmt, int N, int K, int T, int topk);
// Estimated times (us) of a routed call under an even router, epilogue included, on the streaming kernels and on the kernels
// for few pairs: the rule between the two (qgemm_small_w4.hip says how they were measured).
double qgemm_stream_routed_us(int fmt, int N, int K, int E, int T, int topk, int epilogue);
int qgemm_stream_w4_units_per_wave(int N, int K, int E, int64_t M);
int launch_qgemm_stream_w4(const GemmArgs &a, hipStream_t s);
bool qgemm_stream_w4_supported(int N, int K);
bool qgemm_stream_w4_routed_supported(int N, int K, int T, int topk);
// Routed W4A16 / W4A8 calls of a few pairs; combine_w: the COMBINE epilogue, a.out then is its [T][N] output
bool qgemm_small_w4_supported(int N, int K, int T, int topk, int epilogue);
double qgemm_small_w4_us(int fmt, int N, int K, int T, int topk, int epilogue);
int launch_qgemm_small_w4(const GemmArgs &a, const float *combine_w, hipStream_t s);
// The same for FP8 / FP4
bool qgemm_small_fp8_supported(int N, int K, int T, int topk, int epilogue);
double qgemm_small_fp8_us(int fmt, int N, int K, int T, int topk, int epilogue);
int launch_qgemm_small_fp8(const GemmArgs &a, const float *combine_w, hipStream_t s);
int launch_qgemm_tile(const GemmArgs &a, hipStream_t s);
int launch_qgemm_tile_fp8(const GemmArgs &a, hipStream_t s);
// Straight-through backward of the W4A16 grouped GEMM: a.x = dY bf16 [M][N], a.out = dX [M][K]
int launch_qgemm_dx(const GemmArgs &a, hipStream_t s);
int launch_grouped_dw(const void *dy, const void *x, const int32_t *row_map, const int32_t *offsets, int64_t M, int E, int N,
                      int K, void *out, int out_f32, hipStream_t s);
int launch_group_sums(const void *x_bf16, int64_t rows, int K, float *sums, hipStream_t s);
// ids: of the pairs, or null (every row of Y was written)
int launch_combine(const float *y_pair_order, const float *w, const int32_t *ids, int E, int T, int topk, int N, void *out,
                   int out_f32, hipStream_t s);
int launch_logprob(const void *h, const void *wlm, const int32_t *target, int T, int H, int V,
                   float inv_temp, float *logprob, void *ws, size_t ws_bytes, hipStream_t s);
size_t logprob_ws_bytes(int T, int H, int V);
size_t logprob_ws_least(int T, int V);   // enough for every call; up to 128 tokens the size above lets more CUs take part
// Device address, on the current device, of the library's own file-scope scratch array (kLogprobScratchBytes).
constexpr size_t kLogprobScratchBytes = (size_t)4 << 20;
int logprob_static_scratch(void **ptr);
int launch_fill_f32(float *p, int64_t n, float v, hipStream_t s);
int launch_tbpo(const float *lp_cur, const float *lp_old, const float *lp_smp, const int32_t *seq_offsets, int S,
                const float *adv, float eps_low, float eps_high, float delta_low, float delta_high, float c,
                float *r_seq, float *w_clip, float *r_clip, int32_t *in_band, float *obj_seq, float *objective,
                float *grad, hipStream_t s);
int launch_mismatch(const float *lp_a, const float *lp_b, int T, const int32_t *seq_offsets, int S, float c,
                    float *delta, float *token_w, float *seq_w, float *seq_wc, hipStream_t s);

}  // namespace qarl
