// Routing of one token by one wavefront: exact top-k of E <= 256 bf16 logits by (logit desc, expert id asc) and the winners'
// softmax weights.  Shared by the router and by the few-pair GEMMs that route their token themselves.
#pragma once
#include "common.hpp"

namespace qarl {

constexpr int kMaxPerLane = 4;  // E <= 256

// Order-preserving integer image of a bf16 pattern (-0 counted as +0), high half of the key;
// low half = 0xffff - expert id so that the lower id wins among equal logits.
__device__ __forceinline__ uint32_t sort_key(uint32_t h, int id)
{
    if (h == 0x8000u) h = 0;
    uint32_t k = (h & 0x8000u) ? (~h & 0xffffu) : (h | 0x8000u);
    return (k << 16) | (0xffffu - (uint32_t)id);
}

// Wavefront reductions on the data-parallel-primitive path (row shifts inside 16-lane rows, then two
// row broadcasts); the result is read from lane 63 into a scalar, so it is uniform.  `ident` fills the
// lanes a shift has no source for.
#define QARL_DPP_STEP(T, OP, CTRL, ROWMASK)                                                                   \
    v = OP(v, (T)__builtin_bit_cast(T, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, ident),             \
                                                                   __builtin_bit_cast(int, v), CTRL, ROWMASK, 0xf, false)))
__device__ __forceinline__ uint32_t umax2(uint32_t a, uint32_t b) { return a > b ? a : b; }
__device__ __forceinline__ float fadd2(float a, float b) { return a + b; }
__device__ __forceinline__ uint32_t wave_max_u32_dpp(uint32_t v)
{
    const uint32_t ident = 0;
    QARL_DPP_STEP(uint32_t, umax2, 0x111, 0xf);  // row_shr:1
    QARL_DPP_STEP(uint32_t, umax2, 0x112, 0xf);  // row_shr:2
    QARL_DPP_STEP(uint32_t, umax2, 0x114, 0xf);  // row_shr:4
    QARL_DPP_STEP(uint32_t, umax2, 0x118, 0xf);  // row_shr:8
    QARL_DPP_STEP(uint32_t, umax2, 0x142, 0xa);  // row_bcast:15 into rows 1 and 3
    QARL_DPP_STEP(uint32_t, umax2, 0x143, 0xc);  // row_bcast:31 into rows 2 and 3
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}
// Sum in the fixed order the shifts imply; every lane gets the same value.
__device__ __forceinline__ float wave_sum_f32_dpp(float v)
{
    const float ident = 0.f;
    QARL_DPP_STEP(float, fadd2, 0x111, 0xf);
    QARL_DPP_STEP(float, fadd2, 0x112, 0xf);
    QARL_DPP_STEP(float, fadd2, 0x114, 0xf);
    QARL_DPP_STEP(float, fadd2, 0x118, 0xf);
    QARL_DPP_STEP(float, fadd2, 0x142, 0xa);
    QARL_DPP_STEP(float, fadd2, 0x143, 0xc);
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}
#undef QARL_DPP_STEP

// Logits of the token, one per lane and 64 experts.  PER: 64-expert groups (E = 192 takes four).
template <int PER>
struct TokenLogits {
    uint32_t key[PER];
    float val[PER];
    __device__ __forceinline__ TokenLogits() {}
    __device__ __forceinline__ TokenLogits(const uint16_t *logits, int E)
    {
        const int lane = threadIdx.x & 63;
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            key[j] = 0;
            val[j] = -INFINITY;
            if (PER < kMaxPerLane || 64 * j < E) {
                const int e = lane + 64 * j;
                const uint32_t h = logits[e];
                key[j] = sort_key(h, e);
                val[j] = bf16_bits_to_f32(h);
            }
        }
    }
    // The keys of the first n winners, lane r the r-th; a key holds both the logit and the id.  Retires them.
    __device__ __forceinline__ uint32_t select(int n)
    {
        const int lane = threadIdx.x & 63;
        uint32_t mine = 0;
        for (int r = 0; r < n; ++r) {
            uint32_t best = 0;
#pragma unroll
            for (int j = 0; j < PER; ++j) best = max(best, key[j]);
            best = wave_max_u32_dpp(best);
#pragma unroll
            for (int j = 0; j < PER; ++j)
                if (key[j] == best) key[j] = 0;   // the owner retires it
            if (lane == r) mine = best;
        }
        return mine;
    }
    static __device__ __forceinline__ int expert(uint32_t k) { return 0xffff - (int)(k & 0xffffu); }
};

// The token's topk experts and weights, written by the wavefront: the probabilities are formed behind the rounds, all at once.
template <int PER>
__device__ __forceinline__ void route_token(TokenLogits<PER> l, int E, int topk, int renorm, int32_t *ids, float *wts)
{
    const int lane = threadIdx.x & 63;
    float m = -INFINITY;
#pragma unroll
    for (int j = 0; j < PER; ++j) m = fmaxf(m, l.val[j]);
    m = wave_max(m);   // (a number or an infinity: a lane starts from -inf)
    float z = 0.f;
#pragma unroll
    for (int j = 0; j < PER; ++j)
        if (PER < kMaxPerLane || 64 * j < E) z += expf(l.val[j] - m);
    z = wave_sum_f32_dpp(z);
    const uint32_t mine = l.select(topk), k = mine >> 16;
    const float p = expf(bf16_bits_to_f32((k & 0x8000u) ? k ^ 0x8000u : ~k & 0xffffu) - m) / z;
    float psum = 0.f;
    for (int r = 0; r < topk; ++r)
        psum += __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, p), r));
    if (lane < topk) {
        ids[lane] = TokenLogits<PER>::expert(mine);
        wts[lane] = renorm ? p / psum : p;
    }
}

}  // namespace qarl
