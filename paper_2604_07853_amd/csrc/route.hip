// MoE router: fp32 softmax over bf16 logits, exact top-k by (logit desc, expert id asc),
// renormalised weights, then a stable grouping of the (token, slot) pairs by expert.
// One wavefront owns one token: E <= 256 logits sit 1..4 per lane, the arg-max of every
// round is a 6-step shuffle reduction on an integer key, so equal bf16 logits resolve to
// the lower expert id exactly as a full stable sort would.
#include "route_token.hpp"

namespace qarl {

constexpr int kRouteThreads = 256;

// PER: 64-expert groups, logits per lane (E = 192 takes the kernel of four).  Bound by issue: a round of the selection is
// the arg-max reduction and little else.  The winning keys are kept, one per lane (a key holds both the logit and the id),
// and the probabilities are formed behind the rounds, all at once.  128 experts, top-8: 16384 tokens 20.2 -> 11.0 us with
// an exponential and a division in every round and four logits per lane before.
template <int PER>
__global__ __launch_bounds__(kRouteThreads) void route_topk_kernel(const uint16_t *__restrict__ logits, int T,
                                                                  int E, int topk, int renorm,
                                                                  int32_t *__restrict__ ids,
                                                                  float *__restrict__ wts)
{
    const int t = blockIdx.x * (kRouteThreads / 64) + (threadIdx.x >> 6);
    if (t >= T) return;
    route_token<PER>(TokenLogits<PER>(logits + (int64_t)t * E, E), E, topk, renorm, ids + (int64_t)t * topk, wts + (int64_t)t * topk);
}

// Grouping of large batches: one workgroup per expert, no counters, no pass in front.  Every wavefront owns a contiguous
// range of the pairs and sweeps it once, eight 16-byte loads per lane in flight, counting the ids below its expert's (their
// sum over the workgroup is the expert's offset) and noting the expert's own as bits.  Behind the only barrier it places
// them in ascending pair order, which keeps (t, slot) order: a pair's rank in a step comes from four ballots.  The bits of
// the first four batches (131072 pairs of a workgroup) stay in registers, later ones are read again (cache hits).
// Bound by the VALU work of the sweep, four operations per pair and expert (a comparison that adds its carry takes as
// many and two wait states).  Top-8 of 128: 11.5 us at 8192 tokens and 17.8 at 16384 (medians), where a counting kernel
// with one counter per expert and two sweeps with prefix sums by shuffles took 4.5 + 22.8 at 16384.
constexpr int kGroupThreads = 1024;
constexpr int kGroupWaves = kGroupThreads / 64;
constexpr int kGroupStep = 256;               // pairs per wavefront and step: four consecutive ones per lane
constexpr int kGroupBatch = 8 * kGroupStep;   // pairs per wavefront whose loads are in flight together
constexpr int kGroupKeep = 4;                 // batches whose bits are kept

typedef int i32x4_u __attribute__((ext_vector_type(4), aligned(4)));   // the caller's ids may lie at any element

__global__ __launch_bounds__(kGroupThreads) void group_by_expert_kernel(const int32_t *__restrict__ ids,
                                                                       uint32_t n_pairs, int E, uint32_t topk_magic,
                                                                       int topk_shift, int32_t *__restrict__ counts,
                                                                       int32_t *__restrict__ offsets,
                                                                       int32_t *__restrict__ pairs,
                                                                       int32_t *__restrict__ tokens)
{
    __shared__ int s_cnt[kGroupWaves], s_less[kGroupWaves];
    const int e = blockIdx.x;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    // pairs in whole groups of four; the up to three behind them are the last wavefront's
    const uint32_t n4 = n_pairs & ~3u;
    const uint32_t steps = (n4 + kGroupWaves * kGroupStep - 1) / (kGroupWaves * kGroupStep);
    const uint32_t lo = wave * steps * kGroupStep;
    const uint32_t hi = min(n4, lo + steps * kGroupStep);

    int less = 0;
    auto sweep = [&](uint32_t p0) -> uint32_t {   // bit 4 s + j: pair p0 + 256 s + 4 lane + j goes to this expert
        i32x4_u v[8];
        const uint32_t p = p0 + lane * 4;
#pragma unroll
        for (int s = 0; s < 8; ++s) v[s] = *(const i32x4_u *)(ids + min(p + s * kGroupStep, n4 - 4));
        uint32_t lt = 0, le = 0;   // ids below e, below e + 1: a difference's sign bit is shifted in by one instruction
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const int es = p + s * kGroupStep < hi ? e : -1;   // past the range: no id is below 0
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                lt = __builtin_amdgcn_alignbit(lt, (uint32_t)(v[s][j] - es), 31);
                le = __builtin_amdgcn_alignbit(le, (uint32_t)(v[s][j] - (es + 1)), 31);
            }
        }
        less += __popc(lt);
        return __brev(le & ~lt);
    };
    uint32_t kept[kGroupKeep];
    int cnt = 0;
#pragma unroll
    for (int b = 0; b < kGroupKeep; ++b) {
        kept[b] = lo + b * kGroupBatch < hi ? sweep(lo + b * kGroupBatch) : 0u;
        cnt += __popc(kept[b]);
    }
    for (uint32_t p0 = lo + kGroupKeep * kGroupBatch; p0 < hi; p0 += kGroupBatch) cnt += __popc(sweep(p0));
    const bool tail = wave == kGroupWaves - 1 && lane == 0;
    if (tail)
        for (uint32_t p = n4; p < n_pairs; ++p) {
            cnt += ids[p] == e;
            less += ids[p] < e;
        }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        cnt += __shfl_xor(cnt, o, 64);
        less += __shfl_xor(less, o, 64);
    }
    if (lane == 0) {
        s_cnt[wave] = cnt;
        s_less[wave] = less;
    }
    __syncthreads();
    int base = 0, total = 0, running = 0;
#pragma unroll
    for (int i = 0; i < kGroupWaves; ++i) {
        base += s_less[i];
        running += i < wave ? s_cnt[i] : 0;
        total += s_cnt[i];
    }
    running += base;
    if (threadIdx.x == 0) {
        counts[e] = total;
        offsets[e] = base;
        if (e == E - 1) offsets[E] = base + total;
    }
    auto put = [&](int pos, uint32_t p) {
        pairs[pos] = (int32_t)p;
        tokens[pos] = (int32_t)(__umulhi(2 * p, topk_magic) >> topk_shift);   // p / topk
    };
    auto place = [&](uint32_t p0, uint32_t w) {
        for (int s = 0; s < 8; ++s, w >>= 4) {
            uint32_t h = w & 15u;
            if (__ballot(h != 0) == 0) continue;
            int before = 0, here = 0;   // hits of the lanes below, of the step
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const unsigned long long m = __ballot((h >> j) & 1u);
                before = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, before));
                here += __popcll(m);
            }
            int pos = running + before;
            for (; h; h &= h - 1) put(pos++, p0 + s * kGroupStep + lane * 4 + __builtin_ctz(h));
            running += here;
        }
    };
#pragma unroll
    for (int b = 0; b < kGroupKeep; ++b) place(lo + b * kGroupBatch, kept[b]);
    for (uint32_t p0 = lo + kGroupKeep * kGroupBatch; p0 < hi; p0 += kGroupBatch) place(p0, sweep(p0));
    if (tail)
        for (uint32_t p = n4; p < n_pairs; ++p)
            if (ids[p] == e) put(running++, p);
}

// Grouping for small batches (decode) by ONE workgroup, with no zeroing pass and no global atomics.
// A token selects an expert at most once, so the pairs of an expert are ordered by token alone: the
// workgroup builds a bit matrix B[expert][token] in LDS (atomic OR, order-free), prefix pop-counts per
// 32-token word give every word's start inside its expert, a scan over the experts gives the offsets, and
// a pair (t, slot) of expert e lands at offsets[e] + start[e][t / 32] + popcount(B[e][t / 32] below bit t):
// the same stable order (expert, token, slot) the large-batch kernels produce.
constexpr int kSmallThreads = 1024;
constexpr int kSmallMaxT = 512;
constexpr int kSmallWords = kSmallMaxT / 32;
constexpr int kSmallMaxPairs = 4096;

__global__ __launch_bounds__(kSmallThreads) void group_small_kernel(const int32_t *__restrict__ ids, int T, int E,
                                                                   int topk, int32_t *__restrict__ counts,
                                                                   int32_t *__restrict__ offsets,
                                                                   int32_t *__restrict__ pairs,
                                                                   int32_t *__restrict__ tokens)
{
    __shared__ uint32_t s_bits[256 * kSmallWords];
    __shared__ uint16_t s_start[256 * kSmallWords];
    __shared__ int s_off[257];
    const int tid = threadIdx.x, lane = tid & 63;
    const int n_pairs = T * topk, words = (T + 31) / 32;
    for (int i = tid; i < E * words; i += kSmallThreads) s_bits[i] = 0;
    __syncthreads();
    constexpr int kMine = kSmallMaxPairs / kSmallThreads;
    int my_e[kMine];
#pragma unroll
    for (int u = 0; u < kMine; ++u) {
        const int pidx = tid + u * kSmallThreads;
        my_e[u] = -1;
        if (pidx < n_pairs) {
            const int e = ids[pidx], t = pidx / topk;
            my_e[u] = e;
            atomicOr(&s_bits[e * words + (t >> 5)], 1u << (t & 31));
        }
    }
    __syncthreads();
    if (tid < E) {
        int run = 0;
        for (int w = 0; w < words; ++w) {
            s_start[tid * words + w] = (uint16_t)run;
            run += __popc(s_bits[tid * words + w]);
        }
        counts[tid] = run;
        s_off[tid + 1] = run;
    }
    if (tid == 0) s_off[0] = 0;
    __syncthreads();
    if (tid < 64) {   // inclusive scan of the counts over the experts, four per lane
        int v[4], sum = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            v[j] = (lane * 4 + j < E) ? s_off[lane * 4 + j + 1] : 0;
            sum += v[j];
        }
        int incl = sum;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int up = __shfl_up(incl, o, 64);
            if (lane >= o) incl += up;
        }
        int run = incl - sum;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            run += v[j];
            if (lane * 4 + j < E) s_off[lane * 4 + j + 1] = run;
        }
    }
    __syncthreads();
    if (tid <= E) offsets[tid] = s_off[tid];
#pragma unroll
    for (int u = 0; u < kMine; ++u) {
        const int pidx = tid + u * kSmallThreads;
        const int e = my_e[u];
        if (e >= 0) {
            const int t = pidx / topk;
            const uint32_t below = s_bits[e * words + (t >> 5)] & ((1u << (t & 31)) - 1u);
            const int pos = s_off[e] + s_start[e * words + (t >> 5)] + __popc(below);
            pairs[pos] = pidx;
            tokens[pos] = t;
        }
    }
}

int launch_route_only(const void *logits, int T, int E, int topk, int renorm, int32_t *ids, float *w, hipStream_t s)
{
    const int per_block = kRouteThreads / 64;
    const dim3 grid((T + per_block - 1) / per_block), block(kRouteThreads);
    const uint16_t *lg = (const uint16_t *)logits;
    if (E == 64)
        route_topk_kernel<1><<<grid, block, 0, s>>>(lg, T, E, topk, renorm, ids, w);
    else if (E == 128)
        route_topk_kernel<2><<<grid, block, 0, s>>>(lg, T, E, topk, renorm, ids, w);
    else
        route_topk_kernel<kMaxPerLane><<<grid, block, 0, s>>>(lg, T, E, topk, renorm, ids, w);
    return check_hip(hipGetLastError(), "route_topk_kernel");
}

int launch_route(const void *logits, int T, int E, int topk, int renorm, int32_t *ids, float *w,
                 int32_t *counts, int32_t *offsets, int32_t *pairs, int32_t *tokens, hipStream_t s)
{
    const int64_t n_pairs = (int64_t)T * topk;
    if (T > 0 && T <= kSmallMaxT && n_pairs <= kSmallMaxPairs) {
        int rc = launch_route_only(logits, T, E, topk, renorm, ids, w, s);
        if (rc) return rc;
        group_small_kernel<<<dim3(1), dim3(kSmallThreads), 0, s>>>(ids, T, E, topk, counts, offsets, pairs, tokens);
        return check_hip(hipGetLastError(), "group_small_kernel");
    }
    if (T > 0) {
        int rc = launch_route_only(logits, T, E, topk, renorm, ids, w, s);
        if (rc) return rc;
    }
    // p / topk == (p * magic) >> (31 + shift) for p < 2^31, magic = ceil(2^(31 + shift) / topk), shift = ceil(log2 topk)
    int shift = 0;
    while ((1 << shift) < topk) ++shift;
    const uint32_t magic = (uint32_t)(((1ULL << (31 + shift)) + topk - 1) / topk);
    group_by_expert_kernel<<<dim3(E), dim3(kGroupThreads), 0, s>>>(ids, (uint32_t)n_pairs, E, magic, shift, counts, offsets,
                                                                   pairs, tokens);
    return check_hip(hipGetLastError(), "group_by_expert_kernel");
}

}  // namespace qarl
