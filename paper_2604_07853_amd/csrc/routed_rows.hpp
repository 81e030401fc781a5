// Routed mode of the weight-streaming kernels (qarl_qgemm_routed): a workgroup of 512 threads finds the rows of its expert
// among the router's ids, and the row blocks of popular experts are dealt to all workgroups.
#pragma once
#include "common.hpp"

namespace qarl {

constexpr int kListWaves = 8;
constexpr int kIdsMax = 4096;    // pairs a workgroup scans (8 per thread)
constexpr int kIdsRows = 512;    // rows of one expert it can list: one per token, T <= 512
constexpr int kSpreadExperts = 256;   // experts the counts per expert have room for
// LDS of the routed mode behind the token tile: activation rows and pair ids of the expert, counts per wavefront, rows per expert
constexpr int kIdsBytes = 8 * kIdsRows + 4 * kListWaves + 4 * kSpreadExperts;

// The thread's share of the router's ids: pairs 8 tid .. 8 tid + 7 (-1 past the end).
__device__ __forceinline__ void load_ids(const int32_t *ids, int n_ids, int (&idv)[8])
{
    const int base = threadIdx.x * 8;
#pragma unroll
    for (int q4 = 0; q4 < 2; ++q4) {
        const int b4 = base + 4 * q4;
        i32x4 v4 = {-1, -1, -1, -1};
        if (b4 + 3 < n_ids) {
            v4 = *(const i32x4 *)(ids + b4);
        } else {
            for (int k = 0; b4 + k < n_ids; ++k) v4[k] = ids[b4 + k];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) idv[4 * q4 + k] = v4[k];
    }
}

// The pairs of expert e among the router's ids by increasing pair id, the (token, slot) order a stable grouping gives:
// activation rows to list[0 ..], pair ids to list[kIdsRows ..]; returns their number.  list[2 kIdsRows ..] is scratch of
// kListWaves counts.  The caller puts a barrier in front of its reads of the list, and one between two calls.
__device__ __forceinline__ int list_pairs(const int (&idv)[8], int e, int x_per_token, int topk, int *list)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, base = tid * 8;
    // hits of the lanes below, of the whole wavefront: eight ballots (a scan by shuffles is six dependent LDS operations)
    uint32_t hits = 0;
    int below = 0, in_wave = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const uint64_t b = __ballot(idv[k] == e);
        hits |= (idv[k] == e) ? (1u << k) : 0u;
        below = __builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, below));
        in_wave += __popcll(b);
    }
    int *s_wcnt = list + 2 * kIdsRows;
    if (lane == 0) s_wcnt[wave] = in_wave;
    lds_barrier();
    int before = 0, total = 0;
#pragma unroll
    for (int w = 0; w < kListWaves; ++w) {
        const int cw = s_wcnt[w];
        before += w < wave ? cw : 0;
        total += cw;
    }
    int rank = before + below;
    for (uint32_t hm = hits; hm; hm &= hm - 1) {
        const int pr = base + __builtin_ctz(hm);
        if (rank < kIdsRows) {
            list[rank] = x_per_token ? pr / topk : pr;
            list[kIdsRows + rank] = pr;
        }
        ++rank;
    }
    return min(total, kIdsRows);
}
__device__ __forceinline__ int list_pairs(const int32_t *ids, int n_ids, int e, int x_per_token, int topk, int *list)
{
    int idv[8];
    load_ids(ids, n_ids, idv);
    return list_pairs(idv, e, x_per_token, topk, list);
}

// Rows of every expert, s_hist[0 .. kSpreadExperts - 1]; ends with a barrier.
__device__ __forceinline__ void count_rows(const int32_t *ids, int n_ids, int E, int *s_hist)
{
    const int tid = threadIdx.x;
    int idv[8];
    load_ids(ids, n_ids, idv);
    if (tid < kSpreadExperts) s_hist[tid] = 0;
    lds_barrier();
#pragma unroll
    for (int k = 0; k < 8; ++k)
        if ((uint32_t)idv[k] < (uint32_t)E) atomicAdd(s_hist + idv[k], 1);
    lds_barrier();
}

// ---- Row blocks of popular experts.  The grid gives every expert m_split row blocks (what an even router needs) times
// `slices` workgroups.  What an expert has beyond them is dealt to the workgroups that find no row in their own block, and
// to those of the popular experts themselves; they count the ids per expert and ask spread_item() for their k-th share.
// Shares are sub-items, 1 / subs of a (row block, slice): workgroups without rows take a whole slice first, the rest goes
// round all takers one sub-item each.  All compute the same assignment from the same counts, nothing is exchanged.  The
// other workgroups, i.e. all of them under an even router, neither count nor ask (counting in all of them costs a layer
// 1.2 us).  As passes of the popular expert's own workgroups, its CUs worked alone while the rest of the chip was idle.
// Layers of 128 experts 2048 x 768, top-8, Zipf 1.1, 64 / 256 / 512 tokens, before -> after in us: W4A16 108 / 392 / 593 ->
// 69 / 82 / 166, W4A8 130 / 483 / 783 -> 76 / 88 / 152, FP8 323 / 720 / 1290 -> 99 / 119 / 213, FP4 207 / 486 / 830 -> 69 / 87 / 177.

// A kernel's argument, thread and workgroup ids read anew: what is computed from them belongs to the shares alone and is not kept
// in registers through the workgroup's own block (kept, it cost the launches of an even router 1-2 %).
template <typename P>
struct FreshArgs {
    P p;
    int tid;
    unsigned bid;
    __device__ __forceinline__ FreshArgs()
    {
        auto a = (const __attribute__((address_space(4))) P *)__builtin_amdgcn_kernarg_segment_ptr();   // P is the only argument
        tid = threadIdx.x;
        bid = blockIdx.x;
        asm volatile("" : "+s"(a), "+s"(bid), "+v"(tid));
        __builtin_memcpy(&p, (const void *)a, sizeof(P));
    }
};

struct SpreadItem {
    int e, block, sub, n_sub;   // row block of expert e; sub-items sub .. sub + n_sub - 1 of the expert's slices * subs
};
// Whether an expert of the call may have more rows than the grid gives it: a router names an expert once per token (an
// expert that is named more often has its further blocks as passes of its own workgroups).
inline int spread_blocks(const GemmArgs &a, int grid_rows)
{
    return a.ids && a.spread && a.E <= kSpreadExperts && a.M / a.topk > grid_rows;
}
// m_split row blocks of 1 << rows_sh rows, workgroup (e, mh, slice); false: no k-th share.
__device__ __forceinline__ bool spread_item(const int *s_hist, int E, int rows_sh, int m_split, int slices, int subs, int e,
                                            int mh, int slice, int k, SpreadItem &it)
{
    const int lane = threadIdx.x & 63, up_to = (1 << rows_sh) - 1;
    int over[4], osum = 0, isum = 0, before = 0;   // row blocks to deal; blocks of the grid without rows; with a share to take
#pragma unroll
    for (int q = 0; q < 4; ++q) {   // four experts per lane
        const int ex = lane * 4 + q, nb = ex < E ? (s_hist[ex] + up_to) >> rows_sh : 0;
        const int idle = ex < E ? max(0, m_split - nb) : 0;
        over[q] = max(0, nb - m_split);
        const int pop = over[q] > 0 ? m_split : 0;
        if (q < (e & 3)) before += idle + (pop << 16);
        osum += over[q];
        isum += idle + (pop << 16);   // both counts below 2^15: at most 256 experts x 8 row blocks
    }
    if (__ballot(osum > 0) == 0) return false;
    int incl_o = osum, incl_i = isum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int up_o = __shfl_up(incl_o, o, 64), up_i = __shfl_up(incl_i, o, 64);
        if (lane >= o) {
            incl_o += up_o;
            incl_i += up_i;
        }
    }
    const int n_over = __builtin_amdgcn_readlane(incl_o, 63), all = __builtin_amdgcn_readlane(incl_i, 63);
    const int mine = __builtin_amdgcn_readlane(incl_i - isum + before, __builtin_amdgcn_readfirstlane(e >> 2));
    const int nb_e = __builtin_amdgcn_readfirstlane((s_hist[e] + up_to) >> rows_sh);
    const int n_idle = (all & 0xffff) * slices, n_pop = (all >> 16) * slices, n_all = n_idle + n_pop;
    int i;
    it.n_sub = 1;
    if (mh >= nb_e) {
        const int rank = ((mine & 0xffff) + mh - nb_e) * slices + slice;
        if (k == 0) it.n_sub = subs;
        i = k == 0 ? rank * subs : n_idle * subs + n_pop + rank + (k - 1) * n_all;
    } else {
        i = n_idle * subs + ((mine >> 16) + mh) * slices + slice + k * n_all;
    }
    const int per_block = slices * subs;
    if (i >= n_over * per_block) return false;
    const int b = i / per_block;
    it.sub = i - b * per_block;
    int base = incl_o - osum, found = -1, blk = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        if (b >= base && b < base + over[q]) {
            found = lane * 4 + q;
            blk = b - base;
        }
        base += over[q];
    }
    const int src = __ffsll((long long)__ballot(found >= 0)) - 1;   // b < n_over: exactly one lane has it
    it.e = __builtin_amdgcn_readlane(found, src);
    it.block = m_split + __builtin_amdgcn_readlane(blk, src);
    return true;
}

}  // namespace qarl
