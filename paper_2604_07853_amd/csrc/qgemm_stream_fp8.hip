// Weight-streaming grouped GEMM: the e4m3 instantiations of qgemm_stream_fp8.hpp, the grid of both code formats, and the dispatch
// of the streaming path.
#include <math.h>

#include <algorithm>

#include "qgemm_stream_fp8.hpp"

namespace qarl {

namespace {

using namespace stream8;

// Rows (in 16-row tiles, row blocks) and slices of the weight tiles that a launch gives every expert; MT 0: K too large.
struct StreamGrid {
    int MT, m_split, n_slices;
};
StreamGrid stream_grid(int N, int K, int E, int64_t M, bool routed, bool w4)
{
    StreamGrid g;
    // rows per expert the grid should cover in one pass: mean + 4 sigma of a uniform router
    const double mean = (double)M / (double)E;
    const double need = mean + 4.0 * sqrt(mean);
    // token tiles per workgroup: limited by the LDS tile, which holds the whole K of every row, and by the gather (16 blocks of 16
    // bytes per thread).  More rows per expert go to further row blocks (m_split), each a pass over the expert's weights.  Blocks of
    // 64 rows where the slices alone fill the chip (routed layers, top-8 of 128, two blocks of 32 -> one of 64: 300 tokens FP8
    // 196 -> 148 us, FP4 137 -> 107, 512 tokens 203 -> 160 and 144 -> 118); with few experts blocks of 32 run side by side
    // (16 experts 1536 x 2048, 48 rows each: FP8 30 against 33 us, FP4 24 against 28).
    // FP4, routed: where the ring in LDS fits beside 32 rows and not beside 64, two blocks of 32, the second reading the weights out of L2 (300 / 400 /
    // 512 tokens, even router, layer 102 / 108 / 113 -> 102 / 106 / 111 us, Zipf 114 / 116 / 163 -> 113 / 115 / 134; FP8, whose codes are twice as
    // many: 141 / 147 / 153 -> 152 / 159 / 164).  K an odd multiple of 128 has no ring in LDS at either height and keeps 64 rows (128 experts, top-8,
    // 32 -> 64 rows, 270 / 400 / 512 tokens: 1408 x 768 111 / 117 / 119 -> 84 / 90 / 93 us, Zipf 119 / 120 / 136 -> 98 / 101 / 140; 1664 x 1408
    // 247 / 253 / 256 -> 166 / 175 / 181, Zipf 243 / 244 / 246 -> 176 / 179 / 242; 1920 x 768, Zipf, 512 tokens 139 -> 155).
    auto ring_in_lds = [&](int MT) { return lr_shape_fits(w4, K, MT, kLrStages, N / 32, 1); };
    const bool mt4 = stream_lds_bytes(K, 4, routed) <= 160 * 1024 && K <= 2048 && !(routed && w4 && ring_in_lds(2) && !ring_in_lds(4));
    const int mt_fit = mt4 ? 4 : stream_lds_bytes(K, 2, routed) <= 160 * 1024 ? 2
                       : stream_lds_bytes(K, 1, routed) <= 160 * 1024 ? 1 : 0;
    const int max_slices = (N / 32 + kSWaves - 1) / kSWaves;
    g.MT = need <= 16.0 ? 1 : need <= 32.0 || mt_fit < 4 || E * max_slices < 256 ? 2 : 4;
    if (g.MT > mt_fit) g.MT = mt_fit < 1 ? 0 : 1;
    const int ms = g.MT ? (int)ceil(need / (16.0 * g.MT)) : 1;
    g.m_split = ms < 1 ? 1 : (ms > 8 ? 8 : ms);
    // slices per expert: aim at one workgroup per CU, at least one pair of tiles per wavefront
    g.n_slices = (256 + E * g.m_split - 1) / (E * g.m_split);
    if (g.n_slices > max_slices) g.n_slices = max_slices;
    if (g.n_slices < 1) g.n_slices = 1;
    return g;
}

int launch_one(const GemmArgs &a, hipStream_t s)
{
    StreamParams p;
    p.codes = (const uint32_t *)a.codes;
    p.scales = (const float *)a.scales;
    p.x = a.x;
    p.x_scales = a.x_scales;
    p.row_map = a.row_map;
    p.out_row_map = a.out_row_map;
    p.offsets = a.offsets;
    p.out = a.out;
    p.E = a.E;
    p.N = a.N;
    p.K = a.K;
    p.out_f32 = a.out_f32;
    p.w4 = (a.fmt == QARL_FP4_E2M1_CH);
    p.ids = a.ids;
    p.n_ids = (int)a.M;
    p.topk = a.topk;
    p.x_per_token = a.x_per_token;
    const bool routed = a.ids != nullptr;
    if (routed && (a.M > kIdsMax || a.topk <= 0 || a.M % a.topk != 0 || a.M / a.topk > kIdsRows || ((uintptr_t)a.ids & 15) != 0)) {
        set_error("qgemm (routed decode path): needs T <= %d, T * topk <= %d and 16-byte aligned ids", kIdsRows, kIdsMax);
        return QARL_ERR_UNSUPPORTED;
    }
    p.n_units = a.N / 32;   // SILU_MUL: (N / 2) / 16
    const StreamGrid g = stream_grid(a.N, a.K, a.E, a.M, routed, p.w4);
    if (g.MT < 1) {
        set_error("qgemm (decode path): K=%d does not fit the LDS tile", a.K);
        return QARL_ERR_UNSUPPORTED;
    }
    p.m_split = g.m_split;
    p.n_slices = g.n_slices;
    p.spread = spread_blocks(a, 16 * g.MT * g.m_split);
    return p.w4 ? launch_fp4(p, a.epilogue, g.MT, s) : launch_codes<false>(p, a.epilogue, g.MT, s);
}

}  // namespace

bool qgemm_stream_routed_supported(int fmt, int N, int K, int T, int topk)
{
    if (fmt == QARL_W4A16_G128 || fmt == QARL_W4A8_G128) return qgemm_stream_w4_routed_supported(N, K, T, topk);
    if (fmt != QARL_FP8_E4M3_CH && fmt != QARL_FP4_E2M1_CH) return false;
    if (!qgemm_stream_supported(fmt, N, K) || T <= 0 || topk <= 0) return false;
    if (T > kIdsRows || (int64_t)T * topk > kIdsMax) return false;
    return stream_lds_bytes(K, 1, true) <= 160 * 1024;
}

// See qgemm_small_w4_us: start-up, a wavefront's pairs of tiles one after the other, the weights of the experts that have
// rows, the results, the combine's launch, and the rows such an expert has.
double qgemm_stream_routed_us(int fmt, int N, int K, int E, int T, int topk, int epilogue)
{
    const int64_t M = (int64_t)T * topk;
    const double G = K / kGroup, comb = epilogue == QARL_EPI_COMBINE;
    const double used = E * (1. - pow(1. - std::min(1., (double)topk / E), T)), rows = M / used;
    const double w = used * N * K * 1e-6, y = (double)M * N * 1e-6;
    if (fmt == QARL_W4A16_G128 || fmt == QARL_W4A8_G128) {
        const double c = qgemm_stream_w4_units_per_wave(N, K, E, M);
        return fmt == QARL_W4A16_G128 ? 5.9 + c * (0.61 + 0.436 * G) + 0.035 * w + 13 * y + 2.25 * comb + 0.05 * rows
                                      : 6.5 + c * (0.39 + 0.476 * G) + 0.033 * w + 12 * y + 2.1 * comb + rows * (0.17 + 0.0015 * G);
    }
    const StreamGrid g = stream_grid(N, K, E, M, true, fmt == QARL_FP4_E2M1_CH);
    const double c = (N / 32 + g.n_slices * kSWaves - 1) / (g.n_slices * kSWaves);
    // (the ring in LDS; 19 000 calls, half of them layer shapes of 64 and 128 experts with rotating weights: off by 9 % and 6 %)
    return fmt == QARL_FP8_E4M3_CH ? 4.0 + c * (0.25 + 0.47 * G) + 0.061 * w + 6.1 * y + 2.55 * comb + rows * (0.034 + 0.0126 * G)
                                   : 4.0 + c * (0.43 + 0.367 * G) + 0.018 * w + 6.9 * y + 2.4 * comb + rows * (0.058 + 0.009 * G);
}

bool qgemm_stream_supported(int fmt, int N, int K)
{
    if (fmt == QARL_W4A16_G128 || fmt == QARL_W4A8_G128) return qgemm_stream_w4_supported(N, K);
    if (N % 32 != 0 || K % kGroup != 0 || K > 4096) return false;  // the gather sweeps >= 2 rows per step
    return stream_lds_bytes(K, 1) <= 160 * 1024;
}

int launch_qgemm_stream(const GemmArgs &a, hipStream_t s)
{
    if (!qgemm_stream_supported(a.fmt, a.N, a.K)) {
        set_error("qgemm (decode path): unsupported shape N=%d K=%d (needs N %% 32 == 0; W4A16: K %% 256 == 0, K <= 4096; "
                  "FP8: K %% 128 == 0, K <= 4096; the token tile of one row block must fit LDS)", a.N, a.K);
        return QARL_ERR_UNSUPPORTED;
    }
    if (a.fmt == QARL_W4A16_G128 || a.fmt == QARL_W4A8_G128) return launch_qgemm_stream_w4(a, s);
    return launch_one(a, s);
}

}  // namespace qarl
