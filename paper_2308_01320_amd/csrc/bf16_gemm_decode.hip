// bf16 path: the launchers and plans of the decode GEMMs and of the LM head.
#include "bf16_decode_kernels.h"

namespace {

// One block per sequence: combines the LM-head partials of the workgroups (or wavefronts) in their order
// (deterministic), writes token id and its untempered log-probability; advance: the step ends here.  One trip over the
// partials, a thread's first requested with the state it needs at the end (4.8 -> 3.4 us for one sequence of 225 partials).
struct LmBest { float score; int id; float z; };
__device__ __forceinline__ void lm_take(LmBest& b, float s, int id, float z) {
    if (s > b.score || (s == b.score && id < b.id)) { b.score = s; b.id = id; b.z = z; }
}
template <int CTRL>
__device__ __forceinline__ void lm_take_dpp(LmBest& b) {
    lm_take(b, lane_dpp<CTRL>(b.score), __builtin_amdgcn_mov_dpp(b.id, CTRL, 0xF, 0xF, false), lane_dpp<CTRL>(b.z));
}
__device__ __forceinline__ void lm_take_apart(LmBest& b, int o) { lm_take(b, __shfl_xor(b.score, o), __shfl_xor(b.id, o), __shfl_xor(b.z, o)); }
__global__ __launch_bounds__(256) void lm_reduce_kernel(const float4* __restrict__ stats, const int* __restrict__ stats_idx, int n_tiles,
                                 he_dev_state* st, int32_t* __restrict__ ids_out,
                                 float* __restrict__ lp_out, int out_stride, int out_at_step,
                                 int32_t* __restrict__ cur_ids, int advance) {
    __shared__ float2 sms[4];
    __shared__ LmBest sbest[4];
    const int b = blockIdx.x, wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const float4* sp = stats + (size_t)b * n_tiles;
    const int* ip = stats_idx + (size_t)b * n_tiles;
    const int q = row_seq(st, b, 1);  // outputs and the next input belong to the row's sequence
    const int step = st->step;
    // soft-max of a thread's partials as it meets them: (largest, sum of exponentials below it)
    float mx = -INFINITY, sum = 0.f;
    LmBest best{-INFINITY, 0x7FFFFFFF, 0.f};
    for (int t = threadIdx.x; t < n_tiles; t += 256) {
        const float4 e = sp[t];
        const int id = ip[t];
        const float top = fmaxf(mx, e.x);
        // (a slice of nothing above -inf adds its sum as it is: 0, or the NaN of a logit)
        sum = (mx > -INFINITY ? sum * expf(mx - top) : sum) + (e.x > -INFINITY ? e.y * expf(e.x - top) : e.y);
        mx = top;
        lm_take(best, e.z, id, e.w);
    }
    const float wmax = lane_max<64>(mx);
    sum = lane_sum<64>(mx > -INFINITY ? sum * expf(mx - wmax) : sum);
    lm_take_dpp<0xB1>(best); lm_take_dpp<0x4E>(best); lm_take_dpp<0x141>(best); lm_take_dpp<0x140>(best);
    lm_take_apart(best, 16); lm_take_apart(best, 32);
    if (lane == 0) { sms[wave] = make_float2(wmax, sum); sbest[wave] = best; }
    __syncthreads();
    if (threadIdx.x == 0) {
        mx = fmaxf(fmaxf(sms[0].x, sms[1].x), fmaxf(sms[2].x, sms[3].x));
        sum = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            sum += sms[w].x > -INFINITY ? sms[w].y * expf(sms[w].x - mx) : sms[w].y;
            if (w) lm_take(best, sbest[w].score, sbest[w].id, sbest[w].z);
        }
        if (!(mx > -INFINITY)) sum = __builtin_nanf("");  // no logit above -inf: no probabilities
        const size_t at = (size_t)q * out_stride + (out_at_step ? step : 0);
        ids_out[at] = best.id;
        lp_out[at] = (best.z - mx) - logf(sum);
        if (cur_ids) cur_ids[q] = best.id;
    }
    if (advance) advance_state_by_last(st, 1, 1);
}

#ifndef HE_SKINNY_U
#define HE_SKINNY_U(NT) ((NT) <= 4 ? 4 : 2)
#endif
#ifndef HE_SKINNY_W8_MAXNT
#define HE_SKINNY_W8_MAXNT 2
#endif
template <int MODE, int NT>
void launch_skinny_nt(hipStream_t s, const void* Wp, const void* Xhi, int KB, int n_tiles,
                      int m_tiles, const Epi& p) {
    constexpr int U = HE_SKINNY_U(NT);
    dim3 grid(1, (n_tiles + NT - 1) / NT, m_tiles);
    if (MODE == MODE_LMHEAD && m_tiles > 1) grid.y = (grid.y + 7) / 8 * 8;  // see the kernel: slices of a tile group share an XCD
    // What bounds a wavefront is its serial chain of load rounds (K/16 blocks / wavefronts / U
    // rounds, about 1.7 us each under load): eight wavefronts halve the chain when K leaves each
    // of them two rounds (and their accumulators still fit in LDS for the final reduction).
    const bool eight = NT <= HE_SKINNY_W8_MAXNT && KB / 8 >= 2 * U;
    const int parts = eight ? 8 : 4;
    // Ask for more than half of a CU's LDS so that no two workgroups share a CU: with at most one
    // workgroup per CU the dispatcher has to spread a launch of <= #CUs workgroups evenly.
    constexpr size_t kWant = 84 * 1024;
    if (eight) {
        constexpr size_t kStatic = (size_t)8 * NT * 16 * 64 * sizeof(float);
        const size_t pad = kStatic >= kWant ? 0 : kWant - kStatic;
        gemm_skinny_kernel<MODE, NT <= HE_SKINNY_W8_MAXNT ? NT : 1, U, 8><<<grid, 512, pad, s>>>(
            (const u32x4*)Wp, (const u32x4*)Xhi, KB, n_tiles, 1, KB / parts, KB % parts, p);
    } else {
        constexpr size_t kStatic = (size_t)4 * NT * 16 * 64 * sizeof(float);
        const size_t pad = kStatic >= kWant ? 0 : kWant - kStatic;
        gemm_skinny_kernel<MODE, NT, U, 4><<<grid, 256, pad, s>>>((const u32x4*)Wp, (const u32x4*)Xhi,
                                                                  KB, n_tiles, 1, KB / parts, KB % parts, p);
    }
}

// nt weight tiles per workgroup (1..8)
template <int MODE>
void launch_skinny(hipStream_t s, const void* Wp, const void* Xhi, int KB, int n_tiles, int m_tiles,
                   int nt, const Epi& p) {
    switch (nt) {
        case 1: launch_skinny_nt<MODE, 1>(s, Wp, Xhi, KB, n_tiles, m_tiles, p); break;
        case 2: launch_skinny_nt<MODE, 2>(s, Wp, Xhi, KB, n_tiles, m_tiles, p); break;
        case 3: launch_skinny_nt<MODE, 3>(s, Wp, Xhi, KB, n_tiles, m_tiles, p); break;
        case 4: launch_skinny_nt<MODE, 4>(s, Wp, Xhi, KB, n_tiles, m_tiles, p); break;
        case 5: launch_skinny_nt<MODE, 5>(s, Wp, Xhi, KB, n_tiles, m_tiles, p); break;
        case 6: launch_skinny_nt<MODE, 6>(s, Wp, Xhi, KB, n_tiles, m_tiles, p); break;
        case 7: launch_skinny_nt<MODE, 7>(s, Wp, Xhi, KB, n_tiles, m_tiles, p); break;
        default: launch_skinny_nt<MODE, 8>(s, Wp, Xhi, KB, n_tiles, m_tiles, p); break;
    }
}

// Tiles per workgroup for a GEMM whose epilogue needs the whole sum in one workgroup: the
// smallest count that fits all workgroups on the chip at once (one per CU), at most 8.
int skinny_nt_fused(int n_tiles, int m_tiles) {
    const int cus = plan_cus();
    int nt = (n_tiles * m_tiles + cus - 1) / cus;
    return nt < 1 ? 1 : (nt > 8 ? 8 : nt);
}

}  // namespace

// ------------------------------------------------------------------ launchers

// How a decode-shaped GEMM is cut up: weight rows in units of 32 (the skinny kernel) or 16 (the
// half-tile kernel), `per_wg` units per workgroup, ks k-splits.  The launch waits for its most
// loaded workgroup, so the plan with the fewest weight bytes per workgroup wins, as long as all of
// its workgroups fit on the chip at once and every wavefront keeps at least 8 k-blocks.
struct GemmPlan { bool half; int per_wg, ks; };

static GemmPlan plan_fused(int M, int N) {  // epilogue needs the whole sum: no k-split
    const int n_tiles = (N + 31) / 32, m_tiles = (M + 31) / 32, cus = plan_cus();
    GemmPlan g{false, skinny_nt_fused(n_tiles, m_tiles), 1};
    if (m_tiles > 2 || N % 16) return g;
    const int n_half = N / 16, ht = (n_half + cus - 1) / cus;
    if (m_tiles == 2) {  // two row slices per workgroup (16-row-unit kernel only): the weights are streamed once
        if (ht <= kHalfMax2) g = GemmPlan{true, ht, 1};
        return g;
    }
    // (a matrix of no more units than CUs: a unit each; 3072 x 1024 in units 4.1 us, in twos 4.5)
    // up to 16 rows the 16-row-unit kernel also leaves out the unused half of the activation panel: it wins ties
    if (ht <= kHalfMax && (16 * ht < 32 * g.per_wg || (M <= 16 && 16 * ht == 32 * g.per_wg)))
        g = GemmPlan{true, ht, 1};
    return g;
}

// The out-projection and FC2, whose sums are added to the residual rows: always 16-row units, per_wg of them to a workgroup, in ks k
// ranges.  Microseconds of a plan beyond what all have in common, fitted to launches of 16 shapes from 512 x 512 to 9216 x 36864
// with 1 .. 64 rows (at most 5 % between the plan chosen and the fastest; a median of nothing):
//   the weight rows and the activation rows of a workgroup's k range at what a CU pulls of each, but never less than the whole
//   matrix takes from HBM, CUs without a workgroup not asking for anything;
//   the hand-off between k ranges, and the quads of outputs a thread finishes;
//   the statistics of one column group per workgroup, which every workgroup of the next GEMM reads for all of its rows.
// One range on a single unit per workgroup has no hand-off and its tail needs no barrier; against the plans before it (at least two units),
// 1 .. 16 rows: 2048 x 2048 7.0 -> 5.0 us, 4096 x 4096 10.1 -> 8.0, 2048 x 8192 (two ranges) 10.8 -> 9.2, 512 x 512 3.4 -> 2.5.
// Two slices (33 .. 64 rows) were planned by weight rows per workgroup alone: 48 rows, 4096 x 4096 20.9 (eight units, eight ranges) -> 12.4.
static double store_cost_us(int N, int K, int ht, int ks, int mh, bool w8, int cus) {
    const double bytes = w8 ? 1.0 : 2.0, w_rate = w8 ? 56.5e3 : 31.5e3, x_rate = w8 ? 82.1e3 : 102.6e3, hbm_rate = w8 ? 9.2e6 : 6.37e6;
    const double meet = w8 ? 0.81 : 1.02, per_range = w8 ? 0.31 : 0.33, per_quad = w8 ? 1.5 : 1.31, idle = w8 ? 0.11 : 1.4;
    const int groups = (N / 16 + ht - 1) / ht, waves = ht <= 4 && mh <= 2 ? 8 : 4;
    const double per_cu = (double)K / ks * (16.0 * bytes * ht / w_rate + 32.0 * mh / x_rate);
    const double hbm = bytes * N * K / hbm_rate * (1.0 + idle * std::max(0.0, 1.0 - (double)groups * ks / cus));
    return std::max(per_cu, hbm) + (ks > 1 ? meet + per_range * ks : 0.0) + per_quad * ((ht * mh + waves - 1) / waves) +
           0.0013 * mh * mh * groups;
}

// capacity: floats the k-split scratch can hold (0 = not checked)
static GemmPlan plan_store(int M, int N, int K, size_t capacity, bool w8) {
    const int m_tiles = (M + 31) / 32, slices = std::min(m_tiles, 2), mh = std::min((M + 15) / 16, 4), cus = plan_cus();
    // (more units to a workgroup: their accumulators do not fit the LDS that adds them up)
    const int most = slices == 2 ? kHalfMax2 : kHalfMax, rows = 2 * slices;
    const int step = w8 ? 64 : 16, least = w8 ? 4 : 8;  // k blocks, and how many of them a wavefront is left with at least
    GemmPlan g{true, most, 1};
    double best = 1e30;
    for (int ht = 1; ht <= most; ++ht) {
        const int groups = (N / 16 + ht - 1) / ht;
        if (groups > cus && ht < most) continue;
        for (int ks = 1; ks <= 8; ++ks) {
            if (ks > 1 && (groups * ks > cus || K / step / (ks * 4) < least)) break;
            // scratch the kernel will index: groups x splits x (items rounded up to the wavefronts) x 256 words
            if (ks > 1 && capacity && (size_t)groups * ks * (size_t)(rows * ht + 7) * 256 * ((m_tiles + slices - 1) / slices) > capacity) break;
            const double cost = store_cost_us(N, K, ht, ks, mh, w8, cus);
            if (cost < best) { best = cost; g = GemmPlan{true, ht, ks}; }
        }
    }
    return g;
}

// 8-bit weights: always the 16-row-unit kernel
static GemmPlan plan_fused_w8(int M, int N) {
    const int cus = plan_cus(), ht = (N / 16 + cus - 1) / cus;
    return GemmPlan{true, std::min(ht, M > 32 ? kHalfMax2 : kHalfMax), 1};
}

void bf16_plan_query(int M, int N, int K, int store, size_t capacity, int cus, int* unit_rows, int* per_wg, int* ks) {
    plan_cus_override = cus;
    const GemmPlan g = store ? plan_store(M, N, K, capacity, false) : plan_fused(M, N);
    plan_cus_override = 0;
    *unit_rows = g.half ? 16 : 32;
    *per_wg = g.per_wg;
    *ks = g.ks;
}

// What the MODE_STORE_LN launch of this shape indexes (host logic only): floats of k-split scratch, arrival
// counters, column groups of statistics per 32-row slice, and its k-split.
void bf16_store_footprint(int M, int N, int K, size_t capacity, int w8, int cus, size_t* scratch_floats,
                          size_t* need_floats, int* cells, int* stat_groups, int* ksplit) {
    StoreFootprint f{};
    plan_cus_override = cus;
    bf16_gemm_args a{};
    a.out_capacity = capacity;
    float one = 1.f;
    if (w8) a.wscale = &one;  // (never read: nothing is launched)
    g_dry = &f;
    bf16_gemm_skinny(nullptr, EPI_STORE_LN, nullptr, nullptr, M, N, K, 0, a);
    g_dry = nullptr;
    *need_floats = bf16_store_need(M, N, K, capacity, w8);
    plan_cus_override = 0;
    *scratch_floats = f.scratch_floats;
    *cells = f.cells;
    *stat_groups = f.stat_groups;
    *ksplit = f.ksplit;
}

void bf16_store_plan(int M, int N, int K, size_t capacity, int w8, int* group_cols, int* ks) {
    const GemmPlan g = plan_store(M, N, K, capacity, w8);
    *group_cols = g.per_wg * 16;
    *ks = g.ks;
}

// Floats of k-split scratch the EPI_STORE_LN launch of this shape may index (an upper bound: per column
// group, row-slice pair and split, one 256-float run per item, items rounded up to whole wavefronts).
size_t bf16_store_need(int M, int N, int K, size_t capacity, int w8) {
    const int m_tiles = (M + 31) / 32, slices = std::min(m_tiles, 2);
    const GemmPlan g = plan_store(M, N, K, capacity, w8);
    const size_t groups = (size_t)(N / 16 + g.per_wg - 1) / g.per_wg;
    return groups * ((m_tiles + slices - 1) / slices) * g.ks * (size_t)(2 * slices * g.per_wg + 7) * 256;
}

void bf16_gemm_skinny(hipStream_t s, int mode, const void* Wp, const void* Xhi, int M, int N, int K,
                      int ksplit, const bf16_gemm_args& a) {
    (void)ksplit;
    const Epi p = make_epi(M, N, a);
    const int KB = K / 16, n_tiles = (N + 31) / 32, m_tiles = (M + 31) / 32;
    if (a.wscale) {  // 8-bit weights: Wp holds E4M3 units
        const GemmPlan g = mode == EPI_STORE_LN ? plan_store(M, N, K, a.out_capacity, true) : plan_fused_w8(M, N);
        bf16_gemm_units8(s, mode, Wp, Xhi, M, N, K, g.per_wg, g.ks, a);
        return;
    }
    if (mode == EPI_STORE_LN) {  // the k-split is the one bf16_store_plan reports for this shape
        const GemmPlan g = plan_store(M, N, K, a.out_capacity, false);
        launch_half<MODE_STORE_LN, false>(s, Wp, Xhi, KB, N / 16, m_tiles, g.per_wg, g.ks, p);
        return;
    }
    const GemmPlan g = plan_fused(M, N);
    if (mode == EPI_BIAS_RELU) {
        if (g.half) launch_half<MODE_BIAS_RELU, false>(s, Wp, Xhi, KB, N / 16, m_tiles, g.per_wg, 1, p);
        else launch_skinny<MODE_BIAS_RELU>(s, Wp, Xhi, KB, n_tiles, m_tiles, g.per_wg, p);
    } else {
        if (g.half) launch_half<MODE_QKV, false>(s, Wp, Xhi, KB, N / 16, m_tiles, g.per_wg, 1, p);
        else launch_skinny<MODE_QKV>(s, Wp, Xhi, KB, n_tiles, m_tiles, g.per_wg, p);
    }
}

// (a matrix of 16 MiB at most, half of what the L2 caches hold: of a larger one the part that fits was fetched for nothing, a step of 7 rows,
// hidden 4096, 1 % slower)
bf16_ahead bf16_store_ahead(const void* Wp, int M, int N, int K, size_t capacity, bool w8) {
    bf16_ahead a;
    if ((size_t)N * K * (w8 ? 1 : 2) > (size_t)16 << 20) return a;
    bf16_gemm_args args{};
    args.out_capacity = capacity;
    float one = 1.f;
    if (w8) args.wscale = &one;  // (never read: nothing is launched)
    g_dry_ahead = &a;
    bf16_gemm_skinny(nullptr, EPI_STORE_LN, nullptr, nullptr, M, N, K, 0, args);
    g_dry_ahead = nullptr;
    a.w = Wp; a.n_units = N / 16; a.kb = K / 16; a.w8 = w8;
    return a;
}

// Tiles per workgroup of the streamed LM head.  All slices of a group of tiles run on one XCD, so a launch is one round where
// every XCD's groups times slices fit its CUs (32 here; a launch that only fits the chip as a whole waited for the XCDs that got a
// group more: 96 rows of 16000 x 5120 +31 us).
static int lm_stream_nt(int tiles, int slices) {
    if (slices == 1) return skinny_nt_fused(tiles, 1);
    const int groups = 8 * std::max(1, plan_cus() / 8 / slices);
    return (tiles + groups - 1) / groups;
}

// Whether the LM head of B rows streams the matrix once per 32 rows (gemm_skinny_kernel; slices after the first find it in L2)
// or takes all rows in 256-wide tiles (gemm_ring_kernel).  A small vocabulary gives the tiles a few workgroups only, each
// walking the whole of K (2000 ids: eight of 256 CUs); the line is where the 32-wide tiles of all slices no longer fit one
// round of at most eight per workgroup.  Measured a decode step, streamed / tiled, us, sampled where not said otherwise:
// K 1024, 64 rows: 2000 ids 50 / 75, 27000 65 / 79 (greedy 62 / 68); 192 rows, greedy: 6000 93 / 100.  K 5120, 64 rows: 12000
// 156 / 183, 20000 173 / 185 (greedy 173 / 175), 27000 192 / 211, beyond the line 50272 269 / 237; 96 rows: 20000 230 / 249; 160:
// 12000 257 / 270; 250: 6000 272 / 304.
bool bf16_lm_head_streams(int B, int V) { return B <= 32 || lm_stream_nt((V + 31) / 32, (B + 31) / 32) <= 8; }

// (streamed: one per workgroup of at least one 32-wide tile; tiled: one per wavefront of a 256-wide tile)
int bf16_lm_parts_max(int V) { return std::max((V + 31) / 32, 2 * ((V + 255) / 256)); }

void bf16_lm_head(hipStream_t s, const void* Wp, const void* Xhi, int B, int V, int K,
                  he_dev_state* st, float* logits_opt, float* stats, int* stats_idx, int32_t* ids_out,
                  float* lp_out, int out_stride, int out_at_step, int32_t* cur_ids, bool advance, const bf16_gemm_args* fold) {
    int parts;  // soft-max partials per row
    if (!bf16_lm_head_streams(B, V)) {
        parts = bf16_lm_head_tiles(s, Wp, Xhi, B, V, K, fold, st, logits_opt, stats, stats_idx);
    } else {
        Epi p{};
        if (fold) p = make_epi(B, V, *fold);
        const int tiles = (V + 31) / 32, m_tiles = (B + 31) / 32, nt = lm_stream_nt(tiles, m_tiles);
        p.M = B; p.N = V; p.st = st; p.logits = logits_opt; p.stats = stats; p.stats_idx = stats_idx;
        p.n_tiles = parts = (tiles + nt - 1) / nt;  // one per workgroup
        launch_skinny<MODE_LMHEAD>(s, Wp, Xhi, K / 16, tiles, m_tiles, nt, p);
    }
    lm_reduce_kernel<<<B, 256, 0, s>>>((const float4*)stats, stats_idx, parts, st, ids_out, lp_out, out_stride, out_at_step,
                                       cur_ids, advance ? 1 : 0);
}

