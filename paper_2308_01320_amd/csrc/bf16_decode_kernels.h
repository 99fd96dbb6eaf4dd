// bf16 path: the weight-streaming GEMM kernels of a decode step (at most 32 rows per slice) and of the LM head fused with
// log-softmax and sampling.  Weights and activations are tiled blocks of IEEE halves.  (A header: the launchers of 16-bit and of
// 8-bit weights are two files, compiled side by side.)
#pragma once
#include "bf16_common.h"

namespace he_bf16 {
// Host-side account of a MODE_STORE_LN launch: when `g_dry` is set the launchers below (called from the same thread) go through
// their choice of kernel variant and grid as usual, then record what that launch would index instead of launching it.
struct StoreFootprint { size_t scratch_floats; int cells; int stat_groups; int ksplit; };
inline thread_local StoreFootprint* g_dry = nullptr;
inline thread_local bf16_ahead* g_dry_ahead = nullptr;  // the same for who reads which weights
}  // namespace he_bf16
using namespace he_bf16;

namespace {

// Quads of outputs a thread of a workgroup holds after the k loop: the workgroup's (tile or unit, row part) items
// dealt out over its wavefronts.  One definition for the kernels and for the launchers' account of the scratch a
// launch indexes.
constexpr int items_per_wave(int items, int waves) { return (items + waves - 1) / waves; }
// Floats of k-split scratch one split of one column group covers (store_ln_tail's layout).
constexpr size_t tail_floats_per_split(int items, int waves) { return (size_t)items * 4 * waves * 64; }

// ----------------------------------------------------------------- k-split GEMM -> residual rows + next LayerNorm's input
//
// Tail of the decode-shaped out-projection / FC2 GEMMs (MODE_STORE_LN).  On entry every thread holds ITEMS quads
// v[i][0..3]: this workgroup's k-split partial sums of outputs n0[i]..n0[i]+3 of row mrow[i] (live[i]: the quad exists).
// rslot[i] says which of the lane's two rows per slice the quad belongs to: lanes with equal lane % LG hold different
// columns of the same rows.
//
// The partial sums cross workgroups (and XCDs, each with an L2 of its own) inside one launch.  They
// travel as agent-scope atomic words -- written through to, and read from, the level every XCD shares
// -- so no cache has to be flushed or invalidated (an agent-scope fence does that to whole L2s and cost
// 45 us per launch).  The 64-bit words of one (split, item, pair) are laid out thread after thread: every
// access is a contiguous 512 bytes per wavefront.  Each workgroup publishes its partial sums, waits for the
// stores to be acknowledged and counts itself in; whoever counts last for the column group reads all splits
// back -- its own included -- and adds them in split order, so the sum does not depend on which
// workgroup that was.  Nobody waits for anybody: the others are done.  The last one adds bias and
// residual, writes the residual rows back, gamma * x as half blocks, and the group's statistics
// (mean and sum of squared deviations per row over the group's `cnt` columns, fixed summation order).
// Returns to the caller, who returns.
// MT: 32-row slices the workgroup holds (rows mt*32 .. mt*32 + 32 MT - 1; mt = its first slice).
// residual, bias and gain of a thread's quads (TailOps): requested here, or by the caller ahead of its k loop where no
// hand-off lies in between (early)
template <int ITEMS>
struct TailOps { float4 resid[ITEMS]; uint2 bias[ITEMS], gamma[ITEMS]; };
// every lane loads (rows and columns past the end are clamped, their results never stored): no per-lane branches around the loads
template <int ITEMS>
__device__ __forceinline__ void tail_request(TailOps<ITEMS>& t, const Epi& p, int i, int mrow, int n0) {
    const int mc = min(mrow, p.M - 1), nc = min(n0, p.N - 4);
    t.resid[i] = *reinterpret_cast<const float4*>(p.resid + (size_t)mc * p.N + nc);
    t.bias[i] = *reinterpret_cast<const uint2*>(p.bias + nc);
    t.gamma[i] = *reinterpret_cast<const uint2*>(p.gamma + nc);
}
template <int ITEMS, int WAVES, int MT = 1, bool LONE = false>
__device__ __forceinline__ void store_ln_tail(const Epi& p, int ksplit, int ks, int grp, int groups, int mt, float cnt,
                                              const float (&v)[ITEMS][4], const int (&mrow)[ITEMS],
                                              const int (&n0)[ITEMS], const bool (&live)[ITEMS],
                                              const int (&rslot)[ITEMS], TailOps<ITEMS>& ops, bool early) {
    constexpr int LG = 16, NSLOT = 32 * MT / LG;
    __shared__ int s_last;
    __shared__ float sred[2][WAVES][32 * MT];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const size_t cell = (size_t)grp * gridDim.z + blockIdx.z;
    constexpr size_t kPer = tail_floats_per_split(ITEMS, WAVES);  // words of one split of one column group
    // 64-bit words (two sums each): a wavefront can have 63 loads outstanding, and the wider they are, the more
    // of the last workgroup's read-back is in flight at once
    uint64_t* scratch = reinterpret_cast<uint64_t*>(p.out + cell * ksplit * kPer) + threadIdx.x;
    constexpr size_t kPer2 = kPer / 2;
    auto pair_bits = [](float a, float b) { return (uint64_t)__float_as_uint(a) | ((uint64_t)__float_as_uint(b) << 32); };
    if (ksplit > 1) {
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            if (!live[i]) continue;
#pragma unroll
            for (int h = 0; h < 2; ++h)
                __hip_atomic_store(scratch + (ks * kPer2 + (size_t)(i * 2 + h) * WAVES * 64), pair_bits(v[i][2 * h], v[i][2 * h + 1]),
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (threadIdx.x == 0)
            s_last = __hip_atomic_fetch_add(p.counters + cell, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == ksplit - 1;
        __syncthreads();
        if (!s_last) return;
    }
    float x[ITEMS][4];
    float srow[NSLOT];
#pragma unroll
    for (int r = 0; r < NSLOT; ++r) srow[r] = 0.f;
    // The splits' partial sums come from the level all XCDs share, a microsecond or two away.  All loads of
    // a chunk of items are issued before anything is stored: with loads and stores outstanding together the
    // hardware counter no longer tells which have returned, and every wait would drain them all.
    constexpr int CH = ITEMS < 4 ? ITEMS : 4;
    auto lo32 = [](uint64_t w) { return __uint_as_float((uint32_t)w); };
    auto hi32 = [](uint64_t w) { return __uint_as_float((uint32_t)(w >> 32)); };
#pragma unroll
    for (int c0 = 0; c0 < ITEMS; c0 += CH) {
        uint64_t y[CH][8][2];
        uint2 hh[CH];
        if (!early) {
#pragma unroll
            for (int c = 0; c < CH; ++c)
                if (c0 + c < ITEMS) tail_request(ops, p, c0 + c, mrow[c0 + c], n0[c0 + c]);
        }
        if (ksplit > 1) {  // every split's sums, this workgroup's own included: one uniform test per split
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                if (k >= ksplit) break;
#pragma unroll
                for (int c = 0; c < CH; ++c) {
                    const int i = c0 + c;
                    if (i >= ITEMS) continue;
#pragma unroll
                    for (int h = 0; h < 2; ++h)
                        y[c][k][h] = __hip_atomic_load(scratch + (k * kPer2 + (size_t)(i * 2 + h) * WAVES * 64),
                                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
        }
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            const int i = c0 + c;
            if (i >= ITEMS) continue;
            x[i][0] = x[i][1] = x[i][2] = x[i][3] = 0.f;
            if (!live[i]) continue;
            float4 tot = make_float4(v[i][0], v[i][1], v[i][2], v[i][3]);
            if (ksplit > 1) {  // in split order, whichever split this workgroup was
                tot = make_float4(lo32(y[c][0][0]), hi32(y[c][0][0]), lo32(y[c][0][1]), hi32(y[c][0][1]));
#pragma unroll
                for (int k = 1; k < 8; ++k)
                    if (k < ksplit) {
                        tot.x += lo32(y[c][k][0]); tot.y += hi32(y[c][k][0]);
                        tot.z += lo32(y[c][k][1]); tot.w += hi32(y[c][k][1]);
                    }
            }
            const float4 rr = ops.resid[i];
            const uint2 bb = ops.bias[i], gg = ops.gamma[i];
            x[i][0] = rr.x + (tot.x + bf_lo(bb.x));
            x[i][1] = rr.y + (tot.y + bf_hi(bb.x));
            x[i][2] = rr.z + (tot.z + bf_lo(bb.y));
            x[i][3] = rr.w + (tot.w + bf_hi(bb.y));
            hh[c].x = pack2(x[i][0] * bf_lo(gg.x), x[i][1] * bf_hi(gg.x));
            hh[c].y = pack2(x[i][2] * bf_lo(gg.y), x[i][3] * bf_hi(gg.y));
            const float part = (x[i][0] + x[i][1]) + (x[i][2] + x[i][3]);
#pragma unroll
            for (int r = 0; r < NSLOT; ++r)
                if (rslot[i] == r) srow[r] += part;
        }
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            const int i = c0 + c;
            if (i >= ITEMS || !live[i]) continue;
            *reinterpret_cast<float4*>(p.resid + (size_t)mrow[i] * p.N + n0[i]) = make_float4(x[i][0], x[i][1], x[i][2], x[i][3]);
            const size_t slot = block_slot(mrow[i], n0[i] & ~7, p.N >> 4);
            reinterpret_cast<uint2*>(p.out_blocks + slot)[(n0[i] >> 2) & 1] = hh[c];
        }
    }
    // row sums over the lanes that share a row, then over the wavefronts
    if constexpr (LONE) {  // a group of one unit: its four lanes per row hold all of it (item 0 of a wavefront is its only one)
        const float sum = lane_sum_apart<LG>((x[0][0] + x[0][1]) + (x[0][2] + x[0][3]));
        const float mean = sum * (1.f / 16.f), d0 = x[0][0] - mean, d1 = x[0][1] - mean, d2 = x[0][2] - mean, d3 = x[0][3] - mean;
        const float m2 = lane_sum_apart<LG>((d0 * d0 + d1 * d1) + (d2 * d2 + d3 * d3));
        if (live[0] && lane < LG)
            p.stats_out[((size_t)(mrow[0] >> 5) * groups + grp) * 32 + (mrow[0] & 31)] = make_float2(mean, m2);
        if (threadIdx.x == 0 && ksplit > 1)
            __hip_atomic_store(p.counters + cell, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return;
    }
#pragma unroll
    for (int r = 0; r < NSLOT; ++r) {
        srow[r] = lane_sum_apart<LG>(srow[r]);
        if (lane < LG) sred[0][wave][LG * r + lane] = srow[r];
    }
    __syncthreads();
    float mean[NSLOT], q[NSLOT];
#pragma unroll
    for (int r = 0; r < NSLOT; ++r) {
        float tot = 0.f;
#pragma unroll
        for (int ww = 0; ww < WAVES; ++ww) tot += sred[0][ww][LG * r + (lane & (LG - 1))];
        mean[r] = tot / cnt;
        q[r] = 0.f;
    }
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        if (!live[i]) continue;
#pragma unroll
        for (int r = 0; r < NSLOT; ++r)
            if (rslot[i] == r) {
                const float d0 = x[i][0] - mean[r], d1 = x[i][1] - mean[r], d2 = x[i][2] - mean[r], d3 = x[i][3] - mean[r];
                q[r] += (d0 * d0 + d1 * d1) + (d2 * d2 + d3 * d3);
            }
    }
#pragma unroll
    for (int r = 0; r < NSLOT; ++r) {
        q[r] = lane_sum_apart<LG>(q[r]);
        if (lane < LG) sred[1][wave][LG * r + lane] = q[r];
    }
    __syncthreads();
    if (threadIdx.x < 32 * MT) {  // (wavefront 0: lane = row)
        float m2 = 0.f, tot = 0.f;
#pragma unroll
        for (int ww = 0; ww < WAVES; ++ww) { m2 += sred[1][ww][lane]; tot += sred[0][ww][lane]; }
        p.stats_out[((size_t)(mt + (lane >> 5)) * groups + grp) * 32 + (lane & 31)] = make_float2(tot / cnt, m2);
    }
    if (threadIdx.x == 0 && ksplit > 1)  // ready for the next launch
        __hip_atomic_store(p.counters + cell, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ----------------------------------------------------------------- skinny GEMM (decode, LM head)
//
// At most 32 rows per grid.z slice: weights are streamed exactly once from HBM,
// straight from global memory into MFMA operand registers.  A workgroup of four
// or eight wavefronts owns NT consecutive 32-row weight tiles; its
// wavefronts divide the k range, keep U blocks per stream in flight (NT weight
// streams plus the activation stream out of L2, which every weight
// tile reuses from registers), and combine their accumulators through LDS.
//
// The launcher picks NT to put one equally loaded workgroup on
// as many of the CUs as the shape allows: more workgroups than CUs double up
// on some CUs and the whole launch waits for those.  Measured on the 13B shapes:
// the stream itself runs at the HBM rate; what it competes for is the path from
// L2 to the CU, which carries the activation panel (half as many bytes again as the
// weights when NT = 2) next to the weights.  Everything executed once per launch
// (prologue, epilogue) is instruction-bound -- a wavefront issues one vector
// instruction per four cycles -- so the code around the loop is kept short and
// what the epilogue needs is requested behind the first round of weight loads.

template <int NT, int U>
struct SkinnyRegs {
    u32x4 w[NT][U], x[U];
};

template <int NT, int U>
__device__ __forceinline__ void skinny_load(SkinnyRegs<NT, U>& r, const u32x4* (&w)[NT], const u32x4*& xh) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
        for (int t = 0; t < NT; ++t) r.w[t][u] = __builtin_nontemporal_load(w[t] + u * 64);
        r.x[u] = xh[u * 64];
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) w[t] += U * 64;
    xh += U * 64;
}

template <int NT, int U>
__device__ __forceinline__ void skinny_mma(const SkinnyRegs<NT, U>& r, f32x16 (&acc)[NT]) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t] = mfma_f16(r.w[t][u], r.x[u], acc[t]);
    }
}

// The k steps of a GEMM are dealt out to its wavefronts `kbase` to each and one more to the first `kmore`; column group, k range (of the
// 16-row units' kernel) and row slices are the grid's y, x and z.  All worked out by the launcher: divisions ahead of the first load are time in
// which a short launch requests nothing.

// Where the keys and values of a decode step's row go (QKV): cache position of its sequence, and the sequence; t < 0: nowhere
struct RowSlot { int b, t; };
__device__ __forceinline__ RowSlot row_slot(const Epi& p, int m, int cur_len) {
    if (cur_len >= 0) return {m, cur_len};
    const int b = row_seq(p.st, min(m, p.M - 1), 1), pad = row_pad(p.st, b), len = seq_len(p.st, b);
    return {b, pad > 0 ? -1 : len};  // (a padding row appends nothing)
}
// epilogue4<MODE_QKV> for one row per sequence and the head dimensions of this path, 64 and 128
__device__ __forceinline__ void qkv_out(const Epi& p, int m, int n0, float v0, float v1, float v2, float v3, uint2 bb, RowSlot r) {
    if (m >= p.M) return;
    v0 += bf_lo(bb.x); v1 += bf_hi(bb.x); v2 += bf_lo(bb.y); v3 += bf_hi(bb.y);
    if (n0 < p.H) {
        *reinterpret_cast<float4*>(p.out + (size_t)m * p.H + n0) = make_float4(v0 * p.qscale, v1 * p.qscale, v2 * p.qscale, v3 * p.qscale);
    } else if (r.t >= 0) {
        const int which = n0 >= 2 * p.H, c = n0 - (which ? 2 * p.H : p.H), sh = p.d == 64 ? 6 : 7;
        half_t* dst = p.kv + kv_index(p.layer, which, r.b, c >> sh, r.t, p.max_batch, p.n_heads, p.max_seq, p.d) + (c & (p.d - 1));
        *reinterpret_cast<uint2*>(dst) = make_uint2(pack2(v0, v1), pack2(v2, v3));
    }
}

// (one k range: ksplit is 1 and blockIdx.x 0.  Without the argument and the term a step of 7 rows, hidden 4096, measured 1.3 us longer.)
template <int MODE, int NT, int U, int WAVES>
__global__ __launch_bounds__(WAVES * 64) void gemm_skinny_kernel(const u32x4* __restrict__ Wp,
                                                                 const u32x4* __restrict__ Xhi, int KB, int n_tiles,
                                                                 int ksplit, int kbase, int kmore, Epi p) {
    __shared__ float red[WAVES][NT][16][64];
    __shared__ float4 lnp[WAVES * 32];  // folded LayerNorm: the wavefronts' partial sums of the row statistics
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    int bx = blockIdx.y, mt = blockIdx.z;
    if (MODE == MODE_LMHEAD && gridDim.z > 1) {
        // Several 32-row slices each stream the whole matrix.  Workgroups go round the XCDs by index: the slices
        // of one group of tiles are placed on ONE XCD, next to each other in dispatch order, so that they run
        // side by side and all but the first of them find the weights in that XCD's L2 (the grid's x is padded
        // to a multiple of eight for this).
        const int lid = blockIdx.z * gridDim.y + blockIdx.y, span = 8 * gridDim.z;
        bx = (lid / span) * 8 + (lid % span) % 8;
        mt = (lid % span) / 8;
        if (bx >= (n_tiles + NT - 1) / NT) return;  // the whole workgroup
    }
    const int grp = bx, ks = blockIdx.x;
    const int part = ks * WAVES + wave, kb0 = part * kbase + min(part, kmore), kb1 = kb0 + kbase + (part < kmore);
    constexpr bool FOLDABLE = MODE == MODE_BIAS_RELU || MODE == MODE_QKV || MODE == MODE_LMHEAD;
    const u32x4* w[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t)  // tiles past the last one are computed from the last one, never stored
        w[t] = Wp + ((size_t)min(grp * NT + t, n_tiles - 1) * KB + kb0) * 64 + lane;
    const u32x4* xh = Xhi + ((size_t)mt * KB + kb0) * 64 + lane;
    // After the k loop the NT*4 (tile, row-quad) items of the workgroup are shared out over its
    // wavefronts: item = wave + i*WAVES -> tile item/4, rows 8*(item%4) + 4*(lane/32) + 0..3.
    constexpr int ITEMS = items_per_wave(NT * 4, WAVES);
    // What the epilogue needs (bias, the folded LayerNorm's vectors and statistics, the cache length) is
    // requested right behind the first round of weight loads: long before it is used, and without holding
    // up the start of the weight stream, which then waits for three pointers and three sizes only.
    uint2 bias_w[ITEMS];
    float4 c1w[ITEMS], c2w[ITEMS];
    LnLoads<WAVES> lnl;
    bool fold = false;
    int cur_len = 0;
    auto request_epilogue_operands = [&]() {
        fold = FOLDABLE && p.ln_stats != nullptr;
        if (fold) ln_issue<WAVES>(lnl, p, mt, wave, lane);
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            const int item = wave + i * WAVES, tile = grp * NT + (item >> 2);
            const int n0 = tile * 32 + 8 * (item & 3) + 4 * (lane >> 5);
            const bool live = item < NT * 4 && tile < n_tiles;
            bias_w[i] = live ? epilogue_bias<MODE>(p, n0) : make_uint2(0, 0);
            if (FOLDABLE) {
                c1w[i] = c2w[i] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (fold && live) {  // c1 and c2 are padded to whole tiles
                    c1w[i] = *reinterpret_cast<const float4*>(p.c1 + n0);
                    c2w[i] = *reinterpret_cast<const float4*>(p.c2 + n0);
                }
            }
        }
        cur_len = epilogue_len<MODE>(p);
    };
    // the folded LayerNorm's partial sums and, for the QKV epilogue, where the rows' keys and values go
    [[maybe_unused]] RowSlot slot{0, 0};
    auto use_statistics = [&]() {
        if (fold) ln_partial<WAVES>(lnl, p, mt, wave, lane, lnp);
        if constexpr (MODE == MODE_QKV) slot = row_slot(p, mt * 32 + (lane & 31), cur_len);
    };
    f32x16 acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = f32x16{};
    // LM head with sampling: the noise of this thread's own outputs (a Philox block and two logarithms each, 11 of a
    // 50272 x 5120 head's 97 us when formed at the end, 5 of 92 here) is formed between the load rounds, while the vector units are idle,
    // and waits in the part of LDS that takes the accumulators after the loop.
    constexpr int NOISE = MODE == MODE_LMHEAD ? ITEMS * 4 : 0;
    [[maybe_unused]] float* nz = &red[0][0][0][0] + threadIdx.x;
    [[maybe_unused]] uint32_t nz_step = 0, nz_seq = 0, nz_k0 = 0, nz_k1 = 0;
    [[maybe_unused]] bool gumbel = false;
    [[maybe_unused]] int nz_next = 0, nz_per_round = 0;
    int n = kb1 - kb0;
    auto noise_round = [&](int count) {
        if constexpr (MODE == MODE_LMHEAD) {
            for (int c = 0; c < count && nz_next < NOISE; ++c, ++nz_next) {
                const int item = wave + (nz_next >> 2) * WAVES;
                const int vid = (grp * NT + (item >> 2)) * 32 + 8 * (item & 3) + 4 * (lane >> 5) + (nz_next & 3);
                nz[nz_next * WAVES * 64] = gumbel_from_word(philox_word0((uint32_t)vid, nz_step, nz_seq, nz_k0, nz_k1));
            }
        }
    };
    auto noise_setup = [&](int blocks) {
        if constexpr (MODE == MODE_LMHEAD) {
            gumbel = p.st->mode == 1;
            nz_step = (uint32_t)p.st->step; nz_k0 = p.st->seed_lo; nz_k1 = p.st->seed_hi;
            nz_seq = (uint32_t)row_seq(p.st, min(mt * 32 + (lane & 31), p.M - 1), 1);  // the noise is keyed by the sequence, not by its row
            nz_per_round = gumbel ? (NOISE * U + blocks - 1) / max(blocks, 1) : 0;
        }
    };
    if (n >= U) {
        SkinnyRegs<NT, U> ra;
        skinny_load<NT, U>(ra, w, xh);
        n -= U;
        request_epilogue_operands();
        noise_setup(n);
        // the statistics are used once the second round is on its way as well (first trip peeled off
        // the loop: a test inside it cost the loop its schedule)
        if (n >= U) {
            SkinnyRegs<NT, U> rb;
            skinny_load<NT, U>(rb, w, xh);
            n -= U;
            use_statistics();
            skinny_mma<NT, U>(ra, acc);
            ra = rb;
        } else {
            use_statistics();
        }
        while (n >= U) {
            SkinnyRegs<NT, U> rb;
            skinny_load<NT, U>(rb, w, xh);
            n -= U;
            noise_round(nz_per_round);
            skinny_mma<NT, U>(ra, acc);
            ra = rb;
        }
        skinny_mma<NT, U>(ra, acc);
    } else {
        request_epilogue_operands();
        noise_setup(0);
        use_statistics();
    }
    for (; n > 0; --n) {
        SkinnyRegs<NT, 1> r1;
        skinny_load<NT, 1>(r1, w, xh);
        skinny_mma<NT, 1>(r1, acc);
    }
    [[maybe_unused]] float noise[ITEMS][4];
    if constexpr (MODE == MODE_LMHEAD) {
        if (gumbel) {
            noise_round(NOISE);
#pragma unroll
            for (int i = 0; i < ITEMS; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) noise[i][r] = nz[(i * 4 + r) * WAVES * 64];
            __syncthreads();
        }
    }
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) red[wave][t][r][lane] = acc[t][r];
    __syncthreads();
    const int m = mt * 32 + (lane & 31);
    float v[ITEMS][4];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const int item = wave + i * WAVES, t = item >> 2, q = item & 3;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            float sum = 0.f;
            if (item < NT * 4) {
#pragma unroll
                for (int ww = 0; ww < WAVES; ww += 2) sum += red[ww][t][q * 4 + r][lane] + red[ww + 1][t][q * 4 + r][lane];
            }
            v[i][r] = sum;
        }
    }
    if (fold) {  // W LN(x) = rstd * (W (gamma x) - mean * W gamma) + W beta
        const float2 mr = ln_finish<WAVES>(lnp, lane & 31, p);
        const float mean = mr.x, rstd = mr.y;
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            v[i][0] = rstd * (v[i][0] - mean * c1w[i].x) + c2w[i].x;
            v[i][1] = rstd * (v[i][1] - mean * c1w[i].y) + c2w[i].y;
            v[i][2] = rstd * (v[i][2] - mean * c1w[i].z) + c2w[i].z;
            v[i][3] = rstd * (v[i][3] - mean * c1w[i].w) + c2w[i].w;
        }
    }
    if constexpr (MODE != MODE_LMHEAD) {
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            const int item = wave + i * WAVES, tile = grp * NT + (item >> 2);
            if (item >= NT * 4 || tile >= n_tiles) continue;
            const int n0 = tile * 32 + 8 * (item & 3) + 4 * (lane >> 5);
            if constexpr (MODE == MODE_QKV) qkv_out(p, m, n0, v[i][0], v[i][1], v[i][2], v[i][3], bias_w[i], slot);
            else epilogue4<MODE>(p, m, n0, ks, v[i][0], v[i][1], v[i][2], v[i][3], bias_w[i], cur_len);
        }
    } else {
        // Soft-max and arg-max partials per (row, workgroup).  All of a thread's outputs belong to one row: reduced in its
        // registers, with the lane 32 away, then over the wavefronts.
        __shared__ float4 part[WAVES][32];
        __shared__ int part_idx[WAVES][32];
        const float temp = p.st->temperature;
        float mx = -INFINITY, best = -INFINITY, bestz = 0.f;
        int besti = 0x7FFFFFFF;
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            const int item = wave + i * WAVES, tile = grp * NT + (item >> 2);
            const int n0 = tile * 32 + 8 * (item & 3) + 4 * (lane >> 5);  // ascending in i
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                if (item >= NT * 4 || n0 + r >= p.N) { v[i][r] = -INFINITY; continue; }
                const float z = v[i][r];
                if (p.logits && m < p.M) p.logits[(size_t)m * p.N + n0 + r] = z;
                mx = fmaxf(mx, z);
                const float s = gumbel ? z / temp + noise[i][r] : z;
                if (s > best) { best = s; besti = n0 + r; bestz = z; }  // strict: the lowest id of equals
            }
        }
        auto take_better = [&](float s, int id, float z) {
            if (s > best || (s == best && id < besti)) { best = s; besti = id; bestz = z; }
        };
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        take_better(__shfl_xor(best, 32), __shfl_xor(besti, 32), __shfl_xor(bestz, 32));
        float sum = 0.f;
        const float base = mx > -INFINITY ? mx : 0.f;  // (nothing above -inf: ids past the vocabulary add 0, a NaN stays one)
#pragma unroll
        for (int i = 0; i < ITEMS; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) sum += expf(v[i][r] - base);
        sum += __shfl_xor(sum, 32);
        if (lane < 32) { part[wave][lane] = make_float4(mx, sum, best, bestz); part_idx[wave][lane] = besti; }
        __syncthreads();
        if (threadIdx.x < 32 && m < p.M) {
            float4 e[WAVES];
#pragma unroll
            for (int x = 0; x < WAVES; ++x) { e[x] = part[x][lane]; mx = fmaxf(mx, e[x].x); }
            sum = 0.f;
#pragma unroll
            for (int x = 0; x < WAVES; ++x) {
                sum += e[x].x > -INFINITY ? e[x].y * expf(e[x].x - mx) : e[x].y;
                take_better(e[x].z, part_idx[x][lane], e[x].w);
            }
            reinterpret_cast<float4*>(p.stats)[(size_t)m * p.n_tiles + grp] = make_float4(mx, sum, best, bestz);
            p.stats_idx[(size_t)m * p.n_tiles + grp] = besti;
        }
    }
}

// ----------------------------------------------------------------- skinny GEMM on 16-row units
//
// The kernel above hands out weight rows in units of 32, so a launch can only be balanced over
// the CUs when the number of 32-row tiles happens to divide well: 640 tiles (FC1 of the 13B
// shape) give 214 workgroups of three, and 42 CUs idle.  This variant hands out units of 16 rows
// -- 1280 of them are five per CU on all 256 -- using the 16x16x32 matrix instruction: its A
// operand is 16 rows x 32 k, i.e. one half (rows 0-15 or 16-31) of two consecutive 32x16 blocks,
// which a wavefront gathers from the unchanged tiled layout as four 256-byte runs (lane l: k-block
// l/32, k half (l/16)%2, row l%16).  The activations are gathered the same way, 16 of the 32 rows
// per instruction.  Lane l ends up with D[n = 16 g + 4 (l/16) + 0..3][m = 16 mh + l%16]: four
// consecutive outputs of one row, as the epilogues want them.  Everything else -- k split over the
// wavefronts, double-buffered loads, reduction through LDS, folded LayerNorm, last-arriving
// workgroup for the k-split modes -- is as above.

typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f32x4 mfma16_f16(const u32x4& a, const u32x4& b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}

// 16 E4M3 codes -> two half operand registers (exact: an E4M3 value has four significant bits and lies in
// 2^-9 .. 448).  Bytes 0-7 are the lane's eight k values of the first 32-wide k range, bytes 8-15 those of the second.
__device__ __forceinline__ uint32_t e4m3x2_to_f16x2(uint32_t word, bool upper) {
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    const f32x2 f = upper ? __builtin_amdgcn_cvt_pk_f32_fp8(word, true) : __builtin_amdgcn_cvt_pk_f32_fp8(word, false);
    return pack2(f.x, f.y);
}
__device__ __forceinline__ void e4m3x16_to_f16(const u32x4& w, u32x4& a0, u32x4& a1) {
    a0 = u32x4{e4m3x2_to_f16x2(w.x, false), e4m3x2_to_f16x2(w.x, true), e4m3x2_to_f16x2(w.y, false),
               e4m3x2_to_f16x2(w.y, true)};
    a1 = u32x4{e4m3x2_to_f16x2(w.z, false), e4m3x2_to_f16x2(w.z, true), e4m3x2_to_f16x2(w.w, false),
               e4m3x2_to_f16x2(w.w, true)};
}

// One loop step of a wavefront covers KU = 1 (bf16 weights) or 2 (8-bit weights: one 16-byte load holds
// two) k ranges of 32, U steps per round of loads.
// MH: 16-row halves of the activation rows a workgroup multiplies its weights by: 2 = one 32-row slice, 4 = two
// slices (decode steps of 33..64 sequences: the weights are still streamed once), 1 = the first half only (at
// most 16 sequences: the other half's loads and products would be thrown away); xstride = 16-byte units
// between two slices
template <int HT, int U, bool W8, int MH = 2>
struct HalfRegs {
    static constexpr int KU = W8 ? 2 : 1;
    u32x4 w[HT][U], xh[MH][U * KU];
};

// one step (of 32 k, or 64 with 8-bit weights) out of the U a round has room for
template <int HT, int U, bool W8, int MH>
__device__ __forceinline__ void half_load_step(HalfRegs<HT, U, W8, MH>& r, const u32x4* const (&w)[HT], const u32x4* xh, size_t xstride, int u) {
    constexpr int KU = W8 ? 2 : 1, WSTEP = W8 ? 64 : 128;
#pragma unroll
    for (int t = 0; t < HT; ++t) r.w[t][u] = __builtin_nontemporal_load(w[t] + u * WSTEP);
#pragma unroll
    for (int kp = 0; kp < KU; ++kp)
#pragma unroll
        for (int mh = 0; mh < MH; ++mh)
            r.xh[mh][u * KU + kp] = xh[(u * KU + kp) * 128 + (mh & 1) * 16 + (mh >> 1) * xstride];
}
// the first n < U steps only (n is the same for the whole wavefront)
template <int HT, int U, bool W8, int MH>
__device__ __forceinline__ void half_load_some(HalfRegs<HT, U, W8, MH>& r, const u32x4* const (&w)[HT], const u32x4* xh, size_t xstride, int n) {
#pragma unroll
    for (int u = 0; u < U - 1; ++u)
        if (u < n) half_load_step<HT, U, W8, MH>(r, w, xh, xstride, u);
}

template <int HT, int U, bool W8, int MH = 2>
__device__ __forceinline__ void half_load(HalfRegs<HT, U, W8, MH>& r, const u32x4* (&w)[HT], const u32x4*& xh,
                                          size_t xstride = 0) {
    constexpr int KU = W8 ? 2 : 1, WSTEP = W8 ? 64 : 128;
#pragma unroll
    for (int u = 0; u < U; ++u) half_load_step<HT, U, W8, MH>(r, w, xh, xstride, u);
#pragma unroll
    for (int t = 0; t < HT; ++t) w[t] += U * WSTEP;
    xh += U * KU * 128;
}

template <int HT, int U, bool W8, int MH>
__device__ __forceinline__ void half_mma_step(const HalfRegs<HT, U, W8, MH>& r, f32x4 (&acc)[HT][MH], int u) {
    if constexpr (W8) {
#pragma unroll
        for (int t = 0; t < HT; ++t) {
            u32x4 a[2];
            e4m3x16_to_f16(r.w[t][u], a[0], a[1]);
#pragma unroll
            for (int kp = 0; kp < 2; ++kp)
#pragma unroll
                for (int mh = 0; mh < MH; ++mh) acc[t][mh] = mfma16_f16(a[kp], r.xh[mh][u * 2 + kp], acc[t][mh]);
        }
    } else {
#pragma unroll
        for (int t = 0; t < HT; ++t)
#pragma unroll
            for (int mh = 0; mh < MH; ++mh) acc[t][mh] = mfma16_f16(r.w[t][u], r.xh[mh][u], acc[t][mh]);
    }
}
template <int HT, int U, bool W8, int MH>
__device__ __forceinline__ void half_mma(const HalfRegs<HT, U, W8, MH>& r, f32x4 (&acc)[HT][MH]) {
#pragma unroll
    for (int u = 0; u < U; ++u) half_mma_step<HT, U, W8, MH>(r, acc, u);
}
template <int HT, int U, bool W8, int MH>
__device__ __forceinline__ void half_mma_some(const HalfRegs<HT, U, W8, MH>& r, f32x4 (&acc)[HT][MH], int n) {
#pragma unroll
    for (int u = 0; u < U - 1; ++u)
        if (u < n) half_mma_step<HT, U, W8, MH>(r, acc, u);
}

// n_half = number of 16-row units of the weight matrix (N / 16); a workgroup owns HT of them.
// W8: the weights are E4M3 codes in units of [16 rows][64 k] -- lane l holds, for row l%16, the eight k
// values 8 (l/16) + 0..7 of the unit's first 32 k in bytes 0-7 and those of its second 32 k in bytes
// 8-15: one contiguous 1 KiB load per unit, two matrix-instruction operands after conversion.
template <int MODE, int HT, int U, int WAVES, bool W8, int MT = 1, int HALVES = 0>
__global__ __launch_bounds__(WAVES * 64) void gemm_half_kernel(const u32x4* __restrict__ Wp, const u32x4* __restrict__ Xhi,
                                                               int KB, int n_half, int ksplit, int kbase, int kmore, int m_rows,
                                                               Epi p) {
    // 16-row halves of the activation rows: both of every slice, or only the first HALVES of them when no more
    // are in use (at most 16 rows of one slice, at most 48 of two): the rest would be loaded and multiplied for nothing
    static_assert(HALVES == 0 || (HALVES < 2 * MT && HALVES > 2 * (MT - 1)), "HALVES ends inside the last slice");
    constexpr int MH = HALVES ? HALVES : 2 * MT;
    constexpr int NI = HT * MH;  // (unit, row half) items of a workgroup
    __shared__ f32x4 red[WAVES][NI][64];
    __shared__ float4 lnp[MT][WAVES * 32];  // folded LayerNorm: the wavefronts' partial sums of the row statistics
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int grp = blockIdx.y, ks = blockIdx.x;
    const int mt = blockIdx.z * MT;  // first 32-row slice
    const size_t xstride = (size_t)KB * 64;
    constexpr int KU = W8 ? 2 : 1;       // 32-wide k ranges per loop step
    const int KP = KB / (2 * KU);        // loop steps over the whole of k
    const int part = ks * WAVES + wave, kp0 = part * kbase + min(part, kmore), kp1 = kp0 + kbase + (part < kmore);
    constexpr bool FOLDABLE = MODE == MODE_BIAS_RELU || MODE == MODE_QKV;
    // this lane's 16 bytes inside a pair of 32x16 blocks: k-block lane/32, slot 32*(k half) + row
    const int in_pair = (lane >> 5) * 64 + 32 * ((lane >> 4) & 1) + (lane & 15);
    const u32x4* w[HT];
#pragma unroll
    for (int t = 0; t < HT; ++t) {  // units past the last one are computed from the last one, never stored
        const int g = min(grp * HT + t, n_half - 1);
        if (W8) w[t] = Wp + ((size_t)g * KP + kp0) * 64 + lane;
        else w[t] = Wp + ((size_t)(g >> 1) * KB + 2 * kp0) * 64 + in_pair + 16 * (g & 1);
    }
    // (of the first 16 rows only those in use: a load then touches half the lines where they are at most eight)
    const int x_in_pair = MH == 1 ? in_pair - (lane & 15) + min(lane & 15, m_rows - 1) : in_pair;
    const u32x4* xh = Xhi + ((size_t)mt * KB + 2 * KU * kp0) * 64 + x_in_pair;
    constexpr int ITEMS = items_per_wave(NI, WAVES);  // item = wave + i*WAVES -> unit item/MH, row half item%MH
    // epilogue operands: requested right behind the first round of weight loads (see gemm_skinny_kernel)
    uint2 bias_w[ITEMS];
    float4 c1w[ITEMS], c2w[ITEMS], wsc[ITEMS];
    constexpr int kLnRows = MH == 1 ? 16 : 32;
    LnLoads<WAVES> lnl[MT];
    bool fold = false;
    int cur_len = 0;
    // out-projection and FC2 without k ranges of several workgroups: what the tail adds to the sums
    constexpr bool EARLY = MODE == MODE_STORE_LN && ITEMS <= 2;
    [[maybe_unused]] TailOps<MODE == MODE_STORE_LN ? ITEMS : 1> tail_ops;
    auto request_epilogue_operands = [&]() {
        if constexpr (EARLY) {
            if (ksplit == 1) {
#pragma unroll
                for (int i = 0; i < ITEMS; ++i) {
                    const int item = wave + i * WAVES;
                    tail_request(tail_ops, p, i, mt * 32 + 16 * (item % MH) + (lane & 15), (grp * HT + item / MH) * 16 + 4 * (lane >> 4));
                }
            }
        }
        fold = FOLDABLE && p.ln_stats != nullptr;
        if (fold) {
#pragma unroll
            for (int s2 = 0; s2 < MT; ++s2) ln_issue<WAVES, kLnRows>(lnl[s2], p, mt + s2, wave, lane);
        }
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            const int item = wave + i * WAVES, g = grp * HT + item / MH;
            const int n0 = g * 16 + 4 * (lane >> 4);
            const bool live = item < NI && g < n_half;
            bias_w[i] = live ? epilogue_bias<MODE>(p, n0) : make_uint2(0, 0);
            wsc[i] = make_float4(1.f, 1.f, 1.f, 1.f);
            if (W8 && live) wsc[i] = *reinterpret_cast<const float4*>(p.wscale + n0);
            c1w[i] = c2w[i] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (FOLDABLE && fold && live) {
                c1w[i] = *reinterpret_cast<const float4*>(p.c1 + n0);
                c2w[i] = *reinterpret_cast<const float4*>(p.c2 + n0);
            }
        }
        cur_len = epilogue_len<MODE>(p);
    };
    f32x4 acc[HT][MH];
#pragma unroll
    for (int t = 0; t < HT; ++t)
#pragma unroll
        for (int mh = 0; mh < MH; ++mh) acc[t][mh] = f32x4{0.f, 0.f, 0.f, 0.f};
    // the folded LayerNorm's partial sums and, for the QKV epilogue, where the rows' keys and values go
    [[maybe_unused]] RowSlot slot[MODE == MODE_QKV ? ITEMS : 1];
    auto use_statistics = [&]() {
        if (fold) {
#pragma unroll
            for (int s2 = 0; s2 < MT; ++s2) ln_partial<WAVES, kLnRows>(lnl[s2], p, mt + s2, wave, lane, lnp[s2]);
        }
        if constexpr (MODE == MODE_QKV) {
#pragma unroll
            for (int i = 0; i < ITEMS; ++i) slot[i] = row_slot(p, mt * 32 + 16 * ((wave + i * WAVES) % MH) + (lane & 15), cur_len);
        }
    };
    int n = kp1 - kp0;
    // Where every workgroup's ranges begin at multiples of 32 KiB and more, workgroups that walk them in step ask the same memory
    // channels at the same time.  With ROTATE each starts its rounds at another one and wraps around: 8-bit 16384 x 4096
    // 19.0 -> 14.9 us, 20480 x 5120 21.9 -> 20.0, 4096 x 16384 (four ranges) 22.7 -> 18.6, 16-bit 4096 x 16384 (two) 28.9 -> 26.9.
    // The 16-bit GEMMs with one range lose by it (16384 x 4096 27.2 -> 29.8).  At other widths it is done for nothing: a layer's
    // decode GEMMs together, rotated less not, us: 8-bit hidden 4096 -7.5, 5120 -2.7, 2048 -0.2, 5184 -0.6, 4160 +0.2, 2112 +0.7, 1088
    // and 1024 +0.4; 16-bit 4096 -1.7, 5120 and 5184 +0.2, 4160 +0.4, 2112 +0.2, 1088 +0.4, 1024 +0.1.
    constexpr bool ROTATE = W8 || MODE == MODE_STORE_LN;
    constexpr int WSTEP = W8 ? 64 : 128;
    const int rounds = n / U;
    int round = 0;  // the round the pointers are at
    auto move = [&](int by) {
#pragma unroll
        for (int t = 0; t < HT; ++t) w[t] += by * U * WSTEP;
        xh += by * U * KU * 128;
    };
    if (ROTATE && rounds > 0) {
        round = (int)((unsigned)(grp * ksplit + ks) * 5u % (unsigned)rounds);
        move(round);
    }
    auto next_round = [&]() {
        if (ROTATE) {
            const bool wrap = ++round == rounds;
            move(wrap ? -rounds : 0);
            round = wrap ? 0 : round;
        }
    };
    if (n >= U) {
        HalfRegs<HT, U, W8, MH> ra;
        half_load<HT, U, W8, MH>(ra, w, xh, xstride);
        next_round();
        n -= U;
        request_epilogue_operands();
        // the statistics are used once the second round is on its way as well (first trip peeled off the loop)
        if (n >= U) {
            HalfRegs<HT, U, W8, MH> rb;
            half_load<HT, U, W8, MH>(rb, w, xh, xstride);
            next_round();
            n -= U;
            use_statistics();
            half_mma<HT, U, W8, MH>(ra, acc);
            ra = rb;
        } else {
            use_statistics();
        }
        while (n >= U) {
            HalfRegs<HT, U, W8, MH> rb;
            half_load<HT, U, W8, MH>(rb, w, xh, xstride);
            next_round();
            n -= U;
            half_mma<HT, U, W8, MH>(ra, acc);
            ra = rb;
        }
        if (ROTATE) move(rounds - round);
        HalfRegs<HT, U, W8, MH> rest;  // the steps behind the last whole round, on their way before its products
        half_load_some<HT, U, W8, MH>(rest, w, xh, xstride, n);
        half_mma<HT, U, W8, MH>(ra, acc);
        half_mma_some<HT, U, W8, MH>(rest, acc, n);
    } else {
        HalfRegs<HT, U, W8, MH> rest;
        half_load_some<HT, U, W8, MH>(rest, w, xh, xstride, n);
        request_epilogue_operands();
        use_statistics();
        half_mma_some<HT, U, W8, MH>(rest, acc, n);
    }
#pragma unroll
    for (int t = 0; t < HT; ++t)
#pragma unroll
        for (int mh = 0; mh < MH; ++mh) red[wave][t * MH + mh][lane] = acc[t][mh];
    __syncthreads();
    float v[ITEMS][4];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const int item = wave + i * WAVES;
        f32x4 sum = {0.f, 0.f, 0.f, 0.f};
        if (item < NI) {
            f32x4 e[WAVES];
#pragma unroll
            for (int ww = 0; ww < WAVES; ++ww) e[ww] = red[ww][item][lane];
#pragma unroll
            for (int ww = 0; ww < WAVES; ww += 2) sum += e[ww] + e[ww + 1];
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) v[i][r] = sum[r];
    }
    if (W8) {  // sums over codes -> sums over weights: exact, the scales are powers of two
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            v[i][0] *= wsc[i].x; v[i][1] *= wsc[i].y; v[i][2] *= wsc[i].z; v[i][3] *= wsc[i].w;
        }
    }
    if (fold) {  // W LN(x) = rstd * (W (gamma x) - mean * W gamma) + W beta; a lane's items sit in two rows
        // (selected, not indexed: an array indexed at run time would live in LDS, whose addressing
        // reads the dispatch packet -- microseconds, here in the tail of the kernel)
        const float2 mr0 = ln_finish<WAVES>(lnp[0], lane & 15, p), mr1 = MH == 1 ? mr0 : ln_finish<WAVES>(lnp[0], 16 + (lane & 15), p);
        float2 mr2 = mr0, mr3 = mr1;
        if (MT == 2) {
            mr2 = ln_finish<WAVES>(lnp[MT - 1], lane & 15, p);
            mr3 = ln_finish<WAVES>(lnp[MT - 1], 16 + (lane & 15), p);
        }
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            const int rh = (wave + i * WAVES) % MH;
            const bool odd = rh & 1, second = rh >= 2;
            const float mean = second ? (odd ? mr3.x : mr2.x) : (odd ? mr1.x : mr0.x);
            const float rstd = second ? (odd ? mr3.y : mr2.y) : (odd ? mr1.y : mr0.y);
            v[i][0] = rstd * (v[i][0] - mean * c1w[i].x) + c2w[i].x;
            v[i][1] = rstd * (v[i][1] - mean * c1w[i].y) + c2w[i].y;
            v[i][2] = rstd * (v[i][2] - mean * c1w[i].z) + c2w[i].z;
            v[i][3] = rstd * (v[i][3] - mean * c1w[i].w) + c2w[i].w;
        }
    }
    if constexpr (MODE == MODE_STORE_LN) {
        int mrow[ITEMS], n0[ITEMS], rslot[ITEMS];
        bool live[ITEMS];
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            const int item = wave + i * WAVES, g = grp * HT + item / MH;
            mrow[i] = mt * 32 + 16 * (item % MH) + (lane & 15);
            n0[i] = g * 16 + 4 * (lane >> 4);
            live[i] = item < NI && g < n_half && mrow[i] < p.M;
            rslot[i] = item % MH;
        }
        store_ln_tail<ITEMS, WAVES, MT, NI <= WAVES && HT == 1>(p, ksplit, ks, grp, (n_half + HT - 1) / HT, mt,
                                                                16.f * (float)min(HT, n_half - grp * HT), v, mrow, n0, live, rslot,
                                                                    tail_ops, EARLY && ksplit == 1);
        return;
    }
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const int item = wave + i * WAVES, g = grp * HT + item / MH;
        if (item >= NI || g >= n_half) continue;
        const int m = mt * 32 + 16 * (item % MH) + (lane & 15), n0 = g * 16 + 4 * (lane >> 4);
        if constexpr (MODE == MODE_QKV) qkv_out(p, m, n0, v[i][0], v[i][1], v[i][2], v[i][3], bias_w[i], slot[i]);
        else epilogue4<MODE>(p, m, n0, ks, v[i][0], v[i][1], v[i][2], v[i][3], bias_w[i], cur_len);
    }
}

// grid: the launch's (k range, column group, row slices); items, waves: of the kernel variant chosen.  True if the launch is to be left out.
inline bool dry_run(const dim3& grid, int ksplit, int items, int waves, int units, int steps) {
    if (bf16_ahead* a = g_dry_ahead) {
        a->wgs = grid.x * grid.y;
        a->ks = ksplit; a->units = units; a->waves = waves;
        a->kbase = steps / (ksplit * waves); a->kmore = steps % (ksplit * waves);
        return true;
    }
    if (!g_dry) return false;
    g_dry->cells = grid.y * grid.z;
    g_dry->stat_groups = grid.y;
    g_dry->ksplit = ksplit;
    g_dry->scratch_floats = ksplit > 1 ? (size_t)g_dry->cells * ksplit * tail_floats_per_split(items, waves) : 0;
    return true;
}

template <int MODE, int HT, bool W8>
void launch_half_ht(hipStream_t s, const void* Wp, const void* Xhi, int KB, int n_half, int m_tiles,
                    int ksplit, const Epi& p) {
    // loads per wavefront and round: (HT + 4) U 16-byte loads with bf16 weights, (HT + 8) U with 8-bit ones
    // (with the activations' second term gone there are registers for deeper rounds at four to six units; three or
    // four blocks per round measured 1-3 % slower than two on the 13B shapes)
    constexpr int U = W8 ? (HT <= 3 ? 2 : 1) : (HT <= 3 ? 4 : 2);
    constexpr int KU = W8 ? 2 : 1;
    const int steps = KB / (2 * KU);
    const int parts4 = ksplit * 4, parts8 = ksplit * 8;
    dim3 grid(ksplit, (n_half + HT - 1) / HT, m_tiles);
    if constexpr (HT <= 8) {  // (the accumulators of more units than that do not fit in LDS for the reduction)
        if (m_tiles == 2) {  // both 32-row slices in one workgroup: the weights are streamed once
            constexpr int U2 = !W8 && HT <= 6 ? 2 : 1;
            constexpr size_t kWant2 = 84 * 1024;
            grid.z = 1;
            if (dry_run(grid, ksplit, items_per_wave(HT * (p.M <= 48 ? 3 : 4), 4), 4, HT, steps)) return;
            if (p.M <= 48) {  // the last 16 of the 64 rows are not in use
                constexpr size_t kStatic = (size_t)4 * HT * 3 * 4 * 64 * sizeof(float);
                const size_t pad = kStatic >= kWant2 ? 0 : kWant2 - kStatic;
                gemm_half_kernel<MODE, HT, U2, 4, W8, 2, 3><<<grid, 256, pad, s>>>(
                    (const u32x4*)Wp, (const u32x4*)Xhi, KB, n_half, ksplit, steps / parts4, steps % parts4, p.M, p);
                return;
            }
            constexpr size_t kStatic = (size_t)4 * HT * 4 * 4 * 64 * sizeof(float);
            const size_t pad = kStatic >= kWant2 ? 0 : kWant2 - kStatic;
            gemm_half_kernel<MODE, HT, U2, 4, W8, 2><<<grid, 256, pad, s>>>((const u32x4*)Wp, (const u32x4*)Xhi,
                                                                               KB, n_half, ksplit, steps / parts4, steps % parts4, p.M, p);
            return;
        }
    }
    // eight wavefronts have 256 registers each: three units with four rounds of operands twice over do not fit
    constexpr int U8 = (!W8 && HT == 3) ? 2 : U;
    // (five and six units of 8-bit weights: four wavefronts are one per SIMD, whose conversions nothing covers.  Up to 16 rows eight
    // are 5 to 15 % faster, 20480 x 5120 20.3 -> 18.6 us; with 32 only where all sums stay in the workgroup, 21.9 -> 21.3 against
    // 24.0 -> 24.5 for 5120 x 20480 in four ranges.)
    constexpr int kEight = W8 ? 6 : 4;
    const int eight_most = W8 && (p.M <= 16 || (HT == 5 && MODE != MODE_STORE_LN)) ? kEight : 4;
    const bool eight = HT <= eight_most && (KB / (2 * KU)) / (ksplit * 8) >= 2 * U8;  // short chains per wavefront, as above
    constexpr size_t kWant = 84 * 1024;                                      // one workgroup per CU
    if (m_tiles == 1 && p.M <= 16) {  // the second half of the 32 activation rows is not in use: leave it out
        if (dry_run(grid, ksplit, items_per_wave(HT, eight ? 8 : 4), eight ? 8 : 4, HT, steps)) return;
        if (eight) {
            constexpr size_t kStatic = (size_t)8 * HT * 4 * 64 * sizeof(float);
            const size_t pad = kStatic >= kWant ? 0 : kWant - kStatic;
            gemm_half_kernel<MODE, HT <= kEight ? HT : 2, U8, 8, W8, 1, 1><<<grid, 512, pad, s>>>(
                (const u32x4*)Wp, (const u32x4*)Xhi, KB, n_half, ksplit, steps / parts8, steps % parts8, p.M, p);
        } else {
            constexpr size_t kStatic = (size_t)4 * HT * 4 * 64 * sizeof(float);
            const size_t pad = kStatic >= kWant ? 0 : kWant - kStatic;
            gemm_half_kernel<MODE, HT, U, 4, W8, 1, 1><<<grid, 256, pad, s>>>(
                (const u32x4*)Wp, (const u32x4*)Xhi, KB, n_half, ksplit, steps / parts4, steps % parts4, p.M, p);
        }
        return;
    }
    if (dry_run(grid, ksplit, items_per_wave(HT * 2, eight ? 8 : 4), eight ? 8 : 4, HT, steps)) return;
    if (eight) {
        constexpr size_t kStatic = (size_t)8 * HT * 2 * 4 * 64 * sizeof(float);
        const size_t pad = kStatic >= kWant ? 0 : kWant - kStatic;
        gemm_half_kernel<MODE, HT <= kEight ? HT : 2, U8, 8, W8><<<grid, 512, pad, s>>>(
            (const u32x4*)Wp, (const u32x4*)Xhi, KB, n_half, ksplit, steps / parts8, steps % parts8, p.M, p);
    } else {
        constexpr size_t kStatic = (size_t)4 * HT * 2 * 4 * 64 * sizeof(float);
        const size_t pad = kStatic >= kWant ? 0 : kWant - kStatic;
        gemm_half_kernel<MODE, HT, U, 4, W8><<<grid, 256, pad, s>>>((const u32x4*)Wp, (const u32x4*)Xhi,
                                                                    KB, n_half, ksplit, steps / parts4, steps % parts4, p.M, p);
    }
}

constexpr int kHalfMax = 10;  // 16-row units per workgroup the half-tile kernel is built for at most
constexpr int kHalfMax2 = 8;                // ... with two 32-row activation slices per workgroup

template <int MODE, bool W8>
void launch_half(hipStream_t s, const void* Wp, const void* Xhi, int KB, int n_half, int m_tiles, int ht,
                 int ksplit, const Epi& p) {
    switch (ht) {
        case 1: launch_half_ht<MODE, 1, W8>(s, Wp, Xhi, KB, n_half, m_tiles, ksplit, p); break;
        case 2: launch_half_ht<MODE, 2, W8>(s, Wp, Xhi, KB, n_half, m_tiles, ksplit, p); break;
        case 3: launch_half_ht<MODE, 3, W8>(s, Wp, Xhi, KB, n_half, m_tiles, ksplit, p); break;
        case 4: launch_half_ht<MODE, 4, W8>(s, Wp, Xhi, KB, n_half, m_tiles, ksplit, p); break;
        case 5: launch_half_ht<MODE, 5, W8>(s, Wp, Xhi, KB, n_half, m_tiles, ksplit, p); break;
        case 6: launch_half_ht<MODE, 6, W8>(s, Wp, Xhi, KB, n_half, m_tiles, ksplit, p); break;
        case 7: launch_half_ht<MODE, 7, W8>(s, Wp, Xhi, KB, n_half, m_tiles, ksplit, p); break;
        case 8: launch_half_ht<MODE, 8, W8>(s, Wp, Xhi, KB, n_half, m_tiles, ksplit, p); break;
        case 9: launch_half_ht<MODE, 9, W8>(s, Wp, Xhi, KB, n_half, m_tiles, ksplit, p); break;
        default: launch_half_ht<MODE, 10, W8>(s, Wp, Xhi, KB, n_half, m_tiles, ksplit, p); break;
    }
}

}  // namespace
