// bf16 path: the LDS-tiled MFMA GEMM of prompt rows, scoring passes and wide decode steps.
#include "bf16_common.h"

using namespace he_bf16;

namespace {

// A wavefront's share of the scoring head, NA column blocks x MJ row blocks from row m0 and column n0 on.  The logits
// never leave the registers: per row, the soft-max partials of the wavefront's 32 NA vocabulary entries (slice `part` of
// the row) and, if the row's next token is among them, its logit.  (The next token is looked for only where one of the rows has it.  The
// hardware's 2^x of an argument multiplied by log2 e, 2976 us instead of 3161 for 16384 x 50272 x 2048, rounds the argument first: terms six
// below the largest are off by up to five ulps, which many additions in one direction made 5e-6 of a sum.)
template <int NA, int MJ, bool BIG = false>
__device__ __forceinline__ void score_tile(const Epi& p, f32x16 (&acc)[NA][MJ], int m0, int n0, int part, int lane) {
    const int nl = n0 + 4 * (lane >> 5);
    const bool whole = n0 + 32 * NA <= p.N;  // (uniform) no entry past the vocabulary
#pragma unroll
    for (int j = 0; j < MJ; ++j) {
        const int m = m0 + j * 32 + (lane & 31);
        int tgt = -1;
        if (m < p.M && m % p.S != p.S - 1) {
            tgt = p.ids[m + 1];
            tgt = tgt < 0 ? 0 : (tgt >= p.N ? p.N - 1 : tgt);  // clamped like the embedding's ids
        }
        if constexpr (BIG) {  // (see store_tile)
#pragma unroll
            for (int i = 0; i < NA; ++i) asm volatile("" : "+a"(acc[i][j]));
        }
        // the next token's logit: few wavefronts hold one of their rows'
        if (__any(tgt >= n0 && tgt < n0 + 32 * NA)) {
            const int at = tgt - nl;  // (this lane's entries: 32 i + 8 (r / 4) + r % 4)
            float hit = 0.f;
#pragma unroll
            for (int i = 0; i < NA; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r) hit = at == i * 32 + 8 * (r >> 2) + (r & 3) ? acc[i][j][r] : hit;
            if (at >= 0 && at < 32 * NA && !(at & 4)) p.sc_tgt[m] = hit;
        }
        float mx = -INFINITY, sum = 0.f;
        auto reduce = [&](auto logit) {
#pragma unroll
            for (int i = 0; i < NA; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r) mx = fmaxf(mx, logit(i, r));
            mx = fmaxf(mx, __shfl_xor(mx, 32));
            if (mx > -INFINITY) {
#pragma unroll
                for (int i = 0; i < NA; ++i)
#pragma unroll
                    for (int r = 0; r < 16; ++r) sum += expf(logit(i, r) - mx);
            }
        };
        if (whole) reduce([&](int i, int r) { return acc[i][j][r]; });
        else reduce([&](int i, int r) { return nl + i * 32 + 8 * (r >> 2) + (r & 3) < p.N ? acc[i][j][r] : -INFINITY; });
        sum += __shfl_xor(sum, 32);
        if (lane < 32 && m < p.M) p.sc_stats[(size_t)m * p.sc_parts + part] = make_float2(mx, sum);
        __builtin_amdgcn_sched_barrier(0);  // (one row block's values in registers at a time)
    }
}

// A wavefront's share of the LM head of a decode step of more than 32 rows, 4 column blocks x MJ row blocks from row m0 and
// column n0 on: per row, soft-max partials of its 128 logits, the best score (with the sampler's noise) and its id, and
// the logits themselves where the caller wants them.  fold: mean and 1/sqrt(var + eps) of the lane's row of each block;
// zl: 64 x 64 floats of LDS of the wavefront's own.
template <int MJ>
__device__ __forceinline__ void lm_head_tile(const Epi& p, const f32x16 (&acc)[4][MJ], const float2 (&fold)[MJ], int m0, int n0, int part,
                                             int lane, float* zl) {
    const int hh = lane >> 5;
    const int mode = p.st->mode, step = p.st->step;
    const float temp = p.st->temperature;
    const uint32_t k0 = p.st->seed_lo, k1 = p.st->seed_hi;
    const bool folded = MJ == 1 && p.ln_stats != nullptr;  // (more rows to a tile: never folded)
#pragma unroll
    for (int j = 0; j < MJ; ++j) {
        if (m0 + j * 32 < p.M) {  // (wave-uniform)
            const int m = m0 + j * 32 + (lane & 31);
            const uint32_t seq = (uint32_t)row_seq(p.st, min(m, p.M - 1), 1);  // the noise is keyed by the sequence, not by its row
            float mx = -INFINITY;
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int nq = n0 + i * 32 + 8 * q + 4 * hh;
                    float4 c1 = make_float4(0.f, 0.f, 0.f, 0.f), c2 = c1;
                    if (folded && nq < p.N) {  // (c1 and c2 are padded to whole 32s)
                        c1 = *reinterpret_cast<const float4*>(p.c1 + nq);
                        c2 = *reinterpret_cast<const float4*>(p.c2 + nq);
                    }
                    const float c1v[4] = {c1.x, c1.y, c1.z, c1.w}, c2v[4] = {c2.x, c2.y, c2.z, c2.w};
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        float v = acc[i][j][4 * q + e];
                        if (folded) v = fold[j].y * (v - fold[j].x * c1v[e]) + c2v[e];
                        if (nq + e >= p.N) v = -INFINITY;
                        else if (p.logits && m < p.M) p.logits[(size_t)m * p.N + nq + e] = v;
                        zl[(i * 16 + 4 * q + e) * 64 + lane] = v;  // (read back by this lane only)
                        mx = fmaxf(mx, v);
                    }
                }
            mx = fmaxf(mx, __shfl_xor(mx, 32));
            // the sampler's noise is some forty multiplications per logit: a loop of its own, short enough to stay in the
            // instruction cache (written out 64 times over it is not)
            float best = -INFINITY, bestz = 0.f, sum = 0.f;
            int besti = 0x7FFFFFFF;
            const float base = mx > -INFINITY ? mx : 0.f;  // (nothing above -inf: ids past the vocabulary add 0, a NaN stays one)
#pragma unroll 4
            for (int x = 0; x < 64; ++x) {
                const float v = zl[x * 64 + lane];
                const int n = n0 + (x >> 4) * 32 + 8 * ((x >> 2) & 3) + 4 * hh + (x & 3);
                sum += expf(v - base);
                float s = v;
                if (mode == 1) s = v / temp + gumbel_from_word(philox_word0((uint32_t)n, (uint32_t)step, seq, k0, k1));
                if (n < p.N && s > best) { best = s; besti = n; bestz = v; }  // ascending ids: strict > keeps the lowest
            }
            sum += __shfl_xor(sum, 32);
            const float os = __shfl_xor(best, 32), oz = __shfl_xor(bestz, 32);
            const int oi = __shfl_xor(besti, 32);
            if (os > best || (os == best && oi < besti)) { best = os; besti = oi; bestz = oz; }
            if (hh == 0 && m < p.M) {
                reinterpret_cast<float4*>(p.stats)[(size_t)m * p.n_tiles + part] = make_float4(mx, sum, best, bestz);
                p.stats_idx[(size_t)m * p.n_tiles + part] = besti;
            }
        }
    }
}

// ----------------------------------------------------------------- 256 x 128 tiles, two workgroups per CU (scoring head)
//
// 256 (n) x 128 (m) output tile per workgroup, four wavefronts in a 2x2 grid of
// 128x64 sub-tiles (4x2 MFMA tiles each: 6 LDS operand reads feed 8 MFMAs per
// k-block).  Operands arrive as 1 KiB blocks whose layout is the lane order, so
// they are moved global -> LDS directly (global_load_lds, 16 bytes per lane, no
// staging registers) into a ring of five stages of one k-block (80 KiB); one barrier per stage.
// At most 256 registers, so that TWO workgroups share a CU: while one of them sits at its barrier, waits
// for operands or reduces its logits, the other one's MFMAs keep the matrix cores busy.  Most passes take the big tile's kernel all the
// same, which loads a third less per product (score_tile, the planner, has both sides); this one is for the row and column counts that
// leave that kernel's last round nearly empty.
constexpr int TN = 256;
constexpr int TNB = TN / 32;  // 32-row operand blocks on the n side
constexpr int TMB = 4;        // ... and on the m side
constexpr int NSTG = 5;       // ring depth

__global__ __launch_bounds__(256, 2) void gemm_score_kernel(const u32x4* __restrict__ Wp, const u32x4* __restrict__ Xhi, int KB, int NT32,
                                                            int MT32, int tiles_n, int tiles_m, Epi p) {
    __shared__ u32x4 ring[NSTG][TNB + TMB][64];  // ring[stage][block][lane]: W row-tiles, then X row-tiles
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    // XCD-aware order: consecutive workgroups land on different XCDs, so give each XCD a
    // contiguous run of tiles; within a run, tiles sharing an m panel are neighbours.
    const int nitem = tiles_n * tiles_m, per_xcd = (nitem + 7) / 8;
    const int lin = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
    if (lin >= nitem) return;
    constexpr int GROUP = 8;  // m-tiles per super-row: the 8 x 8 tiles an XCD works on at once use the same few W and X panels
    const int gsize = GROUP * tiles_n;
    const int g = lin / gsize, first_m = g * GROUP;
    const int gm = min(GROUP, tiles_m - first_m);
    const int tm = first_m + (lin % gsize) % gm, tn = (lin % gsize) / gm;
    const int wn = wave & 1, wm = wave >> 1;  // this wavefront's 128 (n) x 64 (m) sub-tile
    f32x16 acc[4][2];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x16{};
    // this wavefront brings in W row-tiles 2w, 2w+1 and X row-tile w per k-block
    const u32x4* wsrc[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) wsrc[i] = Wp + (size_t)min(tn * TNB + wave * 2 + i, NT32 - 1) * KB * 64 + lane;
    const u32x4* hsrc = Xhi + (size_t)min(tm * TMB + wave, MT32 - 1) * KB * 64 + lane;
    const int nstage = KB;  // (even: K is a multiple of 32)
    auto issue = [&](int st) {
        u32x4 (*slot)[64] = ring[st % NSTG];
        const size_t off = (size_t)st * 64;
        load_block_to_lds(wsrc[0] + off, &slot[wave * 2 + 0][0]);
        load_block_to_lds(wsrc[1] + off, &slot[wave * 2 + 1][0]);
        load_block_to_lds(hsrc + off, &slot[TNB + wave][0]);
    };
    constexpr int kLoadsPerStage = 3;  // per wavefront
    // operand registers of one k-block: 4 weight blocks, 2 activation tiles
    struct Ops { u32x4 a[4], b[2]; };
    auto read_ops = [&](Ops& o, int st) {
        u32x4 (*slot)[64] = ring[st % NSTG];
#pragma unroll
        for (int i = 0; i < 4; ++i) o.a[i] = slot[wn * 4 + i][lane];
#pragma unroll
        for (int i = 0; i < 2; ++i) o.b[i] = slot[TNB + wm * 2 + i][lane];
    };
    auto mma_ops = [&](const Ops& o) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
#pragma unroll
            for (int jj = 0; jj < 2; ++jj) acc[i][jj] = mfma_f16(o.a[i], o.b[jj], acc[i][jj]);
        }
    };
#pragma unroll
    for (int st = 0; st < NSTG - 1; ++st)
        if (st < nstage) issue(st);
    // Two operand register sets, used in turn: even stages from A, odd ones from B.  No set is ever copied into the
    // other: a copy would have to wait for the LDS reads it copies, in the middle of the MFMAs.  A stage's slot is
    // refilled behind the barrier that every wavefront passes only after its MFMAs of that stage.  In the steady
    // state a stage is opened while the NSTG-3 stages issued after it are still in flight, and the slot just finished
    // with is refilled.
    Ops opa, opb;
    constexpr int kAhead = (NSTG - 3) * kLoadsPerStage;
    int s = 0;
    if (nstage > NSTG) {  // then the prologue has issued NSTG-1 stages
        wait_vmcnt<(NSTG - 2) * kLoadsPerStage>();
        __syncthreads();
        read_ops(opa, 0);
        for (; s + NSTG < nstage; s += 2) {
            wait_vmcnt<kAhead>();
            __syncthreads();
            issue(s + NSTG - 1);
            read_ops(opb, s + 1);
            mma_ops(opa);
            wait_vmcnt<kAhead>();
            __syncthreads();
            issue(s + NSTG);
            read_ops(opa, s + 2);
            mma_ops(opb);
        }
    }
    // the last stages: issue the one that may still be missing (into the slot of stage s-1, which
    // every wavefront has left once it is past the barrier), then one wait covers them all
    __syncthreads();
    if (s + NSTG - 1 < nstage) issue(s + NSTG - 1);
    wait_vmcnt<0>();
    __syncthreads();
    if (s == 0) read_ops(opa, 0);
    for (; s < nstage; s += 2) {
        read_ops(opb, s + 1);
        mma_ops(opa);
        if (s + 2 < nstage) read_ops(opa, s + 2);
        mma_ops(opb);
    }
    score_tile<4, 2>(p, acc, (tm * TMB + wm * 2) * 32, tn * TN + wn * 128, tn * 2 + wn, lane);
}

// ----------------------------------------------------------------- 256 x 256 tiles (prompt and scoring passes)
//
// With one half term per activation a 256 x 128 tile no longer keeps the matrix cores busy: it pulls
// 12 KiB of operands out of L2 for every 32 matrix instructions, and at eight rounds of 512 tiles on 256 CUs that
// is 10 TB/s -- what the L2s deliver.  This kernel takes 16 KiB for 64: a 256 x 256 tile per workgroup, four
// wavefronts with a 128 x 128 sub-tile each (16 accumulator tiles: the whole accumulator file, so one workgroup
// per CU).  Nothing else runs on a CU while its four wavefronts sit at a barrier or issue loads, so the schedule is
// laid out by hand: a stage is two k-blocks (32 KiB, ring of four); LDS reads and global -> LDS copies are dealt out
// between pairs of matrix instructions, every read at least eight matrix instructions ahead of the wait that
// covers it.  Measured on the 8160 x 20480 x 5120 product (loop only): matrix instructions alone on random operands
// 1015 us (the clock drops under data toggling), + LDS reads 1082 us, + copies 1280 us = 1.34 PFLOP/s (1310 us with
// one read per pair all through a half: the compiler's wait at the top of a half is for all reads, the newest
// included); with reads and copies issued in bursts after the barrier, as a compiler left to itself schedules
// them, 1690 us.  Copies issued by odd and even wavefronts behind different pairs: no change.
// A lane of a 32x32 accumulator tile holds columns 8q + 4 (lane / 32) + 0..3 of row lane % 32: four halves of an
// eight-column slot, the other four in the lane 32 away.  For a pair of slots (q even, q odd) packed as x, y: the
// lower lane gets the whole even slot, the upper lane the whole odd one -- 16-byte stores instead of 8-byte ones
// (the epilogue is bound by the number of store instructions).
__device__ __forceinline__ u32x4 join_halves(uint2 x, uint2 y) {
    const auto a = __builtin_amdgcn_permlane32_swap(x.x, y.x, false, false);  // [x low lanes | y low lanes], [x high | y high]
    const auto b = __builtin_amdgcn_permlane32_swap(x.y, y.y, false, false);
    return u32x4{a[0], b[0], a[1], b[1]};
}

// The big kernel's result stores, 16 bytes per lane.  (Nontemporal stores were tried: no gain for the half blocks,
// 6 % slower for the float rows.)
typedef float f32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void store16(void* dst, u32x4 v) { *reinterpret_cast<u32x4*>(dst) = v; }
__device__ __forceinline__ void store16(void* dst, float a, float b, float c, float d) {
    *reinterpret_cast<f32x4*>(dst) = f32x4{a, b, c, d};
}

// A wavefront's results, NA column blocks x MJ row blocks of 32 x 32 accumulators from row m0 and column n0 on.
// BIG: the big kernel's accumulators, which fill the accumulation registers (a fifth column block the vector registers) and are to
// stay there until a block of them is turned into results: copied to vector registers all at once they push the next tile's addresses
// into scratch memory.
template <int MODE, int NA, int MJ, bool BIG = false>
__device__ __forceinline__ void store_tile(const Epi& p, const u32x4* __restrict__ bias8, f32x16 (&acc)[NA][MJ], int m0,
                                           int n0, int ks, int cur_len, int lane) {
    // Epilogue.  The CU runs nothing else meanwhile, so it is written out per mode with everything that depends on
    // the row alone (sequence, cache position, row base address) computed once per 32-row block and everything
    // that depends on the column alone wave-uniform (the generic per-quad form recomputes both, with run-time
    // integer divisions, for each of a lane's 64 quads: 22 us per tile for FC1, 44 us for QKV, against 130 us of
    // matrix instructions).  N is a multiple of 32 here, so a 32-column block is inside or outside as a whole.
    // Columns outside, rows inside: a column block's bias is fetched and unpacked once.
    const int hh = lane >> 5;
    size_t row[MJ];                   // MODE_STORE: float index of (m, 4 hh); BIAS_RELU: 16-byte slot of (m, k half hh) in
                                      // the first block of its row of blocks; QKV: float index into q
    [[maybe_unused]] size_t kvrow[MJ];  // QKV: half index of (sequence, head 0, position, 0) inside one (layer, k|v) plane
    bool live[MJ];
    [[maybe_unused]] bool append[MJ];   // QKV: the row is a token (not padding): its key and value go into the cache
#pragma unroll
    for (int j = 0; j < MJ; ++j) {
        const int m = m0 + j * 32 + (lane & 31);
        live[j] = m < p.M;
        if (MODE == MODE_STORE) {
            row[j] = (size_t)ks * p.out_split + (size_t)m * p.N + 4 * hh;
        } else if (MODE == MODE_BIAS_RELU) {
            row[j] = (size_t)(m >> 5) * (p.N >> 4) * 64 + 32 * hh + (m & 31);
        } else {
            row[j] = (size_t)m * p.H + 4 * hh;
            append[j] = false;
            kvrow[j] = 0;
            if (live[j]) {
                const int b = row_seq(p.st, m, p.S), r = m % p.S;
                int t = cur_len + r;
                append[j] = true;
                if (cur_len < 0) {  // sequences of different lengths; padding rows append nothing
                    const int tr = r - row_pad(p.st, b);
                    append[j] = tr >= 0;
                    t = seq_len(p.st, b) + tr;
                }
                kvrow[j] = ((size_t)b * p.n_heads * p.max_seq + t) * p.d;
            }
        }
    }
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        const int n32 = n0 + i * 32;  // wave-uniform
        if (n32 >= p.N) break;
        float bv[MODE == MODE_STORE ? 1 : 4][4];
        if (MODE != MODE_STORE) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const u32x4 b8 = bias8[(n32 >> 3) + q];  // wave-uniform address: a scalar load
                const uint2 bb = hh ? make_uint2(b8.z, b8.w) : make_uint2(b8.x, b8.y);
                bv[q][0] = bf_lo(bb.x); bv[q][1] = bf_hi(bb.x); bv[q][2] = bf_lo(bb.y); bv[q][3] = bf_hi(bb.y);
            }
        }
        const int part = MODE != MODE_QKV ? 0 : (n32 >= 2 * p.H ? 2 : (n32 >= p.H ? 1 : 0));  // query, key or value columns (uniform)
        half_t* kvcol = nullptr;
        if (part) {
            const int c32 = n32 - part * p.H, head = c32 / p.d;
            kvcol = p.kv + (((size_t)(p.layer * 2 + (part - 1)) * p.max_batch) * p.n_heads + head) * p.max_seq * (size_t)p.d +
                    (c32 - head * p.d);
        }
#pragma unroll
        for (int j = 0; j < MJ; ++j) {
            if constexpr (BIG) {
                if (i < 4) asm volatile("" : "+a"(acc[i][j]));
            }
            if (!live[j]) continue;
            if (MODE == MODE_STORE) {
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    store16(p.out + row[j] + n32 + 8 * q, acc[i][j][q * 4 + 0], acc[i][j][q * 4 + 1], acc[i][j][q * 4 + 2],
                            acc[i][j][q * 4 + 3]);
                continue;
            }
            uint2 h4[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float v[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    v[e] = acc[i][j][q * 4 + e] + bv[MODE == MODE_STORE ? 0 : q][e];
                    if (MODE == MODE_BIAS_RELU) v[e] = fmaxf(v[e], 0.f);
                }
                if (MODE == MODE_QKV && !part)
                    store16(p.out + row[j] + n32 + 8 * q, v[0] * p.qscale, v[1] * p.qscale, v[2] * p.qscale, v[3] * p.qscale);
                else
                    h4[q] = make_uint2(pack2(v[0], v[1]), pack2(v[2], v[3]));
            }
            if (MODE == MODE_BIAS_RELU || part) {  // (uniform) halves: eight of a row per lane
                u32x4* ob = p.out_blocks + row[j] + (size_t)(n32 >> 4) * 64;
#pragma unroll
                for (int qq = 0; qq < 2; ++qq) {
                    const u32x4 v8 = join_halves(h4[2 * qq], h4[2 * qq + 1]);
                    if (MODE == MODE_BIAS_RELU) store16(ob + qq * 64, v8);
                    else if (append[j]) store16(kvcol + kvrow[j] + 8 * (2 * qq + hh), v8);
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);  // (a column block's values in registers at a time)
    }
}

// One matrix instruction with the accumulator tile pinned to a register file: the accumulation registers (VG =
// false) or the vector registers.  Twenty accumulator tiles do not fit into the 256 accumulation registers, and left
// to itself the compiler keeps them all there and moves the overflow in and out around every instruction (832 moves
// per stage).  Written as assembly the instruction is opaque to the compiler's hazard recogniser: nothing but these
// instructions touches an accumulator inside the k loop, and the caller waits out the matrix pipeline before the
// epilogue reads them.
template <bool VG>
__device__ __forceinline__ void mfma_f16_pinned(f32x16& c, const u32x4& a, const u32x4& b) {
    if constexpr (VG) asm volatile("v_mfma_f32_32x32x16_f16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b));
    else asm volatile("v_mfma_f32_32x32x16_f16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
}

constexpr int BM = 256;  // rows of X per tile of the big kernel; its width is 64 NA columns (NA = 4 or 5)
constexpr int BSTAGES = 4;

// NA: 32-column blocks of a wavefront's sub-tile (its 32 NA x 128 accumulators: 4 NA tiles of 32 x 32).  NA = 4 is the
// 256-column tile described above.  NA = 5, a 320-column tile, takes 18 KiB of operands for 80 matrix instructions
// (a tenth fewer bytes per flop), keeps a fifth of its accumulators in the vector registers, and is chosen where
// its tiles divide the matrix and the CUs better: at hidden size 5120 the QKV GEMM is six full rounds instead of
// seven and a half, FC1 eight instead of ten, and the out-projection and FC2 two, with nothing left to cut along k.
// Measured on 8192 rows with the same operands launch after launch: FC1 1506 -> 1391 us, the QKV shape 1187 -> 1048;
// inside the prompt pass, where every launch streams new weights, 180.2 -> 177.2 ms for the pass on one box (with
// the wide tile for QKV and FC1 only: 178.9).
template <int MODE, int NA>
__global__ __launch_bounds__(256, 1) void gemm_tiled256_kernel(const u32x4* __restrict__ Wp, const u32x4* __restrict__ X,
                                                               const u32x4* __restrict__ bias8, int KB, int NT32, int MT32,
                                                               int tiles_n, int tiles_m, int ksplit, int split_tn, Epi p) {
    constexpr int BN = 64 * NA;       // columns of the tile
    constexpr int XOFF = 4 * NA;      // blocks of a stage: W row-tile i, k-block j at 2 i + j; X row-tile i at XOFF + 2 i + j
    constexpr int SB = 4 * NA + 16;   // blocks of a stage (two k-blocks of 2 NA W row-tiles and 8 X row-tiles)
    __shared__ u32x4 ring[BSTAGES][SB][64];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int wn = wave & 1, wm = wave >> 1;  // this wavefront's 32 NA (n) x 128 (m) sub-tile
    const int cur_len = epilogue_len<MODE>(p);
    // Work items, in the order of `slot`: the tiles of the first split_tn columns of tiles with their whole k range, then
    // the tiles of the other columns once per k range (k range after k range).  Each of the two parts is dealt out
    // so that an XCD gets a contiguous run of it.  A workgroup takes every gridDim.x-th slot.
    const int n_whole = split_tn * tiles_m, whole_pad = (n_whole + 7) / 8 * 8;
    const int n_cut = (tiles_n - split_tn) * tiles_m * ksplit, slots = whole_pad + (n_cut + 7) / 8 * 8;
    struct Item { int tm, tn, ks, st0, nstage; };
    Item it;
    auto decode = [&](int slot) {  // false: a slot of padding
        const bool cut = slot >= whole_pad;
        const int idx = cut ? slot - whole_pad : slot;
        const int cols = cut ? tiles_n - split_tn : split_tn;  // columns of tiles of this part
        const int nblk = cols * tiles_m;
        const int nitem = cut ? n_cut : nblk;
        const int per_xcd = (nitem + 7) / 8;
        const int item = (idx % 8) * per_xcd + idx / 8;
        if (item >= nitem) return false;
        const int lin = item % nblk, ks = item / nblk;
        const int nks = cut ? ksplit : 1;  // k ranges of this tile
        constexpr int GROUP = 4;  // m-tiles per super-row: the 32 tiles an XCD works on at once share 4 X panels and 8 W panels
        const int gsize = GROUP * cols;
        const int g = lin / gsize, first_m = g * GROUP;
        const int gm = min(GROUP, tiles_m - first_m);
        const int nst_all = KB / 2;  // KB is even (K % 32 == 0)
        const int st0 = (int)((long)ks * nst_all / nks);
        it = Item{first_m + (lin % gsize) % gm, (cut ? split_tn : 0) + (lin % gsize) / gm, ks, st0,
                  (int)((long)(ks + 1) * nst_all / nks) - st0};
        return true;
    };
    int slot = blockIdx.x;
    auto next_item = [&]() {  // the next slot from `slot` on that holds an item
        while (slot < slots && !decode(slot)) slot += gridDim.x;
        return slot < slots;
    };
    if (!next_item()) return;
    // The SB blocks of a stage are copied by the four wavefronts, CW each: wavefront w copies blocks w CW .. w CW + CW - 1
    // (block c < XOFF: W row-tile c / 2, k-block c % 2; else X row-tile (c - XOFF) / 2).  Row-tiles past the matrix:
    // the last one (computed, never stored).
    constexpr int CW = NA + 4;  // copies per wavefront and stage
    const u32x4* src[CW];
    auto set_sources = [&]() {
#pragma unroll
        for (int q = 0; q < CW; ++q) {
            const int c = wave * CW + q;
            const bool isw = c < XOFF;
            const int rt = isw ? min(it.tn * 2 * NA + (c >> 1), NT32 - 1) : min(it.tm * 8 + ((c - XOFF) >> 1), MT32 - 1);
            src[q] = (isw ? Wp : X) + ((size_t)rt * KB + (size_t)it.st0 * 2 + (c & 1)) * 64 + lane;
        }
    };
    auto copy1 = [&](int st, int q) {
        load_block_to_lds(src[q] + (size_t)st * 128, &ring[st & (BSTAGES - 1)][wave * CW + q][0]);
    };
    auto issue = [&](int st) {
#pragma unroll
        for (int q = 0; q < CW; ++q) copy1(st, q);
    };
    constexpr int C2 = CW / 2;  // copies 0 .. C2-1 of a stage go out in the second half of stage t-3, the rest in the first of t-2
    f32x16 acc[NA][4];
    struct Ops { u32x4 a[NA], b[4]; };
    // LDS read q (0 .. NA+3) of a k-block, in the order the matrix instructions below first need the operands:
    // a0, b0, b1, b2, b3, a1, a2, ...
    constexpr int NR = NA + 4;
    auto read1 = [&](Ops& o, int st, int j, int q) {
        u32x4 (*slot)[64] = ring[st & (BSTAGES - 1)];
        if (q == 0) o.a[0] = slot[(wn * NA) * 2 + j][lane];
        else if (q <= 4) o.b[q - 1] = slot[XOFF + (wm * 4 + q - 1) * 2 + j][lane];
        else o.a[q - 4] = slot[(wn * NA + q - 4) * 2 + j][lane];
    };
    auto read_ops = [&](Ops& o, int st, int j) {
#pragma unroll
        for (int q = 0; q < NR; ++q) read1(o, st, j, q);
    };
    // matrix instruction n (0 .. 4 NA - 1) of a k-block: accumulator tile (n / 4, n % 4)
    // (NA = 5: the tiles of the first four column blocks live in the accumulation registers, the fifth block's in
    // the vector registers)
    auto mma1 = [&](const Ops& o, int n) {
        if constexpr (NA > 4) {
            if ((n >> 2) < 4) mfma_f16_pinned<false>(acc[n >> 2][n & 3], o.a[n >> 2], o.b[n & 3]);
            else mfma_f16_pinned<true>(acc[n >> 2][n & 3], o.a[n >> 2], o.b[n & 3]);
        } else {
            acc[n >> 2][n & 3] = mfma_f16(o.a[n >> 2], o.b[n & 3], acc[n >> 2][n & 3]);
        }
    };
    auto mma_all = [&](const Ops& o) {
#pragma unroll
        for (int n = 0; n < 4 * NA; ++n) mma1(o, n);
    };
    // The prologue issues what would fall before stage 0.
    auto prologue = [&]() {
        issue(0);
        if (it.nstage >= 2) issue(1);
        if (it.nstage >= 3) {
#pragma unroll
            for (int q = 0; q < C2; ++q) copy1(2, q);
        }
    };
    set_sources();
    prologue();
    if (it.nstage >= 3) wait_vmcnt<CW + C2>();
    else if (it.nstage == 2) wait_vmcnt<CW>();
    else wait_vmcnt<0>();
    // One tile after another.  Between two of them nothing but this workgroup runs on the CU: the next tile's first stages are requested
    // as soon as everybody has read the last stage, ahead of the epilogue that covers their way.  (A workgroup per tile before, and an
    // epilogue of rows outside, columns inside: a four-layer prompt pass of 8192 rows, hidden 5120, 13.91 -> 13.68 ms, one of 2560
    // rows 5.24 -> 5.15, six layers of 16384 rows, hidden 2048, and the scoring head 13.08 -> 12.42.)
    for (;;) {
        const int nstage = it.nstage, tm = it.tm, tn = it.tn, ks = it.ks;
#pragma unroll
        for (int i = 0; i < NA; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[i][j] = f32x16{};
        __syncthreads();
        Ops opa, opb;
        read_ops(opa, 0, 0);
        int s = 0;
        // Steady state: stage s+1 and the first copies of stage s+2 are in flight; the first half of stage s requests the
        // rest of stage s+2 (into the slot stage s-2 left: everybody passed the barrier of stage s-1 since), the second
        // half the first copies of stage s+3 (into the slot of stage s-1, behind this stage's barrier).  Scheduling
        // barriers keep the order written here.  The workgroup barrier is the bare instruction: what it orders are the
        // copies, which the wait before it covers -- the LDS reads in flight across it belong to the stage in use, not to
        // the slot about to be refilled (a fence would wait for them).
        // In each half of a stage (2 NA pairs of matrix instructions) the first pairs are followed by two LDS reads each
        // (the operands of the other half: the last of them is at least eight matrix instructions old when the half
        // ends, so the wait for the reads at the top of a half finds them done), the last ones by one copy each.
        constexpr int NP = 2 * NA;  // pairs of matrix instructions per half
        static_assert((NR + 1) / 2 + (CW - C2) <= NP, "reads and copies of a half fit behind its pairs");
        for (; s + 3 < nstage; ++s) {
#pragma unroll
            for (int q = 0; q < NP; ++q) {
                mma1(opa, 2 * q);
                mma1(opa, 2 * q + 1);
                if (2 * q < NR) {
                    read1(opb, s, 1, 2 * q);
                    if (2 * q + 1 < NR) read1(opb, s, 1, 2 * q + 1);
                } else if (q >= NP - (CW - C2)) {
                    copy1(s + 2, C2 + q - (NP - (CW - C2)));
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            wait_vmcnt<CW>();  // this wavefront's copies of stage s+1 have landed ...
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_barrier();  // ... and everybody's; everybody is done with stage s-1
            asm volatile("" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int q = 0; q < NP; ++q) {
                mma1(opb, 2 * q);
                mma1(opb, 2 * q + 1);
                if (2 * q < NR) {
                    read1(opa, s + 1, 0, 2 * q);
                    if (2 * q + 1 < NR) read1(opa, s + 1, 0, 2 * q + 1);
                } else if (q >= NP - C2) {
                    copy1(s + 3, q - (NP - C2));
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        for (; s < nstage; ++s) {  // the last three stages: only the late copies of the last one are left to request
            if (s + 2 < nstage) {
#pragma unroll
                for (int q = C2; q < CW; ++q) copy1(s + 2, q);
            }
            read_ops(opb, s, 1);
            mma_all(opa);
            if (s + 1 < nstage) {
                if (s + 2 < nstage) wait_vmcnt<CW>();
                else wait_vmcnt<0>();
                __syncthreads();
                read_ops(opa, s + 1, 0);
            }
            mma_all(opb);
        }
        slot += gridDim.x;
        const bool more = next_item();
        if (more) {
            __syncthreads();  // (the reads of the last stage have been waited for: its matrix instructions are issued)
            set_sources();
            prologue();
        }
        if constexpr (NA > 4) asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");  // the last matrix instructions' results are in
        if constexpr (MODE == MODE_SCORE) {
            // (the lane's number formed anew: kept through the loop it is a register too many)
            const int lane1 = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
            score_tile<NA, 4, true>(p, acc, tm * BM + wm * 128, tn * BN + wn * 32 * NA, tn * 2 + wn, lane1);
        } else store_tile<MODE, NA, 4, true>(p, bias8, acc, tm * BM + wm * 128, tn * BN + wn * 32 * NA, ks, cur_len, lane);
        if (!more) return;
        wait_vmcnt<0>();
    }
}

// ----------------------------------------------------------------- 256 x 64..192 tiles, and halved ones of up to 256 rows, on a deep ring (few rows)
//
// Prompt passes of too few rows to give every CU a 256 x 256 tile, and the wide decode steps.  What bounds these is not
// the matrix cores but how fast one CU pulls operands in: about 64 KB can be outstanding per CU whatever the ring's depth,
// a weight block takes 1.3 us from HBM and an activation block 0.45 us out of L2, so a stage (two k-blocks: 16 KiB of
// weights, 4 MW KiB of activations) takes 0.33 / 0.39 / 0.43 us for MW = 1 / 2 / 3, and a launch is fast when it has
// a workgroup on every CU.  Hence: tiles of 64 MW rows so that few rows are padding, each cut into k ranges until the
// CUs are covered (ring_plan), and as many stages in flight as LDS holds (8 / 6 / 5).  The schedule is the big
// kernel's -- LDS reads and copies dealt out behind the matrix instructions, a bare workgroup barrier per stage -- with
// one difference: a slot is refilled behind the barrier of its own stage (every wavefront waits for its own LDS reads
// before it), so all but one of the slots are in flight.
// Halved tiles -- two workgroups to 256 columns, 128 each (NW = 2) -- give narrow matrices and few rows more workgroups for the same number of k ranges, or leave them out
// (launches on one set of operands; inside the engine: ring_plan):
// 250 x 8192 x 2048 27.6 -> 18.8 us with whole sums, 250 x 16384 x 4096 53.9 -> 45.9, 96 x 2048 x 8192 14.4 (13 ranges) -> 11.8 (8),
// 180 x 1024 x 1024 6.5 -> 5.1; 384 rows and more of wide matrices go better on 256 columns (12288 x 4096 46.4 / 53.6).  (A CU has some 64 KB of
// copies on their way whatever they hit: prefetching the weights into L2 with scalar loads, 50 lines a microsecond and CU, is too slow by
// a factor of four.)
// Measured, the kernel before this (four stages, one range) -> this one with one k range per tile -> with the planned ones:
// 250 x 4096 x 16384: 269 -> 203 -> 45 us; 250 x 16384 x 4096: 79 -> 56, the plan (one range on 64-row tiles; ranges would
// need finish_kernel, 8 us); 250 x 12288 x 4096: 41 and 8 for finish_kernel; 96 x 5120 x 20480: 52 (eight ranges) -> 44 (twelve);
// 768 x 12288 x 4096: 150 -> 76 (192-row tiles, one range).
template <int NW, int MW> struct RingShape {
    static constexpr int TN = 64 * NW, TM = 64 * MW;         // rows of W (columns) and of X per tile
    static constexpr int SB = (2 * NW + 2 * MW) * 2;         // blocks per stage (two k-blocks)
    static constexpr int NST = 160 / SB < 8 ? 160 / SB : 8;  // stages that fit into 160 KiB
    static constexpr int CW = SB / 4;                        // copies per wavefront and stage
};

// s_waitcnt vmcnt(N) lgkmcnt(0)
template <int N>
__device__ __forceinline__ void wait_vmcnt_lgkm0() {
    __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | (0x7 << 4));
}

// STREAM: the weights' copies are non-temporal
template <int MODE, int NW, int MW, bool STREAM>
__global__ __launch_bounds__(256, 1) void gemm_ring_kernel(const u32x4* __restrict__ Wp, const u32x4* __restrict__ X,
                                                           const u32x4* __restrict__ bias8, int KB, int NT32, int MT32,
                                                           int tiles_n, int tiles_m, int ksplit, Epi p) {
    typedef RingShape<NW, MW> Sh;
    constexpr int SB = Sh::SB, NST = Sh::NST, CW = Sh::CW;
    constexpr int NM = NW * MW, NR = NW + MW;  // matrix instructions, LDS reads per wavefront and k-block
    static_assert((NST - 1) * CW <= 63, "the wait counter holds every copy in flight");
    constexpr int XOFF = 4 * NW;
    __shared__ u32x4 ring[NST][SB][64];  // block c of a stage: W row-tile c / 2, k-block c % 2; from XOFF on X row-tile (c - XOFF) / 2
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    // A contiguous run of items per XCD; the row tiles of one (column tile, k range) are neighbours and share its weights
    const int nitem = tiles_n * tiles_m * ksplit, per_xcd = (nitem + 7) / 8;
    const int item = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
    if (item >= nitem) return;
    const int tm = item % tiles_m, rest = item / tiles_m;
    const int tn = rest % tiles_n, ks = rest / tiles_n;
    const int wn = wave & 1, wm = wave >> 1;  // this wavefront's 32 NW (n) x 32 MW (m) sub-tile
    [[maybe_unused]] const int cur_len = epilogue_len<MODE>(p);
    // LM head with the final LayerNorm folded in (decode steps of up to 64 rows, whose rows are one tile of 64: MW = 1): this
    // wavefront's share of the rows' statistics
    constexpr bool FOLDS = MODE == MODE_LMHEAD && MW == 1;
    [[maybe_unused]] LnLoads<4> lnl[FOLDS ? 2 : 1];
    if constexpr (FOLDS) {
        if (p.ln_stats) {
#pragma unroll
            for (int x = 0; x < 2; ++x) ln_issue<4>(lnl[x], p, min(tm * 2 + x, MT32 - 1), wave, lane);
        }
    }
    f32x16 acc[NW][MW];
#pragma unroll
    for (int i = 0; i < NW; ++i)
#pragma unroll
        for (int j = 0; j < MW; ++j) acc[i][j] = f32x16{};
    const int nst_all = KB / 2;  // KB is even (K % 32 == 0)
    const int st0 = (int)((long)ks * nst_all / ksplit);
    const int nstage = (int)((long)(ks + 1) * nst_all / ksplit) - st0;
    // a wavefront's copies of a stage: NW blocks of W, then MW of X
    auto block_of = [&](int q) { return q < NW ? wave * NW + q : XOFF + wave * MW + q - NW; };
    const u32x4* src[CW];  // row-tiles past the matrix: the last one (computed, never stored)
#pragma unroll
    for (int q = 0; q < CW; ++q) {
        const bool isw = q < NW;
        const int c = block_of(q);
        const int rt = isw ? min(tn * 2 * NW + (c >> 1), NT32 - 1) : min(tm * 2 * MW + ((c - XOFF) >> 1), MT32 - 1);
        src[q] = (isw ? Wp : X) + ((size_t)rt * KB + (size_t)st0 * 2 + (c & 1)) * 64 + lane;
    }
    auto copy1 = [&](int st, int slot, int q) {
        u32x4* dst = &ring[slot][block_of(q)][0];
        if (STREAM && q < NW) load_block_to_lds<true>(src[q] + (size_t)st * 128, dst);
        else load_block_to_lds(src[q] + (size_t)st * 128, dst);
    };
    struct Ops { u32x4 a[NW], b[MW]; };
    // LDS read q of a k-block, in the order the matrix instructions first need the operands: a0, b0 .., a1 ..
    auto read1 = [&](Ops& o, int slot, int j, int q) {
        if (q == 0) o.a[0] = ring[slot][wn * NW * 2 + j][lane];
        else if (q <= MW) o.b[q - 1] = ring[slot][XOFF + (wm * MW + q - 1) * 2 + j][lane];
        else o.a[q - MW] = ring[slot][(wn * NW + q - MW) * 2 + j][lane];
    };
    auto mma1 = [&](const Ops& o, int n) { acc[n / MW][n % MW] = mfma_f16(o.a[n / MW], o.b[n % MW], acc[n / MW][n % MW]); };
    // Two reads behind each matrix instruction until all are out, then the copies, spread over the remaining ones.
    constexpr int R2 = (NR + 1) / 2 < NM - 1 ? (NR + 1) / 2 : NM - 1;
    constexpr int C2 = (CW + 1) / 2;  // copies of a stage that go out in the second half of a loop trip; the rest in the next first half
    auto read_behind = [](int q) { return q / 2 < NM - 1 ? q / 2 : NM - 1; };
    auto copy_behind = [](int q, int n) { return R2 + q * (NM - R2) / n; };
    auto barrier = []() {  // the bare instruction: the waits before it say what it orders
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    // this wavefront's LDS reads are done, and its copies of all but the `later` youngest stages have landed
    auto wait_stage = [&](int later) {
        if (later >= NST - 1) wait_vmcnt_lgkm0<(NST - 1) * CW>();
        else if (NST > 7 && later == 6) wait_vmcnt_lgkm0<6 * CW <= 63 ? 6 * CW : 0>();
        else if (NST > 6 && later == 5) wait_vmcnt_lgkm0<5 * CW <= 63 ? 5 * CW : 0>();
        else if (NST > 5 && later == 4) wait_vmcnt_lgkm0<4 * CW>();
        else if (later == 3) wait_vmcnt_lgkm0<3 * CW>();
        else if (later == 2) wait_vmcnt_lgkm0<2 * CW>();
        else if (later == 1) wait_vmcnt_lgkm0<CW>();
        else wait_vmcnt_lgkm0<0>();
    };
    const int n_pro = min(NST, nstage);
    for (int st = 0; st < n_pro; ++st)
#pragma unroll
        for (int q = 0; q < CW; ++q) copy1(st, st, q);
    wait_stage(n_pro - 1);
    barrier();
    Ops opa, opb;
#pragma unroll
    for (int q = 0; q < NR; ++q) read1(opa, 0, 0, q);
    int s = 0, slot = 0;             // the stage in use and its slot
    int late = 0, late_slot = 0;     // the stage whose last copies are still to be requested
    for (; s + NST < nstage; ++s) {  // steady state: stages s+1 .. s+NST-1 are in flight
        const int nslot = slot + 1 == NST ? 0 : slot + 1;
        const bool have_late = s > 0;
#pragma unroll
        for (int n = 0; n < NM; ++n) {
            mma1(opa, n);
#pragma unroll
            for (int q = 0; q < NR; ++q)
                if (read_behind(q) == n) read1(opb, slot, 1, q);
            if (have_late) {
#pragma unroll
                for (int q = C2; q < CW; ++q)
                    if (copy_behind(q - C2, CW - C2) == n) copy1(late, late_slot, q);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        wait_vmcnt_lgkm0<(NST - 2) * CW>();  // stage s+1 has landed, this stage's slot has been read: by everybody behind the barrier
        barrier();
        late = s + NST; late_slot = slot;
#pragma unroll
        for (int n = 0; n < NM; ++n) {
            mma1(opb, n);
#pragma unroll
            for (int q = 0; q < NR; ++q)
                if (read_behind(q) == n) read1(opa, nslot, 0, q);
#pragma unroll
            for (int q = 0; q < C2; ++q)
                if (copy_behind(q, C2) == n) copy1(late, late_slot, q);
            __builtin_amdgcn_sched_barrier(0);
        }
        slot = nslot;
    }
    if (s > 0) {
#pragma unroll
        for (int q = C2; q < CW; ++q) copy1(late, late_slot, q);
    }
    for (; s < nstage; ++s) {  // the last stages: everything has been requested
        const int nslot = slot + 1 == NST ? 0 : slot + 1;
#pragma unroll
        for (int q = 0; q < NR; ++q) read1(opb, slot, 1, q);
#pragma unroll
        for (int n = 0; n < NM; ++n) mma1(opa, n);
        if (s + 1 < nstage) {
            wait_stage(nstage - 2 - s);
            barrier();
#pragma unroll
            for (int q = 0; q < NR; ++q) read1(opa, nslot, 0, q);
        }
#pragma unroll
        for (int n = 0; n < NM; ++n) mma1(opb, n);
        slot = nslot;
    }
    static_assert(NW == 4 || (MODE != MODE_LMHEAD && MODE != MODE_SCORE), "a wavefront's 128 vocabulary entries are one partial");
    if constexpr (MODE == MODE_LMHEAD) {
        float2 fold[MW];
#pragma unroll
        for (int j = 0; j < MW; ++j) fold[j] = make_float2(0.f, 1.f);
        float* lds = reinterpret_cast<float*>(&ring[0][0][0]);  // the ring is free: statistics and logits go through it
        __syncthreads();
        if constexpr (FOLDS) {
            if (p.ln_stats) {
                float4* lnp = reinterpret_cast<float4*>(lds + 4 * 64 * 64);
#pragma unroll
                for (int x = 0; x < 2; ++x) ln_partial<4>(lnl[x], p, min(tm * 2 + x, MT32 - 1), wave, lane, lnp + x * 4 * 32);
                __syncthreads();
                fold[0] = ln_finish<4>(lnp + wm * 4 * 32, lane & 31, p);
            }
        }
        lm_head_tile<MW>(p, acc, fold, tm * Sh::TM + wm * 32 * MW, tn * Sh::TN + wn * 128, tn * 2 + wn, lane,
                         lds + wave * 64 * 64);
    } else if constexpr (MODE == MODE_SCORE) score_tile<4, MW>(p, acc, tm * Sh::TM + wm * 32 * MW, tn * Sh::TN + wn * 128, tn * 2 + wn, lane);
    else store_tile<MODE, NW, MW>(p, bias8, acc, tm * Sh::TM + wm * 32 * MW, tn * Sh::TN + wn * 32 * NW, ks, cur_len, lane);
}

// One wavefront per scored row: log-sum-exp over the vocabulary slices in slice order, then
// out[b][t] = z[next token] - lse  (out is [B][S-1]; the last position of a sequence scores nothing).
__global__ __launch_bounds__(256) void score_reduce_kernel(const float2* __restrict__ stats, const float* __restrict__ tgt,
                                                           int parts, int M, int S, float* __restrict__ out) {
    const int m = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (m >= M || m % S == S - 1) return;
    const float2* sp = stats + (size_t)m * parts;
    float mx = -INFINITY;
    for (int i = lane; i < parts; i += 64) mx = fmaxf(mx, sp[i].x);
    for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
    float sum = 0.f;
    for (int i = lane; i < parts; i += 64) {
        const float2 e = sp[i];
        if (e.x > -INFINITY) sum += e.y * expf(e.x - mx);
    }
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
    if (lane == 0) out[(size_t)(m / S) * (S - 1) + m % S] = tgt[m] - (mx + logf(sum));
}


constexpr int kMaxTiledKSplit = 16;  // k ranges a tile of a few-row GEMM is cut into at most
// Many rows (a prompt or scoring pass): 256 x 256 tiles, one workgroup per CU, once there are enough of them to
// give every CU one.
static bool use_big_tile(int M, int N) {
    return M >= 1024 && (long)((N + TN - 1) / TN) * ((M + 255) / 256) >= plan_cus();
}

// How a many-row GEMM is cut into tiles of 256 rows: 64 na columns wide (na = 4 or 5), and, where the partial sums
// may go through scratch (may_cut), the tiles of the columns from split_col on in ks = 2 k ranges.  The tiles come in
// rounds of one per CU and a partly empty round costs a full one; the cost is in units of a whole 256-column tile.
struct BigPlan { int na, ks, split_col; };
static BigPlan big_plan(int M, int N, int KB, bool may_cut) {
    const long cus = plan_cus(), tm = (M + BM - 1) / BM;
    may_cut = may_cut && KB % 4 == 0 && KB / 2 >= 8 * BSTAGES;
    BigPlan best{4, 1, 0};
    double best_cost = 1e30;
    for (int na = 4; na <= 5; ++na) {
        const long tn = (N + 64 * na - 1) / (64 * na);
        // a 320-column tile is five quarters of the work, done with a tenth fewer operand bytes per flop
        const double unit = na == 5 ? 1.25 * 0.98 : 1.0;
        for (long s = 0; s <= (may_cut ? tn : 0); ++s) {  // s columns of tiles cut in two
            const long whole = (tn - s) * tm, cutn = 2 * s * tm;
            // a cut tile costs a little more than half (its own ramp and epilogue), and every cut column a second
            // set of partial sums for the LayerNorm to read
            const double cost = ((double)((whole + cus - 1) / cus) + 0.52 * (double)((cutn + cus - 1) / cus) + 0.004 * s) * unit;
            if (cost < best_cost - 1e-9) {
                best_cost = cost;
                best = BigPlan{na, s ? 2 : 1, s ? (int)(tn - s) * 64 * na : 0};
            }
        }
    }
    return best;
}

// How a GEMM of too few rows or tiles for whole rounds of big tiles is cut: tiles of 256 columns x 64 mw rows (mw = 1, 2, 3:
// the ring kernel; 4: the big one, which at 5 takes 320 columns), every tile in ks k ranges.  One workgroup per CU, so
// a launch costs its rounds of ramp plus stages, and on top of that: the weights' way from HBM, writing the partial
// sums (fused = false: of a GEMM whose consumer, a LayerNorm, adds them up and pays for reading them), and, for an
// epilogue that needs the whole sum (fused), the pass of finish_kernel.  Microseconds fitted to launches of M = 96 ..
// 768 rows and the 1.3B .. 13B matrices (uncontended stages 0.33 / 0.39 / 0.43 / 0.53 / 0.68 us; a second, partly empty
// round: 4096 x 4096 and 768 rows, 240 workgroups 33.6 us, 288: 54.1).
// (tile: mw, or 10 + mw for halved tiles)
struct RingPlan { int tile, ks; };
static RingPlan ring_plan_256(int M, int N, int KB, bool fused, size_t capacity_floats, int max_mw = 5) {
    constexpr double kStage[5] = {0.33, 0.39, 0.43, 0.53, 0.68}, kRamp[5] = {6.0, 7.0, 8.5, 12.0, 14.0};
    const long cus = plan_cus(), stages = KB / 2;
    const double sums = 4.0 * M * N / 5e6, weights = 32.0 * N * KB / 14e6;
    RingPlan best{2, 1};
    double best_cost = 1e30;
    for (int mw = 1; mw <= max_mw; ++mw) {
        const int tm = mw < 4 ? 64 * mw : 256, tn = mw < 5 ? 256 : 320;
        const long tiles = (long)((N + tn - 1) / tn) * ((M + tm - 1) / tm);
        for (int ks = 1; ks <= kMaxTiledKSplit; ++ks) {
            if (ks > 1 && (stages / ks < 4 || (size_t)ks * M * N > capacity_floats)) break;
            const double rounds = (double)((tiles * ks + cus - 1) / cus);
            double cost = rounds * (kRamp[mw - 1] + (double)((stages + ks - 1) / ks) * kStage[mw - 1]) + weights;
            if (!fused) cost += 2.0 * ks * sums;
            else if (ks > 1) cost += 2.0 * ks * sums + 5.0;
            if (cost < best_cost) {
                best_cost = cost;
                best = RingPlan{mw, ks};
            }
        }
    }
    return best;
}

// The same with halved tiles among the candidates, by a cost fitted inside the engine: prompt passes of 33 .. 1000 rows through models of
// hidden 1024 .. 9216 whose weights no cache holds, one GEMM's plan forced at a time (408 GEMMs, some 18 plans each: the plan chosen costs 0.2 us
// more than the fastest on average, 4.6 at most).  The stages and the epilogue of a CU's rounds, and the weights' way from HBM, which they
// cover in part; the partial sums' writes; and what reads them.  (A fit to launches that reuse one set of operands took those out of the
// caches for nothing and priced whole sums too low: QKV of hidden 5120 and 80 rows in tiles of 64 x 128 47 us, in four ranges of 128 x 256 37 and
// 6 for what adds them up.  A layer of a decode step, the plan above / that fit / this: hidden 5120, 80 rows 200.3 / 207.9 / 199.5 us, 112 rows
// 215.8 / 221.9 / 216.9; 7168, 160 rows 398 / 400 / 379; 4096, 65 rows 146 / 146 / 143, 200 rows 204 / 193 / 192; 1024,
// 160 rows 69 / 52 / 52.)
// All of the fit's matrices have a multiple of 512 rows.  Others keep the plan above, which the tests' table of tiles (4480 wide) is drawn up for.
// That is no crossing: this one is ahead there too, a prompt pass or a wide decode step by 6 to 25 % at hidden 768, 4 to 24 at 1344, -1 to 8 at 4480, 0 to 6 at
// 4096 with an FFN of 10944.
static RingPlan ring_plan(int M, int N, int KB, bool fused, size_t capacity_floats) {
    if (N % 512) return ring_plan_256(M, N, KB, fused, capacity_floats);
    struct Tile { int id, nw, mw; double stage; };
    static constexpr Tile kTiles[] = {{1, 4, 1, 0.372}, {2, 4, 2, 0.363}, {3, 4, 3, 0.40}, {4, 4, 4, 0.497}, {5, 5, 4, 0.85},
                                      {11, 2, 1, 0.193}, {12, 2, 2, 0.243}, {13, 2, 3, 0.296}, {14, 2, 4, 0.348}};
    const double sums = 4.0 * M * N, weights = 32.0 * N * KB / 6.8e6;
    const double tail_of_range = sums / 3.7e6 + sums / (fused ? 5.45e6 : 4.6e6), idle = 0.03 * weights;
    const int cus = plan_cus(), stages = KB / 2;
    RingPlan best{2, 1};
    double best_cost = 1e30;
    for (const Tile& t : kTiles) {
        const int tiles = ((N + 64 * t.nw - 1) / (64 * t.nw)) * ((M + 64 * t.mw - 1) / (64 * t.mw));
        for (int ks = 1; ks <= kMaxTiledKSplit; ++ks) {
            if (ks > 1 && (stages < 4 * ks || (size_t)ks * M * N > capacity_floats)) break;
            const double tail = fused && ks == 1 ? sums / 3.7e6 : ks * tail_of_range + (fused ? 3.0 : 0.0), left = best_cost - tail;
            if (left <= 0) break;  // (it grows with the ranges)
            // a second round costs more than its share (nothing covers its ramp), a partly empty one more than a whole one
            const int full = (tiles * ks + cus - 1) / cus;
            const double rounds = (double)(tiles * ks) / cus;
            const double turns = full == 1 ? 1.0 : 1.0 + 2.1 * (full - 1) - 1.1 * (rounds - 1.0);
            const double core = turns * (t.stage * ((stages + ks - 1) / ks) + 0.425 * t.nw * t.mw);
            const double hbm = full == 1 ? weights + idle * (1.0 - rounds) : weights;
            // (compared as cubes: a launch that no graph replays is planned anew, and a root for each candidate was most of what
            // that costs the host: 96 rows of 5120 x 20480 5.0 us, so 1.6, 0.5 of it the measuring call)
            const double cubes = core * core * core + hbm * hbm * hbm;
            if (cubes < left * left * left) {
                best_cost = std::cbrt(cubes) + tail;
                best = RingPlan{t.id, ks};
            }
        }
    }
    return best;
}

// Workgroups of the big kernel: one per CU, each XCD the same number
static int big_grid(int slots) { return std::min(slots, std::max(8, plan_cus() / 8 * 8)); }

// Whether the weights' copies of the ring kernel are non-temporal.  A copy of what comes from HBM then moves 6.6 - 7.1 TB/s on 256 CUs instead
// of 5.8, and the activations stay in L2.  Matrices of 96 MB and more: a layer of such is more than the 256 MiB cache in front of memory holds,
// while a model of narrower layers may be in there as a whole (two layers of hidden 2048, 384 rows: 155 us, streamed 169; twelve of 768, 64 rows 581 and
// 608).  And several rows of tiles share what one of them fetched only while they keep together.  Plain / streamed per launch, measured
// alternately in one process, such matrices of hidden 3584 .. 7168, 34 .. 1000 rows:
//   one row of tiles                                  0.92 - 1.26, mean 1.07 (28672 x 7168 and 80 rows 88.5 / 75.4 us, 4096 x 16384 and 100 rows 33.4 / 25.7);
//   several, 128 columns to a workgroup, whole sums:
//     64 tile rows                                    0.95 - 1.32, mean 1.17 (12288 x 4096 and 96 rows 1.23, 14336 x 3584 and 120 rows 1.31);
//     128 to 256, the last row of tiles at least seven eighths full  0.98 - 1.06, mean 1.01;
//       or less                                       0.81 - 1.07: a row of padding runs ahead of the others (14336 x 3584 and 160 rows 34.4 / 42.3);
//   several, k ranges or 256 columns                  0.77 - 1.05.
static bool ring_streams(int M, int N, int KB, int tile_rows, int wg_cols, int ksplit) {
    if ((size_t)N * KB * 32 < 96000000) return false;
    const int tiles_m = (M + tile_rows - 1) / tile_rows;
    if (tiles_m == 1) return true;
    if (wg_cols != 128 || ksplit > 1) return false;
    return tile_rows == 64 ? N > 63 * 128 : 8 * (M - (tiles_m - 1) * tile_rows) >= 7 * tile_rows;  // (columns: fewer lost, of smaller matrices)
}
template <int MODE, int NW, int MW>
static void launch_ring(hipStream_t s, int grid, const u32x4* W, const u32x4* X, const u32x4* bias8, int KB, int NT32, int MT32, int tiles_n, int tiles_m,
                        int ksplit, const Epi& p) {
    if (ring_streams(p.M, p.N, KB, 64 * MW, 64 * NW, ksplit)) gemm_ring_kernel<MODE, NW, MW, true><<<grid, 256, 0, s>>>(W, X, bias8, KB, NT32, MT32, tiles_n, tiles_m, ksplit, p);
    else gemm_ring_kernel<MODE, NW, MW, false><<<grid, 256, 0, s>>>(W, X, bias8, KB, NT32, MT32, tiles_n, tiles_m, ksplit, p);
}

// tile: 1 .. 3 the ring kernel with 64 tile rows, 11 .. 14 halved tiles of 64 (tile - 10) rows (128 columns to a workgroup), 4 / 5 the big tiles.  Columns from split_col on are cut into ksplit k
// ranges (with one range none are; the ring kernel cuts every tile).
template <int MODE>
void launch_tiled(hipStream_t s, const void* Wp, const void* Xhi, int KB, int N, int M, const Epi& p, int tile, int ksplit,
                  int split_col) {
    const int NT32 = (N + 31) / 32, MT32 = (M + 31) / 32;
    // (the bias through a pointer of its own: declared never to alias the outputs, its values can be fetched
    // with scalar loads, which do not queue behind the epilogue's stores)
    const u32x4 *W = (const u32x4*)Wp, *X = (const u32x4*)Xhi, *bias8 = (const u32x4*)p.bias;
    if (tile < 4) {
        const int tiles_n = (N + 255) / 256, tiles_m = (M + 64 * tile - 1) / (64 * tile);
        const int grid = (tiles_n * tiles_m * ksplit + 7) / 8 * 8;
        if (tile == 1) launch_ring<MODE, 4, 1>(s, grid, W, X, bias8, KB, NT32, MT32, tiles_n, tiles_m, ksplit, p);
        else if (MODE == MODE_SCORE || tile == 2)  // (score_tile knows no 192-row tile)
            launch_ring<MODE, 4, 2>(s, grid, W, X, bias8, KB, NT32, MT32, tiles_n, tiles_m, ksplit, p);
        else launch_ring<MODE, 4, MODE == MODE_SCORE ? 2 : 3>(s, grid, W, X, bias8, KB, NT32, MT32, tiles_n, tiles_m, ksplit, p);
        return;
    }
    if constexpr (MODE == MODE_SCORE) {
        const int tiles_n = (N + TN - 1) / TN, tiles_m = (M + BM - 1) / BM, grid = big_grid((tiles_n * tiles_m + 7) / 8 * 8);
        gemm_tiled256_kernel<MODE, 4><<<grid, 256, 0, s>>>(W, X, bias8, KB, NT32, MT32, tiles_n, tiles_m, 1, tiles_n, p);
    } else if constexpr (MODE != MODE_LMHEAD) {
        if (tile > 10) {
            const int tiles_n = (N + 127) / 128, tiles_m = (M + 64 * (tile - 10) - 1) / (64 * (tile - 10));
            const int grid = (tiles_n * tiles_m * ksplit + 7) / 8 * 8;
            if (tile == 11) launch_ring<MODE, 2, 1>(s, grid, W, X, bias8, KB, NT32, MT32, tiles_n, tiles_m, ksplit, p);
            else if (tile == 12) launch_ring<MODE, 2, 2>(s, grid, W, X, bias8, KB, NT32, MT32, tiles_n, tiles_m, ksplit, p);
            else if (tile == 13) launch_ring<MODE, 2, 3>(s, grid, W, X, bias8, KB, NT32, MT32, tiles_n, tiles_m, ksplit, p);
            else launch_ring<MODE, 2, 4>(s, grid, W, X, bias8, KB, NT32, MT32, tiles_n, tiles_m, ksplit, p);
            return;
        }
        const int bn = 64 * tile, tiles_n = (N + bn - 1) / bn, tiles_m = (M + BM - 1) / BM;
        const int split_tn = ksplit > 1 ? split_col / bn : tiles_n;  // without a k-split every tile is whole
        const int whole = split_tn * tiles_m, cutn = (tiles_n - split_tn) * tiles_m * ksplit;
        const int grid = big_grid((whole + 7) / 8 * 8 + (cutn + 7) / 8 * 8);
        if (tile == 5) gemm_tiled256_kernel<MODE, 5><<<grid, 256, 0, s>>>(W, X, bias8, KB, NT32, MT32, tiles_n, tiles_m, ksplit, split_tn, p);
        else gemm_tiled256_kernel<MODE, 4><<<grid, 256, 0, s>>>(W, X, bias8, KB, NT32, MT32, tiles_n, tiles_m, ksplit, split_tn, p);
    }
}

// After a k-split MODE_STORE GEMM whose epilogue needs the whole sum: adds the partial sums in split
// order and applies the epilogue of MODE (bias + ReLU into blocks, or the QKV hand-out).
template <int MODE>
__global__ __launch_bounds__(256) void finish_kernel(const float* __restrict__ part, int ksplit, size_t split, Epi p) {
    const int quads = p.N >> 2;  // N is a multiple of 4 here
    const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (size_t)p.M * quads) return;
    const int m = (int)(idx / quads), n0 = (int)(idx % quads) * 4;
    float4 v = *reinterpret_cast<const float4*>(part + (size_t)m * p.N + n0);
    for (int k0 = 1; k0 < ksplit; k0 += 4) {  // in split order, four loads on their way at a time
        float4 y[4];
#pragma unroll
        for (int k = 0; k < 4; ++k)
            y[k] = *reinterpret_cast<const float4*>(part + (size_t)min(k0 + k, ksplit - 1) * split + (size_t)m * p.N + n0);
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (k0 + k < ksplit) { v.x += y[k].x; v.y += y[k].y; v.z += y[k].z; v.w += y[k].w; }
    }
    epilogue4<MODE>(p, m, n0, 0, v.x, v.y, v.z, v.w, epilogue_bias<MODE>(p, n0), epilogue_len<MODE>(p));
}

}  // namespace

// ------------------------------------------------------------------ launchers

// Floats of scratch the k ranges of a few-row GEMM can make use of: at most a round of tiles' sums (256 tiles of
// 256 x 256), and never more than kMaxTiledKSplit sets of the matrix.
size_t bf16_tiled_scratch_floats(int rows, int widest) {
    return std::min((size_t)256 * 256 * 256, (size_t)kMaxTiledKSplit * rows * widest);
}

// Out-projection and FC2 (the following LayerNorm adds the partial sums): which tile, *ks k ranges for the tiles of
// columns >= *split_col and one for the columns before.  With enough rows and columns for rounds of big tiles
// these come whole first, in rounds of one per CU, and the cut ones fill the last, shorter round: 640 tiles of 256
// columns on 256 CUs are two rounds of whole tiles and one of 256 half tiles, with a second set of partial sums for a
// fifth of the columns only (and 512 tiles of 320 columns are two rounds with nothing to cut).  With fewer, ring_plan
// cuts every tile.
void bf16_tiled_store_plan(int M, int N, int K, size_t capacity_floats, int* tile, int* ks, int* split_col, bool few_rows_whole) {
    if (use_big_tile(M, N)) {
        const BigPlan g = big_plan(M, N, K / 16, (size_t)2 * M * N <= capacity_floats);
        *tile = g.na; *ks = g.ks; *split_col = g.split_col;
        return;
    }
    const RingPlan g = ring_plan(M, N, K / 16, false, few_rows_whole ? 0 : capacity_floats);
    *tile = g.tile; *ks = g.ks; *split_col = 0;
}

void bf16_tiled_plan_query(int M, int N, int K, int may_cut, size_t capacity_floats, int cus, int* tile_cols, int* ks,
                           int* split_col) {
    plan_cus_override = cus;
    *tile_cols = 0; *ks = 1; *split_col = 0;
    const size_t room = capacity_floats ? capacity_floats : (size_t)-1;
    if (use_big_tile(M, N)) {
        const BigPlan g = big_plan(M, N, K / 16, may_cut && (size_t)2 * M * N <= room);
        *tile_cols = 64 * g.na; *ks = g.ks; *split_col = g.split_col;
    } else if (may_cut) {
        *ks = ring_plan(M, N, K / 16, false, room).ks;
    }
    plan_cus_override = 0;
}

// QKV and FC1, whose epilogue needs the whole sum: with k ranges finish_kernel applies it.
static RingPlan fused_plan(int M, int N, int KB, size_t capacity_floats) {
    if (use_big_tile(M, N)) return RingPlan{big_plan(M, N, KB, false).na, 1};
    return ring_plan(M, N, KB, true, capacity_floats);
}

// The LM head's tiles (no scratch: whole k ranges; 192 rows at most to a tile).  Up to 64 rows one row of 64-row tiles: there the
// final LayerNorm may come folded in.
static RingPlan lm_head_plan(int M, int V, int K) { return ring_plan_256(M, V, K / 16, true, 0, M <= 64 ? 1 : 3); }

// The scoring head: 0 for gemm_score_kernel (two workgroups per CU) or 4, the big tiles, from two rounds of the former's on, else the
// ring kernel's tile.  Microseconds of rounds, fitted to 640 .. 16384 rows of 5000 .. 50272 ids at k = 1024 .. 5120: a big tile loads a
// third less for its products (16 KiB to 64 of them), where two of the others reduce the logits of one behind the products of the other and
// a last round of at most one workgroup to a CU takes seven tenths.  Rows x ids x k, two workgroups / big, us of the product: 16384 x 50272 x
// 2048 3614 / 3161, x 5120 8265 / 6706, x 1024 1909 / 1944; 2048 x 50272 x 1024 245 / 277, x 2048 494 / 472; 1300 x 50272 x 1024 175 / 195; 700 x 50272
// x 5120 487 / 398.  (The same slices of 128 entries and the same order of sums: the results are the same to the bit.)
static int score_tile(int M, int V, int K) {
    const long cus = plan_cus(), tn = (V + TN - 1) / TN, tiles = tn * ((M + 127) / 128), big = tn * ((M + BM - 1) / BM);
    if (tiles < 2 * cus) return M <= 64 ? 1 : 2;
    const long rest = tiles % (2 * cus);
    const double two = (double)(tiles / (2 * cus)) + (rest == 0 ? 0.0 : (rest <= cus ? 0.7 : 1.0));
    return (double)((big + cus - 1) / cus) * (15.0 + 0.0238 * K) < two * (5.3 + 0.0335 * K) ? 4 : 0;
}

bool bf16_ring_streams(int M, int N, int K, int tile_rows, int wg_cols, int ksplit) { return ring_streams(M, N, K / 16, tile_rows, wg_cols, ksplit); }

void bf16_pass_plan_query(int use, int M, int N, int K, size_t capacity_floats, int cus, int* tile_rows, int* tile_cols, int* wg_cols, int* ks,
                          int* split_col) {
    plan_cus_override = cus;
    int tile = 0;
    *ks = 1; *split_col = 0;
    if (use == TILED_STORE || use == TILED_STORE_WHOLE) {
        bf16_tiled_store_plan(M, N, K, capacity_floats, &tile, ks, split_col, use == TILED_STORE_WHOLE);
    } else if (use == TILED_FUSED) {
        const RingPlan g = fused_plan(M, N, K / 16, capacity_floats);
        tile = g.tile; *ks = g.ks;
    } else if (use == TILED_SCORE_HEAD) {
        tile = score_tile(M, N, K);
    } else {
        tile = bf16_lm_head_streams(M, N) ? -1 : lm_head_plan(M, N, K).tile;
    }
    plan_cus_override = 0;
    *tile_rows = tile < 0 ? 32 : (tile == 0 ? 128 : (tile > 10 ? 64 * (tile - 10) : (tile < 4 ? 64 * tile : 256)));
    *tile_cols = tile < 0 ? 32 : (tile == 5 ? 320 : 256);
    *wg_cols = tile > 10 ? 128 : *tile_cols;
}

void bf16_gemm_tiled_store(hipStream_t s, const void* Wp, const void* Xhi, int M, int N, int K, float* part, int tile, int ks,
                           int split_col) {
    bf16_gemm_args a;
    a.out = part; a.out_split = (size_t)M * N;
    launch_tiled<MODE_STORE>(s, Wp, Xhi, K / 16, N, M, make_epi(M, N, a), tile, ks, split_col);
}

void bf16_gemm_tiled(hipStream_t s, int mode, const void* Wp, const void* Xhi, int M, int N, int K, const bf16_gemm_args& a,
                     float* part, size_t part_floats) {
    const Epi p = make_epi(M, N, a);
    const RingPlan g = fused_plan(M, N, K / 16, part_floats);
    if (g.ks == 1) {  // the epilogue runs in the GEMM
        if (mode == EPI_BIAS_RELU) launch_tiled<MODE_BIAS_RELU>(s, Wp, Xhi, K / 16, N, M, p, g.tile, 1, 0);
        else launch_tiled<MODE_QKV>(s, Wp, Xhi, K / 16, N, M, p, g.tile, 1, 0);
        return;
    }
    bf16_gemm_tiled_store(s, Wp, Xhi, M, N, K, part, g.tile, g.ks, 0);
    const unsigned grid = (unsigned)(((size_t)M * (N / 4) + 255) / 256);
    if (mode == EPI_BIAS_RELU) finish_kernel<MODE_BIAS_RELU><<<grid, 256, 0, s>>>(part, g.ks, (size_t)M * N, p);
    else finish_kernel<MODE_QKV><<<grid, 256, 0, s>>>(part, g.ks, (size_t)M * N, p);
}

// The LM head of a decode step of more than 32 rows and a large vocabulary (bf16_lm_head_streams): the matrix is read once for all
// of them (the weight-streaming kernel takes 32 rows at a time and rereads it: 96 rows of 50272 x 5120 took 222 us, this 151, of
// which 23 are the noise).  Returns the soft-max partials per row.
int bf16_lm_head_tiles(hipStream_t s, const void* Wp, const void* X, int M, int V, int K, const bf16_gemm_args* fold, const he_dev_state* st,
                       float* logits_opt, float* stats, int* stats_idx) {
    Epi p{};
    if (fold) p = make_epi(M, V, *fold);
    p.M = M; p.N = V; p.st = st; p.logits = logits_opt; p.stats = stats; p.stats_idx = stats_idx;
    p.n_tiles = 2 * ((V + 255) / 256);
    launch_tiled<MODE_LMHEAD>(s, Wp, X, K / 16, V, M, p, lm_head_plan(M, V, K).tile, 1, 0);
    return p.n_tiles;
}

int bf16_score_parts(int V) { return 2 * ((V + TN - 1) / TN); }

void bf16_score_head(hipStream_t s, const void* Wp, const void* Xhi, int M, int S, int V, int K,
                     const int32_t* ids, float* stats, float* tgt, float* out) {
    Epi p{};
    p.M = M; p.N = V; p.S = S; p.ids = ids; p.sc_stats = (float2*)stats; p.sc_tgt = tgt; p.sc_parts = bf16_score_parts(V);
    const int NT32 = (V + 31) / 32, MT32 = (M + 31) / 32, KB = K / 16;
    const int tiles_n = (V + TN - 1) / TN, tiles_m = (M + 127) / 128, tiles = tiles_n * tiles_m, tile = score_tile(M, V, K);
    if (tile == 0)
        gemm_score_kernel<<<(tiles + 7) / 8 * 8, 256, 0, s>>>((const u32x4*)Wp, (const u32x4*)Xhi, KB, NT32, MT32, tiles_n, tiles_m, p);
    else
        launch_tiled<MODE_SCORE>(s, Wp, Xhi, KB, V, M, p, tile, 1, 0);
    score_reduce_kernel<<<(M + 3) / 4, 256, 0, s>>>((const float2*)stats, tgt, p.sc_parts, M, S, out);
}

