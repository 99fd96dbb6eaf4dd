// bf16 path: attention over the KV cache of IEEE halves (decode rows, short prompts, prompt rows on the matrix cores).
#include "../../include/he.h"
#include "bf16_common.h"

using namespace he_bf16;

namespace {

// ----------------------------------------------------------------- attention over the KV cache
//
// One workgroup per (row m, head h); the query at position cur_len + (m % S)
// sees keys 0..that position.  D/8 adjacent lanes own one key (16 bytes each, a
// whole row of K or V per group, coalesced); scores are reduced with wavefront
// shuffles, kept in LDS, soft-maxed, then the same lanes accumulate p_j * V[j].
// The output goes out as tiled half blocks for the out-projection GEMM.
//
// Two passes with a score buffer: the form for many (row, head) pairs and long caches, which run at the HBM rate (6.2 TB/s at 32
// sequences x 40 heads x 384 positions) -- four wavefronts where several workgroups share a CU, eight where two do.  attn_few_kernel below is the
// other.
template <int D, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void attn_kernel(const float* __restrict__ q, const half_t* __restrict__ kv,
                                                          u32x4* __restrict__ o,
                                                          const he_dev_state* __restrict__ st, int S, int layer, int H,
                                                          int n_heads, int max_batch, int max_seq) {
    constexpr int LPK = D / 8;     // lanes per key
    constexpr int KPW = 64 / LPK;  // keys per wavefront load
    constexpr int KR = WAVES * KPW;  // keys per workgroup round
    constexpr int U = 4;
    extern __shared__ float sc[];  // [max_seq] scores, then probabilities
    __shared__ float red[2][WAVES];
    __shared__ float ored[WAVES][LPK * 8];
    const int m = blockIdx.x, h = blockIdx.y;
    const int b = row_seq(st, m, S), T = seq_len(st, b) + (m % S) - row_pad(st, b) + 1;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int sub = lane % LPK, grp = lane / LPK;
    if (seq_done(st, b)) return;  // the sequence has ended: its row's output is not used any more
    if (T <= 0) {                 // a padding row: nothing to attend to, nothing reads the output; keep it finite
        if (wave == 0 && grp == 0) {
            const size_t slot = block_slot(m, h * D + sub * 8, H >> 4);
            o[slot] = u32x4{0u, 0u, 0u, 0u};
        }
        return;
    }
    const float4 qa = *reinterpret_cast<const float4*>(q + (size_t)m * H + h * D + sub * 8);
    const float4 qb = *reinterpret_cast<const float4*>(q + (size_t)m * H + h * D + sub * 8 + 4);
    const u32x4* Kp = reinterpret_cast<const u32x4*>(kv + kv_index(layer, 0, b, h, 0, max_batch, n_heads, max_seq, D));
    const u32x4* Vp = reinterpret_cast<const u32x4*>(kv + kv_index(layer, 1, b, h, 0, max_batch, n_heads, max_seq, D));
    const int jw = wave * KPW + grp;
    constexpr int STEP = KR * U;  // keys per workgroup iteration
    auto load_rows = [&](u32x4 (&dst)[U], const u32x4* src, int base) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int j = base + u * KR + jw;
            dst[u] = j < T ? __builtin_nontemporal_load(src + (size_t)j * LPK + sub) : u32x4{0u, 0u, 0u, 0u};
        }
    };
    // loads run one iteration ahead of the arithmetic, and the first values are requested
    // before the soft-max barrier, so the memory pipe never drains between the phases
    float mx = -INFINITY;
    u32x4 cur[U], nxt[U];
    load_rows(cur, Kp, 0);
    for (int base = 0; base < T; base += STEP) {
        if (base + STEP < T) load_rows(nxt, Kp, base + STEP);
        else load_rows(nxt, Vp, 0);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int j = base + u * KR + jw;
            float s = qa.x * half_lo(cur[u].x);
            s = fmaf(qa.y, half_hi(cur[u].x), s);
            s = fmaf(qa.z, half_lo(cur[u].y), s);
            s = fmaf(qa.w, half_hi(cur[u].y), s);
            s = fmaf(qb.x, half_lo(cur[u].z), s);
            s = fmaf(qb.y, half_hi(cur[u].z), s);
            s = fmaf(qb.z, half_lo(cur[u].w), s);
            s = fmaf(qb.w, half_hi(cur[u].w), s);
#pragma unroll
            for (int o2 = 1; o2 < LPK; o2 <<= 1) s += __shfl_xor(s, o2);
            if (j < T) {
                if (sub == 0) sc[j] = s;
                mx = fmaxf(mx, s);
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) cur[u] = nxt[u];
    }
    // cur now holds the first values
    for (int o2 = 32; o2 > 0; o2 >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o2));
    if (lane == 0) red[0][wave] = mx;
    __syncthreads();  // also publishes sc[]
    mx = red[0][0];
#pragma unroll
    for (int w = 1; w < WAVES; ++w) mx = fmaxf(mx, red[0][w]);
    float sum = 0.f;
    for (int j = threadIdx.x; j < T; j += 64 * WAVES) {
        const float pj = expf(sc[j] - mx);
        sc[j] = pj;
        sum += pj;
    }
    for (int o2 = 32; o2 > 0; o2 >>= 1) sum += __shfl_xor(sum, o2);
    if (lane == 0) red[1][wave] = sum;
    __syncthreads();  // also publishes the probabilities
    sum = 0.f;
#pragma unroll
    for (int w = 0; w < WAVES; w += 2) sum += red[1][w] + red[1][w + 1];
    float acc[8] = {};
    for (int base = 0; base < T; base += STEP) {
        if (base + STEP < T) load_rows(nxt, Vp, base + STEP);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int j = base + u * KR + jw;
            const float pj = j < T ? sc[j] : 0.f;
            acc[0] = fmaf(pj, half_lo(cur[u].x), acc[0]);
            acc[1] = fmaf(pj, half_hi(cur[u].x), acc[1]);
            acc[2] = fmaf(pj, half_lo(cur[u].y), acc[2]);
            acc[3] = fmaf(pj, half_hi(cur[u].y), acc[3]);
            acc[4] = fmaf(pj, half_lo(cur[u].z), acc[4]);
            acc[5] = fmaf(pj, half_hi(cur[u].z), acc[5]);
            acc[6] = fmaf(pj, half_lo(cur[u].w), acc[6]);
            acc[7] = fmaf(pj, half_hi(cur[u].w), acc[7]);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) cur[u] = nxt[u];
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {
#pragma unroll
        for (int o2 = LPK; o2 < 64; o2 <<= 1) acc[e] += __shfl_xor(acc[e], o2);
    }
    if (grp == 0) {
#pragma unroll
        for (int e = 0; e < 8; ++e) ored[wave][sub * 8 + e] = acc[e];
    }
    __syncthreads();
    if (threadIdx.x < LPK) {
        float ov[8];
        const float inv = 1.0f / sum;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int i = threadIdx.x * 8 + e;
            float t = 0.f;
#pragma unroll
            for (int w = 0; w < WAVES; w += 2) t += ored[w][i] + ored[w + 1][i];
            ov[e] = t * inv;
        }
        const size_t slot = block_slot(m, h * D + threadIdx.x * 8, H >> 4);
        o[slot] = u32x4{pack2(ov[0], ov[1]), pack2(ov[2], ov[3]), pack2(ov[4], ov[5]), pack2(ov[6], ov[7])};
    }
}

// The same in one pass, for few (row, head) pairs and short caches: what bounds those is not the stream but the chain from the state
// to the output, so there is one barrier and no score buffer.  Every group of D/8 lanes keeps the soft-max state of its own keys (largest
// score, sum, weighted values), K and V of a round are on their way together, one round ahead; the groups of a wavefront are
// merged with data-parallel moves, the wavefronts through LDS.  us, attn_kernel with the number of wavefronts that suited it -> this:
// 1 x 32 heads of 64, 516 keys 8.3 -> 6.9, 130 keys 5.0 -> 3.9; 7 x 32 heads of 128, 180 keys 8.5 -> 7.0; 2 x 40 of 128, 1999 keys
// 26.9 -> 24.5; 16 x 32 of 64, 56 keys 5.6 -> 4.6; 32 x 32 of 64, 64 keys 7.5 -> 5.9; 96 x 40 of 128, 80 keys 31.0 -> 29.0; but 32 x 40
// of 128: 160 keys 19.6 -> 19.4, 384 keys 39.6 -> 41.2.  (The line between the two: decode_attn_plan below.)
//
// Behind the pairs' workgroups come those that fetch the out-projection's weights meanwhile (bf16_ahead): memory has little to do here, the
// L2 caches keep what is read from one launch to the next, and workgroup j of every launch runs on XCD j mod 8.  A step, us, without ->
// with: 16 x 32 heads of 64, 56 keys, hidden 2048 (attention 5.0 -> 5.2, the out-projection 5.2 -> 4.1) 230.3 -> 224.4.  A cache that may hold
// more than 32 MiB is a stream of its own that this is in the way of: 16 x 32, 400 keys 268 -> 278.  The line goes by what the cache can
// hold, not by the keys in use: an engine with room for long answers does without.  Generations of 64 tokens, eight layers, without / with
// (two runs differ by 0.3 %): hidden 2048, 1 row 8 keys 1.013, 500 keys 1.006, 16 rows 1.029, 32 rows 1.034; 768, 1024 and 2560 0.993 .. 1.033, mean 1.01;
// 8-bit weights of hidden 1024 .. 4096, 1 .. 48 rows 0.997 .. 1.031, mean 1.015.
template <int THREADS>
__device__ __forceinline__ void fetch_ahead(const bf16_ahead& a, int j) {
    const bf16_ahead_share s = bf16_ahead_of(a, j);
    uint32_t got = 0;
    for (int l0 = threadIdx.x; l0 < s.lines; l0 += 4 * THREADS) {  // a line to a lane
        uint32_t v[4];
#pragma unroll
        for (int x = 0; x < 4; ++x)
            v[x] = *reinterpret_cast<const uint32_t*>((const char*)a.w + bf16_ahead_line(a, s, min(l0 + x * THREADS, s.lines - 1)));
        got ^= (v[0] ^ v[1]) ^ (v[2] ^ v[3]);
    }
    asm volatile("" ::"v"(got));  // (all that matters is where the lines are now)
}

template <int D, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void attn_few_kernel(const float* __restrict__ q, const half_t* __restrict__ kv,
                                                       u32x4* __restrict__ o, const he_dev_state* __restrict__ st, int S, int layer,
                                                       int H, int n_heads, int max_batch, int max_seq, bf16_ahead ahead) {
    constexpr int LPK = D / 8, KPW = 64 / LPK, KR = WAVES * KPW, U = 4, STEP = KR * U;
    static_assert(D <= 64 * WAVES, "an output value per thread");
    if ((int)blockIdx.y >= n_heads) {  // (whole rows of the grid: the last workgroups of them have nothing to fetch)
        const int j = (int)(blockIdx.y * gridDim.x + blockIdx.x) - (n_heads * (int)gridDim.x + 7) / 8 * 8;
        if (j >= 0 && j < ahead.wgs) fetch_ahead<64 * WAVES>(ahead, j);
        return;
    }
    __shared__ float2 ml[WAVES];          // a wavefront's largest score and sum
    __shared__ float ored[WAVES][D];      // ... and its weighted values
    const int m = blockIdx.x, h = blockIdx.y;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int sub = lane % LPK, grp = lane / LPK;
    const float4 qa = *reinterpret_cast<const float4*>(q + (size_t)m * H + h * D + sub * 8);
    const float4 qb = *reinterpret_cast<const float4*>(q + (size_t)m * H + h * D + sub * 8 + 4);
    const int b = row_seq(st, m, S), t = S == 1 ? 0 : m % S, T = seq_len(st, b) + t - row_pad(st, b) + 1;
    if (seq_done(st, b)) return;  // the sequence has ended: its row's output is not used any more
    if (T <= 0) {                 // a padding row: nothing to attend to, nothing reads the output; keep it finite
        if (wave == 0 && grp == 0) o[block_slot(m, h * D + sub * 8, H >> 4)] = u32x4{0u, 0u, 0u, 0u};
        return;
    }
    const u32x4* Kp = reinterpret_cast<const u32x4*>(kv + kv_index(layer, 0, b, h, 0, max_batch, n_heads, max_seq, D));
    const u32x4* Vp = reinterpret_cast<const u32x4*>(kv + kv_index(layer, 1, b, h, 0, max_batch, n_heads, max_seq, D));
    const int jw = wave * KPW + grp;
    auto load_rows = [&](u32x4 (&dst)[U], const u32x4* src, int base) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int j = base + u * KR + jw;
            dst[u] = j < T ? __builtin_nontemporal_load(src + (size_t)j * LPK + sub) : u32x4{0u, 0u, 0u, 0u};
        }
    };
    float mx = -INFINITY, sum = 0.f, acc[8] = {};
    u32x4 k[U], v[U];
    load_rows(k, Kp, 0);
    load_rows(v, Vp, 0);
    for (int base = 0; base < T; base += STEP) {
        float s[U];
        float top = mx;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            float x = qa.x * half_lo(k[u].x);
            x = fmaf(qa.y, half_hi(k[u].x), x);
            x = fmaf(qa.z, half_lo(k[u].y), x);
            x = fmaf(qa.w, half_hi(k[u].y), x);
            x = fmaf(qb.x, half_lo(k[u].z), x);
            x = fmaf(qb.y, half_hi(k[u].z), x);
            x = fmaf(qb.z, half_lo(k[u].w), x);
            x = fmaf(qb.w, half_hi(k[u].w), x);
            x = lane_sum<LPK>(x);
            s[u] = base + u * KR + jw < T ? x : -INFINITY;
            top = fmaxf(top, s[u]);
        }
        const bool more = base + STEP < T;  // (the same for the whole workgroup)
        if (more) load_rows(k, Kp, base + STEP);
        // (nothing above -inf yet: the state stays what it is)
        const float ref = top > -INFINITY ? top : 0.f, keep = expf(mx - ref);
        float pr[U];
#pragma unroll
        for (int u = 0; u < U; ++u) pr[u] = base + u * KR + jw < T ? expf(s[u] - ref) : 0.f;
        mx = top;
        sum = fmaf(sum, keep, (pr[0] + pr[1]) + (pr[2] + pr[3]));
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] *= keep;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            acc[0] = fmaf(pr[u], half_lo(v[u].x), acc[0]);
            acc[1] = fmaf(pr[u], half_hi(v[u].x), acc[1]);
            acc[2] = fmaf(pr[u], half_lo(v[u].y), acc[2]);
            acc[3] = fmaf(pr[u], half_hi(v[u].y), acc[3]);
            acc[4] = fmaf(pr[u], half_lo(v[u].z), acc[4]);
            acc[5] = fmaf(pr[u], half_hi(v[u].z), acc[5]);
            acc[6] = fmaf(pr[u], half_lo(v[u].w), acc[6]);
            acc[7] = fmaf(pr[u], half_hi(v[u].w), acc[7]);
        }
        if (more) load_rows(v, Vp, base + STEP);
    }
    // the groups of the wavefront
    float wmx = mx;
    if (LPK <= 8) wmx = fmaxf(wmx, lane_xor8(wmx));
    wmx = lane_max32_apart(lane_max16_apart(wmx));
    const float own = mx > -INFINITY ? expf(mx - wmx) : 0.f;
    sum = lane_sum_apart<LPK>(sum * own);
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = lane_sum_apart<LPK>(acc[e] * own);
    if (lane == 0) ml[wave] = make_float2(wmx, sum);
    if (grp == 0) {
        float4* dst = reinterpret_cast<float4*>(&ored[wave][sub * 8]);
        dst[0] = make_float4(acc[0], acc[1], acc[2], acc[3]);
        dst[1] = make_float4(acc[4], acc[5], acc[6], acc[7]);
    }
    __syncthreads();
    if (threadIdx.x >= D) return;
    // the wavefronts: lane i of 16 knows wavefront i's weight
    const float2 e = ml[min(lane & 15, WAVES - 1)];
    const bool counts = (lane & 15) < WAVES && e.x > -INFINITY;
    const float all = lane_max<16>(e.x);
    const float w = counts ? expf(e.x - all) : 0.f, total = lane_sum<16>(counts ? e.y * w : 0.f);
    float out = 0.f;
#pragma unroll
    for (int x = 0; x < WAVES; ++x) out = fmaf(__uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(w), x)), ored[x][threadIdx.x], out);
    out *= 1.0f / total;
    const float next = lane_xor1(out);
    if ((threadIdx.x & 1) == 0) {
        const int i = threadIdx.x, n = h * D + i;
        reinterpret_cast<uint32_t*>(o + block_slot(m, n & ~7, H >> 4))[(n & 7) >> 1] = pack2(out, next);
    }
}

// ----------------------------------------------------------------- attention, prompt rows
//
// Same arithmetic as attn_kernel for a block of QB consecutive queries of one (sequence, head):
// every K and V row fetched once serves all QB queries, which cuts the L2 traffic of the prompt
// pass by QB.  The QB partial dot products of a key are reduced over the D/8 lanes that share
// the key with a halving butterfly (each step sends half of the values and keeps the other
// half), so the lanes end up owning different queries.  Query t0+i sees keys <= cur_len + t0 + i.
constexpr int QB = 8;

template <int D>
__global__ __launch_bounds__(256) void attn_prompt_kernel(const float* __restrict__ q, const half_t* __restrict__ kv,
                                                          u32x4* __restrict__ o,
                                                          const he_dev_state* __restrict__ st, int S, int layer, int H,
                                                          int n_heads, int max_batch, int max_seq) {
    constexpr int LPK = D / 8, KPW = 64 / LPK, KR = 4 * KPW, U = 2, STEP = KR * U;
    extern __shared__ float sc[];  // [QB][max_seq] scores, then probabilities
    __shared__ float ored[4][QB][D];
    __shared__ float inv_sum[QB];
    const int t0 = blockIdx.x * QB, h = blockIdx.y, b = blockIdx.z;
    const int nq = min(QB, S - t0);
    const int cur = seq_len(st, b) - row_pad(st, b);  // cache position of row 0: negative while rows are padding
    const int T = cur + t0 + nq;  // keys any query of the block may see
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int sub = lane % LPK, grp = lane / LPK;
    float qv[QB][8];
#pragma unroll
    for (int i = 0; i < QB; ++i) {
        float4 a = make_float4(0.f, 0.f, 0.f, 0.f), c = a;
        if (i < nq) {
            const float* qp = q + (size_t)(b * S + t0 + i) * H + h * D + sub * 8;
            a = *reinterpret_cast<const float4*>(qp);
            c = *reinterpret_cast<const float4*>(qp + 4);
        }
        qv[i][0] = a.x; qv[i][1] = a.y; qv[i][2] = a.z; qv[i][3] = a.w;
        qv[i][4] = c.x; qv[i][5] = c.y; qv[i][6] = c.z; qv[i][7] = c.w;
    }
    const u32x4* Kp = reinterpret_cast<const u32x4*>(kv + kv_index(layer, 0, b, h, 0, max_batch, n_heads, max_seq, D));
    const u32x4* Vp = reinterpret_cast<const u32x4*>(kv + kv_index(layer, 1, b, h, 0, max_batch, n_heads, max_seq, D));
    const int jw = wave * KPW + grp;
    auto load_rows = [&](u32x4 (&dst)[U], const u32x4* src, int base) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int j = base + u * KR + jw;
            dst[u] = j < T ? src[(size_t)j * LPK + sub] : u32x4{0u, 0u, 0u, 0u};
        }
    };
    // which query this lane owns after the butterfly
    int qown = 0;
    {
        int nval = QB;
#pragma unroll
        for (int off = LPK / 2; off >= 1; off >>= 1)
            if (nval > 1) { nval >>= 1; if (sub & off) qown += nval; }
    }
    constexpr bool kPairs = LPK > QB;  // two lanes end up with the same query: the even one stores
    u32x4 cur_r[U], nxt_r[U];
    load_rows(cur_r, Kp, 0);
    for (int base = 0; base < T; base += STEP) {
        if (base + STEP < T) load_rows(nxt_r, Kp, base + STEP);
        else load_rows(nxt_r, Vp, 0);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int j = base + u * KR + jw;
            const float k0 = half_lo(cur_r[u].x), k1 = half_hi(cur_r[u].x);
            const float k2 = half_lo(cur_r[u].y), k3 = half_hi(cur_r[u].y);
            const float k4 = half_lo(cur_r[u].z), k5 = half_hi(cur_r[u].z);
            const float k6 = half_lo(cur_r[u].w), k7 = half_hi(cur_r[u].w);
            float part[QB];
#pragma unroll
            for (int i = 0; i < QB; ++i) {
                float s = qv[i][0] * k0;
                s = fmaf(qv[i][1], k1, s); s = fmaf(qv[i][2], k2, s); s = fmaf(qv[i][3], k3, s);
                s = fmaf(qv[i][4], k4, s); s = fmaf(qv[i][5], k5, s); s = fmaf(qv[i][6], k6, s);
                part[i] = fmaf(qv[i][7], k7, s);
            }
            int nval = QB;
#pragma unroll
            for (int off = LPK / 2; off >= 1; off >>= 1) {
                if (nval > 1) {
                    nval >>= 1;
                    const bool upper = (sub & off) != 0;
#pragma unroll
                    for (int c = 0; c < QB / 2; ++c) {
                        if (c < nval) {
                            const float send = upper ? part[c] : part[c + nval];
                            const float keep = upper ? part[c + nval] : part[c];
                            part[c] = keep + __shfl_xor(send, off);
                        }
                    }
                } else {
                    part[0] += __shfl_xor(part[0], off);
                }
            }
            if (j < T && (!kPairs || (sub & 1) == 0))
                sc[qown * max_seq + j] = j <= max(cur + t0 + qown, 0) ? part[0] : -INFINITY;  // a padding row looks at key 0
        }
#pragma unroll
        for (int u = 0; u < U; ++u) cur_r[u] = nxt_r[u];
    }
    __syncthreads();
    {   // soft-max of query 2*wave + (lane / 32) over its 32 lanes
        const int qi = 2 * wave + (lane >> 5), l32 = lane & 31;
        float* row = sc + qi * max_seq;
        float mx = -INFINITY;
        for (int j = l32; j < T; j += 32) mx = fmaxf(mx, row[j]);
        for (int o2 = 16; o2 > 0; o2 >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o2));
        float sum = 0.f;
        for (int j = l32; j < T; j += 32) {
            const float pj = expf(row[j] - mx);
            row[j] = pj;
            sum += pj;
        }
        for (int o2 = 16; o2 > 0; o2 >>= 1) sum += __shfl_xor(sum, o2);
        if (l32 == 0) inv_sum[qi] = sum > 0.f ? 1.0f / sum : 0.f;  // no keys at all: a block of padding rows
    }
    __syncthreads();
    float acc[QB][8] = {};
    for (int base = 0; base < T; base += STEP) {
        if (base + STEP < T) load_rows(nxt_r, Vp, base + STEP);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int j = base + u * KR + jw;
            if (j < T) {
                const float v0 = half_lo(cur_r[u].x), v1 = half_hi(cur_r[u].x);
                const float v2 = half_lo(cur_r[u].y), v3 = half_hi(cur_r[u].y);
                const float v4 = half_lo(cur_r[u].z), v5 = half_hi(cur_r[u].z);
                const float v6 = half_lo(cur_r[u].w), v7 = half_hi(cur_r[u].w);
#pragma unroll
                for (int i = 0; i < QB; ++i) {
                    const float pj = sc[i * max_seq + j];
                    acc[i][0] = fmaf(pj, v0, acc[i][0]); acc[i][1] = fmaf(pj, v1, acc[i][1]);
                    acc[i][2] = fmaf(pj, v2, acc[i][2]); acc[i][3] = fmaf(pj, v3, acc[i][3]);
                    acc[i][4] = fmaf(pj, v4, acc[i][4]); acc[i][5] = fmaf(pj, v5, acc[i][5]);
                    acc[i][6] = fmaf(pj, v6, acc[i][6]); acc[i][7] = fmaf(pj, v7, acc[i][7]);
                }
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) cur_r[u] = nxt_r[u];
    }
#pragma unroll
    for (int i = 0; i < QB; ++i)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
#pragma unroll
            for (int o2 = LPK; o2 < 64; o2 <<= 1) acc[i][e] += __shfl_xor(acc[i][e], o2);
        }
    if (grp == 0) {
#pragma unroll
        for (int i = 0; i < QB; ++i)
#pragma unroll
            for (int e = 0; e < 8; ++e) ored[wave][i][sub * 8 + e] = acc[i][e];
    }
    __syncthreads();
    for (int idx = threadIdx.x; idx < QB * LPK; idx += 256) {
        const int i = idx / LPK, c = idx % LPK;
        if (i >= nq) continue;
        float ov[8];
        const float inv = inv_sum[i];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int d0 = c * 8 + e;
            ov[e] = ((ored[0][i][d0] + ored[1][i][d0]) + (ored[2][i][d0] + ored[3][i][d0])) * inv;
        }
        const size_t slot = block_slot(b * S + t0 + i, h * D + c * 8, H >> 4);
        o[slot] = u32x4{pack2(ov[0], ov[1]), pack2(ov[2], ov[3]), pack2(ov[4], ov[5]), pack2(ov[6], ov[7])};
    }
}

// ----------------------------------------------------------------- attention, prompt rows, on the matrix cores
//
// Flash-style causal attention for the prompt pass.  One wavefront owns 32 queries of one
// (sequence, head); the four wavefronts of a workgroup share each 32-key tile of K and V through
// LDS.  Everything is computed transposed so that a lane owns ONE query: S^T = K Q^T puts the
// scores of query lane%32 in that lane's 16 accumulators (online soft-max needs one exchange
// with lane^32), and O^T = V^T P^T accumulates that query's output column, so the soft-max
// rescaling is a per-lane scalar.  Q and P enter the MFMA as two half terms (hi + lo).  The
// keys of a PV step are taken in the order the score accumulators already hold them.
//
// 32 matrix instructions per tile and wavefront (1024 cycles; head dimension 128) set the pace only if nothing else
// takes longer.  V is transposed on its way into LDS -- a thread brings eight dimensions of two consecutive keys and writes
// eight words -- so that an operand of V^T is two 8-byte reads (reading it out of untransposed rows took 64 16-bit reads per
// tile and wavefront, and the LDS pipe was the bottleneck); its pitch of 18 words puts both the writes (16 keys pairs x 4
// dimension groups) and the reads (32 dimensions) on all banks.  Two buffers: one barrier per tile.  The running maximum is
// kept in units of log2, so a probability is one multiply-add (score times log2 e less the maximum) and the hardware's 2^x.
// (log2 e multiplied into Q instead, ahead of its rounding to halves, takes a third off the largest query: 65504 -> 45403.)
// Measured: 2 x 1999 queries, 40 heads of 128: 405 -> 390 us with the above, -> 230 with the order of the workgroups below;
// 32 x 512, 32 heads of 64: 183 -> 174 -> 126; 32 x 256, 40 heads of 128: 132 -> 131 -> 121 (of which reading q in float,
// K and V and writing the output take 76).
template <int D>
__global__ __launch_bounds__(256, 2) void attn_prompt_mfma_kernel(const float* __restrict__ q,
                                                               const half_t* __restrict__ kv, u32x4* __restrict__ o,
                                                               const he_dev_state* __restrict__ st, int S, int layer,
                                                               int H, int n_heads, int max_batch, int max_seq, int batch) {
    constexpr int KBD = D / 16;      // k-blocks over the head dimension
    constexpr int DB = D / 32;       // 32-wide blocks of output dimensions
    constexpr int KPITCH = D + 8;    // halves per K row in LDS (16 bytes of padding)
    constexpr int VPITCH = 36;       // halves per V^T row: 32 keys and 8 bytes of padding
    __shared__ __align__(16) half_t ks[2][32 * KPITCH];
    __shared__ __align__(16) half_t vt[2][D * VPITCH];
    // Workgroups go round the XCDs by index, and one of late queries has many times the keys of one of early ones: with the
    // query blocks along the grid an XCD got the same blocks of every (sequence, head), and the launch waited for the XCD
    // with the last ones (up to 1.6 times the mean).  Here a (sequence, head) belongs to one XCD, and the blocks go out
    // longest first.
    const int qblocks = (S + 127) / 128, pairs = batch * n_heads, per_xcd = (pairs + 7) / 8, slot = blockIdx.x >> 3;
    const int pair = (slot % per_xcd) * 8 + (blockIdx.x & 7), qblock = qblocks - 1 - slot / per_xcd;
    if (pair >= pairs) return;  // the whole workgroup
    const int h = pair % n_heads, b = pair / n_heads;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int j = lane & 31, hh = lane >> 5;
    const int cur = seq_len(st, b) - row_pad(st, b);  // cache position of row 0: negative while rows are padding
    const int T = cur + S;                          // keys in the cache once this pass is stored
    const int t0 = (qblock * 4 + wave) * 32;        // this wavefront's first query
    const bool live = t0 < S;
    const int qpos = max(cur + t0 + j, 0);          // last key this lane's query may see (a padding row looks at key 0)
    const int wg_last = min(T - 1, cur + min(S, (qblock * 4 + 4) * 32) - 1);
    const int n_tiles = wg_last / 32 + 1;
    const int my_last_tile = live ? min(T - 1, cur + t0 + 31) / 32 : -1;

    const half_t* Kg = kv + kv_index(layer, 0, b, h, 0, max_batch, n_heads, max_seq, D);
    const half_t* Vg = kv + kv_index(layer, 1, b, h, 0, max_batch, n_heads, max_seq, D);
    // A tile's K and V rows are requested one tile ahead and wait in registers while the tile before
    // them is multiplied, so that their latency is not paid between two barriers.
    constexpr int NI = 32 * (D / 8) / 256;  // 16-byte pieces of K per thread and tile
    const bool has_v = (int)threadIdx.x < 2 * D;  // V: keys 2 vp, 2 vp + 1, dimensions 8 vc .. 8 vc + 7
    const int vp = threadIdx.x & 15, vc = threadIdx.x >> 4;
    u32x4 kreg[NI], vreg[2];
    auto request_tile = [&](int kt) {
#pragma unroll
        for (int n = 0; n < NI; ++n) {
            const int c = threadIdx.x + n * 256;
            const int key = c / (D / 8), d0 = (c % (D / 8)) * 8, kabs = kt * 32 + key;
            kreg[n] = u32x4{0u, 0u, 0u, 0u};
            if (kabs < T) kreg[n] = *reinterpret_cast<const u32x4*>(Kg + (size_t)kabs * D + d0);
        }
#pragma unroll
        for (int n = 0; n < 2; ++n) {
            const int kabs = kt * 32 + 2 * vp + n;
            vreg[n] = u32x4{0u, 0u, 0u, 0u};
            if (has_v && kabs < T) vreg[n] = *reinterpret_cast<const u32x4*>(Vg + (size_t)kabs * D + vc * 8);
        }
    };
    auto store_tile = [&](int buf) {
#pragma unroll
        for (int n = 0; n < NI; ++n) {
            const int c = threadIdx.x + n * 256;
            *reinterpret_cast<u32x4*>(&ks[buf][(c / (D / 8)) * KPITCH + (c % (D / 8)) * 8]) = kreg[n];
        }
        if (has_v) {
            const uint32_t a[4] = {vreg[0].x, vreg[0].y, vreg[0].z, vreg[0].w}, c[4] = {vreg[1].x, vreg[1].y, vreg[1].z, vreg[1].w};
            uint32_t* dst = reinterpret_cast<uint32_t*>(&vt[buf][0]) + vc * 8 * (VPITCH / 2) + vp;
#pragma unroll
            for (int e = 0; e < 4; ++e) {  // (key 2 vp, key 2 vp + 1) of dimensions 2 e and 2 e + 1
                dst[(2 * e) * (VPITCH / 2)] = (a[e] & 0xFFFFu) | (c[e] << 16);
                dst[(2 * e + 1) * (VPITCH / 2)] = (a[e] >> 16) | (c[e] & 0xFFFF0000u);
            }
        }
    };
    if (n_tiles > 0) request_tile(0);

    u32x4 qhi[KBD], qlo[KBD];
    {
        const bool ok = t0 + j < S;
        const float* qp = q + (size_t)(b * S + (ok ? t0 + j : 0)) * H + h * D + hh * 8;
#pragma unroll
        for (int kb = 0; kb < KBD; ++kb) {
            float4 a = make_float4(0.f, 0.f, 0.f, 0.f), c = a;
            if (ok) {
                a = *reinterpret_cast<const float4*>(qp + kb * 16);
                c = *reinterpret_cast<const float4*>(qp + kb * 16 + 4);
            }
            uint32_t h0, h1, h2, h3, l0, l1, l2, l3;
            split2(a.x, a.y, h0, l0); split2(a.z, a.w, h1, l1);
            split2(c.x, c.y, h2, l2); split2(c.z, c.w, h3, l3);
            qhi[kb] = u32x4{h0, h1, h2, h3};
            qlo[kb] = u32x4{l0, l1, l2, l3};
        }
    }
    f32x16 oacc[DB];
#pragma unroll
    for (int i = 0; i < DB; ++i) oacc[i] = f32x16{};
    constexpr float kLog2e = 1.44269504f;
    float m_run = -INFINITY, l_run = 0.f;  // m_run: in units of log2
    if (n_tiles > 0) {
        store_tile(0);
        if (n_tiles > 1) request_tile(1);
    }
    __syncthreads();
    for (int kt = 0; kt < n_tiles; ++kt) {
        const int buf = kt & 1;
        if (kt <= my_last_tile) {  // (else wholly above the diagonal for this wavefront; uniform per wavefront)
            f32x16 sacc = f32x16{};
#pragma unroll
            for (int kb = 0; kb < KBD; ++kb) {
                const u32x4 kblk = *reinterpret_cast<const u32x4*>(&ks[buf][j * KPITCH + kb * 16 + hh * 8]);
                sacc = mfma_f16(kblk, qlo[kb], sacc);
                sacc = mfma_f16(kblk, qhi[kb], sacc);
            }
            float mx = -INFINITY;
            if (kt * 32 + 31 > cur + t0) {  // the tile reaches past the first query's last key: mask per query
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int kabs = kt * 32 + 8 * (r >> 2) + 4 * hh + (r & 3);
                    if (kabs > qpos) sacc[r] = -INFINITY;
                }
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) mx = fmaxf(mx, sacc[r]);
            mx = fmaxf(mx, __shfl_xor(mx, 32));
            const float m_new = fmaxf(m_run, mx * kLog2e);  // finite from the first tile on: key 0 is visible to every query
            const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
            float psum = 0.f;
            float pr[16];
#pragma unroll
            for (int r = 0; r < 16; ++r) { pr[r] = __builtin_amdgcn_exp2f(fmaf(sacc[r], kLog2e, -m_new)); psum += pr[r]; }
            l_run = l_run * alpha + psum;
            if (__any(m_new != m_run)) {  // no query of this wavefront met a larger score: nothing to rescale
#pragma unroll
                for (int i = 0; i < DB; ++i)
#pragma unroll
                    for (int r = 0; r < 16; ++r) oacc[i][r] *= alpha;
            }
            m_run = m_new;
#pragma unroll
            for (int s2 = 0; s2 < 2; ++s2) {
                uint32_t ph[4], pl[4];
#pragma unroll
                for (int x = 0; x < 4; ++x) split2(pr[8 * s2 + 2 * x], pr[8 * s2 + 2 * x + 1], ph[x], pl[x]);
                const u32x4 phi = u32x4{ph[0], ph[1], ph[2], ph[3]}, plo = u32x4{pl[0], pl[1], pl[2], pl[3]};
                u32x4 vblk[DB];
#pragma unroll
                for (int i = 0; i < DB; ++i) {
                    // V^T operand: this lane's output dimension, the eight keys in the order the score accumulators hold them
                    const half_t* vrow = &vt[buf][(i * 32 + j) * VPITCH + s2 * 16 + 4 * hh];
                    const uint2 v0 = *reinterpret_cast<const uint2*>(vrow), v1 = *reinterpret_cast<const uint2*>(vrow + 8);
                    vblk[i] = u32x4{v0.x, v0.y, v1.x, v1.y};
                }
#pragma unroll
                for (int i = 0; i < DB; ++i) oacc[i] = mfma_f16(vblk[i], plo, oacc[i]);
#pragma unroll
                for (int i = 0; i < DB; ++i) oacc[i] = mfma_f16(vblk[i], phi, oacc[i]);
            }
        }
        if (kt + 1 < n_tiles) {
            store_tile(buf ^ 1);  // (everybody has left that buffer: the barrier that opened this tile)
            if (kt + 2 < n_tiles) request_tile(kt + 2);
            __syncthreads();
        }
    }
    if (!live || t0 + j >= S) return;
    const float l_tot = l_run + __shfl_xor(l_run, 32);
    const float inv = l_tot > 0.f ? 1.0f / l_tot : 0.f;  // 0: a wavefront of padding rows saw no tile
    const int m = b * S + t0 + j;
#pragma unroll
    for (int i = 0; i < DB; ++i)
#pragma unroll
        for (int qd = 0; qd < 4; ++qd) {
            const int dim = h * D + i * 32 + 8 * qd + 4 * hh;  // four consecutive output dimensions
            const size_t slot = block_slot(m, dim & ~7, H >> 4);
            reinterpret_cast<uint2*>(o + slot)[(dim >> 2) & 1] =
                make_uint2(pack2(oacc[i][qd * 4 + 0] * inv, oacc[i][qd * 4 + 1] * inv),
                           pack2(oacc[i][qd * 4 + 2] * inv, oacc[i][qd * 4 + 3] * inv));
        }
}

// The same for passes that leave CUs idle: the four wavefronts of a workgroup take one block of 32 queries together, every
// fourth tile of keys each, and merge their sums in LDS at the end.  What bounds such a pass is the serial chain of a block's
// tiles (1.7 us each with the tile's way through registers, LDS and a barrier); here it is a quarter as long and has no barrier: a
// wavefront reads its K operands straight from the cache (the register image of one is a row's 16 bytes per lane) and
// transposes V in LDS of its own.  The keys are read by four times as many workgroups, out of L2.  us, one workgroup per 128 queries ->
// this: 250 queries, 32 heads of 128 16.2 -> 11.9; 500, 32 of 64 19.1 -> 12.1; 1000, 16 of 64 33.0 -> 17.5; 4 x 879, 2 of 64 29.1 -> 12.0.  (Where a second
// round of workgroups loses: prompt_splits below.)
template <int D>
__global__ __launch_bounds__(256, 1) void attn_prompt_split_kernel(const float* __restrict__ q, const half_t* __restrict__ kv,
                                                                u32x4* __restrict__ o, const he_dev_state* __restrict__ st, int S, int layer,
                                                                int H, int n_heads, int max_batch, int max_seq, int batch) {
    constexpr int WAVES = 4;
    constexpr int KBD = D / 16, DB = D / 32, VPITCH = 36, NV = D / 32;  // NV: groups of eight dimensions a lane transposes per tile
    __shared__ __align__(16) half_t vt[WAVES][D * VPITCH];
    __shared__ f32x16 red[WAVES][DB][64];
    __shared__ float2 ml[WAVES][32];
    const int qblocks = (S + 31) / 32, pairs = batch * n_heads, per_xcd = (pairs + 7) / 8, slot = blockIdx.x >> 3;
    const int pair = (slot % per_xcd) * 8 + (blockIdx.x & 7), qblock = qblocks - 1 - slot / per_xcd;  // longest first
    if (pair >= pairs) return;  // the whole workgroup
    const int h = pair % n_heads, b = pair / n_heads;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int j = lane & 31, hh = lane >> 5, t0 = qblock * 32;
    const bool ok = t0 + j < S;
    float4 qa[KBD], qc[KBD];
    const float* qp = q + (size_t)(b * S + (ok ? t0 + j : 0)) * H + h * D + hh * 8;
#pragma unroll
    for (int kb = 0; kb < KBD; ++kb) {
        qa[kb] = *reinterpret_cast<const float4*>(qp + kb * 16);
        qc[kb] = *reinterpret_cast<const float4*>(qp + kb * 16 + 4);
    }
    const int cur = seq_len(st, b) - row_pad(st, b);  // cache position of row 0: negative while rows are padding
    const int T = cur + S;                          // keys in the cache once this pass is stored
    const int qpos = max(cur + t0 + j, 0);          // last key this lane's query may see (a padding row looks at key 0)
    const int n_tiles = min(T - 1, cur + t0 + 31) / 32 + 1;
    const half_t* Kg = kv + kv_index(layer, 0, b, h, 0, max_batch, n_heads, max_seq, D);
    const half_t* Vg = kv + kv_index(layer, 1, b, h, 0, max_batch, n_heads, max_seq, D);
    const int vp = lane & 15, vc = lane >> 4;  // V: keys 2 vp, 2 vp + 1, dimensions 8 (vc + 4 n) .. + 7
    u32x4 kreg[KBD], vreg[NV][2];
    auto request_tile = [&](int kt) {
        const int key = kt * 32 + j;
#pragma unroll
        for (int kb = 0; kb < KBD; ++kb) {
            kreg[kb] = u32x4{0u, 0u, 0u, 0u};
            if (key < T) kreg[kb] = *reinterpret_cast<const u32x4*>(Kg + (size_t)key * D + kb * 16 + hh * 8);
        }
#pragma unroll
        for (int n = 0; n < NV; ++n)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int kabs = kt * 32 + 2 * vp + e;
                vreg[n][e] = u32x4{0u, 0u, 0u, 0u};
                if (kabs < T) vreg[n][e] = *reinterpret_cast<const u32x4*>(Vg + (size_t)kabs * D + (vc + 4 * n) * 8);
            }
    };
    if (wave < n_tiles) request_tile(wave);
    u32x4 qhi[KBD], qlo[KBD];
#pragma unroll
    for (int kb = 0; kb < KBD; ++kb) {
        float4 a = qa[kb], c = qc[kb];
        if (!ok) a = c = make_float4(0.f, 0.f, 0.f, 0.f);
        uint32_t h0, h1, h2, h3, l0, l1, l2, l3;
        split2(a.x, a.y, h0, l0); split2(a.z, a.w, h1, l1);
        split2(c.x, c.y, h2, l2); split2(c.z, c.w, h3, l3);
        qhi[kb] = u32x4{h0, h1, h2, h3};
        qlo[kb] = u32x4{l0, l1, l2, l3};
    }
    f32x16 oacc[DB];
#pragma unroll
    for (int i = 0; i < DB; ++i) oacc[i] = f32x16{};
    constexpr float kLog2e = 1.44269504f;
    float m_run = -INFINITY, l_run = 0.f;  // m_run: in units of log2
    uint32_t* vw = reinterpret_cast<uint32_t*>(&vt[wave][0]);
    for (int kt = wave; kt < n_tiles; kt += WAVES) {
        f32x16 sacc = f32x16{};
#pragma unroll
        for (int kb = 0; kb < KBD; ++kb) {
            sacc = mfma_f16(kreg[kb], qlo[kb], sacc);
            sacc = mfma_f16(kreg[kb], qhi[kb], sacc);
        }
#pragma unroll
        for (int n = 0; n < NV; ++n) {
            const uint32_t a[4] = {vreg[n][0].x, vreg[n][0].y, vreg[n][0].z, vreg[n][0].w};
            const uint32_t c[4] = {vreg[n][1].x, vreg[n][1].y, vreg[n][1].z, vreg[n][1].w};
            uint32_t* dst = vw + (vc + 4 * n) * 8 * (VPITCH / 2) + vp;
#pragma unroll
            for (int e = 0; e < 4; ++e) {  // (key 2 vp, key 2 vp + 1) of dimensions 2 e and 2 e + 1
                dst[(2 * e) * (VPITCH / 2)] = (a[e] & 0xFFFFu) | (c[e] << 16);
                dst[(2 * e + 1) * (VPITCH / 2)] = (a[e] >> 16) | (c[e] & 0xFFFF0000u);
            }
        }
        if (kt + WAVES < n_tiles) request_tile(kt + WAVES);
        if (kt * 32 + 31 > cur + t0) {  // the tile reaches past the first query's last key: mask per query
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int kabs = kt * 32 + 8 * (r >> 2) + 4 * hh + (r & 3);
                if (kabs > qpos) sacc[r] = -INFINITY;
            }
        }
        float mx = -INFINITY;
#pragma unroll
        for (int r = 0; r < 16; ++r) mx = fmaxf(mx, sacc[r]);
        mx = lane_max32_apart(mx);
        const float m_new = fmaxf(m_run, mx * kLog2e);
        const float ref = m_new > -INFINITY ? m_new : 0.f;  // (no key of this tile visible to the query, and none before)
        const float alpha = __builtin_amdgcn_exp2f(m_run - ref);
        float psum = 0.f, pr[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) { pr[r] = __builtin_amdgcn_exp2f(fmaf(sacc[r], kLog2e, -ref)); psum += pr[r]; }
        l_run = l_run * alpha + psum;
        if (__any(m_new != m_run)) {
#pragma unroll
            for (int i = 0; i < DB; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r) oacc[i][r] *= alpha;
        }
        m_run = m_new;
        asm volatile("" ::: "memory");  // (the wavefront's own LDS accesses stay in this order)
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2) {
            uint32_t ph[4], pl[4];
#pragma unroll
            for (int x = 0; x < 4; ++x) split2(pr[8 * s2 + 2 * x], pr[8 * s2 + 2 * x + 1], ph[x], pl[x]);
            const u32x4 phi = u32x4{ph[0], ph[1], ph[2], ph[3]}, plo = u32x4{pl[0], pl[1], pl[2], pl[3]};
            u32x4 vblk[DB];
#pragma unroll
            for (int i = 0; i < DB; ++i) {
                const half_t* vrow = &vt[wave][(i * 32 + j) * VPITCH + s2 * 16 + 4 * hh];
                const uint2 v0 = *reinterpret_cast<const uint2*>(vrow), v1 = *reinterpret_cast<const uint2*>(vrow + 8);
                vblk[i] = u32x4{v0.x, v0.y, v1.x, v1.y};
            }
#pragma unroll
            for (int i = 0; i < DB; ++i) oacc[i] = mfma_f16(vblk[i], plo, oacc[i]);
#pragma unroll
            for (int i = 0; i < DB; ++i) oacc[i] = mfma_f16(vblk[i], phi, oacc[i]);
        }
        asm volatile("" ::: "memory");
    }
    // the wavefronts' sums, each against the largest score of all
    const float l_tot = lane_sum32_apart(l_run);
    if (hh == 0) ml[wave][j] = make_float2(m_run, l_tot);
    __syncthreads();
    float2 e[WAVES];
    float all = -INFINITY, total = 0.f;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) { e[w] = ml[w][j]; all = fmaxf(all, e[w].x); }
    const float ref = all > -INFINITY ? all : 0.f;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) total = fmaf(e[w].y, __builtin_amdgcn_exp2f(e[w].x - ref), total);
    const float own = __builtin_amdgcn_exp2f(m_run - ref);
#pragma unroll
    for (int i = 0; i < DB; ++i) {
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[i][r] *= own;
        red[wave][i][lane] = oacc[i];
    }
    __syncthreads();
    if (!ok || wave >= DB) return;
    const float inv = total > 0.f ? 1.0f / total : 0.f;  // 0: a block of padding rows saw no tile
    const int m = b * S + t0 + j;
    f32x16 sum = red[0][wave][lane];
#pragma unroll
    for (int w = 1; w < WAVES; ++w) sum += red[w][wave][lane];
#pragma unroll
    for (int qd = 0; qd < 4; ++qd) {
        const int dim = h * D + wave * 32 + 8 * qd + 4 * hh;  // four consecutive output dimensions
        const size_t slot2 = block_slot(m, dim & ~7, H >> 4);
        reinterpret_cast<uint2*>(o + slot2)[(dim >> 2) & 1] =
            make_uint2(pack2(sum[qd * 4 + 0] * inv, sum[qd * 4 + 1] * inv), pack2(sum[qd * 4 + 2] * inv, sum[qd * 4 + 3] * inv));
    }
}

}  // namespace

// ------------------------------------------------------------------ launchers

// The form and the wavefronts of a (row, head).  The rule looks at the cache's size and not at how far it is filled: a captured
// step must add up like the eager one.  us of a layer's step (attention, GEMMs of a short FFN) with the cache three quarters full, both
// sides in turn on one engine, 256 CUs; a "row" is what a head caches of a sequence, in keys of 128 values (heads of 64: twice the keys):
//   Up to a pair per CU: one pass, as many wavefronts as one round over a full cache takes, at most eight.  (32 to 256 pairs, rows of 64 to 2048:
//   4 to 30 % less than two passes of 4 to 16.)
//   Up to two: at most four, but two passes of eight (the launch is the HBM stream then, and wants more of it requested) where nearly
//   every CU has two and the cache is long.  One pass of four / two passes of eight: 512 pairs, row 384 61.8 / 62.7, 512 64.6 / 64.3, 767 71.8 / 70.1, 1024 80.7 /
//   77.5, 1536 94.0 / 92.3; 480, row 512 62.5 / 63.6, 640 65.2 / 65.0, 1536 90.4 / 89.0; 448, 511 63.3 / 63.7, 767 68.9 / 67.2, 1000 73.5 / 72.8; 400, 768 79.5 / 79.8, 1280 91.4 /
//   90.7; 384, 768 65.1 / 65.4, 1024 72.3 / 70.9, 2048 93.0 / 91.8; 352, 1000 68.7 / 69.4, 1536 81.3 / 81.1; 320, 1280 73.0 / 74.3, 2048 87.6 / 88.9.  (Half
//   full: 512 pairs, row 512 +1.1, 1000 -0.1, 1536 -0.7, 2500 -2.0; one size stands out, 512 pairs and a row of 1999: +0.3 and +0.8 where full.)
//   More: one pass of two while the cache is short; four from 8 pairs per CU and a row of 128 on.  All three lie within 2 % of each other from rows of
//   112 to 192.  One pass of two / four / two passes of four: 640 pairs, row 112 61.7 / 61.9 / 62.5, 160 61.9 / 61.1 / 62.2, 192 63.6 / 63.8 / 64.3;
//   768, 136 63.0 / 62.1 / 62.4, 160 63.3 / 62.3 / 62.8, 192 65.6 / 66.2 / 65.2; 1280, 112 79.5 / 81.1 / 80.4, 160 83.3 / 83.0 / 82.9, 192 85.6 / 85.6 / 85.1; 1920,
//   112 97.8 / 99.3 / 99.5, 160 102.7 / 102.2 / 102.5; 2560, 112 110.3 / 110.0 / 111.4, 128 112.4 / 110.6 / 113.0, 160 117.1 / 115.7 / 116.4, 192 122.1 / 120.5 / 122.3; 3840, 112
//   137.5 / 138.5 / 139.9, 160 148.4 / 147.6 / 147.9; heads of 64, 1024 pairs, cache 224 41.2 / 42.4 / 42.0, 256 45.0 / 47.6 / 46.3, 320 45.0 / 44.7 / 44.8; 2048, 256 66.3 / 63.3 / 66.4,
//   384 71.8 / 70.8 / 71.0.  (Heads of 64 could go on to a row of 160, 320 of theirs, within that 2 %.)
struct AttnPlan { int form, waves; };  // form: HE_ATTN_ in he.h
static AttnPlan decode_attn_plan(long pairs, int max_seq, int d) {
    const long cus = plan_cus(), row = (long)max_seq * d;
    if (pairs > 2 * cus) {
        if (max_seq > (d == 128 ? 160 : 256)) return {HE_ATTN_TWO_PASSES, 4};
        return {HE_ATTN_ONE_PASS, pairs >= 8 * cus && row >= 128 * 128 ? 4 : 2};
    }
    if (8 * pairs >= 11 * cus && (pairs - cus) * row >= 512 * 128 * cus) return {HE_ATTN_TWO_PASSES, 8};
    const int keys_per_wave = 4 * 64 / (d / 8), most = pairs <= cus ? 8 : 4;  // of one round
    int waves = 2;
    while (waves < most && waves * keys_per_wave < max_seq) waves *= 2;
    return {HE_ATTN_ONE_PASS, waves};
}

template <int D>
static void launch_attn(hipStream_t s, const float* q, const void* kv, void* o_blocks, const he_dev_state* st, int M, int S, int layer,
                        int H, int n_heads, int max_batch, int max_seq, AttnPlan g, const bf16_ahead* ahead) {
    dim3 grid(M, n_heads);
    const half_t* c = (const half_t*)kv;
    u32x4* o = (u32x4*)o_blocks;
    if (g.form == HE_ATTN_TWO_PASSES) {
        const size_t shm = (size_t)max_seq * sizeof(float);
        if (g.waves == 8) attn_kernel<D, 8><<<grid, 512, shm, s>>>(q, c, o, st, S, layer, H, n_heads, max_batch, max_seq);
        else attn_kernel<D, 4><<<grid, 256, shm, s>>>(q, c, o, st, S, layer, H, n_heads, max_batch, max_seq);
        return;
    }
    bf16_ahead after;
    if (ahead && (size_t)M * n_heads * max_seq * D * 4 <= (size_t)32 << 20) after = *ahead;
    if (after.wgs) grid.y += (after.wgs + 7 + M - 1) / M;
    switch (g.waves) {
        case 8: attn_few_kernel<D, 8><<<grid, 512, 0, s>>>(q, c, o, st, S, layer, H, n_heads, max_batch, max_seq, after); break;
        case 4: attn_few_kernel<D, 4><<<grid, 256, 0, s>>>(q, c, o, st, S, layer, H, n_heads, max_batch, max_seq, after); break;
        default: attn_few_kernel<D, 2><<<grid, 128, 0, s>>>(q, c, o, st, S, layer, H, n_heads, max_batch, max_seq, after);
    }
}

// Prompt rows whose workgroups of 128 queries occupy half of the CUs or fewer, with more than one block of keys to share out: 32 queries
// to a workgroup, as long as these do not come in rounds that cost more than a longer block does.  Heads of 128 leave room for one of
// them to a CU (LDS), heads of 64 for three.  `blocks`: workgroups of an XCD, which takes every eighth (sequence, head) pair whole.  us a
// launch, 128 queries to a workgroup -> 32, 256 CUs.  Heads of 128, one round: 96 queries x 64 pairs 10.9 -> 10.9, 250 x 32 17.9 -> 13.7, 1500 x 5 66.6 ->
// 33.3; up to two: 96 x 96 11.1 -> 16.7, 192 x 48 14.4 -> 17.2, 250 x 48 18.0 -> 20.0, 320 x 40 20.0 -> 22.3, but of four pairs to an XCD 320 x 32
// 17.7 -> 16.8, 500 x 32 28.4 -> 25.6, 1000 x 16 48.4 -> 34.1; beyond: 384 x 42 23.4 -> 30.0, 640 x 25 33.4 -> 36.4, but of three pairs to an XCD
// 765 x 20 38.4 -> 36.9, 829 x 18 39.3 -> 41.0, 2000 x 8 86.7 -> 49.2.  Heads of 64, more than a round, difference: 65 queries +0.4, 96 +0.9,
// 112 x 80 and 128 pairs -0.7 and -0.1, 128 +0.1, 160 0.0, 192 -0.8, 250 -2.4, 500 -6.8.
static bool prompt_splits(int pairs, int S, int d) {
    const long cus = plan_cus(), per_xcd = (pairs + 7) / 8, blocks = (S + 31) / 32 * per_xcd, round = cus / 8;
    if (S <= 64 || (long)((S + 127) / 128) * pairs * 2 > cus) return false;
    if (blocks <= round) return true;
    return d == 128 ? per_xcd <= 3 || (per_xcd == 4 && blocks <= 2 * round) : S > 96;
}

// The kernel that M rows of S per sequence take and the wavefronts of its workgroups.
static AttnPlan attn_plan(int M, int S, int n_heads, int d, int max_seq) {
    if (S >= 32) return {prompt_splits(M / S * n_heads, S, d) ? HE_ATTN_PROMPT_SPLIT : HE_ATTN_PROMPT, 4};
    if (S >= QB && (size_t)QB * max_seq * sizeof(float) <= 96 * 1024) return {HE_ATTN_SHORT_PROMPT, 4};
    return decode_attn_plan((long)M * n_heads, max_seq, d);
}

void bf16_attn_plan_query(int M, int S, int n_heads, int d, int max_seq, int cus, int* form, int* waves) {
    plan_cus_override = cus;
    const AttnPlan g = attn_plan(M, S, n_heads, d, max_seq);
    plan_cus_override = 0;
    *form = g.form;
    *waves = g.waves;
}

void bf16_attn(hipStream_t s, const float* q, const void* kv, void* o_blocks, const he_dev_state* st, int M, int S, int layer, int H, int n_heads, int max_batch, int max_seq,
               const bf16_ahead* ahead) {
    const half_t* c = (const half_t*)kv;
    u32x4* o = (u32x4*)o_blocks;
    const int d = H / n_heads, batch = M / S;
    const unsigned pairs8 = (unsigned)((batch * n_heads + 7) / 8) * 8;
    const AttnPlan g = attn_plan(M, S, n_heads, d, max_seq);
    if (g.form == HE_ATTN_PROMPT_SPLIT) {
        const unsigned grid = (unsigned)((S + 31) / 32) * pairs8;
        if (d == 128) attn_prompt_split_kernel<128><<<grid, 256, 0, s>>>(q, c, o, st, S, layer, H, n_heads, max_batch, max_seq, batch);
        else attn_prompt_split_kernel<64><<<grid, 256, 0, s>>>(q, c, o, st, S, layer, H, n_heads, max_batch, max_seq, batch);
    } else if (g.form == HE_ATTN_PROMPT) {  // 32 queries per wavefront on the matrix cores
        const unsigned grid = (unsigned)((S + 127) / 128) * pairs8;
        if (d == 128) attn_prompt_mfma_kernel<128><<<grid, 256, 0, s>>>(q, c, o, st, S, layer, H, n_heads, max_batch, max_seq, batch);
        else attn_prompt_mfma_kernel<64><<<grid, 256, 0, s>>>(q, c, o, st, S, layer, H, n_heads, max_batch, max_seq, batch);
    } else if (g.form == HE_ATTN_SHORT_PROMPT) {  // blocks of QB queries per workgroup
        const size_t shm = (size_t)QB * max_seq * sizeof(float);
        const dim3 grid((S + QB - 1) / QB, n_heads, batch);
        if (d == 128) attn_prompt_kernel<128><<<grid, 256, shm, s>>>(q, c, o, st, S, layer, H, n_heads, max_batch, max_seq);
        else attn_prompt_kernel<64><<<grid, 256, shm, s>>>(q, c, o, st, S, layer, H, n_heads, max_batch, max_seq);
    } else {
        if (d == 128) launch_attn<128>(s, q, kv, o_blocks, st, M, S, layer, H, n_heads, max_batch, max_seq, g, ahead);
        else launch_attn<64>(s, q, kv, o_blocks, st, M, S, layer, H, n_heads, max_batch, max_seq, g, ahead);
    }
}
