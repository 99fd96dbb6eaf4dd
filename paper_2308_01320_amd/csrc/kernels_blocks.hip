// Decode steps of small float models: an attention block and an FFN block per layer, a launch each.
//
// A step of a small model is nothing but launches: five a layer, 3.3 to 4.4 us each for a microsecond's work.  Here a workgroup
// takes a whole head of a row (LayerNorm, its queries, keys and values, attention, and the head's share of the out-projection), or
// 32 columns of the FFN's width (LayerNorm, FC1, and their share of FC2).  The shares are partial sums of the residual rows;
// whoever reads the rows next adds them up, in order, with the bias, the row itself last (each of the others rounds at the sums' size, not
// the row's): no hand-off inside a launch, none left over.  What the blocks
// pay is work done more than once -- a row's sum and LayerNorm per head or slice, a head's weights per row -- so they are for models
// a head of which one CU reads in two or three microseconds (plain_blocks_fit).  Weights and cached keys are requested behind the row
// (loads return in order) and before anything that has to be waited for; sums over lanes are data-parallel moves; the products of an
// FFN block are float matrix instructions, those of a single row are not (fifteen of sixteen rows would be padding).
//
// A generation of 16 tokens, two layers of width 256, FFN 1024, 1024 ids, prompts of 32, us, a launch per matrix -> this: 1 row 836 -> 657, 4
// rows 910 -> 695, 16 rows 1022 -> 867; width 192, FFN 768, 16 rows 940 -> 730; width 128, FFN 512, 4 rows 802 -> 608.  A launch here is
// 5 to 8 us, bound by what one CU reads (260 KB of weights for a head of 64 at width 256) and the chain behind it.  (FFN slices of 64 columns:
// 8.5 us against 6; attention blocks of four or sixteen wavefronts: 738 and 745 us where eight take 695.)
// Long caches gain as well, a step of two layers, a launch per matrix -> this: width 256, 4 rows, 512 keys 60 -> 48 us, 4096 keys 153 -> 129, 8000
// keys 257 -> 216; 1 row, 8000 keys 248 -> 205; 16 rows, 4096 keys 194 -> 172; width 128, 1 row, 4096 keys 128 -> 101.
// Error against 64 bits, twelve models of width 128 to 256, a launch per matrix -> this: logits 2.45e-7 -> 2.40e-7, log-probabilities 7.7e-8 both.
#include "he_common.h"
#include "kernels.h"

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr int kBlockThreads = 512, kBlockWaves = 8, kAttnWaves = 8;
constexpr int kMaxWidth = 256, kMaxRows = 16, kMaxHead = 64, kSlice = 32, kMaxHeads = 8, kMaxSlices = 32;

__device__ __forceinline__ f32x4 ldv(const float* p) { return *reinterpret_cast<const f32x4*>(p); }
__device__ __forceinline__ float dot4(const f32x4& a, const f32x4& b, float c) {
    return fmaf(a[3], b[3], fmaf(a[2], b[2], fmaf(a[1], b[1], fmaf(a[0], b[0], c))));
}
__device__ __forceinline__ float sum4(const f32x4& v) { return (v[0] + v[1]) + (v[2] + v[3]); }

// a lane's four values of a row of H (H <= 256: lane l holds 4 l ..) -> normalised; lanes past the row hold zeros
__device__ __forceinline__ f32x4 norm_row(const f32x4& x, int H, int lane, float eps, const f32x4& g, const f32x4& b) {
    const float mean = lane_sum<64>(sum4(x)) / H;
    f32x4 d = x - mean;
    if (4 * lane >= H) d = f32x4{0.f, 0.f, 0.f, 0.f};
    const float rstd = 1.0f / sqrtf(lane_sum<64>(sum4(d * d)) / H + eps);
    return d * rstd * g + b;
}

// One workgroup per (row, head).  Sixteen lanes share a row of weights or a key.
template <bool EMBED>
__global__ __launch_bounds__(64 * kAttnWaves) void attn_block_kernel(const float* __restrict__ wqkv, const float* __restrict__ wo,
                                                                   const float* __restrict__ x, const float* __restrict__ part,
                                                                   float* __restrict__ kv, he_dev_state* __restrict__ st, plain_block_args a) {
    constexpr int NK = kMaxWidth / 64, ROWS = 4 * kAttnWaves, NQ = 3 * kMaxHead / ROWS, NO = kMaxWidth / ROWS, U = 64 / ROWS;
    __shared__ __align__(16) float red[kAttnWaves][kMaxWidth], xs[kMaxWidth], qkv[3 * kMaxHead];
    __shared__ float2 ml[kAttnWaves];
    __shared__ f32x4 ored[kAttnWaves][16];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, l16 = lane & 15, grp = lane >> 4;
    const int m = blockIdx.x, h = blockIdx.y, B = gridDim.x, H = a.H, d = H / a.n_heads;
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    if (EMBED && m == 0 && h == 0 && threadIdx.x == 0) store_sampling(st, a.sp);
    const bool in = 4 * lane < H;
    const int len = seq_len(st, m) - row_pad(st, m);  // cached positions
    // the row: embedding, or residual row + bias + the FFN slices' shares
    f32x4 xv = zero, gv = zero, bv = zero, first = zero;
    if (EMBED) {
        int id = a.ids[(size_t)m * a.id_stride];
        id = id < 0 ? 0 : (id >= a.V ? a.V - 1 : id);  // out-of-range ids are clamped, never read out of bounds
        if (in) xv = ldv(a.tok + (size_t)id * H + 4 * lane) + ldv(a.pos + (size_t)(len + a.pos_offset) * H + 4 * lane);
    } else if (in) {
        f32x4 pb = zero;
        if (wave == 0) { xv = ldv(x + (size_t)m * H + 4 * lane); pb = ldv(a.pbias + 4 * lane); }
        f32x4 p[kMaxSlices / kAttnWaves];
#pragma unroll
        for (int i = 0; i < kMaxSlices / kAttnWaves; ++i) {
            const int s = wave + i * kAttnWaves;
            p[i] = s < a.n_part ? ldv(part + ((size_t)s * B + m) * H + 4 * lane) : zero;
        }
#pragma unroll
        for (int i = 0; i < kMaxSlices / kAttnWaves; ++i) pb += p[i];
        if (wave) xv = pb;
        else first = pb;
    }
    if (in) { gv = ldv(a.gamma + 4 * lane); bv = ldv(a.beta + 4 * lane); }
    // weights and cached keys and values
    const int row0 = wave * 4 + grp;
    f32x4 w[NQ][NK], ow[NO], kr[U], vr[U];
    float bias[NQ];
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
        const int r = row0 + ROWS * i, which = (r >= d) + (r >= 2 * d), n = which * H + h * d + r - which * d;
        bias[i] = r < 3 * d ? a.bqkv[n] : 0.f;
#pragma unroll
        for (int k = 0; k < NK; ++k) w[i][k] = r < 3 * d && 64 * k + 4 * l16 < H ? ldv(wqkv + (size_t)n * H + 64 * k + 4 * l16) : zero;
    }
    const float* Kp = kv + kv_index(a.layer, 0, m, h, 0, a.max_batch, a.n_heads, a.max_seq, d);
    const float* Vp = kv + kv_index(a.layer, 1, m, h, 0, a.max_batch, a.n_heads, a.max_seq, d);
    const bool dim = 4 * l16 < d;
    auto load_keys = [&](int base) {  // (past the cached ones: some row of the cache, not used)
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const size_t at = (size_t)min(base + u * ROWS + row0, a.max_seq - 1) * d + 4 * l16;
            kr[u] = dim ? ldv(Kp + at) : zero;
            vr[u] = dim ? ldv(Vp + at) : zero;
        }
    };
    load_keys(0);
#pragma unroll
    for (int i = 0; i < NO; ++i) ow[i] = row0 + ROWS * i < H && dim ? ldv(wo + (size_t)(row0 + ROWS * i) * H + h * d + 4 * l16) : zero;
    if (!EMBED) {
        if (wave) *reinterpret_cast<f32x4*>(&red[wave][4 * lane]) = xv;
        __syncthreads();
        if (wave == 0) {
#pragma unroll
            for (int i = 1; i < kAttnWaves; ++i) first += ldv(&red[i][4 * lane]);
            xv += first;
        }
    }
    if (wave == 0) {
        *reinterpret_cast<f32x4*>(xs + 4 * lane) = norm_row(xv, H, lane, a.eps, gv, bv);  // (zeros past the row)
        if (h == 0 && in) *reinterpret_cast<f32x4*>(a.x_out + (size_t)m * H + 4 * lane) = xv;
    }
    __syncthreads();
    f32x4 xk[NK];
#pragma unroll
    for (int k = 0; k < NK; ++k) xk[k] = ldv(xs + 64 * k + 4 * l16);
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
        float s = 0.f;
#pragma unroll
        for (int k = 0; k < NK; ++k) s = dot4(w[i][k], xk[k], s);
        s = lane_sum<16>(s) + bias[i];
        const int r = row0 + ROWS * i;
        if (l16 == 0 && r < 3 * d) qkv[r] = r < d ? s * a.qscale : s;
    }
    __syncthreads();
    if ((int)threadIdx.x < d / 2) {  // the new key, then the new value, into the cache
        const int which = (int)threadIdx.x >= d / 4, c = 4 * ((int)threadIdx.x - which * (d / 4));
        const float* src = qkv + (1 + which) * d + c;
        float* dst = kv + kv_index(a.layer, which, m, h, len, a.max_batch, a.n_heads, a.max_seq, d) + c;
        *reinterpret_cast<f32x4*>(dst) = f32x4{src[0], src[1], src[2], src[3]};
    }
    const bool done = seq_done(st, m);  // (nothing reads this row's output)
    f32x4 qv = zero, kn = zero, vn = zero, acc = zero;
    if (dim) {
#pragma unroll
        for (int e = 0; e < 4; ++e) { qv[e] = qkv[4 * l16 + e]; kn[e] = qkv[d + 4 * l16 + e]; vn[e] = qkv[2 * d + 4 * l16 + e]; }
    }
    float mx = -INFINITY, sum = 0.f;
    for (int base = 0; base <= len && !done; base += U * ROWS) {
        if (base) load_keys(base);
        float s[U], top = mx;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int j = base + u * ROWS + row0;
            if (j == len) { kr[u] = kn; vr[u] = vn; }
            if (j > len) vr[u] = zero;
            const float v = lane_sum<16>(dot4(qv, kr[u], 0.f));
            s[u] = j <= len ? v : -INFINITY;
            top = fmaxf(top, s[u]);
        }
        // (nothing above -inf yet: the state stays what it is)
        const float ref = top > -INFINITY ? top : 0.f, keep = expf(mx - ref);
        mx = top;
        sum *= keep;
        acc *= keep;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const float pr = base + u * ROWS + row0 <= len ? expf(s[u] - ref) : 0.f;
            sum += pr;
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[e] = fmaf(pr, vr[u][e], acc[e]);
        }
    }
    // the lane groups of a wavefront, then the wavefronts
    const float wmx = lane_max32_apart(lane_max16_apart(mx)), own = mx > -INFINITY ? expf(mx - wmx) : 0.f;
    sum = lane_sum_apart<16>(sum * own);
    if (lane == 0) ml[wave] = make_float2(wmx, sum);
    f32x4 t;
#pragma unroll
    for (int e = 0; e < 4; ++e) t[e] = lane_sum_apart<16>(acc[e] * own);
    if (grp == 0) ored[wave][l16] = t;
    __syncthreads();
    float all = -INFINITY, total = 0.f;
#pragma unroll
    for (int i = 0; i < kAttnWaves; ++i) all = fmaxf(all, ml[i].x);
    f32x4 o = zero;
#pragma unroll
    for (int i = 0; i < kAttnWaves; ++i) {
        const float2 e = ml[i];
        const float f = e.x > -INFINITY ? expf(e.x - all) : 0.f;
        total += e.x > -INFINITY ? e.y * f : 0.f;
        o += ored[i][l16] * f;
    }
    o = done ? zero : o / total;
    float* out = a.part_out + ((size_t)h * B + m) * H;
#pragma unroll
    for (int i = 0; i < NO; ++i) {
        const float s = lane_sum<16>(dot4(ow[i], o, 0.f));
        if (l16 == 0 && row0 + ROWS * i < H) out[row0 + ROWS * i] = s;
    }
}

// Residual rows x + bias + the n partial sums of each, normalised, into LDS: xs[row][..].  Two threads share a quad of values where
// there are threads for that.  raw: where the rows themselves go (null: nowhere).  What a thread needs of its first quad comes from
// request_rows, ahead of the weights: loads return in order.
constexpr int kLdsRow = kMaxWidth + 4;
struct BlockRows { float xs[kMaxRows][kLdsRow], half[2][kMaxRows][kLdsRow]; };
template <int NP> struct RowRequest { f32x4 x, bias, part[NP]; };
__device__ __forceinline__ bool rows_by_two(int B, int H) { return 2 * B * (H / 4) <= kBlockThreads; }
template <int NP>
__device__ __forceinline__ void request_quad(RowRequest<NP>& q, const float* x, const float* part, int n, const float* bias, int B, int H, int e,
                                             bool two, int second) {
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    const int m = e / (H / 4), c = 4 * (e - m * (H / 4));
    const bool live = m < B;
    const float* p = part + (size_t)m * H + c;
    q.x = q.bias = zero;
    if (live && !second) { q.x = ldv(x + (size_t)m * H + c); q.bias = ldv(bias + c); }
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        const int s = two ? second + 2 * i : i;
        q.part[i] = live && s < n ? ldv(p + (size_t)s * B * H) : zero;
    }
}
template <int NP>
__device__ __forceinline__ void request_rows(RowRequest<NP>& q, const float* x, const float* part, int n, const float* bias, int B, int H) {
    const bool two = rows_by_two(B, H);
    const int second = two && (int)threadIdx.x >= kBlockThreads / 2;
    request_quad(q, x, part, n, bias, B, H, threadIdx.x - second * (kBlockThreads / 2), two, second);
}
// (ends with a barrier)
template <int NP>
__device__ __forceinline__ void block_rows(BlockRows& L, RowRequest<NP>& q, const float* x, const float* part, int n, const float* bias, int B,
                                           int H, float eps, const float* gamma, const float* beta, float* raw, int wave, int lane) {
    const int quads = B * (H / 4), c4 = H / 4;
    const bool two = rows_by_two(B, H);
    const int second = two && (int)threadIdx.x >= kBlockThreads / 2;
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    f32x4 g = zero, b = zero;
    if (4 * lane < H) { g = ldv(gamma + 4 * lane); b = ldv(beta + 4 * lane); }
    for (int e = threadIdx.x - second * (kBlockThreads / 2); e < quads; e += kBlockThreads) {
        if (e >= kBlockThreads) request_quad(q, x, part, n, bias, B, H, e, two, second);
        const int m = e / c4, c = 4 * (e - m * c4);
        f32x4 v = q.bias;
#pragma unroll
        for (int i = 0; i < NP; ++i) v += q.part[i];
        if (two) *reinterpret_cast<f32x4*>(L.half[second][m] + c) = v;
        if (!second) *reinterpret_cast<f32x4*>(L.xs[m] + c) = two ? q.x : q.x + v;
    }
    __syncthreads();
    for (int m = wave; m < B; m += kBlockWaves) {
        f32x4 v = zero;
        if (4 * lane < H) {
            v = ldv(L.xs[m] + 4 * lane);
            if (two) v += ldv(L.half[0][m] + 4 * lane) + ldv(L.half[1][m] + 4 * lane);
            if (raw) *reinterpret_cast<f32x4*>(raw + (size_t)m * H + 4 * lane) = v;
        }
        const f32x4 nv = norm_row(v, H, lane, eps, g, b);
        if (4 * lane < H) *reinterpret_cast<f32x4*>(L.xs[m] + 4 * lane) = nv;
    }
    __syncthreads();
}

__device__ __forceinline__ f32x4 mma4(const f32x4& w, const f32x4& x, f32x4 c) {
#pragma unroll
    for (int e = 0; e < 4; ++e) c = __builtin_amdgcn_mfma_f32_16x16x4f32(w[e], x[e], c, 0, 0, 0);
    return c;
}

// One workgroup per 32 columns of the FFN's width, all rows.  Lane l of a product holds row l % 16, columns 4 (l / 16) .. + 3.
__global__ __launch_bounds__(kBlockThreads) void ffn_block_kernel(const float* __restrict__ w1, const float* __restrict__ w2,
                                                                  const float* __restrict__ x, const float* __restrict__ part,
                                                                  const float* __restrict__ b1, plain_block_args a, int B, int F) {
    constexpr int T1 = kSlice / 16, KW = kBlockWaves / T1, S1 = kMaxWidth / 16 / KW, S2 = kSlice / 16, T2 = kMaxWidth / 16 / kBlockWaves;
    __shared__ __align__(16) BlockRows L;
    __shared__ __align__(16) float hs[kMaxRows][kSlice + 4];
    __shared__ f32x4 red[KW][T1][64];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, l16 = lane & 15, kq = 4 * (lane >> 4);
    const int slice = blockIdx.x, H = a.H, tile = wave % T1, kw = wave / T1;
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    RowRequest<kMaxHeads> q;
    request_rows(q, x, part, a.n_part, a.pbias, B, H);
    // FC1: tiles of 16 columns, KW wavefronts to each, every KW-th step of 16 k to a wavefront (S1 at most); FC2: tiles of 16 columns, a wavefront each
    f32x4 wa[S1], wb[T2][S2];
    const float* r1 = w1 + (size_t)(slice * kSlice + tile * 16 + l16) * H + kq;
#pragma unroll
    for (int i = 0; i < S1; ++i) wa[i] = 16 * (kw + i * KW) < H ? ldv(r1 + 16 * (kw + i * KW)) : zero;
    const f32x4 bias = ldv(b1 + slice * kSlice + tile * 16 + kq);
#pragma unroll
    for (int t = 0; t < T2; ++t) {
        const int n = (wave + t * kBlockWaves) * 16;
#pragma unroll
        for (int i = 0; i < S2; ++i) wb[t][i] = n < H ? ldv(w2 + (size_t)(n + l16) * F + slice * kSlice + 16 * i + kq) : zero;
    }
    block_rows<kMaxHeads>(L, q, x, part, a.n_part, a.pbias, B, H, a.eps, a.gamma, a.beta, slice == 0 ? a.x_out : nullptr, wave, lane);
    const int m = min(l16, B - 1);  // (rows past the batch: its last one, never stored)
    f32x4 acc = zero;
#pragma unroll
    for (int i = 0; i < S1; ++i)
        if (16 * (kw + i * KW) < H) acc = mma4(wa[i], ldv(&L.xs[m][16 * (kw + i * KW) + kq]), acc);
    red[kw][tile][lane] = acc;
    __syncthreads();
    if (kw == 0) {
        acc = bias;
#pragma unroll
        for (int i = 0; i < KW; ++i) acc += red[i][tile][lane];
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] = fmaxf(acc[e], 0.f);
        *reinterpret_cast<f32x4*>(&hs[l16][tile * 16 + kq]) = acc;
    }
    __syncthreads();
    f32x4 hv[S2];
#pragma unroll
    for (int i = 0; i < S2; ++i) hv[i] = ldv(&hs[l16][16 * i + kq]);
#pragma unroll
    for (int t = 0; t < T2; ++t) {
        const int n = (wave + t * kBlockWaves) * 16;
        f32x4 v = zero;
#pragma unroll
        for (int i = 0; i < S2; ++i) v = mma4(wb[t][i], hv[i], v);
        if (n < H && l16 < B) *reinterpret_cast<f32x4*>(a.part_out + ((size_t)slice * B + l16) * H + n + kq) = v;
    }
}

// One workgroup per 16 vocabulary entries, all rows, k split over the wavefronts.
__global__ __launch_bounds__(kBlockThreads) void head_block_kernel(const float* __restrict__ w, const float* __restrict__ x,
                                                                   const float* __restrict__ part, float* __restrict__ logits,
                                                                   plain_block_args a, int B, int vec_out) {
    constexpr int S = kMaxWidth / 16 / kBlockWaves;
    __shared__ __align__(16) BlockRows L;
    __shared__ f32x4 red[kBlockWaves][64];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, l16 = lane & 15, kq = 4 * (lane >> 4);
    const int H = a.H, n0 = blockIdx.x * 16;
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    RowRequest<kMaxSlices> q;
    request_rows(q, x, part, a.n_part, a.pbias, B, H);
    f32x4 wv[S];
#pragma unroll
    for (int i = 0; i < S; ++i) {  // entries past the vocabulary: its last one, never stored
        const int k = 16 * (wave + i * kBlockWaves);
        wv[i] = k < H ? ldv(w + (size_t)min(n0 + l16, a.V - 1) * H + k + kq) : zero;
    }
    block_rows<kMaxSlices>(L, q, x, part, a.n_part, a.pbias, B, H, a.eps, a.gamma, a.beta, nullptr, wave, lane);
    const int m = min(l16, B - 1);
    f32x4 acc = zero;
#pragma unroll
    for (int i = 0; i < S; ++i)
        if (16 * (wave + i * kBlockWaves) < H) acc = mma4(wv[i], ldv(&L.xs[m][16 * (wave + i * kBlockWaves) + kq]), acc);
    red[wave][lane] = acc;
    __syncthreads();
    if (wave != 0 || l16 >= B) return;
    f32x4 v = zero;
#pragma unroll
    for (int i = 0; i < kBlockWaves; ++i) v += red[i][lane];
    const int n = n0 + kq;
    float* dst = logits + (size_t)l16 * a.V + n;
    if (vec_out && n + 4 <= a.V) *reinterpret_cast<f32x4*>(dst) = v;
    else
        for (int e = 0; e < 4; ++e)
            if (n + e < a.V) dst[e] = v[e];
}

}  // namespace

// ------------------------------------------------------------------ launchers

// A head's weights are 16 H d bytes, read once per row; an FFN slice's 256 H.  part_heads, part_slices: floats the two sets of partial
// sums can hold.
bool plain_blocks_fit(int B, int H, int n_heads, int F, size_t part_heads, size_t part_slices) {
    return H % 16 == 0 && H <= kMaxWidth && H / n_heads <= kMaxHead && n_heads <= kMaxHeads && F % kSlice == 0 && F / kSlice <= kMaxSlices &&
           B <= kMaxRows && (size_t)n_heads * B * H <= part_heads && (size_t)(F / kSlice) * B * H <= part_slices;
}

void plain_attn_block(hipStream_t s, bool embed, const float* wqkv, const float* wo, const float* x, const float* part, float* kv, he_dev_state* st,
                      int B, const plain_block_args& a) {
    const dim3 grid(B, a.n_heads);
    if (embed) attn_block_kernel<true><<<grid, 64 * kAttnWaves, 0, s>>>(wqkv, wo, x, part, kv, st, a);
    else attn_block_kernel<false><<<grid, 64 * kAttnWaves, 0, s>>>(wqkv, wo, x, part, kv, st, a);
}

int plain_ffn_slices(int F) { return F / kSlice; }

void plain_ffn_block(hipStream_t s, const float* w1, const float* w2, const float* x, const float* part, const float* b1, int B, int F,
                     const plain_block_args& a) {
    ffn_block_kernel<<<F / kSlice, kBlockThreads, 0, s>>>(w1, w2, x, part, b1, a, B, F);
}

void plain_head_block(hipStream_t s, const float* w, const float* x, const float* part, float* logits, int B, const plain_block_args& a) {
    head_block_kernel<<<(a.V + 15) / 16, kBlockThreads, 0, s>>>(w, x, part, logits, a, B, a.V % 4 == 0 && (uintptr_t)logits % 16 == 0);
}
