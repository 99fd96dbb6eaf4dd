// Plain kernels: the f32 path of the engine (and, instantiated for bf16 storage,
// a slow comparator for the tuned bf16 kernels).  One obvious kernel per step of
// the decoder; activations are float, row-major [rows, features].
#include "he_common.h"
#include "../../include/he.h"
#include "kernels.h"

namespace {

constexpr int kThreads = 256;
typedef float f32x4 __attribute__((ext_vector_type(4)));

// four consecutive values, aligned
__device__ __forceinline__ f32x4 load4(const float* p) { return *reinterpret_cast<const f32x4*>(p); }
__device__ __forceinline__ f32x4 load4(const bf16_t* p) {
    const uint2 w = *reinterpret_cast<const uint2*>(p);
    return f32x4{__uint_as_float(w.x << 16), __uint_as_float(w.x & 0xFFFF0000u), __uint_as_float(w.y << 16), __uint_as_float(w.y & 0xFFFF0000u)};
}
// the caller's tables and vectors may start anywhere
template <typename ST>
bool aligned4(const void* q) { return (uintptr_t)q % (4 * sizeof(ST)) == 0; }

__device__ __forceinline__ float block_sum(float v, float* red) {
    v = lane_sum<64>(v);
    const int w = threadIdx.x >> 6, nw = blockDim.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[w] = v;
    __syncthreads();
    float t = 0.f;
    for (int i = 0; i < nw; ++i) t += red[i];
    return t;
}

// Row m = b*S + t:  x[m,:] = tok_emb[ids[b*id_stride + t],:] + pos_emb[cur_len + t + pos_offset,:]
// VEC: H is a multiple of four and the tables are aligned for four values at a time (96 rows of 5120: 11.2 -> 6.8 us).
template <typename ST, bool VEC>
__global__ __launch_bounds__(256) void embed_kernel(const int32_t* __restrict__ ids, int id_stride, const ST* __restrict__ tok,
                                                    const ST* __restrict__ pos, float* __restrict__ x, he_dev_state* __restrict__ st,
                                                    int S, int H, int V, int pos_offset, he_step_sampling sp) {
    if (blockIdx.x == 0 && threadIdx.x == 0) store_sampling(st, sp);
    const int m = blockIdx.x, b = sp.start ? m / S : row_seq(st, m, S), t = m % S - (sp.start ? 0 : row_pad(st, b));
    const bool token = t >= 0;  // else a padding row: zeros, nothing downstream uses it
    int id = ids[(size_t)b * id_stride + (m % S)];
    id = id < 0 ? 0 : (id >= V ? V - 1 : id);  // out-of-range ids are clamped, never read out of bounds
    const size_t p = token ? (size_t)((sp.start ? 0 : seq_len(st, b)) + t + pos_offset) : 0;
    if (VEC) {
        for (int i = threadIdx.x * 4; i < H; i += blockDim.x * 4) {
            f32x4 v = {0.f, 0.f, 0.f, 0.f};
            if (token) v = load4(tok + (size_t)id * H + i) + load4(pos + p * H + i);
            *reinterpret_cast<f32x4*>(x + (size_t)m * H + i) = v;
        }
    } else {
        for (int i = threadIdx.x; i < H; i += blockDim.x)
            x[(size_t)m * H + i] = token ? ld_f32(tok, (size_t)id * H + i) + ld_f32(pos, p * H + i) : 0.f;
    }
}

// a[m,:] = LayerNorm of row m*in_mul + in_add of the residual stream.  (Many rows; a few are normalised inside the GEMM.)
template <typename ST>
__global__ void ln_kernel(const float* __restrict__ r, const ST* __restrict__ gamma, const ST* __restrict__ beta,
                          float* __restrict__ a, int H, float eps, int in_mul, int in_add) {
    __shared__ float red[8];
    const int m = blockIdx.x;
    const float* rr = r + ((size_t)m * in_mul + in_add) * H;
    float s = 0.f;
    for (int i = threadIdx.x; i < H; i += blockDim.x) s += rr[i];
    const float mean = block_sum(s, red) / H;
    float q = 0.f;
    for (int i = threadIdx.x; i < H; i += blockDim.x) {
        const float dlt = rr[i] - mean;
        q += dlt * dlt;
    }
    const float rstd = 1.0f / sqrtf(block_sum(q, red) / H + eps);
    for (int i = threadIdx.x; i < H; i += blockDim.x)
        a[(size_t)m * H + i] = (rr[i] - mean) * rstd * ld_f32(gamma, i) + ld_f32(beta, i);
}

// ----------------------------------------------------------------- GEMM
//
// C[m,n] = sum_k A[m,k] W[n,k] in float on the matrix cores (16x16x4: 4 KFLOP per wavefront and four k, float operands and
// accumulators).  A wavefront holds T x T tiles of 16 x 16; lane l loads W[n0 + l%16][k .. k+3] and A[m0 + l%16][k .. k+3], k = 16 step + 4 (l/16),
// 16 bytes each, and instruction i of a step multiplies element i of both: the four lane groups' k values differ, but
// by the same rule on both sides.  No LDS staging: the models of this path are small and their rows come out of L2.
// What bounds it is the length of the dependent chain -- a launch, a load or two, a few matrix instructions -- so the k
// range is split over the wavefronts of a workgroup (partial sums added in wavefront order through LDS) and the few rows
// of a decode step go 16 columns to a workgroup.
//   few rows (at most 64, 256   gemm_few_kernel: 16 columns x 16 rows per workgroup, LayerNorm of the rows folded in (plain_gemm_form)
//   of small matrices):
//   many tiles (from 256 on):   KW = 1: 64 x 64 per workgroup of four wavefronts
//   else:                       KW = 8: 32 x 32 per workgroup
// VEC: K is a multiple of four and the rows are aligned for 16-byte loads (8-byte ones for bf16 storage).
template <bool VEC, typename ST>
__device__ __forceinline__ f32x4 load_k4(const ST* row, int k, int K) {
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if (VEC) {
        if (k < K) v = load4(row + k);
        return v;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (k + i < K) v[i] = ld_f32(row, k + i);
    return v;
}

struct PlainGemm {
    int M, N, K, epi;
    float* out;
    float* kv;
    const he_dev_state* st;
    int S, layer, H, n_heads, max_batch, max_seq;
    float qscale;
    float eps;           // folded LayerNorm: row m of A is row m*in_mul + in_add of the residual stream, not normalised
    int in_mul, in_add;
    int vec_out;         // four consecutive outputs may be stored at once
};

template <typename ST>
__device__ __forceinline__ void plain_epilogue4(const PlainGemm& p, const ST* __restrict__ bias, int m, int n0, f32x4 v) {
    if (m >= p.M) return;
    const int nv = min(4, p.N - n0);
    if (p.epi != EPI_STORE)
        for (int i = 0; i < nv; ++i) v[i] += ld_f32(bias, n0 + i);
    float* dst = p.out + (size_t)m * p.N + n0;
    if (p.epi == EPI_BIAS_RELU) {
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = fmaxf(v[i], 0.f);
    } else if (p.epi == EPI_RESID) {
        for (int i = 0; i < nv; ++i) v[i] = dst[i] + v[i];
    } else if (p.epi == EPI_QKV) {  // q scaled to `out`, k and v appended to the cache (H and the head dimension are multiples of 8)
        const int d = p.H / p.n_heads;
        if (n0 < p.H) {
            dst = p.out + (size_t)m * p.H + n0;
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] *= p.qscale;
        } else if (n0 < p.N) {
            const int which = n0 >= 2 * p.H, c = n0 - (which ? 2 * p.H : p.H);
            const int b = row_seq(p.st, m, p.S), tr = m % p.S - row_pad(p.st, b);
            if (tr < 0) return;  // padding rows append nothing
            dst = p.kv + kv_index(p.layer, which, b, c / d, seq_len(p.st, b) + tr, p.max_batch, p.n_heads, p.max_seq, d) + (c % d);
        }
    }
    if (p.vec_out && nv == 4) {
        *reinterpret_cast<f32x4*>(dst) = v;
    } else {
        for (int i = 0; i < nv; ++i) dst[i] = v[i];
    }
}

template <typename ST, int KW, int WN, int WM, bool VEC>
__global__ __launch_bounds__(64 * KW * WN * WM) void gemm_kernel(const float* __restrict__ A, const ST* __restrict__ W,
                                                                 const ST* __restrict__ bias, PlainGemm p) {
    constexpr int T = 2, U = 2;  // U: steps of 16 k requested together
    __shared__ float red[KW > 1 ? KW : 1][T * T][4][64];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, l16 = lane & 15, kq = 4 * (lane >> 4);
    const int kw = wave % KW, wn = (wave / KW) % WN, wm = wave / (KW * WN);
    const int n0 = (blockIdx.x * WN + wn) * 16 * T, m0 = (blockIdx.y * WM + wm) * 16 * T;
    const int steps = (p.K + 15) / 16;
    const int s0 = kw * steps / KW, s1 = (kw + 1) * steps / KW;
    const ST* wr[T];
    const float* ar[T];
#pragma unroll
    for (int t = 0; t < T; ++t) {  // rows past the end: the last one (computed, never stored)
        wr[t] = W + (size_t)min(n0 + 16 * t + l16, p.N - 1) * p.K;
        ar[t] = A + (size_t)min(m0 + 16 * t + l16, p.M - 1) * p.K;
    }
    f32x4 acc[T][T];
#pragma unroll
    for (int i = 0; i < T; ++i)
#pragma unroll
        for (int j = 0; j < T; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    f32x4 w[U][T], a[U][T];
    for (int s = s0; s < s1; s += U) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = s + u < s1 ? 16 * (s + u) + kq : p.K;  // (past this wavefront's range: zeros)
#pragma unroll
            for (int t = 0; t < T; ++t) {
                w[u][t] = load_k4<VEC>(wr[t], k, p.K);
                a[u][t] = load_k4<VEC>(ar[t], k, p.K);
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int i = 0; i < T; ++i)
#pragma unroll
                    for (int j = 0; j < T; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[u][i][e], a[u][j][e], acc[i][j], 0, 0, 0);
    }
    if (KW > 1) {
#pragma unroll
        for (int i = 0; i < T; ++i)
#pragma unroll
            for (int j = 0; j < T; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) red[kw][i * T + j][r][lane] = acc[i][j][r];
        __syncthreads();
        for (int t = kw; t < T * T; t += KW) {
            f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int x = 0; x < KW; ++x)
#pragma unroll
                for (int r = 0; r < 4; ++r) v[r] += red[x][t][r][lane];
            plain_epilogue4(p, bias, m0 + 16 * (t % T) + l16, n0 + 16 * (t / T) + kq, v);
        }
    } else {
#pragma unroll
        for (int i = 0; i < T; ++i)
#pragma unroll
            for (int j = 0; j < T; ++j) plain_epilogue4(p, bias, m0 + 16 * j + l16, n0 + 16 * i + kq, acc[i][j]);
    }
}

// The few rows of a decode step: 16 columns x 16 rows per workgroup of eight wavefronts, the LayerNorm of the rows folded in (LN).
// Nothing here takes as long as a launch; what does is the chain of everything that waits for something else, so all that the
// epilogue needs (bias, residual, where a key or value goes) is requested behind the first weights, a row's values are read
// once and its sums are data-parallel moves.  4 rows, a captured decode step: 256 x 256 and 256 x 1024 5.2 -> 4.0 us,
// 768 x 256 and 1024 x 256 with their LayerNorm 6.4 and 5.7 -> 4.1.
template <typename ST, bool VEC, bool LN>
__global__ __launch_bounds__(512) void gemm_few_kernel(const float* __restrict__ A, const ST* __restrict__ W, const ST* __restrict__ bias,
                                                       const ST* __restrict__ gamma, const ST* __restrict__ beta, PlainGemm p) {
    constexpr int KW = 8, U = 4, C = 4;  // U: steps of 16 k requested together; C: 256-value pieces of a row kept in registers
    __shared__ f32x4 red[KW][64];
    __shared__ float2 smr[16];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, l16 = lane & 15, kq = 4 * (lane >> 4);
    const int n0 = blockIdx.x * 16, m0 = blockIdx.y * 16;
    const int steps = (p.K + 15) / 16, s0 = wave * steps / KW, s1 = (wave + 1) * steps / KW;
    const ST* wr = W + (size_t)min(n0 + l16, p.N - 1) * p.K;  // rows past the end: the last one (computed, never stored)
    auto a_row = [&](int m) { return A + (LN ? (size_t)m * p.in_mul + p.in_add : (size_t)m) * p.K; };
    const float* ar = a_row(min(m0 + l16, p.M - 1));
    f32x4 acc = {0.f, 0.f, 0.f, 0.f}, w[U], a[U], g[U], be[U];
    auto load = [&](int s) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = s + u < s1 ? 16 * (s + u) + kq : p.K;  // (past this wavefront's range: zeros)
            w[u] = load_k4<VEC>(wr, k, p.K);
            a[u] = load_k4<VEC>(ar, k, p.K);
            if (LN) { g[u] = load_k4<VEC>(gamma, k, p.K); be[u] = load_k4<VEC>(beta, k, p.K); }
        }
    };
    load(s0);
    // rows of the tile: a wavefront takes row `wave` and row `wave` + 8
    const int rows = min(16, p.M - m0);
    f32x4 x[C];
    auto load_row = [&](const float* row) {
#pragma unroll
        for (int c = 0; c < C; ++c) {
            if (256 * c >= p.K) break;
            x[c] = load_k4<VEC>(row, 256 * c + 4 * lane, p.K);
        }
    };
    if (LN && wave < rows) load_row(a_row(m0 + wave));
    // the first wavefront finishes the tile: lane -> row l16, columns n0 + kq .. + 3
    const int m = m0 + l16, n = n0 + kq;
    const bool live = wave == 0 && m < p.M && n < p.N;
    f32x4 badd = {0.f, 0.f, 0.f, 0.f}, old = {0.f, 0.f, 0.f, 0.f};
    float* dst = p.out + (size_t)m * p.N + n;
    float scale = 1.f;
    bool store = live;
    if (live) {
        if (p.epi != EPI_STORE) badd = load_k4<false>(bias, n, p.N);
        if (p.epi == EPI_RESID) {
            if (p.vec_out) old = *reinterpret_cast<const f32x4*>(dst);
            else old = load_k4<false>(dst - n, n, p.N);
        } else if (p.epi == EPI_QKV) {  // q scaled to `out`, k and v appended to the cache (H and the head dimension are multiples of 8)
            if (n < p.H) {
                dst = p.out + (size_t)m * p.H + n;
                scale = p.qscale;
            } else {
                const int d = p.H / p.n_heads, which = n >= 2 * p.H, c = n - (which ? 2 * p.H : p.H);
                const int b = row_seq(p.st, m, p.S), tr = (p.S == 1 ? 0 : m % p.S) - row_pad(p.st, b);
                store = tr >= 0;  // padding rows append nothing
                dst = p.kv + kv_index(p.layer, which, b, c / d, seq_len(p.st, b) + tr, p.max_batch, p.n_heads, p.max_seq, d) + (c % d);
            }
        }
    }
    float mean = 0.f, rstd = 0.f;
    if (LN) {  // mean and 1/sqrt(var + eps) of the tile's rows
        for (int r = wave; r < rows; r += KW) {
            const float* row = a_row(m0 + r);
            if (r != wave) load_row(row);
            float t = 0.f;
#pragma unroll
            for (int c = 0; c < C; ++c) {
                if (256 * c >= p.K) break;
                t += (x[c][0] + x[c][1]) + (x[c][2] + x[c][3]);
            }
            for (int k = 256 * C + lane; k < p.K; k += 64) t += row[k];
            const float mu = lane_sum<64>(t) / p.K;
            float q = 0.f;
#pragma unroll
            for (int c = 0; c < C; ++c) {
                if (256 * c >= p.K) break;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float dlt = 256 * c + 4 * lane + e < p.K ? x[c][e] - mu : 0.f;
                    q += dlt * dlt;
                }
            }
            for (int k = 256 * C + lane; k < p.K; k += 64) { const float dlt = row[k] - mu; q += dlt * dlt; }
            q = lane_sum<64>(q);
            if (lane == 0) smr[r] = make_float2(mu, 1.0f / sqrtf(q / p.K + p.eps));
        }
        __syncthreads();
        const float2 mr = smr[min(l16, rows - 1)];
        mean = mr.x; rstd = mr.y;
    }
    for (int s = s0; s < s1; s += U) {
        if (s > s0) load(s);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (s + u >= s1) break;
            if (LN) a[u] = (a[u] - mean) * rstd * g[u] + be[u];
#pragma unroll
            for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(w[u][e], a[u][e], acc, 0, 0, 0);
        }
    }
    red[wave][lane] = acc;
    __syncthreads();
    if (wave != 0) return;
    f32x4 v = {0.f, 0.f, 0.f, 0.f}, part[KW];
#pragma unroll
    for (int i = 0; i < KW; ++i) part[i] = red[i][lane];
#pragma unroll
    for (int i = 0; i < KW; ++i) v += part[i];
    v += badd;
    if (p.epi == EPI_BIAS_RELU) {
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = fmaxf(v[i], 0.f);
    }
    v = (v + old) * scale;
    if (!store) return;
    const int nv = min(4, p.N - n);
    if (p.vec_out && nv == 4) {
        *reinterpret_cast<f32x4*>(dst) = v;
    } else {
        for (int i = 0; i < nv; ++i) dst[i] = v[i];
    }
}

// One block per (row m, head h).  16 lanes share a key, CH times four of its dimensions each, and keep the soft-max state of their
// keys (largest score, sum, weighted values) in one pass; K and V are on their way together, a round ahead.  The lane groups of a
// wavefront are merged with data-parallel moves, the four wavefronts through LDS behind the only barrier.  (4 rows x 4 heads of 64, up to
// 48 keys: 3.3 us; with a score buffer, two block-wide reductions and serial sums 6.1.)
template <int CH>
__global__ __launch_bounds__(256) void attn_kernel(const float* __restrict__ q, const float* __restrict__ kv,
                                                   float* __restrict__ o, const he_dev_state* __restrict__ st, int S, int layer,
                                                   int H, int n_heads, int max_batch, int max_seq) {
    constexpr int WAVES = 4, U = CH == 1 ? 4 : (CH == 2 ? 2 : 1), KR = WAVES * 4, STEP = KR * U;
    __shared__ float2 ml[WAVES];             // a wavefront's largest score and sum
    __shared__ f32x4 ored[WAVES][16 * CH];   // ... and its weighted values
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, sub = lane & 15, grp = lane >> 4;
    const int d = H / n_heads, d4 = d / 4;  // (d is a multiple of 8, at most 256)
    const int m = blockIdx.x, h = blockIdx.y;
    const f32x4* Q = reinterpret_cast<const f32x4*>(q + (size_t)m * H + h * d);
    f32x4 qv[CH];
#pragma unroll
    for (int c = 0; c < CH; ++c) qv[c] = sub + 16 * c < d4 ? Q[sub + 16 * c] : f32x4{0.f, 0.f, 0.f, 0.f};
    const int b = S == 1 ? m : m / S, T = seq_len(st, b) + (S == 1 ? 0 : m % S) - row_pad(st, b) + 1;
    f32x4* out = reinterpret_cast<f32x4*>(o + (size_t)m * H + h * d);
    if (T <= 0 || seq_done(st, b)) {  // a padding row, or a sequence that has ended: nothing reads this output
        for (int e = threadIdx.x; e < d4; e += 256) out[e] = f32x4{0.f, 0.f, 0.f, 0.f};
        return;
    }
    const f32x4* Kp = reinterpret_cast<const f32x4*>(kv + kv_index(layer, 0, b, h, 0, max_batch, n_heads, max_seq, d));
    const f32x4* Vp = reinterpret_cast<const f32x4*>(kv + kv_index(layer, 1, b, h, 0, max_batch, n_heads, max_seq, d));
    const int jw = wave * 4 + grp;
    auto load_rows = [&](f32x4 (&dst)[U][CH], const f32x4* src, int base) {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                const int j = base + u * KR + jw;
                dst[u][c] = j < T && sub + 16 * c < d4 ? src[(size_t)j * d4 + sub + 16 * c] : f32x4{0.f, 0.f, 0.f, 0.f};
            }
    };
    float mx = -INFINITY, sum = 0.f;
    f32x4 acc[CH], k[U][CH], v[U][CH];
#pragma unroll
    for (int c = 0; c < CH; ++c) acc[c] = f32x4{0.f, 0.f, 0.f, 0.f};
    load_rows(k, Kp, 0);
    load_rows(v, Vp, 0);
    for (int base = 0; base < T; base += STEP) {
        float s[U], top = mx;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            float x = 0.f;
#pragma unroll
            for (int c = 0; c < CH; ++c)
#pragma unroll
                for (int e = 0; e < 4; ++e) x = fmaf(qv[c][e], k[u][c][e], x);
            x = lane_sum<16>(x);
            s[u] = base + u * KR + jw < T ? x : -INFINITY;
            top = fmaxf(top, s[u]);
        }
        const bool more = base + STEP < T;  // (the same for the whole workgroup)
        if (more) load_rows(k, Kp, base + STEP);
        // (nothing above -inf yet: the state stays what it is)
        const float ref = top > -INFINITY ? top : 0.f, keep = expf(mx - ref);
        mx = top;
        sum *= keep;
#pragma unroll
        for (int c = 0; c < CH; ++c) acc[c] *= keep;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const float pr = base + u * KR + jw < T ? expf(s[u] - ref) : 0.f;
            sum += pr;
#pragma unroll
            for (int c = 0; c < CH; ++c)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[c][e] = fmaf(pr, v[u][c][e], acc[c][e]);
        }
        if (more) load_rows(v, Vp, base + STEP);
    }
    const float wmx = lane_max32_apart(lane_max16_apart(mx)), own = mx > -INFINITY ? expf(mx - wmx) : 0.f;
    sum = lane_sum_apart<16>(sum * own);
    if (lane == 0) ml[wave] = make_float2(wmx, sum);
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        f32x4 t;
#pragma unroll
        for (int e = 0; e < 4; ++e) t[e] = lane_sum_apart<16>(acc[c][e] * own);
        if (grp == 0) ored[wave][sub + 16 * c] = t;
    }
    __syncthreads();
    if ((int)threadIdx.x >= d4) return;
    float2 e[WAVES];
#pragma unroll
    for (int w = 0; w < WAVES; ++w) e[w] = ml[w];
    const float all = fmaxf(fmaxf(e[0].x, e[1].x), fmaxf(e[2].x, e[3].x));
    float total = 0.f;
    f32x4 t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
        const float f = e[w].x > -INFINITY ? expf(e[w].x - all) : 0.f;
        total += e[w].x > -INFINITY ? e[w].y * f : 0.f;
        t += ored[w][threadIdx.x] * f;
    }
    out[threadIdx.x] = t / total;
}

// One block per sequence: token = argmax of z (greedy) or of z/temperature + Gumbel noise, ties
// to the lowest id; logprob = z[token] - logsumexp(z).
// advance > 0: the pass fed that many tokens per sequence and ends here.
__global__ __launch_bounds__(kThreads) void sample_kernel(const float* __restrict__ logits, int V, he_dev_state* st,
                              int32_t* __restrict__ ids_out, float* __restrict__ lp_out, int out_stride,
                              int out_at_step, int32_t* __restrict__ cur_ids, int advance) {
    constexpr int C = 8, WAVES = kThreads / 64;  // logits of a thread kept in registers, the rest read again
    __shared__ float2 sms[WAVES];
    __shared__ float bs[WAVES];
    __shared__ int bi[WAVES];
    const int b = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const float* z = logits + (size_t)b * V;
    float zc[C];
#pragma unroll
    for (int c = 0; c < C; ++c) zc[c] = (int)threadIdx.x + c * kThreads < V ? z[threadIdx.x + c * kThreads] : -INFINITY;
    const int mode = st->mode, n = st->step;
    const float temp = st->temperature;
    const uint32_t k0 = st->seed_lo, k1 = st->seed_hi;
    float best = -INFINITY, mx = -INFINITY;
    int besti = 0x7FFFFFFF;
    auto look = [&](float zv, int v) {
        mx = fmaxf(mx, zv);
        float s = zv;
        if (mode == 1) s = zv / temp + gumbel_from_word(philox_word0((uint32_t)v, (uint32_t)n, (uint32_t)b, k0, k1));
        if (s > best || (s == best && v < besti)) { best = s; besti = v; }
    };
#pragma unroll
    for (int c = 0; c < C; ++c)
        if ((int)threadIdx.x + c * kThreads < V) look(zc[c], threadIdx.x + c * kThreads);
    for (int v = threadIdx.x + C * kThreads; v < V; v += kThreads) look(z[v], v);
    // a wavefront's exponentials against its own largest logit
    mx = lane_max<64>(mx);
    const float ref = mx > -INFINITY ? mx : 0.f;
    float sum = 0.f;
#pragma unroll
    for (int c = 0; c < C; ++c) sum += expf(zc[c] - ref);  // (past the vocabulary: -inf, adds 0)
    for (int v = threadIdx.x + C * kThreads; v < V; v += kThreads) sum += expf(z[v] - ref);
    sum = lane_sum<64>(sum);
    auto take = [&](float os, int oi) {
        if (os > best || (os == best && oi < besti)) { best = os; besti = oi; }
    };
    take(lane_xor1(best), __builtin_amdgcn_mov_dpp(besti, 0xB1, 0xF, 0xF, false));
    take(lane_xor2(best), __builtin_amdgcn_mov_dpp(besti, 0x4E, 0xF, 0xF, false));
    take(lane_mirror8(best), __builtin_amdgcn_mov_dpp(besti, 0x141, 0xF, 0xF, false));
    take(lane_mirror16(best), __builtin_amdgcn_mov_dpp(besti, 0x140, 0xF, 0xF, false));
    take(__shfl_xor(best, 16), __shfl_xor(besti, 16));
    take(__shfl_xor(best, 32), __shfl_xor(besti, 32));
    if (lane == 0) { sms[wave] = make_float2(mx, sum); bs[wave] = best; bi[wave] = besti; }
    __syncthreads();
    if (threadIdx.x == 0) {
        sum = 0.f;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) { mx = fmaxf(mx, sms[w].x); take(bs[w], bi[w]); }
#pragma unroll
        for (int w = 0; w < WAVES; ++w) sum += sms[w].x > -INFINITY ? sms[w].y * expf(sms[w].x - mx) : sms[w].y;
        if (!(mx > -INFINITY)) sum = __builtin_nanf("");  // no logit above -inf: no probabilities
        const size_t at = (size_t)b * out_stride + (out_at_step ? n : 0);
        ids_out[at] = besti;
        // (a row of nothing but NaN has no best token: besti is no vocabulary id then, and the sum is NaN)
        lp_out[at] = ((besti < V ? z[besti] : 0.f) - mx) - logf(sum);  // (in this order one rounding less of what is large)
        if (cur_ids) cur_ids[b] = besti;
    }
    if (advance) advance_state_by_last(st, advance, 1);
}

// Empty cache, greedy sampling; the arrival counters of the k-split GEMMs (null: none) and of the step's last kernel cleared
// with it.
__global__ __launch_bounds__(256) void reset_state_kernel(he_dev_state* st, int* __restrict__ counters, int n_counters) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i == 0) {
        st->cur_len = 0; st->step = 0; st->ragged = 0; st->arrivals = 0;
        st->mode = 0; st->temperature = 1.f; st->seed_lo = st->seed_hi = 0u;
    }
    if (i < n_counters) counters[i] = 0;
}

__global__ void init_state_kernel(he_dev_state* st, int max_batch) {
    for (int i = threadIdx.x; i < 4 * max_batch; i += blockDim.x) st->seq[i] = 0;
    for (int i = threadIdx.x; i < max_batch; i += blockDim.x) st->seq[4 * max_batch + i] = i;
    if (threadIdx.x == 0) {
        st->cur_len = 0; st->step = 0; st->mode = 0; st->temperature = 1.f; st->seed_lo = st->seed_hi = 0u;
        st->ragged = 0; st->max_batch = max_batch; st->eos_id = -1; st->pad_id = 0; st->n_active = 0; st->arrivals = 0;
    }
}

// Start of a ragged batch: B left-padded prompt rows of S entries, lens[b] of them tokens.
__global__ void set_ragged_kernel(he_dev_state* st, const int32_t* __restrict__ lens, int B, int S, int eos_id,
                                  int pad_id) {
    const int mb = st->max_batch;
    for (int b = threadIdx.x; b < mb; b += blockDim.x) {
        int n = b < B ? lens[b] : S;
        n = n < 1 ? 1 : (n > S ? S : n);  // lengths are clamped to what the rows can hold
        st->seq[b] = 0;
        st->seq[mb + b] = S - n;
        st->seq[2 * mb + b] = 0;
        st->seq[3 * mb + b] = 0;
        st->seq[4 * mb + b] = b;
    }
    if (threadIdx.x == 0) {
        st->cur_len = 0; st->step = 0;  // (a replay of a captured pass finds what the last one left)
        st->ragged = 1; st->eos_id = eos_id; st->pad_id = pad_id; st->n_active = B;
    }
}

__global__ void advance_state_kernel(he_dev_state* st, int tokens, int steps) { advance_state(st, tokens, steps); }

// he_generate_ragged, after a step's sampling: a sequence that has ended keeps producing the
// filler (log-probability 0); one that has just produced eos_id ends here.
__global__ void ragged_post_kernel(he_dev_state* st, int32_t* __restrict__ gen_ids, float* __restrict__ gen_lp,
                                   int32_t* __restrict__ cur_ids, int G, int B) {
    __shared__ int active;
    if (threadIdx.x == 0) active = 0;
    __syncthreads();
    const int mb = st->max_batch, n = st->step;
    for (int r = threadIdx.x; r < B; r += blockDim.x) {  // the B rows of the step (sequences without a row have ended)
        const int b = st->seq[4 * mb + r];
        const size_t at = (size_t)b * G + n;
        if (st->seq[2 * mb + b]) {
            gen_ids[at] = st->pad_id;
            gen_lp[at] = 0.f;
            cur_ids[b] = st->pad_id;
        } else {
            st->seq[3 * mb + b] = n + 1;
            if (gen_ids[at] == st->eos_id) st->seq[2 * mb + b] = 1;
            else atomicAdd(&active, 1);
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) st->n_active = active;
}

// he_generate_ragged, between two steps: the rows of sequences that have ended are dropped, the others move up
// in order.  rows: rows of the steps so far (new count = the running sequences: st->n_active).  One thread: the
// order has to be the same every time, and there are a few hundred rows at most.
__global__ void compact_rows_kernel(he_dev_state* st, int rows) {
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    const int mb = st->max_batch;
    int k = 0;
    for (int r = 0; r < rows; ++r) {
        const int b = st->seq[4 * mb + r];
        if (!st->seq[2 * mb + b]) st->seq[4 * mb + k++] = b;
    }
    for (; k < mb; ++k) st->seq[4 * mb + k] = k;  // (not in use: any valid sequence number)
}
// ... and back to one row per sequence, in sequence order.
__global__ void identity_rows_kernel(he_dev_state* st) {
    const int mb = st->max_batch;
    for (int i = threadIdx.x; i < mb; i += blockDim.x) st->seq[4 * mb + i] = i;
}

__global__ void fill_gen_kernel(int32_t* ids, float* lp, int count, const he_dev_state* st) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) { ids[i] = st->pad_id; lp[i] = 0.f; }
}

__global__ void copy_lens_kernel(const he_dev_state* st, int32_t* out, int B) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b < B) out[b] = st->seq[3 * st->max_batch + b];
}

__global__ void rng_words_kernel(uint32_t* out, int count, uint32_t v0, uint32_t n, uint32_t b, uint32_t k0,
                                 uint32_t k1) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) out[i] = philox_word0(v0 + (uint32_t)i, n, b, k0, k1);
}

// plain 16-byte-per-thread copy: the known-size reference that profiler byte counters are scaled by
__global__ void calibration_copy_kernel(const uint4* __restrict__ src, uint4* __restrict__ dst, size_t n16) {
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += stride) dst[i] = src[i];
}

__global__ void copy_out_kernel(const int32_t* __restrict__ ids, const float* __restrict__ lp,
                                int32_t* __restrict__ out_ids, float* __restrict__ out_lp, int count) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) { out_ids[i] = ids[i]; out_lp[i] = lp[i]; }
}

}  // namespace

// ------------------------------------------------------------------ launchers

template <typename ST>
static void plain_embed_t(hipStream_t s, const int32_t* ids, int id_stride, const void* tok, const void* pos,
                          float* x, he_dev_state* st, int M, int S, int H, int V, int pos_offset, const he_step_sampling& sp) {
    if (H % 4 == 0 && aligned4<ST>(tok) && aligned4<ST>(pos))
        embed_kernel<ST, true><<<M, kThreads, 0, s>>>(ids, id_stride, (const ST*)tok, (const ST*)pos, x, st, S, H, V, pos_offset, sp);
    else
        embed_kernel<ST, false><<<M, kThreads, 0, s>>>(ids, id_stride, (const ST*)tok, (const ST*)pos, x, st, S, H, V, pos_offset, sp);
}
void plain_embed(hipStream_t s, int bf16, const int32_t* ids, int id_stride, const void* tok, const void* pos, float* x,
                 he_dev_state* st, int M, int S, int H, int V, int pos_offset, const he_step_sampling& sp) {
    if (bf16) plain_embed_t<bf16_t>(s, ids, id_stride, tok, pos, x, st, M, S, H, V, pos_offset, sp);
    else plain_embed_t<float>(s, ids, id_stride, tok, pos, x, st, M, S, H, V, pos_offset, sp);
}

void plain_ln(hipStream_t s, int bf16, const float* r, const plain_ln_args& ln, float* a, int rows, int H) {
    if (bf16)
        ln_kernel<bf16_t><<<rows, kThreads, 0, s>>>(r, (const bf16_t*)ln.gamma, (const bf16_t*)ln.beta, a, H, ln.eps, ln.in_mul,
                                                    ln.in_add);
    else
        ln_kernel<float><<<rows, kThreads, 0, s>>>(r, (const float*)ln.gamma, (const float*)ln.beta, a, H, ln.eps, ln.in_mul,
                                                   ln.in_add);
}

// Rows up to which the LayerNorm is folded into the GEMM: every workgroup of 16 columns then normalises its 16 rows for itself,
// which costs rows x width x columns / 16.  Measured, decode steps of two layers (us, folded / a LayerNorm kernel and the 32 x 32
// tiles): width 256: 1 row 62 / 84, 64 rows 74 / 94; 512: 77 / 117, 117 / 130; 1024: 1 row 122 / 184, 32 rows 187 / 202, 33 220 / 198, 64
// 287 / 201; 2048: 1 row 255 / 358, 16 367 / 362, 64 974 / 477.  So the line is right for models up to 512 wide, whose steps this path
// is for, and too high for wider ones from 33 (1024) or 17 (2048) rows on.
// Small matrices go this way up to 256 rows: the 32 x 32 tiles are too few workgroups there (128 rows: 32 of them for 256 columns).  A
// prompt pass of two layers, tiles / this: width 256, FFN 1024: 128 rows 98 / 73, 256 rows 99 / 92, 272 106 / 104, 384 114 / 119, 512
// 119 / 135; width 128: 320 rows 139 / 73.  Up to 2^27 multiply-adds: what a workgroup's 16 rows and 16 columns load for them is four
// times what a tile loads.  Four layers, tiles / this: width 512, FFN 2048 (2^20 weights): 65 rows 233 / 170, 128 rows 244 / 208, 192 rows 298 / 303, 256
// rows 314 / 353; width 1024, FFN 1024: 65 rows 299 / 252, 128 rows 325 / 295, 256 rows 416 / 490; 768, FFN 768: 128 rows 269 / 239, 256
// rows 345 / 354.
constexpr int kFewRows = 64, kSmallRows = 256, kSmallMatrix = 1024 * 1024, kSmallWork = 128 * kSmallMatrix;
int plain_gemm_form(int M, int N, int K) {
    if (M <= kFewRows) return HE_PLAIN_FEW_ROWS;
    if (M <= kSmallRows && (long)N * K <= kSmallMatrix && (long)M * N * K <= kSmallWork) return HE_PLAIN_FEW_ROWS;
    return (long)((N + 63) / 64) * ((M + 63) / 64) >= 256 ? HE_PLAIN_TILES_64 : HE_PLAIN_TILES_32;
}

template <typename ST, bool VEC>
static void launch_gemm(hipStream_t s, const float* A, const ST* W, const ST* bias, const plain_ln_args* ln, const PlainGemm& p) {
    const ST *gamma = ln ? (const ST*)ln->gamma : nullptr, *beta = ln ? (const ST*)ln->beta : nullptr;
    const int form = plain_gemm_form(p.M, p.N, p.K);
    if (form == HE_PLAIN_FEW_ROWS) {
        const dim3 grid((p.N + 15) / 16, (p.M + 15) / 16);
        if (ln) gemm_few_kernel<ST, VEC, true><<<grid, 512, 0, s>>>(A, W, bias, gamma, beta, p);
        else gemm_few_kernel<ST, VEC, false><<<grid, 512, 0, s>>>(A, W, bias, gamma, beta, p);
        return;
    }
    if (form == HE_PLAIN_TILES_64)
        gemm_kernel<ST, 1, 2, 2, VEC><<<dim3((p.N + 63) / 64, (p.M + 63) / 64), 256, 0, s>>>(A, W, bias, p);
    else
        gemm_kernel<ST, 8, 1, 1, VEC><<<dim3((p.N + 31) / 32, (p.M + 31) / 32), 512, 0, s>>>(A, W, bias, p);
}

template <typename ST>
static void plain_gemm_t(hipStream_t s, const float* A, const void* W, const void* bias, const plain_ln_args* ln, float* scratch,
                         PlainGemm& p) {
    if (ln && plain_gemm_form(p.M, p.N, p.K) != HE_PLAIN_FEW_ROWS) {
        plain_ln(s, sizeof(ST) == 2, A, *ln, scratch, p.M, p.K);
        A = scratch;
        ln = nullptr;
    }
    // (the engine's activations are aligned)
    p.vec_out = p.N % 4 == 0 && (uintptr_t)p.out % 16 == 0;
    const bool vec = p.K % 4 == 0 && aligned4<ST>(W) && (!ln || (aligned4<ST>(ln->gamma) && aligned4<ST>(ln->beta)));
    if (ln) { p.eps = ln->eps; p.in_mul = ln->in_mul; p.in_add = ln->in_add; }
    if (vec) launch_gemm<ST, true>(s, A, (const ST*)W, (const ST*)bias, ln, p);
    else launch_gemm<ST, false>(s, A, (const ST*)W, (const ST*)bias, ln, p);
}

void plain_gemm(hipStream_t s, int bf16, const float* A, const void* W, const void* bias, int M, int N, int K, int epi,
                float* out, void* kv, const he_dev_state* st, int S, int layer, int H, int n_heads, int max_batch,
                int max_seq, float qscale, const plain_ln_args* ln, float* scratch) {
    PlainGemm p{M, N, K, epi, out, (float*)kv, st, S, layer, H, n_heads, max_batch, max_seq, qscale, 0.f, 1, 0, 0};
    if (bf16) plain_gemm_t<bf16_t>(s, A, W, bias, ln, scratch, p);
    else plain_gemm_t<float>(s, A, W, bias, ln, scratch, p);
}

void plain_attn(hipStream_t s, int bf16, const float* q, const void* kv, float* o, const he_dev_state* st, int M, int S,
                int layer, int H, int n_heads, int max_batch, int max_seq) {
    dim3 grid(M, n_heads);
    (void)bf16;  // the plain kernels keep keys and values as floats whatever the weights' type
    const float* c = (const float*)kv;
    const int ch = (H / n_heads / 4 + 15) / 16;  // (1 to 4: heads of up to 256)
    if (ch == 1) attn_kernel<1><<<grid, 256, 0, s>>>(q, c, o, st, S, layer, H, n_heads, max_batch, max_seq);
    else if (ch == 2) attn_kernel<2><<<grid, 256, 0, s>>>(q, c, o, st, S, layer, H, n_heads, max_batch, max_seq);
    else attn_kernel<4><<<grid, 256, 0, s>>>(q, c, o, st, S, layer, H, n_heads, max_batch, max_seq);
}

// one workgroup per row: log-sum-exp of the row's logits, then the next token's log-probability
__global__ void score_rows_kernel(const float* __restrict__ logits, const int32_t* __restrict__ ids, int row0, int S,
                                  int V, float* __restrict__ out) {
    __shared__ float red[kThreads];
    const int m = row0 + blockIdx.x;
    if (m % S == S - 1) return;
    const float* z = logits + (size_t)blockIdx.x * V;
    float mx = -INFINITY;
    for (int i = threadIdx.x; i < V; i += blockDim.x) mx = fmaxf(mx, z[i]);
    red[threadIdx.x] = mx;
    __syncthreads();
    for (int o = blockDim.x / 2; o > 0; o >>= 1) {
        if (threadIdx.x < o) red[threadIdx.x] = fmaxf(red[threadIdx.x], red[threadIdx.x + o]);
        __syncthreads();
    }
    mx = red[0];
    __syncthreads();
    float sum = 0.f;
    for (int i = threadIdx.x; i < V; i += blockDim.x) sum += expf(z[i] - mx);
    red[threadIdx.x] = sum;
    __syncthreads();
    for (int o = blockDim.x / 2; o > 0; o >>= 1) {
        if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        int t = ids[m + 1];
        t = t < 0 ? 0 : (t >= V ? V - 1 : t);
        out[(size_t)(m / S) * (S - 1) + m % S] = z[t] - (mx + logf(red[0]));
    }
}

void plain_score_rows(hipStream_t s, const float* logits, const int32_t* ids, int row0, int n, int S, int V, float* out) {
    score_rows_kernel<<<n, kThreads, 0, s>>>(logits, ids, row0, S, V, out);
}

void launch_sample(hipStream_t s, const float* logits, int B, int V, he_dev_state* st, int32_t* ids_out,
                   float* lp_out, int out_stride, int out_at_step, int32_t* cur_ids, int advance) {
    sample_kernel<<<B, kThreads, 0, s>>>(logits, V, st, ids_out, lp_out, out_stride, out_at_step, cur_ids, advance);
}

void launch_reset_state(hipStream_t s, he_dev_state* st, int* counters, int n_counters) {
    reset_state_kernel<<<(n_counters + 255) / 256 + (n_counters == 0), 256, 0, s>>>(st, counters, n_counters);
}

void launch_init_state(hipStream_t s, he_dev_state* st, int max_batch) { init_state_kernel<<<1, 256, 0, s>>>(st, max_batch); }
void launch_set_ragged(hipStream_t s, he_dev_state* st, const int32_t* lens, int B, int S, int eos_id, int pad_id) {
    set_ragged_kernel<<<1, 256, 0, s>>>(st, lens, B, S, eos_id, pad_id);
}
void launch_ragged_post(hipStream_t s, he_dev_state* st, int32_t* gen_ids, float* gen_lp, int32_t* cur_ids, int G, int B) {
    ragged_post_kernel<<<1, 256, 0, s>>>(st, gen_ids, gen_lp, cur_ids, G, B);
}
void launch_compact_rows(hipStream_t s, he_dev_state* st, int rows) { compact_rows_kernel<<<1, 64, 0, s>>>(st, rows); }
void launch_identity_rows(hipStream_t s, he_dev_state* st) { identity_rows_kernel<<<1, 256, 0, s>>>(st); }
void launch_fill_gen(hipStream_t s, int32_t* ids, float* lp, int count, const he_dev_state* st) {
    fill_gen_kernel<<<(count + 255) / 256, 256, 0, s>>>(ids, lp, count, st);
}
void launch_copy_lens(hipStream_t s, const he_dev_state* st, int32_t* out, int B) {
    copy_lens_kernel<<<(B + 255) / 256, 256, 0, s>>>(st, out, B);
}
void launch_advance_state(hipStream_t s, he_dev_state* st, int tokens, int steps) {
    advance_state_kernel<<<1, 64, 0, s>>>(st, tokens, steps);
}

void launch_rng_words(hipStream_t s, uint64_t seed, uint32_t b, uint32_t n, uint32_t v0, int count, uint32_t* out) {
    rng_words_kernel<<<(count + 255) / 256, 256, 0, s>>>(out, count, v0, n, b, (uint32_t)(seed & 0xFFFFFFFFu),
                                                         (uint32_t)(seed >> 32));
}

void launch_calibration_copy(hipStream_t s, const void* src, void* dst, size_t bytes) {
    calibration_copy_kernel<<<4096, 256, 0, s>>>((const uint4*)src, (uint4*)dst, bytes / 16);
}

void launch_copy_out(hipStream_t s, const int32_t* ids, const float* lp, int32_t* out_ids, float* out_lp, int count) {
    copy_out_kernel<<<(count + 255) / 256, 256, 0, s>>>(ids, lp, out_ids, out_lp, count);
}
