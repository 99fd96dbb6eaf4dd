// bf16 path: LayerNorm kernels, and the producer side of LayerNorms folded into the next GEMM.
#include "bf16_common.h"

using namespace he_bf16;

namespace {

// ----------------------------------------------------------------- LayerNorm (+ residual update)
//
// Row `src = m*in_mul + in_add`: r += sum of k-split partials + bias (fixed order),
// written back when asked; a = LayerNorm(r) is emitted as tiled half blocks.
__global__ __launch_bounds__(1024) void ln_blocks_kernel(float* __restrict__ r, const float* __restrict__ part,
                                                        int ksplit, size_t part_split,
                                                        const bf16_t* __restrict__ pbias,
                                                        const bf16_t* __restrict__ gamma,
                                                        const bf16_t* __restrict__ beta, u32x4* __restrict__ a,
                                                        int H, float eps, int in_mul, int in_add, int writeback,
                                                        int split_col) {
    extern __shared__ __align__(16) float row[];
    __shared__ float red[16];
    const int m = blockIdx.x, wave = threadIdx.x >> 6, lane = threadIdx.x & 63, nwave = blockDim.x >> 6;
    const size_t src = (size_t)m * in_mul + in_add;
    float4* rr = reinterpret_cast<float4*>(r + src * H);
    float s = 0.f;
    for (int i = threadIdx.x; i < H / 4; i += blockDim.x) {
        float4 v = rr[i];
        if (part) {
            for (int k = 0; k < ksplit; ++k) {
                if (k > 0 && 4 * i < split_col) break;  // columns before split_col have one whole sum
                const float4 y = *reinterpret_cast<const float4*>(part + (size_t)k * part_split + src * H + 4 * i);
                v.x += y.x; v.y += y.y; v.z += y.z; v.w += y.w;
            }
            const uint2 bb = *reinterpret_cast<const uint2*>(pbias + 4 * i);
            v.x += bf_lo(bb.x); v.y += bf_hi(bb.x);
            v.z += bf_lo(bb.y); v.w += bf_hi(bb.y);
            if (writeback) rr[i] = v;
        }
        reinterpret_cast<float4*>(row)[i] = v;
        s += (v.x + v.y) + (v.z + v.w);
    }
    s = lane_sum<64>(s);
    if (lane == 0) red[wave] = s;
    __syncthreads();
    float tot = 0.f;
    for (int i = 0; i < nwave; ++i) tot += red[i];
    const float mean = tot / H;
    float q = 0.f;
    for (int i = threadIdx.x; i < H; i += blockDim.x) { const float dlt = row[i] - mean; q += dlt * dlt; }
    q = lane_sum<64>(q);
    __syncthreads();
    if (lane == 0) red[wave] = q;
    __syncthreads();
    tot = 0.f;
    for (int i = 0; i < nwave; ++i) tot += red[i];
    const float rstd = 1.0f / sqrtf(tot / H + eps);
    const int KB = H >> 4;
    for (int c = threadIdx.x; c < H / 8; c += blockDim.x) {
        const int k0 = c * 8;
        const u32x4 gg = *reinterpret_cast<const u32x4*>(gamma + k0), bb = *reinterpret_cast<const u32x4*>(beta + k0);
        const uint32_t gw[4] = {gg.x, gg.y, gg.z, gg.w}, bw[4] = {bb.x, bb.y, bb.z, bb.w};
        uint32_t o[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float e0 = (row[k0 + 2 * j] - mean) * rstd * bf_lo(gw[j]) + bf_lo(bw[j]);
            const float e1 = (row[k0 + 2 * j + 1] - mean) * rstd * bf_hi(gw[j]) + bf_hi(bw[j]);
            o[j] = pack2(e0, e1);
        }
        a[block_slot(m, k0, KB)] = u32x4{o[0], o[1], o[2], o[3]};
    }
}

// The same operation with every value of the row held in registers (NV float4 per thread) and all
// loads -- residual, k-split partials, bias, gamma, beta -- issued before the first reduction.
// For the few rows of a decode step one 1024-thread workgroup per row (the kernel's time is then the
// length of its dependent-load chain); for the many rows of a prompt pass 256 threads per row.
template <int NV, int THREADS>
__global__ __launch_bounds__(THREADS) void ln_row_kernel(float* __restrict__ r, const float* __restrict__ part, int ksplit,
                                                      size_t part_split, const bf16_t* __restrict__ pbias,
                                                      const bf16_t* __restrict__ gamma,
                                                      const bf16_t* __restrict__ beta, u32x4* __restrict__ a,
                                                      int H, float eps, int in_mul, int in_add, int writeback,
                                                      int rows, int split_col) {
    constexpr int NW = THREADS / 64;
    __shared__ float red[2][NW];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    int m = blockIdx.x;
    if (THREADS == 256) {
        // Many rows: a row writes 16-byte slots of the 32-row blocks, 512 bytes apart, and the 32 rows of a block
        // together fill whole cache lines.  Workgroups go round the eight XCDs by index, so the rows of one block
        // are kept on one XCD (block b on XCD b mod 8): its L2 then holds complete lines to write back.
        const int x = blockIdx.x & 7, j = blockIdx.x >> 3;
        m = (((j >> 5) << 3) + x) * 32 + (j & 31);
        if (m >= rows) return;  // the whole workgroup: the grid is padded to eight blocks
    }
    const size_t src = (size_t)m * in_mul + in_add;
    const int nq = H >> 2;  // float4 per row
    float4 v[NV];
    uint2 gg[NV], bb[NV];
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const int i = threadIdx.x + j * THREADS;
        v[j] = make_float4(0.f, 0.f, 0.f, 0.f);
        gg[j] = bb[j] = make_uint2(0, 0);
        if (i < nq) {
            v[j] = *reinterpret_cast<const float4*>(r + src * H + 4 * i);
            gg[j] = *reinterpret_cast<const uint2*>(gamma + 4 * i);
            bb[j] = *reinterpret_cast<const uint2*>(beta + 4 * i);
        }
    }
    if (part && ksplit <= 2) {  // the usual cases, with every load of the row requested before the first is used
        float4 y0[NV], y1[NV];
        uint2 pb[NV];
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            const int i = threadIdx.x + j * THREADS;
            y0[j] = y1[j] = make_float4(0.f, 0.f, 0.f, 0.f);
            pb[j] = make_uint2(0, 0);
            if (i >= nq) continue;
            y0[j] = *reinterpret_cast<const float4*>(part + src * H + 4 * i);
            // (columns before split_col have one whole sum; a multiple of 256 or 320)
            if (ksplit == 2 && 4 * i >= split_col) y1[j] = *reinterpret_cast<const float4*>(part + part_split + src * H + 4 * i);
            pb[j] = *reinterpret_cast<const uint2*>(pbias + 4 * i);
        }
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            const int i = threadIdx.x + j * THREADS;
            if (i >= nq) continue;
            v[j].x += (y0[j].x + y1[j].x) + bf_lo(pb[j].x);
            v[j].y += (y0[j].y + y1[j].y) + bf_hi(pb[j].x);
            v[j].z += (y0[j].z + y1[j].z) + bf_lo(pb[j].y);
            v[j].w += (y0[j].w + y1[j].w) + bf_hi(pb[j].y);
            if (writeback) *reinterpret_cast<float4*>(r + src * H + 4 * i) = v[j];
        }
    } else if (part) {
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            const int i = threadIdx.x + j * THREADS;
            if (i >= nq) continue;
            float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
            for (int k0 = 0; k0 < ksplit; k0 += 4) {  // fixed order: the sum does not depend on scheduling
                float4 y[4];  // four loads on their way at a time
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    y[k] = *reinterpret_cast<const float4*>(part + (size_t)min(k0 + k, ksplit - 1) * part_split + src * H + 4 * i);
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (k0 + k < ksplit) { acc.x += y[k].x; acc.y += y[k].y; acc.z += y[k].z; acc.w += y[k].w; }
            }
            const uint2 pb = *reinterpret_cast<const uint2*>(pbias + 4 * i);
            v[j].x += acc.x + bf_lo(pb.x);
            v[j].y += acc.y + bf_hi(pb.x);
            v[j].z += acc.z + bf_lo(pb.y);
            v[j].w += acc.w + bf_hi(pb.y);
            if (writeback) *reinterpret_cast<float4*>(r + src * H + 4 * i) = v[j];
        }
    }
#pragma unroll
    for (int j = 0; j < NV; ++j) s += (v[j].x + v[j].y) + (v[j].z + v[j].w);  // lanes past the row hold zeros
    s = lane_sum<64>(s);
    if (lane == 0) red[0][wave] = s;
    __syncthreads();
    float tot = 0.f;
#pragma unroll
    for (int i = 0; i < NW; ++i) tot += red[0][i];
    const float mean = tot / H;
    float q = 0.f;
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        if (threadIdx.x + j * THREADS < nq) {
            const float d0 = v[j].x - mean, d1 = v[j].y - mean, d2 = v[j].z - mean, d3 = v[j].w - mean;
            q += (d0 * d0 + d1 * d1) + (d2 * d2 + d3 * d3);
        }
    }
    q = lane_sum<64>(q);
    if (lane == 0) red[1][wave] = q;
    __syncthreads();
    tot = 0.f;
#pragma unroll
    for (int i = 0; i < NW; ++i) tot += red[1][i];
    const float rstd = 1.0f / sqrtf(tot / H + eps);
    const int KB = H >> 4;
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const int i = threadIdx.x + j * THREADS;
        if (i >= nq) continue;
        const float e0 = (v[j].x - mean) * rstd * bf_lo(gg[j].x) + bf_lo(bb[j].x);
        const float e1 = (v[j].y - mean) * rstd * bf_hi(gg[j].x) + bf_hi(bb[j].x);
        const float e2 = (v[j].z - mean) * rstd * bf_lo(gg[j].y) + bf_lo(bb[j].y);
        const float e3 = (v[j].w - mean) * rstd * bf_hi(gg[j].y) + bf_hi(bb[j].y);
        const int k0 = 4 * i;  // four values: half of a 16-byte slot
        const size_t slot = block_slot(m, k0 & ~7, KB);
        reinterpret_cast<uint2*>(a + slot)[(k0 >> 2) & 1] = make_uint2(pack2(e0, e1), pack2(e2, e3));
    }
}

// ----------------------------------------------------------------- LayerNorm folded into the next GEMM (decode rows)
//
// For the few rows of a decode step a LayerNorm kernel of its own is all latency.  Instead
//   W LN(x) + b = rstd * (W (gamma . x) - mean * (W gamma)) + W beta + b,
// so the kernel that produces x (the embedding below, or the out-projection / FC2 GEMM
// through its last-arriving workgroup) writes gamma . x as half blocks plus per-column-
// group statistics of x, the consuming GEMM multiplies those blocks by the unchanged
// weights and applies mean and rstd in its epilogue, and W gamma, W beta are vectors computed
// once per weight update.

// Row m of a decode step: x = tok_emb[id] + pos_emb[cur_len + pos_offset], four columns per lane.  A wavefront takes the
// column groups that fit its lanes whole (gw <= 256; one lane group of gw / 4 lanes to each).  What bounds it is the chain
// from the state and the ids to the table rows; the sums over a group's lanes are data-parallel moves where gw / 4 is a power of two.
__device__ __forceinline__ float group_sum(float v, int lanes, int first) {
    switch (lanes) {  // (the same for the whole launch)
        case 4: return lane_sum<4>(v);
        case 8: return lane_sum<8>(v);
        case 16: return lane_sum<16>(v);
        case 32: return lane_sum<32>(v);
        case 64: return lane_sum<64>(v);
    }
    float t = 0.f;
    for (int i = 0; i < lanes; ++i) t += __shfl(v, first + i);
    return t;
}
__global__ __launch_bounds__(64) void embed_ln_kernel(const int32_t* __restrict__ ids, int id_stride,
                                                      const bf16_t* __restrict__ tok, const bf16_t* __restrict__ pos,
                                                      he_dev_state* __restrict__ st, int V, int pos_offset,
                                                      int H, int gw, int groups, int per_wave, const bf16_t* __restrict__ gamma,
                                                      float* __restrict__ r, u32x4* __restrict__ xb,
                                                      float2* __restrict__ stats, he_step_sampling sp) {
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) store_sampling(st, sp);
    const int m = blockIdx.y, lane = threadIdx.x, lanes = gw >> 2;
    const int sub = min(lane / lanes, per_wave), in_group = lane - sub * lanes;  // (lanes past the last whole group: idle)
    const int g = blockIdx.x * per_wave + sub, cols = g < groups ? min(gw, H - g * gw) : 0, c0 = g * gw + 4 * in_group;
    const bool live = sub < per_wave && 4 * in_group < cols;
    uint2 gg = make_uint2(0, 0);
    if (live) gg = *reinterpret_cast<const uint2*>(gamma + c0);
    const int b = sp.start ? m : row_seq(st, m, 1);  // one row per running sequence here
    int id = ids[(size_t)b * id_stride];
    id = id < 0 ? 0 : (id >= V ? V - 1 : id);
    const size_t prow = (size_t)((sp.start ? 0 : seq_len(st, b)) + pos_offset);
    float x0 = 0.f, x1 = 0.f, x2 = 0.f, x3 = 0.f;
    if (live) {
        const uint2 t = *reinterpret_cast<const uint2*>(tok + (size_t)id * H + c0);
        const uint2 q = *reinterpret_cast<const uint2*>(pos + prow * H + c0);
        x0 = bf_lo(t.x) + bf_lo(q.x);
        x1 = bf_hi(t.x) + bf_hi(q.x);
        x2 = bf_lo(t.y) + bf_lo(q.y);
        x3 = bf_hi(t.y) + bf_hi(q.y);
        *reinterpret_cast<float4*>(r + (size_t)m * H + c0) = make_float4(x0, x1, x2, x3);
        const size_t slot = block_slot(m, c0 & ~7, H >> 4);
        reinterpret_cast<uint2*>(xb + slot)[(c0 >> 2) & 1] =
            make_uint2(pack2(x0 * bf_lo(gg.x), x1 * bf_hi(gg.x)), pack2(x2 * bf_lo(gg.y), x3 * bf_hi(gg.y)));
    }
    const int first = sub * lanes;
    const float mean = group_sum((x0 + x1) + (x2 + x3), lanes, first) / (float)max(cols, 1);
    float q2 = 0.f;
    if (live) {
        const float d0 = x0 - mean, d1 = x1 - mean, d2 = x2 - mean, d3 = x3 - mean;
        q2 = (d0 * d0 + d1 * d1) + (d2 * d2 + d3 * d3);
    }
    q2 = group_sum(q2, lanes, first);
    if (live && in_group == 0) stats[((size_t)(m >> 5) * groups + g) * 32 + (m & 31)] = make_float2(mean, q2);
}

// c1[n] = sum_k W[n][k] gamma[k], c2[n] = sum_k W[n][k] beta[k] from the tiled weights: a workgroup per T 32-row tiles (lane =
// row and k half), its eight wavefronts each with a share of k, float accumulation in k order, the shares' sums added in
// wavefront order.  Bound by reading the matrix once: the next round of four blocks of each tile is on its way while one is
// added up, and two tiles share their gamma and beta, where that leaves each CU a workgroup.  Right behind the kernel that
// wrote the tiles part of them is read from the memory side's cache.  us with the matrix in its place in the pass over a model's
// weights, one round of one tile after all matrices were written -> this:
// 16384 x 4096 39.3 -> 28.0, 12288 x 4096 36.4 -> 22.1, 50272 x 4096 96 -> 83.
constexpr int kWvecWaves = 8;
template <int T>
__global__ __launch_bounds__(64 * kWvecWaves) void wvec_kernel(const u32x4* __restrict__ Wp, int KB, int n_tiles,
                                                               const bf16_t* __restrict__ gamma,
                                                               const bf16_t* __restrict__ beta, float* __restrict__ c1,
                                                               float* __restrict__ c2) {
    __shared__ float red[2][kWvecWaves][T * 32];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, tile = blockIdx.x * T;
    const int kb0 = wave * KB / kWvecWaves, kb1 = (wave + 1) * KB / kWvecWaves;
    constexpr int U = 4;
    struct Round { u32x4 w[T][U], g[U], b[U]; };
    auto load = [&](Round& r, int kb) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = min(kb + u, kb1 - 1);
#pragma unroll
            for (int t = 0; t < T; ++t)  // (past the last tile: it again, never stored)
                r.w[t][u] = __builtin_nontemporal_load(Wp + ((size_t)min(tile + t, n_tiles - 1) * KB + k) * 64 + lane);
            r.g[u] = *reinterpret_cast<const u32x4*>(gamma + k * 16 + (lane >> 5) * 8);
            r.b[u] = *reinterpret_cast<const u32x4*>(beta + k * 16 + (lane >> 5) * 8);
        }
    };
    float a1[T], a2[T];
#pragma unroll
    for (int t = 0; t < T; ++t) a1[t] = a2[t] = 0.f;
    Round cur, nxt;
    if (kb0 < kb1) load(cur, kb0);
    for (int kb = kb0; kb < kb1; kb += U) {
        if (kb + U < kb1) load(nxt, kb + U);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (kb + u >= kb1) break;
            const uint32_t gg[4] = {cur.g[u].x, cur.g[u].y, cur.g[u].z, cur.g[u].w}, bb[4] = {cur.b[u].x, cur.b[u].y, cur.b[u].z, cur.b[u].w};
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const uint32_t ww[4] = {cur.w[t][u].x, cur.w[t][u].y, cur.w[t][u].z, cur.w[t][u].w};
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    const float w0 = half_lo(ww[x]), w1 = half_hi(ww[x]);
                    a1[t] = fmaf(w0, bf_lo(gg[x]), a1[t]);
                    a1[t] = fmaf(w1, bf_hi(gg[x]), a1[t]);
                    a2[t] = fmaf(w0, bf_lo(bb[x]), a2[t]);
                    a2[t] = fmaf(w1, bf_hi(bb[x]), a2[t]);
                }
            }
        }
        cur = nxt;
    }
#pragma unroll
    for (int t = 0; t < T; ++t) {
        a1[t] = lane_sum32_apart(a1[t]);
        a2[t] = lane_sum32_apart(a2[t]);
        if (lane < 32) { red[0][wave][t * 32 + lane] = a1[t]; red[1][wave][t * 32 + lane] = a2[t]; }
    }
    __syncthreads();
    if (threadIdx.x < 64 * T) {  // rows past the matrix are zero blocks: their entries come out zero
        const int which = threadIdx.x >= 32 * T, r = threadIdx.x - which * 32 * T;
        float sum = 0.f;
#pragma unroll
        for (int x = 0; x < kWvecWaves; ++x) sum += red[which][x][r];
        if (tile + (r >> 5) < n_tiles) (which ? c2 : c1)[tile * 32 + r] = sum;
    }
}

// Rows b*S + S-1 (each sequence's last prompt row) of two [B*S][H] float arrays -> rows b of two [B][H] arrays.  Reads nothing of
// the state, so the first workgroup also advances it (one launch less).
__global__ __launch_bounds__(256) void gather_last_rows_kernel(const float* __restrict__ r, const float* __restrict__ q,
                                                               float* __restrict__ r_out, float* __restrict__ q_out, int S,
                                                               int H, he_dev_state* st, int advance) {
    const size_t src = ((size_t)blockIdx.x * S + S - 1) * H, dst = (size_t)blockIdx.x * H;
    for (int i = threadIdx.x; i < H / 4; i += 256) {
        reinterpret_cast<float4*>(r_out + dst)[i] = reinterpret_cast<const float4*>(r + src)[i];
        reinterpret_cast<float4*>(q_out + dst)[i] = reinterpret_cast<const float4*>(q + src)[i];
    }
    if (blockIdx.x == 0) advance_state(st, advance, 0);
}

}  // namespace

// ------------------------------------------------------------------ launchers

void bf16_gather_last_rows(hipStream_t s, const float* r, const float* q, float* r_out, float* q_out, int B, int S, int H, he_dev_state* st,
                           int advance) {
    gather_last_rows_kernel<<<B, 256, 0, s>>>(r, q, r_out, q_out, S, H, st, advance);
}

void bf16_embed_ln(hipStream_t s, const int32_t* ids, int id_stride, const void* tok, const void* pos,
                   he_dev_state* st, int B, int H, int V, int pos_offset, int gw, const void* gamma, float* r,
                   void* x_blocks, float* stats, const he_step_sampling& sp) {
    const int groups = (H + gw - 1) / gw, per_wave = 256 / gw;
    embed_ln_kernel<<<dim3((groups + per_wave - 1) / per_wave, B), 64, 0, s>>>(ids, id_stride, (const bf16_t*)tok, (const bf16_t*)pos, st, V,
                                                   pos_offset, H, gw, groups, per_wave, (const bf16_t*)gamma, r,
                                                   (u32x4*)x_blocks, (float2*)stats, sp);
}

void bf16_wvec(hipStream_t s, const void* Wp, int N, int K, const void* gamma, const void* beta, float* c1, float* c2) {
    const int tiles = (N + 31) / 32;  // two to a workgroup where every CU keeps one (12288 rows x 4096: 22.1 us with one each)
    if (tiles >= 2 * num_cus())
        wvec_kernel<2><<<(tiles + 1) / 2, 64 * kWvecWaves, 0, s>>>((const u32x4*)Wp, K / 16, tiles, (const bf16_t*)gamma, (const bf16_t*)beta, c1, c2);
    else
        wvec_kernel<1><<<tiles, 64 * kWvecWaves, 0, s>>>((const u32x4*)Wp, K / 16, tiles, (const bf16_t*)gamma, (const bf16_t*)beta, c1, c2);
}

void bf16_ln(hipStream_t s, float* r, const float* part, int ksplit, size_t part_split, const void* pbias,
             const void* gamma, const void* beta, void* a_blocks, int rows, int H, float eps, int in_mul, int in_add,
             int writeback, int split_col) {
    if (ksplit != 2) split_col = 0;  // (only the two-range form knows partly cut rows)
    const int nv = (H / 4 + 1023) / 1024, nv256 = (H / 4 + 255) / 256;
#define HE_LN_ROW(NV, T)                                                                                                \
    ln_row_kernel<NV, T><<<(T == 256 ? (rows + 255) / 256 * 256 : rows), T, 0, s>>>(                                    \
        r, part, ksplit, part_split, (const bf16_t*)pbias, (const bf16_t*)gamma, (const bf16_t*)beta, (u32x4*)a_blocks, \
        H, eps, in_mul, in_add, writeback, rows, split_col)
    if (rows <= 256 && nv <= 3) {  // a decode step
        if (nv == 1) HE_LN_ROW(1, 1024);
        else if (nv == 2) HE_LN_ROW(2, 1024);
        else HE_LN_ROW(3, 1024);
        return;
    }
    if (nv256 <= 10) {  // prompt rows, hidden sizes up to 10240
        switch (nv256) {
            case 1: HE_LN_ROW(1, 256); break;
            case 2: HE_LN_ROW(2, 256); break;
            case 3: HE_LN_ROW(3, 256); break;
            case 4: HE_LN_ROW(4, 256); break;
            case 5: HE_LN_ROW(5, 256); break;
            case 6: HE_LN_ROW(6, 256); break;
            case 7: HE_LN_ROW(7, 256); break;
            case 8: HE_LN_ROW(8, 256); break;
            case 9: HE_LN_ROW(9, 256); break;
            default: HE_LN_ROW(10, 256); break;
        }
        return;
    }
#undef HE_LN_ROW
    ln_blocks_kernel<<<rows, 256, (size_t)H * sizeof(float), s>>>(
        r, part, ksplit, part_split, (const bf16_t*)pbias, (const bf16_t*)gamma, (const bf16_t*)beta, (u32x4*)a_blocks,
        H, eps, in_mul, in_add, writeback, split_col);
}

