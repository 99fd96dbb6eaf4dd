// bf16 path: weight preparation -- the caller's bf16 matrices converted to IEEE half and tiled into MFMA
// operand blocks (optionally with low-rank adapters folded in), and 8-bit E4M3 row quantisation.
#include "bf16_common.h"

using namespace he_bf16;

namespace {

// ----------------------------------------------------------------- weight tiling

// eight bf16 values -> eight halves: exact for magnitudes 2^-14 .. 65504 (8 significant bits into 11), nearest
// multiple of 2^-24 (ties to even) below that
__device__ __forceinline__ u32x4 bf16x8_to_half(const u32x4& w) {
    return u32x4{pack2(bf_lo(w.x), bf_hi(w.x)), pack2(bf_lo(w.y), bf_hi(w.y)), pack2(bf_lo(w.z), bf_hi(w.z)),
                 pack2(bf_lo(w.w), bf_hi(w.w))};
}
// two floats -> two bf16 in one word, round to nearest even (the LoRA merge rounds to the model's own format)
__device__ __forceinline__ uint32_t pack2_bf16(float lo, float hi) { return f32x2_to_bf16x2(lo, hi); }

// The same with a low-rank adapter folded in: dst = tiled half(bf16(W + scale * B A)), A [rank, K], B [R, rank].
// The sum fixes a bf16 rounding, so its order is part of the definition: products B[r][j] A[j][k] are added one by one for
// j = 0..rank-1, then W + scale * that, every operation a float rounding of its own.  The products of two bf16 values have 16
// significant bits: they are floats, and adding one by a fused multiply-add rounds just as a separate addition does.  (Products
// below 2^-134, which a float would round, leave a sum that is zero as a half for every scale below 2^75; products above 2^127
// need adapter entries of 2^63.)  So the sums are formed on the matrix cores: a float instruction of depth one, a fused multiply-add
// per element, for each rank.  scale * t is no such product: it and the addition to W round separately.
//
// Where the matrix follows a LayerNorm (FOLD), W gamma and W beta of its rows are formed from the values on their way, or, TILED,
// from tiles that are there already (the caller's, or dequantised ones), in one order whatever the weights came as, part of the
// definition too (a last bit of them can decide how an activation rounds, layers later): a workgroup has 32 rows, its eight wavefronts each
// a share of k, in blocks of 16 columns; a wavefront adds up the two halves of its blocks apart, k ascending, then the one to the other,
// and the wavefronts' sums are added in their order.
//
// Bound by the memory rate.  Without the vectors a workgroup takes 32 rows x 512 columns, neighbours next to each other along k, so that the
// workgroups in flight sweep source and destination in order.  With them a wavefront goes over its share 64 columns at a time, whose
// gamma and beta go through LDS (a wavefront's own loads of them cost as much as its weights').  The k side of the products is permuted so
// that a lane's accumulators are its own eight columns of each block.
// us a launch with others around it, a kernel that tiles or merges on the vector units, then one that reads the tiles again for the vectors -> this:
// 16384 x 4096, rank 16 61.7 + 28.9 -> 64.5, 12288 x 4096 49.2 + 23.9 -> 61 (384 workgroups on 256 CUs), 50272 x 4096 without an adapter 152 + 82 -> 164;
// without vectors, plain 52.6 -> 47.3, rank 16 (4096 x 16384) 61.4 -> 50, (4096 x 4096) 21 -> 15.5.  (Workgroups of 32 rows x 512 columns that leave partial sums
// for another kernel to add, 67, 54 and 146 us, sum in another order: outputs of whole models moved by 5e-4.  The next 64 columns requested
// ahead, then the adapter's values: 68, 63 and 165.)  The tiles are stored non-temporally: four layers of hidden 4096 with adapters and the head 1248 -> 1216 us, twelve of hidden
// 2048 650 -> 616, and with a decode step behind it 1061 -> 1025; the sources must not be loaded so (1248 -> 1434: four loads share a cache line).
typedef float f32x32 __attribute__((ext_vector_type(32)));
constexpr int kMergeBlocks = 4;                               // blocks of 16 columns at a time: two accumulator tiles
constexpr int kMergeWaves = 8;
constexpr int kMergeSpan = kMergeBlocks * kMergeWaves;        // ... to a workgroup without the vectors
constexpr int kMergeRanks = 32;                               // ranks whose B values are in LDS at a time
// LORA, how B's rows come: in loads of 16 bytes (rank a multiple of eight, B so aligned); a value at a time, up to eight; through
// LDS, where the eight wavefronts would each wait for more than eight such loads.  16384 x 4096, rank 17: 81 us a value at a time, 67 through
// LDS; rank 3: 48 and 57; rank 16: 53 by 16 bytes, 69 through LDS.
enum { LORA_NONE = 0, LORA_WIDE = 1, LORA_FEW = 2, LORA_LDS = 3 };
template <int LORA, bool FOLD, bool TILED>
__global__ __launch_bounds__(64 * kMergeWaves) void tile_merge_kernel(const bf16_t* __restrict__ src, u32x4* __restrict__ dst, int R, int K,
                                                                      const bf16_t* __restrict__ A, const bf16_t* __restrict__ B, int rank,
                                                                      float scale, const bf16_t* __restrict__ gamma,
                                                                      const bf16_t* __restrict__ beta, float* __restrict__ c1, float* __restrict__ c2,
                                                                      int spans) {
#pragma clang fp contract(off)  // scale * t and the addition to W round separately, as stated
    constexpr int U = kMergeBlocks;
    static_assert(!TILED || LORA == LORA_NONE, "tiles hold merged weights");
    __shared__ float red[2][kMergeWaves][32];
    __shared__ u32x4 vec[kMergeWaves][4 * U];  // a wavefront's gamma, then beta, of the blocks at hand
    __shared__ float bs[LORA == LORA_LDS ? 32 : 1][kMergeRanks + 1];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, half = lane >> 5;
    const int KB = K >> 4, tile = FOLD ? blockIdx.x : blockIdx.x / spans;
    // the wavefront's blocks (the bounds are the same for all of its lanes; there may be none)
    const int kb0 = FOLD ? (int)((long)wave * KB / kMergeWaves) : min(((int)(blockIdx.x % spans) * kMergeWaves + wave) * U, KB);
    const int kb1 = FOLD ? (int)((long)(wave + 1) * KB / kMergeWaves) : min(kb0 + U, KB);
    const int rounds = FOLD ? ((KB + kMergeWaves - 1) / kMergeWaves + U - 1) / U : 1;  // ... U at a time, the most that any wavefront has
    const int r = tile * 32 + (lane & 31), rr = min(r, R - 1);
    u32x4* out = dst + (size_t)tile * KB * 64 + lane;
    struct Round { u32x4 w[U], v; };
    auto load = [&](Round& q, int kb) {  // (past the share: its last block, not used)
        if (kb >= kb1) return;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = min(kb + u, kb1 - 1);
            q.w[u] = TILED ? out[(size_t)k * 64] : *reinterpret_cast<const u32x4*>(src + (size_t)rr * K + k * 16 + 8 * half);
        }
        if (FOLD) q.v = reinterpret_cast<const u32x4*>(lane & 2 * U ? beta : gamma)[min(2 * kb + (lane & (2 * U - 1)), 2 * kb1 - 1)];
    };
    Round cur;
    float a1 = 0.f, a2 = 0.f;
    for (int round = 0; round < rounds; ++round) {
        const int kb = kb0 + round * U, nb = min(U, kb1 - kb);
        [[maybe_unused]] f32x32 t = {};
        // (the adapter's first values ahead of the weights: loads return in order, and its products need not wait for them)
        if constexpr (LORA == LORA_NONE) load(cur, kb);
        if constexpr (LORA == LORA_NONE && !FOLD) {  // (all four loads before the first of them is used)
#pragma unroll
            for (int u = 0; u < U; ++u) asm volatile("" : "+v"(cur.w[u]));
        }
        if constexpr (LORA != LORA_NONE) {
            // accumulator 4 q + e of a lane belongs to column 8 q + 4 (lane / 32) + e of the instruction: that is fed column
            // 16 (q / 2) + 8 (lane / 32) + 4 (q % 2) + e of the matrix
            const int i = lane & 31, col = 32 * half + 16 * (i >> 4) + 8 * ((i >> 2) & 1) + 4 * ((i >> 3) & 1) + (i & 3);
            const bf16_t* ap = A + min(kb * 16 + col, K - 1);  // (past the matrix: its last column, not used)
            const bf16_t* bp = B + (size_t)rr * rank;
            constexpr int G = 8;                               // ranks whose values are requested together
            if constexpr (LORA == LORA_LDS) {
                bf16_t aj[G], an[G];
                auto load_a = [&](bf16_t (&v)[G], int j0) {
#pragma unroll
                    for (int x = 0; x < G; ++x) v[x] = ap[(size_t)min(j0 + x, rank - 1) * K];
                };
                load_a(aj, 0);
                load(cur, kb);
                for (int j0 = 0; j0 < rank; j0 += kMergeRanks) {  // (every wavefront, with blocks left or not: there are barriers)
                    const int n = min(kMergeRanks, rank - j0);
                    if (round == 0 || rank > kMergeRanks) {
                        if (round || j0) __syncthreads();
                        for (int x = threadIdx.x; x < 32 * kMergeRanks; x += 64 * kMergeWaves) {
                            const int br = x / kMergeRanks, j = x % kMergeRanks;
                            if (j < n) bs[br][j] = bf16_to_f32(B[(size_t)min(tile * 32 + br, R - 1) * rank + j0 + j]);
                        }
                        __syncthreads();
                    }
                    for (int j = 0; j < n; j += G) {
                        if (j0 + j + G < rank) load_a(an, j0 + j + G);
#pragma unroll
                        for (int x = 0; x < G; ++x) {
                            if (j + x >= n) break;
                            t = __builtin_amdgcn_mfma_f32_32x32x1f32(bf16_to_f32(aj[x]), bs[lane & 31][j + x], t, 0, 0, 0);
                        }
#pragma unroll
                        for (int x = 0; x < G; ++x) aj[x] = an[x];
                    }
                }
            } else if (nb > 0) {
                for (int j0 = 0; j0 < rank; j0 += G) {
                    bf16_t aj[G], bj[G];
                    u32x4 b8;
                    if constexpr (LORA == LORA_WIDE) b8 = *reinterpret_cast<const u32x4*>(bp + j0);
#pragma unroll
                    for (int x = 0; x < G; ++x) {
                        const int j = min(j0 + x, rank - 1);
                        aj[x] = ap[(size_t)j * K];
                        if constexpr (LORA == LORA_FEW) bj[x] = bp[j];
                    }
                    if (j0 == 0) load(cur, kb);
                    const uint32_t bw[4] = {b8.x, b8.y, b8.z, b8.w};
#pragma unroll
                    for (int x = 0; x < G; ++x) {
                        if (LORA == LORA_FEW && j0 + x >= rank) break;
                        const float bv = LORA == LORA_WIDE ? (x & 1 ? bf_hi(bw[x >> 1]) : bf_lo(bw[x >> 1])) : bf16_to_f32(bj[x]);
                        t = __builtin_amdgcn_mfma_f32_32x32x1f32(bf16_to_f32(aj[x]), bv, t, 0, 0, 0);
                    }
                }
            }
        }
        if (FOLD && lane < 4 * U) vec[wave][lane] = cur.v;
        __builtin_amdgcn_wave_barrier();  // (a wavefront's LDS operations are in order)
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (u < nb) {
                u32x4 h = cur.w[u];
                if constexpr (LORA != LORA_NONE) {
                    const uint32_t ww[4] = {h.x, h.y, h.z, h.w};
                    uint32_t o[4];
#pragma unroll
                    for (int x = 0; x < 4; ++x) {
                        const float s0 = scale * t[8 * u + 2 * x], s1 = scale * t[8 * u + 2 * x + 1];  // plain operators: the pragma above covers them
                        const float lo = bf_lo(ww[x]) + s0;
                        const float hi = bf_hi(ww[x]) + s1;
                        o[x] = pack2_bf16(lo, hi);  // the merged weight is a bf16 value ...
                    }
                    h = u32x4{o[0], o[1], o[2], o[3]};
                }
                if constexpr (!TILED) {
                    h = bf16x8_to_half(h);  // ... held as a half like every other weight; rows past the matrix are zeros
                    if (r >= R) h = u32x4{0u, 0u, 0u, 0u};
                    __builtin_nontemporal_store(h, out + (size_t)(kb + u) * 64);
                }
                if constexpr (FOLD) {
                    const u32x4 g = vec[wave][2 * u + half], b = vec[wave][2 * U + 2 * u + half];
                    const uint32_t ww[4] = {h.x, h.y, h.z, h.w}, gg[4] = {g.x, g.y, g.z, g.w}, bb[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
                    for (int x = 0; x < 4; ++x) {
                        const float w0 = half_lo(ww[x]), w1 = half_hi(ww[x]);
                        a1 = fmaf(w0, bf_lo(gg[x]), a1);
                        a1 = fmaf(w1, bf_hi(gg[x]), a1);
                        a2 = fmaf(w0, bf_lo(bb[x]), a2);
                        a2 = fmaf(w1, bf_hi(bb[x]), a2);
                    }
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
    if constexpr (FOLD) {
        a1 = lane_sum32_apart(a1);
        a2 = lane_sum32_apart(a2);
        if (lane < 32) { red[0][wave][lane] = a1; red[1][wave][lane] = a2; }
        __syncthreads();
        if (threadIdx.x < 64) {
            float sum = 0.f;
#pragma unroll
            for (int x = 0; x < kMergeWaves; ++x) sum += red[half][x][lane & 31];
            (half ? c2 : c1)[tile * 32 + (lane & 31)] = sum;
        }
    }
}

// ----------------------------------------------------------------- 8-bit weight storage
//
// Row n of a weight matrix is kept as E4M3 codes q[n][:] and a power-of-two scale 2^e[n], e[n] the
// smallest integer with max|W[n][:]| 2^-e[n] <= 448; q = nearest E4M3 value of W 2^-e (ties to even).
// Scaling by a power of two is exact, so the codes are a rounding decision on the weights' own values.

// one wavefront per row: e[n] and 2^e[n]
__global__ __launch_bounds__(256) void row_exp_kernel(const bf16_t* __restrict__ src, int R, int K, int* __restrict__ exps,
                                                      float* __restrict__ scales) {
    const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (row >= R) return;
    float amax = 0.f;
    for (int k = lane * 8; k < K; k += 512) {
        const u32x4 v = *reinterpret_cast<const u32x4*>(src + (size_t)row * K + k);
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            amax = fmaxf(amax, fabsf(bf_lo(w[j])));
            amax = fmaxf(amax, fabsf(bf_hi(w[j])));
        }
    }
    for (int o = 32; o > 0; o >>= 1) amax = fmaxf(amax, __shfl_xor(amax, o));
    if (lane == 0) {
        int x = 0, e = 0;
        if (amax > 0.f) {
            const float f = frexpf(amax, &x);  // amax = f 2^x, f in [0.5, 1); 448 = 0.875 2^9
            e = f <= 0.875f ? x - 9 : x - 8;
        }
        exps[row] = e;
        scales[row] = ldexpf(1.0f, e);
    }
}

// eight bf16 values (one 16-byte load) -> eight E4M3 codes
__device__ __forceinline__ uint2 quant8_e4m3(const u32x4& v, float inv_scale) {
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
    float f[8];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        f[2 * j] = bf_lo(w[j]) * inv_scale;
        f[2 * j + 1] = bf_hi(w[j]) * inv_scale;
    }
    int lo = 0, hi = 0;
    lo = __builtin_amdgcn_cvt_pk_fp8_f32(f[0], f[1], lo, false);
    lo = __builtin_amdgcn_cvt_pk_fp8_f32(f[2], f[3], lo, true);
    hi = __builtin_amdgcn_cvt_pk_fp8_f32(f[4], f[5], hi, false);
    hi = __builtin_amdgcn_cvt_pk_fp8_f32(f[6], f[7], hi, true);
    return make_uint2((uint32_t)lo, (uint32_t)hi);
}

// row-major codes (a utility, and what the tests compare bit for bit)
__global__ void quant_rows_kernel(const bf16_t* __restrict__ src, const int* __restrict__ exps, uint2* __restrict__ codes,
                                  int R, int K) {
    const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (size_t)R * (K / 8)) return;
    const int row = (int)(idx / (K / 8));
    codes[idx] = quant8_e4m3(reinterpret_cast<const u32x4*>(src)[idx], ldexpf(1.0f, -exps[row]));
}

// codes in the half-tile kernel's units: [R/16][K/64][64 lanes][16 bytes]
__global__ void quant_units_kernel(const bf16_t* __restrict__ src, const int* __restrict__ exps, u32x4* __restrict__ dst,
                                   int R, int K, size_t total) {
    const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= total) return;
    const int KQ = K >> 6;
    const int lane = (int)(idx & 63);
    const int j = (int)((idx >> 6) % KQ), g = (int)((idx >> 6) / KQ);
    const int row = g * 16 + (lane & 15), k0 = j * 64 + 8 * (lane >> 4);
    u32x4 out = u32x4{0u, 0u, 0u, 0u};
    if (row < R) {
        const float inv = ldexpf(1.0f, -exps[row]);
        const uint2 a = quant8_e4m3(*reinterpret_cast<const u32x4*>(src + (size_t)row * K + k0), inv);
        const uint2 b = quant8_e4m3(*reinterpret_cast<const u32x4*>(src + (size_t)row * K + k0 + 32), inv);
        out = u32x4{a.x, a.y, b.x, b.y};
    }
    dst[idx] = out;
}

// units -> the half 32x16 blocks the tiled GEMMs read (a dequantised weight q 2^e has four significant bits: exact
// as a half down to 2^-24, which only rows whose largest weight is below 448 * 2^-15 = 0.014 can undercut)
__global__ void dequant_units_kernel(const u32x4* __restrict__ units, const float* __restrict__ scales,
                                     u32x4* __restrict__ dst, int R, int K, size_t total) {
    const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= total) return;
    const int KB = K >> 4, KQ = K >> 6;
    const int lane = (int)(idx & 63);
    const int kb = (int)((idx >> 6) % KB), rt = (int)((idx >> 6) / KB);
    const int row = rt * 32 + (lane & 31), k0 = kb * 16 + 8 * (lane >> 5);
    u32x4 out = u32x4{0u, 0u, 0u, 0u};
    if (row < R) {
        const int g = row >> 4, j = k0 >> 6, off = k0 & 63;
        const u32x4 u = units[((size_t)g * KQ + j) * 64 + 16 * ((off & 31) >> 3) + (row & 15)];
        const uint32_t c0 = off & 32 ? u.z : u.x, c1 = off & 32 ? u.w : u.y;
        const float sc = scales[row];
        typedef float f32x2 __attribute__((ext_vector_type(2)));
        const f32x2 f0 = __builtin_amdgcn_cvt_pk_f32_fp8(c0, false), f1 = __builtin_amdgcn_cvt_pk_f32_fp8(c0, true);
        const f32x2 f2 = __builtin_amdgcn_cvt_pk_f32_fp8(c1, false), f3 = __builtin_amdgcn_cvt_pk_f32_fp8(c1, true);
        out = u32x4{pack2(f0.x * sc, f0.y * sc), pack2(f1.x * sc, f1.y * sc), pack2(f2.x * sc, f2.y * sc),
                    pack2(f3.x * sc, f3.y * sc)};
    }
    dst[idx] = out;
}

}  // namespace

// ------------------------------------------------------------------ launchers

size_t bf16_tiled_bytes(int rows, int K) { return (size_t)((rows + 31) / 32) * (K / 16) * 1024; }

size_t fp8_units_bytes(int rows, int K) { return (size_t)((rows + 15) / 16) * (K / 64) * 1024; }

void fp8_row_exponents(hipStream_t s, const void* src, int R, int K, int* exps, float* scales) {
    row_exp_kernel<<<(R + 3) / 4, 256, 0, s>>>((const bf16_t*)src, R, K, exps, scales);
}

void fp8_quant_rows(hipStream_t s, const void* src, const int* exps, void* codes, int R, int K) {
    const size_t total = (size_t)R * (K / 8);
    quant_rows_kernel<<<(unsigned)((total + 255) / 256), 256, 0, s>>>((const bf16_t*)src, exps, (uint2*)codes, R, K);
}

void fp8_quant_units(hipStream_t s, const void* src, const int* exps, void* units, int R, int K) {
    const size_t total = (size_t)((R + 15) / 16) * (K / 64) * 64;
    quant_units_kernel<<<(unsigned)((total + 255) / 256), 256, 0, s>>>((const bf16_t*)src, exps, (u32x4*)units, R, K, total);
}

void fp8_dequant_units(hipStream_t s, const void* units, const float* scales, void* dst_blocks, int R, int K) {
    const size_t total = (size_t)((R + 31) / 32) * (K / 16) * 64;
    dequant_units_kernel<<<(unsigned)((total + 255) / 256), 256, 0, s>>>((const u32x4*)units, scales, (u32x4*)dst_blocks, R, K,
                                                                        total);
}

// dst: the tiles, written, or (src null) read
template <bool FOLD>
static void launch_tile_merge(hipStream_t s, const void* src, void* dst, int R, int K, const void* A, const void* B, int rank, float scale,
                              const void* gamma, const void* beta, float* c1, float* c2) {
    const int spans = FOLD ? 1 : (K / 16 + kMergeSpan - 1) / kMergeSpan, grid = (R + 31) / 32 * spans;
    auto launch = [&](auto kernel) {
        kernel<<<grid, 64 * kMergeWaves, 0, s>>>((const bf16_t*)src, (u32x4*)dst, R, K, (const bf16_t*)A, (const bf16_t*)B, rank, scale,
                                                 (const bf16_t*)gamma, (const bf16_t*)beta, c1, c2, spans);
    };
    if (A && B && rank > 0) {
        if (rank % 8 == 0 && (reinterpret_cast<uintptr_t>(B) & 15) == 0) launch(tile_merge_kernel<LORA_WIDE, FOLD, false>);
        else if (rank <= 8) launch(tile_merge_kernel<LORA_FEW, FOLD, false>);
        else launch(tile_merge_kernel<LORA_LDS, FOLD, false>);
    } else if (!FOLD || src) launch(tile_merge_kernel<LORA_NONE, FOLD, false>);
    else if constexpr (FOLD) launch(tile_merge_kernel<LORA_NONE, true, true>);
}

void bf16_tile_fold(hipStream_t s, const void* src, void* dst, int R, int K, const void* A, const void* B, int rank, float scale,
                    const void* gamma, const void* beta, float* c1, float* c2) {
    launch_tile_merge<true>(s, src, dst, R, K, A, B, rank, scale, gamma, beta, c1, c2);
}

void bf16_tile_rows(hipStream_t s, const void* src, void* dst, int R, int K) {
    launch_tile_merge<false>(s, src, dst, R, K, nullptr, nullptr, 0, 0.f, nullptr, nullptr, nullptr, nullptr);
}

void bf16_tile_rows_lora(hipStream_t s, const void* src, void* dst, int R, int K, const void* A, const void* B, int rank,
                         float scale) {
    launch_tile_merge<false>(s, src, dst, R, K, A, B, rank, scale, nullptr, nullptr, nullptr, nullptr);
}
