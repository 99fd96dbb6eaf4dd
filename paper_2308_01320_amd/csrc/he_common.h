// Internal definitions shared by the engine and its kernels (not part of the ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

typedef uint16_t bf16_t;  // raw bfloat16: the upper 16 bits of an IEEE float
typedef uint16_t half_t;  // raw IEEE half (what the bf16 path's matrix-core operands and KV cache hold)

// Device-resident generation state.  Every kernel reads positions, step
// numbers and sampling parameters from here rather than from launch
// arguments, so a captured decode step can be replayed unchanged.
struct he_dev_state {
    int cur_len;       // positions already in the KV cache, per sequence (uniform batches)
    int step;          // generation step n of the token about to be sampled
    int mode;          // 0 greedy, 1 Gumbel-max
    float temperature;
    uint32_t seed_lo, seed_hi;
    int ragged;        // 1: sequences differ in length -- per-sequence numbers live in seq[]
    int max_batch;
    int eos_id, pad_id;  // end-of-sequence stop (eos_id < 0: none) and the filler written after it
    int n_active;      // sequences that have not produced eos_id yet
    int arrivals;      // workgroups of the step's last kernel that are done with this state (zero between launches)
    int reserved[4];
    // [0 .. max_batch): cached positions of sequence b;  [max_batch .. 2 max_batch): left padding of
    // the rows now going through the model (0 outside a prompt pass);  [2 .. 3 max_batch): 1 once the
    // sequence has produced eos_id;  [3 .. 4 max_batch): tokens produced so far;  [4 .. 5 max_batch): the
    // sequence whose token goes through row r of a decode step (r itself, until he_generate_ragged drops the
    // rows of sequences that have ended)
    int seq[1];
};

__host__ __device__ inline size_t he_dev_state_bytes(int max_batch) {
    return sizeof(he_dev_state) + (size_t)5 * max_batch * sizeof(int);
}
// positions of sequence b already in the cache
__device__ __forceinline__ int seq_len(const he_dev_state* st, int b) { return st->ragged ? st->seq[b] : st->cur_len; }
// leading rows of sequence b in this pass that are padding, not tokens
__device__ __forceinline__ int row_pad(const he_dev_state* st, int b) { return st->ragged ? st->seq[st->max_batch + b] : 0; }
__device__ __forceinline__ bool seq_done(const he_dev_state* st, int b) {
    return st->ragged && st->seq[2 * st->max_batch + b] != 0;
}
// The sequence of row m of a pass of S rows per sequence.  Rows of a decode step (S = 1) go through the map;
// cache slot, per-sequence state, sampling noise and outputs belong to the sequence, activations to the row.
__device__ __forceinline__ int row_seq(const he_dev_state* st, int m, int S) {
    if (S != 1) return m / S;
    return st->ragged ? st->seq[4 * st->max_batch + m] : m;
}

// Sampling parameters that come with a step: stored by its first kernel, which does not read them.  start: the step is a
// prompt pass over sequences of one length, which begins at position 0 and generation step 0 whatever the state holds (a
// captured pass is replayed with the state its last replay left); its first kernel stores that as well and, because its other
// workgroups may look before or after, reads nothing of the state.  (Ragged passes: set_ragged_kernel.)
struct he_step_sampling { int set, mode; float temperature; uint32_t seed_lo, seed_hi; int start; };
__device__ __forceinline__ void store_sampling(he_dev_state* st, const he_step_sampling& sp) {
    if (sp.set) { st->mode = sp.mode; st->temperature = sp.temperature; st->seed_lo = sp.seed_lo; st->seed_hi = sp.seed_hi; }
    if (sp.start) { st->cur_len = 0; st->step = 0; st->ragged = 0; }
}

// End of a pass that fed `tokens` rows per sequence (padding included) and sampled `steps` tokens; by a whole workgroup.
__device__ __forceinline__ void advance_state(he_dev_state* st, int tokens, int steps) {
    if (st->ragged) {
        const int mb = st->max_batch;
        for (int b = threadIdx.x; b < mb; b += blockDim.x) {
            if (!st->seq[2 * mb + b]) st->seq[b] += tokens - st->seq[mb + b];
            st->seq[mb + b] = 0;
        }
    }
    if (threadIdx.x == 0) {
        st->cur_len += tokens;
        st->step += steps;
    }
}
// The same at the end of a kernel of many workgroups (a launch of its own for these few words costs 5 us): each counts itself
// in once it has used what it read of the state -- the values went into addresses of stores that were issued before --
// and whoever is last advances it.  All threads call it.
__device__ __forceinline__ void advance_state_by_last(he_dev_state* st, int tokens, int steps) {
    __shared__ int last;
    __syncthreads();
    if (gridDim.x == 1) {  // nobody to wait for
        advance_state(st, tokens, steps);
        return;
    }
    if (threadIdx.x == 0) {
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        last = __hip_atomic_fetch_add(&st->arrivals, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (int)gridDim.x - 1;
    }
    __syncthreads();
    if (!last) return;
    advance_state(st, tokens, steps);
    if (threadIdx.x == 0) __hip_atomic_store(&st->arrivals, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ---- sums and maxima over lanes
//
// Data-parallel moves inside the vector unit: some ten cycles a step, where a shuffle goes through LDS (a hundred).  The last
// steps of the kernels are chains of these.  Every lane of the wavefront takes part.
// The lane l ^ 8 of a row of 16, l ^ 16 and l ^ 32 for any values; xor_1/2 likewise; the two mirrors stand for l ^ 4 and l ^ 8 where
// the four (eight) lanes below already hold the same value.
template <int CTRL>
__device__ __forceinline__ float lane_dpp(float v) {
    return __uint_as_float((uint32_t)__builtin_amdgcn_mov_dpp((int)__float_as_uint(v), CTRL, 0xF, 0xF, false));
}
__device__ __forceinline__ float lane_xor1(float v) { return lane_dpp<0xB1>(v); }          // quad_perm [1, 0, 3, 2]
__device__ __forceinline__ float lane_xor2(float v) { return lane_dpp<0x4E>(v); }          // quad_perm [2, 3, 0, 1]
__device__ __forceinline__ float lane_mirror8(float v) { return lane_dpp<0x141>(v); }      // l ^ 7
__device__ __forceinline__ float lane_mirror16(float v) { return lane_dpp<0x140>(v); }     // l ^ 15
__device__ __forceinline__ float lane_xor8(float v) { return lane_dpp<0x128>(v); }         // row_ror 8
// v of the lower and of the upper lane of the pair (l, l ^ 16) or (l, l ^ 32)
struct LanePair { float lo, hi; };
__device__ __forceinline__ LanePair lane_pair16(float v) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return {__uint_as_float(r[0]), __uint_as_float(r[1])};
}
__device__ __forceinline__ LanePair lane_pair32(float v) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return {__uint_as_float(r[0]), __uint_as_float(r[1])};
}
__device__ __forceinline__ float lane_sum16_apart(float v) { const LanePair p = lane_pair16(v); return p.lo + p.hi; }
__device__ __forceinline__ float lane_sum32_apart(float v) { const LanePair p = lane_pair32(v); return p.lo + p.hi; }
__device__ __forceinline__ float lane_max16_apart(float v) { const LanePair p = lane_pair16(v); return fmaxf(p.lo, p.hi); }
__device__ __forceinline__ float lane_max32_apart(float v) { const LanePair p = lane_pair32(v); return fmaxf(p.lo, p.hi); }
// over the N lanes of an aligned group (all of them get it)
template <int N>
__device__ __forceinline__ float lane_sum(float v) {
    if (N >= 2) v += lane_xor1(v);
    if (N >= 4) v += lane_xor2(v);
    if (N >= 8) v += lane_mirror8(v);
    if (N >= 16) v += lane_mirror16(v);
    if (N >= 32) v = lane_sum16_apart(v);
    if (N >= 64) v = lane_sum32_apart(v);
    return v;
}
template <int N>
__device__ __forceinline__ float lane_max(float v) {
    if (N >= 2) v = fmaxf(v, lane_xor1(v));
    if (N >= 4) v = fmaxf(v, lane_xor2(v));
    if (N >= 8) v = fmaxf(v, lane_mirror8(v));
    if (N >= 16) v = fmaxf(v, lane_mirror16(v));
    if (N >= 32) v = lane_max16_apart(v);
    if (N >= 64) v = lane_max32_apart(v);
    return v;
}
// over the lanes N (8, 16 or 32) apart
template <int N>
__device__ __forceinline__ float lane_sum_apart(float v) {
    if (N <= 8) v += lane_xor8(v);
    if (N <= 16) v = lane_sum16_apart(v);
    if (N <= 32) v = lane_sum32_apart(v);
    return v;
}

__device__ __forceinline__ float bf16_to_f32(bf16_t v) { return __uint_as_float(((uint32_t)v) << 16); }

// Two floats -> two bf16 in one word (first argument in the low half), round to nearest, ties to even:
// the hardware's packed conversion, one instruction for the pair.
__device__ __forceinline__ uint32_t f32x2_to_bf16x2(float lo, float hi) {
    typedef float he_f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 he_bf16x2 __attribute__((ext_vector_type(2)));
    const he_f32x2 v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, he_bf16x2));
}
__device__ __forceinline__ bf16_t f32_to_bf16(float f) { return (bf16_t)(f32x2_to_bf16x2(f, 0.f) & 0xFFFFu); }

__device__ __forceinline__ float ld_f32(const float* p, size_t i) { return p[i]; }
__device__ __forceinline__ float ld_f32(const bf16_t* p, size_t i) { return bf16_to_f32(p[i]); }
__device__ __forceinline__ void st_val(float* p, size_t i, float v) { p[i] = v; }
__device__ __forceinline__ void st_val(bf16_t* p, size_t i, float v) { p[i] = f32_to_bf16(v); }

// ---- Philox-4x32-10 (Salmon et al., SC'11): word 0 for counter (v, n, b, 0), key = seed ----
__device__ __forceinline__ uint32_t philox_word0(uint32_t v, uint32_t n, uint32_t b, uint32_t k0, uint32_t k1) {
    uint32_t c0 = v, c1 = n, c2 = b, c3 = 0u;
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        // (64-bit products: one multiplication instruction for both halves)
        const uint64_t p0 = (uint64_t)0xD2511F53u * c0, p1 = (uint64_t)0xCD9E8D57u * c2;
        const uint32_t hi0 = (uint32_t)(p0 >> 32), lo0 = (uint32_t)p0, hi1 = (uint32_t)(p1 >> 32), lo1 = (uint32_t)p1;
        const uint32_t n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
        c0 = n0; c1 = lo1; c2 = n2; c3 = lo0;
        k0 += 0x9E3779B9u; k1 += 0xBB67AE85u;
    }
    return c0;
}

// Gumbel noise for vocabulary id v: u = ((x >> 9) + 1/2) 2^-23 lies strictly in (0,1)
__device__ __forceinline__ float gumbel_from_word(uint32_t x) {
    const float u = ((float)(x >> 9) + 0.5f) * 1.1920928955078125e-07f;  // 2^-23
    return -logf(-logf(u));
}

// KV arena: [layer][k|v][max_batch][head][max_seq_len][head_dim]
__host__ __device__ __forceinline__ size_t kv_index(int layer, int kv, int b, int h, int t, int max_batch, int n_heads,
                                                    int max_seq, int d) {
    return ((((size_t)(layer * 2 + kv) * max_batch + b) * n_heads + h) * max_seq + t) * (size_t)d;
}
