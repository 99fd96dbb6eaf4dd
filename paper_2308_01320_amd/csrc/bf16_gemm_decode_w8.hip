// bf16 path: the decode GEMMs on 8-bit weights.
#include "bf16_decode_kernels.h"

void bf16_gemm_units8(hipStream_t s, int mode, const void* Wp, const void* X, int M, int N, int K, int units, int ksplit,
                      const bf16_gemm_args& a) {
    const Epi p = make_epi(M, N, a);
    const int KB = K / 16, m_tiles = (M + 31) / 32;
    if (mode == EPI_STORE_LN) launch_half<MODE_STORE_LN, true>(s, Wp, X, KB, N / 16, m_tiles, units, ksplit, p);
    else if (mode == EPI_BIAS_RELU) launch_half<MODE_BIAS_RELU, true>(s, Wp, X, KB, N / 16, m_tiles, units, 1, p);
    else launch_half<MODE_QKV, true>(s, Wp, X, KB, N / 16, m_tiles, units, 1, p);
}
