// binary16 matrix-core form of the layer for larger batches (gemm_mfma.hip):
// what the entry points of shiftadd.hip need to choose and launch it.
#ifndef SHIFTADD_GEMM_MFMA_H
#define SHIFTADD_GEMM_MFMA_H

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sa_mfma {

struct Args {
    const uint16_t* x;         // activations [B][K]
    const uint8_t* packed;     // planes, packed layout
    const int8_t* exps;        // row-wise [q][N][K/G]; additive [q][N][K/G][T]
    const int8_t* term_signs;  // additive [q][N][K/G][T]
    int q, N, K, G, B, terms;  // terms = 0: row-wise
    void* y;                   // [B][N] fp32, or binary16 when out_half
    int out_half;
};

// Whether this form takes a call with row-wise or additive factors.
bool takes(int q, int N, int K, int G, int B, bool additive);

void launch(const Args& a, hipStream_t s);

}  // namespace sa_mfma

#endif
