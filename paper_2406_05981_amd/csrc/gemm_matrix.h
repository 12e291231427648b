// The matrix-core forms of the layer for batches: what the entry points of
// shiftadd.hip need to choose and launch them (gemm_mx.hip, gemm_mfma.hip).
#ifndef SHIFTADD_GEMM_MATRIX_H
#define SHIFTADD_GEMM_MATRIX_H

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "shiftadd.h"

namespace sa_matrix {

struct Args {
    const uint16_t* x;         // activations [B][K]
    const uint8_t* packed;     // planes, packed layout
    const int8_t* exps;        // row-wise [q][N][K/G]; additive [q][N][K/G][T]
    const int8_t* term_signs;  // additive [q][N][K/G][T]
    int q, N, K, G, B, terms;  // terms = 0: row-wise
    void* y;                   // [B][N] fp32, or binary16 when out_half
    int out_half;
};

constexpr double kNever = 1e30;

// A 128-column block J lies in exponent group (J * magic) >> 32 (0: one block per
// group): J / d exactly while J * d < 2^32, d = G / 128 (K is at most 2^22).
inline uint32_t group_magic(int G) {
    const uint32_t d = (uint32_t)(G / 128);
    return d == 1 ? 0u : (uint32_t)(((1ull << 32) + d - 1) / d);
}

__device__ inline int group_of(int J, uint32_t magic) {
    return magic ? (int)__umulhi((uint32_t)J, magic) : J;
}

}  // namespace sa_matrix

// plan(): the estimated time (us) of a call with at most 4 planes, batch >= 2 and
// group % 128 == 0, and its geometry; kNever where the form does not take it.
// launch(): the call with that geometry.
namespace sa_mx {
double plan(int q, int N, int K, int G, int B, int terms, sa_matrix_plan* p);
void launch(const sa_matrix::Args& a, const sa_matrix_plan& p, hipStream_t s);
}  // namespace sa_mx

namespace sa_mfma {
double plan(int q, int N, int K, int G, int B, int terms, sa_matrix_plan* p);
void launch(const sa_matrix::Args& a, const sa_matrix_plan& p, hipStream_t s);
}  // namespace sa_mfma

#endif
