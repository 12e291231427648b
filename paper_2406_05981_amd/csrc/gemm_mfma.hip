// The layer for larger batches on the binary16 matrix cores (gfx950).
//
//   y[b][n] = sum_i sum_g 2^e[i][n][g] * sum_{k in g} s_i[n][k] x[b][k]
//
// For a batch the inner sums are a contraction of +-1 planes with binary16
// activations, and v_mfma_f32_16x16x32_f16 computes them as they are stated:
// the products +-x are exact, the sums are fp32, and each 128-column sum is
// multiplied by its row's power of two in fp32 before it is added up.  The
// planes stay packed in memory (one bit per weight) and are expanded to +-1.0
// in registers, two VALU operations per two weights.
//
// Two kernels with the same tiles: k_gemm_split shares a row's columns among
// the waves of a workgroup (few batch rows: the rows alone would not fill the
// chip), k_gemm_tile shares the activations of a workgroup through LDS (many
// batch rows: an expanded plane serves up to 64 of them).  2-norm error against
// 64 bits at most the table kernel's on ordinary activations (4096x4096 q=3 batch 16
// 7.9e-8 against 8.9e-8, 8001x512 q=4 batch 60 5.8e-8 against 5.9e-8); with massive
// outliers (x1000) on fewer than 1700 columns up to 1.14 times it.
//
// Measured against the table batch kernel (us, graph replay, weights rotated
// over 300 MB): split: 4096x4096 q=3 batch 16 13.3 -> 7.6, batch 32 21.4 -> 10.4,
// 11008x4096 q=2 batch 16 20.7 -> 11.5, 28672x8192 batch 16 122 -> 60, additive
// factors of two terms 4096x11008 q=2 batch 16 26.2 -> 19.1; tile: 11003x4096 q=3
// batch 250 345 -> 81.5, 11008x4096 q=2 batch 128 132 -> 46, 4096x11008 q=4 batch
// 256 450 -> 148.
// What bounds them (counters, share of SIMD cycles): the split kernel latency --
// VALU instructions 27-29%, matrix cores 5-6%, and its waves wait 42% (11008x4096
// q=2 batch 16) to 65% (4096x11008) of their cycles: activations are requested
// one 128-column block ahead, 0.2-0.4 us of work at two waves a SIMD.  The tile
// kernel (4096x4096 q=3 batch 250) issues VALU in 26% and keeps the matrix cores
// busy 18% of the cycles at one workgroup a CU: a block's LDS reads, products and
// barrier follow each other.  k_gemm_tile<3, 4, 4> spills 10 registers (44 bytes a
// lane) to stay at three waves a SIMD; without that cap 11003x4096 batch 250 takes
// 88 us.
#include "gemm_matrix.h"
#include "keys.h"

namespace sa_mfma {
namespace {

using sa_matrix::Args;

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef float float4_t __attribute__((ext_vector_type(4)));

constexpr int kWaves = 8;          // split kernel
constexpr int kThreads = 64 * kWaves;
constexpr int kTileWaves = 4;      // tile kernel
constexpr int kTileThreads = 64 * kTileWaves;
constexpr int kTile = 16;          // rows and batch rows of one MFMA tile
constexpr int kGroupBlocks = 4;    // 128-column blocks per group: one 16-byte key load per lane

struct KernelArgs {
    Args a;
    int row_wgs, col_wgs;  // grid
    int ksplit;            // split kernel: waves that share the columns (power of two)
    int NG;                // exponent groups of a row
    uint32_t group_magic;  // sa_matrix::group_magic
    int vec;               // the exponents of 4 consecutive blocks load as one word (or two)
};

// Word b of the result holds byte b of the four words.
__device__ inline void transpose_bytes(uint32_t w[4]) {
    const uint32_t p01 = __builtin_amdgcn_perm(w[1], w[0], 0x05010400u);
    const uint32_t q01 = __builtin_amdgcn_perm(w[1], w[0], 0x07030602u);
    const uint32_t p23 = __builtin_amdgcn_perm(w[3], w[2], 0x05010400u);
    const uint32_t q23 = __builtin_amdgcn_perm(w[3], w[2], 0x07030602u);
    w[0] = __builtin_amdgcn_perm(p23, p01, 0x05040100u);
    w[1] = __builtin_amdgcn_perm(p23, p01, 0x07060302u);
    w[2] = __builtin_amdgcn_perm(q23, q01, 0x05040100u);
    w[3] = __builtin_amdgcn_perm(q23, q01, 0x07060302u);
}

// 4x4 transpose between the four 16-lane groups and the four words: on entry
// lane group p holds the words 0..3 of block p, on return word g of block b is
// w[b] of lane group g.
__device__ inline void transpose4(uint32_t w[4]) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const auto s = __builtin_amdgcn_permlane32_swap(w[i], w[i + 2], false, false);
        w[i] = s[0];
        w[i + 2] = s[1];
    }
#pragma unroll
    for (int i = 0; i < 4; i += 2) {
        const auto s = __builtin_amdgcn_permlane16_swap(w[i], w[i + 1], false, false);
        w[i] = s[0];
        w[i + 1] = s[1];
    }
}

// The 32 signs of a key word as +-1.0 halves: register t holds (column t,
// column 16 + t) of the word's 32 columns.  A bit at position 10..14 of a half
// is the binary16 value 2^-14, 2^-13, 2^-11, 2^-7 or 2, so one AND and one
// packed fma (bit * 2 / value - 1, exact) give both signs of a register; the
// bit at position 15 is the sign bit itself.  Two shifted copies of the word
// bring every bit to one of these positions.
__device__ inline void expand(uint32_t w, half2_t out[16]) {
    const half2_t one = {(_Float16)1.0f, (_Float16)1.0f};
    // bits 10..15 of w are columns 10..15; of w << 6 columns 4..9; of w << 12 columns 0..3
    const uint32_t src[3] = {w << 12, w << 6, w};
#pragma unroll
    for (int t = 0; t < 16; ++t) {
        const int s = t < 4 ? 0 : t < 10 ? 1 : 2;
        const int pos = t < 4 ? t + 12 : t < 10 ? t + 6 : t;
        if (pos == 15) {
            out[t] = __builtin_bit_cast(half2_t, (src[s] & 0x80008000u) ^ 0xBC00BC00u);
        } else {
            const float mul = pos == 10 ? 32768.0f : pos == 11 ? 16384.0f : pos == 12 ? 4096.0f
                              : pos == 13 ? 256.0f : 1.0f;
            const half2_t m = {(_Float16)mul, (_Float16)mul};
            const half2_t b = __builtin_bit_cast(half2_t, src[s] & (0x00010001u << pos));
            out[t] = __builtin_elementwise_fma(b, m, -one);
        }
    }
}

__device__ inline half8_t cat(half2_t a, half2_t b, half2_t c, half2_t d) {
    return half8_t{a[0], a[1], b[0], b[1], c[0], c[1], d[0], d[1]};
}

// Activations of one block for this lane: four chunks of one batch row,
// re-paired so that register t holds (column t, column 16 + t).
__device__ inline void pair_columns(const uint4 raw[4], uint32_t out[16]) {
    const uint32_t d[16] = {raw[0].x, raw[0].y, raw[0].z, raw[0].w, raw[1].x, raw[1].y,
                            raw[1].z, raw[1].w, raw[2].x, raw[2].y, raw[2].z, raw[2].w,
                            raw[3].x, raw[3].y, raw[3].z, raw[3].w};
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        out[2 * i] = __builtin_amdgcn_perm(d[8 + i], d[i], 0x05040100u);
        out[2 * i + 1] = __builtin_amdgcn_perm(d[8 + i], d[i], 0x07060302u);
    }
}

// ---------------------------------------------------------------- columns shared by waves

// One group (4 blocks) of RT row tiles: keys as loaded, exponents of the four blocks.
template <int Q, int RT, bool ADD>
struct Group {
    uint4 w[RT][Q];
    // exponents: row-wise a byte per block of one word, additive T bytes per block
    uint32_t e[RT][Q][ADD ? 4 : 1];
    uint32_t s[RT][Q][ADD ? 4 : 1];  // additive: T term signs per block
};

// Work split.  A workgroup owns 16*RT*(8/ksplit) rows and 16 batch rows;
// `ksplit` of its waves share the input dimension, wave k taking the
// 512-column groups k, k + ksplit, ..., and the other factor of the 8 waves
// takes further rows.  No partial sum leaves a workgroup: the ksplit waves'
// sums meet in LDS and are added in wave order (deterministic).
//
// Tiles.  One MFMA is 16 batch rows x 16 rows x 32 columns with the
// activations as the first operand, so that a lane's four results belong to
// one row and take one exponent.  The order of the columns inside a block is
// free as long as both operands agree: lane group g holds the block's chunks g,
// 4 + g, 8 + g and 12 + g (so that a load of activations touches 64 contiguous
// bytes a row), and register t the pair (t, 16 + t) of those 32 columns, which
// is what a key word masked with one constant gives (expand).
//
// Loads.  A lane reads 16 key bytes of one row in one of the group's four
// blocks (256-byte runs); the bytes are put in chunk order, transposed in the
// lane and then between the lane groups, in registers.  The block loop stays
// rolled: its code runs four times a group and would be fetched cold.  The next group's keys are requested
// before the current group's products; activations one block ahead.
template <int Q, int RT, bool ADD>
__device__ __forceinline__ void split_body(const KernelArgs& ka, float* red) {
    const Args& a = ka.a;
    constexpr int kE = ADD ? 4 : 1;
    const int C = a.K >> 3, C16 = C >> 4, NG = ka.NG;
    auto group_of = [&](int J) { return sa_matrix::group_of(J, ka.group_magic); };
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int r = lane & 15, g = lane >> 4;
    // workgroups are dealt to the 8 XCDs round-robin; the batch tiles of a row
    // range land on one XCD and share its L2
    const int xcd = (int)blockIdx.x & 7, idx = (int)blockIdx.x >> 3;
    const int row_wg = xcd + 8 * (idx / ka.col_wgs), col_wg = idx % ka.col_wgs;
    if (row_wg >= ka.row_wgs) return;  // whole workgroup: padding of the grid
    const int ksl = wave & (ka.ksplit - 1), rset = wave / ka.ksplit;
    const int sets = kWaves / ka.ksplit;
    const int row0 = kTile * RT * (row_wg * sets + rset);  // first row of this wave
    const int b0 = kTile * col_wg;
    const int groups = (C16 + kGroupBlocks - 1) / kGroupBlocks;

    float4_t tot[RT];
#pragma unroll
    for (int t = 0; t < RT; ++t) tot[t] = float4_t{0.0f, 0.0f, 0.0f, 0.0f};

    // this lane's row in each tile (rows past N repeat the last one)
    int n[RT];
    uint32_t key_off[RT];  // of block 0; block J adds 16 * J * R
    int key_step[RT];      // bytes per block: 16 * R
#pragma unroll
    for (int t = 0; t < RT; ++t) {
        n[t] = imin(row0 + kTile * t + r, a.N - 1);
        const int T = n[t] >> 6;
        key_step[t] = 16 * imin(64, a.N - 64 * T);
        key_off[t] = (uint32_t)(64 * T * C + 16 * (n[t] & 63));
    }
    const uint16_t* xrow = a.x + (int64_t)imin(b0 + r, a.B - 1) * a.K + 8 * g;

    auto load_group = [&](int jg, Group<Q, RT, ADD>& k) {
        const int J0 = kGroupBlocks * jg;
        const int J = imin(J0 + g, C16 - 1);
#pragma unroll
        for (int t = 0; t < RT; ++t) {
            const uint32_t off = key_off[t] + (uint32_t)(J * key_step[t]);
#pragma unroll
            for (int i = 0; i < Q; ++i) {
                const int64_t erow = ((int64_t)i * a.N + n[t]) * NG;
                if constexpr (ADD) {
                    if (ka.vec) {  // two terms: the 8 bytes of 4 blocks at once
                        const uint2 e = *reinterpret_cast<const uint2*>(a.exps + (erow + J0) * 2);
                        const uint2 s =
                            *reinterpret_cast<const uint2*>(a.term_signs + (erow + J0) * 2);
                        k.e[t][i][0] = e.x & 0xffffu;
                        k.e[t][i][1] = e.x >> 16;
                        k.e[t][i][2] = e.y & 0xffffu;
                        k.e[t][i][3] = e.y >> 16;
                        k.s[t][i][0] = s.x & 0xffffu;
                        k.s[t][i][1] = s.x >> 16;
                        k.s[t][i][2] = s.y & 0xffffu;
                        k.s[t][i][3] = s.y >> 16;
                    } else
#pragma unroll
                    for (int b = 0; b < 4; ++b) {
                        const int64_t eo = (erow + group_of(imin(J0 + b, C16 - 1))) * a.terms;
                        k.e[t][i][b] = load_terms(a.exps + eo, a.terms);
                        k.s[t][i][b] = load_terms(a.term_signs + eo, a.terms);
                    }
                } else {
                    const uint8_t* p = reinterpret_cast<const uint8_t*>(a.exps) + erow;
                    if (ka.vec) {
                        k.e[t][i][0] = *reinterpret_cast<const uint32_t*>(p + J0);
                    } else {
                        uint32_t e = 0;
#pragma unroll
                        for (int b = 0; b < 4; ++b)
                            e |= (uint32_t)p[group_of(imin(J0 + b, C16 - 1))] << (8 * b);
                        k.e[t][i][0] = e;
                    }
                }
                k.w[t][i] =
                    *reinterpret_cast<const uint4*>(a.packed + (size_t)i * a.N * C + off);
            }
        }
    };
    auto load_x = [&](int J, uint4 (&raw)[4]) {
        const uint16_t* p = xrow + 128 * (int64_t)imin(J, C16 - 1);
#pragma unroll
        for (int d = 0; d < 4; ++d) raw[d] = *reinterpret_cast<const uint4*>(p + 32 * d);
    };

    if (ksl < groups) {
        Group<Q, RT, ADD> k;
        uint4 raw[4];
        load_group(ksl, k);
        load_x(kGroupBlocks * ksl, raw);
        for (int jg = ksl; jg < groups; jg += ka.ksplit) {
            const int next = jg + ka.ksplit < groups ? jg + ka.ksplit : jg;
            // the words of block 0, 1, 2, 3 and their exponents, taken one block
            // after the other from index 0
            uint32_t kw[RT][Q][4], e[RT][Q][kE], s[RT][Q][kE];
#pragma unroll
            for (int t = 0; t < RT; ++t)
#pragma unroll
                for (int i = 0; i < Q; ++i) {
                    rotate16(k.w[t][i], 16 - r, kw[t][i]);
                    transpose_bytes(kw[t][i]);
                    transpose4(kw[t][i]);
#pragma unroll
                    for (int b = 0; b < kE; ++b) {
                        e[t][i][b] = k.e[t][i][b];
                        s[t][i][b] = k.s[t][i][b];
                    }
                }
            if (next != jg) load_group(next, k);
            const int nb = imin(kGroupBlocks, C16 - kGroupBlocks * jg);
#pragma unroll 1
            for (int b = 0; b < nb; ++b) {
                uint32_t p[16];
                pair_columns(raw, p);
                half8_t X[4];
#pragma unroll
                for (int m = 0; m < 4; ++m)
                    X[m] = cat(__builtin_bit_cast(half2_t, p[4 * m]),
                               __builtin_bit_cast(half2_t, p[4 * m + 1]),
                               __builtin_bit_cast(half2_t, p[4 * m + 2]),
                               __builtin_bit_cast(half2_t, p[4 * m + 3]));
                if (b + 1 < nb || next != jg)
                    load_x(b + 1 < nb ? kGroupBlocks * jg + b + 1 : kGroupBlocks * next, raw);
#pragma unroll
                for (int t = 0; t < RT; ++t) {
                    // a block's planes and terms first: shorter chains of additions
                    float sum[4];
#pragma unroll
                    for (int i = 0; i < Q; ++i) {
                        half2_t A[16];
                        expand(kw[t][i][0], A);
                        float4_t acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                        for (int m = 0; m < 4; ++m)
                            acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                                X[m], cat(A[4 * m], A[4 * m + 1], A[4 * m + 2], A[4 * m + 3]), acc,
                                0, 0, 0);
                        if constexpr (ADD) {
#pragma unroll
                            for (int u = 0; u < SA_MAX_TERMS; ++u) {
                                if (u >= a.terms) break;
                                // sign 0: no term, whatever its exponent byte or the
                                // activations hold (a select: 0 * inf is a NaN)
                                const float sg = (float)(int8_t)(s[t][i][0] >> (8 * u));
                                const float f = ldexpf(sg, (int)(int8_t)(e[t][i][0] >> (8 * u)));
#pragma unroll
                                for (int v = 0; v < 4; ++v) {
                                    const float z = i == 0 && u == 0 ? 0.0f : sum[v];
                                    sum[v] = sg != 0.0f ? fmaf(acc[v], f, z) : z;
                                }
                            }
                        } else {
                            const float f = ldexpf(1.0f, (int)(int8_t)e[t][i][0]);
#pragma unroll
                            for (int v = 0; v < 4; ++v)
                                sum[v] = i == 0 ? acc[v] * f : fmaf(acc[v], f, sum[v]);
                        }
#pragma unroll
                        for (int d = 0; d < 3; ++d) kw[t][i][d] = kw[t][i][d + 1];
                        if constexpr (ADD) {
#pragma unroll
                            for (int d = 0; d < 3; ++d) {
                                e[t][i][d] = e[t][i][d + 1];
                                s[t][i][d] = s[t][i][d + 1];
                            }
                        } else {
                            e[t][i][0] >>= 8;
                        }
                    }
#pragma unroll
                    for (int v = 0; v < 4; ++v) tot[t][v] += sum[v];
                }
            }
        }
    }

    // sums of the ksplit waves, added in wave order: red[wave][t][v][lane]
    constexpr int kVals = RT * 256;
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) red[wave * kVals + (t * 4 + v) * 64 + lane] = tot[t][v];
    __syncthreads();
    for (int o = threadIdx.x; o < sets * kVals; o += kThreads) {
        const int set = o / kVals, q = o - set * kVals;
        const int l = q & 63, v = (q >> 6) & 3, t = q >> 8;
        const int row = kTile * RT * (row_wg * sets + set) + kTile * t + (l & 15);
        const int b = b0 + 4 * (l >> 4) + v;
        if (row < a.N && b < a.B) {
            const float* p = red + set * ka.ksplit * kVals + q;
            float s = p[0];
            for (int w = 1; w < ka.ksplit; ++w) s += p[w * kVals];
            if (a.out_half)
                static_cast<uint16_t*>(a.y)[(int64_t)b * a.N + row] =
                    __builtin_bit_cast(uint16_t, (_Float16)s);
            else
                static_cast<float*>(a.y)[(int64_t)b * a.N + row] = s;
        }
    }
}

template <int Q, int RT, bool ADD>
__global__ __launch_bounds__(kThreads, RT == 1 && Q <= (ADD ? 2 : 3) ? 4 : 2)
void k_gemm_split(KernelArgs a) {
    __shared__ float red[kWaves * RT * 256];
    split_body<Q, RT, ADD>(a, red);
}

// ---------------------------------------------------------------- activations shared in LDS
//
// Four waves are RW row tiles times 4 / RW shares of the columns; a wave has 16
// rows and all 16 * CT batch rows of the workgroup.  The activations of one
// 128-column block lie in LDS in operand order, double buffered: the next
// block's are loaded before a block's products and written, re-paired, after
// them, one barrier a block.  A block's planes are expanded once and multiplied
// by every column tile.  Up to 3 planes the kernel is held to three waves a SIMD:
// reading a column tile ahead and adding one behind hides the LDS reads but costs
// that third wave (11003x4096 q=3 batch 250: 80 us as it is, 88 with them).
template <int Q>
struct TileKeys {
    uint4 w[Q];
    uint32_t e[Q];  // exponents of the group's four blocks, a byte each
};

template <int Q, int CT, int RW>
__device__ __forceinline__ void tile_body(const KernelArgs& ka, uint4* xbuf) {
    const Args& a = ka.a;
    constexpr int KW = kTileWaves / RW;
    constexpr int kBuf = CT * 256;  // uint4 of one block's operand: [ct][m][lane]
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int r = lane & 15, g = lane >> 4;
    const int rw = wave % RW, kw = wave / RW;
    const int C = a.K >> 3, C16 = C >> 4, NG = ka.NG;
    const int groups = (C16 + kGroupBlocks - 1) / kGroupBlocks;
    const int gper = (groups + KW - 1) / KW;  // groups of a column share
    const int blk0 = imin(kGroupBlocks * gper * kw, C16);
    const int blk1 = imin(blk0 + kGroupBlocks * gper, C16);
    const int xcd = (int)blockIdx.x & 7, idx = (int)blockIdx.x >> 3;
    const int row_wg = xcd + 8 * (idx / ka.col_wgs);
    if (row_wg >= ka.row_wgs) return;  // whole workgroup: padding of the grid
    const int row0 = kTile * (RW * row_wg + rw), b0 = kTile * CT * (idx % ka.col_wgs);

    const int n = imin(row0 + r, a.N - 1);
    const int T = n >> 6, R = imin(64, a.N - 64 * T);
    const uint32_t key_off = (uint32_t)(64 * T * C + 16 * (n & 63));
    auto load_keys = [&](int J0, TileKeys<Q>& k) {
        const uint32_t off = key_off + (uint32_t)(16 * imin(J0 + g, C16 - 1) * R);
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            const uint8_t* p =
                reinterpret_cast<const uint8_t*>(a.exps) + ((int64_t)i * a.N + n) * NG;
            if (ka.vec) {
                k.e[i] = *reinterpret_cast<const uint32_t*>(p + J0);
            } else {
                uint32_t e = 0;
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    const int J = imin(J0 + b, C16 - 1);
                    e |= (uint32_t)p[sa_matrix::group_of(J, ka.group_magic)] << (8 * b);
                }
                k.e[i] = e;
            }
        }
#pragma unroll
        for (int i = 0; i < Q; ++i)
            k.w[i] = *reinterpret_cast<const uint4*>(a.packed + (size_t)i * a.N * C + off);
    };

    // this wave stages the column tiles rw, rw + RW, ... of its column share
    constexpr int kStage = (CT + RW - 1) / RW;
    const uint16_t* xrow[kStage];
#pragma unroll
    for (int t = 0; t < kStage; ++t)
        xrow[t] = a.x + (int64_t)imin(b0 + kTile * (rw + RW * t) + r, a.B - 1) * a.K + 8 * g;
    uint4 raw[kStage][4];
    auto load_x = [&](int J) {
#pragma unroll
        for (int t = 0; t < kStage; ++t)
            if (rw + RW * t < CT)
#pragma unroll
                for (int d = 0; d < 4; ++d)
                    raw[t][d] = *reinterpret_cast<const uint4*>(xrow[t] + 128 * (int64_t)J + 32 * d);
    };
    uint4* xk = xbuf + kw * 2 * kBuf;
    auto store_x = [&](int buf) {
#pragma unroll
        for (int t = 0; t < kStage; ++t)
            if (rw + RW * t < CT) {
                uint32_t p[16];
                pair_columns(raw[t], p);
                uint4* o = xk + buf * kBuf + (rw + RW * t) * 256 + lane;
#pragma unroll
                for (int m = 0; m < 4; ++m)
                    o[64 * m] = uint4{p[4 * m], p[4 * m + 1], p[4 * m + 2], p[4 * m + 3]};
            }
    };

    // the sums of one group, and over the groups: shorter chains of fp32 additions
    float4_t part[CT], tot[CT];
#pragma unroll
    for (int c = 0; c < CT; ++c) part[c] = tot[c] = float4_t{0.0f, 0.0f, 0.0f, 0.0f};

    TileKeys<Q> k;
    uint32_t w[Q][4], e[Q];
    if (blk0 < blk1) {
        load_x(blk0);
        load_keys(blk0, k);
        store_x(0);
    }
    __syncthreads();
    // every wave runs the same number of steps: the barriers match
    const int steps = kGroupBlocks * gper;
#pragma unroll 1
    for (int s = 0; s < steps; ++s) {
        const int J = blk0 + s;
        const bool next = J + 1 < blk1;
        if (next) load_x(J + 1);
        if (J < blk1) {
            if ((s & 3) == 0) {
#pragma unroll
                for (int i = 0; i < Q; ++i) {
                    rotate16(k.w[i], 16 - r, w[i]);
                    transpose_bytes(w[i]);
                    transpose4(w[i]);
                    e[i] = k.e[i];
                    asm volatile("" : "+v"(w[i][0]), "+v"(w[i][1]), "+v"(w[i][2]), "+v"(w[i][3]),
                                      "+v"(e[i]));
                }
                if (J + 4 < blk1) load_keys(J + 4, k);
            }
            half2_t A[Q][16];
            float f[Q];
#pragma unroll
            for (int i = 0; i < Q; ++i) {
                expand(w[i][0], A[i]);
                f[i] = ldexpf(1.0f, (int)(int8_t)e[i]);
                e[i] >>= 8;
#pragma unroll
                for (int d = 0; d < 3; ++d) w[i][d] = w[i][d + 1];
            }
            const uint4* xs = xk + (s & 1) * kBuf + lane;
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                half8_t X[4];
#pragma unroll
                for (int m = 0; m < 4; ++m)
                    X[m] = __builtin_bit_cast(half8_t, xs[(4 * c + m) * 64]);
                float4_t acc[Q];
#pragma unroll
                for (int m = 0; m < 4; ++m)
#pragma unroll
                    for (int i = 0; i < Q; ++i)
                        acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                            X[m], cat(A[i][4 * m], A[i][4 * m + 1], A[i][4 * m + 2], A[i][4 * m + 3]),
                            m == 0 ? float4_t{0.0f, 0.0f, 0.0f, 0.0f} : acc[i], 0, 0, 0);
                // a block's planes first: shorter chains of additions
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    float sum = acc[0][v] * f[0];
#pragma unroll
                    for (int i = 1; i < Q; ++i) sum = fmaf(acc[i][v], f[i], sum);
                    part[c][v] += sum;
                }
            }
            if ((s & 3) == 3 || J + 1 == blk1) {
#pragma unroll
                for (int c = 0; c < CT; ++c) {
                    tot[c] += part[c];
                    part[c] = float4_t{0.0f, 0.0f, 0.0f, 0.0f};
                }
            }
        }
        if (next) store_x((s + 1) & 1);
        __syncthreads();
    }

    if constexpr (KW > 1) {
        // the column shares' sums, added in order by the first share's waves
        float* red = reinterpret_cast<float*>(xbuf);
        constexpr int kVals = CT * 256;
#pragma unroll
        for (int c = 0; c < CT; ++c)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                red[(kw * RW + rw) * kVals + (c * 4 + v) * 64 + lane] = tot[c][v];
        __syncthreads();
        if (kw > 0) return;
#pragma unroll
        for (int c = 0; c < CT; ++c)
#pragma unroll
            for (int v = 0; v < 4; ++v)
#pragma unroll
                for (int u = 1; u < KW; ++u)
                    tot[c][v] += red[(u * RW + rw) * kVals + (c * 4 + v) * 64 + lane];
    }
    const int row = row0 + r;
    if (row >= a.N) return;
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int b = b0 + kTile * c + 4 * g + v;
            if (b < a.B) {
                if (a.out_half)
                    static_cast<uint16_t*>(a.y)[(int64_t)b * a.N + row] =
                        __builtin_bit_cast(uint16_t, (_Float16)tot[c][v]);
                else
                    static_cast<float*>(a.y)[(int64_t)b * a.N + row] = tot[c][v];
            }
        }
}

template <int Q, int CT, int RW>
__global__ __launch_bounds__(kTileThreads, Q <= 3 ? 3 : 2) void k_gemm_tile(KernelArgs a) {
    __shared__ uint4 xbuf[(kTileWaves / RW) * 2 * CT * 256];
    tile_body<Q, CT, RW>(a, xbuf);
}

// ---------------------------------------------------------------- choice and launch

// Rounds of workgroups over the 256 CUs; a partial round counts half as a whole
// one, since several workgroups of a CU overlap.
double rounds(int64_t wgs) {
    const double r = (double)wgs / 256;
    if (r <= 1) return r;
    return 0.5 * (r + (double)((wgs + 255) / 256));
}

template <int RT, bool ADD>
void launch_split(const KernelArgs& ka, int grid, hipStream_t s) {
    const dim3 g(grid), b(kThreads);
    switch (ka.a.q) {
        case 1: hipLaunchKernelGGL((k_gemm_split<1, RT, ADD>), g, b, 0, s, ka); break;
        case 2: hipLaunchKernelGGL((k_gemm_split<2, RT, ADD>), g, b, 0, s, ka); break;
        case 3: hipLaunchKernelGGL((k_gemm_split<3, RT, ADD>), g, b, 0, s, ka); break;
        default:
            // (more row tiles with 4 planes would spill: plan())
            if constexpr (RT <= (ADD ? 1 : 3))
                hipLaunchKernelGGL((k_gemm_split<4, RT, ADD>), g, b, 0, s, ka);
            break;
    }
}

template <int CT, int RW>
void launch_tile(const KernelArgs& ka, int grid, hipStream_t s) {
    const dim3 g(grid), b(kTileThreads);
    switch (ka.a.q) {
        case 1: hipLaunchKernelGGL((k_gemm_tile<1, CT, RW>), g, b, 0, s, ka); break;
        case 2: hipLaunchKernelGGL((k_gemm_tile<2, CT, RW>), g, b, 0, s, ka); break;
        case 3: hipLaunchKernelGGL((k_gemm_tile<3, CT, RW>), g, b, 0, s, ka); break;
        default: hipLaunchKernelGGL((k_gemm_tile<4, CT, RW>), g, b, 0, s, ka); break;
    }
}

}  // namespace

// The kernel and tiles with the least estimated time.  Up to 4 planes (registers);
// the index bounds: exact division by multiplication (K), 32-bit key offsets (a
// plane holds fewer than 2^31 bytes).
// The estimates are fitted to every kernel's time on 2986 drawn layers of N
// 60..28672, K 128..28672, q 1..4, batch 2..256, weights rotated over 320 MB (5th
// and 95th percentile of estimate / measured: split 0.75 and 1.4, tile 0.82 and
// 1.2).  Split: a workgroup alone takes a latency per 512-column group of a wave
// (its activations are requested one 128-column block ahead), more of them on a CU
// their issue time.  Tile: the same per 128-column block of a column share.
// Row tiles that spill (4 planes x 4 tiles, additive 4 x 2) are left out.
double plan(int q, int N, int K, int G, int B, int terms, sa_matrix_plan* p) {
    *p = sa_matrix_plan{};
    const bool add = terms > 0;
    if (K > (1 << 22) || (add && B < 5)) return sa_matrix::kNever;
    double best = sa_matrix::kNever;
    auto offer = [&](double us, int kernel, int row_tiles, int col_tiles, int shares, int rows,
                     int threads, size_t lds) {
        if (us >= best) return;
        best = us;
        p->kernel = kernel;
        p->rows_per_wg = rows;
        p->batch_per_wg = kTile * col_tiles;
        p->workgroups = 8 * ((B + kTile * col_tiles - 1) / (kTile * col_tiles)) *
                        (((N + rows - 1) / rows + 7) / 8);
        p->threads = threads;
        p->row_tiles = row_tiles;
        p->col_tiles = col_tiles;
        p->column_shares = shares;
        p->lds_bytes = lds;
    };
    auto workgroups = [&](int rows, int col_tiles) {
        return (int64_t)((N + rows - 1) / rows) *
               ((B + kTile * col_tiles - 1) / (kTile * col_tiles));
    };
    const int blocks = K / 128, groups = (blocks + kGroupBlocks - 1) / kGroupBlocks;
    int ksplit = 1;
    while (ksplit < kWaves && ksplit < groups) ksplit *= 2;
    const int sets = kWaves / ksplit, per_wave = (groups + ksplit - 1) / ksplit;
    // the part of a wave's blocks that exist
    const double fill = (double)blocks / (kGroupBlocks * ksplit * per_wave);
    // base, alone (per group: least, fixed, per plane and row tile), shared (fixed, per
    // group, per plane and row tile; what a missing block saves): row-wise; one term,
    // two that load as words, two that do not, three, four
    static const double kSplit[6][8] = {
        {2.7, 2.4, 0.96, 1.1, 0.24, 0.89, 1.2, 0},   {1.7, 0.6, 1.5, 2.1, 1.5, 0, 3.3, 0.8},
        {2.6, 2.8, 1.0, 1.6, 1.4, 0.71, 1.9, 0.57},  {2.2, 3.2, 1.5, 1.6, 1.2, 0.3, 2.8, 1},
        {0, 1.4, 2.8, 3.8, 1.3, 0.46, 5.9, 0.94},    {0, 1, 2.3, 5.0, 3.1, 0, 8.7, 1}};
    const bool bytes = G != 128 || K % 512;
    const double* f = kSplit[!add ? 0 : terms == 1 ? 1 : terms == 2 ? 2 + bytes : terms + 1];
    for (int rt = 1; rt <= (add ? 2 : 4) && rt * q <= (add ? 6 : 12); ++rt) {
        const int rows = kTile * rt * sets, qr = q * rt;
        const double alone = f[2] + f[3] * qr;
        const double t0 = per_wave * (alone > f[1] ? alone : f[1]);
        const double t1 = rounds(workgroups(rows, 1)) *
                          (f[4] + per_wave * (f[5] + f[6] * qr) * (1 - f[7] * (1 - fill)));
        const double us = f[0] + (t0 > t1 ? t0 : t1);
        // the estimates of additive layers spread wider: 9% against them
        offer(add ? 1.09 * us : us, 2, rt, 1, ksplit, rows, kThreads,
              sizeof(float) * kWaves * rt * 256);
    }
    if (add) return best;
    struct Fit {
        int ct, rw;
        double base, alone, alone_q, shared, shared_q;
    };
    static const Fit kFit[] = {{1, 4, 2.7, 0.37, 0.15, 0.22, 0.13},
                               {2, 4, 3.0, 0.38, 0.19, 0.16, 0.21},
                               {4, 4, 3.6, 0.43, 0.30, 0.46, 0.22},
                               {1, 2, 3.1, 0.39, 0.17, 0.20, 0.15},
                               {2, 2, 3.5, 0.54, 0.17, 0.35, 0.17}};
    for (const Fit& f : kFit) {
        if (f.ct > 1 && B <= 8 * f.ct) continue;
        const int rows = kTile * f.rw, steps = (blocks * f.rw + kTileWaves - 1) / kTileWaves;
        const double t0 = steps * (f.alone + f.alone_q * q);
        const double t1 = rounds(workgroups(rows, f.ct)) * steps * (f.shared + f.shared_q * q);
        offer(f.base + (t0 > t1 ? t0 : t1), 3, f.rw, f.ct, kTileWaves / f.rw, rows, kTileThreads,
              sizeof(uint4) * (kTileWaves / f.rw) * 2 * f.ct * 256);
    }
    return best;
}

void launch(const Args& a, const sa_matrix_plan& p, hipStream_t s) {
    const bool add = a.terms > 0;
    KernelArgs ka{};
    ka.a = a;
    ka.row_wgs = (a.N + p.rows_per_wg - 1) / p.rows_per_wg;
    ka.col_wgs = (a.B + p.batch_per_wg - 1) / p.batch_per_wg;
    ka.ksplit = p.column_shares;
    ka.NG = a.K / a.G;
    ka.group_magic = sa_matrix::group_magic(a.G);
    const uintptr_t e = reinterpret_cast<uintptr_t>(a.exps) |
                        (add ? reinterpret_cast<uintptr_t>(a.term_signs) : 0);
    ka.vec = a.G == 128 && a.K % 512 == 0 && (e & (add ? 7u : 3u)) == 0 && (!add || a.terms == 2);
    const int grid = p.workgroups;
    if (p.kernel == 3) {
        if (p.row_tiles == 4) {
            if (p.col_tiles == 1) launch_tile<1, 4>(ka, grid, s);
            else if (p.col_tiles == 2) launch_tile<2, 4>(ka, grid, s);
            else launch_tile<4, 4>(ka, grid, s);
        } else {
            if (p.col_tiles == 1) launch_tile<1, 2>(ka, grid, s);
            else launch_tile<2, 2>(ka, grid, s);
        }
        return;
    }
    if (add) {
        if (p.row_tiles == 1) launch_split<1, true>(ka, grid, s);
        else launch_split<2, true>(ka, grid, s);
    } else if (p.row_tiles == 1) {
        launch_split<1, false>(ka, grid, s);
    } else if (p.row_tiles == 2) {
        launch_split<2, false>(ka, grid, s);
    } else if (p.row_tiles == 3) {
        launch_split<3, false>(ka, grid, s);
    } else {
        launch_split<4, false>(ka, grid, s);
    }
}

}  // namespace sa_mfma
