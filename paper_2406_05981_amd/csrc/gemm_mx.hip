// The layer for a few batch rows on the block-scaled matrix cores (gfx950).
//
//   y[b][n] = sum_i sum_g 2^e[i][n][g] * sum_{k in g} s_i[n][k] x[b][k]
//
// v_mfma_scale_f32_16x16x128_f8f6f4 multiplies fp4 by fp8 operands in blocks of
// 32 columns, each block of each operand row with a power of two of its own.
// That is this layer's form: the planes are +-1.0 in fp4, one VALU operation per
// eight weights after a shift, and the factor 2^e of a (row, 128 columns) is
// the operand's block scale, so nothing is shifted or added outside the matrix
// core over the whole input dimension.
//
// Activations.  A binary16 activation is split into four fp8 (e4m3) pieces of
// four significand bits each, x = S (p0 + p1 / 2^5 + p2 / 2^10 + p3 / 2^15), S the
// power of two that brings the largest of 32 columns into [8, 16); the pieces are
// the four matrix columns of a batch row, so they cost no extra products.  The last
// piece's smallest step is 2^-24 S, below half of which bits are dropped: a block
// whose largest is below 16 loses none (2^-24 is binary16's own step), in any other
// block a value above 2^-17 of the largest is exact and the rest is off by at most
// 2^-28 of the largest, which fp32 sums with that largest do not resolve.
// The core adds products of eight consecutive columns in a window of 13 bits
// below the largest (measured: 2^8 + 2^-5 is kept, 2^8 + 2^-6 is not, further
// apart fp32); below 16 and down to e4m3's 2^-9 the pieces stay inside that
// window, so these sums are exact and everything after them is fp32.
// Measured against 64 bits (2-norm, 3 planes, batch 8, the table batch kernel's
// error in brackets): 4170x4096 N(0,1) 6.2e-8 (8.5e-8), four columns x1000 9.1e-8
// (1.1e-7), x30000 1.2e-7 (1.3e-7), 28672 columns 8.2e-8 (1.7e-7).  With three pieces
// 3.0e-7 at x16000; the fourth costs 8192x28672 batch 8 40.1 -> 44.3 us.
//
// What bounds it: per 16 rows x 128 columns x plane a SIMD needs 25 ns (batch <= 4: 8
// VALU operations and one MFMA), the table kernel's queries about 100.  VALU
// instructions take 56% of the SIMD cycles at 28672x8192 batch 8 and 60% at
// 8192x28672, where every workgroup splits all activations for two row tiles; the
// matrix cores are busy 23 and 16%, the LDS 12 and 28%, two thirds of it in bank
// conflicts of the 528-byte columns (counters).
// Measured against the table batch kernel (us, graph replay, weights rotated over
// 300 MB): 4096x4096 q=3 batch 2 7.8 -> 5.5, batch 4 7.8 -> 6.4; 28672x8192 batch 4
// 38.0 -> 24.4, batch 8 67.3 -> 32.0; 8192x28672 batch 8 68.1 -> 47.3; 11008x4096 q=4
// batch 8 23.3 -> 13.4; two terms 4096x11008 q=4 batch 8 32.2 -> 29.7.
#include <type_traits>

#include "gemm_matrix.h"
#include "keys.h"

namespace sa_mx {
namespace {

using sa_matrix::Args;

typedef int int4_t __attribute__((ext_vector_type(4)));
typedef int int8v_t __attribute__((ext_vector_type(8)));
typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef short short2_t __attribute__((ext_vector_type(2)));
typedef float float4_t __attribute__((ext_vector_type(4)));

constexpr int kWaves = 8;
constexpr int kThreads = 64 * kWaves;
constexpr int kTile = 16;
constexpr int kGroupBlocks = 4;   // 128-column blocks per group
constexpr int kPieces = 4;        // fp8 pieces of an activation
constexpr int kColBytes = 528;    // LDS bytes of one piece of one batch row over a group (512 + 16)
constexpr int kMaxTiles = 8;      // row tiles of one wave
// Factors above 2^100 (scale bytes above this one): sums over 512 columns and 4
// planes of |x| < 2^16 may leave fp32 before their terms cancel, and the byte of
// 2^127 is a NaN.  A wave that meets one runs its columns a second time for these
// factors alone, with activations scaled by 2^-kTopShift (28672x8192 q=3 batch 8:
// 43 us with one such factor, 64 us with exponents over all of int8, 34 without).
constexpr uint32_t kTopByte = 228;
constexpr int kTopShift = 64;

struct KernelArgs {
    Args a;
    int tiles;             // 16-row tiles, spread over (workgroup, row set)
    int shares;            // workgroups * row sets
    int ksplit;            // waves that share the columns (power of two <= kWaves)
    int sets;              // row sets of a workgroup: it has ksplit * sets waves
    int NG;                // exponent groups of a row
    uint32_t group_magic;  // sa_matrix::group_magic
};

// 32 signs as fp4 (e2m1) +-1.0: register v, nibble n holds bit 4n + v of the
// word.  A set bit is +1.0 (0010), a clear one -1.0 (1010); the masks of a
// negated term give the opposite, those of an absent one zero.
constexpr uint32_t kAnd = 0x88888888u, kXor = 0xAAAAAAAAu, kXorNeg = 0x22222222u;

__device__ inline int8v_t expand(uint32_t w, uint32_t and_mask = kAnd, uint32_t xor_mask = kXor) {
    int8v_t a = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int v = 0; v < 4; ++v) a[v] = (int)(((w << (3 - v)) & and_mask) ^ xor_mask);
    return a;
}

// Activations that are not finite stay out of the matrix core: what they add to an
// output follows from signs alone.  For batch row b the workgroup lists the chunks of
// 8 columns that hold one (masks of the columns that are +inf and -inf; a NaN is
// both), and every output of the row collects over the list which infinities reach
// it: bit 0 +inf, bit 1 -inf, both a NaN.  A lane stops at both, so a row full of them
// costs a few keys an output (28672x8192 q=3 batch 8: 41 us with one infinity, 41
// with a row of NaNs, 34 without).
struct Chunk {
    uint32_t c, masks;  // +inf columns | -inf columns << 8
};
struct ChunkList {
    uint32_t count;
    Chunk chunk[kThreads];
};

__device__ inline uint32_t infinity_masks(const uint4 v) {
    const uint32_t d[4] = {v.x, v.y, v.z, v.w};
    uint32_t m = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const uint32_t h = (d[j >> 1] >> (16 * (j & 1))) & 0xffffu;
        if (h == 0x7c00u || (h & 0x7fffu) > 0x7c00u) m |= 1u << j;
        if (h == 0xfc00u || (h & 0x7fffu) > 0x7c00u) m |= 256u << j;
    }
    return m;
}

// The infinities that reach output row n over the listed chunks, added to `f`.
template <bool ADD>
__device__ inline uint32_t collect(const Args& a, const ChunkList* list, int n, uint32_t f) {
    const int C = a.K >> 3, NG = a.K / a.G, r = n & 63;
    const int64_t first = n - r;
    const int R = imin(64, a.N - (n - r));
    const uint32_t count = list->count;
    for (uint32_t k = 0; k < count && f != 3; ++k) {
        const int c = (int)list->chunk[k].c;
        const uint32_t pos = list->chunk[k].masks & 0xffu, neg = list->chunk[k].masks >> 8;
        for (int i = 0; i < a.q; ++i) {
            const uint32_t key = a.packed[((int64_t)i * a.N + first) * C + 16 * r +
                                          (int64_t)(c >> 4) * 16 * R + ((c - r) & 15)];
            const bool p = (key & pos) | (~key & neg), m = (key & neg) | (~key & pos);
            const uint32_t plus = (uint32_t)p | (uint32_t)m << 1;
            if constexpr (ADD) {
                const uint32_t minus = (uint32_t)m | (uint32_t)p << 1;
                const int8_t* sg =
                    a.term_signs + (((int64_t)i * a.N + n) * NG + 8 * c / a.G) * a.terms;
                for (int u = 0; u < a.terms; ++u) f |= sg[u] > 0 ? plus : sg[u] < 0 ? minus : 0u;
            } else {
                f |= plus;
            }
        }
    }
    return f;
}

// Work split.  Every workgroup owns whole rows: its waves are ksplit shares of
// the input dimension (512-column groups ksl, ksl + ksplit, ...) times `sets`
// sets of row tiles, so no partial sum leaves a workgroup.  One 8-wave
// workgroup per CU: a second one would hide more latency but splits the
// activations once more (28672x8192 batch 4: 23.2 us against 26.7 with 512
// workgroups).  A wave splits the activations of its group into LDS that only
// it reads (no barrier), keeps them as matrix operands in registers and runs
// its row tiles through them, the next tile's keys requested before the
// current tile's products.  The loops stay rolled: a workgroup runs them few
// times and unrolled code would be fetched cold.
//
// Columns.  Lane (row r, block g) loads the 16 key bytes of one row and one of
// the group's four blocks, rotates them to chunk order, and step m multiplies
// 32 columns of each of the four blocks: register v, nibble n of the operand is
// bit 4n + v of key word m.  The activations are stored in that order; the
// second operand's lanes hold columns 16g..16g+15 and 64+16g.. of a step, which
// is half a block's 32 columns each.
template <int Q>
struct Keys {
    uint4 w[Q];
    uint32_t e[Q];  // exponent byte of this lane's row and block; additive: T bytes
    uint32_t s[Q];  // additive: T term signs
};

template <int Q, int CT, int NP, bool ADD>
__device__ __forceinline__ void body(const KernelArgs& ka, char* lds) {
    const Args& a = ka.a;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int ksl = wave & (ka.ksplit - 1);
    const int C = a.K >> 3, C16 = C >> 4, NG = ka.NG;
    const int groups = (C16 + kGroupBlocks - 1) / kGroupBlocks;

    // activations of this lane: 16 columns of batch rows (lane >> 5), + 2, + 4, ...
    const int xp = (lane >> 3) & 3, xm = (lane >> 1) & 3, xh = lane & 1;
    auto load_x = [&](int jg, uint4 (&raw)[NP][2]) {
        const int64_t off = 128 * (int64_t)imin(kGroupBlocks * jg + xp, C16 - 1) + 16 * (lane & 7);
#pragma unroll
        for (int t = 0; t < NP; ++t) {
            const uint16_t* p = a.x + (int64_t)imin(2 * t + (lane >> 5), a.B - 1) * a.K + off;
            raw[t][0] = *reinterpret_cast<const uint4*>(p);
            raw[t][1] = *reinterpret_cast<const uint4*>(p + 8);
        }
    };
    uint4 raw[NP][2];
    if (ksl < groups) load_x(ksl, raw);
    __builtin_amdgcn_sched_barrier(0);

    const int r = lane & 15, g = lane >> 4;
    const int sets = ka.sets, rset = wave / ka.ksplit;
    // row tiles of this wave: the first `extra` shares take one more
    const int share = (int)blockIdx.x * sets + rset;
    const int base = ka.tiles / ka.shares, extra = ka.tiles - base * ka.shares;
    const int ntiles = base + (share < extra ? 1 : 0);
    const int tile0 = share * base + imin(share, extra);

    // this wave's pieces [4 B][528 bytes], then its scales [B][4 blocks] words
    constexpr int kMaxB = 4 * CT;
    constexpr int kWaveBytes = kPieces * kMaxB * kColBytes + kMaxB * 16;
    char* px = lds + wave * kWaveBytes;
    char* ps = px + kPieces * kMaxB * kColBytes;

    auto load_keys = [&](int jg, int t, Keys<Q>& k) {
        const int n = imin(kTile * (tile0 + t) + r, a.N - 1);
        const int J = imin(kGroupBlocks * jg + g, C16 - 1);
        const uint32_t eoff = (uint32_t)(n * NG + sa_matrix::group_of(J, ka.group_magic));
        const int T = n >> 6, R = imin(64, a.N - 64 * T);
        const uint32_t off = (uint32_t)(64 * T * C + 16 * (n & 63) + 16 * J * R);
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            if constexpr (ADD) {
                const size_t o = ((size_t)i * a.N * NG + eoff) * a.terms;
                k.e[i] = load_terms(a.exps + o, a.terms);
                k.s[i] = load_terms(a.term_signs + o, a.terms);
            } else {
                k.e[i] = (reinterpret_cast<const uint8_t*>(a.exps) + (size_t)i * a.N * NG)[eoff];
            }
        }
#pragma unroll
        for (int i = 0; i < Q; ++i)
            k.w[i] = *reinterpret_cast<const uint4*>(a.packed + (size_t)i * a.N * C + off);
    };
    uint32_t not_finite = 0;  // batch rows with an activation that is not finite
    auto split_x = [&](int jg) {
        const bool in = kGroupBlocks * jg + xp < C16;
        const bool short_group = kGroupBlocks * (jg + 1) > C16;  // uniform
#pragma unroll
        for (int t = 0; t < NP; ++t) {
            const int b = 2 * t + (lane >> 5);
            uint32_t d[8] = {raw[t][0].x, raw[t][0].y, raw[t][0].z, raw[t][0].w,
                             raw[t][1].x, raw[t][1].y, raw[t][1].z, raw[t][1].w};
            if (short_group) {
#pragma unroll
                for (int u = 0; u < 8; ++u) d[u] = in ? d[u] : 0u;
            }
            // exponent field of the largest of the block's 32 columns
            auto largest = [&] {
                half2_t hm = {(_Float16)0.0f, (_Float16)0.0f};
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const half2_t h = __builtin_bit_cast(half2_t, d[u]);
                    hm = __builtin_elementwise_maximum(__builtin_elementwise_maximum(hm, h), -h);
                }
                uint32_t mx = __builtin_bit_cast(uint32_t, hm);
                mx = max(mx & 0x7fffu, (mx >> 16) & 0x7fffu);
                mx = max(mx, (uint32_t)__builtin_amdgcn_mov_dpp((int)mx, 0xB1, 0xf, 0xf, true));
                return max(mx >> 10, 1u);
            };
            uint32_t E = largest();
            // From 63488 on the first piece would round up past the binary16 range: a
            // block in the top binade is halved (exact but for subnormals, far below
            // the last piece's step) and only its scale byte keeps the exponent.
            if (__any(E >= 30u)) {
                if (E == 31u) not_finite |= 1u << b;
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    if ((d[u] & 0x7c00u) == 0x7c00u) d[u] &= 0xffff0000u;
                    if ((d[u] & 0x7c000000u) == 0x7c000000u) d[u] &= 0xffffu;
                }
                E = largest();
                const _Float16 f = E >= 30u ? (_Float16)0.5f : (_Float16)1.0f;
                const half2_t h = {f, f};
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    d[u] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(half2_t, d[u]) * h);
            }
            const uint32_t F = min(E, 29u);
            float S[kPieces];
#pragma unroll
            for (int p = 0; p < kPieces; ++p)
                S[p] = __builtin_bit_cast(float, (F + 109u - 5u * p) << 23);
            uint32_t out[kPieces][2][2];  // [piece][s][v & 1]
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int o = 0; o < 2; ++o) {
                    const uint32_t sel = o ? 0x07060302u : 0x05040100u;
                    // columns v = 2s + o and v + 4 of the lane's two chunks
                    const uint32_t c0 = __builtin_amdgcn_perm(d[2 + s], d[s], sel);
                    const uint32_t c1 = __builtin_amdgcn_perm(d[6 + s], d[4 + s], sel);
                    half2_t f0 = __builtin_bit_cast(half2_t, c0);
                    half2_t f1 = __builtin_bit_cast(half2_t, c1);
#pragma unroll
                    for (int p = 0; p < kPieces; ++p) {
                        short2_t w = {0, 0};
                        w = __builtin_amdgcn_cvt_scalef32_pk_fp8_f16(w, f0, S[p], false);
                        w = __builtin_amdgcn_cvt_scalef32_pk_fp8_f16(w, f1, S[p], true);
                        const int wi = __builtin_bit_cast(int, w);
                        out[p][s][o] = (uint32_t)wi;
                        if (p + 1 < kPieces) {
                            f0 -= __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(wi, S[p], false);
                            f1 -= __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(wi, S[p], true);
                        }
                    }
                }
            if (b < a.B) {
#pragma unroll
                for (int p = 0; p < kPieces; ++p)
#pragma unroll
                    for (int s = 0; s < 2; ++s) {
                        uint32_t* o = reinterpret_cast<uint32_t*>(
                            px + (kPieces * b + p) * kColBytes + (xm * 8 + xp * 2 + s) * 16 +
                            4 * xh);
                        o[0] = out[p][s][0];
                        o[2] = out[p][s][1];
                    }
                if (xh == 0)
                    *reinterpret_cast<uint8_t*>(ps + (b * 4 + xp) * 4 + xm) = (uint8_t)(E + 108u);
            }
        }
    };
    auto wave_fence = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };

    float tot[kMaxTiles][CT];
#pragma unroll
    for (int t = 0; t < kMaxTiles; ++t)
#pragma unroll
        for (int c = 0; c < CT; ++c) tot[t][c] = 0.0f;

    uint32_t top = 0;  // the largest scale byte
    const int passes = ksl < groups && ntiles > 0 ? 2 : 0;
#pragma unroll 1
    for (int pass = 0; pass < passes; ++pass) {
        Keys<Q> k;
        int jg0 = ksl, t0 = 0;
        // opaque: the addresses of the first loads are not kept over the passes
        asm volatile("" : "+s"(jg0), "+s"(t0));
        if (pass) {
            if (!__any(top > kTopByte)) break;
            load_x(jg0, raw);
        }
        load_keys(jg0, t0, k);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll 1
        for (int jg = ksl; jg < groups; jg += ka.ksplit) {
            const bool more = jg + ka.ksplit < groups;
            split_x(jg);
            wave_fence();
            if (more) load_x(jg + ka.ksplit, raw);
            // matrix column r is piece r & 3 of batch row r >> 2 (+ 4 per column
            // tile); columns of batch rows past the last repeat it
            int8v_t X[CT][4];
            uint32_t xs[CT];
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                const int b = imin(4 * c + (r >> 2), a.B - 1), piece = r & 3;
                const char* p = px + (kPieces * b + piece) * kColBytes + g * 16;
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    const int4_t lo = *reinterpret_cast<const int4_t*>(p + m * 128);
                    const int4_t hi = *reinterpret_cast<const int4_t*>(p + m * 128 + 64);
                    X[c][m] = int8v_t{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
                }
                xs[c] = *reinterpret_cast<const uint32_t*>(ps + (b * 4 + g) * 4) -
                        0x05050505u * (uint32_t)piece -
                        0x01010101u * (uint32_t)(pass * kTopShift);
            }
            // The scale byte of a factor in this pass.  In the other pass its byte is 0:
            // 2^-127 of its product beside the product itself, and nothing at all with
            // the activations of the second pass.
            auto scale = [&](uint32_t es) {
                top = max(top, es);
                return (es > kTopByte) == (pass != 0) ? es - (uint32_t)pass : 0u;
            };
#pragma unroll 1
            for (int t = 0; t < ntiles; ++t) {
                uint32_t w[Q][4], e[Q], sg[Q];
#pragma unroll
                for (int i = 0; i < Q; ++i) {
                    rotate16(k.w[i], 16 - r, w[i]);
                    if constexpr (ADD) {
                        e[i] = k.e[i] ^ 0x80808080u;
                        sg[i] = k.s[i];
                        asm volatile("" : "+v"(sg[i]));
                    } else {
                        e[i] = scale(k.e[i] ^ 0x80u);
                    }
                    asm volatile("" : "+v"(w[i][0]), "+v"(w[i][1]), "+v"(w[i][2]), "+v"(w[i][3]),
                                      "+v"(e[i]));
                }
                __builtin_amdgcn_sched_barrier(0);
                if (t + 1 < ntiles)
                    load_keys(jg, t + 1, k);
                else if (more)
                    load_keys(jg + ka.ksplit, 0, k);
                __builtin_amdgcn_sched_barrier(0);
                // Every 32 columns' products are 4 roundings of fp32 behind the largest,
                // so the chains are kept short: row-wise one accumulator a step, over
                // the planes; additive two, whose first piece (the others are 2^-5 of
                // it) is taken out after every term.
                constexpr int NA = ADD ? 2 : 4;
                float4_t acc[CT][NA];
                float first[CT];
                auto step = [&](auto mc, const int8v_t W, uint32_t es) {
                    constexpr int m = decltype(mc)::value;
#pragma unroll
                    for (int c = 0; c < CT; ++c)
                        acc[c][m % NA] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(
                            X[c][m], W, acc[c][m % NA], 0, 4, m, (int)xs[c], 0, (int)es);
                };
#pragma unroll
                for (int c = 0; c < CT; ++c) {
                    first[c] = 0.0f;
#pragma unroll
                    for (int d = 0; d < NA; ++d) acc[c][d] = float4_t{0.0f, 0.0f, 0.0f, 0.0f};
                }
#pragma unroll
                for (int i = 0; i < Q; ++i) {
                    if constexpr (ADD) {
                        // a term's sign goes into the expansion: no term, no weight
#pragma unroll 1
                        for (int u = 0; u < a.terms; ++u) {
                            const int s8 = (int)(int8_t)sg[i];
                            const uint32_t es = scale(s8 ? e[i] & 0xffu : 0x80u);
                            const uint32_t am = s8 ? kAnd : 0u;
                            const uint32_t xm8 = s8 ? (s8 < 0 ? kXorNeg : kXor) : 0u;
                            step(std::integral_constant<int, 0>{}, expand(w[i][0], am, xm8), es);
                            step(std::integral_constant<int, 1>{}, expand(w[i][1], am, xm8), es);
                            step(std::integral_constant<int, 2>{}, expand(w[i][2], am, xm8), es);
                            step(std::integral_constant<int, 3>{}, expand(w[i][3], am, xm8), es);
                            e[i] >>= 8;
                            sg[i] >>= 8;
#pragma unroll
                            for (int c = 0; c < CT; ++c) {
                                first[c] += acc[c][0][0] + acc[c][1][0];
                                acc[c][0][0] = acc[c][1][0] = 0.0f;
                            }
                        }
                    } else {
                        step(std::integral_constant<int, 0>{}, expand(w[i][0]), e[i]);
                        step(std::integral_constant<int, 1>{}, expand(w[i][1]), e[i]);
                        step(std::integral_constant<int, 2>{}, expand(w[i][2]), e[i]);
                        step(std::integral_constant<int, 3>{}, expand(w[i][3]), e[i]);
                    }
                }
                // a lane's results are the pieces of one (row, batch row)
#pragma unroll
                for (int c = 0; c < CT; ++c) {
                    float4_t s = acc[c][0] + acc[c][1];
                    if constexpr (!ADD) s += acc[c][2] + acc[c][3];
                    float v = ((s[3] + s[2]) + s[1]) + (s[0] + first[c]);
                    if (pass) v = ldexpf(v, kTopShift + 1);
#pragma unroll
                    for (int u = 0; u < kMaxTiles; ++u)
                        if (u == t) tot[u][c] += v;
                }
            }
            wave_fence();
        }
    }

    // the waves' sums meet in LDS, red[wave][t][c][lane], and are added in wave order
    uint32_t inf = 0;  // of this lane's outputs: two bits each, in the order of the last loop
    const int klog = __builtin_ctz(ka.ksplit);
    if (__syncthreads_or(not_finite != 0)) {
        ChunkList* list = reinterpret_cast<ChunkList*>(lds);
        for (int b = 0; b < a.B; ++b) {
            if (!__syncthreads_or((not_finite >> b) & 1u)) continue;
            for (int c0 = 0; c0 < C; c0 += (int)blockDim.x) {
                if (threadIdx.x == 0) list->count = 0;
                __syncthreads();
                const int c = c0 + (int)threadIdx.x;
                if (c < C) {
                    const uint32_t m = infinity_masks(
                        *reinterpret_cast<const uint4*>(a.x + (int64_t)b * a.K + 8 * c));
                    if (m) list->chunk[atomicAdd(&list->count, 1u)] = {(uint32_t)c, m};
                }
                __syncthreads();
                for (int t = 0; t < ntiles; ++t) {
                    const int o = t * CT + (b >> 2), row = kTile * (tile0 + t) + r;
                    if ((o & (ka.ksplit - 1)) != ksl || g != (b & 3) || row >= a.N) continue;
                    const int at = 2 * (o >> klog);
                    inf |= collect<ADD>(a, list, row, (inf >> at) & 3u) << at;
                }
                __syncthreads();
            }
        }
    }
    float* red = reinterpret_cast<float*>(lds);
    constexpr int kVals = kMaxTiles * CT * 64;
#pragma unroll
    for (int t = 0; t < kMaxTiles; ++t)
        if (t < ntiles)
#pragma unroll
            for (int c = 0; c < CT; ++c)
                red[wave * kVals + (t * CT + c) * 64 + lane] = tot[t][c];
    __syncthreads();
    // outputs of this wave's row set: its ksplit waves take every ksplit-th vector
    for (int o = ksl; o < ntiles * CT; o += ka.ksplit) {
        const int t = o / CT, c = o - t * CT;
        const int row = kTile * (tile0 + t) + r, b = 4 * c + g;
        const float* v = red + rset * ka.ksplit * kVals + o * 64 + lane;
        float p[kWaves];
#pragma unroll
        for (int w = 0; w < kWaves; ++w) p[w] = w < ka.ksplit ? v[w * kVals] : 0.0f;
        float y = p[0];
#pragma unroll
        for (int w = 1; w < kWaves; ++w) y += p[w];
        if (row < a.N && b < a.B) {
            const uint32_t f = (inf >> (2 * (o >> klog))) & 3u;
            if (f & 1u) y += __builtin_inff();
            if (f & 2u) y -= __builtin_inff();
            if (a.out_half)
                static_cast<uint16_t*>(a.y)[(int64_t)b * a.N + row] =
                    __builtin_bit_cast(uint16_t, (_Float16)y);
            else
                static_cast<float*>(a.y)[(int64_t)b * a.N + row] = y;
        }
    }
}

template <int CT>
constexpr int lds_bytes() {
    const int pieces = kWaves * (kPieces * 4 * CT * kColBytes + 4 * CT * 16);
    const int red = kWaves * kMaxTiles * CT * 256;
    return pieces > red ? pieces : red;
}

template <int Q, int CT, int NP, bool ADD>
__global__ __launch_bounds__(kThreads, 2) void k_gemm_mx(KernelArgs a) {
    __shared__ uint4 lds[(lds_bytes<CT>() + 15) / 16];
    body<Q, CT, NP, ADD>(a, reinterpret_cast<char*>(lds));
}

// ---------------------------------------------------------------- choice and launch

template <int CT, int NP, bool ADD>
void launch_q(const KernelArgs& ka, int grid, hipStream_t s) {
    const dim3 g(grid), b(64 * ka.ksplit * ka.sets);
    switch (ka.a.q) {
        case 1: hipLaunchKernelGGL((k_gemm_mx<1, CT, NP, ADD>), g, b, 0, s, ka); break;
        case 2: hipLaunchKernelGGL((k_gemm_mx<2, CT, NP, ADD>), g, b, 0, s, ka); break;
        case 3: hipLaunchKernelGGL((k_gemm_mx<3, CT, NP, ADD>), g, b, 0, s, ka); break;
        default: hipLaunchKernelGGL((k_gemm_mx<4, CT, NP, ADD>), g, b, 0, s, ka); break;
    }
}

template <bool ADD>
void launch_batch(const KernelArgs& ka, int grid, hipStream_t s) {
    if (ka.a.B <= 2) launch_q<1, 1, ADD>(ka, grid, s);
    else if (ka.a.B <= 4) launch_q<1, 2, ADD>(ka, grid, s);
    else launch_q<2, 4, ADD>(ka, grid, s);
}

}  // namespace

// Batch 2 to 8.  The index bounds: exact division by multiplication (K), 32-bit
// offsets into a plane's exponents.
// The estimate is fitted (5th and 95th percentile of estimate / measured 0.9 and
// 1.2) to 1590 drawn layers of N 60..28672, K 128..28672, q 1..4, weights rotated
// over 320 MB: per 512-column group of a wave a fixed part (splitting the
// activations) and a part per row tile, plane and term; waves left out by a short
// K cost their share.
double plan(int q, int N, int K, int G, int B, int terms, sa_matrix_plan* p) {
    *p = sa_matrix_plan{};
    if (B > 8 || K > (1 << 22) || (int64_t)N * (K / 128) >= (int64_t)1 << 31)
        return sa_matrix::kNever;
    (void)G;
    const int groups = (K / 128 + kGroupBlocks - 1) / kGroupBlocks;
    int ksplit = 1;
    while (ksplit < kWaves && ksplit < groups) ksplit *= 2;
    const int tiles = (N + kTile - 1) / kTile;
    int sets = 1;
    while (sets * ksplit < kWaves && tiles > 256 * sets) sets *= 2;
    int wgs = imin((tiles + sets - 1) / sets, 256);
    if ((tiles + wgs * sets - 1) / (wgs * sets) > kMaxTiles)
        wgs = (tiles + kMaxTiles * sets - 1) / (kMaxTiles * sets);
    const int share = (tiles + wgs * sets - 1) / (wgs * sets);
    const int ct = B <= 4 ? 1 : 2;
    p->kernel = 1;
    p->rows_per_wg = kTile * sets * share;
    p->batch_per_wg = B;
    p->workgroups = wgs;
    p->threads = 64 * ksplit * sets;
    p->row_tiles = share;
    p->col_tiles = ct;
    p->column_shares = ksplit;
    p->lds_bytes = (size_t)(ct == 1 ? lds_bytes<1>() : lds_bytes<2>());
    // [batch 2, 3-4, 5-8][row-wise, additive]
    static const double kFit[3][2][6] = {
        {{3.0, 0.52, 0.50, 0.33, 0, 0.30}, {3.3, 0.41, 0.43, 0.53, 0.44, 0.50}},
        {{3.4, 1.2, 0.48, 0.31, 0, 0.26}, {3.7, 1.0, 0.33, 0.59, 0.43, 0.39}},
        {{3.9, 2.3, 0.45, 0.42, 0, 0.31}, {4.0, 2.2, 0.13, 0.80, 0.48, 0.45}}};
    const double* f = kFit[B <= 2 ? 0 : B <= 4 ? 1 : 2][terms > 0];
    const double rounds = wgs > 256 ? wgs / 256.0 : 1.0;
    const int per_wave = (groups + ksplit - 1) / ksplit;
    const double tile = f[2] + f[3] * q * (terms > 1 ? 1 + f[4] * (terms - 1) : 1);
    // the factors of three terms load by the byte
    return f[0] + rounds * per_wave * (f[1] + share * tile) *
                      (f[5] + (1 - f[5]) * p->threads / kThreads) * (terms == 3 ? 1.12 : 1);
}

void launch(const Args& a, const sa_matrix_plan& p, hipStream_t s) {
    KernelArgs ka{};
    ka.a = a;
    ka.ksplit = p.column_shares;
    ka.sets = p.threads / (64 * ka.ksplit);
    ka.tiles = (a.N + kTile - 1) / kTile;
    ka.shares = p.workgroups * ka.sets;
    ka.NG = a.K / a.G;
    ka.group_magic = sa_matrix::group_magic(a.G);
    if (a.terms) launch_batch<true>(ka, p.workgroups, s);
    else launch_batch<false>(ka, p.workgroups, s);
}

}  // namespace sa_mx
