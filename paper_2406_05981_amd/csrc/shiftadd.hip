// gfx950 kernels and C ABI of the shift-add linear layer (ShiftAddLLM, Sec. 4.1).
//
//   y[b][n] = sum_i sum_g 2^e[i][n][g] * sum_{k in g} s_i[n][k] x[b][k]
//
// computed as: 256-entry tables of signed partial sums per 8 activations
// (built in LDS), one table query per packed weight byte, fp32 adds, and one
// ldexp per (plane, row, 128-column block) folded into the fp32 accumulation.
// The path is an HBM stream of packed bits, not a dense contraction: no MFMA.
#include <hip/hip_runtime.h>

#include <stdint.h>

#include "gemm_matrix.h"
#include "keys.h"
#include "shiftadd.h"

#define SA_VERSION_STRING "0.1.0 gfx950"

namespace {

constexpr int kThreads = 256;     // 4 waves of 64
constexpr int kTileRows = 64;     // rows per tile: one row per lane
constexpr int kBlockChunks = 16;  // chunks (8 columns each) per block: 128 columns
constexpr int kKeyStride = 64;    // floats per key in the LDS tables (256 bytes)

// Byte offset of the key of (plane i, row n, chunk c) in the packed layout.
// Rows come in tiles of 64 and chunks in blocks of 16; a 64-row tile of one
// block is a contiguous piece, 16 bytes per row.  Inside a full block the 16
// keys of row r are rotated by r: position p holds chunk (p + r) mod 16, so
// that the lanes of a wave querying position p touch 16 different tables.
__host__ __device__ inline int64_t layout_offset(int i, int n, int c, int N, int C) {
    const int T = n >> 6, r = n & 63;
    const int R = imin(kTileRows, N - kTileRows * T);
    const int J = c >> 4, u = c & 15;
    const int U = imin(kBlockChunks, C - kBlockChunks * J);
    const int p = (U == kBlockChunks) ? ((u - r) & 15) : u;
    return ((int64_t)i * N + (int64_t)kTileRows * T) * C + (int64_t)kBlockChunks * J * R +
           (int64_t)r * U + p;
}

// One output: fp32, or IEEE binary16 rounded to nearest even when `half` (the
// fp16 output activations of Sec. 4.1; y then holds binary16 bit patterns).
__device__ inline void store_out(float* y, int64_t i, float v, int half) {
    if (half)
        reinterpret_cast<uint16_t*>(y)[i] = __builtin_bit_cast(uint16_t, (_Float16)v);
    else
        y[i] = v;
}

__device__ inline float half_bits_to_float(uint32_t h) {
    return (float)__builtin_bit_cast(_Float16, (uint16_t)h);
}

// The 8 activations x[8c..8c+7] of one chunk (16 bytes, 16-byte aligned).
__device__ inline void load_chunk(const uint16_t* p, float f[8]) {
    const uint4 v = *reinterpret_cast<const uint4*>(p);
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        f[2 * j] = half_bits_to_float(w[j] & 0xffffu);
        f[2 * j + 1] = half_bits_to_float(w[j] >> 16);
    }
}

// Signed sums of 4 activations for every 4-bit pattern a (bit j set -> +x_j):
// out[a] = (+-x0 +-x1) + (+-x2 +-x3).  Flipping every bit of a negates the
// result exactly, so table entries m and 255-m are exact negatives.
__device__ inline void nibble_sums(float x0, float x1, float x2, float x3, float out[16]) {
    const float s01 = x0 + x1, d01 = x0 - x1, s23 = x2 + x3, d23 = x2 - x3;
    const float p01[4] = {-s01, d01, -d01, s01};
    const float p23[4] = {-s23, d23, -d23, s23};
#pragma unroll
    for (int a = 0; a < 16; ++a) out[a] = p01[a & 3] + p23[a >> 2];
}

// One high-nibble sum (activations 4..7 of the chunk) for pattern h.
__device__ inline float nibble_sum(float x4, float x5, float x6, float x7, int h) {
    const float a = (h & 1) ? x4 : -x4;
    const float b = (h & 2) ? x5 : -x5;
    const float c = (h & 4) ? x6 : -x6;
    const float d = (h & 8) ? x7 : -x7;
    return (a + b) + (c + d);
}
// Table entry m of a chunk = low-nibble sum of (m & 15) + high-nibble sum of (m >> 4).

// ---------------------------------------------------------------- pack / unpack

__global__ void k_pack(const int8_t* __restrict__ signs, int q, int N, int C,
                       uint8_t* __restrict__ packed) {
    const int64_t total = (int64_t)q * N * C;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < total; t += stride) {
        const int c = (int)(t % C);
        const int64_t rest = t / C;
        const int n = (int)(rest % N);
        const int i = (int)(rest / N);
        const int8_t* s = signs + t * 8;
        uint32_t v = 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) v |= (s[j] > 0 ? 1u : 0u) << j;
        packed[layout_offset(i, n, c, N, C)] = (uint8_t)v;
    }
}

__global__ void k_unpack(const uint8_t* __restrict__ packed, int q, int N, int C,
                         int8_t* __restrict__ signs) {
    const int64_t total = (int64_t)q * N * C;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < total; t += stride) {
        const int c = (int)(t % C);
        const int64_t rest = t / C;
        const int n = (int)(rest % N);
        const int i = (int)(rest / N);
        const uint32_t v = packed[layout_offset(i, n, c, N, C)];
        int8_t* s = signs + t * 8;
#pragma unroll
        for (int j = 0; j < 8; ++j) s[j] = ((v >> j) & 1u) ? (int8_t)1 : (int8_t)-1;
    }
}

// ---------------------------------------------------------------- tables

// One item = (batch row b, chunk c, high nibble h): the 16 entries 16h..16h+15.
__global__ void k_build_lut(const uint16_t* __restrict__ x, int K, int B, float* __restrict__ lut) {
    const int C = K >> 3;
    const int64_t total = (int64_t)B * C * 16;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < total; t += stride) {
        const int h = (int)(t & 15);
        const int64_t bc = t >> 4;  // b * C + c
        const int b = (int)(bc / C), c = (int)(bc % C);
        float f[8];
        load_chunk(x + (int64_t)b * K + 8 * c, f);
        float lo[16];
        nibble_sums(f[0], f[1], f[2], f[3], lo);
        const float hi = nibble_sum(f[4], f[5], f[6], f[7], h);
        float4* out = reinterpret_cast<float4*>(lut + bc * 256 + 16 * h);
#pragma unroll
        for (int a = 0; a < 4; ++a)
            out[a] = make_float4(lo[4 * a] + hi, lo[4 * a + 1] + hi, lo[4 * a + 2] + hi,
                                 lo[4 * a + 3] + hi);
    }
}

// ---------------------------------------------------------------- generic kernel
//
// Any group size (group % 8 == 0).  One workgroup = 256 output rows of one
// batch row; K is walked in blocks of 16 chunks whose tables are staged in LDS.
// Each row keeps one fp32 partial per plane (in LDS) across blocks and shifts it
// into its total when a group ends.
__global__ __launch_bounds__(kThreads) void k_gemm_generic(
    const uint16_t* __restrict__ x, const uint8_t* __restrict__ packed,
    const int8_t* __restrict__ exps, int q, int N, int K, int G, float* __restrict__ y,
    int out_half) {
    __shared__ float lut[kBlockChunks][256];
    __shared__ float part[SA_MAX_Q][kThreads];
    const int C = K >> 3, NG = K / G, b = blockIdx.y;
    const int n = blockIdx.x * kThreads + threadIdx.x;
    const bool active = n < N;
    const uint16_t* xb = x + (int64_t)b * K;
    for (int i = 0; i < SA_MAX_Q; ++i) part[i][threadIdx.x] = 0.0f;
    float total = 0.0f;
    for (int J = 0; J * kBlockChunks < C; ++J) {
        const int U = imin(kBlockChunks, C - kBlockChunks * J);
        {
            const int u = threadIdx.x >> 4, h = threadIdx.x & 15;
            if (u < U) {
                float f[8];
                load_chunk(xb + 8 * (kBlockChunks * J + u), f);
                float lo[16];
                nibble_sums(f[0], f[1], f[2], f[3], lo);
                const float hi = nibble_sum(f[4], f[5], f[6], f[7], h);
#pragma unroll
                for (int a = 0; a < 16; ++a) lut[u][16 * h + a] = lo[a] + hi;
            }
        }
        __syncthreads();
        if (active) {
            for (int i = 0; i < q; ++i) {
                float acc = part[i][threadIdx.x];
                for (int u = 0; u < U; ++u) {
                    const int c = kBlockChunks * J + u;
                    acc += lut[u][packed[layout_offset(i, n, c, N, C)]];
                    if ((8 * (c + 1)) % G == 0) {
                        const int g = (8 * c) / G;
                        total += ldexpf(acc, (int)exps[((int64_t)i * N + n) * NG + g]);
                        acc = 0.0f;
                    }
                }
                part[i][threadIdx.x] = acc;
            }
        }
        __syncthreads();
    }
    if (active) store_out(y, (int64_t)b * N + n, total, out_half);
}

// ---------------------------------------------------------------- row kernel
//
// group % 128 == 0.  Each workgroup owns a contiguous range of 16-row groups
// over the whole input dimension, so no partial sums ever leave a workgroup.
// The row groups are spread evenly over the workgroups (counts differ by at
// most one), so no compute unit carries more rows than the average rounded up.
//
// Tables.  The 256-entry table of chunk c (Sec. 4.1) is stored factored into
// its two 16-entry halves: lo_c[v] = sum_{j<4} (bit j of v ? +x : -x)[8c+j] and
// hi_c[v] likewise over columns 8c+4..8c+7, so entry m = lo_c[m & 15] +
// hi_c[m >> 4].  A query of key m reads both halves and adds them.  32 stored
// values per chunk instead of 256 let one workgroup hold the tables of 4096
// columns in 64 KB of LDS and build them in a fraction of the time the
// queries take.
//
// LDS layout of a 4096-column piece: 256 rows of 64 four-byte slots.  The 32
// chunks of region rho (blocks 2rho and 2rho+1) keep their low halves in row
// (rho << 4) | v, slot 16*(block & 1) + u for chunk u of the block, and their
// high halves in row (v << 4) | rho, slot 32 + 16*(block & 1) + u.  A query
// address is one v_perm_b32: byte 1 = the key byte masked to the wanted
// nibble and or-ed with the region (one v_and_or_b32 per 4 keys and half),
// byte 0 = 4*slot.
//
// Work split.  Row r of a 16-row group is handled by lanes r, r+16, r+32,
// r+48 of all eight waves: part = 4*wave + (lane >> 4) owns block `part` of
// each piece.  Keys are stored rotated by row (position t of a row's 16 bytes
// holds chunk (t + row) mod 16).  A 4-byte LDS read is served one half-wave
// (32 lanes) at a time, and those lanes must touch 32 different slots mod 32
// (measured on gfx950 with SQ_LDS_BANK_CONFLICT); the two parts of a
// half-wave query 2 x 16 different chunks, i.e. 32 different slots: no bank
// conflicts by construction.
//
// Jobs.  A job is (batch row, piece, row group), row group fastest; a lane's
// share of a job is one 16-byte key load per plane and one exponent per plane.
//
// Each lane adds the 32 half-entries of its block, shifts the sum by the
// block's exponent (ldexp) and accumulates in fp32; the 32 lanes of a row are
// then combined in a fixed order (two xor-shuffles, then the eight waves via
// LDS).  The result is deterministic.

constexpr int kRowThreads = 512;     // 8 waves: 2 per SIMD
constexpr int kRowWaves = kRowThreads / 64;
constexpr int kGroupRows = 16;       // rows per row group
constexpr int kPieceBlocks = 32;     // 128-column blocks per table piece (4096 columns)
constexpr int kPieceChunks = kPieceBlocks * kBlockChunks;
constexpr int kRegionFloats = 1024;  // 4 KB: 16 values x 64 slots
constexpr int kMaxRG = 4;            // row groups per workgroup
static_assert(kRowThreads == kPieceChunks, "one table chunk per thread");
static_assert(4 * kRowWaves == kPieceBlocks, "one block per lane per piece");

struct RowsArgs {
    const uint16_t* x;  // activations [B][K]
    const uint8_t* packed;
    const int8_t* exps;      // row-wise: [q][N][K/G]
    const int8_t* col_exps;  // column-wise: [q][K]
    const int8_t* blk_exps;  // block-wise: [q][NB][K/8], NB = ceil(N / row_block)
    int q, N, K, G, B;
    float* y;           // [B][N]
    int groups;         // 16-row groups of N, spread over the grid
    int row_block, NB;  // block-wise: rows per block, blocks
    const int8_t* term_signs;  // additive: [q][N][K/G][T], with exps [q][N][K/G][T]
    int terms;                 // additive: T
};

// Where the power-of-two factors sit: one per (plane, row, group of G columns),
// one per (plane, column), one per (plane, block of rows, 8-column key), or a
// sum of T signed terms per (plane, row, group) (additive, Eq. 2).
enum ScaleMode { kRowWise = 0, kColWise = 1, kBlockWise = 2, kAdditive = 3 };
constexpr int kMaxTerms = 4;

// Keys and exponents of one job for this lane (Q planes of one block), and the
// activations of the lane's table chunk when the job starts a piece.
template <int Q>
struct JobRegs {
    uint4 w[Q];
    uint32_t e[Q];  // exponent byte, zero-extended; sign-extended where it is used
    uint4 xr;
    uint2 xe;       // column-wise: the exponents of the table chunk's 8 columns
    uint4 eb[Q];    // block-wise: the exponents of the block's 16 keys, per plane
    uint32_t et[Q]; // additive: the T exponent bytes of the plane's group, one per byte
    uint32_t st[Q]; // additive: the T term signs, one per byte
};

// Position of a job inside the workgroup's sequence: row group g (fastest),
// piece pc, plane i (column-wise layers only; 0 otherwise), batch row b.
struct JobPos {
    int g, pc, i, b;
};

__device__ inline void next_pos(JobPos& j, int nrg, int pieces, int planes) {
    if (++j.g == nrg) {
        j.g = 0;
        if (++j.pc == pieces) {
            j.pc = 0;
            if (++j.i == planes) {
                j.i = 0;
                ++j.b;
            }
        }
    }
}

// Exponents are requested before keys: whatever the compiler hoists onto the
// exponents then waits for them alone, never for the keys behind them.
// Per-lane offsets are 32-bit (a plane holds fewer than 2^31 bytes) on
// workgroup-uniform plane bases, so no 64-bit address arithmetic per load.
template <int Q>
__device__ inline void load_job_exps(const RowsArgs& a, int n, int J, int NG, int bpg,
                                     JobRegs<Q>& j) {
    const uint32_t off = (uint32_t)(n * NG + (bpg == 1 ? J : J / bpg));
#pragma unroll
    for (int i = 0; i < Q; ++i)
        j.e[i] = reinterpret_cast<const uint8_t*>(a.exps + (size_t)i * a.N * NG)[off];
}

// PLANE_ORDER: a workgroup barrier between the planes' requests, so that a
// CU asks for plane i of every wave before plane i + 1 of any (a CU's loads
// return in request order); only where every wave of the workgroup runs it.
template <int Q, bool PLANE_ORDER = false>
__device__ inline void load_job_keys(const RowsArgs& a, int n, int J, int C, int plane0,
                                     JobRegs<Q>& j) {
    const int T = n >> 6;
    const int R = imin(kTileRows, a.N - kTileRows * T);
    const uint32_t off = (uint32_t)(kTileRows * T * C + 16 * (n & 63) + kBlockChunks * J * R);
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        j.w[i] = *reinterpret_cast<const uint4*>(a.packed + (size_t)(plane0 + i) * a.N * C + off);
        if constexpr (PLANE_ORDER) {
            if (i + 1 < Q) {
                __builtin_amdgcn_sched_barrier(0);
                asm volatile("s_barrier" ::: "memory");  // no wait on the loads in flight
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
}

// Additive: the T exponents and term signs of the lane's group in every plane,
// T consecutive bytes each (one load of 1, 2 or 4 bytes; three bytes for T = 3).
template <int Q>
__device__ inline void load_job_terms(const RowsArgs& a, int n, int J, int NG, int bpg,
                                      JobRegs<Q>& j) {
    const uint32_t off = (uint32_t)(n * NG + (bpg == 1 ? J : J / bpg)) * (uint32_t)a.terms;
    const size_t plane = (size_t)a.N * NG * a.terms;
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        j.et[i] = load_terms(a.exps + i * plane + off, a.terms);
        j.st[i] = load_terms(a.term_signs + i * plane + off, a.terms);
    }
}

// Block-wise: the 16 exponents of the lane's 128-column block J in its row's
// block of rows, per plane (16 bytes; a row of the exponent array is K/8
// bytes, a multiple of 16).
template <int Q>
__device__ inline void load_job_blk_exps(const RowsArgs& a, int n, int J, int C, JobRegs<Q>& j) {
    const int rb = n / a.row_block;
#pragma unroll
    for (int i = 0; i < Q; ++i)
        j.eb[i] = *reinterpret_cast<const uint4*>(a.blk_exps +
                                                  ((size_t)i * a.NB + rb) * C + 16 * J);
}

// Empty asm that "may modify" one plane's job registers: their consumers
// cannot be hoisted above this point, so the wait for that plane's loads lands
// here -- after the tables are built and after the previous plane's queries.
template <int Q>
__device__ inline void pin_plane(JobRegs<Q>& j, int i) {
    asm volatile("" : "+v"(j.w[i].x), "+v"(j.w[i].y), "+v"(j.w[i].z), "+v"(j.w[i].w),
                 "+v"(j.e[i]));
}

template <int Q>
__device__ inline void pin_terms(JobRegs<Q>& j, int i) {
    asm volatile("" : "+v"(j.et[i]), "+v"(j.st[i]));
}

// Software-pipelined table reads need 8 more registers: used where they stay
// within the 128 registers of four waves per SIMD (up to 3 planes, one shift
// per plane); block-wise shifts per key keep the plain order.
template <int Q, bool BLK>
constexpr bool kPipelineWords = Q <= 3 && !BLK;

// Queries and adds of one job: sum over planes of ldexp(block sum, exponent).
// Planes are consumed in load order, so a plane's queries run while later
// planes are still arriving.
// Block-wise (BLK): every key has its own exponent, so each queried entry is
// shifted (ldexp) before it is added and the plane sum needs no shift; r is the
// lane's row mod 16.  Additive (terms > 0): the plane sum is shifted once per
// term and added with the term's sign (0: no term).
template <int Q, bool BLK = false>
__device__ inline float job_sum(JobRegs<Q>& j, uint32_t rgn_lo, uint32_t rgn_hi,
                                const uint32_t offs[8], const char* lut_bytes, int r = 0,
                                int terms = 0) {
    float tot = 0.0f;
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        __builtin_amdgcn_sched_barrier(0);
        pin_plane<Q>(j, i);
        const uint32_t words[4] = {j.w[i].x, j.w[i].y, j.w[i].z, j.w[i].w};
        uint32_t ek[4];
        if constexpr (BLK) rotate16(j.eb[i], r, ek);
        float acc;
        auto add_key = [&](int wd, int t, float L, float H) {
            if constexpr (BLK) {
                const float v = ldexpf(L + H, (int)(int8_t)(ek[wd] >> (8 * t)));
                if (wd == 0 && t == 0)
                    acc = v;
                else
                    acc += v;
            } else if (wd == 0 && t == 0) {
                acc = L + H;
            } else {
                acc += L;
                acc += H;
            }
        };
        // the 8 table reads of key word wd (4 keys, low and high half)
        auto fetch = [&](int wd, float* Lo, float* Ho) {
            // row byte of each of 4 keys: low nibble | region << 4, and
            // high nibble (in place) | region
            const uint32_t lo = (words[wd] & 0x0f0f0f0fu) | rgn_lo;
            const uint32_t hi = (words[wd] & 0xf0f0f0f0u) | rgn_hi;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                // byte 0: slot offset (offs[2wd + t/2] byte t%2); byte 1:
                // row (byte t); byte 2: the 64 KB half of the tables; the
                // high halves sit 32 slots (128 bytes) further: the read's
                // immediate offset
                const uint32_t sel = 0x03020000u | ((4u + t) << 8) | (uint32_t)(t & 1);
                const uint32_t o = offs[2 * wd + (t >> 1)];
                Lo[t] = *reinterpret_cast<const float*>(
                    lut_bytes + __builtin_amdgcn_perm(lo, o, sel));
                Ho[t] = *reinterpret_cast<const float*>(
                    lut_bytes + 128 + __builtin_amdgcn_perm(hi, o, sel));
            }
        };
        if constexpr (kPipelineWords<Q, BLK>) {
            // Word wd + 1's reads go out before word wd's adds: a wave keeps
            // up to 16 table reads in flight instead of draining 8 at a time.
            float Lw[2][4], Hw[2][4];
            fetch(0, Lw[0], Hw[0]);
#pragma unroll
            for (int wd = 0; wd < 4; ++wd) {
                if (wd + 1 < 4) fetch(wd + 1, Lw[(wd + 1) & 1], Hw[(wd + 1) & 1]);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int t = 0; t < 4; ++t) add_key(wd, t, Lw[wd & 1][t], Hw[wd & 1][t]);
                __builtin_amdgcn_sched_barrier(0);
            }
        } else {
#pragma unroll
            for (int wd = 0; wd < 4; ++wd) {
                const uint32_t lo = (words[wd] & 0x0f0f0f0fu) | rgn_lo;
                const uint32_t hi = (words[wd] & 0xf0f0f0f0u) | rgn_hi;
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const uint32_t sel = 0x03020000u | ((4u + t) << 8) | (uint32_t)(t & 1);
                    const uint32_t o = offs[2 * wd + (t >> 1)];
                    const float L = *reinterpret_cast<const float*>(
                        lut_bytes + __builtin_amdgcn_perm(lo, o, sel));
                    const float H = *reinterpret_cast<const float*>(
                        lut_bytes + 128 + __builtin_amdgcn_perm(hi, o, sel));
                    add_key(wd, t, L, H);
                }
            }
        }
        if constexpr (BLK) {
            tot += acc;
        } else if (terms > 0) {
            pin_terms<Q>(j, i);
#pragma unroll
            for (int t = 0; t < kMaxTerms; ++t) {
                const int sg = (int)(int8_t)(j.st[i] >> (8 * t));
                if (t < terms && sg != 0) {
                    const float v = ldexpf(acc, (int)(int8_t)(j.et[i] >> (8 * t)));
                    tot += sg < 0 ? -v : v;
                }
            }
        } else {
            tot += ldexpf(acc, (int)(int8_t)j.e[i]);
        }
    }
    return tot;
}

// MODE kColWise: the layer with column-wise factors (one exponent per plane and
// column).  Then a job covers one plane (Q = 1) and the plane is a job
// dimension; each plane's tables are built from the activations shifted by
// that plane's column exponents (exact in fp32), and the queried sums need no
// shift.  MODE kBlockWise: one exponent per (plane, block of rows, key); each
// queried entry is shifted (job_sum).
// H = 2 (layers of several pieces with at most one workgroup per CU): 16
// waves, the second 8 taking the odd pieces with their own 64 KB of tables, so
// two pieces are in flight per CU; the 16 waves' row sums meet at the end.
// OUT16: y holds binary16 outputs (row-wise layer only).
template <int Q, int U, int MODE, int H = 1, bool OUT16 = false>
__device__ __forceinline__ void gemm_rows_body(const RowsArgs& a, float* lut,
                                               float (*red)[kGroupRows * kMaxRG]) {
    constexpr bool COL = MODE == kColWise;
    constexpr bool BLK = MODE == kBlockWise;
    constexpr bool ADD = MODE == kAdditive;
    const int C = a.K >> 3, C16 = C >> 4, NG = a.K / a.G, bpg = a.G >> 7;
    const int lane = threadIdx.x & 63, wave_all = threadIdx.x >> 6;
    const int half = H == 1 ? 0 : wave_all / kRowWaves;  // pieces half, half + H, ...
    const int wave = wave_all - half * kRowWaves;
    const int r = lane & 15, p = lane >> 4, part = 4 * wave + p;
    // row groups of this workgroup: the first `extra` workgroups take one more
    const int wgs = (int)gridDim.x, wg = (int)blockIdx.x;
    const int base = a.groups / wgs, extra = a.groups - base * wgs;
    const int nrg = base + (wg < extra ? 1 : 0);
    const int rg0 = wg * base + imin(wg, extra);
    const int pieces_all = (C16 + kPieceBlocks - 1) / kPieceBlocks;
    const int pieces = (pieces_all - half + H - 1) / H;  // this half's pieces
    const int planes = COL ? a.q : 1;
    const int jobs = a.B * planes * pieces * nrg;

    // LDS address parts of this lane's 16 key positions, two positions per
    // register: bytes 0 and 1 of offs[k] are 4*slot of positions 2k and
    // 2k+1 (low half: slot = 16*(p & 1) + ((pos + r) & 15); the high half is
    // 32 slots further), byte 2 is the 64 KB half of the tables this wave
    // queries.  A query address is then one v_perm_b32 up to 128 KB, with no
    // add for the second half.
    uint32_t offs[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const uint32_t s0 = 16 * (p & 1) + ((2 * k + r) & 15);
        const uint32_t s1 = 16 * (p & 1) + ((2 * k + 1 + r) & 15);
        offs[k] = (4 * s0) | ((4 * s1) << 8) | ((uint32_t)half << 16);
    }
    const uint32_t rgn_lo = (uint32_t)((part >> 1) << 4) * 0x01010101u;
    const uint32_t rgn_hi = (uint32_t)(part >> 1) * 0x01010101u;

    float acc[kMaxRG];
#pragma unroll
    for (int g = 0; g < kMaxRG; ++g) acc[g] = 0.0f;

    // queries address all of the tables (the half is in the perm's byte 2);
    // the build writes this half
    const char* lut_bytes = reinterpret_cast<const char*>(lut);
    lut += half * (16 * kRegionFloats);
    // j.pc counts this half's pieces; the piece itself is H * j.pc + half
    auto row_of = [&](const JobPos& j) { return imin(kGroupRows * (rg0 + j.g) + r, a.N - 1); };
    auto block_of = [&](const JobPos& j) {
        return imin(kPieceBlocks * (H * j.pc + half) + part, C16 - 1);
    };
    // Tables are wave-local: the 64 lanes of a wave build the 64 chunks of the
    // four blocks that wave queries (lane (r, p) builds chunk r of block
    // `part`), so no table write is ever read by another wave and the only
    // workgroup barrier is the final combination of the waves' row sums.
    const int my_rho = part >> 1;
    const int slot_lo = 16 * (p & 1) + r;
    const int slot_hi = 32 + slot_lo;
    // activations of this lane's table chunk (and, column-wise, their
    // exponents in the job's plane)
    auto chunk_of = [&](const JobPos& j) {
        return imin(kPieceChunks * (H * j.pc + half) + kBlockChunks * part + r, C - 1);
    };
    auto load_x = [&](const JobPos& j) {
        return *reinterpret_cast<const uint4*>(a.x + (int64_t)j.b * a.K + 8 * chunk_of(j));
    };
    auto load_xe = [&](const JobPos& j) {
        return *reinterpret_cast<const uint2*>(a.col_exps + (int64_t)j.i * a.K + 8 * chunk_of(j));
    };
    // tables of this wave's four blocks of one piece for one batch row
    auto build = [&](const uint4 xr, const uint2 xe) {
        const uint32_t w4[4] = {xr.x, xr.y, xr.z, xr.w};
        float f[8];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            f[2 * t] = half_bits_to_float(w4[t] & 0xffffu);
            f[2 * t + 1] = half_bits_to_float(w4[t] >> 16);
        }
        if constexpr (COL) {
            const uint32_t e2[2] = {xe.x, xe.y};
#pragma unroll
            for (int t = 0; t < 8; ++t)
                f[t] = ldexpf(f[t], (int)(int8_t)(e2[t >> 2] >> (8 * (t & 3))));
        }
        float lo[16], hi[16];
        nibble_sums(f[0], f[1], f[2], f[3], lo);
        nibble_sums(f[4], f[5], f[6], f[7], hi);
        // low half: row (rho << 4) | v; high half: row (v << 4) | rho
        float* t_lo = lut + my_rho * kRegionFloats + slot_lo;
        float* t_hi = lut + my_rho * 64 + slot_hi;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            t_lo[v * 64] = lo[v];
            t_hi[v * kRegionFloats] = hi[v];
        }
        // the wave's own queries follow; LDS accesses of one wave complete in order
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    // Requests of one job: the activations when the job starts a piece (its
    // tables are built just before its queries, so they are asked for first),
    // then exponents, then keys.
    auto load_job = [&](const JobPos& j, JobRegs<Q>& regs) {
        const int n = row_of(j), J = block_of(j);
        if constexpr (COL) {
            if (j.g == 0) {
                regs.xr = load_x(j);
                regs.xe = load_xe(j);
            }
            __builtin_amdgcn_sched_barrier(0);
            regs.e[0] = 0u;
            load_job_keys<Q>(a, n, J, C, j.i, regs);
        } else {
            if (j.g == 0) regs.xr = load_x(j);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (BLK)
                load_job_blk_exps<Q>(a, n, J, C, regs);
            else if constexpr (ADD)
                load_job_terms<Q>(a, n, J, NG, bpg, regs);
            else
                load_job_exps<Q>(a, n, J, NG, bpg, regs);
            __builtin_amdgcn_sched_barrier(0);
            load_job_keys<Q>(a, n, J, C, 0, regs);
        }
    };
    // queries of one job, accumulation into its row group, and -- when the job
    // completes batch row b -- the combination of the 32 lanes of every row
    auto run_job = [&](const JobPos& j, JobRegs<Q>& regs) {
        const bool valid = kPieceBlocks * (H * j.pc + half) + part < C16;
        const float v = job_sum<Q, BLK>(regs, rgn_lo, rgn_hi, offs, lut_bytes, r,
                                        ADD ? a.terms : 0);
#pragma unroll
        for (int gg = 0; gg < kMaxRG; ++gg)
            if (gg == j.g && valid) acc[gg] += v;
        if (j.pc == pieces - 1 && j.g == nrg - 1 && j.i == planes - 1) {
#pragma unroll
            for (int gg = 0; gg < kMaxRG; ++gg) {
                if (gg < nrg) {
                    float s = acc[gg];
                    s += __shfl_xor(s, 16);
                    s += __shfl_xor(s, 32);
                    if (lane < kGroupRows) red[wave_all][kGroupRows * gg + r] = s;
                }
                acc[gg] = 0.0f;
            }
            __syncthreads();
            for (int t = threadIdx.x; t < kGroupRows * nrg; t += kRowThreads * H) {
                const int n = kGroupRows * rg0 + t;
                if (n < a.N) {
                    float s = red[0][t];
#pragma unroll
                    for (int w = 1; w < kRowWaves * H; ++w) s += red[w][t];
                    store_out(a.y, (int64_t)j.b * a.N + n, s, OUT16);
                }
            }
            // red is rewritten by the next batch row
            if (j.b + 1 < a.B) __syncthreads();
        }
    };

    // One job at a time: its requests (activations first, then exponents,
    // then keys), the table build when the job starts a piece, the queries.
    // Latency is hidden by the other waves resident on the SIMD rather than by
    // prefetching into a second register set: a loop-carried set of pending
    // loads makes the compiler copy registers at the loop back-edge, which
    // waits for every outstanding load and costs more than it hides.
    JobPos j{0, 0, 0, 0};
    // (additive: only when every workgroup has a single job; with one or two
    // jobs per workgroup the general order below measured faster)
    if ((MODE == kRowWise || (ADD && a.groups <= (int)gridDim.x)) && jobs == 1) {
        // A single job (a layer of at most 4096 columns and 16 rows per
        // workgroup): every request goes out at once, with no ordering
        // constraint, and the table build waits for the activations only.
        JobRegs<Q> regs;
        regs.xr = load_x(j);
        if constexpr (ADD)
            load_job_terms<Q>(a, row_of(j), block_of(j), NG, bpg, regs);
        else
            load_job_exps<Q>(a, row_of(j), block_of(j), NG, bpg, regs);
        // 8 waves (H = 1): plane-ordered requests, so every wave's first
        // plane arrives before any wave's second and all waves query while
        // the later planes stream in
        load_job_keys<Q, H == 1>(a, row_of(j), block_of(j), C, 0, regs);
        __builtin_amdgcn_sched_barrier(0);
        build(regs.xr, regs.xe);
        __builtin_amdgcn_sched_barrier(0);
        run_job(j, regs);
        return;
    }
    // Several jobs: U jobs per iteration.  All their requests go out at the
    // top of the iteration (past the last job they repeat it), then the jobs
    // are worked through in order, each waiting only for its own loads.  No
    // load is pending across the loop back-edge, so the compiler keeps every
    // register set in place, and a wave has U jobs of keys in flight per
    // round trip to memory.
    for (int job = 0; job < jobs; job += U) {
        JobRegs<Q> regs[U];
        JobPos pos[U];
        pos[0] = j;
#pragma unroll
        for (int u = 1; u < U; ++u) {
            pos[u] = pos[u - 1];
            if (job + u < jobs) next_pos(pos[u], nrg, pieces, planes);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) load_job(pos[u], regs[u]);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (job + u < jobs) {
                __builtin_amdgcn_sched_barrier(0);
                if (pos[u].g == 0) build(regs[u].xr, regs[u].xe);
                __builtin_amdgcn_sched_barrier(0);
                run_job(pos[u], regs[u]);
            }
        }
        j = pos[U - 1];
        next_pos(j, nrg, pieces, planes);
    }
}

// Jobs per loop iteration.  One: requesting several jobs' keys at once
// measured slower on gfx950 (the layer is bound by LDS and VALU issue, not by
// memory latency, and the extra registers only add pressure).
template <int Q>
constexpr int rows_jobs_per_iter() { return 1; }

// Up to 4 planes: two 8-wave workgroups per CU (4 waves per SIMD, <= 128
// VGPRs).  More planes need more registers: one workgroup per CU.
template <int Q, int H = 1, bool OUT16 = false>
__global__ __launch_bounds__(kRowThreads * H) __attribute__((amdgpu_waves_per_eu(4)))
void k_gemm_rows(RowsArgs a) {
    __shared__ float lut[H * 16 * kRegionFloats];  // 64 KB per half
    __shared__ float red[kRowWaves * H][kGroupRows * kMaxRG];
    gemm_rows_body<Q, rows_jobs_per_iter<Q>(), kRowWise, H, OUT16>(a, lut, red);
}

template <int Q, bool OUT16 = false>
__global__ __launch_bounds__(kRowThreads) void k_gemm_rows_wide(RowsArgs a) {
    __shared__ float lut[16 * kRegionFloats];  // 64 KB
    __shared__ float red[kRowWaves][kGroupRows * kMaxRG];
    gemm_rows_body<Q, rows_jobs_per_iter<Q>(), kRowWise, 1, OUT16>(a, lut, red);
}

// Column-wise factors: one plane per job, registers of a one-plane job.
template <int H = 1>
__global__ __launch_bounds__(kRowThreads * H) __attribute__((amdgpu_waves_per_eu(4)))
void k_gemm_rows_col(RowsArgs a) {
    __shared__ float lut[H * 16 * kRegionFloats];  // 64 KB per half
    __shared__ float red[kRowWaves * H][kGroupRows * kMaxRG];
    gemm_rows_body<1, 1, kColWise, H>(a, lut, red);
}

// Block-wise factors: the row kernel with a shift per queried key.
template <int Q, int H = 1>
__global__ __launch_bounds__(kRowThreads * H) __attribute__((amdgpu_waves_per_eu(4)))
void k_gemm_rows_blk(RowsArgs a) {
    __shared__ float lut[H * 16 * kRegionFloats];  // 64 KB per half
    __shared__ float red[kRowWaves * H][kGroupRows * kMaxRG];
    gemm_rows_body<Q, 1, kBlockWise, H>(a, lut, red);
}

template <int Q>
__global__ __launch_bounds__(kRowThreads) void k_gemm_rows_blk_wide(RowsArgs a) {
    __shared__ float lut[16 * kRegionFloats];  // 64 KB
    __shared__ float red[kRowWaves][kGroupRows * kMaxRG];
    gemm_rows_body<Q, 1, kBlockWise>(a, lut, red);
}

// Additive factors: the row kernel with T signed shifts per plane sum.
template <int Q, int H = 1>
__global__ __launch_bounds__(kRowThreads * H) __attribute__((amdgpu_waves_per_eu(4)))
void k_gemm_rows_add(RowsArgs a) {
    __shared__ float lut[H * 16 * kRegionFloats];  // 64 KB per half
    __shared__ float red[kRowWaves * H][kGroupRows * kMaxRG];
    gemm_rows_body<Q, 1, kAdditive, H>(a, lut, red);
}

template <int Q>
__global__ __launch_bounds__(kRowThreads) void k_gemm_rows_add_wide(RowsArgs a) {
    __shared__ float lut[16 * kRegionFloats];  // 64 KB
    __shared__ float red[kRowWaves][kGroupRows * kMaxRG];
    gemm_rows_body<Q, 1, kAdditive>(a, lut, red);
}

// ---------------------------------------------------------------- K-slice kernel with full tables
//
// Row-wise factors, batch 1.  The 256-entry table of each chunk (Sec. 4.1) is
// stored whole, so a query is one LDS read and one add per key instead of two
// of each.  Rebuilding 256 entries per chunk for every piece of a row kernel
// costs more LDS time than the halved reads save (LDS writes cost about twice
// what reads do on gfx950), so here a workgroup owns one 1024-column slice of
// K, builds its 128 KB of tables once, and streams every row of its row range
// through them.  Each workgroup writes one fp32 partial per (slice, row) to a
// workspace; a second kernel adds the slices of a row in slice order
// (deterministic).
//
// LDS layout (128 chunks): half h (chunks 64h..64h+63) holds 256 rows of 64
// four-byte slots, entry m of chunk 64h + s at float h*16384 + m*64 + s.  The
// bank of a read is its slot alone, whatever the key, so a query address is
// one v_perm_b32 (byte 0 = 4*slot, byte 1 = the key byte itself, byte 2 = h),
// and a half-wave's reads are conflict-free when its 32 lanes ask for 32
// different chunks.
//
// Build: thread t writes the 32 entries of chunk 64*((t >> 6) & 1) + (t & 63)
// whose high nibble is 2*(t >> 7) or 2*(t >> 7) + 1, entry m = lo[m & 15] +
// hi[m >> 4] with the nibble sums of the row kernel (entries m and 255 - m
// are exact negatives).  A wave's writes of one entry fill one 256-byte row.
//
// Queries: a job is 8 consecutive rows (starting at a multiple of 8) of the
// slice; lane (r = lane & 7, b = lane >> 3) of the wave owns row r, block b
// (blocks 0-3 in half 0, 4-7 in half 1).  Keys are stored rotated by row
// (position t of a row's 16 bytes holds chunk (t + row) mod 16), so the 8
// rows x 4 blocks of a half-wave ask for 32 different chunks.  Wave w takes
// jobs w, w + 16, ... of its range; every job of a wave has the same row
// parity, so the lane's slot offsets are fixed.  The next job's keys and
// exponents are requested before the current job's queries.
constexpr int kSliceBlocks = 8;                             // 1024 columns per slice
constexpr int kSliceCols = kSliceBlocks * 128;
constexpr int kSliceHalfFloats = 256 * 64;                  // 64 KB
constexpr int kSliceThreads = 1024;                         // 16 waves
constexpr int kSliceWaves = kSliceThreads / 64;
constexpr int kSliceJobRows = 8;

struct SliceArgs {
    const uint16_t* x;
    const uint8_t* packed;
    const int8_t* exps;
    int q, N, K, G;
    int slices, ranges;  // grid = slices * ranges
    int jobs;            // ceil(N / 8)
    float* part;         // [slices][N]
};

template <int Q>
struct SliceRegs {
    uint4 w[Q];
    int e[Q];  // exponent, sign-extended by the load
};

template <int Q>
__global__ __launch_bounds__(kSliceThreads) void k_gemm_kslice(SliceArgs a) {
    __shared__ float tab[2 * kSliceHalfFloats];
    const int C = a.K >> 3, NG = a.K / a.G, bpg = a.G >> 7;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int slice = (int)blockIdx.x % a.slices, range = (int)blockIdx.x / a.slices;
    // jobs [j0, j1) of this range, spread evenly over the ranges
    const int jbase = a.jobs / a.ranges, jextra = a.jobs - jbase * a.ranges;
    const int j0 = range * jbase + imin(range, jextra);
    const int j1 = j0 + jbase + (range < jextra ? 1 : 0);
    const int nj = j1 - j0 > wave ? (j1 - j0 - wave + kSliceWaves - 1) / kSliceWaves : 0;

    const int r = lane & 7, b = lane >> 3;
    const int rr = r + 8 * ((j0 + wave) & 1);  // row mod 16 of this lane's rows
    const int J = kSliceBlocks * slice + b;    // block of the whole row
    uint32_t offs[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const uint32_t s0 = 16 * (b & 3) + ((2 * k + rr) & 15);
        const uint32_t s1 = 16 * (b & 3) + ((2 * k + 1 + rr) & 15);
        offs[k] = (4 * s0) | ((4 * s1) << 8) | ((uint32_t)(b >> 2) << 16);
    }
    const char* tab_bytes = reinterpret_cast<const char*>(tab);

    auto row_of = [&](int k) {  // row of this lane in the wave's k-th job (clamped)
        const int n = kSliceJobRows * (j0 + wave + kSliceWaves * imin(k, nj - 1)) + r;
        return n < 0 ? 0 : imin(n, a.N - 1);
    };
    auto load_job = [&](int k, SliceRegs<Q>& g) {
        const int n = row_of(k);
        const uint32_t eoff = (uint32_t)(n * NG + (bpg == 1 ? J : J / bpg));
#pragma unroll
        for (int i = 0; i < Q; ++i) g.e[i] = (a.exps + (size_t)i * a.N * NG)[eoff];
        const int T = n >> 6;
        const int R = imin(kTileRows, a.N - kTileRows * T);
        const uint32_t off = (uint32_t)(kTileRows * T * C + 16 * (n & 63) + kBlockChunks * J * R);
#pragma unroll
        for (int i = 0; i < Q; ++i)
            g.w[i] = *reinterpret_cast<const uint4*>(a.packed + (size_t)i * a.N * C + off);
    };
    // queries of one job, then the row's 8 blocks combined in a fixed order
    auto run_job = [&](int k, SliceRegs<Q>& g) {
        float tot = 0.0f;
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            const uint32_t words[4] = {g.w[i].x, g.w[i].y, g.w[i].z, g.w[i].w};
            float s = 0.0f;
#pragma unroll
            for (int wd = 0; wd < 4; ++wd) {
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const uint32_t sel = 0x03020000u | ((4u + t) << 8) | (uint32_t)(t & 1);
                    const float v = *reinterpret_cast<const float*>(
                        tab_bytes + __builtin_amdgcn_perm(words[wd], offs[2 * wd + (t >> 1)], sel));
                    s = (wd == 0 && t == 0) ? v : s + v;
                }
            }
            tot += ldexpf(s, g.e[i]);
        }
        tot += __shfl_xor(tot, 8);
        tot += __shfl_xor(tot, 16);
        tot += __shfl_xor(tot, 32);
        const int n = kSliceJobRows * (j0 + wave + kSliceWaves * k) + r;
        if (lane < kSliceJobRows && k < nj && n < a.N) a.part[(size_t)slice * a.N + n] = tot;
    };

    // the slice's tables, built once: activations requested first, then the
    // first job's keys, so the build waits for the activations only
    const int slot = threadIdx.x & 63, half = (threadIdx.x >> 6) & 1, kq = threadIdx.x >> 7;
    const uint4 xr = *reinterpret_cast<const uint4*>(a.x + kSliceCols * slice +
                                                     8 * (64 * half + slot));
    __builtin_amdgcn_sched_barrier(0);
    SliceRegs<Q> ga, gb;
    load_job(0, ga);  // (a valid row even for a wave without jobs)
    __builtin_amdgcn_sched_barrier(0);
    {
        const uint32_t w4[4] = {xr.x, xr.y, xr.z, xr.w};
        float f[8];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            f[2 * t] = half_bits_to_float(w4[t] & 0xffffu);
            f[2 * t + 1] = half_bits_to_float(w4[t] >> 16);
        }
        float lo[16];
        nibble_sums(f[0], f[1], f[2], f[3], lo);
        float* t0 = tab + half * kSliceHalfFloats + slot;
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
            const int h = 2 * kq + hh;
            const float hv = nibble_sum(f[4], f[5], f[6], f[7], h);
#pragma unroll
            for (int l = 0; l < 16; ++l) t0[(16 * h + l) * 64] = lo[l] + hv;
        }
    }
    // LDS writes done, then the barrier; the first job's loads stay in flight
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    // Two jobs per iteration, each job's loads issued one job ahead into the
    // other register set (past the last job the request repeats it), no
    // branch around the loads, so the compiler keeps both sets in place.
    for (int k = 0; k < nj; k += 2) {
        load_job(k + 1, gb);
        run_job(k, ga);
        load_job(k + 2, ga);
        run_job(k + 1, gb);
    }
}

// y[n] = sum over slices of part[s][n], in slice order (eight loads in flight
// per thread, the adds in order).
__global__ void k_sum_slices(const float* __restrict__ part, int slices, int N,
                             float* __restrict__ y) {
    const int n = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (n >= N) return;
    float s = 0.0f;
    for (int i0 = 0; i0 < slices; i0 += 8) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            v[u] = i0 + u < slices ? part[(size_t)(i0 + u) * N + n] : 0.0f;
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (i0 + u < slices) s = i0 + u == 0 ? v[u] : s + v[u];
    }
    y[n] = s;
}

constexpr int kRowsResidentQ = 4;  // largest q launched two workgroups per CU

// ---------------------------------------------------------------- batch kernel
//
// batch >= 2, group % 128 == 0.  A key byte is shared by every batch row, so
// the tables of four batch rows (a quad) are interleaved: value v of a
// half-table is a float4 over the quad, and one query reads the four entries
// with one 16-byte LDS load and adds them into four accumulators.  The address
// arithmetic of a query is paid once per four batch rows.
//
// Work split.  A workgroup owns 16*KW output rows (KW = 1, 2 or 4) and one
// quad; it walks the input dimension in pieces of 1024 columns, one 128-column
// block per wave.  Each lane handles one row and KW of the 4 key words (4 keys
// each) of that row's block, so a wave covers its block for all 16*KW rows.
// Each wave builds the tables of its own block for the quad, one (chunk, batch
// row) per lane: lane l builds chunk (l & 7) + 8*(l >> 5) for batch row
// (l >> 3) & 3, so the 32 lanes of a half-wave write 32 different 4-byte
// banks.  Tables are wave-local and the only workgroup barrier is the final
// combination of the partial sums.
//
// LDS layout of a wave's tables (8 KB): float v*128 + h*64 + c*4 + u holds
// value v of half h (0: columns 8c..8c+3, 1: 8c+4..8c+7) of chunk c for batch
// row u of the quad.  A query address is one v_perm_b32: byte 1 = (wave << 5)
// | (v << 1) | h, byte 0 = 16*c.
//
// Bank groups.  A 16-byte LDS read is served 16 lanes at a time: the lanes
// that agree in lane bit 5 and in the parity of lane bits 2..4 (measured on
// gfx950 with SQ_LDS_BANK_CONFLICT), and those 16 must touch 16 different
// 16-byte bank groups (address bits 4..7), i.e. 16 different chunks.  With
// keys rotated by row, a query at key position pos touches chunk
// (pos + row) mod 16.  Lane (r, p) (r = lane & 15, p = lane >> 4) therefore
// takes, for KW = 4: row 16p + r, all words; KW = 2: row 16(p & 1) + r, words
// 2(p >> 1)..+1 (the two lanes of a half that share r read the same position
// of different rows); KW = 1: row (r - 4p) mod 16, word p (every lane then
// queries chunk r + t at step t).  Each 16-lane set covers every chunk once.

constexpr int kQuad = 4;                                          // batch rows per table word
constexpr int kWaveTableFloats = 16 * 2 * kBlockChunks * kQuad;  // 2048 floats = 8 KB
constexpr int kBatchRows = 64;                                    // most rows per workgroup

struct BatchArgs {
    const uint16_t* x;  // activations [B][K]
    const uint8_t* packed;
    const int8_t* exps;        // row-wise [q][N][K/G]; additive [q][N][K/G][T]
    int q, N, K, G, B;
    float* y;     // [B][N]
    int n_tiles;  // row tiles of 16*KW rows
    int n_quads;  // ceil(B / 4)
    const int8_t* term_signs;  // additive: [q][N][K/G][T]
    int terms;                 // additive: T
    const int8_t* blk_exps;    // block-wise: [q][NB][K/8]
    int row_block, NB;         // block-wise
    const int8_t* col_exps;    // column-wise: [q][K]
    int pre_bytes;             // PRE: bytes of a lane's exponents over all its pieces
};

// One piece for this lane: KW key words of Q planes, their exponents, and the
// activations of the table chunk the lane builds.
template <int Q, int KW>
struct BatchJob {
    uint32_t w[Q][KW];
    int e[Q];
    uint4 xr;
    uint32_t et[Q], st[Q];  // additive: T exponent bytes, T term signs
    uint4 eb[Q];            // block-wise: the 16 exponents of the block in the row's block of rows
    uint2 xe[Q];            // column-wise: the exponents of the table chunk's 8 columns
};

template <int KW>
__device__ inline void load_words(const uint8_t* p, uint32_t* w) {
    if constexpr (KW == 4) {
        const uint4 v = *reinterpret_cast<const uint4*>(p);
        w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = v.w;
    } else if constexpr (KW == 2) {
        const uint2 v = *reinterpret_cast<const uint2*>(p);
        w[0] = v.x; w[1] = v.y;
    } else {
        w[0] = *reinterpret_cast<const uint32_t*>(p);
    }
}

template <int Q, int KW>
__device__ inline void pin_batch_plane(BatchJob<Q, KW>& j, int i) {
#pragma unroll
    for (int k = 0; k < KW; ++k) asm volatile("" : "+v"(j.w[i][k]));
    asm volatile("" : "+v"(j.e[i]));
}

// MODE: kRowWise, kAdditive (each plane's group sums shifted by T signed terms),
// kBlockWise (each queried entry shifted by its key's exponent) or kColWise
// (each plane queries its own tables, built in turn from the activations
// shifted by that plane's column exponents; the queried sums need no shift).
// UNI (block-wise): the workgroup's rows lie in one block of rows, so the
// block exponents are the same for all its lanes and come in by scalar loads,
// which keeps them out of the vector registers.
// Every wave owns consecutive blocks (J = pieces * wave + pc).  PRE
// (additive, G = 128, K % 1024 == 0): a lane's T exponent bytes and T term
// signs of all its pieces are then pieces * T consecutive bytes of its row,
// fetched by one 4-, 8- or 16-byte load each at the start instead of two
// scattered loads per piece and plane (these touch one cache line per lane
// and were a third of the additive kernel's time on large layers; the
// row-wise kernel's one byte per piece measured no gain from it).
// OUT16: y holds binary16 outputs (row-wise layer only).
template <int Q, int KW, int MODE, bool UNI = false, bool PRE = false, bool OUT16 = false>
__device__ __forceinline__ void gemm_batch_body(const BatchArgs& a, float* lut, float* red) {
    constexpr int DS = 4 / KW;  // lanes sharing one row, KW key words each
    constexpr bool ADD = MODE == kAdditive;
    constexpr bool BLK = MODE == kBlockWise;
    constexpr bool COL = MODE == kColWise;
    static_assert(!PRE || (ADD && Q <= 3), "preloaded exponents: additive mode, up to 3 planes");
    const int C = a.K >> 3, C16 = C >> 4, NG = a.K / a.G, bpg = a.G >> 7;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r = lane & 15, p = lane >> 4;
    // key-word slice, 16-row group and row (mod 16) of this lane (see above)
    const int dsl = KW == 4 ? 0 : KW == 2 ? p >> 1 : p;
    const int rsub = KW == 4 ? p : KW == 2 ? p & 1 : 0;
    const int rr = KW == 1 ? (r - 4 * p) & 15 : r;
    // Workgroup -> (row tile, quad).  Workgroups are dealt to the 8 XCDs
    // round-robin; the quads of one tile land on one XCD and share its L2.
    const int xcd = blockIdx.x & 7, idx = blockIdx.x >> 3;
    const int tile = xcd + 8 * (idx / a.n_quads), quad = idx % a.n_quads;
    if (tile >= a.n_tiles) return;  // whole workgroup: padding of the grid
    const int row0 = 16 * KW * tile;
    const int row_local = 16 * rsub + rr;
    const int n = imin(row0 + row_local, a.N - 1);
    const int pieces = (C16 + kRowWaves - 1) / kRowWaves;

    // byte t of offs[k] = 16 * (chunk at key position 4*(KW*dsl + k) + t of row r)
    uint32_t offs[KW];
#pragma unroll
    for (int k = 0; k < KW; ++k) {
        uint32_t o = 0;
#pragma unroll
        for (int t = 0; t < 4; ++t)
            o |= (uint32_t)(((4 * (KW * dsl + k) + t + rr) & 15) << 4) << (8 * t);
        offs[k] = o;
    }
    const uint32_t rgn_lo = (uint32_t)(wave << 5) * 0x01010101u;
    const uint32_t rgn_hi = (uint32_t)((wave << 5) | 1) * 0x01010101u;
    const char* lut_bytes = reinterpret_cast<const char*>(lut);

    // this lane's table chunk and batch row of the quad (see above)
    const int bc = (lane & 7) + 8 * (lane >> 5), bu = (lane >> 3) & 3;
    const int bx = imin(kQuad * quad + bu, a.B - 1);
    const int T = n >> 6;
    const int R = imin(kTileRows, a.N - kTileRows * T);
    const uint8_t* key_row = a.packed + (int64_t)kTileRows * T * C + 16 * (n & 63) + 4 * KW * dsl;
    const int8_t* exp_row = a.exps + (int64_t)n * NG;

    // PRE: bytes [pieces * wave * T, (pieces * wave + pieces) * T) of the row
    constexpr int QP = PRE ? Q : 1, QS = PRE ? Q : 1;
    uint32_t pe[QP][4] = {}, ps[QS][4] = {};
    if constexpr (PRE) {
        const int64_t off0 = ((int64_t)n * NG + (int64_t)pieces * wave) * a.terms;
        const int64_t plane = (int64_t)a.N * NG * a.terms;
        auto fetch = [&](const int8_t* src, uint32_t* w) {
            if (a.pre_bytes == 16) {
                const uint4 v = *reinterpret_cast<const uint4*>(src);
                w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = v.w;
            } else if (a.pre_bytes == 8) {
                const uint2 v = *reinterpret_cast<const uint2*>(src);
                w[0] = v.x; w[1] = v.y;
            } else {
                w[0] = *reinterpret_cast<const uint32_t*>(src);
            }
        };
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            fetch(a.exps + i * plane + off0, pe[i]);
            fetch(a.term_signs + i * plane + off0, ps[i]);
        }
    }
    // PRE: the T bytes of piece pc in a lane's preloaded words (T divides 4)
    auto pre_field = [&](const uint32_t* w, int pc) {
        const int bo = pc * a.terms;
        const int wi = bo >> 2;
        const uint32_t v = wi == 0 ? w[0] : wi == 1 ? w[1] : wi == 2 ? w[2] : w[3];
        return v >> (8 * (bo & 3));
    };

    auto load_job = [&](int pc, BatchJob<Q, KW>& j) {
        const int J = imin(pieces * wave + pc, C16 - 1);
        if constexpr (PRE) {
            // exponents come from the preloaded words at query time
        } else if constexpr (ADD) {
            const int64_t off = ((int64_t)n * NG + (bpg == 1 ? J : J / bpg)) * a.terms;
            const int64_t plane = (int64_t)a.N * NG * a.terms;
#pragma unroll
            for (int i = 0; i < Q; ++i) {
                j.et[i] = load_terms(a.exps + i * plane + off, a.terms);
                j.st[i] = load_terms(a.term_signs + i * plane + off, a.terms);
            }
        } else if constexpr (BLK && UNI) {
            const int Ju = __builtin_amdgcn_readfirstlane(J);  // J is uniform per wave
            const int8_t* eb = a.blk_exps + (int64_t)(row0 / a.row_block) * C + 16 * Ju;
#pragma unroll
            for (int i = 0; i < Q; ++i)
                j.eb[i] = *reinterpret_cast<const uint4*>(eb + (int64_t)i * a.NB * C);
        } else if constexpr (BLK) {
            const int rb = n / a.row_block;
#pragma unroll
            for (int i = 0; i < Q; ++i)
                j.eb[i] = *reinterpret_cast<const uint4*>(a.blk_exps +
                                                          ((int64_t)i * a.NB + rb) * C + 16 * J);
        } else if constexpr (COL) {
#pragma unroll
            for (int i = 0; i < Q; ++i)
                j.xe[i] = *reinterpret_cast<const uint2*>(a.col_exps + (int64_t)i * a.K +
                                                          8 * (kBlockChunks * J + bc));
        } else {
            const int8_t* e = exp_row + (bpg == 1 ? J : J / bpg);
#pragma unroll
            for (int i = 0; i < Q; ++i) j.e[i] = e[(int64_t)i * a.N * NG];
        }
        j.xr = *reinterpret_cast<const uint4*>(a.x + (int64_t)bx * a.K +
                                               8 * (kBlockChunks * J + bc));
        const uint8_t* kp = key_row + (int64_t)kBlockChunks * J * R;
#pragma unroll
        for (int i = 0; i < Q; ++i) load_words<KW>(kp + (int64_t)i * a.N * C, j.w[i]);
    };
    auto build = [&](const uint4 xr, const uint2 xe) {
        const uint32_t w4[4] = {xr.x, xr.y, xr.z, xr.w};
        float f[8];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            f[2 * t] = half_bits_to_float(w4[t] & 0xffffu);
            f[2 * t + 1] = half_bits_to_float(w4[t] >> 16);
        }
        if constexpr (COL) {
            const uint32_t e2[2] = {xe.x, xe.y};
#pragma unroll
            for (int t = 0; t < 8; ++t)
                f[t] = ldexpf(f[t], (int)(int8_t)(e2[t >> 2] >> (8 * (t & 3))));
        }
        float lo[16], hi[16];
        nibble_sums(f[0], f[1], f[2], f[3], lo);
        nibble_sums(f[4], f[5], f[6], f[7], hi);
        float* t = lut + wave * kWaveTableFloats + bc * kQuad + bu;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            t[v * 128] = lo[v];
            t[v * 128 + 64] = hi[v];
        }
        // the wave's own queries follow; LDS accesses of one wave complete in order
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };

    float tot[kQuad] = {0.0f, 0.0f, 0.0f, 0.0f};
    auto query_job = [&](int pc, BatchJob<Q, KW>& j) {
        // blocks past the end (last piece) repeat the last block and are left out
        // (a select: 0 * inf is a NaN)
        const bool keep = pieces * wave + pc < C16;
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            __builtin_amdgcn_sched_barrier(0);
            // column-wise: this plane's tables replace the previous plane's
            // (the wave's LDS reads and writes complete in order)
            if constexpr (COL) build(j.xr, j.xe[i]);
            pin_batch_plane<Q, KW>(j, i);
            float s[kQuad];
            // block-wise: the exponents of this lane's KW key words (4 keys each),
            // rotated to the row's key order
            uint32_t ekw[KW];
            if constexpr (BLK) {
                uint32_t ek[4];
                rotate16(j.eb[i], rr, ek);
#pragma unroll
                for (int k = 0; k < KW; ++k) {
                    const int wsel = KW * dsl + k;
                    ekw[k] = wsel == 0 ? ek[0] : wsel == 1 ? ek[1] : wsel == 2 ? ek[2] : ek[3];
                }
            }
#pragma unroll
            for (int k = 0; k < KW; ++k) {
                // one key word at a time: its 8 loads go out together, then
                // its adds (32 registers of loads in flight)
                if (k > 0) __builtin_amdgcn_sched_barrier(0);
                const uint32_t lo = ((j.w[i][k] << 1) & 0x1e1e1e1eu) | rgn_lo;
                const uint32_t hi = ((j.w[i][k] >> 3) & 0x1e1e1e1eu) | rgn_hi;
                float4 L[4], H[4];
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const uint32_t sel = 0x0c0c0000u | ((4u + t) << 8) | (uint32_t)t;
                    L[t] = *reinterpret_cast<const float4*>(
                        lut_bytes + __builtin_amdgcn_perm(lo, offs[k], sel));
                    H[t] = *reinterpret_cast<const float4*>(
                        lut_bytes + __builtin_amdgcn_perm(hi, offs[k], sel));
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    if constexpr (BLK) {
                        const int ex = (int)(int8_t)(ekw[k] >> (8 * t));
                        const float v0 = ldexpf(L[t].x + H[t].x, ex);
                        const float v1 = ldexpf(L[t].y + H[t].y, ex);
                        const float v2 = ldexpf(L[t].z + H[t].z, ex);
                        const float v3 = ldexpf(L[t].w + H[t].w, ex);
                        if (k == 0 && t == 0) {
                            s[0] = v0; s[1] = v1; s[2] = v2; s[3] = v3;
                        } else {
                            s[0] += v0; s[1] += v1; s[2] += v2; s[3] += v3;
                        }
                    } else if (k == 0 && t == 0) {
                        s[0] = L[0].x + H[0].x;
                        s[1] = L[0].y + H[0].y;
                        s[2] = L[0].z + H[0].z;
                        s[3] = L[0].w + H[0].w;
                    } else {
                        s[0] += L[t].x; s[0] += H[t].x;
                        s[1] += L[t].y; s[1] += H[t].y;
                        s[2] += L[t].z; s[2] += H[t].z;
                        s[3] += L[t].w; s[3] += H[t].w;
                    }
                }
                // the word's adds complete here, so its loads' registers free up
                asm volatile("" : "+v"(s[0]), "+v"(s[1]), "+v"(s[2]), "+v"(s[3]));
            }
            if constexpr (BLK || COL) {
#pragma unroll
                for (int u = 0; u < kQuad; ++u) tot[u] += keep ? s[u] : 0.0f;
            } else if constexpr (ADD) {
                if constexpr (PRE) {
                    j.et[i] = pre_field(pe[i], pc);
                    j.st[i] = pre_field(ps[i], pc);
                }
                asm volatile("" : "+v"(j.et[i]), "+v"(j.st[i]));
                // the plane's signed terms (sign -1, 0 or +1: the products are
                // exact), then the piece's weight once.  A sign of 0 means no
                // term, whatever its exponent byte or the activations hold (a
                // select, no branch: 0 * inf would be a NaN).
                float pl[kQuad] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int tt = 0; tt < kMaxTerms; ++tt) {
                    if (tt < a.terms) {
                        const float sg = (float)(int8_t)(j.st[i] >> (8 * tt));
                        const int ex = (int)(int8_t)(j.et[i] >> (8 * tt));
#pragma unroll
                        for (int u = 0; u < kQuad; ++u) {
                            const float v = fmaf(sg, ldexpf(s[u], ex), pl[u]);
                            pl[u] = sg != 0.0f ? v : pl[u];
                        }
                    }
                }
#pragma unroll
                for (int u = 0; u < kQuad; ++u) tot[u] += keep ? pl[u] : 0.0f;
            } else {
#pragma unroll
                for (int u = 0; u < kQuad; ++u) tot[u] += keep ? ldexpf(s[u], j.e[i]) : 0.0f;
            }
        }
    };

    // Two register sets alternate; a piece's keys and activations are
    // requested before the previous piece's queries, unconditionally (past
    // the last piece they repeat it), so no register set depends on a branch.
    BatchJob<Q, KW> ja, jb;
    load_job(0, ja);
    for (int pc = 0; pc < pieces; pc += 2) {
        if constexpr (!COL) build(ja.xr, uint2{});
        load_job(imin(pc + 1, pieces - 1), jb);
        query_job(pc, ja);
        if (pc + 1 >= pieces) break;
        if constexpr (!COL) build(jb.xr, uint2{});
        load_job(imin(pc + 2, pieces - 1), ja);
        query_job(pc + 1, jb);
    }

    // Partial sums of (wave, row, word slice) meet in LDS and are added in a
    // fixed order: waves outer, word slices inner.
    *reinterpret_cast<float4*>(red + (wave * kBatchRows + row_local * DS + dsl) * kQuad) =
        make_float4(tot[0], tot[1], tot[2], tot[3]);
    __syncthreads();
    const int t = threadIdx.x;
    if (t < 16 * KW * kQuad) {
        const int row = t >> 2, u = t & 3;
        const int nn = row0 + row, b = kQuad * quad + u;
        if (nn < a.N && b < a.B) {
            float s = red[row * DS * kQuad + u];
#pragma unroll
            for (int d = 1; d < DS; ++d) s += red[(row * DS + d) * kQuad + u];
#pragma unroll
            for (int w = 1; w < kRowWaves; ++w)
#pragma unroll
                for (int d = 0; d < DS; ++d)
                    s += red[(w * kBatchRows + row * DS + d) * kQuad + u];
            store_out(a.y, (int64_t)b * a.N + nn, s, OUT16);
        }
    }
}

// UNI (block-wise only): every workgroup's rows lie in one block of rows
// (row_block is a multiple of the 16*KW rows of a workgroup).
template <int Q, int KW, int MODE = kRowWise, bool UNI = false, bool PRE = false,
          bool OUT16 = false>
__global__ __launch_bounds__(kRowThreads) __attribute__((amdgpu_waves_per_eu(4)))
void k_gemm_batch(BatchArgs a) {
    __shared__ float4 lut[kRowWaves * kWaveTableFloats / 4];  // 64 KB
    __shared__ float4 red[kRowWaves * kBatchRows];            // 8 KB
    gemm_batch_body<Q, KW, MODE, UNI, PRE, OUT16>(a, reinterpret_cast<float*>(lut),
                                                  reinterpret_cast<float*>(red));
}

template <int Q, int KW, int MODE = kRowWise, bool UNI = false, bool OUT16 = false>
__global__ __launch_bounds__(kRowThreads) void k_gemm_batch_wide(BatchArgs a) {
    __shared__ float4 lut[kRowWaves * kWaveTableFloats / 4];
    __shared__ float4 red[kRowWaves * kBatchRows];
    gemm_batch_body<Q, KW, MODE, UNI, false, OUT16>(a, reinterpret_cast<float*>(lut),
                                                    reinterpret_cast<float*>(red));
}

// ---------------------------------------------------------------- read probe
//
// Measurement aid, not part of the layer: every thread reads kProbePer 16-byte
// words of the buffer (grid-strided, so each request of a wave is 1 KiB of
// contiguous memory) and folds them with xor, and each wave folds its lanes.
// Its time is that of a plain read of the same bytes -- the practical floor a
// layer streaming that many bytes is measured against.  The shape (256-thread
// workgroups, one word per thread, as many workgroups as words / 256) was the
// fastest of a sweep over 256, 512 and 1024 threads, 1 to 16 words per thread,
// one-shot and persistent grids, at 6.7, 18 and 94 MB on gfx950.

constexpr int kProbeThreads = 256;
constexpr int kProbePer = 1;

__global__ __launch_bounds__(kProbeThreads) void k_read_probe(const uint4* __restrict__ p,
                                                              int64_t n16, float* out) {
    const int64_t tid = (int64_t)blockIdx.x * kProbeThreads + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * kProbeThreads;
    uint4 v[kProbePer];
#pragma unroll
    for (int k = 0; k < kProbePer; ++k) {
        const int64_t i = tid + k * stride;
        v[k] = p[i < n16 ? i : n16 - 1];
    }
    uint32_t acc = 0;
#pragma unroll
    for (int k = 0; k < kProbePer; ++k) acc ^= v[k].x ^ v[k].y ^ v[k].z ^ v[k].w;
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) acc ^= __shfl_xor(acc, m);
    // one store per wave for the first 256 waves; later waves store only on a
    // data pattern, so every wave's loads stay live without a burst of stores
    const int gw = (int)blockIdx.x * (kProbeThreads / 64) + (int)(threadIdx.x >> 6);
    if ((threadIdx.x & 63) == 0 && (gw < 256 || acc == 0x9e3779b9u)) out[gw & 255] = (float)acc;
}

// ---------------------------------------------------------------- host side

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

int check_dims(int q, int N, int K) {
    if (q < 1 || q > SA_MAX_Q) return SA_ERR_Q;
    if (N < 1 || K < 8 || (K & 7)) return SA_ERR_SHAPE;
    // every element count that the kernels index must fit comfortably; one
    // plane of packed keys stays below 2^31 bytes (32-bit per-lane offsets)
    if ((int64_t)q * N * K > (int64_t)1 << 36) return SA_ERR_SHAPE;
    if ((int64_t)N * (K / 8) >= (int64_t)1 << 31) return SA_ERR_SHAPE;
    return SA_OK;
}

int validate_gemm(const void* x, const void* packed, const void* exps, int q, int N, int K,
                  int group, int batch, const void* y) {
    if (!x || !packed || !exps || !y) return SA_ERR_NULL;
    int st = check_dims(q, N, K);
    if (st != SA_OK) return st;
    if (batch < 1 || batch > SA_MAX_BATCH) return SA_ERR_SHAPE;
    if (group < 8 || (group & 7) || (K % group)) return SA_ERR_GROUP;
    if (!aligned16(x) || !aligned16(packed) || !aligned16(y)) return SA_ERR_ALIGN;
    return SA_OK;
}

// Row kernel grid: as many workgroups as are resident at once (two per CU up
// to kRowsResidentQ planes, one beyond), or fewer when there are fewer row
// groups; more only when a workgroup would otherwise hold more than kMaxRG
// row groups.  The kernel spreads the row groups evenly over the grid.
int rows_workgroups(int q, int N) {
    const int resident = q <= kRowsResidentQ ? 512 : 256;
    const int groups = (N + kGroupRows - 1) / kGroupRows;
    int w = groups < resident ? groups : resident;
    if ((groups + w - 1) / w > kMaxRG) w = (groups + kMaxRG - 1) / kMaxRG;
    return w;
}

// Batch kernel geometry: rows per workgroup 16*KW.  Every (row tile, quad)
// pair is one workgroup, and the kernel is bound by LDS work, which the
// workgroups resident on a CU share: per workgroup and piece the queries cost
// about 16.5*rows*q LDS cycles (two 16-byte reads per key and quad) and the
// table build about 1144 (eight waves of 32 four-byte writes, which cost about
// four times as much per byte as the reads); a CU runs ceil(workgroups / 256)
// workgroups.  The KW with the least LDS work on the busiest CU wins.
int batch_kw(int q, int N, int batch, int builds = 1, int max_kw = 4) {
    const int64_t quads = (batch + kQuad - 1) / kQuad;
    int best_kw = 1;
    double best = -1;
    for (int kw = 1; kw <= max_kw; kw <<= 1) {
        const int64_t rows = 16 * kw;
        const int64_t wgs = (N + rows - 1) / rows * quads;
        const double cost =
            (double)((wgs + 255) / 256) * (16.5 * (double)rows * q + 1144.0 * builds);
        if (best < 0 || cost < best) {
            best = cost;
            best_kw = kw;
        }
    }
    return best_kw;
}

void make_plan(int q, int N, int K, int group, int batch, sa_plan* p, int builds = 1,
               int max_kw = 4) {
    *p = sa_plan{};
    p->threads = kThreads;
    if (group % 128 == 0 && batch >= 2) {
        const int kw = batch_kw(q, N, batch, builds, max_kw);
        const int tiles = (N + 16 * kw - 1) / (16 * kw);
        const int quads = (batch + kQuad - 1) / kQuad;
        p->path = 2;
        p->rows_per_wg = 16 * kw;
        p->workgroups = 8 * quads * ((tiles + 7) / 8);
        p->pieces = (K / 128 + kRowWaves - 1) / kRowWaves;
        p->threads = kRowThreads;
        p->lds_bytes = sizeof(float) * (kRowWaves * kWaveTableFloats + kRowWaves * kBatchRows * kQuad);
        return;
    }
    if (group % 128 != 0) {
        p->path = 0;
        p->rows_per_wg = kThreads;
        p->workgroups = ((N + kThreads - 1) / kThreads) * batch;
        p->pieces = (K / 8 + kBlockChunks - 1) / kBlockChunks;
        p->lds_bytes = sizeof(float) * (kBlockChunks * 256 + SA_MAX_Q * kThreads);
        return;
    }
    const int groups = (N + kGroupRows - 1) / kGroupRows;
    int wgs = rows_workgroups(q, N);
    p->pieces = (K / 128 + kPieceBlocks - 1) / kPieceBlocks;
    // Several pieces and 449..512 row groups: two groups per workgroup on 225
    // to 256 workgroups (16 waves, below), so each piece's tables serve 32
    // rows instead of 16 (8192x28672 q=3: 27.2 -> 25.1 us); fewer groups would
    // leave CUs idle
    if (q <= kRowsResidentQ && p->pieces >= 2 && groups > 448 && groups <= 512)
        wgs = (groups + 1) / 2;
    p->path = 1;
    p->rows_per_wg = kGroupRows * ((groups + wgs - 1) / wgs);  // the largest share
    p->workgroups = wgs;
    // Two pieces in flight per workgroup (16 waves, 128 KB of tables) where
    // the workgroups leave a CU to each: up to 4 planes (128 registers at four
    // waves per SIMD), at most 256 workgroups, several pieces.
    const int split = (q <= kRowsResidentQ && wgs <= 256 && p->pieces >= 2) ? 2 : 1;
    p->threads = kRowThreads * split;
    p->lds_bytes = sizeof(float) * split * (16 * kRegionFloats + kRowWaves * kGroupRows * kMaxRG);
}

// Column-wise factors: the row kernel with one plane per job (path 3, batch
// 1), or the batch kernel building each plane's tables in turn (path 6).
void make_plan_colwise(int q, int N, int K, int batch, sa_plan* p) {
    if (batch >= 2) {
        make_plan(q, N, K, 128, batch, p, q);
        p->path = 6;
        return;
    }
    *p = sa_plan{};
    const int groups = (N + kGroupRows - 1) / kGroupRows;
    int wgs = rows_workgroups(1, N);
    p->pieces = (K / 128 + kPieceBlocks - 1) / kPieceBlocks;
    if (p->pieces >= 2 && groups > 448 && groups <= 512) wgs = (groups + 1) / 2;  // as in make_plan
    p->path = 3;
    p->rows_per_wg = kGroupRows * ((groups + wgs - 1) / wgs);
    p->workgroups = wgs;
    const int split = (wgs <= 256 && p->pieces >= 2) ? 2 : 1;  // as in make_plan
    p->threads = kRowThreads * split;
    p->lds_bytes = sizeof(float) * split * (16 * kRegionFloats + kRowWaves * kGroupRows * kMaxRG);
}

// Block-wise factors: the row kernel (batch 1, path 4) or the batch kernel
// (batch >= 2, path 5) with a shift per key.  The batch kernel holds each
// job's 16 key exponents per plane in scalar registers when row_block is a
// multiple of its 16*KW rows, else in vector registers.  With 4 planes KW is
// capped at 2: at 4 key words per lane the variant does not fit the vector
// registers of four waves per SIMD (measured slower than 2 key words).
void make_plan_blockwise(int q, int N, int K, int row_block, int batch, sa_plan* p) {
    (void)row_block;
    make_plan(q, N, K, 128, batch, p, 1, q == 4 ? 2 : 4);
    if (batch < 2 && q == 4 && p->threads == 2 * kRowThreads) {
        // the 16-wave row kernel with 4 planes and a shift per key spills
        p->threads = kRowThreads;
        p->lds_bytes /= 2;
    }
    p->path = batch >= 2 ? 5 : 4;
}

// Estimated time (us) of the batch table kernel on a row-wise (terms = 0) or
// additive layer: rounds of workgroups over the CUs times the pieces a workgroup
// walks, or the latency of those pieces.  Fitted to 2986 drawn layers, weights
// rotated over 320 MB (5th and 95th percentile of estimate / measured 0.85 and 1.16
// row-wise, 0.75 and 1.28 additive).
double table_us(int q, int N, int K, int batch, int terms) {
    const int kw = batch_kw(q, N, batch);
    const int rows = 16 * kw;
    const double rounds = (double)((N + rows - 1) / rows) * ((batch + kQuad - 1) / kQuad) / 256;
    const double pieces = (K / 128 + kRowWaves - 1) / kRowWaves;
    // base, walk (fixed, per plane), work (fixed, per plane and row tile), by terms
    static const double kFit[SA_MAX_TERMS + 1][5] = {{2.6, 0.016, 0.31, 0.44, 0.18},
                                                     {3.0, 0.40, 0.39, 0.64, 0.195},
                                                     {2.9, 0.28, 0.49, 0.59, 0.24},
                                                     {2.8, 0.18, 1.01, 0.52, 0.33},
                                                     {2.9, 0.38, 0.58, 0.63, 0.27}};
    const double* f = kFit[terms];
    const double walk = f[1] + f[2] * q;
    const double work = (rounds > 1 ? rounds : 1) * (f[3] + f[4] * q * kw);
    return f[0] + pieces * (walk > work ? walk : work);
}

// The kernel of a row-wise (terms = 0) or additive batch: the least estimated time,
// a matrix-core kernel where it is 7% below the table kernel's (kernel 0: the
// geometry of make_plan).  On 4576 drawn layers 1% of the calls are more than 3%
// slower than the table kernel, 0.4% more than 10%, and the geometric mean is 0.85
// of its time (0.82 would be the best kernel for every layer).
void make_matrix_plan(int q, int N, int K, int group, int terms, int batch, sa_matrix_plan* p) {
    *p = sa_matrix_plan{};
    if (batch < 2 || q > 4 || group % 128) return;
    double best = 0.93 * table_us(q, N, K, batch, terms);
    sa_matrix_plan c;
    double us = sa_mx::plan(q, N, K, group, batch, terms, &c);
    if (us < best) {
        best = us;
        *p = c;
    }
    us = sa_mfma::plan(q, N, K, group, batch, terms, &c);
    if (us < best) *p = c;
}

int launch_status() { return hipGetLastError() == hipSuccess ? SA_OK : SA_ERR_HIP; }

int grid_for(int64_t items) {
    int64_t g = (items + kThreads - 1) / kThreads;
    if (g > 16384) g = 16384;
    if (g < 1) g = 1;
    return (int)g;
}

template <bool OUT16 = false>
void launch_rows(int q, const RowsArgs& a, int workgroups, int split, hipStream_t s) {
    const dim3 g(workgroups), b(kRowThreads * split);
    if (split == 2) {
        switch (q) {
            case 1: hipLaunchKernelGGL((k_gemm_rows<1, 2, OUT16>), g, b, 0, s, a); break;
            case 2: hipLaunchKernelGGL((k_gemm_rows<2, 2, OUT16>), g, b, 0, s, a); break;
            case 3: hipLaunchKernelGGL((k_gemm_rows<3, 2, OUT16>), g, b, 0, s, a); break;
            default: hipLaunchKernelGGL((k_gemm_rows<4, 2, OUT16>), g, b, 0, s, a); break;
        }
        return;
    }
    switch (q) {
        case 1: hipLaunchKernelGGL((k_gemm_rows<1, 1, OUT16>), g, b, 0, s, a); break;
        case 2: hipLaunchKernelGGL((k_gemm_rows<2, 1, OUT16>), g, b, 0, s, a); break;
        case 3: hipLaunchKernelGGL((k_gemm_rows<3, 1, OUT16>), g, b, 0, s, a); break;
        case 4: hipLaunchKernelGGL((k_gemm_rows<4, 1, OUT16>), g, b, 0, s, a); break;
        case 5: hipLaunchKernelGGL((k_gemm_rows_wide<5, OUT16>), g, b, 0, s, a); break;
        case 6: hipLaunchKernelGGL((k_gemm_rows_wide<6, OUT16>), g, b, 0, s, a); break;
        case 7: hipLaunchKernelGGL((k_gemm_rows_wide<7, OUT16>), g, b, 0, s, a); break;
        default: hipLaunchKernelGGL((k_gemm_rows_wide<8, OUT16>), g, b, 0, s, a); break;
    }
}

template <int KW, int MODE, bool UNI, bool OUT16 = false>
void launch_batch_kw(int q, const BatchArgs& a, int workgroups, hipStream_t s) {
    const dim3 g(workgroups), b(kRowThreads);
    switch (q) {
        case 1: hipLaunchKernelGGL((k_gemm_batch<1, KW, MODE, UNI, false, OUT16>), g, b, 0, s, a); break;
        case 2: hipLaunchKernelGGL((k_gemm_batch<2, KW, MODE, UNI, false, OUT16>), g, b, 0, s, a); break;
        case 3: hipLaunchKernelGGL((k_gemm_batch<3, KW, MODE, UNI, false, OUT16>), g, b, 0, s, a); break;
        case 4: hipLaunchKernelGGL((k_gemm_batch<4, KW, MODE, UNI, false, OUT16>), g, b, 0, s, a); break;
        case 5: hipLaunchKernelGGL((k_gemm_batch_wide<5, KW, MODE, UNI, OUT16>), g, b, 0, s, a); break;
        case 6: hipLaunchKernelGGL((k_gemm_batch_wide<6, KW, MODE, UNI, OUT16>), g, b, 0, s, a); break;
        case 7: hipLaunchKernelGGL((k_gemm_batch_wide<7, KW, MODE, UNI, OUT16>), g, b, 0, s, a); break;
        default: hipLaunchKernelGGL((k_gemm_batch_wide<8, KW, MODE, UNI, OUT16>), g, b, 0, s, a); break;
    }
}

template <int MODE = kRowWise, bool UNI = false, bool OUT16 = false>
void launch_batch(int q, int kw, const BatchArgs& a, int workgroups, hipStream_t s) {
    if (kw == 4) launch_batch_kw<4, MODE, UNI, OUT16>(q, a, workgroups, s);
    else if (kw == 2) launch_batch_kw<2, MODE, UNI, OUT16>(q, a, workgroups, s);
    else launch_batch_kw<1, MODE, UNI, OUT16>(q, a, workgroups, s);
}

// Preloaded exponents and term signs (additive batch kernel, up to 3 planes
// within 128 registers): the bytes a lane needs over all its pieces, or 0
// where the per-piece loads are used.  Needs G = 128 and K % 1024 == 0 (every
// wave owns whole blocks, so a lane's bytes stay inside its row), a load of
// 4, 8 or 16 bytes, and base pointers aligned to it.
int pre_bytes(int q, int K, int G, int T, const void* p0, const void* p1) {
    if (G != 128 || K % 1024 || q > 3) return 0;
    const int pieces = K / 1024;
    const int lw = pieces * T;
    if (lw != 4 && lw != 8 && lw != 16) return 0;
    if ((reinterpret_cast<uintptr_t>(p0) % lw) || (p1 && reinterpret_cast<uintptr_t>(p1) % lw))
        return 0;
    return lw;
}

// q in [1, 3] (pre_bytes is 0 otherwise)
template <int KW, int MODE>
void launch_batch_pre_kw(int q, const BatchArgs& a, int workgroups, hipStream_t s) {
    const dim3 g(workgroups), b(kRowThreads);
    if (q == 1) hipLaunchKernelGGL((k_gemm_batch<1, KW, MODE, false, true>), g, b, 0, s, a);
    else if (q == 2) hipLaunchKernelGGL((k_gemm_batch<2, KW, MODE, false, true>), g, b, 0, s, a);
    else if (q == 3) hipLaunchKernelGGL((k_gemm_batch<3, KW, MODE, false, true>), g, b, 0, s, a);
}

template <int MODE>
void launch_batch_pre(int q, int kw, const BatchArgs& a, int workgroups, hipStream_t s) {
    if (kw == 4) launch_batch_pre_kw<4, MODE>(q, a, workgroups, s);
    else if (kw == 2) launch_batch_pre_kw<2, MODE>(q, a, workgroups, s);
    else launch_batch_pre_kw<1, MODE>(q, a, workgroups, s);
}

}  // namespace

extern "C" {

SA_API size_t sa_packed_bytes(int q, int N, int K) {
    if (check_dims(q, N, K) != SA_OK) return 0;
    return (size_t)q * N * (K / 8);
}

SA_API int64_t sa_packed_offset(int q, int N, int K, int i, int n, int c) {
    if (check_dims(q, N, K) != SA_OK) return -1;
    if (i < 0 || i >= q || n < 0 || n >= N || c < 0 || c >= K / 8) return -1;
    return layout_offset(i, n, c, N, K / 8);
}

SA_API int sa_pack_weights(const int8_t* signs, int q, int N, int K, uint8_t* packed_bits,
                           void* stream) {
    if (!signs || !packed_bits) return SA_ERR_NULL;
    const int st = check_dims(q, N, K);
    if (st != SA_OK) return st;
    if (!aligned16(packed_bits)) return SA_ERR_ALIGN;
    const int64_t items = (int64_t)q * N * (K / 8);
    hipLaunchKernelGGL(k_pack, dim3(grid_for(items)), dim3(kThreads), 0,
                       reinterpret_cast<hipStream_t>(stream), signs, q, N, K / 8, packed_bits);
    return launch_status();
}

SA_API int sa_unpack_weights(const uint8_t* packed_bits, int q, int N, int K, int8_t* signs,
                             void* stream) {
    if (!signs || !packed_bits) return SA_ERR_NULL;
    const int st = check_dims(q, N, K);
    if (st != SA_OK) return st;
    if (!aligned16(packed_bits)) return SA_ERR_ALIGN;
    const int64_t items = (int64_t)q * N * (K / 8);
    hipLaunchKernelGGL(k_unpack, dim3(grid_for(items)), dim3(kThreads), 0,
                       reinterpret_cast<hipStream_t>(stream), packed_bits, q, N, K / 8, signs);
    return launch_status();
}

SA_API int sa_build_lut(const uint16_t* x, int K, int batch, float* lut, void* stream) {
    if (!x || !lut) return SA_ERR_NULL;
    if (K < 8 || (K & 7) || batch < 1 || batch > SA_MAX_BATCH) return SA_ERR_SHAPE;
    if (!aligned16(x) || !aligned16(lut)) return SA_ERR_ALIGN;
    const int64_t items = (int64_t)batch * (K / 8) * 16;
    hipLaunchKernelGGL(k_build_lut, dim3(grid_for(items)), dim3(kThreads), 0,
                       reinterpret_cast<hipStream_t>(stream), x, K, batch, lut);
    return launch_status();
}

SA_API int sa_plan_gemm(int q, int N, int K, int group, int batch, sa_plan* plan) {
    if (!plan) return SA_ERR_NULL;
    int st = check_dims(q, N, K);
    if (st != SA_OK) return st;
    if (batch < 1 || batch > SA_MAX_BATCH) return SA_ERR_SHAPE;
    if (group < 8 || (group & 7) || (K % group)) return SA_ERR_GROUP;
    make_plan(q, N, K, group, batch, plan);
    return SA_OK;
}

SA_API int sa_plan_gemm_matrix(int q, int N, int K, int group, int terms, int batch,
                               sa_matrix_plan* plan) {
    if (!plan) return SA_ERR_NULL;
    const int st = check_dims(q, N, K);
    if (st != SA_OK) return st;
    if (batch < 1 || batch > SA_MAX_BATCH || terms < 0 || terms > SA_MAX_TERMS) return SA_ERR_SHAPE;
    if (group < 8 || (group & 7) || (K % group) || (terms && group % 128)) return SA_ERR_GROUP;
    make_matrix_plan(q, N, K, group, terms, batch, plan);
    return SA_OK;
}

// The layer with fp32 (out_half = 0) or binary16 (out_half = 1) outputs.
int shiftadd_gemm(const uint16_t* x, const uint8_t* packed_bits, const int8_t* exps, int q, int N,
                  int K, int group, int batch, float* y, int out_half, void* stream) {
    const int st = validate_gemm(x, packed_bits, exps, q, N, K, group, batch, y);
    if (st != SA_OK) return st;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    sa_matrix_plan mp;
    make_matrix_plan(q, N, K, group, 0, batch, &mp);
    if (mp.kernel) {
        const sa_matrix::Args a = {x, packed_bits, exps, nullptr, q, N, K, group, batch, 0, y, out_half};
        if (mp.kernel == 1) sa_mx::launch(a, mp, s);
        else sa_mfma::launch(a, mp, s);
        return launch_status();
    }
    sa_plan plan;
    make_plan(q, N, K, group, batch, &plan);
    if (plan.path == 0) {
        hipLaunchKernelGGL(k_gemm_generic, dim3((N + kThreads - 1) / kThreads, batch),
                           dim3(kThreads), 0, s,
                           x, packed_bits, exps, q, N, K, group, y, out_half);
        return launch_status();
    }
    if (plan.path == 2) {
        BatchArgs a{};
        a.x = x;
        a.packed = packed_bits;
        a.exps = exps;
        a.q = q;
        a.N = N;
        a.K = K;
        a.G = group;
        a.B = batch;
        a.y = y;
        const int kw = plan.rows_per_wg / 16;
        a.n_tiles = (N + plan.rows_per_wg - 1) / plan.rows_per_wg;
        a.n_quads = (batch + kQuad - 1) / kQuad;
        if (out_half)
            launch_batch<kRowWise, false, true>(q, kw, a, plan.workgroups, s);
        else
            launch_batch(q, kw, a, plan.workgroups, s);
        return launch_status();
    }
    RowsArgs a{};
    a.x = x;
    a.packed = packed_bits;
    a.exps = exps;
    a.q = q;
    a.N = N;
    a.K = K;
    a.G = group;
    a.B = batch;
    a.y = y;
    a.groups = (N + kGroupRows - 1) / kGroupRows;
    if (out_half)
        launch_rows<true>(q, a, plan.workgroups, plan.threads / kRowThreads, s);
    else
        launch_rows(q, a, plan.workgroups, plan.threads / kRowThreads, s);
    return launch_status();
}

SA_API int sa_shiftadd_gemm(const uint16_t* x, const uint8_t* packed_bits, const int8_t* exps,
                            int q, int N, int K, int group, int batch, float* y, void* stream) {
    return shiftadd_gemm(x, packed_bits, exps, q, N, K, group, batch, y, 0, stream);
}

SA_API int sa_shiftadd_gemm_f16(const uint16_t* x, const uint8_t* packed_bits, const int8_t* exps,
                                int q, int N, int K, int group, int batch, uint16_t* y,
                                void* stream) {
    return shiftadd_gemm(x, packed_bits, exps, q, N, K, group, batch,
                         reinterpret_cast<float*>(y), 1, stream);
}

// K-slice grid: one workgroup per (slice, row range); the ranges fill one
// workgroup per CU (256) where there are enough 8-row jobs, at least 16 jobs
// (one per wave) per range otherwise.
void kslice_geometry(int N, int K, int* slices, int* ranges, int* jobs) {
    *slices = K / kSliceCols;
    *jobs = (N + kSliceJobRows - 1) / kSliceJobRows;
    int r = 256 / *slices;
    const int by_jobs = (*jobs + kSliceWaves - 1) / kSliceWaves;
    if (r > by_jobs) r = by_jobs;
    *ranges = r < 1 ? 1 : r;
}

SA_API size_t sa_kslice_workspace_bytes(int N, int K) {
    if (N < 1 || K < kSliceCols || K % kSliceCols) return 0;
    return sizeof(float) * (size_t)(K / kSliceCols) * (size_t)N;
}

SA_API int sa_shiftadd_gemm_kslice(const uint16_t* x, const uint8_t* packed_bits,
                                   const int8_t* exps, int q, int N, int K, int group, float* y,
                                   float* workspace, size_t workspace_bytes, void* stream) {
    const int st = validate_gemm(x, packed_bits, exps, q, N, K, group, 1, y);
    if (st != SA_OK) return st;
    if (!workspace) return SA_ERR_NULL;
    if (reinterpret_cast<uintptr_t>(workspace) & 3) return SA_ERR_ALIGN;
    if (group % 128) return SA_ERR_GROUP;
    if (K % kSliceCols) return SA_ERR_SHAPE;
    SliceArgs a{};
    kslice_geometry(N, K, &a.slices, &a.ranges, &a.jobs);
    if (workspace_bytes < sizeof(float) * (size_t)a.slices * (size_t)N) return SA_ERR_SHAPE;
    a.x = x;
    a.packed = packed_bits;
    a.exps = exps;
    a.q = q;
    a.N = N;
    a.K = K;
    a.G = group;
    a.part = workspace;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    const dim3 g(a.slices * a.ranges), b(kSliceThreads);
    switch (q) {
        case 1: hipLaunchKernelGGL(k_gemm_kslice<1>, g, b, 0, s, a); break;
        case 2: hipLaunchKernelGGL(k_gemm_kslice<2>, g, b, 0, s, a); break;
        case 3: hipLaunchKernelGGL(k_gemm_kslice<3>, g, b, 0, s, a); break;
        case 4: hipLaunchKernelGGL(k_gemm_kslice<4>, g, b, 0, s, a); break;
        case 5: hipLaunchKernelGGL(k_gemm_kslice<5>, g, b, 0, s, a); break;
        case 6: hipLaunchKernelGGL(k_gemm_kslice<6>, g, b, 0, s, a); break;
        case 7: hipLaunchKernelGGL(k_gemm_kslice<7>, g, b, 0, s, a); break;
        default: hipLaunchKernelGGL(k_gemm_kslice<8>, g, b, 0, s, a); break;
    }
    hipLaunchKernelGGL(k_sum_slices, dim3((N + 255) / 256), dim3(256), 0, s, workspace, a.slices,
                       N, y);
    return launch_status();
}

SA_API int sa_plan_gemm_blockwise(int q, int N, int K, int row_block, int batch,
                                  sa_plan* plan) {
    if (!plan) return SA_ERR_NULL;
    const int st = check_dims(q, N, K);
    if (st != SA_OK) return st;
    if (batch < 1 || batch > SA_MAX_BATCH || (K % 128) || row_block < 1) return SA_ERR_SHAPE;
    make_plan_blockwise(q, N, K, row_block, batch, plan);
    return SA_OK;
}

SA_API int sa_shiftadd_gemm_blockwise(const uint16_t* x, const uint8_t* packed_bits,
                                      const int8_t* blk_exps, int q, int N, int K, int row_block,
                                      int batch, float* y, void* stream) {
    if (!x || !packed_bits || !blk_exps || !y) return SA_ERR_NULL;
    const int st = check_dims(q, N, K);
    if (st != SA_OK) return st;
    if (batch < 1 || batch > SA_MAX_BATCH || (K % 128) || row_block < 1) return SA_ERR_SHAPE;
    if (!aligned16(x) || !aligned16(packed_bits) || !aligned16(y) || !aligned16(blk_exps))
        return SA_ERR_ALIGN;
    sa_plan plan;
    make_plan_blockwise(q, N, K, row_block, batch, &plan);
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    if (plan.path == 5) {
        BatchArgs a{};
        a.x = x;
        a.packed = packed_bits;
        a.exps = blk_exps;  // not read in this mode
        a.blk_exps = blk_exps;
        a.q = q;
        a.N = N;
        a.K = K;
        a.G = K;
        a.B = batch;
        a.y = y;
        a.row_block = row_block;
        a.NB = (N + row_block - 1) / row_block;
        const int kw = plan.rows_per_wg / 16;
        a.n_tiles = (N + plan.rows_per_wg - 1) / plan.rows_per_wg;
        a.n_quads = (batch + kQuad - 1) / kQuad;
        if (row_block % plan.rows_per_wg == 0)
            launch_batch<kBlockWise, true>(q, kw, a, plan.workgroups, s);
        else
            launch_batch<kBlockWise, false>(q, kw, a, plan.workgroups, s);
        return launch_status();
    }
    RowsArgs a{};
    a.x = x;
    a.packed = packed_bits;
    a.blk_exps = blk_exps;
    a.q = q;
    a.N = N;
    a.K = K;
    a.G = K;
    a.B = batch;
    a.y = y;
    a.groups = (N + kGroupRows - 1) / kGroupRows;
    a.row_block = row_block;
    a.NB = (N + row_block - 1) / row_block;
    const dim3 g(plan.workgroups), b(plan.threads);
    if (plan.threads == 2 * kRowThreads) {
        switch (q) {
            case 1: hipLaunchKernelGGL((k_gemm_rows_blk<1, 2>), g, b, 0, s, a); break;
            case 2: hipLaunchKernelGGL((k_gemm_rows_blk<2, 2>), g, b, 0, s, a); break;
            case 3: hipLaunchKernelGGL((k_gemm_rows_blk<3, 2>), g, b, 0, s, a); break;
            default: hipLaunchKernelGGL((k_gemm_rows_blk<4, 2>), g, b, 0, s, a); break;
        }
        return launch_status();
    }
    switch (q) {
        case 1: hipLaunchKernelGGL(k_gemm_rows_blk<1>, g, b, 0, s, a); break;
        case 2: hipLaunchKernelGGL(k_gemm_rows_blk<2>, g, b, 0, s, a); break;
        case 3: hipLaunchKernelGGL(k_gemm_rows_blk<3>, g, b, 0, s, a); break;
        case 4: hipLaunchKernelGGL(k_gemm_rows_blk<4>, g, b, 0, s, a); break;
        case 5: hipLaunchKernelGGL(k_gemm_rows_blk_wide<5>, g, b, 0, s, a); break;
        case 6: hipLaunchKernelGGL(k_gemm_rows_blk_wide<6>, g, b, 0, s, a); break;
        case 7: hipLaunchKernelGGL(k_gemm_rows_blk_wide<7>, g, b, 0, s, a); break;
        default: hipLaunchKernelGGL(k_gemm_rows_blk_wide<8>, g, b, 0, s, a); break;
    }
    return launch_status();
}

SA_API int sa_shiftadd_gemm_terms(const uint16_t* x, const uint8_t* packed_bits,
                                  const int8_t* exps, const int8_t* term_signs, int q, int N,
                                  int K, int group, int terms, int batch, float* y,
                                  void* stream) {
    if (!term_signs) return SA_ERR_NULL;
    const int st = validate_gemm(x, packed_bits, exps, q, N, K, group, batch, y);
    if (st != SA_OK) return st;
    if (group % 128) return SA_ERR_GROUP;
    if (terms < 1 || terms > SA_MAX_TERMS) return SA_ERR_SHAPE;
    // the T bytes of a group are loaded at once: 2- and 4-byte loads need that alignment
    const uintptr_t al = terms == 2 ? 1u : (terms == 4 ? 3u : 0u);
    if ((reinterpret_cast<uintptr_t>(exps) & al) || (reinterpret_cast<uintptr_t>(term_signs) & al))
        return SA_ERR_ALIGN;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    sa_matrix_plan mp;
    make_matrix_plan(q, N, K, group, terms, batch, &mp);
    if (mp.kernel) {
        const sa_matrix::Args a = {x, packed_bits, exps, term_signs, q, N, K, group, batch, terms, y, 0};
        if (mp.kernel == 1) sa_mx::launch(a, mp, s);
        else sa_mfma::launch(a, mp, s);
        return launch_status();
    }
    sa_plan plan;
    make_plan(q, N, K, group, batch, &plan);  // row kernel (batch 1) or batch kernel
    if (plan.path == 2) {
        BatchArgs a{};
        a.x = x;
        a.packed = packed_bits;
        a.exps = exps;
        a.term_signs = term_signs;
        a.terms = terms;
        a.q = q;
        a.N = N;
        a.K = K;
        a.G = group;
        a.B = batch;
        a.y = y;
        const int kw = plan.rows_per_wg / 16;
        a.n_tiles = (N + plan.rows_per_wg - 1) / plan.rows_per_wg;
        a.n_quads = (batch + kQuad - 1) / kQuad;
        a.pre_bytes = pre_bytes(q, K, group, terms, exps, term_signs);
        if (a.pre_bytes && q <= 3)
            launch_batch_pre<kAdditive>(q, kw, a, plan.workgroups, s);
        else
            launch_batch<kAdditive>(q, kw, a, plan.workgroups, s);
        return launch_status();
    }
    RowsArgs a{};
    a.x = x;
    a.packed = packed_bits;
    a.exps = exps;
    a.term_signs = term_signs;
    a.terms = terms;
    a.q = q;
    a.N = N;
    a.K = K;
    a.G = group;
    a.B = batch;
    a.y = y;
    a.groups = (N + kGroupRows - 1) / kGroupRows;
    const dim3 g(plan.workgroups), b(plan.threads);
    if (plan.threads == 2 * kRowThreads) {
        switch (q) {
            case 1: hipLaunchKernelGGL((k_gemm_rows_add<1, 2>), g, b, 0, s, a); break;
            case 2: hipLaunchKernelGGL((k_gemm_rows_add<2, 2>), g, b, 0, s, a); break;
            case 3: hipLaunchKernelGGL((k_gemm_rows_add<3, 2>), g, b, 0, s, a); break;
            default: hipLaunchKernelGGL((k_gemm_rows_add<4, 2>), g, b, 0, s, a); break;
        }
        return launch_status();
    }
    switch (q) {
        case 1: hipLaunchKernelGGL(k_gemm_rows_add<1>, g, b, 0, s, a); break;
        case 2: hipLaunchKernelGGL(k_gemm_rows_add<2>, g, b, 0, s, a); break;
        case 3: hipLaunchKernelGGL(k_gemm_rows_add<3>, g, b, 0, s, a); break;
        case 4: hipLaunchKernelGGL(k_gemm_rows_add<4>, g, b, 0, s, a); break;
        case 5: hipLaunchKernelGGL(k_gemm_rows_add_wide<5>, g, b, 0, s, a); break;
        case 6: hipLaunchKernelGGL(k_gemm_rows_add_wide<6>, g, b, 0, s, a); break;
        case 7: hipLaunchKernelGGL(k_gemm_rows_add_wide<7>, g, b, 0, s, a); break;
        default: hipLaunchKernelGGL(k_gemm_rows_add_wide<8>, g, b, 0, s, a); break;
    }
    return launch_status();
}

SA_API int sa_plan_gemm_colwise(int q, int N, int K, int batch, sa_plan* plan) {
    if (!plan) return SA_ERR_NULL;
    const int st = check_dims(q, N, K);
    if (st != SA_OK) return st;
    if (batch < 1 || batch > SA_MAX_BATCH || (K % 128)) return SA_ERR_SHAPE;
    make_plan_colwise(q, N, K, batch, plan);
    return SA_OK;
}

SA_API int sa_shiftadd_gemm_colwise(const uint16_t* x, const uint8_t* packed_bits,
                                    const int8_t* col_exps, int q, int N, int K, int batch,
                                    float* y, void* stream) {
    if (!x || !packed_bits || !col_exps || !y) return SA_ERR_NULL;
    const int st = check_dims(q, N, K);
    if (st != SA_OK) return st;
    if (batch < 1 || batch > SA_MAX_BATCH || (K % 128)) return SA_ERR_SHAPE;
    if (!aligned16(x) || !aligned16(packed_bits) || !aligned16(y) ||
        (reinterpret_cast<uintptr_t>(col_exps) & 7u))
        return SA_ERR_ALIGN;
    sa_plan plan;
    make_plan_colwise(q, N, K, batch, &plan);
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    if (plan.path == 6) {
        BatchArgs a{};
        a.x = x;
        a.packed = packed_bits;
        a.exps = col_exps;  // not read in this mode
        a.col_exps = col_exps;
        a.q = q;
        a.N = N;
        a.K = K;
        a.G = K;
        a.B = batch;
        a.y = y;
        const int kw = plan.rows_per_wg / 16;
        a.n_tiles = (N + plan.rows_per_wg - 1) / plan.rows_per_wg;
        a.n_quads = (batch + kQuad - 1) / kQuad;
        launch_batch<kColWise>(q, kw, a, plan.workgroups, s);
        return launch_status();
    }
    RowsArgs a{};
    a.x = x;
    a.packed = packed_bits;
    a.exps = nullptr;
    a.col_exps = col_exps;
    a.q = q;
    a.N = N;
    a.K = K;
    a.G = K;
    a.B = batch;
    a.y = y;
    a.groups = (N + kGroupRows - 1) / kGroupRows;
    if (plan.threads == 2 * kRowThreads)
        hipLaunchKernelGGL(k_gemm_rows_col<2>, dim3(plan.workgroups), dim3(plan.threads), 0, s, a);
    else
        hipLaunchKernelGGL(k_gemm_rows_col<1>, dim3(plan.workgroups), dim3(plan.threads), 0, s, a);
    return launch_status();
}

SA_API int sa_read_probe(const void* buf, size_t bytes, float* out, void* stream) {
    if (!buf || !out) return SA_ERR_NULL;
    if (bytes < 16 || (bytes & 15) || bytes > ((size_t)1 << 40)) return SA_ERR_SHAPE;
    if (!aligned16(buf)) return SA_ERR_ALIGN;
    const int64_t n16 = (int64_t)(bytes / 16);
    const int64_t per_wg = (int64_t)kProbeThreads * kProbePer;
    const int64_t grid = (n16 + per_wg - 1) / per_wg;
    hipLaunchKernelGGL(k_read_probe, dim3((unsigned)grid), dim3(kProbeThreads), 0,
                       reinterpret_cast<hipStream_t>(stream),
                       reinterpret_cast<const uint4*>(buf), n16, out);
    return launch_status();
}

SA_API const char* sa_status_string(int status) {
    switch (status) {
        case SA_OK: return "ok";
        case SA_ERR_NULL: return "a required pointer is NULL";
        case SA_ERR_SHAPE: return "invalid shape (N, K, batch or sizes out of range, or K % 8 != 0)";
        case SA_ERR_Q: return "q must be in [1, 8]";
        case SA_ERR_GROUP: return "group must be a multiple of 8 that divides K";
        case SA_ERR_ALIGN: return "x, packed_bits, y and lut must be 16-byte aligned";
        case SA_ERR_HIP: return "HIP runtime error or kernel launch failure";
        default: return "unknown status";
    }
}

SA_API const char* sa_version(void) { return SA_VERSION_STRING; }

}  // extern "C"
