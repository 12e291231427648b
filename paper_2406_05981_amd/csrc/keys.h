// What every kernel of the layer needs to read keys and exponents of the packed
// layout (16-byte key rows, rotated by the row).
#ifndef SHIFTADD_KEYS_H
#define SHIFTADD_KEYS_H

#include <hip/hip_runtime.h>
#include <stdint.h>

__host__ __device__ inline int imin(int a, int b) { return a < b ? a : b; }

// Bytes of v rotated so that byte p of the result is byte (p + r) mod 16 of v.  The
// key at position p of a row is chunk (p + row) mod 16 of its block: rotating 16
// exponents in chunk order by the row lines them up with the keys, rotating the
// keys by 16 - row puts them in chunk order.
__device__ inline void rotate16(const uint4 v, int r, uint32_t out[4]) {
    const uint32_t in[4] = {v.x, v.y, v.z, v.w};
    const uint32_t b = (uint32_t)(r & 3);
    uint32_t t[4], u[4];
#pragma unroll
    for (int d = 0; d < 4; ++d) t[d] = __builtin_amdgcn_alignbyte(in[(d + 1) & 3], in[d], b);
#pragma unroll
    for (int d = 0; d < 4; ++d) u[d] = (r & 4) ? t[(d + 1) & 3] : t[d];
#pragma unroll
    for (int d = 0; d < 4; ++d) out[d] = (r & 8) ? u[(d + 2) & 3] : u[d];
}

// T consecutive bytes (exponents or signs of a group's terms), one per byte of the
// result; 2 and 4 are aligned to their size (checked on the host).
__device__ inline uint32_t load_terms(const int8_t* p, int T) {
    const uint8_t* b = reinterpret_cast<const uint8_t*>(p);
    if (T == 4) return *reinterpret_cast<const uint32_t*>(b);
    if (T == 2) return *reinterpret_cast<const uint16_t*>(b);
    if (T == 3) return (uint32_t)b[0] | ((uint32_t)b[1] << 8) | ((uint32_t)b[2] << 16);
    return b[0];
}

#endif
