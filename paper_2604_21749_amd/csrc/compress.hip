// Compression of mesh geometry for gfx950 (Sec. 4.6): index range and position bounding box
// (a partial result per workgroup, then one workgroup), bit packing of indices relative to their minimum
// and 16-bit quantization of positions relative to the bounding box.  The decoding side lives in
// device.h (packed_index, mesh_vertex); the host entry points in runtime.hip.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "device.h"

namespace curast {

// Order-preserving map of binary32 to uint32 (negative values reversed below the positive ones).
__device__ __forceinline__ uint32_t ordered_bits(float f)
{
    const uint32_t u = __builtin_bit_cast(uint32_t, f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ uint32_t wave_min(uint32_t v)
{
    for (int off = 32; off > 0; off >>= 1) v = min(v, (uint32_t)__shfl_xor((int)v, off));
    return v;
}

__device__ __forceinline__ uint32_t wave_max(uint32_t v)
{
    for (int off = 32; off > 0; off >>= 1) v = max(v, (uint32_t)__shfl_xor((int)v, off));
    return v;
}

// Index range and position bounding box: blocks [0, gi) reduce the indices, the other gp blocks the
// positions, each into its own partial result; range_final_kernel joins them.  Bound by reading both
// arrays once (16-byte loads, four in flight per lane).  One atomic per wavefront on the eight result
// words, as this was before, serialized at the memory side: 573 us for the box of 9.0 M vertices and
// 235 us for the range of 54 M indices; the two launches here take 67 us together
// (324 MB, 52 us at the streaming read rate).
typedef float f32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));
struct RangeAcc {
    uint32_t lo[3], hi[3];
};

__device__ __forceinline__ void block_reduce(RangeAcc& r, uint32_t (&s)[4][6])
{
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        r.lo[c] = wave_min(r.lo[c]);
        r.hi[c] = wave_max(r.hi[c]);
    }
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            s[threadIdx.x >> 6][c] = r.lo[c];
            s[threadIdx.x >> 6][3 + c] = r.hi[c];
        }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        r.lo[c] = min(min(s[0][c], s[1][c]), min(s[2][c], s[3][c]));
        r.hi[c] = max(max(s[0][3 + c], s[1][3 + c]), max(s[2][3 + c], s[3][3 + c]));
    }
}

// part[6 b ..]: block b's {lo, lo, lo, hi, hi, hi} (three index lanes, or the ordered x, y, z)
__global__ void __launch_bounds__(256) range_kernel(const uint32_t* __restrict__ idx, uint64_t n_idx, uint32_t gi,
                                                    const float* __restrict__ pos, uint64_t n_pos, uint32_t gp,
                                                    uint32_t* __restrict__ part)
{
    __shared__ uint32_t s[4][6];
    RangeAcc r = {{0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu}, {0u, 0u, 0u}};
    if (blockIdx.x < gi) {
        const uint64_t n4 = n_idx >> 2, stride = (uint64_t)gi * 256;
        const CURAST_GLOBAL u32x4_a4* p = (const CURAST_GLOBAL u32x4_a4*)gl(idx);
        const uint64_t t = (uint64_t)blockIdx.x * 256 + threadIdx.x;
#pragma unroll 4
        for (uint64_t i = t; i < n4; i += stride) {
            const u32x4_a4 v = p[i];
            r.lo[0] = min(min(r.lo[0], min(v.x, v.y)), min(v.z, v.w));
            r.hi[0] = max(max(r.hi[0], max(v.x, v.y)), max(v.z, v.w));
        }
        if (t < (n_idx & 3)) {
            const uint32_t v = gl(idx)[4 * n4 + t];
            r.lo[0] = min(r.lo[0], v);
            r.hi[0] = max(r.hi[0], v);
        }
    } else {
        // 16-byte group i starts at component (4 i) % 3 = i % 3; the stride is a multiple of 3, so a lane
        // meets the same rotation of x, y, z in all its groups and undoes it once at the end
        const uint64_t n4 = n_pos >> 2, stride = (uint64_t)gp * 256;
        const CURAST_GLOBAL f32x4_a4* p = (const CURAST_GLOBAL f32x4_a4*)gl(pos);
        const uint64_t t = (uint64_t)(blockIdx.x - gi) * 256 + threadIdx.x;
        uint32_t lo[3] = {0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu}, hi[3] = {0u, 0u, 0u};
#pragma unroll 4
        for (uint64_t i = t; i < n4; i += stride) {
            const f32x4_a4 v = p[i];
            const uint32_t b[4] = {ordered_bits(v.x), ordered_bits(v.y), ordered_bits(v.z), ordered_bits(v.w)};
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                lo[c % 3] = min(lo[c % 3], b[c]);
                hi[c % 3] = max(hi[c % 3], b[c]);
            }
        }
        const uint32_t rot = (uint32_t)(t % 3);   // lo[k] belongs to component (k + rot) % 3
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            r.lo[c] = rot == 0 ? lo[c] : rot == 1 ? lo[(c + 2) % 3] : lo[(c + 1) % 3];
            r.hi[c] = rot == 0 ? hi[c] : rot == 1 ? hi[(c + 2) % 3] : hi[(c + 1) % 3];
        }
        if (t < (n_pos & 3)) {
            const uint64_t i = 4 * n4 + t;
            const uint32_t b = ordered_bits(gl(pos)[i]), comp = (uint32_t)(i % 3);
#pragma unroll
            for (uint32_t c = 0; c < 3; ++c)
                if (comp == c) {
                    r.lo[c] = min(r.lo[c], b);
                    r.hi[c] = max(r.hi[c], b);
                }
        }
    }
    block_reduce(r, s);
    if (threadIdx.x < 6) gl(part)[6 * (uint64_t)blockIdx.x + threadIdx.x] =
        threadIdx.x < 3 ? (threadIdx.x == 0 ? r.lo[0] : threadIdx.x == 1 ? r.lo[1] : r.lo[2])
                        : (threadIdx.x == 3 ? r.hi[0] : threadIdx.x == 4 ? r.hi[1] : r.hi[2]);
}

// out[0..7] = {index min, index max, ordered min x, y, z, ordered max x, y, z}; `out` is host memory
__global__ void __launch_bounds__(256) range_final_kernel(const uint32_t* __restrict__ part, uint32_t gi, uint32_t gp,
                                                          uint32_t* out)
{
    __shared__ uint32_t s[4][6];
    for (uint32_t kind = 0; kind < 2; ++kind) {
        RangeAcc r = {{0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu}, {0u, 0u, 0u}};
        const uint32_t first = kind ? gi : 0u, n = kind ? gp : gi;
        for (uint32_t b = threadIdx.x; b < n; b += 256)
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                r.lo[c] = min(r.lo[c], gl(part)[6 * (first + b) + c]);
                r.hi[c] = max(r.hi[c], gl(part)[6 * (first + b) + 3 + c]);
            }
        block_reduce(r, s);
        if (threadIdx.x == 0) {
            if (kind == 0) {
                out[0] = r.lo[0];
                out[1] = r.hi[0];
            } else {
                for (int c = 0; c < 3; ++c) {
                    out[2 + c] = r.lo[c];
                    out[5 + c] = r.hi[c];
                }
            }
        }
        __syncthreads();
    }
}

// Four 32-bit output words per lane: ORs in every value whose bits overlap the word (words past the
// last value, the padding, are 0).  Bit positions are 64-bit once per workgroup and 32-bit per lane
// (with two 64-bit divisions per word it took 138 us for 54 M
// 24-bit indices, here 113; reading 216 MB and writing 162 MB takes 73 us at the copy rate).
constexpr uint32_t kPackWords = 1024;          // words per workgroup

__global__ void __launch_bounds__(256) pack_kernel(const uint32_t* __restrict__ idx, uint64_t n, uint32_t bits,
                                                   uint32_t base, uint32_t* __restrict__ out, uint64_t words)
{
    const uint64_t w0 = (uint64_t)blockIdx.x * kPackWords;
    const uint64_t first = 32 * w0 / bits;                       // value holding the workgroup's first bit
    const uint32_t r0 = (uint32_t)(32 * w0 - first * bits);      // its bits before that one
    const CURAST_GLOBAL uint32_t* src = gl(idx) + first;
    const uint64_t left = first < n ? n - first : 0;
    const uint32_t avail = left < 0xFFFFFFFFull ? (uint32_t)left : 0xFFFFFFFFu;
#pragma unroll
    for (uint32_t k = 0; k < kPackWords / 256; ++k) {
        const uint32_t lw = k * 256 + threadIdx.x;
        if (w0 + lw >= words) break;
        const uint32_t o = r0 + 32 * lw;
        uint32_t i = o / bits;
        int32_t shift = (int32_t)(i * bits - o);                 // position of value i in the word
        uint32_t word = 0;
        for (; shift < 32 && i < avail; ++i, shift += (int32_t)bits) {
            const uint32_t v = src[i] - base;
            word |= shift >= 0 ? v << shift : v >> -shift;
        }
        gl(out)[w0 + lw] = word;
    }
}

// Position components in pairs, one 4-byte store per pair: q = clamp(rint((p - lo) * scale), 0, 65535)
// in binary32; element n, the padding, is 0.  59 us with one component and a 2-byte store per lane, 41 us
// here, for 9.0 M vertices (31 us at the copy rate).
constexpr uint32_t kQuantPairs = 1024;         // pairs per workgroup

__global__ void __launch_bounds__(256) quantize_kernel(const float* __restrict__ pos, uint64_t n, float lx, float ly,
                                                       float lz, float sx, float sy, float sz,
                                                       uint16_t* __restrict__ out)
{
    const uint64_t e0 = 2ull * kQuantPairs * blockIdx.x;         // the workgroup's first element
    const uint32_t c0 = (uint32_t)(e0 % 3);
#pragma unroll
    for (uint32_t k = 0; k < kQuantPairs / 256; ++k) {
        const uint32_t j = 2 * (k * 256 + threadIdx.x);
        const uint64_t e = e0 + j;
        if (e > n) break;
        uint32_t q[2] = {0, 0};
#pragma unroll
        for (uint32_t h = 0; h < 2; ++h)
            if (e + h < n) {
                const uint32_t c = (c0 + j + h) % 3;
                const float lo = c == 0 ? lx : c == 1 ? ly : lz;
                const float sc = c == 0 ? sx : c == 1 ? sy : sz;
                const float t = __builtin_rintf((gl(pos)[e + h] - lo) * sc);
                q[h] = (uint32_t)(uint16_t)(t < 0.0f ? 0.0f : t > 65535.0f ? 65535.0f : t);
            }
        if (e + 1 <= n) *(CURAST_GLOBAL uint32_t*)(gl(out) + e) = q[0] | q[1] << 16;
        else gl(out)[e] = (uint16_t)q[0];
    }
}

// part: kRangeWords words of device scratch; out: 8 words of pinned host memory
hipError_t launch_compress_ranges(const uint32_t* idx, uint64_t n_idx, const float* pos, uint32_t V, uint32_t* part,
                                  uint32_t* out, hipStream_t s)
{
    // a workgroup reads 4096 values in one round of its unrolled loop
    auto blocks = [](uint64_t n) {
        return n ? (uint32_t)std::min<uint64_t>((n + 4095) / 4096 + 2, kRangeBlocks) / 3 * 3 : 0u;
    };
    const uint32_t gi = blocks(n_idx), gp = blocks(3ull * V);
    if (gi + gp) range_kernel<<<gi + gp, 256, 0, s>>>(idx, n_idx, gi, pos, 3ull * V, gp, part);
    range_final_kernel<<<1, 256, 0, s>>>(part, gi, gp, out);
    return hipGetLastError();
}

hipError_t launch_compress(const uint32_t* idx, uint64_t n_idx, uint32_t bits, uint32_t base, uint32_t* packed,
                           uint64_t words, const float* pos, uint32_t V, const float lo[3], const float scale[3],
                           uint16_t* qpos, hipStream_t s)
{
    auto blocks = [](uint64_t n, uint32_t per) { return (uint32_t)((n + per - 1) / per); };
    if (words) pack_kernel<<<blocks(words, kPackWords), 256, 0, s>>>(idx, n_idx, bits, base, packed, words);
    const uint64_t n = 3ull * V;
    quantize_kernel<<<blocks(n + 1, 2 * kQuantPairs), 256, 0, s>>>(pos, n, lo[0], lo[1], lo[2], scale[0], scale[1],
                                                                   scale[2], qpos);
    return hipGetLastError();
}

}  // namespace curast
