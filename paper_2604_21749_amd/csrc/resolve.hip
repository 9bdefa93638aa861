// Resolve kernels for gfx950 (Sec. 4.4): one lane per pixel decodes the 28-bit depth / 36-bit
// global triangle ID, finds the (mesh, instance) by binary search over the int64 exclusive
// prefix of triangle counts, reloads and re-projects the triangle, and interpolates its vertex
// attributes perspective-correctly at the pixel centre.  The paper shades in world space with a
// ray-plane intersection; the equivalent screen-space form used here is
//   b_k = q_k / (q0 + q1 + q2), q_k = lambda_k / w_k,
// lambda_k the 2-D cross products of the pixel-relative projected vertices, which stays valid for
// vertices behind the camera (the resolve uses the unclipped triangle).  The backward kernel
// differentiates that expression with visibility held fixed.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "device.h"

namespace curast {

struct Interp {
    float d[3][2];   // pixel-relative window positions
    float zI[3];
    float lam[3];
    float s;
    float b[3];
};

// fp32 interpolation weights in a fixed operation order (no contraction).
__device__ __forceinline__ void interp_weights(const float sx[3], const float sy[3], const float w[3], int32_t px,
                                               int32_t py, Interp& r)
{
    const float cx = (float)px + 0.5f, cy = (float)py + 0.5f;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        r.d[k][0] = sx[k] - cx;
        r.d[k][1] = sy[k] - cy;
        r.zI[k] = 1.0f / w[k];
    }
    r.lam[0] = r.d[1][0] * r.d[2][1] - r.d[1][1] * r.d[2][0];
    r.lam[1] = r.d[2][0] * r.d[0][1] - r.d[2][1] * r.d[0][0];
    r.lam[2] = r.d[0][0] * r.d[1][1] - r.d[0][1] * r.d[1][0];
    const float q0 = r.lam[0] * r.zI[0], q1 = r.lam[1] * r.zI[1], q2 = r.lam[2] * r.zI[2];
    r.s = (q0 + q1) + q2;
    r.b[0] = q0 / r.s;
    r.b[1] = q1 / r.s;
    r.b[2] = q2 / r.s;
}

// The pixel of a lane: workgroups of 256 lanes take 16 x 16 tiles, wavefronts 8 x 8, so that a
// wavefront's pixels share index, vertex and texel lines in both directions (256 pixels of a row
// before: textured resolve at 2557 x 1439 80 -> 51 us, RGB at 1600 x 900 47 -> 39, no gain where
// triangles are much smaller than pixels).  Tiles in launch order: an eighth of the image per XCD was
// 30% slower, since images are covered unevenly.
__device__ __forceinline__ bool tile_pixel(uint32_t W, uint32_t H, uint32_t& x, uint32_t& y)
{
    const uint32_t tx = (W + 15) / 16, by = blockIdx.x / tx, bx = blockIdx.x - by * tx;
    const uint32_t wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    x = bx * 16 + (wave & 1) * 8 + (lane & 7);
    y = by * 16 + (wave >> 1) * 8 + (lane >> 3);
    return x < W && y < H;
}

// Calls f with the channel count as a constant for the counts that have kernels of their own, 0 for
// the others; with MORE also for 5 to 7, which the resolves without supersampling take (differentiable
// resolve of 5 channels at 1280 x 720 16.5 us in groups of four, 10.1 with the constant).
template <bool MORE = false, class F>
static auto with_channels(uint32_t C, F&& f)
{
    if constexpr (MORE) switch (C) {
    case 5: return f(std::integral_constant<int, 5>());
    case 6: return f(std::integral_constant<int, 6>());
    case 7: return f(std::integral_constant<int, 7>());
    }
    switch (C) {
    case 1: return f(std::integral_constant<int, 1>());
    case 2: return f(std::integral_constant<int, 2>());
    case 3: return f(std::integral_constant<int, 3>());
    case 4: return f(std::integral_constant<int, 4>());
    case 8: return f(std::integral_constant<int, 8>());
    case 16: return f(std::integral_constant<int, 16>());
    default: return f(std::integral_constant<int, 0>());
    }
}

// put(c, value) for every interpolated channel (b0 a0 + b1 a1) + b2 a2 of three attribute rows, CC
// channels (0: C).  The rows' loads are issued four channels at a time (or all of a count that four does not
// divide) before any arithmetic.
template <int CC, class Put>
__device__ __forceinline__ void blend(const float* const (&a)[3], const float (&b)[3], uint32_t C, Put&& put)
{
    constexpr uint32_t G = CC == 0 || CC % 4 == 0 ? 4 : CC;
    const uint32_t n = CC ? (uint32_t)CC : C;
    auto group = [&](uint32_t c0) __attribute__((always_inline)) {
        float v[3][G];
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
            for (uint32_t c = 0; c < G; ++c) v[k][c] = CC || c0 + c < n ? gl(a[k])[c0 + c] : 0.0f;
#pragma unroll
        for (uint32_t c = 0; c < G; ++c)
            if (CC || c0 + c < n) put(c0 + c, (b[0] * v[0][c] + b[1] * v[1][c]) + b[2] * v[2][c]);
    };
    if constexpr (CC != 0) {
#pragma unroll
        for (uint32_t c0 = 0; c0 < (uint32_t)CC; c0 += G) group(c0);
    } else {
        for (uint32_t c0 = 0; c0 < n; c0 += G) group(c0);
    }
}

template <int CC>
__device__ __forceinline__ void write_zero(uint32_t C, float* o)
{
    const uint32_t n = CC ? (uint32_t)CC : C;
#pragma unroll
    for (uint32_t c = 0; c < n; ++c) gl(o)[c] = 0.0f;
}

// ----------------------------------------------------------------------------------------------
// Window positions of one mesh instance: pos_ss[v] = (sx, sy, w) before snapping
// ----------------------------------------------------------------------------------------------
struct ProjectArgs {
    MeshDesc mesh;                // plain or compressed positions
    float A[12];
    float hW, hH;
    float* out;
};

__global__ void __launch_bounds__(256) project_kernel(ProjectArgs a)
{
    const uint64_t v = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= a.mesh.V) return;
    float p[3];
    mesh_vertex(a.mesh, (uint32_t)v, p);
    const Clip c = transform(a.A, p[0], p[1], p[2]);
    const float zI = 1.0f / c.w;
    a.out[3 * v + 0] = __builtin_fmaf(c.x * zI, a.hW, a.hW);
    a.out[3 * v + 1] = __builtin_fmaf(c.y * zI, a.hH, a.hH);
    a.out[3 * v + 2] = c.w;
}

// ----------------------------------------------------------------------------------------------
// Resolve of a multi-mesh, multi-instance visibility buffer
// ----------------------------------------------------------------------------------------------
constexpr uint32_t kLdsBases = 2048;   // per-mesh first IDs staged in LDS for the binary search

// Where a resolve reads its descriptors: device memory, with the meshes' first IDs staged in LDS when
// they fit (kDescDevice); an LDS copy of the descriptor block that came with the kernel argument
// (kDescInline); or the argument itself, through scalar loads, for one mesh with one instance, whose
// descriptors are the same for every pixel (kDescOne).
enum DescMode : int { kDescDevice, kDescInline, kDescOne };

struct ResolveDesc {
    const uint64_t* bases;
    const uint32_t* mesh_pair;
    const DrawDesc* pairs;
    const MeshDesc* meshes;
    const float* const* attrs;
    const TexDesc* tex;
};

template <int MODE>
struct ResolveLds {
    uint64_t w[MODE == kDescOne ? 1 : MODE == kDescInline ? kResolveWords / 2 : kLdsBases + 1];
};

// All threads of the workgroup take part.  The argument's block is read where it lies (the first
// argument starts the kernel argument segment).
template <int MODE, int WORDS>
__device__ __forceinline__ ResolveDesc stage_desc(const ResolveBlock<WORDS>& blk, ResolveLds<MODE>& lds)
{
    ResolveDesc d;
    if constexpr (MODE == kDescDevice) {
        const ResolveArgs& a = blk.a;
        const bool staged = a.n_meshes <= kLdsBases;
        if (staged) {
            for (uint32_t i = threadIdx.x; i <= a.n_meshes; i += 256) lds.w[i] = gl(a.bases)[i];
            __syncthreads();
        }
        d.bases = staged ? lds.w : a.bases;
        d.mesh_pair = a.mesh_pair;
        d.pairs = a.pairs;
        d.meshes = a.meshes;
        d.attrs = a.attrs;
        d.tex = a.tex;
    } else {
        using Arg = const __attribute__((address_space(4))) ResolveBlock<WORDS>;
        Arg* k = (Arg*)__builtin_amdgcn_kernarg_segment_ptr();
        const char* base;
        if constexpr (MODE == kDescInline) {
            uint32_t* dst = reinterpret_cast<uint32_t*>(lds.w);
            const uint32_t n = k->words;
            for (uint32_t i = threadIdx.x; i < n; i += 256) dst[i] = k->w[i];
            __syncthreads();
            base = reinterpret_cast<const char*>(lds.w);
        } else {
            base = (const char*)(const __attribute__((address_space(4))) char*)k->w;
        }
        d.bases = reinterpret_cast<const uint64_t*>(base);
        d.mesh_pair = reinterpret_cast<const uint32_t*>(base + blk.off_mpair);
        d.pairs = reinterpret_cast<const DrawDesc*>(base + blk.off_pairs);
        d.meshes = reinterpret_cast<const MeshDesc*>(base + blk.off_meshes);
        d.attrs = reinterpret_cast<const float* const*>(base + blk.off_attrs);
        d.tex = reinterpret_cast<const TexDesc*>(base + blk.off_tex);
    }
    return d;
}

// floor(off / T) for T >= 1, off / T < 2^36: an approximate reciprocal with one Newton step (relative
// error below 2^-40) gives it to within one; a 64-bit division takes four times the instructions.
__device__ __forceinline__ uint64_t instance_of(uint64_t off, uint64_t T)
{
    const double t = (double)T;
    double r = __builtin_amdgcn_rcp(t);
    r = __builtin_fma(__builtin_fma(-t, r, 1.0), r, r);
    uint64_t q = (uint64_t)((double)off * r);
    if (q * T > off) --q;
    else if ((q + 1) * T <= off) ++q;
    return q;
}

// The (mesh, instance) pair and vertex indices of the triangle stored at pixel p; false for an
// empty pixel or an invalid triangle.
template <int MODE>
__device__ __forceinline__ bool pixel_triangle(const ResolveArgs& a, const ResolveDesc& d, uint32_t p, uint32_t& pair,
                                               uint32_t (&vi)[3])
{
    if constexpr (MODE == kDescOne) {
        const MeshDesc& M = d.meshes[0];
        const unsigned long long key = gl(a.vis)[p];
        const uint64_t id = key & kIdMask;
        if (key == kEmptyKey || id >= M.T) return false;
        mesh_triangle(M, id, vi);
        pair = 0;
        return vi[0] < M.V && vi[1] < M.V && vi[2] < M.V;
    }
    // the int64 prefix of triangle counts over (mesh, instance) pairs (Sec. 4.4) is searched at
    // mesh granularity: the instances of mesh m hold IDs B[m] + i T_m .. B[m] + (i + 1) T_m - 1,
    // so the instance is one exact integer division (the last mesh with B[m] <= id has T_m > 0)
    const uint32_t nm = a.n_meshes;
    const unsigned long long key = gl(a.vis)[p];
    const uint64_t id = key & kIdMask;
    if (key == kEmptyKey || id >= d.bases[nm]) return false;
    uint32_t lo = 0, hi = nm;
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (d.bases[mid] <= id) lo = mid;
        else hi = mid;
    }
    const MeshDesc& M = d.meshes[lo];
    const uint64_t off = id - d.bases[lo];
    const uint64_t inst = off >= M.T ? instance_of(off, M.T) : 0;
    mesh_triangle(M, off - inst * M.T, vi);
    pair = d.mesh_pair[lo] + (uint32_t)inst;
    return vi[0] < M.V && vi[1] < M.V && vi[2] < M.V;
}

// Window positions of a triangle's vertices under a pair's draw matrix, in the rasterizer's fp32
// operations before snapping.
__device__ __forceinline__ void pixel_windows(const ResolveArgs& a, const DrawDesc& D, const MeshDesc& M,
                                              const uint32_t (&vi)[3], float (&sx)[3], float (&sy)[3], float (&w)[3])
{
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        float q[3];
        mesh_vertex(M, vi[k], q);
        const Clip c = transform(D.A, q[0], q[1], q[2]);
        const float zI = 1.0f / c.w;
        sx[k] = __builtin_fmaf(c.x * zI, a.hW, a.hW);
        sy[k] = __builtin_fmaf(c.y * zI, a.hH, a.hH);
        w[k] = c.w;
    }
}

// put(c, value) for every channel of pixel (x, y) of the view; false for an empty pixel
// or an invalid triangle.
template <int CC, int MODE, class Put>
__device__ __forceinline__ bool resolve_pixel(const ResolveArgs& a, const ResolveDesc& d, uint32_t x, uint32_t y,
                                              Put&& put)
{
    uint32_t pair, vi[3];
    if (!pixel_triangle<MODE>(a, d, y * (uint32_t)a.W + x, pair, vi)) return false;
    const DrawDesc& D = d.pairs[pair];
    const uint32_t m = MODE == kDescOne ? 0u : D.mesh;
    const float* at = d.attrs[m];
    const float* rows[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) rows[k] = at + (size_t)vi[k] * (CC ? (uint32_t)CC : a.C);
    float sx[3], sy[3], w[3];
    pixel_windows(a, D, d.meshes[m], vi, sx, sy, w);
    Interp r;
    interp_weights(sx, sy, w, (int32_t)x, (int32_t)y, r);
    blend<CC>(rows, r.b, a.C, put);
    return true;
}

// Bound by gathering, through a chain of three dependent loads (key, indices, vertices and attribute
// rows), from triangles that neighbouring pixels of a dense mesh do not share.  The channel count is
// a constant for the usual counts, so that the attribute rows load together with the vertices instead
// of one channel per round trip (1080p RGB of a 33.5M-triangle scan 85 -> 68 us, 8 channels over
// instances 41 -> 20 us).
template <int CC, int MODE, int WORDS>
__global__ void __launch_bounds__(256) resolve_kernel(ResolveBlock<WORDS> blk)
{
    __shared__ ResolveLds<MODE> lds;
    const ResolveDesc d = stage_desc<MODE>(blk, lds);
    const ResolveArgs& a = blk.a;
    uint32_t x, y;
    if (!tile_pixel((uint32_t)a.W, (uint32_t)a.H, x, y)) return;
    float* o = a.out + (size_t)(y * (uint32_t)a.W + x) * (CC ? (uint32_t)CC : a.C);
    if (!resolve_pixel<CC, MODE>(a, d, x, y, [&](uint32_t c, float v) { gl(o)[c] = v; })) write_zero<CC>(a.C, o);
}

// Supersampled resolve: the view holds ss x ss samples per output pixel (a visibility buffer of
// ss W_out x ss H_out).  One lane per sample, a pixel's samples on
// neighbouring lanes (one lane per pixel walked its samples one after the other: 25 -> 15.5 us for
// 960 x 540 pixels of 2 x 2 samples); the samples' channels meet in LDS, where one lane per (pixel, channel) sums them in fp32 row by row
// (empty samples add 0) and scales by 1 / ss^2 (exact).
constexpr uint32_t kMaxChannels = 16;

template <int CC, int MODE, int WORDS>
__global__ void __launch_bounds__(256) resolve_ss_kernel(ResolveBlock<WORDS> blk)
{
    constexpr uint32_t kStride = (CC ? (uint32_t)CC : kMaxChannels) | 1u;   // odd: no bank conflicts
    __shared__ ResolveLds<MODE> lds;
    __shared__ float s_val[256 * kStride];
    const ResolveDesc d = stage_desc<MODE>(blk, lds);
    const ResolveArgs& a = blk.a;
    const uint32_t C = CC ? (uint32_t)CC : a.C;
    const uint32_t ls = a.ss == 2 ? 1u : 2u, k = a.ss, kk = k * k;          // 2 x 2 or 4 x 4 samples
    const uint32_t lt = 4 - ls, T = 1u << lt;                               // T x T output pixels per workgroup
    const uint32_t Wo = (uint32_t)a.W >> ls, Ho = (uint32_t)a.H >> ls;
    const uint32_t tx = (Wo + T - 1) >> lt, by = blockIdx.x / tx, bx = blockIdx.x - by * tx;
    const uint32_t q = threadIdx.x >> (2 * ls), s = threadIdx.x & (kk - 1);  // pixel of the tile, sample of the pixel
    const uint32_t px = (bx << lt) + (q & (T - 1)), py = (by << lt) + (q >> lt);
    float* mine = s_val + threadIdx.x * kStride;
    bool hit = false;
    if (px < Wo && py < Ho)
        hit = resolve_pixel<CC, MODE>(a, d, (px << ls) + (s & (k - 1)), (py << ls) + (s >> ls),
                                      [&](uint32_t c, float v) { mine[c] = v; });
    if (!hit)
        for (uint32_t c = 0; c < C; ++c) mine[c] = 0.0f;
    __syncthreads();
    const float scale = 1.0f / (float)kk;
    for (uint32_t it = threadIdx.x; it < T * T * C; it += 256) {
        const uint32_t o = it / C, c = it - o * C;
        const uint32_t ox = (bx << lt) + (o & (T - 1)), oy = (by << lt) + (o >> lt);
        if (ox >= Wo || oy >= Ho) continue;
        const float* v = s_val + (o << (2 * ls)) * kStride + c;
        float acc = 0.0f;
        for (uint32_t i = 0; i < kk; ++i) acc += v[i * kStride];
        gl(a.out)[(size_t)(oy * Wo + ox) * C + c] = acc * scale;
    }
}

// ----------------------------------------------------------------------------------------------
// Textured resolve (Sec. 4.4, "Shading and Mip Mapping").  Rays through the pixel and its right,
// top and top-right neighbours hit the triangle's plane; their barycentrics are solved in clip
// space (the world-to-clip map is affine, so they equal the world-space ones, and no vertex is
// divided by its w):
//   n = ((sx - W/2) / (W/2), (sy - H/2) / (H/2)),  a_k = fmaf(-n.x, w_k, x_k),  c_k likewise,
//   e = a x c,  s = (e0 + e1) + e2,  uv = ((e0 uv0 + e1 uv1) + e2 uv2) / s.
// lod = log2 of the larger UV extent of the four hits in texels, clamped to the chain; the colour
// is the trilinear, wrap-around sample at the pixel's own hit.
// ----------------------------------------------------------------------------------------------
struct Footprint {
    uint32_t t00, t10, t01, t11;   // the four texels
    float ax, ay;                  // their weights
};

__device__ __forceinline__ Footprint texels_at(const TexDesc& T, uint32_t l, float u, float v)
{
    const uint32_t wl = max(1u, T.w >> l), hl = max(1u, T.h >> l);
    const CURAST_GLOBAL uint32_t* L = gl(T.texels) + T.off[l];
    const float fu = u - floorf(u), fv = v - floorf(v);
    const float x = fu * (float)wl - 0.5f, y = fv * (float)hl - 0.5f;
    const float x0 = floorf(x), y0 = floorf(y);
    // x0 lies in [-1, wl - 1] and y0 in [-1, hl - 1]; the clamps only guard the addressing
    const int32_t ix = (int32_t)x0, iy = (int32_t)y0;
    const uint32_t i0 = min(ix < 0 ? wl - 1 : (uint32_t)ix, wl - 1), i1 = ix + 1 >= (int32_t)wl ? 0u : (uint32_t)(ix + 1);
    const uint32_t j0 = min(iy < 0 ? hl - 1 : (uint32_t)iy, hl - 1), j1 = iy + 1 >= (int32_t)hl ? 0u : (uint32_t)(iy + 1);
    Footprint f;
    f.t00 = L[(size_t)j0 * wl + i0];
    f.t10 = L[(size_t)j0 * wl + min(i1, wl - 1)];
    f.t01 = L[(size_t)min(j1, hl - 1) * wl + i0];
    f.t11 = L[(size_t)min(j1, hl - 1) * wl + min(i1, wl - 1)];
    f.ax = x - x0;
    f.ay = y - y0;
    return f;
}

__device__ __forceinline__ float4 bilinear(const Footprint& f)
{
    const float k = 1.0f / 255.0f;
    float r[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const float c00 = (float)((f.t00 >> (8 * c)) & 0xFFu) * k, c10 = (float)((f.t10 >> (8 * c)) & 0xFFu) * k;
        const float c01 = (float)((f.t01 >> (8 * c)) & 0xFFu) * k, c11 = (float)((f.t11 >> (8 * c)) & 0xFFu) * k;
        const float r0 = c00 + f.ax * (c10 - c00);
        const float r1 = c01 + f.ax * (c11 - c01);
        r[c] = r0 + f.ay * (r1 - r0);
    }
    return make_float4(r[0], r[1], r[2], r[3]);
}

template <int MODE, int WORDS>
__global__ void __launch_bounds__(256) resolve_textured_kernel(ResolveBlock<WORDS> blk)
{
    __shared__ ResolveLds<MODE> lds;
    const ResolveDesc d = stage_desc<MODE>(blk, lds);
    const ResolveArgs& a = blk.a;
    uint32_t x, y;
    if (!tile_pixel((uint32_t)a.W, (uint32_t)a.H, x, y)) return;
    const uint32_t p = y * (uint32_t)a.W + x;
    CURAST_GLOBAL float4* o = (CURAST_GLOBAL float4*)gl(a.out) + p;
    uint32_t pr, vi[3];
    if (!pixel_triangle<MODE>(a, d, p, pr, vi)) {
        *o = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        return;
    }
    const DrawDesc& D = d.pairs[pr];
    const uint32_t m = MODE == kDescOne ? 0u : D.mesh;
    const MeshDesc& M = d.meshes[m];
    float cx[3], cy[3], cw[3], tu[3], tv[3];
    const CURAST_GLOBAL float* uv = gl(d.attrs[m]);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        float q[3];
        mesh_vertex(M, vi[k], q);
        const Clip c = transform(D.A, q[0], q[1], q[2]);
        cx[k] = c.x;
        cy[k] = c.y;
        cw[k] = c.w;
        tu[k] = uv[2 * (size_t)vi[k]];
        tv[k] = uv[2 * (size_t)vi[k] + 1];
    }
    const int32_t px = (int32_t)x, py = (int32_t)y;
    float su[4], sv[4];
    bool finite = true;
#pragma unroll
    for (int smp = 0; smp < 4; ++smp) {
        const float sx = (float)px + ((smp & 1) ? 1.5f : 0.5f), sy = (float)py + ((smp & 2) ? 1.5f : 0.5f);
        const float nx = (sx - a.hW) / a.hW, ny = (sy - a.hH) / a.hH;
        float e_a[3], e_c[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            e_a[k] = __builtin_fmaf(-nx, cw[k], cx[k]);
            e_c[k] = __builtin_fmaf(-ny, cw[k], cy[k]);
        }
        const float e0 = e_a[1] * e_c[2] - e_a[2] * e_c[1];
        const float e1 = e_a[2] * e_c[0] - e_a[0] * e_c[2];
        const float e2 = e_a[0] * e_c[1] - e_a[1] * e_c[0];
        const float s = (e0 + e1) + e2;
        su[smp] = ((e0 * tu[0] + e1 * tu[1]) + e2 * tu[2]) / s;
        sv[smp] = ((e0 * tv[0] + e1 * tv[1]) + e2 * tv[2]) / s;
        finite = finite && __builtin_isfinite(su[smp]) && __builtin_isfinite(sv[smp]);
    }
    if (!__builtin_isfinite(su[0]) || !__builtin_isfinite(sv[0])) {
        *o = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        return;
    }
    const TexDesc& T = d.tex[m];
    const float top = (float)(T.levels - 1);
    float lod = top;
    if (finite) {
        float umin = su[0], umax = su[0], vmin = sv[0], vmax = sv[0];
#pragma unroll
        for (int smp = 1; smp < 4; ++smp) {
            umin = fminf(umin, su[smp]);
            umax = fmaxf(umax, su[smp]);
            vmin = fminf(vmin, sv[smp]);
            vmax = fmaxf(vmax, sv[smp]);
        }
        const float du = (umax - umin) * (float)T.w, dv = (vmax - vmin) * (float)T.h;
        lod = log2f(fmaxf(du, dv));
        lod = lod > 0.0f ? lod : 0.0f;
        lod = lod > top ? top : lod;
    }
    const uint32_t l0 = (uint32_t)floorf(lod);
    const float t = lod - (float)l0;
    // the texels of both levels are loaded before either is filtered
    const bool two = t > 0.0f && l0 + 1 < T.levels;
    const Footprint f0 = texels_at(T, l0, su[0], sv[0]);
    Footprint f1 = f0;
    if (two) f1 = texels_at(T, l0 + 1, su[0], sv[0]);
    float4 c = bilinear(f0);
    if (two) {
        const float4 c1 = bilinear(f1);
        c.x = c.x + t * (c1.x - c.x);
        c.y = c.y + t * (c1.y - c.y);
        c.z = c.z + t * (c1.z - c.z);
        c.w = c.w + t * (c1.w - c.w);
    }
    *o = c;
}

// Level l + 1 of a chain from level l: per-channel rounded mean of a 2 x 2 block, coordinates
// clamped to level l.
__global__ void __launch_bounds__(256) mip_kernel(const uint32_t* __restrict__ src, uint32_t pw, uint32_t ph,
                                                  uint32_t* __restrict__ dst, uint32_t cw, uint32_t ch)
{
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (uint64_t)cw * ch) return;
    const uint32_t x = (uint32_t)(i % cw), y = (uint32_t)(i / cw);
    const uint32_t x0 = 2 * x, y0 = 2 * y, x1 = min(2 * x + 1, pw - 1), y1 = min(2 * y + 1, ph - 1);
    const CURAST_GLOBAL uint32_t* S = gl(src);
    const uint32_t q0 = S[(size_t)y0 * pw + x0], q1 = S[(size_t)y0 * pw + x1];
    const uint32_t q2 = S[(size_t)y1 * pw + x0], q3 = S[(size_t)y1 * pw + x1];
    uint32_t out = 0;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const uint32_t sum = 2 + ((q0 >> (8 * c)) & 0xFFu) + ((q1 >> (8 * c)) & 0xFFu) + ((q2 >> (8 * c)) & 0xFFu) +
                             ((q3 >> (8 * c)) & 0xFFu);
        out |= (sum >> 2) << (8 * c);
    }
    gl(dst)[i] = out;
}

// ----------------------------------------------------------------------------------------------
// Screen-space (differentiable) resolve of one mesh and its backward pass
// ----------------------------------------------------------------------------------------------
__device__ __forceinline__ bool screen_tri(const ScreenArgs& a, uint32_t p, uint32_t (&vi)[3])
{
    const unsigned long long key = gl(a.vis)[p];
    if (key == kEmptyKey) return false;
    const uint64_t id = key & kIdMask;
    if (id < a.id_base || id - a.id_base >= a.T) return false;
    const CURAST_GLOBAL uint32_t* ip = gl(a.idx) + 3 * (id - a.id_base);
    vi[0] = ip[0];
    vi[1] = ip[1];
    vi[2] = ip[2];
    return vi[0] < a.V && vi[1] < a.V && vi[2] < a.V;
}

__device__ __forceinline__ void screen_windows(const ScreenArgs& a, const uint32_t (&vi)[3], float (&sx)[3],
                                               float (&sy)[3], float (&w)[3])
{
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const CURAST_GLOBAL float* q = gl(a.pos_ss) + 3 * (size_t)vi[k];
        sx[k] = q[0];
        sy[k] = q[1];
        w[k] = q[2];
    }
}

template <int CC>
__global__ void __launch_bounds__(256) resolve_screen_kernel(ScreenArgs a)
{
    uint32_t x, y;
    if (!tile_pixel((uint32_t)a.W, (uint32_t)a.H, x, y)) return;
    const uint32_t p = y * (uint32_t)a.W + x;
    const uint32_t C = CC ? (uint32_t)CC : a.C;
    float* o = a.out + (size_t)p * C;
    uint32_t vi[3];
    if (!screen_tri(a, p, vi)) {
        write_zero<CC>(C, o);
        return;
    }
    const float* rows[3] = {a.attrs + (size_t)vi[0] * C, a.attrs + (size_t)vi[1] * C, a.attrs + (size_t)vi[2] * C};
    float sx[3], sy[3], w[3];
    screen_windows(a, vi, sx, sy, w);
    Interp r;
    interp_weights(sx, sy, w, (int32_t)x, (int32_t)y, r);
    blend<CC>(rows, r.b, C, [&](uint32_t c, float v) { gl(o)[c] = v; });
}

// Backward with visibility held fixed.  The chain rule of one pixel has cancelling terms
// (G_j - sum_k G_k b_k, the cross-product partials of sliver triangles), so it is evaluated in
// fp64 from the fp32 inputs:
//   dL/da_k = g b_k;  G_k = g . a_k;  dL/dq_j = (G_j - sum_k G_k b_k) / s;
//   dL/dlambda_j = dL/dq_j zI_j;  dL/dw_j = -(dL/dq_j lambda_j) zI_j^2;
//   lambda_0 = d1 x d2, lambda_1 = d2 x d0, lambda_2 = d0 x d1 with d_k = s_k - pixel centre.
//
// Each contribution is rounded once to fp32.  Device-scope fp32 atomics are performed at the memory
// side, one request per 64-byte sector and instruction, about 17 G requests/s: that rate bounds the
// kernels, not the bytes.  So a workgroup adds the contributions of its 16 x 16 pixel tile in LDS first,
// one table row (C attribute and 3 position components) per vertex, and then issues one atomic per
// touched row and component, neighbouring lanes on neighbouring components and rows.  A vertex's row is
// its low bits where it can be, so that the rows of neighbouring vertices, which share sectors, stay neighbours
// in the table.  1.80 M requests (2.25 M with one staged row per pixel and vertex) for 0.46 M pixels of a
// 10M-triangle mesh take 103 us, 143 before; 0.2 M pixels of coarser meshes, 4 channels and positions,
// 269 us with an atomic per value and 57 here.
constexpr uint32_t kBwdSlots = 1024;           // at most 3 x 256 vertices per tile: never full

// The fp64 terms of one pixel's chain rule, from the fp32 window positions (sx, sy, w) of its
// triangle's vertices and the pixel (x, y).
struct BwdTerms {
    double d[3][2];   // pixel-relative positions
    double zI[3];
    double lam[3];
    double b[3];
    double inv_sum;   // 1 / (q0 + q1 + q2)
};

__device__ __forceinline__ void bwd_terms(const float (&sx)[3], const float (&sy)[3], const float (&w)[3], uint32_t x,
                                          uint32_t y, BwdTerms& t)
{
    const double cx = (double)x + 0.5, cy = (double)y + 0.5;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        t.d[k][0] = (double)sx[k] - cx;
        t.d[k][1] = (double)sy[k] - cy;
        t.zI[k] = 1.0 / (double)w[k];
    }
    t.lam[0] = t.d[1][0] * t.d[2][1] - t.d[1][1] * t.d[2][0];
    t.lam[1] = t.d[2][0] * t.d[0][1] - t.d[2][1] * t.d[0][0];
    t.lam[2] = t.d[0][0] * t.d[1][1] - t.d[0][1] * t.d[1][0];
    const double q[3] = {t.lam[0] * t.zI[0], t.lam[1] * t.zI[1], t.lam[2] * t.zI[2]};
    t.inv_sum = 1.0 / (q[0] + q[1] + q[2]);
#pragma unroll
    for (int k = 0; k < 3; ++k) t.b[k] = q[k] * t.inv_sum;
}

// Gradients to (sx, sy, w) of the three vertices from G_k = g . a_k, each rounded once to fp32.
__device__ __forceinline__ void bwd_pos(const BwdTerms& t, const double (&G)[3], float (&gpos)[3][3])
{
    const double Gb = G[0] * t.b[0] + G[1] * t.b[1] + G[2] * t.b[2];
    double L[3], dw[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        const double Q = (G[j] - Gb) * t.inv_sum;
        L[j] = Q * t.zI[j];
        dw[j] = -(Q * t.lam[j]) * t.zI[j] * t.zI[j];
    }
    const double gx[3] = {L[2] * t.d[1][1] - L[1] * t.d[2][1], L[0] * t.d[2][1] - L[2] * t.d[0][1],
                          L[1] * t.d[0][1] - L[0] * t.d[1][1]};
    const double gy[3] = {L[1] * t.d[2][0] - L[2] * t.d[1][0], L[2] * t.d[0][0] - L[0] * t.d[2][0],
                          L[0] * t.d[1][0] - L[1] * t.d[0][0]};
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        gpos[k][0] = (float)gx[k];
        gpos[k][1] = (float)gy[k];
        gpos[k][2] = (float)dw[k];
    }
}

// Table rows of a pixel's three vertices, inserted where they are new (`first`).  A vertex's row is the low bits
// of its index; if that is taken, a row among those of its group of 8 vertices, which the group's hash places; from
// there on odd steps, which reach every row and are the same for all vertices of a block of the table's size.  Low
// bits alone, with the steps right after them, made the rows of a lat-long sphere's tile share an eighth of the table
// wherever a row of the mesh has 2^k + 1 vertices (4.2 M triangles, 130 K pixels, 3 channels and positions 46 us, 28
// with the groups; 16.8 M triangles 95 and 50); hashed groups alone cost a mesh of rows that do not collide their
// neighbourhood (train step of a 10M-triangle scan 290 us, 283 with the low bits first).  Steps by the group's hash
// instead scatter what the blocks hold together: a frame of 38 meshes at 28 triangles a pixel 61 us, 35 with the
// blocks' steps, 32 without the groups.  The three are probed together, a placed one again at its own row, so that
// a round costs one LDS round trip instead of three.
template <class Key>
__device__ __forceinline__ void bwd_slots(Key* keys, const Key (&key)[3], const uint32_t (&v)[3], uint32_t (&slot)[3],
                                          bool (&first)[3])
{
    constexpr Key kFree = (Key)~(Key)0;
    uint32_t move[3], step[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        slot[k] = v[k] & (kBwdSlots - 1);
        move[k] = (((v[k] >> 3) * 2654435761u >> 25) << 3 | (v[k] & 7)) - slot[k];
        step[k] = ((v[k] / kBwdSlots) * 2654435761u >> 20) | 1u;
        first[k] = false;
    }
    bool more;
    do {
        Key prev[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) prev[k] = atomicCAS(keys + slot[k], kFree, key[k]);
        more = false;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const bool other = prev[k] != kFree && prev[k] != key[k];
            first[k] |= prev[k] == kFree;
            slot[k] = other ? (slot[k] + move[k]) & (kBwdSlots - 1) : slot[k];
            move[k] = other ? step[k] : move[k];
            more |= other;
        }
    } while (more);
}

// A pixel's upstream gradient and the attribute rows of its three vertices, G channels from c0 on,
// loaded together.
template <int CC, bool POS>
struct BwdChannels {
    static constexpr uint32_t G = CC == 0 || CC > 4 ? 4 : CC;
    float g[G], at[3][G];
    __device__ __forceinline__ void load(const float* const (&rows)[3], const float* grad, uint32_t c0, uint32_t n)
    {
#pragma unroll
        for (uint32_t c = 0; c < G; ++c) {
            const bool in = CC || c0 + c < n;
            g[c] = in ? gl(grad)[c0 + c] : 0.0f;
#pragma unroll
            for (int k = 0; k < 3; ++k) at[k][c] = POS && in ? gl(rows[k])[c0 + c] : 0.0f;
        }
    }
};

// The table rows of one pixel's vertices, and the contributions it adds to them: attribute gradients
// g b_k and, with POS and `pos`, the position gradients.  The pixel that inserted a row stores into it
// (`store`, which also makes clearing the rows unnecessary), then, after a barrier, the others add
// (`add`): LDS float atomics are slow, and most rows of a dense mesh have one pixel.
template <int CC, bool POS>
struct BwdPixel {
    static constexpr uint32_t G4 = BwdChannels<CC, POS>::G;
    static constexpr bool kKeep = CC >= 1 && CC <= 4;   // attribute gradients kept in registers until `add`
    uint32_t slot[3];
    bool first[3], pos;
    double b[3];
    float gatt[kKeep ? 3 : 1][G4], gpos[3][3];

    __device__ __forceinline__ void store(const BwdTerms& t, const float* const (&rows)[3], const float* grad,
                                          uint32_t C, BwdChannels<CC, POS> ch, float* val)
    {
        const uint32_t n = CC ? (uint32_t)CC : C, S = n + 3;
        double G[3] = {0.0, 0.0, 0.0};
#pragma unroll
        for (uint32_t c0 = 0; c0 < n; c0 += G4) {
            if (c0) ch.load(rows, grad, c0, n);
#pragma unroll
            for (uint32_t c = 0; c < G4; ++c)
                if (CC || c0 + c < n)
#pragma unroll
                    for (int k = 0; k < 3; ++k) {
                        G[k] += (double)ch.g[c] * (double)ch.at[k][c];
                        const float v = (float)((double)ch.g[c] * t.b[k]);
                        if constexpr (kKeep) gatt[k][c] = v;
                        if (first[k]) val[slot[k] * S + c0 + c] = v;
                    }
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) b[k] = t.b[k];
        if constexpr (POS) {
#pragma unroll
            for (int k = 0; k < 3; ++k)
#pragma unroll
                for (int j = 0; j < 3; ++j) gpos[k][j] = 0.0f;
            if (pos) bwd_pos(t, G, gpos);
#pragma unroll
            for (int k = 0; k < 3; ++k)
                if (first[k])
#pragma unroll
                    for (int j = 0; j < 3; ++j) val[slot[k] * S + n + j] = gpos[k][j];
        }
    }

    __device__ __forceinline__ void add(const float* grad, uint32_t C, float* val) const
    {
        const uint32_t n = CC ? (uint32_t)CC : C, S = n + 3;
#pragma unroll
        for (int k = 0; k < 3; ++k)
            if (!first[k]) {
                float* row = val + slot[k] * S;
                if constexpr (kKeep) {
#pragma unroll
                    for (uint32_t c = 0; c < n; ++c) unsafeAtomicAdd(row + c, gatt[k][c]);
                } else {
                    for (uint32_t c = 0; c < n; ++c) unsafeAtomicAdd(row + c, (float)((double)gl(grad)[c] * b[k]));
                }
                if (POS && pos)
#pragma unroll
                    for (int j = 0; j < 3; ++j) unsafeAtomicAdd(row + n + j, gpos[k][j]);
            }
    }
};

extern __shared__ __align__(16) unsigned char s_bwd[];   // keys, then kBwdSlots rows of C + 3 floats

template <int CC, bool POS>
__global__ void __launch_bounds__(256) resolve_backward_kernel(ScreenArgs a)
{
    uint32_t* keys = reinterpret_cast<uint32_t*>(s_bwd);
    float* val = reinterpret_cast<float*>(keys + kBwdSlots);
    const uint32_t C = CC ? (uint32_t)CC : a.C, S = C + 3;
    uint32_t x, y, vi[3];
    const bool in = tile_pixel((uint32_t)a.W, (uint32_t)a.H, x, y);
    const uint32_t p = in ? y * (uint32_t)a.W + x : 0;
    const bool have = in && screen_tri(a, p, vi);
    if (!__syncthreads_or(have)) return;
    for (uint32_t i = threadIdx.x; i < kBwdSlots; i += 256) keys[i] = ~0u;
    __syncthreads();
    BwdPixel<CC, POS> px;
    const float* grad = a.grad_out + (size_t)p * C;
    if (have) {
        float sx[3], sy[3], w[3];
        screen_windows(a, vi, sx, sy, w);
        const float* rows[3] = {a.attrs + (size_t)vi[0] * C, a.attrs + (size_t)vi[1] * C, a.attrs + (size_t)vi[2] * C};
        BwdChannels<CC, POS> ch;
        ch.load(rows, grad, 0, C);
        px.pos = true;
        bwd_slots(keys, vi, vi, px.slot, px.first);
        BwdTerms t;
        bwd_terms(sx, sy, w, x, y, t);
        px.store(t, rows, grad, C, ch, val);
    }
    __syncthreads();
    if (have) px.add(grad, C, val);
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < kBwdSlots * C; i += 256) {
        const uint32_t s = i / C, c = i - s * C, v = keys[s];
        if (v != ~0u) unsafeAtomicAdd(a.grad_attr + (size_t)v * C + c, val[s * S + c]);
    }
    if (POS)
        for (uint32_t i = threadIdx.x; i < kBwdSlots * 3; i += 256) {
            const uint32_t s = i / 3, c = i - s * 3, v = keys[s];
            if (v != ~0u) unsafeAtomicAdd(a.grad_pos + 3 * (size_t)v + c, val[s * S + C + c]);
        }
}

// Backward of the multi-mesh resolve (resolve_kernel) with visibility held fixed: one lane per
// pixel finds the (mesh, instance) and triangle as the forward does, projects its three vertices
// with the same fp32 operations, and applies the chain rule above; attribute gradients of every
// instance of a mesh add into the mesh's rows, position gradients (to the unsnapped window
// positions of one-instance meshes) where the mesh has a gradient buffer.  Table keys are
// (mesh, vertex).
template <int CC, bool POS>
__global__ void __launch_bounds__(256) resolve_backward_meshes_kernel(ResolveBlock<kResolveWordsOne> blk)
{
    unsigned long long* keys = reinterpret_cast<unsigned long long*>(s_bwd);
    float* val = reinterpret_cast<float*>(keys + kBwdSlots);
    const ResolveArgs& a = blk.a;
    const ResolveDesc d = {a.bases, a.mesh_pair, a.pairs, a.meshes, a.attrs, nullptr};
    const uint32_t C = CC ? (uint32_t)CC : a.C, S = C + 3;
    uint32_t x, y, pair = 0, vi[3];
    const bool in = tile_pixel((uint32_t)a.W, (uint32_t)a.H, x, y);
    const uint32_t p = in ? y * (uint32_t)a.W + x : 0;
    const bool have = in && pixel_triangle<kDescDevice>(a, d, p, pair, vi);
    if (!__syncthreads_or(have)) return;
    for (uint32_t i = threadIdx.x; i < kBwdSlots; i += 256) keys[i] = ~0ull;
    __syncthreads();
    BwdPixel<CC, POS> px;
    const float* grad = a.grad_out + (size_t)p * C;
    if (have) {
        const DrawDesc& D = d.pairs[pair];
        const uint32_t m = D.mesh;
        float sx[3], sy[3], w[3];
        pixel_windows(a, D, d.meshes[m], vi, sx, sy, w);
        const float* at = d.attrs[m];
        const float* rows[3] = {at + (size_t)vi[0] * C, at + (size_t)vi[1] * C, at + (size_t)vi[2] * C};
        BwdChannels<CC, POS> ch;
        ch.load(rows, grad, 0, C);
        px.pos = POS && a.grad_pos[m] != nullptr;
        unsigned long long key[3];
        uint32_t hash[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            key[k] = (unsigned long long)m << 32 | vi[k];
            hash[k] = vi[k] + m * 0x9E3779B9u;
        }
        bwd_slots(keys, key, hash, px.slot, px.first);
        BwdTerms t;
        bwd_terms(sx, sy, w, x, y, t);
        px.store(t, rows, grad, C, ch, val);
    }
    __syncthreads();
    if (have) px.add(grad, C, val);
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < kBwdSlots * C; i += 256) {
        const uint32_t s = i / C, c = i - s * C;
        const unsigned long long key = keys[s];
        if (key == ~0ull) continue;
        float* ga = a.grad_attrs[key >> 32];
        if (ga) unsafeAtomicAdd(ga + (size_t)(uint32_t)key * C + c, val[s * S + c]);
    }
    if (POS)
        for (uint32_t i = threadIdx.x; i < kBwdSlots * 3; i += 256) {
            const uint32_t s = i / 3, c = i - s * 3;
            const unsigned long long key = keys[s];
            if (key == ~0ull) continue;
            float* gp = a.grad_pos[key >> 32];
            if (gp) unsafeAtomicAdd(gp + 3 * (size_t)(uint32_t)key + c, val[s * S + C + c]);
        }
}

// ----------------------------------------------------------------------------------------------
// Launch wrappers
// ----------------------------------------------------------------------------------------------
static uint32_t blocks_for(uint64_t n) { return (uint32_t)((n + 255) / 256); }

// 16 x 16 pixel tiles of a view (at most 16384 x 16384 pixels).
static uint32_t tiles_for(int32_t W, int32_t H) { return (((uint32_t)W + 15u) / 16u) * (((uint32_t)H + 15u) / 16u); }

hipError_t launch_project(const MeshDesc& mesh, const float A[12], float hW, float hH, float* out, hipStream_t s)
{
    ProjectArgs a;
    a.mesh = mesh;
    for (int i = 0; i < 12; ++i) a.A[i] = A[i];
    a.hW = hW;
    a.hH = hH;
    a.out = out;
    if (mesh.V == 0) return hipSuccess;
    project_kernel<<<blocks_for(mesh.V), 256, 0, s>>>(a);
    return hipGetLastError();
}

template <int MODE, int WORDS>
static hipError_t resolve_any(const ResolveBlock<WORDS>& b, hipStream_t s)
{
    const ResolveArgs& a = b.a;
    if (a.textured) {
        resolve_textured_kernel<MODE, WORDS><<<tiles_for(a.W, a.H), 256, 0, s>>>(b);
    } else {
        if (a.ss > 1)
            with_channels(a.C, [&](auto cc) {
                resolve_ss_kernel<decltype(cc)::value, MODE, WORDS><<<tiles_for(a.W, a.H), 256, 0, s>>>(b);
            });
        else
            with_channels<true>(a.C, [&](auto cc) {
                resolve_kernel<decltype(cc)::value, MODE, WORDS><<<tiles_for(a.W, a.H), 256, 0, s>>>(b);
            });
    }
    return hipGetLastError();
}

// Descriptors in device memory (`words` 0) or as part of the argument.
hipError_t launch_resolve(const ResolveBlock<kResolveWords>& b, hipStream_t s)
{
    if (b.words && !(b.a.n_meshes == 1 && b.a.n_pairs == 1)) return resolve_any<kDescInline>(b, s);
    ResolveBlock<kResolveWordsOne> o;
    if (b.words > (uint32_t)kResolveWordsOne) return hipErrorInvalidValue;
    for (uint32_t i = 0; i < b.words; ++i) o.w[i] = b.w[i];
    o.words = b.words;
    o.off_mpair = b.off_mpair;
    o.off_pairs = b.off_pairs;
    o.off_meshes = b.off_meshes;
    o.off_attrs = b.off_attrs;
    o.off_tex = b.off_tex;
    o.a = b.a;
    return b.words ? resolve_any<kDescOne>(o, s) : resolve_any<kDescDevice>(o, s);
}

// Levels 1 .. levels - 1 from level 0, one launch per level (each reads the previous one).
hipError_t launch_build_mips(uint32_t* texels, uint32_t w, uint32_t h, uint32_t levels, hipStream_t s)
{
    uint64_t off = 0;
    for (uint32_t l = 0; l + 1 < levels; ++l) {
        const uint32_t pw = max(1u, w >> l), ph = max(1u, h >> l), cw = max(1u, w >> (l + 1)), ch = max(1u, h >> (l + 1));
        uint32_t* src = texels + off;
        off += (uint64_t)pw * ph;
        mip_kernel<<<blocks_for((uint64_t)cw * ch), 256, 0, s>>>(src, pw, ph, texels + off, cw, ch);
    }
    return hipGetLastError();
}

hipError_t launch_resolve_screen(const ScreenArgs& a, hipStream_t s)
{
    with_channels<true>(a.C, [&](auto cc) {
        resolve_screen_kernel<decltype(cc)::value><<<tiles_for(a.W, a.H), 256, 0, s>>>(a);
    });
    return hipGetLastError();
}

// LDS of a backward workgroup: at most 4 or 8 bytes of key and 19 floats for each of 1024 rows, 84 KB.
static size_t bwd_lds(uint32_t C, size_t key) { return kBwdSlots * (key + sizeof(float) * (C + 3)); }

hipError_t launch_resolve_backward(const ScreenArgs& a, hipStream_t s)
{
    with_channels(a.C, [&](auto cc) {
        constexpr int CC = decltype(cc)::value;
        const size_t lds = bwd_lds(a.C, sizeof(uint32_t));
        if (a.grad_pos) resolve_backward_kernel<CC, true><<<tiles_for(a.W, a.H), 256, lds, s>>>(a);
        else resolve_backward_kernel<CC, false><<<tiles_for(a.W, a.H), 256, lds, s>>>(a);
    });
    return hipGetLastError();
}

hipError_t launch_resolve_backward_meshes(const ResolveBlock<kResolveWordsOne>& b, hipStream_t s)
{
    with_channels(b.a.C, [&](auto cc) {
        constexpr int CC = decltype(cc)::value;
        const size_t lds = bwd_lds(b.a.C, sizeof(unsigned long long));
        const uint32_t tiles = tiles_for(b.a.W, b.a.H);
        if (b.a.grad_pos) resolve_backward_meshes_kernel<CC, true><<<tiles, 256, lds, s>>>(b);
        else resolve_backward_meshes_kernel<CC, false><<<tiles, 256, lds, s>>>(b);
    });
    return hipGetLastError();
}

}  // namespace curast
