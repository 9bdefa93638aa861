// Descriptors shared by the host runtime and the gfx950 kernels of the rasterizer.
//
// Memory layout in HBM (all written by the host runtime each frame, read-only in kernels):
//   FrameHeader | ViewDesc[n_views] | MeshDesc[M] | Segment[n_segs] | DrawDesc[n_draws]
// plus context-owned scratch: the stage queues (Q2, large-triangle records, Q3) and counters.
// Per-vertex and per-index data stay in the caller's buffers ([V][3] float, [T][3] uint32) and are
// streamed once per frame by stage 1 (the paper's bandwidth-bound hot loop, Sec. 4.5).
#pragma once

#include <stdint.h>

namespace curast {

constexpr float kGuardBand = 16.0f;               // |x|, |y| <= 16 w needs no clipping
constexpr uint64_t kIdMask = (uint64_t(1) << 36) - 1;
constexpr uint64_t kEmptyKey = ~uint64_t(0);
constexpr int kTileSize = 64;                     // stage-3 screen tile (Sec. 4.2)
constexpr int kMaxDim = 16384;
constexpr uint32_t kNullRecord = 0xFFFFFFFFu;
constexpr uint32_t kNoPart = 0xFFFFFFFFu;         // end of a tile's list of stage-3 parts
// Stage 1 keeps triangles whose snapped bounding box spans less than this many 1/256-px units in
// x and y: every edge-function value at a pixel centre of the box (and one step past it) then
// fits in int32 (|E| <= 2 * ext * (ext + 384) < 2^31).
constexpr int32_t kSmallExtent = 32768 - 512;
// Twice the area, in 1/256 px squared, from which a triangle samples a stored depth (see raster_small): 1.5 px.
// It reads before its atomics where at least kSampleLanes lanes of the wavefront are to: each read costs the whole
// wavefront a round trip, and saves one atomic per lane.
constexpr int32_t kSampleArea = 3 << 16, kNeverSample = 0x7FFFFFFF, kSampleLanes = 24;

struct FrameHeader {              // 48 B
    uint64_t total_batches;       // stage-1 work items over all segments
    uint32_t n_segs;
    uint32_t n_views;
    uint32_t draws_per_item;      // draws per work item
    uint32_t n_tiles;             // 64x64 screen tiles over all views (stage-3 bins)
    uint64_t shared_batches;      // work items [0, shared_batches) belong to meshes drawn more than once
    uint64_t pad[2];
};

struct ViewDesc {                 // 48 B
    unsigned long long* vis;      // [H][W]
    int32_t W, H;
    float hW, hH;                 // W/2, H/2 (exact)
    float near_plane;
    uint32_t tile_base;           // first stage-3 tile of this view; its tiles are row-major
    float wmax, hmax;             // W - 1, H - 1 (exact)
    float reach;                  // DrawDesc::reach of the view's general draws (on the device: of the current draw)
    uint32_t pad;
};

struct MeshDesc {                 // 80 B
    const float* pos;             // [V][3], or NULL when compressed
    const uint32_t* idx;          // [T][3], or the packed index stream when compressed
    const uint16_t* qpos;         // [3 V + 1] quantized positions (+1 padding) when compressed, else NULL
    uint64_t T;
    uint32_t V;
    uint32_t idx_bits;            // 0: plain indices; else bits per packed index
    uint32_t idx_min;             // added to every packed index
    float lo[3], step[3];         // position = fmaf(q, step, lo) when compressed
    uint32_t pad;
};

// A run of stage-1 work items over one mesh: work item j of the segment covers the triangle batch
// j / n_groups and the draw group j % n_groups (consecutive items share triangles, so the
// index/vertex lines they read are still in L2 when the next draw group needs them).
struct Segment {                  // 32 B
    uint64_t batch_begin;         // first global work item of the segment
    uint32_t mesh;
    uint32_t draw_begin;          // first draw of the mesh
    uint32_t draw_count;          // draws of the mesh that survived the host cull
    uint32_t n_groups;            // ceil(draw_count / draws_per_item)
    uint32_t batch_tris;          // triangles per work item of this segment
    uint32_t pad;
};

// One (mesh, instance, view): rows x, y, w of VP * X, the global ID of triangle 0, the view.
// Bit 31 of `view` (kDrawInterior) marks draws whose bounding sphere the host proved to lie in
// front of the near plane and inside |x|, |y| <= 1.99 w: no vertex of such a draw needs the
// per-vertex near/guard tests of the fast stage-1 path.
struct DrawDesc {                 // 128 B, aligned to them: one cache line holds all that a fragment of the draw needs
    float A[12];                  // rows x, y, w of VP * X (the exact transform)
    float R[8];                   // interior draws: hW (row x + row w), hH (row y + row w)
    uint64_t id_base;
    uint32_t view;                // view index | kDrawInterior
    uint32_t mesh;
    float scale;                  // interior draws: pixels per unit of length at most; 0: bound too loose;
                                  // < 0: triangles too large for strip spheres
    float grow;                   // interior draws: pixels added to a strip sphere's projected radius
    float wmax, hmax;             // W - 1, H - 1 of the view (exact)
    unsigned long long* vis;      // visibility buffer of the view
    float near_plane;             // of the view
    float reach;                  // 1/2 px + the fast positions' error bound (see the stage-1 kernels)
};
static_assert(sizeof(DrawDesc) == 128, "one cache line");
constexpr uint32_t kDrawInterior = 0x80000000u;
constexpr uint32_t kDrawViewMask = 0x7FFFFFFFu;

struct Q2Entry {                  // triangle forwarded by stage 1
    uint32_t draw;
    uint32_t tri;
};

struct LargeTri {                 // snapped (sub-)triangle forwarded by stage 2, 48 B
    int32_t X[3], Y[3];
    float zI[3];
    uint32_t view;
    uint64_t id;
};

struct Q3Entry {                  // one 64x64 tile part of a large triangle
    uint32_t rec;                 // LargeTri index or kNullRecord
    uint16_t tx, ty;
};

enum Counter : int {
    kCntQ2 = 0,                   // entries appended to Q2 (may exceed its capacity)
    kCntLarge = 1,                // large records reserved
    kCntQ3 = 2,                   // Q3 entries reserved
    kCntTiles = 3,                // screen tiles with parts
    kNumCounters = 4
};

enum Stat : int {
    kStTriDraws = 0, kStDrawsCulled, kStCulledNear, kStCulledFrustum, kStCulledTiny,
    kStCulledBack, kStS1Raster, kStQ2, kStQ2Overflow, kStS2Raster, kStQ3, kStQ3Overflow,
    kStFragments, kStAtomics, kStStripDraws, kStStripPass, kStSpherePass, kNumStats
};

// Option flags mirrored from the public header.
constexpr uint32_t kFlagNoTinyCull = 0x1u;
constexpr uint32_t kFlagNoEarlyOut = 0x2u;
constexpr uint32_t kFlagNoMeshCull = 0x4u;
constexpr uint32_t kFlagStats = 0x8u;
constexpr uint32_t kFlagNoGraph = 0x10u;
constexpr uint32_t kFlagS3PerPart = 0x40u;          // stage 3 per tile part instead of per binned tile
constexpr uint32_t kFlagNoFastInterior = 0x80u;     // no prescaled interior draws in stage 1
constexpr uint32_t kFlagNoStrips = 0x100u;          // no triangle strips in stage 1
constexpr uint32_t kFlagSingleStrips = 0x200u;      // strips in the single-draw stage-1 launch too
constexpr uint32_t kFlagS1Overlap = 0x400u;         // the two stage-1 launches on two streams at once
constexpr uint32_t kFlagEarlyOutAll = 0x800u;       // read the stored key before the atomic in every stage
constexpr uint32_t kFlagZeroQueues = 0x80000000u;   // testing aid: queue capacities of zero

struct RasterArgs {
    const FrameHeader* hdr;
    const ViewDesc* views;
    const MeshDesc* meshes;
    const Segment* segs;
    const DrawDesc* draws;
    Q2Entry* q2;
    LargeTri* large;
    Q3Entry* q3;
    unsigned long long* counters;
    unsigned long long* stats;
    uint32_t q2_cap, large_cap, q3_cap;
    uint32_t small_px, medium_px;
    uint32_t s2_blocks;           // workgroups that walk the stage-2 queue
    uint32_t flags;
    uint32_t s1_mode;             // 0 auto (= 2), 1 exact only, 2 fast reject (strip spheres in the
                                  // multi-draw launch), 3 vertex sharing for every mesh, 4 as 2 without spheres
    int32_t sample_area;          // stage 1: a triangle's twice-area, in 1/256 px squared, from which its lane samples
                                  // the stored depth to decide whether to read before its atomics
    uint32_t part;                // stage-1 work items: 0 all, 1 the shared prefix, 2 the rest
    uint32_t* tile_head;          // [n_tiles] last part linked to each tile (kNoPart: none; clear kernel)
    uint32_t* tile_list;          // [n_tiles] the tiles that have parts, kCntTiles of them
    uint32_t* q3_next;            // [q3_cap] the next part of the same tile, or kNoPart
    uint32_t compressed_parts;    // bit p: stage-1 part p has a compressed mesh; bit p + 8: every
                                  // mesh of part p is compressed (host-side kernel choice)
};

// A frame's descriptor block as a kernel argument (at most 4 KB in all), with what the clear needs.  Of a
// block that is too large, the argument holds the first WORDS and `tail` the rest in pinned host memory.
constexpr int kBlockWordsSmall = 240, kBlockWords = 960;
template <int WORDS>
struct FrameBlock {
    uint32_t* dst;                // device copy of w[0 .. words)
    unsigned long long* counters;
    uint32_t* tile_head;
    uint32_t words, views_word;   // words of the block in use; the first word of its views
    uint32_t n_views, n_tiles;
    const uint32_t* tail;         // pinned host memory: words WORDS, WORDS + 1, ... of the block
    uint32_t tail_words;
    uint32_t pad[3];
    alignas(16) uint32_t w[WORDS];
};
static_assert(sizeof(FrameBlock<kBlockWords>) <= 4096 - 128, "fits a kernel argument");

// Compression's index range and bounding box: workgroups per reduction (a multiple of 3) and words of
// their partial results.
constexpr uint32_t kRangeBlocks = 1536, kRangeWords = 2 * 6 * kRangeBlocks;

// A mip-mapped RGBA8 texture: level l is max(1, w >> l) x max(1, h >> l) texels from off[l].
struct TexDesc {
    const uint32_t* texels;
    uint32_t w, h, levels, pad;
    uint32_t off[16];
};

struct ResolveArgs {
    const unsigned long long* vis;
    int32_t W, H;
    float hW, hH;
    const uint64_t* bases;        // [n_meshes + 1] first global ID of each mesh (its instances follow
                                  // one another, T IDs apart); the last entry is the ID count
    const uint32_t* mesh_pair;    // [n_meshes] index of each mesh's first (mesh, instance) pair
    const DrawDesc* pairs;        // [n_pairs] draw matrix of every (mesh, instance) for this view
    const MeshDesc* meshes;
    const float* const* attrs;    // [M] per-mesh attribute pointers
    uint32_t n_pairs;
    uint32_t n_meshes;
    uint32_t C;
    float* out;                   // [H][W][C], or [H/ss][W/ss][C] when supersampled
    uint32_t ss;                  // samples per axis and output pixel (1: no supersampling)
    uint32_t textured;            // the textured resolve, with:
    const TexDesc* tex;           // [M] textures of the textured resolve (attrs are then the UVs)
    const float* grad_out;        // backward input [H][W][C]
    float* const* grad_attrs;     // [M] per-mesh attribute gradients [V][C] (accumulated), entries may be null
    float* const* grad_pos;       // [M] per-mesh window-position gradients [V][3], or null (one-instance meshes)
};

// A resolve's descriptor block (bases | mesh_pair | pairs | meshes | attrs | textures) as part of the
// kernel argument, or its device pointers in `a` (words 0).
constexpr int kResolveWords = 880, kResolveWordsOne = 96;   // the latter holds one mesh's block
template <int WORDS>
struct ResolveBlock {
    alignas(16) uint32_t w[WORDS];
    uint32_t words, off_mpair, off_pairs, off_meshes, off_attrs, off_tex;   // byte offsets into w
    ResolveArgs a;
};
static_assert(sizeof(ResolveBlock<kResolveWords>) <= 4096 - 128, "fits a kernel argument");

struct ScreenArgs {
    const unsigned long long* vis;
    int32_t W, H;
    const uint32_t* idx;
    uint64_t T;
    uint64_t id_base;
    const float* pos_ss;          // [V][3]
    uint32_t V;
    const float* attrs;           // [V][C]
    uint32_t C;
    float* out;                   // forward output [H][W][C]
    const float* grad_out;        // backward input [H][W][C]
    float* grad_attr;             // [V][C]
    float* grad_pos;              // [V][3] or null
};

}  // namespace curast
