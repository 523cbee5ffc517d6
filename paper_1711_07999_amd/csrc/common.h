// Internal declarations shared by the HIP translation units of libtrack.
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <cstdint>
#include <algorithm>
#include <type_traits>

namespace trk {

constexpr int kMaxJoints = 127;
constexpr int kMaxLinks = 255;
constexpr int kPPMax = 128;          // padded Gram size (P + 1 rounded up to 16)
constexpr float kZNear = 1e-3f;      // vertices at z <= kZNear are not candidates
constexpr double kFix = 4294967296.0;  // 2^32: fixed-point quantum of the offsets (m)
constexpr int kNeRows = 128;         // vertices per normal-equation chunk
constexpr int kNeGrid = 512;         // normal-equation workgroups at most
constexpr int kNeCols = kPPMax;      // entries of a workgroup's column list
constexpr int kRedGroups = 16;       // groups of partial Gram matrices summed apart
constexpr int kRedPer = 32;          // a group's entries in the rank table

// Joint and link tables (device copy, built once per model on the host).
struct JointTable {
    int P, L;
    int parent[kMaxJoints + 1];
    int type[kMaxJoints + 1];
    double axis[kMaxJoints + 1][3];
    double off[kMaxJoints + 1][8];     // fixed offset O_j as a dual quaternion
    int link_joint[kMaxLinks + 1];
    double binv[kMaxLinks + 1][8];     // (H^0_{0,link joint})^{-1}
    uint32_t anc[kMaxLinks + 1][4];    // joints on the chain of each link
    double prior[kMaxJoints + 1];      // (lambda_s S_k)^2
    int active[kMaxJoints + 1];
    int rounds;                        // ceil(log2(longest joint chain))
};

// Tree-ordered factorisation of the pose system (built on the host from the
// skeleton and the skin weights, read by the pose-solve kernel).  Joints are
// eliminated children first; chains of the elimination tree form supernodes,
// each with a dense front: its pivot rows, the later rows they touch, and the
// right-hand side as a last row, stored row-major with `fw` columns.
constexpr int kFrontRows = 32;       // rows of a front, right-hand side included
constexpr int kSolveWaves = 8;       // waves of the tree-form pose-solve workgroup
constexpr int kSolveThreads = 64 * kSolveWaves;
constexpr int kFrontWords = 8;       // words of a front record in the blob

// A front record: storage offset, pivots, rows (without the right-hand
// side), row width, byte offset of its row-to-joint map in the blob.
struct FrontRec { int off, np, f, fw, row0, pad[3]; };
// The assembly of a level's fronts: its first entry's word in the blob,
// parent entries, those of more than one word, words of the longest.
struct AsmRec { int map0, n, n1, words; };

// What the kernels read of a stream's tree plan (in its slot, so that no
// read waits on another).
struct TreeRef {
    const uint32_t* blob;            // TreePlan::blob
    double* fimg;                    // [elems] the fronts as the solve starts them, written by the
                                     // Gram reduction (damped, frozen); zero outside the entries
    const int* gfmap;                // [PP*PP] Gram position (at or above the diagonal, or the
                                     // right-hand side) -> front storage index, -1 none; null: dense form
    int nwords, nlev, elems, o_lev, o_front;
};

struct alignas(16) TreePlan {
    int ok;                          // the tree form applies to this model
    int nsn, nlev, elems;            // supernodes, levels, front storage (elements)
    int nwords;                      // words of `blob`
    int o_lev, o_front;              // word offsets of the assembly and the front records
    // what the kernel copies to LDS: per level and wave the first front
    // (wstart, kSolveWaves * nlev + 1 words), the levels' assembly records,
    // the front records in that order, the assembly entries, then the row
    // maps (bytes).  A parent entry's words: its storage index | a child's
    // storage index << 16, then two more children's a word, in child order,
    // 0xFFFF = none.  A level's entries are sorted, those of most words first,
    // and stored word by word (all first words, then the second words of the
    // entries that have one, ...), so none is padded to the longest; before
    // them, the number of entries with a third word, a fourth, ...
    const uint32_t* blob;
};

constexpr int kFanInline = 8;   // incident faces of a vertex held in the inline (per-slot) table

// The columns of [J | r] that the normal equations' workgroups touch.
struct NeRef {
    const uint8_t* cols;     // [negrid][kNeCols] a workgroup's columns, increasing, the residual (column P)
                             // last, then 0xFF
    const uint32_t* mask;    // [chunks][4] joints on the chains of the chunk's links
    const uint8_t* rank;     // [PP][kRedGroups][kRedPer] column's place in the list of the group's workgroups, or 0xFF
    int width;               // longest list, rounded up to 16
};

// Mesh, weights and tables in structure-of-arrays device form.
constexpr int kBlendLinear = 1;   // TRACK_BLEND_LINEAR

struct DevModel {
    int P, L, V, F;
    const float *rx, *ry, *rz;     // template vertices
    const float4 *w;               // weights, padded to four
    const uint32_t *links;         // four link bytes per vertex, 0xFF = unused
    const int4 *nbr;               // neighbours, -1 = none
    // the faces around each vertex i: (b, c) with face (i, b, c) counter-clockwise
    const int2 *fan8;              // [kFanInline][V] the first kFanInline, padded with (i, i)
    const uint32_t *rest_off;      // [V+1] the others: vertex i's in rest[rest_off[i]..rest_off[i + 1])
    const int2 *rest;
    // the same by blocks of 64 vertices: the vertices outside a block that its
    // faces reach (its rim), and the fans in places of a block and its rim
    // (b below 64: the block's vertex b, else entry b - 64 of the rim)
    const uint32_t *rim_off;       // [blocks+1]
    const uint32_t *rim;
    const uint4 *fan_at;           // [V] kFanInline pairs of bytes, padded with (i, i)
    const uint16_t *rest_at;       // like `rest`, b | c << 8
};
constexpr int kRim = 192;          // vertices of a rim at most (places are bytes)

struct DevCam {
    int W, H, tiles_x, tiles_y;
    float fx, fy, cx, cy;
    float lb_c1;   // lower bound of the 3-D distance per pixel ring, per metre of depth
};

// DevStats::status set by a kernel: -4 the pose system is not positive
// definite; kStatusBucketOverflow a count found the overflow list full
// (counters not cleared: an internal error).
constexpr int kStatusBucketOverflow = -16;

// Per-iteration bookkeeping written by the kernels and read back per frame.
struct DevStats {
    int n_valid_px, n_assoc_px, n_obs_verts, status;
    float energy[256];
    float step_norm[256];
};

// Offset and normal buffers: SoA x, y, z of V floats each (skinned vertices
// are float4 (x, y, z, 0) so that neighbour gathers are single loads).
struct Vec3Buf { float *x, *y, *z; };

// Fixed-point per-vertex accumulators of the association.
struct Accum {
    uint32_t* cnt;           // pixels per vertex
    long long *sx, *sy, *sz; // sum of (p - v) in units of 2^-32 m
};

// Bucket (index/z-buffer) storage.  Pixels are numbered tile-major (8x8
// tiles in row-major order, 64 pixels per tile in Morton order), so a 4x4
// quadrant of a tile ("cell") is 16 consecutive pixels and pixel k lies in
// cell k >> 4.  Every counted vertex goes straight into its cell's region of
// `cellv`; the regions were laid out by the previous association from the
// counts it read (with room for the surface to move, see layout_tiles), and
// a vertex that finds its cell's region full goes to the overflow list after
// the regions.  The counters are double-buffered: the association reads one
// parity and writes the other's layout (counters cleared), which the next
// count fills.
struct Buckets {
    uint4* cells[2];   // [cells + 1] per parity: (zmin bits, zmax bits, vertices counted, first slot
                       // of the cell's region); entry `cells` holds the end of the last region in .w
    uint32_t* tsum[2]; // [tiles] per parity: vertices counted per tile
    uint32_t* ovfn;    // [2] vertices in the overflow list, per parity
    float4* cellv;     // [ncap + V] (x, y, vertex id bits, z): the cells' regions, then the overflow list
                       // (id before z: the search forms (id, d2) in the registers of (id, z))
    int ncap;          // slots of the regions (bucket_capacity bounds every layout)
    int4* bstat;       // [tiles] valid, matched, newly observed pixels per tile
    const int* torder; // [ntorder] the tile (column | row << 16) each association workgroup takes, -1 none (see
                       // tile_order in track.hip: entry k runs on XCD k % 8, each XCD's tiles
                       // nearest the image centre first)
    int ntorder;       // a multiple of 8
};

// Summary of one frame, written by the frame-end kernel.
struct DevSummary {
    int status, n_valid_px, n_assoc_px, n_obs_verts;
    float energy_first, energy_last, step_norm_last;
    int reason;   // 0 ok, 1 not positive definite, 2 no valid pixel, 3 nothing matched, 4/5 diverged,
                  // 6 bucket index overflow
};

// ---------------------------------------------------------------------------
// Slot table.  Every kernel works on a batch of tracking streams ("slots"):
// its grid is the concatenation of each slot's own grid, and a workgroup finds
// its slot by a binary search of the per-kind workgroup prefix.  A single
// tracker is a batch of one.  The table is rewritten by the host before each
// frame; kernels address the double-buffered vertices and the triple-buffered
// offsets relative to the frame-start indices held in the table, so one
// captured frame serves every starting state.
// ---------------------------------------------------------------------------
constexpr int kSlotBeginFrame = 1;    // the launch starts a frame of this slot
constexpr int kSlotEndFrame = 2;      // the launch ends a frame of this slot
constexpr int kSlotRefreshPose = 4;   // redo forward kinematics at frame start

struct alignas(16) Slot {
    DevModel m;
    DevCam c;
    const JointTable* jt;
    TreeRef tree;                 // tree form of the pose solve
    const uint32_t* anc;          // [L*4] joints on each link's chain
    NeRef ne;
    Buckets b;
    Accum a;
    float* dq;                    // [L*8] link offsets
    float* xi;                    // [P*8] world joint generators
    double *theta, *theta_backup, *step, *gram;
    float* partials;              // [negrid][width*width] (NeRef)
    float4* verts[2];
    Vec3Buf normals;
    Vec3Buf phi[3];
    const float* depth;           // frame input: depth image ...
    const float* xyz;             // ... or organised point cloud (the other is null)
    int32_t* assoc;
    DevStats* st;
    DevSummary* summary;
    int PP, negrid, flags;
    float tau, lambda_k, lphi, lnbr, lt, lw;
    int v_cur;                    // current vertex buffer when the launch starts
    int phi_cur, phi_prev;        // current and previous-frame offset buffers
    int iter;                     // iteration of the frame the launch starts at
    int blend;                    // 0 dual-quaternion blend, kBlendLinear: linear blend of the links' motions
    int bpar;                     // bucket counters filled by the next count when the launch starts
};

// Offset buffer written by the step after `src` (never the previous frame's
// buffer, so a failed frame can return to it).
__host__ __device__ __forceinline__ int phi_next(int src, int prev) {
    int n = 0;
    while (n == src || n == prev) ++n;
    return n;
}

// offset buffer current after `n` offset steps of the frame
__host__ __device__ __forceinline__ int phi_index(const Slot& S, int n) {
    int q = S.phi_cur;
    for (int k = 0; k < n; ++k) q = phi_next(q, S.phi_prev);
    return q;
}

enum KernelKind {
    KK_ONE = 0,     // one workgroup per slot (frame bookkeeping, FK, solve)
    KK_VERT,        // ceil(V / 256) workgroups
    KK_CLEAR,       // ceil(max(2 (cells + 1), V) / 256)
    KK_LAYOUT,      // ceil(tiles / kLayoutTiles): bucket layout
    KK_ASSOC,       // association: layout + normals + one search workgroup per entry of the tile order
    KK_NE,          // normal-equation workgroups
    KK_REDUCE,      // Gram reduction workgroups
    KK_VERT64,      // ceil(V / 64) workgroups
    KK_VERT512,     // ceil(V / 512) workgroups
    KK_COUNT_
};

template <int NT>
constexpr KernelKind kVertKind = NT == 512 ? KK_VERT512 : NT == 256 ? KK_VERT : KK_VERT64;

struct Batch {
    const Slot* slots;   // [n] device table
    const int* pre;      // [KK_COUNT_][n + 1] exclusive prefix of workgroups per slot
    int n;
};

// host-side launch description: the batch and its grid per kernel kind
struct Launch {
    Batch B;
    int grid[KK_COUNT_];
    int solve_n;        // largest padded pose-system size of the batch
    int solve_elems;    // largest tree-form front storage of the batch; 0: dense form
    int solve_words;    // largest tree-form plan blob of the batch
    int rims;           // every slot's blocks have their rims laid out
    int ne_cols, ne_pp, ne_l;   // widest column list, largest padded Gram size and link count of the batch
    hipStream_t s;
    const Slot* stage_src;   // the window in pinned memory (device view)
    const int* stage_pre;
    // a timed pass: its first kernel stamps t_start and its last kernel
    // t_stop with the kernels' own dispatch timestamps
    hipEvent_t t_start = nullptr, t_stop = nullptr;
};

// Launch `kernel` on L's stream; `first` / `last` mark the kernel's place in
// its pass, so a timed pass's events go to the dispatch packets themselves.
template <typename F, typename... Args>
inline void launch_kernel(const Launch& L, bool first, bool last, F kernel, dim3 grid, dim3 block, uint32_t lds,
                          Args... args) {
    hipEvent_t e0 = first ? L.t_start : nullptr, e1 = last ? L.t_stop : nullptr;
    if (e0 || e1) hipExtLaunchKernelGGL(kernel, grid, block, lds, L.s, e0, e1, 0u, args...);
    else hipLaunchKernelGGL(kernel, grid, block, lds, L.s, args...);
}

// n (>= 1) floats from global memory to LDS, every load of a thread issued
// before its first store (a one-wave workgroup copies the link table in one
// round of loads rather than one round per 64 entries)
__device__ __forceinline__ void copy_to_lds(float* dst, const float* __restrict__ src, int n) {
    for (int base = threadIdx.x; base < n; base += 8 * blockDim.x) {
        float t[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) t[j] = src[min(base + j * (int)blockDim.x, n - 1)];   // past n: not stored
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (base + j * (int)blockDim.x < n) dst[base + j * blockDim.x] = t[j];
    }
}

// Global memory read, written and updated as such.  Through a generic
// pointer the compiler emits flat instructions, which also count as LDS
// accesses: the next wait for LDS (a shuffle, an LDS read, a barrier) or for
// a scalar load then waits for every one of them still in flight.
template <class T>
__device__ __forceinline__ T ldg(const T* p) {
    return *(const __attribute__((address_space(1))) T*)p;
}
__device__ __forceinline__ float4 ldg(const float4* p) {
    typedef float v4f __attribute__((ext_vector_type(4)));
    const v4f t = *(const __attribute__((address_space(1))) v4f*)p;
    return make_float4(t.x, t.y, t.z, t.w);
}
__device__ __forceinline__ int4 ldg(const int4* p) {
    typedef int v4i __attribute__((ext_vector_type(4)));
    const v4i t = *(const __attribute__((address_space(1))) v4i*)p;
    return make_int4(t.x, t.y, t.z, t.w);
}
__device__ __forceinline__ int2 ldg(const int2* p) {
    typedef int v2i __attribute__((ext_vector_type(2)));
    const v2i t = *(const __attribute__((address_space(1))) v2i*)p;
    return make_int2(t.x, t.y);
}
__device__ __forceinline__ uint4 ldg(const uint4* p) {
    typedef unsigned v4u __attribute__((ext_vector_type(4)));
    const v4u t = *(const __attribute__((address_space(1))) v4u*)p;
    return make_uint4(t.x, t.y, t.z, t.w);
}
__device__ __forceinline__ uint2 ldg(const uint2* p) {
    typedef unsigned v2u __attribute__((ext_vector_type(2)));
    const v2u t = *(const __attribute__((address_space(1))) v2u*)p;
    return make_uint2(t.x, t.y);
}
// x, y, z of a float4 (w = 0): an unused fourth register of a load in
// flight would be taken for other values, which must then wait for the load
__device__ __forceinline__ float4 ldg_xyz(const float4* p) {
    typedef float v3f __attribute__((ext_vector_type(3)));
    const v3f t = *(const __attribute__((address_space(1))) v3f*)p;
    return make_float4(t.x, t.y, t.z, 0.0f);
}
template <class T>
__device__ __forceinline__ void stg(T* p, T v) {
    *(__attribute__((address_space(1))) T*)p = v;
}
__device__ __forceinline__ void stg(float4* p, float4 v) {
    typedef float v4f __attribute__((ext_vector_type(4)));
    v4f t;
    t.x = v.x; t.y = v.y; t.z = v.z; t.w = v.w;
    *(__attribute__((address_space(1))) v4f*)p = t;
}
// relaxed device-scope atomics
__device__ __forceinline__ uint32_t atomic_add_g(uint32_t* p, uint32_t v) {
    return __hip_atomic_fetch_add((__attribute__((address_space(1))) uint32_t*)p, v, __ATOMIC_RELAXED,
                                  __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long atomic_add_g(unsigned long long* p, unsigned long long v) {
    return __hip_atomic_fetch_add((__attribute__((address_space(1))) unsigned long long*)p, v, __ATOMIC_RELAXED,
                                  __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void atomic_min_g(uint32_t* p, uint32_t v) {
    __hip_atomic_fetch_min((__attribute__((address_space(1))) uint32_t*)p, v, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void atomic_max_g(uint32_t* p, uint32_t v) {
    __hip_atomic_fetch_max((__attribute__((address_space(1))) uint32_t*)p, v, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
}

// Keeps a loaded value where it stands: the compiler would otherwise move a
// load into the branch that alone uses it, to be waited for there on its
// own instead of together with the loads issued before it.  Emits nothing.
__device__ __forceinline__ void pin_load(int& x) { asm volatile("" : "+v"(x)); }
__device__ __forceinline__ void pin_load(uint32_t& x) { asm volatile("" : "+v"(x)); }
__device__ __forceinline__ void pin_load(int2& x) { pin_load(x.x); pin_load(x.y); }

// A value the whole wave holds alike (a field of its workgroup's slot), in
// scalar registers: where the compiler cannot tell that it is uniform (a
// value carried through a loop that also copies into LDS) it would keep a
// copy per lane in vector registers.
template <class T>
__device__ __forceinline__ T* wave_uniform(T* p) {
    const unsigned long long a = (unsigned long long)p;
    const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)a);
    const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(a >> 32));
    return (T*)(((unsigned long long)hi << 32) | lo);
}
__device__ __forceinline__ uint32_t wave_uniform(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
}
__device__ __forceinline__ int wave_uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ float wave_uniform(float v) {
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}

// slot of workgroup `blk` of kernel kind `kind`, and its index in that slot
__device__ __forceinline__ int slot_of(const Batch& B, int kind, int blk, int& local) {
    const int* p = B.pre + kind * (B.n + 1);
    int lo = 0, hi = B.n - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (p[mid] <= blk) lo = mid; else hi = mid - 1;
    }
    local = lo == 0 ? blk : blk - p[lo];  // every prefix starts at 0
    return lo;
}

// returns the launch's own status (an error that an earlier call of the
// thread's left is the caller's)
hipError_t launch_pack_state(hipStream_t s, const double* theta, int P, Vec3Buf phi, const float4* verts, int V,
                             double* out_theta, float* out_phi, float* out_verts);
int ne_grid(int V);

// Association launch: layout workgroups, normal workgroups, then (from a
// multiple of 8, so that workgroup k runs on XCD k % 8) the tiles' search
// workgroups, one per entry of the tile order (entry k on XCD k % 8)
constexpr int kAssocThreads = 256;
constexpr int kXcds = 8;             // workgroups are dealt to the chip's XCDs in turn
constexpr int kLayoutTiles = kAssocThreads;   // tiles per layout workgroup (one per thread)
__host__ __device__ inline int layout_blocks(int ntiles) { return (ntiles + kLayoutTiles - 1) / kLayoutTiles; }
__host__ __device__ inline int assoc_normal_blocks(int V) { return (V + kAssocThreads - 1) / kAssocThreads; }
// the layout and normal workgroups, rounded up to a multiple of kXcds
__host__ __device__ inline int assoc_extra_blocks(int ntiles, int V) {
    return (layout_blocks(ntiles) + assoc_normal_blocks(V) + kXcds - 1) / kXcds * kXcds;
}
// Slots of the cells' regions.  A layout gives tile t d + d/2 + 32 slots, d
// the largest count of the 3x3 tiles around it; the d sum to about 2 V on a
// body (9 V at most), so 4 V + 32 per tile leaves room to spare.  Regions
// past the end are cut to nothing (their vertices take the overflow list):
// a layout never writes outside the buffer, whatever the counts.
inline int bucket_capacity(int V, int ntiles) { return 4 * V + 32 * ntiles; }

// workgroups of each kind for one slot (host side)
inline int slot_blocks(const Slot& s, int kind) {
    const int V = s.m.V, ntiles = s.c.tiles_x * s.c.tiles_y;
    switch (kind) {
        case KK_ONE: return 1;
        case KK_VERT: return (V + 255) / 256;
        case KK_CLEAR: { const int n = 2 * (4 * ntiles + 1); return ((n > V ? n : V) + 255) / 256; }
        case KK_LAYOUT: return layout_blocks(ntiles);
        case KK_ASSOC: return assoc_extra_blocks(ntiles, V) + s.b.ntorder;
        case KK_NE: return s.negrid;
        case KK_VERT64: return (V + 63) / 64;
        case KK_VERT512: return (V + 511) / 512;
        case KK_REDUCE: { int nb = s.PP >> 4; return nb * (nb + 1) / 2 * 8; }
    }
    return 0;
}

// Threads of a workgroup of the per-vertex passes that count their surface
// (each workgroup counts in LDS before its atomics go out).  Larger
// workgroups send fewer atomics to a cell -- a mesh's next ring of vertices
// falls into the same cells as the last -- but fill fewer compute units: 512
// where that leaves each of the 256 a workgroup (offset step of 200,000
// vertices: 256 threads 20.5 us, 512 16.5, 1024 15.3; of 32 x 50,000: 99.4,
// 96.1, 127; of 50,000 alone: 9.0, 9.6, 12.6), 64 where 256 would leave three
// quarters of them without (10,000 vertices: 7.4 us, 64 threads 6.5; 2,000:
// 7.5, 6.9).  (One wave a workgroup, grouping its lanes one cell after
// another: 200,000 22.1, 32 x 50,000 106.7, 50,000 11.5, 2,000 8.8.)
inline int vert_threads(const Launch& L) {
    return L.grid[KK_VERT512] >= 256 ? 512 : L.grid[KK_VERT] >= 64 ? 256 : 64;
}
// The largest of them for an offset step that skins the new pose's surface
// itself: a wave's block and rim take 4 KB of LDS, and with 512 threads two
// workgroups fill a CU's instead of five.  The results are the same to the
// bit, and 512 threads gain nothing over 256 (a pass of 32 streams of 50 000
// vertices 15.30 ms against 15.34 on one box, two runs of either differ by as
// much): no instance is kept for them.
constexpr int kSkinThreads = 256;
// calls f with the size chosen, as an integral constant
template <class F>
inline void with_vert_threads(const Launch& L, F f) {
    switch (vert_threads(L)) {
        case 512: f(std::integral_constant<int, 512>()); break;
        case 256: f(std::integral_constant<int, 256>()); break;
        default: f(std::integral_constant<int, 64>()); break;
    }
}

// ---- launchers (each defined next to its kernels) -------------------------
// vsel: 0 = the slot's vertex buffer at the launch's start, 1 = the other;
// pn: number of offset steps taken so far (see phi_index).
// Which slots take the optional part of a kernel:
enum SlotSel { SEL_NONE = 0, SEL_ALL = 1, SEL_BEGIN = 2, SEL_NOT_END = 3 };
__device__ __forceinline__ bool selected(const Slot& S, int sel) {
    return sel == SEL_ALL || (sel == SEL_BEGIN && (S.flags & kSlotBeginFrame)) ||
           (sel == SEL_NOT_END && !(S.flags & kSlotEndFrame));
}
// copy a table window (slots and prefix rows) from host-visible pinned memory
void launch_stage(hipStream_t s, const Slot* src, Slot* dst, int n, const int* psrc, int* pdst, int npre);
void launch_frame_begin(const Launch& L);
void launch_frame_end(const Launch& L, int first_pose, int last_pose);  // iterations of the frame, -1 = none
void launch_fk(const Launch& L);
// bsel: 0 = the bucket counters of parity Slot::bpar, 1 = the other.
// skin into vsel for the slots selected by `which`; `count` of them also
// enter the buckets of bsel (count_only: the counts alone, for a layout);
// `clear_acc` slots have their accumulators zeroed
void launch_skin(const Launch& L, int vsel, int pn, int which, int count, int bsel, int count_only,
                 int clear_acc);  // count: a SlotSel
void launch_normals(const Launch& L, int vsel);
void launch_clear(const Launch& L);                 // both parities' bucket records (no layout), accumulators,
                                                    // front image
void launch_clear_acc(const Launch& L);             // accumulators only
void launch_clear_counts(const Launch& L, int bsel);  // bsel's counters, its layout kept
void launch_bucket_count(const Launch& L, int vsel, int which, int bsel);
void launch_layout(const Launch& L, int bsel);      // bsel's counts -> the other parity's layout
// association of the surface vsel counted into bsel; the same launch forms
// the surface's normals and lays out the other parity from bsel's counts
void launch_associate(const Launch& L, int vsel, int bsel);
void launch_normal_eq(const Launch& L, int gram_mode, int vsel, int pn);
void launch_gram_reduce(const Launch& L);
void launch_pose_solve(const Launch& L, int fp64, int iter);
bool tree_solve_fits(int elems, int words);   // the tree form's LDS fits the kernel in both precisions
bool prepare_pose_solve();   // once per process, before the first launch
bool prepare_normal_eq();    // likewise
// offset step from v_old / v_new (normals of v_new formed in place); the
// slots selected by `next` also skin the new offsets into v_new ^ 1 and count
// them into the buckets of bsel
// skin: the offset step skins the new pose's surface itself (L.rims)
void launch_shape(const Launch& L, int fp64, int v_old, int v_new, int pn, int next, int bsel, bool skin);

}  // namespace trk
