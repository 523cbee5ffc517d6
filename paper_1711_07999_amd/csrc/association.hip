// Projective data association (Section 4.1).
//
// Vertices are projected into pixel buckets (a point-rasterised index kept
// per 4x4-pixel cell, see Buckets) together with each cell's and tile's z
// range (the z-buffer).  Every valid pixel then finds the nearest vertex
// closer than tau: cells are visited in rings around the pixel's cell and
// skipped when a lower bound on the distance of anything inside them (from
// the pixel distance to the cell, or from its z range) cannot beat the best
// distance so far, so the result equals the exhaustive nearest-vertex search.
// The matched offsets are summed per vertex in 64-bit fixed point
// (deterministic).
//
// Float32 decisions follow one operation order, compiled without contraction:
//   point       x = ((u - cx) * d) / fx, y = ((v - cy) * d) / fy, z = d
//   bucket      floor((fx * x) / z + cx + 0.5), floor((fy * y) / z + cy + 0.5)
//   distance    (dx*dx + dy*dy) + dz*dz, accepted if < tau*tau,
//               ties to the lower vertex index.
#include "common.h"
#include "surface.h"

#pragma clang fp contract(off)

namespace trk {

__device__ __forceinline__ int wave_lane() { return threadIdx.x & 63; }

constexpr uint32_t kInfBits = 0x7F800000u;   // +inf: the z minimum of an empty cell or tile

// ---------------------------------------------------------------------------
// clear both parities' bucket records (counters and layout: every region
// empty, so the first count sends its vertices to the overflow list), the
// per-vertex accumulators and the solve's front image
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_clear(const Slot* __restrict__ bs, const int* __restrict__ bp, int bn) {
    const Batch B{bs, bp, bn};
    int local;
    const Slot& S = B.slots[slot_of(B, KK_CLEAR, blockIdx.x, local)];
    const Buckets& b = S.b;
    const Accum& a = S.a;
    const int V = S.m.V, ntiles = S.c.tiles_x * S.c.tiles_y, ncells = 4 * ntiles;
    const int i = local * blockDim.x + threadIdx.x;
    if (i <= ncells) {
        b.cells[0][i] = make_uint4(kInfBits, 0u, 0u, 0u);
        b.cells[1][i] = make_uint4(kInfBits, 0u, 0u, 0u);
    }
    if (i < ntiles) {
        b.tsum[0][i] = 0u;
        b.tsum[1][i] = 0u;
    }
    if (i < 2) b.ovfn[i] = 0u;
    if (i < V) {
        a.cnt[i] = 0u;
        a.sx[i] = 0; a.sy[i] = 0; a.sz[i] = 0;
    }
    // the tree solve's front image: zero outside the entries the Gram
    // reduction writes
    if (S.tree.gfmap) {
        const int n = 2 * (ncells + 1) > V ? 2 * (ncells + 1) : V;
        const int stride = (n + 255) / 256 * 256;
        for (int e = i; e < S.tree.elems; e += stride) S.tree.fimg[e] = 0.0;
    }
}

void launch_clear(const Launch& L) {
    launch_kernel(L, true, true, k_clear, dim3(L.grid[KK_CLEAR]), dim3(256), 0, L.B.slots, L.B.pre, L.B.n);
}

// the counters of one parity, its layout kept
__global__ void __launch_bounds__(256) k_clear_counts(const Slot* __restrict__ bs, const int* __restrict__ bp, int bn, int bsel) {
    const Batch B{bs, bp, bn};
    int local;
    const Slot& S = B.slots[slot_of(B, KK_CLEAR, blockIdx.x, local)];
    const Buckets& b = S.b;
    const int par = S.bpar ^ bsel;
    const int ntiles = S.c.tiles_x * S.c.tiles_y, ncells = 4 * ntiles;
    const int i = local * blockDim.x + threadIdx.x;
    if (i <= ncells) {
        uint4* c = &b.cells[par][i];
        c->x = kInfBits; c->y = 0u; c->z = 0u;
    }
    if (i < ntiles) b.tsum[par][i] = 0u;
    if (i == 0) b.ovfn[par] = 0u;
}

void launch_clear_counts(const Launch& L, int bsel) {
    launch_kernel(L, true, true, k_clear_counts, dim3(L.grid[KK_CLEAR]), dim3(256), 0, L.B.slots, L.B.pre, L.B.n, bsel);
}

__global__ void __launch_bounds__(256) k_clear_acc(const Slot* __restrict__ bs, const int* __restrict__ bp, int bn) {
    const Batch B{bs, bp, bn};
    int local;
    const Slot& S = B.slots[slot_of(B, KK_VERT, blockIdx.x, local)];
    const int i = local * blockDim.x + threadIdx.x;
    if (i >= S.m.V) return;
    S.a.cnt[i] = 0u;
    S.a.sx[i] = 0; S.a.sy[i] = 0; S.a.sz[i] = 0;
}

void launch_clear_acc(const Launch& L) {
    launch_kernel(L, true, true, k_clear_acc, dim3(L.grid[KK_VERT]), dim3(256), 0, L.B.slots, L.B.pre, L.B.n);
}

// count a given surface into the buckets (the producing kernels count their
// own output instead)
__global__ void __launch_bounds__(256) k_bucket_count(const Slot* __restrict__ bs, const int* __restrict__ bp, int bn, int vsel, int which, int bsel) {
    const Batch B{bs, bp, bn};
    __shared__ CountTable<256> ct;
    int local;
    const Slot& S = B.slots[slot_of(B, KK_VERT, blockIdx.x, local)];
    if (!selected(S, which)) return;
    const int i = local * blockDim.x + threadIdx.x;
    const bool live = i < S.m.V;
    count_clear(ct);
    __syncthreads();
    count_vertex(count_refs(S, bsel), i, S.verts[S.v_cur ^ vsel][live ? i : 0], live, false, ct);
}

void launch_bucket_count(const Launch& L, int vsel, int which, int bsel) {
    launch_kernel(L, true, true, k_bucket_count, dim3(L.grid[KK_VERT]), dim3(256), 0, L.B.slots, L.B.pre, L.B.n, vsel, which, bsel);
}

// ---------------------------------------------------------------------------
// Bucket layout for the next count, from the counts of parity `par`, with
// room for the surface to move: tile t gets d + d/2 + 32 slots, d the largest
// count among the 3x3 tiles around it (so a tile the surface moves into has
// room), placed after the tiles before it; inside it, cell c gets its own
// count n + n/2 + 8 plus a quarter of what the tile has beyond the sum of
// those (the last cell the rest).  Written into the other parity with its
// counters cleared.  A workgroup takes kLayoutTiles tiles (one per thread)
// and sums the shares of all tiles before them itself, from the tile counts
// staged in LDS (a stretch of rows at a time when they do not fit).
// ---------------------------------------------------------------------------
constexpr int kLayoutStage = 5056;   // tile counts staged in LDS at a time (of the candidates' 20 KB)

__device__ __forceinline__ uint32_t tile_share(uint32_t d) { return d + (d >> 1) + 32u; }

__device__ __forceinline__ void layout_tiles(const Slot& S, int par, int lblk, uint32_t* stage, uint32_t* sred) {
    const Buckets& b = S.b;
    const int tx = S.c.tiles_x, ty = S.c.tiles_y, ntiles = tx * ty;
    const uint32_t* __restrict__ tin = b.tsum[par];
    const uint4* __restrict__ cin = b.cells[par];
    uint4* __restrict__ cout = b.cells[par ^ 1];
    uint32_t* __restrict__ tout = b.tsum[par ^ 1];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nthr = blockDim.x, nw = nthr / 64;
    const int t0 = lblk * kLayoutTiles;
    // this thread's tile: its cells' counts, issued first
    const int t = t0 + threadIdx.x;
    const bool live = t < ntiles;
    const int tl = live ? t : 0;
    uint32_t c4[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) c4[q] = cin[4 * tl + q].z;
    // tiles [c0, ce) are summed, or laid out, from the counts [lo, hi) in the
    // stage (a row and a tile more on either side)
    uint32_t part = 0u, R = 0u;
    for (int c0 = 0;;) {
        const int lo = max(c0 - tx - 1, 0), hi = min(ntiles, lo + kLayoutStage);
        for (int u = lo + threadIdx.x; u < hi; u += nthr * 10) {
            uint32_t a[10];
#pragma unroll
            for (int k = 0; k < 10; ++k) a[k] = tin[min(u + nthr * k, hi - 1)];
#pragma unroll
            for (int k = 0; k < 10; ++k)
                if (u + nthr * k < hi) stage[u + nthr * k - lo] = a[k];
        }
        __syncthreads();
        // largest count of column x over rows y-1..y+1 (0 outside the image);
        // the largest count of the 3x3 tiles around (x, y) is that of columns
        // x-1, x, x+1
        auto column = [&](int x, int y) {
            uint32_t d = 0u;
            if (x >= 0 && x < tx)
                for (int yy = max(y - 1, 0); yy <= min(y + 1, ty - 1); ++yy) d = max(d, stage[yy * tx + x - lo]);
            return d;
        };
        const int ce = hi == ntiles ? ntiles : hi - tx - 1;
        // shares of the tiles before this workgroup's: a contiguous run per
        // thread, walked along its rows with the three columns carried over
        const int pe = min(ce, t0);
        const int chunk = (pe - c0 + nthr - 1) / nthr;
        int u = c0 + threadIdx.x * chunk;
        const int ue = min(u + chunk, pe);
        if (u < ue) {
            int x = u % tx, y = u / tx;
            uint32_t cl = column(x - 1, y), cm = column(x, y), cr = column(x + 1, y);
            for (; u < ue; ++u) {
                part += tile_share(max(cl, max(cm, cr)));
                if (++x == tx) {
                    x = 0;
                    ++y;
                    cl = 0u; cm = column(0, y); cr = column(1, y);
                } else {
                    cl = cm; cm = cr; cr = column(x + 1, y);
                }
            }
        }
        // this thread's tile, from the stage that holds all of the workgroup's
        if (min(t0 + kLayoutTiles, ntiles) <= ce) {
            const int xl = tl % tx, yl = tl / tx;
            if (live) R = tile_share(max(column(xl - 1, yl), max(column(xl, yl), column(xl + 1, yl))));
            break;
        }
        c0 = pe;
        __syncthreads();   // the stage is consumed
    }
    for (int o = 32; o > 0; o >>= 1) part += (uint32_t)__shfl_xor((int)part, o);
    // the tiles' shares scanned over the wave
    uint32_t incl = R;
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = (uint32_t)__shfl_up((int)incl, o);
        if (lane >= o) incl += y;
    }
    if (lane == 63) { sred[wid] = part; sred[nw + wid] = incl; }
    __syncthreads();
    uint32_t base = 0u;
    for (int w = 0; w < nw; ++w) base += sred[w] + (w < wid ? sred[nw + w] : 0u);
    if (live) {
        // R >= the cells' own shares: d >= the tile's count, and the cells'
        // halves sum to at most the tile's half
        uint32_t own[4], sum = 0u;
#pragma unroll
        for (int q = 0; q < 4; ++q) { own[q] = c4[q] + (c4[q] >> 1) + 8u; sum += own[q]; }
        const uint32_t extra = (R - sum) >> 2;
        // counts of one count phase sum to at most V, so the regions end by
        // ncap; the clamp only keeps every region inside the buffer
        const uint32_t ncap = (uint32_t)b.ncap;
        uint32_t o = base + incl - R;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            cout[4 * t + q] = make_uint4(kInfBits, 0u, 0u, min(o, ncap));
            o += own[q] + extra;
        }
        tout[t] = 0u;
        if (t == ntiles - 1) cout[4 * ntiles] = make_uint4(kInfBits, 0u, 0u, min(base + incl, ncap));
    }
    if (lblk == 0 && threadIdx.x == 0) b.ovfn[par ^ 1] = 0u;
}

__global__ void __launch_bounds__(kAssocThreads) k_layout(const Slot* __restrict__ bs, const int* __restrict__ bp, int bn, int bsel) {
    const Batch B{bs, bp, bn};
    __shared__ uint32_t stage[kLayoutStage];
    __shared__ uint32_t sred[2 * (kAssocThreads / 64)];
    int local;
    const Slot& S = B.slots[slot_of(B, KK_LAYOUT, blockIdx.x, local)];
    layout_tiles(S, S.bpar ^ bsel, local, stage, sred);
}

void launch_layout(const Launch& L, int bsel) {
    launch_kernel(L, true, true, k_layout, dim3(L.grid[KK_LAYOUT]), dim3(kAssocThreads), 0, L.B.slots, L.B.pre, L.B.n, bsel);
}

// ---------------------------------------------------------------------------
// association
// ---------------------------------------------------------------------------
// Lower bound on the distance from the pixel's point (depth d) to any vertex
// whose bucket is m >= 1 rings away: the vertex's ray makes an angle of at
// least (m - 1/2) pixels with the pixel's ray, so the distance is at least
// d * (m - 1/2) / (f_max * R_max), R_max bounding |(b, 1)| over the image.
// lb_c1 = (1 - 1e-4) / (f_max R_max); the 0.001 and 1e-6 terms absorb the
// float32 rounding of the bucket and of the back-projected point.
__device__ __forceinline__ float ring_lb(const DevCam& c, float d, int m) {
    float t = ((float)m - 0.501f) * c.lb_c1 - 1e-6f;
    return t > 0.0f ? d * t : 0.0f;
}

// z-range test: true if no vertex with z in [zmn, zmx] can have a squared
// distance that beats (or, with no match yet, reaches) the current bound.
__device__ __forceinline__ bool z_pruned(float zmn, float zmx, float pz, float bound, bool found) {
    float g1 = zmn - pz, g2 = pz - zmx;
    float g = fmaxf(g1, g2);
    if (!(g > 0.0f)) return false;
    float g2s = g * g;
    return g2s > bound || (!found && g2s >= bound);
}

// One workgroup per 8x8 tile, one wave per 4x4 quadrant of it (one cell of
// the bucket index).  Lane = pixel (16) x slot (4): candidate vertices, copied
// into the wave's LDS, go through the wave four at a time, each lane comparing
// its pixel's point with the candidate of its slot and keeping the key
// (d2 bits << 32 | vertex id), whose minimum is the nearest vertex with ties
// to the lower index; the slots of a pixel are combined across lanes.  The
// same launch also runs the layout of the next count (its first workgroups,
// from the counts read here) and the vertex normals of the surface (the
// workgroups after them).
constexpr int kAssocWaves = kAssocThreads / 64;
constexpr int kAssocPass = 304;   // candidates per pass
// Vertices of a cell that is compared on its own first: its vertices lie so
// close that most pixels need none of the eight cells around it, whose
// thousands of candidates would take pass after pass.  Nine cells at once
// against this, us a frame of five iterations: 200,000 vertices on 96x80
// pixels (1,300 a cell) 2968 / 1721, on 160x120 1558 / 999, 50,000 on 160x120
// 557 / 444, 10,000 on 64x48 434 / 347; 200,000 on 512x424 (100 a cell) 571 /
// 565, 50,000 on 640x480 (25 a cell) 323 / 322.  At 512 the third and fourth
// are lost again; at 128 cells of middling size pay for a third round of loads
// in the launch's longest waves (23,457 vertices on 333x251 1308 -> 1334 us a
// pass, point clouds of 31,113 on 424x320 1227 -> 1246).
constexpr int kDenseCell = 256;
constexpr int kWindowCells = 5;   // cells from a quadrant's to the last of the 5x5 tiles around its own
constexpr int kAssocBuf = kAssocPass + 16;   // and what is read past them (20 KB of LDS a workgroup: eight fit a compute unit)
static_assert(kAssocWaves == 4, "a wave per quadrant of a tile");
static_assert(kAssocPass % 16 == 0, "a pass is whole trips of four slots x four steps");

// Keys compare as doubles: a key's high word is the bits of a squared
// distance (>= 0, at most +inf), so its bits are those of a finite positive
// double, whose order is the order of the bits (as integers a minimum takes a
// 64-bit compare and two selects).  Never given a NaN: counted vertices and
// valid points are finite where d2 could be one.
__device__ __forceinline__ double key_of(uint32_t d2, uint32_t id) {
    return __hiloint2double((int)d2, (int)id);
}
__device__ __forceinline__ uint32_t key_d2(double k) { return (uint32_t)__double2hiint(k); }
__device__ __forceinline__ uint32_t key_id(double k) { return (uint32_t)__double2loint(k); }
__device__ __forceinline__ double key_min(double a, double b) {
    double r;   // (fmin would first quiet both operands)
    asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// A lane swap must not read a register in the two cycles after a vector
// instruction wrote it; the compiler sees to that for its own instructions,
// not for key_min's.
__device__ __forceinline__ double key_settled(double k) {
    asm("s_nop 1" : "+v"(k));
    return k;
}

// Lanes l, l ^ 16, l ^ 32, l ^ 48: the four lanes (slots) of a pixel.  Each
// swap leaves the two halves' values side by side in every lane.
typedef unsigned int u2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ double slot_min(double k) {
    k = key_settled(k);
    u2v lo = __builtin_amdgcn_permlane16_swap(key_id(k), key_id(k), false, false);
    u2v hi = __builtin_amdgcn_permlane16_swap(key_d2(k), key_d2(k), false, false);
    k = key_settled(key_min(key_of(hi.x, lo.x), key_of(hi.y, lo.y)));
    lo = __builtin_amdgcn_permlane32_swap(key_id(k), key_id(k), false, false);
    hi = __builtin_amdgcn_permlane32_swap(key_d2(k), key_d2(k), false, false);
    return key_min(key_of(hi.x, lo.x), key_of(hi.y, lo.y));
}

__device__ __forceinline__ float4 lds_volatile(const float4* p) {
    typedef float v4f __attribute__((ext_vector_type(4)));
    const v4f t = *(const volatile __attribute__((address_space(3))) v4f*)p;
    return make_float4(t.x, t.y, t.z, t.w);
}

// minimum over the lanes l, l ^ 16, l ^ 32, l ^ 48
__device__ __forceinline__ float rows_min(float v) {
    u2v t = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = fminf(__uint_as_float(t.x), __uint_as_float(t.y));
    t = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fminf(__uint_as_float(t.x), __uint_as_float(t.y));
}

// minimum over the 16 lanes of a row, in every lane of it
template <int ROR>
__device__ __forceinline__ float row_step_min(float v) {
    return fminf(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x120 | ROR, 0xF, 0xF, false)));
}
__device__ __forceinline__ float row_min(float v) {
    return row_step_min<1>(row_step_min<2>(row_step_min<4>(row_step_min<8>(v))));
}

// The pixel's depth z from the depth image or the organised cloud (then with
// the point's x and y); false if the pixel has no measurement.
__device__ __forceinline__ bool pixel_depth(const DevCam& c, const float* __restrict__ depth,
                                            const float* __restrict__ xyz, int u, int v, float& px, float& py,
                                            float& pz) {
    px = py = pz = 0.0f;
    if (u >= c.W || v >= c.H) return false;
    const uint32_t k = (uint32_t)(v * c.W + u);
    if (xyz) {
        px = ldg(xyz + 3 * k); py = ldg(xyz + 3 * k + 1); pz = ldg(xyz + 3 * k + 2);
        return isfinite(px) && isfinite(py) && isfinite(pz) && pz > 0.0f;
    }
    const float d = ldg(depth + k);
    if (!(d > 0.0f && isfinite(d))) return false;
    pz = d;
    return true;
}
// x and y of a depth image's pixel (back-projected), apart from its depth: a
// wave of background does not need them
__device__ __forceinline__ void back_project(const DevCam& c, int u, int v, float d, float& px, float& py) {
#pragma clang fp contract(off)
    px = (((float)u - c.cx) * d) / c.fx;
    py = (((float)v - c.cy) * d) / c.fy;
}

// Tile rings that can hold a vertex closer than tau to a point at depth z or
// beyond, capped by the image.  An over-estimate is harmless: the estimates
// of the reciprocals (1 ulp) are made up for by the last factor.
__device__ __forceinline__ int window_tiles(const DevCam& c, float tau, float z) {
    const float mf = 0.501f + (tau * __builtin_amdgcn_rcpf(z) + 1e-6f) * __builtin_amdgcn_rcpf(c.lb_c1) * 1.00001f;
    return ((int)fminf(mf, (float)max(c.W, c.H)) + 8) >> 3;
}

// A cell's record as a search holds it, one or two per lane: the cell, its
// z range and its region; `more` where vertices beyond the region went to
// the overflow list.
struct CellRec {
    int cx, cy;
    float zmn, zmx;
    uint32_t first, n;
    bool more;
};

// The cell's record and the end of its region, as they are: cell q of tile
// (x, y), or cell 0 where there is none (`in` false or outside the image).
struct RawCell {
    uint4 r;
    uint32_t end;
    bool in;
};
__device__ __forceinline__ RawCell load_cell(const DevCam& c, const uint4* __restrict__ cells, int x, int y, int q,
                                             bool in) {
    RawCell k;
    k.in = in && (uint32_t)x < (uint32_t)c.tiles_x && (uint32_t)y < (uint32_t)c.tiles_y;
    const uint32_t ci = k.in ? (uint32_t)(4 * (y * c.tiles_x + x) + q) : 0u;
    k.r = ldg(cells + ci);
    k.end = ldg(&cells[ci + 1].w);
    return k;
}
// a cell with a z range (an empty one holds (+inf, 0)) that is not as far as
// the cutoff from all depths in [pmin, pmax].  The gap is subtracted and
// squared as a candidate's z difference is, and rounding keeps the order: a
// vertex of the cell has that z difference or a larger one to every pixel,
// and a squared distance no smaller than its square.
__device__ __forceinline__ bool cell_meets(const RawCell& k, float pmin, float pmax, float tau2) {
    const float zmn = __uint_as_float(k.r.x), zmx = __uint_as_float(k.r.y);
    const float g = fmaxf(fmaxf(zmn - pmax, pmin - zmx), 0.0f);
    return k.in && zmn <= zmx && g * g < tau2;
}
__device__ __forceinline__ CellRec cell_rec(const RawCell& w, int x, int y, int q) {
    CellRec k;
    k.cx = 2 * x + (q & 1);
    k.cy = 2 * y + (q >> 1);
    k.zmn = __uint_as_float(w.r.x);
    k.zmx = __uint_as_float(w.r.y);
    k.first = w.r.w;
    const uint32_t cap = w.end > w.r.w ? w.end - w.r.w : 0u;
    k.n = min(w.r.z, cap);
    k.more = w.r.z > cap;
    return k;
}

// The search of one quadrant (4x4 pixels, one cell of the bucket index) of a
// tile by one wave with an LDS buffer of kAssocPass candidates: the pixels'
// matches, the per-vertex sums, and the quadrant's counts of (valid, matched,
// newly observed) pixels.
//
// The cells of the 5x5 tiles around the tile come with the pixels, in one
// round of loads (two records per lane).  A wave none of whose cells has a z
// range within tau of its points' is done (the background).  Otherwise the
// quadrant's cell and the eight around it are compared first (a dense cell by
// itself, then what is still needed of the eight), then, with the bounds they
// leave, whatever cell some pixel still needs.  Only a window wider than 16
// pixels goes on, ring by ring of tiles.
//
// A background wave is bound by one round of loads, and all of them together
// by instruction issue, so it forms no more than the depths and two range
// tests (a wave per quadrant rather than per two rows: half as many); a
// searching wave by its rounds of loads (pixels and cells, candidates, the
// match's vertex, its sums: about 6 us together under the launch's load) and
// 7 ns a candidate.  50,000 vertices at 640x480 (19,200 waves, 1,680 of
// which search, 226 candidates on average, 700 at most): with eight waves a
// tile that reloaded the window and then the cell records, 31.7 us a launch
// and 15.1 M vector instructions; so 18.2 us and 5.2 M.  A batch of 32 such
// streams: 541 us behind a screen that queued the tiles to search, 350 us
// without one.
__device__ __forceinline__ int3 search_quadrant(const Slot& S, int par, int vsel, int tx, int ty, int quad, float4* cand) {
    const DevCam& c = S.c;
    const Buckets& b = S.b;
    const uint4* __restrict__ cells = b.cells[par];
    const int lane = wave_lane();
    const int q = lane & 15, slot = lane >> 4;
    const int ccx = 2 * tx + (quad & 1), ccy = 2 * ty + (quad >> 1);   // the quadrant's cell
    const int u = ccx * 4 + (q & 3), v = ccy * 4 + (q >> 2);
    const bool inimg = u < c.W && v < c.H;
    // the 5x5 tiles' cells: entry e is cell e & 3 of tile e >> 2, row-major
    const int qc = lane & 3, e0 = lane >> 2, e1 = 16 + (lane >> 2);
    const int ey0 = (e0 * 13) >> 6, ey1 = (e1 * 13) >> 6;   // e / 5 for e < 32
    const int wx0 = e0 - 5 * ey0 - 2, wy0 = ey0 - 2, wx1 = e1 - 5 * ey1 - 2, wy1 = ey1 - 2;
    const RawCell raw0 = load_cell(c, cells, tx + wx0, ty + wy0, qc, true);
    const RawCell raw1 = load_cell(c, cells, tx + wx1, ty + wy1, qc, e1 < 25);
    float px, py, pz;
    const bool valid = pixel_depth(c, S.depth, S.xyz, u, v, px, py, pz);
    const float tau = S.tau, tau2 = tau * tau;
    const uint32_t tau2_bits = __float_as_uint(tau2);
    // key of the best candidate so far (this lane's slot; all slots' after a
    // slot_min); an unmatched valid pixel holds (tau^2, 0), which no candidate
    // at distance >= tau can undercut, an invalid one 0, which nothing
    // undercuts
    double key = valid ? key_of(tau2_bits, 0u) : 0.0;
    const unsigned long long vb = __ballot(slot == 0 && valid);
    if (vb) {
        // z range of the wave's points (every row of 16 lanes holds all of
        // them), the tile rings of its window, and the cells within reach in
        // both
        const float pmin = row_min(valid ? pz : INFINITY), pmax = -row_min(valid ? -pz : INFINITY);
        const int tr = wave_uniform(window_tiles(c, tau, pmin));
        const unsigned long long in0 = __ballot(cell_meets(raw0, pmin, pmax, tau2) && max(abs(wx0), abs(wy0)) <= tr);
        const unsigned long long in1 = __ballot(cell_meets(raw1, pmin, pmax, tau2) && max(abs(wx1), abs(wy1)) <= tr);
        if ((in0 | in1) != 0ull || tr > 2) {
            CellRec r0 = cell_rec(raw0, tx + wx0, ty + wy0, qc), r1 = cell_rec(raw1, tx + wx1, ty + wy1, qc);
            if (S.depth) back_project(c, u, v, pz, px, py);
            // held in scalar registers: read through the slot inside the copy
            // loops, they would be reloaded after every copy into LDS (which
            // the compiler takes as a store that may alias them), each reload
            // waiting for every copy still in flight
            const float4* __restrict__ cellv = wave_uniform(b.cellv);
            const uint32_t ovf_at = wave_uniform((uint32_t)b.ncap);
            // the overflow list: compared whole, once, by a wave that needs one
            // of the cells whose region was full
            const uint32_t novf = wave_uniform(min(b.ovfn[par], (uint32_t)S.m.V));
            bool ovf_done = false;
            auto nearer = [&](const float4& s) {
                const float dx = s.x - px, dy = s.y - py, dz = s.w - pz;
                const float d2 = (dx * dx + dy * dy) + dz * dz;
                key = key_min(key, key_of(__float_as_uint(d2), __float_as_uint(s.z)));
            };
            // compare every pixel with the cells of the masks (of the records
            // a and b), in passes of kAssocPass candidates copied from the
            // cells' regions straight into LDS (one DMA load per cell, all in
            // flight together); extra candidates are real vertices, so the
            // minimum stays exact
            auto compare = [&](unsigned long long ma, const CellRec& ra, unsigned long long mb, const CellRec& rb) {
                const bool take_ovf = !ovf_done && ((ma & __ballot(ra.more)) | (mb & __ballot(rb.more))) != 0ull;
                ovf_done = ovf_done || take_ovf;
                for (uint32_t pass = 0;; pass += kAssocPass) {
                    const uint32_t pend = pass + (uint32_t)kAssocPass;
                    uint32_t pre = 0u;
                    // candidates [off, off + cnt) of `cellv` as the segment after `pre`
                    auto segment = [&](uint32_t off, uint32_t cnt) {
                        const uint32_t a0 = max(pre, pass), a1 = min(pre + cnt, pend);
                        for (uint32_t s0 = a0; s0 < a1; s0 += 64u) {
                            if ((uint32_t)lane < a1 - s0)
                                __builtin_amdgcn_global_load_lds(
                                    (const void*)(cellv + (off + (s0 - pre) + (uint32_t)lane)),
                                    (__attribute__((address_space(3))) void*)&cand[s0 - pass], 16, 0, 0);
                        }
                        pre += cnt;
                    };
                    for (unsigned long long m = ma; m; m &= m - 1ull) {
                        const int k = __builtin_ctzll(m);
                        segment((uint32_t)__builtin_amdgcn_readlane((int)ra.first, k),
                                (uint32_t)__builtin_amdgcn_readlane((int)ra.n, k));
                    }
                    for (unsigned long long m = mb; m; m &= m - 1ull) {
                        const int k = __builtin_ctzll(m);
                        segment((uint32_t)__builtin_amdgcn_readlane((int)rb.first, k),
                                (uint32_t)__builtin_amdgcn_readlane((int)rb.n, k));
                    }
                    if (take_ovf) segment(ovf_at, novf);
                    if (pre <= pass) break;   // (pre: the total)
                    const int n = (int)min((uint32_t)kAssocPass, pre - pass);
                    // the pass's last trip filled up with entries at +inf: for
                    // a finite pixel their d2 is +inf, whose bits no key of a
                    // valid pixel (at most tau^2, 0) or of an invalid one (0)
                    // exceeds
                    const int ntrip = (n + 15) & ~15;
                    if (lane < ntrip - n) cand[n + lane] = make_float4(INFINITY, INFINITY, 0.0f, INFINITY);
                    __builtin_amdgcn_s_waitcnt(0);   // the copies have landed in LDS
                    __builtin_amdgcn_wave_barrier();
                    // four slots x four steps per trip, the LDS reads two
                    // steps ahead (past the end: unused)
                    // (the first ones read as volatile, so that they and those
                    // of the loop's end are not made one read at its start)
                    const float4* const mine = cand + slot;
                    float4 s0 = lds_volatile(mine), s1 = lds_volatile(mine + 4);
                    for (int i0 = 0; i0 < ntrip; i0 += 16) {
                        const float4 s2 = mine[i0 + 8], s3 = mine[i0 + 12];
                        nearer(s0);
                        nearer(s1);
                        s0 = mine[i0 + 16];
                        s1 = mine[i0 + 20];
                        nearer(s2);
                        nearer(s3);
                    }
                    __builtin_amdgcn_wave_barrier();
                    if (pre <= pend) break;
                }
                key = slot_min(key);
            };
            // is every vertex outside the square of cells [x0, x1] x [y0, y1]
            // (the pixel inside it) too far to be the pixel's?
            auto settled = [&](int x0, int x1, int y0, int y1) {
                const int m_next = min(min(u - 4 * x0, 4 * x1 + 3 - u), min(v - 4 * y0, 4 * y1 + 3 - v)) + 1;
                const float lb = ring_lb(c, pz, m_next);
                return !valid || lb * lb >= __uint_as_float(key_d2(key));
            };
            // lane = cell: does one of the wave's open pixels need it (the
            // pixel-distance and z-range bounds cannot exclude a better
            // vertex)?  One open pixel a round.
            auto needed = [&](unsigned long long open, const CellRec& k) {
                bool need = false;
                for (unsigned long long m = open; m; m &= m - 1ull) {
                    const int pq = __builtin_ctzll(m);
                    const int up = ccx * 4 + (pq & 3), vp = ccy * 4 + (pq >> 2);
                    const float pzp = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(pz), pq));
                    const uint32_t bp = (uint32_t)__builtin_amdgcn_readlane((int)key_d2(key), pq);
                    const float bound = __uint_as_float(bp);
                    const int X0 = k.cx * 4, Y0 = k.cy * 4;
                    const int mx = max(max(X0 - up, up - (X0 + 3)), 0), my = max(max(Y0 - vp, vp - (Y0 + 3)), 0);
                    const float lb = ring_lb(c, pzp, max(mx, my));
                    need = need || (!(lb * lb >= bound) && !z_pruned(k.zmn, k.zmx, pzp, bound, bp < tau2_bits));
                }
                return need;
            };
            // z range of the cells in reach
            const float wmin = row_min(rows_min(fminf((in0 >> lane) & 1ull ? r0.zmn : INFINITY, (in1 >> lane) & 1ull ? r1.zmn : INFINITY)));
            const float wmax = -row_min(rows_min(fminf((in0 >> lane) & 1ull ? -r0.zmx : INFINITY, (in1 >> lane) & 1ull ? -r1.zmx : INFINITY)));
            // first the quadrant's cell (cell `quad` of the window's middle
            // tile) with the eight around it, or, where it is dense, that cell
            // and then what of the eight some pixel still needs; then what some
            // pixel still needs of the rest of the 5x5 tiles (`reach`: cells
            // from the quadrant's that are through with)
            auto within = [&](const CellRec& k, int a, int b) {
                const int d = max(abs(k.cx - ccx), abs(k.cy - ccy));
                return d > a && d <= b;
            };
            int reach = __builtin_amdgcn_readlane((int)r0.n, 4 * 12 + quad) < kDenseCell ? 1 : 0;
            unsigned long long m0 = in0 & __ballot(within(r0, -1, reach)), m1 = in1 & __ballot(within(r1, -1, reach));
            // ring of tiles whose cells r0 and r1 hold (2: the 5x5 tiles), and
            // where its next 32 tiles start (past its end: none left)
            int ring = 2, t0 = 0;
            for (;;) {
                if ((m0 | m1) != 0ull) compare(m0, r0, m1, r1);
                if (reach < kWindowCells) {
                    // (a pixel of the background beside the subject needs nothing)
                    const unsigned long long open = __ballot(!settled(ccx - reach, ccx + reach, ccy - reach, ccy + reach) &&
                                                             !z_pruned(wmin, wmax, pz, __uint_as_float(key_d2(key)), key_d2(key) < tau2_bits)) & 0xFFFFull;
                    const int next = open && reach == 0 ? 1 : kWindowCells;
                    if (open) {
                        m0 = in0 & __ballot(within(r0, reach, next) && needed(open, r0));
                        m1 = in1 & __ballot(within(r1, reach, next) && needed(open, r1));
                    }
                    reach = next;
                    if (open) continue;
                }
                if (tr <= 2) break;
                // a wider window: the rings of tiles from the third on, 32
                // tiles (two records per lane) at a time
                if (ring == 2 || t0 >= 8 * ring) { ++ring; t0 = 0; }
                const unsigned long long open =
                    __ballot(!settled(2 * (tx - ring) + 2, 2 * (tx + ring) - 1, 2 * (ty - ring) + 2, 2 * (ty + ring) - 1)) & 0xFFFFull;
                if (ring > tr || !open) break;
                const int side = 2 * ring + 1;
                auto ring_cell = [&](int k, CellRec& rec) {
                    // the ring's tiles: upper row, lower row, left, right column
                    int x, y;
                    if (k < side) { x = tx - ring + k; y = ty - ring; }
                    else if (k < 2 * side) { x = tx - ring + (k - side); y = ty + ring; }
                    else if (k < 3 * side - 2) { x = tx - ring; y = ty - ring + 1 + (k - 2 * side); }
                    else { x = tx + ring; y = ty - ring + 1 + (k - (3 * side - 2)); }
                    const RawCell raw = load_cell(c, cells, x, y, qc, k < 8 * ring);
                    rec = cell_rec(raw, x, y, qc);
                    return cell_meets(raw, pmin, pmax, tau2);
                };
                const bool meets0 = ring_cell(t0 + (lane >> 2), r0), meets1 = ring_cell(t0 + 16 + (lane >> 2), r1);
                t0 += 32;
                m0 = __ballot(meets0);
                m1 = __ballot(meets1);
                if (m0) m0 &= __ballot(needed(open, r0));
                if (m1) m1 &= __ballot(needed(open, r1));
            }
        }
    }
    // slot 0 lanes hold the pixels
    int bestv = -1;
    bool first = false;
    const bool mine = slot == 0;
    if (mine && valid && key_d2(key) < tau2_bits) {
        const Accum& a = S.a;
        bestv = (int)key_id(key);
        const float4 sv = ldg_xyz(S.verts[S.v_cur ^ vsel] + bestv);
        const float dx = sv.x - px, dy = sv.y - py, dz = sv.z - pz;
        uint32_t old = atomic_add_g(a.cnt + bestv, 1u);
        atomic_add_g((unsigned long long*)&a.sx[bestv], (unsigned long long)(long long)rintf(-dx * 4294967296.0f));
        atomic_add_g((unsigned long long*)&a.sy[bestv], (unsigned long long)(long long)rintf(-dy * 4294967296.0f));
        atomic_add_g((unsigned long long*)&a.sz[bestv], (unsigned long long)(long long)rintf(-dz * 4294967296.0f));
        first = old == 0u;
    }
    if (mine && inimg) stg(S.assoc + v * c.W + u, bestv);
    const unsigned long long ab = __ballot(bestv >= 0), fb = __ballot(first);
    return make_int3(__popcll(vb), __popcll(ab), __popcll(fb));
}

__global__ void __launch_bounds__(kAssocThreads, 8) k_associate(const Slot* __restrict__ bs, const int* __restrict__ bp, int bn, int vsel, int bsel) {
    const Batch B{bs, bp, bn};
    __shared__ float4 scand[kAssocWaves][kAssocBuf];
    int local;
    const Slot& S = B.slots[slot_of(B, KK_ASSOC, blockIdx.x, local)];
    const DevCam& c = S.c;
    const Buckets& b = S.b;
    const int par = S.bpar ^ bsel;
    {
        const int nlay = layout_blocks(c.tiles_x * c.tiles_y), nnorm = assoc_normal_blocks(S.m.V);
        if (local < nlay) {
            static_assert(sizeof(scand) >= (kLayoutStage + 2 * kAssocWaves) * sizeof(uint32_t),
                          "layout stage fits the candidate LDS");
            uint32_t* const stage = reinterpret_cast<uint32_t*>(&scand[0][0]);
            layout_tiles(S, par, local, stage, stage + kLayoutStage);
            return;
        }
        if (local < nlay + nnorm) {
            const int i = (local - nlay) * kAssocThreads + threadIdx.x;
            const bool live = i < S.m.V;
            float nx, ny, nz;
            vertex_normal_lean(S.m, S.verts[S.v_cur ^ vsel], i, live, nx, ny, nz);   // the whole wave
            if (live) { S.normals.x[i] = nx; S.normals.y[i] = ny; S.normals.z[i] = nz; }
            return;
        }
        // workgroups rounding the extras up to a multiple of kXcds: none
        const int nextra = assoc_extra_blocks(c.tiles_x * c.tiles_y, S.m.V);
        if (local < nextra) return;
        local -= nextra;
    }
    const int at = b.torder[local];   // the tile's column and row
    if (at < 0) return;   // an XCD with fewer tiles than the others
    const int tx = at & 0xFFFF, ty = at >> 16, tile = ty * c.tiles_x + tx;
    const int wid = threadIdx.x >> 6;
    const int3 r = search_quadrant(S, par, vsel, tx, ty, wid, scand[wid]);
    // per-workgroup counts go to this workgroup's own slot (no shared counter:
    // device-wide atomics on one address serialise across the chip), through
    // the waves' own buffers, done with
    if ((threadIdx.x & 63) == 0) *reinterpret_cast<int4*>(scand[wid]) = make_int4(r.x, r.y, r.z, 0);
    __syncthreads();
    if (threadIdx.x == 0) {
        int4 t = make_int4(0, 0, 0, 0);
        for (int w = 0; w < kAssocWaves; ++w) {
            const int4 n = *reinterpret_cast<const int4*>(scand[w]);
            t.x += n.x; t.y += n.y; t.z += n.z;
        }
        b.bstat[tile] = t;
    }
}

void launch_associate(const Launch& L, int vsel, int bsel) {
    launch_kernel(L, true, true, k_associate, dim3(L.grid[KK_ASSOC]), dim3(kAssocThreads), 0, L.B.slots, L.B.pre, L.B.n, vsel, bsel);
}

}  // namespace trk
