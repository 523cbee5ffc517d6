// Residuals, pose Jacobian rows and the normal equations (Eq. 6-8).
//
// For each observed vertex i (at least one associated pixel and a non-zero
// normal) the residual is r_i = n_i . delta_i with delta_i the mean offset of
// its points (Eq. 6).  Its Jacobian row follows the chain rule of Section 4.2;
// with dH_{l,Delta}/dtheta_k = Xi_k H_{l,Delta} (see the FK kernel) and
// dT/dH collapsed against the normal into one dual quaternion c = (c_r, c_d),
//   c_d = (2/N) n r,   c_r = -(2/N) (n r x + n d + (n . v) r),   N = |r|^2
// for the blend H = (r, d), template point x = v0 + phi and skinned point v,
// every entry is a dot product of 6-vectors:
//   J_ik = - sum over influences m whose link chain holds joint k of
//          w_m [ vec(c_r H_m,r^* + c_d H_m,d^*) . Xi_k,r + vec(c_d H_m,r^*) . Xi_k,d ].
// Rows are built in LDS as [J | r] (never written to HBM) and the Gram matrix
// G = [J r]^T [J r] (which holds J^T J, J^T r and r^T r) is accumulated with
// MFMA with float32 accumulation, from one of three operand forms:
//   mode 0: float32 operands (v_mfma_f32_16x16x4_f32);
//   mode 1: each entry split as hi + lo in bfloat16, G ~ hi.hi + hi.lo + lo.hi
//           (3 bfloat16 products, about 2^-17 relative error per product);
//   mode 2: hi + mid + lo, G ~ hi.hi + hi.mid + mid.hi + hi.lo + lo.hi + mid.mid
//           (6 products, about 2^-24: float32 accuracy at bfloat16 rate).
// Each workgroup writes one partial G; partials are summed in workgroup
// order (deterministic) by a second kernel.
//
// A row is zero outside the chains of its vertex' links, and neighbouring
// vertices share them: 128 vertices of the 75-joint body touch 15 columns or
// so.  Which ones follows from the links alone, so the host lists each
// workgroup's columns (NeRef) and the tile, the MFMA blocks and the partial
// hold just these: of the 15 block products of 75 joints mostly one or three
// are left, and a partial shrinks from 15 KB to one or three.  Its sums are
// those of the full form to the bit (each entry takes the same products in
// the same order).
//
// Bound by the chain of one chunk -- the vertices' reads, their 6-vectors,
// the rows, the products, each behind a barrier -- for one stream, and by how
// many chunks a CU holds for many.  Full rows against column lists, with the
// reduction's share in brackets: one frame of 50 000 vertices 12.4 (5.0) ->
// 7.4 (5.9) us, 200 000 vertices 26.5 (5.0) -> 16.8 (6.4) us, 32 streams of
// 50 000 229 (52) -> 106 (29) us, 2 000 vertices 7.1 (3.9) -> 5.6 (4.7) us.
#include "common.h"
#include "dq.h"

namespace trk {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));

constexpr int kJTStride = kNeRows + 8;  // floats per LDS column of the row tile
constexpr int kGStride = 25;            // floats per row of per-influence 6-vectors
// upper 16x16 Gram blocks each of a workgroup's waves owns at most
constexpr int ne_blocks(int waves) { return ((kPPMax / 16) * (kPPMax / 16 + 1) / 2 + waves - 1) / waves; }
static_assert(kNeCols == kPPMax, "two column entries a lane, a byte each");
static_assert(kNeGrid <= kRedGroups * kRedPer, "the rank table's groups");

__device__ __forceinline__ void block_of(int idx, int nb, int& I, int& J) {
    int q = idx;
    for (I = 0; I < nb; ++I) {
        int len = nb - I;
        if (q < len) { J = I + q; return; }
        q -= len;
    }
    I = J = 0;
}

// what a vertex's row needs, read in one round of loads
struct VertexIn {
    float4 w, v;
    uint32_t links, cnt;
    float nx, ny, nz, x0, x1, x2;   // normal; template point + offset
    long long sx, sy, sz;           // fixed-point sums of its points' offsets
};

__device__ __forceinline__ void vertex_load(const DevModel& m, int i, const float4* v, const Vec3Buf& n,
                                            const Vec3Buf& phi, const Accum& a, VertexIn& in) {
    // global reads: as flat reads they would also count as LDS and scalar
    // accesses, and the first wait for one of those would wait for them
    in.w = ldg(m.w + i);
    in.links = ldg(m.links + i);
    in.v = ldg(v + i);
    in.nx = ldg(n.x + i); in.ny = ldg(n.y + i); in.nz = ldg(n.z + i);
    in.cnt = ldg(a.cnt + i);
    in.sx = (long long)ldg(a.sx + i); in.sy = (long long)ldg(a.sy + i); in.sz = (long long)ldg(a.sz + i);
    const float rx = ldg(m.rx + i), ry = ldg(m.ry + i), rz = ldg(m.rz + i);
    const float px = ldg(phi.x + i), py = ldg(phi.y + i), pz = ldg(phi.z + i);
    // every read issued before the first use of one
    __builtin_amdgcn_sched_barrier(0);
    in.x0 = rx + px;
    in.x1 = ry + py;
    in.x2 = rz + pz;
}

// The quaternion products of a vertex' row, with the order and the rounding
// of every step written out: left to the compiler, which product of a sum is
// rounded apart would change with the code around it, and with it the last
// bits of a frame's results.
// (0, n) q
__device__ __forceinline__ void vec_qmul(float nx, float ny, float nz, const float* q, float* o) {
    o[0] = fmaf(-nz, q[3], fmaf(-ny, q[2], -(nx * q[1])));
    o[1] = fmaf(-nz, q[2], fmaf(ny, q[3], nx * q[0]));
    o[2] = fmaf(nz, q[1], fmaf(ny, q[0], -(nx * q[3])));
    o[3] = fmaf(nz, q[0], fmaf(-ny, q[1], nx * q[2]));
}
// vector part of a b
__device__ __forceinline__ void qmul_vec(const float* a, const float* b, float* o) {
    o[0] = fmaf(-a[3], b[2], fmaf(a[2], b[3], fmaf(a[1], b[0], a[0] * b[1])));
    o[1] = fmaf(a[3], b[1], fmaf(a[2], b[0], fmaf(a[0], b[2], -(a[1] * b[3]))));
    o[2] = fmaf(a[3], b[0], fmaf(-a[2], b[1], fmaf(a[1], b[2], a[0] * b[3])));
}

// per-vertex 6-vectors of the Jacobian (one per influence, an unused one's
// left as it was) and the residual
__device__ __forceinline__ void vertex_terms(const float* sdq, const VertexIn& in, float* G, float& r_out,
                                             bool linear) {
    float H[8], sg[4];
    const float4 w = in.w;
    const uint32_t lk = in.links;
    const float inv = 1.0f / ((float)in.cnt * 4294967296.0f);
    const float dx = (float)in.sx * inv, dy = (float)in.sy * inv, dz = (float)in.sz * inv;
    if (linear) {
        // the linear blend: influence m moves the template point rigidly to
        // y_m = T(H_m, x), and dy_m/dtheta_k = Xi_k acting on y_m, so its
        // 6-vector is 2 w_m (y_m x n, n) (the one-influence case of the
        // collapsed form above)
        const float nx = in.nx, ny = in.ny, nz = in.nz;
        const float ws[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int l = (lk >> (8 * k)) & 0xFF;
            float* g = G + 6 * k;
            if (l == 0xFF) continue;
            float yx, yy, yz;
            dq_apply(sdq + 8 * l, in.x0, in.x1, in.x2, yx, yy, yz);
            const float s2 = 2.0f * ws[k];
            g[0] = s2 * det2(yy, nz, yz, ny);
            g[1] = s2 * det2(yz, nx, yx, nz);
            g[2] = s2 * det2(yx, ny, yy, nx);
            g[3] = s2 * nx;
            g[4] = s2 * ny;
            g[5] = s2 * nz;
        }
        r_out = dot3(nx, dx, ny, dy, nz, dz);
        return;
    }
    dq_blend(sdq, w, lk, H, sg);
    const float nx = in.nx, ny = in.ny, nz = in.nz;
    const float vx = in.v.x, vy = in.v.y, vz = in.v.z;
    const float N = fma_of(H[3], H[3], dot3(H[0], H[0], H[1], H[1], H[2], H[2]));
    const float s2 = 2.0f / N;
    float nr[4], nd[4];
    vec_qmul(nx, ny, nz, H, nr);
    vec_qmul(nx, ny, nz, H + 4, nd);
    const float x1 = in.x0, x2 = in.x1, x3 = in.x2;
    const float nrx[4] = {fmaf(-nr[3], x3, fmaf(-nr[2], x2, -(nr[1] * x1))), fmaf(-nr[3], x2, fmaf(nr[2], x3, nr[0] * x1)),
                          fmaf(nr[3], x1, fmaf(nr[0], x2, -(nr[1] * x3))), fmaf(-nr[2], x1, fmaf(nr[1], x2, nr[0] * x3))};
    const float ndotv = fmaf(nz, vz, fmaf(ny, vy, nx * vx));
    float cr[4], cd[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        cd[c] = s2 * nr[c];
        cr[c] = -s2 * fmaf(ndotv, H[c], nrx[c] + nd[c]);
    }
    const float ws[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        int l = (lk >> (8 * k)) & 0xFF;
        float* g = G + 6 * k;
        if (l == 0xFF) continue;
        const float* D = sdq + 8 * l;
        const float s = sg[k];
        const float rc[4] = {s * D[0], -s * D[1], -s * D[2], -s * D[3]};
        const float dc[4] = {s * D[4], -s * D[5], -s * D[6], -s * D[7]};
        float t1[3], t2[3], t3[3];
        qmul_vec(cr, rc, t1);
        qmul_vec(cd, dc, t2);
        qmul_vec(cd, rc, t3);
        const float ww = ws[k];
#pragma unroll
        for (int e = 0; e < 3; ++e) {
            g[e] = ww * (t1[e] + t2[e]);
            g[3 + e] = ww * t3[e];
        }
    }
    r_out = dot3(nx, dx, ny, dy, nz, dz);
}

// Dynamic LDS of the normal equations for the batch's widest column list
// (ncmax, in blocks of 16), padded size ppmax and link count lmax: the
// [col][row] tile (float32, or two / three bfloat16 planes), the per-row
// 6-vectors, links, residuals and the staged link offsets, generators and
// link chains.  33 KB for lists of up to 32 columns.
template <int MODE>
__host__ __device__ inline size_t ne_tile_bytes(int ncmax) {
    return (size_t)ncmax * kJTStride * (MODE == 0 ? 4 : MODE == 1 ? 4 : 6);
}
template <int MODE>
__host__ __device__ inline size_t ne_lds_bytes(int ncmax, int ppmax, int lmax) {
    return ne_tile_bytes<MODE>(ncmax) + 4 * (size_t)kNeRows * kGStride + 4 * (size_t)kNeRows * 2 + 16 +
           4 * (size_t)(8 * lmax + 8 * ppmax + 4 * lmax);
}

// BIG: an instance allowed more than 64 KB of LDS (column lists of more than
// 64 or so); smaller sizes use the other instance, which launches faster
template <int MODE, bool BIG, int NW>
__global__ void __launch_bounds__(64 * NW) k_normal_eq(const Slot* __restrict__ bs, const int* __restrict__ bp, int bn, int vsel, int pn, int ncmax, int ppmax, int lmax) {
    constexpr int kNeWaves = NW, kNeThreads = 64 * NW, kNeBlocks = ne_blocks(NW);
    const Batch B{bs, bp, bn};
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    unsigned char* q0 = smem;
    // [col][row] tile: float32 (mode 0) or two / three bfloat16 planes
    float* sJT = reinterpret_cast<float*>(q0);
    __bf16* plane0 = reinterpret_cast<__bf16*>(q0);
    __bf16* plane1 = plane0 + ncmax * kJTStride;
    __bf16* plane2 = plane1 + ncmax * kJTStride;
    q0 += ne_tile_bytes<MODE>(ncmax);
    float* sG = reinterpret_cast<float*>(q0);
    q0 += 4 * kNeRows * kGStride;
    uint32_t* slink = reinterpret_cast<uint32_t*>(q0);
    q0 += 4 * kNeRows;
    float* sr = reinterpret_cast<float*>(q0);
    q0 += 4 * kNeRows;
    int* scount = reinterpret_cast<int*>(q0);
    q0 += 16;
    float* sdq = reinterpret_cast<float*>(q0);
    q0 += 4 * 8 * lmax;
    float* sxi = reinterpret_cast<float*>(q0);
    q0 += 4 * 8 * ppmax;
    uint32_t* sanc = reinterpret_cast<uint32_t*>(q0);

    int wg;
    const Slot& S = B.slots[slot_of(B, KK_NE, blockIdx.x, wg)];
    const DevModel& m = S.m;
    const float* __restrict__ dq = S.dq;
    const float* __restrict__ xi = S.xi;
    const uint32_t* __restrict__ anc = S.anc;
    const float4* __restrict__ v = S.verts[S.v_cur ^ vsel];
    const Vec3Buf n = S.normals;
    const Vec3Buf phi = S.phi[phi_index(S, pn)];
    const Accum& a = S.a;
    const NeRef ne = S.ne;
    const bool linear = S.blend == kBlendLinear;
    const int nchunks = (m.V + kNeRows - 1) / kNeRows;
    const int tid = threadIdx.x, lane = tid & 63, wid = wave_uniform(tid >> 6);
    const int P = m.P;
    // this workgroup's columns, increasing, the residual (P) last: two a lane
    const uint8_t* __restrict__ cl = ne.cols + (size_t)kNeCols * wg;
    const int l0 = ldg(cl + lane), l1 = ldg(cl + 64 + lane);
    {
        // the three tables' first rounds read together (clamped indices; the
        // values past a table's end are not stored), the rest after
        const int n1 = 8 * m.L, n2 = 8 * P, n3 = 4 * m.L;
        const float t1 = ldg(dq + min(tid, n1 - 1));
        const float t2 = ldg(xi + min(tid, n2 - 1));
        const uint32_t t3 = ldg(anc + min(tid, n3 - 1));
        if (tid < n1) sdq[tid] = t1;
        if (tid < n2) sxi[tid] = t2;
        if (tid < n3) sanc[tid] = t3;
        for (int q = tid + kNeThreads; q < n1; q += kNeThreads) sdq[q] = dq[q];
        for (int q = tid + kNeThreads; q < n2; q += kNeThreads) sxi[q] = xi[q];
        for (int q = tid + kNeThreads; q < n3; q += kNeThreads) sanc[q] = anc[q];
    }
    const int ncol = __popcll(__ballot(l0 != 0xFF)) + __popcll(__ballot(l1 != 0xFF));
    const int nb = (ncol + 15) >> 4;
    const int nbt = nb * (nb + 1) / 2;
    f4 acc[kNeBlocks];
#pragma unroll
    for (int q = 0; q < kNeBlocks; ++q) acc[q] = f4{0.0f, 0.0f, 0.0f, 0.0f};

    for (int chunk = wg; chunk < nchunks; chunk += S.negrid) {
        // 1. compact the observed vertices of this chunk (every read of a
        //    vertex's row issued before the compaction)
        const uint32_t m0 = ldg(ne.mask + 4 * chunk + min(l0 >> 5, 3)), m1 = ldg(ne.mask + 4 * chunk + min(l1 >> 5, 3));
        bool obs = false;
        int i = chunk * kNeRows + tid;
        VertexIn in;
        if (tid < kNeRows && i < m.V) {
            vertex_load(m, i, v, n, phi, a, in);
            obs = in.cnt > 0u && (in.nx * in.nx + in.ny * in.ny + in.nz * in.nz) > 0.0f;
        }
        const unsigned long long bal = __ballot(obs);
        // the workgroup's columns that this chunk touches (with several
        // chunks a workgroup lists the columns of all)
        const unsigned long long tb0 = __ballot(l0 == P || (l0 < P && ((m0 >> (l0 & 31)) & 1u)));
        const unsigned long long tb1 = __ballot(l1 == P || (l1 < P && ((m1 >> (l1 & 31)) & 1u)));
        auto blk_used = [&](int K) { return ((K < 4 ? tb0 >> (16 * K) : tb1 >> (16 * K - 64)) & 0xFFFFull) != 0ull; };
        if (lane == 0 && wid < 2) scount[wid] = __popcll(bal);
        __syncthreads();   // (also: the tables are staged, the previous chunk's tile is consumed)
        const int nrows = scount[0] + scount[1];
        if (obs) {
            int row = __popcll(bal & ((1ull << lane) - 1ull)) + (wid == 1 ? scount[0] : 0);
            float r;
            vertex_terms(sdq, in, &sG[row * kGStride], r, linear);
            sr[row] = r;
            slink[row] = in.links;
        }
        __syncthreads();
        if (nrows == 0) continue;
        const int kstep = MODE == 0 ? 16 : 32;
        const int npad = (nrows + kstep - 1) / kstep * kstep;

        // 2. rows of [J r] into the [col][row] tile: a lane a row, the
        //    columns dealt to the waves (two waves a column for more than 64
        //    rows).  A row's per-influence 6-vectors stay in registers, the
        //    next column's twists and chain bits are read before this one is
        //    stored.
        {
            const bool two = npad > 64;
            const int row = (two ? (wid & 1) * 64 : 0) + lane;
            const int w0 = two ? wid >> 1 : wid, wstep = two ? kNeWaves / 2 : kNeWaves;
            const bool have = row < nrows;
            const uint32_t lk = have ? slink[row] : 0xFFFFFFFFu;
            const float rr = have ? sr[row] : 0.0f;
            auto columns = [&](auto nk_) {
                constexpr int NK = decltype(nk_)::value;   // influences that some row of the wave has
                struct ColIn { float x[6]; uint32_t bits[NK]; };
                float g[6 * NK];
                int lb[NK];
#pragma unroll
                for (int k = 0; k < NK; ++k) {
                    lb[k] = (lk >> (8 * k)) & 0xFF;
#pragma unroll
                    for (int e = 0; e < 6; ++e) g[6 * k + e] = sG[min(row, kNeRows - 1) * kGStride + 6 * k + e];
                }
                auto column = [&](int c) { return __builtin_amdgcn_readlane(c < 64 ? l0 : l1, c & 63); };
                auto read = [&](int col, ColIn& q) {
                    const int cc = min(col, P - 1);
                    const float4 xa = *reinterpret_cast<const float4*>(sxi + 8 * cc);
                    const float2 xb = *reinterpret_cast<const float2*>(sxi + 8 * cc + 4);
                    q.x[0] = xa.x; q.x[1] = xa.y; q.x[2] = xa.z; q.x[3] = xa.w; q.x[4] = xb.x; q.x[5] = xb.y;
#pragma unroll
                    for (int k = 0; k < NK; ++k) q.bits[k] = sanc[lb[k] == 0xFF ? 0 : 4 * lb[k] + (cc >> 5)];
                };
                ColIn cur, nxt;
                int col = column(min(w0, ncol - 1));
                read(col, cur);
                for (int c = w0; c < ncol; c += wstep) {
                    const int coln = column(min(c + wstep, ncol - 1));
                    read(coln, nxt);
                    float val = 0.0f;
                    if (col == P) {
                        val = rr;
                    } else if (((c < 64 ? tb0 >> c : tb1 >> (c - 64)) & 1ull) != 0ull) {
#pragma unroll
                        for (int k = 0; k < NK; ++k) {
                            const float* gk = g + 6 * k;
                            // (written out, so that the forms for fewer influences round alike)
                            float dt = fmaf(gk[0], cur.x[0], gk[1] * cur.x[1]);
#pragma unroll
                            for (int e = 2; e < 6; ++e) dt = fmaf(gk[e], cur.x[e], dt);
                            const float nv = val - dt;
                            val = (lb[k] != 0xFF && ((cur.bits[k] >> (col & 31)) & 1u)) ? nv : val;
                        }
                    }
                    const int at = c * kJTStride + row;
                    if (row < npad) {
                        if (MODE == 0) {
                            sJT[at] = val;
                        } else {
                            const __bf16 h = (__bf16)val;
                            const float rem = val - (float)h;
                            const __bf16 md = (__bf16)rem;
                            plane0[at] = h;
                            plane1[at] = md;
                            if (MODE == 2) plane2[at] = (__bf16)(rem - (float)md);
                        }
                    }
                    col = coln;
                    cur = nxt;
                }
            };
            if (__ballot((lk >> 16) != 0xFFFFu)) columns(std::integral_constant<int, 4>{});
            else if (__ballot((lk >> 8) != 0xFFFFFFu)) columns(std::integral_constant<int, 2>{});
            else columns(std::integral_constant<int, 1>{});
        }
        __syncthreads();

        // 3. Gram blocks (I <= J) owned by this wave.  (The entries of the
        //    last block past the column list are whatever the tile held: they
        //    touch no other entry's sum and are not read.)
#pragma unroll
        for (int q = 0; q < kNeBlocks; ++q) {
            const int idx = wid + kNeWaves * q;
            int I = 0, J = 0;
            if (idx < nbt) block_of(idx, nb, I, J);
            // a block of columns the chunk does not touch is zero in the
            // tile: its products are skipped
            if (idx < nbt && blk_used(I) && blk_used(J)) {
                const int ca = (I * 16 + (lane & 15)) * kJTStride;
                const int cb = (J * 16 + (lane & 15)) * kJTStride;
                if (MODE == 0) {
                    for (int k0 = 0; k0 < npad; k0 += 16) {
                        const int ro = k0 + 4 * (lane >> 4);
                        f4 av = *reinterpret_cast<const f4*>(&sJT[ca + ro]);
                        f4 bv = *reinterpret_cast<const f4*>(&sJT[cb + ro]);
                        acc[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(av.x, bv.x, acc[q], 0, 0, 0);
                        acc[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(av.y, bv.y, acc[q], 0, 0, 0);
                        acc[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(av.z, bv.z, acc[q], 0, 0, 0);
                        acc[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(av.w, bv.w, acc[q], 0, 0, 0);
                    }
                } else {
                    for (int k0 = 0; k0 < npad; k0 += 32) {
                        const int ro = k0 + 8 * (lane >> 4);
                        bf8 ah = *reinterpret_cast<const bf8*>(&plane0[ca + ro]);
                        bf8 am = *reinterpret_cast<const bf8*>(&plane1[ca + ro]);
                        bf8 bh = *reinterpret_cast<const bf8*>(&plane0[cb + ro]);
                        bf8 bm = *reinterpret_cast<const bf8*>(&plane1[cb + ro]);
                        // smallest products first
                        if (MODE == 2) {
                            bf8 al = *reinterpret_cast<const bf8*>(&plane2[ca + ro]);
                            bf8 bl = *reinterpret_cast<const bf8*>(&plane2[cb + ro]);
                            acc[q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, bh, acc[q], 0, 0, 0);
                            acc[q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bl, acc[q], 0, 0, 0);
                            acc[q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(am, bm, acc[q], 0, 0, 0);
                        }
                        acc[q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(am, bh, acc[q], 0, 0, 0);
                        acc[q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bm, acc[q], 0, 0, 0);
                        acc[q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bh, acc[q], 0, 0, 0);
                    }
                }
            }
        }
    }

    // 4. this workgroup's partial Gram: the upper blocks of its columns, each
    //    as the products left it (a lane's four rows of a column together)
    f4* out = reinterpret_cast<f4*>(S.partials + (size_t)wg * ne.width * ne.width);
#pragma unroll
    for (int q = 0; q < kNeBlocks; ++q) {
        const int idx = wid + kNeWaves * q;
        if (idx < nbt) {
            int I, J;
            block_of(idx, nb, I, J);
            out[64 * (I * (ne.width >> 4) + J) + lane] = acc[q];
        }
    }
}

// one chunk per workgroup up to kNeGrid workgroups; larger meshes loop over chunks
int ne_grid(int V) {
    int nchunks = (V + kNeRows - 1) / kNeRows;
    return nchunks < kNeGrid ? nchunks : kNeGrid;
}

constexpr size_t kSmallLds = 64 * 1024;

template <int MODE, int NW>
bool prepare_normal_eq_t() {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(k_normal_eq<MODE, true, NW>),
                               hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)ne_lds_bytes<MODE>(kNeCols, kPPMax, kMaxLinks + 1)) == hipSuccess;
}

bool prepare_normal_eq() {
    bool ok = true;
    ok = prepare_normal_eq_t<0, 4>() && ok;
    ok = prepare_normal_eq_t<1, 4>() && ok;
    ok = prepare_normal_eq_t<2, 4>() && ok;
    ok = prepare_normal_eq_t<0, 8>() && ok;
    ok = prepare_normal_eq_t<1, 8>() && ok;
    ok = prepare_normal_eq_t<2, 8>() && ok;
    return ok;
}

template <int MODE, int NW>
void launch_normal_eq_w(const Launch& L, int vsel, int pn) {
    const dim3 g(L.grid[KK_NE]);
    const int nc = L.ne_cols, pp = L.ne_pp, lm = L.ne_l;
    const size_t bytes = ne_lds_bytes<MODE>(nc, pp, lm);
    if (bytes <= kSmallLds)
        launch_kernel(L, true, true, k_normal_eq<MODE, false, NW>, g, dim3(64 * NW), bytes, L.B.slots, L.B.pre, L.B.n, vsel, pn, nc, pp, lm);
    else
        launch_kernel(L, true, true, k_normal_eq<MODE, true, NW>, g, dim3(64 * NW), bytes, L.B.slots, L.B.pre, L.B.n, vsel, pn, nc, pp, lm);
}

// Eight waves a workgroup while the workgroups start nearly together (one
// chunk's chain is then all that counts, and eight waves shorten it), four
// when the launch has many times what the CUs hold (the registers let a CU
// hold twice the workgroups of four).  Eight against four waves: 391
// workgroups 7.3 / 9.2 us, 782 12.4 / 12.3, 1 173 16.0 / 15.7, 1 564 19.4 /
// 17.7, 12 512 131 / 106.
constexpr int kNeFew = 1024;

template <int MODE>
void launch_normal_eq_t(const Launch& L, int vsel, int pn) {
    if (L.grid[KK_NE] <= kNeFew) launch_normal_eq_w<MODE, 8>(L, vsel, pn);
    else launch_normal_eq_w<MODE, 4>(L, vsel, pn);
}

void launch_normal_eq(const Launch& L, int gram_mode, int vsel, int pn) {
    if (gram_mode == 0) launch_normal_eq_t<0>(L, vsel, pn);
    else if (gram_mode == 1) launch_normal_eq_t<1>(L, vsel, pn);
    else launch_normal_eq_t<2>(L, vsel, pn);
}

// Sum of the partial Gram matrices in workgroup order, in float64; writes the
// full symmetric matrix (the upper triangle is summed and mirrored, so the
// result is exactly symmetric).  A workgroup handles 32 elements of one
// 16x16 block; each element's partials are split into kRedGroups contiguous
// groups summed by as many threads, and the group sums are added in group
// order.  The rank table says where a column lies in each partial (0xFF: not
// in it, its entries are zero); a thread reads its two columns' bytes for the
// whole group, then the entries that are there (a buffer read past the end
// gives zero and reads nothing).
__global__ void __launch_bounds__(32 * kRedGroups) k_gram_reduce(const Slot* __restrict__ bs, const int* __restrict__ bp, int bn) {
    const Batch B{bs, bp, bn};
    __shared__ double part[kRedGroups][32];
    int local;
    const Slot& S = B.slots[slot_of(B, KK_REDUCE, blockIdx.x, local)];
    const int PP = S.PP, nparts = S.negrid;
    float* __restrict__ partials = S.partials;
    double* __restrict__ gram = S.gram;
    const int nb = PP >> 4;
    const int blk = local >> 3;               // 8 workgroups per 16x16 block
    const int el = (local & 7) * 32 + (threadIdx.x & 31);
    const int grp = threadIdx.x >> 5;
    int I, J;
    block_of(blk, nb, I, J);
    const int i = I * 16 + (el >> 4), j = J * 16 + (el & 15);
    // the tree-form pose solve takes this element (damped, frozen) in its front image
    // (its reads unconditional at clamped indices, issued with the partials'
    // below: a read under a condition is waited for inside it)
    const int* __restrict__ gfm = S.tree.gfmap;
    const int P = S.m.P;
    int fe = -1;
    double prior_i = 0.0, theta_i = 0.0;
    int act_i = 0, act_j = 0;
    if (gfm) {   // the same for the whole workgroup
        const int ic = min(i, P - 1), jc = min(j, P - 1);
        const int f0 = gfm[i * PP + j];
        const double pr = S.jt->prior[ic], th = S.theta[ic];
        const int ai = S.jt->active[ic], aj = S.jt->active[jc];
        fe = (grp == 0 && i <= j) ? f0 : -1;
        if (fe >= 0) {
            prior_i = pr;
            act_i = ai;
            act_j = j < P ? aj : 1;
            theta_i = th;
        }
    }
    const NeRef ne = S.ne;
    const int per = (nparts + kRedGroups - 1) / kRedGroups;
    const int q0 = grp * per, q1 = min(nparts, q0 + per);
    const uint4* __restrict__ ri = reinterpret_cast<const uint4*>(ne.rank + ((size_t)i * kRedGroups + grp) * kRedPer);
    const uint4* __restrict__ rj = reinterpret_cast<const uint4*>(ne.rank + ((size_t)j * kRedGroups + grp) * kRedPer);
    uint32_t ci[kRedPer / 4], cj[kRedPer / 4];
#pragma unroll
    for (int t = 0; t < kRedPer / 16; ++t) {
        const uint4 x = ldg(ri + t), y = ldg(rj + t);
        ci[4 * t] = x.x; ci[4 * t + 1] = x.y; ci[4 * t + 2] = x.z; ci[4 * t + 3] = x.w;
        cj[4 * t] = y.x; cj[4 * t + 1] = y.y; cj[4 * t + 2] = y.z; cj[4 * t + 3] = y.w;
    }
    const uint32_t stride = 4u * ne.width * ne.width;
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(partials, 0, nparts * stride, 0x00020000);
    double s = 0.0;
#pragma unroll
    for (int t = 0; t < kRedPer; t += 8) {
        // (a wave whose elements none of these partials hold goes on)
        if (__ballot((ci[t / 4] & ci[t / 4 + 1]) != ~0u && (cj[t / 4] & cj[t / 4 + 1]) != ~0u) == 0) continue;
        float a[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const uint32_t a0 = (ci[(t + u) / 4] >> (8 * (u & 3))) & 0xFF, a1 = (cj[(t + u) / 4] >> (8 * (u & 3))) & 0xFF;
            const uint32_t at = (uint32_t)(q0 + t + u) * stride +
                                4u * (((a0 >> 4) * (ne.width >> 4) + (a1 >> 4)) * 256u + ((a0 & 15) >> 2) * 64u +
                                      (a1 & 15) * 4u + (a0 & 3));
            a[u] = __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(
                rsrc, (int)(a0 == 0xFF || a1 == 0xFF ? 0x80000000u : at), 0, 0));
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) s += (double)a[u];
    }
    part[grp][threadIdx.x & 31] = s;
    __syncthreads();
    if (grp == 0 && i <= j) {
        double tot = 0.0;
        for (int g = 0; g < kRedGroups; ++g) tot += part[g][threadIdx.x & 31];
        gram[i * PP + j] = tot;
        gram[j * PP + i] = tot;
        if (fe >= 0) {
            // as the dense solve sets up its matrix: a joint with no weight
            // (zero diagonal: its whole row is zero) or masked inactive is
            // frozen to an identity row with a zero right-hand side
            double v;
            if (j == P) v = act_i ? tot + prior_i * theta_i : 0.0;
            else if (i == j) v = (tot + prior_i == 0.0 || !act_i) ? 1.0 : (tot + prior_i) * (1.0 + (double)S.lambda_k);
            else v = (act_i && act_j) ? tot : 0.0;
            S.tree.fimg[fe] = v;
        }
    }
}

void launch_gram_reduce(const Launch& L) {
    launch_kernel(L, true, true, k_gram_reduce, dim3(L.grid[KK_REDUCE]), dim3(32 * kRedGroups), 0, L.B.slots, L.B.pre, L.B.n);
}

}  // namespace trk
