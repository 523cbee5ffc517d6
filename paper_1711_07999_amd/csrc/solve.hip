// Pose step (Section 4.2) and per-vertex offset step (Section 4.3).
#include "common.h"
#include "dq.h"
#include "fk.h"
#include "surface.h"

namespace trk {

// ---------------------------------------------------------------------------
// Damped least squares (Marquardt): (A + lambda_k diag(A)) x = b with
// A = J^T J + (lambda_s S)^2 and b = J^T r + (lambda_s S)^2 Theta, solved by
// Cholesky; Theta <- Theta - x.  Parameters with A_kk == 0 (no observed vertex
// moves them) or marked inactive are frozen (x_k = 0).  A failed
// factorisation leaves Theta unchanged and flags the frame.
//
// One workgroup per stream.  The damped matrix (padded with identity rows to
// a multiple of 16) sits in LDS with b appended as an extra row, and is
// factored left-looking in 16-column panels: all four waves first subtract
// the contribution of the finished panels from the new one (dot products out
// of LDS), then wave 0 factors the panel in registers -- one row per lane,
// columns broadcast between lanes with readlane, so the column-to-column
// chain has no barrier.  The appended row becomes y = L^-1 b on the way
// (forward substitution for free).  Back substitution runs panel by panel in
// wave 0; the same workgroup then runs forward kinematics at the new pose.
// ---------------------------------------------------------------------------
constexpr int kPanel = 16;
constexpr int kNMax = kMaxJoints + 1;   // 128
static_assert(4 * kMaxJoints <= kSolveThreads, "forward kinematics takes four threads a joint");

// Dynamic LDS of the solve for padded size n (row stride n + 4, so rows are
// 16-byte aligned for vector access): the matrix with the right-hand-side
// row (reused for forward kinematics afterwards), x, 1 / L_jj, the frozen
// flags and the failure flag.
template <class T>
__host__ __device__ inline size_t solve_lds_bytes(int n) {
    size_t mat = sizeof(T) * (size_t)(n + 1) * (n + 4);
    if (mat < sizeof(FkScratch)) mat = sizeof(FkScratch);
    mat = (mat + 15) & ~size_t(15);
    return mat + 2 * sizeof(T) * n + sizeof(int) * (n + 1);
}

// 1/sqrt(d): the hardware estimate for float (1 ulp), IEEE for double
__device__ __forceinline__ float rsqrt_of(float d) { return __builtin_amdgcn_rsqf(d); }
__device__ __forceinline__ double rsqrt_of(double d) { return 1.0 / sqrt(d); }

// four consecutive elements from 16-byte aligned LDS
__device__ __forceinline__ void load4(const float* p, float* o) {
    const float4 v = *reinterpret_cast<const float4*>(p);
    o[0] = v.x; o[1] = v.y; o[2] = v.z; o[3] = v.w;
}
__device__ __forceinline__ void load4(const double* p, double* o) {
    const double2 a = *reinterpret_cast<const double2*>(p);
    const double2 b = *reinterpret_cast<const double2*>(p + 2);
    o[0] = a.x; o[1] = a.y; o[2] = b.x; o[3] = b.y;
}

__device__ __forceinline__ float lane_bcast(float v, int lane) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}
__device__ __forceinline__ double lane_bcast(double v, int lane) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffll), lane);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

__device__ __forceinline__ void store4(float* p, const float* v) {
    *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
}
__device__ __forceinline__ void store4(double* p, const double* v) {
    *reinterpret_cast<double2*>(p) = make_double2(v[0], v[1]);
    *reinterpret_cast<double2*>(p + 2) = make_double2(v[2], v[3]);
}

constexpr size_t kSmallLds = 64 * 1024;

// BIG: an instance allowed more than 64 KB of LDS (P > 112 in float64); a
// kernel allowed that much is launched more slowly, so sizes below use the
// other instance
template <class T, bool BIG>
__global__ void __launch_bounds__(256) k_pose_solve(const Slot* __restrict__ bs, const int* __restrict__ bp, int bn, int iter, int nmax) {
    const Batch B{bs, bp, bn};
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int ld = nmax + 4;   // row stride shared by the batch
    size_t mat = sizeof(T) * (size_t)(nmax + 1) * ld;
    if (mat < sizeof(FkScratch)) mat = sizeof(FkScratch);
    mat = (mat + 15) & ~size_t(15);
    T* M = reinterpret_cast<T*>(smem);
    FkScratch& fk_ws = *reinterpret_cast<FkScratch*>(smem);
    T* sx = reinterpret_cast<T*>(smem + mat);
    T* sdinv = sx + nmax;
    int* sfrozen = reinterpret_cast<int*>(sdinv + nmax);
    int& sfail = sfrozen[nmax];
    int local;
    const Slot& S = B.slots[slot_of(B, KK_ONE, blockIdx.x, local)];
    const JointTable* __restrict__ jt = S.jt;
    const int PP = S.PP;
    const double* __restrict__ gram = S.gram;
    const float lambda_k = S.lambda_k;
    double* __restrict__ theta = S.theta;
    DevStats* st = S.st;
    const int P = S.m.P;   // (the table's copy: no dependent load through jt)
    const int n = (P + kPanel - 1) / kPanel * kPanel;
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;

    // Every global read of the set-up is issued before any is used: the
    // strictly lower triangle (a quarter-wave per row, four rows at a time)
    // and, per parameter, its diagonal, right-hand side, prior and flags.
    const int q = tid & 15, row0 = tid >> 4;
    constexpr int kRows = 4;
    T raw[2][kRows][kNMax / 16];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int a = 0; a < kRows; ++a) {
            const int r = row0 + 16 * (kRows * h + a);
#pragma unroll
            for (int u = 0; u < kNMax / 16; ++u) {
                const int c = q + 16 * u;
                raw[h][a][u] = (r < P && c < r) ? T(gram[r * PP + c]) : T(0);
            }
        }
    double gkk = 0.0, gkb = 0.0, prk = 0.0, thk = 0.0;
    int actk = 0;
    if (tid < P) {
        gkk = gram[tid * PP + tid];
        gkb = gram[tid * PP + P];
        prk = jt->prior[tid];
        thk = theta[tid];
        actk = jt->active[tid];
    }
    if (tid == 0) sfail = 0;
    if (tid < n) {
        const int fz = tid >= P || (gkk + prk == 0.0) || !actk;
        sfrozen[tid] = fz;
        M[n * ld + tid] = fz ? T(0) : T(gkb + prk * thk);
        M[tid * ld + tid] = fz ? T(1) : T((gkk + prk) * (1.0 + (double)lambda_k));
    }
    __syncthreads();
    // the damped, frozen and padded matrix (lower triangle)
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int a = 0; a < kRows; ++a) {
            const int r = row0 + 16 * (kRows * h + a);
            if (r >= n) continue;
            const bool fr = sfrozen[r] != 0;
#pragma unroll
            for (int u = 0; u < kNMax / 16; ++u) {
                const int c = q + 16 * u;
                if (c < r) M[r * ld + c] = (fr || sfrozen[c]) ? T(0) : raw[h][a][u];
            }
        }
    __syncthreads();

    for (int c0 = 0; c0 < n; c0 += kPanel) {
        // (1) A[r][c] -= sum_{k < c0} L[r][k] L[c][k] for the panel's columns,
        //     rows c0..n (row n: b -> y)
        if (c0 > 0) {
            const int rows = n + 1 - c0;
            for (int e = tid; e < rows * kPanel; e += 256) {
                const int r = c0 + e / kPanel, c = c0 + (e & (kPanel - 1));
                if (c > r) continue;
                const T* Lr = M + r * ld;
                const T* Lc = M + c * ld;
                T acc[4] = {T(0), T(0), T(0), T(0)};
                for (int k = 0; k < c0; k += 4) {
                    T xr[4], xc[4];
                    load4(Lr + k, xr);
                    load4(Lc + k, xc);
#pragma unroll
                    for (int t = 0; t < 4; ++t) acc[t] += xr[t] * xc[t];
                }
                M[r * ld + c] -= (acc[0] + acc[1]) + (acc[2] + acc[3]);
            }
            __syncthreads();
        }
        // (2) factor the panel in wave 0: lane l holds rows c0 + l and
        //     c0 + 64 + l; every lane carries the right-hand-side row
        if (wid == 0) {
            const int r0 = c0 + lane, r1 = c0 + 64 + lane;
            const bool h0 = r0 < n, h1 = r1 < n;
            T a0[kPanel], a1[kPanel], ab[kPanel];
#pragma unroll
            for (int j = 0; j < kPanel; j += 4) {
                if (h0) load4(M + r0 * ld + c0 + j, a0 + j);
                else a0[j] = a0[j + 1] = a0[j + 2] = a0[j + 3] = T(0);
                if (h1) load4(M + r1 * ld + c0 + j, a1 + j);
                else a1[j] = a1[j + 1] = a1[j + 2] = a1[j + 3] = T(0);
                load4(M + n * ld + c0 + j, ab + j);
            }
            const bool two = c0 + 64 < n;   // the second row set holds rows
            bool ok = true;
#pragma unroll
            for (int j = 0; j < kPanel; ++j) {
                const T d = lane_bcast(a0[j], j);
                ok = ok && (d > T(0));
                const T inv = ok ? rsqrt_of(d) : T(1);
                // column j of L: the diagonal, then the rows below it; y_j.
                // Lanes at or above the diagonal keep their (unused) entries.
                const T lj = lane > j ? a0[j] * inv : T(0);
                a0[j] = lane == j ? d * inv : (lane > j ? lj : a0[j]);
                a1[j] *= inv;
                ab[j] *= inv;
                if (lane == 0) sdinv[c0 + j] = inv;
                if (two) {
#pragma unroll
                    for (int c = j + 1; c < kPanel; ++c) {
                        const T lcj = lane_bcast(lj, c);
                        a0[c] -= lj * lcj;
                        a1[c] -= a1[j] * lcj;
                        ab[c] -= ab[j] * lcj;
                    }
                } else {
#pragma unroll
                    for (int c = j + 1; c < kPanel; ++c) {
                        const T lcj = lane_bcast(lj, c);
                        a0[c] -= lj * lcj;
                        ab[c] -= ab[j] * lcj;
                    }
                }
            }
#pragma unroll
            for (int j = 0; j < kPanel; ++j) {
                if (h0 && r0 >= c0 + j) M[r0 * ld + c0 + j] = a0[j];
                if (h1) M[r1 * ld + c0 + j] = a1[j];
                if (lane == 0) M[n * ld + c0 + j] = ab[j];
            }
            if (!ok && lane == 0) sfail = 1;
        }
        __syncthreads();
        if (sfail) break;
    }
    const bool fail = sfail != 0;
    if (!fail && wid == 0) {
        // back substitution L^T x = y, panel by panel from the last
        for (int c0 = n - kPanel; c0 >= 0; c0 -= kPanel) {
            // t_c = y_c - sum_{r >= c0 + 16} L[r][c] x_r for the panel's 16 columns:
            // lanes 16 g + l take rows r = c0 + 16 + g, +4, ...
            const int l = lane & (kPanel - 1), g = lane >> 4;
            T t = T(0);
            for (int r = c0 + kPanel + g; r < n; r += 4) t += M[r * ld + c0 + l] * sx[r];
            t += __shfl_xor(t, 16);
            t += __shfl_xor(t, 32);
            t = M[n * ld + c0 + l] - t;
            // upper-triangular 16x16 solve with L_pp^T in registers (column l)
            T lc[kPanel];
#pragma unroll
            for (int j = 0; j < kPanel; ++j) lc[j] = j >= l ? M[(c0 + j) * ld + c0 + l] : T(0);
#pragma unroll
            for (int j = kPanel - 1; j >= 0; --j) {
                const T xj = lane_bcast(t, j) * sdinv[c0 + j];
                t = l < j ? t - lc[j] * xj : (l == j ? xj : t);
            }
            if (lane < kPanel) sx[c0 + lane] = t;
            __builtin_amdgcn_wave_barrier();
        }
    }
    __syncthreads();
    if (!fail) {
        if (wid == 0) {
            double part = 0.0;
            for (int k = lane; k < P; k += 64) {
                const double x = sfrozen[k] ? 0.0 : (double)sx[k];
                S.step[k] = x;
                theta[k] -= x;
                part += x * x;
            }
            for (int o = 32; o > 0; o >>= 1) part += __shfl_xor(part, o);
            if (lane == 0) {
                st->step_norm[S.iter + iter] = (float)sqrt(part);
                st->energy[S.iter + iter] = (float)gram[P * PP + P];
            }
        }
    } else if (tid == 0) {
        st->status = -4;
        st->energy[S.iter + iter] = (float)gram[P * PP + P];
        st->step_norm[S.iter + iter] = 0.0f;
    }
    __syncthreads();
    fk_block(jt, P, S.m.L, theta, S.dq, S.xi, fk_ws);
}

// ---------------------------------------------------------------------------
// Tree form of the same solve.  J_ik vanishes unless joint k lies on the
// chain of a link weighting vertex i (Section 4.2), so A_kj vanishes unless
// some vertex's chains hold both joints: limbs do not touch each other, only
// their common ancestors.  Eliminated children first, the factor stays
// inside that pattern and its elimination tree follows the skeleton (the
// host plan, TreePlan).  Each supernode -- a chain of the elimination tree --
// owns a dense front: its pivot rows, the later rows they touch, and the
// right-hand side as one more row.  Level by level, all waves add the
// children's update blocks to the level's fronts (an entry per thread), then
// each wave takes its fronts, a row in two lanes' registers, and factors them
// (the right-hand-side row turns into y on the way, the rest of the front into
// the update block for the parent); 1 / L_jj goes into the front's spare last
// column.  Back substitution walks
// the levels downwards; a wave reads its next front's columns into registers
// while the levels above are solved.  Only structural zeros are skipped: the
// arithmetic per entry is that of the dense form.
//
// One workgroup, bound by the chain of dependent steps from the limbs' first
// pivot to the last round of forward kinematics: so no step of that chain
// goes through LDS that can do without (the next pivot's column takes its one
// multiplier by a lane broadcast, ahead of the others, which are read from LDS
// meanwhile; solutions are broadcast into scalar registers), and what waves
// wait for the others they use to read ahead.  75 joints (seven fronts on three levels), float32
// 18.5 -> 14.7 us, float64 (200 000 vertices, the same joints) 24.4 -> 19.4 us.
// ---------------------------------------------------------------------------
// Dynamic LDS of the tree form: the fronts (reused for forward kinematics),
// a copy of the plan, x, the waves' buffers (reused for the new pose and x^2),
// the failure flag.
template <class T>
__host__ __device__ inline size_t tree_front_bytes(int elems) {
    size_t mat = sizeof(T) * (size_t)elems;
    if (mat < sizeof(FkScratch)) mat = sizeof(FkScratch);
    return (mat + 15) & ~size_t(15);
}
template <class T>
__host__ __device__ inline size_t tree_lds_bytes(int elems, int words) {
    return tree_front_bytes<T>(elems) + 16 * (size_t)((words + 3) / 4) + sizeof(T) * kNMax +
           sizeof(T) * 64 * kSolveWaves + 16;
}

bool tree_solve_fits(int elems, int words) { return tree_lds_bytes<double>(elems, words) <= kSmallLds; }

// The value of lane l & 31 (a), and that of lane l | 32 (b), in every lane l.
__device__ __forceinline__ void halves(float v, float& a, float& b) {
    const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    a = __uint_as_float(h[0]);
    b = __uint_as_float(h[1]);
}
__device__ __forceinline__ void halves(double v, double& a, double& b) {
    const unsigned lo = (unsigned)__double2loint(v), hi = (unsigned)__double2hiint(v);
    const auto l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
    const auto h = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    a = __hiloint2double((int)h[0], (int)l[0]);
    b = __hiloint2double((int)h[1], (int)l[1]);
}

// A front as it is factored.  Lane i (< 32) holds the first 16 columns of row
// i that are left, lane 32 + i the next 16, the pivot column first; finished
// rows are carried along, unread.
template <class T>
struct FactorState {
    T* col;             // where the lane's entry of the next column of L goes
    int col_step;       // (both halves store it; rows past f where nothing is read)
    T* wb;              // the wave's buffer: a column's entries for the rows still to come from its
                        // start, the finished rows' in its second half, unread
    T first, inv;       // the pivot column (in both halves) and 1 / sqrt of the pivot
    T myinv, worst;     // 1 / L_ii of row i; -1 once a pivot was not positive
};

template <class T>
__device__ __forceinline__ void tree_pivot_ahead(FactorState<T>& s, T column, int row, int j) {
    const T d = lane_bcast(column, j);
    T other;
    halves(column, s.first, other);
    s.inv = rsqrt_of(d);
    s.myinv = row == j ? s.inv : s.myinv;
    s.worst = d > T(0) ? s.worst : T(-1);
}

// Pivot j, its broadcast and reciprocal root made by the step before: every
// lane reads its columns' multipliers from the buffer (wide broadcast reads)
// and every row moves one column to the left (from r into q).  The next
// pivot's own column is updated ahead of the others, by a lane broadcast, so
// that its root is on its way while the rest of this pivot's update waits for
// LDS.  HW: the columns of a lane that are still in use.  Nothing branches,
// and nothing but the pivots and multipliers crosses to the scalar unit.
template <class T, int HW>
__device__ __forceinline__ void tree_pivot(FactorState<T>& s, const T (&r)[16], T (&q)[16], int lane, int j) {
    const int row = lane & 31;
    const T lj = s.first * s.inv;   // L_jj = d / sqrt(d) in row j, y_j in the right-hand side's
    T other, across;   // the column that comes from the upper half
    halves(r[0], other, across);
    s.wb[(row - j - 1) & 63] = lj;
    T m[HW];
#pragma unroll
    for (int c = 0; c < HW; c += 4) load4(s.wb + (HW == 16 ? (lane & 32) / 2 : 0) + c, m + c);
    *s.col = lj;
    s.col += s.col_step;
    const T next = r[1] - lj * lane_bcast(lj, (j + 1) & 31);
    tree_pivot_ahead(s, next, row, (j + 1) & 31);
#pragma unroll
    for (int c = 0; c < HW - 1; ++c) q[c] = r[c + 1] - lj * m[c];
    q[HW - 1] = HW == 16 ? across - lj * m[HW - 1] : T(0);
}

// Factor the np pivots of a front of f rows (+ the right-hand-side row f),
// row-major with fw columns, fw > f.  Column j of L is stored as it is found,
// the update block (columns np..f-1 of rows np..f) at the end, and 1 / L_jj
// into the spare column fw - 1.
template <class T>
__device__ __forceinline__ void tree_factor(T* Fr, T* wb, int np, int f, int fw, int lane, bool& ok) {
    const int row = lane & 31, c16 = (lane & 32) / 2;
    T r[16], q[16];
    // (rows past f repeat it, columns past fw the last ones: unread)
    const T* mine = Fr + min(row, f) * fw;
#pragma unroll
    for (int c = 0; c < 16; c += 4) load4(mine + min(c16 + c, fw - 4), r + c);
    FactorState<T> s;
    s.col = row <= f ? Fr + row * fw : wb + 63;
    s.col_step = row <= f ? 1 : 0;
    s.wb = wb;
    s.myinv = T(0);
    s.worst = T(1);
    tree_pivot_ahead(s, r[0], row, 0);
    // two pivots a trip: the rows move from one set of registers to the other
    // and back
    int j = 0;
    const int je = min(np, f - 8);   // past the last pivot with more than 8 columns left
    T worst = s.worst;
    while (j < je) {
        worst = s.worst;
        tree_pivot<T, 16>(s, r, q, lane, j);
        ++j;
        if (j < je) {
            worst = s.worst;
            tree_pivot<T, 16>(s, q, r, lane, j);
            ++j;
        } else {
#pragma unroll
            for (int c = 0; c < 16; ++c) r[c] = q[c];
        }
    }
    while (j < np) {
        worst = s.worst;
        tree_pivot<T, 8>(s, r, q, lane, j);
        ++j;
        if (j < np) {
            worst = s.worst;
            tree_pivot<T, 8>(s, q, r, lane, j);
            ++j;
        } else {
#pragma unroll
            for (int c = 0; c < 8; ++c) r[c] = q[c];
        }
    }
    const int nU = f - np;
    T* const out = Fr + row * fw + np + c16;
    const int left = row >= np && row <= f ? nU - c16 : 0;   // the lane's columns of the update block
#pragma unroll
    for (int c = 0; c < 16; ++c) *(c < left ? out + c : wb + 63) = r[c];
    if (lane < np) Fr[lane * fw + fw - 1] = s.myinv;
    ok = ok && !__any(worst < T(0));   // (the look ahead past the last pivot does not count)
}

// What a wave holds of a front for its back substitution, lane c < np of
// pivot c: column c of L below the diagonal (zero above and past np, so that
// what a finished lane or a step past the last pivot does leaves t as it is),
// its first later rows (zero past nU), 1 / L_cc, y_c and its joint; lane k
// the joint of later row k.
constexpr int kBackLater = 16;
template <class T>
struct BackRegs {
    T col[kFrontRows], later[kBackLater], dinv, y;
    int joint, later_joint;
};

template <class T>
__device__ __forceinline__ void tree_back_load(BackRegs<T>& b, const T* Fr, const FrontRec& F, const unsigned char* row,
                                               int lane) {
    const int np = F.np, f = F.f, fw = F.fw, nU = f - np;
    const int cl = lane < np ? lane : 0;
    b.joint = row[cl];
    b.later_joint = row[lane < nU ? np + lane : 0];
    b.dinv = Fr[cl * fw + fw - 1];
    b.y = Fr[f * fw + cl];
    // eight rows at a time (row f again past it: unused)
    const unsigned below = lane < np ? (unsigned)(np - lane - 1) : 0u;   // rows of the pivots' triangle
    const T* at = Fr + cl;
#pragma unroll
    for (int k0 = 0; k0 < kFrontRows; k0 += 8)
        if (k0 < np) {
            T v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) { v[k] = *at; at += k0 + k < f ? fw : 0; }
#pragma unroll
            for (int k = 0; k < 8; ++k) b.col[k0 + k] = (unsigned)(k0 + k - lane - 1) < below ? v[k] : T(0);
        }
    at = Fr + np * fw + cl;
#pragma unroll
    for (int k0 = 0; k0 < kBackLater; k0 += 8)
        if (k0 < nU) {
            T v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) { v[k] = *at; at += np + k0 + k < f ? fw : 0; }
#pragma unroll
            for (int k = 0; k < 8; ++k) b.later[k0 + k] = k0 + k < nU ? v[k] : T(0);
        }
}

// L^T x = y for the front's pivots, given x of its later rows.  Without
// branches inside a run of eight steps: the code is run once a launch, and a
// jump to instructions that are not there yet costs more than a few steps
// with zeros.
template <class T>
__device__ __forceinline__ void tree_back(const BackRegs<T>& b, const T* Fr, const FrontRec& F, T* sx, int lane) {
    const int np = F.np, fw = F.fw, nU = F.f - np;
    T t = b.y;
    if (nU > 0) {
        const T xk = sx[b.later_joint];
        const T xl = lane < nU ? xk : T(0);   // x of later row k in lane k
        // four independent partial sums, the rows past the last whole four
        // into the first
        T t1 = T(0), t2 = T(0), t3 = T(0);
#pragma unroll
        for (int k0 = 0; k0 < kBackLater; k0 += 8)
            if (k0 < nU) {
#pragma unroll
                for (int k = k0; k < k0 + 8; k += 4) {
                    const bool whole = k + 4 <= nU;
                    const T x0 = lane_bcast(xl, k), x1 = lane_bcast(xl, k + 1), x2 = lane_bcast(xl, k + 2),
                            x3 = lane_bcast(xl, k + 3);
                    t -= b.later[k] * x0;
                    t -= (whole ? T(0) : b.later[k + 1]) * x1;
                    t -= (whole ? T(0) : b.later[k + 2]) * x2;
                    t1 -= (whole ? b.later[k + 1] : T(0)) * x1;
                    t2 -= (whole ? b.later[k + 2] : T(0)) * x2;
                    t3 -= b.later[k + 3] * x3;   // zero where the four are not whole
                }
            }
        const int cl = lane < np ? lane : 0;
        int k = kBackLater;
        for (; k + 4 <= nU; k += 4) {
            const T* R = Fr + (np + k) * fw + cl;
            t -= R[0] * lane_bcast(xl, k);
            t1 -= R[fw] * lane_bcast(xl, k + 1);
            t2 -= R[2 * fw] * lane_bcast(xl, k + 2);
            t3 -= R[3 * fw] * lane_bcast(xl, k + 3);
        }
        for (; k < nU; ++k) t -= Fr[(np + k) * fw + cl] * lane_bcast(xl, k);
        t = (t + t1) + (t2 + t3);
    }
    // the pivots' own triangle, last pivot first
#pragma unroll
    for (int j0 = kFrontRows - 8; j0 >= 0; j0 -= 8)
        if (j0 < np) {
#pragma unroll
            for (int j = j0 + 7; j >= j0; --j) {
                const T xj = lane_bcast(t * b.dinv, j);
                t -= b.col[j] * xj;
            }
        }
    if (lane < np) sx[b.joint] = t * b.dinv;
}

template <class T>
__global__ void __launch_bounds__(kSolveThreads) k_pose_solve_tree(const Slot* __restrict__ bs, int elems_max, int words_max, int iter) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const size_t mat = tree_front_bytes<T>(elems_max);
    T* Fs = reinterpret_cast<T*>(smem);
    FkScratch& fk_ws = *reinterpret_cast<FkScratch*>(smem);
    uint32_t* lb = reinterpret_cast<uint32_t*>(smem + mat);   // the plan's blob, copied to LDS
    T* sx = reinterpret_cast<T*>(smem + mat + 16 * (size_t)((words_max + 3) / 4));
    T* wbase = sx + kNMax;
    static_assert(sizeof(T) * 64 * kSolveWaves >= sizeof(double) * 2 * kNMax, "the new pose and x^2 fit the waves' buffers");
    double* sth = reinterpret_cast<double*>(wbase);            // the new pose (the factorisation done)
    double* spart = sth + kNMax;                               // x^2
    int& sfail = *reinterpret_cast<int*>(wbase + 64 * kSolveWaves);
    const Slot& S = bs[blockIdx.x];   // one workgroup per slot
    const TreeRef& tr = S.tree;
    const int P = S.m.P, NL = S.m.L, elems = tr.elems, nwords = tr.nwords;
    const JointTable* __restrict__ jt = S.jt;
    double* __restrict__ theta = S.theta;
    const int tid = threadIdx.x, lane = tid & 63, wid = wave_uniform(tid >> 6);
    T* wb = wbase + 64 * wid;   // this wave's broadcast buffer

    // set-up: every global read is issued before any is used -- the fronts'
    // starting image (from the Gram reduction), the plan, and per joint the
    // pose and whether it is frozen
    // (elems is even: rows are multiples of 8 wide)
    const double2* __restrict__ img = reinterpret_cast<const double2*>(tr.fimg);
    // (unconditional loads at clamped indices, the unused ones dropped after:
    // a load under a condition is waited for inside it, one after another)
    constexpr int kPre = 8;
    double2 iv[kPre];
#pragma unroll
    for (int k = 0; k < kPre; ++k) iv[k] = img[min(tid + kSolveThreads * k, elems / 2 - 1)];
    const uint4* __restrict__ bsrc = reinterpret_cast<const uint4*>(tr.blob);
    const int nw4 = (nwords + 3) / 4;
    const uint4 bw = bsrc[min(tid, nw4 - 1)];
    const int tp = min(tid, P - 1);
    const double th0 = theta[tp], prior = jt->prior[tp];
    const int act = jt->active[tp];
    const int rounds = wave_uniform(jt->rounds);
    // forward kinematics' constants, needed last
    FkJoint fj;
    FkLink fl;
    fk_prefetch(jt, P, NL, fj, fl);
    // (waited for much later)
    const int PP = S.PP;
    const double* __restrict__ gram = S.gram;
    DevStats* const st = S.st;
    const double gdiag = ldg(gram + tp * PP + tp), energy = ldg(gram + P * PP + P);
    const double thk = tid < P ? th0 : 0.0;
#pragma unroll
    for (int k = 0; k < kPre; ++k) {
        const int e = tid + kSolveThreads * k;
        if (2 * e < elems) {
            Fs[2 * e] = T(iv[k].x);
            Fs[2 * e + 1] = T(iv[k].y);
        }
    }
    for (int e = tid + kSolveThreads * kPre; 2 * e < elems; e += kSolveThreads) {
        const double2 v = img[e];
        Fs[2 * e] = T(v.x);
        Fs[2 * e + 1] = T(v.y);
    }
    if (tid < nw4) reinterpret_cast<uint4*>(lb)[tid] = bw;
    for (int i = tid + kSolveThreads; i < nw4; i += kSolveThreads) reinterpret_cast<uint4*>(lb)[i] = bsrc[i];
    if (tid == 0) sfail = 0;
    __syncthreads();

    // factor, level by level
    const int nlev = wave_uniform(tr.nlev);
    const int* wstart = reinterpret_cast<const int*>(lb);
    const AsmRec* levels = reinterpret_cast<const AsmRec*>(lb + tr.o_lev);
    const FrontRec* fronts = reinterpret_cast<const FrontRec*>(lb + tr.o_front);
    const unsigned char* lbytes = reinterpret_cast<const unsigned char*>(lb);
    // this wave's fronts on level l (lane l): the first one and how many; a
    // plan has at most 64 levels
    const int wl = min(lane, nlev - 1) * kSolveWaves + wid;
    const int wfirst = wstart[wl], wcount = lane < nlev ? wstart[wl + 1] - wfirst : 0;
    const unsigned long long my_levels = __ballot(wcount > 0);
    auto front = [&](int q) {   // (read from LDS: the same for the whole wave)
        FrontRec F = fronts[q];
        F.off = wave_uniform(F.off); F.np = wave_uniform(F.np); F.f = wave_uniform(F.f);
        F.fw = wave_uniform(F.fw); F.row0 = wave_uniform(F.row0);
        return F;
    };
    // the record of the wave's next front and the level's assembly entry of
    // this thread are read before the level is reached; what the back
    // substitution needs of a finished front (`back`, of front G on level
    // `next`) while higher levels are factored
    int level = my_levels ? __builtin_ctzll(my_levels) : nlev, next = -1, q = 0, q1 = 0;
    FrontRec F = front(level < nlev ? __builtin_amdgcn_readlane(wfirst, level) : 0), G = F;
    BackRegs<T> back;
    bool held = true;   // `back` is G's
    auto hold = [&]() {
        tree_back_load<T>(back, Fs + G.off, G, lbytes + G.row0, lane);
        held = true;
    };
    bool ok = true;
    for (int l = 0; l < nlev; ++l) {
        // the children's update blocks: an entry of a front per thread, its
        // shares in child order
        const AsmRec A = levels[l];
        const int an = wave_uniform(A.n), an1 = wave_uniform(A.n1), aw = wave_uniform(A.words);
        const uint32_t* m = lb + A.map0;
        uint32_t w0 = 0u, w1 = 0xFFFFFFFFu;
        if (tid < an) w0 = m[tid];
        if (tid < an1) w1 = m[an + tid];
        if (l > 0) __syncthreads();   // the level below is done
        for (int e = tid; e < an; e += kSolveThreads) {
            if (e != tid) {
                w0 = m[e];
                w1 = e < an1 ? m[an + e] : 0xFFFFFFFFu;
            }
            const uint32_t dst = w0 & 0xFFFFu;
            uint32_t s1 = w1 & 0xFFFFu, s2 = w1 >> 16;
            T v = Fs[dst];
            const T v0 = Fs[w0 >> 16], v1 = Fs[s1 == 0xFFFFu ? dst : s1], v2 = Fs[s2 == 0xFFFFu ? dst : s2];
            v += v0;
            v = s1 == 0xFFFFu ? v : v + v1;
            v = s2 == 0xFFFFu ? v : v + v2;
            for (int k = 2, at = an + an1; k < aw; ++k) {
                const int nk = (int)m[k - aw];   // entries of more than k words: the first ones
                if (e < nk) {
                    const uint32_t w = m[at + e];
                    s1 = w & 0xFFFFu;
                    s2 = w >> 16;
                    v += Fs[s1];
                    if (s2 != 0xFFFFu) v += Fs[s2];
                }
                at += nk;
            }
            Fs[dst] = v;
        }
        if (l > 0) __syncthreads();
        if (l == level) {
            next = l;
            q = __builtin_amdgcn_readlane(wfirst, l);
            q1 = q + __builtin_amdgcn_readlane(wcount, l);
            G = F;
            held = false;
            tree_factor<T>(Fs + F.off, wb, F.np, F.f, F.fw, lane, ok);
            for (int k = q + 1; k < q1; ++k) {
                F = front(k);
                tree_factor<T>(Fs + F.off, wb, F.np, F.f, F.fw, lane, ok);
            }
            const unsigned long long above = l < 63 ? my_levels >> (l + 1) : 0ull;
            if (above) {
                level = l + 1 + __builtin_ctzll(above);
                F = front(__builtin_amdgcn_readlane(wfirst, level));
            }
        } else if (sizeof(T) == 4 && !held) {   // (float64: not the registers for it)
            hold();
        }
    }
    if (!held) hold();
    if (!ok && lane == 0) sfail = 1;
    __syncthreads();
    const bool fail = sfail != 0;
    if (!fail) {
        unsigned long long left = next >= 0 ? my_levels & ~(1ull << next) : 0ull;
        for (int l = nlev - 1; l >= 0; --l) {
            while (next == l) {
                tree_back<T>(back, Fs + G.off, G, sx, lane);
                if (++q >= q1) {
                    next = left ? 63 - __builtin_clzll(left) : -1;
                    if (next < 0) break;
                    left &= ~(1ull << next);
                    q = __builtin_amdgcn_readlane(wfirst, next);
                    q1 = q + __builtin_amdgcn_readlane(wcount, next);
                }
                G = front(q);
                hold();
            }
            __syncthreads();
        }
    }
    // the step: Theta <- Theta - x (frozen parameters keep their value)
    const bool frozen = tid >= P || gdiag + prior == 0.0 || !act;
    const double x = (!fail && !frozen) ? (double)sx[tid] : 0.0;
    if (tid < P) {
        const double th = thk - x;
        sth[tid] = th;
        if (!fail) {
            stg(S.step + tid, x);
            stg(theta + tid, th);
        }
    }
    if (tid < kNMax) spart[tid] = x * x;   // (zero past P)
    __syncthreads();
    fk_block_pre(jt, P, NL, rounds, sth, fj, fl, S.dq, S.xi, fk_ws);
    if (wid == 5) {
        // the step's norm, by a wave that forward kinematics leaves idle for
        // up to 80 joints
        double norm2 = 0.0;
        for (int k = 0; k < kNMax; k += 64) {
            double part = spart[k + lane];
            for (int o = 32; o > 0; o >>= 1) part += __shfl_xor(part, o);
            norm2 += part;
        }
        if (lane == 0) {
            st->energy[S.iter + iter] = (float)energy;
            st->step_norm[S.iter + iter] = fail ? 0.0f : (float)sqrt(norm2);
            if (fail) st->status = -4;
        }
    }
}

// let the BIG instances take the largest system (P = 127, float64: about
// 136 KB of LDS)
bool prepare_pose_solve() {
    bool ok = hipFuncSetAttribute(reinterpret_cast<const void*>(k_pose_solve<double, true>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize,
                                  (int)solve_lds_bytes<double>(kNMax)) == hipSuccess;
    ok = hipFuncSetAttribute(reinterpret_cast<const void*>(k_pose_solve<float, true>),
                             hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)solve_lds_bytes<float>(kNMax)) == hipSuccess && ok;
    return ok;
}

template <class T>
void launch_pose_solve_t(const Launch& L, int iter) {
    if (L.solve_elems > 0) {
        const size_t bytes = tree_lds_bytes<T>(L.solve_elems, L.solve_words);
        launch_kernel(L, true, true, k_pose_solve_tree<T>, dim3(L.grid[KK_ONE]), dim3(kSolveThreads), bytes, L.B.slots,
                      L.solve_elems, L.solve_words, iter);
        return;
    }
    const int n = L.solve_n;
    const size_t bytes = solve_lds_bytes<T>(n);
    if (bytes <= kSmallLds)
        launch_kernel(L, true, true, k_pose_solve<T, false>, dim3(L.grid[KK_ONE]), dim3(256), bytes, L.B.slots, L.B.pre, L.B.n, iter, n);
    else
        launch_kernel(L, true, true, k_pose_solve<T, true>, dim3(L.grid[KK_ONE]), dim3(256), bytes, L.B.slots, L.B.pre, L.B.n, iter, n);
}

void launch_pose_solve(const Launch& L, int fp64, int iter) {
    if (fp64) launch_pose_solve_t<double>(L, iter);
    else launch_pose_solve_t<float>(L, iter);
}

// ---------------------------------------------------------------------------
// Per-vertex offset step (reading of Eq. 9 as a sum of squared residuals with
// the neighbours held fixed, the independence approximation of Section 4.3):
//   u_i = -R_i^T n_i (0 if unobserved),  r_i = n_i . delta_i,
//   g_i = u_i r_i + lam_phi phi_i + lam_N sum_n (phi_i - phi_n)
//         + lam_T (phi_i - phi_i^prev),
//   A_i = u_i u_i^T + (lam_phi + lam_N |N(i)| + lam_T) I,
//   (A_i + lam_w diag A_i) x_i = g_i,  phi_i <- phi_i - x_i,
// with delta_i = (sum of p - v at association) / c_i + (v_old - v_new) after
// a pose step.  One vertex per lane; the 3x3 solve in float32 or float64.
// ---------------------------------------------------------------------------
template <class T>
__device__ __forceinline__ void solve3(const T M[9], const T g[3], T x[3]) {
    const T c00 = det2(M[4], M[8], M[5], M[7]), c01 = det2(M[5], M[6], M[3], M[8]), c02 = det2(M[3], M[7], M[4], M[6]);
    const T det = dot3(M[0], c00, M[1], c01, M[2], c02);
    if (!(fabs(det) > T(0))) { x[0] = x[1] = x[2] = T(0); return; }
    const T i0[3] = {c00, det2(M[7], M[2], M[1], M[8]), det2(M[1], M[5], M[2], M[4])};
    const T i1[3] = {c01, det2(M[0], M[8], M[2], M[6]), det2(M[2], M[3], M[0], M[5])};
    const T i2[3] = {c02, det2(M[6], M[1], M[0], M[7]), det2(M[0], M[4], M[1], M[3])};
    x[0] = dot3(i0[0], g[0], i0[1], g[1], i0[2], g[2]) / det;
    x[1] = dot3(i1[0], g[0], i1[1], g[1], i1[2], g[2]) / det;
    x[2] = dot3(i2[0], g[0], i2[1], g[1], i2[2], g[2]) / det;
}

//
// SKIN: the surface at the new pose (v_new) is skinned here instead of by a
// launch of its own.  The step's normals need the neighbours' vertices: a wave
// skins its block of 64 vertices and the block's rim (about two rows of the
// mesh, 130 vertices) into LDS, unless none of its vertices is observed.
// Bound by the rounds of reads of one wave (the rim's vertices wait for its
// list); a launch of skinning, its gap and a pass over the surface go away.
// Skinning and this step apart against together: 50 000 vertices 5.6 + 9.0 ->
// 11.4 us, 2 000 4.8 + 6.6 -> 8.5 us; a pass of 32 streams of 50 000 14.5 ->
// 14.0 ms.  Meshes of longer rims (more than kRim vertices) keep them apart,
// and with them every stream of their launch: both forms give the same bits
// (each sum of products is written out, see dq.h), so a stream does not show
// which one it went through.
template <class T, int NT, bool SKIN>
__global__ void __launch_bounds__(NT) k_shape(const Slot* __restrict__ bs, const int* __restrict__ bp, int bn, int vo_sel, int vn_sel, int pn, int next, int bsel) {
    const Batch B{bs, bp, bn};
    __shared__ float sdq[8 * (kMaxLinks + 1)];
    __shared__ CountTable<NT> ct;
    __shared__ float4 spos[SKIN ? NT / 64 : 1][SKIN ? 64 + kRim : 1];
    int local;
    const Slot& S = B.slots[slot_of(B, kVertKind<NT>, blockIdx.x, local)];
    const DevModel& m = S.m;
    const float4* __restrict__ v_old = S.verts[S.v_cur ^ vo_sel];
    const float4* __restrict__ v_new = S.verts[S.v_cur ^ vn_sel];
    const Accum& a = S.a;
    const int src = phi_index(S, pn);
    const Vec3Buf phi = S.phi[src];
    const Vec3Buf phi_prev = S.phi[S.phi_prev];
    const Vec3Buf phi_out = S.phi[phi_next(src, S.phi_prev)];
    const float lphi = S.lphi, lnbr = S.lnbr, lt = S.lt, lw = S.lw;
    const bool counted = selected(S, next);
    const CountRefs cr = count_refs(S, bsel);
    // the slot fields used after the first loads, read here (into scalar
    // registers) rather than each where it is used, behind its own wait
    const bool linear = wave_uniform(S.blend) == kBlendLinear;
    uint32_t* const acnt = wave_uniform(a.cnt);
    long long* const asx = wave_uniform(a.sx);
    long long* const asy = wave_uniform(a.sy);
    long long* const asz = wave_uniform(a.sz);
    float* const pox = wave_uniform(phi_out.x);
    float* const poy = wave_uniform(phi_out.y);
    float* const poz = wave_uniform(phi_out.z);
    float4* const vnext = wave_uniform(S.verts[S.v_cur ^ vn_sel ^ 1]);
    const int i = local * NT + threadIdx.x;
    const bool live = i < m.V;
    const int ii = live ? i : 0;   // lanes past the end read vertex 0 and store nothing
    // every per-vertex load that does not wait on another goes out first,
    // ahead of the link table's copy (global reads: the barrier does not wait
    // for them), so their latencies overlap the copy's and each other's
    const uint32_t c0 = ldg(a.cnt + ii);
    const float px0 = ldg(phi.x + ii), py0 = ldg(phi.y + ii), pz0 = ldg(phi.z + ii);
    const float qx0 = ldg(phi_prev.x + ii), qy0 = ldg(phi_prev.y + ii), qz0 = ldg(phi_prev.z + ii);
    const int4 nb = ldg(m.nbr + ii);
    const float4 vo = ldg_xyz(v_old + ii);
    float4 vn;
    // this wave's block and rim (a wave past the end: none)
    const int blk = wave_uniform(i >> 6), lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const bool some = SKIN && 64 * blk < m.V;
    uint32_t r0 = 0u, nrim = 0u, rim[3];
    if (SKIN) {
        if (some) {
            r0 = wave_uniform(ldg(m.rim_off + blk));
            nrim = wave_uniform(ldg(m.rim_off + blk + 1)) - r0;
        }
    } else {
        vn = ldg_xyz(v_new + ii);
    }
    const long long ax = ldg(a.sx + ii), ay = ldg(a.sy + ii), az = ldg(a.sz + ii);
    const float4 wv = ldg(m.w + ii);
    const uint32_t lk = ldg(m.links + ii);
    const float rx = ldg(m.rx + ii), ry = ldg(m.ry + ii), rz = ldg(m.rz + ii);
    FanIn fan;
    uint4 at;
    uint32_t e0, e1;
    if (SKIN) {
        at = ldg(m.fan_at + ii);
        e0 = ldg(m.rest_off + ii);
        e1 = ldg(m.rest_off + ii + 1);
#pragma unroll
        for (int k = 0; k < 3; ++k) rim[k] = nrim ? ldg(m.rim + r0 + min(64u * k + lane, nrim - 1u)) : 0u;
    } else {
        vertex_fan_load(m, v_new, i, live, fan);   // not waiting for the count
    }
    copy_to_lds(sdq, S.dq, 8 * m.L);
    if (counted) count_clear(ct);
    __syncthreads();
    if (!SKIN) vertex_fan_settle(fan, live);
    const uint32_t c = live ? c0 : 0u;
    const T px = px0, py = py0, pz = pz0;
    const T qx = qx0, qy = qy0, qz = qz0;
    const int nbs[4] = {nb.x, nb.y, nb.z, nb.w};
    T nphi[4][3];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int j = nbs[q] < 0 ? ii : nbs[q];
        nphi[q][0] = (T)ldg(phi.x + j); nphi[q][1] = (T)ldg(phi.y + j); nphi[q][2] = (T)ldg(phi.z + j);
    }
    float nx = 0.0f, ny = 0.0f, nz = 0.0f;
    if (SKIN) {
        float4* const pos = spos[wid];
        auto skin = [&](float4 w, uint32_t links, float x, float y, float z) {
            float4 o = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            if (linear) {
                lbs_apply(sdq, w, links, x, y, z, o.x, o.y, o.z);
            } else {
                float Hs[8];
                dq_blend(sdq, w, links, Hs);
                dq_apply(Hs, x, y, z, o.x, o.y, o.z);
            }
            return o;
        };
        vn = skin(wv, lk, rx + px0, ry + py0, rz + pz0);
        if (__ballot(c > 0u) != 0ull) {
            pos[lane] = vn;
            // (every read of the rim issued before the first is skinned)
            struct RimIn { float4 w; uint32_t links; float x, y, z, fx, fy, fz; } in[3];
#pragma unroll
            for (int k = 0; k < 3; ++k)
                if (64u * k < nrim) {   // the same for the whole wave
                    const uint32_t j = rim[k];
                    in[k].w = ldg(m.w + j);
                    in[k].links = ldg(m.links + j);
                    in[k].x = ldg(m.rx + j); in[k].y = ldg(m.ry + j); in[k].z = ldg(m.rz + j);
                    in[k].fx = ldg(phi.x + j); in[k].fy = ldg(phi.y + j); in[k].fz = ldg(phi.z + j);
                }
#pragma unroll
            for (int k = 0; k < 3; ++k)
                if (64u * k < nrim)
                    pos[64 + 64 * k + lane] = skin(in[k].w, in[k].links, in[k].x + in[k].fx, in[k].y + in[k].fy, in[k].z + in[k].fz);
            // (a wave's LDS accesses are in order)
            asm volatile("" ::: "memory");
            __builtin_amdgcn_wave_barrier();
            vertex_normal_rim(m, pos, at, e0, e1, c > 0u, nx, ny, nz);   // the whole wave
        }
        if (!counted && live) stg(const_cast<float4*>(v_new) + i, vn);
    } else {
        vertex_normal_fan(m, v_new, i, live && c > 0u, fan, nx, ny, nz);   // the whole wave
    }
    // lanes past the end go on with vertex 0's values (count 0) and store nothing
    T u[3] = {T(0), T(0), T(0)};
    T r = T(0);
    float H[8];
    if (!linear) dq_blend(sdq, wv, lk, H);
    if (c > 0u) {
        if ((nx * nx + ny * ny + nz * nz) > 0.0f) {
            // dr/dphi = -(dv/dx)^T n: the blend's rotation, or for the linear
            // blend the weighted sum of the links' rotations
            T R[9];
            if (!linear) {
                quat_matrix<T>(H, R);
            } else {
                const float ws[4] = {wv.x, wv.y, wv.z, wv.w};
                for (int q = 0; q < 9; ++q) R[q] = T(0);
                for (int k = 0; k < 4; ++k) {
                    const int l = (lk >> (8 * k)) & 0xFF;
                    if (l == 0xFF) continue;
                    T Rl[9];
                    quat_matrix<T>(sdq + 8 * l, Rl);
                    for (int q = 0; q < 9; ++q) R[q] = fma_of((T)ws[k], Rl[q], R[q]);
                }
            }
            for (int q = 0; q < 3; ++q) u[q] = -dot3(R[q], (T)nx, R[3 + q], (T)ny, R[6 + q], (T)nz);
            const T inv = T(1) / ((T)c * T(4294967296.0));
            const T dx = fma_of((T)ax, inv, (T)vo.x - (T)vn.x);
            const T dy = fma_of((T)ay, inv, (T)vo.y - (T)vn.y);
            const T dz = fma_of((T)az, inv, (T)vo.z - (T)vn.z);
            r = dot3((T)nx, dx, (T)ny, dy, (T)nz, dz);
        }
    }
    // this is the association's last reader: clear for the next one
    if (live) {
        stg(acnt + i, 0u);
        stg(asx + i, 0ll); stg(asy + i, 0ll); stg(asz + i, 0ll);
    }
    T alpha = (T)lphi + (T)lt;
    T g[3] = {dot3((T)lphi, px, u[0], r, (T)lt, px - qx),
              dot3((T)lphi, py, u[1], r, (T)lt, py - qy),
              dot3((T)lphi, pz, u[2], r, (T)lt, pz - qz)};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        if (nbs[q] < 0) continue;
        alpha += (T)lnbr;
        g[0] = fma_of((T)lnbr, px - nphi[q][0], g[0]);
        g[1] = fma_of((T)lnbr, py - nphi[q][1], g[1]);
        g[2] = fma_of((T)lnbr, pz - nphi[q][2], g[2]);
    }
    T M[9];
    for (int p = 0; p < 3; ++p)
        for (int q = p; q < 3; ++q) M[3 * p + q] = M[3 * q + p] = fma_of(u[p], u[q], p == q ? alpha : T(0));
    for (int p = 0; p < 3; ++p) M[4 * p] *= (T(1) + (T)lw);
    T xs[3];
    solve3(M, g, xs);
    const float fx = (float)(px - xs[0]), fy = (float)(py - xs[1]), fz = (float)(pz - xs[2]);
    if (live) {
        stg(pox + i, fx);
        stg(poy + i, fy);
        stg(poz + i, fz);
    }
    if (counted) {
        // the next iteration's surface: skin the new offsets (same blend) into
        // the buffer not read here by other vertices, and count it
        float ox, oy, oz;
        if (linear) lbs_apply(sdq, wv, lk, rx + fx, ry + fy, rz + fz, ox, oy, oz);
        else dq_apply(H, rx + fx, ry + fy, rz + fz, ox, oy, oz);
        const float4 q = make_float4(ox, oy, oz, 0.0f);
        if (live) stg(vnext + i, q);
        count_vertex(cr, i, q, live, false, ct);   // the whole workgroup
    }
}

void launch_shape(const Launch& L, int fp64, int v_old, int v_new, int pn, int next, int bsel, bool skin) {
    with_vert_threads(L, [&](auto nt) {
        constexpr int NT = decltype(nt)::value;
        const dim3 g(L.grid[kVertKind<NT>]);
        auto go = [&](auto k) { launch_kernel(L, true, true, k, g, dim3(NT), 0, L.B.slots, L.B.pre, L.B.n, v_old, v_new, pn, next, bsel); };
        if (skin) {
            constexpr int NS = NT < kSkinThreads ? NT : kSkinThreads;
            auto gs = [&](auto k) { launch_kernel(L, true, true, k, dim3(L.grid[kVertKind<NS>]), dim3(NS), 0, L.B.slots, L.B.pre, L.B.n, v_old, v_new, pn, next, bsel); };
            return fp64 ? gs(k_shape<double, NS, true>) : gs(k_shape<float, NS, true>);
        }
        fp64 ? go(k_shape<double, NT, false>) : go(k_shape<float, NT, false>);
    });
}

}  // namespace trk
