// Forward kinematics of one pose in one workgroup (Section 3.1), shared by
// the FK kernel and the pose-step kernel.
#pragma once
#include "common.h"
#include "dq.h"

namespace trk {

// ---------------------------------------------------------------------------
// Forward kinematics (Section 3.1) in float64, one workgroup.
//
// Each joint first forms its local transform O_j H_j(theta_j) (Eq. 1 or 2);
// the chain products H_{0,j} = H_{0,P(j)} O_j H_j are then formed by pointer
// jumping: every joint repeatedly left-multiplies by the product held at its
// current ancestor and jumps to that ancestor's ancestor, so a tree of depth
// D needs ceil(log2 D) rounds (jt->rounds) instead of D dependent steps.
//
// Outputs (float32): the link offsets H_{l,Delta} = H_{0,l} (H^0_{0,l})^{-1}
// (8 per link) and, per joint k, the world-frame generator
//   Xi_k = H_{0,k} (dH_k/dtheta H_k^{-1}) H_{0,k}^{-1},
// i.e. H_{0,k} (z/2) H_{0,k}^* for a hinge and H_{0,k} (eps z/2) H_{0,k}^* for
// a prismatic, stored as its 6 vector components (real xyz, dual xyz) + pad.
// dH_{l,Delta}/dtheta_k = Xi_k H_{l,Delta} for every joint k on the chain of
// link l (the derivative blocks of Section 4.2).
// ---------------------------------------------------------------------------
// LDS workspace of fk_block (callers provide it, so that a kernel can
// overlay it on memory it no longer needs)
struct FkScratch {
    double M[2][kMaxJoints + 1][8];   // (fk_block_pre: a quad's entry for each quad of the workgroup)
    int A[2][kMaxJoints + 1];
};

__device__ __forceinline__ void fk_block(const JointTable* __restrict__ jt, int P, int L,
                                         const double* __restrict__ theta, float* __restrict__ dq,
                                         float* __restrict__ xi, FkScratch& ws) {
    double (*M)[kMaxJoints + 1][8] = ws.M;
    int (*A)[kMaxJoints + 1] = ws.A;
    const int t = threadIdx.x;
    for (int j = t; j < P; j += blockDim.x) {
        double th = theta[j];
        double Hj[8] = {1, 0, 0, 0, 0, 0, 0, 0};
        const double* z = jt->axis[j];
        if (jt->type[j] == 0) {
            double s, c;
            sincos(0.5 * th, &s, &c);
            Hj[0] = c; Hj[1] = s * z[0]; Hj[2] = s * z[1]; Hj[3] = s * z[2];
        } else {
            Hj[5] = 0.5 * th * z[0]; Hj[6] = 0.5 * th * z[1]; Hj[7] = 0.5 * th * z[2];
        }
        double loc[8];
        dqmul(jt->off[j], Hj, loc);
        for (int c = 0; c < 8; ++c) M[0][j][c] = loc[c];
        A[0][j] = jt->parent[j];
    }
    __syncthreads();
    int cur = 0;
    for (int round = 0; round < jt->rounds; ++round) {
        int nxt = cur ^ 1;
        for (int j = t; j < P; j += blockDim.x) {
            int a = A[cur][j];
            if (a >= 0) {
                double o[8];
                dqmul(M[cur][a], M[cur][j], o);
                for (int c = 0; c < 8; ++c) M[nxt][j][c] = o[c];
                A[nxt][j] = A[cur][a];
            } else {
                for (int c = 0; c < 8; ++c) M[nxt][j][c] = M[cur][j][c];
                A[nxt][j] = -1;
            }
        }
        __syncthreads();
        cur = nxt;
    }
    for (int j = t; j < P; j += blockDim.x) {
        const double* H = M[cur][j];
        double g[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        const double* z = jt->axis[j];
        if (jt->type[j] == 0) { g[1] = 0.5 * z[0]; g[2] = 0.5 * z[1]; g[3] = 0.5 * z[2]; }
        else { g[5] = 0.5 * z[0]; g[6] = 0.5 * z[1]; g[7] = 0.5 * z[2]; }
        double hc[8], tmp[8], o[8];
        dqconj(H, hc);
        dqmul(H, g, tmp);
        dqmul(tmp, hc, o);
        float* dst = xi + 8 * j;
        dst[0] = (float)o[1]; dst[1] = (float)o[2]; dst[2] = (float)o[3];
        dst[3] = (float)o[5]; dst[4] = (float)o[6]; dst[5] = (float)o[7];
        dst[6] = 0.0f; dst[7] = 0.0f;
    }
    for (int l = t; l < L; l += blockDim.x) {
        double o[8];
        dqmul(M[cur][jt->link_joint[l]], jt->binv[l], o);
        for (int c = 0; c < 8; ++c) dq[8 * l + c] = (float)o[c];
    }
}

// The same forward kinematics by four lanes a joint (or link): lane c of the
// quad holds component c of the real and of the dual part.  A product's
// operands go round the quad in registers, so of a round of pointer jumping
// only the ancestor's product comes from LDS (one 16-byte read a lane).  The
// constants are read ahead of time (a kernel issues fk_prefetch early, so the
// reads overlap other work), the pose comes from LDS.  Joint j's quad is
// threads 4 j .. 4 j + 3 (the workgroup has at least 4 P threads); the links
// go to the quads from the last one on, which the joints mostly leave idle.
// The rounds do not branch: a quad past the joints, or done, goes through
// the motions.
struct FkJoint { double r, d, z; int type, parent; };   // z: the axis's component c - 1
struct FkLink { double r, d; int joint; };

__device__ __forceinline__ void fk_link_load(const JointTable* __restrict__ jt, int l, FkLink& fl) {
    const int c = threadIdx.x & 3;
    fl.r = ldg(&jt->binv[l][c]);
    fl.d = ldg(&jt->binv[l][4 + c]);
    fl.joint = ldg(&jt->link_joint[l]);
}

__device__ __forceinline__ void fk_prefetch(const JointTable* __restrict__ jt, int P, int L, FkJoint& fj, FkLink& fl) {
    // every thread reads (at clamped indices; the others' values go unused),
    // so that no read waits under a branch, and as global reads, so that the
    // LDS work in between does not wait for them
    const int c = threadIdx.x & 3;
    const int tj = min((int)threadIdx.x >> 2, P - 1);
    fj.r = ldg(&jt->off[tj][c]);
    fj.d = ldg(&jt->off[tj][4 + c]);
    fj.z = ldg(&jt->axis[tj][max(c - 1, 0)]);
    fj.type = ldg(&jt->type[tj]);
    fj.parent = ldg(&jt->parent[tj]);
    fk_link_load(jt, min((int)(blockDim.x - 1 - threadIdx.x) >> 2, L - 1), fl);
}

// value of another lane of the quad
template <int CTRL>
__device__ __forceinline__ double quad_perm(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_mov_dpp((int)(b & 0xffffffffll), CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xF, 0xF, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
// v with its sign flipped where flip (0 or the sign bit) says so
__device__ __forceinline__ double signed_by(double v, unsigned flip) {
    return __hiloint2double(__double2hiint(v) ^ (int)flip, __double2loint(v));
}

// Component c of the quaternion product a b, from the quad's components of
// both: sum over k of s_k(c) a_k b_{k ^ c}, the signs of k = 1, 2, 3 in `flip`.
struct QuadSigns { unsigned s1, s2, s3; };
__device__ __forceinline__ QuadSigns quad_signs() {
    const int c = threadIdx.x & 3;
    QuadSigns q;
    q.s1 = (c & 1) ? 0u : 0x80000000u;              // - + - +
    q.s2 = (c == 0 || c == 3) ? 0x80000000u : 0u;   // - + + -
    q.s3 = c < 2 ? 0x80000000u : 0u;                // - - + +
    return q;
}
__device__ __forceinline__ double quad_mul(double a, double b, const QuadSigns& q) {
    double t = quad_perm<0x00>(a) * b;
    t += signed_by(quad_perm<0x55>(a), q.s1) * quad_perm<0xB1>(b);
    t += signed_by(quad_perm<0xAA>(a), q.s2) * quad_perm<0x4E>(b);
    t += signed_by(quad_perm<0xFF>(a), q.s3) * quad_perm<0x1B>(b);
    return t;
}
// dual quaternion product (a.r b.r, a.r b.d + a.d b.r)
__device__ __forceinline__ double2 quad_dqmul(double2 a, double2 b, const QuadSigns& q) {
    return make_double2(quad_mul(a.x, b.x, q), quad_mul(a.x, b.y, q) + quad_mul(a.y, b.x, q));
}

__device__ __forceinline__ void fk_block_pre(const JointTable* __restrict__ jt, int P, int L, int rounds,
                                             const double* __restrict__ sth, const FkJoint& fj, FkLink fl,
                                             float* __restrict__ dq, float* __restrict__ xi, FkScratch& ws) {
    double2 (*M)[4 * (kMaxJoints + 1)] = reinterpret_cast<double2(*)[4 * (kMaxJoints + 1)]>(ws.M);
    int (*A)[kMaxJoints + 1] = ws.A;
    const int t = threadIdx.x, j = t >> 2, c = t & 3;
    const QuadSigns sg = quad_signs();
    const bool live = j < P;
    double2 m;
    {
        const double half = 0.5 * sth[min(j, P - 1)];
        double s, co;
        sincos(half, &s, &co);
        const bool hinge = fj.type == 0;
        const double2 h = make_double2(c == 0 ? (hinge ? co : 1.0) : (hinge ? s * fj.z : 0.0),
                                       c == 0 || hinge ? 0.0 : half * fj.z);
        m = quad_dqmul(make_double2(fj.r, fj.d), h, sg);
    }
    int a = live ? fj.parent : -1;
    M[0][t] = m;
    A[0][j] = a;
    __syncthreads();
    int cur = 0;
    for (int round = 0; round < rounds; ++round) {
        const int nxt = cur ^ 1, up = max(a, 0);
        const double2 mu = M[cur][4 * up + c];
        const int au = A[cur][up];
        const double2 p = quad_dqmul(mu, m, sg);
        m.x = a >= 0 ? p.x : m.x;
        m.y = a >= 0 ? p.y : m.y;
        a = a >= 0 ? au : -1;
        M[nxt][t] = m;
        A[nxt][j] = a;
        __syncthreads();
        cur = nxt;
    }
    if (live) {
        // H (z / 2) H^* in the real part (hinge) or the dual part (prismatic)
        const double half_z = c == 0 ? 0.0 : 0.5 * fj.z;
        const double2 g = fj.type == 0 ? make_double2(half_z, 0.0) : make_double2(0.0, half_z);
        const double2 hc = c == 0 ? m : make_double2(-m.x, -m.y);
        const double2 o = quad_dqmul(quad_dqmul(m, g, sg), hc, sg);
        // six components, then two of padding: lane 0 has the padding
        float* dst = xi + 8 * j;
        if (c != 0) {
            stg(dst + (c - 1), (float)o.x);
            stg(dst + 3 + (c - 1), (float)o.y);
        } else {
            stg(dst + 6, 0.0f);
            stg(dst + 7, 0.0f);
        }
    }
    const int nq = (int)blockDim.x >> 2;
    for (int l = nq - 1 - j; l < L; l += nq) {   // a quad has all of its lanes in or none
        if (l >= nq) fk_link_load(jt, l, fl);
        const double2 o = quad_dqmul(M[cur][4 * fl.joint + c], make_double2(fl.r, fl.d), sg);
        stg(dq + 8 * l + c, (float)o.x);
        stg(dq + 8 * l + 4 + c, (float)o.y);
    }
}

}  // namespace trk
