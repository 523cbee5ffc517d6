// Quaternion and dual-quaternion arithmetic on the device (Section 3.1).
// A dual quaternion H = r + eps d is held as 8 numbers: r.w r.x r.y r.z,
// d.w d.x d.y d.z.
#pragma once
#include <hip/hip_runtime.h>

namespace trk {

template <class T>
__device__ __forceinline__ void qmul(const T* a, const T* b, T* o) {
    T w = a[0] * b[0] - a[1] * b[1] - a[2] * b[2] - a[3] * b[3];
    T x = a[0] * b[1] + a[1] * b[0] + a[2] * b[3] - a[3] * b[2];
    T y = a[0] * b[2] - a[1] * b[3] + a[2] * b[0] + a[3] * b[1];
    T z = a[0] * b[3] + a[1] * b[2] - a[2] * b[1] + a[3] * b[0];
    o[0] = w; o[1] = x; o[2] = y; o[3] = z;
}

// o = a * b for dual quaternions: (a.r b.r, a.r b.d + a.d b.r)
template <class T>
__device__ __forceinline__ void dqmul(const T* a, const T* b, T* o) {
    T r[4], d1[4], d2[4];
    qmul(a, b, r);
    qmul(a, b + 4, d1);
    qmul(a + 4, b, d2);
    o[0] = r[0]; o[1] = r[1]; o[2] = r[2]; o[3] = r[3];
    o[4] = d1[0] + d2[0]; o[5] = d1[1] + d2[1]; o[6] = d1[2] + d2[2]; o[7] = d1[3] + d2[3];
}

// Conjugate of both parts; the inverse of a unit dual quaternion.
template <class T>
__device__ __forceinline__ void dqconj(const T* a, T* o) {
    o[0] = a[0]; o[1] = -a[1]; o[2] = -a[2]; o[3] = -a[3];
    o[4] = a[4]; o[5] = -a[5]; o[6] = -a[6]; o[7] = -a[7];
}

// Sums of products with every rounding written out.  Left to the compiler,
// which product of a sum is rounded apart differs from one instance of a
// kernel to the next (of q.x below, the offset step that skins the new pose
// rounded q_y y apart with 256 threads and q_x x with 512), and with it the
// last bits of a stream's results would depend on the launch that it is in.
__device__ __forceinline__ float fma_of(float a, float b, float c) { return fmaf(a, b, c); }
__device__ __forceinline__ double fma_of(double a, double b, double c) { return fma(a, b, c); }
// a b + c d, the second product rounded
template <class T>
__device__ __forceinline__ T dot2(T a, T b, T c, T d) {
#pragma clang fp contract(off)
    return fma_of(a, b, c * d);
}
// a b - c d, the second product rounded
template <class T>
__device__ __forceinline__ T det2(T a, T b, T c, T d) {
#pragma clang fp contract(off)
    return fma_of(a, b, -(c * d));
}
// a b + c d + e f, the second product rounded
template <class T>
__device__ __forceinline__ T dot3(T a, T b, T c, T d, T e, T f) {
    return fma_of(e, f, dot2(a, b, c, d));
}

// Point transform by a possibly non-unit (blended) dual quaternion:
//   T(H, x) = (r x r* + 2 vec(d r*)) / |r|^2,
// with r x r* = (w^2 - q.q) x + 2 (q.x) q + 2 w (q cross x) for r = (w, q)
// and vec(d r*) = w d_v - d_w q + q cross d_v.
__device__ __forceinline__ void dq_apply(const float* H, float x, float y, float z, float& ox,
                                         float& oy, float& oz) {
#pragma clang fp contract(off)
    const float w = H[0], qx = H[1], qy = H[2], qz = H[3];
    const float dw = H[4], dx = H[5], dy = H[6], dz = H[7];
    const float qq = dot3(qx, qx, qy, qy, qz, qz);
    const float nn = fma_of(w, w, qq);
    const float s = fma_of(w, w, -qq);
    const float qdx2 = 2.0f * dot3(qx, x, qy, y, qz, z), w2 = 2.0f * w;
    const float cx = det2(qy, z, qz, y), cy = det2(qz, x, qx, z), cz = det2(qx, y, qy, x);
    const float ax = fma_of(w2, cx, dot2(s, x, qdx2, qx));
    const float ay = fma_of(w2, cy, dot2(s, y, qdx2, qy));
    const float az = fma_of(w2, cz, dot2(s, z, qdx2, qz));
    const float bx = det2(w, dx, dw, qx) + det2(qy, dz, qz, dy);
    const float by = det2(w, dy, dw, qy) + det2(qz, dx, qx, dz);
    const float bz = det2(w, dz, dw, qz) + det2(qx, dy, qy, dx);
    const float inv = 1.0f / nn;
    ox = fma_of(2.0f, bx, ax) * inv;
    oy = fma_of(2.0f, by, ay) * inv;
    oz = fma_of(2.0f, bz, az) * inv;
}

// Blend of up to four link offsets with the weights of one vertex, each
// signed to the hemisphere of the largest-weight influence (ties: lower
// link index).  dq holds 8 floats per link.
__device__ __forceinline__ void dq_blend(const float* dq, float4 w, uint32_t links, float* H,
                                         float* sgn_out = nullptr) {
    const float ws[4] = {w.x, w.y, w.z, w.w};
    int piv = -1;
    float wb = -1.0f;
    int lb = 0x7fffffff;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        int l = (links >> (8 * k)) & 0xFF;
        if (l == 0xFF) continue;
        if (ws[k] > wb || (ws[k] == wb && l < lb)) { wb = ws[k]; lb = l; piv = l; }
    }
#pragma unroll
    for (int c = 0; c < 8; ++c) H[c] = 0.0f;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        int l = (links >> (8 * k)) & 0xFF;
        float sg = 1.0f;
        if (l != 0xFF) {
            const float* a = dq + 8 * l;
            const float* p = dq + 8 * piv;
            const float d = fma_of(a[3], p[3], dot3(a[0], p[0], a[1], p[1], a[2], p[2]));
            sg = d < 0.0f ? -1.0f : 1.0f;
            float ww = ws[k] * sg;
#pragma unroll
            for (int c = 0; c < 8; ++c) H[c] = fma_of(ww, a[c], H[c]);
        }
        if (sgn_out) sgn_out[k] = sg;
    }
}

// The linear variant of the blend (matrix linear blend skinning): the point
// moved rigidly by each influence's unit link offset, averaged with the
// weights.  No hemisphere signs: each link's motion is applied on its own.
__device__ __forceinline__ void lbs_apply(const float* dq, float4 w, uint32_t links, float x, float y, float z,
                                          float& ox, float& oy, float& oz) {
    const float ws[4] = {w.x, w.y, w.z, w.w};
    ox = 0.0f; oy = 0.0f; oz = 0.0f;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int l = (links >> (8 * k)) & 0xFF;
        if (l == 0xFF) continue;
        float tx, ty, tz;
        dq_apply(dq + 8 * l, x, y, z, tx, ty, tz);
        ox = fma_of(ws[k], tx, ox);
        oy = fma_of(ws[k], ty, oy);
        oz = fma_of(ws[k], tz, oz);
    }
}

// Rotation matrix (row-major) of the quaternion r / |r|.
template <class T>
__device__ __forceinline__ void quat_matrix(const float* q, T R[9]) {
#pragma clang fp contract(off)
    const T w = q[0], x = q[1], y = q[2], z = q[3];
    const T s = T(2) / fma_of(z, z, dot3(w, w, x, x, y, y));
    const T wy = w * y, wz = w * z, yz = y * z;
    R[0] = fma_of(-s, dot2(y, y, z, z), T(1)); R[1] = s * fma_of(x, y, -wz); R[2] = s * fma_of(x, z, wy);
    R[3] = s * fma_of(x, y, wz); R[4] = fma_of(-s, dot2(x, x, z, z), T(1)); R[5] = s * fma_of(-w, x, yz);
    R[6] = s * fma_of(x, z, -wy); R[7] = s * fma_of(w, x, yz); R[8] = fma_of(-s, dot2(x, x, y, y), T(1));
}

}  // namespace trk
