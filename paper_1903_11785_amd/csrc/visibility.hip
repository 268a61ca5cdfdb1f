// Depth images and visibility of a triangle mesh in every camera (Sec. II-D,
// Eq. (4)) on gfx950, with the readings stated in include/fvv.h
// (fvv_visibility): a triangle covers the pixels whose centres lie on the same
// side of its three projected edges, at the camera-plane distance of its
// centroid; a pixel keeps the minimum; a triangle is visible in a camera when
// its centroid projects into the image and its distance exceeds the depth
// there by at most T_v.
//
// Depth: one thread per triangle, its vertices loaded once and rastered in
// every camera in turn (a wave's triangles, listed cell by cell, touch
// neighbouring pixels of each image); the minimum is an atomicMin on the
// float's bits (the distances are positive, so their bit patterns order like
// the values and the result does not depend on the order of the updates).  Visibility: one thread per triangle
// over all cameras, one mask word each.  All arithmetic is fp32 in a fixed
// order with IEEE division, as the reading defines it.
#include <algorithm>

#include "fvv_internal.h"

namespace fvv {

constexpr uint32_t kInfBits = 0x7f800000u;   // +inf
constexpr int kVisCams = 4;                  // cameras whose depth loads are in flight

__global__ __launch_bounds__(kBlock) void depth_clear_kernel(uint32_t* __restrict__ depth,
                                                             size_t n) {
    for (size_t q = (size_t)blockIdx.x * kBlock + threadIdx.x; q < n;
         q += (size_t)gridDim.x * kBlock)
        depth[q] = kInfBits;
}

__device__ __forceinline__ void project3(const float* p, const float X[3], float& a, float& b,
                                         float& w) {
    a = __builtin_fmaf(p[2], X[2], __builtin_fmaf(p[1], X[1], __builtin_fmaf(p[0], X[0], p[3])));
    b = __builtin_fmaf(p[6], X[2], __builtin_fmaf(p[5], X[1], __builtin_fmaf(p[4], X[0], p[7])));
    w = __builtin_fmaf(p[10], X[2], __builtin_fmaf(p[9], X[1], __builtin_fmaf(p[8], X[0], p[11])));
}

// The IEEE quotients a[k] / w[k] and b[k] / w[k] of K points: per point the
// reciprocal refined once for both, then for each quotient Markstein's two
// corrections by the exactly computed remainder, which round correctly while no
// intermediate leaves the normal range (operands of magnitude 2^-60 to 2^60);
// anything else in the wave is divided.
__device__ __forceinline__ float quotient(float a, float w, float r) {
    float q = a * r;
    q = __builtin_fmaf(__builtin_fmaf(-w, q, a), r, q);
    return __builtin_fmaf(__builtin_fmaf(-w, q, a), r, q);
}

template <int K>
__device__ __forceinline__ void quotients(const float* a, const float* b, const float* w,
                                          float* qa, float* qb) {
    float lo = INFINITY, hi = 0.0f;
    bool nan = false;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const float fa = __builtin_fabsf(a[k]), fb = __builtin_fabsf(b[k]);
        const float fw = __builtin_fabsf(w[k]);
        lo = fminf(lo, fminf(fa, fminf(fb, fw)));
        hi = fmaxf(hi, fmaxf(fa, fmaxf(fb, fw)));
        // (a NaN in a sum stays one; fminf and fmaxf pass over it)
        nan |= !(fa + fb + fw <= INFINITY);
        float r = __builtin_amdgcn_rcpf(w[k]);
        r = __builtin_fmaf(__builtin_fmaf(-w[k], r, 1.0f), r, r);
        qa[k] = quotient(a[k], w[k], r);
        qb[k] = quotient(b[k], w[k], r);
    }
    const bool odd = nan || lo <= 0x1p-60f || hi >= 0x1p60f;
    if (__builtin_expect(__ballot(odd) != 0ull, 0)) {
        if (odd) {
#pragma unroll
            for (int k = 0; k < K; ++k) {
                qa[k] = a[k] / w[k];
                qb[k] = b[k] / w[k];
            }
        }
    }
}

// The triangle's vertices, or false when it names a vertex past nv.
__device__ __forceinline__ bool load_triangle(const float* __restrict__ xyz,
                                              const uint32_t* __restrict__ tris, uint32_t m,
                                              uint32_t nv, float V[3][3]) {
    const uint32_t t0 = tris[3 * (size_t)m], t1 = tris[3 * (size_t)m + 1],
                   t2 = tris[3 * (size_t)m + 2];
    if (t0 >= nv || t1 >= nv || t2 >= nv)
        return false;
    const uint32_t t[3] = {t0, t1, t2};
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int a = 0; a < 3; ++a)
            V[k][a] = xyz[3 * (size_t)t[k] + a];
    return true;
}

// The triangle's centroid ((v0 + v1) + v2) / 3.
__device__ __forceinline__ void centroid(const float V[3][3], float G[3]) {
#pragma unroll
    for (int k = 0; k < 3; ++k)
        G[k] = ((V[0][k] + V[1][k]) + V[2][k]) / 3.0f;
}

__device__ __forceinline__ float edge_fn(float x0, float y0, float x1, float y1, float px,
                                         float py) {
    return (x1 - x0) * (py - y0) - (y1 - y0) * (px - x0);
}

// The pixels of one triangle (vertices V, centroid G) in one camera: skipped
// when a vertex is behind the camera, the projected area is zero, the
// centroid's distance is not positive or the box misses the image; else
// atomicMin of the distance's bits into each covered pixel of the camera's
// depth image D.
//
// The edge tests decide; the box only has to hold every pixel they accept.
// [floor(min), floor(max)] does by definition.  For a triangle that is no
// sliver, so does the box of the pixels whose centres lie within t = 2^-6 of
// its bounds: a centre p farther out has a barycentric coordinate of at most
// -t / (2 S) (S the larger side of the bounds), so one edge function is
// |A| t / (2 S) on the wrong side (A the area's, twice the area), and another
// at least |A| / 3 on the right one; the tests' rounding is below 8 2^-24 S (S
// + 1).  |A| above 2^-12 S (S + 1)^2 leaves a factor of four.  Coordinates up
// to 8192 round by less than t / 8.  A mesh's triangles are about a pixel
// wide: three times fewer pixels are tested, and with the shared reciprocals
// 4.7e5 triangles in 16 cameras of 1920 x 1080 take 45 us, before 61 (with
// plain stores for the atomics, 57 then).  Large triangles spend their time on
// the pixels: with the row terms formed once per row a mesh of 200 mm edges in 4
// cameras of 3840 x 2160 takes the call 1050 us, formed at each pixel 1150.
__device__ __forceinline__ void raster_one(const float* p, const float V[3][3], const float G[3],
                                           int W, int H, uint32_t* __restrict__ D) {
    float u[3], v[3], a[3], b[3], w[3];
    bool front = true;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        project3(p, V[k], a[k], b[k], w[k]);
        front &= w[k] > 0.0f;
    }
    quotients<3>(a, b, w, u, v);
    const float area = edge_fn(u[0], v[0], u[1], v[1], u[2], v[2]);
    if (!front || area == 0.0f)
        return;
    float ga, gb, d;
    project3(p, G, ga, gb, d);
    if (!(d > 0.0f))
        return;
    const float lo_u = fminf(u[0], fminf(u[1], u[2])), hi_u = fmaxf(u[0], fmaxf(u[1], u[2]));
    const float lo_v = fminf(v[0], fminf(v[1], v[2])), hi_v = fmaxf(v[0], fmaxf(v[1], v[2]));
    if (!(hi_u >= 0.0f && hi_v >= 0.0f && lo_u < (float)W && lo_v < (float)H))
        return;
    const float S = fmaxf(hi_u - lo_u, hi_v - lo_v);
    const bool tight = W <= 8192 && H <= 8192 &&
                       __builtin_fabsf(area) > 0x1p-12f * S * (S + 1.0f) * (S + 1.0f);
    // (NaN bounds keep the whole range, as the comparisons above leave it)
    const float in = tight ? 0.5f - 0x1p-6f : 0.0f;
    const float fx0 = tight ? __builtin_ceilf(lo_u - 0.5f - 0x1p-6f) : lo_u;
    const float fy0 = tight ? __builtin_ceilf(lo_v - 0.5f - 0x1p-6f) : lo_v;
    const float fx1 = hi_u - in, fy1 = hi_v - in;
    const int x0 = fx0 < 0.0f ? 0 : (int)fx0;
    const int y0 = fy0 < 0.0f ? 0 : (int)fy0;
    const int x1 = fx1 >= (float)(W - 1) ? W - 1 : fx1 < 0.0f ? -1 : (int)fx1;
    const int y1 = fy1 >= (float)(H - 1) ? H - 1 : fy1 < 0.0f ? -1 : (int)fy1;
    const uint32_t dbits = __float_as_uint(d);
    if (x0 > x1 || y0 > y1)
        return;
    const float cx0 = (float)x0 + 0.5f, cx1 = (float)x1 + 0.5f, cy1 = (float)y1 + 0.5f;
    float px = cx0, py = (float)y0 + 0.5f;       // pixel centres, exact
    uint32_t* row = D + (size_t)y0 * W + x0;
    uint32_t* at = row;
    // the edge functions' row terms, by edge_fn's own operations
    auto row_term = [&](int i, int j) { return (u[j] - u[i]) * (py - v[i]); };
    float r0 = row_term(0, 1), r1 = row_term(1, 2), r2 = row_term(2, 0);
    for (;;) {                                   // one loop over rows and columns
        const float e0 = r0 - (v[1] - v[0]) * (px - u[0]);
        const float e1 = r1 - (v[2] - v[1]) * (px - u[1]);
        const float e2 = r2 - (v[0] - v[2]) * (px - u[2]);
        const bool in = (e0 >= 0.0f && e1 >= 0.0f && e2 >= 0.0f) ||
                        (e0 <= 0.0f && e1 <= 0.0f && e2 <= 0.0f);
        if (in)
            atomicMin(at, dbits);
        ++at;
        px += 1.0f;
        if (px > cx1) {
            px = cx0;
            py += 1.0f;
            row += W;
            at = row;
            if (py > cy1)
                break;
            r0 = row_term(0, 1);
            r1 = row_term(1, 2);
            r2 = row_term(2, 0);
        }
    }
}

__global__ __launch_bounds__(kBlock) void depth_raster_kernel(
    const CamSet cams, const float* __restrict__ xyz, const uint32_t* __restrict__ n_vert_p,
    uint32_t max_vert, const uint32_t* __restrict__ tris, const uint32_t* __restrict__ n_tris_p,
    uint32_t max_tris, uint32_t* __restrict__ depth) {
    const uint32_t nv_all = *n_vert_p, nt_all = *n_tris_p;
    const uint32_t nv = nv_all < max_vert ? nv_all : max_vert;
    const uint32_t T = nt_all < max_tris ? nt_all : max_tris;
    const int W = cams.W, H = cams.H;
    for (uint64_t mm = (uint64_t)blockIdx.x * kBlock + threadIdx.x; mm < T;
         mm += (uint64_t)gridDim.x * kBlock) {
        float V[3][3];
        if (!load_triangle(xyz, tris, (uint32_t)mm, nv, V))
            continue;
        float G[3];
        centroid(V, G);
        for (int c = 0; c < cams.n; ++c)
            raster_one(cams.P[c], V, G, W, H, depth + (size_t)c * W * H);
    }
}

__global__ __launch_bounds__(kBlock) void visibility_kernel(
    const CamSet cams, const float* __restrict__ xyz, const uint32_t* __restrict__ n_vert_p,
    uint32_t max_vert, const uint32_t* __restrict__ tris, const uint32_t* __restrict__ n_tris_p,
    uint32_t max_tris, const float* __restrict__ depth, float t_v, uint32_t* __restrict__ vis) {
    const uint32_t nv_all = *n_vert_p, nt_all = *n_tris_p;
    const uint32_t nv = nv_all < max_vert ? nv_all : max_vert;
    const uint32_t T = nt_all < max_tris ? nt_all : max_tris;
    const int W = cams.W, H = cams.H;
    for (uint32_t m = blockIdx.x * kBlock + threadIdx.x; m < T; m += gridDim.x * kBlock) {
        float V[3][3];
        uint32_t mask = 0;
        if (load_triangle(xyz, tris, m, nv, V)) {
            float G[3];
            centroid(V, G);
            // four cameras at a time, their depth loads in flight together (one
            // after the other: 19.4 us for 4.7e5 triangles in 16 cameras, so
            // 16.9; a camera past the last repeats it)
            for (int c0 = 0; c0 < cams.n; c0 += kVisCams) {
                float d[kVisCams], D[kVisCams];
                bool seen[kVisCams];
#pragma unroll
                for (int k = 0; k < kVisCams; ++k) {
                    const int c = min(c0 + k, cams.n - 1);
                    float a, b, u, v;
                    project3(cams.P[c], G, a, b, d[k]);
                    quotients<1>(&a, &b, &d[k], &u, &v);
                    const float fx = __builtin_floorf(u), fy = __builtin_floorf(v);
                    seen[k] = d[k] > 0.0f && fx >= 0.0f && fy >= 0.0f && fx < (float)W &&
                              fy < (float)H;
                    D[k] = seen[k] ? depth[((size_t)c * H + (size_t)fy) * W + (size_t)fx] : 0.0f;
                }
#pragma unroll
                for (int k = 0; k < kVisCams; ++k)
                    if (seen[k] && c0 + k < cams.n && d[k] - D[k] <= t_v)
                        mask |= 1u << (c0 + k);
            }
        }
        vis[m] = mask;
    }
}

hipError_t launch_visibility(fvv_ctx* ctx, const CamSet& cams, const float* xyz,
                             const uint32_t* n_vert, uint32_t max_vert, const uint32_t* tris,
                             const uint32_t* n_tris, uint32_t max_tris, float t_v, float* depth,
                             uint32_t* vis, hipStream_t s) {
    const size_t n = (size_t)cams.n * cams.W * cams.H;
    const int64_t cap = (int64_t)ctx->n_cus * 8;
    hipLaunchKernelGGL(depth_clear_kernel,
                       dim3((unsigned)std::min<int64_t>(((int64_t)n + kBlock - 1) / kBlock, cap)),
                       dim3(kBlock), 0, s, reinterpret_cast<uint32_t*>(depth), n);
    hipLaunchKernelGGL(depth_raster_kernel,
                       dim3((unsigned)std::min<int64_t>(((int64_t)max_tris + kBlock - 1) / kBlock,
                                                        cap)),
                       dim3(kBlock), 0, s, cams, xyz, n_vert, max_vert, tris, n_tris, max_tris,
                       reinterpret_cast<uint32_t*>(depth));
    hipLaunchKernelGGL(visibility_kernel,
                       dim3((unsigned)std::min<int64_t>(((int64_t)max_tris + kBlock - 1) / kBlock,
                                                        cap)),
                       dim3(kBlock), 0, s, cams, xyz, n_vert, max_vert, tris, n_tris, max_tris,
                       depth, t_v, vis);
    return hipGetLastError();
}

}  // namespace fvv
