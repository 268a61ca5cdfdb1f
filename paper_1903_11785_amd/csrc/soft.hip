// Differentiable soft visual hull on gfx950: a smooth relative of the binary
// hull of Sec. II-B-1 (every camera must see a point inside its silhouette)
// for refining silhouettes and camera poses by gradient descent.
//
//   camera c: X_c = R_c X + t_c, R_c = exp([omega_c]x) R0_c, t_c = t0_c + tau_c;
//             u = fx X_c.x / X_c.z + cx, v = fy X_c.y / X_c.z + cy (pixel (x, y)
//             covers [x, x+1) x [y, y+1), centre at (x + 0.5, y + 0.5));
//   p_c(X)  = bilinear interpolation of sigmoid(L_c) between pixel centres at
//             (u, v), off-image pixels 0, and 0 behind the camera;
//   o(X)    = prod_c p_c(X), loss = sum_v (o_v - target_v)^2.
//
// The adjoint recomputes every sample's projections instead of storing them
// (one lattice at a time), takes d o / d p_c as the product of the other
// cameras' p from prefix and suffix products (no division by a p that may be
// 0), scatters the logit gradient into the four taps, and reduces each
// camera's pose gradient over the lattice: with g = d loss / d X_c,
// d loss / d tau = sum g and d loss / d omega = J_l(omega)^T sum (R X) x g,
// J_l being the left Jacobian of SO(3) (exp([omega + d]x) = exp([J_l d]x)
// exp([omega]x) to first order).
#include <limits.h>
#include <math.h>
#include <string.h>

#include <algorithm>

#include "fvv_internal.h"

namespace fvv {

// ------------------------------------------------------------------ host: rotations
// exp([w]x) = I + a [w]x + b [w]x^2 and J_l(w) = I + b [w]x + c [w]x^2 with
// a = sin t / t, b = (1 - cos t) / t^2, c = (t - sin t) / t^3 (t = |w|), by
// their series below t = 1e-3 (where the closed forms cancel).
void so3_exp_and_left_jacobian(const float w_in[3], double R[9], double J[9]) {
    const double w[3] = {w_in[0], w_in[1], w_in[2]};
    const double t2 = w[0] * w[0] + w[1] * w[1] + w[2] * w[2], t = sqrt(t2);
    double a, b, c;
    if (t < 1e-3) {
        a = 1.0 - t2 / 6.0 + t2 * t2 / 120.0;
        b = 0.5 - t2 / 24.0 + t2 * t2 / 720.0;
        c = 1.0 / 6.0 - t2 / 120.0 + t2 * t2 / 5040.0;
    } else {
        a = sin(t) / t;
        b = (1.0 - cos(t)) / t2;
        c = (t - sin(t)) / (t2 * t);
    }
    const double K[9] = {0, -w[2], w[1], w[2], 0, -w[0], -w[1], w[0], 0};
    double K2[9];
    for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 3; ++j) {
            double s = 0;
            for (int k = 0; k < 3; ++k)
                s += K[3 * i + k] * K[3 * k + j];
            K2[3 * i + j] = s;
        }
    for (int i = 0; i < 9; ++i) {
        const double I = (i % 4 == 0) ? 1.0 : 0.0;
        R[i] = I + a * K[i] + b * K2[i];
        J[i] = I + b * K[i] + c * K2[i];
    }
}

bool make_soft_cams(int n, int W, int H, const fvv_soft_camera* in, SoftCamSet* cs,
                    SoftJacobians* jac) {
    memset(cs, 0, sizeof(*cs));
    cs->n = n;
    cs->W = W;
    cs->H = H;
    for (int c = 0; c < n; ++c) {
        const fvv_soft_camera& s = in[c];
        const float* all[5] = {s.K, s.R0, s.t0, s.omega, s.tau};
        const int cnt[5] = {4, 9, 3, 3, 3};
        for (int q = 0; q < 5; ++q)
            for (int k = 0; k < cnt[q]; ++k)
                if (!isfinite(all[q][k]))
                    return false;
        if (!(s.K[0] > 0.0f) || !(s.K[1] > 0.0f))
            return false;
        double E[9], J[9];
        so3_exp_and_left_jacobian(s.omega, E, J);
        SoftCam& d = cs->c[c];
        d.fx = s.K[0];
        d.fy = s.K[1];
        d.cx = s.K[2];
        d.cy = s.K[3];
        for (int i = 0; i < 3; ++i) {
            for (int j = 0; j < 3; ++j) {
                double r = 0;
                for (int k = 0; k < 3; ++k)
                    r += E[3 * i + k] * (double)s.R0[3 * k + j];
                d.R[3 * i + j] = (float)r;
            }
            d.t[i] = (float)((double)s.t0[i] + (double)s.tau[i]);
        }
        for (int i = 0; i < 9; ++i)
            jac->Jl[c][i] = J[i];
    }
    return true;
}

// ------------------------------------------------------------------ device: one camera
struct SoftSample {
    float p;            // bilinear sigmoid value (0 behind the camera)
    float Xc[3];        // camera-space point
    float sg[4];        // sigmoid of taps (x0,y0), (x0+1,y0), (x0,y0+1), (x0+1,y0+1); 0 off-image
    float ax, ay;       // bilinear fractions
    int x0, y0;
    bool front;
};

__device__ __forceinline__ float sigmoidf(float L) { return 1.0f / (1.0f + expf(-L)); }

// The projection, and the taps' logits into s.sg.  Neither the loads nor, below,
// the sigmoids are behind a branch (an address off the image is moved onto it,
// and its value dropped), so that several cameras' loads are in flight at once
// where they are called in two loops.
__device__ __forceinline__ SoftSample soft_taps(const SoftCam& k, const float* __restrict__ L,
                                                int W, int H, float X, float Y, float Z) {
    SoftSample s;
    s.Xc[0] = __builtin_fmaf(k.R[2], Z, __builtin_fmaf(k.R[1], Y, __builtin_fmaf(k.R[0], X, k.t[0])));
    s.Xc[1] = __builtin_fmaf(k.R[5], Z, __builtin_fmaf(k.R[4], Y, __builtin_fmaf(k.R[3], X, k.t[1])));
    s.Xc[2] = __builtin_fmaf(k.R[8], Z, __builtin_fmaf(k.R[7], Y, __builtin_fmaf(k.R[6], X, k.t[2])));
    s.front = s.Xc[2] > 0.0f;
    const float inv = 1.0f / s.Xc[2], rz = s.front ? inv : 0.0f;
    // pixel-centre coordinates, clamped where every tap is off-image anyway
    const float su = fminf(fmaxf(k.fx * s.Xc[0] * rz + k.cx - 0.5f, -2.0f), (float)W + 1.0f);
    const float sv = fminf(fmaxf(k.fy * s.Xc[1] * rz + k.cy - 0.5f, -2.0f), (float)H + 1.0f);
    const float fx0 = floorf(su), fy0 = floorf(sv);
    s.ax = su - fx0;
    s.ay = sv - fy0;
    s.x0 = (int)fx0;
    s.y0 = (int)fy0;
    const int xa = min(max(s.x0, 0), W - 1), xb = min(max(s.x0 + 1, 0), W - 1);
    const float* const r0 = L + (int64_t)min(max(s.y0, 0), H - 1) * W;
    const float* const r1 = L + (int64_t)min(max(s.y0 + 1, 0), H - 1) * W;
    s.sg[0] = r0[xa];
    s.sg[1] = r0[xb];
    s.sg[2] = r1[xa];
    s.sg[3] = r1[xb];
    return s;
}

__device__ __forceinline__ void soft_value(SoftSample& s, int W, int H) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int x = s.x0 + (q & 1), y = s.y0 + (q >> 1);
        const float v = sigmoidf(s.sg[q]);
        s.sg[q] = s.front & (x >= 0) & (x < W) & (y >= 0) & (y < H) ? v : 0.0f;
    }
    const float p = (1.0f - s.ax) * (1.0f - s.ay) * s.sg[0] + s.ax * (1.0f - s.ay) * s.sg[1] +
                    (1.0f - s.ax) * s.ay * s.sg[2] + s.ax * s.ay * s.sg[3];
    s.p = s.front ? p : 0.0f;
}

__device__ __forceinline__ void sample_coords(const fvv_grid& g, uint32_t idx, float& X, float& Y,
                                              float& Z) {
    const uint32_t nx = (uint32_t)g.dims[0], ny = (uint32_t)g.dims[1];
    const uint32_t r = idx / nx;
    X = lattice_coord(g.lo[0] + (int)(idx - r * nx), g.h, g.origin[0]);
    Y = lattice_coord(g.lo[1] + (int)(r % ny), g.h, g.origin[1]);
    Z = lattice_coord(g.lo[2] + (int)(r / ny), g.h, g.origin[2]);
}

// Sum over the wave (DPP row shifts and broadcasts; lane 63 holds the total).
__device__ __forceinline__ float wave_sum(float v) {
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x111, 0xf, 0xf, true));
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x112, 0xf, 0xf, true));
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x114, 0xf, 0xf, true));
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x118, 0xf, 0xf, true));
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x142, 0xa, 0xf, false));
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x143, 0xc, 0xf, false));
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), kWave - 1));
}

// ------------------------------------------------------------------ kernels
__global__ __launch_bounds__(kBlock) void soft_zero_kernel(float* __restrict__ f, int64_t nf,
                                                           double* __restrict__ d, int nd) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    for (int64_t q = i; q < nf; q += (int64_t)gridDim.x * kBlock)
        f[q] = 0.0f;
    for (int64_t q = i; q < nd; q += (int64_t)gridDim.x * kBlock)
        d[q] = 0.0;
}

// kSplit waves share 64 samples, each taking every kSplit-th camera of them,
// four cameras' loads in flight at once; with kSplit > 1 the p meet in LDS and
// the first of the waves multiplies them in the cameras' order.  A lattice of
// one person's box is some 5e4 samples, a wave per SIMD with a thread a sample,
// whose cameras' loads and sigmoids then run one after the other: split in four
// 4.8e4 samples of 16 cameras of 320 x 240 take 15 us, in turn 23.  A large
// lattice has the waves without, and is left early where a camera sees nothing.
// One atomic per workgroup: they go one after the other, 7 ns each, so the
// workgroups are large (1024 threads) and at most two per CU.
constexpr int kSoftWaves = kBlock / kWave;
constexpr int fwd_block(int split) { return split > 1 ? 1024 : kBlock; }

template <bool kLoss, int kSplit>
__global__ __launch_bounds__(fwd_block(kSplit)) void soft_fwd_kernel(const SoftCamSet cams,
                                                             const fvv_grid g,
                                                             const float* __restrict__ logits,
                                                             const float* __restrict__ target,
                                                             float* __restrict__ occ,
                                                             double* __restrict__ loss) {
    constexpr int kFwdBlock = fwd_block(kSplit), kSamples = kFwdBlock / kSplit;
    __shared__ float s_p[kSplit > 1 ? FVV_MAX_CAMS : 1][kSplit > 1 ? kSamples : 1];
    __shared__ double s_part[kFwdBlock / kWave];
    const uint32_t V = (uint32_t)((int64_t)g.dims[0] * g.dims[1] * g.dims[2]);
    const int64_t cam_px = (int64_t)cams.W * cams.H;
    const uint32_t at = threadIdx.x % kSamples;
    const int share = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kSamples));
    double acc = 0.0;
    for (uint32_t base = blockIdx.x * kSamples; base < V; base += gridDim.x * kSamples) {
        const uint32_t idx = min(base + at, V - 1u);
        float X, Y, Z, o = 1.0f;
        sample_coords(g, idx, X, Y, Z);
        for (int c0 = share; c0 < cams.n; c0 += 4 * kSplit) {
            SoftSample sm[4];
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const int c = min(c0 + m * kSplit, cams.n - 1);
                sm[m] = soft_taps(cams.c[c], logits + c * cam_px, cams.W, cams.H, X, Y, Z);
            }
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const int c = c0 + m * kSplit;
                if (kSplit > 1) {
                    // (cameras beyond the last are the last, and their p dropped)
                    soft_value(sm[m], cams.W, cams.H);
                    if (c < cams.n)
                        s_p[c][at] = sm[m].p;
                } else if (c < cams.n && __any(o != 0.0f)) {
                    soft_value(sm[m], cams.W, cams.H);
                    const float next = o * sm[m].p;
                    o = o != 0.0f ? next : o;
                }
            }
            if (kSplit == 1 && !__any(o != 0.0f))
                break;
        }
        if (kSplit > 1) {
            __syncthreads();
            if (share == 0)
                for (int c = 0; c < cams.n; ++c) {
                    const float next = o * s_p[c][at];
                    o = o != 0.0f ? next : o;
                }
        }
        if (share == 0 && base + at < V) {
            if (occ)
                occ[idx] = o;
            if (kLoss) {
                const double d = (double)o - (double)target[idx];
                acc += d * d;
            }
        }
        if (kSplit > 1)
            __syncthreads();
    }
    if (kLoss) {
        // block sum in double (wave partials through LDS), one atomic per block
        for (int off = kWave / 2; off >= 1; off >>= 1)
            acc += __shfl_xor(acc, off);
        if (lane_id() == 0)
            s_part[threadIdx.x / kWave] = acc;
        __syncthreads();
        if (threadIdx.x == 0) {
            double t = 0.0;
            for (int w = 0; w < kFwdBlock / kWave; ++w)
                t += s_part[w];
            unsafeAtomicAdd(loss, t);
        }
    }
}

// Minimum over the wave (as wave_sum; a lane without a source keeps its own).
__device__ __forceinline__ int wave_min_i32(int v) {
    v = min(v, __builtin_amdgcn_update_dpp(v, v, 0x111, 0xf, 0xf, false));
    v = min(v, __builtin_amdgcn_update_dpp(v, v, 0x112, 0xf, 0xf, false));
    v = min(v, __builtin_amdgcn_update_dpp(v, v, 0x114, 0xf, 0xf, false));
    v = min(v, __builtin_amdgcn_update_dpp(v, v, 0x118, 0xf, 0xf, false));
    v = min(v, __builtin_amdgcn_update_dpp(v, v, 0x142, 0xa, 0xf, false));
    v = min(v, __builtin_amdgcn_update_dpp(v, v, 0x143, 0xc, 0xf, false));
    return __builtin_amdgcn_readlane(v, kWave - 1);
}

// The adjoint.  A workgroup takes a brick of 4 x 4 x 4 lattice samples, one per
// lane, and its wave w the cameras c = w mod 4: each wave samples its own
// cameras once and keeps what the gradient needs of them in registers, the p of
// all cameras meet in LDS, and every wave forms the prefix and suffix products
// of its cameras in the cameras' order from them (kPer: cameras per wave).  Per
// camera, the brick's logit-gradient contributions fall in a small pixel window
// (the brick spans a few pixels): the wave sums them there with LDS atomics and
// adds the window to the gradient image with one global atomic per touched
// pixel, instead of four contended global atomics per sample (all samples along
// a camera ray hit the same pixels).  Windows larger than kWin pixels fall back
// to global atomics.  The windows are the waves' own, so cameras need no
// barrier between them.  acc [kSoftSlots][FVV_MAX_CAMS][6]: per camera sum of
// g = d loss / d X_c and of (R X) x g (DPP wave sums, then double over the
// workgroup's bricks, then an atomic each per workgroup, to one of kSoftSlots
// copies: the workgroups end together).
// What bounds it is latency and the sigmoids: bricks of 256 samples whose four
// camera groups sampled all 16 cameras each (80 samplings per lattice sample for
// the 16 needed here) with six barriers per camera took 67 us on 4.8e4 samples
// of 16 cameras of 320 x 240, 37 now (of 56 us at 8.6e4 samples 16 are the rate of the LDS
// atomics themselves: copies of the
// window against their conflicts gave nothing).
constexpr int kBrick = 4;
static_assert(kBrick * kBrick * kBrick == kWave, "a sample per lane");
constexpr int kWin = 1024;

template <int kPer, bool kL2>
__global__ __launch_bounds__(kBlock, 2) void soft_bwd_kernel(const SoftCamSet cams, const fvv_grid g,
                                                          const float* __restrict__ logits,
                                                          const float* __restrict__ target,
                                                          const float* __restrict__ grad_occ,
                                                          const double* __restrict__ scale_p,
                                                          float* __restrict__ grad_logits,
                                                          double* __restrict__ acc) {
    constexpr int kN = kPer * kSoftWaves;
    __shared__ double s_acc[kN][6];
    __shared__ float s_p[kN][kWave];
    __shared__ float s_win_all[kSoftWaves][kWin];
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave)), lane = lane_id();
    float* const s_win = s_win_all[wave];
    for (int q = threadIdx.x; q < kN * 6; q += kBlock)
        s_acc[q / 6][q % 6] = 0.0;
    for (int q = threadIdx.x; q < kN * kWave; q += kBlock)
        s_p[q / kWave][q % kWave] = 1.0f;      // (cameras beyond the rig's stay at 1)
    __syncthreads();
    const int nx = g.dims[0], ny = g.dims[1], nz = g.dims[2];
    const int nbx = (nx + kBrick - 1) / kBrick, nby = (ny + kBrick - 1) / kBrick;
    const int nbz = (nz + kBrick - 1) / kBrick;
    const int64_t bricks = (int64_t)nbx * nby * nbz;
    const int64_t cam_px = (int64_t)cams.W * cams.H;
    const float scale = scale_p ? (float)*scale_p : 1.0f;
    const int lx = lane % kBrick, ly = (lane / kBrick) % kBrick, lz = lane / (kBrick * kBrick);
    for (int64_t br = blockIdx.x; br < bricks; br += gridDim.x) {
        const int bx = (int)(br % nbx), by = (int)((br / nbx) % nby), bz = (int)(br / nbx / nby);
        const int i = bx * kBrick + lx, j = by * kBrick + ly, k = bz * kBrick + lz;
        const bool act = i < nx && j < ny && k < nz;
        const uint32_t idx = act ? (uint32_t)(((int64_t)k * ny + j) * nx + i) : 0u;
        float X, Y, Z;
        sample_coords(g, idx, X, Y, Z);
        SoftSample sm[kPer];
#pragma unroll
        for (int m = 0; m < kPer; ++m) {
            const int c = min(wave + m * kSoftWaves, cams.n - 1);
            sm[m] = soft_taps(cams.c[c], logits + c * cam_px, cams.W, cams.H, X, Y, Z);
        }
#pragma unroll
        for (int m = 0; m < kPer; ++m)
            soft_value(sm[m], cams.W, cams.H);
#pragma unroll
        for (int m = 0; m < kPer; ++m)
            if (wave + m * kSoftWaves < cams.n)
                s_p[wave + m * kSoftWaves][lane] = sm[m].p;
        __syncthreads();
        float gp[kPer], run = 1.0f;
#pragma unroll
        for (int c = kN - 1; c >= 0; --c) {
            if (c % kSoftWaves == wave)
                gp[c / kSoftWaves] = run;      // the later cameras' product
            run *= s_p[c][lane];
        }
        float go = 0.0f;
        if (act)
            go = (kL2 ? 2.0f * (run - target[idx]) : grad_occ[idx]) * scale;
        run = 1.0f;
#pragma unroll
        for (int c = 0; c < kN; ++c) {
            if (c % kSoftWaves == wave)
                gp[c / kSoftWaves] = go * run * gp[c / kSoftWaves];
            run *= s_p[c][lane];
        }
#pragma unroll
        for (int m = 0; m < kPer; ++m) {
            const int c = wave + m * kSoftWaves;
            if (c >= cams.n)
                break;
            const SoftSample& t = sm[m];
            const bool live = gp[m] != 0.0f && t.front;
            if (!__any(live))
                continue;                      // the whole brick has no gradient here
            const SoftCam& cm = cams.c[c];
            // the brick's tap window
            const int wx0 = wave_min_i32(live ? t.x0 : INT_MAX);
            const int wy0 = wave_min_i32(live ? t.y0 : INT_MAX);
            const int wxn = 1 - wave_min_i32(live ? -(t.x0 + 1) : INT_MAX) - wx0;
            const int wyn = 1 - wave_min_i32(live ? -(t.y0 + 1) : INT_MAX) - wy0;
            const bool in_lds = (int64_t)wxn * wyn <= kWin;   // uniform
            float* gl = grad_logits + c * cam_px;
            const float w4[4] = {(1.0f - t.ax) * (1.0f - t.ay), t.ax * (1.0f - t.ay),
                                 (1.0f - t.ax) * t.ay, t.ax * t.ay};
            if (in_lds) {
                for (int q = lane; q < wxn * wyn; q += kWave)
                    s_win[q] = 0.0f;
                wave_lds_sync();
            }
            float gx = 0.0f, gy = 0.0f, gz = 0.0f, bxv = 0.0f, byv = 0.0f, bzv = 0.0f;
            if (live) {
                // logits: d p / d L_tap = weight * sigmoid' (taps off-image have sg = 0)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int x = t.x0 + (q & 1), y = t.y0 + (q >> 1);
                    if (x >= 0 && x < cams.W && y >= 0 && y < cams.H) {
                        const float v = gp[m] * w4[q] * t.sg[q] * (1.0f - t.sg[q]);
                        if (in_lds)
                            atomicAdd(&s_win[(y - wy0) * wxn + (x - wx0)], v);
                        else
                            unsafeAtomicAdd(&gl[(int64_t)y * cams.W + x], v);
                    }
                }
                // pose: d p / d u and d p / d v, then through the projection
                const float du = (1.0f - t.ay) * (t.sg[1] - t.sg[0]) + t.ay * (t.sg[3] - t.sg[2]);
                const float dv = (1.0f - t.ax) * (t.sg[2] - t.sg[0]) + t.ax * (t.sg[3] - t.sg[1]);
                const float rz = 1.0f / t.Xc[2];
                gx = gp[m] * du * cm.fx * rz;
                gy = gp[m] * dv * cm.fy * rz;
                gz = -(gx * t.Xc[0] + gy * t.Xc[1]) * rz;
                // R X = X_c - t
                const float rx = t.Xc[0] - cm.t[0], ry = t.Xc[1] - cm.t[1],
                            rzv = t.Xc[2] - cm.t[2];
                bxv = ry * gz - rzv * gy;
                byv = rzv * gx - rx * gz;
                bzv = rx * gy - ry * gx;
            }
            const float v6[6] = {gx, gy, gz, bxv, byv, bzv};
            float mine = 0.0f;
#pragma unroll
            for (int q = 0; q < 6; ++q) {
                const float sum = wave_sum(v6[q]);
                mine = lane == q ? sum : mine;
            }
            if (lane < 6)
                s_acc[c][lane] += (double)mine;        // (the wave's own cameras)
            if (in_lds) {
                wave_lds_sync();
                for (int q = lane; q < wxn * wyn; q += kWave) {
                    const float v = s_win[q];
                    if (v != 0.0f) {    // only in-image taps were added
                        const int y = q / wxn;
                        unsafeAtomicAdd(&gl[(int64_t)(wy0 + y) * cams.W + (wx0 + q - y * wxn)], v);
                    }
                }
                wave_lds_sync();       // the next camera's window is cleared after these reads
            }
        }
        __syncthreads();   // every wave has read s_p
    }
    acc += (blockIdx.x % kSoftSlots) * (FVV_MAX_CAMS * 6);
    for (int q = threadIdx.x; q < cams.n * 6; q += kBlock)
        if (s_acc[q / 6][q % 6] != 0.0)
            unsafeAtomicAdd(&acc[q], s_acc[q / 6][q % 6]);
}

// grad_pose[c] = (J_l^T sum (R X) x g, sum g).
__global__ void soft_pose_kernel(const double* __restrict__ acc, const SoftJacobians jac, int n,
                                 double* __restrict__ grad_pose) {
    const int c = threadIdx.x;
    if (c >= n)
        return;
    double a[6] = {};
#pragma unroll
    for (int q = 0; q < kSoftSlots; ++q)
        for (int i = 0; i < 6; ++i)
            a[i] += acc[(q * FVV_MAX_CAMS + c) * 6 + i];
    const double* J = jac.Jl[c];
    for (int i = 0; i < 3; ++i)
        grad_pose[6 * c + i] = J[i] * a[3] + J[3 + i] * a[4] + J[6 + i] * a[5];
    for (int i = 0; i < 3; ++i)
        grad_pose[6 * c + 3 + i] = a[i];
}

// ------------------------------------------------------------------ launchers
hipError_t launch_soft_forward(fvv_ctx* ctx, const SoftCamSet& cams, const fvv_grid& g,
                               const float* logits, const float* target, float* occ,
                               double* loss, hipStream_t s) {
    const int64_t V = (int64_t)g.dims[0] * g.dims[1] * g.dims[2];
    // split where a thread a sample gives fewer than four waves per SIMD and
    // there is more than one batch of cameras to share
    const bool split = V < (int64_t)ctx->n_cus * 16 * kWave && cams.n > 4;
    const int block = fwd_block(split ? 4 : 1), per = split ? block / 4 : block;
    const unsigned blocks = (unsigned)std::min<int64_t>((V + per - 1) / per,
                                                        (int64_t)ctx->n_cus * (split ? 2 : 16));
#define X(LOSS, SPLIT)                                                                          \
    hipLaunchKernelGGL((soft_fwd_kernel<LOSS, SPLIT>), dim3(blocks), dim3(block), 0, s,         \
                       cams, g, logits, target, occ, loss);
    if (loss) {
        hipLaunchKernelGGL(soft_zero_kernel, dim3(1), dim3(kBlock), 0, s, nullptr, (int64_t)0,
                           loss, 1);
        if (split) {
            X(true, 4)
        } else {
            X(true, 1)
        }
    } else if (split) {
        X(false, 4)
    } else {
        X(false, 1)
    }
#undef X
    return hipGetLastError();
}

hipError_t launch_soft_backward(fvv_ctx* ctx, const SoftCamSet& cams, const SoftJacobians& jac,
                                const fvv_grid& g, const float* logits, const float* target,
                                const float* grad_occ, const double* scale, float* grad_logits,
                                double* grad_pose, hipStream_t s) {
    const int64_t npx = (int64_t)cams.n * cams.W * cams.H;
    const unsigned zb = (unsigned)std::min<int64_t>((npx + kBlock - 1) / kBlock, 4096);
    hipLaunchKernelGGL(soft_zero_kernel, dim3(zb), dim3(kBlock), 0, s, grad_logits, npx,
                       ctx->d_soft_acc, kSoftSlots * FVV_MAX_CAMS * 6);
    const int64_t bricks = (int64_t)((g.dims[0] + kBrick - 1) / kBrick) *
                           ((g.dims[1] + kBrick - 1) / kBrick) * ((g.dims[2] + kBrick - 1) / kBrick);
    const unsigned blocks = (unsigned)std::min<int64_t>(bricks, (int64_t)ctx->n_cus * 8);
#define X(KP)                                                                                   \
    if (target)                                                                                 \
        hipLaunchKernelGGL((soft_bwd_kernel<KP, true>), dim3(blocks), dim3(kBlock), 0, s, cams, \
                           g, logits, target, grad_occ, scale, grad_logits, ctx->d_soft_acc);   \
    else                                                                                        \
        hipLaunchKernelGGL((soft_bwd_kernel<KP, false>), dim3(blocks), dim3(kBlock), 0, s,      \
                           cams, g, logits, target, grad_occ, scale, grad_logits,               \
                           ctx->d_soft_acc);
    if (cams.n <= 4 * kSoftWaves) {
        X(4)
    } else {
        X(FVV_MAX_CAMS / kSoftWaves)
    }
#undef X
    hipLaunchKernelGGL(soft_pose_kernel, dim3(1), dim3(kWave), 0, s, ctx->d_soft_acc, jac, cams.n,
                       grad_pose);
    return hipGetLastError();
}

}  // namespace fvv
