// Depth-image preparation for the render-accelerated point-to-plane ICP of
// Sec. V: downsampling with the far-point filter, Gaussian smoothing, the
// depth-image normals of Eq. (2) and per-vertex normals of a meshified view.
// These run once per depth image, outside the per-iteration render loop; the
// association and the point-to-plane blocks are fused into the tile pass.
#include "rm_internal.h"

namespace rm {

namespace {

// out(i, j) = depth(f i, f j) when it is a finite positive depth up to z_max,
// NaN otherwise.
__global__ void k_downsample(const float* __restrict__ depth, int32_t H, int32_t W, int32_t f, int32_t H2,
                             int32_t W2, float z_max, float* __restrict__ out) {
    const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= (int64_t)H2 * W2) return;
    const int i = (int)(n / W2), j = (int)(n % W2);
    const float z = depth[(int64_t)(i * f) * W + (int64_t)j * f];
    out[n] = (z > 0.0f && z <= z_max) ? z : __int_as_float(0x7fc00000);   // NaN and +inf fail both tests
}

// Eq. (2): with the central differences dz_x, dz_y of the smoothed depth and
// the metric steps dx = 2 z/fx, dy = 2 z/fy at the centre, the normal is
// (0, dy, dz_y) x (dx, 0, dz_x) = (dy dz_x, dx dz_y, -dx dy), normalized
// (camera frame).  s: the smoothed depth at the pixel, rows `row` apart; NaN
// inputs give NaN.
__device__ __forceinline__ float3 depth_normal(const double* s, int row, double fx, double fy) {
    const double c = *s;
    const double dzx = s[1] - s[-1];
    const double dzy = s[row] - s[-row];
    const double dx = 2.0 * c / fx, dy = 2.0 * c / fy;
    const double a = dy * dzx, b = dx * dzy, e = -dx * dy;
    const double inv = 1.0 / sqrt(a * a + b * b + e * e);
    return make_float3((float)(a * inv), (float)(b * inv), (float)(e * inv));
}

// Gaussian smoothing over the valid pixels of the (2R+1)^2 window, weights
// w_a w_b renormalized over them (FP64); an invalid centre stays NaN.  Then
// Eq. (2); NaN on the border and where an input is invalid.
// One workgroup per 32x8 pixels: depths with a border of R + 1 and smoothed
// depths with a border of one stay in LDS (340 smoothed pixels for 256
// normals); the radius is known when compiled, so that a window's loads and
// sums are straight code (latency bounds the pass).  320x240, R = 2: 6.0 us;
// 13.8 us in two launches with the smoothed image in memory.  Windows up to
// R = 5 are written out whole, of larger ones five rows at a time: the products
// of all their weights, kept in registers, leave too few waves (640x480, R = 8:
// 51 us a call, 110 us with 362 registers, 63 us in two launches; 1280x960, R =
// 6: 97, 113 and 129 us, though 320x240 took 17.2 us whole and takes 19.2).
constexpr int kNrmW = 32, kNrmH = 8;
constexpr int kNrmPW = kNrmW + 2 * (RM_MAX_NORMAL_RADIUS + 1), kNrmPH = kNrmH + 2 * (RM_MAX_NORMAL_RADIUS + 1);

constexpr int kUnrolled = 5, kPartUnroll = 5;
template <int R>
constexpr int kRowUnroll = R <= kUnrolled ? 2 * R + 1 : kPartUnroll;

template <int R>
__global__ void __launch_bounds__(kWG) k_depth_normals(const float* __restrict__ depth, int32_t H, int32_t W, GaussW g,
                                                       double fx, double fy, float* __restrict__ nrm) {
    __shared__ float z[kNrmPH * kNrmPW];
    __shared__ double zs[(kNrmH + 2) * (kNrmW + 2)];
    static_assert(kNrmW * kNrmH == kWG, "a thread per normal");
    // (blocks of all rows in one grid dimension: images may be taller than the others reach)
    const unsigned nbx = (unsigned)(W + kNrmW - 1) / kNrmW;
    const int bx = (int)(blockIdx.x % nbx) * kNrmW, by = (int)(blockIdx.x / nbx) * kNrmH;
    const float q = __int_as_float(0x7fc00000);
    const int pw = kNrmW + 2 * (R + 1), ph = kNrmH + 2 * (R + 1), ox = bx - R - 1, oy = by - R - 1;
    for (int p = threadIdx.x; p < pw * ph; p += kWG) {
        const int y = oy + p / pw, x = ox + p % pw;
        z[p] = y >= 0 && y < H && x >= 0 && x < W ? depth[(int64_t)y * W + x] : q;   // (outside: invalid)
    }
    __syncthreads();
    for (int p = threadIdx.x; p < (kNrmH + 2) * (kNrmW + 2); p += kWG) {
        const int y = p / (kNrmW + 2), x = p % (kNrmW + 2);
        const float* c = z + (y + R) * pw + x + R;
        double s = (double)q;
        if (*c == *c) {
            double num = 0.0, den = 0.0;
#pragma unroll kRowUnroll<R>
            for (int a = -R; a <= R; ++a) {
                const double wa = g.w[a + R];
#pragma unroll
                for (int b = -R; b <= R; ++b) {
                    // (an invalid pixel adds +0, which changes neither sum)
                    const float v = c[a * pw + b];
                    const double w = wa * g.w[b + R], t = w * (double)v;
                    num += v == v ? t : 0.0;
                    den += v == v ? w : 0.0;
                }
            }
            s = num / den;
        }
        zs[p] = s;
    }
    __syncthreads();
    const int lx = threadIdx.x % kNrmW, ly = threadIdx.x / kNrmW, x = bx + lx, y = by + ly;
    if (x >= W || y >= H) return;
    float3 o = make_float3(q, q, q);
    if (x > 0 && x < W - 1 && y > 0 && y < H - 1)
        o = depth_normal(zs + (ly + 1) * (kNrmW + 2) + lx + 1, kNrmW + 2, fx, fy);
    float* n = nrm + 3 * ((int64_t)y * W + x);
    n[0] = o.x; n[1] = o.y; n[2] = o.z;
}

// The same in two launches, the smoothed image in memory, for long images that
// fill little of a 32x8 tile (normals_in_two).
__global__ void __launch_bounds__(kWG) k_smooth(const float* __restrict__ depth, int32_t H, int32_t W, GaussW g,
                                                double* __restrict__ out) {
    const int64_t n = (int64_t)blockIdx.x * kWG + threadIdx.x;
    if (n >= (int64_t)H * W) return;
    const int y = (int)(n / W), x = (int)(n % W);
    double s = (double)__int_as_float(0x7fc00000);
    if (depth[n] == depth[n]) {
        double num = 0.0, den = 0.0;
        for (int a = -g.radius; a <= g.radius; ++a) {
            const int yy = y + a;
            if (yy < 0 || yy >= H) continue;
            const double wa = g.w[a + g.radius];
            for (int b = -g.radius; b <= g.radius; ++b) {
                const int xx = x + b;
                if (xx < 0 || xx >= W) continue;
                const float z = depth[(int64_t)yy * W + xx];
                if (!(z == z)) continue;
                const double w = wa * g.w[b + g.radius];
                num += w * (double)z;
                den += w;
            }
        }
        s = num / den;
    }
    out[n] = s;
}

__global__ void __launch_bounds__(kWG) k_normals(const double* __restrict__ zs, int32_t H, int32_t W, double fx, double fy,
                                                 float* __restrict__ nrm) {
    const int64_t n = (int64_t)blockIdx.x * kWG + threadIdx.x;
    if (n >= (int64_t)H * W) return;
    const int y = (int)(n / W), x = (int)(n % W);
    const float q = __int_as_float(0x7fc00000);
    float3 o = make_float3(q, q, q);
    if (x > 0 && x < W - 1 && y > 0 && y < H - 1) o = depth_normal(zs + n, W, fx, fy);
    nrm[3 * n] = o.x; nrm[3 * n + 1] = o.y; nrm[3 * n + 2] = o.z;
}

struct Rot9 { double r[9]; };

// World normal of meshify node (i, j): the camera-frame normal at pixel
// (j s, i s) rotated by the view's rotation, in FP64, rounded to f32.
__global__ void k_vertex_normals(const float* __restrict__ nrm, int32_t W, int32_t s, int32_t gh, int32_t gw,
                                 Rot9 R, float* __restrict__ out) {
    const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= (int64_t)gh * gw) return;
    const int i = (int)(n / gw), j = (int)(n % gw);
    const float* p = nrm + 3 * ((int64_t)(i * s) * W + (int64_t)j * s);
    const double a = p[0], b = p[1], c = p[2];
#pragma unroll
    for (int k = 0; k < 3; ++k) out[3 * n + k] = (float)(R.r[3 * k] * a + R.r[3 * k + 1] * b + R.r[3 * k + 2] * c);
}

unsigned blocks_for(int64_t n) { return (unsigned)((n + kWG - 1) / kWG); }

}  // namespace

hipError_t launch_downsample(hipStream_t st, const float* depth, int32_t H, int32_t W, int32_t f, float z_max,
                             float* out) {
    const int32_t H2 = (H + f - 1) / f, W2 = (W + f - 1) / f;
    hipLaunchKernelGGL(k_downsample, dim3(blocks_for((int64_t)H2 * W2)), dim3(kWG), 0, st, depth, H, W, f, H2, W2,
                       z_max, out);
    return hipGetLastError();
}

// Images of at least 2^16 pixels that are less than 8 pixels wide, or with R > 2
// less than 24 wide or 8 high: 3 x 200,000 pixels take 14 us in two launches
// and 32 in one at R = 0, 59 and 677 at R = 8; 15 x 20,000 13.5 and 12.9 at R = 2,
// 23 and 29 at R = 4; 31 x 9,000 60 and 51 at R = 8; 200,000 x 3 15.0 and 15.4 at
// R = 2, 28 and 106 at R = 8.
bool normals_in_two(int32_t H, int32_t W, int32_t radius) {
    return (int64_t)H * W >= 65536 && (W < 8 || (radius > 2 && (W < 24 || H < 8)));
}

hipError_t launch_depth_normals(hipStream_t st, const float* depth, int32_t H, int32_t W, double fx, double fy,
                                const GaussW& g, double* smoothed, float* normals) {
    if (smoothed) {
        const unsigned nb = blocks_for((int64_t)H * W);
        hipLaunchKernelGGL(k_smooth, dim3(nb), dim3(kWG), 0, st, depth, H, W, g, smoothed);
        hipLaunchKernelGGL(k_normals, dim3(nb), dim3(kWG), 0, st, smoothed, H, W, fx, fy, normals);
        return hipGetLastError();
    }
    const dim3 grid((unsigned)((W + kNrmW - 1) / kNrmW) * (unsigned)((H + kNrmH - 1) / kNrmH));
#define RM_NRM(R)                                                                                                  \
    case R: hipLaunchKernelGGL(k_depth_normals<R>, grid, dim3(kWG), 0, st, depth, H, W, g, fx, fy, normals); break;
    static_assert(RM_MAX_NORMAL_RADIUS == 8, "a kernel per radius");
    switch (g.radius) {
        RM_NRM(0)
        RM_NRM(1)
        RM_NRM(2)
        RM_NRM(3)
        RM_NRM(4)
        RM_NRM(5)
        RM_NRM(6)
        RM_NRM(7)
        RM_NRM(8)
    }
#undef RM_NRM
    return hipGetLastError();
}

hipError_t launch_vertex_normals(hipStream_t st, const float* normals, int32_t H, int32_t W, int32_t stride,
                                 const double* T_wc, float* out) {
    const int32_t gh = (H + stride - 1) / stride, gw = (W + stride - 1) / stride;
    Rot9 R;
    for (int r = 0; r < 3; ++r)
        for (int c = 0; c < 3; ++c) R.r[3 * r + c] = T_wc[4 * r + c];
    hipLaunchKernelGGL(k_vertex_normals, dim3(blocks_for((int64_t)gh * gw)), dim3(kWG), 0, st, normals, W, stride,
                       gh, gw, R, out);
    return hipGetLastError();
}

}  // namespace rm
