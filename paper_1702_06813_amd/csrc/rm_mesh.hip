// Scan image, meshification and cluster bounds (Sec. IV-A of the paper).
#include "rm_internal.h"

namespace rm {

namespace {

enum { kDead = 0, kNoReturn = 1, kValid = 2 };

// Range pixel class: dead (NaN, negative, or a positive range below z_min),
// no-return (0, +inf, or beyond z_max: free space up to the sensor maximum),
// or valid.
__device__ __forceinline__ int range_class(float z, float z_min, float z_max) {
    if (isnan(z) || z < 0.0f) return kDead;
    if (z == 0.0f || isinf(z) || z > z_max) return kNoReturn;
    if (z < z_min) return kDead;
    return kValid;
}

__global__ void k_scan_image(const float* __restrict__ depth, int64_t n, float z_min, float z_max,
                             float* __restrict__ d_out, uint8_t* __restrict__ c_out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float z = depth[i];
    const int k = range_class(z, z_min, z_max);
    d_out[i] = k == kValid ? z : (k == kNoReturn ? z_max : __int_as_float(0x7fc00000));
    c_out[i] = k == kValid ? RM_FO : (k == kNoReturn ? RM_FU : RM_NONE);
}

struct Pose12 { double m[12]; };

// Grid node (i, j) sits at pixel (j*s, i*s).  A valid node's depth is the
// FP64 mean of the valid pixels of the (2R+1)^2 window around it whose depth
// is within RM_SMOOTH_REL of the node pixel's (R = 0: the node pixel); the
// kept depths differ by 3 % at most, so their FP64 sum (at most 1,089 of them)
// is exact and its order free.  Back-projection in FP64 at that depth (z_max
// for a no-return), world transform in FP64, one rounding to f32 at the end.
// Dead nodes get NaN.  G lanes share a node's window, row by row.
struct MeshArgs {
    const float* depth;
    int32_t H, W, s, R, gh, gw;
    float fx, fy, cx, cy, z_min, z_max;
    Pose12 T;
};

// WIN: depths are averaged over the window.
template <int G, bool WIN>
__device__ __forceinline__ int mesh_node(const MeshArgs& m, int i, int j, int sub, float out[3]) {
    const int py = i * m.s, px = j * m.s;
    const float z = m.depth[(int64_t)py * m.W + px];
    const int k = range_class(z, m.z_min, m.z_max);
    double zd = (k == kNoReturn) ? (double)m.z_max : (double)z;
    if (WIN) {
        const double zc = (double)z, tol = RM_SMOOTH_REL * zc;
        double sum = 0.0;
        int cnt = 0;
        if (k == kValid)
            for (int yy = max(py - m.R, 0) + sub; yy <= min(py + m.R, m.H - 1); yy += G) {
                const int x1 = min(px + m.R, m.W - 1);
#pragma unroll 4
                for (int xx = max(px - m.R, 0); xx <= x1; ++xx) {
                    const float zn = m.depth[(int64_t)yy * m.W + xx];
                    // (valid, without branches; NaN fails every test)
                    const bool in = (zn > 0.0f) & (zn >= m.z_min) & (zn <= m.z_max) & (fabs((double)zn - zc) <= tol);
                    sum += in ? (double)zn : 0.0;
                    cnt += in;
                }
            }
#pragma unroll
        for (int off = G / 2; off > 0; off >>= 1) {
            sum += __shfl_xor(sum, off);
            cnt += __shfl_xor(cnt, off);
        }
        if (k == kValid) zd = sum / (double)cnt;
    }
    const double xc = zd * (((double)px - (double)m.cx) / (double)m.fx);
    const double yc = zd * (((double)py - (double)m.cy) / (double)m.fy);
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        const double w = ((m.T.m[4 * r] * xc + m.T.m[4 * r + 1] * yc) + m.T.m[4 * r + 2] * zd) + m.T.m[4 * r + 3];
        out[r] = k == kDead ? __int_as_float(0x7fc00000) : (float)w;
    }
    return k;
}

// Quad between the nodes c[0..3] in perimeter order: dropped (keep = false) with
// a dead corner, free-unknown (fu) with a no-return corner or a side beyond the
// limit.  kind(n), pos(n): a node's class and world position.
template <typename I, typename Kind, typename Pos>
__device__ __forceinline__ void quad_test(const I (&c)[4], Kind kind, Pos pos, double lim2, bool& keep, bool& fu) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int kk = kind(c[k]);
        keep &= kk != kDead;
        fu |= kk == kNoReturn;
        const float* p = pos(c[k]);
        const float* q = pos(c[(k + 1) & 3]);
        const double dx = (double)p[0] - (double)q[0];
        const double dy = (double)p[1] - (double)q[1];
        const double dz = (double)p[2] - (double)q[2];
        fu |= ((dx * dx + dy * dy) + dz * dz) > lim2;
    }
}

// Nodes without windows: one workgroup per 8x8 block of quads computes the
// nodes of its 9x9 corners (a corner on a shared side is computed by each block
// that needs it and written by the one to its lower right), then a wave
// classifies the quads, lane = row*8 + col.  masks[2 blk] = quads kept,
// masks[2 blk + 1] = free-unknown ones.  Latency sets the time of small grids,
// and one launch less counts: a view of 300 blocks takes 31 us whole, 33 us
// with launches of their own for nodes and quads.
constexpr int kNodeSide = kQuadBlock + 1;

__global__ void __launch_bounds__(kWG) k_mesh_block(MeshArgs m, int bw, double lim2, float* __restrict__ xyz,
                                                    uint64_t* __restrict__ masks) {
    __shared__ float v[kNodeSide * kNodeSide][3];
    __shared__ int kind[kNodeSide * kNodeSide];
    constexpr int kNodes = kNodeSide * kNodeSide;
    static_assert(kNodes <= kWG, "a thread per node");
    const int blk = blockIdx.x;
    const int i0 = blk / bw * kQuadBlock, j0 = blk % bw * kQuadBlock;
    const int n = threadIdx.x, na = n / kNodeSide, nb = n % kNodeSide, i = i0 + na, j = j0 + nb;
    if (n < kNodes && i < m.gh && j < m.gw) {
        float p[3];
        kind[n] = mesh_node<1, false>(m, i, j, 0, p);
#pragma unroll
        for (int r = 0; r < 3; ++r) v[n][r] = p[r];
        if ((na < kQuadBlock || i == m.gh - 1) && (nb < kQuadBlock || j == m.gw - 1)) {
            float* o = xyz + 3 * ((int64_t)i * m.gw + j);
#pragma unroll
            for (int r = 0; r < 3; ++r) o[r] = p[r];
        }
    }
    __syncthreads();
    if (threadIdx.x >= 64) return;
    const int lane = threadIdx.x, a = lane / kQuadBlock, b = lane % kQuadBlock;
    bool keep = i0 + a < m.gh - 1 && j0 + b < m.gw - 1, fu = false;
    const int n00 = a * kNodeSide + b;
    const int c[4] = {n00, n00 + 1, n00 + kNodeSide + 1, n00 + kNodeSide};   // perimeter order
    if (keep) quad_test(c, [&](int n) { return kind[n]; }, [&](int n) { return v[n]; }, lim2, keep, fu);
    const uint64_t mk = __ballot(keep), mf = __ballot(keep && fu);
    if (lane == 0) { masks[2 * (int64_t)blk] = mk; masks[2 * (int64_t)blk + 1] = mf; }
}

// Nodes by themselves, G lanes each: all that have windows, large grids, and
// grids without quads (a single row or column of nodes; kind null, the triangle
// total is zero).
template <int G, bool WIN>
__global__ void __launch_bounds__(kWG) k_mesh_nodes(MeshArgs m, float* __restrict__ xyz, uint8_t* __restrict__ kind,
                                                    int32_t* __restrict__ total) {
    const int64_t t = (int64_t)blockIdx.x * kWG + threadIdx.x, n = t / G;
    if (!kind && t == 0) *total = 0;
    if (n >= (int64_t)m.gh * m.gw) return;
    float p[3];
    const int k = mesh_node<G, WIN>(m, (int)(n / m.gw), (int)(n % m.gw), (int)(t % G), p);
    if (t % G) return;
    if (kind) kind[n] = (uint8_t)k;
#pragma unroll
    for (int r = 0; r < 3; ++r) xyz[3 * n + r] = p[r];
}

// A window's rows go to as many lanes as leave the launch within about half a
// million threads: 9x9 windows of 300 / 1,200 / 2,451 / 4,800 blocks take 35.9 /
// 43.9 / 49.7 / 73.5 us a view with eight lanes, 36.2 / 39.5 / 45.2 / 60.2 with
// two and 38.6 / 41.9 / 46.2 / 58.5 with one; 33x33 windows of 300 / 2,451 /
// 4,800 blocks 58 / 127 / 326, 66 / 118 / 212 and 94 / 130 / 181 us.  Whole
// blocks in one workgroup with their windows staged in LDS took 38 / 45 / 54 /
// 77 and 64 / 134 / 222 us: corners on shared sides computed twice to four
// times, and at large strides more pixels staged than used.
constexpr int64_t kEightLanes = 512, kTwoLanes = 4096;

// The masks of k_mesh_block from nodes in memory, a wave per block of quads;
// counts (may be null): its triangles.
__global__ void __launch_bounds__(kWG) k_mesh_quads(const float* __restrict__ xyz, const uint8_t* __restrict__ kind,
                                                    int gh, int gw, int bw, int64_t n_blocks, double lim2,
                                                    uint64_t* __restrict__ masks, int32_t* __restrict__ counts) {
    const int64_t blk = (int64_t)blockIdx.x * (kWG / 64) + threadIdx.x / 64;
    const int lane = threadIdx.x & 63;
    if (blk >= n_blocks) return;
    const int qi = (int)(blk / bw) * kQuadBlock + lane / kQuadBlock, qj = (int)(blk % bw) * kQuadBlock + lane % kQuadBlock;
    bool keep = qi < gh - 1 && qj < gw - 1, fu = false;
    const int64_t n00 = (int64_t)qi * gw + qj;
    const int64_t c[4] = {n00, n00 + 1, n00 + gw + 1, n00 + gw};
    if (keep) quad_test(c, [&](int64_t n) { return (int)kind[n]; }, [&](int64_t n) { return xyz + 3 * n; }, lim2, keep, fu);
    const uint64_t mk = __ballot(keep), mf = __ballot(keep && fu);
    if (lane == 0) {
        masks[2 * blk] = mk;
        masks[2 * blk + 1] = mf;
        if (counts) counts[blk] = 2 * __popcll(mk);
    }
}

// Exclusive prefix sum of the block counts in place (one workgroup of 1024
// threads), for grids of more than kDirectBlocks blocks.
constexpr int64_t kDirectBlocks = 4096;

__global__ void k_mesh_scan(int32_t* __restrict__ offsets, int64_t n) {
    __shared__ int64_t part[1024];
    const int t = threadIdx.x;
    const int64_t per = (n + 1023) / 1024;
    const int64_t b = t * per, e = b + per < n ? b + per : n;
    int64_t s = 0;
    for (int64_t k = b; k < e; ++k) s += offsets[k];
    part[t] = s;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        const int64_t v = t >= off ? part[t - off] : 0;
        __syncthreads();
        part[t] += v;
        __syncthreads();
    }
    int64_t run = part[t] - s;
    for (int64_t k = b; k < e; ++k) {
        const int32_t c = offsets[k];
        offsets[k] = (int32_t)run;
        run += c;
    }
}

// Triangles of four blocks per workgroup, a wave each.  Without offsets
// (grids of up to kDirectBlocks blocks) each workgroup sums the counts before
// its own blocks, which is cheaper than a launch of its own.  The last wave
// writes the total to pinned host memory.
__global__ void __launch_bounds__(kWG) k_mesh_emit(const uint64_t* __restrict__ masks, int gw, int bw, int64_t n_blocks,
                                                   const int32_t* __restrict__ offsets, int64_t cap_t,
                                                   int32_t* __restrict__ tri, uint8_t* __restrict__ cls,
                                                   int32_t* __restrict__ total) {
    __shared__ int part[kWG / 64];
    const int wave = threadIdx.x / 64, lane = threadIdx.x & 63;
    const int64_t b0 = (int64_t)blockIdx.x * (kWG / 64), blk = b0 + wave;
    int64_t base = 0;
    if (!offsets) {
        int s = 0;
        for (int64_t k = threadIdx.x; k < b0; k += kWG) s += 2 * __popcll(masks[2 * k]);
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
        if (lane == 0) part[wave] = s;
        __syncthreads();
        base = part[0] + part[1] + part[2] + part[3];
        for (int64_t k = b0; k < min(blk, n_blocks); ++k) base += 2 * __popcll(masks[2 * k]);
    }
    if (blk >= n_blocks) return;
    if (offsets) base = offsets[blk];
    const uint64_t m = masks[2 * blk], mf = masks[2 * blk + 1];
    if (blk == n_blocks - 1 && lane == 0) *total = (int32_t)(base + 2 * __popcll(m));
    if (!((m >> lane) & 1)) return;
    const int qi = (int)(blk / bw) * kQuadBlock + lane / kQuadBlock;
    const int qj = (int)(blk % bw) * kQuadBlock + lane % kQuadBlock;
    const int64_t t0 = base + 2 * __popcll(m & ((1ull << lane) - 1ull));
    if (t0 + 2 > cap_t) return;                 // host reports RM_ERR_CAPACITY from the total
    const int32_t n00 = qi * gw + qj, n01 = n00 + 1, n10 = n00 + gw, n11 = n10 + 1;
    const uint8_t c = (mf >> lane) & 1 ? RM_FU : RM_FO;
    tri[3 * t0] = n00; tri[3 * t0 + 1] = n01; tri[3 * t0 + 2] = n11;
    tri[3 * t0 + 3] = n00; tri[3 * t0 + 4] = n11; tri[3 * t0 + 5] = n10;
    cls[t0] = c;
    cls[t0 + 1] = c;
}

// Cluster bounds: one workgroup per cluster of kClusterTris triangles.
__global__ void __launch_bounds__(kWG) k_clusters(const float* __restrict__ xyz, uint32_t vmax,
                                                  const int32_t* __restrict__ tri, int64_t n_tris,
                                                  ClusterBounds* __restrict__ out) {
    __shared__ float red[6][kWG / 64];
    const int64_t t = (int64_t)blockIdx.x * kClusterTris + threadIdx.x;
    float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    if (t < n_tris) {
        for (int k = 0; k < 3; ++k) {
            const float* p = xyz + 3 * (int64_t)min((uint32_t)tri[3 * t + k], vmax);
            for (int d = 0; d < 3; ++d) { lo[d] = fminf(lo[d], p[d]); hi[d] = fmaxf(hi[d], p[d]); }
        }
    }
    for (int off = 32; off > 0; off >>= 1)
        for (int d = 0; d < 3; ++d) {
            lo[d] = fminf(lo[d], __shfl_xor(lo[d], off));
            hi[d] = fmaxf(hi[d], __shfl_xor(hi[d], off));
        }
    const int w = threadIdx.x / 64;
    if ((threadIdx.x & 63) == 0)
        for (int d = 0; d < 3; ++d) { red[d][w] = lo[d]; red[3 + d][w] = hi[d]; }
    __syncthreads();
    if (threadIdx.x == 0) {
        ClusterBounds b;
        for (int d = 0; d < 3; ++d) {
            float l = red[d][0], h = red[3 + d][0];
            for (int k = 1; k < kWG / 64; ++k) { l = fminf(l, red[d][k]); h = fmaxf(h, red[3 + d][k]); }
            b.lo[d] = l; b.hi[d] = h;
        }
        const int64_t rem = n_tris - (int64_t)blockIdx.x * kClusterTris;
        b.n_tris = (int32_t)(rem < kClusterTris ? rem : kClusterTris);
        b.pad = 0;
        out[blockIdx.x] = b;
    }
}

// World-frame unit normal of every triangle: cross product of the FP32
// vertices' differences in FP64, normalized, rounded to f32.
__global__ void k_normals(const float* __restrict__ xyz, uint32_t vmax, const int32_t* __restrict__ tri,
                          int64_t n_tris, float* __restrict__ nrm) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n_tris) return;
    const float* p0 = xyz + 3 * (int64_t)min((uint32_t)tri[3 * t], vmax);
    const float* p1 = xyz + 3 * (int64_t)min((uint32_t)tri[3 * t + 1], vmax);
    const float* p2 = xyz + 3 * (int64_t)min((uint32_t)tri[3 * t + 2], vmax);
    const double ax = (double)p1[0] - p0[0], ay = (double)p1[1] - p0[1], az = (double)p1[2] - p0[2];
    const double bx = (double)p2[0] - p0[0], by = (double)p2[1] - p0[1], bz = (double)p2[2] - p0[2];
    const double nx = ay * bz - az * by, ny = az * bx - ax * bz, nz = ax * by - ay * bx;
    const double l = sqrt(nx * nx + ny * ny + nz * nz);
    const double il = l > 0.0 ? 1.0 / l : 0.0;
    nrm[3 * t] = (float)(nx * il);
    nrm[3 * t + 1] = (float)(ny * il);
    nrm[3 * t + 2] = (float)(nz * il);
}

__global__ void k_zero_i32(int32_t* p, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

}  // namespace

int64_t meshify_blocks(int32_t H, int32_t W, int32_t stride) {
    const int64_t gh = (H + stride - 1) / stride, gw = (W + stride - 1) / stride;
    const int64_t qh = gh > 1 ? gh - 1 : 0, qw = gw > 1 ? gw - 1 : 0;
    return ((qh + kQuadBlock - 1) / kQuadBlock) * ((qw + kQuadBlock - 1) / kQuadBlock);
}

hipError_t launch_scan_image(hipStream_t st, const float* depth, int32_t H, int32_t W, float z_min,
                             float z_max, float* d_out, uint8_t* c_out) {
    const int64_t n = (int64_t)H * W;
    hipLaunchKernelGGL(k_scan_image, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, depth, n, z_min,
                       z_max, d_out, c_out);
    return hipGetLastError();
}

hipError_t launch_meshify(hipStream_t st, const float* depth, rm_camera cam, const double* T,
                          int32_t stride, int32_t smooth_radius, float z_min, float z_max, float max_edge,
                          float* xyz, int32_t* tri, uint8_t* cls, int64_t cap_t, uint64_t* masks,
                          uint8_t* kind, int32_t* block_offsets, int32_t* total) {
    MeshArgs m;
    m.depth = depth;
    m.H = cam.height; m.W = cam.width; m.s = stride; m.R = smooth_radius;
    m.gh = (cam.height + stride - 1) / stride; m.gw = (cam.width + stride - 1) / stride;
    m.fx = cam.fx; m.fy = cam.fy; m.cx = cam.cx; m.cy = cam.cy;
    m.z_min = z_min; m.z_max = z_max;
    for (int k = 0; k < 12; ++k) m.T.m[k] = T[k];
    const int64_t nn = (int64_t)m.gh * m.gw;
    const int64_t nb = meshify_blocks(m.H, m.W, stride);
    const int bw = (m.gw - 1 + kQuadBlock - 1) / kQuadBlock;
    const double lim2 = (double)max_edge * (double)max_edge;
    auto blocks = [&](int lanes) { return dim3((unsigned)((lanes * nn + kWG - 1) / kWG)); };
    if (nb == 0) {
        hipLaunchKernelGGL((k_mesh_nodes<8, true>), blocks(8), dim3(kWG), 0, st, m, xyz, (uint8_t*)nullptr, total);
        return hipGetLastError();
    }
    const bool direct = nb <= kDirectBlocks;
    const dim3 waves((unsigned)((nb + 3) / 4));
    if (smooth_radius == 0 && direct) {
        hipLaunchKernelGGL(k_mesh_block, dim3((unsigned)nb), dim3(kWG), 0, st, m, bw, lim2, xyz, masks);
    } else {
        if (smooth_radius == 0) hipLaunchKernelGGL((k_mesh_nodes<1, false>), blocks(1), dim3(kWG), 0, st, m, xyz, kind, total);
        else if (nb <= kEightLanes) hipLaunchKernelGGL((k_mesh_nodes<8, true>), blocks(8), dim3(kWG), 0, st, m, xyz, kind, total);
        else if (nb <= kTwoLanes) hipLaunchKernelGGL((k_mesh_nodes<2, true>), blocks(2), dim3(kWG), 0, st, m, xyz, kind, total);
        else hipLaunchKernelGGL((k_mesh_nodes<1, true>), blocks(1), dim3(kWG), 0, st, m, xyz, kind, total);
        hipLaunchKernelGGL(k_mesh_quads, waves, dim3(kWG), 0, st, xyz, kind, m.gh, m.gw, bw, nb, lim2, masks,
                           direct ? nullptr : block_offsets);
    }
    if (!direct) hipLaunchKernelGGL(k_mesh_scan, dim3(1), dim3(1024), 0, st, block_offsets, nb);
    hipLaunchKernelGGL(k_mesh_emit, waves, dim3(kWG), 0, st, masks, m.gw, bw, nb,
                       direct ? nullptr : block_offsets, cap_t, tri, cls, total);
    return hipGetLastError();
}

int64_t prepared_normals_offset(int64_t n_tris) {
    const int64_t nc = (n_tris + kClusterTris - 1) / kClusterTris;
    return (nc * (int64_t)sizeof(ClusterBounds) + 255) & ~(int64_t)255;
}

hipError_t launch_prepare(hipStream_t st, const float* xyz, int64_t n_vertices, const int32_t* tri,
                          int64_t n_tris, void* out) {
    const int64_t nc = (n_tris + kClusterTris - 1) / kClusterTris;
    if (nc == 0 || n_vertices < 1) return hipSuccess;
    const uint32_t vmax = (uint32_t)(n_vertices - 1);
    hipLaunchKernelGGL(k_clusters, dim3((unsigned)nc), dim3(kWG), 0, st, xyz, vmax, tri, n_tris,
                       static_cast<ClusterBounds*>(out));
    float* nrm = reinterpret_cast<float*>(static_cast<char*>(out) + prepared_normals_offset(n_tris));
    hipLaunchKernelGGL(k_normals, dim3((unsigned)((n_tris + 255) / 256)), dim3(256), 0, st, xyz, vmax, tri, n_tris,
                       nrm);
    return hipGetLastError();
}

hipError_t launch_zero_i32(hipStream_t st, int32_t* p, int64_t n) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_zero_i32, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, p, n);
    return hipGetLastError();
}

}  // namespace rm
