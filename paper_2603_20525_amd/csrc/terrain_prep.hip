// Terrain preparation kernels, off the per-plan path (run once per map):
//   * level-of-detail smoothing (section "Terrain Smoothing"): the heightmap
//     convolved with a Gaussian of standard deviation sigma, truncated at
//     r = ceil(3 sigma / res) nodes, clamp-to-edge; the kernel is separable,
//     so it runs as a row pass and a column pass, each staging its tile and
//     halo in LDS (HBM-bound: one read and one write of the grid per pass);
//   * the distance-constraint costmap (sections "OCP Formulation" and
//     "Real-Time Implementation": sdist pre-computed and summed over all
//     features, interpolated at run time): at each node the sum over
//     perimeters of sigma * max(0, 1 - sdist / eps)^2, sdist negative inside
//     an obstacle and outside a path boundary, inside by the even-odd rule.
#include "plan_internal.h"

namespace plan {
namespace {

constexpr int ROW_OUT = 4;                      // outputs per thread, row pass
constexpr int ROW_TILE = 256 * ROW_OUT;         // outputs per workgroup, row pass
constexpr int COL_W = 32;                       // columns per workgroup, column pass
constexpr int COL_RUN = 8;                      // consecutive rows per thread, column pass
constexpr int COL_T = (256 / COL_W) * COL_RUN;  // rows per workgroup, column pass (64)

// Row pass: tmp[j][i] = sum_k w[k] h[j][clamp(i + k - r)], k = 0 .. 2r in
// order. Each thread produces ROW_OUT neighbouring outputs from one sliding
// window of the LDS row tile.
__global__ __launch_bounds__(256) void smooth_rows(const float *__restrict__ h, int W, int H,
                                                   const SmoothTaps taps,
                                                   float *__restrict__ tmp) {
    __shared__ float tile[ROW_TILE + 2 * MAX_SMOOTH_RADIUS];
    const int r = taps.r;
    const int j = blockIdx.y;
    if (j >= H) return;  // whole workgroup (grid rows = H)
    const int i0 = blockIdx.x * ROW_TILE;
    const float *row = h + (size_t)j * W;
    for (int q = threadIdx.x; q < ROW_TILE + 2 * r; q += 256) {
        const int i = min(max(i0 + q - r, 0), W - 1);
        tile[q] = row[i];
    }
    __syncthreads();
    const int base = threadIdx.x * ROW_OUT;  // first output of this thread in the tile
    float acc[ROW_OUT];
#pragma unroll
    for (int o = 0; o < ROW_OUT; ++o) acc[o] = 0.0f;
    float win[ROW_OUT];
#pragma unroll
    for (int o = 0; o < ROW_OUT - 1; ++o) win[o + 1] = tile[base + o];
    for (int k = 0; k <= 2 * r; ++k) {
        // window = tile[base + k .. base + k + ROW_OUT - 1]
#pragma unroll
        for (int o = 0; o < ROW_OUT - 1; ++o) win[o] = win[o + 1];
        win[ROW_OUT - 1] = tile[base + k + ROW_OUT - 1];
        const float w = taps.w[k];
#pragma unroll
        for (int o = 0; o < ROW_OUT; ++o) acc[o] = fmaf(w, win[o], acc[o]);
    }
    float *dst = tmp + (size_t)j * W + i0 + base;
#pragma unroll
    for (int o = 0; o < ROW_OUT; ++o)
        if (i0 + base + o < W) dst[o] = acc[o];
}

// Column pass: out[j][i] = sum_k w[k] tmp[clamp(j + k - r)][i]; a tile of
// COL_T rows x COL_W columns plus the vertical halo is staged in LDS (at most
// 318 x 32 floats, 40.7 KB). Thread t owns column t % COL_W and the COL_RUN
// consecutive rows starting at (t / COL_W) * COL_RUN, swept with a sliding
// window of the column.
__global__ __launch_bounds__(256) void smooth_cols(const float *__restrict__ tmp, int W, int H,
                                                   const SmoothTaps taps,
                                                   float *__restrict__ out) {
    __shared__ float tile[(COL_T + 2 * MAX_SMOOTH_RADIUS) * COL_W];
    const int r = taps.r;
    const int i0 = blockIdx.x * COL_W, j0 = blockIdx.y * COL_T;
    const int rows = COL_T + 2 * r;
    const int c = threadIdx.x & (COL_W - 1);
    const int i = min(i0 + c, W - 1);
    for (int q = threadIdx.x / COL_W; q < rows; q += 256 / COL_W) {
        const int j = min(max(j0 + q - r, 0), H - 1);
        tile[q * COL_W + c] = tmp[(size_t)j * W + i];
    }
    __syncthreads();
    if (i0 + c >= W) return;
    const int t0 = (threadIdx.x / COL_W) * COL_RUN;  // first output row in the tile
    float acc[COL_RUN];
#pragma unroll
    for (int o = 0; o < COL_RUN; ++o) acc[o] = 0.0f;
    float win[COL_RUN];
#pragma unroll
    for (int o = 0; o < COL_RUN - 1; ++o) win[o + 1] = tile[(t0 + o) * COL_W + c];
    for (int k = 0; k <= 2 * r; ++k) {
#pragma unroll
        for (int o = 0; o < COL_RUN - 1; ++o) win[o] = win[o + 1];
        win[COL_RUN - 1] = tile[(t0 + k + COL_RUN - 1) * COL_W + c];
        const float w = taps.w[k];
#pragma unroll
        for (int o = 0; o < COL_RUN; ++o) acc[o] = fmaf(w, win[o], acc[o]);
    }
#pragma unroll
    for (int o = 0; o < COL_RUN; ++o) {
        const int j = j0 + t0 + o;
        if (j < H) out[(size_t)j * W + i0 + c] = acc[o];
    }
}

// Squared distance from (px, py) to the segment a-b (FP32). The root is
// monotonic, so the root of the smallest square is the smallest root.
__device__ __forceinline__ float seg_dist2(float px, float py, float ax, float ay, float bx,
                                           float by) {
    const float ex = bx - ax, ey = by - ay;
    const float len2 = fmaf(ex, ex, ey * ey);
    float t = 0.0f;
    if (len2 > 0.0f) t = fminf(fmaxf(fmaf(px - ax, ex, (py - ay) * ey) / len2, 0.0f), 1.0f);
    const float qx = fmaf(t, ex, ax) - px, qy = fmaf(t, ey, ay) - py;
    return fmaf(qx, qx, qy * qy);
}

// A tile of CM_TILE x CM_TILE nodes per workgroup, CM_ROWS nodes of a column
// per thread. Most tiles lie on the safe side of a perimeter (outside an
// obstacle, inside a path boundary) by more than eps, where every node's term
// is exactly zero, so the workgroup first decides which perimeters can touch
// it and then evaluates those alone, node by node as before and in the order
// of the list: the sums are the same bits. Bound before: the vector ALUs, on
// every node against every edge (2048 x 2048 nodes, 244 edges: 950-990 us);
// now the writes and, per tile, one pass over the edges (the same map: 23 us).
// 32 x 32 nodes keep that pass (one edge per thread and a barrier) small
// against the tile's work while the tile stays small against an obstacle.
constexpr int CM_TILE = 32;
constexpr int CM_BLOCK = 512;
constexpr int CM_ROWS = CM_TILE * CM_TILE / CM_BLOCK;

// Whether the perimeter e's edge a-b can come within reach of the tile with
// centre (cx, cy) and half diagonal rho: a lower bound of the distance of
// every node of the tile from the edge, at least 0 (0 also for a non-finite
// or huge vertex, whose perimeter is then never skipped). The slack, 4e-6 of
// the coordinates' size, is an order of magnitude above the rounding of the
// distances and crossings here and at the nodes.
__device__ __forceinline__ float tile_gap(float cx, float cy, float rho, float2 a, float2 b) {
    const float size = fabsf(cx) + fabsf(cy) + rho + fabsf(a.x) + fabsf(a.y) + fabsf(b.x) +
                       fabsf(b.y);
    const float gap = sqrtf(seg_dist2(cx, cy, a.x, a.y, b.x, b.y)) - rho - 4e-6f * size;
    return size < 1e15f ? fmaxf(gap, 0.0f) : 0.0f;
}

__device__ __forceinline__ bool crosses(float px, float py, float2 v0, float2 v1) {
    if ((v0.y > py) == (v1.y > py)) return false;
    const float xc = v0.x + (py - v0.y) * (v1.x - v0.x) / (v1.y - v0.y);
    return px < xc;
}

__global__ __launch_bounds__(CM_BLOCK) void costmap_polygons(const float2 *__restrict__ verts,
                                                        const PolygonSet ps, int W, int H,
                                                        float x0, float y0, float res,
                                                        float sigma, float eps, float inv_eps,
                                                        int accumulate,
                                                        float *__restrict__ cm) {
    __shared__ int off[MAX_POLYGONS + 1];
    __shared__ unsigned gap[MAX_POLYGONS];     // smallest tile_gap over the perimeter's edges
    __shared__ unsigned parity[MAX_POLYGONS];  // crossings seen from the tile's centre
    __shared__ unsigned long long touched;
    const int tid = threadIdx.x;
    const int i0 = blockIdx.x * CM_TILE, j0 = blockIdx.y * CM_TILE;
    if (tid <= MAX_POLYGONS) off[tid] = ps.offsets[tid];
    if (tid < MAX_POLYGONS) {
        gap[tid] = 0x7f800000u;  // +inf
        parity[tid] = 0u;
    }
    __syncthreads();
    {
        // the tile as its centre and half diagonal, from its corner nodes
        const float xa = fmaf((float)i0, res, x0), ya = fmaf((float)j0, res, y0);
        const float xb = fmaf((float)min(i0 + CM_TILE - 1, W - 1), res, x0);
        const float yb = fmaf((float)min(j0 + CM_TILE - 1, H - 1), res, y0);
        const float cx = 0.5f * (xa + xb), cy = 0.5f * (ya + yb);
        const float hx = 0.5f * (xb - xa), hy = 0.5f * (yb - ya);
        const float rho = sqrtf(fmaf(hx, hx, hy * hy));
        const int V = ps.count > 0 ? off[ps.count] : 0;
        for (int e = tid; e < V; e += CM_BLOCK) {
            int lo = 0, hi = ps.count - 1;  // the perimeter of vertex e
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (off[mid] <= e)
                    lo = mid;
                else
                    hi = mid - 1;
            }
            const float2 v1 = verts[e], v0 = verts[e == off[lo] ? off[lo + 1] - 1 : e - 1];
            // distances are >= 0, so their bits order as the values do
            atomicMin(&gap[lo], __float_as_uint(tile_gap(cx, cy, rho, v0, v1)));
            if (crosses(cx, cy, v0, v1)) atomicXor(&parity[lo], 1u);
        }
    }
    __syncthreads();
    if (tid < 64) {
        // beyond eps of every edge, all nodes are on the centre's side: the
        // term is zero outside an obstacle and inside a path boundary
        bool touch = tid < ps.count;
        if (touch) {
            const bool safe = (parity[tid] != 0u) == (ps.kinds[tid] == 1);
            touch = !(safe && __uint_as_float(gap[tid]) > 1.00001f * eps);
        }
        const unsigned long long m = __ballot(touch);
        if (tid == 0) touched = m;
    }
    __syncthreads();
    const int i = i0 + (tid & (CM_TILE - 1)), jt = j0 + tid / CM_TILE;
    const float px = fmaf((float)i, res, x0);
    float py[CM_ROWS], c[CM_ROWS];
#pragma unroll
    for (int q = 0; q < CM_ROWS; ++q) {
        py[q] = fmaf((float)(jt + q * (CM_BLOCK / CM_TILE)), res, y0);
        c[q] = 0.0f;
    }
    unsigned long long todo = touched;
    // wave-uniform, in scalar registers
    todo = ((unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((int)(todo >> 32)) << 32) |
           (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)todo);
    while (todo) {
        const int p = __builtin_ctzll(todo);
        todo &= todo - 1;
        const int a = ps.offsets[p], m = ps.offsets[p + 1] - a;
        float dmin[CM_ROWS];
        bool inside[CM_ROWS];
#pragma unroll
        for (int q = 0; q < CM_ROWS; ++q) {
            dmin[q] = __builtin_inff();
            inside[q] = false;
        }
        float2 v0 = verts[a + m - 1];
        for (int e = 0; e < m; ++e) {
            const float2 v1 = verts[a + e];
#pragma unroll
            for (int q = 0; q < CM_ROWS; ++q) {
                dmin[q] = fminf(dmin[q], seg_dist2(px, py[q], v0.x, v0.y, v1.x, v1.y));
                if (crosses(px, py[q], v0, v1)) inside[q] = !inside[q];
            }
            v0 = v1;
        }
#pragma unroll
        for (int q = 0; q < CM_ROWS; ++q) {
            // obstacle: negative inside; path boundary: negative outside
            const float d = sqrtf(dmin[q]);
            const float sd = (inside[q] == (ps.kinds[p] == 0)) ? -d : d;
            const float mm = fmaxf(0.0f, fmaf(-sd, inv_eps, 1.0f));
            c[q] = fmaf(sigma * mm, mm, c[q]);
        }
    }
    if (i >= W) return;
#pragma unroll
    for (int q = 0; q < CM_ROWS; ++q) {
        const int j = jt + q * (CM_BLOCK / CM_TILE);
        if (j >= H) break;
        const size_t o = (size_t)j * W + i;
        cm[o] = accumulate ? cm[o] + c[q] : c[q];
    }
}

}  // namespace

hipError_t launch_smooth(const float *h, int W, int H, const SmoothTaps &taps, float *tmp,
                         float *out, hipStream_t s) {
    hipLaunchKernelGGL(smooth_rows, dim3((W + ROW_TILE - 1) / ROW_TILE, H), dim3(256), 0, s, h, W,
                       H, taps, tmp);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(smooth_cols, dim3((W + COL_W - 1) / COL_W, (H + COL_T - 1) / COL_T),
                       dim3(256), 0, s, tmp, W, H, taps, out);
    return hipGetLastError();
}

hipError_t launch_costmap_polygons(const float *verts, const PolygonSet &ps, int W, int H,
                                   float x0, float y0, float res, float sigma, float eps,
                                   int accumulate, float *cm, hipStream_t s) {
    dim3 grid((W + CM_TILE - 1) / CM_TILE, (H + CM_TILE - 1) / CM_TILE);
    hipLaunchKernelGGL(costmap_polygons, grid, dim3(CM_BLOCK), 0, s, (const float2 *)verts, ps, W, H,
                       x0, y0, res, sigma, eps, 1.0f / eps, accumulate, cm);
    return hipGetLastError();
}

}  // namespace plan
