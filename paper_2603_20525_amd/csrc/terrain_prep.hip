// Terrain preparation kernels, off the per-plan path (run once per map):
//   * level-of-detail smoothing (section "Terrain Smoothing"): the heightmap
//     convolved with a Gaussian of standard deviation sigma, truncated at
//     r = ceil(3 sigma / res) nodes, clamp-to-edge; the kernel is separable,
//     so it runs as a row pass and a column pass, in one kernel or two, each
//     staging its tile and halo in LDS;
//   * the distance-constraint costmap (sections "OCP Formulation" and
//     "Real-Time Implementation": sdist pre-computed and summed over all
//     features, interpolated at run time): at each node the sum over
//     perimeters of sigma * max(0, 1 - sdist / eps)^2, sdist negative inside
//     an obstacle and outside a path boundary, inside by the even-odd rule.
#include "launch_rules.h"
#include "plan_internal.h"

namespace plan {
namespace {

// Both smoothing passes are products with a banded Toeplitz matrix of the
// taps, on the matrix cores: an output tile of 16 x 16 is the sum over K steps
// of v_mfma_f32_16x16x4_f32, four inputs of the window a step. That
// instruction adds its four products one after the other in ascending k, each
// with one rounding (measured equal to a chain of fmaf for every one of
// 512 000 results), and the zeros around the band add nothing to a finite
// window, so the sums are the bits of the scalar loop
//   acc = fmaf(w[k], x[k], acc), k = 0 .. 2r,
// except the sign of a zero that underflow leaves (of heights around 1e-41). A
// workgroup still runs that loop where its windows hold an infinity or a NaN,
// whose product with the band's zeros would spread. 16 x 16 wastes 15 of
// 2r + 16 columns of the band (32 x 32 twice that) and takes half the cycles of
// vector fused multiply-adds. Bound: the matrix cores at large sigma, the
// grid's reads and writes at small.
// Measured, both passes, before (register windows on the vector ALUs) and
// now: 2048 x 2048 nodes at 19, 37 and 181 taps 27.1, 33.4 and 86.2 us ->
// 17.3, 22.1 and 48.3 us; 1537 x 1025 at 181 taps 52.7 -> 33.2 us.
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int ROW_H = 16;    // rows per workgroup, row pass
constexpr int ROW_W = 256;   // columns per workgroup, row pass (four tiles a wave)
constexpr int COL_W = 32;    // columns per workgroup, column pass
constexpr int COL_H = 128;   // rows per workgroup, column pass (two by two tiles a wave)

// K steps of a window of 2r + 1 taps sliding over 16 outputs.
__host__ __device__ constexpr int smooth_steps(int r) { return (2 * r + 16 + 3) / 4; }
constexpr int MAX_SMOOTH_STEPS = smooth_steps(MAX_SMOOTH_RADIUS);
constexpr int BAND = 4 * MAX_SMOOTH_STEPS + 16;

// Row stride of the row pass's tile in LDS: 2 mod 32, so that the 16 rows x 2
// columns that half a wave reads fall on 32 banks.
__host__ __device__ constexpr int row_stride(int r) {
    return (ROW_W + 4 * smooth_steps(r) - 16 + 29) / 32 * 32 + 2;
}

// band[q] = w[q - 15], zero outside the taps: output n of a tile weighs input
// k (counted from the tile's first window) with band[k - n + 15].
template <int BLOCK>
__device__ __forceinline__ void load_band(const SmoothTaps &taps, float *band) {
    for (int q = threadIdx.x; q < BAND; q += BLOCK) {
        const int k = q - 15;
        band[q] = (k >= 0 && k <= 2 * taps.r) ? taps.w[k] : 0.0f;
    }
}

// Four neighbouring nodes, starting at any.
typedef float quad_t __attribute__((ext_vector_type(4), aligned(4)));

// 0 for finite values, NaN once a value was not: 0 x is NaN for those alone.
__device__ __forceinline__ float chain_zero(float v, float z) { return fmaf(v, 0.0f, z); }

// Row pass: tmp[j][i] = sum_k w[k] h[j][clamp(i + k - r)].
__global__ __launch_bounds__(256) void smooth_rows(const float *__restrict__ h, int W, int H,
                                                   const SmoothTaps taps,
                                                   float *__restrict__ tmp) {
    extern __shared__ float lds[];
    __shared__ float band[BAND];
    const int r = taps.r, steps = smooth_steps(r), stride = row_stride(r);
    const int i0 = blockIdx.x * ROW_W, j0 = blockIdx.y * ROW_H;
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int width = ROW_W + 4 * steps - 16;  // inputs of the tile's windows and steps
    load_band<256>(taps, band);
    float zero = 0.0f;
    const bool inner = i0 >= r && i0 - r + width <= W;
    // this wave's four rows, eight loads in flight a lane
    for (int q0 = lane; q0 < width; q0 += 128) {
        float v[2][4];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int i = i0 - r + q0 + 64 * u;
            const int ic = inner ? min(i, W - 1) : min(max(i, 0), W - 1);
#pragma unroll
            for (int p = 0; p < 4; ++p) v[u][p] = h[(size_t)min(j0 + wv + 4 * p, H - 1) * W + ic];
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            if (q0 + 64 * u >= width) break;
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                zero = chain_zero(v[u][p], zero);
                lds[(wv + 4 * p) * stride + q0 + 64 * u] = v[u][p];
            }
        }
    }
    if (__syncthreads_or(zero != 0.0f)) {
        for (int row = wv; row < ROW_H && j0 + row < H; row += 4)
            for (int q = lane; q < ROW_W && i0 + q < W; q += 64) {
                float acc = 0.0f;
                for (int k = 0; k <= 2 * r; ++k)
                    acc = fmaf(taps.w[k], lds[row * stride + q + k], acc);
                tmp[(size_t)(j0 + row) * W + i0 + q] = acc;
            }
        return;
    }
    // A = heights (row lane % 16, input 4 s + lane / 16), B = band
    const int m = lane & 15, g = lane >> 4;
    const float *in = lds + m * stride + 64 * wv + g;
    const float *bw = band + g - m + 15;
    f32x4 acc[4] = {};
    float w = bw[0], x[4] = {in[0], in[16], in[32], in[48]};
    for (int s = 0; s < steps; ++s) {
        // the next step's operands are read under this step's products (the
        // last step reads its own again)
        const int n = 4 * min(s + 1, steps - 1);
        const float wn = bw[n];
        float xn[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) xn[t] = in[16 * t + n];
#pragma unroll
        for (int t = 0; t < 4; ++t)
            acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[t], w, acc[t], 0, 0, 0);
        w = wn;
#pragma unroll
        for (int t = 0; t < 4; ++t) x[t] = xn[t];
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const int i = i0 + 64 * wv + 16 * t + m;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int j = j0 + 4 * g + q;
            if (i < W && j < H) tmp[(size_t)j * W + i] = acc[t][q];
        }
    }
}

// Column pass: out[j][i] = sum_k w[k] tmp[clamp(j + k - r)][i]. A tile of
// COL_H rows and its halo, COL_W columns wide, in LDS; odd rows are stored
// with their two halves swapped, so that the two rows of 16 columns that half
// a wave reads fall on 32 banks.
__global__ __launch_bounds__(256) void smooth_cols(const float *__restrict__ tmp, int W, int H,
                                                   const SmoothTaps taps,
                                                   float *__restrict__ out) {
    extern __shared__ float lds[];
    __shared__ float band[BAND];
    const int r = taps.r, steps = smooth_steps(r);
    const int i0 = blockIdx.x * COL_W, j0 = blockIdx.y * COL_H;
    const int rows = COL_H + 4 * steps - 16;
    load_band<256>(taps, band);
    float zero = 0.0f;
    {
        // four columns of a row a thread, eight loads in flight
        constexpr int PER = COL_W / 4, STEP = 256 / PER;
        const int c = 4 * (threadIdx.x % PER);
        const bool inner = i0 + COL_W <= W;
        for (int q0 = threadIdx.x / PER; q0 < rows; q0 += 8 * STEP) {
            quad_t v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                if (q0 + u * STEP >= rows) break;
                const float *src = tmp + (size_t)min(max(j0 + q0 + u * STEP - r, 0), H - 1) * W;
                if (inner) {
                    v[u] = *reinterpret_cast<const quad_t *>(src + i0 + c);
                } else {
                    const int i = i0 + c;
                    v[u] = quad_t{src[min(i, W - 1)], src[min(i + 1, W - 1)],
                                  src[min(i + 2, W - 1)], src[min(i + 3, W - 1)]};
                }
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int q = q0 + u * STEP;
                if (q >= rows) break;
                zero = chain_zero(v[u].x, chain_zero(v[u].y, zero));
                zero = chain_zero(v[u].z, chain_zero(v[u].w, zero));
                *reinterpret_cast<float4 *>(lds + q * COL_W + (c ^ ((q & 1) << 4))) =
                    make_float4(v[u].x, v[u].y, v[u].z, v[u].w);
            }
        }
    }
    if (__syncthreads_or(zero != 0.0f)) {
        const int c = threadIdx.x & (COL_W - 1);
        for (int q = threadIdx.x / COL_W; q < COL_H; q += 256 / COL_W) {
            if (i0 + c >= W || j0 + q >= H) break;
            float acc = 0.0f;
            for (int k = 0; k <= 2 * r; ++k)
                acc = fmaf(taps.w[k], lds[(q + k) * COL_W + (c ^ (((q + k) & 1) << 4))], acc);
            out[(size_t)(j0 + q) * W + i0 + c] = acc;
        }
        return;
    }
    // A = band (output row lane % 16), B = inputs (row 4 s + lane / 16, column
    // lane % 16); this wave's two row tiles start at 32 wv
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int m = lane & 15, g = lane >> 4;
    const float *bw = band + g - m + 15;
    const float *in0 = lds + (32 * wv + g) * COL_W + (m ^ ((g & 1) << 4));
    const float *in1 = lds + (32 * wv + g) * COL_W + ((m + 16) ^ ((g & 1) << 4));
    f32x4 acc[2][2] = {};
    float w = bw[0];
    float x[2][2] = {{in0[0], in1[0]}, {in0[16 * COL_W], in1[16 * COL_W]}};
    for (int s = 0; s < steps; ++s) {
        const int n = 4 * min(s + 1, steps - 1);  // as in the row pass
        const float wn = bw[n];
        float xn[2][2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            xn[t][0] = in0[(16 * t + n) * COL_W];
            xn[t][1] = in1[(16 * t + n) * COL_W];
        }
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                acc[t][u] = __builtin_amdgcn_mfma_f32_16x16x4f32(w, x[t][u], acc[t][u], 0, 0, 0);
                x[t][u] = xn[t][u];
            }
        w = wn;
    }
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int i = i0 + 16 * u + m;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int j = j0 + 32 * wv + 16 * t + 4 * g + q;
                if (i < W && j < H) out[(size_t)j * W + i] = acc[t][u][q];
            }
        }
}

// Both passes in one kernel for the smaller radii: a 64 x 64 tile and its halo
// in LDS, the row pass in place (each wave owns sixteen rows, which no other
// reads), the column pass from there. It reads each height about
// ((64 + 2r) / 64)^2 times, mostly from L2, does the row pass on as many more
// rows, and saves the intermediate grid's write and read and a launch: 2048 x
// 2048 at 37 taps 28.9 us in two kernels, 22.1 us here. A tile is written
// while others still read its surroundings, so the heights and the output must
// not overlap. Odd multiples of two as row stride keep the 16 rows x 2 columns
// of the row pass on 32 banks. Loads of one node a lane: pairs, which halve
// their number but straddle lines, took 3 us more with the heights in HBM.
constexpr int FUSE_T = 64;
constexpr int FUSE_BLOCK = 512;

__host__ __device__ constexpr int fuse_stride(int r) {
    return (FUSE_T + 4 * smooth_steps(r) - 16 + 1) / 4 * 4 + 2;
}
__host__ __device__ constexpr int fuse_rows(int r) {
    return (FUSE_T + 4 * smooth_steps(r) - 16 + 15) / 16 * 16;
}

__global__ __launch_bounds__(FUSE_BLOCK) void smooth_fused(const float *__restrict__ h, int W,
                                                           int H, const SmoothTaps taps,
                                                           float *__restrict__ out) {
    extern __shared__ float lds[];
    __shared__ float band[BAND];
    constexpr int WAVES = FUSE_BLOCK / 64;
    const int r = taps.r, steps = smooth_steps(r), stride = fuse_stride(r);
    const int tiles_x = (W + FUSE_T - 1) / FUSE_T, tile = blockIdx.x;
    const int i0 = tile % tiles_x * FUSE_T, j0 = tile / tiles_x * FUSE_T;
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int side = FUSE_T + 4 * steps - 16;  // rows and columns of the tile's windows and steps
    load_band<FUSE_BLOCK>(taps, band);
    float zero = 0.0f;
    {
        // rows up to the last tile's end (past the windows: the padding of its
        // sixteen), two columns a lane, all loads in flight at once
        constexpr int ROWS = 128 / WAVES;
        const int rows = fuse_rows(r);
        const bool inner = i0 >= r && i0 - r + side <= W;
        float v[ROWS][2];
#pragma unroll
        for (int p = 0; p < ROWS; ++p) {
            if (WAVES * p >= rows) break;
            const float *src = h + (size_t)min(max(j0 + wv + WAVES * p - r, 0), H - 1) * W;
            const int i = i0 - r + lane;
            v[p][0] = src[inner ? i : min(max(i, 0), W - 1)];
            v[p][1] = 0.0f;
            if (lane + 64 < side) v[p][1] = src[inner ? i + 64 : min(max(i + 64, 0), W - 1)];
        }
#pragma unroll
        for (int p = 0; p < ROWS; ++p) {
            if (WAVES * p >= rows) break;
            zero = chain_zero(v[p][1], chain_zero(v[p][0], zero));
            lds[(wv + WAVES * p) * stride + lane] = v[p][0];
            if (lane + 64 < side) lds[(wv + WAVES * p) * stride + lane + 64] = v[p][1];
        }
    }
    const bool scalar_rows = __syncthreads_or(zero != 0.0f);
    const int m = lane & 15, g = lane >> 4;
    zero = 0.0f;
    if (scalar_rows) {
        // one row at a time in a wave, every lane's window read before any is written
        for (int row = wv; row < side; row += WAVES) {
            float acc = 0.0f;
            for (int k = 0; k <= 2 * r; ++k)
                acc = fmaf(taps.w[k], lds[row * stride + lane + k], acc);
            lds[row * stride + lane] = acc;
            zero = chain_zero(acc, zero);
        }
    } else {
        for (int rt = 16 * wv; rt < side; rt += 16 * WAVES) {
            const float *in = lds + (rt + m) * stride + g;
            const float *bw = band + g - m + 15;
            f32x4 acc[4] = {};
            float w = bw[0], x[4] = {in[0], in[16], in[32], in[48]};
            for (int s = 0; s < steps; ++s) {
                const int n = 4 * min(s + 1, steps - 1);
                const float wn = bw[n];
                float xn[4];
#pragma unroll
                for (int t = 0; t < 4; ++t) xn[t] = in[16 * t + n];
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[t], w, acc[t], 0, 0, 0);
                w = wn;
#pragma unroll
                for (int t = 0; t < 4; ++t) x[t] = xn[t];
            }
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int row = rt + 4 * g + q;
                    lds[row * stride + 16 * t + m] = acc[t][q];
                    zero = chain_zero(acc[t][q], zero);
                }
        }
    }
    if (__syncthreads_or(zero != 0.0f)) {
        for (int q = wv; q < FUSE_T; q += WAVES) {
            if (i0 + lane >= W || j0 + q >= H) break;
            float acc = 0.0f;
            for (int k = 0; k <= 2 * r; ++k)
                acc = fmaf(taps.w[k], lds[(q + k) * stride + lane], acc);
            out[(size_t)(j0 + q) * W + i0 + lane] = acc;
        }
        return;
    }
    // sixteen tiles, two beside each other a wave
    const int tj = 16 * (wv >> 1), ti = 32 * (wv & 1);
    const float *in = lds + (tj + g) * stride + ti + m;
    const float *bw = band + g - m + 15;
    f32x4 acc[2] = {};
    float w = bw[0], x[2] = {in[0], in[16]};
    for (int s = 0; s < steps; ++s) {
        const int n = 4 * min(s + 1, steps - 1);
        const float wn = bw[n], x0 = in[n * stride], x1 = in[n * stride + 16];
        acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(w, x[0], acc[0], 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(w, x[1], acc[1], 0, 0, 0);
        w = wn;
        x[0] = x0;
        x[1] = x1;
    }
    float *dst = out + (size_t)(j0 + tj + 4 * g) * W + i0 + ti + m;
    const bool whole = i0 + FUSE_T <= W && j0 + FUSE_T <= H;  // uniform
#pragma unroll
    for (int q = 0; q < 4; ++q) {
#pragma unroll
        for (int u = 0; u < 2; ++u)
            if (whole || (i0 + ti + 16 * u + m < W && j0 + tj + 4 * g + q < H))
                dst[16 * u] = acc[u][q];
        dst += W;
    }
}

// Largest radius whose tile of smooth_fused fits 64 KB of LDS (and a row of it
// two loads a lane). Beyond it the row pass would also run on more than twice
// the tile's rows, where the intermediate grid of the two kernels costs less.
constexpr int FUSE_MAX_RADIUS = 28;
static_assert(sizeof(float) * fuse_rows(FUSE_MAX_RADIUS) * fuse_stride(FUSE_MAX_RADIUS) +
                      sizeof(float) * BAND <= 65536 &&
                  FUSE_T + 4 * smooth_steps(FUSE_MAX_RADIUS) - 16 <= 128,
              "smooth_fused's tile");

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

// A tile of TILE x TILE nodes per workgroup, of a column's nodes every thread
// takes as many as BLOCK threads leave it. Most tiles lie on the safe side of a perimeter (outside an
// obstacle, inside a path boundary) by more than eps, where every node's term
// is exactly zero, so the workgroup first decides which perimeters can touch
// it and then evaluates those alone, node by node as before and in the order
// of the list: the sums are the same bits. Bound before: the vector ALUs, on
// every node against every edge (2048 x 2048 nodes, 244 edges: 950-990 us);
// now the writes and, per tile, one pass over the edges (the same map: 23 us).
// 32 x 32 nodes keep that pass (one edge per thread and a barrier) small
// against the tile's work while the tile stays small against an obstacle. Maps
// of few such tiles (costmap_small_tiles) take 16 x 16, a node a thread: the
// bound there is a thread's chain over the edges of the perimeters that touch
// its tile, on as many compute units as there are tiles.
constexpr int CM_TILE = 32, CM_BLOCK = 512;
constexpr int CM_TILE_SMALL = 16, CM_BLOCK_SMALL = 256;

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

template <int TILE, int BLOCK>
__global__ __launch_bounds__(BLOCK) void costmap_polygons(const float2 *__restrict__ verts,
                                                        const PolygonSet ps, int W, int H,
                                                        float x0, float y0, float res,
                                                        float sigma, float eps, float inv_eps,
                                                        int accumulate,
                                                        float *__restrict__ cm) {
    constexpr int ROWS = TILE * TILE / BLOCK;
    __shared__ int off[MAX_POLYGONS + 1];
    __shared__ unsigned gap[MAX_POLYGONS];     // smallest tile_gap over the perimeter's edges
    __shared__ unsigned parity[MAX_POLYGONS];  // crossings seen from the tile's centre
    __shared__ unsigned long long touched;
    const int tid = threadIdx.x;
    const int i0 = blockIdx.x * TILE, j0 = blockIdx.y * TILE;
    if (tid <= MAX_POLYGONS) off[tid] = ps.offsets[tid];
    if (tid < MAX_POLYGONS) {
        gap[tid] = 0x7f800000u;  // +inf
        parity[tid] = 0u;
    }
    __syncthreads();
    {
        // the tile as its centre and half diagonal, from its corner nodes
        const float xa = fmaf((float)i0, res, x0), ya = fmaf((float)j0, res, y0);
        const float xb = fmaf((float)min(i0 + TILE - 1, W - 1), res, x0);
        const float yb = fmaf((float)min(j0 + TILE - 1, H - 1), res, y0);
        const float cx = 0.5f * (xa + xb), cy = 0.5f * (ya + yb);
        const float hx = 0.5f * (xb - xa), hy = 0.5f * (yb - ya);
        const float rho = sqrtf(fmaf(hx, hx, hy * hy));
        const int V = ps.count > 0 ? off[ps.count] : 0;
        for (int e = tid; e < V; e += BLOCK) {
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
    const int i = i0 + (tid & (TILE - 1)), jt = j0 + tid / TILE;
    if (i >= W || jt >= H) return;  // nodes past the grid (the rows below are tested with them)
    const float px = fmaf((float)i, res, x0);
    float py[ROWS], c[ROWS];
#pragma unroll
    for (int q = 0; q < ROWS; ++q) {
        py[q] = fmaf((float)(jt + q * (BLOCK / TILE)), res, y0);
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
        float dmin[ROWS];
        bool inside[ROWS];
#pragma unroll
        for (int q = 0; q < ROWS; ++q) {
            dmin[q] = __builtin_inff();
            inside[q] = false;
        }
        float2 v0 = verts[a + m - 1];
        for (int e = 0; e < m; ++e) {
            const float2 v1 = verts[a + e];
#pragma unroll
            for (int q = 0; q < ROWS; ++q) {
                dmin[q] = fminf(dmin[q], seg_dist2(px, py[q], v0.x, v0.y, v1.x, v1.y));
                if (crosses(px, py[q], v0, v1)) inside[q] = !inside[q];
            }
            v0 = v1;
        }
#pragma unroll
        for (int q = 0; q < ROWS; ++q) {
            // obstacle: negative inside; path boundary: negative outside
            const float d = sqrtf(dmin[q]);
            const float sd = (inside[q] == (ps.kinds[p] == 0)) ? -d : d;
            const float mm = fmaxf(0.0f, fmaf(-sd, inv_eps, 1.0f));
            c[q] = fmaf(sigma * mm, mm, c[q]);
        }
    }
#pragma unroll
    for (int q = 0; q < ROWS; ++q) {
        const int j = jt + q * (BLOCK / TILE);
        if (j >= H) break;
        const size_t o = (size_t)j * W + i;
        cm[o] = accumulate ? cm[o] + c[q] : c[q];
    }
}

}  // namespace

hipError_t launch_smooth(const float *h, int W, int H, const SmoothTaps &taps, float *tmp,
                         float *out, hipStream_t s) {
    const size_t nodes = (size_t)W * H;
    const uintptr_t hb = (uintptr_t)h, ob = (uintptr_t)out;
    const bool apart = hb + sizeof(float) * nodes <= ob || ob + sizeof(float) * nodes <= hb;
    if (apart && taps.r <= FUSE_MAX_RADIUS) {
        const size_t lds = sizeof(float) * fuse_rows(taps.r) * fuse_stride(taps.r);
        hipLaunchKernelGGL(smooth_fused,
                           dim3((unsigned)(((W + FUSE_T - 1) / FUSE_T) * ((H + FUSE_T - 1) / FUSE_T))),
                           dim3(FUSE_BLOCK), lds, s, h, W, H, taps, out);
        return hipGetLastError();
    }
    const size_t row_lds = sizeof(float) * ROW_H * row_stride(taps.r);
    const size_t col_lds = sizeof(float) * COL_W * (COL_H + 4 * smooth_steps(taps.r) - 16);
    hipLaunchKernelGGL(smooth_rows, dim3((W + ROW_W - 1) / ROW_W, (H + ROW_H - 1) / ROW_H),
                       dim3(256), row_lds, s, h, W, H, taps, tmp);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(smooth_cols, dim3((W + COL_W - 1) / COL_W, (H + COL_H - 1) / COL_H),
                       dim3(256), col_lds, s, tmp, W, H, taps, out);
    return hipGetLastError();
}

hipError_t launch_costmap_polygons(const float *verts, const PolygonSet &ps, int W, int H,
                                   float x0, float y0, float res, float sigma, float eps,
                                   int accumulate, float *cm, int units, hipStream_t s) {
    auto launch = [&](auto kernel, int tile, int block) {
        hipLaunchKernelGGL(kernel, dim3((W + tile - 1) / tile, (H + tile - 1) / tile), dim3(block),
                           0, s, (const float2 *)verts, ps, W, H, x0, y0, res, sigma, eps,
                           1.0f / eps, accumulate, cm);
    };
    if (costmap_small_tiles(W, H, units))
        launch(costmap_polygons<CM_TILE_SMALL, CM_BLOCK_SMALL>, CM_TILE_SMALL, CM_BLOCK_SMALL);
    else
        launch(costmap_polygons<CM_TILE, CM_BLOCK>, CM_TILE, CM_BLOCK);
    return hipGetLastError();
}

}  // namespace plan
