// Soft silhouette renderer (SoftRas-style; the paper renders its meshes with a
// differentiable soft rasterizer so that losses sit on pixels, Sec. 3 and the
// rendering appendix) and its adjoint, on CDNA4.
//
// Each vertex X is projected by a 3x4 camera matrix P to pixel coordinates
// u = P0.[X,1] / P2.[X,1], v = P1.[X,1] / P2.[X,1].  Triangle j covers pixel p
// (centre (col + 0.5, row + 0.5)) with probability D_j = sigmoid(x_j),
// x_j = +-d_j^2 / sigma (d_j: distance from p to the triangle's edges; + inside);
// the image is I = 1 - prod_j (1 - D_j) = 1 - T with the transmittance
// T = 1 / prod_j (1 + exp(x_j)) (as 1 - sigmoid(x) = 1 / (1 + e^x)).  Terms of
// pixels outside a triangle with d^2 > CUT sigma (D < 1e-6) are dropped.
//
// Adjoint: dI / dx_j = T D_j (prod over the other triangles times D_j (1 - D_j)),
// which needs no division by 1 - D_j, and d(d^2) / d(endpoint) of the nearest edge
// point q = s0 + t (s1 - s0) is -2 (1 - t) (p - q) and -2 t (p - q).
//
// Kernels: triangle records (one thread per triangle: its corners projected, widened
// box, orientation, reciprocal edge lengths, and each chunk's box); forward (an 8 x 8
// or 4 x 4 pixel tile per workgroup: the chunks whose box reaches the tile are listed,
// the records of their triangles that reach it are compacted through LDS in order, and
// the wavefronts share the tile's 4 x 4 quadrants); triangle adjoint (one wavefront, or
// a workgroup, per triangle over the pixels of its widened box, the transmittance recomputed by the
// forward kernels first); vertex gather (one thread per vertex summing its triangle
// corners in a fixed order, then through the projection).  No atomics anywhere: results
// are bitwise repeatable.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <new>
#include <vector>

#include "gsim.h"
#include "gsim_device.h"
#include "gsim_host.h"

namespace gsim {
namespace {

constexpr int RSLICE = 8;         // wavefronts per pixel tile
constexpr int RCHUNK = 64;        // triangles per chunk (one wavefront's)
constexpr int RROUND = 64 * RSLICE;  // triangles a round stages, and chunks a lookup tests
constexpr int RBOX = 4;           // values per triangle box
constexpr int RREC = 10;          // values per triangle record
constexpr int RTERM = 16;         // values per staged record
constexpr int RBOXED = 0x80;      // mark of a staged triangle (see unsafe_term)
const double RCUT = 13.815510557964274;  // -ln(1e-6)

// Per-triangle box and record, written once per frame.  Box: the bounding box widened by
// the cut-off distance (xmin, xmax, ymin, ymax).  Record: [0..5] screen corners a, b, c;
// [6] orientation (+1, -1, 0 for a degenerate triangle); [7..9] reciprocal squared lengths
// of the edges ab, bc, ca.  Boxes stand apart because most triangles are only tested.
template <typename T>
struct RasterArgs {
    const int32_t* tris;   // [nt][3]
    const int32_t* coff;   // [nv + 1] vertex -> corner list
    const int32_t* cent;   // [3 nt] corner = 3 tri + k
    T* trans;              // [H][W]
    T* cg;                 // [nt][6] screen-space gradient of each corner
    T* tbox;               // [nt][RBOX] triangle boxes
    T* trec;               // [nt][RREC] triangle records
    T* cbox;               // [ceil(nt / RCHUNK)][RBOX] widened box of each chunk of triangles
    int64_t nv, nt;
    int32_t H, W;
    T P[12];
    T isigma, cut;         // 1 / sigma; cut = CUT sigma
};

template <typename T, int N>
struct alignas(16) Vec {
    T v[N];
};

template <typename T>
__device__ __forceinline__ T cr2(T ax, T ay, T bx, T by) {
    return ax * by - ay * bx;
}

// Box of the corners q[0..5] widened by r.
template <typename T>
__device__ __forceinline__ void box_of(const T* q, T r, T* b) {
    b[0] = fmin(fmin(q[0], q[2]), q[4]) - r;
    b[1] = fmax(fmax(q[0], q[2]), q[4]) + r;
    b[2] = fmin(fmin(q[1], q[3]), q[5]) - r;
    b[3] = fmax(fmax(q[1], q[3]), q[5]) + r;
}

// A record as tri_term takes it: corners [0..5], edge vectors ab, bc, ca [6..11],
// orientation [12], reciprocal squared edge lengths [13..15].
template <typename T>
__device__ __forceinline__ void term_of(const T* q, T* r) {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const int n = k == 2 ? 0 : k + 1;
        r[2 * k] = q[2 * k];
        r[2 * k + 1] = q[2 * k + 1];
        r[6 + 2 * k] = q[2 * n] - q[2 * k];
        r[7 + 2 * k] = q[2 * n + 1] - q[2 * k + 1];
        r[13 + k] = q[7 + k];
    }
    r[12] = q[6];
}

// Whether tri_term may take a pixel out of reach for one inside, or for one with no
// distance at all: its coordinates are not finite or too far apart to be squared, or it is
// so thin (twice its area against the square of its extent L, r the cut-off distance)
// that the three orientations of a pixel r away may all be roundings.
template <typename T>
__device__ __forceinline__ bool unsafe_term(const T* q, T r) {
    constexpr T eps = sizeof(T) == 4 ? T(0x1p-16) : T(0x1p-45);  // 2^8 roundings
    const T L = (fmax(fmax(q[0], q[2]), q[4]) - fmin(fmin(q[0], q[2]), q[4])) +
                (fmax(fmax(q[1], q[3]), q[5]) - fmin(fmin(q[1], q[3]), q[5]));
    return !(fabs(cr2(q[2] - q[0], q[3] - q[1], q[4] - q[0], q[5] - q[1])) * r > eps * L * L * (L + r));
}

// Squared distance from a point at w from the segment's start to the segment e (inv: 1 /
// |e|^2) and the parameter t of the nearest point.
template <typename T>
__device__ __forceinline__ T seg_d2(T wx, T wy, T ex, T ey, T inv, T& t) {
    t = fmin(fmax((wx * ex + wy * ey) * inv, T(0)), T(1));  // (a zero-length edge: t = 0)
    const T dx = wx - t * ex, dy = wy - t * ey;
    return dx * dx + dy * dy;
}

// Signed scaled distance x = +-d^2 / sigma of pixel p to the triangle of q (see term_of);
// returns false when the term is dropped.  edge / t: the nearest edge (0: ab, 1: bc,
// 2: ca; the first minimum) and its parameter.
template <typename T>
__device__ __forceinline__ bool tri_term(T px, T py, const T* q, T isigma, T cut, T& x, int& edge, T& t) {
    T wx[3], wy[3], d[3], tk[3];
    bool inside = q[12] != T(0);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        wx[k] = px - q[2 * k];
        wy[k] = py - q[2 * k + 1];
        inside = inside & (q[12] * cr2(q[6 + 2 * k], q[7 + 2 * k], wx[k], wy[k]) >= T(0));
        d[k] = seg_d2(wx[k], wy[k], q[6 + 2 * k], q[7 + 2 * k], q[13 + k], tk[k]);
    }
    T m = d[0];
    edge = 0;
    t = tk[0];
    if (d[1] < m) { m = d[1]; edge = 1; t = tk[1]; }
    if (d[2] < m) { m = d[2]; edge = 2; t = tk[2]; }
    if (!inside && m > cut) return false;
    x = (inside ? m : -m) * isigma;
    return true;
}

__device__ __forceinline__ float sigm(float x) { return 1.f / (1.f + expf(-x)); }
__device__ __forceinline__ double sigm(double x) { return 1.0 / (1.0 + exp(-x)); }

// Screen position of vertex i and its depth P2.[X, 1].
template <typename T>
__device__ __forceinline__ V3<T> project(const RasterArgs<T>& A, const T* __restrict__ x, int64_t i) {
    const V3<T> X = ld3(x, A.nv, i);
    const T n0 = A.P[0] * X.x + A.P[1] * X.y + A.P[2] * X.z + A.P[3];
    const T n1 = A.P[4] * X.x + A.P[5] * X.y + A.P[6] * X.z + A.P[7];
    const T dn = A.P[8] * X.x + A.P[9] * X.y + A.P[10] * X.z + A.P[11];
    return {n0 / dn, n1 / dn, dn};
}

// One thread per triangle: its corners projected (a chain of three loads bounds the
// kernel, so projecting a vertex once per triangle costs less than a launch that does it
// once), its box and record, and the union of the boxes of each chunk of RCHUNK
// triangles, one wavefront's (so a tile can skip whole chunks).
template <typename T>
__global__ __launch_bounds__(256) void k_raster_tri_prep(RasterArgs<T> A, const T* __restrict__ x) {
    const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const T r = sqrt(A.cut);
    T b[4] = {T(INFINITY), T(-INFINITY), T(INFINITY), T(-INFINITY)};
    // a triangle with a corner index outside [0, nv) (possible only with a caller's
    // device-side list, which the host cannot check) is not read: its record keeps an
    // empty box, so it covers no pixel and no chunk box grows for it
    bool valid = j < A.nt;
    int32_t ci[3] = {0, 0, 0};
    if (valid)
        for (int k = 0; k < 3; ++k) {
            ci[k] = A.tris[3 * j + k];
            valid = valid && ci[k] >= 0 && ci[k] < A.nv;
        }
    bool nan = false;
    if (j < A.nt) {
        T q[RREC];
#pragma unroll
        for (int k = 0; k < RREC; ++k) q[k] = T(0);
        if (valid) {
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const V3<T> u = project(A, x, ci[k]);
                q[2 * k] = u.x;
                q[2 * k + 1] = u.y;
            }
            const T ax = q[0], ay = q[1], bx = q[2], by = q[3], cx = q[4], cy = q[5];
            box_of(q, r, b);
            nan = b[0] != b[0] || b[2] != b[2];
            const T area = cr2(bx - ax, by - ay, cx - ax, cy - ay);
            q[6] = area > T(0) ? T(1) : (area < T(0) ? T(-1) : T(0));
            q[7] = T(1) / ((bx - ax) * (bx - ax) + (by - ay) * (by - ay));
            q[8] = T(1) / ((cx - bx) * (cx - bx) + (cy - by) * (cy - by));
            q[9] = T(1) / ((ax - cx) * (ax - cx) + (ay - cy) * (ay - cy));
        }
#pragma unroll
        for (int k = 0; k < RBOX; ++k) A.tbox[RBOX * j + k] = b[k];
#pragma unroll
        for (int k = 0; k < RREC; ++k) A.trec[RREC * j + k] = q[k];
    }
    // (a box that is not a number is tested as reached everywhere, and so is its chunk's)
    if (nan) {
        b[0] = b[2] = T(-INFINITY);
        b[1] = b[3] = T(INFINITY);
    }
#pragma unroll
    for (int h = 32; h > 0; h >>= 1) {
        b[0] = fmin(b[0], __shfl_xor(b[0], h));
        b[1] = fmax(b[1], __shfl_xor(b[1], h));
        b[2] = fmin(b[2], __shfl_xor(b[2], h));
        b[3] = fmax(b[3], __shfl_xor(b[3], h));
    }
    const int lane = threadIdx.x & 63;
    if (lane < RBOX && j - lane < A.nt)
        A.cbox[RBOX * (j / RCHUNK) + lane] = lane == 0 ? b[0] : lane == 1 ? b[1] : lane == 2 ? b[2] : b[3];
}

// Entries before this thread's among the workgroup's kept ones (in thread order), and
// their count: the wavefronts' counts through LDS.  Two barriers; `count` must not be in
// use by an earlier call's readers.
__device__ __forceinline__ int rank_of(bool keep, int* count, int& total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const unsigned long long m = __ballot(keep);
    __syncthreads();
    if (lane == 0) count[wave] = __popcll(m);
    __syncthreads();
    int base = 0;
    total = 0;
#pragma unroll
    for (int w = 0; w < RSLICE; ++w) {
        base += w < wave ? count[w] : 0;
        total += count[w];
    }
    return base + __popcll(m & ((1ull << lane) - 1ull));
}

// Every fourth listed triangle from the group's on: Q *= 1 + e^x at its pixel.
template <typename T, bool BOXED>
__device__ __forceinline__ void take_terms(const RasterArgs<T>& A, const Vec<T, RTERM>* rec, const uint16_t* list,
                                           int group, int n, T px, T py, T& Q) {
    for (int k = group; k < n; k += 4) {
        const Vec<T, RTERM> r = rec[list[k]];
        if constexpr (BOXED) {
            T b[RBOX];
            box_of(r.v, sqrt(A.cut), b);
            if ((px < b[0]) | (px > b[1]) | (py < b[2]) | (py > b[3])) continue;
        }
        T x, t;
        int e;
        if (tri_term(px, py, r.v, A.isigma, A.cut, x, e, t)) Q = fma(Q, exp(x), Q);  // Q (1 + e^x)
    }
}

// One pixel tile of QUADS (4 or 1) quadrants of 4 x 4 pixels per workgroup of RSLICE
// wavefronts; writes the transmittance and (if not null) the image.  RROUND chunk boxes at
// a time are tested and the chunks that reach the tile listed in order; RSLICE listed
// chunks at a time, the triangles whose box (widened by the cut-off distance) reaches a
// quadrant are compacted into LDS in triangle order.  Each quadrant has RSLICE / QUADS
// wavefronts: each lists every (RSLICE / QUADS)-th of its quadrant's triangles, and each of
// its four groups of 16 lanes takes every fourth of those for the quadrant's 16 pixels,
// with the product prod (1 + exp(x_j)) per pixel; T = 1 / the product of a pixel's partial
// products, in a fixed order.
//
// Bound by the vector units: a triangle's box is mostly margin (its extent plus twice the
// cut-off distance, 3.7 sqrt(sigma) pixels), so of the (tile, triangle) pairs that survive
// most pixels of a large tile are out of reach.  4 x 4 pixels per step instead of 8 x 8
// do 0.6 of the work at 3-pixel triangles.  Boxes of 64 triangles, and boxes apart from
// records, cut what a tile reads.  Measured with a 64 x 64 cloth (7938 triangles) at
// 256 x 256: 18.7 us with 8 x 8 steps and chunks of 512 records, 12.7 us so.
template <typename T, int QUADS>
__global__ __launch_bounds__(64 * RSLICE) void k_raster_fwd(RasterArgs<T> A, T* __restrict__ image) {
    constexpr int RT = QUADS == 4 ? 8 : 4;     // tile edge
    constexpr int SHARE = RSLICE / QUADS;      // wavefronts per quadrant
    constexpr int PARTS = 4 * SHARE;           // partial products per pixel
    __shared__ Vec<T, RTERM> rec[RROUND];
    __shared__ T part[PARTS][RT * RT];
    __shared__ uint16_t hit[RROUND];
    __shared__ uint16_t mine[RSLICE][RROUND / SHARE];
    __shared__ uint8_t reach[RROUND];  // quadrants a triangle reaches | RBOXED
    __shared__ int count[RSLICE];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int quad = wave & (QUADS - 1), turn = wave / QUADS, group = lane >> 4, pix = lane & 15;
    const int tc = blockIdx.x * RT, tr = blockIdx.y * RT;
    const T px = (T)(tc + 4 * (quad & 1) + (pix & 3)) + T(0.5), py = (T)(tr + 4 * (quad >> 1) + (pix >> 2)) + T(0.5);
    // the tile's pixel-centre extent
    const T tx0 = (T)tc + T(0.5), tx1 = tx0 + T(RT - 1);
    const T ty0 = (T)tr + T(0.5), ty1 = ty0 + T(RT - 1);
    T Q = T(1);
    const int64_t nc = (A.nt + RCHUNK - 1) / RCHUNK;
    for (int64_t c0 = 0; c0 < nc; c0 += RROUND) {
        bool near = false;
        if (c0 + threadIdx.x < nc) {
            const Vec<T, RBOX> cb = *(const Vec<T, RBOX>*)(A.cbox + RBOX * (c0 + threadIdx.x));
            near = !((cb.v[1] < tx0) | (cb.v[0] > tx1) | (cb.v[3] < ty0) | (cb.v[2] > ty1));
        }
        int hits;
        const int at = rank_of(near, count, hits);
        if (near) hit[at] = (uint16_t)threadIdx.x;
        __syncthreads();
        for (int h0 = 0; h0 < hits; h0 += RSLICE) {
            const int64_t j = h0 + wave < hits ? RCHUNK * (c0 + hit[h0 + wave]) + lane : A.nt;
            int to = 0;  // quadrants in reach
            if (j < A.nt) {
                const Vec<T, RBOX> q = *(const Vec<T, RBOX>*)(A.tbox + RBOX * j);
#pragma unroll
                for (int k = 0; k < QUADS; ++k) {
                    const T x0 = tx0 + T(4 * (k & 1)), y0 = ty0 + T(4 * (k >> 1));
                    const bool out = (q.v[1] < x0) | (q.v[0] > x0 + T(3)) | (q.v[3] < y0) | (q.v[2] > y0 + T(3));
                    to |= out ? 0 : 1 << k;
                }
            }
            int total;
            const int k0 = rank_of(to != 0, count, total);  // (its barriers end the last round's reads)
            if (to) {
                T q[RREC];
#pragma unroll
                for (int k = 0; k < RREC; ++k) q[k] = A.trec[RREC * j + k];
                Vec<T, RTERM> r;
                term_of(q, r.v);
                rec[k0] = r;
                reach[k0] = (uint8_t)(unsafe_term(q, sqrt(A.cut)) ? to | RBOXED : to);
            }
            __syncthreads();
            // this wavefront's triangles
            int n = 0;
            unsigned long long boxed = 0;
            for (int k = 0; k < total; k += 64) {
                const int to = k + lane < total ? reach[k + lane] : 0;
                const bool in = to >> quad & 1;
                const unsigned long long m = __ballot(in);
                boxed |= __ballot(to & RBOXED);
                const int o = n + __popcll(m & ((1ull << lane) - 1ull));
                if (in && o % SHARE == turn) mine[wave][o / SHARE] = (uint16_t)(k + lane);
                n += __popcll(m);
            }
            n = (n + SHARE - 1 - turn) / SHARE;
            __builtin_amdgcn_wave_barrier();
            // each pixel against the box too where a term may be wrong about its reach (tested in
            // every round it takes 5-8 % of the kernel, chosen by round 1-4 %)
            if (boxed) take_terms<T, true>(A, rec, mine[wave], group, n, px, py, Q);
            else take_terms<T, false>(A, rec, mine[wave], group, n, px, py, Q);
        }
        __syncthreads();  // the list of chunks is no longer read
    }
    part[4 * turn + group][16 * quad + pix] = Q;
    __syncthreads();
    const int col = tc + 4 * ((lane >> 4) & 1) + (lane & 3), row = tr + 4 * (lane >> 5) + ((lane >> 2) & 3);
    if (wave == 0 && lane < RT * RT && col < A.W && row < A.H) {
        T P = part[0][lane];
#pragma unroll
        for (int w = 1; w < PARTS; ++w) P *= part[w][lane];
        const T tr = T(1) / P;
        A.trans[(int64_t)row * A.W + col] = tr;
        if (image) image[(int64_t)row * A.W + col] = T(1) - tr;
    }
}

// WAVES wavefronts per triangle: d <Ibar, I> / d (screen corners) over the pixels of its
// widened box, strided over the lanes, then summed over them (fixed order).  Needs the
// transmittance of the same x (the forward runs first).  Bound by the chain of one pixel
// after another in a lane (record, pixel, two image loads, exponential): one wavefront
// takes the 110 pixels of a 3-pixel triangle in two steps, and the 8 of a workgroup share
// the thousands of pixels of a triangle where there are few (see raster_backward).
// Measured, 7938 triangles at 256 x 256: 11.7 us with 16 lanes per triangle, 7.6 us so.
template <typename T, int WAVES>
__global__ __launch_bounds__(WAVES == 1 ? 256 : 64 * WAVES) void k_raster_tri_adj(RasterArgs<T> A,
                                                                                   const T* __restrict__ ibar) {
    __shared__ T red[WAVES][6];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t j = WAVES == 1 ? (int64_t)blockIdx.x * 4 + wave : (int64_t)blockIdx.x;
    if (j >= A.nt) return;  // the whole wavefront (WAVES > 1: never)
    T box[RBOX], rec[RREC], q[RTERM];
#pragma unroll
    for (int k = 0; k < RBOX; ++k) box[k] = A.tbox[RBOX * j + k];
#pragma unroll
    for (int k = 0; k < RREC; ++k) rec[k] = A.trec[RREC * j + k];
    term_of(rec, q);
    // pixel index range whose centres lie inside the widened box, clamped into the
    // image before any conversion to int (far or non-finite corners stay in range)
    const int c0 = (int)fmin(T(A.W), fmax(T(0), ceil(box[0] - T(0.5))));
    const int c1 = (int)fmax(T(-1), fmin(T(A.W - 1), floor(box[1] - T(0.5))));
    const int r0 = (int)fmin(T(A.H), fmax(T(0), ceil(box[2] - T(0.5))));
    const int r1 = (int)fmax(T(-1), fmin(T(A.H - 1), floor(box[3] - T(0.5))));
    const int bw = c1 >= c0 ? c1 - c0 + 1 : 0;
    const int npx = r1 >= r0 ? bw * (r1 - r0 + 1) : 0;
    T g[6] = {T(0), T(0), T(0), T(0), T(0), T(0)};
    for (int p = WAVES == 1 ? lane : (int)threadIdx.x; p < npx; p += 64 * WAVES) {
        const int row = r0 + p / bw, col = c0 + p % bw;
        const T px = (T)col + T(0.5), py = (T)row + T(0.5);
        const int64_t pi = (int64_t)row * A.W + col;
        const T ib = ibar[pi], tr = A.trans[pi];
        T x, t;
        int e;
        if (!tri_term(px, py, q, A.isigma, A.cut, x, e, t)) continue;
        const T gx = ib * tr * sigm(x);
        if (gx == T(0)) continue;
        // x = +-d2 / sigma; d2 = |p - q|^2, q on edge e = (s0, s1)
        const T sgn = x >= T(0) ? T(1) : T(-1);
        const T s0x = e == 0 ? q[0] : e == 1 ? q[2] : q[4], s0y = e == 0 ? q[1] : e == 1 ? q[3] : q[5];
        const T ex = e == 0 ? q[6] : e == 1 ? q[8] : q[10], ey = e == 0 ? q[7] : e == 1 ? q[9] : q[11];
        const T qx = s0x + t * ex, qy = s0y + t * ey;
        const T k = gx * sgn * A.isigma * T(-2);
        const T a = k * (T(1) - t), b = k * t;
        if (e == 0) {
            g[0] += a * (px - qx); g[1] += a * (py - qy); g[2] += b * (px - qx); g[3] += b * (py - qy);
        } else if (e == 1) {
            g[2] += a * (px - qx); g[3] += a * (py - qy); g[4] += b * (px - qx); g[5] += b * (py - qy);
        } else {
            g[4] += a * (px - qx); g[5] += a * (py - qy); g[0] += b * (px - qx); g[1] += b * (py - qy);
        }
    }
    wave_sum<T, 6>(g);
    if constexpr (WAVES > 1) {
        if (lane == 0)
#pragma unroll
            for (int k = 0; k < 6; ++k) red[wave][k] = g[k];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            g[k] = red[0][k];
#pragma unroll
            for (int w = 1; w < WAVES; ++w) g[k] += red[w][k];
        }
    }
    if (lane == 0 && (WAVES == 1 || wave == 0)) {
#pragma unroll
        for (int k = 0; k < 6; ++k) A.cg[6 * j + k] = g[k];
    }
}

// One thread per vertex: sum its corners' screen gradients (fixed order), then
// through the projection; adds to xbar (SoA [3][nv]).
template <typename T>
__global__ __launch_bounds__(256) void k_raster_vertex_adj(RasterArgs<T> A, const T* __restrict__ x,
                                                               T* __restrict__ xbar) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= A.nv) return;
    T gu = T(0), gv = T(0);
    for (int32_t k = A.coff[i]; k < A.coff[i + 1]; ++k) {
        const int32_t c = A.cent[k];
        gu += A.cg[6 * (c / 3) + 2 * (c % 3)];
        gv += A.cg[6 * (c / 3) + 2 * (c % 3) + 1];
    }
    const V3<T> at = project(A, x, i);
    const T u = at.x, v = at.y, id = T(1) / at.z;
#pragma unroll
    for (int k = 0; k < 3; ++k) xbar[k * A.nv + i] += (gu * (A.P[k] - u * A.P[8 + k]) + gv * (A.P[4 + k] - v * A.P[8 + k])) * id;
}

}  // namespace
}  // namespace gsim

using namespace gsim;

// ------------------------------------------------------------------ host ---
struct gsim_raster {
    int dtype = GSIM_F32;
    int64_t nv = 0, nt = 0;
    int H = 0, W = 0;
    char* ws = nullptr;
    size_t o_tris = 0, o_coff = 0, o_cent = 0, o_trans = 0, o_cg = 0, o_tbox = 0, o_trec = 0, o_cbox = 0;
};

namespace {

size_t raster_layout(gsim_raster* R, size_t tsize) {
    size_t o = 0;
    auto take = [&](size_t bytes) {
        o = (o + 255) & ~size_t(255);
        const size_t at = o;
        o += std::max<size_t>(bytes, 1);
        return at;
    };
    R->o_tris = take(12 * (size_t)R->nt);
    R->o_coff = take(4 * (size_t)(R->nv + 1));
    R->o_cent = take(12 * (size_t)R->nt);
    R->o_trans = take(tsize * (size_t)R->H * R->W);
    R->o_cg = take(6 * tsize * (size_t)R->nt);
    R->o_tbox = take(RBOX * tsize * (size_t)R->nt);
    R->o_trec = take(RREC * tsize * (size_t)R->nt);
    R->o_cbox = take(RBOX * tsize * (size_t)((R->nt + RCHUNK - 1) / RCHUNK));
    return (o + 255) & ~size_t(255);
}

int raster_check(int dtype, int64_t nv, int64_t nt, int H, int W) {
    if (dtype != GSIM_F32 && dtype != GSIM_F64) return fail(GSIM_E_INVALID, "dtype must be GSIM_F32 or GSIM_F64");
    if (nv < 1 || nt < 1 || nt > (int64_t)INT32_MAX / 3 || nv >= INT32_MAX)
        return fail(GSIM_E_INVALID, "n_verts and n_tris must be >= 1 (and below 2^31 / 3 triangles)");
    if (H < 1 || W < 1 || (int64_t)H * W > (int64_t)1 << 28) return fail(GSIM_E_INVALID, "bad image size");
    return GSIM_OK;
}

template <typename T>
RasterArgs<T> raster_args(const gsim_raster* R, const gsim_camera* cam) {
    RasterArgs<T> A;
    std::memset(&A, 0, sizeof A);
    A.tris = (const int32_t*)(R->ws + R->o_tris);
    A.coff = (const int32_t*)(R->ws + R->o_coff);
    A.cent = (const int32_t*)(R->ws + R->o_cent);
    A.trans = (T*)(R->ws + R->o_trans);
    A.cg = (T*)(R->ws + R->o_cg);
    A.tbox = (T*)(R->ws + R->o_tbox);
    A.trec = (T*)(R->ws + R->o_trec);
    A.cbox = (T*)(R->ws + R->o_cbox);
    A.nv = R->nv;
    A.nt = R->nt;
    A.H = R->H;
    A.W = R->W;
    for (int k = 0; k < 12; ++k) A.P[k] = (T)cam->P[k];
    A.isigma = (T)(1.0 / cam->sigma);
    A.cut = (T)(RCUT * cam->sigma);
    return A;
}

int cam_check(const gsim_camera* cam) {
    if (!cam) return fail(GSIM_E_INVALID, "NULL camera");
    if (!(cam->sigma > 0) || !std::isfinite(cam->sigma)) return fail(GSIM_E_INVALID, "sigma must be > 0");
    for (int k = 0; k < 12; ++k)
        if (!std::isfinite(cam->P[k])) return fail(GSIM_E_NONFINITE, "camera matrix");
    return GSIM_OK;
}

int raster_cam_check(const gsim_raster* R, const gsim_camera* cam) {
    if (!R || !cam) return fail(GSIM_E_INVALID, "NULL renderer or camera");
    if (!(cam->sigma > 0) || !std::isfinite(cam->sigma)) return fail(GSIM_E_INVALID, "sigma must be > 0");
    for (int k = 0; k < 12; ++k)
        if (!std::isfinite(cam->P[k])) return fail(GSIM_E_NONFINITE, "camera matrix");
    return GSIM_OK;
}

// The forward launches.  4 x 4 tiles give four times the workgroups, each staging its
// triangles for a quarter of the pixels: they pay where the 8 x 8 tiles would not cover
// the compute units or hold many triangles each.  Measured (8 x 8 / 4 x 4 tiles, us):
// 7938 triangles at 60 x 60 71 / 24, 160 x 160 20.3 / 10.6, 200 x 200 (12.7 triangles per
// tile) 15.4 / 11.7, 256 x 256 (7.8) 12.3 / 14.7, 512 x 512 (1.9) 14.6 / 36; 32258
// triangles at 256 x 256 (31.5) 33.6 / 26.9, 700 x 700 (4.2) 33.9 / 85; 450 triangles at
// 124 x 124 (256 tiles) 5.3 / 4.7, 98 at 700 x 700 16 / 51.
template <typename T>
hipError_t raster_frame(const gsim_raster* R, const RasterArgs<T>& A, const T* x, T* image, hipStream_t s) {
    hipLaunchKernelGGL(k_raster_tri_prep<T>, dim3((unsigned)((R->nt + 255) / 256)), dim3(256), 0, s, A, x);
    const int64_t tiles = (int64_t)((R->W + 7) / 8) * ((R->H + 7) / 8);
    if (tiles < 256 || R->nt >= 10 * tiles)
        hipLaunchKernelGGL((k_raster_fwd<T, 1>), dim3((R->W + 3) / 4, (R->H + 3) / 4), dim3(64 * RSLICE), 0, s, A, image);
    else
        hipLaunchKernelGGL((k_raster_fwd<T, 4>), dim3((R->W + 7) / 8, (R->H + 7) / 8), dim3(64 * RSLICE), 0, s, A, image);
    return hipGetLastError();
}

template <typename T>
int raster_forward(gsim_raster* R, const gsim_camera* cam, const T* x, T* image, hipStream_t s) {
    RasterArgs<T> A = raster_args<T>(R, cam);
    const hipError_t e = raster_frame<T>(R, A, x, image, s);
    return e == hipSuccess ? GSIM_OK : hip_fail(e, "raster forward");
}

template <typename T>
int raster_backward(gsim_raster* R, const gsim_camera* cam, const T* x, const T* ibar, T* xbar, hipStream_t s) {
    int rc = raster_forward<T>(R, cam, x, nullptr, s);  // transmittance and projection of this x
    if (rc) return rc;
    RasterArgs<T> A = raster_args<T>(R, cam);
    // few triangles: a workgroup each, so that large ones do not leave the card to a few
    // wavefronts (one / eight per triangle: 98 triangles at 700 x 700 70 / 12 us, 450 at
    // 124 x 124 4.8 / 4.0, 1922 at 400 x 300 5.1 / 6.5)
    if (R->nt <= 1024)
        hipLaunchKernelGGL((k_raster_tri_adj<T, 8>), dim3((unsigned)R->nt), dim3(512), 0, s, A, ibar);
    else
        hipLaunchKernelGGL((k_raster_tri_adj<T, 1>), dim3((unsigned)((R->nt + 3) / 4)), dim3(256), 0, s, A, ibar);
    hipLaunchKernelGGL(k_raster_vertex_adj<T>, dim3((unsigned)((R->nv + 255) / 256)), dim3(256), 0, s, A, x, xbar);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? GSIM_OK : hip_fail(e, "raster backward");
}

// ------------------------------------------- forward without allocation ---
// Scratch of gsim_raster_forward_noalloc: one static device array per GPU (each device
// the library runs on holds its own copy until the process ends).  In host code
// `scratch` names a host-side stand-in, not device memory: its device address is taken
// once per device with hipGetSymbolAddress and only that address is passed on.
static __device__ __align__(256) unsigned char scratch[GSIM_RASTER_SCRATCH_BYTES];

const int MAX_DEVICES = 64;
std::mutex g_scratch_mu;
char* g_scratch_ptr[MAX_DEVICES] = {};

// Device address of the current device's scratch (looked up on the first call on it).
int scratch_ptr(char** out) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e, "current device");
    if (dev < 0 || dev >= MAX_DEVICES) return fail(GSIM_E_UNSUPPORTED, "device %d: at most %d devices", dev, MAX_DEVICES);
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) return hip_fail(e == hipSuccess ? hipErrorInvalidSymbol : e, "scratch address");
        g_scratch_ptr[dev] = (char*)p;
    }
    *out = g_scratch_ptr[dev];
    return GSIM_OK;
}

// Offsets of the forward's scratch (transmittance, triangle boxes and records, chunk
// boxes) from one base; returns the bytes it needs.
size_t raster_fwd_layout(gsim_raster* R, size_t tsize) {
    size_t o = 0;
    auto take = [&](size_t bytes) {
        o = (o + 255) & ~size_t(255);
        const size_t at = o;
        o += std::max<size_t>(bytes, 1);
        return at;
    };
    R->o_trans = take(tsize * (size_t)R->H * R->W);
    R->o_tbox = take(RBOX * tsize * (size_t)R->nt);
    R->o_trec = take(RREC * tsize * (size_t)R->nt);
    R->o_cbox = take(RBOX * tsize * (size_t)((R->nt + RCHUNK - 1) / RCHUNK));
    return (o + 255) & ~size_t(255);
}

template <typename T>
int raster_forward_noalloc(gsim_raster* R, const int32_t* d_tris, const gsim_camera* cam, const T* x, T* image,
                           hipStream_t s) {
    RasterArgs<T> A = raster_args<T>(R, cam);
    A.tris = d_tris;  // the caller's device list (coff, cent, cg: only the adjoint uses them)
    A.coff = A.cent = nullptr;
    A.cg = nullptr;
    const hipError_t e = raster_frame<T>(R, A, x, image, s);
    return e == hipSuccess ? GSIM_OK : hip_fail(e, "raster forward (no allocation)");
}

}  // namespace

extern "C" {

int gsim_raster_forward_noalloc(int dtype, int64_t n_verts, int64_t n_tris, const int32_t* d_tris, int height,
                                int width, const gsim_camera* camera, const void* x, void* image, void* stream) {
    if (int rc = raster_check(dtype, n_verts, n_tris, height, width)) return rc;
    if (int rc = cam_check(camera)) return rc;
    if (!d_tris || !x || !image) return fail(GSIM_E_INVALID, "NULL triangle list, positions or image");
    gsim_raster R;  // host-side description only (no workspace of its own)
    R.dtype = dtype;
    R.nv = n_verts;
    R.nt = n_tris;
    R.H = height;
    R.W = width;
    const size_t need = raster_fwd_layout(&R, dtype == GSIM_F64 ? 8 : 4);
    if (need > (size_t)GSIM_RASTER_SCRATCH_BYTES)
        return fail(GSIM_E_WORKSPACE, "%lld vertices, %lld triangles at %dx%d need %zu bytes of scratch; the static "
                    "scratch holds %d (use gsim_raster_init with a workspace)", (long long)n_verts, (long long)n_tris,
                    height, width, need, GSIM_RASTER_SCRATCH_BYTES);
    if (int rc = scratch_ptr(&R.ws)) return rc;
    return dtype == GSIM_F64
               ? raster_forward_noalloc<double>(&R, d_tris, camera, (const double*)x, (double*)image, (hipStream_t)stream)
               : raster_forward_noalloc<float>(&R, d_tris, camera, (const float*)x, (float*)image, (hipStream_t)stream);
}

int gsim_raster_sizes(int dtype, int64_t n_verts, int64_t n_tris, int height, int width, size_t* workspace_bytes) {
    if (int rc = raster_check(dtype, n_verts, n_tris, height, width)) return rc;
    if (!workspace_bytes) return fail(GSIM_E_INVALID, "NULL output");
    gsim_raster R;
    R.nv = n_verts;
    R.nt = n_tris;
    R.H = height;
    R.W = width;
    *workspace_bytes = raster_layout(&R, dtype == GSIM_F64 ? 8 : 4);
    return GSIM_OK;
}

int gsim_raster_init(int dtype, int64_t n_verts, int64_t n_tris, const int32_t* tris, int height, int width,
                     void* d_workspace, size_t bytes, void* stream, gsim_raster** out) {
    if (int rc = raster_check(dtype, n_verts, n_tris, height, width)) return rc;
    if (!tris || !d_workspace || !out) return fail(GSIM_E_INVALID, "NULL argument");
    if (((uintptr_t)d_workspace) & 255) return fail(GSIM_E_INVALID, "workspace must be 256-byte aligned");
    for (int64_t k = 0; k < 3 * n_tris; ++k)
        if (tris[k] < 0 || tris[k] >= n_verts) return fail(GSIM_E_TOPOLOGY, "triangle %lld index out of range", (long long)(k / 3));
    gsim_raster* R = new (std::nothrow) gsim_raster();
    if (!R) return fail(GSIM_E_INVALID, "out of host memory");
    R->dtype = dtype;
    R->nv = n_verts;
    R->nt = n_tris;
    R->H = height;
    R->W = width;
    R->ws = (char*)d_workspace;
    const size_t need = raster_layout(R, dtype == GSIM_F64 ? 8 : 4);
    if (bytes < need) {
        delete R;
        return fail(GSIM_E_WORKSPACE, "workspace of %zu bytes, %zu needed", bytes, need);
    }
    // vertex -> corner lists (corner = 3 tri + k), in increasing corner order
    std::vector<int32_t> coff(n_verts + 1, 0), cent(3 * n_tris);
    for (int64_t k = 0; k < 3 * n_tris; ++k) coff[tris[k] + 1]++;
    for (int64_t i = 0; i < n_verts; ++i) coff[i + 1] += coff[i];
    std::vector<int32_t> fill(coff.begin(), coff.end() - 1);
    for (int64_t k = 0; k < 3 * n_tris; ++k) cent[fill[tris[k]]++] = (int32_t)k;
    hipStream_t s = (hipStream_t)stream;
    hipError_t e = hipMemcpyAsync(R->ws + R->o_tris, tris, 12 * (size_t)n_tris, hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipMemcpyAsync(R->ws + R->o_coff, coff.data(), 4 * coff.size(), hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipMemcpyAsync(R->ws + R->o_cent, cent.data(), 4 * cent.size(), hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) {
        delete R;
        return hip_fail(e, "raster upload");
    }
    *out = R;
    return GSIM_OK;
}

int gsim_raster_destroy(gsim_raster* R) {
    delete R;
    return GSIM_OK;
}

int gsim_raster_forward(gsim_raster* R, const gsim_camera* cam, const void* x, void* image, void* stream) {
    if (int rc = raster_cam_check(R, cam)) return rc;
    if (!x || !image) return fail(GSIM_E_INVALID, "NULL x or image");
    return R->dtype == GSIM_F64 ? raster_forward<double>(R, cam, (const double*)x, (double*)image, (hipStream_t)stream)
                                : raster_forward<float>(R, cam, (const float*)x, (float*)image, (hipStream_t)stream);
}

int gsim_raster_backward(gsim_raster* R, const gsim_camera* cam, const void* x, const void* image_bar, void* x_bar,
                         void* stream) {
    if (int rc = raster_cam_check(R, cam)) return rc;
    if (!x || !image_bar || !x_bar) return fail(GSIM_E_INVALID, "NULL argument");
    return R->dtype == GSIM_F64
               ? raster_backward<double>(R, cam, (const double*)x, (const double*)image_bar, (double*)x_bar,
                                         (hipStream_t)stream)
               : raster_backward<float>(R, cam, (const float*)x, (const float*)image_bar, (float*)x_bar,
                                        (hipStream_t)stream);
}

}  // extern "C"
