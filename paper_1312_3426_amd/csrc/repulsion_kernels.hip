// repulsion_kernels.hip -- soft-sphere repulsion of the mesh nodes (the
// object-object and object-wall collisions of the paper's channel script,
// Section "Implementation details": "inter ... soft-sphere a n cutoff offset"
// between part types and with the channel walls): a (d - offset)^-n for
// offset < d < offset + cutoff, pushing the partners apart.
//
// Per step, before the membrane kernel (which adds the result to each node's
// total force), two launches where the cells hold less than a node and a half on
// average:
//   rep_bin     the positions the membrane kernel takes its forces at (those
//               of the step start, or advanced by the half-step velocity with
//               velocity Verlet), wrapped into the box along periodic axes,
//               and their cells (a regular grid, edge >= the largest pair
//               range); each node is put at the head of its cell's list (in
//               whatever order the atomics go), and the lists of the step
//               before are emptied;
//   rep_force   one thread per node: the lists of its own cell and of the
//               neighbour cells it is within the range of, a cell across a
//               periodic face shifted by the box length (the minimum image:
//               cells are at least the pair range and the box at least twice
//               it); then every obstacle shape and the z walls; FP64
//               arithmetic, each node's terms summed exactly (fixed_point.h),
//               so the result does not depend on the order of the lists.
// What bounds it: the round trips of the atomics (bin) and of the lists (force),
// a few dependent loads a node with all nodes in flight at once.
// With more nodes to a cell (RepDev::sorted: ranges of several mesh edges) the
// lists' nodes, one place in memory each, cost more than a counting sort over the
// few cells: rep_bin counts, a scan, rep_scatter and rep_gather put the nodes in
// cell order, and rep_sorted runs one thread per node in that order, so that a wave
// reads its partners as the same contiguous runs.  Repulsion of 500 spheres of 642
// nodes in 256x128x128 (us a step, lists and sorted): range 1.5 (0.3 nodes a cell) 487
// and 538, 2 (0.6) 903 and 906, 3 (2.1) 1984 and 1656, 5 (9.8) 4759 and 3638; 400
// cells of 393 nodes: range 3 (1.0) 927 and 1024, 5 (4.8) 1925 and 1650.
#include <limits.h>

#include "device_common.h"
#include "fixed_point.h"

namespace oif {
namespace {

using namespace dev;

// x wrapped into [0, L): x - L floor(x / L), without the division where x is
// inside already (x < L makes x / L round below 1)
__device__ __forceinline__ double wrapped(double x, double L) {
    return x >= 0.0 && x < L ? x : x - L * floor(x / L);
}

// Cell of a (wrapped) coordinate.  The product with the reciprocal edge may put
// a node at a cell's face into the cell beside it, which the margin of
// offsets() allows for.
__device__ __forceinline__ int cell_coord(const RepDev& D, int a, double w) {
    const double q = floor(w * D.rhc[a]);
    // also catches a non-finite position (the watchdog reports those)
    if (!(q >= 0.0)) return 0;
    return q >= (double)D.nc[a] ? D.nc[a] - 1 : (int)q;
}

template <typename R>
__global__ void __launch_bounds__(256)
rep_bin_kernel(const ObjDev<R>* __restrict__ objs, const RepDev* __restrict__ Dp, int parity) {
    const ObjDev<R>& O = objs[blockIdx.x];
    const RepDev& D = *Dp;
    const int v = blockIdx.y * blockDim.x + threadIdx.x;
    if (v >= O.t->nv) return;
    const R half_im = R(0.5) * O.inv_mass;
    const int j = O.node0 + v;
    double p[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const int k = 3 * v + c;
        // the same expression as the membrane kernel's staging
        const double x = O.F ? O.X[k] + (double)fmadd(O.F[k], half_im, O.V[k]) : O.X[k];
        p[c] = x + (double)O.anchor[c];
        if (c < 2 || !D.walls_z) p[c] = wrapped(p[c], D.L[c]);
        D.pos[3 * j + c] = p[c];
    }
    if (D.pairs) {
        const int cx = cell_coord(D, 0, p[0]), cy = cell_coord(D, 1, p[1]), cz = cell_coord(D, 2, p[2]);
        const int cell = (cz * D.nc[1] + cy) * D.nc[0] + cx, old = D.cell[j];
        if (D.sorted) {
            D.cell[j] = cell;
            atomicAdd(&D.cnt[cell], 1);
            return;
        }
        if (old >= 0) D.head[parity ^ 1][old] = -1;
        D.cell[j] = cell;
        const int next = atomicExch(&D.head[parity][cell], j);
        D.node[j] = RepNode{(float)p[0], (float)p[1], (float)p[2], next};
    }
}

__device__ __forceinline__ double dot3(const double* a, const double* b) {
    return a[0] * b[0] + a[1] * b[1] + a[2] * b[2];
}

// Distance from x to the surface of a shape and the unit vector from the
// closest surface point to x; false if x is inside (no force then).  For a
// rhomboid the closest point is the nearest of the face interiors (projection
// inside the parallelogram), the edges (clamped projection) and so the
// corners.
__device__ bool shape_distance(const ShapeDev& S, const double x[3], double& dist, double dir[3]) {
    if (S.kind == 1) {
        const double d = dot3(x, S.n) - S.dist;
        if (!(d > 0.0)) return false;
        dist = d;
        for (int c = 0; c < 3; ++c) dir[c] = S.n[c];
        return true;
    }
    double r[3] = {x[0] - S.corner[0], x[1] - S.corner[1], x[2] - S.corner[2]};
    bool inside = true;
    for (int k = 0; k < 3; ++k) {
        const double st = dot3(r, S.cof[k]) / S.det;
        inside = inside && st >= 0.0 && st <= 1.0;
    }
    if (inside) return false;
    double best2 = INFINITY, bp[3] = {0.0, 0.0, 0.0};
    for (int k = 0; k < 3; ++k) {
        const double* u = S.e[(k + 1) % 3];
        const double* v = S.e[(k + 2) % 3];
        const double uu = dot3(u, u), uv = dot3(u, v), vv = dot3(v, v), den = uu * vv - uv * uv;
        for (int side = 0; side < 2; ++side) {  // the two faces with coordinate k fixed
            double q[3];
            for (int c = 0; c < 3; ++c) q[c] = r[c] - side * S.e[k][c];
            const double qu = dot3(q, u), qv = dot3(q, v);
            const double a = (qu * vv - qv * uv) / den, b = (qv * uu - qu * uv) / den;
            if (a >= 0.0 && a <= 1.0 && b >= 0.0 && b <= 1.0) {
                double p[3], d2 = 0.0;
                for (int c = 0; c < 3; ++c) {
                    p[c] = side * S.e[k][c] + a * u[c] + b * v[c];
                    d2 += (r[c] - p[c]) * (r[c] - p[c]);
                }
                if (d2 < best2) {
                    best2 = d2;
                    for (int c = 0; c < 3; ++c) bp[c] = p[c];
                }
            }
        }
        const double ee = dot3(S.e[k], S.e[k]);
        for (int i = 0; i < 4; ++i) {  // the four edges along e_k
            double o[3], q[3];
            for (int c = 0; c < 3; ++c) {
                o[c] = (i & 1) * u[c] + (i >> 1) * v[c];
                q[c] = r[c] - o[c];
            }
            double t = dot3(q, S.e[k]) / ee;
            t = t < 0.0 ? 0.0 : (t > 1.0 ? 1.0 : t);
            double p[3], d2 = 0.0;
            for (int c = 0; c < 3; ++c) {
                p[c] = o[c] + t * S.e[k][c];
                d2 += (r[c] - p[c]) * (r[c] - p[c]);
            }
            if (d2 < best2) {
                best2 = d2;
                for (int c = 0; c < 3; ++c) bp[c] = p[c];
            }
        }
    }
    dist = sqrt(best2);
    for (int c = 0; c < 3; ++c) dir[c] = (r[c] - bp[c]) / dist;
    return true;
}

// Exact sum of a node's force terms (three components).
struct ForceSum {
    long long hi[3] = {0, 0, 0}, lo[3] = {0, 0, 0};
    bool ok = true;
    __device__ void add(double fx, double fy, double fz) {
        const double g[3] = {fx, fy, fz};
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            long long h, l;
            ok = fx_split(g[c], h, l) && ok;
            hi[c] += h;
            lo[c] += l;
        }
    }
};

__device__ __forceinline__ void soft_sphere(const SoftSphereDev& ss, double d, const double dir[3], ForceSum& f) {
    const double e = d - ss.offset;
    if (!(e > 0.0 && e < ss.cutoff)) return;
    const double m = ss.a * ss.n * pow(e, -(ss.n + 1.0));
    f.add(m * dir[0], m * dir[1], m * dir[2]);
}

// Pair force on a node of type tj from the node w of type tw, r their distance
// vector.
__device__ __forceinline__ void pair_force(const RepDev& D, int tj, int tw, const double r[3], ForceSum& f) {
    const double d2 = dot3(r, r);
    if (!(d2 < D.range2)) return;  // beyond every pair range
    const SoftSphereDev& ss = D.pair[tj][tw];
    if (ss.a == 0.0) return;
    const double d = sqrt(d2), id = 1.0 / d;
    const double dir[3] = {r[0] * id, r[1] * id, r[2] * id};
    soft_sphere(ss, d, dir, f);
}

// Forces of the obstacle shapes and the z walls on a node at p (wrapped).
__device__ __forceinline__ void wall_forces(const RepDev& D, const SoftSphereDev& ws, const double p[3], ForceSum& f) {
    for (int k = 0; k < D.n_shape; ++k) {
        double d, dir[3];
        if (shape_distance(D.shape[k], p, d, dir)) soft_sphere(ws, d, dir, f);
    }
    if (D.walls_z) {
        const double up[3] = {0.0, 0.0, 1.0}, down[3] = {0.0, 0.0, -1.0};
        if (p[2] > 0.0) soft_sphere(ws, p[2], up, f);
        if (p[2] < D.L[2]) soft_sphere(ws, D.L[2] - p[2], down, f);
    }
}

// Neighbour cell offsets along one axis that hold nodes within the range of w
// (in cell k): of -1 .. 1 those whose near face is not beyond it (with a margin
// for the rounding of the cell numbers); each cell once when the periodic axis
// has fewer than three cells.
__device__ __forceinline__ void offsets(const RepDev& D, int a, double w, int k, bool periodic, double range, int& lo,
                                        int& hi) {
    if (periodic && D.nc[a] < 3) {
        lo = 0;
        hi = D.nc[a] - 1;
        return;
    }
    const double h = D.hc[a], reach = range + 1e-6 * h, x = w - k * h;
    lo = x < reach ? -1 : 0;
    hi = h - x < reach ? 1 : 0;
}

// One thread per node.  Cells of about 0.9 with a range of 0.3 (16 cells a node
// at most): a node looks into 4.4 cells on average, of the 27 around it.  It
// collects the lists that are not empty (in LDS, [NL][256]: all their heads are
// loads of their own) and then walks them as one chain, so that a wave waits for
// its lane with the most nodes and not for the longest list of each cell; nodes
// that the FP32 positions put beyond the range are passed over by one 16-byte
// load.  500 spheres of 642 nodes, range 0.3: 26 us and 21 us for rep_bin, after
// 76 us and 70 us for the sorted cell list (count, scan over 5 million cells,
// scatter, gather) whose 27 cells every node read.  With 8 or 4 cells a node in
// place of 16 the walk takes 33 or 40 us.
// WALLS: some part type interacts with the walls; without it that code, and its
// registers, are left out.
// NL: cells a node may look into: 8 where every cell is at least twice the range
// (two along an axis), else 27.
constexpr int REP_BLOCK = 256;
template <typename R, bool WALLS, int NL>
__global__ void __launch_bounds__(REP_BLOCK) __attribute__((amdgpu_waves_per_eu(WALLS ? 1 : (NL == 8 ? 6 : 4))))
rep_force_kernel(const RepDev* __restrict__ Dp, int parity) {
    __shared__ int first[NL * REP_BLOCK];             // list heads
    __shared__ unsigned char image[NL * REP_BLOCK];   // their cells' periodic images, 2 bits an axis
    const RepDev& D = *Dp;
    const int j = blockIdx.x * REP_BLOCK + threadIdx.x;
    if (j >= D.M) return;
    const int tj = D.type[j];
    const bool pz = !D.walls_z;
    const double p[3] = {D.pos[3 * j], D.pos[3 * j + 1], D.pos[3 * j + 2]};
    ForceSum f;
    if (D.pairs) {
        const int* __restrict__ head = D.head[parity];
        const double range = sqrt(D.range2);
        const int cell = D.cell[j];
        const int cx = cell % D.nc[0], t = cell / D.nc[0], cy = t % D.nc[1], cz = t / D.nc[1];
        int lx, hx, ly, hy, lz, hz;
        offsets(D, 0, p[0], cx, true, range, lx, hx);
        offsets(D, 1, p[1], cy, true, range, ly, hy);
        offsets(D, 2, p[2], cz, pz, range, lz, hz);
        // an axis with fewer than 3 cells: each cell once, the image by rounding
        const bool round_x = D.nc[0] < 3, round_y = D.nc[1] < 3, round_z = pz && D.nc[2] < 3;
        const bool rounds = round_x || round_y || round_z;
        int n = 0;
        for (int dz = lz; dz <= hz; ++dz) {
            int z = cz + dz, iz = 1;  // image 0, 1, 2: shifted by -L, 0, L
            if (pz) {
                if (z < 0) { z += D.nc[2]; iz = 0; }
                else if (z >= D.nc[2]) { z -= D.nc[2]; iz = 2; }
            } else if (z < 0 || z >= D.nc[2]) {
                continue;
            }
            for (int dy = ly; dy <= hy; ++dy) {
                int y = cy + dy, iy = 1;
                if (y < 0) { y += D.nc[1]; iy = 0; }
                else if (y >= D.nc[1]) { y -= D.nc[1]; iy = 2; }
                for (int dx = lx; dx <= hx; ++dx) {
                    int x = cx + dx, ix = 1;
                    if (x < 0) { x += D.nc[0]; ix = 0; }
                    else if (x >= D.nc[0]) { x -= D.nc[0]; ix = 2; }
                    const int u = head[(z * D.nc[1] + y) * D.nc[0] + x];
                    if (u < 0) continue;
                    first[n * REP_BLOCK + threadIdx.x] = u;
                    image[n * REP_BLOCK + threadIdx.x] = (unsigned char)(ix | iy << 2 | iz << 4);
                    ++n;
                }
            }
        }
        // FP32 coordinates and their difference are off by a few 2^-24 of the
        // box length (of |z| where z is not wrapped)
        const double far = range + 0x1p-20 * (fmax(fmax(D.L[0], D.L[1]), D.L[2]) + fabs(p[2]));
        const float far2 = (float)(far * far) * 1.000001f;
        const float px = (float)p[0], py = (float)p[1], pw = (float)p[2];
        int k = -1, u = -1, im = 0;
        // (a node is in one list once: the bound ends the walk whatever the
        // lists hold)
        for (int steps = 0; steps < D.M + 27; ++steps) {
            if (u < 0) {  // the next list
                if (++k >= n) break;
                u = first[k * REP_BLOCK + threadIdx.x];
                im = image[k * REP_BLOCK + threadIdx.x];
            }
            const RepNode o = D.node[u];
            const int w = u;
            u = o.next;
            const int sx = (im & 3) - 1, sy = ((im >> 2) & 3) - 1, sz = (im >> 4) - 1;
            const float qx = px - (o.x + (float)sx * (float)D.L[0]), qy = py - (o.y + (float)sy * (float)D.L[1]),
                        qz = pw - (o.z + (float)sz * (float)D.L[2]);
            if (w == j || !(rounds || qx * qx + qy * qy + qz * qz < far2)) continue;
            double r[3] = {p[0] - (D.pos[3 * w] + sx * D.L[0]), p[1] - (D.pos[3 * w + 1] + sy * D.L[1]),
                           p[2] - (D.pos[3 * w + 2] + sz * D.L[2])};
            if (round_x) r[0] -= D.L[0] * rint(r[0] / D.L[0]);
            if (round_y) r[1] -= D.L[1] * rint(r[1] / D.L[1]);
            if (round_z) r[2] -= D.L[2] * rint(r[2] / D.L[2]);
            pair_force(D, tj, D.type[w], r, f);
        }
    }
    const SoftSphereDev& ws = D.wall[tj];
    if (WALLS && ws.a != 0.0) wall_forces(D, ws, p, f);
    R* out = (R*)D.frep;
    for (int c = 0; c < 3; ++c) out[3 * j + c] = (R)fx_value(f.hi[c], f.lo[c]);
    if (!f.ok) atomicOr(D.status, ST_OVERFLOW);
}

// ---- the nodes in cell order ----

// exclusive scan of the 1024-thread block's values (wave scans, then the
// wave totals); all threads of the block must call it
__device__ __forceinline__ int block_exclusive_scan(int v, int* wsum) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int incl = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int o = __shfl_up(incl, off, 64);
        if (lane >= off) incl += o;
    }
    if (lane == 63) wsum[w] = incl;
    __syncthreads();
    int before = 0;
    for (int k = 0; k < w; ++k) before += wsum[k];
    return before + incl - v;
}

// The four counts of thread t of a block: cnt[4 (1024 b + t) ...], one 16-byte
// access where all four lie below n (cnt is 16-byte aligned).
__device__ __forceinline__ void load4(const int* cnt, int i, int n, int (&v)[4]) {
    if (i + 3 < n) {
        const int4 q = *(const int4*)(cnt + i);
        v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
    } else {
        for (int k = 0; k < 4; ++k) v[k] = i + k < n ? cnt[i + k] : 0;
    }
}
__device__ __forceinline__ void store4(int* a, int i, int n, const int (&v)[4]) {
    if (i + 3 < n) {
        *(int4*)(a + i) = make_int4(v[0], v[1], v[2], v[3]);
    } else {
        for (int k = 0; k < 4; ++k)
            if (i + k < n) a[i + k] = v[k];
    }
}

// exclusive prefix sum of cnt[0, n) in place, per block of 4096 counts (four
// per thread); the block totals go to bsum
__global__ void __launch_bounds__(1024) scan_block_kernel(int* __restrict__ cnt, int* __restrict__ bsum, int n) {
    __shared__ int wsum[16];
    const int i = 4 * (blockIdx.x * 1024 + threadIdx.x);
    int v[4];
    load4(cnt, i, n, v);
    const int t = v[0] + v[1] + v[2] + v[3];
    int acc = block_exclusive_scan(t, wsum);
    int e[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        e[k] = acc;
        acc += v[k];
    }
    store4(cnt, i, n, e);
    if (threadIdx.x == 1023) bsum[blockIdx.x] = acc;
}

__global__ void __launch_bounds__(1024) scan_top_kernel(int* __restrict__ bsum, int nb) {
    // one workgroup: every thread sums a contiguous run, the run sums are
    // scanned across the block, then every thread writes its run's prefixes
    __shared__ int wsum[16];
    const int per = (nb + 1023) / 1024;
    const int b0 = threadIdx.x * per;
    int s = 0;
    for (int k = b0; k < b0 + per && k < nb; ++k) s += bsum[k];
    int acc = block_exclusive_scan(s, wsum);
    for (int k = b0; k < b0 + per && k < nb; ++k) {
        const int t = bsum[k];
        bsum[k] = acc;
        acc += t;
    }
}

// add the block offsets: cnt = cell starts, cursor = a copy for the scatter;
// cnt[n] = total
__global__ void __launch_bounds__(1024) scan_add_kernel(int* __restrict__ cnt, int* __restrict__ cursor,
                                                        const int* __restrict__ bsum, int n, int total) {
    const int i = 4 * (blockIdx.x * 1024 + threadIdx.x);
    if (i < n) {
        int v[4];
        load4(cnt, i, n, v);
        const int b = bsum[blockIdx.x];
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] += b;
        store4(cnt, i, n, v);
        store4(cursor, i, n, v);
    }
    if (i == 0) cnt[n] = total;
}

__global__ void __launch_bounds__(256) rep_scatter_kernel(const RepDev* __restrict__ Dp) {
    const RepDev& D = *Dp;
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= D.M) return;
    const int slot = atomicAdd(&D.cursor[D.cell[j]], 1);
    D.list[slot] = j;
}

__global__ void __launch_bounds__(256) rep_gather_kernel(const RepDev* __restrict__ Dp) {
    const RepDev& D = *Dp;
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= D.M) return;
    const int j = D.list[s];
    for (int c = 0; c < 3; ++c) D.spos[3 * s + c] = D.pos[3 * j + c];
    D.stype[s] = D.type[j];
}

// One thread per node, in cell order (slot s holds node list[s]): the partners in
// the 27 surrounding cells, a neighbour cell across a periodic face shifted by the
// box length; on an axis of one or two cells each cell once, the image by rounding.
template <typename R>
__global__ void __launch_bounds__(256) rep_sorted_kernel(const RepDev* __restrict__ Dp) {
    const RepDev& D = *Dp;
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= D.M) return;
    const int j = D.list[s], tj = D.stype[s], cell = D.cell[j];
    const bool pz = !D.walls_z;
    const double p[3] = {D.spos[3 * s], D.spos[3 * s + 1], D.spos[3 * s + 2]};
    ForceSum f;
    const int cx = cell % D.nc[0], t = cell / D.nc[0], cy = t % D.nc[1], cz = t / D.nc[1];
    const bool round_x = D.nc[0] < 3, round_y = D.nc[1] < 3, round_z = pz && D.nc[2] < 3;
    const int lx = round_x ? 0 : -1, hx = round_x ? D.nc[0] - 1 : 1, ly = round_y ? 0 : -1, hy = round_y ? D.nc[1] - 1 : 1,
              lz = round_z ? 0 : -1, hz = round_z ? D.nc[2] - 1 : 1;
    // the cells x - 1 .. x + 1 of a row without a wrap are one contiguous run of slots
    const bool run3 = !round_x && cx > 0 && cx + 1 < D.nc[0];
    for (int dz = lz; dz <= hz; ++dz) {
        int z = cz + dz;
        double sz = 0.0;  // shift of the neighbour cell's nodes (periodic image)
        if (pz) {
            if (z < 0) { z += D.nc[2]; sz = -D.L[2]; }
            else if (z >= D.nc[2]) { z -= D.nc[2]; sz = D.L[2]; }
        } else if (z < 0 || z >= D.nc[2]) {
            continue;
        }
        for (int dy = ly; dy <= hy; ++dy) {
            int y = cy + dy;
            double sy = 0.0;
            if (y < 0) { y += D.nc[1]; sy = -D.L[1]; }
            else if (y >= D.nc[1]) { y -= D.nc[1]; sy = D.L[1]; }
            const int row = (z * D.nc[1] + y) * D.nc[0];
            for (int dx = run3 ? 0 : lx; dx <= (run3 ? 0 : hx); ++dx) {
                int x = cx + dx;
                double sx = 0.0;
                if (x < 0) { x += D.nc[0]; sx = -D.L[0]; }
                else if (x >= D.nc[0]) { x -= D.nc[0]; sx = D.L[0]; }
                const int u1 = D.cnt[row + (run3 ? cx + 2 : x + 1)];
                for (int u = D.cnt[row + (run3 ? cx - 1 : x)]; u < u1; ++u) {
                    if (u == s) continue;
                    double r[3] = {p[0] - (D.spos[3 * u] + sx), p[1] - (D.spos[3 * u + 1] + sy),
                                   p[2] - (D.spos[3 * u + 2] + sz)};
                    if (round_x) r[0] -= D.L[0] * rint(r[0] / D.L[0]);
                    if (round_y) r[1] -= D.L[1] * rint(r[1] / D.L[1]);
                    if (round_z) r[2] -= D.L[2] * rint(r[2] / D.L[2]);
                    pair_force(D, tj, D.stype[u], r, f);
                }
            }
        }
    }
    const SoftSphereDev& ws = D.wall[tj];
    if (ws.a != 0.0) wall_forces(D, ws, p, f);
    R* out = (R*)D.frep;
    for (int c = 0; c < 3; ++c) out[3 * j + c] = (R)fx_value(f.hi[c], f.lo[c]);
    if (!f.ok) atomicOr(D.status, ST_OVERFLOW);
}

// a[0, n) = v, four per thread (a 16-byte aligned)
__global__ void __launch_bounds__(256) fill_int_kernel(int* __restrict__ a, int n, int v) {
    const int i = 4 * (blockIdx.x * blockDim.x + threadIdx.x);
    const int f[4] = {v, v, v, v};
    if (i < n) store4(a, i, n, f);
}

template <typename R>
hipError_t launch_rep_t(const RepDev& h, const RepDev* d, const void* objs, int nobj, int max_nv, int parity,
                        hipStream_t s) {
    if (h.M == 0) return hipSuccess;
    if (h.sorted)
        hipLaunchKernelGGL(fill_int_kernel, dim3((h.ncell + 1 + 1023) / 1024), dim3(256), 0, s, h.cnt, h.ncell + 1, 0);
    hipLaunchKernelGGL((rep_bin_kernel<R>), dim3(nobj, (max_nv + 255) / 256), dim3(256), 0, s, (const ObjDev<R>*)objs, d,
                       parity);
    if (h.sorted) {
        const int nb = (h.ncell + 4095) / 4096, gm = (h.M + 255) / 256;
        hipLaunchKernelGGL(scan_block_kernel, dim3(nb), dim3(1024), 0, s, h.cnt, h.bsum, h.ncell);
        hipLaunchKernelGGL(scan_top_kernel, dim3(1), dim3(1024), 0, s, h.bsum, nb);
        hipLaunchKernelGGL(scan_add_kernel, dim3(nb), dim3(1024), 0, s, h.cnt, h.cursor, (const int*)h.bsum, h.ncell, h.M);
        hipLaunchKernelGGL(rep_scatter_kernel, dim3(gm), dim3(256), 0, s, d);
        hipLaunchKernelGGL(rep_gather_kernel, dim3(gm), dim3(256), 0, s, d);
        hipLaunchKernelGGL(rep_sorted_kernel<R>, dim3(gm), dim3(256), 0, s, d);
        return hipGetLastError();
    }
    bool walls = false, two = true;
    for (const SoftSphereDev& w : h.wall) walls = walls || w.a != 0.0;
    for (int a = 0; a < 3; ++a) two = two && (h.nc[a] < 3 || h.hc[a] >= 2.0 * (sqrt(h.range2) + 2e-6 * h.hc[a]));
    const void* f = walls ? (two ? (const void*)rep_force_kernel<R, true, 8> : (const void*)rep_force_kernel<R, true, 27>)
                          : (two ? (const void*)rep_force_kernel<R, false, 8> : (const void*)rep_force_kernel<R, false, 27>);
    void* args[] = {(void*)&d, (void*)&parity};
    const hipError_t e = hipLaunchKernel(f, dim3((h.M + REP_BLOCK - 1) / REP_BLOCK), dim3(REP_BLOCK), args, 0, s);
    if (e != hipSuccess) return e;
    return hipGetLastError();
}

}  // namespace

hipError_t launch_repulsion(const RepDev& h, const RepDev* d, const void* objs, int nobj, int max_nv, int parity,
                            int precision, hipStream_t s) {
    return precision == PREC_FP64 ? launch_rep_t<double>(h, d, objs, nobj, max_nv, parity, s)
                                  : launch_rep_t<float>(h, d, objs, nobj, max_nv, parity, s);
}

}  // namespace oif
