// lb_kernels.hip -- lattice kernels of the coupled step (paper, Section
// "Method": the D3Q19 propagation/collision update with an external force
// term, eq. lbequation, and the moment definitions of density and velocity).
//
//   lb_kernel   one lattice node per thread: decode the 19 stored deviations,
//               BGK collision with Guo forcing (force density g + G, the
//               step's G read only where the node's mask bit is set, the bit
//               cleared; the membrane kernel zeroes G in the next step), push the
//               19 post-collision values to the neighbours (halfway
//               bounce-back at z walls), encode.  HBM bound: every node reads
//               and writes 19 stored values once, 2 x 19 x sizeof(storage)
//               bytes per node; the force read adds 24 bytes only at nodes
//               touched by the spreading.
//   diag_kernel FP64 sums of mass and momentum (lattice and membranes) and a
//               non-finite watchdog, with a fixed summation order (deterministic).
//   *_to_*      conversions between the storage form and canonical FP64 fields.
#include <algorithm>

#include "lb_device.h"

namespace oif {
namespace {

using namespace dev;

// the lattice update of one node: lb_device.h

template <int P, bool OBST, bool ALL, bool MRT, bool NT>
__global__ void __launch_bounds__(1024)
lb_kernel(const BoxDev* __restrict__ boxes, const int2* __restrict__ work, int nblocks, int parity,
          int remap, int mode) {
    int bid = blockIdx.x;
    if (remap) {
        // workgroups are dispatched round-robin over the 8 XCDs; give each XCD
        // a contiguous range of lattice blocks so neighbouring planes share an L2
        const int full = nblocks & ~7;
        if (bid < full) bid = (bid & 7) * (full >> 3) + (bid >> 3);
    }
    int box = 0, blk = bid;
    if (work) {
        const int2 w = work[bid];
        box = w.x;
        blk = w.y;
    }
    lb_node<P, OBST, ALL, MRT, NT>(boxes + box, blk * (int)blockDim.x + (int)threadIdx.x, parity, mode);
}

// The sums of a state in one launch: blocks below `nlat` take lattice nodes,
// each of the others `per` objects, and the last block to end adds the partials
// up and writes the ten totals and the status word to host memory.  Every sum
// has a fixed order (a thread's nodes in turn, a tree over the wave, the waves
// in turn; the partials likewise), so which block comes last does not show in
// the bits.  A chain of latencies on all but the largest boxes, which is why
// it is one launch: a call takes 23 us at half a million nodes (12 of them the
// kernel), as three kernels and two copies 50.  1024 threads per block: sixteen
// waves per compute unit keep enough population loads in flight over the
// grid-stride loop.  Objects share blocks where there are too many for blocks of
// their own to start together: 20000 meshes of 42 nodes in four million lattice nodes
// 80 us a call, 314 with a block each.
template <int P>
__global__ void __launch_bounds__(1024)
diag_kernel(const BoxDev* __restrict__ B, const ObjDev<typename Prec<P>::R>* __restrict__ objs, int nlat, int nobj,
            int per, int parity, double* part, double* out) {
    typedef typename Prec<P>::S S;
    __shared__ double red[5][16];
    __shared__ bool last;
    const int t = threadIdx.x, wave = t >> 6, blk = blockIdx.x;
    double s[5] = {0, 0, 0, 0, 0};
    double scale = 1.0;
    if (blk < nlat) {
        const S* __restrict__ src = (const S*)B->f[parity];
        const int N = B->N;
        const float inv = B->st_inv;
        for (int p = blk * 1024 + t; p < N; p += nlat * 1024) {
            double d[19];
#pragma unroll
            for (int i = 0; i < 19; ++i) {
                d[i] = (double)dec<P>(pop_load(src, i, p), inv);
                if (!isfinite(d[i])) s[4] = 1.0;
            }
#pragma unroll
            for (int i = 0; i < 19; ++i) {
                s[0] += d[i];
                s[1] += cx(i) * d[i];
                s[2] += cy(i) * d[i];
                s[3] += cz(i) * d[i];
            }
        }
    } else if (const int w = 16 / per, o = (blk - nlat) * per + wave / w; o < nobj) {  // w waves an object
        const ObjDev<typename Prec<P>::R>& O = objs[o];
        const int nv = O.t->nv;
        for (int v = (wave % w) * 64 + (t & 63); v < nv; v += 64 * w) {
            const double a = O.V[3 * v], b = O.V[3 * v + 1], c = O.V[3 * v + 2];
            s[1] += a;
            s[2] += b;
            s[3] += c;
            if (!isfinite(a + b + c) || !isfinite(O.X[3 * v] + O.X[3 * v + 1] + O.X[3 * v + 2])) s[4] = 1.0;
        }
        scale = O.mass;
    }
#pragma unroll
    for (int c = 0; c < 5; ++c) {
        const double w = wave_sum(s[c]);
        if ((t & 63) == 63) red[c][wave] = c > 0 && c < 4 ? scale * w : w;
    }
    __syncthreads();
    if (t < 5) {
        double tot = 0.0;
        for (int k = 0; k < 16; ++k) tot += red[t][k];
        // an exchange whose old value has come back is in device memory, so no
        // fence is needed before the count (a release here writes each XCD's L2
        // back, and with it what the step left there: 84 us instead of 12 at half a
        // million nodes)
        const double old = __hip_atomic_exchange(part + 5 * (size_t)blk + t, tot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("" ::"v"(old));
    }
    __syncthreads();
    unsigned* ctr = B->status + STATUS_DIAG_CTR;
    if (t == 0) {
        last = __hip_atomic_fetch_add(ctr, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1;
        if (last) __hip_atomic_store(ctr, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // for the next launch
    }
    __syncthreads();
    if (!last) return;
    // the lower half of the block adds the lattice's partials, the upper half the objects'
    const int g = t >> 9, n = g ? (int)gridDim.x - nlat : nlat;
    const double* p = part + (g ? 5 * (size_t)nlat : 0);
    double q[5] = {0, 0, 0, 0, 0};
    for (int k = t & 511; k < n; k += 512)
#pragma unroll
        for (int c = 0; c < 5; ++c)
            q[c] += __hip_atomic_load(p + 5 * (size_t)k + c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
    for (int c = 0; c < 5; ++c) {
        const double w = wave_sum(q[c]);
        if ((t & 63) == 63) red[c][wave] = w;
    }
    __syncthreads();
    double* word = out + t;
    if (t < 10) {
        const int c = t % 5, w0 = t / 5 * 8;
        double tot = 0.0;
        for (int k = 0; k < 8; ++k) tot += red[c][w0 + k];
        __hip_atomic_store(word, tot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    } else if (t == 10) {
        const unsigned st = __hip_atomic_load(B->status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(word, (double)st, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

__device__ inline double weight_of(int i) { return i == 0 ? 1.0 / 3.0 : (i <= 6 ? 1.0 / 18.0 : 1.0 / 36.0); }

// full populations n_i = w_i rho0 + d_i (dev = 0), or the stored deviations
// d_i alone (dev = 1), which FP64 holds exactly in every storage form
template <int P>
__global__ void pops_to_f64_kernel(const BoxDev* __restrict__ B, int parity, double* __restrict__ out, int dev) {
    typedef typename Prec<P>::S S;
    const int N = B->N;
    const size_t k = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= (size_t)19 * N) return;
    const int i = (int)(k / N), p = (int)(k - (size_t)i * N);
    const S* src = (const S*)B->f[parity];
    const double d = (double)dec<P>(pop_load(src, i, p), B->st_inv);
    out[k] = dev ? d : weight_of(i) * B->rho0 + d;
}

template <int P>
__global__ void f64_to_pops_kernel(const BoxDev* __restrict__ B, int parity, const double* __restrict__ in,
                                   int dev) {
    typedef typename Prec<P>::S S;
    typedef typename Prec<P>::R R;
    const int N = B->N;
    const size_t k = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= (size_t)19 * N) return;
    const int i = (int)(k / N), p = (int)(k - (size_t)i * N);
    S* dst = (S*)B->f[parity];
    pop_store(dst, i, p, enc<P>((R)(dev ? in[k] : in[k] - weight_of(i) * B->rho0), B->st_scale));
}

template <int P>
__global__ void moments_kernel(const BoxDev* __restrict__ B, int first, int count, int parity,
                               double* __restrict__ rho, double* __restrict__ u) {
    typedef typename Prec<P>::S S;
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= count) return;
    const int p = first + k;
    if (B->btype && B->btype[p]) {  // obstacle node: rho0 and the wall velocity
        const double* uw = B->wall_u + 3 * B->btype[p];
        if (rho) rho[k] = B->rho0;
        if (u) {
            u[k] = uw[0];
            u[count + k] = uw[1];
            u[2 * count + k] = uw[2];
        }
        return;
    }
    const S* src = (const S*)B->f[parity];
    double d[19];
#pragma unroll
    for (int i = 0; i < 19; ++i) d[i] = (double)dec<P>(pop_load(src, i, p), B->st_inv);
    double dr = 0, jx = 0, jy = 0, jz = 0;
#pragma unroll
    for (int i = 0; i < 19; ++i) {
        dr += d[i];
        jx += cx(i) * d[i];
        jy += cy(i) * d[i];
        jz += cz(i) * d[i];
    }
    const double r = B->rho0 + dr;
    if (rho) rho[k] = r;
    if (u) {
        u[k] = (jx + 0.5 * B->g[0]) / r;
        u[count + k] = (jy + 0.5 * B->g[1]) / r;
        u[2 * count + k] = (jz + 0.5 * B->g[2]) / r;
    }
}

// device arrays into a slot of host memory in one launch
__global__ void __launch_bounds__(256) gather_kernel(GatherSrc src, unsigned* __restrict__ dst) {
    unsigned base = 0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const unsigned* __restrict__ q = (const unsigned*)src.p[a];
        for (unsigned i = blockIdx.x * 256 + threadIdx.x; i < src.n[a]; i += gridDim.x * 256) dst[base + i] = q[i];
        base += src.n[a];
    }
}

// plain streaming copy, 16 bytes per thread (bandwidth reference)
__global__ void __launch_bounds__(256) copy_kernel(const float4* __restrict__ src, float4* __restrict__ dst,
                                                   size_t n) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = src[i];
}

}  // namespace

hipError_t launch_copy(const void* src, void* dst, size_t bytes, hipStream_t s) {
    const size_t n = bytes / 16;
    hipLaunchKernelGGL(copy_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, (const float4*)src,
                       (float4*)dst, n);
    return hipGetLastError();
}

#define OIF_DISPATCH_P(prec, KER, grid, blk, s, ...)                                               \
    switch (prec) {                                                                              \
        case PREC_FP64: hipLaunchKernelGGL(KER<PREC_FP64>, grid, blk, 0, s, __VA_ARGS__); break; \
        case PREC_FP32: hipLaunchKernelGGL(KER<PREC_FP32>, grid, blk, 0, s, __VA_ARGS__); break; \
        case PREC_FP16: hipLaunchKernelGGL(KER<PREC_FP16>, grid, blk, 0, s, __VA_ARGS__); break; \
        case PREC_BF16: hipLaunchKernelGGL(KER<PREC_BF16>, grid, blk, 0, s, __VA_ARGS__); break; \
        default: return hipErrorInvalidValue;                                                    \
    }

template <int P>
void launch_lb_p(const LbLaunch& L) {
#define OIF_LB(O, A, M, NT)                                                                                     \
    hipLaunchKernelGGL((lb_kernel<P, O, A, M, NT>), dim3(L.nblocks), dim3(L.block), 0, L.stream, L.boxes, L.work, \
                       L.nblocks, L.parity, L.remap, L.mode)
#define OIF_LB_M(O, A, NT)             \
    if (L.mrt) OIF_LB(O, A, true, NT); \
    else OIF_LB(O, A, false, NT)
    // the split step's two launches keep ordinary reads
    const bool all = L.mode == LB_ALL;
    if (L.obstacles) {
        if (!all) OIF_LB_M(true, false, false);
        else if (L.nt) OIF_LB_M(true, true, true);
        else OIF_LB_M(true, true, false);
    } else {
        if (!all) OIF_LB_M(false, false, false);
        else if (L.nt) OIF_LB_M(false, true, true);
        else OIF_LB_M(false, true, false);
    }
#undef OIF_LB_M
#undef OIF_LB
}

hipError_t launch_lb(const LbLaunch& L) {
    switch (L.precision) {
        case PREC_FP64: launch_lb_p<PREC_FP64>(L); break;
        case PREC_FP32: launch_lb_p<PREC_FP32>(L); break;
        case PREC_FP16: launch_lb_p<PREC_FP16>(L); break;
        case PREC_BF16: launch_lb_p<PREC_BF16>(L); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_diag(const BoxDev* box_dev, int N, const void* objs, int nobj, int max_nv, int precision, int parity,
                       double* partials, double* out, hipStream_t s) {
    const int nlat = diag_lattice_blocks(N);
    // objects a block takes: one while all blocks start together (two to a
    // compute unit), of more as many as leave a thread about four nodes
    const int per = nobj <= 512 || max_nv > 1024 ? 1 : (max_nv > 256 ? 4 : 16);
#define OIF_DIAG(P)                                                                                               \
    case P:                                                                                                       \
        hipLaunchKernelGGL(diag_kernel<P>, dim3(nlat + (nobj + per - 1) / per), dim3(1024), 0, s, box_dev,        \
                           (const ObjDev<typename Prec<P>::R>*)objs, nlat, nobj, per, parity, partials, out);     \
        break
    switch (precision) {
        OIF_DIAG(PREC_FP64);
        OIF_DIAG(PREC_FP32);
        OIF_DIAG(PREC_FP16);
        OIF_DIAG(PREC_BF16);
        default: return hipErrorInvalidValue;
    }
#undef OIF_DIAG
    return hipGetLastError();
}

hipError_t launch_pops_to_f64(const BoxDev* box_dev, int N, int precision, int parity, double* out,
                              int deviations, hipStream_t s) {
    const size_t n = (size_t)19 * N;
    OIF_DISPATCH_P(precision, pops_to_f64_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), s, box_dev,
                   parity, out, deviations);
    return hipGetLastError();
}

hipError_t launch_f64_to_pops(const BoxDev* box_dev, int N, int precision, int parity,
                              const double* in, int deviations, hipStream_t s) {
    const size_t n = (size_t)19 * N;
    OIF_DISPATCH_P(precision, f64_to_pops_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), s, box_dev,
                   parity, in, deviations);
    return hipGetLastError();
}

hipError_t launch_moments(const BoxDev* box_dev, int first, int count, int precision, int parity, double* rho,
                          double* u, hipStream_t s) {
    OIF_DISPATCH_P(precision, moments_kernel, dim3((unsigned)((count + 255) / 256)), dim3(256), s, box_dev, first,
                   count, parity, rho, u);
    return hipGetLastError();
}

hipError_t launch_gather(const GatherSrc& src, void* dst, hipStream_t s) {
    const unsigned n = std::max(src.n[0], std::max(src.n[1], src.n[2]));
    hipLaunchKernelGGL(gather_kernel, dim3(std::min(256u, (n + 255) / 256)), dim3(256), 0, s, src, (unsigned*)dst);
    return hipGetLastError();
}

}  // namespace oif
