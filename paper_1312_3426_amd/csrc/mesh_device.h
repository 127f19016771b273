// mesh_device.h -- device routines of the membrane forces, fluid coupling
// and mesh integration (paper: Section "Elastic interactions" for the
// stretching, bending, local area, global area and volume forces; Section
// "Method" for the IB point dynamics, eq. newton, and the drag coupling,
// eq. dragforce, with linear interpolation of the fluid velocity and
// distribution of the reaction), shared by the membrane kernel and the
// persistent batch kernel.  The outline of the per-object routine is in
// mesh_kernels.hip.
#pragma once

#include <limits.h>
#include <type_traits>

#include "device_common.h"
#include "fixed_point.h"

namespace oif {
namespace dev {

// Accumulation of the reaction force handed to the fluid.  FP32 forms: int64
// fixed point with resolution 2^-e, so sums are exact and independent of the
// order in which mesh nodes add (bitwise reproducible); FP64 form: FP64.
template <int P>
struct Acc {
    // FP32 forms: one int64 word per component, the value times 2^fixed_point_exp
    typedef unsigned long long T;
    static constexpr int WC = 1;    // words per component
    static constexpr int SLOT = 4;  // words per node of G (x, y, z, unused)
    // v * scale is exact (a power of two).  Below 2^51 units the sum with
    // 1.5 * 2^52 rounds it to the nearest integer (ties to even, as the general
    // conversion does) in the low bits of the sum.
    __device__ static void convert(float v, double scale, T* out, unsigned& fl) {
        const double a = (double)v * scale;
        if (__builtin_expect(fabs(a) < 0x1p51, 1)) {
            out[0] = __builtin_bit_cast(T, a + 0x1.8p52) - 0x4338000000000000ull;
            return;
        }
        // below 2^55 units, so a sum of up to 256 values stays in the int64 range
        if (!(fabs(a) < 0x1p55)) {  // out of range or not finite
            fl |= ST_OVERFLOW;
            out[0] = 0ull;
            return;
        }
        out[0] = (T)__double2ll_rn(a);
    }
};

template <>
struct Acc<PREC_FP64> {
    // FP64 form: two int64 words per component, the value split into a
    // multiple of 2^-30 and the remainder in units of 2^-80.  Both integer
    // sums are exact, so the spread force does not depend on the order of the
    // additions (as in the FP32 forms); a value is rounded only below 2^-80,
    // and |value| < 2^25 (else the overflow flag), which leaves room for
    // sums of 256 values.
    typedef unsigned long long T;
    static constexpr int WC = 2;
    static constexpr int SLOT = 8;  // x hi, x lo, y hi, y lo, z hi, z lo, two unused
    __device__ static void convert(double v, double, T* out, unsigned& fl) {
        long long hi, lo;
        if (!fx_split(v, hi, lo)) fl |= ST_OVERFLOW;
        out[0] = (T)hi;
        out[1] = (T)lo;
    }
};

// Add a reaction force to a node's LDS accumulator (3 * WC words).
template <int P>
__device__ __forceinline__ unsigned acc_add(typename Acc<P>::T* acc, typename Prec<P>::R x, typename Prec<P>::R y,
                                            typename Prec<P>::R z, double scale) {
    constexpr int WC = Acc<P>::WC;
    unsigned fl = 0;
    typename Acc<P>::T v[3 * WC];
    Acc<P>::convert(x, scale, v, fl);
    Acc<P>::convert(y, scale, v + WC, fl);
    Acc<P>::convert(z, scale, v + 2 * WC, fl);
#pragma unroll
    for (int w = 0; w < 3 * WC; ++w) atomicAdd(acc + w, v[w]);
    return fl;
}

// Add a node's summed reaction (3 * WC words) to G at lattice node q and set
// its mask bit.
template <int P>
__device__ __forceinline__ void acc_flush(gptr<const BoxDev> B, int parity, int q, const typename Acc<P>::T* v) {
    constexpr int WC = Acc<P>::WC;
    typedef typename Acc<P>::T T;
    T any = 0ull;
#pragma unroll
    for (int w = 0; w < 3 * WC; ++w) any |= v[w];
    if (any == 0ull) return;
    T* G = (T*)B->G[parity] + Acc<P>::SLOT * (size_t)q;
#pragma unroll
    for (int w = 0; w < 3 * WC; ++w)
        if (v[w]) gatomic_add(G + w, v[w]);
    gatomic_or(B->mask + (q >> 6), 1ull << (q & 63));
}

// Lattice index of the (unwrapped) node (gx, gy, gz): periodic in x and y,
// periodic or clamped to the walls in z.
__device__ __forceinline__ int lattice_node(gptr<const BoxDev> B, int gx, int gy, int gz) {
    const int nxb = B->nx, nyb = B->ny, nzb = B->nz;
    gx %= nxb;
    gx += gx < 0 ? nxb : 0;
    gy %= nyb;
    gy += gy < 0 ? nyb : 0;
    if (B->walls_z) {
        gz = gz < 0 ? 0 : (gz >= nzb ? nzb - 1 : gz);
    } else {
        gz %= nzb;
        gz += gz < 0 ? nzb : 0;
    }
    return (gz * nyb + gy) * nxb + gx;
}

// q = a / d, r = a % d for 0 <= a < 2^20 and 0 < d, without an integer
// division: the float estimate a * (1/d) is within one of the quotient.
__device__ __forceinline__ void divmod_small(int a, int d, float rd, int& q, int& r) {
    q = (int)((float)a * rd);
    r = a - q * d;
    if (r < 0) {
        --q;
        r += d;
    } else if (r >= d) {
        ++q;
        r -= d;
    }
}

// a mod n in [0, n)
__device__ __forceinline__ int wrap_mod(int a, int n) {
    const int r = a % n;
    return r < 0 ? r + n : r;
}

// Lower corner of the 2x2x2 stencil of a mesh node at (px, py, pz): nodes sit
// at cell centres, so the stencil starts at floor(x - 1/2) per axis (plus the
// object's integer anchor).  False for a non-finite or runaway position,
// which gets no stencil.
__device__ __forceinline__ bool stencil_corner(double px, double py, double pz, const int* anchor, int (&b)[3]) {
    const double sx = px - 0.5, sy = py - 0.5, sz = pz - 0.5;
    if (!(fabs(sx) < 1e7 && fabs(sy) < 1e7 && fabs(sz) < 1e7)) return false;
    b[0] = anchor[0] + (int)floor(sx);
    b[1] = anchor[1] + (int)floor(sy);
    b[2] = anchor[2] + (int)floor(sz);
    return true;
}

// Arithmetic of the elements.  FP64 form: the library's square root and division.
// FP32 forms: FP64 as well (additions, products and their sums run at the FP32
// rate of unpacked instructions), rounded to FP32 once where a value is stored.
// The hardware's reciprocal and reciprocal square root (good to some 2^-23) are
// refined once, far below that rounding.  The nodes' sums over their corners are
// FP32 in those forms.  Root mean square error of the FP32 form's force over the
// nodes, all moduli: 1.6 units of 2^-24 of the force, where correctly rounded FP32
// operations on the plain rules give 1.9 and FP32 estimates refined once, summed in
// one order or another, 2.3; launch of 500 spheres 56.1 us, with those 55.9 (FP16
// storage 42.8, 41.3).  Sums over the corners in FP64: 0.49 units, 57.2 and 44.1 us
// (5000 cells 565 us, 552 so).
__device__ __forceinline__ double recip(double x) {
    const double r = __builtin_amdgcn_rcp(x);
    return fmadd(r, fmadd(-x, r, 1.0), r);
}
template <typename R>
__device__ __forceinline__ double rsqrt_of(double x) {
    if (sizeof(R) == 8) return 1.0 / sqrt(x);
    const double r = __builtin_amdgcn_rsq(x);
    return fmadd(r, fmadd(-0.5 * x * r, r, 0.5), r);
}
// length L and 1 / L from L^2, both to FP64 in every form (the length's
// difference to the relaxed one cancels): the estimate refined twice
template <typename R>
__device__ __forceinline__ void length_of(double L2, double& L, double& rL) {
    if (sizeof(R) == 8) {
        L = sqrt(L2);
        rL = 1.0 / L;
        return;
    }
    double r = __builtin_amdgcn_rsq(L2);
    const double h = 0.5 * L2;
    r = fmadd(r, fmadd(-h * r, r, 0.5), r);
    r = fmadd(r, fmadd(-h * r, r, 0.5), r);
    L = L2 * r;
    L = fmadd(fmadd(-L, L, L2), 0.5 * r, L);
    rL = r;
}
// 1 / sqrt(x) in the arithmetic type.  FP32: the estimate r refined once with the
// rounding of x r carried along, so that the result is off by half a unit in the
// last place, as the correctly rounded quotient would be
__device__ __forceinline__ double rsqrt_r(double x) { return 1.0 / sqrt(x); }
__device__ __forceinline__ float rsqrt_r(float x) {
    const float r = __builtin_amdgcn_rsqf(x), s = x * r;
    const float e = fmadd(-fmadd(x, r, -s), r, fmadd(-s, r, 1.0f));
    return fmadd(0.5f * r, e, r);
}
// angle of (x, y).  FP32 forms: near the relaxed shape the Taylor series of
// atan (terms to t^7 leave 7e-9 of t at |t| = 1/8), the library's atan2 beyond
template <typename R>
__device__ __forceinline__ R angle_of(double y, double x) {
    if (sizeof(R) == 8) return atan2(y, x);
    if (fabs(y) < 0.125 * x) {
        const float t = (float)(y * recip(x)), t2 = t * t;
        return fmadd(t * t2, fmadd(t2, fmadd(t2, -1.0f / 7.0f, 0.2f), -1.0f / 3.0f), t);
    }
    return atan2f((float)y, (float)x);
}

// Records of a triangle, an edge and a node's corner as loaded (TmplDev), in
// 16- or 32-bit numbers.
struct TriRec {
    int a, b, c;
    double S0;
};
struct EdgeRec {
    int A, B, C, D;
    double L0;
};
struct Corner {
    int a, b, t, ea, eb, o;
    bool t2a, t2b, t2o, valid;  // the triangle is the edge's T2; false: a repeated corner
};
__device__ __forceinline__ double double_of(unsigned lo, unsigned hi) {
    return __builtin_bit_cast(double, (unsigned long long)hi << 32 | lo);
}
template <bool WIDE>
struct Lists;
template <>
struct Lists<false> {
    typedef uint4 Raw;
    const uint4 *tri, *edge, *ring, *rest;
    int rstride;
    template <class TP>
    __device__ __forceinline__ explicit Lists(TP T)
        : tri(T->tri16), edge(T->edge16), ring(T->ring16), rest(T->rest16), rstride(T->rstride) {}
    template <typename V>
    __device__ __forceinline__ static V at(const V* base, int i) { return gat(base, i); }
    __device__ __forceinline__ TriRec triangle(int t) const {
        const uint4 r = gat(tri, t);
        return TriRec{(int)(r.x & 0xffffu), (int)(r.x >> 16), (int)r.y, double_of(r.z, r.w)};
    }
    __device__ __forceinline__ EdgeRec hinge(int e) const {
        const uint4 r = gat(edge, e);
        return EdgeRec{(int)(r.x & 0xffffu), (int)(r.x >> 16), (int)(r.y & 0xffffu), (int)(r.y >> 16), double_of(r.z, r.w)};
    }
    __device__ __forceinline__ Raw raw(int j, int v) const { return gat(ring, j * rstride + v); }
    __device__ __forceinline__ Raw more(int k) const { return gat(rest, k); }
    __device__ __forceinline__ static Corner corner(const Raw& r) {
        return Corner{(int)(r.x & 0xffffu), (int)(r.x >> 16), (int)(r.y & 0xffffu), (int)((r.y >> 16) & 0x7fffu),
                      (int)(r.z & 0x7fffu), (int)((r.z >> 16) & 0x7fffu),
                      (r.y >> 31) != 0u, (r.z & 0x8000u) != 0u, (r.z >> 31) != 0u, r.w != 0u};
    }
};
template <>
struct Lists<true> {
    struct Raw {
        int4 p, q;
    };
    const int4 *tri, *edge, *ring, *rest;
    const double *S0, *L0;
    int rstride;
    template <class TP>
    __device__ __forceinline__ explicit Lists(TP T)
        : tri(T->tri32), edge(T->hinge32), ring(T->ring32), rest(T->rest32), S0(T->S0), L0(T->L0), rstride(T->rstride) {}
    // (64-bit offsets: a mesh that is not in LDS may have arrays beyond 4 GiB)
    template <typename V>
    __device__ __forceinline__ static V at(const V* base, int i) { return gld(base + i); }
    __device__ __forceinline__ TriRec triangle(int t) const {
        const int4 r = gld(tri + t);
        return TriRec{r.x, r.y, r.z, gld(S0 + t)};
    }
    __device__ __forceinline__ EdgeRec hinge(int e) const {
        const int4 r = gld(edge + e);
        return EdgeRec{r.x, r.y, r.z, r.w, gld(L0 + e)};
    }
    __device__ __forceinline__ Raw pair(const int4* p) const { return Raw{gld(p), gld(p + 1)}; }
    __device__ __forceinline__ Raw raw(int j, int v) const { return pair(ring + 2 * ((size_t)j * rstride + v)); }
    __device__ __forceinline__ Raw more(int k) const { return pair(rest + 2 * (size_t)k); }
    __device__ __forceinline__ static Corner corner(const Raw& r) {
        return Corner{r.p.x, r.p.y, r.p.z, r.p.w & 0x7fffffff, r.q.x & 0x7fffffff, r.q.y & 0x7fffffff,
                      r.p.w < 0, r.q.x < 0, r.q.y < 0, r.q.z != 0};
    }
};

// Whether a stencil box of these extents has at most cap nodes (a runaway
// mesh's extents reach 2e7, whose product leaves 64 bits).
__device__ __forceinline__ bool box_fits(long long ex, long long ey, long long ez, int cap) {
    return ex <= cap && ey <= cap && ez <= cap && ex * ey * ez <= cap;  // cap <= 10^6
}

// Stencil marking of one object for split stepping: every lattice node inside
// the 2x2x2 stencil of a finite node position gets its bit in `touch`.  The
// object's stencil box is marked in the bitmask `bits` ((ucap + 31)/32 words)
// first when it fits, so each touched node costs one global atomic however
// many stencils contain it; otherwise every corner goes to `touch` directly.
// Called by the whole workgroup.  The nodes marked: 0 .. nv - 1, or
// order[0 .. nv - 1] when order is not null.
__device__ void mark_object(const double* pos, const int* order, int nv, const int* anchor, gptr<const BoxDev> B,
                            int ucap, unsigned* bits, int* bbox, unsigned long long* touch) {
    __syncthreads();  // earlier users of bits and bbox are done
    if (threadIdx.x == 0) {
        bbox[0] = bbox[1] = bbox[2] = INT_MAX;
        bbox[3] = bbox[4] = bbox[5] = INT_MIN;
    }
    __syncthreads();
    int blo[3] = {INT_MAX, INT_MAX, INT_MAX}, bhi[3] = {INT_MIN, INT_MIN, INT_MIN};
    for (int i = threadIdx.x; i < nv; i += blockDim.x) {
        const int v = order ? gld(order + i) : i;
        const double sx = pos[3 * v] - 0.5, sy = pos[3 * v + 1] - 0.5, sz = pos[3 * v + 2] - 0.5;
        if (!(fabs(sx) < 1e7 && fabs(sy) < 1e7 && fabs(sz) < 1e7)) continue;
        const int bx = anchor[0] + (int)floor(sx), by = anchor[1] + (int)floor(sy),
                  bz = anchor[2] + (int)floor(sz);
        blo[0] = min(blo[0], bx); blo[1] = min(blo[1], by); blo[2] = min(blo[2], bz);
        bhi[0] = max(bhi[0], bx); bhi[1] = max(bhi[1], by); bhi[2] = max(bhi[2], bz);
    }
    wave_bbox_to_block(blo, bhi, bbox);
    __syncthreads();
    const int ox = bbox[0], oy = bbox[1], oz = bbox[2];
    if (bbox[3] < bbox[0]) return;  // no finite node (block-uniform)
    const long long exl = (long long)bbox[3] - ox + 2, eyl = (long long)bbox[4] - oy + 2,
                    ezl = (long long)bbox[5] - oz + 2;
    if (box_fits(exl, eyl, ezl, ucap)) {
        const int ex = (int)exl, exy = (int)(exl * eyl), vol = (int)(exl * eyl * ezl);
        for (int k = threadIdx.x; k < (vol + 31) / 32; k += blockDim.x) bits[k] = 0u;
        __syncthreads();
        for (int i = threadIdx.x; i < nv; i += blockDim.x) {
            const int v = order ? gld(order + i) : i;
            const double sx = pos[3 * v] - 0.5, sy = pos[3 * v + 1] - 0.5, sz = pos[3 * v + 2] - 0.5;
            if (!(fabs(sx) < 1e7 && fabs(sy) < 1e7 && fabs(sz) < 1e7)) continue;
            const int b0 = (anchor[2] + (int)floor(sz) - oz) * exy + (anchor[1] + (int)floor(sy) - oy) * ex +
                           (anchor[0] + (int)floor(sx) - ox);
#pragma unroll
            for (int kk = 0; kk < 8; ++kk) {
                const int k = (kk + (int)threadIdx.x) & 7;
                const int idx = b0 + (k >> 2) * exy + ((k >> 1) & 1) * ex + (k & 1);
                atomicOr(&bits[idx >> 5], 1u << (idx & 31));
            }
        }
        __syncthreads();
        for (int idx = threadIdx.x; idx < vol; idx += blockDim.x) {
            if (!((bits[idx >> 5] >> (idx & 31)) & 1u)) continue;
            const int q = lattice_node(B, ox + idx % ex, oy + (idx / ex) % (int)eyl, oz + idx / exy);
            gatomic_or(touch + (q >> 6), 1ull << (q & 63));
        }
    } else {
        for (int i = threadIdx.x; i < nv; i += blockDim.x) {
            const int v = order ? gld(order + i) : i;
            const double sx = pos[3 * v] - 0.5, sy = pos[3 * v + 1] - 0.5, sz = pos[3 * v + 2] - 0.5;
            if (!(fabs(sx) < 1e7 && fabs(sy) < 1e7 && fabs(sz) < 1e7)) continue;
            const int bx = anchor[0] + (int)floor(sx), by = anchor[1] + (int)floor(sy),
                      bz = anchor[2] + (int)floor(sz);
            for (int k = 0; k < 8; ++k) {
                const int q = lattice_node(B, bx + (k & 1), by + ((k >> 1) & 1), bz + (k >> 2));
                gatomic_or(touch + (q >> 6), 1ull << (q & 63));
            }
        }
    }
}

// The workgroup's fixed LDS besides its dynamic one.
struct MeshShared {
    int bbox[6];      // of mark_object
    int wbox[6][16];  // stencil bounds per wave: low corners, complements of the high ones
};

// CONS: some object of the launch may use the conservative force model (each
// object's template says whether it does); without it that code is left out.
// CPL (meshes too large for LDS only): the coupling area alone sits in LDS, so
// that the stencil-bit ORs and the per-node force sums, whose addresses many
// mesh nodes share, are LDS and not global atomics.
// PH: the whole object in one workgroup (PH_ALL), or one of the two launches
// that split it over T->nslice workgroups (meshes too large for LDS whose
// patches fit there): PH_SUMS, the area and volume sums of slice `slice` of
// the triangles, left in the object's scratch; PH_PATCH, the forces, coupling
// and update of patch `slice` of the nodes, run as an LDS-resident object on
// the patch's sub-template (T->subs[slice]: the patch's nodes first, then the
// other nodes its triangles and hinges reach, with the triangles and hinges
// its nodes' gathers read and corners in local numbering), after the area and
// volume are summed from the slices in a fixed order.
// LISTS: some box of the launch has the membrane kernel clear its coupling
// force (BoxDev::g_by_mesh); without it the list code is left out.
// The membrane forces, coupling and update of object O by the whole
// workgroup; smem is the workgroup's dynamic LDS.
template <int P, bool USE_LDS, bool CONS, bool CPL, int PH = PH_ALL, bool LISTS = true>
__device__ __forceinline__ void mesh_object(const ObjDev<typename Prec<P>::R>& O, unsigned char* smem, MeshShared& sh,
                                            int parity, int mark_next, int slice = 0) {
#pragma clang fp contract(off)
    constexpr bool SPLIT = PH != PH_ALL;
    static_assert(PH != PH_SUMS || (!USE_LDS && CPL), "sums launch: positions alone in LDS");
    static_assert(PH != PH_PATCH || (USE_LDS && !CPL), "patch launch: the patch's sub-template in LDS");
    typedef typename Prec<P>::S S;
    typedef typename Prec<P>::R R;
    typedef Lists<!USE_LDS && PH == PH_ALL> L;  // mesh in the global scratch: 32-bit lists
    const gptr<const TmplDev<R>> Tp = (gptr<const TmplDev<R>>)O.t;  // the object's template
    const gptr<const TmplDev<R>> T = PH == PH_PATCH ? (gptr<const TmplDev<R>>)(Tp->subs + slice) : Tp;
    const gptr<const BoxDev> B = (gptr<const BoxDev>)O.box;
    const int nv = T->nv, nt = T->nt, ne = T->ne;
    const int ucap = T->ucap, ccap = T->ccap;
    const int cons = CONS ? T->conservative : 0;
    const MeshLayout lay = mesh_layout(sizeof(R), nv, nt, ne, ucap, ccap, cons, USE_LDS);
    unsigned char* base = USE_LDS ? smem : O.scratch;
    // node positions (forces phase); the sums launch keeps them alone in LDS
    double* xs = PH == PH_SUMS ? (double*)smem : (double*)(base + lay.xs);
    R* tn = (R*)(base + lay.tn);
    R* tr = (R*)(base + lay.tr);
    R* se = (R*)(base + lay.se);
    R* fh = (R*)(base + lay.fh);
    // area and volume sums of each 64 triangles
    double* sums = PH == PH_SUMS ? (double*)(smem + align16((size_t)nv * 3 * sizeof(double))) : (double*)(base + lay.sums);
    // coupling part: over the forces phase's arrays, alone in LDS (CPL), or
    // beside them in the scratch
    unsigned char* cbase = USE_LDS || CPL ? smem : O.scratch + lay.forces;
    // the nodes this launch updates: all, or the patch (its sub-template's
    // first nodes; T->order maps them to the object's node numbers)
    const int nsl = SPLIT ? T->nslice : 1;
    const int nn = PH == PH_PATCH ? gld(T->slice_off + 1) : nv;
    auto node_of = [&](int i) -> int { return PH == PH_PATCH ? gld(T->order + i) : i; };
    // the slices' area and volume sums, after the object's mesh layout in its scratch
    double* part = SPLIT ? (double*)(O.scratch + split_part_offset(mesh_layout(sizeof(R), Tp->nv, Tp->nt, Tp->ne,
                                                                                ucap, ccap, cons, false)))
                         : nullptr;  // [nslice][2]
    // The staged positions of a split object, in its scratch's forces part: the
    // sums launch leaves them there (each slice its share of the nodes) and the
    // patch launch takes them from there.  A patch stages nodes of its neighbours
    // too, whose workgroups may by then have written their new positions to O.X:
    // not all patches of an object run at once when a launch has more of them than
    // the device holds.
    double* xsplit = SPLIT ? (double*)O.scratch : nullptr;  // [nv of the object][3]

    // When the membrane kernel clears G (B->g_by_mesh): the G slots this object
    // added to in the previous step (G[parity ^ 1], which the lattice kernel
    // has read by now) are zeroed for the step after this one, from the lists
    // the previous step kept (per slice; a whole-object workgroup takes all of
    // them, since the previous step may have run split), and the previous
    // step's flag is reset.  This step's lists start empty.  (Otherwise the
    // lattice kernel clears G and no lists are kept.)
    const bool lists = LISTS && B->g_by_mesh != 0;
    const int kq = T->nslice;
    const size_t qstride = (size_t)ccap + 1;
    if (PH != PH_SUMS && lists) {
        const int np = parity ^ 1;
        unsigned char* Gp = (unsigned char*)B->G[np];
        for (int sl = SPLIT ? slice : 0; sl < (SPLIT ? slice + 1 : kq); ++sl) {
            const int* qo = O.qsave + ((size_t)np * kq + sl) * qstride;
            const int cnt = min(gld(qo), ccap);
            for (int k = threadIdx.x; k < cnt; k += blockDim.x) {
                unsigned long long* g = (unsigned long long*)Gp + Acc<P>::SLOT * (size_t)gld(qo + 1 + k);
#pragma unroll
                for (int w = 0; w < 3 * Acc<P>::WC; ++w) gst(g + w, 0ull);
            }
        }
        if (threadIdx.x == 0) gst(B->gclear + np, 0u);
        if ((int)threadIdx.x < (SPLIT ? 1 : kq))
            gst(O.qsave + ((size_t)parity * kq + (SPLIT ? slice : (int)threadIdx.x)) * qstride, 0);
    }
    unsigned* need = (unsigned*)(cbase + lay.need);
    uint2* pw = (uint2*)(cbase + lay.pw);
    R* ug = (R*)(cbase + lay.ug);
    int* qn = (int*)(cbase + lay.qn);
    typedef typename Acc<P>::T A;
    constexpr int AW = 3 * Acc<P>::WC;  // accumulator words per node
    A* gacc = (A*)(cbase + lay.gacc);
    int(&wbox)[6][16] = sh.wbox;
    const int tid = threadIdx.x, bd = blockDim.x, lane = tid & 63, nwave = (bd + 63) >> 6;
    unsigned flags = 0;

    // Position of node k (component-wise index) the forces and the drag are
    // taken at: X, or with velocity Verlet X + (V + F_last/(2m)), the
    // half-step velocity rounded once.  Staged in LDS for the forces phase and
    // formed again from HBM by the coupling phase (the same expression, so the
    // same bits).
    const R half_im = R(0.5) * O.inv_mass;
    auto stage = [&](int k) -> double {
        const double x = L::at((const double*)O.X, k);
        return O.F ? x + (double)fmadd(L::at((const R*)O.F, k), half_im, L::at((const R*)O.V, k)) : x;
    };
    // The stencil box is found on the way: each wave's bounds are reduced in
    // its lanes and meet in LDS.
    int blo[3] = {INT_MAX, INT_MAX, INT_MAX}, bhi[3] = {INT_MIN, INT_MIN, INT_MIN};
    const int x0 = PH == PH_SUMS ? (int)((long long)nv * slice / nsl) : 0;  // the slice's share of xsplit
    const int x1 = PH == PH_SUMS ? (int)((long long)nv * (slice + 1) / nsl) : 0;
    for (int i = tid; i < nv; i += bd) {
        const int v = PH == PH_PATCH ? gld(T->order + i) : i;
        auto at = [&](int k) -> double { return PH == PH_PATCH ? gat(xsplit, k) : stage(k); };
        const double px = at(3 * v), py = at(3 * v + 1), pz = at(3 * v + 2);
        xs[3 * i] = px;
        xs[3 * i + 1] = py;
        xs[3 * i + 2] = pz;
        if (PH == PH_SUMS && i >= x0 && i < x1) {
            gst(xsplit + 3 * i, px);
            gst(xsplit + 3 * i + 1, py);
            gst(xsplit + 3 * i + 2, pz);
        }
        if (PH == PH_SUMS || i >= nn) continue;
        int b[3];
        if (stencil_corner(px, py, pz, O.anchor, b)) {
            for (int k = 0; k < 3; ++k) {
                blo[k] = min(blo[k], b[k]);
                bhi[k] = max(bhi[k], b[k]);
            }
        } else {
            flags |= ST_NONFINITE;  // no stencil for a non-finite or runaway node
        }
    }
    if (PH != PH_SUMS) {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const int lo = wave_min(blo[k]), hi = wave_min(~bhi[k]);
            if (lane == 63) {
                wbox[k][tid >> 6] = lo;
                wbox[3 + k][tid >> 6] = hi;
            }
        }
    }
    __syncthreads();

    // Coupling, first part: the touched lattice nodes.  The object's stencil
    // box (unwrapped lattice indices [o, o + e)) gets one bit per node that some
    // stencil touches, the touched nodes are numbered compactly, and their
    // lattice indices found.  This needs the positions alone, so it goes first:
    // the populations of the touched nodes (asked for below, one node a thread)
    // then arrive while the forces are computed, a wait of 9 us per object
    // otherwise.  With seven barriers in place of fourteen, the fixed-point
    // conversion by one addition and the mask bits set by rows, the launch of
    // 500 spheres of 642 nodes took 58 us after 72 (FP32), 47 after 59 (FP16),
    // 5000 red cells 732 after 818.
    const int nxb = B->nx, nyb = B->ny, nzb = B->nz;
    int ox = 0, oy = 0, oz = 0, ex = 0, ey = 0, ez = 0, exy = 0, ncomp = 0;
    bool grid = false, compact = false;
    if (PH != PH_SUMS) {
        int v0 = INT_MAX, v1 = INT_MAX;
        if ((lane & 15) < nwave) {
            v0 = wbox[lane >> 4][lane & 15];
            if (lane < 32) v1 = wbox[4 + (lane >> 4)][lane & 15];
        }
        v0 = row_min(v0);
        v1 = row_min(v1);
        ox = __builtin_amdgcn_readlane(v0, 15);
        oy = __builtin_amdgcn_readlane(v0, 31);
        oz = __builtin_amdgcn_readlane(v0, 47);
        const int hx = ~__builtin_amdgcn_readlane(v0, 63), hy = ~__builtin_amdgcn_readlane(v1, 15),
                  hz = ~__builtin_amdgcn_readlane(v1, 31);
        if (hx >= ox) {  // some finite node
            const long long exl = (long long)hx - ox + 2, eyl = (long long)hy - oy + 2, ezl = (long long)hz - oz + 2;
            grid = box_fits(exl, eyl, ezl, ucap);
            if (grid) {
                ex = (int)exl;
                ey = (int)eyl;
                ez = (int)ezl;
                exy = ex * ey;
            }
        }
    }
    if (grid) {
        const int vol = exy * ez, nw = (vol + 31) >> 5;
        for (int k = tid; k < nw; k += bd) need[k] = 0u;
        __syncthreads();
        for (int i = tid; i < nn; i += bd) {
            int b[3];
            if (!stencil_corner(xs[3 * i], xs[3 * i + 1], xs[3 * i + 2], O.anchor, b)) continue;
            const int b0 = (b[2] - oz) * exy + (b[1] - oy) * ex + (b[0] - ox);
            // the rows of the stencil in a lane-rotated order: lanes whose nodes
            // share a cell then hit different words in the same instruction
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
                const int k = (kk + tid) & 3;
                const int idx = b0 + (k >> 1) * exy + (k & 1) * ex;
                const unsigned long long two = 3ull << (idx & 31);
                atomicOr(&need[idx >> 5], (unsigned)two);
                if (two >> 32) atomicOr(&need[(idx >> 5) + 1], (unsigned)(two >> 32));
            }
        }
        __syncthreads();
        // Every wave counts all words and writes the same prefixes, so that it
        // can go on with its own copy, without a barrier.
        int run = 0;
        for (int k0 = 0; k0 < nw; k0 += 64) {
            const int k = k0 + lane;
            const unsigned word = k < nw ? need[k] : 0u;
            const int cnt = __popc(word), incl = wave_scan(cnt);
            if (k < nw) pw[k] = make_uint2(word, (unsigned)(run + incl - cnt));
            run += __builtin_amdgcn_readlane(incl, 63);
        }
        ncomp = run;
        compact = ncomp <= ccap;  // uniform
        if (!USE_LDS && !CPL) __syncthreads();  // the words in global memory
        if (compact) {
            // (the box origin wrapped once, box offsets without integer division)
            const int oxw = wrap_mod(ox, nxb), oyw = wrap_mod(oy, nyb);
            const int ozw = B->walls_z ? oz : wrap_mod(oz, nzb);
            const float rex = 1.0f / (float)ex, rey = 1.0f / (float)ey;
            for (int idx = tid; idx < vol; idx += bd) {
                const uint2 w = pw[idx >> 5];
                if (!((w.x >> (idx & 31)) & 1u)) continue;
                const int c = (int)(w.y + __popc(w.x & ((1u << (idx & 31)) - 1u)));
                int t, dx, dy, dz;
                divmod_small(idx, ex, rex, t, dx);
                divmod_small(t, ey, rey, dz, dy);
                int gx = oxw + dx, gy = oyw + dy, gz = ozw + dz;
                while (gx >= nxb) gx -= nxb;
                while (gy >= nyb) gy -= nyb;
                if (B->walls_z) {
                    if (gz < 0 || gz >= nzb) flags |= ST_CLAMPED;
                    gz = gz < 0 ? 0 : (gz >= nzb ? nzb - 1 : gz);
                } else {
                    while (gz >= nzb) gz -= nzb;
                }
                qn[c] = (gz * nyb + gy) * nxb + gx;
            }
        }
        __syncthreads();
        if (compact && lists) {  // the slots this workgroup adds to, zeroed by it in the next step
            int* qs = O.qsave + ((size_t)parity * kq + (SPLIT ? slice : 0)) * qstride;
            for (int k = tid; k < ncomp; k += bd) gst(qs + 1 + k, qn[k]);
            if (tid == 0) gst(qs, ncomp);
        }
    }
    // corner by corner with lists kept: the lattice kernel clears G[parity]
    // where it reads it in this step
    if (PH != PH_SUMS && lists && !compact && tid == 0) gst(B->gclear + parity, 1u);

    // Fluid velocity u = (sum_i n_i e_i + g/2)/rho at a touched node, in two
    // halves: its populations asked for, and their sums.
    const S* __restrict__ pop = (const S*)B->f[parity];
    const float inv = B->st_inv;
    const R gx_ = (R)B->g[0], gy_ = (R)B->g[1], gz_ = (R)B->g[2];
    const R rho0 = (R)B->rho0, xi = (R)B->xi;
    const unsigned char* bt = B->btype;  // obstacles (null: none)
    auto ask = [&](int q, S(&raw)[19]) {
#pragma unroll
        for (int i = 0; i < 19; ++i) raw[i] = pop_load(pop, i, q);
    };
    auto velocity = [&](int q, const S(&raw)[19], R& x, R& y, R& z) {
#pragma clang fp contract(off)
        if (bt && gld(bt + q)) {  // obstacle node: the wall velocity
            const double* uw = B->wall_u + 3 * gld(bt + q);
            x = (R)gld(uw);
            y = (R)gld(uw + 1);
            z = (R)gld(uw + 2);
            return;
        }
        R dd[19], dr = 0;
#pragma unroll
        for (int i = 0; i < 19; ++i) {
            dd[i] = dec<P>(raw[i], inv);
            dr += dd[i];
        }
        const R jx = dd[1] - dd[2] + dd[7] - dd[8] + dd[9] - dd[10] + dd[11] - dd[12] + dd[13] - dd[14];
        const R jy = dd[3] - dd[4] + dd[7] - dd[8] - dd[9] + dd[10] + dd[15] - dd[16] + dd[17] - dd[18];
        const R jz = dd[5] - dd[6] + dd[11] - dd[12] - dd[13] + dd[14] + dd[15] - dd[16] - dd[17] + dd[18];
        const R ir = R(1) / (rho0 + dr);
        x = (jx + R(0.5) * gx_) * ir;
        y = (jy + R(0.5) * gy_) * ir;
        z = (jz + R(0.5) * gz_) * ir;
    };
    // Triangles, edges and the touched nodes' velocities, side by side: the
    // last waves of the workgroup (a quarter to a third of them) fetch
    // populations, one touched node a lane and up to four rounds, while the
    // others compute the elements, a wave of 64 triangles or edges at a time.
    // Waves of their own because a wave's loads return in order: a fetching
    // wave that also read element records would wait for its populations
    // first.  (The populations of a 642-node sphere lie in some 2000 lines of
    // 128 bytes; all objects of a launch fetch at once: 500 of them read 141 MB and
    // write 23, at the memory's rate half of the launch's time.)  With one 16-byte record
    // per triangle, edge and corner in place of two or three loads, and no
    // branches between a node's corners: 500 spheres FP16 46.7 -> 43.4 us (FP32
    // 58.0 -> 57.3, bound by the fetch), 120 conservative ones FP64 53.1 -> 48.0,
    // 32 uneven boxes 86.6 -> 80.7.
    constexpr int VROUNDS = 4, VDEPTH = sizeof(S) == 8 ? 1 : 2;
    const int nvw = compact ? min((ncomp + 255) >> 8, nwave / 3) : 0;  // fetching waves
    const int cw = nwave - nvw, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    R uv[VROUNDS][3];
    const int vt = tid - 64 * cw, vn = 64 * nvw;  // this lane's first touched node, nodes a round

    const L lists_of(T);
    const double kal = T->kal, ks = T->ks;
    const bool do_s = T->ks != 0.0, do_b = T->kb != 0.0, linear = T->linear != 0;
    auto triangle = [&](int t, const TriRec& q, double r0x, double r0y, double r0z, double& sdarea, double& svol) {
#pragma clang fp contract(off)
        const double ax = xs[3 * q.a], ay = xs[3 * q.a + 1], az = xs[3 * q.a + 2];
        const double abx = xs[3 * q.b] - ax, aby = xs[3 * q.b + 1] - ay, abz = xs[3 * q.b + 2] - az;
        const double acx = xs[3 * q.c] - ax, acy = xs[3 * q.c + 1] - ay, acz = xs[3 * q.c + 2] - az;
        const double nx_ = fmadd(aby, acz, -(abz * acy));
        const double ny_ = fmadd(abz, acx, -(abx * acz));
        const double nz_ = fmadd(abx, acy, -(aby * acx));
        const double n2 = fmadd(nx_, nx_, fmadd(ny_, ny_, nz_ * nz_));  // 4 S^2
        double len, rl;
        length_of<R>(n2, len, rl);
        const double S = 0.5 * len;
        const double dS = sizeof(R) == 8 ? fmadd(0.25, n2, -(q.S0 * q.S0)) / (S + q.S0) : S - q.S0;
        if (PH != PH_SUMS) {  // the sums launch keeps the sums only
            tn[4 * t + 0] = (R)(nx_ * rl);
            tn[4 * t + 1] = (R)(ny_ * rl);
            tn[4 * t + 2] = (R)(nz_ * rl);
            tn[4 * t + 3] = (R)S;
            tr[t] = (R)(-kal * (2.0 * dS * rl));
        }
        sdarea = dS;
        // signed tetrahedron (node 0, a, b, c): a . N = -6 V for inward N
        svol = fmadd(ax - r0x, nx_, fmadd(ay - r0y, ny_, (az - r0z) * nz_));
    };
    // stretching coefficient and bending magnitude of a hinge
    auto edge = [&](int e, const EdgeRec& h, const double2& cs, double kth) {
#pragma clang fp contract(off)
        const double bx = xs[3 * h.B], by = xs[3 * h.B + 1], bz = xs[3 * h.B + 2];
        const double cx_ = xs[3 * h.C], cy_ = xs[3 * h.C + 1], cz_ = xs[3 * h.C + 2];
        const double dx = cx_ - bx, dy = cy_ - by, dz = cz_ - bz;
        const double L2 = fmadd(dx, dx, fmadd(dy, dy, dz * dz));
        double L, rL;
        length_of<R>(L2, L, rL);
        R s = R(0);
        if (do_s) {
            // neo-Hookean kappa = (lam^1/2 + lam^-5/2) / (lam + lam^-3)
            //                   = lam^1/2 (1 + lam^3) / (1 + lam^4)
            double strain, kap = 1.0;
            if (sizeof(R) == 8) {
                // (L - L0)/L0 = (L^2 - L0^2) / (L0 (L + L0))
                strain = fmadd(-h.L0, h.L0, L2) / (h.L0 * (L + h.L0));
                if (!linear) {
                    const double lam = 1.0 + strain, l3 = lam * lam * lam;
                    kap = sqrt(lam) * (1.0 + l3) / fmadd(l3, lam, 1.0);
                }
            } else {
                strain = (L - h.L0) * recip(h.L0);
                if (!linear) {
                    const double lam = 1.0 + strain, l3 = lam * lam * lam;
                    kap = lam * rsqrt_of<R>(lam) * (1.0 + l3) * recip(fmadd(l3, lam, 1.0));
                }
            }
            s = (R)(ks * kap * strain * rL);
        }
        se[e] = s;
        R* q = fh + (cons ? 4 : 1) * e;
        if (!do_b) {
            for (int k = 0; k < (cons ? 4 : 1); ++k) q[k] = R(0);
            return;
        }
        // normals of T1 = (A, B, C) and T2 = (D, C, B) (inward, unnormalised):
        // N1 = (B - A) x (C - B), N2 = (C - B) x (C - D)
        const double ux = bx - xs[3 * h.A], uy = by - xs[3 * h.A + 1], uz = bz - xs[3 * h.A + 2];
        const double wx_ = cx_ - xs[3 * h.D], wy_ = cy_ - xs[3 * h.D + 1], wz_ = cz_ - xs[3 * h.D + 2];
        const double n1x = fmadd(uy, dz, -(uz * dy)), n1y = fmadd(uz, dx, -(ux * dz)), n1z = fmadd(ux, dy, -(uy * dx));
        const double n2x = fmadd(dy, wz_, -(dz * wy_)), n2y = fmadd(dz, wx_, -(dx * wz_)),
                     n2z = fmadd(dx, wy_, -(dy * wx_));
        // theta - pi = atan2((n1 x n2) . e, n1 . n2) for the unit vectors, where
        // N1 x N2 = (C - B) ((B - A) . N2); the difference to theta0 - pi is the
        // angle of the relative rotation, atan2(sin d, cos d), every term scaled
        // by |N1| |N2| > 0
        const double sn = L * fmadd(ux, n2x, fmadd(uy, n2y, uz * n2z));
        const double cn = fmadd(n1x, n2x, fmadd(n1y, n2y, n1z * n2z));
        const R dth = angle_of<R>(fmadd(sn, cs.x, -(cn * cs.y)), fmadd(cn, cs.x, sn * cs.y));
        const R f = (R)kth * dth;
        if (!cons) {
            q[0] = f;
        } else {
            // gradient form: the wing factors w = c / h (c = hbar f, h = |N| / L
            // the wing's distance from the edge line) and the positions a of the
            // wings' feet on the edge, B + a (C - B)
            const R c = (R)lists_of.at(T->hbar, e) * f;
            q[0] = c * (R)(L * rsqrt_of<R>(fmadd(n1x, n1x, fmadd(n1y, n1y, n1z * n1z))));
            q[1] = c * (R)(L * rsqrt_of<R>(fmadd(n2x, n2x, fmadd(n2y, n2y, n2z * n2z))));
            q[2] = (R)(-fmadd(ux, dx, fmadd(uy, dy, uz * dz)) / L2);
            q[3] = (R)((L2 - fmadd(wx_, dx, fmadd(wy_, dy, wz_ * dz))) / L2);
        }
    };
    if (wave >= cw) {
        S raw[VDEPTH][19];
        int qv[VROUNDS];
#pragma unroll
        for (int k = 0; k < VROUNDS + VDEPTH - 1; ++k) {
            if (k < VROUNDS && vt + k * vn < ncomp) {
                qv[k] = qn[vt + k * vn];
                ask(qv[k], raw[k % VDEPTH]);
            }
            const int d = k - (VDEPTH - 1);  // the round whose populations are taken now
            if (d >= 0 && vt + d * vn < ncomp)
                velocity(qv[d], raw[d % VDEPTH], uv[d][0], uv[d][1], uv[d][2]);
        }
    } else {
        // node 0 of the object: the apex of the signed tetrahedra (the patch launch sums none)
        const double r0x = xs[0], r0y = xs[1], r0z = xs[2];
        const int t0 = PH == PH_SUMS ? (int)((long long)nt * slice / nsl) : 0;
        const int t1 = PH == PH_SUMS ? (int)((long long)nt * (slice + 1) / nsl) : nt;
        const int ntc = (t1 - t0 + 63) >> 6;                            // waves of triangles,
        const int nch = ntc + (PH == PH_SUMS ? 0 : (ne + 63) >> 6);     // and of edges after them
        const double2* cs0 = T->cs0;
        const double* kth = T->kth;
        for (int ch = wave; ch < nch; ch += cw) {
            if (ch < ntc) {
                const int t = t0 + 64 * ch + lane;
                double sdarea = 0.0, svol = 0.0;
                if (t < t1) triangle(t, lists_of.triangle(t), r0x, r0y, r0z, sdarea, svol);
                if (PH != PH_PATCH) {
                    sdarea = wave_sum(sdarea);
                    svol = wave_sum(svol);
                    if (lane == 63) {
                        sums[2 * ch] = sdarea;
                        sums[2 * ch + 1] = svol;
                    }
                }
            } else {
                const int e = 64 * (ch - ntc) + lane;
                if (e < ne) edge(e, lists_of.hinge(e), lists_of.at(cs0, e), lists_of.at(kth, e));
            }
        }
    }
    // The object's area and volume: each 64 triangles' sums are taken in the
    // lanes of the wave that computed them and added here in an order of their
    // own, so that the bits do not depend on the number of threads.
    double dSg, Vol;  // Sg - Sg0, volume
    auto block_sums = [&](int n) {
        double s0 = 0.0, s1 = 0.0;
        for (int k = lane; k < n; k += 64) {
            s0 += sums[2 * k];
            s1 += sums[2 * k + 1];
        }
        dSg = lane_value(wave_sum(s0), 63);
        Vol = lane_value(wave_sum(s1), 63) * (-1.0 / 6.0);
    };
    __syncthreads();
    if (PH == PH_SUMS) {
        block_sums(((int)((long long)nt * (slice + 1) / nsl) - (int)((long long)nt * slice / nsl) + 63) >> 6);
        if (tid == 0) {
            gst(part + 2 * slice, dSg);
            gst(part + 2 * slice + 1, Vol);
        }
        return;  // the patch launch reads the slices' sums
    }

    if (PH == PH_ALL) {
        block_sums((nt + 63) >> 6);
    } else {
        // the slices' sums, added in slice order (the same bits in every
        // workgroup of the object)
        dSg = 0.0;
        Vol = 0.0;
        for (int k = 0; k < nsl; ++k) {
            dSg += gld(part + 2 * k);
            Vol += gld(part + 2 * k + 1);
        }
    }
    const double Sg = T->Sg0 + dSg;
    if (tid == 0 && slice == 0 && O.geo) {
        gst(O.geo, Sg);
        gst(O.geo + 1, Vol);
    }
    const double cg = -T->kag * dSg / Sg;                             // global area coefficient
    const double cv3 = -T->kv * (Vol - T->V0) / T->V0 * (1.0 / 3.0);  // volume coefficient, a third
    // (in two parts: their rounding would be the same relative error at every node)
    const R cgh = (R)cg, cgl = (R)(cg - (double)cgh), cvh = (R)cv3, cvl = (R)(cv3 - (double)cvh);

    // 3. nodes (in the patch launch the patch's nodes are the sub-template's
    // first nn nodes, so xs and the corners take the same index).  The
    // node's force from its corners (v, a, b) alone: each hands it the
    // stretching of its edge (v, a), and, as every bending force runs along a
    // triangle's normal, the triangle's normal times the sum of the magnitudes
    // that act on v through it: its own wing (edge (a, b)), the shares of the
    // hinges on (v, a) and (b, v), and the volume force.  (Gathering edges,
    // hinges and triangles by three lists read 24 entries of 8 to 16 bytes and
    // some 150 LDS words per node where the corners take 6 entries of 16 bytes,
    // a wave's entries contiguous, and some 75 words.  Together with the reciprocals
    // of recip and its kin in place of division sequences: launch of 500 spheres
    // of 642 nodes, FP32, 79.2 -> 72.4 us; FP64, 120 conservative ones 64.2 -> 55.8 us.)
    typedef typename L::Raw Raw;
    const int rmax = T->rmax;
    const int* xoff = T->xoff;
    R F0x = 0, F0y = 0, F0z = 0;
    for (int i = tid; i < nn; i += bd) {
        const double px = xs[3 * i], py = xs[3 * i + 1], pz = xs[3 * i + 2];
        // (a corner's terms are one-sided and much larger than the node's force;
        // the host lists opposite corners one after the other, and stretching has a
        // sum of its own, so that the partial sums stay small)
        R Fx = 0, Fy = 0, Fz = 0, Sx = 0, Sy = 0, Sz = 0;
        auto corner = [&](const Raw& raw) {
#pragma clang fp contract(off)
            const Corner c = L::corner(raw);
            const double ax = px - xs[3 * c.a], ay = py - xs[3 * c.a + 1], az = pz - xs[3 * c.a + 2];
            const double bx = px - xs[3 * c.b], by = py - xs[3 * c.b + 1], bz = pz - xs[3 * c.b + 2];
            R s = se[c.ea];
            const R n0 = tn[4 * c.t], n1 = tn[4 * c.t + 1], n2 = tn[4 * c.t + 2], S = tn[4 * c.t + 3];
            // bending: wings along their triangle's normal, edge ends minus
            // half the sum ("Bending force"; conservative model: minus the wing
            // forces split by the positions of the wings' feet)
            R bend;
            if (!cons) {
                bend = fh[c.o] - R(0.5) * (fh[c.ea] + fh[c.eb]);
            } else {
                const R* qa = fh + 4 * c.ea + (c.t2a ? 1 : 0);  // v is the edge's B where the triangle is its T1, else C
                const R* qb = fh + 4 * c.eb + (c.t2b ? 1 : 0);  // v is the edge's C where the triangle is its T1, else B
                bend = fh[4 * c.o + (c.t2o ? 1 : 0)];
                bend = fmadd(c.t2a ? -qa[2] : qa[2] - R(1), qa[0], bend);
                bend = fmadd(c.t2b ? qb[2] - R(1) : -qb[2], qb[0], bend);
            }
            // volume: -kv dV/V0 S n_out / 3
            R cn = fmadd(-cvh, S, fmadd(-cvl, S, bend));
            // local area (-kal dS/S w), global area (-kag dSg/Sg w); w = centroid
            // -> vertex over its length (three times it: (v - a) + (v - b)), or
            // (conservative model) over the RMS length of the triangle's three
            const R wx = (R)(ax + bx), wy = (R)(ay + by), wz = (R)(az + bz);
            R w2 = fmadd(wx, wx, fmadd(wy, wy, wz * wz));
            if (cons) {
                // the mean of |a + b|^2, |b - 2 a|^2 and |a - 2 b|^2, a = v - a and
                // b = v - b: |a + b|^2 / 2 + 3 |b - a|^2 / 2
                const R ux = (R)(bx - ax), uy = (R)(by - ay), uz = (R)(bz - az);
                w2 = fmadd(R(0.5), w2, R(1.5) * fmadd(ux, ux, fmadd(uy, uy, uz * uz)));
            }
            R ct = (tr[c.t] + cgl + cgh) * rsqrt_r(w2);
            // a repeated corner adds nothing (selected, not skipped: without
            // branches the corners' LDS reads overlap)
            ct = c.valid ? ct : R(0);
            cn = c.valid ? cn : R(0);
            s = c.valid ? s : R(0);
            // F_v += ks kappa (L - L0)/L0 (x_a - x_v)/L  ("Stretching force")
            Sx = fmadd(-s, (R)ax, Sx);
            Sy = fmadd(-s, (R)ay, Sy);
            Sz = fmadd(-s, (R)az, Sz);
            Fx = fmadd(ct, wx, fmadd(cn, n0, Fx));
            Fy = fmadd(ct, wy, fmadd(cn, n1, Fy));
            Fz = fmadd(ct, wz, fmadd(cn, n2, Fz));
        };
        if (CONS) {
            // (with the conservative terms six corners side by side spill a
            // hundred registers in the FP32 forms: one ahead instead)
            Raw raw = lists_of.raw(0, i);
#pragma unroll 1
            for (int j = 0; j < rmax; ++j) {
                const Raw cur = raw;
                raw = lists_of.raw(min(j + 1, rmax - 1), i);
                corner(cur);
            }
        } else {
            // the first six corners' entries (most nodes have five to seven) are
            // all in flight before the first is used, and the seventh's with them
            Raw raw[7];
#pragma unroll
            for (int j = 0; j < 7; ++j) raw[j] = lists_of.raw(min(j, rmax - 1), i);
#pragma unroll
            for (int j = 0; j < 6; ++j) corner(raw[j]);
            if (rmax > 6) corner(raw[6]);
        }
        if (xoff) {  // some node has more than seven corners
            const int k1 = gld(xoff + i + 1);
            int k = gld(xoff + i);
            if (k < k1) {
                Raw raw = lists_of.more(k);
#pragma unroll 1
                for (; k < k1; ++k) {
                    const Raw cur = raw;
                    raw = lists_of.more(min(k + 1, k1 - 1));
                    corner(cur);
                }
            }
        }

        Fx += Sx;
        Fy += Sy;
        Fz += Sz;
        // the first node's force stays with its thread
        if (i == tid) {
            F0x = Fx;
            F0y = Fy;
            F0z = Fz;
        } else {
            R* f = O.fel + 3 * node_of(i);
            gst(f, Fx);
            gst(f + 1, Fy);
            gst(f + 2, Fz);
        }
    }

    // Coupling, second part: the reaction forces of all mesh nodes are summed
    // per lattice node in LDS before one global atomic per node and component.
    // The first round's position and velocity are asked for ahead of the
    // barrier.
    double px = 0, py = 0, pz = 0;
    R vx = 0, vy = 0, vz = 0;
    auto fetch = [&](int i) {
        const int v = node_of(i);
        px = lists_of.at((const double*)O.X, 3 * v);
        py = lists_of.at((const double*)O.X, 3 * v + 1);
        pz = lists_of.at((const double*)O.X, 3 * v + 2);
        vx = lists_of.at((const R*)O.V, 3 * v);
        vy = lists_of.at((const R*)O.V, 3 * v + 1);
        vz = lists_of.at((const R*)O.V, 3 * v + 2);
        if (O.F) {  // the half-step velocity, as staged
            vx = fmadd(gld(O.F + 3 * v), half_im, vx);
            vy = fmadd(gld(O.F + 3 * v + 1), half_im, vy);
            vz = fmadd(gld(O.F + 3 * v + 2), half_im, vz);
            px += (double)vx;
            py += (double)vy;
            pz += (double)vz;
        }
    };
    if (tid < nn) fetch(tid);
    __syncthreads();
    if (compact) {
        for (int k = tid; k < AW * ncomp; k += bd) gacc[k] = A(0);
        if (wave >= cw) {
#pragma unroll
            for (int k = 0; k < VROUNDS; ++k) {
                const int c = vt + k * vn;
                if (c < ncomp) {
                    ug[3 * c] = uv[k][0];
                    ug[3 * c + 1] = uv[k][1];
                    ug[3 * c + 2] = uv[k][2];
                }
            }
        }
        for (int c = VROUNDS * vn + tid; c < ncomp; c += bd) {
            const int q = qn[c];
            S raw[19];
            ask(q, raw);
            velocity(q, raw, ug[3 * c], ug[3 * c + 1], ug[3 * c + 2]);
        }
        __syncthreads();
    }

    // per mesh node: interpolate, drag, integrate, spread
    for (int i = tid; i < nn; i += bd) {
        const int v = node_of(i);
        if (i >= bd) {
            fetch(i);
            F0x = lists_of.at((const R*)O.fel, 3 * v);
            F0y = lists_of.at((const R*)O.fel, 3 * v + 1);
            F0z = lists_of.at((const R*)O.fel, 3 * v + 2);
        }
        R dgx = 0, dgy = 0, dgz = 0;
        int sb[3];
        if (stencil_corner(px, py, pz, O.anchor, sb)) {
            const double sx = px - 0.5, sy = py - 0.5, sz = pz - 0.5;
            const R phx = (R)(sx - floor(sx)), phy = (R)(sy - floor(sy)), phz = (R)(sz - floor(sz));
            if (compact) {
                // corners in an order rotated by the node index (the same for
                // any block size): lanes whose nodes share a cell then add to
                // different LDS accumulators in the same instruction; the
                // integer sums do not depend on the order
                const int rot = v & 7;
                const int b0 = (sb[2] - oz) * exy + (sb[1] - oy) * ex + (sb[0] - ox);
                int cr[8];
                R wr[8];
                R ujx = 0, ujy = 0, ujz = 0;
#pragma unroll
                for (int kk = 0; kk < 8; ++kk) {
                    const int k = (kk + rot) & 7;
                    const int dx = k & 1, dy = (k >> 1) & 1, dz = k >> 2;
                    wr[kk] = (dx ? phx : R(1) - phx) * (dy ? phy : R(1) - phy) * (dz ? phz : R(1) - phz);
                    const int idx = b0 + dz * exy + dy * ex + dx;
                    const uint2 w = pw[idx >> 5];
                    cr[kk] = (int)(w.y + __popc(w.x & ((1u << (idx & 31)) - 1u)));
                    ujx = fmadd(wr[kk], ug[3 * cr[kk]], ujx);
                    ujy = fmadd(wr[kk], ug[3 * cr[kk] + 1], ujy);
                    ujz = fmadd(wr[kk], ug[3 * cr[kk] + 2], ujz);
                }
                // eq. dragforce: the fluid receives xi (v - u), the point its opposite
                dgx = xi * (vx - ujx);
                dgy = xi * (vy - ujy);
                dgz = xi * (vz - ujz);
#pragma unroll
                for (int kk = 0; kk < 8; ++kk) {
                    flags |= acc_add<P>(&gacc[AW * cr[kk]], wr[kk] * dgx, wr[kk] * dgy, wr[kk] * dgz,
                                         B->fp_scale);
                }
            } else {
                // stencil box too large for LDS: per-corner loads and atomics
                int ix = sb[0] % nxb;
                ix += ix < 0 ? nxb : 0;
                int iy = sb[1] % nyb;
                iy += iy < 0 ? nyb : 0;
                const int ix1 = ix + 1 == nxb ? 0 : ix + 1;
                const int iy1 = iy + 1 == nyb ? 0 : iy + 1;
                int iz0, iz1;
                const int izr = sb[2];
                if (B->walls_z) {
                    iz0 = izr < 0 ? 0 : (izr >= nzb ? nzb - 1 : izr);
                    iz1 = izr + 1 < 0 ? 0 : (izr + 1 >= nzb ? nzb - 1 : izr + 1);
                    if (izr < 0 || izr + 1 >= nzb) flags |= ST_CLAMPED;
                } else {
                    iz0 = izr % nzb;
                    iz0 += iz0 < 0 ? nzb : 0;
                    iz1 = iz0 + 1 == nzb ? 0 : iz0 + 1;
                }
                R ujx = 0, ujy = 0, ujz = 0;
#pragma unroll 1
                for (int k = 0; k < 8; ++k) {
                    const int dx = k & 1, dy = (k >> 1) & 1, dz = k >> 2;
                    const int qk = ((dz ? iz1 : iz0) * nyb + (dy ? iy1 : iy)) * nxb + (dx ? ix1 : ix);
                    const R wk = (dx ? phx : R(1) - phx) * (dy ? phy : R(1) - phy) * (dz ? phz : R(1) - phz);
                    S raw[19];
                    R ux, uy, uz;
                    ask(qk, raw);
                    velocity(qk, raw, ux, uy, uz);
                    ujx = fmadd(wk, ux, ujx);
                    ujy = fmadd(wk, uy, ujy);
                    ujz = fmadd(wk, uz, ujz);
                }
                dgx = xi * (vx - ujx);
                dgy = xi * (vy - ujy);
                dgz = xi * (vz - ujz);
#pragma unroll 1
                for (int k = 0; k < 8; ++k) {
                    const int dx = k & 1, dy = (k >> 1) & 1, dz = k >> 2;
                    const R wk = (dx ? phx : R(1) - phx) * (dy ? phy : R(1) - phy) * (dz ? phz : R(1) - phz);
                    if (wk == R(0)) continue;
                    A av[AW];
                    Acc<P>::convert(wk * dgx, B->fp_scale, av, flags);
                    Acc<P>::convert(wk * dgy, B->fp_scale, av + AW / 3, flags);
                    Acc<P>::convert(wk * dgz, B->fp_scale, av + 2 * AW / 3, flags);
                    const int qk = ((dz ? iz1 : iz0) * nyb + (dy ? iy1 : iy)) * nxb + (dx ? ix1 : ix);
                    if (bt && gld(bt + qk)) continue;  // an obstacle takes no share
                    acc_flush<P>(B, parity, qk, av);
                }
            }
        }
        // eq. newton.  Symplectic Euler: kick with the total force, then
        // drift.  Velocity Verlet: the second half kick (the drift came
        // first), the total force kept for the next step's first half kick.
        R rx = 0, ry = 0, rz = 0;  // soft-sphere repulsion of this step
        if (O.frep) {
            rx = gld(O.frep + 3 * v);
            ry = gld(O.frep + 3 * v + 1);
            rz = gld(O.frep + 3 * v + 2);
        }
        const R ftx = F0x - dgx + O.fext[0] + rx;
        const R fty = F0y - dgy + O.fext[1] + ry;
        const R ftz = F0z - dgz + O.fext[2] + rz;
        if (O.F) {
            vx = fmadd(ftx, half_im, vx);
            vy = fmadd(fty, half_im, vy);
            vz = fmadd(ftz, half_im, vz);
            gst(O.F + 3 * v, ftx);
            gst(O.F + 3 * v + 1, fty);
            gst(O.F + 3 * v + 2, ftz);
        } else {
            vx = fmadd(ftx, O.inv_mass, vx);
            vy = fmadd(fty, O.inv_mass, vy);
            vz = fmadd(ftz, O.inv_mass, vz);
        }
        gst(O.V + 3 * v, vx);
        gst(O.V + 3 * v + 1, vy);
        gst(O.V + 3 * v + 2, vz);
        const double qx = O.F ? px : px + (double)vx, qy = O.F ? py : py + (double)vy,
                     qz = O.F ? pz : pz + (double)vz;
        gst(O.X + 3 * v, qx);
        gst(O.X + 3 * v + 1, qy);
        gst(O.X + 3 * v + 2, qz);
    }
    if (compact) {
        // one global atomic per touched lattice node and accumulator word
        __syncthreads();
        // (one lane per node and word: a wave's atomics cover the consecutive
        // slots of ~21 nodes (FP32 forms) instead of one component of 64 nodes
        // spread over three arrays)
        for (int k = tid; k < AW * ncomp; k += bd) {
            const int c = k / AW, w = k - AW * c;
            const int q = qn[c];
            const A val = gacc[k];
            if (bt && gld(bt + q)) continue;  // an obstacle takes no share
            if (val != A(0)) gatomic_add((A*)B->G[parity] + Acc<P>::SLOT * (size_t)q + w, val);
        }
        // the mask bits row by row of the stencil box: a row's touched nodes
        // share a mask word or two (a bit where the force is zero only costs a
        // read of that zero)
        for (int r = tid; r < ey * ez; r += bd) {
            const int dz = r / ey, dy = r - dz * ey;
            const int gy = wrap_mod(oy + dy, nyb);
            const int gz = B->walls_z ? min(max(oz + dz, 0), nzb - 1) : wrap_mod(oz + dz, nzb);
            const int row = (gz * nyb + gy) * nxb;
            int gx = wrap_mod(ox, nxb);
            for (int dx = 0; dx < ex;) {
                const int p = row + gx;
                // up to the end of the stencil row, of the lattice row, of the mask word
                const int n = min(min(ex - dx, nxb - gx), min(32, 64 - (p & 63)));
                const int idx = r * ex + dx;
                unsigned long long bits = pw[idx >> 5].x >> (idx & 31);
                if ((idx & 31) + n > 32) bits |= (unsigned long long)pw[(idx >> 5) + 1].x << (32 - (idx & 31));
                bits &= (1ull << n) - 1ull;
                if (bits) gatomic_or(B->mask + (p >> 6), bits << (p & 63));
                dx += n;
                gx = gx + n == nxb ? 0 : gx + n;
            }
        }
    }
    // split stepping: the stencils of the new positions, for the next step
    if (mark_next)  // (mark_object begins with a barrier: every new position is written)
        mark_object(O.X, SPLIT ? T->order : nullptr, nn, O.anchor, B, ucap, need, sh.bbox,
                    B->touch[parity ^ 1]);
    if (flags) gatomic_or(B->status, flags);
}

}  // namespace dev
}  // namespace oif
