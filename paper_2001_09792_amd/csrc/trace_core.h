// trace_core.h -- the per-ray traversal of the two-level hierarchy, shared by
// the trace entry points and the render passes (both in trace.hip / render.hip).
//
// Per ray: test the W child boxes of the current node (robust slab test: the
// far distance is widened by 2*gamma_3, after Ize 2013, so rounding never
// drops a box the ray touches), continue with the nearest hit child and push
// the others far-to-near.  At a top-level leaf the ray is moved into the
// instance's object space: the ray is mapped with the world->object
// matrix in double (t is unchanged by the map), and its origin is slid to
// where it enters the bottom level's root box, so float32 coordinates stay
// box-sized; the slide t0 is added back to every t.  At a bottom-level leaf each
// triangle is tested with the watertight ray/triangle test of Woop, Benthin &
// Wald (JCGT 2013): vertices are sheared into ray space and three 2-D edge
// functions decide inside/outside; evaluated without fused multiply-add, a
// shared edge gives exactly negated values in its two triangles, so no ray
// passes between them.  Edges and vertices count as inside (two-sided,
// closed), a zero determinant (ray parallel to the plane) is a miss.
// Closest hit keeps the least t (ties: lowest instance, then primitive);
// any hit stops at the first triangle in [tmin, tmax].
#pragma once

#include "rg_internal.h"
#include "trace_lds.h"

namespace rgt {

constexpr uint32_t kFlip = 4u;  // in Tracer::cull: the instance flips its facing
// rounds a wave may run without any of its rays finishing: far above any
// traversal of a valid hierarchy (a loop bound, not a limit of the method)
constexpr uint32_t kMaxSteps = 1u << 22;
// The far distance of a slab is widened by 2 gamma_5 (gamma_n = n u / (1 - n u),
// u = 2^-24): the subtraction, the hardware reciprocal (1 ulp) and the product
// each add error to t, and the near distance may err the other way.
constexpr float kFarWiden = 2.0f * (5.0f * 5.9604645e-8f) / (1.0f - 5.0f * 5.9604645e-8f);
// Slab distances are computed as fma(plane, inv, -c): one rounding less in
// the relative error than (plane - o) * inv, but c = o * inv is rounded (by
// up to u |o inv|) and so is the shifted constant (u |c'|).  Shifting c by
// 3 u |o| |inv| (slightly more) towards the side that widens the slab keeps
// the lo-plane and hi-plane distances on the safe side of the exact ones.
constexpr float kSlabShift = 3.0f * 5.9604645e-8f * 1.01f;

#define RG_GLOBAL __attribute__((address_space(1)))
#define RG_LDS __attribute__((address_space(3)))

template <class T>
__device__ inline const RG_GLOBAL T *gptr(const void *p) {
    return (const RG_GLOBAL T *)(p);
}

typedef uint32_t rg_u4 __attribute__((ext_vector_type(4)));
typedef uint32_t rg_u2 __attribute__((ext_vector_type(2)));
typedef uint32_t rg_u4a8 __attribute__((ext_vector_type(4), aligned(8)));  // 16 bytes at 8-byte alignment

// Loads element i of a global array of T with global_load (T's size a
// multiple of 16 bytes and 16-byte aligned, or of 8 bytes for rg_u2 pieces).
template <class T, class V = rg_u4>
__device__ inline T gload(const void *base, uint64_t i) {
    static_assert(sizeof(T) % sizeof(V) == 0, "size");
    T out;
    const RG_GLOBAL V *src = (const RG_GLOBAL V *)((const char *)base + i * sizeof(T));
    V *dst = reinterpret_cast<V *>(&out);
#pragma unroll
    for (uint32_t k = 0; k < sizeof(T) / sizeof(V); ++k) dst[k] = src[k];
    return out;
}

enum Mode { kClosest = 0, kCounts = 1, kRender = 2 };
struct Ray {
    float o[3], d[3], tmin, tmax;
};

// Result of one traversal: which triangle is hit.  For kRender `inst` is the
// top-level record index and `prim` the bottom-level triangle slot (leaf
// order); otherwise they are the input indices.  The hit's t is the
// tracer's `best` (closest hit); the trace entry points recompute t and the
// barycentrics of the chosen triangle in double afterwards (k_refine).
struct Hit {
    uint32_t inst, prim;
    uint32_t n_nodes, n_tris, n_inst;  // visit counts (kCounts)
};

__device__ inline float safe_rcp(float x) {
    // zero components get a huge finite reciprocal of the same sign, so that
    // (lo - o) * inv never evaluates 0 * inf; hardware reciprocal (1 ulp)
    const float tiny = 1e-30f;
    float y = fabsf(x) < tiny ? copysignf(tiny, x) : x;
    return __builtin_amdgcn_rcpf(y);
}

__device__ inline float bsel(uint32_t m, float a, float b) {  // m all ones: a, m zero: b (one v_bfi_b32)
    const uint32_t x = __float_as_uint(a), y = __float_as_uint(b);
    return __uint_as_float((m & x) | (~m & y));
}

// Ray-space shear constants (Woop, Benthin & Wald 2013).  The axes are the
// rotation (kx, ky, kz) = (kz + 1, kz + 2, kz) that puts the direction's
// largest component at z, held as two lane masks (z0: kz = 0, z1: kz = 1,
// neither: kz = 2), so that a vertex is rotated with two bit selects per
// component: compares of an axis number end up as branches, which cost a
// dozen scalar instructions each.  The published form also swaps x and y
// when d[kz] < 0; the swap only negates the edge functions, det and T
// together (exactly: every operation is odd), which no decision here reads
// but the facing (see `cull`).
struct Shear {
    uint32_t z0, z1;
    float sx, sy, sz;
    __device__ inline float z(const float v[3]) const { return bsel(z0, v[0], bsel(z1, v[1], v[2])); }
    __device__ inline float x(const float v[3]) const { return bsel(z0, v[1], bsel(z1, v[2], v[0])); }
    __device__ inline float y(const float v[3]) const { return bsel(z0, v[2], bsel(z1, v[0], v[1])); }
};

// Returns whether d[kz] < 0.
__device__ inline bool make_shear(const float d[3], Shear &s) {
    const float ax = fabsf(d[0]), ay = fabsf(d[1]), az = fabsf(d[2]);
    const bool xy = ax > ay;
    s.z0 = (xy && ax > az) ? ~0u : 0u;
    s.z1 = (!xy && ay > az) ? ~0u : 0u;
    // any consistent constants keep the test watertight: the same values
    // serve every triangle of the instance
    const float dz = s.z(d), rz = __builtin_amdgcn_rcpf(dz);
    s.sx = s.x(d) * rz;
    s.sy = s.y(d) * rz;
    s.sz = rz;
    return dz < 0.0f;
}

// Watertight ray/triangle test in ray space.  Returns true on a hit whose
// t (in the ray's own frame) lies in [lo, hi] (up to a relative 1e-6 slack
// on either side, settled by the caller on the exact quotient), and writes
// T and det (t = T / det) and the edge values V, W (u = V / det, v = W / det).
// No division is done here: most triangles fail the edge or range test.
// Straight-line: the lanes of a wave rarely agree, so an early way out saves
// nothing and each costs an exchange of the lane mask.
__device__ inline bool tri_test(const float tv[9], const float o[3], const Shear &s, float lo, float hi,
                                float &T_out, float &det_out, float &V_out, float &W_out) {
#pragma clang fp contract(off)
    const float a[3] = {tv[0] - o[0], tv[1] - o[1], tv[2] - o[2]};
    const float b[3] = {tv[3] - o[0], tv[4] - o[1], tv[5] - o[2]};
    const float c[3] = {tv[6] - o[0], tv[7] - o[1], tv[8] - o[2]};
    const float az = s.z(a), bz = s.z(b), cz = s.z(c);
    const float Ax = s.x(a) - s.sx * az, Ay = s.y(a) - s.sy * az;
    const float Bx = s.x(b) - s.sx * bz, By = s.y(b) - s.sy * bz;
    const float Cx = s.x(c) - s.sx * cz, Cy = s.y(c) - s.sy * cz;
    const float U = Cx * By - Cy * Bx;
    const float V = Ax * Cy - Ay * Cx;
    const float W = Bx * Ay - By * Ax;
    const float least = fminf(fminf(U, V), W), most = fmaxf(fmaxf(U, V), W);
    const float det = U + V + W;
    const float T = U * (s.sz * az) + V * (s.sz * bz) + W * (s.sz * cz);
    // range test without dividing: t in [lo, hi] <=> T in det*[lo, hi] for
    // det > 0 (reversed for det < 0); a small slack keeps it conservative
    const float ad = fabsf(det), sT = det < 0.0f ? -T : T;
    const float slack = 1e-6f * ad * fmaxf(fabsf(lo), fabsf(hi));
    T_out = T;
    det_out = det;
    V_out = V;
    W_out = W;
    return !((least < 0.0f) & (most > 0.0f)) & (det != 0.0f) & !(sT > hi * ad + slack) & !(sT < lo * ad - slack);
}

// Stack with the first n_lds entries in LDS (lane-interleaved, so the
// 64 lanes of a wave hit 64 different banks) and the rest in private memory.
// LDS: the caller has seen that no lane of the wave needs the private part
// this round, and nothing branches per entry.
struct Stack {
    uint32_t RG_LDS *lds;  // base of this lane's column: lds[e * kThreads]
    uint32_t *priv;        // kPrivStack further entries (a private array of the kernel)
    int sp;
    int n_lds;             // entries kept in LDS (8..kMaxLdsStack)
    template <bool LDS>
    __device__ inline void push_if(uint32_t v, bool keep) {
        if (LDS) {  // the entry goes to the top whether or not it stays
            lds[sp * kThreads] = v;
            sp += keep ? 1 : 0;
        } else if (keep) {
            if (sp < n_lds) lds[sp * kThreads] = v;
            else priv[sp - n_lds] = v;
            ++sp;
        }
    }
    template <bool LDS>
    __device__ inline uint32_t pop() {
        --sp;
        return (LDS || sp < n_lds) ? lds[sp * kThreads] : priv[sp - n_lds];
    }
};

template <int W>
__device__ inline void sort_children(float tn[W], uint32_t ch[W]) {
    // selects of values (not a swap under a branch)
#define RG_CSWAP(i, j)                                            \
    {                                                             \
        const bool s_ = tn[j] < tn[i];                            \
        const float ta_ = s_ ? +tn[j] : +tn[i], tb_ = s_ ? +tn[i] : +tn[j]; \
        const uint32_t ca_ = s_ ? ch[j] + 0u : ch[i] + 0u, cb_ = s_ ? ch[i] + 0u : ch[j] + 0u; \
        tn[i] = ta_; tn[j] = tb_;                                 \
        ch[i] = ca_; ch[j] = cb_;                                 \
    }
    if constexpr (W == 2) {
        RG_CSWAP(0, 1)
    } else if constexpr (W == 4) {
        RG_CSWAP(0, 1) RG_CSWAP(2, 3) RG_CSWAP(0, 2) RG_CSWAP(1, 3) RG_CSWAP(1, 2)
    } else {
        RG_CSWAP(0, 1) RG_CSWAP(2, 3) RG_CSWAP(4, 5) RG_CSWAP(6, 7)
        RG_CSWAP(0, 2) RG_CSWAP(1, 3) RG_CSWAP(4, 6) RG_CSWAP(5, 7)
        RG_CSWAP(1, 2) RG_CSWAP(5, 6) RG_CSWAP(0, 4) RG_CSWAP(3, 7)
        RG_CSWAP(1, 5) RG_CSWAP(2, 6)
        RG_CSWAP(1, 4) RG_CSWAP(3, 6)
        RG_CSWAP(2, 4) RG_CSWAP(3, 5)
        RG_CSWAP(3, 4)
    }
#undef RG_CSWAP
}

// The wave's lanes named by a mask: the compiler takes the mask itself as the
// branch's execution mask (no per-lane flags to keep and to compare).
__device__ inline bool lane_in(uint64_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }
__device__ inline uint64_t ballot(bool b) { return __builtin_amdgcn_ballot_w64(b); }

// Opacity of the micro-triangle holding barycentrics (u, v) of a triangle cut
// into 4^level: cell (floor(n u), floor(n v)), n = 2^level, upright or
// inverted, numbered row by row (row j starts at j (2n - j)).
__device__ inline bool alpha_open(uint64_t mask, uint32_t level, float u, float v) {
    const int n = 1 << level;
    const float U = u * (float)n, V = v * (float)n;
    int i = (int)floorf(U), j = (int)floorf(V);
    i = i < 0 ? 0 : (i > n - 1 ? n - 1 : i);
    j = j < 0 ? 0 : (j > n - 1 - i ? n - 1 - i : j);
    const int inv = ((U - (float)i) + (V - (float)j) > 1.0f && i + j < n - 1) ? 1 : 0;
    return ((mask >> (j * (2 * n - j) + 2 * i + inv)) & 1ull) != 0ull;
}

// Traversal of the 64 rays of a wave as a resumable state machine: begin()
// loads a lane's ray, round() performs one unit of work (an inner node, an
// instance entry, or a leaf's next two triangles, then the pop) for the lanes
// it picks and reports which rays are finished.  The kernels run many rays
// per lane through it, so that lanes whose ray has finished can take a new
// one while the others continue.
//
// What bounds it is the issue of vector instructions under divergence, so the
// round is laid out for few of them:
//  - Which lanes hold a ray, which of those are inside an instance and which
//    run what are wave-wide masks in scalar registers, not per-lane flags.
//  - The unit kinds are separate `if`s one after another, not an if / else
//    chain, and each updates the lane's state in place.  In a chain the old
//    state stays live beside the new one until the join, which then copies
//    every register of it twice per round (56 moves of about 300
//    instructions, and 20 more registers held).
//  - Axis selects are bit selects, and the triangle test has no branch.
//  - A lane knows the stack level at which it entered its instance, so that
//    leaving it takes no marker on the stack and no second pop.
// Measured against the chain form with compares of axis numbers: a 1080p frame
// of the two-level scene at depth 4 2.53 -> 2.02 ms, a 256x256 frame 395 ->
// 241 us, 24 frames together 2.57 -> 1.95 ms, camera and AO rays over 10M
// triangles (12.4M rays) 7.45 -> 6.96 ms, 1,000 rays 149 -> 111 us.
//
// OPT: visibility masks, face culling and opacity masks are compiled in
// (launches whose rays carry options, or whose top levels carry instance
// flags or opacity masks); without it the traversal has none of their
// registers or tests.
template <int W, bool ANY, int MODE, bool OPT>
struct Tracer {
    const RgNode<W> *tlas_nodes;
    const RgInst *recs;
    Ray R;
    Hit h;
    float best;                 // closest: shrinks to the best hit (closed interval)
    float ox, oy, oz, ix, iy, iz;  // current frame: origin and reciprocal direction
    float t0, tlo, thi;         // slide of the frame's origin, interval in the frame
    uint64_t nodes;             // the frame's nodes
    uint64_t leaves;            // what its leaves index: instance records, or the bottom level's triangles
    uint32_t inst_id;
    Shear sh;
    Stack st;
    int isp;             // stack level at the instance's entry
    uint32_t cur;        // the next unit: an inner node, or a leaf (RG_LEAF_BIT)
    uint32_t rmask;      // this ray's visibility mask
    uint32_t call_cull;  // RG_RAY_CULL_* of the launch
    uint32_t cull;       // culling in the current instance: RG_RAY_CULL_* | kFlip
    const uint64_t *alpha;  // opacity masks of the current instance's triangles (null: opaque)
    uint32_t alpha_level;
    // wave-wide
    uint64_t m_has, m_blas;  // lanes holding a ray; lanes inside an instance

    __device__ inline bool found() const { return h.inst != RG_MISS; }

    __device__ inline void world_frame() {
        nodes = (uint64_t)tlas_nodes;
        leaves = (uint64_t)recs;
        ox = R.o[0]; oy = R.o[1]; oz = R.o[2];
        ix = safe_rcp(R.d[0]); iy = safe_rcp(R.d[1]); iz = safe_rcp(R.d[2]);
        t0 = 0.0f;
        tlo = R.tmin;
        thi = best;
    }

    // Returns false if the ray has nothing to do (empty interval).  The
    // caller puts the lane into m_has and takes it out of m_blas.
    __device__ inline bool begin(const Ray &ray) {
        R = ray;
        h.inst = h.prim = RG_MISS;
        h.n_nodes = h.n_tris = h.n_inst = 0;
        best = R.tmax;
        st.sp = 0;
        cur = 0;  // root inner node of the top level
        world_frame();
        return R.tmin <= R.tmax;
    }

    // Slab distances as one fused plane * inv - c each.  The constant
    // c of the lo planes and that of the hi planes sit on either side
    // of o * inv, kSlabShift |o| |inv| apart from it, on the side that
    // widens the slab whatever the sign of inv, so the rounding of
    // o * inv cannot narrow an interval; the far widening covers the
    // relative error as before.
    __device__ inline void slab_consts(float cl[3], float chh[3]) const {
        const float o_[3] = {ox, oy, oz}, i_[3] = {ix, iy, iz};
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const float c = o_[a] * i_[a], sh_ = kSlabShift * fabsf(o_[a]);
            cl[a] = fmaf(sh_, i_[a], c);
            chh[a] = fmaf(-sh_, i_[a], c);
        }
    }
    // Entry distance of a child box in the frame's interval, INFINITY if
    // the ray misses it or the slot is empty.
    __device__ inline float slab(const float lo[3], const float hi[3], const float cl[3], const float chh[3],
                                 uint32_t child) const {
        const float x0 = fmaf(lo[0], ix, -cl[0]), x1 = fmaf(hi[0], ix, -chh[0]);
        const float y0 = fmaf(lo[1], iy, -cl[1]), y1 = fmaf(hi[1], iy, -chh[1]);
        const float z0 = fmaf(lo[2], iz, -cl[2]), z1 = fmaf(hi[2], iz, -chh[2]);
        const float n_ = fmaxf(fmaxf(fminf(x0, x1), fminf(y0, y1)), fmaxf(fminf(z0, z1), tlo));
        float f_ = fminf(fminf(fmaxf(x0, x1), fmaxf(y0, y1)), fmaxf(z0, z1));
        f_ = fmaf(fabsf(f_), kFarWiden, f_);
        f_ = fminf(f_, thi);
        const bool hit = (n_ <= f_) & (child != RG_EMPTY);
        return hit ? n_ : INFINITY;
    }

    // An inner node: tests its children, continues with the nearest hit one
    // and pushes the others far first; cur = RG_EMPTY if none is hit.
    __device__ inline void inner(const uint32_t *w, bool shallow) {
        if (MODE == kCounts) ++h.n_nodes;
        float tn[W];
        uint32_t ch[W];
        float cl[3], chh[3];
        slab_consts(cl, chh);
#pragma unroll
        for (int k = 0; k < W; ++k) {
            const float lo[3] = {__uint_as_float(w[k]), __uint_as_float(w[W + k]), __uint_as_float(w[2 * W + k])};
            const float hi[3] = {__uint_as_float(w[3 * W + k]), __uint_as_float(w[4 * W + k]),
                                 __uint_as_float(w[5 * W + k])};
            ch[k] = w[6 * W + k];
            tn[k] = slab(lo, hi, cl, chh, ch[k]);
        }
        if (!ANY) sort_children<W>(tn, ch);
        if (shallow) cur = push<true>(tn, ch);
        else cur = push<false>(tn, ch);
    }

    // Pushes the hit children but the one to continue with, which it returns
    // (RG_EMPTY: none).
    template <bool LDS>
    __device__ inline uint32_t push(const float *tn, const uint32_t *ch) {
        if (ANY) {
            uint32_t next = RG_EMPTY;
#pragma unroll
            for (int k = 0; k < W; ++k) {
                const bool hk = tn[k] != INFINITY;
                if (k > 0) st.template push_if<LDS>(ch[k], hk & (next != RG_EMPTY));
                next = (hk & (next == RG_EMPTY)) ? ch[k] : next;
            }
            return next;
        }
#pragma unroll
        for (int k = W - 1; k >= 1; --k) st.template push_if<LDS>(ch[k], tn[k] != INFINITY);
        return tn[0] != INFINITY ? ch[0] : RG_EMPTY;
    }

    // A top-level leaf: one instance.  Record words: inv[9] 0..8, p[3]
    // 9..11, nodes 12..13, tris 14..15, hdr 16..17, mat 18, inst 19,
    // root box lo 20..22, hi 23..25, flags 26.
    // w(i) gives word i.
    template <class Words>
    __device__ inline void enter(Words w) {
        if (MODE == kCounts) ++h.n_inst;
        // object-space ray in double: o' = M^-1 (o - p), d' = M^-1 d
        const double q[3] = {(double)R.o[0] - (double)__uint_as_float(w(9)),
                             (double)R.o[1] - (double)__uint_as_float(w(10)),
                             (double)R.o[2] - (double)__uint_as_float(w(11))};
        const double e[3] = {(double)R.d[0], (double)R.d[1], (double)R.d[2]};
        double od[3], dd[3];
#pragma unroll
        for (int r = 0; r < 3; ++r) {
            const double ir0 = __uint_as_float(w(3 * r)), ir1 = __uint_as_float(w(3 * r + 1));
            const double ir2 = __uint_as_float(w(3 * r + 2));
            od[r] = fma(ir2, q[2], fma(ir0, q[0], ir1 * q[1]));
            dd[r] = fma(ir2, e[2], fma(ir0, e[0], ir1 * e[1]));
        }
        // slide the origin to where the ray enters the bottom level's
        // root box (not before tmin); the entry only needs to be near the
        // box, so float suffices
        float ten = -INFINITY, tex = INFINITY;
#pragma unroll
        for (int r = 0; r < 3; ++r) {
            const float of = (float)od[r], df = (float)dd[r], rr = safe_rcp(df);
            const float a = (__uint_as_float(w(20 + r)) - of) * rr, b = (__uint_as_float(w(23 + r)) - of) * rr;
            ten = fmaxf(ten, fminf(a, b));
            tex = fminf(tex, fmaxf(a, b));
        }
        float ts = ((ten <= tex) & (ten > R.tmin)) ? ten : R.tmin;
        ts = ts > R.tmax ? R.tmax : ts;
        float ld_[3];
        ox = (float)fma((double)ts, dd[0], od[0]);
        oy = (float)fma((double)ts, dd[1], od[1]);
        oz = (float)fma((double)ts, dd[2], od[2]);
#pragma unroll
        for (int r = 0; r < 3; ++r) ld_[r] = (float)dd[r];
        ix = safe_rcp(ld_[0]); iy = safe_rcp(ld_[1]); iz = safe_rcp(ld_[2]);
        const bool mirrored = make_shear(ld_, sh);
        t0 = ts;
        tlo = R.tmin - t0;
        tlo = fmaf(fabsf(tlo), -1.2e-7f, tlo);
        thi = best - t0;
        thi = fmaf(fabsf(thi), 2.4e-7f, thi);
        nodes = (uint64_t)w(12) | ((uint64_t)w(13) << 32);
        leaves = (uint64_t)w(14) | ((uint64_t)w(15) << 32);
        inst_id = (MODE == kRender) ? rg_leaf_first(cur) : w(19);
        if (OPT) {
            cull = (w(26) & RG_INST_CULL_DISABLE) ? 0u : call_cull;
            // the facing reads the sign of det in the published axis order,
            // which swaps x and y for a direction with d[kz] < 0
            if (cull) cull ^= (((w(26) & RG_INST_FLIP_FACING) != 0u) != mirrored) ? kFlip : 0u;
            alpha = nullptr;
            if (w(26) & RG_INST_ALPHA) {
                const RgBlasHdr *H = reinterpret_cast<const RgBlasHdr *>((uint64_t)w(16) | ((uint64_t)w(17) << 32));
                alpha = reinterpret_cast<const uint64_t *>(H->alpha);
                alpha_level = H->alpha_level;
            }
        }
        isp = st.sp;
        cur = 0;
    }

    // One triangle (ten words: vertices, input index) in leaf slot `slot`.
    // Returns whether it became the hit.
    __device__ inline bool triangle(const uint32_t *w, uint32_t slot) {
        if (MODE == kCounts) ++h.n_tris;
        const float o3[3] = {ox, oy, oz};
        float tv[9];
#pragma unroll
        for (int k = 0; k < 9; ++k) tv[k] = __uint_as_float(w[k]);
        float T, det, V, Wv;
        bool ok = tri_test(tv, o3, sh, tlo, thi, T, det, V, Wv);
        if (OPT) {
            // facing: det > 0 when the ray travels against the winding
            // normal (the sheared axes keep their handedness)
            const bool front = (det > 0.0f) != ((cull & kFlip) != 0u);
            ok = ok & ((cull & (front ? RG_RAY_CULL_FRONT : RG_RAY_CULL_BACK)) == 0u);
        }
        // t by the hardware reciprocal (1 ulp) and one product: up to
        // 1.5 ulp from T / det, inside the float32 band the parity
        // checks allow around t; the reported t is recomputed in double
        const float tw = fmaf(T, __builtin_amdgcn_rcpf(det), t0);
        ok = ok & (tw >= R.tmin) & (tw <= best);
        const uint32_t pid = (MODE == kRender) ? slot : w[9];
        // ties: lowest instance, then primitive
        if (!ANY)
            ok = ok & ((tw != best) | !found() |
                       !((inst_id > h.inst) | ((inst_id == h.inst) & (pid >= h.prim))));
        if (OPT && ok && alpha) ok = alpha_open(alpha[w[9]], alpha_level, V / det, Wv / det);
        if (ok) {
            h.inst = inst_id;
            h.prim = pid;
            if (!ANY) {
                best = tw;
                thi = best - t0;
                thi = fmaf(fabsf(thi), 2.4e-7f, thi);
            }
        }
        return ok;
    }

    // One round: inner nodes whenever a lane has one; leaves and instance
    // entries (each a long stretch of code that runs for the whole wave if
    // any lane needs it) once enough lanes wait for one, or when nothing
    // else is left.  A lane that waits keeps its state; every round runs at
    // least one kind present.  Every lane of the wave calls it; some lane
    // holds a ray.  Returns the lanes whose ray is finished (taken out of
    // m_has; h holds the result).
    //
    // Whatever the unit -- an inner node, an instance record or two
    // triangles of a leaf -- its bytes are requested before any of them
    // is used, into one register block by the same load instructions (only
    // the address differs), so that a wave whose lanes are at different
    // kinds of units waits for one memory round trip per round.  112 bytes
    // cover a record, two triangles (a leaf of one reads into the next
    // triangle or the arrays after the last: every structure keeps at
    // least 112 bytes of its own buffer after each array) and a node of
    // width 2 or 4; width 8 nodes load their second half separately.
    __device__ inline uint64_t round(int leaf_batch, int inst_batch) {
        constexpr int kNodeU4 = (7 * W + 3) / 4;  // node bytes without padding, in 16 B
        constexpr int kWords = 4 * kNodeU4 > 28 ? 4 * kNodeU4 : 28;
        const uint64_t m_inner = ballot(!rg_is_leaf(cur)) & m_has;
        const uint64_t at_leaf = m_has & ~m_inner & m_blas, at_inst = m_has & ~m_inner & ~m_blas;
        const uint64_t m_leaf = (__popcll(at_leaf) >= leaf_batch || m_inner == 0ull) ? at_leaf : 0ull;
        const uint64_t m_inst = (__popcll(at_inst) >= inst_batch || (m_inner | m_leaf) == 0ull) ? at_inst : 0ull;
        const uint64_t run = m_inner | m_leaf | m_inst;
        // no lane of the wave reaches past the LDS part of its stack this round
        const bool shallow = (ballot(st.sp + W - 1 > st.n_lds) & m_has) == 0ull;
        const uint32_t first = cur & 0x0FFFFFFFu;  // node, record or triangle
        uint32_t w[kWords];
        if (lane_in(run)) {
            const bool in = lane_in(m_inner);
            const uint32_t stride = in ? (uint32_t)sizeof(RgNode<W>)
                                       : (lane_in(m_leaf) ? (uint32_t)sizeof(RgTri) : (uint32_t)sizeof(RgInst));
            // (values made opaque: the compiler would rather select between
            // the two members' addresses, and keep both in scratch memory)
            uint64_t a_nodes = nodes, a_leaves = leaves;
            asm("" : "+v"(a_nodes), "+v"(a_leaves));
            const uint64_t addr = (in ? a_nodes : a_leaves) + (uint64_t)first * stride;
            const RG_GLOBAL rg_u4a8 *src = gptr<rg_u4a8>((const void *)addr);
#pragma unroll
            for (int k = 0; k < 7; ++k) {
                const rg_u4a8 v = src[k];
                w[4 * k] = v.x; w[4 * k + 1] = v.y; w[4 * k + 2] = v.z; w[4 * k + 3] = v.w;
            }
            if (kNodeU4 > 7 && in) {
#pragma unroll
                for (int k = 7; k < kNodeU4; ++k) {
                    const rg_u4a8 v = src[k];
                    w[4 * k] = v.x; w[4 * k + 1] = v.y; w[4 * k + 2] = v.z; w[4 * k + 3] = v.w;
                }
            }
        }
        if (lane_in(m_inner)) inner(w, shallow);
        uint64_t hidden = 0ull, stop = 0ull;
        if (m_inst) {
            if (OPT) hidden = ballot(((w[26] & 0xFFu) & rmask) == 0u) & m_inst;  // not visible: as if missed
            if (lane_in(m_inst & ~hidden)) enter([&](int i) { return w[i]; });
            if (OPT && lane_in(hidden)) cur = RG_EMPTY;
        }
        if (m_leaf) {
            if (lane_in(m_leaf)) {
                // two triangles of the leaf; what it holds beyond them is the lane's next unit
                const uint32_t more = (cur >> 28) & 7u;  // triangles after the first
                triangle(w, first);
                if (more > 0u && !(ANY && found())) triangle(w + 10, first + 1);
                cur = more > 1u ? cur - (2u << 28) + 2u : RG_EMPTY;
            }
            if (ANY) stop = ballot(found()) & m_leaf;
        }
        // lanes whose unit led nowhere take the next entry of their stack
        uint64_t pop = ballot(cur == RG_EMPTY) & run & ~stop;
        const uint64_t end = ballot(st.sp == 0) & pop;
        pop &= ~end;
        m_blas = (m_blas | m_inst) & ~hidden;
        const uint64_t leave = ballot(st.sp == isp) & pop & m_blas;
        if (lane_in(leave)) world_frame();
        m_blas &= ~leave;
        if (lane_in(pop)) {
            if (shallow) cur = st.template pop<true>();
            else cur = st.template pop<false>();
        }
        const uint64_t fin = end | stop;
        m_has &= ~fin;
        return fin;
    }
};

// Orders one wave's LDS accesses across lanes: a compiler fence at
// wavefront scope and a wave barrier (the LDS serves a wave's accesses in
// order).  The barrier alone orders no memory.
__device__ inline void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Value of the lane at `ctrl` (DPP: quad_perm, row_half_mirror); every lane
// read from is active.
template <int CTRL>
__device__ inline uint32_t dpp(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xF, 0xF, true);
}
constexpr int kQuad1 = 0xB1, kQuad2 = 0x4E, kQuad3 = 0x1B;  // quad_perm: lane ^ 1, ^ 2, ^ 3
constexpr int kHalfMirror = 0x141;                          // lane 7 - i of each eight

// The traversal for short launches: W lanes (a group) per ray, one child box
// or one triangle of a leaf per lane, 64 / W rays per wave.  A short launch
// lasts as long as its longest rays, and one ray's time is the latency of the
// instructions of its rounds: with a lane per ray a round of an inner node is
// about 260 vector and 90 scalar instructions (1 us; memory is the smaller
// part: requesting the children's lines early made it 10% slower).  Here the
// box test is one child's, the order of the children is each lane's rank
// among the W entry distances (DPP), and a leaf's triangles are tested side by
// side.  All lanes of a group hold the ray's state alike.  The same units are
// visited as in Tracer::round; children at equal distances go in slot order.
template <int W, bool ANY, int MODE, bool OPT, class Fetch, class Put>
__device__ inline void trace_groups(Tracer<W, ANY, MODE, OPT> &tr, uint32_t first_ray, uint32_t end_ray,
                                    uint32_t RG_LDS *stacks, Fetch fetch, Put put) {
    static_assert(W == 4 || W == 8, "group width");
    constexpr uint32_t G = 64 / W;
    const uint32_t lane = threadIdx.x & 63u, k = lane & (W - 1u), grp = lane / W;
    uint32_t RG_LDS *stk = stacks + grp * kStackCap;
    uint32_t next_ray = first_ray + grp, ray = 0u;
    uint64_t has = 0ull, blas = 0ull;
    uint32_t stalled = 0u;
    while (true) {
        const uint64_t take = ballot(next_ray < end_ray) & ~has;
        if (take) {
            bool live = false;
            if (lane_in(take)) {
                ray = next_ray;
                next_ray += G;
                live = fetch(ray);
                if (!live && k == 0u) put(ray);  // empty interval: a miss without traversal
            }
            has |= ballot(live);
            blas &= ~take;
            stalled = 0u;
        }
        if (has == 0ull) {
            if (ballot(next_ray < end_ray) == 0ull) return;
            continue;
        }
        const uint64_t m_inner = ballot(!rg_is_leaf(tr.cur)) & has;
        const uint64_t m_leaf = has & ~m_inner & blas, m_inst = has & ~m_inner & ~blas;
        const uint32_t first = tr.cur & 0x0FFFFFFFu, count = ((tr.cur >> 28) & 7u) + 1u;
        // every kind's bytes are requested before any is used
        uint32_t w[10];
        const uint64_t m_tri = ballot(k < count) & m_leaf;
        if (lane_in(m_inner)) {
            const RG_GLOBAL uint32_t *src =
                gptr<uint32_t>((const void *)(tr.nodes + (uint64_t)first * sizeof(RgNode<W>) + 4u * k));
#pragma unroll
            for (int r = 0; r < 7; ++r) w[r] = src[r * W];
        }
        if (m_tri && lane_in(m_tri)) {
            const RG_GLOBAL rg_u2 *src =
                gptr<rg_u2>((const void *)(tr.leaves + (uint64_t)(first + k) * sizeof(RgTri)));
#pragma unroll
            for (int r = 0; r < 5; ++r) {
                const rg_u2 v = src[r];
                w[2 * r] = v.x;
                w[2 * r + 1] = v.y;
            }
        }
        if (m_inst && lane_in(m_inst)) {  // a quarter of the record per lane of a quad
            const RG_GLOBAL uint32_t *src =
                gptr<uint32_t>((const void *)(tr.leaves + (uint64_t)first * sizeof(RgInst) + 28u * (k & 3u)));
#pragma unroll
            for (int r = 0; r < 7; ++r) w[r] = src[r];
        }
        if (lane_in(m_inner)) {
            const float lo[3] = {__uint_as_float(w[0]), __uint_as_float(w[1]), __uint_as_float(w[2])};
            const float hi[3] = {__uint_as_float(w[3]), __uint_as_float(w[4]), __uint_as_float(w[5])};
            float cl[3], chh[3];
            tr.slab_consts(cl, chh);
            const float tn = tr.slab(lo, hi, cl, chh, w[6]);
            const bool hit = tn != INFINITY;
            const uint32_t hits = (uint32_t)(ballot(hit) >> (lane & ~(W - 1u))) & ((1u << W) - 1u);
            const int nh = __popc(hits);
            // rank: lanes that come before this one (nearer, or as near and
            // in a lower slot); any hit goes in slot order
            uint32_t rank = (uint32_t)__popc(hits & ((1u << k) - 1u));
            if (!ANY) {
                rank = 0u;
                auto before = [&](uint32_t bits, uint32_t other) {
                    const float t = __uint_as_float(bits);
                    rank += ((t < tn) | ((t == tn) & (other < k))) ? 1u : 0u;
                };
                const uint32_t b = __float_as_uint(tn);
                before(dpp<kQuad1>(b), k ^ 1u);
                before(dpp<kQuad2>(b), k ^ 2u);
                before(dpp<kQuad3>(b), k ^ 3u);
                if constexpr (W == 8) {
                    const uint32_t m = dpp<kHalfMirror>(b);
                    before(m, k ^ 7u);
                    before(dpp<kQuad1>(m), k ^ 6u);
                    before(dpp<kQuad2>(m), k ^ 5u);
                    before(dpp<kQuad3>(m), k ^ 4u);
                }
            }
            // nearest first: it is the next unit, the others lie on the stack
            // farthest first (any hit: first slot next, the others in order)
            if (hit & (rank != 0u)) stk[tr.st.sp + (ANY ? (int)rank - 1 : nh - 1 - (int)rank)] = w[6];
            uint32_t nx = (hit & (rank == 0u)) ? w[6] : 0u;  // no child is node 0
            nx |= dpp<kQuad1>(nx);
            nx |= dpp<kQuad2>(nx);
            if constexpr (W == 8) nx |= dpp<kHalfMirror>(nx);
            tr.cur = nh ? nx : RG_EMPTY;
            tr.st.sp += nh ? nh - 1 : 0;
        }
        uint64_t hidden = 0ull, stop = 0ull;
        if (m_inst) {
            // flags: word 26, the fourth lane's sixth (a mask is only ever set
            // by all lanes together: under a lane's branch it would differ
            // from lane to lane)
            if (OPT) hidden = ballot(((dpp<0xFF>(w[5]) & 0xFFu) & tr.rmask) == 0u) & m_inst;
            if (lane_in(m_inst & ~hidden)) {
                tr.enter([&](int i) {
                    const uint32_t v = w[i % 7];
                    return i < 7 ? dpp<0x00>(v) : (i < 14 ? dpp<0x55>(v) : (i < 21 ? dpp<0xAA>(v) : dpp<0xFF>(v)));
                });
            }
            if (OPT && lane_in(hidden)) tr.cur = RG_EMPTY;
        }
        if (m_leaf) {
            bool ok = false;
            if (lane_in(m_tri)) ok = tr.triangle(w, first + k);
            const uint64_t got = ballot(ok);
            if (ANY) {
                // the first of the group's hits
                stop = ballot(((uint32_t)(got >> (lane & ~(W - 1u))) & ((1u << W) - 1u)) != 0u) & m_leaf;
                if (lane_in(stop)) {
                    const uint32_t bits = (uint32_t)(got >> (lane & ~(W - 1u))) & ((1u << W) - 1u);
                    const int from = (int)(lane & ~(W - 1u)) + __ffs((int)bits) - 1;
                    tr.h.inst = tr.inst_id;
                    tr.h.prim = (uint32_t)__shfl((int)tr.h.prim, from);
                }
            } else if (got) {
                // least (t, instance, primitive) over the group
                if (lane_in(m_leaf)) {
                    auto least = [&](uint32_t ob, uint32_t oi, uint32_t op) {
                        const float t = __uint_as_float(ob);
                        const bool lt = (t < tr.best) |
                                        ((t == tr.best) & ((oi < tr.h.inst) | ((oi == tr.h.inst) & (op < tr.h.prim))));
                        tr.best = lt ? t : tr.best;
                        tr.h.inst = lt ? oi : tr.h.inst;
                        tr.h.prim = lt ? op : tr.h.prim;
                    };
                    least(dpp<kQuad1>(__float_as_uint(tr.best)), dpp<kQuad1>(tr.h.inst), dpp<kQuad1>(tr.h.prim));
                    least(dpp<kQuad2>(__float_as_uint(tr.best)), dpp<kQuad2>(tr.h.inst), dpp<kQuad2>(tr.h.prim));
                    if constexpr (W == 8)
                        least(dpp<kHalfMirror>(__float_as_uint(tr.best)), dpp<kHalfMirror>(tr.h.inst),
                              dpp<kHalfMirror>(tr.h.prim));
                    tr.thi = tr.best - tr.t0;
                    tr.thi = fmaf(fabsf(tr.thi), 2.4e-7f, tr.thi);
                }
            }
            if (lane_in(m_leaf)) tr.cur = count > (uint32_t)W ? tr.cur - ((uint32_t)W << 28) + (uint32_t)W : RG_EMPTY;
        }
        wave_sync();  // the group's pushes come before its pops
        uint64_t pop = ballot(tr.cur == RG_EMPTY) & has & ~stop;
        const uint64_t end = ballot(tr.st.sp == 0) & pop;
        pop &= ~end;
        blas = (blas | m_inst) & ~hidden;
        const uint64_t leave = ballot(tr.st.sp == tr.isp) & pop & blas;
        if (lane_in(leave)) {
            tr.world_frame();
        }
        blas &= ~leave;
        if (lane_in(pop)) tr.cur = stk[--tr.st.sp];
        wave_sync();  // and its pops before the next round's pushes
        uint64_t fin = end | stop;
        // loop bound: see Tracer's callers
        stalled = fin ? 0u : stalled + 1u;
        if (stalled > kMaxSteps) fin = has;
        has &= ~fin;
        if (fin) {
            if (lane_in(fin) && k == 0u) put(ray);
        }
    }
}

}  // namespace rgt

// A top level as the kernels need it.
struct RgTlasRef {
    const void *nodes;
    const RgInst *recs;
};

// Arguments of the trace kernels (passed by value).
struct RgTraceArgs {
    const void *nodes;             // top-level nodes
    const RgInst *recs;            // top-level instance records
    const uint32_t *ray_job;       // per ray: index into jobs (nullable: all rays use nodes/recs)
    uint32_t ray_flags = 0u;       // RG_RAY_CULL_*
    uint32_t mask = RG_INST_MASK_ALL;  // visibility mask of every ray, unless ray_mask
    const uint8_t *ray_mask = nullptr;  // per ray (nullable)
    bool opt = false;              // masks / culling in effect (ray options or instance flags)
    bool lanes = false;            // a lane per ray whatever the number of rays
    const RgTlasRef *jobs;
    const float *ray[8];           // ox oy oz dx dy dz tmin tmax
    int64_t n;                     // number of rays (upper bound if `count` is set)
    const uint32_t *count;         // device count of rays (nullable)
    float *t, *u, *v;              // outputs (nullable)
    uint32_t *inst, *prim;
    uint8_t *occluded;             // any hit
    uint32_t *counts;              // visit counts [n][3]
    uint32_t *work;                // the launch's packet counters, two words (set by rg_trace_launch)
};

// Launches the traversal over a.n rays (or *a.count if set) on `stream`.
// width: 2/4/8; any: any-hit; mode: rgt::Mode.
// scope: the RG_TUNE_* family whose launch parameters apply.
rg_status rg_trace_launch(int width, bool any, int mode, const RgTraceArgs &a, hipStream_t stream, int scope);
// Compute units of the current device (queried once).
int rg_cu_count();
// Largest (W-1)*(top depth + bottom depth) + 1 the traversal stack holds.
bool rg_trace_depth_ok(const rg_tlas *t);
