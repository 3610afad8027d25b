// Immersed-boundary and structure kernels (Secs. 1.2-1.3).
//
// One MLS point (triangle centroid, probe or vertex) is evaluated by a group of 8 lanes (half a
// DPP row), which share the 3x3x3 nodes around the node nearest to the point.  The 4x4 moment matrix
// is accumulated and factorised in FP64 (every lane of the group solves redundantly), so no lane
// waits on another except for the butterfly sums.  The marker kernels run one-wave blocks of eight
// points: few lanes per point keep the instructions per point low, which bounds the batched launches,
// and a lone body's launches are chains of instructions and dependent reads, so they too follow the
// instruction count (below: nodes outside the support dropped first, one window test per wave).
//
// Step order inside the time step n -> n+1:
//   k_centroids  triangle blocks: force window of this step from the vertex bounding box,
//                geometry at x^n (kept for the probes), MLS at centroids on moments of f^n,
//                F_l = U_b - U*, fixed-point spreading into the body's force window, partial
//                enclosed volumes; edge blocks: spring and bending forces of every hinge
//   (sweep)      collide+stream with the spread force
//   (moments)    moments of f^{n+1} in the body's window; a block per body for the volume V^n of
//                membranes with k_v != 0 from the partials
//   k_triangles  one group per probe (geometry from the centroid kernel): stresses on f^{n+1}
//                (Eqs. hydroForP, hydroForNu), volume force per triangle; rigid bodies: FP64
//                partial force and torque per block.  Blocks of their own: the fluid velocity
//                at every membrane vertex from f^{n+1}
//   k_fold_bodies (rigid bodies) FP64 totals and the velocity / pose update
//   k_vertices   gathered forces, membrane update with that velocity, integer bounding boxes
//                of x^{n+1} for the next step's window
#include "lbib_reduce.h"

namespace lbib {

// The same for K values, level by level: a DPP move reads its operand two cycles after it was
// written at the earliest, and the other values' additions fill that time.
template <int K>
__device__ __forceinline__ void gsum8(double v[K]) {
#pragma unroll
    for (int i = 0; i < K; ++i) v[i] += dpp_f64<0xB1>(v[i]);
#pragma unroll
    for (int i = 0; i < K; ++i) v[i] += dpp_f64<0x4E>(v[i]);
#pragma unroll
    for (int i = 0; i < K; ++i) v[i] += dpp_f64<0x141>(v[i]);
}

// Minimum / maximum over the wave: DPP within rows (quad permutes, half-mirror, mirror), then the
// four rows from scalar registers, where the result stays: what is derived from it (the spreading
// box, the force window) is then scalar work too.
template <int CTRL>
__device__ __forceinline__ int dpp_i32(int v) {
    return __builtin_amdgcn_mov_dpp(v, CTRL, 0xF, 0xF, true);
}
template <bool MAX>
__device__ __forceinline__ int wave_minmax(int v) {
    auto op = [](int a, int b) { return MAX ? max(a, b) : min(a, b); };
    v = op(v, dpp_i32<0xB1>(v));
    v = op(v, dpp_i32<0x4E>(v));
    v = op(v, dpp_i32<0x141>(v));
    v = op(v, dpp_i32<0x140>(v));
    return op(op(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)),
              op(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
}


// Nodes of an MLS point.  Every node within r_w < 1.5 of x lies in the 3x3x3 block around the node c
// nearest to x; lane l of the point's 8 owns nodes l, l + 8, l + 16 and l + 24 of the block, its
// class.  About 9 of the 27 are within r_w, so the lane drops the others before it does any work on
// them: a class never holds more than three within r_w < sqrt(2), and rarely more than two.  Per axis
// call c near, the neighbour on x's side second and the other one far, at distances f, 1 - f and
// 1 + f (f <= 1/2).  Of two nodes that are second and far on one axis and far and second on another
// only one can be within r_w, since their squared distances add up to 4 or more, and none is far on
// two axes; that leaves at most two nodes of the classes 0, 1, 2 and 5, and the other classes have
// three nodes.  Slots are filled in the class's order, so the sums over them are those over the whole
// class bit for bit (the dropped nodes have weight zero).  The third slot is skipped in waves that
// do not need it.  WIDE (r_w^2 >= MLS_COMPACT_RW2, with a margin for the FP32 test) keeps all four.
template <bool WIDE>
struct MlsLane {
    static constexpr int N = WIDE ? 4 : 3;   // slots per lane
    int c[3];                    // node nearest to the point (unwrapped)
    int o[N][3];                 // slot's node relative to c
    bool active[N];              // within r_w of the point
    double d0[N], d1[N], d2[N], r2[N];
    double phi[N];
    double gr[N][3];
    bool more;                   // some lane of the wave uses the slots from the third on
};
#define MLS_SLOTS(s, m)                                                     \
    _Pragma("unroll") for (int s = 0; s < MlsLane<WIDE>::N; ++s)            \
        if (s < 2 || (m).more)

template <bool WIDE>
__device__ __forceinline__ void mls_locate(const double xp[3], double rw2, int lane, MlsLane<WIDE>& m) {
    // the point's coordinates are taken as rounded, not fused with the product that formed them
#pragma clang fp contract(off)
    double dn[3];
    float f[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const double n = floor(xp[a] + 0.5);
        m.c[a] = (int)n;
        dn[a] = n - xp[a];   // exact, and so is the offset added to it below
        f[a] = (float)dn[a];
    }
    // the class's nodes within r_w, by their FP32 distance with a margin; FP64 decides below
    unsigned set = WIDE ? 15u : 0u;
    if (!WIDE) {
        const float r2max = (float)rw2 + 1e-4f;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int k = lane + 8 * s, q3 = (k * 171) >> 9, q9 = (k * 57) >> 9;
            const float x = f[0] + (float)(k - 3 * q3 - 1), y = f[1] + (float)(q3 - 3 * q9 - 1), z = f[2] + (float)(q9 - 1);
            set |= (fmaf(z, z, fmaf(y, y, x * x)) <= r2max && k < 27 ? 1u : 0u) << s;
        }
    }
    m.more = WIDE || __any((set & (set - 1u) & ((set & (set - 1u)) - 1u)) != 0u);
    MLS_SLOTS(s, m) {
        const int pick = WIDE ? s : __ffs(set) - 1;   // -1: none left
        const bool some = WIDE ? lane + 8 * s < 27 : set != 0u;
        set &= set - 1u;
        const int k = some ? lane + 8 * pick : 13, q3 = (k * 171) >> 9, q9 = (k * 57) >> 9;
        m.o[s][0] = k - 3 * q3 - 1;
        m.o[s][1] = q3 - 3 * q9 - 1;
        m.o[s][2] = q9 - 1;
        m.d0[s] = dn[0] + (double)m.o[s][0];
        m.d1[s] = dn[1] + (double)m.o[s][1];
        m.d2[s] = dn[2] + (double)m.o[s][2];
        m.r2[s] = fma(m.d2[s], m.d2[s], fma(m.d0[s], m.d0[s], m.d1[s] * m.d1[s]));
        m.active[s] = some && m.r2[s] <= rw2;
    }
}

// 1/x in FP64: hardware reciprocal refined by two Newton steps (x > 0, normal).
__device__ __forceinline__ double rcp64(double x) {
    double r = __builtin_amdgcn_rcp(x);
    r = fma(r, fma(-x, r, 1.0), r);
    r = fma(r, fma(-x, r, 1.0), r);
    return r;
}

// Shape functions phi_k = [A^{-1} W_k p_k]_0 and (optionally) their gradients, A = sum W p p^T,
// p = (1, d), W = exp(-(|d| / (r_w alpha))^2) (Eqs. l2norm, intKernel).  The weights are
// evaluated in FP32; the moment matrix is accumulated and factorised (A = L D L^T, unit L) in
// FP64 on every lane.
template <bool WIDE>
__device__ __forceinline__ void mls_solve(MlsLane<WIDE>& m, float wq, bool want_grad, int& err) {
    double W[MlsLane<WIDE>::N];
    double A[10] = {};   // 00 01 02 03 11 12 13 22 23 33
    MLS_SLOTS(s, m) {
        W[s] = m.active[s] ? (double)expf(-wq * (float)m.r2[s]) : 0.0;
        const double w = W[s], d0 = m.d0[s], d1 = m.d1[s], d2 = m.d2[s];
        A[0] += w; A[1] += w * d0; A[2] += w * d1; A[3] += w * d2;
        A[4] += w * d0 * d0; A[5] += w * d0 * d1; A[6] += w * d0 * d2;
        A[7] += w * d1 * d1; A[8] += w * d1 * d2; A[9] += w * d2 * d2;
    }
    gsum8<10>(A);
    const double a00 = A[0], a01 = A[1], a02 = A[2], a03 = A[3], a11 = A[4], a12 = A[5], a13 = A[6], a22 = A[7],
                 a23 = A[8], a33 = A[9];
    // A = L D L^T
    const double e0 = a00;
    const double i0 = rcp64(e0);
    const double l10 = a01 * i0, l20 = a02 * i0, l30 = a03 * i0;
    const double e1 = a11 - l10 * a01;
    const double i1 = rcp64(e1);
    const double b21 = a12 - l20 * a01, b31 = a13 - l30 * a01;   // D-scaled column entries
    const double l21 = b21 * i1, l31 = b31 * i1;
    const double e2 = a22 - l20 * a02 - l21 * b21;
    const double i2 = rcp64(e2);
    const double b32 = a23 - l30 * a02 - l31 * b21;
    const double l32 = b32 * i2;
    const double e3 = a33 - l30 * a03 - l31 * b31 - l32 * b32;
    const double i3 = rcp64(e3);
    if (!(e0 > 0.0 && e1 > 0.0 && e2 > 0.0 && e3 > 0.0)) err |= FLAG_NONFINITE;
    MLS_SLOTS(s, m) {
        // v = A^{-1} p_k: L y = p, z = D^{-1} y, L^T v = z.  The first column of L, a0j / e0, enters
        // the differences as the unrounded product; every fusion is written out, so that a body alone
        // and in a batch (two instantiations) rounds alike
        const double y1 = fma(-i0, a01, m.d0[s]);
        const double y2 = fma(-l21, y1, fma(-i0, a02, m.d1[s]));
        const double y3 = fma(-l32, y2, fma(-l31, y1, fma(-i0, a03, m.d2[s])));
        const double v3 = y3 * i3;
        const double v2 = fma(y2, i2, -(l32 * v3));
        const double v1 = fma(-l31, v3, fma(y1, i1, -(l21 * v2)));
        const double v0 = fma(-l30, v3, fma(-l20, v2, fma(-l10, v1, i0)));
        m.phi[s] = W[s] * v0;
        if (want_grad) { m.gr[s][0] = W[s] * v1; m.gr[s][1] = W[s] * v2; m.gr[s][2] = W[s] * v3; }
    }
}

// The lane's part of sum_k c_k q_k over the point for per-node coefficients c (phi or a gradient row)
// and field values q (component `comp` of the moments: 0 rho - 1, 1..3 u*)
template <bool WIDE>
__device__ __forceinline__ double point_dot(const MlsLane<WIDE>& m, const double* c, int cstride,
                                            const float4 mom[MlsLane<WIDE>::N], int comp) {
    double acc = 0.0;
    MLS_SLOTS(s, m) {
        const float q = comp == 0 ? mom[s].x : (comp == 1 ? mom[s].y : (comp == 2 ? mom[s].z : mom[s].w));
        acc += c[s * cstride] * (double)q;
    }
    return acc;
}

// Index of every slot's node in a window of layout d (see WinDesc).  Points whose 3x3x3 block lies
// inside the window and the fluid, every point of an ordinary step, take the first form (one vote
// per wave): no wrap, no test per node, and the inactive slots hold valid indices too, so the
// caller loads all of them without a branch.  The second form wraps periodic axes, reports support
// nodes beyond a wall or the window, and gives their slots index 0.  They stay in the point's moment
// system, which would be singular without them and end the job as unstable, not as out of its domain;
// DROP takes them out afterwards, for the spreading.
template <bool WIDE, bool DROP = false>
__device__ __forceinline__ void mls_index(const JobDev& J, const WinDesc& d, MlsLane<WIDE>& m,
                                          unsigned idx[MlsLane<WIDE>::N], int& err) {
    const int n[3] = {J.nx, J.ny, J.nz};
    const int s1 = d.w[0], s2 = d.w[0] * d.w[1];
    bool in = s2 < (1 << 23);   // 24-bit products below
    int lo[3], hi[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const int bc = J.bc[2 * a];
        lo[a] = bc == 0 ? -0x40000000 : (bc == 1 ? 1 : 0);
        hi[a] = bc == 0 ? 0x40000000 : (bc == 1 ? n[a] - 2 : n[a] - 1);
        in = in && m.c[a] > max(lo[a], d.b[a]) && m.c[a] < min(hi[a], d.b[a] + d.w[a] - 1);
    }
    if (__all(in)) {
        const int base = (m.c[0] - d.b[0]) + s1 * (m.c[1] - d.b[1]) + s2 * (m.c[2] - d.b[2]);
        MLS_SLOTS(s, m)
            idx[s] = (unsigned)(base + m.o[s][0] + __mul24(m.o[s][1], s1) + __mul24(m.o[s][2], s2));
        return;
    }
    MLS_SLOTS(s, m) {
        unsigned i = 0, st = 1;
        bool ok = true;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            int u = m.c[a] + m.o[s][a];
            if (J.bc[2 * a] != 0 && (u < lo[a] || u > hi[a])) {
                if (m.active[s]) err |= FLAG_DOMAIN;
                u = u < lo[a] ? lo[a] : hi[a];
            }
            int t = u - d.b[a];
            if (J.bc[2 * a] == 0 && (t < 0 || t >= d.w[a])) {
                t %= n[a];
                if (t < 0) t += n[a];
            }
            ok = ok && t >= 0 && t < d.w[a];
            i += (unsigned)t * st;
            st *= (unsigned)d.w[a];
        }
        if (!ok && m.active[s]) err |= FLAG_WINDOW;
        if (DROP && !ok) m.active[s] = false;
        idx[s] = ok ? i : 0u;
    }
}

__device__ __forceinline__ void load3(const double* p, double v[3]) { v[0] = p[0]; v[1] = p[1]; v[2] = p[2]; }
__device__ __forceinline__ void cross3(const double a[3], const double b[3], double c[3]) {
    c[0] = a[1] * b[2] - a[2] * b[1];
    c[1] = a[2] * b[0] - a[0] * b[2];
    c[2] = a[0] * b[1] - a[1] * b[0];
}
__device__ __forceinline__ double dot3(const double a[3], const double b[3]) {
    return a[0] * b[0] + a[1] * b[1] + a[2] * b[2];
}

// ---------------------------------------------------------------- hinge forces
// Spring (Eq. strainFor) on the edge x1-x2 and bending -k_b sin(theta - theta0) dtheta/dx_r on
// the four hinge vertices, theta the signed angle between the outward normals of (x1,x2,x3)
// and (x2,x1,x4) about x1->x2.  out[0..2] = spring force on x1 (x2 gets the opposite),
// out[3+3r..] = bending force on vertex r.
__device__ void hinge_forces(const Pools& P, const BodyDev& B, int e, double out[15]) {
    const int* hv = P.hinge + 4 * (B.e0 + e);
    double x1[3], x2[3], x3[3], x4[3];
    load3(P.x + 3 * (B.v0 + hv[0]), x1);
    load3(P.x + 3 * (B.v0 + hv[1]), x2);
    load3(P.x + 3 * (B.v0 + hv[2]), x3);
    load3(P.x + 3 * (B.v0 + hv[3]), x4);
    double e12[3], p3[3], p4[3], q[3];
    for (int a = 0; a < 3; ++a) { e12[a] = x2[a] - x1[a]; p3[a] = x3[a] - x1[a]; p4[a] = x4[a] - x2[a]; q[a] = -e12[a]; }
    const double le2 = dot3(e12, e12), le = sqrt(le2);
    const double sp = -P.ks[B.e0 + e] * (le - P.l0[B.e0 + e]) / le;
    for (int a = 0; a < 3; ++a) out[a] = -sp * e12[a];   // r_12 = x1 - x2 = -e12
    if (B.kb == 0.0) {
        for (int i = 3; i < 15; ++i) out[i] = 0.0;
        return;
    }
    double N1[3], N2[3], c12[3];
    cross3(e12, p3, N1);
    cross3(q, p4, N2);
    const double a1 = sqrt(dot3(N1, N1)), a2 = sqrt(dot3(N2, N2));
    const double n1[3] = {N1[0] / a1, N1[1] / a1, N1[2] / a1};
    const double n2[3] = {N2[0] / a2, N2[1] / a2, N2[2] / a2};
    cross3(n1, n2, c12);
    const double theta = atan2(dot3(c12, e12) / le, dot3(n1, n2));
    // opposite vertices rotate their triangle about the edge with lever arm = height over it;
    // the edge vertices carry the reaction split at each opposite vertex's foot point
    const double h3 = a1 / le, h4 = a2 / le;
    const double d4[3] = {x4[0] - x1[0], x4[1] - x1[1], x4[2] - x1[2]};
    const double t3 = dot3(p3, e12) / le2, t4 = dot3(d4, e12) / le2;
    const double sb = -B.kb * sin(theta - P.theta0[B.e0 + e]);
    for (int a = 0; a < 3; ++a) {
        const double g3 = -n1[a] / h3, g4 = -n2[a] / h4;
        out[3 + a] = sb * ((t3 - 1.0) * g3 + (t4 - 1.0) * g4);
        out[6 + a] = sb * (-t3 * g3 - t4 * g4);
        out[9 + a] = sb * g3;
        out[12 + a] = sb * g4;
    }
}

// ---------------------------------------------------------------- fixed point
// Round to nearest even into int64, as __double2ll_rn, without its software sequence: for
// |v| < 2^51, v + 1.5 * 2^52 lies in [2^52, 2^53), where the addition itself rounds v to an
// integer in the low mantissa bits.  The addition must not be fused with the product that
// formed v.  Larger values (small false) are left to the caller, one vote for all of a wave's.
__device__ __forceinline__ long long fix_rn(double v, bool& small) {
#pragma clang fp contract(off)
    small = small && fabs(v) < 2251799813685248.0;
    const double t = v + 6755399441055744.0;
    return __double_as_longlong(t) - 0x4338000000000000LL;
}

// ---------------------------------------------------------------- spreading
// The markers of a block are neighbours on the mesh, so their stencils overlap: about 9 active
// nodes per marker, but far fewer distinct nodes per marker over the block.  The
// block therefore sums its contributions in LDS first (int64, so the order cannot change the
// sum) and sends one global atomic per distinct node and component.  The LDS box is the
// bounding box of the block's 3x3x3 stencils in unwrapped node coordinates, laid out with fixed
// strides of 8 and 64, so its cells are addressed by shifts and a lane keeps its x and y through the
// planes; a block whose box exceeds 8 x 8 x SPREAD_LDS_Z (markers far apart on the lattice) adds
// straight to global memory.
//
// The same block-wide reduction also folds the integer boxes that the vertex blocks wrote for x^n
// into this step's force window (min / max, order independent): every block derives the same
// descriptor and block 0 publishes it for the sweep and the moments.  vb[6] is the box of the
// vertex-block boxes this thread loaded.  Folding once per body in a kernel of its own saved the
// 64-job batch's 30,000 blocks as much as its launch cost (644 us per step either way), and cost
// smaller launches the launch: 12 jobs 86.3 -> 83.2 us, four capsules in one lattice 42.8 -> 41.1.
constexpr int SPREAD_LDS_Z = 6;
// vertex-block boxes a lone body's centroid blocks load ahead (a level-4 icosphere has 161)
template <bool SOLO> constexpr int vbox_early() { return SOLO ? 3 * IB_BLOCK : IB_BLOCK; }

template <bool WIDE>
__device__ __forceinline__ void spread_block(const Pools& P, const JobDev& J, const BodyDev& B, int b,
                                             int blk, const int vb[6], bool live, MlsLane<WIDE>& m,
                                             const long long fx[MlsLane<WIDE>::N][3], int& err) {
    constexpr int N = MlsLane<WIDE>::N;
    static_assert(IB_BLOCK == 64, "the block is one wave: its boxes are wave reductions");
    __shared__ unsigned long long s_acc[3][64 * SPREAD_LDS_Z];
    const long long capn = (long long)B.win_cap[0] * B.win_cap[1] * B.win_cap[2];
    unsigned long long* fw0 = (unsigned long long*)(P.fwin + 3 * B.win_off);
    // stencil box of the block's markers, and the box of the vertex-block boxes
    int o[3], w[3], bmin[3], bmax[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        o[a] = wave_minmax<false>(m.c[a]) - 1;
        w[a] = wave_minmax<true>(m.c[a]) + 2 - o[a];
        bmin[a] = wave_minmax<false>(vb[a]);
        bmax[a] = wave_minmax<true>(vb[3 + a]);
    }
    const WinDesc fd = window_from_box(J, B.win_cap, bmin, bmax, err);
    if (blk == 0 && threadIdx.x == 0) P.fdesc[b] = fd;
    const bool use_lds = w[0] <= 8 && w[1] <= 8 && w[2] <= SPREAD_LDS_Z;   // uniform over the block
    unsigned idx[N];
    if (!use_lds) {
        mls_index<WIDE, true>(J, fd, m, idx, err);
        MLS_SLOTS(s, m)
            if (live && m.active[s])
                for (int c = 0; c < 3; ++c)
                    if (fx[s][c]) atomicAdd(fw0 + c * capn + idx[s], (unsigned long long)fx[s][c]);
        return;
    }
    const int t = threadIdx.x;
    // the lane's column of the box in the window, for the flush.  Only nodes that hold a sum are
    // mapped to the window and added; a support node beyond a wall has raised the domain error and
    // is dropped.
    const int n[3] = {J.nx, J.ny, J.nz};
    const int ux = o[0] + (t & 7), uy = o[1] + (t >> 3);
    bool in = true;
    int l[3] = {ux, uy, 0};
    for (int a = 0; a < 2; ++a) {
        const int u = l[a];
        l[a] = u - fd.b[a];
        if (J.bc[2 * a] == 0) {
            if (l[a] < 0 || l[a] >= fd.w[a]) { l[a] %= n[a]; if (l[a] < 0) l[a] += n[a]; }
        }
        in = in && l[a] >= 0 && l[a] < fd.w[a];
    }
    const unsigned s2 = (unsigned)fd.w[0] * (unsigned)fd.w[1];
    const unsigned col = (unsigned)l[0] + (unsigned)fd.w[0] * (unsigned)l[1];
    for (int z = 0; z < w[2]; ++z)
        for (int c = 0; c < 3; ++c) s_acc[c][64 * z + t] = 0;
    __syncthreads();
    if (live) {
        const int base = (m.c[0] - o[0]) + 8 * (m.c[1] - o[1]) + 64 * (m.c[2] - o[2]);
        MLS_SLOTS(s, m) {
            const int li = base + m.o[s][0] + 8 * m.o[s][1] + 64 * m.o[s][2];
            if (m.active[s])
                for (int c = 0; c < 3; ++c) atomicAdd(&s_acc[c][li], (unsigned long long)fx[s][c]);
        }
    }
    __syncthreads();
    for (int z = 0; z < w[2]; ++z) {
        const unsigned long long v0 = s_acc[0][64 * z + t], v1 = s_acc[1][64 * z + t], v2 = s_acc[2][64 * z + t];
        int lz = o[2] + z - fd.b[2];   // uniform
        if (J.bc[4] == 0 && (lz < 0 || lz >= fd.w[2])) { lz %= n[2]; if (lz < 0) lz += n[2]; }
        if (!(v0 | v1 | v2)) continue;
        if (!in || lz < 0 || lz >= fd.w[2]) {
            err |= FLAG_WINDOW;
            continue;
        }
        unsigned long long* f = fw0 + col + (unsigned long long)s2 * (unsigned)lz;
        if (v0) atomicAdd(f, v0);
        if (v1) atomicAdd(f + capn, v1);
        if (v2) atomicAdd(f + 2 * capn, v2);
    }
}

// ---------------------------------------------------------------- centroids (+ hinges)
template <bool SOLO, bool WIDE>
__global__ void __launch_bounds__(IB_BLOCK, SOLO ? 1 : 4) k_centroids(Pools P, int nblk_tri) {
    constexpr int N = MlsLane<WIDE>::N, PTS = IB_BLOCK / MLS_GROUP, VBOX_EARLY = vbox_early<SOLO>();
    if ((int)blockIdx.x >= nblk_tri) {
        // edge blocks: one thread per hinge of a membrane
        const int eb = blockIdx.x - nblk_tri;
        const int b = block_body<SOLO>(P, P.blk_body_e, eb);
        const BodyDev& B = body_of<SOLO>(P, b);
        const int e = (eb - B.blk_e0) * IB_BLOCK + threadIdx.x;
        if (e >= B.ne) return;
        double f[15];
        hinge_forces(P, B, e, f);
        double* o = P.fedge + 15LL * (B.e0 + e);
        for (int i = 0; i < 15; ++i) o[i] = f[i];
        return;
    }
    const int b = block_body<SOLO>(P, P.blk_body_c, blockIdx.x);
    // Body and job records are copied before the first store: one round of scalar loads.  What is
    // read from them after a store comes through the vector cache and waits for the store, too
    // (bodies of a batch read in place: 604 us per step of 64 jobs, copied in the centroid, probe and
    // vertex kernels 587; four capsules in one lattice 39.0 and 37.8).
    const BodyDev B = body_of<SOLO>(P, b);
    if ((B.rw2 >= MLS_COMPACT_RW2) != WIDE) return;   // the other form's launch
    const JobDev J = body_job<SOLO>(P, B);
    const WinDesc md = P.mdesc[b];
    BodyState& S = P.bstate[b];
    const int grp = threadIdx.x / MLS_GROUP, lane = threadIdx.x % MLS_GROUP;
    const int blk = blockIdx.x - B.blk_c0;
    if (SOLO)
        loaded(P.tri, P.x, P.uv, P.vbox, P.mwin, P.fwin, P.tgeo, B.nt, B.t0, B.v0, B.win_off, B.win_cap[0], B.win_cap[2],
               B.nblk_v, B.vbox0, B.rigid, B.kv, B.shell_h, B.wq, J.nx, J.ny, J.nz, J.bc[0], J.bc[2], J.bc[4], md.w[0],
               md.w[1], md.w[2], md.b[0], md.b[1], md.b[2]);
    const bool live = blk * PTS + grp < B.nt;
    const int t = live ? blk * PTS + grp : B.nt - 1;   // a spare group repeats the last triangle
    int err = 0;
    // everything this block reads before its MLS work is loaded first, so that the latencies
    // overlap: the vertex-block boxes of x^n, the triangle's vertices and the desired-velocity inputs
    double xa[3], xb_[3], xc[3], Ub[3] = {0, 0, 0};
    const int* tv = P.tri + 3 * (B.t0 + t);
    load3(P.x + 3 * (B.v0 + tv[0]), xa);
    load3(P.x + 3 * (B.v0 + tv[1]), xb_);
    load3(P.x + 3 * (B.v0 + tv[2]), xc);
    if (!B.rigid)
        for (int a = 0; a < 3; ++a)
            Ub[a] = (P.uv[3 * (B.v0 + tv[0]) + a] + P.uv[3 * (B.v0 + tv[1]) + a] +
                     P.uv[3 * (B.v0 + tv[2]) + a]) * (1.0 / 3.0);
    // boxes of the first VBOX_EARLY vertex blocks, held until the force window needs them (a box past
    // the last one repeats it)
    const int* box = P.vbox + 6LL * B.vbox0;
    int eb[VBOX_EARLY / IB_BLOCK][6];
#pragma unroll
    for (int i = 0; i < VBOX_EARLY / IB_BLOCK; ++i) {
        const int q = min(IB_BLOCK * i + (int)threadIdx.x, B.nblk_v - 1);
        for (int a = 0; a < 6; ++a) eb[i][a] = box[6 * q + a];
    }
    double cen[3], ab[3], ac[3], nn[3];
    for (int a = 0; a < 3; ++a) {
        cen[a] = (xa[a] + xb_[a] + xc[a]) * (1.0 / 3.0);
        ab[a] = xb_[a] - xa[a];
        ac[a] = xc[a] - xa[a];
    }
    MlsLane<WIDE> m;
    mls_locate<WIDE>(cen, B.rw2, lane, m);
    unsigned idx[N];
    float4 mom[N];
    mls_index<WIDE>(J, md, m, idx, err);
    // a lone body's launch is a latency chain: its moment loads go out before the solve; a
    // batched launch is throughput-bound and loads them after it, to hold fewer registers
    if (SOLO) MLS_SLOTS(s, m) mom[s] = P.mwin[B.win_off + idx[s]];
    cross3(ab, ac, nn);
    const double A = 0.5 * sqrt(dot3(nn, nn));
    if (live && lane == 0) {
        // geometry at x^n for the probes of this step
        double* g = P.tgeo + 6 * (B.t0 + t);
        for (int a = 0; a < 3; ++a) { g[a] = cen[a]; g[3 + a] = nn[a]; }
    }
    double Vt = 0.0;
    if (!B.rigid && B.kv != 0.0) {
        // signed volume of the tetrahedron (r, a, b, c), r = vertex 0 of the body
        double r0[3], pa[3], pb[3], pc[3], bc[3];
        load3(P.x + 3 * B.v0, r0);
        for (int a = 0; a < 3; ++a) { pa[a] = xa[a] - r0[a]; pb[a] = xb_[a] - r0[a]; pc[a] = xc[a] - r0[a]; }
        cross3(pb, pc, bc);
        Vt = dot3(pa, bc) * (1.0 / 6.0);
    }
    mls_solve<WIDE>(m, B.wq, false, err);
    if (!SOLO) MLS_SLOTS(s, m) mom[s] = P.mwin[B.win_off + idx[s]];
    double U[3];
    for (int a = 0; a < 3; ++a) U[a] = point_dot<WIDE>(m, m.phi, 1, mom, 1 + a);
    gsum8<3>(U);
    // desired boundary velocity U_b (Sec. 1.2): membranes average their vertex velocities,
    // rigid bodies move the marker with the body
    if (B.rigid) {
        double rr[3] = {cen[0] - S.X[0], cen[1] - S.X[1], cen[2] - S.X[2]}, w[3];
        cross3(S.om, rr, w);
        for (int a = 0; a < 3; ++a) Ub[a] = S.u[a] + w[a];
    }
    // F_l = (U_b - U*) / dt, spread with c_l = A_l h (Eq. bodyforce), as int64 fixed point
    const double fs = A * B.shell_h * FIX_SCALE;
    long long fx[N][3];   // fixed-point force of each slot's node
    for (int a = 0; a < 3; ++a) U[a] = Ub[a] - U[a];
    bool small = true;
    MLS_SLOTS(s, m)
        for (int a = 0; a < 3; ++a) fx[s][a] = fix_rn(fs * m.phi[s] * U[a], small);
    if (!__all(small)) {
        MLS_SLOTS(s, m)
            for (int a = 0; a < 3; ++a) fx[s][a] = __double2ll_rn(fs * m.phi[s] * U[a]);
    }
    int vb[6];
    for (int a = 0; a < 6; ++a) vb[a] = eb[0][a];
#pragma unroll
    for (int i = 1; i < VBOX_EARLY / IB_BLOCK; ++i)
        for (int a = 0; a < 3; ++a) { vb[a] = min(vb[a], eb[i][a]); vb[3 + a] = max(vb[3 + a], eb[i][3 + a]); }
    for (int q0 = VBOX_EARLY; q0 < B.nblk_v; q0 += 4 * IB_BLOCK) {
        int e[4][6];   // four boxes in flight per lane
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int q = min(q0 + IB_BLOCK * i + (int)threadIdx.x, B.nblk_v - 1);
            for (int a = 0; a < 6; ++a) e[i][a] = box[6 * q + a];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
            for (int a = 0; a < 3; ++a) { vb[a] = min(vb[a], e[i][a]); vb[3 + a] = max(vb[3 + a], e[i][3 + a]); }
    }
    spread_block<WIDE>(P, J, B, b, blk, vb, live, m, fx, err);
    // spare groups report too: they repeat the last triangle, and their lanes take columns of the box
    if (err) atomicOr(P.flags + B.job, err);
    if (B.rigid || B.kv == 0.0) return;
    // one partial of the volume per VOL_GROUP triangles, folded into V by the moments launch
    __shared__ double vol[PTS];
    if (lane == 0) vol[grp] = live ? Vt : 0.0;
    __syncthreads();
    constexpr int PARTS = PTS / VOL_GROUP;
    const int part = blk * PARTS + (int)threadIdx.x;
    if ((int)threadIdx.x < PARTS && part < B.nblk_c) {
        double sv = 0.0;
        for (int g = 0; g < VOL_GROUP; ++g) sv += vol[VOL_GROUP * threadIdx.x + g];
        store_partials(P, B, part, &sv, 1);
    }
}

// ---------------------------------------------------------------- vertex velocities
// Fluid velocity at every membrane vertex from the moments of f^{n+1} (the tentative velocity
// of Eq. verletPos).  It needs nothing from the probes, so its blocks ride in the probe launch
// and the vertex kernel only gathers forces and moves the vertices.  One group per vertex.
template <bool SOLO, bool WIDE>
__device__ void vertex_velocity_block(const Pools& P, int vb) {
    constexpr int N = MlsLane<WIDE>::N, PTS = IB_BLOCK / MLS_GROUP;
    const int b = block_body<SOLO>(P, P.blk_body_u, vb);
    const BodyDev B = body_of<SOLO>(P, b);
    if (B.rigid || (B.rw2 >= MLS_COMPACT_RW2) != WIDE) return;
    const JobDev J = body_job<SOLO>(P, B);
    const WinDesc md = P.mdesc[b];
    if (SOLO)
        loaded(P.x, P.mwin, B.nv, B.v0, B.win_off, B.wq, J.nx, J.ny, J.nz, J.bc[0], J.bc[2], J.bc[4], md.w[0], md.w[1],
               md.w[2], md.b[0], md.b[1], md.b[2]);
    const int grp = threadIdx.x / MLS_GROUP, lane = threadIdx.x % MLS_GROUP;
    const bool live = (vb - B.blk_u0) * PTS + grp < B.nv;
    const long long gv = B.v0 + (live ? (vb - B.blk_u0) * PTS + grp : B.nv - 1);
    int err = 0;
    double x[3];
    load3(P.x + 3 * gv, x);
    MlsLane<WIDE> m;
    unsigned idx[N];
    float4 mom[N];
    mls_locate<WIDE>(x, B.rw2, lane, m);
    mls_index<WIDE>(J, md, m, idx, err);
    MLS_SLOTS(s, m) mom[s] = P.mwin[B.win_off + idx[s]];
    mls_solve<WIDE>(m, B.wq, false, err);
    double u[3];
    for (int a = 0; a < 3; ++a) u[a] = point_dot<WIDE>(m, m.phi, 1, mom, 1 + a);
    gsum8<3>(u);
    if (live && lane < 3) P.u0v[3 * gv + lane] = lane == 0 ? u[0] : (lane == 1 ? u[1] : u[2]);
    if (err && live) atomicOr(P.flags + B.job, err);
}

// ---------------------------------------------------------------- triangles (probes)
// Group 2k evaluates the outer probe of triangle k of the block, group 2k+1 the inner one.
// Blocks from nblk_tri on compute the vertex velocities instead.
template <bool SOLO, bool WIDE>
__global__ void __launch_bounds__(IB_BLOCK, 4) k_triangles(Pools P, int nblk_tri) {
    constexpr int N = MlsLane<WIDE>::N, PTS = IB_BLOCK / MLS_GROUP, TRIS = PTS / 2;
    if ((int)blockIdx.x >= nblk_tri) {
        vertex_velocity_block<SOLO, WIDE>(P, blockIdx.x - nblk_tri);
        return;
    }
    const int b = block_body<SOLO>(P, P.blk_body_t, blockIdx.x);
    // copied before the first store
    const BodyDev B = body_of<SOLO>(P, b);
    if ((B.rw2 >= MLS_COMPACT_RW2) != WIDE) return;   // the other form's launch
    const JobDev J = body_job<SOLO>(P, B);
    const WinDesc md = P.mdesc[b];
    BodyState& S = P.bstate[b];
    const int grp = threadIdx.x / MLS_GROUP, lane = threadIdx.x % MLS_GROUP;
    const int blk = blockIdx.x - B.blk_t0;
    if (SOLO)
        loaded(P.tgeo, P.mwin, P.fext, P.fvol, B.nt, B.t0, B.win_off, B.probe, B.rigid, B.kv, B.wq, J.nx, J.ny, J.nz,
               J.nu, J.bc[0], J.bc[2], J.bc[4], md.w[0], md.w[1], md.w[2], md.b[0], md.b[1], md.b[2]);
    const int k = grp >> 1, side = grp & 1;
    const bool live = blk * TRIS + k < B.nt;
    const int t = live ? blk * TRIS + k : B.nt - 1;   // spare groups repeat the last triangle
    int err = 0;
    // centroid and normal at x^n, as the centroid kernel of this step computed them
    const double* g = P.tgeo + 6 * (B.t0 + t);
    double cen[3], nn[3], nrm[3], xp[3];
    for (int a = 0; a < 3; ++a) { cen[a] = g[a]; nn[a] = g[3 + a]; }
    const double ln = sqrt(dot3(nn, nn)), A = 0.5 * ln;
    const double sg = side == 0 ? B.probe : -B.probe;
    for (int a = 0; a < 3; ++a) {
        nrm[a] = nn[a] / ln;
        xp[a] = cen[a] + sg * nrm[a];
    }
    MlsLane<WIDE> m;
    unsigned idx[N];
    float4 mom[N];
    mls_locate<WIDE>(xp, B.rw2, lane, m);
    mls_index<WIDE>(J, md, m, idx, err);
    MLS_SLOTS(s, m) mom[s] = P.mwin[B.win_off + idx[s]];
    mls_solve<WIDE>(m, B.wq, true, err);
    // interpolated rho - 1 and the gradient rows of u* (diffuse derivatives), here and at the
    // triangle's other probe, in the other half of the 16 lanes
    double pp[10], pm[10];
    pp[0] = point_dot<WIDE>(m, m.phi, 1, mom, 0);
    for (int j = 0; j < 3; ++j) {
        pp[1 + j] = point_dot<WIDE>(m, &m.gr[0][j], 3, mom, 1);
        pp[4 + j] = point_dot<WIDE>(m, &m.gr[0][j], 3, mom, 2);
        pp[7 + j] = point_dot<WIDE>(m, &m.gr[0][j], 3, mom, 3);
    }
    gsum8<10>(pp);
    for (int i = 0; i < 10; ++i) pm[i] = dpp_f64<0x128>(pp[i]);   // row_ror:8
    if (err && live) atomicOr(P.flags + B.job, err);
    // outer minus inner probe (right in the outer probe's lanes): p = c_s^2 rho,
    // tau = rho nu (grad u + grad u^T); grad u [i][j] = pp[1 + 3 i + j]
    double Ft[3], Mt[3] = {0, 0, 0};
    const double nu = J.nu;
    const double rp = 1.0 + pp[0], rm = 1.0 + pm[0];
    const double dp = (pp[0] - pm[0]) * (1.0 / 3.0);
    for (int i = 0; i < 3; ++i) {
        double tn = 0.0;
        for (int j = 0; j < 3; ++j)
            tn += (rp * nu * (pp[1 + 3 * i + j] + pp[1 + 3 * j + i]) -
                   rm * nu * (pm[1 + 3 * i + j] + pm[1 + 3 * j + i])) * nrm[j];
        Ft[i] = (-dp * nrm[i] + tn) * A;
    }
    const bool store = live && side == 0 && lane == 0;
    if (store)
        for (int i = 0; i < 3; ++i) P.fext[3 * (B.t0 + t) + i] = Ft[i];
    if (!B.rigid) {
        // volume penalty (Eq. volFor, restoring): k_v (1 - V/V0) n_t A_t, a third per vertex
        if (B.kv == 0.0) return;
        const double vs = B.kv * (1.0 - S.V / B.V0) * (1.0 / 6.0);
        if (store)
            for (int i = 0; i < 3; ++i) P.fvol[3 * (B.t0 + t) + i] = vs * nn[i];
        return;
    }
    // one partial of force and torque per RED_GROUP triangles, folded, with the pose update, by
    // k_fold_bodies
    __shared__ double red[TRIS][6];
    const double rr[3] = {cen[0] - S.X[0], cen[1] - S.X[1], cen[2] - S.X[2]};
    cross3(rr, Ft, Mt);
    if (side == 0 && lane == 0)
        for (int i = 0; i < 3; ++i) { red[k][i] = live ? Ft[i] : 0.0; red[k][3 + i] = live ? Mt[i] : 0.0; }
    __syncthreads();
    constexpr int PARTS = TRIS / RED_GROUP;
    const int part = (int)threadIdx.x / 8, i = threadIdx.x % 8;
    if (part < PARTS && i < 6 && blk * PARTS + part < B.nblk_t) {
        double sum = 0.0;
        for (int q4 = 0; q4 < RED_GROUP; ++q4) sum += red[RED_GROUP * part + q4][i];
        P.partial[16LL * B.red_slot + i * partial_stride(B) + blk * PARTS + part] = sum;
    }
}

// Rigid body, Eqs. (linearVelRig), (angularVelRig), from the FP64 totals tot = (F, M).  Returns
// false for a non-finite or singular state.
__device__ bool rigid_update(const BodyDev& B, BodyState& S, const double tot[6]) {
    for (int i = 0; i < 3; ++i) { S.F[i] = tot[i]; S.M[i] = tot[3 + i]; }
    // Rigid body, Eqs. (linearVelRig), (angularVelRig): udot = F/m with net weight (m - V0) g,
    // omegadot = I_w^{-1} M with I_w = R I R^T.
    double F[3];
    for (int i = 0; i < 3; ++i) F[i] = tot[i] + (B.mass - B.V0) * B.gravity[i];
    double IR[9], Iw[9];
    for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 3; ++j) {
            double s = 0.0;
            for (int q = 0; q < 3; ++q) s += B.Ib[3 * i + q] * S.R[3 * j + q];  // I R^T
            IR[3 * i + j] = s;
        }
    for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 3; ++j) {
            double s = 0.0;
            for (int q = 0; q < 3; ++q) s += S.R[3 * i + q] * IR[3 * q + j];
            Iw[3 * i + j] = s;
        }
    // omegadot = Iw^{-1} M by the adjugate
    const double c00 = Iw[4] * Iw[8] - Iw[5] * Iw[7], c01 = Iw[5] * Iw[6] - Iw[3] * Iw[8],
                 c02 = Iw[3] * Iw[7] - Iw[4] * Iw[6];
    const double c10 = Iw[2] * Iw[7] - Iw[1] * Iw[8], c11 = Iw[0] * Iw[8] - Iw[2] * Iw[6],
                 c12 = Iw[1] * Iw[6] - Iw[0] * Iw[7];
    const double c20 = Iw[1] * Iw[5] - Iw[2] * Iw[4], c21 = Iw[2] * Iw[3] - Iw[0] * Iw[5],
                 c22 = Iw[0] * Iw[4] - Iw[1] * Iw[3];
    const double det = Iw[0] * c00 + Iw[1] * c01 + Iw[2] * c02;
    const double* M = tot + 3;
    const double wd[3] = {(c00 * M[0] + c10 * M[1] + c20 * M[2]) / det,
                          (c01 * M[0] + c11 * M[1] + c21 * M[2]) / det,
                          (c02 * M[0] + c12 * M[1] + c22 * M[2]) / det};
    double un[3], wn[3];
    for (int i = 0; i < 3; ++i) {
        un[i] = (2.0 / 3.0) * (2.0 * S.u[i] - 0.5 * S.u1[i] + F[i] / B.mass);
        wn[i] = (2.0 / 3.0) * (2.0 * S.om[i] - 0.5 * S.om1[i] + wd[i]);
    }
    for (int i = 0; i < 3; ++i) {
        S.u1[i] = S.u[i]; S.u[i] = un[i];
        S.om1[i] = S.om[i]; S.om[i] = wn[i];
        S.X[i] += un[i];
    }
    // R <- Rot(omega dt) R (Rodrigues)
    const double th = sqrt(dot3(wn, wn));
    double Rw[9] = {1, 0, 0, 0, 1, 0, 0, 0, 1};
    if (th > 0.0) {
        const double kx = wn[0] / th, ky = wn[1] / th, kz = wn[2] / th;
        // one argument reduction for both: less code on the fold's serial tail, which runs it once
        // per launch (1,280 partials: fold 7.96 -> 7.48 us)
        double s, cs;
        sincos(th, &s, &cs);
        const double c = 1.0 - cs;
        Rw[0] = 1.0 + c * (-ky * ky - kz * kz);  Rw[1] = -s * kz + c * kx * ky;  Rw[2] = s * ky + c * kx * kz;
        Rw[3] = s * kz + c * kx * ky;  Rw[4] = 1.0 + c * (-kx * kx - kz * kz);  Rw[5] = -s * kx + c * ky * kz;
        Rw[6] = -s * ky + c * kx * kz;  Rw[7] = s * kx + c * ky * kz;  Rw[8] = 1.0 + c * (-kx * kx - ky * ky);
    }
    double Rn[9];
    for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 3; ++j) {
            double s = 0.0;
            for (int q = 0; q < 3; ++q) s += Rw[3 * i + q] * S.R[3 * q + j];
            Rn[3 * i + j] = s;
        }
    bool fin = isfinite(det) && det != 0.0;
    for (int i = 0; i < 9; ++i) { S.R[i] = Rn[i]; fin = fin && isfinite(Rn[i]); }
    for (int i = 0; i < 3; ++i) fin = fin && isfinite(S.X[i]) && isfinite(un[i]) && isfinite(wn[i]);
    return fin;
}

// ---------------------------------------------------------------- per-body totals
// After the probe kernel, one block per body: hydrodynamic totals and the velocity / pose update of
// rigid bodies; other bodies return at once.
__global__ void __launch_bounds__(FOLD_THREADS) k_fold_bodies(Pools P) {
    const int b = blockIdx.x;
    const BodyDev& B = P.bodies[b];
    if (B.nv == 0 || !B.rigid) return;   // nv: an empty slot of a slotted batch
    double tot[6];
    fold_partials<6, FOLD_THREADS>(P, B, B.nblk_t, tot);
    if (threadIdx.x != 0) return;
    // the state and the body constants are read into registers at once and stored once
    const BodyDev Bc = B;
    BodyState S = P.bstate[b];
    const bool fin = rigid_update(Bc, S, tot);
    P.bstate[b] = S;
    if (!fin) atomicOr(P.flags + Bc.job, FLAG_NONFINITE);
}

// ---------------------------------------------------------------- vertices
template <bool SOLO>
__global__ void __launch_bounds__(VERT_BLOCK) k_vertices(Pools P) {
    const int b = block_body<SOLO>(P, P.blk_body_v, blockIdx.x);
    const BodyDev B = body_of<SOLO>(P, b);
    BodyState& S = P.bstate[b];
    const int grp = threadIdx.x / VERT_GROUP, lane = threadIdx.x % VERT_GROUP;
    const int blk = blockIdx.x - B.blk_v0;
    const int v = blk * VERT_PER_BLOCK + grp;
    if (SOLO)
        loaded(P.vt_list, P.vh_list, P.x, P.u0v, P.fext, P.fvol, P.fedge, P.xprev, P.uv, P.fv, P.vbox, B.nv, B.v0, B.t0,
               B.e0, B.vt_off, B.vh_off, B.vt_w, B.vh_w, B.rigid, B.integrator, B.mv, B.vbox0);
    __shared__ int box[VERT_PER_BLOCK][6];
    int err = 0;
    int bl[3] = {0x7fffffff, 0x7fffffff, 0x7fffffff}, bh[3] = {-0x7fffffff, -0x7fffffff, -0x7fffffff};
    if (v < B.nv) {
        const long long gv = B.v0 + v;
        // incidence entries first (lane j holds entry j when the lists fit in a group), so
        // that the force loads they address go out together with the moment loads
        const bool one = B.vt_w <= VERT_GROUP && B.vh_w <= VERT_GROUP;
        int tl0 = -1, hc0 = -1;
        if (one) {
            if (lane < B.vt_w) tl0 = P.vt_list[B.vt_off + (long long)v * B.vt_w + lane];
            if (!B.rigid && lane < B.vh_w) hc0 = P.vh_list[B.vh_off + (long long)v * B.vh_w + lane];
        }
        double x[3], xn[3], u0[3] = {0.0, 0.0, 0.0};
        load3(P.x + 3 * gv, x);
        if (!B.rigid) load3(P.u0v + 3 * gv, u0);   // fluid velocity, from the probe launch
        // gathered forces: a third of each incident triangle's probe force, its volume force (a
        // membrane without the penalty has none: it is neither written nor read, 641 -> 635 us per
        // step of 64 jobs), the spring and bending forces of every incident hinge; lane j takes entry j
        const bool vol = !B.rigid && B.kv != 0.0;
        double f[3] = {0.0, 0.0, 0.0};
        auto add_tri = [&](int tl) {
            const long long t = B.t0 + tl;
            for (int a = 0; a < 3; ++a) f[a] += P.fext[3 * t + a] * (1.0 / 3.0);
            if (vol)
                for (int a = 0; a < 3; ++a) f[a] += P.fvol[3 * t + a];
        };
        auto add_hinge = [&](int code) {
            const double* fe = P.fedge + 15LL * (B.e0 + (code >> 2));
            const int role = code & 3;
            const double sgn = role == 0 ? 1.0 : (role == 1 ? -1.0 : 0.0);
            for (int a = 0; a < 3; ++a) f[a] += sgn * fe[a] + fe[3 + 3 * role + a];
        };
        if (one) {
            if (tl0 >= 0) add_tri(tl0);
            if (hc0 >= 0) add_hinge(hc0);
        } else {
            for (int j = lane; j < B.vt_w; j += VERT_GROUP) {
                const int tl = P.vt_list[B.vt_off + (long long)v * B.vt_w + j];
                if (tl >= 0) add_tri(tl);
            }
            if (!B.rigid)
                for (int j = lane; j < B.vh_w; j += VERT_GROUP) {
                    const int code = P.vh_list[B.vh_off + (long long)v * B.vh_w + j];
                    if (code >= 0) add_hinge(code);
                }
        }
        const double F0 = gsum<VERT_GROUP>(f[0]), F1 = gsum<VERT_GROUP>(f[1]), F2 = gsum<VERT_GROUP>(f[2]);
        if (!B.rigid) {
            // tentative velocity u0: fluid velocity at the vertex from f^{n+1}
            const double Fv[3] = {F0, F1, F2};
            double un[3];
            for (int a = 0; a < 3; ++a) {
                const double acc = Fv[a] / B.mv;
                double dx;
                if (B.integrator == 1) {
                    // Eqs. (verletPos), (verletVel), (verletPos) as printed, in displacement form
                    un[a] = 1.5 * (u0[a] + 0.5 * acc) - 0.5 * (x[a] - P.xprev[3 * gv + a]);
                    dx = un[a] + 0.5 * acc;
                } else if (B.integrator == 2) {
                    // kinematic IB (Sec. 2.4): advected with the fluid velocity
                    un[a] = u0[a];
                    dx = un[a];
                } else {
                    // Eq. (verletPos); vertex velocity = displacement of the step
                    dx = u0[a] + 0.5 * acc;
                    un[a] = dx;
                }
                xn[a] = x[a] + dx;
            }
            if (lane == 0)
                for (int a = 0; a < 3; ++a) {
                    P.xprev[3 * gv + a] = x[a];
                    P.x[3 * gv + a] = xn[a];
                    P.uv[3 * gv + a] = un[a];
                    P.fv[3 * gv + a] = Fv[a];
                }
        } else {
            double xb[3], w[3];
            load3(P.xb + 3 * gv, xb);
            for (int a = 0; a < 3; ++a)
                xn[a] = S.X[a] + S.R[3 * a] * xb[0] + S.R[3 * a + 1] * xb[1] + S.R[3 * a + 2] * xb[2];
            const double rr[3] = {xn[0] - S.X[0], xn[1] - S.X[1], xn[2] - S.X[2]};
            cross3(S.om, rr, w);
            if (lane == 0)
                for (int a = 0; a < 3; ++a) {
                    P.xprev[3 * gv + a] = x[a];
                    P.x[3 * gv + a] = xn[a];
                    P.uv[3 * gv + a] = S.u[a] + w[a];
                    P.fv[3 * gv + a] = a == 0 ? F0 : (a == 1 ? F1 : F2);
                }
        }
        if (!(isfinite(xn[0]) && isfinite(xn[1]) && isfinite(xn[2])) ||
            fabs(xn[0]) > 1e7 || fabs(xn[1]) > 1e7 || fabs(xn[2]) > 1e7)
            err |= FLAG_NONFINITE;
        for (int a = 0; a < 3; ++a) { bl[a] = box_lo(xn[a]); bh[a] = box_hi(xn[a]); }
    }
    if (lane == 0)
        for (int a = 0; a < 3; ++a) { box[grp][a] = bl[a]; box[grp][3 + a] = bh[a]; }
    if (err) atomicOr(P.flags + B.job, err);
    __syncthreads();
    if (threadIdx.x == 0) {
        int* vb = P.vbox + 6LL * (B.vbox0 + blk);
        for (int a = 0; a < 3; ++a) {
            int lo = box[0][a], hi = box[0][3 + a];
            for (int g = 1; g < VERT_PER_BLOCK; ++g) { lo = min(lo, box[g][a]); hi = max(hi, box[g][3 + a]); }
            vb[a] = lo;
            vb[3 + a] = hi;
        }
    }
}

// ---------------------------------------------------------------- reported totals (membranes)
// FP64 hydrodynamic force and torque of the last step, torque about the vertex mean of x^n
// (held in xprev after the update).  One block, fixed-shape tree: reproducible.
__global__ void __launch_bounds__(256) k_body_totals(Pools P, int b, double* out) {
    const BodyDev& B = P.bodies[b];
    __shared__ double red[7][256];
    const int t = threadIdx.x;
    double c[3] = {0, 0, 0};
    for (int v = t; v < B.nv; v += 256)
        for (int a = 0; a < 3; ++a) c[a] += P.xprev[3 * (B.v0 + v) + a];
    for (int a = 0; a < 3; ++a) red[a][t] = c[a];
    __syncthreads();
    for (int w = 128; w >= 1; w >>= 1) {
        if (t < w) for (int a = 0; a < 3; ++a) red[a][t] += red[a][t + w];
        __syncthreads();
    }
    const double ctr[3] = {red[0][0] / B.nv, red[1][0] / B.nv, red[2][0] / B.nv};
    __syncthreads();
    double F[3] = {0, 0, 0}, M[3] = {0, 0, 0};
    for (int q = t; q < B.nt; q += 256) {
        const int* tv = P.tri + 3 * (B.t0 + q);
        double cen[3], f[3], m[3];
        for (int a = 0; a < 3; ++a) {
            cen[a] = (P.xprev[3 * (B.v0 + tv[0]) + a] + P.xprev[3 * (B.v0 + tv[1]) + a] +
                      P.xprev[3 * (B.v0 + tv[2]) + a]) * (1.0 / 3.0) - ctr[a];
            f[a] = P.fext[3 * (B.t0 + q) + a];
        }
        cross3(cen, f, m);
        for (int a = 0; a < 3; ++a) { F[a] += f[a]; M[a] += m[a]; }
    }
    for (int a = 0; a < 3; ++a) { red[a][t] = F[a]; red[3 + a][t] = M[a]; }
    __syncthreads();
    for (int w = 128; w >= 1; w >>= 1) {
        if (t < w) for (int a = 0; a < 6; ++a) red[a][t] += red[a][t + w];
        __syncthreads();
    }
    if (t < 6) out[t] = red[t][0];
}

// A launch in the compact form and, where a body's support needs it, one in the WIDE form: each
// serves the bodies of its form.  The edge blocks ride in the first.
void launch_centroids(const Pools& P, int nblk_tri, int nblk_edge, bool wide, hipStream_t s) {
    if (!(nblk_tri + nblk_edge > 0)) return;
    const dim3 grid(nblk_tri + nblk_edge), block(IB_BLOCK);
    if (P.solo_job >= 0) {
        hipLaunchKernelGGL((k_centroids<true, false>), grid, block, 0, s, P, nblk_tri);
        if (wide) hipLaunchKernelGGL((k_centroids<true, true>), dim3(nblk_tri), block, 0, s, P, nblk_tri);
    } else {
        hipLaunchKernelGGL((k_centroids<false, false>), grid, block, 0, s, P, nblk_tri);
        if (wide) hipLaunchKernelGGL((k_centroids<false, true>), dim3(nblk_tri), block, 0, s, P, nblk_tri);
    }
}
void launch_fold_bodies(const Pools& P, int nbodies, hipStream_t s) {
    if (nbodies > 0) hipLaunchKernelGGL(k_fold_bodies, dim3(nbodies), dim3(FOLD_THREADS), 0, s, P);
}

void launch_triangles(const Pools& P, int nblk_tri, int nblk_vel, bool wide, hipStream_t s) {
    if (!(nblk_tri + nblk_vel > 0)) return;
    const dim3 grid(nblk_tri + nblk_vel), block(IB_BLOCK);
    if (P.solo_job >= 0) {
        hipLaunchKernelGGL((k_triangles<true, false>), grid, block, 0, s, P, nblk_tri);
        if (wide) hipLaunchKernelGGL((k_triangles<true, true>), grid, block, 0, s, P, nblk_tri);
    } else {
        hipLaunchKernelGGL((k_triangles<false, false>), grid, block, 0, s, P, nblk_tri);
        if (wide) hipLaunchKernelGGL((k_triangles<false, true>), grid, block, 0, s, P, nblk_tri);
    }
}
void launch_vertices(const Pools& P, int nblocks, hipStream_t s) {
    if (!(nblocks > 0)) return;
    if (P.solo_job >= 0) hipLaunchKernelGGL(k_vertices<true>, dim3(nblocks), dim3(VERT_BLOCK), 0, s, P);
    else hipLaunchKernelGGL(k_vertices<false>, dim3(nblocks), dim3(VERT_BLOCK), 0, s, P);
}
void launch_body_totals(const Pools& P, int body, double* out6, hipStream_t s) {
    hipLaunchKernelGGL(k_body_totals, dim3(1), dim3(256), 0, s, P, body, out6);
}

}  // namespace lbib
