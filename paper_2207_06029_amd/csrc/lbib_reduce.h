#pragma once
// Sums over lanes and over the blocks of a body.
#include "lbib_internal.h"

namespace lbib {

template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
    // every control used here reads a valid lane, so no value for the others is set up
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}
// Sum over a group of G = 8 (half a DPP row) or 16 lanes (a row).  Lane exchanges xor 1 and xor 2
// are quad permutes, then the row half-mirror pairs the two quads of 8 lanes and the row mirror
// the two halves of a row (after the previous levels every lane of a block holds the same
// partial, so a mirror acts as an exchange).  Each level adds the same two operands on both
// partners, so every lane ends with the identical sum, and no value leaves the group.
template <int G>
__device__ __forceinline__ double gsum(double v) {
    static_assert(G == 8 || G == 16, "groups of 8 or 16 lanes");
    v += dpp_f64<0xB1>(v);   // quad_perm [1,0,3,2]
    v += dpp_f64<0x4E>(v);   // quad_perm [2,3,0,1]
    v += dpp_f64<0x141>(v);  // row_half_mirror
    if (G == 16) v += dpp_f64<0x140>(v);  // row_mirror
    return v;
}

// Deterministic per-body totals.  Every block of a body stores its partial sums (up to six values, one
// row per value in the body's region); one block per body folds them in a later launch (volumes: in a
// block of the moments launch), whose boundary makes the partials visible without a per-block
// device-scope release (each of which would write back an L2).  Thread t takes blocks t, t+512, ... in
// order, then a fixed tree (DPP within each wave, the eight waves in order) combines the 512 results; a
// block of 256 threads takes the parts of t and t+256.  The order depends only on the body's own block
// count, so totals are bitwise reproducible and independent of other jobs in the launch.
constexpr int FOLD_THREADS = 512;   // threads of the fold block: 2048 partials per load round

// A body's partials: value i of block k at 16 red_slot + i stride + k, stride = the body's larger
// block count (its region holds 16 such rows), so a wave of the fold reads value i of 64
// consecutive blocks from consecutive addresses.
__device__ __forceinline__ long long partial_stride(const BodyDev& B) { return max(B.nblk_c, B.nblk_t); }
__device__ __forceinline__ void store_partials(const Pools& P, const BodyDev& B, int blk, const double* v,
                                               int nval) {
    double* row = P.partial + 16LL * B.red_slot + blk;
    const long long st = partial_stride(B);
    for (int i = 0; i < nval; ++i) row[i * st] = v[i];
}

template <int NVAL, int THREADS>
__device__ __forceinline__ void fold_partials(const Pools& P, const BodyDev& B, int nblk, double* out) {
    constexpr int PASS = FOLD_THREADS / THREADS;
    __shared__ double s_red[NVAL][FOLD_THREADS / 64];
    // four slots per round, loaded together; summed in ascending block order
    const double* rows = P.partial + 16LL * B.red_slot;
    const long long st = partial_stride(B);
#pragma unroll
    for (int p = 0; p < PASS; ++p) {
        const int t = threadIdx.x + p * THREADS;
        double acc[NVAL];
        for (int i = 0; i < NVAL; ++i) acc[i] = 0.0;
        for (int k0 = t; k0 < nblk; k0 += 4 * FOLD_THREADS) {
            double v[4][NVAL];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int k = k0 + u * FOLD_THREADS;
                const double* col = rows + (k < nblk ? k : 0);
#pragma unroll
                for (int i = 0; i < NVAL; ++i) v[u][i] = col[i * st];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (k0 + u * FOLD_THREADS < nblk)
#pragma unroll
                    for (int i = 0; i < NVAL; ++i) acc[i] += v[u][i];
        }
        // each wave sums its 64 lanes (rows by DPP, then the four rows by two exchanges), wave 0's
        // first lane adds the waves in order: a fixed tree, so the totals are reproducible
#pragma unroll
        for (int i = 0; i < NVAL; ++i) {
            double v = gsum<16>(acc[i]);
            v += __shfl_xor(v, 16, 64);
            v += __shfl_xor(v, 32, 64);
            if (t % 64 == 0) s_red[i][t / 64] = v;
        }
    }
    __syncthreads();
    for (int i = 0; i < NVAL; ++i) {
        double v = s_red[i][0];
        for (int w = 1; w < FOLD_THREADS / 64; ++w) v += s_red[i][w];
        out[i] = v;
    }
}

// Enclosed volume V^n of one membrane with a volume penalty; other bodies return at once.
template <int THREADS>
__device__ __forceinline__ void fold_volume(const Pools& P, int b) {
    const BodyDev& B = P.bodies[b];
    if (B.nv == 0 || B.rigid || B.kv == 0.0) return;   // nv: an empty slot of a slotted batch
    double V;
    fold_partials<1, THREADS>(P, B, B.nblk_c, &V);
    if (threadIdx.x == 0) P.bstate[b].V = V;
}

}  // namespace lbib
