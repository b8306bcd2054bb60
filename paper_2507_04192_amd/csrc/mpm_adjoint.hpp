// Adjoint of the MPM step for gfx950 and the checkpointed rollout driver.
//
// Forward (mpm_forward_loss): the state is copied to a checkpoint every k
// steps; at observation frames the extraction operators Q_l and the masked
// squared error are evaluated on the device (loss in binary64).
//
// Backward (mpm_backward), segment by segment from the last: the segment's
// checkpoint is restored and its k steps recomputed into a tape of states
// and a grid tape (each step's sort, nodal mass and nodal velocity before
// and after the walls); then for each step in reverse (Sec. 3.1, eq:dzda;
// Sec. 3.3 recomputation):
//   g2p_adj   per particle: reverse of the constitutive update and of G2P;
//             node adjoints accumulated in LDS and written per tile
//   grid_adj  per node: reverse of the walls (dL/dmu) and of v = P/m + dt g
//             (2-D: inside p2g_adj)
//   p2g_adj   per particle: reverse of P2G, then the sort is undone by
//             writing each particle's adjoint at its slot before the step.
#pragma once

#include <type_traits>

#include "mpm_adjoint_device.hpp"
#include "mpm_kernels.hpp"

namespace mpm {

// threads of the reverse per-tile kernels (2-D: a tile's particles at once)
template <int D> constexpr int kAdjBlock = D == 2 ? 256 : 128;

// Waves per SIMD of the reverse G2P.  The materials without F take two, in 3-D
// binary64 at the price of a few spilled registers (fluid 20, viscous 36,
// hypoelastic 0 bytes a lane; with FLIP 180, 188, 72).  That pays where the
// tiles fill two: a tile is two waves, the chip 1024 SIMDs, so up to 512 tiles
// one wave each with all registers is as fast or faster.  Binary64, one wave and
// two, 97,336 particles: fluid 43 and 49 us, viscous 45 and 52, hypoelastic 56 and
// 56, with FLIP 67 and 82, 69 and 82, 72 and 85; 216,000: 67 and 57, 69 and 60, 63
// and 64, with FLIP 98 and 99, 100 and 99, 107 and 97; 381,216: 93 and 74, 96 and
// 80, 82 and 84, with FLIP 144 and 136, 146 and 139, 152 and 128.
template <int MAT> constexpr int kAdjWaves = mat_has_F(MAT) ? 1 : 2;
// The tiles with particles are not known to the host: at eight particles per
// cell, as most bodies are started, a full tile holds 512, and those at the
// border less; 131,072 fill 256, and reach about 400.
inline bool adj_few_tiles(const mpm_ctx* c) { return c->geo.ntiles <= 512 || c->N <= 131072; }

// Per-slot intermediate of the reverse sweep (mid), component-major with
// stride cap, written by k_g2p_adj and read by k_p2g_adj:
//   [0, D)              position adjoint
//   [D, D + D^2)        adjoint of the stored F_e - I (fluid: [D] holds J;
//                       hypoelastic Drucker-Prager: [D] J, then the
//                       constitutive part of the packed stress adjoint in
//                       [D + 1, D + 1 + D(D+1)/2), which fits the same slots)
//   [D + D^2, 2D + D^2) FLIP: the direct adjoint of the input velocity,
//                       alpha times that of v'
template <int D> struct MidLayout {
    static constexpr int X = 0, G = D, S = D + 1, V = D + D * D, N = D + D * D;
    static_assert(D + 1 + D * (D + 1) / 2 <= D + D * D, "stress adjoint fits the intermediate");
};

// f = x/h - base of a position, and along one axis the weight factors and the
// offset of the stencil's first node in the tile's block (clamped: memory guard).
template <class T>
__device__ __forceinline__ T block_axis_f(const Phys<T>& P, T x)
{
    const T t = mul_exact(x, P.inv);
    return t - floor(t - T(0.5));
}

template <class T, int D>
__device__ __forceinline__ int block_axis(const Geo& g, const Phys<T>& P, int a, T x, int tc, AxisFactors<T, D>& A)
{
    constexpr int TE = TileShape<D>::TE;
    const T t = mul_exact(x, P.inv), fb = floor(t - T(0.5));
    A.set(a, t - fb, P.inv, P.h);
    const int l = (int)fb + g.G - tc * TE;
    return l < 0 ? 0 : (l > TE - 1 ? TE - 1 : l);
}

// A transfer of component a between particle and nodes is
//   T(k) = w_x w_y w_z c + E^x(k_x) w_y w_z + w_x E^y(k_y) w_z + w_x w_y E^z(k_z),
//   E^b(k) = wd_b(k) p_b + dw_b(k) q_b
// (P2G: c = m v_a, p = m C_a, q = -dt V sigma_a; the adjoint of G2P: c, p and q
// the adjoints of the velocity, of C and of the velocity gradient).  axis_vjp
// contracts it with a node field f: R[b][k] = sum of f over the nodes with
// offset k along b, weighted with the other axes' w (the adjoint of E^b(k)), and
// wb[b][k] += the adjoint of w_b(k) through c and the other axes' E.  171
// multiply-adds per component, one reading of the field.
template <class B, class T, int D>
__device__ __forceinline__ void axis_vjp(const T (&f)[B::LN], int n0, const AxisFactors<T, D>& A, T c, const T E[D][3], T R[D][3],
                                         T wb[D][3])
{
    constexpr int LY = B::LY, LZ = B::LZ;
#pragma unroll
    for (int k = 0; k < 3; ++k) R[0][k] = R[1][k] = T(0);
    if constexpr (D == 2) {
#pragma unroll
        for (int ky = 0; ky < 3; ++ky)
#pragma unroll
            for (int kx = 0; kx < 3; ++kx) {
                const T p = f[n0 + ky * LY + kx];
                R[0][kx] = fma(A.w[1][ky], p, R[0][kx]);
                R[1][ky] = fma(A.w[0][kx], p, R[1][ky]);
                wb[0][kx] = fma(E[1][ky], p, wb[0][kx]);
                wb[1][ky] = fma(E[0][kx], p, wb[1][ky]);
            }
    } else {
        T xy[3][3];   // summed along z
#pragma unroll
        for (int ky = 0; ky < 3; ++ky)
#pragma unroll
            for (int kx = 0; kx < 3; ++kx) xy[ky][kx] = T(0);
#pragma unroll
        for (int kz = 0; kz < 3; ++kz) {
            T xz[3] = {T(0), T(0), T(0)};   // summed along y
            R[2][kz] = T(0);
#pragma unroll
            for (int ky = 0; ky < 3; ++ky) {
                T yz = T(0);                // summed along x
#pragma unroll
                for (int kx = 0; kx < 3; ++kx) {
                    const T p = f[n0 + kz * LZ + ky * LY + kx];
                    yz = fma(A.w[0][kx], p, yz);
                    xz[kx] = fma(A.w[1][ky], p, xz[kx]);
                    xy[ky][kx] = fma(A.w[2][kz], p, xy[ky][kx]);
                }
                R[2][kz] = fma(A.w[1][ky], yz, R[2][kz]);
                wb[1][ky] = fma(E[2][kz], yz, wb[1][ky]);
                wb[2][kz] = fma(E[1][ky], yz, wb[2][kz]);
            }
#pragma unroll
            for (int kx = 0; kx < 3; ++kx) {
                wb[0][kx] = fma(E[2][kz], xz[kx], wb[0][kx]);
                wb[2][kz] = fma(E[0][kx], xz[kx], wb[2][kz]);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int ky = 0; ky < 3; ++ky)
#pragma unroll
            for (int kx = 0; kx < 3; ++kx) {
                R[0][kx] = fma(A.w[1][ky], xy[ky][kx], R[0][kx]);
                R[1][ky] = fma(A.w[0][kx], xy[ky][kx], R[1][ky]);
                wb[0][kx] = fma(E[1][ky], xy[ky][kx], wb[0][kx]);
                wb[1][ky] = fma(E[0][kx], xy[ky][kx], wb[1][ky]);
            }
    }
#pragma unroll
    for (int b = 0; b < D; ++b)
#pragma unroll
        for (int k = 0; k < 3; ++k) wb[b][k] = fma(c, R[b][k], wb[b][k]);
}

// E of one component (see axis_vjp).
template <class T, int D>
__device__ __forceinline__ void axis_terms(const AxisFactors<T, D>& A, const T p[D], const T q[D], T E[D][3])
{
#pragma unroll
    for (int b = 0; b < D; ++b)
#pragma unroll
        for (int k = 0; k < 3; ++k) E[b][k] = fma(A.dw[b][k], q[b], A.wd[b][k] * p[b]);
}

// Position adjoint of one component through E: d wd_b / dx = dw_b dd - w_b and
// d dw_b / dx = ddw, the second derivative of the quadratic B-spline,
// (1, -2, 1) / h^2; with p_b = q_b summed against R once: sum_k R_b(k) (p_b
// (dw_b(k) dd(k) - w_b(k)) + q_b ddw(k)).  dwd: dw dd - w.
template <class T>
__device__ __forceinline__ T axis_dx(const T dwd[3], T inv2, T p, T q, const T R[3])
{
    return fma(p, dot3(dwd, R), q * (inv2 * (R[0] - T(2) * R[1] + R[2])));
}

// Reverse of the constitutive update, the kinematics x' = x + dt v and G2P,
// per particle of a tile.  First part: recomputes the G2P velocity and
// velocity gradient from the tile's node block and applies the constitutive
// VJP.  Second part, component by component: node adjoints of the velocity
// (accumulated in binary64 in LDS, then written as the tile's partial block)
// and the position adjoint through the weights and x_i - x_p (see axis_vjp).  The velocity,
// velocity-gradient and partial position adjoints pass between the parts in
// registers; the F (or J) adjoint and the position adjoint go to mid.
// FLIP (FL): v' = sum phi v_i + alpha (v_p - sum phi v_i^n); the adjoint of
// v^n = sum phi v_i^n is scattered to a second node block (binary64 LDS,
// written after the first in the tile's partial block), its weights pass
// an adjoint to the position, and alpha times the adjoint of v' goes to mid
// as the direct adjoint of v_p.
// What bounds it: the arithmetic, at the waves that its registers leave.  The LDS
// atomics (81 per particle) cost nothing measurable: with plain adds in their
// place the dam-break takes 137 us (136) in binary32 and 225 (215) in binary64.
// 3-D dam-break, 1,843,200 particles, by lines along x -> by axis sums: binary32
// 153 -> 133 us, binary64 333 -> 221 at two waves per SIMD (sand would spill: 114 ->
// 190 us on the half cylinder, where by axis sums alone it went 125 -> 114).
// WV: waves per SIMD asked for, see kAdjWaves.
template <class T, int D, int MAT, bool FL, int WV>
__global__ __launch_bounds__((kAdjBlock<D>)) __attribute__((amdgpu_waves_per_eu(WV))) void k_g2p_adj(Geo g, Phys<T> P, const int* __restrict__ meta,
                                                    const ActiveTile* __restrict__ active,
                                                    const int* __restrict__ perm, PView<T> st, PView<T> aout,
                                                    const T* __restrict__ gv, const T* __restrict__ gvo,
                                                    T* __restrict__ part, T* __restrict__ mid)
{
    constexpr int TE = TileShape<D>::TE, BE = TileShape<D>::BE, NB = TileShape<D>::NB;
    constexpr int NS = D * (D + 1) / 2;
    constexpr int NVA = FL ? 2 * D + 1 : D + 1;   // partial block values per node
    using ML = MidLayout<D>;
    // binary32 is faster on the padded block (3-D dam-break 147 -> 134 us);
    // binary64 is not (221 -> 227)
    using B = std::conditional_t<D == 3 && sizeof(T) == 4, PaddedBlock, DenseBlock<D>>;
    constexpr int LY = B::LY, LZ = B::LZ, LN = B::LN;
    constexpr int stride[3] = {1, LY, LZ};
    __shared__ T s_v[D][LN];
    __shared__ double s_b[D][LN];
    __shared__ T s_vo[FL ? D : 1][FL ? LN : 1];
    __shared__ double s_bo[FL ? D : 1][FL ? LN : 1];
    const int n_active = meta[0];
    const int tid = threadIdx.x;
    const long long cap = st.cap;
    const T inv2 = P.inv * P.inv;
    for (int it = 0;; ++it) {
        int e = tile_entry(it, n_active);
        if (e < 0) break;
        ActiveTile at = active[e];
        int tc[3];
        tile_coords(g, at.tile, tc);
        for (int i = tid; i < NB; i += kAdjBlock<D>) {
            int l0 = i % BE, l1 = (i / BE) % BE, l2 = (D == 3) ? i / (BE * BE) : 0;
            const int q = B::at(i);
            long long node = node_index(g, tc[0] * TE + l0, tc[1] * TE + l1, (D == 3) ? tc[2] * TE + l2 : 0);
#pragma unroll
            for (int a = 0; a < D; ++a) {
                s_v[a][q] = gv[a * g.NN + node];
                s_b[a][q] = 0.0;
                if constexpr (FL) {
                    s_vo[a][q] = gvo[a * g.NN + node];
                    s_bo[a][q] = 0.0;
                }
            }
        }
        __syncthreads();
        for (int k = tid; k < at.cnt; k += kAdjBlock<D>) {
            long long s = at.off + k;
            int j = perm[s];
            T xbar_c[D], vt_c[D], Lb_c[D][D], vob_c[FL ? D : 1];
            {
                T xp[D];
                AxisFactors<T, D> A;
                int n0 = 0;
    #pragma unroll
                for (int a = 0; a < D; ++a) {
                    xp[a] = st.x[a * cap + j];
                    n0 += block_axis(g, P, a, xp[a], tc[a], A) * stride[a];
                }
                // forward G2P of this particle: velocity and velocity gradient
                T vn[D], Lm[D][D];
    #pragma unroll
                for (int a = 0; a < D; ++a) {
                    T R[D][3];
                    axis_sums<B>(s_v[a], n0, A, R);
                    vn[a] = dot3(A.w[0], R[0]);
    #pragma unroll
                    for (int b = 0; b < D; ++b) Lm[a][b] = dot3(A.dw[b], R[b]);
                }
                // reverse of the constitutive update
                T Lb[D][D];
                if constexpr (MAT == MAT_FLUID) {
                    T Jb_in;
                    fluid_vjp<T, D>(P, Lm, st.G[j], aout.G[s], aout.S[s], Lb, Jb_in);
                    mid[ML::G * cap + s] = Jb_in;
                } else if constexpr (MAT == MAT_VFLUID) {
                    T sb[NS], Jb_in;
    #pragma unroll
                    for (int q = 0; q < NS; ++q) sb[q] = aout.S[q * cap + s];
                    vfluid_vjp<T, D>(P, Lm, st.G[j], aout.G[s], sb, Lb, Jb_in);
                    mid[ML::G * cap + s] = Jb_in;
                } else if constexpr (MAT == MAT_JAUMANN) {
                    T Sv[NS], sb[NS], sb_in[NS], Jb_in;
    #pragma unroll
                    for (int q = 0; q < NS; ++q) {
                        Sv[q] = st.S[q * cap + j];
                        sb[q] = aout.S[q * cap + s];
                    }
                    jaumann_vjp<T, D>(P, Lm, st.G[j], Sv, aout.G[s], sb, Lb, Jb_in, sb_in);
                    mid[ML::G * cap + s] = Jb_in;
    #pragma unroll
                    for (int q = 0; q < NS; ++q) mid[(ML::S + q) * cap + s] = sb_in[q];
                } else {
                    T G[D][D], Gb[D][D], Gb_in[D][D], sb[NS];
    #pragma unroll
                    for (int a = 0; a < D; ++a)
    #pragma unroll
                        for (int b = 0; b < D; ++b) {
                            G[a][b] = st.G[(a * D + b) * cap + j];
                            Gb[a][b] = aout.G[(a * D + b) * cap + s];
                        }
    #pragma unroll
                    for (int q = 0; q < NS; ++q) sb[q] = aout.S[q * cap + s];
                    hencky_vjp<T, D>(P, MAT == MAT_SAND, Lm, G, Gb, sb, Lb, Gb_in);
    #pragma unroll
                    for (int a = 0; a < D; ++a)
    #pragma unroll
                        for (int b = 0; b < D; ++b) mid[(ML::G + a * D + b) * cap + s] = Gb_in[a][b];
                }
                // x' = clamp(x + dt v'): no gradient through a clamped component
    #pragma unroll
                for (int a = 0; a < D; ++a) {
                    T xb = aout.x[a * cap + s];
                    T xn = xp[a] + P.dt * vn[a];
                    bool free_ = (xn >= T(0)) && (xn <= P.ext[a]);
                    xbar_c[a] = free_ ? xb : T(0);
                    const T vb_out = aout.v[a * cap + s];
                    vt_c[a] = vb_out + (free_ ? P.dt * xb : T(0));
                    if constexpr (FL) {
                        vob_c[a] = -P.flip_alpha * vb_out;
                        mid[(ML::V + a) * cap + s] = P.flip_alpha * vb_out;
                    }
    #pragma unroll
                    for (int b = 0; b < D; ++b) Lb_c[a][b] = Lb[a][b];
                }
            }
            {
                AxisFactors<T, D> A;
                T dwd[D][3];
                int n0 = 0;
    #pragma unroll
                for (int a = 0; a < D; ++a) {
                    const T f = block_axis_f(P, st.x[a * cap + j]);
                    n0 += block_axis(g, P, a, st.x[a * cap + j], tc[a], A) * stride[a];
    #pragma unroll
                    for (int q = 0; q < 3; ++q) dwd[a][q] = A.dw[a][q] * ((T(q) - f) * P.h) - A.w[a][q];
                }
                T xbar[D], vt[D], Cb[D][D], Lb[D][D];
    #pragma unroll
                for (int a = 0; a < D; ++a) {
                    xbar[a] = xbar_c[a];
                    vt[a] = vt_c[a];
    #pragma unroll
                    for (int b = 0; b < D; ++b) {
                        Cb[a][b] = aout.C[(a * D + b) * cap + s];
                        Lb[a][b] = Lb_c[a][b];
                    }
                }
                // the carried matrix of the other transfers: TPIC's C' = L
                // (its adjoint joins that of L), PIC's C' = 0 (none flows back)
                if (P.xfer != XF_APIC) {
    #pragma unroll
                    for (int a = 0; a < D; ++a)
    #pragma unroll
                        for (int b = 0; b < D; ++b) {
                            if (P.xfer == XF_TPIC) Lb[a][b] += Cb[a][b];
                            Cb[a][b] = T(0);
                        }
                }
                // Per component: the node adjoint of the velocity, scattered,
                //   phi (vt + Dinv Cb dd) + Lb grad phi,
                // a transfer of the same form as P2G (see axis_vjp), and its
                // position adjoint against the node velocities.
                T wb[D][3];
    #pragma unroll
                for (int b = 0; b < D; ++b)
    #pragma unroll
                    for (int q = 0; q < 3; ++q) wb[b][q] = T(0);
    #pragma unroll
                for (int a = 0; a < D; ++a) {
                    T E[D][3], R[D][3], pc[D];
    #pragma unroll
                    for (int b = 0; b < D; ++b) pc[b] = P.Dinv * Cb[a][b];
                    axis_terms<T, D>(A, pc, Lb[a], E);
                    axis_vjp<B>(s_v[a], n0, A, vt[a], E, R, wb);
    #pragma unroll
                    for (int b = 0; b < D; ++b) xbar[b] += axis_dx(dwd[b], inv2, pc[b], Lb[a][b], R[b]);
                    constexpr int KZ = (D == 3) ? 3 : 1;
    #pragma unroll
                    for (int kz = 0; kz < KZ; ++kz)
    #pragma unroll
                        for (int ky = 0; ky < 3; ++ky) {
                            T wyz = A.w[1][ky], U = fma(A.w[1][ky], vt[a], E[1][ky]);
                            if constexpr (D == 3) {
                                wyz *= A.w[D - 1][kz];
                                U = fma(A.w[D - 1][kz], U, A.w[1][ky] * E[D - 1][kz]);
                            }
    #pragma unroll
                            for (int kx = 0; kx < 3; ++kx) {
                                const int n = n0 + kz * LZ + ky * LY + kx;
                                atomicAdd(&s_b[a][n], (double)fma(wyz, E[0][kx], A.w[0][kx] * U));
                                if constexpr (FL) atomicAdd(&s_bo[a][n], (double)(A.w[0][kx] * wyz * vob_c[a]));
                            }
                        }
                    if constexpr (FL) {
    #pragma unroll
                        for (int b = 0; b < D; ++b)
    #pragma unroll
                            for (int q = 0; q < 3; ++q) E[b][q] = T(0);
                        axis_vjp<B>(s_vo[a], n0, A, vob_c[a], E, R, wb);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
    #pragma unroll
                for (int b = 0; b < D; ++b) xbar[b] += dot3(wb[b], A.dw[b]);
    #pragma unroll
                for (int a = 0; a < D; ++a) mid[(ML::X + a) * cap + s] = xbar[a];
            }
        }
        __syncthreads();
        // 2-D: by tile, so that the next kernel need not look the block up
        T* dst = part + (long long)(D == 2 ? at.tile : e) * NVA * NB;
        for (int i = tid; i < D * NB; i += kAdjBlock<D>) dst[i] = (T)s_b[i / NB][B::at(i % NB)];
        if constexpr (FL)
            for (int i = tid; i < D * NB; i += kAdjBlock<D>) dst[D * NB + i] = (T)s_bo[i / NB][B::at(i % NB)];
        __syncthreads();
    }
}

// Reverse of a node's update (walls, obstacles, v = P/m + dt g) from the
// adjoint vb of its velocity (overwritten): pb the adjoint of its momentum, mb
// of its mass m.  vt: the velocity before the walls; FLIP (FL): vob, the
// adjoint of the velocity before the update, v^n = Q / m = vo, whose Q gets
// qb.  amu (null: not added): dL/dmu per floor node.
template <class T, int D, bool FL>
__device__ __forceinline__ void node_adjoint(const Geo& g, const Phys<T>& P, const int I[3], T m, const T vt[D], T vb[D],
                                             const T* vo, const T* vob, double* __restrict__ amu, T pb[D], T& mb, T* qb)
{
    mb = T(0);
#pragma unroll
    for (int a = 0; a < D; ++a) pb[a] = T(0);
    if constexpr (FL)
#pragma unroll
        for (int a = 0; a < D; ++a) qb[a] = T(0);
    if (!(m > T(0))) return;
    // the walls forward, the velocity before each kept for its reverse (all
    // indexes are constants after unrolling, so nothing goes to scratch)
    T vin[2 * D][D], vel[D];
#pragma unroll
    for (int a = 0; a < D; ++a) vel[a] = vt[a];
    auto beyond = [&](int face) { const int ip = I[face / 2] - g.G; return face % 2 == 0 ? ip <= 0 : ip >= g.n[face / 2]; };
    auto floor_at = [&] {
        const int fx = min(I[0], g.box[0] - 1);
        return (D == 3) ? min(I[1], g.box[1] - 1) * P.floor_stride + fx : fx;
    };
    auto friction = [&](int face) { return face == 2 * (D - 1) && P.floor_mu ? P.floor_mu[floor_at()] : P.wall_mu[face]; };
#pragma unroll
    for (int face = 0; face < 2 * D; ++face) {
#pragma unroll
        for (int q = 0; q < D; ++q) vin[face][q] = vel[q];
        if (beyond(face))
            wall_node<T, D>(P.wall_mode[face], friction(face), face / 2, face % 2 == 0 ? T(-1) : T(1), vel);
    }
    // resting obstacles after the walls (Sec. 4.2.1): a component that one of
    // them removed passes no adjoint back
    if (P.n_obst > 0) {
        double xi[D];
#pragma unroll
        for (int a = 0; a < D; ++a) xi[a] = double(I[a] - g.G) * P.obst_h;
        for (int o = 0; o < P.n_obst; ++o) {
            const int cut = obstacle_component<T, D>(P, o, xi, vel);
#pragma unroll
            for (int a = 0; a < D; ++a)
                if (cut == a) vel[a] = vb[a] = T(0);
        }
    }
#pragma unroll
    for (int face = 2 * D - 1; face >= 0; --face) {
        if (!beyond(face)) continue;
        const T mub = wall_node_vjp<T, D>(P.wall_mode[face], friction(face), face / 2, face % 2 == 0 ? T(-1) : T(1), vin[face], vb);
        if (amu && face == 2 * (D - 1) && P.floor_mu && mub != T(0)) atomicAdd(&amu[floor_at()], (double)mub);
    }
    T dot = T(0);
#pragma unroll
    for (int a = 0; a < D; ++a) {
        pb[a] = vb[a] / m;
        dot += vb[a] * (vt[a] - P.dt * P.g[a]);
        if constexpr (FL) {
            dot += vob[a] * vo[a];
            qb[a] = vob[a] / m;
        }
    }
    mb = -dot / m;
}

template <class T, int D, bool FL>
__global__ __launch_bounds__((kAdjBlock<D>)) void k_grid_adj(Geo g, Phys<T> P, const int* __restrict__ meta,
                                                     const ActiveTile* __restrict__ active,
                                                     const int* __restrict__ tile_slot, const T* __restrict__ part,
                                                     T* __restrict__ gmass, const T* __restrict__ gvt,
                                                     T* __restrict__ gv, T* __restrict__ gvo,
                                                     double* __restrict__ amu)
{
    // FLIP: the partial blocks also carry the adjoint of the velocity before
    // the update, after the first D
    constexpr int NVA = FL ? 2 * D + 1 : D + 1, NS = FL ? 2 * D : D;
    struct Node {
        T m, vt[D], vo[D];
    };
    __shared__ int s_around[kAdjBlock<D> / 64][27];
    for (int it = 0;; ++it) {
        const int tile = node_tile<kAdjBlock<D> / 64>(it, meta, active, g.ntiles);
        if (tile < 0) break;
        tile_nodes<T, NVA, NS>(
            g, tile, tile_slot, part, s_around[threadIdx.x >> 6],
            [&](long long node) {
                Node in;
                in.m = gmass[node];
#pragma unroll
                for (int a = 0; a < D; ++a) {
                    in.vt[a] = gvt[a * g.NN + node];
                    if constexpr (FL) in.vo[a] = gvo[a * g.NN + node];
                }
                return in;
            },
            [&](const int I[3], long long node, const Node& in, T sum[NS]) {
                T pb[D], qb[D], mb;
                node_adjoint<T, D, FL>(g, P, I, in.m, in.vt, sum, in.vo, sum + NS - D, amu, pb, mb, qb);
#pragma unroll
                for (int a = 0; a < D; ++a) gv[a * g.NN + node] = pb[a];
                gmass[node] = mb;
                // FLIP: the adjoint of Q replaces v^n in the record
                if constexpr (FL)
#pragma unroll
                    for (int a = 0; a < D; ++a) gvo[a * g.NN + node] = qb[a];
            });
    }
}

// 2-D: what the reverse of P2G needs to form its tile's node adjoints itself
// (as k_grid_adj, 1.56 times per node, the owner adding to dL/dmu): a launch
// and its chain of round trips less in a step that is nothing but those.
// 6,000 particles, binary64, per reverse step: g2p_adj 10.3, grid_adj 5.0,
// p2g_adj 6.2 us -> 7.3 (256 threads per tile) and 7.2.
template <class T>
struct NodesAdj2 {
    const T* part;
    const int* tile_slot;
    const T *gmass, *gvt, *gvo;
    double* amu;
};

template <class T, bool FL>
__device__ __forceinline__ void node_adj_block2(const Geo& g, const Phys<T>& P, const NodesAdj2<T>& nd, int tile, int tid,
                                                T (&s_p)[2][TileShape<2>::NB], T (*s_f)[FL ? TileShape<2>::NB : 1], T* s_m)
{
    constexpr int D = 2, NB = TileShape<D>::NB, NV = FL ? 2 * D : D, NS = FL ? 2 * D + 1 : D + 1;
    if (tid >= NB) return;
    int tc[3];
    tile_coords(g, tile, tc);
    const long long node = node_index(g, tc[0] * TileShape<D>::TE + tid % TileShape<D>::BE,
                                      tc[1] * TileShape<D>::TE + tid / TileShape<D>::BE, 0);
    const T m = nd.gmass[node];
    T vt[D], vo[D] = {T(0), T(0)};
#pragma unroll
    for (int a = 0; a < D; ++a) {
        vt[a] = nd.gvt[a * g.NN + node];
        if constexpr (FL) vo[a] = nd.gvo[a * g.NN + node];
    }
    int I[3];
    T sum[NV], pb[D], qb[D], mb;
    const int des = block_sum2<T, NV, NS>(g, nd.tile_slot, nd.part, tile, tid, I, sum);
    node_adjoint<T, D, FL>(g, P, I, m, vt, sum, vo, &sum[FL ? D : 0], des == tile ? nd.amu : nullptr, pb, mb, qb);
    s_m[tid] = mb;
#pragma unroll
    for (int a = 0; a < D; ++a) {
        if constexpr (FL) {
            s_f[a][tid] = pb[a];
            s_p[a][tid] = pb[a] + qb[a];
        } else {
            s_p[a][tid] = pb[a];
        }
    }
}

// At least two waves per SIMD in binary64.  3-D dam-break, 1,843,200 particles,
// by lines along x -> by axis sums: binary32 117 -> 97 us, binary64 191 -> 156;
// it is left with its traffic (the adjoint goes back to the order before the
// sort, partial lines at its ends).
// FLIP (FL): the force-free momentum Q (for v^n = Q / m) shares P's affine
// part, so the affine gathers take p + q (q the adjoint of Q, gqb) and the
// force's gathers p alone; the direct adjoint of v_p comes from mid.
template <class T, int D, int MAT, bool FL>
__global__ __launch_bounds__((kAdjBlock<D>)) __attribute__((amdgpu_waves_per_eu(2))) void k_p2g_adj(Geo g, Phys<T> P, const int* __restrict__ meta,
                                                    const ActiveTile* __restrict__ active,
                                                    const int* __restrict__ perm, PView<T> st,
                                                    const T* __restrict__ gpb, const T* __restrict__ gmb,
                                                    const T* __restrict__ gqb,
                                                    const T* __restrict__ mid, PView<T> ain, NodesAdj2<T> nd)
{
    constexpr int TE = TileShape<D>::TE, BE = TileShape<D>::BE, NB = TileShape<D>::NB;
    using ML = MidLayout<D>;
    using B = DenseBlock<D>;
    constexpr int stride[3] = {1, B::LY, B::LZ};
    __shared__ T s_p[D][NB];     // p (FL: p + q)
    __shared__ T s_f[FL ? D : 1][FL ? NB : 1];   // FL: p
    __shared__ T s_m[NB];
    const int n_active = meta[0];
    const int tid = threadIdx.x;
    const long long cap = st.cap;
    const T inv2 = P.inv * P.inv;
    for (int it = 0;; ++it) {
        int e = tile_entry(it, n_active);
        if (e < 0) break;
        ActiveTile at = active[e];
        int tc[3];
        tile_coords(g, at.tile, tc);
        if constexpr (D == 2) node_adj_block2<T, FL>(g, P, nd, at.tile, tid, s_p, s_f, s_m);
        else
        for (int i = tid; i < NB; i += kAdjBlock<D>) {
            int l0 = i % BE, l1 = (i / BE) % BE, l2 = (D == 3) ? i / (BE * BE) : 0;
            long long node = node_index(g, tc[0] * TE + l0, tc[1] * TE + l1, (D == 3) ? tc[2] * TE + l2 : 0);
            s_m[i] = gmb[node];
#pragma unroll
            for (int a = 0; a < D; ++a) {
                const T pv = gpb[a * g.NN + node];
                if constexpr (FL) {
                    s_f[a][i] = pv;
                    s_p[a][i] = pv + gqb[a * g.NN + node];
                } else {
                    s_p[a][i] = pv;
                }
            }
        }
        __syncthreads();
        for (int k = tid; k < at.cnt; k += kAdjBlock<D>) {
            long long s = at.off + k;
            int j = perm[s];
            AxisFactors<T, D> A;
            T dwd[D][3], vp[D], Cp[D][D], Sp[D][D];
            int n0 = 0;
#pragma unroll
            for (int a = 0; a < D; ++a) {
                const T xa = st.x[a * cap + j], f = block_axis_f(P, xa);
                n0 += block_axis(g, P, a, xa, tc[a], A) * stride[a];
#pragma unroll
                for (int q = 0; q < 3; ++q) dwd[a][q] = A.dw[a][q] * ((T(q) - f) * P.h) - A.w[a][q];
                vp[a] = st.v[a * cap + j];
#pragma unroll
                for (int b2 = 0; b2 < D; ++b2) Cp[a][b2] = st.C[(a * D + b2) * cap + j];
            }
            if constexpr (MAT == MAT_FLUID) {
                T si = st.S[j];
#pragma unroll
                for (int a = 0; a < D; ++a)
#pragma unroll
                    for (int b = 0; b < D; ++b) Sp[a][b] = (a == b) ? si : T(0);
            } else if constexpr (D == 3) {
                Sp[0][0] = st.S[0 * cap + j]; Sp[1][1] = st.S[1 * cap + j]; Sp[2][2] = st.S[2 * cap + j];
                Sp[0][1] = Sp[1][0] = st.S[3 * cap + j];
                Sp[0][2] = Sp[2][0] = st.S[4 * cap + j];
                Sp[1][2] = Sp[2][1] = st.S[5 * cap + j];
            } else {
                Sp[0][0] = st.S[0 * cap + j]; Sp[1][1] = st.S[1 * cap + j];
                Sp[0][1] = Sp[1][0] = st.S[2 * cap + j];
            }
            // With p_i, m_i the node adjoints of momentum and mass, per component
            // (see axis_vjp, c = m v, p = m C, q = -dt S):
            //   vbar = m sum phi p,  Cbar_b = m sum phi p dd_b = m sum_k wd_b R_b,
            //   Sbar_b = -dt sum p d_b phi = -dt sum_k dw_b R_b,
            // and the position adjoint through the weights (wb) and through E.
            // FLIP: the affine part takes p + q (s_p), the force p alone (s_f).
            T xbar[D], vbar[D], Cbar[D][D], Sbar[D][D], wb[D][3];
#pragma unroll
            for (int b = 0; b < D; ++b) {
                xbar[b] = mid[b * cap + s];
#pragma unroll
                for (int q = 0; q < 3; ++q) wb[b][q] = T(0);
            }
#pragma unroll
            for (int a = 0; a < D; ++a) {
                T E[D][3], R[D][3], pc[D], qc[D], none[D];
                const T c = P.mass * vp[a];
#pragma unroll
                for (int b = 0; b < D; ++b) {
                    pc[b] = P.mass * Cp[a][b];
                    qc[b] = -P.dt * Sp[a][b];
                    none[b] = T(0);
                }
                axis_terms<T, D>(A, pc, FL ? none : qc, E);
                axis_vjp<B>(s_p[a], n0, A, c, E, R, wb);
                vbar[a] = P.mass * dot3(A.w[0], R[0]);
                if constexpr (FL) vbar[a] += mid[(ML::V + a) * cap + s];
#pragma unroll
                for (int b = 0; b < D; ++b) {
                    Cbar[a][b] = P.mass * dot3(A.wd[b], R[b]);
                    if constexpr (!FL) Sbar[a][b] = -P.dt * dot3(A.dw[b], R[b]);
                    xbar[b] += axis_dx(dwd[b], inv2, pc[b], FL ? T(0) : qc[b], R[b]);
                }
                if constexpr (FL) {
                    axis_terms<T, D>(A, none, qc, E);
                    axis_vjp<B>(s_f[a], n0, A, T(0), E, R, wb);
#pragma unroll
                    for (int b = 0; b < D; ++b) {
                        Sbar[a][b] = -P.dt * dot3(A.dw[b], R[b]);
                        xbar[b] += axis_dx(dwd[b], inv2, T(0), qc[b], R[b]);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            {
                T R[D][3];
                axis_sums<B>(s_m, n0, A, R);
#pragma unroll
                for (int b = 0; b < D; ++b) {
#pragma unroll
                    for (int q = 0; q < 3; ++q) wb[b][q] = fma(P.mass, R[b][q], wb[b][q]);
                    xbar[b] += dot3(wb[b], A.dw[b]);
                }
            }
            // the particle's adjoint goes to its slot before the step's sort
#pragma unroll
            for (int a = 0; a < D; ++a) {
                ain.x[a * cap + j] = xbar[a];
                ain.v[a * cap + j] = vbar[a];
#pragma unroll
                for (int b = 0; b < D; ++b) ain.C[(a * D + b) * cap + j] = Cbar[a][b];
            }
            if constexpr (MAT == MAT_FLUID) {
                ain.G[j] = mid[D * cap + s];
                T tr = T(0);
#pragma unroll
                for (int a = 0; a < D; ++a) tr += Sbar[a][a];
                ain.S[j] = tr;
            } else if constexpr (MAT == MAT_VFLUID) {
                // J carried; the stress is recomputed from J and L each step,
                // so its input adjoint is the force's part only
                ain.G[j] = mid[D * cap + s];
                if constexpr (D == 3) {
                    ain.S[0 * cap + j] = Sbar[0][0];
                    ain.S[1 * cap + j] = Sbar[1][1];
                    ain.S[2 * cap + j] = Sbar[2][2];
                    ain.S[3 * cap + j] = Sbar[0][1] + Sbar[1][0];
                    ain.S[4 * cap + j] = Sbar[0][2] + Sbar[2][0];
                    ain.S[5 * cap + j] = Sbar[1][2] + Sbar[2][1];
                } else {
                    ain.S[0 * cap + j] = Sbar[0][0];
                    ain.S[1 * cap + j] = Sbar[1][1];
                    ain.S[2 * cap + j] = Sbar[0][1] + Sbar[1][0];
                }
            } else if constexpr (MAT == MAT_JAUMANN) {
                // the force's part of the stress adjoint plus the constitutive part
                constexpr int S0 = MidLayout<D>::S;
                ain.G[j] = mid[D * cap + s];
                if constexpr (D == 3) {
                    ain.S[0 * cap + j] = Sbar[0][0] + mid[(S0 + 0) * cap + s];
                    ain.S[1 * cap + j] = Sbar[1][1] + mid[(S0 + 1) * cap + s];
                    ain.S[2 * cap + j] = Sbar[2][2] + mid[(S0 + 2) * cap + s];
                    ain.S[3 * cap + j] = Sbar[0][1] + Sbar[1][0] + mid[(S0 + 3) * cap + s];
                    ain.S[4 * cap + j] = Sbar[0][2] + Sbar[2][0] + mid[(S0 + 4) * cap + s];
                    ain.S[5 * cap + j] = Sbar[1][2] + Sbar[2][1] + mid[(S0 + 5) * cap + s];
                } else {
                    ain.S[0 * cap + j] = Sbar[0][0] + mid[(S0 + 0) * cap + s];
                    ain.S[1 * cap + j] = Sbar[1][1] + mid[(S0 + 1) * cap + s];
                    ain.S[2 * cap + j] = Sbar[0][1] + Sbar[1][0] + mid[(S0 + 2) * cap + s];
                }
            } else {
#pragma unroll
                for (int a = 0; a < D; ++a)
#pragma unroll
                    for (int b = 0; b < D; ++b) ain.G[(a * D + b) * cap + j] = mid[(D + a * D + b) * cap + s];
                if constexpr (D == 3) {
                    ain.S[0 * cap + j] = Sbar[0][0];
                    ain.S[1 * cap + j] = Sbar[1][1];
                    ain.S[2 * cap + j] = Sbar[2][2];
                    ain.S[3 * cap + j] = Sbar[0][1] + Sbar[1][0];
                    ain.S[4 * cap + j] = Sbar[0][2] + Sbar[2][0];
                    ain.S[5 * cap + j] = Sbar[1][2] + Sbar[2][1];
                } else {
                    ain.S[0 * cap + j] = Sbar[0][0];
                    ain.S[1 * cap + j] = Sbar[1][1];
                    ain.S[2 * cap + j] = Sbar[0][1] + Sbar[1][0];
                }
            }
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// Observation operators and loss (Sec. 3.2, eq:inverse_loss)
// ---------------------------------------------------------------------------

// Lagrangian tracers: Q_l = z of particle l.  Adds m |Q - z_obs|^2 to the
// loss and, when seed != 0, 2 m (Q - z_obs) to the adjoint of z.
template <class T, int D>
__global__ void k_lag_obs(const T* __restrict__ z, T* __restrict__ zb, long long cap, long long N,
                          const int32_t* __restrict__ inv, const int32_t* __restrict__ tracer, int ntr,
                          const T* __restrict__ target, const T* __restrict__ mask, int seed,
                          double* __restrict__ loss)
{
    int l = blockIdx.x * kBlock + threadIdx.x;
    double part = 0.0;
    // an id outside [0, N) is skipped (it names no particle)
    if (l < ntr && tracer[l] >= 0 && tracer[l] < N) {
        int s = inv[tracer[l]];
        T m = mask ? mask[l] : T(1);
        if (m != T(0)) {
#pragma unroll
            for (int a = 0; a < D; ++a) {
                T r = z[a * cap + s] - target[a * ntr + l];
                part += (double)m * (double)r * (double)r;
                if (seed) zb[a * cap + s] += T(2) * m * r;
            }
        }
    }
    // wave reduction, one atomic per wave
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) part += __shfl_xor(part, o);
    if ((threadIdx.x & 63) == 0 && part != 0.0) atomicAdd(loss, part);
}

struct Boxes {
    double lo[kMaxBoxes][3], hi[kMaxBoxes][3];
    int n;
};

template <class T, int D>
__device__ __forceinline__ bool in_box(const Boxes& bx, int b, const T* x, long long cap, long long s)
{
    bool in = true;
#pragma unroll
    for (int a = 0; a < D; ++a) {
        T xv = x[a * cap + s];
        in = in && (xv >= (T)bx.lo[b][a]) && (xv < (T)bx.hi[b][a]);
    }
    return in;
}

// Eulerian boxes, pass 1: per-box sums of z and particle counts (binary64).
template <class T, int D>
__global__ void k_box_sum(Boxes bx, const T* __restrict__ x, const T* __restrict__ z, long long cap, long long N,
                          double* __restrict__ sum, int* __restrict__ cnt)
{
    long long s = (long long)blockIdx.x * kBlock + threadIdx.x;
    for (int b = 0; b < bx.n; ++b) {
        bool in = s < N && in_box<T, D>(bx, b, x, cap, s);
        unsigned long long msk = __ballot(in);
        double acc[D];
#pragma unroll
        for (int a = 0; a < D; ++a) {
            double v = in ? (double)z[a * cap + s] : 0.0;
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
            acc[a] = v;
        }
        if ((threadIdx.x & 63) == 0 && msk) {
            atomicAdd(&cnt[b], __popcll(msk));
#pragma unroll
            for (int a = 0; a < D; ++a) atomicAdd(&sum[b * 3 + a], acc[a]);
        }
    }
}

// Eulerian boxes, pass 2 (one thread per box): Q, the loss and the seed
// coefficient 2 m (Q - z_obs) / |P_l| per box; empty boxes contribute nothing.
template <class T, int D>
__global__ void k_box_loss(int nbox, const double* __restrict__ sum, const int* __restrict__ cnt,
                           const T* __restrict__ target, const T* __restrict__ mask, double* __restrict__ coef,
                           double* __restrict__ loss)
{
    int b = threadIdx.x;
    if (b >= nbox) return;
    double m = mask ? (double)mask[b] : 1.0;
    int c = cnt[b];
    double part = 0.0;
#pragma unroll
    for (int a = 0; a < D; ++a) {
        double cf = 0.0;
        if (c > 0 && m != 0.0) {
            double r = sum[b * 3 + a] / c - (double)target[a * nbox + b];
            part += m * r * r;
            cf = 2.0 * m * r / c;
        }
        coef[b * 3 + a] = cf;
    }
    if (part != 0.0) atomicAdd(loss, part);
}

template <class T, int D>
__global__ void k_box_seed(Boxes bx, const T* __restrict__ x, T* __restrict__ zb, long long cap, long long N,
                           const double* __restrict__ coef)
{
    long long s = (long long)blockIdx.x * kBlock + threadIdx.x;
    if (s >= N) return;
    for (int b = 0; b < bx.n; ++b) {
        if (!in_box<T, D>(bx, b, x, cap, s)) continue;
#pragma unroll
        for (int a = 0; a < D; ++a) zb[a * cap + s] += (T)coef[b * 3 + a];
    }
}

template <class T, int D>
__global__ void k_lag_extract(const T* __restrict__ z, long long cap, long long N, const int32_t* __restrict__ inv,
                              const int32_t* __restrict__ tracer, int ntr, T* __restrict__ q)
{
    int l = blockIdx.x * kBlock + threadIdx.x;
    if (l >= ntr) return;
    int id = tracer[l];
    bool ok = id >= 0 && id < N;
    int s = ok ? inv[id] : 0;
#pragma unroll
    for (int a = 0; a < D; ++a) q[a * ntr + l] = ok ? z[a * cap + s] : T(0);
}

template <class T, int D>
__global__ void k_box_mean(int nbox, const double* __restrict__ sum, const int* __restrict__ cnt, T* __restrict__ q)
{
    int b = threadIdx.x;
    if (b >= nbox) return;
#pragma unroll
    for (int a = 0; a < D; ++a) q[a * nbox + b] = cnt[b] > 0 ? (T)(sum[b * 3 + a] / cnt[b]) : T(0);
}

template <class T>
__global__ void k_mu_out(const double* __restrict__ amu, long long n, T* __restrict__ out)
{
    long long i = (long long)blockIdx.x * kBlock + threadIdx.x;
    if (i < n) out[i] = (T)amu[i];
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------

template <class T, int D>
struct Adjoint {
    using S = Solver<T, D>;

    static PView<T> slot_view(const mpm_ctx* c, char* base, int32_t* pid)
    {
        PView<T> v{};
        T* b = (T*)base;
        long long cap = c->cap;
        v.cap = cap;
        v.x = b;
        v.v = b + D * cap;
        v.C = b + 2 * D * cap;
        v.G = b + (2 * D + D * D) * cap;
        v.S = v.G + (mat_has_F(c->mat) ? D * D : 1) * cap;
        v.pid = pid;
        return v;
    }
    static size_t state_bytes(const mpm_ctx* c) { return (size_t)c->nsc * (size_t)c->cap * sizeof(T); }
    static PView<T> ckpt(const mpm_ctx* c, int i)
    {
        return slot_view(c, c->ckpt + (size_t)i * state_bytes(c), c->ckpt_pid + (size_t)i * c->cap);
    }
    // State i (1..ckpt_every) of tape slot q (one slot per taped segment).
    static PView<T> tape(const mpm_ctx* c, int q, int i)
    {
        const size_t at = (size_t)q * (size_t)c->ckpt_every + (size_t)(i - 1);
        return slot_view(c, c->tape + at * state_bytes(c), c->tape_pid + at * c->cap);
    }
    // State i (0..ckpt_every) of segment seg of a rollout of n steps, its steps
    // on tape slot q.  A segment's ends are the checkpoints themselves: steps
    // read and write them in place.  Forward plus adjoint with copies between
    // checkpoint and tape and a whole last recomputed step, and so: 10 steps of
    // 442,368 particles in binary64, segments of 5, one taped 3457 -> 3343 us;
    // 6 steps of 1.8 M in binary32, segments of 3, 3447 -> 3190 us.
    static PView<T> seg_state(const mpm_ctx* c, int seg, int q, int i, int n)
    {
        const int t = seg * c->ckpt_every + i;
        return t % c->ckpt_every == 0 && t < n ? ckpt(c, t / c->ckpt_every) : tape(c, q, i);
    }
    static PView<T> adj(const mpm_ctx* c, int i) { return slot_view(c, c->adj[i], nullptr); }

    static int copy_state(mpm_ctx* c, const PView<T>& dst, const PView<T>& src)
    {
        hipStream_t st = c->stream;
        if (hipMemcpyAsync(dst.x, src.x, state_bytes(c), hipMemcpyDeviceToDevice, st) != hipSuccess ||
            hipMemcpyAsync(dst.pid, src.pid, sizeof(int32_t) * c->cap, hipMemcpyDeviceToDevice, st) != hipSuccess)
            return S::launch_err(c, "state copy");
        return MPM_OK;
    }

    // The grid-tape record of step i of the segment in tape slot q.
    static typename S::StepBufs rec_bufs(const mpm_ctx* c, int q, int i)
    {
        char* r = c->gtape + ((size_t)q * (size_t)c->ckpt_every + (size_t)i) * c->grec.bytes;
        return {(int32_t*)(r + c->grec.perm), (int32_t*)(r + c->grec.tile_slot), (ActiveTile*)(r + c->grec.active),
                (int32_t*)(r + c->grec.meta), (T*)(r + c->grec.gv), (T*)(r + c->grec.gmass),
                (T*)(r + c->grec.gvt), c->xfer == XF_FLIP ? (T*)(r + c->grec.gvo) : nullptr};
    }

    // Reverse of one step whose sort and grid are in record rb (written by
    // the segment's forward recomputation): aout holds the adjoint of the
    // step's output state, ain receives that of its input state st_in.  The
    // record's nodal velocity and mass are overwritten by their adjoints (3-D).
    template <int MAT>
    static void adjoint_step(mpm_ctx* c, const Phys<T>& P, const PView<T>& st_in, const PView<T>& aout,
                             const PView<T>& ain, const typename S::StepBufs& rb)
    {
        hipStream_t st = c->stream;
        const Geo& g = c->geo;
        prof_mark(c, -1);
        const bool flip = c->xfer == XF_FLIP;
        auto g2p_adj = [&](auto fl) {
            constexpr bool FL = decltype(fl)::value;
            constexpr int WV = kAdjWaves<MAT>, WF = sizeof(T) == 8 && D == 3 ? 1 : WV;
            auto* kernel = adj_few_tiles(c) ? k_g2p_adj<T, D, MAT, FL, WF> : k_g2p_adj<T, D, MAT, FL, WV>;
            kernel<<<tile_wgs(c, kAdjBlock<D>), kAdjBlock<D>, 0, st>>>(g, P, rb.meta, rb.active, rb.perm, st_in, aout, (const T*)rb.gv,
                                                                      FL ? (const T*)rb.gvo : nullptr, (T*)c->part_grid, (T*)c->mid);
        };
        if (flip) g2p_adj(std::true_type{});
        else g2p_adj(std::false_type{});
        prof_mark(c, MPM_PROF_G2P_ADJ);
        double* amu = c->floor_mu ? c->amu : nullptr;
        NodesAdj2<T> nd{};
        if constexpr (D == 2) {
            nd = {(const T*)c->part_grid, rb.tile_slot, rb.gmass, rb.gvt, rb.gvo, amu};
        } else {
            if (flip)
                k_grid_adj<T, D, true><<<tile_wgs(c, kAdjBlock<D>), kAdjBlock<D>, 0, st>>>(
                    g, P, rb.meta, rb.active, rb.tile_slot, (const T*)c->part_grid, rb.gmass, (const T*)rb.gvt, rb.gv, rb.gvo, amu);
            else
                k_grid_adj<T, D, false><<<tile_wgs(c, kAdjBlock<D>), kAdjBlock<D>, 0, st>>>(
                    g, P, rb.meta, rb.active, rb.tile_slot, (const T*)c->part_grid, rb.gmass, (const T*)rb.gvt, rb.gv, nullptr, amu);
            prof_mark(c, MPM_PROF_GRID_ADJ);
        }
        if (flip)
            k_p2g_adj<T, D, MAT, true><<<tile_wgs(c, kAdjBlock<D>), kAdjBlock<D>, 0, st>>>(
                g, P, rb.meta, rb.active, rb.perm, st_in, (const T*)rb.gv, (const T*)rb.gmass, (const T*)rb.gvo,
                (const T*)c->mid, ain, nd);
        else
            k_p2g_adj<T, D, MAT, false><<<tile_wgs(c, kAdjBlock<D>), kAdjBlock<D>, 0, st>>>(
                g, P, rb.meta, rb.active, rb.perm, st_in, (const T*)rb.gv, (const T*)rb.gmass, nullptr,
                (const T*)c->mid, ain, nd);
        prof_mark(c, MPM_PROF_P2G_ADJ);
    }

    static Boxes boxes(const mpm_ctx* c)
    {
        Boxes b{};
        b.n = c->obs_nbox;
        for (int i = 0; i < b.n; ++i)
            for (int a = 0; a < 3; ++a) {
                b.lo[i][a] = c->box_lo[i][a];
                b.hi[i][a] = c->box_hi[i][a];
            }
        return b;
    }

    // Loss of frame fi on state v; with zb_* non-null also the seeds.
    static void observe(mpm_ctx* c, const PView<T>& v, int fi, const PView<T>* ab)
    {
        hipStream_t st = c->stream;
        long long N = c->N;
        if (c->obs_ntr > 0) {
            k_inverse_pid<0><<<nblocks(N), kBlock, 0, st>>>(v.pid, N, c->inv);
            const T* z = c->obs_lag_field == MPM_FIELD_X ? v.x : v.v;
            T* zb = ab ? (c->obs_lag_field == MPM_FIELD_X ? ab->x : ab->v) : nullptr;
            const T* tgt = (const T*)c->obs_lag_target + (size_t)fi * D * c->obs_ntr;
            const T* msk = c->obs_lag_mask ? (const T*)c->obs_lag_mask + (size_t)fi * c->obs_ntr : nullptr;
            k_lag_obs<T, D><<<nblocks(c->obs_ntr), kBlock, 0, st>>>(z, zb, v.cap, N, c->inv, c->obs_tracer,
                                                                    c->obs_ntr, tgt, msk, ab ? 1 : 0, c->loss);
        }
        if (c->obs_nbox > 0) {
            Boxes bx = boxes(c);
            k_fill<double><<<1, kBlock, 0, st>>>(c->box_sum, kMaxBoxes * 3, 0.0);
            k_fill<int><<<1, kBlock, 0, st>>>(c->box_cnt, kMaxBoxes, 0);
            const T* z = c->obs_eul_field == MPM_FIELD_X ? v.x : v.v;
            k_box_sum<T, D><<<nblocks(N), kBlock, 0, st>>>(bx, v.x, z, v.cap, N, c->box_sum, c->box_cnt);
            const T* tgt = (const T*)c->obs_eul_target + (size_t)fi * D * c->obs_nbox;
            const T* msk = c->obs_eul_mask ? (const T*)c->obs_eul_mask + (size_t)fi * c->obs_nbox : nullptr;
            // the seed pass must not add this frame's loss twice
            double* loss_dst = ab ? c->loss_scratch : c->loss;
            k_box_loss<T, D><<<1, kMaxBoxes, 0, st>>>(c->obs_nbox, c->box_sum, c->box_cnt, tgt, msk, c->box_coef,
                                                      loss_dst);
            if (ab) {
                T* zb = c->obs_eul_field == MPM_FIELD_X ? ab->x : ab->v;
                k_box_seed<T, D><<<nblocks(N), kBlock, 0, st>>>(bx, v.x, zb, v.cap, N, c->box_coef);
            }
        }
    }

    static int frame_index(const mpm_ctx* c, int t)
    {
        for (size_t i = 0; i < c->obs_frames.size(); ++i)
            if (c->obs_frames[i] == t) return (int)i;
        return -1;
    }

    template <int MAT, int XF>
    static int forward_loss_mat(mpm_ctx* c, int n, double dt, double* loss)
    {
        hipStream_t st = c->stream;
        Phys<T> P = make_phys<T>(c, dt);
        Phys<T> Pk = P;
        Pk.keep_grid = 1;
        const int k = c->ckpt_every;
        // the trailing tape_segs segments run directly on the tape (states
        // and grid records), so the backward sweep reverses them without
        // recomputing them
        const int nseg = (n + k - 1) / k;
        const int nt = std::max(1, std::min(c->tape_segs, nseg));
        const int first = nseg - nt, tl = first * k;
        c->taped = 0;
        k_fill<double><<<1, kBlock, 0, st>>>(c->loss, 2, 0.0);
        const int cur0 = c->cur;
        PView<T> now = ckpt(c, 0);   // the state at t
        int rc = copy_state(c, now, view<T>(c, c->cur));
        if (rc) return rc;
        for (int t = 0; t < n; ++t) {
            const int seg = t / k, i = t - seg * k, q = seg - first;
            PView<T> nxt;
            if (t < tl) {
                // off the tape: through the context's two states to the next checkpoint
                if (i + 1 < k) c->cur = 1 - c->cur;
                nxt = i + 1 < k ? view<T>(c, c->cur) : ckpt(c, seg + 1);
                S::template step_views<MAT, XF>(c, P, now, nxt);
            } else {
                nxt = seg_state(c, seg, q, i + 1, n);
                S::template step_views<MAT, XF>(c, Pk, now, nxt, rec_bufs(c, q, i));
            }
            now = nxt;
            int fi = frame_index(c, t + 1);
            if (fi >= 0) observe(c, now, fi, nullptr);
        }
        // the context's state, sort and grid again describe the last step; the
        // state buffer is the one that as many steps off the tape end in
        {
            c->cur = tl % 2 == 0 ? cur0 : 1 - cur0;
            S::match_turn(c, true);
            const int ql = nt - 1, il = n - (nseg - 1) * k;
            rc = copy_state(c, view<T>(c, c->cur), now);
            if (rc) return rc;
            typename S::StepBufs last = rec_bufs(c, ql, il - 1);
            const size_t nn = (size_t)c->geo.NN * sizeof(T);
            rc = hip_check(c, hipMemcpyAsync(c->perm, last.perm, (size_t)c->cap * 4, hipMemcpyDeviceToDevice, st),
                           "sort copy");
            if (!rc) rc = hip_check(c, hipMemcpyAsync(c->gv, last.gv, D * nn, hipMemcpyDeviceToDevice, st), "grid copy");
            if (!rc)
                rc = hip_check(c, hipMemcpyAsync(c->tile_slot, last.tile_slot, (size_t)c->geo.ntiles * 4,
                                                 hipMemcpyDeviceToDevice, st), "grid copy");
            if (!rc && c->cfg.keep_grid)
                rc = hip_check(c, hipMemcpyAsync(c->gmass, last.gmass, nn, hipMemcpyDeviceToDevice, st), "grid copy");
            if (rc) return rc;
        }
        c->taped = nt;
        rc = S::launch_err(c, "forward loss");
        if (rc) return rc;
        double h[2];
        rc = hip_check(c, hipMemcpyAsync(h, c->loss, sizeof(h), hipMemcpyDeviceToHost, st), "loss read");
        if (rc) return rc;
        rc = hip_check(c, hipStreamSynchronize(st), "stream synchronize");
        if (rc) return rc;
        *loss = h[0];
        return MPM_OK;
    }

    template <int MAT, int XF>
    static int backward_mat(mpm_ctx* c, void* grad_v0, void* grad_mu)
    {
        hipStream_t st = c->stream;
        const int n = c->fwd_steps, k = c->ckpt_every;
        Phys<T> P = make_phys<T>(c, c->fwd_dt);
        Phys<T> Pk = P;   // the recomputed steps keep their nodal mass
        Pk.keep_grid = 1;
        int a = 0;   // adjoint buffer holding the adjoint of the later state
        k_fill<T><<<4096, kBlock, 0, st>>>((T*)c->adj[0], (long long)c->nsc * c->cap, T(0));
        long long nfl = c->geo.dim == 3 ? (long long)c->geo.box[0] * c->geo.box[1] : c->geo.box[0];
        k_fill<double><<<std::min<long long>(nblocks(nfl), 4096), kBlock, 0, st>>>(c->amu, nfl, 0.0);
        const int nseg = (n + k - 1) / k;
        // the forward pass left its trailing segments on the tape (once: the
        // reverse steps overwrite the grid records with adjoints); earlier
        // segments are recomputed from their checkpoint into slot 0, which the
        // taped segments have released by then
        const int first = nseg - c->taped;
        c->taped = 0;
        for (int seg = nseg - 1; seg >= 0; --seg) {
            int t0 = seg * k, t1 = std::min(t0 + k, n);
            const bool on_tape = seg >= first;
            const int q = on_tape ? seg - first : 0;
            if (!on_tape) {
                prof_mark(c, -1);
                S::new_keys(c, ckpt(c, seg));
                prof_mark(c, MPM_PROF_SCAN);
                // a segment's last step ends at the next checkpoint: only its
                // sort and grid are needed (but the rollout's end has none)
                for (int t = t0; t < t1; ++t)
                    S::template step_views<MAT, XF>(c, Pk, seg_state(c, seg, 0, t - t0, n), tape(c, 0, t - t0 + 1),
                                                    rec_bufs(c, 0, t - t0), t + 1 < t1 || t1 == n);
            }
            for (int t = t1 - 1; t >= t0; --t) {
                int fi = frame_index(c, t + 1);
                PView<T> aout = adj(c, a), ain = adj(c, 1 - a);
                if (fi >= 0) observe(c, seg_state(c, seg, q, t + 1 - t0, n), fi, &aout);
                adjoint_step<MAT>(c, P, seg_state(c, seg, q, t - t0, n), aout, ain, rec_bufs(c, q, t - t0));
                a = 1 - a;
            }
        }
        // dL/dv0 in pid order (S^0 is checkpoint 0)
        if (grad_v0 && c->N > 0)
            k_read_field<T, D><<<nblocks(c->N), kBlock, 0, st>>>(adj(c, a).v, c->cap, ckpt(c, 0).pid, c->N, D,
                                                                CONV_COPY, 1, (T*)grad_v0);
        if (grad_mu) k_mu_out<T><<<nblocks(nfl), kBlock, 0, st>>>(c->amu, nfl, (T*)grad_mu);
        // the step's key and count arrays again describe the current state
        int rc = S::recompute_keys(c);
        if (rc) return rc;
        rc = S::launch_err(c, "backward");
        if (rc) return rc;
        return hip_check(c, hipStreamSynchronize(st), "stream synchronize");
    }

    static int extract(mpm_ctx* c, void* lag_q, void* eul_q)
    {
        hipStream_t st = c->stream;
        PView<T> v = view<T>(c, c->cur);
        long long N = c->N;
        if (lag_q && c->obs_ntr > 0) {
            k_inverse_pid<0><<<nblocks(N), kBlock, 0, st>>>(v.pid, N, c->inv);
            const T* z = c->obs_lag_field == MPM_FIELD_X ? v.x : v.v;
            k_lag_extract<T, D><<<nblocks(c->obs_ntr), kBlock, 0, st>>>(z, v.cap, N, c->inv, c->obs_tracer,
                                                                        c->obs_ntr, (T*)lag_q);
        }
        if (eul_q && c->obs_nbox > 0) {
            Boxes bx = boxes(c);
            k_fill<double><<<1, kBlock, 0, st>>>(c->box_sum, kMaxBoxes * 3, 0.0);
            k_fill<int><<<1, kBlock, 0, st>>>(c->box_cnt, kMaxBoxes, 0);
            const T* z = c->obs_eul_field == MPM_FIELD_X ? v.x : v.v;
            k_box_sum<T, D><<<nblocks(N), kBlock, 0, st>>>(bx, v.x, z, v.cap, N, c->box_sum, c->box_cnt);
            k_box_mean<T, D><<<1, kMaxBoxes, 0, st>>>(c->obs_nbox, c->box_sum, c->box_cnt, (T*)eul_q);
        }
        return S::launch_err(c, "extract");
    }

    // the reverse sweep of each transfer
    template <int MAT>
    static int forward_loss_x(mpm_ctx* c, int n, double dt, double* loss)
    {
        switch (c->xfer) {
        case XF_PIC: return forward_loss_mat<MAT, XF_PIC>(c, n, dt, loss);
        case XF_TPIC: return forward_loss_mat<MAT, XF_TPIC>(c, n, dt, loss);
        case XF_FLIP: return forward_loss_mat<MAT, XF_FLIP>(c, n, dt, loss);
        default: return forward_loss_mat<MAT, XF_APIC>(c, n, dt, loss);
        }
    }
    template <int MAT>
    static int backward_x(mpm_ctx* c, void* gv0, void* gmu)
    {
        switch (c->xfer) {
        case XF_PIC: return backward_mat<MAT, XF_PIC>(c, gv0, gmu);
        case XF_TPIC: return backward_mat<MAT, XF_TPIC>(c, gv0, gmu);
        case XF_FLIP: return backward_mat<MAT, XF_FLIP>(c, gv0, gmu);
        default: return backward_mat<MAT, XF_APIC>(c, gv0, gmu);
        }
    }
    static int forward_loss(mpm_ctx* c, int n, double dt, double* loss)
    {
        switch (c->mat) {
        case MAT_FLUID: return forward_loss_x<MAT_FLUID>(c, n, dt, loss);
        case MAT_VFLUID: return forward_loss_x<MAT_VFLUID>(c, n, dt, loss);
        case MAT_JAUMANN: return forward_loss_x<MAT_JAUMANN>(c, n, dt, loss);
        case MAT_SAND: return forward_loss_x<MAT_SAND>(c, n, dt, loss);
        default: return forward_loss_x<MAT_ELASTIC>(c, n, dt, loss);
        }
    }
    static int backward(mpm_ctx* c, void* gv0, void* gmu)
    {
        switch (c->mat) {
        case MAT_FLUID: return backward_x<MAT_FLUID>(c, gv0, gmu);
        case MAT_VFLUID: return backward_x<MAT_VFLUID>(c, gv0, gmu);
        case MAT_JAUMANN: return backward_x<MAT_JAUMANN>(c, gv0, gmu);
        case MAT_SAND: return backward_x<MAT_SAND>(c, gv0, gmu);
        default: return backward_x<MAT_ELASTIC>(c, gv0, gmu);
        }
    }
};

}  // namespace mpm
