// Explicit-explicit multirate stepping of Eq. (1) (Section III-C): the
// torque of the exchange field is the fast partition, everything else (demag,
// DMI, anisotropy, bias) the slow one, and both time scales use the
// three-stage third-order method of Knoth and Wolke in its multirate
// infinitesimal step form.
//
// Per step and slow stage i = 1..3 the slow torque S_i = R(Y_i, H_eff - H_exch)
// is evaluated once (one FFT convolution); the forcing of the following fast
// interval, r_i = sum_j w_ij S_j, is formed in the same kernel.  The fast ODE
// dv/dtau = R(v, H_exch(v)) + r_i is then advanced in equal substeps, each the
// three stages of the method in Williamson's two-register form
//   q <- A_k q + h F(v),  v <- v + B_k q,
// A = (0, -5/9, -153/128), B = (1/3, 15/16, 8/15).  On thin grids one kernel
// advances a whole substep (mri_substep); otherwise a fast stage is one stencil
// kernel over the grid, and the last one of an interval optionally renormalises
// and performs the forward x pass of the next slow evaluation.
#include "cell_ops.hpp"

namespace magx {

// Slow stage: inverse x pass of the convolution output + slow local terms +
// torque; r = wa*Sa + wb*Sb + wn*S (Sa, Sb earlier slow torques or null).
// V: 0 with a magnetisation profile, 1 without.
template <typename R, int ORD, int LN, int V>
__global__ void __launch_bounds__(kNT) mri_slow_kernel(const cx<R>* __restrict__ Y1, const R* __restrict__ y,
                                                       PG g, Phys<R> ph, int has_demag, R* __restrict__ S_out,
                                                       const R* __restrict__ Sa, const R* __restrict__ Sb, R wa,
                                                       R wb, R wn, R* __restrict__ r_out) {
    pg_fix<LN>(g);
    const bool stream = stream_of<ORD>(g);
    extern __shared__ unsigned char smem_raw[];
    cx<R>* buf = reinterpret_cast<cx<R>*>(smem_raw);
    const int lb = xcd_logical_block(blockIdx.x, gridDim.x);
    const int mb = lb / g.bpm;
    int pen0, npen;
    block_pencils(g, lb - mb * g.bpm, pen0, npen);
    const long long mo = (long long)mb * 3 * g.N;
    y += mo;
    r_out += mo;
    if (S_out) S_out += mo;
    if (Sa) Sa += mo;
    if (Sb) Sb += mo;
    if constexpr (V > 0) ph.msp = nullptr;
    R hbv[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) hbv[c] = ph.hbm ? ph.hbm[mb * 3 + c] : ph.hb[c];
    const bool vec = (g.nx & 1) == 0;
    if (has_demag) c2r_lines<R, ORD, LN>(buf, Y1, g, mb, pen0, npen);
    for (int e = threadIdx.x; e < slots_of<LN>(g, npen); e += kNT) {
        int p, n;
        slot_of<LN>(g, e, p, n);
        const int x0 = 2 * n;
        if (x0 >= g.nx) continue;
        const bool two = x0 + 1 < g.nx;
        int yy, z;
        pen_coords<R>(g, pen0 + p, yy, z);
        const long long id = ((long long)z * g.ny + yy) * g.nx + x0;
        R m[2][3], H[2][3], S[2][3], r[2][3], sw[2] = {(R)1, (R)1};
        if constexpr (V > 0) {
            Stencil<R> t;
            local_field_plain<R>(t, y, g, x0, yy, z, (unsigned)id * (unsigned)sizeof(R), vec, two, ph, H);
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int c = 0; c < 3; ++c) m[q][c] = t.m[q][c];
        } else {
            R ex[2], dm[2], an[2];
            local_field_pair<R>(y, g, x0, yy, z, vec, two, ph, m, H, ex, dm, an, false, sw);
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            // with a profile: no field outside the magnet
            const R inside = (!ph.msp || sw[q] > (R)0) ? (R)1 : (R)0;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                if (has_demag) H[q][c] += inside * demag_at<R>(buf, 3 * p + c, g.Lh, n, q);
                if (ph.terms & MAGX_ZEEMAN) H[q][c] += inside * hbv[c];
            }
            llg_rhs<R>(m[q], H[q], ph.a, ph.alpha, S[q]);
#pragma unroll
            for (int c = 0; c < 3; ++c) r[q][c] = wn * S[q][c];
        }
        if (Sa) {
            R a0[3], a1[3];
            load_pair(Sa, g.N, id, vec, two, a0, a1);
#pragma unroll
            for (int c = 0; c < 3; ++c) { r[0][c] += wa * a0[c]; r[1][c] += wa * a1[c]; }
        }
        if (Sb) {
            R b0[3], b1[3];
            load_pair(Sb, g.N, id, vec, two, b0, b1);
#pragma unroll
            for (int c = 0; c < 3; ++c) { r[0][c] += wb * b0[c]; r[1][c] += wb * b1[c]; }
        }
        if (S_out) store_pair(S_out, g.N, id, vec, two, S[0], S[1], stream);
        store_pair(r_out, g.N, id, vec, two, r[0], r[1], stream);
    }
}

// One fast stage: F = R(v, H_exch(v)) + r; q <- Ak q + h F (q not read when
// first); v_out = v + Bk q, renormalised if norm; r2c of v_out into X1 if fwd.
template <typename R, int ORD, int LN>
__global__ void __launch_bounds__(kNT) mri_fast_kernel(const R* __restrict__ v, R* __restrict__ vout,
                                                       R* __restrict__ qbuf, const R* __restrict__ rbuf, PG g,
                                                       Phys<R> ph, R Ak, R Bk, R h, int first, int norm, int fwd,
                                                       cx<R>* __restrict__ X1) {
    pg_fix<LN>(g);
    const bool stream = stream_of<ORD>(g);
    extern __shared__ unsigned char smem_raw[];
    cx<R>* buf = reinterpret_cast<cx<R>*>(smem_raw);
    const int lb = xcd_logical_block(blockIdx.x, gridDim.x);
    const int mb = lb / g.bpm;
    int pen0, npen;
    block_pencils(g, lb - mb * g.bpm, pen0, npen);
    const long long mo = (long long)mb * 3 * g.N;
    v += mo;
    vout += mo;
    qbuf += mo;
    rbuf += mo;
    const bool vec = (g.nx & 1) == 0;
    // v_out also goes into this thread's LDS line entries for the forward x pass
    // one slot (cell pair) per iteration; kept rolled to keep the kernel small
#pragma unroll 1
    for (int i = 0; i < maxslot<ORD>(); ++i) {
        const int e = threadIdx.x + i * kNT;
        if (e >= slots_of<LN>(g, npen)) continue;
        int p, n;
        slot_of<LN>(g, e, p, n);
        const int x0 = 2 * n;
        if (x0 >= g.nx) {
            if (fwd) {
#pragma unroll
                for (int c = 0; c < 3; ++c) buf[(3 * p + c) * g.Lh + n] = mk<R>((R)0, (R)0);
            }
            continue;
        }
        const bool two = x0 + 1 < g.nx;
        int yy, z;
        pen_coords<R>(g, pen0 + p, yy, z);
        const long long id = ((long long)z * g.ny + yy) * g.nx + x0;
        R m[2][3], H[2][3], ex[2], dm[2], an[2], r[2][3], q[2][3], k[2][3], xn[2][3], sw[2];
        local_field_pair<R>(v, g, x0, yy, z, vec, two, ph, m, H, ex, dm, an, false, sw);
        load_pair(rbuf, g.N, id, vec, two, r[0], r[1]);
        if (!first) load_pair(qbuf, g.N, id, vec, two, q[0], q[1]);
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            llg_rhs<R>(m[s], H[s], ph.a, ph.alpha, k[s]);
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const R F = k[s][c] + r[s][c];
                q[s][c] = first ? h * F : Ak * q[s][c] + h * F;
                xn[s][c] = m[s][c] + Bk * q[s][c];
            }
            if (norm) {
                const R nr = sqrt(dot3(xn[s], xn[s]));
                if (nr > (R)0) {
                    const R inv = (R)1 / nr;
#pragma unroll
                    for (int c = 0; c < 3; ++c) xn[s][c] *= inv;
                }
            }
        }
        store_pair(qbuf, g.N, id, vec, two, q[0], q[1], stream);
        store_pair(vout, g.N, id, vec, two, xn[0], xn[1], stream);
        if (fwd) {
            // demag source of the next slow stage: Ms(r) m = Ms s m
#pragma unroll
            for (int c = 0; c < 3; ++c)
                buf[(3 * p + c) * g.Lh + n] = mk<R>(sw[0] * xn[0][c], two ? sw[1] * xn[1][c] : (R)0);
        }
    }
    if (!fwd) return;
    r2c_lines<R, ORD, LN>(buf, X1, g, mb, pen0, npen);
}

// One fast substep, all three stages, on thin grids (nz <= NZM): a block loads a
// 32 x 16 column tile of v (every z) with a halo of three cells in x and y and
// advances it three stages in LDS and registers, each stage one cell narrower,
// so 26 x 10 columns come out whole.  A thread owns one column: its v, q and r
// stay in registers for all z, and only the x and y neighbours go through LDS.
// The method's first coefficient A is 0, so q never leaves the kernel.  Per
// substep and cell it moves 36 bytes of its own fields (v, r, v'; single
// precision) and the halo, which neighbouring blocks find in L2, where the
// stage kernels move 168, and it is one launch instead of three; the halo costs
// 1.5 times the arithmetic.  At 640x160x4 in single precision three stage
// kernels took 33 us and a substep takes 10.7 us (12 substeps and 3 forward x
// passes in place of 36 stages: 545 -> 310 us a step).
constexpr int kSubX = 32, kSubY = 16, kSubH = 3;

template <typename R, int NZM>
__global__ void __launch_bounds__(kSubX* kSubY)
    mri_substep_kernel(const R* __restrict__ v, R* __restrict__ vout, const R* __restrict__ r, int nx, int ny, int nz,
                       int ntx, int tiles, Phys<R> ph, R A1, R A2, R B0, R B1, R B2, R h, int norm) {
    __shared__ R sv[3][NZM][kSubY][kSubX];
    const int lb = xcd_logical_block(blockIdx.x, gridDim.x);
    const int mb = lb / tiles, tile = lb - mb * tiles;
    const int ty = tile / ntx, tx = tile - ty * ntx;
    const int lx = threadIdx.x & (kSubX - 1), ly = threadIdx.x / kSubX;
    const int x = tx * (kSubX - 2 * kSubH) - kSubH + lx, y = ty * (kSubY - 2 * kSubH) - kSubH + ly;
    const bool in = x >= 0 && x < nx && y >= 0 && y < ny;
    const int plane = nx * ny;
    const long long N = (long long)plane * nz;
    const long long col = (long long)mb * 3 * N + (in ? y * nx + x : 0);
    R V[NZM][3], q[NZM][3], rr[NZM][3];
#pragma unroll
    for (int z = 0; z < NZM; ++z)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const long long o = col + c * N + (long long)min(z, nz - 1) * plane;
            V[z][c] = v[o];
            rr[z][c] = r[o];
        }
    const R kdx = ph.kap * ph.dx, kdy = ph.kap * ph.dy;
    const bool exch = (ph.terms & MAGX_EXCH) != 0;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const R Ak = k == 1 ? A1 : A2, Bk = k == 0 ? B0 : (k == 1 ? B1 : B2);
#pragma unroll
        for (int z = 0; z < NZM; ++z)
            if (z < nz) {
#pragma unroll
                for (int c = 0; c < 3; ++c) sv[c][z][ly][lx] = V[z][c];
            }
        __syncthreads();
        // stage k is complete on the columns at least k + 1 cells inside the tile.
        // Columns beyond the grid in x compute along (nothing reads their values):
        // double-precision arithmetic of a wave with few active lanes ran at about
        // half speed (4x20x6 25 -> 14 us a substep, 27x20x6 25 -> 15, 30x20x6 18 -> 15,
        // 26x20x6 14 either way; single precision 4x20x6 11.7 -> 10.6).
        if (y >= 0 && y < ny && lx > k && lx < kSubX - 1 - k && ly > k && ly < kSubY - 1 - k) {
            R below[3];
#pragma unroll
            for (int z = 0; z < NZM; ++z) {
                if (z >= nz) break;
                const R m[3] = {V[z][0], V[z][1], V[z][2]};
                R H[3] = {(R)0, (R)0, (R)0};
                if (exch) {
                    R xp[3], xm[3], yp[3], ym[3];
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        xp[c] = sv[c][z][ly][lx + 1];
                        xm[c] = sv[c][z][ly][lx - 1];
                        yp[c] = sv[c][z][ly + 1][lx];
                        ym[c] = sv[c][z][ly - 1][lx];
                    }
                    if (x + 1 >= nx) ghost_xp<R>(m, kdx, xp);
                    if (x == 0) ghost_xm<R>(m, kdx, xm);
                    if (y + 1 >= ny) ghost_yp<R>(m, kdy, yp);
                    if (y == 0) ghost_ym<R>(m, kdy, ym);
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        const R m2 = (R)2 * m[c];
                        const R zp = z + 1 < nz ? V[z + 1 < NZM ? z + 1 : z][c] : m[c];
                        const R zm = z > 0 ? below[c] : m[c];
                        H[c] = ph.cex * ((xp[c] - m2 + xm[c]) * ph.idx2 + (yp[c] - m2 + ym[c]) * ph.idy2 +
                                         (zp - m2 + zm) * ph.idz2);
                    }
                }
                R kk[3];
                llg_rhs<R>(m, H, ph.a, ph.alpha, kk);
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    const R F = kk[c] + rr[z][c];
                    q[z][c] = k == 0 ? h * F : Ak * q[z][c] + h * F;
                    below[c] = m[c];
                    V[z][c] = m[c] + Bk * q[z][c];
                }
            }
        }
        __syncthreads();   // the tile is rewritten by the next stage
    }
    if (!in || lx < kSubH || lx >= kSubX - kSubH || ly < kSubH || ly >= kSubY - kSubH) return;
#pragma unroll
    for (int z = 0; z < NZM; ++z) {
        if (z >= nz) break;
        R s = (R)1;
        if (norm) {
            const R nr = sqrt(dot3(V[z], V[z]));
            if (nr > (R)0) s = (R)1 / nr;
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) vout[col + c * N + (long long)z * plane] = s * V[z][c];
    }
}

// lines with an odd factor are compile-time lengths, the others runtime ones
static int odd_line(const Plan& pl) { return odd_part(pl.Lh) > 1 ? pl.Lh : 0; }
#define MAGX_LINE_LAUNCH(KERNEL, VV, LINE, ...)                                                                    \
    do {                                                                                                           \
        const dim3 grid_((unsigned)pl.pencil_blocks), block_(kNT);                                                 \
        if (pl.col) {                                                                                              \
            switch (LINE) {                                                                                        \
                MAGX_ODD_LINES(kColumns, KERNEL, VV, lds, __VA_ARGS__)                                             \
                default:                                                                                           \
                    hipLaunchKernelGGL((KERNEL<R, kColumns, 0 MAGX_UNWRAP VV>), grid_, block_, lds, s, __VA_ARGS__); \
            }                                                                                                      \
            break;                                                                                                 \
        }                                                                                                          \
        switch (LINE) {                                                                                            \
            MAGX_ODD_LINES(kRows, KERNEL, VV, lds, __VA_ARGS__)                                                    \
            default:                                                                                               \
                if constexpr (sizeof(R) == 4) {                                                                    \
                    if (pencil_big(pl)) {                                                                          \
                        hipLaunchKernelGGL((KERNEL<R, kBigRows, 0 MAGX_UNWRAP VV>), grid_, block_, lds, s,         \
                                           __VA_ARGS__);                                                           \
                        break;                                                                                     \
                    }                                                                                              \
                }                                                                                                  \
                hipLaunchKernelGGL((KERNEL<R, kRows, 0 MAGX_UNWRAP VV>), grid_, block_, lds, s, __VA_ARGS__);      \
        }                                                                                                          \
    } while (0)

template <typename R>
hipError_t launch_mri_slow(const Plan& pl, const Phys<R>& ph, const void* Y1, const R* y, int has_demag, R* S_out,
                           const R* Sa, const R* Sb, R wa, R wb, R wn, R* r_out, hipStream_t s) {
    const PG g = make_pg(pl);
    const size_t lds = has_demag ? pencil_lds(pl) : 0;
    const cx<R>* Y = static_cast<const cx<R>*>(Y1);
    if (ph.msp)
        MAGX_LINE_LAUNCH(mri_slow_kernel, (, 0), odd_line(pl), Y, y, g, ph, has_demag, S_out, Sa, Sb, wa, wb, wn, r_out);
    else
        MAGX_LINE_LAUNCH(mri_slow_kernel, (, 1), odd_line(pl), Y, y, g, ph, has_demag, S_out, Sa, Sb, wa, wb, wn, r_out);
    return hipGetLastError();
}

template <typename R>
hipError_t launch_mri_fast(const Plan& pl, const Phys<R>& ph, const R* v, R* vout, R* q, const R* r, R Ak, R Bk,
                           R h, int first, int norm, void* X1, hipStream_t s) {
    const PG g = make_pg(pl);
    const int fwd = X1 != nullptr;
    const size_t lds = fwd ? pencil_lds(pl) : 0;
    MAGX_LINE_LAUNCH(mri_fast_kernel, (), odd_line(pl), v, vout, q, r, g, ph, Ak, Bk, h, first, norm, fwd, static_cast<cx<R>*>(X1));
    return hipGetLastError();
}

// One substep of three stages (A[0] = 0): grids of at most mri_substep_planes
// planes without a profile; hipErrorNotSupported otherwise.
template <typename R>
hipError_t launch_mri_substep(const Plan& pl, const Phys<R>& ph, const R* v, R* vout, const R* r, const double A[3],
                              const double B[3], R h, int norm, hipStream_t s) {
    if (pl.nz > mri_substep_planes<R>() || ph.msp || A[0] != 0.0 || v == vout) return hipErrorNotSupported;
    const int ntx = (pl.nx + kSubX - 2 * kSubH - 1) / (kSubX - 2 * kSubH);
    const int nty = (pl.ny + kSubY - 2 * kSubH - 1) / (kSubY - 2 * kSubH);
    const dim3 grid((unsigned)(ntx * nty * pl.nbatch)), block(kSubX * kSubY);
#define MAGX_SUBSTEP(NZM)                                                                                        \
    hipLaunchKernelGGL((mri_substep_kernel<R, NZM>), grid, block, 0, s, v, vout, r, pl.nx, pl.ny, pl.nz, ntx,    \
                       ntx * nty, ph, (R)A[1], (R)A[2], (R)B[0], (R)B[1], (R)B[2], h, norm)
    if (pl.nz == 1) MAGX_SUBSTEP(1);
    else if (pl.nz == 2) MAGX_SUBSTEP(2);
    else if (pl.nz <= 4) MAGX_SUBSTEP(4);
    else MAGX_SUBSTEP((sizeof(R) == 4 ? 8 : 6));
#undef MAGX_SUBSTEP
    return hipGetLastError();
}

template hipError_t launch_mri_substep<float>(const Plan&, const Phys<float>&, const float*, float*, const float*,
                                              const double*, const double*, float, int, hipStream_t);
template hipError_t launch_mri_substep<double>(const Plan&, const Phys<double>&, const double*, double*, const double*,
                                               const double*, const double*, double, int, hipStream_t);
template hipError_t launch_mri_slow<float>(const Plan&, const Phys<float>&, const void*, const float*, int, float*,
                                           const float*, const float*, float, float, float, float*, hipStream_t);
template hipError_t launch_mri_slow<double>(const Plan&, const Phys<double>&, const void*, const double*, int,
                                            double*, const double*, const double*, double, double, double, double*,
                                            hipStream_t);
template hipError_t launch_mri_fast<float>(const Plan&, const Phys<float>&, const float*, float*, float*,
                                           const float*, float, float, float, int, int, void*, hipStream_t);
template hipError_t launch_mri_fast<double>(const Plan&, const Phys<double>&, const double*, double*, double*,
                                            const double*, double, double, double, int, int, void*, hipStream_t);

MAGX_TW_INIT(init_tw_mri)

}  // namespace magx
