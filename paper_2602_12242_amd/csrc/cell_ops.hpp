// Device helpers shared by the x-pass kernels and the multirate kernels:
// cell-pair accesses, the local field terms with the boundary ghost rule,
// the LLG torque and its transpose, and the x-line transforms in LDS.
//
// Boundary condition (Eq. (10) with the outward normal n): one ghost per face,
// m_ghost = m_b + h (-D/2A) (e_z x n) x m_b, shared by the exchange and DMI
// stencils; on z faces and without DMI it is plain zero-flux Neumann.
#pragma once

#include "magx_internal.hpp"

namespace magx {

// ORD: order of X1/Y1 and register budget of a pencil kernel.  kRows and kColumns
// hold 16 FFT elements and 4 cell-pair slots per thread (np * Lh <= 1024, every
// grid with nx <= 1024); kBigRows holds 32 and 8 (nx up to 2048, float only).
// kColumns is the order of the column convolution (see x_row); it is a constant
// of the kernel because an order chosen at run time cost the small row-order
// grids 4 % (10 RK4 steps at 128x32x1 in double precision 577 -> 600 us).
constexpr int kRows = 0, kBigRows = 1, kColumns = 2;
template <int ORD> constexpr int pemax() { return ORD == kBigRows ? 32 : 16; }
template <int ORD> constexpr int maxslot() { return ORD == kBigRows ? 8 : 4; }

struct PG {
    int nx, ny, nz, Lh, lgLh, Hx, Sx, lgPx, np, npen_total;   // npen_total: pencils of one member
    // log2 of the cell-pair slots per line (of their power-of-two factor, see
    // slot_of), max(Lh/2, 1): the cells fill the lower half of a packed line
    // (x < nx <= Px/2); the upper half is the zero padding, which the forward
    // pass never reads and nothing writes
    int lgLq;
    int bpm;                                                 // blocks per member
    int zmajor;                                              // block order: z fastest (see block_pencils)
    int ks;                                                  // column order of X1: stride of four kx
    int stream;                                              // streaming cell-pair stores (see store_pair;
                                                             // kernels read it once, as stream_of)
    long long N;                                             // cells of one member
    FastDiv div_ny, div_hx;                                  // n / ny and n / Hx
};

// LDS bytes of a pencil block (3 np lines of Lh complex values) and its register budget
inline size_t pencil_lds(const Plan& pl) { return (size_t)3 * pl.np * pl.Lh * pl.esize * 2; }
inline bool pencil_big(const Plan& pl) { return pl.np * pl.Lh > 1024; }

// Compile-time line geometry: the kernels are instantiated with the transform
// length LN = Lh (a multiple of 16, so Hx = LN + 1, Sx = LN + 16) as a constant
// for the lengths with an odd factor, and for the power-of-two lines 128 ... 1024
// of grids with nx = Lh, where nx is a constant too; that turns the FFT strides
// and row offsets into immediates.  LN = 0 keeps runtime values (powers of two).
constexpr bool pencil_exact(int LN) { return LN > 0 && odd_part(LN) == 1; }

inline int pencil_line(const Plan& pl) {
    if (pl.np * pl.Lh > 1024) return 0;
    if (odd_part(pl.Lh) > 1) return pl.Lh;
    return pl.nx == pl.Lh && pl.Lh >= 128 && pl.Lh <= 1024 ? pl.Lh : 0;
}

template <int LN>
__device__ __forceinline__ void pg_fix(PG& g) {
    if constexpr (LN > 0) {
        constexpr int lg = ilog2c(LN / odd_part(LN));
        g.lgLh = lg;
        g.lgLq = lg - 1;
        g.Lh = LN;
        g.lgPx = lg + 1;
        if (pencil_exact(LN)) g.nx = LN;
        g.Hx = LN + 1;
        g.Sx = LN + 16;
    }
}

// Cases of a launch switch over the line length: the lengths with an odd factor
// (_512: those of at most 512 values).
// VV: further template arguments in parentheses, "()" or "(, value)".
#define MAGX_UNWRAP(...) __VA_ARGS__
#define MAGX_LINE_CASE(ORD, LN, KERNEL, VV, LDS, ...)                                                     \
    case LN:                                                                                              \
        hipLaunchKernelGGL((KERNEL<R, ORD, LN MAGX_UNWRAP VV>), grid_, block_, LDS, s, __VA_ARGS__);      \
        break;
#define MAGX_ODD_LINES_512(ORD, KERNEL, VV, LDS, ...)      \
    MAGX_LINE_CASE(ORD, 80, KERNEL, VV, LDS, __VA_ARGS__)  \
    MAGX_LINE_CASE(ORD, 96, KERNEL, VV, LDS, __VA_ARGS__)  \
    MAGX_LINE_CASE(ORD, 160, KERNEL, VV, LDS, __VA_ARGS__) \
    MAGX_LINE_CASE(ORD, 192, KERNEL, VV, LDS, __VA_ARGS__) \
    MAGX_LINE_CASE(ORD, 320, KERNEL, VV, LDS, __VA_ARGS__) \
    MAGX_LINE_CASE(ORD, 384, KERNEL, VV, LDS, __VA_ARGS__)
#define MAGX_ODD_LINES(ORD, KERNEL, VV, LDS, ...)          \
    MAGX_ODD_LINES_512(ORD, KERNEL, VV, LDS, __VA_ARGS__)  \
    MAGX_LINE_CASE(ORD, 640, KERNEL, VV, LDS, __VA_ARGS__) \
    MAGX_LINE_CASE(ORD, 768, KERNEL, VV, LDS, __VA_ARGS__)

// log2 of the largest radix of a line transform.  Radix 8 in place of 16 costs a
// pass at 256 (4 8 8 in place of 16 16) but spreads over twice the threads: a
// gradient at 256x256x8 7100 -> 6870 us, at 190x75x9 in double precision (lines of
// 192: 8 8 3 in place of 4 16 3) 2610 -> 2567; four RK4 steps at lines of 96 and 160
// (4 8 3 and 4 8 5 in place of 2 16 3 and 2 16 5) in single precision 90x60x1 257 -> 239,
// 150x60x1 264 -> 245, 90x150x7 697 -> 674, 150x150x7 750 -> 724, in double precision up
// to 8 %, equal at 90x300x12 and above; films (128) and 1024-cell lines were 2 and 1 %
// slower with it, 320 and 512 equal.
template <int ORD, int LN> constexpr int line_lgm() {
    return ORD == kBigRows ? 5 : (LN == 256 || LN == 192 || LN == 160 || LN == 96 ? 3 : 4);
}

// Cell-pair slots of npen lines (Lh/2 each) and the line p and pair n of slot e.
template <int LN> constexpr int line_odd() { return LN > 0 ? odd_part(LN) : 1; }
template <int LN> __device__ __forceinline__ int slots_of(const PG& g, int npen) {
    return line_odd<LN>() > 1 ? npen * (LN / 2) : npen << g.lgLq;
}
template <int LN> __device__ __forceinline__ void slot_of(const PG& g, int e, int& p, int& n) {
    if constexpr (line_odd<LN>() > 1) {
        p = (int)((unsigned)e / (unsigned)(LN / 2));
        n = e - p * (LN / 2);
    } else {
        p = e >> g.lgLq;
        n = e & ((1 << g.lgLq) - 1);
    }
}

// The streaming flag of a kernel, read once into a register: the 32-element
// register budget (kBigRows) leaves no room for the second store path, so those
// kernels never stream.
template <int ORD>
__device__ __forceinline__ bool stream_of(const PG& g) {
    return ORD != kBigRows && g.stream != 0;
}

inline PG make_pg(const Plan& pl) {
    PG g;
    g.nx = pl.nx; g.ny = pl.ny; g.nz = pl.nz;
    g.Lh = pl.Lh; g.lgLh = pl.lgLh; g.Hx = pl.Hx; g.Sx = pl.Sx; g.lgPx = pl.lgPx;
    g.lgLq = pl.lgLh > 0 ? pl.lgLh - 1 : 0;
    g.np = pl.np; g.npen_total = pl.ny * pl.nz; g.bpm = pl.blocks_per_member; g.N = pl.ncell;
    g.div_ny = make_fastdiv(pl.ny);
    g.div_hx = make_fastdiv(pl.Hx);
    g.zmajor = pl.pencil_zmajor;
    g.ks = 12 * g.npen_total;
    // fields of 64 MiB and more (a batch counts whole) are far larger than the caches
    g.stream = !pencil_big(pl) && 3.0 * (double)pl.ncell * pl.nbatch * pl.esize >= 64.0 * (1 << 20) ? 1 : 0;
    return g;
}

// Pencils of block lbm of a member: np consecutive rows y of one plane z.
// With zmajor the blocks run through z fastest ((y group, z) -> lbm =
// group * nz + z), so the blocks holding a row's z neighbours run right
// before and after it on the same XCD and the stencil finds them in L2;
// otherwise pencils are numbered z * ny + y and a block takes np of them.
// Either way its pencils are consecutive in the z * ny + y numbering.
__device__ __forceinline__ void block_pencils(const PG& g, int lbm, int& pen0, int& npen) {
    if (g.zmajor) {
        const int grp = lbm / g.nz;
        const int z = lbm - grp * g.nz;
        const int y0 = grp * g.np;
        pen0 = z * g.ny + y0;
        npen = min(g.np, g.ny - y0);
    } else {
        pen0 = lbm * g.np;
        npen = min(g.np, g.npen_total - pen0);
    }
}

template <typename R>
__device__ __forceinline__ void load3(const R* __restrict__ f, long long N, long long id, R v[3]) {
    v[0] = f[id];
    v[1] = f[N + id];
    v[2] = f[2 * N + id];
}

template <typename R>
__device__ __forceinline__ void store3(R* __restrict__ f, long long N, long long id, const R v[3]) {
    f[id] = v[0];
    f[N + id] = v[1];
    f[2 * N + id] = v[2];
}

// ---- cell pairs (2n, 2n+1) along x ------------------------------------------------
// With nx even every pair is complete and 8-byte (float) / 16-byte (double)
// aligned, so a pair is one vector access per component; with nx odd the last
// pair of a row has a single cell and scalar accesses are used.  Fields that a
// pencil kernel writes are read again a whole convolution later at the
// earliest; on grids whose fields are far larger than the caches (PG::stream)
// pairs are stored with streaming stores (see st_stream), and a field read
// once (stream) is loaded the same way.  Measured at 512 x 512 x 32: the
// reverse start kernel 186 -> 178 us, the forward y pass that follows a stage
// 126 -> 122 us; at 256 x 256 x 16, whose fields stay in the caches, the same
// accesses cost 3 % of an RK4 step.
template <typename R>
__device__ __forceinline__ void load_pair(const R* __restrict__ f, long long N, long long id, bool vec, bool two,
                                          R a[3], R b[3], bool stream = false) {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const R* p = f + c * N + id;
        if (vec) {
            const cx<R> v = stream ? ld_stream<R>(reinterpret_cast<const cx<R>*>(p))
                                   : *reinterpret_cast<const cx<R>*>(p);
            a[c] = v.x;
            b[c] = v.y;
        } else {
            a[c] = p[0];
            const R v1 = p[two ? 1 : 0];   // unconditional load: no wait behind a branch
            b[c] = two ? v1 : (R)0;
        }
    }
}

template <typename R>
__device__ __forceinline__ void store_pair(R* __restrict__ f, long long N, long long id, bool vec, bool two,
                                           const R a[3], const R b[3], bool stream = false) {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        R* p = f + c * N + id;
        if (vec) {
            if (stream) st_stream<R>(reinterpret_cast<cx<R>*>(p), mk<R>(a[c], b[c]));
            else *reinterpret_cast<cx<R>*>(p) = mk<R>(a[c], b[c]);
        } else {
            p[0] = a[c];
            if (two) p[1] = b[c];
        }
    }
}

// Ghost values of the boundary condition (Eq. (10)) for a cell c on a face
// with outward normal -x, +x, -y, +y (kd = -D/(2A) times the cell size; on z
// faces the ghost is c itself).
template <typename R> __device__ __forceinline__ void ghost_xm(const R c[3], R kd, R o[3]) {
    o[0] = c[0] - kd * c[2]; o[1] = c[1]; o[2] = c[2] + kd * c[0];
}
template <typename R> __device__ __forceinline__ void ghost_xp(const R c[3], R kd, R o[3]) {
    o[0] = c[0] + kd * c[2]; o[1] = c[1]; o[2] = c[2] - kd * c[0];
}
template <typename R> __device__ __forceinline__ void ghost_ym(const R c[3], R kd, R o[3]) {
    o[0] = c[0]; o[1] = c[1] - kd * c[2]; o[2] = c[2] + kd * c[1];
}
template <typename R> __device__ __forceinline__ void ghost_yp(const R c[3], R kd, R o[3]) {
    o[0] = c[0]; o[1] = c[1] + kd * c[2]; o[2] = c[2] - kd * c[1];
}

template <typename R>
__device__ __forceinline__ void load_s_pair(const R* __restrict__ s, long long id, bool vec, bool two, R o[2]) {
    if (vec) {
        const cx<R> v = *reinterpret_cast<const cx<R>*>(s + id);
        o[0] = v.x;
        o[1] = v.y;
    } else {
        o[0] = s[id];
        const R v1 = s[id + (two ? 1 : 0)];
        o[1] = two ? v1 : (R)0;
    }
}

// Exchange + DMI + anisotropy of the linear field f for the pair of cells
// (x0 = 2n, x0 + 1) of row (y, z); h*[0] belongs to cell x0, h*[1] to x0 + 1.
// A neighbour outside the grid, or (with a magnetisation profile ph.msp)
// outside the magnet, is replaced by the ghost of the boundary condition built
// from the cell itself.  With a profile the local prefactors are divided by the
// cell's s = Ms(r)/Ms and cells with s = 0 get no field; sw returns s of the
// two cells (1 without a profile).
template <typename R>
__device__ __forceinline__ void local_field_pair(const R* __restrict__ f, const PG& g, int x0, int y, int z,
                                                 bool vec, bool two, const Phys<R>& ph, R m[2][3], R h[2][3],
                                                 R hex_dot[2], R hdmi_dot[2], R hani_dot[2], bool want_parts,
                                                 R sw[2]) {
    const long long N = g.N;
    const long long id = ((long long)z * g.ny + y) * g.nx + x0;
    const R* __restrict__ sp = ph.msp;
    load_pair(f, N, id, vec, two, m[0], m[1]);
    sw[0] = sw[1] = (R)1;
    if (sp) load_s_pair(sp, id, vec, two, sw);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
#pragma unroll
        for (int c = 0; c < 3; ++c) h[q][c] = (R)0;
        hex_dot[q] = hdmi_dot[q] = hani_dot[q] = (R)0;
    }
    if (ph.terms & (MAGX_EXCH | MAGX_DMI)) {
        const R kdx = ph.kap * ph.dx, kdy = ph.kap * ph.dy;
        R xl[3], xr[3], yp[2][3], ym[2][3], zp[2][3], zm[2][3];
        // Neighbour availability: in the grid and (with a profile) in the
        // magnet.  Every neighbour is loaded, at the cell itself where it lies
        // outside the grid (so the address is valid), and replaced by its ghost
        // value afterwards: no load sits behind a branch, so all of them are in
        // flight together.
        const int xr_off = two ? 2 : 1;
        const long long pz = (long long)g.nx * g.ny;
        const bool gxl = x0 > 0, gxr = x0 + xr_off < g.nx;
        const bool gyp = y + 1 < g.ny, gym = y > 0, gzp = z + 1 < g.nz, gzm = z > 0;
        const long long il = gxl ? id - 1 : id, ir = gxr ? id + xr_off : id;
        const long long iyp = gyp ? id + g.nx : id, iym = gym ? id - g.nx : id;
        const long long izp = gzp ? id + pz : id, izm = gzm ? id - pz : id;
        R xlv[3], xrv[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            xlv[c] = f[c * N + il];
            xrv[c] = f[c * N + ir];
        }
        load_pair(f, N, iyp, vec, two, yp[0], yp[1]);
        load_pair(f, N, iym, vec, two, ym[0], ym[1]);
        load_pair(f, N, izp, vec, two, zp[0], zp[1]);
        load_pair(f, N, izm, vec, two, zm[0], zm[1]);
        bool okxl = gxl, okxr = gxr;
        bool okyp[2], okym[2], okzp[2], okzm[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            okyp[q] = gyp;
            okym[q] = gym;
            okzp[q] = gzp;
            okzm[q] = gzm;
        }
        if (sp) {
            const R sl = sp[il], sr = sp[ir];
            R t0[2], t1[2], t2[2], t3[2];
            load_s_pair(sp, iyp, vec, two, t0);
            load_s_pair(sp, iym, vec, two, t1);
            load_s_pair(sp, izp, vec, two, t2);
            load_s_pair(sp, izm, vec, two, t3);
            okxl = okxl && sl > (R)0;
            okxr = okxr && sr > (R)0;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                okyp[q] = okyp[q] && t0[q] > (R)0;
                okym[q] = okym[q] && t1[q] > (R)0;
                okzp[q] = okzp[q] && t2[q] > (R)0;
                okzm[q] = okzm[q] && t3[q] > (R)0;
            }
        }
        // outer x neighbours of the pair: cell x0 - 1 and cell x0 + 2 (or x0 + 1 if alone)
        R last[3], gl[3], gr[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) last[c] = two ? m[1][c] : m[0][c];
        ghost_xm<R>(m[0], kdx, gl);
        ghost_xp<R>(last, kdx, gr);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            xl[c] = okxl ? xlv[c] : gl[c];
            xr[c] = okxr ? xrv[c] : gr[c];
        }
        // the two cells of the pair see each other unless one is outside the magnet
        const bool in0 = sw[0] > (R)0, in1 = sw[1] > (R)0;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const R* mc = m[q];
            R xp[3], xm[3], ypq[3], ymq[3], zpq[3], zmq[3];
            if (q == 0) {
#pragma unroll
                for (int c = 0; c < 3; ++c) xm[c] = xl[c];
                if (!two) {
#pragma unroll
                    for (int c = 0; c < 3; ++c) xp[c] = xr[c];
                } else if (in1) {
#pragma unroll
                    for (int c = 0; c < 3; ++c) xp[c] = m[1][c];
                } else {
                    ghost_xp<R>(m[0], kdx, xp);
                }
            } else {
#pragma unroll
                for (int c = 0; c < 3; ++c) xp[c] = xr[c];
                if (in0) {
#pragma unroll
                    for (int c = 0; c < 3; ++c) xm[c] = m[0][c];
                } else {
                    ghost_xm<R>(m[1], kdx, xm);
                }
            }
            if (okyp[q]) { ypq[0] = yp[q][0]; ypq[1] = yp[q][1]; ypq[2] = yp[q][2]; }
            else ghost_yp<R>(mc, kdy, ypq);
            if (okym[q]) { ymq[0] = ym[q][0]; ymq[1] = ym[q][1]; ymq[2] = ym[q][2]; }
            else ghost_ym<R>(mc, kdy, ymq);
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                zpq[c] = okzp[q] ? zp[q][c] : mc[c];
                zmq[c] = okzm[q] ? zm[q][c] : mc[c];
            }
            R hx[3] = {(R)0, (R)0, (R)0}, hd[3] = {(R)0, (R)0, (R)0};
            if (ph.terms & MAGX_EXCH) {
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    const R m2 = (R)2 * mc[c];
                    hx[c] = ph.cex * ((xp[c] - m2 + xm[c]) * ph.idx2 + (ypq[c] - m2 + ymq[c]) * ph.idy2 +
                                      (zpq[c] - m2 + zmq[c]) * ph.idz2);
                }
            }
            if (ph.terms & MAGX_DMI) {
                hd[0] = ph.cdmi * (xp[2] - xm[2]) * ph.h2x;
                hd[1] = ph.cdmi * (ypq[2] - ymq[2]) * ph.h2y;
                hd[2] = -ph.cdmi * ((xp[0] - xm[0]) * ph.h2x + (ypq[1] - ymq[1]) * ph.h2y);
            }
            if (sp) {
                const R inv = sw[q] > (R)0 ? (R)1 / sw[q] : (R)0;
#pragma unroll
                for (int c = 0; c < 3; ++c) { hx[c] *= inv; hd[c] *= inv; }
            }
#pragma unroll
            for (int c = 0; c < 3; ++c) h[q][c] = hx[c] + hd[c];
            if (want_parts) {
                hex_dot[q] = mc[0] * hx[0] + mc[1] * hx[1] + mc[2] * hx[2];
                hdmi_dot[q] = mc[0] * hd[0] + mc[1] * hd[1] + mc[2] * hd[2];
            }
        }
    }
    if (ph.terms & MAGX_ANIS) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const R pr = m[q][0] * ph.eK[0] + m[q][1] * ph.eK[1] + m[q][2] * ph.eK[2];
            R ca = ph.cani;
            if (sp) ca = sw[q] > (R)0 ? ca / sw[q] : (R)0;
#pragma unroll
            for (int c = 0; c < 3; ++c) h[q][c] += ca * pr * ph.eK[c];
            if (want_parts) hani_dot[q] = ca * pr * pr;
        }
    }
}

// The same without a magnetisation profile, for the cell pair at element id =
// pen nx + x0 of row pen = z ny + y.  Accesses are a uniform base per component
// plus one 32-bit byte offset per neighbour (a component of a member is below
// 2^32 bytes: the plan's limits keep N below 2^29 elements), and a neighbour
// outside the grid is loaded at the cell itself, which is its ghost already
// except for the DMI rotation, added on the boundary cells.
template <typename R>
__device__ __forceinline__ void load_pair32(const R* __restrict__ f, long long N, unsigned off, bool vec, bool two,
                                            R a[3], R b[3], bool stream = false) {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const char* p = reinterpret_cast<const char*>(f + c * N);
        if (vec) {
            const cx<R>* q = reinterpret_cast<const cx<R>*>(p + off);
            const cx<R> v = stream ? ld_stream<R>(q) : *q;
            a[c] = v.x;
            b[c] = v.y;
        } else {
            a[c] = *reinterpret_cast<const R*>(p + off);
            const R v1 = *reinterpret_cast<const R*>(p + (off + (two ? (unsigned)sizeof(R) : 0u)));
            b[c] = two ? v1 : (R)0;
        }
    }
}

template <typename R>
__device__ __forceinline__ void store_pair32(R* __restrict__ f, long long N, unsigned off, bool vec, bool two,
                                             const R a[3], const R b[3], bool stream = false) {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        char* p = reinterpret_cast<char*>(f + c * N);
        if (vec) {
            cx<R>* q = reinterpret_cast<cx<R>*>(p + off);
            if (stream) st_stream<R>(q, mk<R>(a[c], b[c]));
            else *q = mk<R>(a[c], b[c]);
        } else {
            R* q = reinterpret_cast<R*>(p + off);
            q[0] = a[c];
            if (two) q[1] = b[c];
        }
    }
}

// The values of the pair and of its neighbours, their loads and the exchange and
// DMI field computed from them (h; both only with an exchange or DMI term).
template <typename R> struct Stencil {
    R m[2][3], xl[3], xr[3], yp[2][3], ym[2][3], zp[2][3], zm[2][3];
};

template <typename R>
__device__ __forceinline__ void neighbours_load(Stencil<R>& t, const R* __restrict__ f, const PG& g, int x0, int y,
                                                int z, unsigned off, bool vec, bool two) {
    constexpr unsigned es = (unsigned)sizeof(R);
    const long long N = g.N;
    const unsigned rowb = (unsigned)g.nx * es, planeb = (unsigned)g.ny * rowb;
    const unsigned ol = x0 > 0 ? off - es : off;
    const unsigned orr = off + ((two ? 1u : 0u) + (x0 + (two ? 2 : 1) < g.nx ? 1u : 0u)) * es;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const char* p = reinterpret_cast<const char*>(f + c * N);
        t.xl[c] = *reinterpret_cast<const R*>(p + ol);
        t.xr[c] = *reinterpret_cast<const R*>(p + orr);
    }
    load_pair32(f, N, y + 1 < g.ny ? off + rowb : off, vec, two, t.yp[0], t.yp[1]);
    load_pair32(f, N, y > 0 ? off - rowb : off, vec, two, t.ym[0], t.ym[1]);
    load_pair32(f, N, z + 1 < g.nz ? off + planeb : off, vec, two, t.zp[0], t.zp[1]);
    load_pair32(f, N, z > 0 ? off - planeb : off, vec, two, t.zm[0], t.zm[1]);
}

template <typename R>
__device__ __forceinline__ void neighbours_field(Stencil<R>& t, const PG& g, int x0, int y, bool two,
                                                 const Phys<R>& ph, R h[2][3]) {
    if (ph.terms & MAGX_DMI) {
        const R kdx = ph.kap * ph.dx, kdy = ph.kap * ph.dy;
        if (x0 == 0) ghost_xm<R>(t.m[0], kdx, t.xl);
        if (x0 + (two ? 2 : 1) >= g.nx) {
            if (two) ghost_xp<R>(t.m[1], kdx, t.xr);
            else ghost_xp<R>(t.m[0], kdx, t.xr);
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            if (y + 1 >= g.ny) ghost_yp<R>(t.m[q], kdy, t.yp[q]);
            if (y == 0) ghost_ym<R>(t.m[q], kdy, t.ym[q]);
        }
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const R* mc = t.m[q];
        R xp[3], xm[3], hx[3] = {(R)0, (R)0, (R)0}, hd[3] = {(R)0, (R)0, (R)0};
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            xm[c] = q == 0 ? t.xl[c] : t.m[0][c];
            xp[c] = q == 1 || !two ? t.xr[c] : t.m[1][c];
        }
        if (ph.terms & MAGX_EXCH) {
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const R m2 = (R)2 * mc[c];
                hx[c] = ph.cex * ((xp[c] - m2 + xm[c]) * ph.idx2 + (t.yp[q][c] - m2 + t.ym[q][c]) * ph.idy2 +
                                  (t.zp[q][c] - m2 + t.zm[q][c]) * ph.idz2);
            }
        }
        if (ph.terms & MAGX_DMI) {
            hd[0] = ph.cdmi * (xp[2] - xm[2]) * ph.h2x;
            hd[1] = ph.cdmi * (t.yp[q][2] - t.ym[q][2]) * ph.h2y;
            hd[2] = -ph.cdmi * ((xp[0] - xm[0]) * ph.h2x + (t.yp[q][1] - t.ym[q][1]) * ph.h2y);
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) h[q][c] = hx[c] + hd[c];
    }
}

// Exchange, DMI and anisotropy field of the pair.  LOADED: t holds the pair and
// its neighbours already (loaded ahead, with stencil_load); otherwise they are
// loaded here, next to their use, which keeps fewer registers live.
template <typename R, bool LOADED = false>
__device__ __forceinline__ void local_field_plain(Stencil<R>& t, const R* __restrict__ f, const PG& g, int x0, int y,
                                                  int z, unsigned off, bool vec, bool two, const Phys<R>& ph,
                                                  R h[2][3]) {
    if constexpr (!LOADED) load_pair32(f, g.N, off, vec, two, t.m[0], t.m[1]);
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int c = 0; c < 3; ++c) h[q][c] = (R)0;
    if (ph.terms & (MAGX_EXCH | MAGX_DMI)) {
        if constexpr (!LOADED) neighbours_load<R>(t, f, g, x0, y, z, off, vec, two);
        neighbours_field<R>(t, g, x0, y, two, ph, h);
    }
    if (ph.terms & MAGX_ANIS) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const R pr = t.m[q][0] * ph.eK[0] + t.m[q][1] * ph.eK[1] + t.m[q][2] * ph.eK[2];
#pragma unroll
            for (int c = 0; c < 3; ++c) h[q][c] += ph.cani * pr * ph.eK[c];
        }
    }
}

template <typename R>
__device__ __forceinline__ void stencil_load(Stencil<R>& t, const R* __restrict__ f, const PG& g, int x0, int y, int z,
                                             unsigned off, bool vec, bool two, unsigned terms) {
    load_pair32(f, g.N, off, vec, two, t.m[0], t.m[1]);
    if (terms & (MAGX_EXCH | MAGX_DMI)) neighbours_load<R>(t, f, g, x0, y, z, off, vec, two);
}

// Non-finite detection (calls made with check_finite): true if any of the
// n values is NaN or infinite; note_nonfinite sets the flag word with one
// atomic from the first lane of every wave that met such a value (called by
// all active lanes of the wave).
template <typename R, int n>
__device__ __forceinline__ bool any_nonfinite(const R* v) {
    bool bad = false;
#pragma unroll
    for (int i = 0; i < n; ++i) bad = bad || !isfinite(v[i]);
    return bad;
}

__device__ __forceinline__ void note_nonfinite(unsigned* flag, bool bad) {
    const unsigned long long b = __ballot(bad);
    if (b != 0ull && __lane_id() == (unsigned)(__ffsll((long long)b) - 1)) atomicOr(flag, 1u);
}

template <typename R>
__device__ __forceinline__ void cross3(const R a[3], const R b[3], R o[3]) {
    o[0] = a[1] * b[2] - a[2] * b[1];
    o[1] = a[2] * b[0] - a[0] * b[2];
    o[2] = a[0] * b[1] - a[1] * b[0];
}

template <typename R> __device__ __forceinline__ R dot3(const R a[3], const R b[3]) {
    return a[0] * b[0] + a[1] * b[1] + a[2] * b[2];
}

// Eq. (1) for unit m: a [m x H + alpha m x (m x H)].
template <typename R>
__device__ __forceinline__ void llg_rhs(const R m[3], const R H[3], R a, R alpha, R k[3]) {
    R mxH[3], mmH[3];
    cross3(m, H, mxH);
    cross3(m, mxH, mmH);
#pragma unroll
    for (int c = 0; c < 3; ++c) k[c] = a * (mxH[c] + alpha * mmH[c]);
}

// Cotangent of H for a cotangent kappa of R(y): a [kappa x y + alpha y x (y x kappa)].
template <typename R>
__device__ __forceinline__ void rhs_mu(const R y[3], const R kap[3], R a, R alpha, R mu[3]) {
    R kxy[3], yxk[3], yyk[3];
    cross3(kap, y, kxy);
    cross3(y, kap, yxk);
    cross3(y, yxk, yyk);
#pragma unroll
    for (int c = 0; c < 3; ++c) mu[c] = a * (kxy[c] + alpha * yyk[c]);
}

// ---- x-line transforms in LDS --------------------------------------------------
// LDS line for (pencil p, component c) starts at (3p + c) * Lh.

template <typename R>
__device__ __forceinline__ void pen_coords(const PG& g, int pen, int& y, int& z) {
    z = fdiv(pen, g.div_ny);
    y = pen - z * g.ny;
}

// Split/merge items per thread and chunk (3 np Lh/2 <= 1536 items per block
// for np Lh <= 1024).
constexpr int kXIt = 6;

// Offset of kx in a row of X1/Y1 (signed: the row order's Lh - t then splits into
// an immediate offset and the thread's address; as an unsigned number it cost the
// 512x512x32 stage 211 -> 216 us and the double-precision field kernel 186 -> 216).
template <int ORD>
__device__ __forceinline__ int col_off(const PG& g, int kx) {
    return ORD == kColumns ? (int)(umul24((unsigned)kx >> 2, (unsigned)g.ks) + ((unsigned)kx & 3u)) : kx;
}

// Row of X1/Y1 holding component c of pencil p (32-bit element offset: the
// spectral arrays of a whole batch stay below 2^31 elements).
// Column order: [kx / 4][y][c][z][kx % 4], the real X[0] and X[Lh] stored together
// at kx = 0.
template <int ORD>
__device__ __forceinline__ unsigned x_row(const PG& g, int mb, int c, int pen) {
    if constexpr (ORD == kColumns) {
        const int z = fdiv(pen, g.div_ny), y = pen - z * g.ny;
        return (unsigned)mb * (unsigned)(g.Lh >> 2) * (unsigned)g.ks + 4u * (unsigned)((y * 3 + c) * g.nz + z);
    }
    return ((unsigned)(mb * 3 + c) * (unsigned)g.npen_total + (unsigned)pen) * (unsigned)g.Sx;
}

// The half-length real-FFT split and merge steps pair bin k with its mirror
// Lh - k: both come from the same two values and the same twiddle
// W^k = exp(-2 pi i k / Px), since W^(Lh-k) = -conj(W^k).  Item t < Lq
// (Lq = max(Lh/2, 1)) of a line takes k = t and Lh - t; t = 0 also takes
// k = Lh/2 (its own mirror).

// Inverse x pass: Y1 rows -> real lines; afterwards the real value of cell x
// of line l is buf[l*Lh + x/2].x (x even) or .y (x odd).  Split step of the
// half-length inverse, Z[k] = (X[k] + X*[Lh-k]) + i (X[k] - X*[Lh-k]) w^-k
// (w^-k = conj(W^k)), into LDS; then the inverse FFT of every line in LDS.
template <typename R, int ORD, int LN>
__device__ void c2r_lines(cx<R>* buf, const cx<R>* Y1, const PG& g, int mb, int pen0, int npen) {
    constexpr int ODD = line_odd<LN>();
    const int Lh = g.Lh;
    const int lgq = g.lgLh > 0 ? g.lgLh - 1 : 0;
    const int twsh = tw_log(ODD) - g.lgPx;
    auto split = [](cx<R> a, cx<R> b, cx<R> wc) {   // a = X[k], b = X[Lh-k], wc = conj(W^k)
        const cx<R> bc = cconj<R>(b);
        const cx<R> A = cadd<R>(a, bc);
        const cx<R> B = cmul<R>(csub<R>(a, bc), wc);
        return mk<R>(A.x - B.y, A.y + B.x);
    };
    tw_lds_fill<R, ODD>();   // pass twiddles, read after the barrier below
    if (ODD == 1 && (1 << lgq) >= kNT) {
        // at least one item per thread and line: thread tid takes items
        // t = tid + k kNT of every line, so its twiddles are the same for all
        // lines and each line's row address is uniform (scalar registers).
        // A chunk holds kXIt items per thread: with one item per line the six
        // lines of a two-pencil block are one chunk and their loads make one
        // round trip (measured at 512-cell lines: stage 224 -> 211 us).
        auto chunks = [&](auto ipl_c) {
            constexpr int IPL = decltype(ipl_c)::value;   // items per thread and line
            constexpr int LC = kXIt / IPL;                // lines per chunk
            cx<R> wc[IPL];
#pragma unroll
            for (int k = 0; k < IPL; ++k) wc[k] = cconj<R>(tw_fwd<R>(((int)threadIdx.x + k * kNT) << twsh));
            const int nl = npen * 3;
            for (int l0 = 0; l0 < nl; l0 += LC) {
                cx<R> A[LC][IPL], B[LC][IPL], C[LC];
#pragma unroll
                for (int i = 0; i < LC; ++i) {
                    const int l = min(l0 + i, nl - 1);
                    const int p = l / 3, c = l - 3 * p;
                    const cx<R>* row = Y1 + x_row<ORD>(g, mb, c, pen0 + p);
#pragma unroll
                    for (int k = 0; k < IPL; ++k) {
                        const int t = (int)threadIdx.x + k * kNT;
                        A[i][k] = row[col_off<ORD>(g, t)];
                        // column order: X[0] and X[Lh] are real and stored together
                        B[i][k] = row[col_off<ORD>(g, ORD == kColumns && t == 0 ? 0 : Lh - t)];
                    }
                    // X[Lh/2] for item 0 of a line (loaded by the first wave only)
                    C[i] = mk<R>((R)0, (R)0);
                    if (threadIdx.x < 64) C[i] = row[col_off<ORD>(g, threadIdx.x == 0 ? (Lh >> 1) : (int)threadIdx.x)];
                }
#pragma unroll
                for (int i = 0; i < LC; ++i) {
                    const int l = l0 + i;
                    if (l >= nl) break;
                    cx<R>* out = buf + l * Lh;
#pragma unroll
                    for (int k = 0; k < IPL; ++k) {
                        const int t = (int)threadIdx.x + k * kNT;
                        if (t == 0) {
                            if (ORD == kColumns) {
                                B[i][k] = mk<R>(A[i][k].y, (R)0);
                                A[i][k].y = (R)0;
                            }
                            out[0] = split(A[i][k], B[i][k], mk<R>((R)1, (R)0));
                            out[Lh >> 1] = split(C[i], C[i], mk<R>((R)0, (R)1));   // conj(W^(Lh/2)) = i
                        } else {
                            out[t] = split(A[i][k], B[i][k], wc[k]);
                            out[Lh - t] = split(B[i][k], A[i][k], mk<R>(-wc[k].x, wc[k].y));   // conj(W^(Lh-t)) = -W^t
                        }
                    }
                }
            }
        };
        // Lh <= 2048: one, two or four items per thread and line
        if ((1 << lgq) == kNT) chunks(IntC<1>{});
        else if ((1 << lgq) == 2 * kNT) chunks(IntC<2>{});
        else chunks(IntC<4>{});
    } else {
    // items in chunks of kXIt per thread: all loads of a chunk are issued
    // before any is used (no load behind a branch or a loop-carried wait)
    const int count = slots_of<LN>(g, npen * 3);
    for (int base = 0; base < count; base += kXIt * kNT) {
        cx<R> A[kXIt], B[kXIt], C[kXIt], W[kXIt];
        const int wave0 = base + ((int)threadIdx.x & ~63);
#pragma unroll
        for (int i = 0; i < kXIt; ++i) {
            const int e = min(base + (int)threadIdx.x + i * kNT, count - 1);
            int line, t;
            slot_of<LN>(g, e, line, t);
            const int p = line / 3, c = line - 3 * p;
            const cx<R>* row = Y1 + x_row<ORD>(g, mb, c, pen0 + p);
            A[i] = row[col_off<ORD>(g, t)];
            B[i] = row[col_off<ORD>(g, ORD == kColumns && t == 0 ? 0 : Lh - t)];
            W[i] = tw_fwd<R, ODD>(t << twsh);
            C[i] = mk<R>((R)0, (R)0);
            // X[Lh/2] for item 0 of a line, loaded only by waves holding such an item
            bool has0;
            if constexpr (ODD > 1) {
                const unsigned w = (unsigned)(wave0 + i * kNT) % (unsigned)(LN / 2);
                has0 = w == 0 || w + 64u > (unsigned)(LN / 2);
            } else {
                has0 = lgq < 6 || ((wave0 + i * kNT) & ((1 << lgq) - 1)) == 0;
            }
            if (has0) C[i] = row[col_off<ORD>(g, t == 0 ? (Lh >> 1) : t)];
        }
#pragma unroll
        for (int i = 0; i < kXIt; ++i) {
            const int e = base + (int)threadIdx.x + i * kNT;
            if (e >= count) break;
            int line, t;
            slot_of<LN>(g, e, line, t);
            cx<R>* out = buf + line * Lh;
            if (t == 0) {
                if (ORD == kColumns) {
                    B[i] = mk<R>(A[i].y, (R)0);
                    A[i].y = (R)0;
                }
                out[0] = split(A[i], B[i], mk<R>((R)1, (R)0));
                if (Lh > 1) out[Lh >> 1] = split(C[i], C[i], mk<R>((R)0, (R)1));   // conj(W^(Lh/2)) = i
            } else {
                const cx<R> wc = cconj<R>(W[i]);
                out[t] = split(A[i], B[i], wc);
                out[Lh - t] = split(B[i], A[i], mk<R>(-wc.x, wc.y));            // conj(W^(Lh-t)) = -W^t
            }
        }
    }
    }
    __syncthreads();
    auto none_load = [&](int, int) -> cx<R> { return mk<R>(0, 0); };
    auto none_store = [&](int, int, cx<R>) {};
    fft_io<R, true, pemax<ORD>(), true, true, kLines, 1, false, true, line_lgm<ORD, LN>(), kNT, true, ODD>(
        buf, g.lgLh, 0, npen * 3, none_load, none_store);
}

// Forward x pass: buf holds packed lines z[n] = x[2n] + i x[2n+1]; writes the
// Hx-column half spectrum of every line to X1.  Merge step: with P = Z[k],
// Q = Z[Lh-k], E = (P + Q*)/2, O = (P - Q*)/(2i) and T = W^k O,
// X[k] = E + T and X[Lh-k] = (E - T)*.
template <typename R, int ORD, int LN>
__device__ void r2c_lines(cx<R>* buf, cx<R>* X1, const PG& g, int mb, int pen0, int npen) {
    constexpr int ODD = line_odd<LN>();
    const int Lh = g.Lh;
    const int lgq = g.lgLh > 0 ? g.lgLh - 1 : 0;
    const int twsh = tw_log(ODD) - g.lgPx;
    auto none_load = [&](int, int) -> cx<R> { return mk<R>(0, 0); };
    auto none_store = [&](int, int, cx<R>) {};
    tw_lds_fill<R, ODD>();   // pass twiddles (same values if c2r_lines filled them)
    __syncthreads();
    fft_io<R, false, pemax<ORD>(), true, true, kLines, 1, true, false, line_lgm<ORD, LN>(), kNT, true, ODD>(
        buf, g.lgLh, 0, npen * 3, none_load, none_store);
    const R half = (R)0.5;
    if (ODD == 1 && (1 << lgq) >= kNT) {
        // as in the split step: fixed items t = tid + k kNT of every line,
        // uniform row addresses
        auto lines = [&](auto ipl_c) {
            constexpr int IPL = decltype(ipl_c)::value;   // items per thread and line
            cx<R> W[IPL];
#pragma unroll
            for (int k = 0; k < IPL; ++k) W[k] = tw_fwd<R>(((int)threadIdx.x + k * kNT) << twsh);
            const int nl = npen * 3;
            for (int l = 0; l < nl; ++l) {
                const int p = l / 3, c = l - 3 * p;
                cx<R>* row = X1 + x_row<ORD>(g, mb, c, pen0 + p);
                const cx<R>* in = buf + l * Lh;
#pragma unroll
                for (int k = 0; k < IPL; ++k) {
                    const int t = (int)threadIdx.x + k * kNT;
                    if (t == 0) {
                        const cx<R> P = in[0];
                        row[0] = mk<R>(P.x + P.y, ORD == kColumns ? P.x - P.y : (R)0);
                        if (ORD != kColumns) row[Lh] = mk<R>(P.x - P.y, (R)0);
                        row[col_off<ORD>(g, Lh >> 1)] = cconj<R>(in[Lh >> 1]);   // W^(Lh/2) = -i
                    } else {
                        const cx<R> P = in[t], Q = in[Lh - t];
                        const cx<R> E = mk<R>(half * (P.x + Q.x), half * (P.y - Q.y));
                        const cx<R> O = mk<R>(half * (P.y + Q.y), half * (Q.x - P.x));
                        const cx<R> T = cmul<R>(W[k], O);
                        row[col_off<ORD>(g, t)] = cadd<R>(E, T);
                        row[col_off<ORD>(g, Lh - t)] = mk<R>(E.x - T.x, T.y - E.y);
                    }
                }
            }
        };
        if ((1 << lgq) == kNT) lines(IntC<1>{});
        else if ((1 << lgq) == 2 * kNT) lines(IntC<2>{});
        else lines(IntC<4>{});
        return;
    }
    const int count = slots_of<LN>(g, npen * 3);
    for (int base = 0; base < count; base += kXIt * kNT) {
        cx<R> W[kXIt];
#pragma unroll
        for (int i = 0; i < kXIt; ++i) {
            const int e = min(base + (int)threadIdx.x + i * kNT, count - 1);
            int line, t;
            slot_of<LN>(g, e, line, t);
            W[i] = tw_fwd<R, ODD>(t << twsh);
        }
#pragma unroll
        for (int i = 0; i < kXIt; ++i) {
            const int e = base + (int)threadIdx.x + i * kNT;
            if (e >= count) break;
            int line, t;
            slot_of<LN>(g, e, line, t);
            const int p = line / 3, c = line - 3 * p;
            cx<R>* row = X1 + x_row<ORD>(g, mb, c, pen0 + p);
            const cx<R>* in = buf + line * Lh;
            if (t == 0) {
                const cx<R> P = in[0];
                row[0] = mk<R>(P.x + P.y, ORD == kColumns ? P.x - P.y : (R)0);
                if (ORD != kColumns) row[Lh] = mk<R>(P.x - P.y, (R)0);
                if (Lh > 1) row[col_off<ORD>(g, Lh >> 1)] = cconj<R>(in[Lh >> 1]);   // W^(Lh/2) = -i
            } else {
                const cx<R> P = in[t], Q = in[Lh - t];
                const cx<R> E = mk<R>(half * (P.x + Q.x), half * (P.y - Q.y));
                const cx<R> O = mk<R>(half * (P.y + Q.y), half * (Q.x - P.x));
                const cx<R> T = cmul<R>(W[i], O);
                row[col_off<ORD>(g, t)] = cadd<R>(E, T);
                row[col_off<ORD>(g, Lh - t)] = mk<R>(E.x - T.x, T.y - E.y);
            }
        }
    }
}

template <typename R>
__device__ __forceinline__ R demag_at(const cx<R>* buf, int line, int Lh, int n, int h) {
    const cx<R> v = buf[line * Lh + n];
    return h ? v.y : v.x;
}

__device__ __forceinline__ double block_sum(double v, double* sh) {
    sh[threadIdx.x] = v;
    __syncthreads();
    for (int s = kNT / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
        __syncthreads();
    }
    const double r = sh[0];
    __syncthreads();
    return r;
}


}  // namespace magx
