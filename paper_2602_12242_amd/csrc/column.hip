// Column convolution: forward y pass, z pass with the spectral product and inverse
// y pass of one kx column in one kernel, for thin grids whose column (all y and z
// of the three components) fits in LDS (plan.col).
//
// The x passes write and read X1 in column order here, [kx / 4][y][c][z][kx % 4]:
// a block reads one column out of a contiguous piece of four, and an x pass touches
// 32 bytes at a time; X2 and its two round trips through memory
// (192 of the 264 bytes per cell of the three separate passes) do not exist.
// The half spectrum of a real line has real values at kx = 0 and kx = Lh: the x
// passes store them as one complex column kx = 0, which leaves exactly Lh
// columns; the two are told apart after the y pass by the symmetry of a real
// sequence's transform.
//
//  * y: Stockham passes of radix 8 (a factor 3 or 5 last) over the 3 nz
//    sequences of a column in LDS, element (y, b) at y st + b with st = 3 nz T | 1
//    (odd: a row per lane and a sequence per lane are both free of bank conflicts).
//  * z: one thread per ky row, in registers.  The even and the odd kz are each a
//    length-Pz/2 DFT of the (for odd kz twiddled) inputs, of which only z < Pz/2
//    are not zero; each half is multiplied by the tensor and transformed back, and
//    the two accumulate: Pz/2 values of three components at a time, no exchange.
//  * The tensor is read from a copy in column order, [Lh + 1][6][Hz][Hy].
//
// What bounds it: a block is a chain of memory, LDS and register phases with one
// to four blocks per CU by LDS and registers, and the block of column 0 runs its z
// phase twice.  At 300x300x1 in single precision 12.3 us a launch for what took
// 20.6 + 15.4 + 16.0 (event-timed), at 640x160x4 28 for 45, at 256x256x8 31 for 43.
#include <mutex>

#include "magx_internal.hpp"

namespace magx {

template <int PY> struct ColCfg {
    static constexpr int ODD = odd_part(PY);
    static constexpr int LG = ilog2c(PY / ODD);
    static constexpr int T = column_width(PY);                          // columns per block
    static constexpr int NT = (T * PY + 63) / 64 * 64;                  // one thread per (column, ky)
};

// One Stockham pass of radix RAD over nseq sequences of length L in LDS (see
// the header of this file for the layout); NS: product of the radices so far.
// SRC_FN / DST_FN: load(b, j) / store(b, j, v) in place of LDS; HIN, HOUT: only
// the lower half of the inputs is not zero / of the outputs is wanted.
template <typename R, int RAD, int L, int NS, bool INV, int EM, int NT, bool SRC_FN, bool DST_FN, bool HIN, bool HOUT,
          class Load, class Store>
__device__ __forceinline__ void col_pass(cx<R>* buf, unsigned st, unsigned nseq, const FastDiv& fd, Load& load,
                                         Store& store) {
    constexpr int ODD = odd_part(L);
    constexpr bool LAST_ODD = RAD == 3 || RAD == 5;
    constexpr unsigned nb = L / RAD;
    constexpr int PER = (EM + RAD - 1) / RAD;
    constexpr int RIN = HIN ? RAD / 2 : RAD, ROUT = HOUT ? (RAD + 1) / 2 : RAD;
    constexpr int twshift = tw_log(ODD) - (LAST_ODD ? 0 : ilog2c(RAD)) - ilog2c(NS);
    const unsigned total = nb * nseq;
    cx<R> v[PER][RAD];
    unsigned bb[PER], pp[PER];
    const unsigned tid = (unsigned)tid_opaque<NT>();
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const unsigned t = tid + (unsigned)(i * NT);
        if (t < total) {
            const unsigned j = (unsigned)fdiv((int)t, fd), b = t - j * nseq;
#pragma unroll
            for (int r = 0; r < RIN; ++r) {
                if constexpr (SRC_FN) v[i][r] = load(b, j + r * nb);
                else v[i][r] = buf[umul24(j + r * nb, st) + b];
            }
#pragma unroll
            for (int r = RIN; r < RAD; ++r) v[i][r] = mk<R>((R)0, (R)0);
            const unsigned k = j % (unsigned)NS;
            bb[i] = b;
            pp[i] = (j / (unsigned)NS) * (unsigned)(NS * RAD) + k;
            if constexpr (NS > 1) twiddle_apply<R, INV, RAD, true, ODD>(v[i], (int)k, twshift);
            dft<R, RAD, INV>(v[i]);
        }
    }
    if constexpr (!SRC_FN && !DST_FN) __syncthreads();
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const unsigned t = tid + (unsigned)(i * NT);
        if (t < total) {
#pragma unroll
            for (int r = 0; r < ROUT; ++r) {
                if constexpr (DST_FN) store(bb[i], pp[i] + (unsigned)(r * NS), v[i][r]);
                else buf[umul24(pp[i] + (unsigned)(r * NS), st) + bb[i]] = v[i][r];
            }
        }
    }
    if constexpr (!DST_FN) __syncthreads();
}

// The passes of a transform of length L from the product NS on: the remainder of
// log2 by 3 first, radix 8, the odd factor last.
template <typename R, int L, int NS, bool INV, int EM, int NT, class Load, class Store>
__device__ __forceinline__ void col_fft(cx<R>* buf, unsigned st, unsigned nseq, const FastDiv& fd, Load& load,
                                        Store& store) {
    constexpr int ODD = odd_part(L), P2 = L / ODD, LEFT = P2 / NS;
    constexpr int RAD = NS == P2 ? ODD : (NS == 1 && ilog2c(P2) % 3 ? 1 << (ilog2c(P2) % 3) : 8);
    if constexpr (NS < L) {
        constexpr bool first = NS == 1, last = NS * RAD == L;
        static_assert(NS == P2 || LEFT % RAD == 0, "radix plan");
        // forward: the first pass loads, the last stays in LDS; inverse: the last stores
        col_pass<R, RAD, L, NS, INV, EM, NT, first && !INV, last && INV, first && !INV, last && INV>(buf, st, nseq, fd,
                                                                                                    load, store);
        if constexpr (!last) col_fft<R, L, NS * RAD, INV, EM, NT>(buf, st, nseq, fd, load, store);
    }
}

template <typename R, int PY, int PZ>
__global__ void __launch_bounds__((ColCfg<PY>::NT))
    column_kernel(cx<R>* __restrict__ X1, const R* __restrict__ tens, R Ms, int ny, int nz, int Lh, int st_,
                  FastDiv fd) {
    constexpr int ODD = ColCfg<PY>::ODD, T = ColCfg<PY>::T, NT = ColCfg<PY>::NT, EM = 3 * PZ / 2;
    constexpr int Hy = PY / 2 + 1, Hz = PZ / 2 + 1;
    constexpr int S = PZ / 2, NQ = 2;
    tw_lds_fill<R, ODD>();
    extern __shared__ unsigned char smem_raw[];
    cx<R>* buf = reinterpret_cast<cx<R>*>(smem_raw);
    const unsigned st = (unsigned)st_;
    const unsigned n3 = 3u * (unsigned)nz, nseq = n3 * T;
    const int cpm = Lh / T;                                   // column groups of a member
    // (most groups of four columns, which share lines, stay on one XCD: its range of
    // blocks need not end at a group, then two XCDs hold parts of its lines)
    const int lb = xcd_logical_block(blockIdx.x, gridDim.x);
    const int mb = lb / cpm, kx0 = (lb - mb * cpm) * T;
    cx<R>* base = X1 + ((long long)mb * Lh + (kx0 & ~3)) * ny * n3 + (kx0 & 3);
    auto off = [&](unsigned b, unsigned j) {
        if constexpr (T == 1) return 4u * (j * n3 + b);
        const unsigned t = b / n3;                            // T = 2: columns kx0, kx0 + 1 of one group of four
        return 4u * (j * n3 + (b - t * n3)) + t;
    };
    auto load = [&](unsigned b, unsigned j) -> cx<R> {
        return (int)j < ny ? base[off(b, j)] : mk<R>((R)0, (R)0);
    };
    auto store = [&](unsigned b, unsigned j, cx<R> v) {
        if ((int)j < ny) base[off(b, j)] = v;
    };
    __syncthreads();   // the twiddle table
    col_fft<R, PY, 1, false, EM, NT>(buf, st, nseq, fd, load, store);
    // z
    cx<R> acc[3][S];
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int n = 0; n < S; ++n) acc[c][n] = mk<R>((R)0, (R)0);
    const int tid = threadIdx.x;
    const int tc = tid / PY, ky = tid - tc * PY;
    const bool act = NT == T * PY || tid < T * PY;
    const int kx = kx0 + tc;
    cx<R>* row = buf + (unsigned)ky * st + (unsigned)tc * n3;
    if (act) {
        const cx<R>* mir = buf + (unsigned)(ky == 0 ? 0 : PY - ky) * st + (unsigned)tc * n3;
        const int kyo = ky <= PY / 2 ? ky : PY - ky;
        const R sy = ky <= PY / 2 ? (R)1 : (R)-1;
        // kx = 0 holds the columns 0 (rep 0) and Lh (rep 1): of Z = A + i B with
        // real sequences' transforms A and B, A = (Z + Z*')/2 and i B = (Z - Z*')/2,
        // Z*' the conjugate at -ky
        const int nrep = kx == 0 ? 2 : 1;
#pragma unroll 1
        for (int rep = 0; rep < nrep; ++rep) {
            const R* ten = tens + (long long)(rep ? Lh : kx) * (6 * Hz * Hy) + kyo;
            auto value = [&](int c, int z) -> cx<R> {
                if (z >= nz) return mk<R>((R)0, (R)0);
                const cx<R> a = row[c * nz + z];
                if (kx != 0) return a;
                const cx<R> b = cconj<R>(mir[c * nz + z]);
                const cx<R> d = rep ? csub<R>(a, b) : cadd<R>(a, b);
                return cscale<R>(d, (R)0.5);
            };
            auto residue = [&](auto qc) {
                constexpr int q = decltype(qc)::value;
                R tv[S][6];
#pragma unroll
                for (int k = 0; k < S; ++k) {
                    const int kz = NQ * k + q, kzo = kz <= PZ / 2 ? kz : PZ - kz;
#pragma unroll
                    for (int c6 = 0; c6 < 6; ++c6) tv[k][c6] = ten[(c6 * Hz + kzo) * Hy];
                }
                cx<R> u[3][S];
#pragma unroll
                for (int c = 0; c < 3; ++c) {
#pragma unroll
                    for (int n = 0; n < S; ++n) u[c][n] = value(c, n);
                    twist<R, false, q, PZ, S>(u[c]);
                    if constexpr (S > 1) dft<R, S, false>(u[c]);
                }
#pragma unroll
                for (int k = 0; k < S; ++k) {
                    const int kz = NQ * k + q;
                    const R sz = kz <= PZ / 2 ? (R)1 : (R)-1;
                    const R nxx = tv[k][0], nyy = tv[k][1], nzz = tv[k][2];
                    const R nxy = sy * tv[k][3], nxz = sz * tv[k][4], nyz = sy * sz * tv[k][5];
                    const cx<R> mx = u[0][k], my = u[1][k], mz = u[2][k];
                    u[0][k] = mk<R>(nxx * mx.x + nxy * my.x + nxz * mz.x, nxx * mx.y + nxy * my.y + nxz * mz.y);
                    u[1][k] = mk<R>(nxy * mx.x + nyy * my.x + nyz * mz.x, nxy * mx.y + nyy * my.y + nyz * mz.y);
                    u[2][k] = mk<R>(nxz * mx.x + nyz * my.x + nzz * mz.x, nxz * mx.y + nyz * my.y + nzz * mz.y);
                }
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    if constexpr (S > 1) dft<R, S, true>(u[c]);
                    twist<R, true, q, PZ, S>(u[c]);
#pragma unroll
                    for (int n = 0; n < S; ++n) acc[c][n] = cadd<R>(acc[c][n], u[c][n]);
                }
            };
            residue(IntC<0>{});
            residue(IntC<1>{});
        }
    }
    __syncthreads();   // column 0 reads the mirrored rows
    if (act) {
        const R s = -Ms;
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
            for (int n = 0; n < S; ++n)
                if (n < nz) row[c * nz + n] = cscale<R>(acc[c][n], s);
    }
    __syncthreads();
    col_fft<R, PY, 1, true, EM, NT>(buf, st, nseq, fd, load, store);
}

// The tensor in column order from the tile-major spectrum [Hy][ntz][6][Hz][tz].
template <typename R>
static __global__ void column_tensor_kernel(const R* __restrict__ spec, R* __restrict__ out, int Hx, int Hy, int Hz,
                                            int tz, int ntz, long long n) {
    const long long e = (long long)blockIdx.x * kNT + threadIdx.x;
    if (e >= n) return;
    const int ky = (int)(e % Hy);
    const long long r = e / Hy;
    const int kz = (int)(r % Hz), c6 = (int)(r / Hz % 6), kx = (int)(r / Hz / 6);
    out[e] = spec[((((long long)ky * ntz + kx / tz) * 6 + c6) * Hz + kz) * tz + kx % tz];
}

template <typename R>
hipError_t launch_column_tensor(const Plan& pl, void* spectrum, hipStream_t s) {
    const long long n = 6LL * pl.Hx * pl.Hy * pl.Hz;
    R* sp = static_cast<R*>(spectrum);
    hipLaunchKernelGGL(column_tensor_kernel<R>, dim3((unsigned)((n + kNT - 1) / kNT)), dim3(kNT), 0, s, sp,
                       sp + pl.tc_off, pl.Hx, pl.Hy, pl.Hz, pl.tz, pl.ntz, n);
    return hipGetLastError();
}

template <typename R, int PY, int PZ>
static hipError_t run_column(const Plan& pl, void* X1, const void* spec, R Ms, hipStream_t s) {
    using C = ColCfg<PY>;
    const int nseq = 3 * pl.nz * C::T, st = nseq | 1;
    const size_t lds = (size_t)st * PY * sizeof(cx<R>);
    if (pl.Py != PY || pl.Pz != PZ || 2 * pl.nz > PZ || pl.Lh % C::T != 0 || lds > (size_t)kColumnLds)
        return hipErrorInvalidValue;
    const void* k = reinterpret_cast<const void*>(&column_kernel<R, PY, PZ>);
    {
        // more than 64 KiB of dynamic LDS has to be allowed per kernel and device
        static std::mutex mu;
        static bool done[64];
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return hipErrorInvalidDevice;
        std::lock_guard<std::mutex> lk(mu);
        if (!done[dev]) {
            if (hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, kColumnLds) != hipSuccess)
                return hipErrorInvalidValue;
            done[dev] = true;
        }
    }
    hipLaunchKernelGGL((column_kernel<R, PY, PZ>), dim3((unsigned)(pl.Lh / C::T * pl.nbatch)), dim3(C::NT), lds, s,
                       static_cast<cx<R>*>(X1), static_cast<const R*>(spec) + pl.tc_off, Ms, pl.ny, pl.nz, pl.Lh, st,
                       make_fastdiv(nseq));
    return hipGetLastError();
}

template <typename R, int PZ>
static hipError_t run_column_py(const Plan& pl, void* X1, const void* spec, R Ms, hipStream_t s) {
    if constexpr (PZ == 16) {   // the lengths it is the faster path at
        if (pl.Py == 256) return run_column<R, 256, PZ>(pl, X1, spec, Ms, s);
        if (pl.Py == 512) return run_column<R, 512, PZ>(pl, X1, spec, Ms, s);
        return hipErrorInvalidValue;
    } else {
        switch (pl.Py) {
            case 32: return run_column<R, 32, PZ>(pl, X1, spec, Ms, s);
            case 64: return run_column<R, 64, PZ>(pl, X1, spec, Ms, s);
            case 128: return run_column<R, 128, PZ>(pl, X1, spec, Ms, s);
            case 160: return run_column<R, 160, PZ>(pl, X1, spec, Ms, s);
            case 192: return run_column<R, 192, PZ>(pl, X1, spec, Ms, s);
            case 256: return run_column<R, 256, PZ>(pl, X1, spec, Ms, s);
            case 320: return run_column<R, 320, PZ>(pl, X1, spec, Ms, s);
            case 384: return run_column<R, 384, PZ>(pl, X1, spec, Ms, s);
            case 512: return run_column<R, 512, PZ>(pl, X1, spec, Ms, s);
            default: break;
        }
        // longer columns: more than 512 threads leave 128 (1024) or 168 registers
        if (pl.Py == 640) return run_column<R, 640, PZ>(pl, X1, spec, Ms, s);
        if (pl.Py == 768) return run_column<R, 768, PZ>(pl, X1, spec, Ms, s);
        if constexpr (PZ <= (sizeof(R) == 4 ? 8 : 4)) {
            if (pl.Py == 1024) return run_column<R, 1024, PZ>(pl, X1, spec, Ms, s);
        }
        return hipErrorInvalidValue;
    }
}

template <typename R>
hipError_t launch_column(const Plan& pl, void* X1, const void* spec, R Ms, hipStream_t s) {
    switch (pl.Pz) {
        case 2: return run_column_py<R, 2>(pl, X1, spec, Ms, s);
        case 4: return run_column_py<R, 4>(pl, X1, spec, Ms, s);
        case 8: return run_column_py<R, 8>(pl, X1, spec, Ms, s);
        case 16:
            if constexpr (sizeof(R) == 4) return run_column_py<R, 16>(pl, X1, spec, Ms, s);
            return hipErrorInvalidValue;
        default: return hipErrorInvalidValue;
    }
}

#define MAGX_INST(R)                                                                        \
    template hipError_t launch_column<R>(const Plan&, void*, const void*, R, hipStream_t);  \
    template hipError_t launch_column_tensor<R>(const Plan&, void*, hipStream_t);

#if MAGX_REAL == 32
MAGX_INST(float)
MAGX_TW_INIT(init_tw_column32)
#else
MAGX_INST(double)
MAGX_TW_INIT(init_tw_column64)
#endif

}  // namespace magx
