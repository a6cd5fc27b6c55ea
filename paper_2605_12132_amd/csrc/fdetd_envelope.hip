// Fused stages of the FP64 envelope propagator: S consecutive Horner stages in one pass over memory.
//
// A stage (section 4.2) reads the stage vector (a, a~), the state psi_a and chi and writes the next stage
// vector, 6.5 complex values per cell, and the stages of a step are bound by exactly those bytes.  A group of S
// stages reads the same planes once and keeps the S - 1 vectors between its stages on the chip.
//
// Layout of the work.  A block owns COLS consecutive z columns, of which the middle OC = COLS - 2 (S - 1) N_D are
// output (the columns beside them are formed by the neighbouring blocks as well: stage t is needed N_D columns
// beyond stage t + 1), and marches down a segment of rho rows; stage t + 1 runs N_D rows behind stage t.  Each
// lane keeps, per stage, the window of 2 N_D + 1 rows of a for the rho stencils, whose newest row is the stage
// before's output of the same iteration, and a delay line of N_D + 1 rows of a~.  The current row of a of every
// stage is shared through LDS for the z stencils, two rows per barrier (the windows hold the next row as well;
// N_D = 1: one).  Columns beside the grid and rows beyond it are read at the nearest cell of the grid and replaced
// by zeros.
//
// What bounds it (order 8, 4096 x 512, a step of 4 stages: 137 us stage by stage, 109 us fused; 6000 x 700, whose
// planes leave the caches: 355 and 217 us; order 2: 345 and 134 us): no longer the bytes (249 MB per group past
// the L2, 4.5 TB/s) but issue, with two wavefronts per SIMD and the vector unit busy 42 % of the time, and the rows
// and columns formed twice (a fifth at this size).  Two blocks of four wavefronts per CU are as fast as one of eight
// (867 and 877 us per 8 steps) and faster than three (910: shorter segments) or one of twelve (934); one barrier per
// row 867, per two rows 836.
#include "fdetd_envelope.h"
#include "fdetd_lanes.h"

namespace fdetd {
namespace {

using L_ = lv<double, 1>;  // a lane's part of a complex value

// Lane access at a byte offset from a wave-uniform address (scalar base, 32-bit lane offset).
#define FDETD_GLOBAL __attribute__((address_space(1)))
using GBytes = FDETD_GLOBAL char;
__device__ __forceinline__ double rld(const GBytes *p, unsigned off) { return *(const FDETD_GLOBAL double *)(p + off); }
__device__ __forceinline__ void rst(GBytes *p, unsigned off, double v) { *(FDETD_GLOBAL double *)(p + off) = v; }
// Barrier of the block that orders its LDS accesses only: loads in flight from global memory stay in flight.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}
// Holds a wave-uniform value in scalar registers from here on.
__device__ __forceinline__ void keep(double &x) { asm volatile("" : "+s"(x)); }
// This lane's part of i s x, of which the lane holds the real (even lanes) or imaginary part
__device__ __forceinline__ L_ rotate(double s, L_ x)
{
    const unsigned long long u = __builtin_bit_cast(unsigned long long, x.p[0]);
    const unsigned lo = __builtin_amdgcn_mov_dpp((int)(unsigned)u, 0xB1, 0xf, 0xf, true);
    const unsigned hi = __builtin_amdgcn_mov_dpp((int)(unsigned)(u >> 32), 0xB1, 0xf, 0xf, true);
    const double o = __builtin_bit_cast(double, (unsigned long long)hi << 32 | lo);
    return L_{{(threadIdx.x & 1) ? s * o : -s * o}};
}

struct EnvGroup {  // one problem's vectors (a, a~) of a group; wave-uniform
    CDesc *D;
    const char *va, *vt, *pa, *pt, *chi;
    char *oa, *ot;
    const double *coef;
};

template <int ND, int S>
struct EnvGeo {
    static constexpr int SL = 2, CPW = WAVE / SL, COLS = kEnvWaves * CPW;  // lanes per column, columns
    static constexpr int OC = COLS - 2 * (S - 1) * ND, ROW = (COLS + 2 * ND) * SL;
    static constexpr int RB = ND > 1 ? 2 : 1;                     // rows that share a barrier
    static constexpr int TAB = 2 * RB * S * ROW;                  // in doubles: offset of the row table
    static constexpr int LDS = TAB + 3 * kEnvRows;                // 1 / rho, m^2 / rho^2, sigma_rho per row
};

// Output rows k0 .. k1 - 1, columns o0 .. o0 + OC - 1.
template <int ND, int S>
__device__ __forceinline__ void env_group(const EnvGroup &C, int o0, int k0, int k1, double *lds)
{
    using G = EnvGeo<ND, S>;
    constexpr int SL = G::SL, ROW = G::ROW, W = 2 * ND + 1, PF = 2, U = 4, RB = G::RB;
    CDesc &D = *C.D;
    const int nz = __builtin_amdgcn_readfirstlane(D.nz), nr = __builtin_amdgcn_readfirstlane(D.nr);
    const int lane = threadIdx.x % WAVE, strip = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
    static_assert((long long)kEnvColumns * SL * (int)sizeof(double) <= 0x7fffffff, "bytes of a row");
    const int rb = nz * SL * (int)sizeof(double), rbc = nz * (int)sizeof(double);
    const int base = max(0, k0 - (S - 1) * ND), niter = k1 - base + (S - 1) * ND;
    const int col = o0 - (S - 1) * ND + strip * G::CPW + lane / SL, ccol = min(max(col, 0), nz - 1);
    const bool in_grid = col == ccol, out_col = in_grid && col >= o0 && col < o0 + G::OC;
    const unsigned off = (unsigned)((ccol * SL + lane % SL) * (int)sizeof(double)), coff = (unsigned)(ccol * (int)sizeof(double));
    // halo columns of the input row: N_D to the left by the first wavefront, to the right by the last
    const bool hl = lane < ND * SL && (strip == 0 || strip == kEnvWaves - 1);
    const int hcol = (strip == 0 ? o0 - S * ND : o0 - (S - 1) * ND + G::COLS) + lane / SL, hcc = min(max(hcol, 0), nz - 1);
    const unsigned hoff = (unsigned)((hcc * SL + lane % SL) * (int)sizeof(double));
    const bool h_in = hl && hcol == hcc;
    const int hidx = (strip == 0 ? 0 : (ND + G::COLS) * SL) + lane, own = ND * SL + strip * WAVE + lane;
    const L_ zero = zero_lv<double, 1>();
    const double pS = D.pS, k2 = 2.0 * D.k0;
    const double szi = in_grid ? gld<double>(D.sz, (unsigned)col) : 0.0;  // absorbing layer: sigma_z of this column

    // row table: row j is the row that the last stage has in iteration j
    double *tab = lds + G::TAB;
    for (int j = threadIdx.x; j < kEnvRows; j += kEnvWaves * WAVE) {
        const int r = min(max(base - (S - 1) * ND + j, 0), nr - 1);
        tab[3 * j] = D.rinv_p[r];
        tab[3 * j + 1] = D.m2rinv2[r];
        tab[3 * j + 2] = D.sr[r];
    }
    // the taps stay in scalar registers: left to the compiler they are loaded again in every row, and the wait for
    // scalar loads is one with the wait for the LDS reads
    double bz[ND + 1], br[ND + 1], dzc[ND], drc[ND];
#pragma unroll
    for (int j = 0; j <= ND; ++j) {
        bz[j] = D.bz[j];
        br[j] = D.br[j];
        keep(bz[j]);
        keep(br[j]);
        if (j < ND) {
            dzc[j] = D.dzc[j];
            drc[j] = D.drc[j];
            keep(dzc[j]);
            keep(drc[j]);
        }
    }

    // running pointers to the rows that the next fetch reads; each stays within the rows that its stage forms
    // (of the input vector: within the grid), where it reads a row again that nothing needs
    const GBytes *pw = (const GBytes *)C.va + (long long)min(base + ND, nr - 1) * rb;
    const GBytes *ph = (const GBytes *)C.va + (long long)base * rb, *pt = (const GBytes *)C.vt + (long long)base * rb;
    const GBytes *pa[S], *pb[S], *pc[S];
    int sf[S], sn[S];  // first row and number of rows that a stage has to form
#pragma unroll
    for (int t = 0; t < S; ++t) {
        sf[t] = max(0, k0 - (S - 1 - t) * ND);
        sn[t] = min(nr, k1 + (S - 1 - t) * ND) - sf[t];
        pa[t] = (const GBytes *)C.pa + (long long)sf[t] * rb;
        pb[t] = (const GBytes *)C.pt + (long long)sf[t] * rb;
        pc[t] = (const GBytes *)C.chi + (long long)sf[t] * rbc;
    }
    GBytes *oa = (GBytes *)C.oa + (long long)k0 * rb, *ot = (GBytes *)C.ot + (long long)k0 * rb;
    const int last = __builtin_amdgcn_readfirstlane(nr - 1);
    int fr = base;
    struct In {
        double w, t, pa[S], pt[S], chi[S];
    };
    auto fetch = [&]() -> In {
        In x;
        x.w = rld(pw, off);
        x.t = rld(pt, off);
        pw += fr + ND < last ? rb : 0;
        const int step = fr < last ? rb : 0;
        pt += step;
#pragma unroll
        for (int t = 0; t < S; ++t) {
            const bool on = (unsigned)(fr - t * ND - sf[t]) < (unsigned)(sn[t] - 1);
            const int st = on ? rb : 0;
            x.pa[t] = rld(pa[t], off);
            x.pt[t] = rld(pb[t], off);
            x.chi[t] = rld(pc[t], coff);
            pa[t] += st;
            pb[t] += st;
            pc[t] += on ? rbc : 0;
        }
        ++fr;
        return x;
    };
    int hr = base;
    auto fetch_h = [&]() -> double {
        const double x = rld(ph, hoff);
        ph += hr < last ? rb : 0;
        ++hr;
        return x;
    };
    double halo[U];
#pragma unroll
    for (int p = 0; p < U; ++p) halo[p] = fetch_h();
    In ring[PF];
#pragma unroll
    for (int p = 0; p < PF; ++p) ring[p] = fetch();

    // windows: rows r_t - N_D .. r_t + N_D while row r_t of stage t is formed; at the top of an iteration they sit
    // one slot higher and slide down first
    L_ Wa[S][W], T[S][ND + 1];
#pragma unroll
    for (int t = 0; t < S; ++t) {
#pragma unroll
        for (int q = 0; q < W; ++q) Wa[t][q] = zero;
#pragma unroll
        for (int q = 0; q <= ND; ++q) T[t][q] = zero;
    }
    {
        double f[W - 1];
#pragma unroll
        for (int t = 0; t < W - 1; ++t) {
            const int q = base - ND + t, r = q < 0 ? -1 - q : q;
            f[t] = rld((const GBytes *)C.va + (long long)min(r, nr - 1) * rb, off);
        }
#pragma unroll
        for (int t = 0; t < W - 1; ++t) {
            const int q = base - ND + t;
            Wa[0][t + 1] = keep_if(in_grid && q < nr, (q < 0 ? pS : 1.0) * L_{{f[t]}});
        }
    }
    // everything loaded so far has arrived: otherwise the loop's first wait, which serves the entry as well, would
    // wait for the newest loads in every iteration
    __builtin_amdgcn_s_waitcnt(0x0f70);
    const double *rt = tab;
    auto row = [&](const In &cu, int i, int u) {
        const int par = u % (2 * RB);
#pragma unroll
        for (int t = 0; t < S; ++t) {
#pragma unroll
            for (int q = 0; q < W - 1; ++q) Wa[t][q] = Wa[t][q + 1];
#pragma unroll
            for (int q = 0; q < ND; ++q) T[t][q] = T[t][q + 1];
        }
        Wa[0][W - 1] = keep_if(in_grid && base + i + ND < nr, L_{{cu.w}});
        // the rows of this barrier: the windows hold the next row of every stage as well (N_D > 1)
        if (u % RB == 0) {
#pragma unroll
            for (int x = 0; x < RB; ++x) {
                double *z = lds + (par + x) * S * ROW;
#pragma unroll
                for (int t = 0; t < S; ++t) {
                    z[t * ROW + own] = t == 0 || in_grid ? Wa[t][ND + x].p[0] : 0.0;
                }
                if (hl) z[hidx] = keep_if(h_in, L_{{halo[u + x]}}).p[0];
            }
            lds_barrier();
        }
#pragma unroll
        for (int t = 0; t < S; ++t) {
            const double *z = lds + (par * S + t) * ROW + own;
            const int r = base + i - t * ND;
            const L_ a0 = Wa[t][ND], tin = t == 0 ? L_{{cu.t}} : T[t][0];
            L_ lz = bz[0] * a0, d1z = zero, lr = br[0] * a0, d1r = zero;
#pragma unroll
            for (int j = 1; j <= ND; ++j) {
                const L_ zp = {{z[j * SL]}}, zm = {{z[-j * SL]}};
                lz = fmav(bz[j], zp + zm, lz);
                d1z = fmav(dzc[j - 1], zp - zm, d1z);
            }
#pragma unroll
            for (int j = 1; j <= ND; ++j) {
                const L_ rp = Wa[t][ND + j], rm = Wa[t][ND - j];
                lr = fmav(br[j], rp + rm, lr);
                d1r = fmav(drc[j - 1], rp - rm, d1r);
            }
            const double *e = rt + 3 * (S - 1 - t) * ND;
            const double sig = szi + e[2], pot = fma(sig, sig, e[1] + cu.chi[t]);
            const L_ dtv = lr + e[0] * d1r + lz - pot * a0 + rotate(k2, d1z + tin);
            const L_ na = L_{{cu.pa[t]}} + C.coef[t] * tin, nt = L_{{cu.pt[t]}} + C.coef[t] * dtv;
            if (t < S - 1) {
                Wa[t + 1][W - 1] = keep_if(r < nr, na);
                T[t + 1][ND] = nt;
                // first row of the next stage at the axis: the rows below the axis are the mirrored ones
                if (u % 2 == (t + 1) * ND % 2 && base == 0 && i == (t + 1) * ND) {
#pragma unroll
                    for (int j = 1; j <= ND; ++j) Wa[t + 1][ND - j] = pS * Wa[t + 1][ND + j - 1];
                }
            } else if (r >= k0 && r < k1) {
                if (out_col) {
                    rst(oa, off, na.p[0]);
                    rst(ot, off, nt.p[0]);
                }
                oa += rb;
                ot += rb;
            }
        }
        rt += 3;
    };
    for (int ib = 0; ib < niter; ib += U) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            row(ring[u % PF], ib + u, u);
            ring[u % PF] = fetch();
            halo[u] = fetch_h();
        }
    }
}

// Vector `sel` of problem p: 0 the caller's planes, 1 and 2 the plan's two stage vectors.
__device__ __forceinline__ void env_vector(const EnvFuseArgs &A, CDesc &D, int p, int sel, char *&a, char *&t)
{
    a = sel == 0 ? (char *)A.psi[p] : (char *)D.buf[sel - 1];
    t = sel == 0 ? (char *)A.aux[p] : (char *)D.buf[sel - 1] + D.plane * sizeof(double2);
}

template <int ND, int S>
__global__ __launch_bounds__(kEnvWaves *WAVE) void k_envelope_group(EnvFuseArgs A)
{
    using G = EnvGeo<ND, S>;
    __shared__ __align__(16) double lds[G::LDS];
    // each XCD (the blocks with b % 8 == x) gets a contiguous range of tiles
    const int per = (A.ntiles + NXCD - 1) / NXCD, t = (int)(blockIdx.x % NXCD) * per + (int)(blockIdx.x / NXCD);
    if (t >= A.ntiles) return;
    int p = 0;
    while (p + 1 < A.nprob && A.begin[p + 1] <= t) ++p;
    CDesc &D = ((CDesc *)A.probs)[p];
    FuseTile ft;
    if (!decode_fused(D.nz, D.nr, t - A.begin[p], A.seg, G::OC, ft)) return;
    // (the tile's divisions run in vector instructions: back to scalars)
    const int o0 = __builtin_amdgcn_readfirstlane(ft.o0), k0 = __builtin_amdgcn_readfirstlane(ft.k0),
              k1 = __builtin_amdgcn_readfirstlane(ft.k1);
    EnvGroup C;
    C.D = &D;
    char *a, *b;
    env_vector(A, D, p, A.sel_in, a, b);
    C.va = a;
    C.vt = b;
    env_vector(A, D, p, A.sel_psi, a, b);
    C.pa = a;
    C.pt = b;
    env_vector(A, D, p, A.sel_out, C.oa, C.ot);
    C.chi = (const char *)A.chi[p];
    C.coef = A.coefs;
    env_group<ND, S>(C, o0, k0, k1, lds);
}

template <int ND>
hipError_t go_fused(const EnvFuseArgs &a, hipStream_t s)
{
    const dim3 grid(NXCD * ((a.ntiles + NXCD - 1) / NXCD)), block(kEnvWaves * WAVE);
    hipLaunchKernelGGL((k_envelope_group<ND, env_depth(ND)>), grid, block, 0, s, a);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_envelope_fused(int nd, const EnvFuseArgs &a, hipStream_t s)
{
    switch (nd) {
    case 1: return go_fused<1>(a, s);
    case 2: return go_fused<2>(a, s);
    case 3: return go_fused<3>(a, s);
    case 4: return go_fused<4>(a, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace fdetd
