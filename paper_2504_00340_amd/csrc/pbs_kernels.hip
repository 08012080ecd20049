// HIP kernels of libpbsplit for gfx950 (CDNA4, wave64).
//
//   epass   energy CN half-steps (section 3.2 DG-P1 operator eq:(0041-d); section 3.3 CN), one
//           thread per (lateral cell, angle) line sweeping the groups from the top; the closing
//           half of step s-1 and the opening half of step s are done in the same sweep (one read
//           and one write of the fluence).  Also the catastrophic-source energy scan for the
//           next generation and the FP64 deposit of eq:(en_d).
//   tpass   lateral transport CN half-step (section 3.4, eq:(distansport), superbee slopes frozen
//           at the old level), one wave per (x, y) plane walking the rows in the upwind order;
//           the implicit upwind solve along a row is a first-order linear recurrence done as a
//           64-lane affine scan.
//   apass   angular diffusion CN step (section 3.4, eq:(sd), eq:(eqn_fly)) by the discrete sine
//           transform with the even/odd split of the sine matrix, staged through LDS.
//   qgemm   angular part of the catastrophic source: Q = P2^T W for every (state, group,
//           lateral tile).
//   dose    deterministic per-voxel reduction of the per-line deposits.
#include <type_traits>

#include "pbs_common.h"

namespace pbs {

typedef unsigned short u16x8v __attribute__((ext_vector_type(8)));

__device__ __forceinline__ float fast_rcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ double fast_rcp(double x) { return 1.0 / x; }

// Per-group table entries are the same for every lane: read through the constant address space they
// become scalar loads (one per wave, kept apart from the vector memory counter) instead of a vector load
// per lane that the group step then waits for.
template <typename T>
__device__ __forceinline__ T tab(const T *p, long i)
{
    return ((const __attribute__((address_space(4))) T *)p)[i];
}

// v of lane l (uniform)
template <typename T>
__device__ __forceinline__ T lane_of(T v, int l)
{
    if constexpr (sizeof(T) == 4) {
        return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l));
    } else {
        const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
        const unsigned lo = __builtin_amdgcn_readlane((int)(unsigned)u, l);
        const unsigned hi = __builtin_amdgcn_readlane((int)(unsigned)(u >> 32), l);
        return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
    }
}

// ------------------------------------------------------------------------------- energy pass
// The pipeline form of the smallest grids (defined below) and the blocks of 64 threads up to which they take it: about
// three blocks per CU, what its LDS lets run at once.  With one line per thread it still wins at 784 blocks (32 x 32 cells,
// 7 x 7 angles 36 -> 29 us) and loses at 1687 (20 x 24, 15 x 15, FP64 60 -> 82); with four at 605 (12 x 12, 31 x 31 104 -> 89
// us) and loses at 928 (32 x 32, 15 x 15 150 -> 200).
constexpr long EP_PIPE_BLOCKS = 800;
template <typename T, int L> static long epass_pipe_blocks(const EParams<T> &P);
template <typename T, int L> static hipError_t launch_epass_pipe(const EParams<T> &P, int mode, hipStream_t st);

// 2 x 2 CN solve of one group for one line: coefficients of the cell's half-step a.  The fused multiply-adds are
// spelled out, so that every pass that solves a line this way has the same bits.
template <typename T>
struct ECoef {
    T d11, d12, d21, d22, c1, c2, m11, m12, m21, m22, inv, a;
    __device__ __forceinline__ void set(T sm, T sp, T kp, T a_)
    {
#pragma clang fp contract(off)
        a = a_;
        d11 = -(sm + kp), d12 = sm, d21 = T(-3) * sp, d22 = -(fma(T(2), sm, sp) + kp);
        c1 = sp, c2 = T(3) * sp;
        m11 = fma(-a, d11, T(1)), m12 = -a * d12, m21 = -a * d21, m22 = fma(-a, d22, T(1));
        inv = fast_rcp(fma(m11, m22, -(m12 * m21)));
    }
    __device__ __forceinline__ void solve(T x1, T x2, T f, T q, T &y1, T &y2) const
    {
#pragma clang fp contract(off)
        const T r1 = fma(a, fma(c1, f, fma(d12, x2, d11 * x1)) + q, x1);
        const T r2 = fma(a, fma(c2, f, fma(d21, x1, d22 * x2)), x2);
        y1 = fma(r1, m22, -(m12 * r2)) * inv;
        y2 = fma(m11, r2, -(m21 * r1)) * inv;
    }
};

// One thread per line (FP64 contexts, and FP32 contexts whose source product takes the plain scan W):
// block = one lateral tile pb and one octet of angular lines a = 8*oct + e (e = tid/32), 32 cells
// pt = tid%32.  FP32 contexts with the split-BF16 product use epass8_body below.
//
// What bounds it at the sizes that take it (short angular grids, FP64): the serial chain over the groups.  A
// wave's next loads used to wait for its own stores (one memory counter, in order), so a group cost a store
// plus a load round trip.  EP_RING groups are now in flight in a register ring, every load issued before the
// stores of the groups ahead of it and without a branch (past the last group it re-reads group 0): 44 -> 28 us
// at 4 x 4 cells, 11 x 11 angles, 60 groups; 47 -> 29 us at 16 x 16, 7 x 7, 48 groups in FP64; 81 -> 58 us at
// 20 x 24, 15 x 15, 60 groups in FP64; unchanged where the grid fills the chip (64 x 64 cells).  A ring of 1
// gives 31 / 36 / 67 us there, one of 4 the same as 2 but 6 % less at 64 x 64 cells for its registers.
constexpr int EP_RING = 2;
template <typename T, int MODE, bool BANDS, bool HASQ>
__device__ __forceinline__ void epass_body(const EParams<T> &P, int bx)
{
    constexpr bool CL = (MODE & MODE_CLOSE) != 0;
    constexpr bool OP = (MODE & MODE_OPEN) != 0;
    const int NA = (int)(P.NAPT / PBS_PT);
    const int pbk = bx / P.NOCT, oct = bx % P.NOCT;
    const int e = threadIdx.x >> 5, ptc = threadIdx.x & 31;
    const int a = oct * 8 + e;
    if (a >= NA) return;
    const long line = ((long)pbk * NA + a) * PBS_PT + ptc;
    const long pq = (line / P.NAPT) * PBS_PT + (line % PBS_PT);
    const long S = P.NLINE;
    const long QS = (long)P.G * S;
    const double rc = CL ? (double)P.rho_c[pq] : 0.0;
    const double ro = OP ? (double)P.rho_o[pq] : 0.0;
    const double dac = 0.5 * (double)P.h * rc, dao = 0.5 * (double)P.h * ro;
    const T ac = (T)dac, ao = (T)dao;
    T fin = 0, fcl = 0, fop = 0;    // psi1 - psi2 of group g+1: input, after close, after open
    T U0 = 0, U1 = 0, U2 = 0;       // re-emission energy scans of states 0, 1, 2
    T U0b[4] = {}, U1b[4] = {}, U2b[4] = {};   // per-band scans (BANDS)
    double ph0 = 0, ph1 = 0, ph2 = 0, injc = 0, injo = 0;
    T fic = 0, fio = 0, fme = 0, fmn = 0;   // surrogate records (energy sent to the next generation, moments)
    const bool hasW = P.W != nullptr;
    const bool feat = P.inj_c != nullptr;
    T rx1[EP_RING], rx2[EP_RING], rqc[EP_RING], rqo[EP_RING];
    auto fetch = [&](int g, T &f1, T &f2, T &fqc, T &fqo) {
        const long gc = max(g, 0);
        const T *p = P.psi + (2L * gc) * S + line;
        f1 = p[0];
        f2 = p[S];
        // trapezoidal sources of the two half-steps: Q^n + Q* (close), Q^n + Q* (open)
        fqc = fqo = T(0);
        if constexpr (HASQ) {
            const long o = gc * S + line;
            if (CL) fqc = P.Q[o];
            if (OP) fqo = P.Q[QS + o];
        }
    };
#pragma unroll
    for (int u = 0; u < EP_RING; ++u) fetch(P.G - 1 - u, rx1[u], rx2[u], rqc[u], rqo[u]);
    // multiply-adds spelled out as in the pipeline of waves below: recording or not leaves the same bits
    auto group = [&](const int g, const int u) {
#pragma clang fp contract(off)
        T *p1 = P.psi + (2L * g) * S + line;
        T *p2 = p1 + S;
        const T x1 = rx1[u], x2 = rx2[u], qc = rqc[u], qo = rqo[u];
        fetch(g - EP_RING, rx1[u], rx2[u], rqc[u], rqo[u]);
        const T sm = tab(P.Sm, g), sp = tab(P.Sp, g), kp = tab(P.kap, g);
        // rho-free operator: psi1 row [-(S-+k), S-], psi2 row [-3S+, -(S+ + 2S- + k)], coupling S+[1,3]
        T y1 = x1, y2 = x2;
        ECoef<T> K;
        if (CL) {
            K.set(sm, sp, kp, ac);
            K.solve(x1, x2, fin + fcl, qc, y1, y2);
        }
        T z1 = y1, z2 = y2;
        if (OP) {
            K.set(sm, sp, kp, ao);
            K.solve(y1, y2, (CL ? fcl : fin) + fop, qo, z1, z2);
        }
        *p1 = z1;
        *p2 = z2;
        // deposit functional (FP64): stopping + removal of every state, bottom-face outflow
        const double A = tab(P.dA, g), B = tab(P.dB, g);
        if (CL) ph0 += fma(A, (double)x1, B * (double)x2);
        ph1 += fma(A, (double)y1, B * (double)y2);
        if (OP) ph2 += fma(A, (double)z1, B * (double)z2);
        if (g == 0) {
            if (CL) ph0 = fma(P.dBot, (double)x1 - (double)x2, ph0);
            ph1 = fma(P.dBot, (double)y1 - (double)y2, ph1);
            if (OP) ph2 = fma(P.dBot, (double)z1 - (double)z2, ph2);
        }
        if constexpr (HASQ) {
            const double wi = tab(P.dInj, g);
            if (CL) injc = fma(wi, (double)qc, injc);
            if (OP) injo = fma(wi, (double)qo, injo);
        }
        if (hasW || feat) {
            // energy scans of the three states; the next generation needs the sums 0+1 and 1+2
            const T w = tab(P.wc, g), dec = tab(P.wdec, g), idE = tab(P.invdE, g);
            const long o = (long)g * S + line;
            if constexpr (BANDS) {
                // the sum of one scan per band, each with its band's decay; group g feeds its own band
                const int bg = tab(P.band, g);
                U0 = U1 = U2 = T(0);
#pragma unroll
                for (int b = 0; b < 4; ++b)
                    if (b < P.NB) {
                        const T d = tab(P.wdecb, (long)b * P.G + g), wb = b == bg ? w : T(0);
                        if (CL) U0 += (U0b[b] = fma(wb, x1, d * U0b[b]));
                        U1 += (U1b[b] = fma(wb, y1, d * U1b[b]));
                        if (OP) U2 += (U2b[b] = fma(wb, z1, d * U2b[b]));
                    }
            } else {
                if (CL) U0 = fma(w, x1, dec * U0);
                U1 = fma(w, y1, dec * U1);
                if (OP) U2 = fma(dec, U2, w * z1);
            }
            if (feat) {
                // energy the re-emission puts into the next generation (the dInj functional of its
                // source summed over destination angles, which the angular law conserves), moments
                const T wi = (T)tab(P.dInj, g);
                if (CL) fic = fma(wi, (U0 + U1) * idE, fic);
                if (OP) {
                    fio = fma(wi, (U1 + U2) * idE, fio);
                    fme += fma((T)tab(P.wmom, g), z1, (T)tab(P.wmom, 2L * P.G + g) * z2);
                    fmn = fma((T)tab(P.wmom, (long)P.G + g), z1, fmn);
                }
            }
            if (hasW) {
                if (CL) P.W[o] = (U0 + U1) * idE;
                if (OP) P.W[QS + o] = (U1 + U2) * idE;
            }
        }
        fin = x1 - x2;
        fcl = y1 - y2;
        fop = z1 - z2;
    };
    int g0 = P.G - 1;
    for (; g0 >= EP_RING - 1; g0 -= EP_RING) {
#pragma unroll
        for (int u = 0; u < EP_RING; ++u) group(g0 - u, u);
    }
#pragma unroll
    for (int u = 0; u < EP_RING - 1; ++u)
        if (g0 - u >= 0) group(g0 - u, u);
    if (CL) P.dep_c[line] = dac * (ph0 + ph1 - injc) * P.scale;
    if (OP) P.dep_o[line] = dao * (ph1 + ph2 - injo) * P.scale;
    if (feat) {
        if (CL) P.inj_c[line] = dac * (double)fic * P.scale;
        if (OP) {
            P.inj_o[line] = dao * (double)fio * P.scale;
            P.mom_e[line] = (double)fme * P.scale;
            P.mom_n[line] = (double)fmn * P.scale;
        }
    }
}

template <typename T, int MODE, bool BANDS, bool HASQ>
__global__ __launch_bounds__(256) void epass_kernel(EParams<T> P)
{
    epass_body<T, MODE, BANDS, HASQ>(P, blockIdx.x);
}

template <typename T, bool BANDS, bool HASQ>
static void launch_epass_t(const EParams<T> &P, int mode, unsigned nb, hipStream_t st)
{
    if (mode == MODE_PAIR)
        hipLaunchKernelGGL((epass_kernel<T, MODE_PAIR, BANDS, HASQ>), dim3(nb), dim3(256), 0, st, P);
    else if (mode == MODE_OPEN)
        hipLaunchKernelGGL((epass_kernel<T, MODE_OPEN, BANDS, HASQ>), dim3(nb), dim3(256), 0, st, P);
    else
        hipLaunchKernelGGL((epass_kernel<T, MODE_CLOSE, BANDS, HASQ>), dim3(nb), dim3(256), 0, st, P);
}

template <typename T>
hipError_t launch_epass(const EParams<T> &P, int mode, hipStream_t st)
{
    if (P.Wh != nullptr) return hipErrorInvalidValue;   // split scans: launch_epass8
    if (P.NB > 4) return hipErrorInvalidValue;
    if (P.inj_c == nullptr && epass_pipe_blocks<T, 1>(P) <= EP_PIPE_BLOCKS) return launch_epass_pipe<T, 1>(P, mode, st);
    const unsigned nb = (unsigned)((P.NLINE / P.NAPT) * P.NOCT);
    if (P.NB > 1) {
        if (P.Q) launch_epass_t<T, true, true>(P, mode, nb, st);
        else launch_epass_t<T, true, false>(P, mode, nb, st);
    } else {
        if (P.Q) launch_epass_t<T, false, true>(P, mode, nb, st);
        else launch_epass_t<T, false, false>(P, mode, nb, st);
    }
    return hipGetLastError();
}

// ------------------------------------------------------------------ energy pass with straggling
// With straggling (section 3.2's (1/2) d^2/dE^2 (T psi)) every energy line is block-tridiagonal:
//   (I - a D0_g) X*_g - a Lo_g X*_{g-1} - a Up_g X*_{g+1} = X_g + a (D0 X)_g + a [q_g, 0],   a = h rho / 2,
// with the rho-free 2x2 blocks Lo (to g-1), Di (D0_gg), Up (to g+1) of the host tables.  The matrix
// depends only on the cell's density, so the elimination from the top,
//   Dt_g = (I - a Di_g) - a^2 Up_g Dt_{g+1}^-1 Lo_{g+1},   F_g = a Up_g Dt_{g+1}^-1,
// is done once per cell (factor kernel, FP64, stored as [g][8][NPpad]: Dt_g^-1 row-major, then F_g); each
// line then sweeps down (bt_g = b_g + F_g bt_{g+1}, kept in place of X_g) and back up
// (X*_g = Dt_g^-1 (bt_g + a Lo_g X*_{g-1})).  The energy scans of the next generation's source take a
// third sweep down over X*.

// One thread per cell, both half-steps of a chain in one launch (blockIdx.y), once for all generations.  It is a
// serial FP64 chain over the groups, so what counts is its length: the table entries arrive as scalar loads and
// the determinant is inverted once (four divisions before): 69 us per half-step and generation, four
// times a step of two generations, -> 59 us once (24 x 24 cells, 110 groups).
template <typename T>
__global__ __launch_bounds__(64) void strag_factor_kernel(EParams<T> P, int first)
{
    const long pq = (long)blockIdx.x * 64 + threadIdx.x, NPpad = P.NPpad;
    if (pq >= NPpad) return;
    const bool open = first + (int)blockIdx.y == 1;
    const T *rho = open ? P.rho_o : P.rho_c;
    T *sfac = open ? P.sfac_o : P.sfac_c;
    const double a = 0.5 * (double)P.h * (double)rho[pq];
    double di[4] = {0, 0, 0, 0};     // Dt_{g+1}^-1
    double L[4] = {0, 0, 0, 0};      // a Lo of group g+1
    for (int g = P.G - 1; g >= 0; --g) {
        double B[12];
#pragma unroll
        for (int i = 0; i < 12; ++i) B[i] = a * (double)tab(P.blk, 12L * g + i);
        // F = a Up Dt_{g+1}^-1; zero above the top group, where di is
        const double F0 = B[8] * di[0] + B[9] * di[2], F1 = B[8] * di[1] + B[9] * di[3];
        const double F2 = B[10] * di[0] + B[11] * di[2], F3 = B[10] * di[1] + B[11] * di[3];
        const double m0 = (1.0 - B[4]) - (F0 * L[0] + F1 * L[2]), m1 = -B[5] - (F0 * L[1] + F1 * L[3]);
        const double m2 = -B[6] - (F2 * L[0] + F3 * L[2]), m3 = (1.0 - B[7]) - (F2 * L[1] + F3 * L[3]);
        const double det = m0 * m3 - m1 * m2, idet = 1.0 / det;
        auto over_det = [&](double m) {   // FP64: corrected once, as accurate as a division
            const double q = m * idet;
            return sizeof(T) == 8 ? fma(fma(-q, det, m), idet, q) : q;
        };
        di[0] = over_det(m3), di[1] = -over_det(m1), di[2] = -over_det(m2), di[3] = over_det(m0);
#pragma unroll
        for (int i = 0; i < 4; ++i) L[i] = B[i];
        T *o = sfac + (size_t)g * 8 * NPpad + pq;
#pragma unroll
        for (int q = 0; q < 4; ++q) o[q * NPpad] = (T)di[q];
        o[4 * NPpad] = (T)F0;
        o[5 * NPpad] = (T)F1;
        o[6 * NPpad] = (T)F2;
        o[7 * NPpad] = (T)F3;
    }
}

// one step of the re-emission scan (single law, or the sum over bands) at group g; returns the scan value
template <typename T, bool BANDS>
__device__ __forceinline__ T scan_step(const EParams<T> &P, int g, T x, T &U, T (&Ub)[4])
{
    const T w = tab(P.wc, g);
    if constexpr (BANDS) {
        const int bg = tab(P.band, g);
        T u = T(0);
#pragma unroll
        for (int b = 0; b < 4; ++b)
            if (b < P.NB) u += (Ub[b] = (b == bg ? w : T(0)) * x + tab(P.wdecb, (long)b * P.G + g) * Ub[b]);
        return u;
    } else {
        U = w * x + tab(P.wdec, g) * U;
        return U;
    }
}

// The sweeps of one line, each with EP_RING groups in flight (as the plain pass: a group's loads are issued before
// the stores of the groups ahead of it, without a branch; past the last group they re-read it and are not used).
// Three sweeps a half-step, but the scan of a closing half-step's result is the scan of the opening one's start:
// a fused pair takes that sum along in the opening sweep down, five sweeps instead of six.
// Measured with the factors, us per generation: 24 x 24 cells, 15 x 15 angles, 110 groups 426 -> 294 (FP64 936 ->
// 630); 10 x 12, 9 x 9, 60 174 -> 84; 64 x 64, 11 x 11, 60 664 -> 496.
template <typename T, bool BANDS, bool HASQ>
struct StragLine {
    const EParams<T> &P;
    const long line, pq, S, FS;

    template <typename F>
    __device__ __forceinline__ void groups(F &&step) const   // step(k, slot) for k = 0 .. G-1
    {
        int k = 0;
        for (; k + EP_RING <= P.G; k += EP_RING) {
#pragma unroll
            for (int u = 0; u < EP_RING; ++u) step(k + u, u);
        }
#pragma unroll
        for (int u = 0; u < EP_RING - 1; ++u)
            if (k + u < P.G) step(k + u, u);
    }

    // right-hand side and elimination from the top (bt kept in place of X), deposit and scan of X^n; ADDPREV adds the
    // scan to the closing half-step's sum as well
    template <bool ADDPREV>
    __device__ __forceinline__ void down(int half, T a, double &phn, double &inj) const
    {
        const T *sf = (half ? P.sfac_o : P.sfac_c) + pq;
        const bool hasW = P.W != nullptr;
        const long QS = (long)P.G * S;
        T *W = hasW ? P.W + (long)half * QS + line : nullptr, *W0 = P.W + line;
        T xl1[EP_RING], xl2[EP_RING], f[EP_RING][4], q[EP_RING], wp[EP_RING];
        auto fetch = [&](int k, int u) {   // k-th group from the top
            const long g = max(P.G - 1 - k, 0), gl = max(P.G - 2 - k, 0);
            const T *p = P.psi + 2 * gl * S + line;
            xl1[u] = p[0];
            xl2[u] = p[S];
            const T *F = sf + g * 8 * FS + 4 * FS;
#pragma unroll
            for (int i = 0; i < 4; ++i) f[u][i] = F[i * FS];
            if constexpr (HASQ) q[u] = P.Q[(long)half * QS + g * S + line];
            if constexpr (ADDPREV) wp[u] = W0[g * S];
        };
        T xu1 = 0, xu2 = 0, bu1 = 0, bu2 = 0;   // X^n and bt of group g+1
        T x1 = P.psi[2L * (P.G - 1) * S + line], x2 = P.psi[(2L * (P.G - 1) + 1) * S + line];
        T U = 0, Ub[4] = {};
#pragma unroll
        for (int u = 0; u < EP_RING; ++u) fetch(u, u);
        groups([&](int k, int u) {
            const int g = P.G - 1 - k;
            const T l1 = g > 0 ? xl1[u] : T(0), l2 = g > 0 ? xl2[u] : T(0);   // X^n of group g-1
            const T F[4] = {f[u][0], f[u][1], f[u][2], f[u][3]};
            const T qg = HASQ ? q[u] : T(0), w0 = ADDPREV ? wp[u] : T(0);
            fetch(k + EP_RING, u);
            T B[12];
#pragma unroll
            for (int i = 0; i < 12; ++i) B[i] = tab(P.blk, 12L * g + i);
            T b1 = x1 + a * (B[0] * l1 + B[1] * l2 + B[4] * x1 + B[5] * x2 + B[8] * xu1 + B[9] * xu2 + qg);
            T b2 = x2 + a * (B[2] * l1 + B[3] * l2 + B[6] * x1 + B[7] * x2 + B[10] * xu1 + B[11] * xu2);
            b1 += F[0] * bu1 + F[1] * bu2;
            b2 += F[2] * bu1 + F[3] * bu2;
            P.psi[2L * g * S + line] = b1;
            P.psi[(2L * g + 1) * S + line] = b2;
            phn += tab(P.dA2, g) * (double)x1 + tab(P.dB2, g) * (double)x2;
            if constexpr (HASQ) inj += tab(P.dInj, g) * (double)qg;
            if (hasW) {
                const T u1 = scan_step<T, BANDS>(P, g, x1, U, Ub), idE = tab(P.invdE, g);
                W[(long)g * S] = u1 * idE;
                if constexpr (ADDPREV) W0[(long)g * S] = w0 + u1 * idE;
            }
            xu1 = x1, xu2 = x2, bu1 = b1, bu2 = b2;
            x1 = l1, x2 = l2;
        });
    }

    // back-substitution, deposit of X*
    __device__ __forceinline__ void up(int half, T a, double &phs) const
    {
        const T *sf = (half ? P.sfac_o : P.sfac_c) + pq;
        T c1[EP_RING], c2[EP_RING], d[EP_RING][4];
        auto fetch = [&](int k, int u) {
            const long g = min(k, P.G - 1);
            c1[u] = P.psi[2 * g * S + line];
            c2[u] = P.psi[(2 * g + 1) * S + line];
#pragma unroll
            for (int i = 0; i < 4; ++i) d[u][i] = sf[g * 8 * FS + i * FS];
        };
        T y1p = 0, y2p = 0;
#pragma unroll
        for (int u = 0; u < EP_RING; ++u) fetch(u, u);
        groups([&](int g, int u) {
            T b1 = c1[u], b2 = c2[u];
            const T D[4] = {d[u][0], d[u][1], d[u][2], d[u][3]};
            fetch(g + EP_RING, u);
            b1 += a * (tab(P.blk, 12L * g) * y1p + tab(P.blk, 12L * g + 1) * y2p);
            b2 += a * (tab(P.blk, 12L * g + 2) * y1p + tab(P.blk, 12L * g + 3) * y2p);
            const T y1 = D[0] * b1 + D[1] * b2, y2 = D[2] * b1 + D[3] * b2;
            P.psi[2L * g * S + line] = y1;
            P.psi[(2L * g + 1) * S + line] = y2;
            phs += tab(P.dA2, g) * (double)y1 + tab(P.dB2, g) * (double)y2;
            y1p = y1, y2p = y2;
        });
    }

    // the scan of X*, added to that of X^n
    __device__ __forceinline__ void rescan(int half) const
    {
        if (P.W == nullptr) return;
        T *W = P.W + (long)half * P.G * S + line;
        T x[EP_RING], w[EP_RING];
        auto fetch = [&](int k, int u) {
            const long g = max(P.G - 1 - k, 0);
            x[u] = P.psi[2 * g * S + line];
            w[u] = W[g * S];
        };
        T U = 0, Ub[4] = {};
#pragma unroll
        for (int u = 0; u < EP_RING; ++u) fetch(u, u);
        groups([&](int k, int u) {
            const int g = P.G - 1 - k;
            const T xg = x[u], wg = w[u];
            fetch(k + EP_RING, u);
            W[(long)g * S] = wg + scan_step<T, BANDS>(P, g, xg, U, Ub) * tab(P.invdE, g);
        });
    }
};

template <typename T, int MODE, bool BANDS, bool HASQ>
__global__ __launch_bounds__(256) void epass_strag_kernel(EParams<T> P)
{
    const int NA = (int)(P.NAPT / PBS_PT);
    const int bx = blockIdx.x, pbk = bx / P.NOCT, oct = bx % P.NOCT;
    const int e = threadIdx.x >> 5, ptc = threadIdx.x & 31;
    const int a = oct * 8 + e;
    if (a >= NA) return;
    const long line = ((long)pbk * NA + a) * PBS_PT + ptc;
    const long pq = (long)pbk * PBS_PT + ptc;
    const StragLine<T, BANDS, HASQ> L{P, line, pq, P.NLINE, P.NPpad};
    if (MODE & MODE_CLOSE) {
        const double ad = 0.5 * (double)P.h * (double)P.rho_c[pq];
        double phn = 0, phs = 0, inj = 0;
        L.template down<false>(0, (T)ad, phn, inj);
        L.up(0, (T)ad, phs);
        if (MODE == MODE_CLOSE) L.rescan(0);
        P.dep_c[line] = ad * (phn + phs - inj) * P.scale;
    }
    if (MODE & MODE_OPEN) {
        const double ad = 0.5 * (double)P.h * (double)P.rho_o[pq];
        double phn = 0, phs = 0, inj = 0;
        if (MODE == MODE_PAIR && P.W != nullptr)
            L.template down<true>(1, (T)ad, phn, inj);
        else
            L.template down<false>(1, (T)ad, phn, inj);
        L.up(1, (T)ad, phs);
        L.rescan(1);
        P.dep_o[line] = ad * (phn + phs - inj) * P.scale;
    }
}

template <typename T, bool BANDS, bool HASQ>
static void launch_epass_strag_t(const EParams<T> &P, int mode, unsigned nb, hipStream_t st)
{
    if (mode == MODE_PAIR)
        hipLaunchKernelGGL((epass_strag_kernel<T, MODE_PAIR, BANDS, HASQ>), dim3(nb), dim3(256), 0, st, P);
    else if (mode == MODE_OPEN)
        hipLaunchKernelGGL((epass_strag_kernel<T, MODE_OPEN, BANDS, HASQ>), dim3(nb), dim3(256), 0, st, P);
    else
        hipLaunchKernelGGL((epass_strag_kernel<T, MODE_CLOSE, BANDS, HASQ>), dim3(nb), dim3(256), 0, st, P);
}

template <typename T>
hipError_t launch_epass_strag(const EParams<T> &P, int mode, bool factors, hipStream_t st)
{
    if (!P.blk || !P.dA2 || !P.dB2 || P.Wh != nullptr || P.inj_c != nullptr || P.NB > 4) return hipErrorInvalidValue;
    if (factors)
        hipLaunchKernelGGL(strag_factor_kernel<T>, dim3((unsigned)((P.NPpad + 63) / 64), mode == MODE_PAIR ? 2 : 1),
                           dim3(64), 0, st, P, mode == MODE_OPEN ? 1 : 0);
    const unsigned nb = (unsigned)((P.NLINE / P.NAPT) * P.NOCT);
    if (P.NB > 1) {
        if (P.Q) launch_epass_strag_t<T, true, true>(P, mode, nb, st);
        else launch_epass_strag_t<T, true, false>(P, mode, nb, st);
    } else {
        if (P.Q) launch_epass_strag_t<T, false, true>(P, mode, nb, st);
        else launch_epass_strag_t<T, false, false>(P, mode, nb, st);
    }
    return hipGetLastError();
}
template hipError_t launch_epass_strag<float>(const EParams<float> &, int, bool, hipStream_t);
template hipError_t launch_epass_strag<double>(const EParams<double> &, int, bool, hipStream_t);

// Energy pass of FP32 contexts with the split-BF16 source product: one thread per (lateral cell,
// group of PBS_EPASS_LPT consecutive angular lines of an octet a = 8 oct + e).  The thread sweeps the
// groups of its lines together, so the scans of consecutive source nodes form one chunk (8 or 16
// bytes) of the [oct][cell][8] split layout that the thread writes itself (no exchange between
// threads, no barrier).  The FP64 deposits (and surrogate records) of those lines are summed into
// one partial per (cell, line group), stored at line slot a = line group; the dose reduction then
// sums NOCT * 8 / PBS_EPASS_LPT slots per cell instead of NA.  Lanes 0-31 hold the 32 cells of one
// tile.
// The energy pass streams the fluence (and the source) through once: non-temporal loads and stores
// keep it from displacing what the caches hold for others (measured 11.1 -> 10.9 ms per depth step of a
// 64 x 64-cell, 31 x 31-angle, 128-group, 4-generation beam).
#define EP_LD(p) __builtin_nontemporal_load(p)
#define EP_ST(v, p) __builtin_nontemporal_store(v, p)
__device__ __forceinline__ float bf16_to_f32(unsigned short h) { return __builtin_bit_cast(float, (unsigned)h << 16); }
// FEAT / LO = false compile out the surrogate records and the lo half of the split scans.
// RING > 0 keeps that many groups in flight in a register ring (HASQ: with the BF16 source), as the
// one-line-per-thread pass does: for grids with too few waves to hide a group's store and load round trip.
// The arithmetic is the same either way, bit for bit.
template <int MODE, bool FEAT = true, bool LO = true, bool BANDS = false, int RING = 0, bool HASQ = false>
__device__ __forceinline__ void epass8_body(const EParams<float> &P, long gid)
{
    constexpr int L = PBS_EPASS_LPT;
    constexpr int NSUB = 8 / L;
    constexpr bool CL = (MODE & MODE_CLOSE) != 0;
    constexpr bool OP = (MODE & MODE_OPEN) != 0;
    const int NA = (int)(P.NAPT / PBS_PT);
    const long NPB = P.NLINE / P.NAPT;
    const int pt = (int)(gid & 31);
    const long r = gid >> 5;
    const int grp = (int)(r % (P.NOCT * NSUB));   // line group: octet grp / NSUB, lines 8 oct + L sub + e
    const int oct = grp / NSUB, sub = grp % NSUB;
    const long pbk = r / (P.NOCT * NSUB);
    if (pbk >= NPB) return;
    const int nval = min(L, NA - 8 * oct - L * sub);   // lines of this group that exist (may be <= 0)
    const long S = P.NLINE;
    const long QS = (long)P.G * S;
    const long line0 = ((long)pbk * NA + 8 * oct + L * sub) * PBS_PT + pt;   // line of e = 0; e adds PBS_PT
    const long pq = pbk * PBS_PT + pt;
    const double rc = CL ? (double)P.rho_c[pq] : 0.0;
    const double ro = OP ? (double)P.rho_o[pq] : 0.0;
    const double dac = 0.5 * (double)P.h * rc, dao = 0.5 * (double)P.h * ro;
    const float ac = (float)dac, ao = (float)dao;
    float fin[L], fcl[L], fop[L], U0[L], U1[L], U2[L];
#pragma unroll
    for (int e = 0; e < L; ++e) fin[e] = fcl[e] = fop[e] = U0[e] = U1[e] = U2[e] = 0.f;
    float U0b[BANDS ? 4 : 1][L] = {}, U1b[BANDS ? 4 : 1][L] = {}, U2b[BANDS ? 4 : 1][L] = {};   // per-band scans
    // rounding residue of the BF16 scans carried from group g+1 into group g (hi-only products)
    float rcc[L] = {}, rco[L] = {};
    double ph0 = 0, ph1 = 0, ph2 = 0, injc = 0, injo = 0;
    float fic = 0, fio = 0, fme = 0, fmn = 0;
    const bool hasQ = RING ? HASQ : P.Q != nullptr, hasW = P.Wh != nullptr, hasL = LO && P.Wl != nullptr,
               feat = FEAT && P.inj_c != nullptr;
    const bool qbf = hasQ && P.Qb != nullptr;
    const int NAq = (NA + 3) & ~3;
    const long QSb = (long)P.G * NPB * NAq * PBS_PT;
    typedef unsigned short u16x4 __attribute__((ext_vector_type(4)));
    static_assert(L == 4, "the BF16 source is read as 4-line chunks");
    const long SB = (long)P.G * NPB * P.NOCT * (PBS_PT * 8);
    // ring loads: no branch (a line past the last node reads the last one's value, dropped at its use; a
    // group past the last one re-reads group 0)
    constexpr int R = RING ? RING : 1;
    float rx1[R][L], rx2[R][L];
    u16x4 rqc[R], rqo[R];
    const float *lp[L];
    const unsigned short *qp = nullptr;
    if constexpr (RING > 0) {
#pragma unroll
        for (int e = 0; e < L; ++e) lp[e] = P.psi + ((long)pbk * NA + min(8 * oct + L * sub + e, NA - 1)) * PBS_PT + pt;
        if constexpr (HASQ) qp = P.Qb + ((long)pbk * NAq + min(8 * oct + L * sub, NAq - L)) * PBS_PT + pt * L;
    }
    auto fetch = [&](int g, int u) {
        const long gc = max(g, 0);
#pragma unroll
        for (int e = 0; e < L; ++e) {
            rx1[u][e] = EP_LD(lp[e] + 2 * gc * S);
            rx2[u][e] = EP_LD(lp[e] + (2 * gc + 1) * S);
        }
        if constexpr (HASQ) {
            const unsigned short *q = qp + gc * NPB * NAq * PBS_PT;
            if (CL) rqc[u] = EP_LD(reinterpret_cast<const u16x4 *>(q));
            if (OP) rqo[u] = EP_LD(reinterpret_cast<const u16x4 *>(q + QSb));
        }
    };
    auto group = [&](const int g, const int u) {
#pragma clang fp contract(off)
        // every fused operation is written out: the variants of this pass (and the batched one) then give the
        // same bits whatever the compiler would contract in each
        const float sm = tab(P.Sm, g), sp = tab(P.Sp, g), kp = tab(P.kap, g);
        const float d11 = -(sm + kp), d12 = sm, d21 = -3.f * sp, d22 = -(fmaf(2.f, sm, sp) + kp);
        const float c1 = sp, c2 = 3.f * sp;
        const float mc11 = fmaf(-ac, d11, 1.f), mc12 = -ac * d12, mc21 = -ac * d21, mc22 = fmaf(-ac, d22, 1.f);
        const float mo11 = fmaf(-ao, d11, 1.f), mo12 = -ao * d12, mo21 = -ao * d21, mo22 = fmaf(-ao, d22, 1.f);
        const float ic = CL ? fast_rcp(fmaf(mc11, mc22, -(mc12 * mc21))) : 0.f;
        const float io = OP ? fast_rcp(fmaf(mo11, mo22, -(mo12 * mo21))) : 0.f;
        float *p1 = P.psi + (2L * g) * S + line0;
        float *p2 = p1 + S;
        float x1[L], x2[L], qc[L], qo[L];
        if constexpr (RING > 0) {
#pragma unroll
            for (int e = 0; e < L; ++e) {
                const bool v = e < nval;
                x1[e] = v ? rx1[u][e] : 0.f;
                x2[e] = v ? rx2[u][e] : 0.f;
                qc[e] = HASQ && CL && v ? bf16_to_f32(rqc[u][e]) : 0.f;
                qo[e] = HASQ && OP && v ? bf16_to_f32(rqo[u][e]) : 0.f;
            }
            fetch(g - RING, u);
        } else {
#pragma unroll
            for (int e = 0; e < L; ++e) {
                const bool v = e < nval;
                x1[e] = v ? EP_LD(&p1[e * PBS_PT]) : 0.f;
                x2[e] = v ? EP_LD(&p2[e * PBS_PT]) : 0.f;
                qc[e] = qo[e] = 0.f;
                if (hasQ && !qbf && v) {
                    const long o = (long)g * S + line0 + e * PBS_PT;
                    if (CL) qc[e] = EP_LD(&P.Q[o]);
                    if (OP) qo[e] = EP_LD(&P.Q[QS + o]);
                }
            }
            if (qbf && nval > 0) {
                // the BF16 source holds the thread's 4 lines of one cell as one 8-byte chunk
                const long o = (((long)g * NPB + pbk) * NAq + 8 * oct + L * sub) * PBS_PT + pt * L;
                if (CL) {
                    const u16x4 c = EP_LD(reinterpret_cast<const u16x4 *>(P.Qb + o));
#pragma unroll
                    for (int e = 0; e < L; ++e) qc[e] = e < nval ? bf16_to_f32(c[e]) : 0.f;
                }
                if (OP) {
                    const u16x4 c = EP_LD(reinterpret_cast<const u16x4 *>(P.Qb + QSb + o));
#pragma unroll
                    for (int e = 0; e < L; ++e) qo[e] = e < nval ? bf16_to_f32(c[e]) : 0.f;
                }
            }
        }
        const float w = tab(P.wc, g), dec = tab(P.wdec, g), idE = tab(P.invdE, g);
        double s0a = 0, s0b = 0, s1a = 0, s1b = 0, s2a = 0, s2b = 0, sqc = 0, sqo = 0;
        typedef unsigned short chunk_t __attribute__((ext_vector_type(L)));
        chunk_t hc, lc, ho, lo;
#pragma unroll
        for (int e = 0; e < L; ++e) {
            float y1 = x1[e], y2 = x2[e];
            if (CL) {
                const float f = fin[e] + fcl[e];
                const float r1 = fmaf(ac, fmaf(c1, f, fmaf(d12, x2[e], d11 * x1[e])) + qc[e], x1[e]);
                const float r2 = fmaf(ac, fmaf(c2, f, fmaf(d21, x1[e], d22 * x2[e])), x2[e]);
                y1 = fmaf(r1, mc22, -(mc12 * r2)) * ic;
                y2 = fmaf(mc11, r2, -(mc21 * r1)) * ic;
            }
            float z1 = y1, z2 = y2;
            if (OP) {
                const float f = (CL ? fcl[e] : fin[e]) + fop[e];
                const float r1 = fmaf(ao, fmaf(c1, f, fmaf(d12, y2, d11 * y1)) + qo[e], y1);
                const float r2 = fmaf(ao, fmaf(c2, f, fmaf(d21, y1, d22 * y2)), y2);
                z1 = fmaf(r1, mo22, -(mo12 * r2)) * io;
                z2 = fmaf(mo11, r2, -(mo21 * r1)) * io;
            }
            if (e < nval) {
                EP_ST(z1, &p1[e * PBS_PT]);
                EP_ST(z2, &p2[e * PBS_PT]);
            }
            if (CL) {
                s0a += (double)x1[e];
                s0b += (double)x2[e];
                sqc += (double)qc[e];
            }
            s1a += (double)y1;
            s1b += (double)y2;
            if (OP) {
                s2a += (double)z1;
                s2b += (double)z2;
                sqo += (double)qo[e];
            }
            if (hasW || feat) {
                if constexpr (BANDS) {
                    // the sum of one scan per band, each with its band's decay; group g feeds its own band
                    const int bg = tab(P.band, g);
                    U0[e] = U1[e] = U2[e] = 0.f;
#pragma unroll
                    for (int b = 0; b < 4; ++b)
                        if (b < P.NB) {
                            const float d = tab(P.wdecb, (long)b * P.G + g), wb = b == bg ? w : 0.f;
                            if (CL) U0[e] += (U0b[b][e] = fmaf(wb, x1[e], d * U0b[b][e]));
                            U1[e] += (U1b[b][e] = fmaf(wb, y1, d * U1b[b][e]));
                            if (OP) U2[e] += (U2b[b][e] = fmaf(wb, z1, d * U2b[b][e]));
                        }
                } else {
                    if (CL) U0[e] = fmaf(w, x1[e], dec * U0[e]);
                    U1[e] = fmaf(w, y1, dec * U1[e]);
                    if (OP) U2[e] = fmaf(dec, U2[e], w * z1);
                }
                const float uc = CL ? U0[e] + U1[e] : 0.f, uo = OP ? U1[e] + U2[e] : 0.f, vc = uc * idE;
                const float vo = uo * idE;
                if (hasL) {
                    const __bf16 bc = (__bf16)vc, bo = (__bf16)vo;
                    hc[e] = __builtin_bit_cast(unsigned short, bc);
                    ho[e] = __builtin_bit_cast(unsigned short, bo);
                    if constexpr (LO) {
                        lc[e] = __builtin_bit_cast(unsigned short, (__bf16)(vc - (float)bc));
                        lo[e] = __builtin_bit_cast(unsigned short, (__bf16)(vo - (float)bo));
                    }
                } else {
                    // only the rounded value enters the product: round with error feedback along the
                    // groups, so that the line's rounding errors telescope in the number and energy of
                    // the re-emitted protons instead of adding up
                    const float tc = fmaf(uc, idE, rcc[e]), to = fmaf(uo, idE, rco[e]);
                    const __bf16 bc = (__bf16)tc, bo = (__bf16)to;
                    hc[e] = __builtin_bit_cast(unsigned short, bc);
                    ho[e] = __builtin_bit_cast(unsigned short, bo);
                    rcc[e] = tc - (float)bc;
                    rco[e] = to - (float)bo;
                }
                if (feat) {
                    const float wi = (float)tab(P.dInj, g);
                    if (CL) fic = fmaf(wi, vc, fic);
                    if (OP) {
                        fio = fmaf(wi, vo, fio);
                        fme += fmaf((float)tab(P.wmom, g), z1, (float)tab(P.wmom, 2L * P.G + g) * z2);
                        fmn = fmaf((float)tab(P.wmom, (long)P.G + g), z1, fmn);
                    }
                }
            }
            fin[e] = x1[e] - x2[e];
            fcl[e] = y1 - y2;
            fop[e] = z1 - z2;
        }
        // deposit functional (FP64), summed over the lines: A, B depend on the energy group only
        const double A = tab(P.dA, g), B = tab(P.dB, g);
        if (CL) ph0 += fma(A, s0a, B * s0b);
        ph1 += fma(A, s1a, B * s1b);
        if (OP) ph2 += fma(A, s2a, B * s2b);
        if (g == 0) {
            if (CL) ph0 = fma(P.dBot, s0a - s0b, ph0);
            ph1 = fma(P.dBot, s1a - s1b, ph1);
            if (OP) ph2 = fma(P.dBot, s2a - s2b, ph2);
        }
        if (hasQ) {
            const double wi = tab(P.dInj, g);
            if (CL) injc = fma(wi, sqc, injc);
            if (OP) injo = fma(wi, sqo, injo);
        }
        if (hasW) {
            const long ob = (((long)g * NPB + pbk) * P.NOCT + oct) * (PBS_PT * 8) + pt * 8 + L * sub;
            if (CL) *reinterpret_cast<chunk_t *>(P.Wh + ob) = hc;
            if (OP) *reinterpret_cast<chunk_t *>(P.Wh + SB + ob) = ho;
            if constexpr (LO) {
                if (hasL) {
                    if (CL) *reinterpret_cast<chunk_t *>(P.Wl + ob) = lc;
                    if (OP) *reinterpret_cast<chunk_t *>(P.Wl + SB + ob) = lo;
                }
            }
        }
    };
    if constexpr (RING > 0) {
#pragma unroll
        for (int u = 0; u < R; ++u) fetch(P.G - 1 - u, u);
        int g0 = P.G - 1;
        for (; g0 >= R - 1; g0 -= R) {
#pragma unroll
            for (int u = 0; u < R; ++u) group(g0 - u, u);
        }
#pragma unroll
        for (int u = 0; u < R - 1; ++u)
            if (g0 - u >= 0) group(g0 - u, u);
    } else {
        for (int g = P.G - 1; g >= 0; --g) group(g, 0);
    }
    const long slot = ((long)pbk * NA + grp) * PBS_PT + pt;
    if (CL) P.dep_c[slot] = dac * (ph0 + ph1 - injc) * P.scale;
    if (OP) P.dep_o[slot] = dao * (ph1 + ph2 - injo) * P.scale;
    if (feat) {
        if (CL) P.inj_c[slot] = dac * (double)fic * P.scale;
        if (OP) {
            P.inj_o[slot] = dao * (double)fio * P.scale;
            P.mom_e[slot] = (double)fme * P.scale;
            P.mom_n[slot] = (double)fmn * P.scale;
        }
    }
}

// 5 waves per SIMD for the plain kernels (96 VGPRs, a few spilled registers): measured faster than 4
// waves without spills
// Minimum waves per SIMD of the plain energy passes (compile-time knob).  At 5 the compiler held the
// pair-mode kernel to 96 VGPRs and spilled 80 bytes per thread, reloaded in every group step; at 4 it
// takes 114 VGPRs with no scratch (config-2 energy pass 2.94 -> 2.71 ms per launch, config 3 -1 %).
#ifndef EP_WPE
#define EP_WPE 4
#endif
template <int MODE, bool FEAT, bool LO, bool BANDS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(FEAT || BANDS ? 1 : EP_WPE))) void epass8_kernel(
    EParams<float> P)
{
    epass8_body<MODE, FEAT, LO, BANDS>(P, (long)blockIdx.x * 256 + threadIdx.x);
}

template <bool FEAT, bool LO, bool BANDS = false>
static void launch_epass8_t(const EParams<float> &P, int mode, unsigned nb, hipStream_t st)
{
    if (mode == MODE_PAIR)
        hipLaunchKernelGGL((epass8_kernel<MODE_PAIR, FEAT, LO, BANDS>), dim3(nb), dim3(256), 0, st, P);
    else if (mode == MODE_OPEN)
        hipLaunchKernelGGL((epass8_kernel<MODE_OPEN, FEAT, LO, BANDS>), dim3(nb), dim3(256), 0, st, P);
    else
        hipLaunchKernelGGL((epass8_kernel<MODE_CLOSE, FEAT, LO, BANDS>), dim3(nb), dim3(256), 0, st, P);
}

// Ring of the 4-line pass and the grids that take it.  Up to EP8_RING_WAVES waves (two rounds of the plain
// kernel's 4 waves per SIMD) the chip is short of loads in flight and the ring wins: 279 -> 146 us per launch at
// 32 x 32 cells, 15 x 15 angles, 131 groups (928 waves); 446 -> 353 us at 45 x 70, 19 x 19, 75 groups (4554);
// 403 -> 354 us at 40 x 40, 31 x 31, 64 groups (6050).  At 64 x 64 cells and 31 x 31 angles (15488 waves) the two
// take the same time.  A ring of 3 is slower than 2 everywhere (fewer waves).
constexpr int EP8_RING = 2;
constexpr long EP8_RING_WAVES = 8192;
template <int MODE, bool FEAT, bool BANDS, bool HASQ>
__global__ __launch_bounds__(256) void epass8_ring_kernel(EParams<float> P)
{
    epass8_body<MODE, FEAT, false, BANDS, EP8_RING, HASQ>(P, (long)blockIdx.x * 256 + threadIdx.x);
}

template <bool FEAT, bool BANDS, bool HASQ>
static void launch_epass8_ring_t(const EParams<float> &P, int mode, unsigned nb, hipStream_t st)
{
    if (mode == MODE_PAIR)
        hipLaunchKernelGGL((epass8_ring_kernel<MODE_PAIR, FEAT, BANDS, HASQ>), dim3(nb), dim3(256), 0, st, P);
    else if (mode == MODE_OPEN)
        hipLaunchKernelGGL((epass8_ring_kernel<MODE_OPEN, FEAT, BANDS, HASQ>), dim3(nb), dim3(256), 0, st, P);
    else
        hipLaunchKernelGGL((epass8_ring_kernel<MODE_CLOSE, FEAT, BANDS, HASQ>), dim3(nb), dim3(256), 0, st, P);
}

hipError_t launch_epass8(const EParams<float> &P, int mode, hipStream_t st)
{
    const long nthreads = (P.NLINE / P.NAPT) * P.NOCT * (8 / PBS_EPASS_LPT) * PBS_PT;
    const unsigned nb = (unsigned)((nthreads + 255) / 256);
    if (P.NB > 4) return hipErrorInvalidValue;
    if (P.NB > 1 && P.inj_c != nullptr) return hipErrorInvalidValue;   // banded nuclear data: no surrogate records
    if (P.inj_c == nullptr && P.Wl == nullptr && (P.Q == nullptr || P.Qb != nullptr) &&
        epass_pipe_blocks<float, 4>(P) <= EP_PIPE_BLOCKS)
        return launch_epass_pipe<float, 4>(P, mode, st);
    if (nthreads / 64 <= EP8_RING_WAVES && P.Wl == nullptr && (P.Q == nullptr || P.Qb != nullptr)) {
        const bool q = P.Q != nullptr;
        if (P.NB > 1) {
            if (q) launch_epass8_ring_t<false, true, true>(P, mode, nb, st);
            else launch_epass8_ring_t<false, true, false>(P, mode, nb, st);
        } else if (P.inj_c != nullptr) {
            if (q) return hipErrorInvalidValue;   // the records are the primaries', which have no source
            launch_epass8_ring_t<true, false, false>(P, mode, nb, st);
        } else {
            if (q) launch_epass8_ring_t<false, false, true>(P, mode, nb, st);
            else launch_epass8_ring_t<false, false, false>(P, mode, nb, st);
        }
        return hipGetLastError();
    }
    if (P.NB > 1) {
        if (P.Wl != nullptr)
            launch_epass8_t<false, true, true>(P, mode, nb, st);
        else
            launch_epass8_t<false, false, true>(P, mode, nb, st);
    } else if (P.inj_c != nullptr)
        launch_epass8_t<true, true>(P, mode, nb, st);
    else if (P.Wl != nullptr)
        launch_epass8_t<false, true>(P, mode, nb, st);
    else
        launch_epass8_t<false, false>(P, mode, nb, st);
    return hipGetLastError();
}

// ----------------------------------------------------------------- energy pass as a pipeline of waves
// The smallest grids hold fewer line groups than the chip has SIMDs, and a wave's own instruction stream is what
// bounds the sweep there (about 120 vector instructions a group for one line, 370 for four).  A block therefore
// runs the sweep of 64 threads as four waves, each with a quarter of the work, two to four groups (a chunk) behind
// the one before it, handing values on through LDS:
//   0  loads the fluence and the closing source, solves the closing half-step
//   1  loads the opening source, solves the opening half-step, stores the fluence
//   2  scans the three states for the next generation's source
//   3  sums the FP64 deposits
// The arithmetic of a line is that of the passes above (for four lines per thread bit for bit).  One barrier per
// chunk, which waits for LDS only: loads and stores stay in flight across it.  Three chunk buffers: one being
// written by each of waves 0 and 1, one being read by 2 and 3.
// Measured, us per launch, before -> after: 4 x 4 cells, 11 x 11 angles, 60 groups 27 -> 19 (FP64 31 -> 22); 16 x 16, 7 x 7, 48
// 24 -> 18 (FP64 26 -> 20); 6 x 6, 15 x 15, 60 59 -> 37; 16 x 16, 15 x 15, 131 125 -> 74; 24 x 24, 15 x 15, 131 133 -> 105.
template <typename T, int L>
struct EPipe {
    static constexpr int C = L == 1 ? 4 : 2;   // groups per chunk
    static constexpr int PF = 2;               // chunks loaded ahead
    typedef T V __attribute__((ext_vector_type(L)));
    struct Group { V x1[64], x2[64], y1[64], y2[64], z1[64], z2[64], qc[64], qo[64]; };
};

__device__ __forceinline__ void epipe_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Three per-group tables of a chunk's C groups in the lanes of one vector load, read back by lane: scalar loads share
// their counter with LDS, whose every wait would then wait for them.
template <typename X, int C>
struct EPipeTab {
    const X *p;
    int top;
    X v;
    __device__ __forceinline__ EPipeTab(const X *a, const X *b, const X *c, int G, int lane)
        : p(lane < C ? a : lane < 2 * C ? b : c), top(G - 1 - lane % C), v(X(0))
    {
    }
    __device__ __forceinline__ void fetch(int n) { v = p[max(top - n * C, 0)]; }
};

template <typename T, int L, int MODE, bool BANDS, bool HASQ>
__global__ __launch_bounds__(256) void epass_pipe_kernel(EParams<T> P)
{
    using E = EPipe<T, L>;
    using V = typename E::V;
    constexpr int C = E::C, PF = E::PF;
    constexpr bool CL = (MODE & MODE_CLOSE) != 0, OP = (MODE & MODE_OPEN) != 0;
    typedef unsigned short u16x4 __attribute__((ext_vector_type(4)));
    __shared__ typename E::Group buf[3][C];
    const int lane = threadIdx.x & 63, role = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int G = P.G, NA = (int)(P.NAPT / PBS_PT);
    const long S = P.NLINE, NPB = S / P.NAPT;
    // this thread's lines: L = 1 the line itself, L = 4 a line group of an octet (as in the 4-line pass)
    const long gid = (long)blockIdx.x * 64 + lane;
    const int pt = (int)(gid & 31);
    const long rows = L == 1 ? NPB * NA : NPB * P.NOCT * 2;
    // L = 1: the last block's missing row repeats the last one (same wave, same values); L = 4: rows are even
    const long r = min(gid >> 5, rows - 1);
    const int per = L == 1 ? NA : P.NOCT * 2, grp = (int)(r % per);
    const long pbk = r / per;
    const int nval = min(L, NA - L * grp);   // lines of this thread that exist
    const long pq = pbk * PBS_PT + pt;
    const double rc = CL ? (double)P.rho_c[pq] : 0.0, ro = OP ? (double)P.rho_o[pq] : 0.0;
    const double dac = 0.5 * (double)P.h * rc, dao = 0.5 * (double)P.h * ro;
    const T ac = (T)dac, ao = (T)dao;
    const int nch = (G + C - 1) / C, NI = (nch + 2 + PF - 1) / PF * PF;   // chunks; barriers of every wave
    // line e of this thread (one past the last node reads the last one's and is dropped)
    auto line_of = [&](int e) { return ((long)pbk * NA + min(L * grp + e, NA - 1)) * PBS_PT + pt; };
    const int NAq = (NA + 3) & ~3;
    const long QS = (long)G * S, QSb = (long)G * NPB * NAq * PBS_PT;
    auto top = [&](int n, int u) { return G - 1 - (n * C + u); };   // group u of chunk n (< 0 past the last)

    // one half-step: wave 0 from the fluence, wave 1 from wave 0's result
    auto half_step = [&](auto first) {
        constexpr bool closing = decltype(first)::value, ACT = closing ? CL : OP;
        const T ah = closing ? ac : ao;
        V rx1[PF][C], rx2[PF][C];
        std::conditional_t<L == 1, V, u16x4> rq[PF][C];
        auto fetch = [&](int n, int sl) {
#pragma unroll
            for (int u = 0; u < C; ++u) {
                const long g = max(top(n, u), 0);
                if constexpr (closing) {
#pragma unroll
                    for (int e = 0; e < L; ++e) {
                        const T *p = P.psi + 2 * g * S + line_of(e);
                        rx1[sl][u][e] = p[0];
                        rx2[sl][u][e] = p[S];
                    }
                }
                if constexpr (HASQ && ACT) {
                    if constexpr (L == 1)
                        rq[sl][u] = P.Q[(closing ? 0L : QS) + g * S + line_of(0)];
                    else
                        rq[sl][u] = *reinterpret_cast<const u16x4 *>(
                            P.Qb + (closing ? 0L : QSb) + ((g * NPB + pbk) * NAq + min(L * grp, NAq - L)) * PBS_PT + pt * L);
                }
            }
        };
        V fi = V(T(0)), fo = V(T(0));   // psi1 - psi2 of the group above: the state before this half-step, after it
        EPipeTab<T, C> tb(P.Sm, P.Sp, P.kap, G, lane);
        auto chunk = [&](int n, int sl, auto whole) {
            constexpr bool FULL = decltype(whole)::value;   // no group past the last one
            typename E::Group *B = buf[n % 3];
            T cm[C], cp[C], ck[C];
#pragma unroll
            for (int u = 0; u < C; ++u)
                cm[u] = lane_of(tb.v, u), cp[u] = lane_of(tb.v, C + u), ck[u] = lane_of(tb.v, 2 * C + u);
            tb.fetch(n + 1);
            V q[C], a1[C], a2[C];
#pragma unroll
            for (int u = 0; u < C; ++u) {
                if constexpr (closing) {
#pragma unroll
                    for (int e = 0; e < L; ++e) {
                        a1[u][e] = e < nval ? rx1[sl][u][e] : T(0);
                        a2[u][e] = e < nval ? rx2[sl][u][e] : T(0);
                    }
                } else {
                    a1[u] = B[u].y1[lane];
                    a2[u] = B[u].y2[lane];
                }
                q[u] = V(T(0));
                if constexpr (HASQ && ACT) {
#pragma unroll
                    for (int e = 0; e < L; ++e) {
                        if constexpr (L == 1) q[u][e] = rq[sl][u][e];
                        else q[u][e] = e < nval ? (T)bf16_to_f32(rq[sl][u][e]) : T(0);
                    }
                }
            }
            fetch(n + PF, sl);
#pragma unroll
            for (int u = 0; u < C; ++u) {
                const int g = top(n, u);
                if (!FULL && g < 0) break;
                V b1 = a1[u], b2 = a2[u];
                if constexpr (ACT) {
                    ECoef<T> K;
                    K.set(cm[u], cp[u], ck[u], ah);
#pragma unroll
                    for (int e = 0; e < L; ++e) {
                        T s1, s2;
                        K.solve(a1[u][e], a2[u][e], fi[e] + fo[e], q[u][e], s1, s2);
                        b1[e] = s1;
                        b2[e] = s2;
                    }
                }
                fi = a1[u] - a2[u];
                fo = b1 - b2;
                if constexpr (closing) {
                    B[u].x1[lane] = a1[u];
                    B[u].x2[lane] = a2[u];
                    B[u].y1[lane] = b1;
                    B[u].y2[lane] = b2;
                    if constexpr (HASQ && ACT) B[u].qc[lane] = q[u];
                } else {
#pragma unroll
                    for (int e = 0; e < L; ++e)
                        if (e < nval) {
                            T *p = P.psi + 2L * g * S + line_of(e);
                            p[0] = b1[e];
                            p[S] = b2[e];
                        }
                    B[u].z1[lane] = b1;
                    B[u].z2[lane] = b2;
                    if constexpr (HASQ && ACT) B[u].qo[lane] = q[u];
                }
            }
        };
        tb.fetch(0);
#pragma unroll
        for (int k = 0; k < PF; ++k) fetch(k, k);
        if constexpr (!closing) epipe_barrier();   // one chunk behind wave 0
        for (int n0 = 0; n0 < NI; n0 += PF) {
#pragma unroll
            for (int k = 0; k < PF; ++k) {
                if (n0 + k < G / C) chunk(n0 + k, k, std::true_type());
                else if (n0 + k < nch) chunk(n0 + k, k, std::false_type());
                if (closing || n0 + k < NI - 1) epipe_barrier();
            }
        }
    };
    if (role == 0) {
        half_step(std::true_type());
    } else if (role == 1) {
        half_step(std::false_type());
    } else if (role == 2) {
        const bool hasW = L == 1 ? P.W != nullptr : P.Wh != nullptr;
        V U0 = V(T(0)), U1 = V(T(0)), U2 = V(T(0));
        V U0b[BANDS ? 4 : 1], U1b[BANDS ? 4 : 1], U2b[BANDS ? 4 : 1], ec = V(T(0)), eo = V(T(0));
#pragma unroll
        for (int b = 0; b < (BANDS ? 4 : 1); ++b) U0b[b] = U1b[b] = U2b[b] = V(T(0));
        const long SB = (long)G * NPB * P.NOCT * (PBS_PT * 8);
        EPipeTab<T, C> tb(P.wc, P.wdec, P.invdE, G, lane);
        auto chunk = [&](int n, auto whole) {
#pragma clang fp contract(off)
            constexpr bool FULL = decltype(whole)::value;
            const typename E::Group *B = buf[n % 3];
            T cw[C], cd[C], ci[C];
#pragma unroll
            for (int u = 0; u < C; ++u)
                cw[u] = lane_of(tb.v, u), cd[u] = lane_of(tb.v, C + u), ci[u] = lane_of(tb.v, 2 * C + u);
            tb.fetch(n + 1);
#pragma unroll
            for (int u = 0; u < C; ++u) {
                const int g = top(n, u);
                if (!FULL && g < 0) break;
                const V x = B[u].x1[lane], y = B[u].y1[lane], z = B[u].z1[lane];
                unsigned short hc[L], ho[L];
#pragma unroll
                for (int e = 0; e < L; ++e) {
                    if constexpr (BANDS) {
                        const int bg = tab(P.band, g);
                        U0[e] = U1[e] = U2[e] = T(0);
#pragma unroll
                        for (int b = 0; b < 4; ++b)
                            if (b < P.NB) {
                                const T d = tab(P.wdecb, (long)b * G + g), wb = b == bg ? cw[u] : T(0);
                                if (CL) U0[e] += (U0b[b][e] = fma(wb, x[e], d * U0b[b][e]));
                                U1[e] += (U1b[b][e] = fma(wb, y[e], d * U1b[b][e]));
                                if (OP) U2[e] += (U2b[b][e] = fma(wb, z[e], d * U2b[b][e]));
                            }
                    } else {
                        if (CL) U0[e] = fma(cw[u], x[e], cd[u] * U0[e]);
                        U1[e] = fma(cw[u], y[e], cd[u] * U1[e]);
                        if (OP) U2[e] = fma(cd[u], U2[e], cw[u] * z[e]);
                    }
                    const T uc = CL ? U0[e] + U1[e] : T(0), uo = OP ? U1[e] + U2[e] : T(0);
                    if constexpr (L == 1) {
                        if (CL) P.W[(long)g * S + line_of(0)] = uc * ci[u];
                        if (OP) P.W[QS + (long)g * S + line_of(0)] = uo * ci[u];
                    } else {
                        // rounded with error feedback along the groups, as in the 4-line pass
                        const float tc = fma(uc, ci[u], ec[e]), to = fma(uo, ci[u], eo[e]);
                        const __bf16 bc = (__bf16)tc, bo = (__bf16)to;
                        hc[e] = __builtin_bit_cast(unsigned short, bc);
                        ho[e] = __builtin_bit_cast(unsigned short, bo);
                        ec[e] = tc - (float)bc;
                        eo[e] = to - (float)bo;
                    }
                }
                if constexpr (L == 4) {
                    const long ob = (((long)g * NPB + pbk) * P.NOCT + grp / 2) * (PBS_PT * 8) + pt * 8 + L * (grp % 2);
                    if (CL) *reinterpret_cast<u16x4 *>(P.Wh + ob) = u16x4{hc[0], hc[1], hc[2], hc[3]};
                    if (OP) *reinterpret_cast<u16x4 *>(P.Wh + SB + ob) = u16x4{ho[0], ho[1], ho[2], ho[3]};
                }
            }
        };
        tb.fetch(0);
        epipe_barrier();
        epipe_barrier();   // two chunks behind wave 0
        for (int n = 0; n < NI - 2; ++n) {
            if (hasW && n < G / C) chunk(n, std::true_type());
            else if (hasW && n < nch) chunk(n, std::false_type());
            epipe_barrier();
        }
    } else {
        double ph0 = 0, ph1 = 0, ph2 = 0, injc = 0, injo = 0;
        EPipeTab<double, C> tb(P.dA, P.dB, P.dInj, G, lane);
        auto sum = [&](const V &v) {
            double s = 0;
#pragma unroll
            for (int e = 0; e < L; ++e) s += (double)v[e];
            return s;
        };
        auto chunk = [&](int n, auto whole) {
#pragma clang fp contract(off)
            constexpr bool FULL = decltype(whole)::value;
            const typename E::Group *B = buf[n % 3];
            double cA[C], cB[C], cw[C];
#pragma unroll
            for (int u = 0; u < C; ++u)
                cA[u] = lane_of(tb.v, u), cB[u] = lane_of(tb.v, C + u), cw[u] = lane_of(tb.v, 2 * C + u);
            tb.fetch(n + 1);
#pragma unroll
            for (int u = 0; u < C; ++u) {
                const int g = top(n, u);
                if (!FULL && g < 0) break;
                const double s0a = sum(B[u].x1[lane]), s0b = sum(B[u].x2[lane]), s1a = sum(B[u].y1[lane]),
                             s1b = sum(B[u].y2[lane]), s2a = sum(B[u].z1[lane]), s2b = sum(B[u].z2[lane]);
                if (CL) ph0 += fma(cA[u], s0a, cB[u] * s0b);
                ph1 += fma(cA[u], s1a, cB[u] * s1b);
                if (OP) ph2 += fma(cA[u], s2a, cB[u] * s2b);
                if (g == 0) {
                    if (CL) ph0 = fma(P.dBot, s0a - s0b, ph0);
                    ph1 = fma(P.dBot, s1a - s1b, ph1);
                    if (OP) ph2 = fma(P.dBot, s2a - s2b, ph2);
                }
                if constexpr (HASQ) {
                    if (CL) injc = fma(cw[u], sum(B[u].qc[lane]), injc);
                    if (OP) injo = fma(cw[u], sum(B[u].qo[lane]), injo);
                }
            }
        };
        tb.fetch(0);
        epipe_barrier();
        epipe_barrier();
        for (int n = 0; n < NI - 2; ++n) {
            if (n < G / C) chunk(n, std::true_type());
            else if (n < nch) chunk(n, std::false_type());
            epipe_barrier();
        }
        const long slot = L == 1 ? line_of(0) : ((long)pbk * NA + grp) * PBS_PT + pt;
        if (CL) P.dep_c[slot] = dac * (ph0 + ph1 - injc) * P.scale;
        if (OP) P.dep_o[slot] = dao * (ph1 + ph2 - injo) * P.scale;
    }
}

// blocks of the pipeline form of a grid (64 threads each)
template <typename T, int L>
static long epass_pipe_blocks(const EParams<T> &P)
{
    const long rows = L == 1 ? P.NLINE / PBS_PT : P.NLINE / P.NAPT * P.NOCT * 2;
    return (rows * PBS_PT + 63) / 64;
}
template <typename T, int L, bool BANDS, bool HASQ>
static void launch_epass_pipe_t(const EParams<T> &P, int mode, hipStream_t st)
{
    const dim3 nb((unsigned)(epass_pipe_blocks<T, L>(P)));
    if (mode == MODE_PAIR)
        hipLaunchKernelGGL((epass_pipe_kernel<T, L, MODE_PAIR, BANDS, HASQ>), nb, dim3(256), 0, st, P);
    else if (mode == MODE_OPEN)
        hipLaunchKernelGGL((epass_pipe_kernel<T, L, MODE_OPEN, BANDS, HASQ>), nb, dim3(256), 0, st, P);
    else
        hipLaunchKernelGGL((epass_pipe_kernel<T, L, MODE_CLOSE, BANDS, HASQ>), nb, dim3(256), 0, st, P);
}
template <typename T, int L>
static hipError_t launch_epass_pipe(const EParams<T> &P, int mode, hipStream_t st)
{
    if (P.NB > 1) {
        if (P.Q) launch_epass_pipe_t<T, L, true, true>(P, mode, st);
        else launch_epass_pipe_t<T, L, true, false>(P, mode, st);
    } else {
        if (P.Q) launch_epass_pipe_t<T, L, false, true>(P, mode, st);
        else launch_epass_pipe_t<T, L, false, false>(P, mode, st);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------- transport pass
// Superbee-limited face slope without division: delta = Dface * eta(Dup / Dface).
// max(min(2|u|, |f|), min(|u|, 2|f|)) is the median of |u|, |f| and 2 min(|u|, |f|) (exact: doubling, min and
// max do not round); it is 0 when either difference is, so the sign test needs only the two sign bits.
template <typename T>
__device__ __forceinline__ T superbee_slope(T dup, T dface)
{
    const T au = fabs(dup), af = fabs(dface);
    if constexpr (sizeof(T) == 4) {
        const float v = __builtin_amdgcn_fmed3f(au, af, 2.f * fminf(au, af));
        // v <= 2|dup|, so clamping copysign(v, dface) between 0 and 2 dup keeps it when the two differences
        // agree in sign and gives 0 when they do not (no compare, no condition register)
        return __builtin_amdgcn_fmed3f(copysignf(v, dface), 0.f, 2.f * dup);
    } else {
        const T v = fmin(fmax(au, af), T(2) * fmin(au, af));
        return signbit(dup) == signbit(dface) ? copysign(v, dface) : T(0);
    }
}

// The transport sweep reads and writes every plane once: non-temporal loads and stores (both are needed:
// either alone measured no gain; together 12.6 -> 12.1 ms per depth step of a 64 x 64-cell, 31 x 31-angle,
// 128-group, 4-generation beam, 5.3 TB/s).
#define TP_LD(p) __builtin_nontemporal_load(p)
#define TP_ST(v, p) __builtin_nontemporal_store(v, p)
template <typename T, int NSEG>
__device__ __forceinline__ void tpass_body(const TParams<T> &P, long plane)
{
    const int lane = threadIdx.x & 63;
    if (plane >= P.nplanes) return;   // uniform per wave
    const int a = (int)(plane % P.NA);
    const long slab = plane / P.NA;
    const T cx = P.theta[a / P.m], cy = P.theta[a % P.m];
    const bool mx = cx < T(0), my = cy < T(0);   // sweep frames mirrored so the velocity is >= 0
    const T ax = fabs(cx) * P.h_half_over_dx, ay = fabs(cy) * P.h_half_over_dy;
    const T idiag = T(1) / (T(1) + ax + ay);
    const T cq = ay * idiag;
    T *base = P.psi + slab * P.NLINE + (long)a * PBS_PT;
    const long NAPT = (long)P.NA * PBS_PT;
    const int nx = P.nx, ny = P.ny;

    int qcol[NSEG];
    bool valid[NSEG];
#pragma unroll
    for (int s = 0; s < NSEG; ++s) {
        const int qq = s * 64 + lane;
        valid[s] = qq < ny;
        qcol[s] = my ? ny - 1 - qq : qq;
    }
    // powers of the scan multiplier: cp[i] = cq^(2^i); cl = cq^(lane+1)
    T cp[7];
    cp[0] = cq;
#pragma unroll
    for (int i = 1; i < 7; ++i) cp[i] = cp[i - 1] * cp[i - 1];
    T cl = T(1);
#pragma unroll
    for (int i = 0; i < 7; ++i)
        if (((lane + 1) >> i) & 1) cl *= cp[i];

    auto load_row = [&](int r, T (&v)[NSEG]) {
        const int p = mx ? nx - 1 - r : r;
#pragma unroll
        for (int s = 0; s < NSEG; ++s) {
            T x = T(0);
            if (r < nx && valid[s]) {
                const long pq = (long)p * ny + qcol[s];
                x = TP_LD(&base[(pq / PBS_PT) * NAPT + (pq % PBS_PT)]);
            }
            v[s] = x;
        }
    };

    T pm1[NSEG], p0[NSEG], p1[NSEG], p2[NSEG], dxm[NSEG], ym1[NSEG];
#pragma unroll
    for (int s = 0; s < NSEG; ++s) pm1[s] = dxm[s] = ym1[s] = T(0);
    load_row(0, p0);
    load_row(1, p1);
    for (int r = 0; r < nx; ++r) {
        load_row(r + 2, p2);
        T left[NSEG], dyp[NSEG];
#pragma unroll
        for (int s = 0; s < NSEG; ++s) {
            const T up = __shfl_up(p0[s], 1);
            const T dn = __shfl_down(p0[s], 1);
            const T prev_last = s > 0 ? __shfl(p0[s > 0 ? s - 1 : 0], 63) : T(0);
            const T next_first = s + 1 < NSEG ? __shfl(p0[s + 1 < NSEG ? s + 1 : 0], 0) : T(0);
            left[s] = lane == 0 ? prev_last : up;
            const T right = lane == 63 ? next_first : dn;
            dyp[s] = superbee_slope(p0[s] - left[s], right - p0[s]);
        }
        T b[NSEG];
#pragma unroll
        for (int s = 0; s < NSEG; ++s) {
            const T up = __shfl_up(dyp[s], 1);
            const T prev_last = s > 0 ? __shfl(dyp[s > 0 ? s - 1 : 0], 63) : T(0);
            const T dym = lane == 0 ? prev_last : up;
            const T dxp = superbee_slope(p0[s] - pm1[s], p1[s] - p0[s]);
            const T R = p0[s] - ax * ((p0[s] - pm1[s]) + (dxp - dxm[s])) - ay * ((p0[s] - left[s]) + (dyp[s] - dym));
            b[s] = (R + ax * ym1[s]) * idiag;
            dxm[s] = dxp;
        }
        // implicit recurrence along the row: y_q = b_q + cq * y_{q-1}
        T carry = T(0);
        const int p = mx ? nx - 1 - r : r;
#pragma unroll
        for (int s = 0; s < NSEG; ++s) {
            T y = b[s];
#pragma unroll
            for (int i = 0; i < 6; ++i) {
                const int d = 1 << i;
                const T t = __shfl_up(y, d);
                if (lane >= d) y += cp[i] * t;
            }
            y += cl * carry;
            carry = __shfl(y, 63);
            ym1[s] = y;
            if (valid[s]) {
                const long pq = (long)p * ny + qcol[s];
                TP_ST(y, &base[(pq / PBS_PT) * NAPT + (pq % PBS_PT)]);
            }
        }
#pragma unroll
        for (int s = 0; s < NSEG; ++s) {
            pm1[s] = p0[s];
            p0[s] = p1[s];
            p1[s] = p2[s];
        }
    }
}

template <typename T, int NSEG>
__global__ __launch_bounds__(256) void tpass_kernel(TParams<T> P)
{
    tpass_body<T, NSEG>(P, (long)blockIdx.x * 4 + (threadIdx.x >> 6));
}

// The sweeps below move neighbours by DPP (wave_shr/shl:1 in y) and solve a row by a row_shr / row_bcast affine scan.
// All lanes written, lanes without a source read 0: the form the compiler folds into the DPP operand of the
// consuming VALU op (a row-scan step becomes one v_fmac_f32_dpp).
template <int CTRL>
__device__ __forceinline__ float dpp_z(float x)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), CTRL, 0xF, 0xF, true));
}
// DPP controls (GFX9): row_shr:n = 0x110 + n, wave_shl:1 = 0x130, wave_shr:1 = 0x138,
// row_bcast:15 = 0x142, row_bcast:31 = 0x143.  Lanes without a source receive 0 (the ghost value).

// One step of a row scan, y += c * y[source lane of the DPP pattern], as a single v_fmac_f32_dpp (rows
// outside the row mask keep y; lanes without a source read 0 and keep y).  The compiler does not fold a
// DPP move into a multiply-accumulate (a move plus an FMA per step), so the step is written out; the
// leading s_nop gives the two wait states a DPP read needs after a VALU write of its source.  Only used
// where the whole wave is active.
#define PBS_FMAC_DPP(y, c, ctrl, rmask) \
    asm volatile("s_nop 1\n\tv_fmac_f32_dpp %0, %0, %1 " ctrl " row_mask:" rmask " bank_mask:0xf bound_ctrl:1" \
                 : "+v"(y) : "v"(c))

// y_q = b_q + c y_{q-1} within each 16-lane row: Kogge-Stone over distances 1, 2, 4, 8 (multipliers c^d)
__device__ __forceinline__ void scan_rows16(float &y, float c1, float c2, float c4, float c8)
{
    PBS_FMAC_DPP(y, c1, "row_shr:1", "0xf");
    PBS_FMAC_DPP(y, c2, "row_shr:2", "0xf");
    PBS_FMAC_DPP(y, c4, "row_shr:4", "0xf");
    PBS_FMAC_DPP(y, c8, "row_shr:8", "0xf");
}
// ... then lane 15 of rows 0 and 2 into rows 1 and 3 (m16 = c^((lane & 15) + 1)) ...
__device__ __forceinline__ void scan_join32(float &y, float m16) { PBS_FMAC_DPP(y, m16, "row_bcast:15", "0xa"); }
// ... then lane 31 into rows 2 and 3 (m32 = c^((lane & 31) + 1))
__device__ __forceinline__ void scan_join64(float &y, float m32) { PBS_FMAC_DPP(y, m32, "row_bcast:31", "0xc"); }
// two wait states after the last scan step, for any DPP read of y that the compiler places next
__device__ __forceinline__ void scan_done() { asm volatile("s_nop 1"); }

constexpr int TPASS_PF = 8;   // rows of the row-affine sweep loaded ahead (nx must be a multiple)

// Same sweep when ny is 32 or 64 and nx a multiple of TPASS_PF: a lane's address is affine in the row
// (row stride = ny/32 lateral tiles), so each row costs one pointer increment and no guards; lanes
// beyond ny (ny = 32) read a clamped in-range column and are zeroed.
template <int NY>
__device__ __forceinline__ void tpass_affine_body(const TParams<float> &P, long plane)
{
    if (plane >= P.nplanes) return;   // uniform per wave
    const int lane = threadIdx.x & 63;
    const int a = (int)(plane % P.NA);
    const long slab = plane / P.NA;
    const float cx = P.theta[a / P.m], cy = P.theta[a % P.m];
    const bool mx = cx < 0.f, my = cy < 0.f;
    const float ax = fabsf(cx) * P.h_half_over_dx, ay = fabsf(cy) * P.h_half_over_dy;
    const float idiag = 1.f / (1.f + ax + ay);
    const float cq = ay * idiag;
    const long NAPT = (long)P.NA * PBS_PT;
    const int nx = P.nx;
    constexpr bool FULL = NY == 64;
    const bool valid = FULL || lane < NY;
    const int ql = FULL ? lane : (lane < NY ? lane : NY - 1);
    const int qc = my ? NY - 1 - ql : ql;
    const long RS = (long)(NY / 32) * NAPT;   // elements from row p to row p+1
    float *row0 = P.psi + slab * P.NLINE + (long)a * PBS_PT + (long)(qc >> 5) * NAPT + (qc & 31);
    const long step = mx ? -RS : RS;
    float *ptr = mx ? row0 + (long)(nx - 1) * RS : row0;
    const float c1 = cq, c2 = c1 * c1, c4 = c2 * c2, c8 = c4 * c4;
    float m16 = 1.f, m32 = 1.f;
    {
        const int e16 = (lane & 15) + 1, e32 = (lane & 31) + 1;
        float pw = cq;
#pragma unroll
        for (int i = 0; i < 6; ++i) {
            if ((e16 >> i) & 1) m16 *= pw;
            if ((e32 >> i) & 1) m32 *= pw;
            pw *= pw;
        }
        // the broadcasts write every row: rows 0 and 2 (row_bcast15) and lanes 0-31 (row_bcast31) add nothing
        if (!((lane >> 4) & 1)) m16 = 0.f;
        if (lane < 32) m32 = 0.f;
    }
    const float vmask = valid ? 1.f : 0.f;
    constexpr int PF = TPASS_PF;   // rows loaded ahead of the sweep
    float rb[2 * PF];
    const float *ld = ptr;
#pragma unroll
    for (int i = 0; i < PF; ++i) {
        rb[i] = i < nx ? TP_LD(ld) * vmask : 0.f;
        if (i < nx) ld += step;
    }
    float *st = ptr;
    float pm1 = 0.f, dxm = 0.f, ym1 = 0.f;
    for (int r0 = 0; r0 < nx; r0 += PF) {
        const bool more = r0 + PF < nx;
#pragma unroll
        for (int i = 0; i < PF; ++i) {
            rb[PF + i] = more ? TP_LD(ld) * vmask : 0.f;
            if (more) ld += step;
        }
#pragma unroll
        for (int i = 0; i < PF; ++i) {
            const float p0 = rb[i], p1 = rb[i + 1];
            const float left = dpp_z<0x138>(p0);
            const float right = dpp_z<0x130>(p0);
            const float dyp = superbee_slope(p0 - left, right - p0);
            const float dym = dpp_z<0x138>(dyp);
            const float dxp = superbee_slope(p0 - pm1, p1 - p0);
            const float R = p0 - ax * ((p0 - pm1) + (dxp - dxm)) - ay * ((p0 - left) + (dyp - dym));
            float y = (R + ax * ym1) * idiag;
            scan_rows16(y, c1, c2, c4, c8);
            scan_join32(y, m16);
            scan_join64(y, m32);
            scan_done();
            if (FULL || valid) TP_ST(y, st);
            st += step;
            pm1 = p0;
            dxm = dxp;
            ym1 = y;
        }
#pragma unroll
        for (int i = 0; i < PF; ++i) rb[i] = rb[PF + i];
    }
}

template <int NY>
__global__ __launch_bounds__(256) void tpass_affine_kernel(TParams<float> P)
{
    tpass_affine_body<NY>(P, (long)blockIdx.x * 4 + (threadIdx.x >> 6));
}

// Same sweep for ny = 32 with two planes per wave: lanes 0-31 sweep plane 2w, lanes 32-63 plane 2w+1, each
// half with its own angle, mirroring and pointer. Neighbour moves that would cross the halves are zeroed,
// the row scan stops at the 16-lane broadcast (it never crosses lane 31/32), and a half without a plane
// (odd plane count) repeats its neighbour's loads and stores nothing. Every lane carries a cell, where the
// one-plane sweep left half of them idle.
__device__ __forceinline__ void tpass_pair_body(const TParams<float> &P, long pair)
{
    if (pair * 2 >= P.nplanes) return;   // uniform per wave
    const int lane = threadIdx.x & 63;
    const int ql = lane & 31;
    const long plane = pair * 2 + (lane >> 5);
    const bool live = plane < P.nplanes;
    const long pl = live ? plane : plane - 1;
    const int a = (int)(pl % P.NA);
    const long slab = pl / P.NA;
    const float cx = P.theta[a / P.m], cy = P.theta[a % P.m];
    const bool mx = cx < 0.f, my = cy < 0.f;
    const float ax = fabsf(cx) * P.h_half_over_dx, ay = fabsf(cy) * P.h_half_over_dy;
    const float idiag = 1.f / (1.f + ax + ay);
    const float cq = ay * idiag;
    const long NAPT = (long)P.NA * PBS_PT;
    const int nx = P.nx;
    const int qc = my ? 31 - ql : ql;
    const long RS = NAPT;   // one lateral tile per row
    float *row0 = P.psi + slab * P.NLINE + (long)a * PBS_PT + qc;
    const long step = mx ? -RS : RS;
    float *ptr = mx ? row0 + (long)(nx - 1) * RS : row0;
    const float c1 = cq, c2 = c1 * c1, c4 = c2 * c2, c8 = c4 * c4;
    float m16 = 1.f;
    {
        const int e16 = (lane & 15) + 1;
        float pw = cq;
#pragma unroll
        for (int i = 0; i < 5; ++i) {
            if ((e16 >> i) & 1) m16 *= pw;
            pw *= pw;
        }
        // row_bcast15 writes every row: rows 0 and 2 of the wave (the first 16 lanes of each half) add nothing
        if (!((lane >> 4) & 1)) m16 = 0.f;
    }
    // 0 on the lanes whose neighbour move would cross into the other half, else 1.  Kept opaque so that
    // the compiler does not turn "move, then zero some lanes" into a move under a partial exec mask, where
    // the lanes switched off would also stop serving as move sources.
    float keep_l = ql == 0 ? 0.f : 1.f, keep_r = ql == 31 ? 0.f : 1.f;
    asm volatile("" : "+v"(keep_l), "+v"(keep_r));
    constexpr int PF = TPASS_PF;   // rows loaded ahead of the sweep
    float rb[2 * PF];
    const float *ld = ptr;
#pragma unroll
    for (int i = 0; i < PF; ++i) {
        rb[i] = i < nx ? TP_LD(ld) : 0.f;
        if (i < nx) ld += step;
    }
    float *st = ptr;
    float pm1 = 0.f, dxm = 0.f, ym1 = 0.f;
    for (int r0 = 0; r0 < nx; r0 += PF) {
        const bool more = r0 + PF < nx;
#pragma unroll
        for (int i = 0; i < PF; ++i) {
            rb[PF + i] = more ? TP_LD(ld) : 0.f;
            if (more) ld += step;
        }
#pragma unroll
        for (int i = 0; i < PF; ++i) {
            const float p0 = rb[i], p1 = rb[i + 1];
            const float left = keep_l * dpp_z<0x138>(p0);
            const float right = keep_r * dpp_z<0x130>(p0);
            const float dyp = superbee_slope(p0 - left, right - p0);
            const float dym = keep_l * dpp_z<0x138>(dyp);
            const float dxp = superbee_slope(p0 - pm1, p1 - p0);
            const float R = p0 - ax * ((p0 - pm1) + (dxp - dxm)) - ay * ((p0 - left) + (dyp - dym));
            float y = (R + ax * ym1) * idiag;
            scan_rows16(y, c1, c2, c4, c8);
            scan_join32(y, m16);
            scan_done();
            if (live) TP_ST(y, st);
            st += step;
            pm1 = p0;
            dxm = dxp;
            ym1 = y;
        }
#pragma unroll
        for (int i = 0; i < PF; ++i) rb[i] = rb[PF + i];
    }
}

__global__ __launch_bounds__(256) void tpass_pair_kernel(TParams<float> P)
{
    tpass_pair_body(P, (long)blockIdx.x * 4 + (threadIdx.x >> 6));
}

constexpr int TPASS_WIDE_PF = 4;   // rows loaded ahead per segment (4 measured faster than 8 or 2 at ny = 96)

// Same sweep for ny = 96 or 128 (two 64-lane segments per row, ny a multiple of the 32-column lateral
// tile, so every segment's address stays affine in the row): neighbours at a segment seam and the carry of
// the implicit row recurrence cross it by readlane; lanes beyond ny read a clamped column and are zeroed.
template <int NY>
__device__ __forceinline__ void tpass_wide_body(const TParams<float> &P, long plane)
{
    static_assert(NY % 32 == 0 && NY > 64 && NY <= 128, "two segments of whole lateral tiles");
    constexpr int NS = 2;
    if (plane >= P.nplanes) return;   // uniform per wave
    const int lane = threadIdx.x & 63;
    const int a = (int)(plane % P.NA);
    const long slab = plane / P.NA;
    const float cx = P.theta[a / P.m], cy = P.theta[a % P.m];
    const bool mx = cx < 0.f, my = cy < 0.f;
    const float ax = fabsf(cx) * P.h_half_over_dx, ay = fabsf(cy) * P.h_half_over_dy;
    const float idiag = 1.f / (1.f + ax + ay);
    const float cq = ay * idiag;
    const long NAPT = (long)P.NA * PBS_PT;
    const int nx = P.nx;
    const long RS = (long)(NY / 32) * NAPT;   // elements from row p to row p+1
    const long step = mx ? -RS : RS;
    float vmask[NS];
    bool valid[NS];
    const float *ld[NS];
    float *st[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const int q = s * 64 + lane;
        valid[s] = q < NY;
        const int ql = valid[s] ? q : NY - 1;
        const int qc = my ? NY - 1 - ql : ql;
        float *row0 = P.psi + slab * P.NLINE + (long)a * PBS_PT + (long)(qc >> 5) * NAPT + (qc & 31);
        st[s] = mx ? row0 + (long)(nx - 1) * RS : row0;
        ld[s] = st[s];
        vmask[s] = valid[s] ? 1.f : 0.f;
    }
    // scan multipliers: cq^(2^i) for the row shifts, cq^((lane&15)+1), cq^((lane&31)+1) for the row
    // broadcasts and cq^(lane+1) for the carry from the previous segment
    const float c1 = cq, c2 = c1 * c1, c4 = c2 * c2, c8 = c4 * c4;
    float m16 = 1.f, m32 = 1.f, m64 = 1.f;
    {
        const int e16 = (lane & 15) + 1, e32 = (lane & 31) + 1, e64 = lane + 1;
        float pw = cq;
#pragma unroll
        for (int i = 0; i < 7; ++i) {
            if ((e16 >> i) & 1) m16 *= pw;
            if ((e32 >> i) & 1) m32 *= pw;
            if ((e64 >> i) & 1) m64 *= pw;
            pw *= pw;
        }
        // the broadcasts write every row: rows 0 and 2 (row_bcast15) and lanes 0-31 (row_bcast31) add nothing
        if (!((lane >> 4) & 1)) m16 = 0.f;
        if (lane < 32) m32 = 0.f;
    }
    auto lane_of = [](float v, int l) {
        return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l));
    };
    constexpr int PF = TPASS_WIDE_PF;   // rows loaded ahead of the sweep
    float rb[2 * PF][NS];
#pragma unroll
    for (int i = 0; i < PF; ++i)
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            rb[i][s] = i < nx ? TP_LD(ld[s]) * vmask[s] : 0.f;
            if (i < nx) ld[s] += step;
        }
    float pm1[NS], dxm[NS], ym1[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) pm1[s] = dxm[s] = ym1[s] = 0.f;
    for (int r0 = 0; r0 < nx; r0 += PF) {
        const bool more = r0 + PF < nx;
#pragma unroll
        for (int i = 0; i < PF; ++i)
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                rb[PF + i][s] = more ? TP_LD(ld[s]) * vmask[s] : 0.f;
                if (more) ld[s] += step;
            }
#pragma unroll
        for (int i = 0; i < PF; ++i) {
            float left[NS], dyp[NS];
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                const float p0 = rb[i][s];
                const float up = dpp_z<0x138>(p0), dn = dpp_z<0x130>(p0);
                left[s] = (s > 0 && lane == 0) ? lane_of(rb[i][s > 0 ? s - 1 : 0], 63) : up;
                const float right = (s + 1 < NS && lane == 63) ? lane_of(rb[i][s + 1 < NS ? s + 1 : 0], 0) : dn;
                dyp[s] = superbee_slope(p0 - left[s], right - p0);
            }
            float carry = 0.f;
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                const float p0 = rb[i][s], p1 = rb[i + 1][s];
                const float up = dpp_z<0x138>(dyp[s]);
                const float dym = (s > 0 && lane == 0) ? lane_of(dyp[s > 0 ? s - 1 : 0], 63) : up;
                const float dxp = superbee_slope(p0 - pm1[s], p1 - p0);
                const float R = p0 - ax * ((p0 - pm1[s]) + (dxp - dxm[s])) - ay * ((p0 - left[s]) + (dyp[s] - dym));
                float y = (R + ax * ym1[s]) * idiag;
                scan_rows16(y, c1, c2, c4, c8);
                scan_join32(y, m16);
                scan_join64(y, m32);
                scan_done();
                if (s > 0) y += m64 * carry;
                carry = lane_of(y, 63);
                if (valid[s]) TP_ST(y, st[s]);
                st[s] += step;
                pm1[s] = p0;
                dxm[s] = dxp;
                ym1[s] = y;
            }
        }
#pragma unroll
        for (int i = 0; i < PF; ++i)
#pragma unroll
            for (int s = 0; s < NS; ++s) rb[i][s] = rb[PF + i][s];
    }
}

template <int NY>
__global__ __launch_bounds__(256) void tpass_wide_kernel(TParams<float> P)
{
    tpass_wide_body<NY>(P, (long)blockIdx.x * 4 + (threadIdx.x >> 6));
}

constexpr int TPASS_W2_PF = 4;   // rows loaded ahead per operation in the two-plane ny = 96 sweep
// LDS reserved per block of the two-plane sweep, which uses none: it caps the sweep at 3 blocks (12 waves)
// per CU.  Fewer concurrent plane streams suit the memory system: a copy with the sweep's addresses runs
// 5.18 -> 5.43 TB/s at 2 blocks per CU, and the config-3 sweep 8.76 -> 8.47 ms per launch at 2 or 3.
#ifndef TP_W2_LDS
#define TP_W2_LDS 54000
#endif

// ny = 96 with two planes per wave (A = plane 2w, B = plane 2w + 1; the plane count is even).  A row of
// both planes is three full 64-lane operations: A columns 0-63, B columns 0-63, then A columns 64-95 in
// lanes 0-31 beside B columns 64-95 in lanes 32-63.  The one-plane sweep of this width spends two
// operations per row with a quarter of its lanes idle and is instruction-bound; here no lane idles.
// The third operation carries each half's own angle coefficients; its row scan stops at the 16-lane
// broadcast (it never crosses lane 31/32) and takes the carry y_63 of its plane's first operation.
// Neighbours across the seams (A 63|64, B 63|64) move by readlane and masked products; column 96 is the
// ghost.
// Addresses are 32-bit byte offsets in a buffer resource based at plane A's slab (plane B lies in the
// same slab or the next); each lane steps by its plane's signed row stride.
__device__ __forceinline__ void tpass_wide2_body(const TParams<float> &P, int pair)
{
    constexpr int NY = 96;
    if (2L * pair >= P.nplanes) return;   // uniform per wave
    const int lane = threadIdx.x & 63;
    const int ql = lane & 31;
    const bool hi = lane >= 32;
    const long NAPT = (long)P.NA * PBS_PT;
    const int nx = P.nx;
    const long plA = 2L * pair, plB = plA + 1;
    const int aA = (int)(plA % P.NA), aB = (int)(plB % P.NA);
    const long slabA = plA / P.NA, slabB = plB / P.NA;
    const float cxA = P.theta[aA / P.m], cyA = P.theta[aA % P.m];
    const float cxB = P.theta[aB / P.m], cyB = P.theta[aB % P.m];
    const bool mxA = cxA < 0.f, myA = cyA < 0.f, mxB = cxB < 0.f, myB = cyB < 0.f;
    const float axA = fabsf(cxA) * P.h_half_over_dx, ayA = fabsf(cyA) * P.h_half_over_dy;
    const float axB = fabsf(cxB) * P.h_half_over_dx, ayB = fabsf(cyB) * P.h_half_over_dy;
    const float idA = 1.f / (1.f + axA + ayA), idB = 1.f / (1.f + axB + ayB);
    const float cqA = ayA * idA, cqB = ayB * idB;
    // byte offsets from plane A's slab: plane origin + column (mirrored) + first row (mirrored)
    const long RSB = 3 * NAPT * 4;   // bytes from row p to row p + 1
    const long originA = (long)aA * PBS_PT * 4;
    const long originB = ((slabB - slabA) * P.NLINE + (long)aB * PBS_PT) * 4;
    auto col = [&](int q, bool my) -> long {
        const int qc = my ? NY - 1 - q : q;
        return ((long)(qc >> 5) * NAPT + (qc & 31)) * 4;
    };
    const long row0A = mxA ? (long)(nx - 1) * RSB : 0, row0B = mxB ? (long)(nx - 1) * RSB : 0;
    const int stepA = (int)(mxA ? -RSB : RSB), stepB = (int)(mxB ? -RSB : RSB);
    unsigned ld[3], st[3];
    int step[3];
    ld[0] = (unsigned)(originA + col(lane, myA) + row0A);
    ld[1] = (unsigned)(originB + col(lane, myB) + row0B);
    ld[2] = (unsigned)(hi ? originB + col(64 + ql, myB) + row0B : originA + col(64 + ql, myA) + row0A);
    step[0] = stepA;
    step[1] = stepB;
    step[2] = hi ? stepB : stepA;
#pragma unroll
    for (int o = 0; o < 3; ++o) st[o] = ld[o];
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(P.psi + slabA * P.NLINE), (short)0, (int)(2 * P.NLINE * 4 < 0x7fffffffL ? 2 * P.NLINE * 4 : 0x7fffffffL),
        0x00020000);
    // scan multipliers per operation: cq^(2^i) for the row shifts, cq^((lane & 15) + 1) and
    // cq^((lane & 31) + 1) for the broadcasts; in the third operation each half has its own cq, and
    // cq^(ql + 1) takes the carry of its plane's first operation (zero in the other half)
    auto powers = [](float cq, int e) {
        float m = 1.f, pw = cq;
#pragma unroll
        for (int i = 0; i < 7; ++i) {
            if ((e >> i) & 1) m *= pw;
            pw *= pw;
        }
        return m;
    };
    float c1[3], c2[3], c4[3], c8[3], m16[3], ax[3], ay[3], idg[3];
    const float cq3 = hi ? cqB : cqA;
    const float cqs[3] = {cqA, cqB, cq3};
#pragma unroll
    for (int o = 0; o < 3; ++o) {
        c1[o] = cqs[o];
        c2[o] = c1[o] * c1[o];
        c4[o] = c2[o] * c2[o];
        c8[o] = c4[o] * c4[o];
        m16[o] = powers(cqs[o], (lane & 15) + 1);
    }
    const float m32A = powers(cqA, (lane & 31) + 1), m32B = powers(cqB, (lane & 31) + 1);
    const float mcA = hi ? 0.f : powers(cqA, ql + 1), mcB = hi ? powers(cqB, ql + 1) : 0.f;
    ax[0] = axA; ay[0] = ayA; idg[0] = idA;
    ax[1] = axB; ay[1] = ayB; idg[1] = idB;
    ax[2] = hi ? axB : axA; ay[2] = hi ? ayB : ayA; idg[2] = hi ? idB : idA;
    // lane masks for the seam corrections, kept opaque (a select would run the DPP moves next to it under
    // a partial exec mask, where the switched-off lanes would stop serving as move sources)
    float e63 = lane == 63 ? 1.f : 0.f, e0 = lane == 0 ? 1.f : 0.f, e32 = lane == 32 ? 1.f : 0.f;
    float keep_l = ql == 0 ? 0.f : 1.f, keep_r = ql == 31 ? 0.f : 1.f;
    asm volatile("" : "+v"(e63), "+v"(e0), "+v"(e32), "+v"(keep_l), "+v"(keep_r));
    auto lane_of = [](float v, int l) {
        return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l));
    };
    // the left neighbour in the third operation: the lane below, but plane A's and plane B's column 63
    // (scalars sa, sb) in lanes 0 and 32 -- exact, as every other term is a product with 0
    auto left3 = [&](float v, float sa, float sb) { return keep_l * dpp_z<0x138>(v) + e0 * sa + e32 * sb; };
    constexpr int PF = TPASS_W2_PF;
    float rb[3][2 * PF];
#pragma unroll
    for (int i = 0; i < PF; ++i)
#pragma unroll
        for (int o = 0; o < 3; ++o) {
            rb[o][i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, ld[o], 0, 2));
            ld[o] += step[o];
        }
    float dxb[3], dxm[3], ym1[3];
#pragma unroll
    for (int o = 0; o < 3; ++o) {
        dxb[o] = rb[o][0];   // p0 - p_{-1} with the ghost row upstream
        dxm[o] = ym1[o] = 0.f;
    }
    for (int r0 = 0; r0 < nx; r0 += PF) {
        const bool more = r0 + PF < nx;
        if (more) {
#pragma unroll
            for (int i = 0; i < PF; ++i)
#pragma unroll
                for (int o = 0; o < 3; ++o) {
                    rb[o][PF + i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, ld[o], 0, 2));
                    ld[o] += step[o];
                }
        } else {
#pragma unroll
            for (int i = 0; i < PF; ++i)
#pragma unroll
                for (int o = 0; o < 3; ++o) rb[o][PF + i] = 0.f;
        }
#pragma unroll
        for (int i = 0; i < PF; ++i) {
            float p0[3], dy[3], ayv[3];
#pragma unroll
            for (int o = 0; o < 3; ++o) p0[o] = rb[o][i];
            // lateral differences p0 - left and right - p0, seams patched
            const float rA = lane_of(p0[2], 0), rB = lane_of(p0[2], 32);
            const float lA = lane_of(p0[0], 63), lB = lane_of(p0[1], 63);
            float bf[3];
            ayv[0] = p0[0] - dpp_z<0x138>(p0[0]);
            bf[0] = dpp_z<0x130>(p0[0]) - p0[0] + e63 * rA;
            ayv[1] = p0[1] - dpp_z<0x138>(p0[1]);
            bf[1] = dpp_z<0x130>(p0[1]) - p0[1] + e63 * rB;
            ayv[2] = p0[2] - left3(p0[2], lA, lB);
            bf[2] = keep_r * dpp_z<0x130>(p0[2]) - p0[2];
#pragma unroll
            for (int o = 0; o < 3; ++o) dy[o] = superbee_slope(ayv[o], bf[o]);
            // dyp - dym, the seams taking the upstream plane's lane-63 slope
            float dd[3];
            dd[0] = dy[0] - dpp_z<0x138>(dy[0]);
            dd[1] = dy[1] - dpp_z<0x138>(dy[1]);
            dd[2] = dy[2] - left3(dy[2], lane_of(dy[0], 63), lane_of(dy[1], 63));
            float y[3];
#pragma unroll
            for (int o = 0; o < 3; ++o) {
                const float dxf = rb[o][i + 1] - p0[o];
                const float dxp = superbee_slope(dxb[o], dxf);
                const float R = p0[o] - ax[o] * (dxb[o] + (dxp - dxm[o])) - ay[o] * (ayv[o] + dd[o]);
                y[o] = (R + ax[o] * ym1[o]) * idg[o];
                dxb[o] = dxf;
                dxm[o] = dxp;
            }
            scan_rows16(y[0], c1[0], c2[0], c4[0], c8[0]);
            scan_join32(y[0], m16[0]);
            scan_join64(y[0], m32A);
            scan_rows16(y[1], c1[1], c2[1], c4[1], c8[1]);
            scan_join32(y[1], m16[1]);
            scan_join64(y[1], m32B);
            scan_rows16(y[2], c1[2], c2[2], c4[2], c8[2]);
            scan_join32(y[2], m16[2]);
            scan_done();
            y[2] += mcA * lane_of(y[0], 63);
            y[2] += mcB * lane_of(y[1], 63);
#pragma unroll
            for (int o = 0; o < 3; ++o) {
                __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, y[o]), rs, st[o], 0, 2);
                st[o] += step[o];
                ym1[o] = y[o];
            }
        }
#pragma unroll
        for (int i = 0; i < PF; ++i)
#pragma unroll
            for (int o = 0; o < 3; ++o) rb[o][i] = rb[o][PF + i];
    }
}

__global__ __launch_bounds__(256) void tpass_wide2_kernel(TParams<float> P)
{
    tpass_wide2_body(P, __builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + (threadIdx.x >> 6))));
}

// --- The same sweep for any ny <= 128 and any nx, FP32 and FP64 (every grid that no aligned variant above
// takes).  What bounds the general case is instructions and idle lanes, not memory: the sweep it replaces spent
// one wave per plane whatever its width, moved neighbours and the row scan through LDS shuffles and waited for
// each row's loads.  Here the width picks how planes share a wave --
//   ny <= 16: four planes, one per 16-lane row;  <= 32: two;  <= 64: one;
//   ny <= 96: two planes in three operations (tpass_wide2_body's arrangement);  <= 128: one in two
// -- neighbours and scan move by DPP, and TPASS_PK_PF rows are loaded ahead.  A row need not start a lateral
// tile, so a lane's address is not affine in the row: its cell pq = p ny + q sits at 4|8 x (pq + (pq / 32) 32
// (NA - 1)) bytes from the plane's first cell, three operations in a buffer resource based at the wave's first
// slab.  Lanes without a cell carry offset 2^31, past the resource: their loads read the ghost value 0 and their
// stores are dropped.
// Measured, us per step half of two generations, before -> after: 4 x 4 cells, 11 x 11 angles, 60 groups 21 -> 7;
// 24 x 24, 15 x 15, 110 groups 237 -> 88; 50 x 50, 15 x 15, 64 groups 309 -> 218; 45 x 70, 19 x 19, 75 groups (three
// generations) 1867 -> 860; FP64 20 x 24, 15 x 15, 60 groups 224 -> 73 (5.7 TB/s) and 64 x 64, 15 x 15, 64 groups
// 860 -> 685.  Eight rows ahead instead of four: 5 % slower at 4 x 4 and 50 x 50, the same elsewhere.
constexpr int TPASS_PK_PF = 4;

template <int CTRL, typename T>
__device__ __forceinline__ T dpp_zt(T x)
{
    if constexpr (sizeof(T) == 4) {
        return dpp_z<CTRL>(x);
    } else {
        const unsigned long long u = __builtin_bit_cast(unsigned long long, x);
        const unsigned lo = __builtin_amdgcn_mov_dpp((int)(unsigned)u, CTRL, 0xF, 0xF, true);
        const unsigned hi = __builtin_amdgcn_mov_dpp((int)(unsigned)(u >> 32), CTRL, 0xF, 0xF, true);
        return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
    }
}
// y_q = b_q + c y_{q-1} over W lanes (16, 32 or 64): the multipliers of the 16-lane rows, then of the joins, which
// must be 0 in the lanes a join does not change (m16: rows 0 and 2, m32: lanes 0-31)
template <int W, typename T>
__device__ __forceinline__ void scan_lanes(T &y, T c1, T c2, T c4, T c8, T m16, T m32)
{
    if constexpr (sizeof(T) == 4) {
        scan_rows16(y, c1, c2, c4, c8);
        if constexpr (W >= 32) scan_join32(y, m16);
        if constexpr (W >= 64) scan_join64(y, m32);
        scan_done();
    } else {
        y = fma(c1, dpp_zt<0x111>(y), y);
        y = fma(c2, dpp_zt<0x112>(y), y);
        y = fma(c4, dpp_zt<0x114>(y), y);
        y = fma(c8, dpp_zt<0x118>(y), y);
        if constexpr (W >= 32) y = fma(m16, dpp_zt<0x142>(y), y);
        if constexpr (W >= 64) y = fma(m32, dpp_zt<0x143>(y), y);
    }
}
// c^e for 1 <= e <= 64
template <typename T>
__device__ __forceinline__ T pow_lane(T c, int e)
{
    T m = T(1), pw = c;
#pragma unroll
    for (int i = 0; i < 7; ++i) {
        if ((e >> i) & 1) m *= pw;
        pw *= pw;
    }
    return m;
}
template <typename T, int AUX>
__device__ __forceinline__ T buf_ld(__amdgpu_buffer_rsrc_t rs, unsigned o)
{
    if constexpr (sizeof(T) == 4) {
        return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, o, 0, AUX));
    } else {
        typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
        return __builtin_bit_cast(double, (u32x2)__builtin_amdgcn_raw_buffer_load_b64(rs, o, 0, AUX));
    }
}
template <int AUX, typename T>
__device__ __forceinline__ void buf_st(T v, __amdgpu_buffer_rsrc_t rs, unsigned o)
{
    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
    if constexpr (sizeof(T) == 4)
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), rs, o, 0, AUX);
    else
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), rs, o, 0, AUX);
}

// What the packed sweeps need: 32-bit plane numbers, two slabs inside a 31-bit buffer resource.
template <typename T>
static inline bool tpass_packed_fits(const TParams<T> &P)
{
    return P.ny <= 128 && P.nplanes < (1L << 31) - 256 && 2 * P.NLINE * (long)sizeof(T) < 0x7fffffffL;
}

// One plane per W lanes (W = 16, 32, 64; ny <= W); wave number from the caller, the same in all lanes.
// make(first slab) -> {load(byte offset), store(value, byte offset)} of two slabs (W = 64: of one); NONE is no cell's
// offset: the load gives 0, the store is dropped.
template <typename T, int W, typename MAKE>
__device__ __forceinline__ void tpass_pack_planes(const TParams<T> &P, unsigned wave, MAKE make)
{
    constexpr unsigned NPW = 64 / W, TS = sizeof(T), SH = TS == 4 ? 2 : 3;
    const unsigned pl0 = wave * NPW, nplanes = (unsigned)P.nplanes, NA = P.NA, m = P.m;
    if (pl0 >= nplanes) return;   // uniform per wave
    const int lane = threadIdx.x & 63, q = lane % W, sub = lane / W;
    const int nx = P.nx, ny = P.ny;
    const unsigned slab0 = pl0 / NA;
    unsigned a = pl0 - slab0 * NA + sub;
    const bool next = a >= NA;
    if (next) a -= NA;
    const unsigned ai = a / m, aj = a - ai * m;
    const bool live = pl0 + sub < nplanes && q < ny;
    const T cx = P.theta[ai], cy = P.theta[aj];
    const bool mx = cx < T(0), my = cy < T(0);   // sweep frames mirrored so the velocity is >= 0
    const T ax = fabs(cx) * P.h_half_over_dx, ay = fabs(cy) * P.h_half_over_dy;
    const T idiag = T(1) / (T(1) + ax + ay);
    const T c1 = ay * idiag, c2 = c1 * c1, c4 = c2 * c2, c8 = c4 * c4;
    T m16 = T(0), m32 = T(0);
    if constexpr (W >= 32)
        if ((lane >> 4) & 1) m16 = pow_lane(c1, (lane & 15) + 1);
    if constexpr (W >= 64)
        if (lane >= 32) m32 = pow_lane(c1, (lane & 31) + 1);
    const auto mem = make(slab0);
    using MEM = decltype(make(slab0));
    using Off = typename MEM::Off;
    const Off K = PBS_PT * TS * (NA - 1);
    const Off base = live ? (Off)a * (PBS_PT * TS) + (next ? (Off)(P.NLINE * TS) : Off(0)) : MEM::NONE;
    const int step = live ? (mx ? -ny : ny) : 0;
    int pld = live ? (mx ? nx - 1 : 0) * ny + (my ? ny - 1 - q : q) : 0, pst = pld;   // cell loaded / stored next
    auto addr = [&](int pq) { return base + ((Off)pq << SH) + ((Off)pq >> 5) * K; };
    // neighbour moves inside the plane's W lanes: 16-lane rows shift by themselves; two planes need the lanes at
    // the seam masked (opaque factors: a select would run the move under a partial exec mask)
    T keep_l = T(1), keep_r = T(1);
    if constexpr (W == 32) {
        keep_l = q == 0 ? T(0) : T(1);
        keep_r = q == 31 ? T(0) : T(1);
        asm volatile("" : "+v"(keep_l), "+v"(keep_r));
    }
    auto from_left = [&](T v) {
        if constexpr (W == 16) return dpp_zt<0x111>(v);
        else if constexpr (W == 32) return keep_l * dpp_zt<0x138>(v);
        else return dpp_zt<0x138>(v);
    };
    auto from_right = [&](T v) {
        if constexpr (W == 16) return dpp_zt<0x101>(v);
        else if constexpr (W == 32) return keep_r * dpp_zt<0x130>(v);
        else return dpp_zt<0x130>(v);
    };
    constexpr int PF = TPASS_PK_PF;
    T rb[2 * PF];
#pragma unroll
    for (int i = 0; i < PF; ++i) {
        rb[i] = T(0);
        if (i < nx) {
            rb[i] = mem.load(addr(pld));
            pld += step;
        }
    }
    T dxb = rb[0], dxm = T(0), ym1 = T(0);   // p0 - p_{-1} with the ghost row upstream
    auto row = [&](T p0, T p1) {
        const T dyb = p0 - from_left(p0), dyf = from_right(p0) - p0;
        const T dyp = superbee_slope(dyb, dyf);
        const T dym = from_left(dyp);
        const T dxf = p1 - p0;
        const T dxp = superbee_slope(dxb, dxf);
        const T R = p0 - ax * (dxb + (dxp - dxm)) - ay * (dyb + (dyp - dym));
        T y = (R + ax * ym1) * idiag;
        scan_lanes<W>(y, c1, c2, c4, c8, m16, m32);
        mem.store(y, addr(pst));
        pst += step;
        dxb = dxf;
        dxm = dxp;
        ym1 = y;
    };
    int r0 = 0;
    for (; r0 + 2 * PF <= nx; r0 += PF) {
#pragma unroll
        for (int i = 0; i < PF; ++i) {
            rb[PF + i] = mem.load(addr(pld));
            pld += step;
        }
#pragma unroll
        for (int i = 0; i < PF; ++i) row(rb[i], rb[i + 1]);
#pragma unroll
        for (int i = 0; i < PF; ++i) rb[i] = rb[PF + i];
    }
    // the last rows: fewer than PF left to load, then the ghost row
    {
#pragma unroll
        for (int i = 0; i < PF; ++i) {
            rb[PF + i] = T(0);
            if (r0 + PF + i < nx) {
                rb[PF + i] = mem.load(addr(pld));
                pld += step;
            }
        }
#pragma unroll
        for (int i = 0; i < 2 * PF; ++i)
            if (r0 + i < nx) row(rb[i], i + 1 < 2 * PF ? rb[i + 1 < 2 * PF ? i + 1 : 0] : T(0));
    }
}

template <typename T, int AUX>
struct SlabBuf {
    using Off = unsigned;
    static constexpr Off NONE = 0x80000000u;   // past every resource
    __amdgpu_buffer_rsrc_t rs;
    __device__ __forceinline__ SlabBuf(T *slab, long bytes)
        : rs(__builtin_amdgcn_make_buffer_rsrc((void *)slab, (short)0, (int)bytes, 0x00020000))
    {
    }
    __device__ __forceinline__ T load(unsigned o) const { return buf_ld<T, AUX>(rs, o); }
    __device__ __forceinline__ void store(T v, unsigned o) const { buf_st<AUX>(v, rs, o); }
};
// a slab of any size
template <typename T>
struct SlabFar {
    using Off = long;
    static constexpr Off NONE = -(1L << 62);
    T *p;
    __device__ __forceinline__ T *at(Off o) const { return reinterpret_cast<T *>(reinterpret_cast<char *>(p) + o); }
    __device__ __forceinline__ T load(Off o) const { return o >= 0 ? *at(o) : T(0); }
    __device__ __forceinline__ void store(T v, Off o) const
    {
        if (o >= 0) *at(o) = v;
    }
};
template <typename T, int W, int AUX>
__device__ __forceinline__ void tpass_pack_body(const TParams<T> &P, unsigned wave)
{
    tpass_pack_planes<T, W>(P, wave, [&](unsigned slab0) {
        return SlabBuf<T, AUX>(P.psi + slab0 * P.NLINE, 2 * P.NLINE * (long)sizeof(T));
    });
}

// 64 < ny <= 96 (TWO: two planes in three operations, as tpass_wide2_body) or ny <= 128 (one plane in two).
template <typename T, bool TWO, int AUX>
__device__ __forceinline__ void tpass_packw_body(const TParams<T> &P, unsigned wave)
{
    constexpr unsigned TS = sizeof(T), SH = TS == 4 ? 2 : 3;
    constexpr int NO = TWO ? 3 : 2, NPL = TWO ? 2 : 1;
    const unsigned pl0 = wave * NPL, nplanes = (unsigned)P.nplanes, NA = P.NA, m = P.m;
    if (pl0 >= nplanes) return;   // uniform per wave
    const int lane = threadIdx.x & 63, ql = TWO ? lane & 31 : lane;
    const bool hi = TWO && lane >= 32;
    const int nx = P.nx, ny = P.ny;
    const unsigned slab0 = pl0 / NA, a0 = pl0 - slab0 * NA;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(P.psi + slab0 * P.NLINE), (short)0, (int)(2 * P.NLINE * TS), 0x00020000);
    const unsigned K = PBS_PT * TS * (NA - 1);
    // per plane (uniform): angle, mirroring, slab
    T axp[NPL], ayp[NPL], idp[NPL];
    bool mxp[NPL], myp[NPL];
    unsigned bsp[NPL];
#pragma unroll
    for (int k = 0; k < NPL; ++k) {
        unsigned a = a0 + k;
        const bool next = a >= NA;
        if (next) a -= NA;
        const unsigned ai = a / m;
        const T cx = P.theta[ai], cy = P.theta[a - ai * m];
        mxp[k] = cx < T(0);
        myp[k] = cy < T(0);
        axp[k] = fabs(cx) * P.h_half_over_dx;
        ayp[k] = fabs(cy) * P.h_half_over_dy;
        idp[k] = T(1) / (T(1) + axp[k] + ayp[k]);
        bsp[k] = pl0 + k < nplanes ? a * (PBS_PT * TS) + (next ? (unsigned)(P.NLINE * TS) : 0u) : 0x80000000u;
    }
    // per operation and lane: column, coefficients, cell walked
    T ax[NO], ay[NO], idg[NO], c1[NO], c2[NO], c4[NO], c8[NO], m16[NO], m32[NO];
    unsigned base[NO];
    int step[NO], pld[NO], pst[NO];
#pragma unroll
    for (int o = 0; o < NO; ++o) {
        const bool b = TWO && (o == 1 || (o == 2 && hi));   // plane B
        const int q = TWO ? (o == 2 ? 64 + ql : lane) : o * 64 + lane;
        const bool mx = b ? mxp[NPL - 1] : mxp[0], my = b ? myp[NPL - 1] : myp[0];
        ax[o] = b ? axp[NPL - 1] : axp[0];
        ay[o] = b ? ayp[NPL - 1] : ayp[0];
        idg[o] = b ? idp[NPL - 1] : idp[0];
        c1[o] = ay[o] * idg[o];
        c2[o] = c1[o] * c1[o];
        c4[o] = c2[o] * c2[o];
        c8[o] = c4[o] * c4[o];
        m16[o] = (lane >> 4) & 1 ? pow_lane(c1[o], (lane & 15) + 1) : T(0);
        m32[o] = lane >= 32 ? pow_lane(c1[o], (lane & 31) + 1) : T(0);
        const bool ok = q < ny;
        base[o] = ok ? (b ? bsp[NPL - 1] : bsp[0]) : 0x80000000u;
        step[o] = ok ? (mx ? -ny : ny) : 0;
        pld[o] = ok ? (mx ? nx - 1 : 0) * ny + (my ? ny - 1 - q : q) : 0;
        pst[o] = pld[o];
    }
    // carry of a plane's first operation into the columns from 64 on: c^(column - 63), by plane
    const T mcA = hi ? T(0) : pow_lane(c1[0], ql + 1);
    const T mcB = TWO && hi ? pow_lane(c1[NO - 1], ql + 1) : T(0);
    T e63 = lane == 63 ? T(1) : T(0), e0 = lane == 0 ? T(1) : T(0), e32 = lane == 32 ? T(1) : T(0);
    T keep_l = TWO && ql == 0 ? T(0) : T(1), keep_r = TWO && ql == 31 ? T(0) : T(1);
    asm volatile("" : "+v"(e63), "+v"(e0), "+v"(e32), "+v"(keep_l), "+v"(keep_r));
    auto addr = [&](int o, int pq) { return base[o] + ((unsigned)pq << SH) + ((unsigned)pq >> 5) * K; };
    // left neighbour in the last operation: the lane below, but column 63 of its plane in the seam lanes (exact:
    // every other term is a product with 0)
    auto left_last = [&](T v, T sa, T sb) {
        T l = keep_l * dpp_zt<0x138>(v) + e0 * sa;
        if constexpr (TWO) l += e32 * sb;
        return l;
    };
    constexpr int PF = TS == 8 ? 2 : TPASS_PK_PF;   // rows ahead, within the registers of two waves per SIMD
    T rb[NO][2 * PF];
    auto load = [&](int i) {
#pragma unroll
        for (int o = 0; o < NO; ++o) {
            rb[o][i] = buf_ld<T, AUX>(rs, addr(o, pld[o]));
            pld[o] += step[o];
        }
    };
    auto ghost = [&](int i) {
#pragma unroll
        for (int o = 0; o < NO; ++o) rb[o][i] = T(0);
    };
#pragma unroll
    for (int i = 0; i < PF; ++i) {
        if (i < nx) load(i);
        else ghost(i);
    }
    T dxb[NO], dxm[NO], ym1[NO];
#pragma unroll
    for (int o = 0; o < NO; ++o) {
        dxb[o] = rb[o][0];
        dxm[o] = ym1[o] = T(0);
    }
    constexpr int LAST = NO - 1;
    auto row = [&](int i, bool end) {
        T p0[NO], ayv[NO], bf[NO], dy[NO], dd[NO], y[NO];
#pragma unroll
        for (int o = 0; o < NO; ++o) p0[o] = rb[o][i];
        const T lA = lane_of(p0[0], 63), lB = TWO ? lane_of(p0[1], 63) : T(0);
        ayv[0] = p0[0] - dpp_zt<0x138>(p0[0]);
        bf[0] = dpp_zt<0x130>(p0[0]) - p0[0] + e63 * lane_of(p0[LAST], 0);
        if constexpr (TWO) {
            ayv[1] = p0[1] - dpp_zt<0x138>(p0[1]);
            bf[1] = dpp_zt<0x130>(p0[1]) - p0[1] + e63 * lane_of(p0[LAST], 32);
        }
        ayv[LAST] = p0[LAST] - left_last(p0[LAST], lA, lB);
        bf[LAST] = keep_r * dpp_zt<0x130>(p0[LAST]) - p0[LAST];
#pragma unroll
        for (int o = 0; o < NO; ++o) dy[o] = superbee_slope(ayv[o], bf[o]);
        dd[0] = dy[0] - dpp_zt<0x138>(dy[0]);
        if constexpr (TWO) dd[1] = dy[1] - dpp_zt<0x138>(dy[1]);
        dd[LAST] = dy[LAST] - left_last(dy[LAST], lane_of(dy[0], 63), TWO ? lane_of(dy[1], 63) : T(0));
#pragma unroll
        for (int o = 0; o < NO; ++o) {
            const T dxf = (end ? T(0) : rb[o][i + 1]) - p0[o];
            const T dxp = superbee_slope(dxb[o], dxf);
            const T R = p0[o] - ax[o] * (dxb[o] + (dxp - dxm[o])) - ay[o] * (ayv[o] + dd[o]);
            y[o] = (R + ax[o] * ym1[o]) * idg[o];
            dxb[o] = dxf;
            dxm[o] = dxp;
        }
        scan_lanes<64>(y[0], c1[0], c2[0], c4[0], c8[0], m16[0], m32[0]);
        if constexpr (TWO) {
            scan_lanes<64>(y[1], c1[1], c2[1], c4[1], c8[1], m16[1], m32[1]);
            scan_lanes<32>(y[2], c1[2], c2[2], c4[2], c8[2], m16[2], m32[2]);
            y[2] += mcA * lane_of(y[0], 63);
            y[2] += mcB * lane_of(y[1], 63);
        } else {
            scan_lanes<64>(y[1], c1[1], c2[1], c4[1], c8[1], m16[1], m32[1]);
            y[1] += mcA * lane_of(y[0], 63);
        }
#pragma unroll
        for (int o = 0; o < NO; ++o) {
            buf_st<AUX>(y[o], rs, addr(o, pst[o]));
            pst[o] += step[o];
            ym1[o] = y[o];
        }
    };
    int r0 = 0;
    for (; r0 + 2 * PF <= nx; r0 += PF) {
#pragma unroll
        for (int i = 0; i < PF; ++i) load(PF + i);
#pragma unroll
        for (int i = 0; i < PF; ++i) row(i, false);
#pragma unroll
        for (int i = 0; i < PF; ++i)
#pragma unroll
            for (int o = 0; o < NO; ++o) rb[o][i] = rb[o][PF + i];
    }
#pragma unroll
    for (int i = 0; i < PF; ++i) {
        if (r0 + PF + i < nx) load(PF + i);
        else ghost(PF + i);
    }
#pragma unroll
    for (int i = 0; i < 2 * PF; ++i)
        if (r0 + i < nx) row(i, i + 1 == 2 * PF);
}

// planes that share a wave in the packed sweeps
static inline int tpass_packed_planes(int ny) { return ny <= 16 ? 4 : ny <= 32 ? 2 : ny <= 64 ? 1 : ny <= 96 ? 2 : 1; }

// V: 16, 32, 64 (lanes per plane), 96 (two planes in three operations), 128 (one plane in two).
// NT: rows of whole lateral tiles pass the caches by (as the aligned sweeps; FP64, 64 x 64 cells: 685 us against
// 708); where a row ends inside a tile, its 128-byte line is written by two rows and has to meet in the cache
// (50 x 50 cells: 218 us against 293, 45 x 70: 860 against 1096).
template <typename T, int V, bool NT>
__device__ __forceinline__ void tpass_packed_body(const TParams<T> &P, unsigned wave)
{
    wave = __builtin_amdgcn_readfirstlane(wave);
    if constexpr (V <= 64)
        tpass_pack_body<T, V, NT ? 2 : 0>(P, wave);
    else
        tpass_packw_body<T, V == 96, NT ? 2 : 0>(P, wave);
}

template <typename T, int V, bool NT>
__global__ __launch_bounds__(256) void tpass_packed_kernel(TParams<T> P)
{
    tpass_packed_body<T, V, NT>(P, blockIdx.x * 4 + (threadIdx.x >> 6));
}

// FP32, ny <= 64, slabs past the packed sweep's buffer resources (1 GiB): the same sweep, one plane per wave, by pointers.
// Half the time of the shuffle sweep: 31 x 31 angles, 2 groups, ms, 8500 x 33 cells (slabs of 1.08 GB) 6.9 -> 3.4, 14000 x 20
// 10.4 -> 5.4, 8801 x 64 (2.2 GB) 7.5 -> 3.8.
static inline bool tpass_far_fits(const TParams<float> &P) { return P.ny <= 64 && P.nplanes < (1L << 31) - 256; }
__device__ __forceinline__ void tpass_far_body(const TParams<float> &P, unsigned wave)
{
    tpass_pack_planes<float, 64>(P, __builtin_amdgcn_readfirstlane(wave),
                                 [&](unsigned slab) { return SlabFar<float>{P.psi + slab * P.NLINE}; });
}
__global__ __launch_bounds__(256) void tpass_far_kernel(TParams<float> P)
{
    tpass_far_body(P, blockIdx.x * 4 + (threadIdx.x >> 6));
}

// One instantiation per width and cache policy: f(V, NT) as compile-time constants.
template <typename F>
static void tpass_packed_select(int ny, F &&f)
{
    using std::integral_constant;
    if (ny <= 16) f(integral_constant<int, 16>(), std::false_type());
    else if (ny < 32) f(integral_constant<int, 32>(), std::false_type());
    else if (ny == 32) f(integral_constant<int, 32>(), std::true_type());
    else if (ny < 64) f(integral_constant<int, 64>(), std::false_type());
    else if (ny == 64) f(integral_constant<int, 64>(), std::true_type());
    else if (ny < 96) f(integral_constant<int, 96>(), std::false_type());
    else if (ny == 96) f(integral_constant<int, 96>(), std::true_type());
    else if (ny < 128) f(integral_constant<int, 128>(), std::false_type());
    else f(integral_constant<int, 128>(), std::true_type());
}

template <typename T>
hipError_t launch_tpass(const TParams<T> &P, hipStream_t st)
{
    if constexpr (sizeof(T) == 4) {
        const dim3 grid((unsigned)((P.nplanes + 3) / 4));
        if (P.nx % TPASS_PF == 0 && P.ny == 64) {
            hipLaunchKernelGGL(tpass_affine_kernel<64>, grid, dim3(256), 0, st, P);
            return hipGetLastError();
        }
        if (P.nx % TPASS_PF == 0 && P.ny == 32) {
            const long pairs = (P.nplanes + 1) / 2;
            hipLaunchKernelGGL(tpass_pair_kernel, dim3((unsigned)((pairs + 3) / 4)), dim3(256), 0, st, P);
            return hipGetLastError();
        }
        if (P.nx % TPASS_W2_PF == 0 && P.ny == 96 && P.nplanes % 2 == 0 && 2 * P.NLINE * 4 < 0x7fffffffL &&
            P.nplanes / 2 < 0x7fffffffL) {
            const long pairs = P.nplanes / 2;
            hipLaunchKernelGGL(tpass_wide2_kernel, dim3((unsigned)((pairs + 3) / 4)), dim3(256), TP_W2_LDS, st, P);
            return hipGetLastError();
        }
        if (P.nx % TPASS_PF == 0 && P.ny == 96) {
            hipLaunchKernelGGL(tpass_wide_kernel<96>, grid, dim3(256), 0, st, P);
            return hipGetLastError();
        }
        if (P.nx % TPASS_PF == 0 && P.ny == 128) {
            hipLaunchKernelGGL(tpass_wide_kernel<128>, grid, dim3(256), 0, st, P);
            return hipGetLastError();
        }
    }
    if (tpass_packed_fits(P)) {
        const long waves = (P.nplanes + tpass_packed_planes(P.ny) - 1) / tpass_packed_planes(P.ny);
        const dim3 grid((unsigned)((waves + 3) / 4));
        tpass_packed_select(P.ny, [&](auto v, auto nt) {
            hipLaunchKernelGGL((tpass_packed_kernel<T, decltype(v)::value, decltype(nt)::value>), grid, dim3(256), 0, st, P);
        });
        return hipGetLastError();
    }
    const unsigned nb = (unsigned)((P.nplanes + 3) / 4);
    if constexpr (sizeof(T) == 4) {
        if (tpass_far_fits(P)) {
            hipLaunchKernelGGL(tpass_far_kernel, dim3(nb), dim3(256), 0, st, P);
            return hipGetLastError();
        }
    }
    const int nseg = (P.ny + 63) / 64;
    switch (nseg) {
    case 1: hipLaunchKernelGGL((tpass_kernel<T, 1>), dim3(nb), dim3(256), 0, st, P); break;
    case 2: hipLaunchKernelGGL((tpass_kernel<T, 2>), dim3(nb), dim3(256), 0, st, P); break;
    case 3: hipLaunchKernelGGL((tpass_kernel<T, 3>), dim3(nb), dim3(256), 0, st, P); break;
    case 4: hipLaunchKernelGGL((tpass_kernel<T, 4>), dim3(nb), dim3(256), 0, st, P); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// ----------------------------------------------------------------------------- angular pass
// y_M = sum_n sin(pi M n / N) x_n over the interior nodes n, M = 1..N-1, with the even/odd split
// sin(pi M (N-n)/N) = (-1)^(M+1) sin(pi M n/N).  S[(M-1)*(N-1) + (n-1)] holds the sines.
// They are scalar loads by tab(): left to the compiler, a kernel that stores before them reads them per lane and spills.
template <typename T, int N>
__device__ __forceinline__ void dst1(const T (&x)[N - 1], T (&y)[N - 1], const T *__restrict__ S)
{
    constexpr int H = N / 2;
    T sp[H], dm[H];
#pragma unroll
    for (int n = 1; n < H; ++n) {
        sp[n - 1] = x[n - 1] + x[N - n - 1];
        dm[n - 1] = x[n - 1] - x[N - n - 1];
    }
    sp[H - 1] = x[H - 1];
#pragma unroll
    for (int M = 1; M < N; M += 2) {   // odd modes: symmetric part + centre node
        T acc = T(0);
#pragma unroll
        for (int n = 1; n <= H; ++n) acc += tab(S, (M - 1) * (N - 1) + (n - 1)) * sp[n - 1];
        y[M - 1] = acc;
    }
#pragma unroll
    for (int M = 2; M < N; M += 2) {   // even modes: antisymmetric part
        T acc = T(0);
#pragma unroll
        for (int n = 1; n < H; ++n) acc += tab(S, (M - 1) * (N - 1) + (n - 1)) * dm[n - 1];
        y[M - 1] = acc;
    }
}

// The angular step of ntile lateral tiles (ONE: one) in LDS, L0 = [tile][NA][PC], rho their densities;
// all nt threads of the block, which sees the results after the barrier that ends it.
template <typename T, int N, bool ONE>
__device__ __forceinline__ void apass_cells(const AParams<T> &P, T *L0, const T *rho, int g, int ntile, int nt)
{
    constexpr int m = N - 1, NA = m * m, PC = PBS_PT;
    constexpr T inv2N = T(2) / T(N);
    // forward transform over the first angular index for every (j, column)
    for (int it = threadIdx.x; it < ntile * m * PC; it += nt) {
        T *L = ONE ? L0 : L0 + it / (m * PC) * (NA * PC);
        const int j = (ONE ? it : it % (m * PC)) / PC, c = it % PC;
        T x[m], y[m];
#pragma unroll
        for (int i = 0; i < m; ++i) x[i] = L[(i * m + j) * PC + c];
        dst1<T, N>(x, y, P.S);
#pragma unroll
        for (int k = 0; k < m; ++k) L[(k * m + j) * PC + c] = y[k];
    }
    __syncthreads();
    // over the second index: forward, CN factor (1 + a lam)/(1 - a lam), inverse
    const T coef = T(0.25) * P.h * P.sig[g];   // (h/2) * sigma_tr/2, times rho
    for (int it = threadIdx.x; it < ntile * m * PC; it += nt) {
        T *L = ONE ? L0 : L0 + it / (m * PC) * (NA * PC);
        const int k = (ONE ? it : it % (m * PC)) / PC, c = it % PC;
        const T al = coef * rho[ONE ? c : it / (m * PC) * PC + c];
        const T lk = P.lam[k];
        T x[m], y[m];
#pragma unroll
        for (int j = 0; j < m; ++j) x[j] = L[(k * m + j) * PC + c];
        dst1<T, N>(x, y, P.S);
#pragma unroll
        for (int n = 0; n < m; ++n) {
            const T lm = al * (lk + P.lam[n]);
            y[n] = y[n] * (T(1) + lm) * fast_rcp(T(1) - lm);
        }
        dst1<T, N>(y, x, P.S);
#pragma unroll
        for (int j = 0; j < m; ++j) L[(k * m + j) * PC + c] = x[j] * inv2N;
    }
    __syncthreads();
    // inverse over the first index
    for (int it = threadIdx.x; it < ntile * m * PC; it += nt) {
        T *L = ONE ? L0 : L0 + it / (m * PC) * (NA * PC);
        const int j = (ONE ? it : it % (m * PC)) / PC, c = it % PC;
        T x[m], y[m];
#pragma unroll
        for (int k = 0; k < m; ++k) x[k] = L[(k * m + j) * PC + c];
        dst1<T, N>(x, y, P.S);
#pragma unroll
        for (int i = 0; i < m; ++i) L[(i * m + j) * PC + c] = y[i] * inv2N;
    }
    __syncthreads();
}

// one lateral tile of one slab per block
template <typename T, int N>
__global__ __launch_bounds__(256) void apass_kernel(AParams<T> P)
{
    constexpr int NA = (N - 1) * (N - 1), NV = NA * PBS_PT;
    __shared__ T L[NV];              // [NA][PBS_PT]
    const int tid = threadIdx.x;
    const long stack = blockIdx.y;   // (k*G + g)*2 + l
    const int g = (int)((stack / 2) % P.G), pb = blockIdx.x;
    T *blk = P.psi + stack * P.NLINE + (long)pb * NV;
    // 8 loads in flight per thread before their LDS stores (a load-store loop waits for each in turn)
    for (int i0 = tid; i0 < NV; i0 += 8 * 256) {
        T v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int idx = i0 + u * 256;
            if (idx < NV) v[u] = blk[idx];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int idx = i0 + u * 256;
            if (idx < NV) L[idx] = v[u];
        }
    }
    __syncthreads();
    apass_cells<T, N, true>(P, L, P.rho + (long)pb * PBS_PT, g, 1, 256);
    for (int idx = tid; idx < NV; idx += 256) blk[idx] = L[idx];
}

template <typename T, int N>
static hipError_t launch_apass_n(const AParams<T> &P, long nstack, hipStream_t st)
{
    hipLaunchKernelGGL((apass_kernel<T, N>), dim3(P.NPB, (unsigned)nstack), dim3(256), 0, st, P);
    return hipGetLastError();
}

// ------------------------------------------- transport, angular step, transport of a small slab in one launch
// The three passes between two energy sweeps read and write the fluence once each, and on the smallest grids each
// of them is a launch of a few microseconds that waits for its loads.  One block holds a whole (group, coefficient)
// slab of a generation in LDS: the transport sweeps of its planes read it from memory, the angular step of its
// cells works in place, the second transport writes it back.  The arithmetic is that of the passes by themselves.
// 1024 threads, for the loads in flight: 512 cost 2 us more.  Whole steps, us, three launches -> one:
// 4 x 4 cells, 11 x 11 angles, 60 groups, 2 generations 64 -> 59 (FP64 84 -> 76); 16 x 16, 7 x 7, 48 71 -> 61
// (FP64 86 -> 73); 32 x 32, 5 x 5, 60 97 -> 80; 16 x 16, 11 x 11, 48 90 (two streams) -> 86.
constexpr int TAT_NT = 1024;
constexpr long TAT_SLAB = 131072;   // bytes of a slab held in LDS (of 160 KB)
template <typename T>
struct SlabLds {
    using Off = unsigned;
    char *p;
    unsigned zero, dump;   // beyond the slab: a zero to load, a place to store to, for lanes without a cell
    __device__ __forceinline__ T load(unsigned o) const { return *reinterpret_cast<const T *>(p + min(o, zero)); }
    __device__ __forceinline__ void store(T v, unsigned o) const { *reinterpret_cast<T *>(p + min(o, dump)) = v; }
};
template <typename T, typename FROM, typename TO>
struct SlabMove {
    using Off = unsigned;
    static constexpr Off NONE = 0x80000000u;
    FROM from;
    TO to;
    __device__ __forceinline__ T load(unsigned o) const { return from.load(o); }
    __device__ __forceinline__ void store(T v, unsigned o) const { to.store(v, o); }
};

__device__ __forceinline__ void dose_reduce_body(double *edep, const double *dep, int ngen, int NA, int nslot,
                                                 long NLINE, int NP, int pb);

// blocks 0 .. nstack - 1: one slab each; those after them: the step's dose reductions, a job and lateral tile each
template <typename T, int N, int W>
__global__ __launch_bounds__(TAT_NT) void tat_kernel(TParams<T> P, AParams<T> A, int nstack, DoseJobs J)
{
    constexpr int NA = (N - 1) * (N - 1);
    if ((int)blockIdx.x >= nstack) {
        const int q = blockIdx.x - nstack, j = q / A.NPB;
        dose_reduce_body(J.row[j], J.dep[j], J.ngen[j], NA, J.nslot, P.NLINE, P.nx * P.ny, q % A.NPB);
        return;
    }
    extern __shared__ char smem_raw[];
    const long stack = blockIdx.x;   // (k*G + g)*2 + l
    const unsigned bytes = (unsigned)(P.NLINE * (long)sizeof(T));
    const SlabLds<T> lds{smem_raw, bytes, bytes + 8};
    const SlabBuf<T, 0> buf(P.psi + stack * P.NLINE, bytes);
    T *L = reinterpret_cast<T *>(smem_raw);
    // cells that pad the last tile, and the zero
    const int np = P.nx * P.ny, npad = A.NPB * PBS_PT - np;
    for (int i = threadIdx.x; i < npad * NA; i += TAT_NT)
        L[((long)(A.NPB - 1) * NA + i / npad) * PBS_PT + PBS_PT - npad + i % npad] = T(0);
    if (threadIdx.x == 0) *reinterpret_cast<T *>(smem_raw + bytes) = T(0);
    P.nplanes = NA;
    const unsigned wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    for (unsigned w = wave; w < (NA * W + 63) / 64; w += TAT_NT / 64)
        tpass_pack_planes<T, W>(P, w, [&](unsigned) { return SlabMove<T, SlabBuf<T, 0>, SlabLds<T>>{buf, lds}; });
    __syncthreads();
    apass_cells<T, N, false>(A, L, A.rho, (int)((stack / 2) % A.G), A.NPB, TAT_NT);
    for (unsigned w = wave; w < (NA * W + 63) / 64; w += TAT_NT / 64)
        tpass_pack_planes<T, W>(P, w, [&](unsigned) { return SlabMove<T, SlabLds<T>, SlabBuf<T, 0>>{lds, buf}; });
}

// What the kernel can take: the angular grids it is built for, registers of 1024 threads, a slab in LDS.
template <typename T>
static bool tat_takes(int nth, int ny, long nline)
{
    if (nth != 6 && nth != 8 && nth != 10 && nth != 12) return false;
    return ny <= (sizeof(T) == 8 && nth >= 10 ? 16 : 32) && nline * (long)sizeof(T) <= TAT_SLAB;
}

// Where it pays.  A CU holds one block (77-127 registers of 1024 threads), so 256 slabs are one round; fewer than 96
// leave too many CUs idle (5 x 7, 11 x 11, 40, one generation: 80 slabs, 32 against 31 us; 60: 36.7 against 37.7).  A
// second round still beats the passes on one stream by 5 to 15 % (16 x 16, 7 x 7, 120, two generations 93 against 108
// us; 12 x 16, 7 x 7, 60, four, FP64 149 against 163), except for wide grids of large slabs (8 x 20, 11 x 11, 160, one
// generation of 77 KB 93 against 87).  With two generations the passes on two streams, if they may take them (overlap),
// are the better ones where the slabs take long: us a step here | there, 16 x 20, 7 x 7, 100 (63 KB) 104 | 98; 12 x 20,
// 7 x 7, 100 (50 KB) 95 | 98; 10 x 16, 11 x 11, 128 (77 KB) 129 | 123; 8 x 16, 11 x 11, 100 (62 KB) 101 | 108; 24 x 32, 5 x 5,
// 128 (77 KB) 120 | 130; FP64 16 x 20, 5 x 5, 100 (64 KB) 108 | 104; 8 x 20, 7 x 7, 100 (63 KB) 109 | 112; 4 x 4, 11 x 11,
// 100 (31 KB) 105 | 100.
template <typename T>
bool tat_fits(int nth, int ny, long nline, long nstack, int ngen, bool overlap)
{
    if (!tat_takes<T>(nth, ny, nline) || nstack < 96 || nstack > 512) return false;
    if (nstack <= 256) return true;
    constexpr bool F64 = sizeof(T) == 8;
    long lim = 80000;   // bytes of a slab in two rounds
    if (F64 || nth > 6) {
        if (ngen == 1 && ny > 16) lim = 64000;
        if (ngen == 2 && overlap) lim = F64 && nth == 12 ? 0 : !F64 && ny > 16 ? 51000 : 64000;
    }
    return nline * (long)sizeof(T) < lim;
}
template <typename T, int N>
static void launch_tat_n(const TParams<T> &P, const AParams<T> &A, long nstack, const DoseJobs &J, hipStream_t st)
{
    const dim3 grid((unsigned)(nstack + (long)J.n * A.NPB));
    const size_t sh = P.NLINE * sizeof(T) + 16;
    if (P.ny <= 16) {
        hipLaunchKernelGGL((tat_kernel<T, N, 16>), grid, dim3(TAT_NT), sh, st, P, A, (int)nstack, J);
    } else {
        if constexpr (sizeof(T) == 4 || N < 10)
            hipLaunchKernelGGL((tat_kernel<T, N, 32>), grid, dim3(TAT_NT), sh, st, P, A, (int)nstack, J);
    }
}
template <typename T>
hipError_t launch_tat(const TParams<T> &P, const AParams<T> &A, int nth, long nstack, const DoseJobs &J, hipStream_t st)
{
    if (!tat_takes<T>(nth, P.ny, P.NLINE) || P.NA != (nth - 1) * (nth - 1)) return hipErrorInvalidValue;
    switch (nth) {
    case 6: launch_tat_n<T, 6>(P, A, nstack, J, st); break;
    case 8: launch_tat_n<T, 8>(P, A, nstack, J, st); break;
    case 10: launch_tat_n<T, 10>(P, A, nstack, J, st); break;
    default: launch_tat_n<T, 12>(P, A, nstack, J, st); break;
    }
    return hipGetLastError();
}

// MFMA version for nth = 32 (31 interior nodes), FP32.  Each of the four 31-point sine transforms
// is split by mode parity into two 16 x 16 blocks (odd modes act on x_n + x_{32-n} plus the centre
// node, even modes on x_n - x_{32-n}); the inverse uses the transposed blocks with the output
// butterflies x_n = u + v, x_{32-n} = u - v.  Every block product is a chain of four
// v_mfma_f32_16x16x4_f32 whose 16 columns are 16 lateral cells of one angular line.  The block's
// 31 x 31 x 16 values stay in LDS between the passes over the two indices (a block barrier after each);
// within a pass each wave owns whole lines and works in place.
// LDS banks: an MFMA result holds rows 4 (lane / 16) + q in lane groups of 16, so writing row r of the
// result with r = 4 (lane / 16) + q puts the four lane groups of one store 4 rows apart, a multiple of
// the bank count at every row stride here (4-way conflicts).  The operand rows are therefore permuted,
// result row 4 g + q holding output index 4 q + g, so one store's lane groups are one row apart; and
// the modes are kept de-interleaved (odd block in rows 0-15, even block in rows 16-30, in both angular
// directions), so consecutive odd (even) modes are adjacent.  Every LDS access then reaches 32
// distinct banks per half wave.  The same permutation makes a result the next product's operand: element
// q of lane group g holds index 4 q + g, which lane group g supplies at chain step q, so the modes of the
// second index go from the forward product to the inverse one in registers.
//   Ktab[(mat*4 + s)*64 + lane] = A_mat[perm(lane % 16)][4 s + lane / 16] for mat = Sodd, Seven and
//   A_mat[4 s + lane / 16][perm(lane % 16)] for mat = Sodd^T, Seven^T, perm(4 g + q) = 4 q + g.
typedef float floatx4 __attribute__((ext_vector_type(4)));

typedef double doublex4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ floatx4 mfma16(float a, float b, floatx4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ doublex4 mfma16(double a, double b, doublex4 c)
{
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// 16 waves per block: the dependent MFMA chains of a line are short, so latency is hidden by the
// number of lines in flight (2 blocks of 61.5 KB LDS per CU = 32 waves)
constexpr int APASS32_NT = 1024;
__device__ __forceinline__ void apass_mfma32_body(const AParams<float> &P, const float *__restrict__ Ktab, long stack,
                                                  int pb, int half)
{
    constexpr int m = 31, NA = 961, PC = 16;
    __shared__ float L[NA * PC];   // L[a*16 + c], a = i*31 + j
    const int c0 = half * PC;
    const int g = (int)((stack / 2) % P.G);
    float *blk = P.psi + stack * P.NLINE + (long)pb * NA * PBS_PT + c0;
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int r4 = lane >> 4, cc = lane & 15;
    for (int idx = tid; idx < NA * 4; idx += APASS32_NT) {
        const int a = idx >> 2, q = idx & 3;
        *reinterpret_cast<float4 *>(&L[a * PC + q * 4]) = *reinterpret_cast<const float4 *>(blk + (long)a * PBS_PT + q * 4);
    }
    float Ao[4], Ae[4], Bo[4], Be[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        Ao[s] = Ktab[(0 * 4 + s) * 64 + lane];
        Ae[s] = Ktab[(1 * 4 + s) * 64 + lane];
        Bo[s] = Ktab[(2 * 4 + s) * 64 + lane];
        Be[s] = Ktab[(3 * 4 + s) * 64 + lane];
    }
    // result row 4 r4 + q holds mode (or node) block index 4 q + r4
    float lamO[4], lamE[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int r = 4 * q + r4;
        lamO[q] = P.lam[2 * r];
        lamE[q] = r < 15 ? P.lam[2 * r + 1] : 0.f;
    }
    const float al = 0.25f * P.h * P.sig[g] * P.rho[(long)pb * PBS_PT + c0 + cc];
    __syncthreads();

    // forward over the first angular index; line = column j.  Odd mode r -> row r, even mode r -> row 16 + r.
    for (int j = wid; j < m; j += APASS32_NT / 64) {
        floatx4 yo = {0.f, 0.f, 0.f, 0.f}, ye = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int ip = 4 * s + r4;
            const float xa = L[(ip * m + j) * PC + cc];
            const float xb = ip < 15 ? L[((30 - ip) * m + j) * PC + cc] : 0.f;
            yo = mfma16(Ao[s], ip < 15 ? xa + xb : xa, yo);
            ye = mfma16(Ae[s], xa - xb, ye);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int r = 4 * q + r4;
            L[(r * m + j) * PC + cc] = yo[q];
            if (r < 15) L[((16 + r) * m + j) * PC + cc] = ye[q];
        }
    }
    __syncthreads();
    // over the second index: forward, CN factor, inverse; line = row k (odd mode k, or even mode k - 16, of
    // the first index)
    for (int k = wid; k < m; k += APASS32_NT / 64) {
        floatx4 zo = {0.f, 0.f, 0.f, 0.f}, ze = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int jp = 4 * s + r4;
            const float ya = L[(k * m + jp) * PC + cc];
            const float yb = jp < 15 ? L[(k * m + 30 - jp) * PC + cc] : 0.f;
            zo = mfma16(Ao[s], jp < 15 ? ya + yb : ya, zo);
            ze = mfma16(Ae[s], ya - yb, ze);
        }
        const float lk = P.lam[k < 16 ? 2 * k : 2 * (k - 16) + 1];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int r = 4 * q + r4;
            const float to = al * (lk + lamO[q]);
            zo[q] = zo[q] * (1.f + to) * __builtin_amdgcn_rcpf(1.f - to);
            const float te = al * (lk + lamE[q]);
            ze[q] = r < 15 ? ze[q] * (1.f + te) * __builtin_amdgcn_rcpf(1.f - te) : 0.f;
        }
        // the scaled modes are already the inverse's B operands: element s of lane group r4 holds mode
        // 4 s + r4, the operand of step s (the permuted rows make the MFMA result layout the operand layout)
        floatx4 u = {0.f, 0.f, 0.f, 0.f}, v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            u = mfma16(Bo[s], zo[s], u);
            v = mfma16(Be[s], ze[s], v);
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int jp = 4 * q + r4;
            if (jp < 15) {
                L[(k * m + jp) * PC + cc] = u[q] + v[q];
                L[(k * m + 30 - jp) * PC + cc] = u[q] - v[q];
            } else {
                L[(k * m + 15) * PC + cc] = u[q];
            }
        }
    }
    __syncthreads();
    // inverse over the first index, with the (2/N)^2 normalisation
    constexpr float sc = (2.f / 32.f) * (2.f / 32.f);
    for (int j = wid; j < m; j += APASS32_NT / 64) {
        floatx4 u = {0.f, 0.f, 0.f, 0.f}, v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int r = 4 * s + r4;
            const float bo = L[(r * m + j) * PC + cc];
            const float be = r < 15 ? L[((16 + r) * m + j) * PC + cc] : 0.f;
            u = mfma16(Bo[s], bo, u);
            v = mfma16(Be[s], be, v);
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int ip = 4 * q + r4;
            if (ip < 15) {
                L[(ip * m + j) * PC + cc] = (u[q] + v[q]) * sc;
                L[((30 - ip) * m + j) * PC + cc] = (u[q] - v[q]) * sc;
            } else {
                L[(15 * m + j) * PC + cc] = u[q] * sc;
            }
        }
    }
    __syncthreads();
    for (int idx = tid; idx < NA * 4; idx += APASS32_NT) {
        const int a = idx >> 2, q = idx & 3;
        *reinterpret_cast<float4 *>(blk + (long)a * PBS_PT + q * 4) = *reinterpret_cast<const float4 *>(&L[a * PC + q * 4]);
    }
}

// Blocks of the 16-cell forms per stack, and a block's lateral tile and first cell.  From 8 tiles on the two halves of one tile
// are 8 workgroups apart (one XCD, shared L2 lines), in whole groups of 8 tiles; fewer tiles are packed, as most of
// such a group would be empty blocks (2 tiles, 15 x 15 angles, 60 groups: 33 -> 21 us).
__host__ __device__ constexpr int apass_half_blocks(int npb) { return npb < 8 ? 2 * npb : (npb + 7) / 8 * 16; }
__device__ __forceinline__ void apass_half_tile(int bid, int npb, int &pb, int &half)
{
    pb = npb < 8 ? bid >> 1 : (bid >> 4) * 8 + (bid & 7);
    half = npb < 8 ? bid & 1 : (bid >> 3) & 1;
}

// two blocks per CU need <= 64 VGPRs (8 waves per SIMD)
__global__ __launch_bounds__(APASS32_NT) __attribute__((amdgpu_waves_per_eu(8))) void apass_mfma32_kernel(
    AParams<float> P, const float *__restrict__ Ktab, int npb)
{
    int pb, half;
    apass_half_tile(blockIdx.x, npb, pb, half);
    if (pb >= npb) return;
    apass_mfma32_body(P, Ktab, blockIdx.y, pb, half);
}

hipError_t launch_apass_mfma32(const AParams<float> &P, const float *Ktab, long nstack, hipStream_t st)
{
    hipLaunchKernelGGL(apass_mfma32_kernel, dim3(apass_half_blocks(P.NPB), (unsigned)nstack), dim3(APASS32_NT), 0, st, P, Ktab, P.NPB);
    return hipGetLastError();
}

// The other matrix forms: N = 16 (one dense 16 x 16 product per line, zero-padded, a chain of four), 20 and 24 (split by
// mode parity as above), and N = 32 in FP64.  What bounded the vector transform they replace was its set-up around the
// arithmetic, not the arithmetic: half a wave's lanes per line, the sine table through scalar loads in every line, a
// block barrier per phase with 12 waves per CU.  A block holds 16 cells of one lateral tile; its waves take whole lines
// and work in place.  As in the 32-node pass the FP32 operand rows are permuted, so that result element q of lane
// group g holds index 4 q + g: a store's lane groups land in adjacent rows, and the modes of the second index feed the
// inverse product straight from registers.  FP64 results come out in that order by themselves (row 4 q + lane / 16).
//   Ktab: dense, [s*64 + lane] = S[perm(lane % 16)][4 s + lane / 16], S[r][k] = sin(pi (r+1)(k+1) / N) (symmetric: the
//   inverse uses it too); split as above.
// Measured, us per launch of two generations, before -> after: FP32 40 x 40 cells, 60 groups, N = 20 686 -> 343 and N =
// 24 1144 -> 432; 45 x 70, N = 20, 75, three generations 2487 -> 1060; 64 x 64, N = 16, 96 657 -> 640 (4.4 TB/s; the four
// loads of a thread in flight before their LDS stores); FP64 64 x 64, N = 16, 64 1311 -> 881; 40 x 40, 60, N = 20 970 -> 775
// and N = 24 1161 -> 1000; 32 x 32, 32, N = 32 828 -> 700.  Tried and dropped: both 16-cell groups of a tile in one block (1-18 %
// slower), 4 or 16 waves instead of 8 for the split forms (5-25 %), 8 instead of 4 for N = 16 in FP32 (7 %; in FP64 8 are
// 3 % faster), blocks that stay and load their next tile while they transform the present one (N = 16: 5-15 % slower, the
// registers of the tile cost more waves than the overlap gains).  Below 16 nodes the vector transform stays: its
// lines are short enough that its blocks keep 32 waves per CU, and the matrix form took 1.3-1.7 times as long at N = 8 and
// 10 and 1.25 times at N = 12.
template <typename T, int N>
struct AngMfma {
    static constexpr int m = N - 1, NA = m * m;
    static constexpr bool SPLIT = N > 16;
    static constexpr int H = SPLIT ? N / 2 : m;       // odd (or all) modes and operand nodes
    static constexpr int HE = SPLIT ? N / 2 - 1 : 0;  // even modes
    static constexpr int KS = (H + 3) / 4;            // 4-node steps
    static constexpr int NT = !SPLIT && sizeof(T) == 4 ? 256 : 512;
    static constexpr int CH = 16 / (int)sizeof(T);    // values per 16-byte access
    typedef T T4 __attribute__((ext_vector_type(4)));
    typedef T TC __attribute__((ext_vector_type(CH)));
};

template <typename T, int N>
__device__ __forceinline__ void apass_mfma_body(const AParams<T> &P, const T *__restrict__ Ktab, long stack, int pb, int c0)
{
    using C = AngMfma<T, N>;
    using T4 = typename C::T4;
    using TC = typename C::TC;
    constexpr int m = C::m, NA = C::NA, H = C::H, HE = C::HE, KS = C::KS, NT = C::NT, CH = C::CH;
    constexpr bool SPLIT = C::SPLIT;
    __shared__ T L[NA * 16];   // [a][cell]
    const int g = (int)((stack / 2) % P.G);
    T *blk = P.psi + stack * P.NLINE + (long)pb * NA * PBS_PT + c0;
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int r4 = lane >> 4, cc = lane & 15;
    // tile to LDS and back, 16 bytes per lane, several loads in flight
    constexpr int CPR = 16 / CH, NCHK = NA * CPR, UL = 4;
    auto lds_at = [&](int idx) { return reinterpret_cast<TC *>(&L[idx * CH]); };
    auto mem_at = [&](int idx) { return reinterpret_cast<TC *>(blk + (long)(idx / CPR) * PBS_PT + (idx % CPR) * CH); };
    for (int i0 = tid; i0 < NCHK; i0 += UL * NT) {
        TC v[UL];
#pragma unroll
        for (int u = 0; u < UL; ++u)
            if (i0 + u * NT < NCHK) v[u] = *mem_at(i0 + u * NT);
#pragma unroll
        for (int u = 0; u < UL; ++u)
            if (i0 + u * NT < NCHK) *lds_at(i0 + u * NT) = v[u];
    }
    // operand rows: forward odd (or dense) and even, inverse odd and even (dense: the sine matrix is symmetric)
    T Ao[KS], Ae[KS], Bo[KS], Be[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        Ao[s] = Ktab[(0 * 4 + s) * 64 + lane];
        if constexpr (SPLIT) {
            Ae[s] = Ktab[(1 * 4 + s) * 64 + lane];
            Bo[s] = Ktab[(2 * 4 + s) * 64 + lane];
            Be[s] = Ktab[(3 * 4 + s) * 64 + lane];
        }
    }
    // result element q of lane group r4 holds index 4 q + r4
    T lamO[KS], lamE[KS];
#pragma unroll
    for (int q = 0; q < KS; ++q) {
        const int r = 4 * q + r4;
        lamO[q] = r < H ? P.lam[SPLIT ? 2 * r : r] : T(0);
        lamE[q] = SPLIT && r < HE ? P.lam[2 * r + 1] : T(0);
    }
    constexpr T sc = T(2) / T(N);   // after each inverse: values below the normal range round as in the other passes
    const T al = T(0.25) * P.h * P.sig[g] * P.rho[(long)pb * PBS_PT + c0 + cc];
    // a line's operand at step s: node ip, and its mirror image folded in by parity
    auto fold = [&](const T *x, int stride, int s, T &o, T &e) {
        const int ip = 4 * s + r4;
        const T xa = ip < H ? x[ip * stride] : T(0);
        if constexpr (SPLIT) {
            const T xb = ip < HE ? x[(m - 1 - ip) * stride] : T(0);
            o = xa + xb;
            e = xa - xb;   // the centre node (ip = H - 1) meets a zero column of the even matrix
        } else {
            o = xa;
        }
    };
    __syncthreads();
    // forward over the first angular index, line = column j: odd mode r to row r, even mode r to row H + r
    for (int j = wid; j < m; j += NT / 64) {
        T *x = &L[j * 16 + cc];
        T4 yo = {0, 0, 0, 0}, ye = {0, 0, 0, 0};
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            T o, e;
            fold(x, m * 16, s, o, e);
            yo = mfma16(Ao[s], o, yo);
            if constexpr (SPLIT) ye = mfma16(Ae[s], e, ye);
        }
#pragma unroll
        for (int q = 0; q < KS; ++q) {
            const int r = 4 * q + r4;
            if (r < H) x[r * m * 16] = yo[q];
            if (SPLIT && r < HE) x[(H + r) * m * 16] = ye[q];
        }
    }
    __syncthreads();
    // over the second index: forward, CN factor, inverse; line = row k (odd or even mode of the first index)
    for (int k = wid; k < m; k += NT / 64) {
        T *x = &L[k * m * 16 + cc];
        T4 zo = {0, 0, 0, 0}, ze = {0, 0, 0, 0};
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            T o, e;
            fold(x, 16, s, o, e);
            zo = mfma16(Ao[s], o, zo);
            if constexpr (SPLIT) ze = mfma16(Ae[s], e, ze);
        }
        const T lk = P.lam[!SPLIT ? k : k < H ? 2 * k : 2 * (k - H) + 1];
#pragma unroll
        for (int q = 0; q < KS; ++q) {
            const int r = 4 * q + r4;
            const T to = al * (lk + lamO[q]);
            zo[q] = r < H ? zo[q] * (T(1) + to) * fast_rcp(T(1) - to) : T(0);
            if constexpr (SPLIT) {
                const T te = al * (lk + lamE[q]);
                ze[q] = r < HE ? ze[q] * (T(1) + te) * fast_rcp(T(1) - te) : T(0);
            }
        }
        // the scaled modes are already the inverse's operands
        T4 u = {0, 0, 0, 0}, v = {0, 0, 0, 0};
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            u = mfma16(SPLIT ? Bo[s] : Ao[s], zo[s], u);
            if constexpr (SPLIT) v = mfma16(Be[s], ze[s], v);
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int q = 0; q < KS; ++q) {
            const int jp = 4 * q + r4;
            if constexpr (SPLIT) {
                if (jp < HE) {
                    x[jp * 16] = (u[q] + v[q]) * sc;
                    x[(m - 1 - jp) * 16] = (u[q] - v[q]) * sc;
                } else if (jp == H - 1) {
                    x[jp * 16] = u[q] * sc;
                }
            } else if (jp < m) {
                x[jp * 16] = u[q] * sc;
            }
        }
    }
    __syncthreads();
    // inverse over the first index
    for (int j = wid; j < m; j += NT / 64) {
        T *x = &L[j * 16 + cc];
        T4 u = {0, 0, 0, 0}, v = {0, 0, 0, 0};
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const int r = 4 * s + r4;
            const T bo = r < H ? x[r * m * 16] : T(0);
            u = mfma16(SPLIT ? Bo[s] : Ao[s], bo, u);
            if constexpr (SPLIT) {
                const T be = r < HE ? x[(H + r) * m * 16] : T(0);
                v = mfma16(Be[s], be, v);
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int q = 0; q < KS; ++q) {
            const int ip = 4 * q + r4;
            if constexpr (SPLIT) {
                if (ip < HE) {
                    x[ip * m * 16] = (u[q] + v[q]) * sc;
                    x[(m - 1 - ip) * m * 16] = (u[q] - v[q]) * sc;
                } else if (ip == H - 1) {
                    x[ip * m * 16] = u[q] * sc;
                }
            } else if (ip < m) {
                x[ip * m * 16] = u[q] * sc;
            }
        }
    }
    __syncthreads();
    for (int idx = tid; idx < NCHK; idx += NT) *mem_at(idx) = *lds_at(idx);
}

template <typename T, int N>
__device__ __forceinline__ void apass_mfma_block(const AParams<T> &P, const T *__restrict__ Ktab, int bid, long stack, int npb)
{
    int pb, half;
    apass_half_tile(bid, npb, pb, half);
    if (pb >= npb) return;
    apass_mfma_body<T, N>(P, Ktab, stack, pb, 16 * half);
}

template <typename T, int N>
__global__ __launch_bounds__((AngMfma<T, N>::NT)) void apass_mfma_kernel(AParams<T> P, const T *__restrict__ Ktab)
{
    apass_mfma_block<T, N>(P, Ktab, blockIdx.x, blockIdx.y, P.NPB);
}

template <typename T, int N>
static hipError_t launch_apass_mfma_n(const AParams<T> &P, const T *Ktab, long nstack, hipStream_t st)
{
    hipLaunchKernelGGL((apass_mfma_kernel<T, N>), dim3((unsigned)(apass_half_blocks(P.NPB)), (unsigned)nstack),
                       dim3(AngMfma<T, N>::NT), 0, st, P, Ktab);
    return hipGetLastError();
}

bool apass_supported(int nth)
{
    switch (nth) {
    case 4: case 6: case 8: case 10: case 12: case 16: case 20: case 24: case 32: return true;
    default: return false;
    }
}

template <typename T>
hipError_t launch_apass(const AParams<T> &P, const T *Ktab, int nth, long nstack, hipStream_t st)
{
    if constexpr (sizeof(T) == 4) {
        if (nth == 32) return launch_apass_mfma32(P, Ktab, nstack, st);
    }
    switch (nth) {
    case 4: return launch_apass_n<T, 4>(P, nstack, st);
    case 6: return launch_apass_n<T, 6>(P, nstack, st);
    case 8: return launch_apass_n<T, 8>(P, nstack, st);
    case 10: return launch_apass_n<T, 10>(P, nstack, st);
    case 12: return launch_apass_n<T, 12>(P, nstack, st);
    case 16: return launch_apass_mfma_n<T, 16>(P, Ktab, nstack, st);
    case 20: return launch_apass_mfma_n<T, 20>(P, Ktab, nstack, st);
    case 24: return launch_apass_mfma_n<T, 24>(P, Ktab, nstack, st);
    case 32:
        if constexpr (sizeof(T) == 8) return launch_apass_mfma_n<T, 32>(P, Ktab, nstack, st);
        [[fallthrough]];
    default: return hipErrorInvalidValue;
    }
}

// ------------------------------------------------------------------- source angular product
// Q[s][g][pb][a][pt] = sum_a' P2T[a][a'] W[s][g][pb][a'][pt].
// FP32 MFMA version (v_mfma_f32_32x32x2_f32).  Block tile 128 destination nodes x 128 columns
// (4 lateral tiles of one (half-step, group) panel); 4 waves in 2 x 2, each 64 x 64 = 2 x 2
// MFMA tiles.  A is the zero-padded P2 [Kp][Mp] (source-major), staged k-major in LDS like B.
typedef float floatx16 __attribute__((ext_vector_type(16)));

__global__ __launch_bounds__(256) void qgemm_mfma_f32_kernel(QParams<float> P, int nmt, int nnt, long nlogical,
                                                             long per_xcd)
{
    // Workgroups are dispatched round-robin over the 8 XCDs; give every XCD a contiguous range of
    // logical tiles so the M tiles that share one B panel run back to back on the same L2.
    const long bid = blockIdx.x;
    const long logical = (bid & 7) * per_xcd + (bid >> 3);
    if (logical >= nlogical) return;
    const int mt = (int)(logical % nmt);
    const long rest = logical / nmt;
    const int nt = (int)(rest % nnt);
    const long batch = rest / nnt;
    const int s = P.s0 + (int)(batch / P.G), g = (int)(batch % P.G);
    const long off = ((long)s * P.G + g) * P.NLINE;
    const float *__restrict__ P2p = P.P2p + (P.band ? (long)P.band[g] * P.Kp * P.Mp : 0L);
    const float *__restrict__ B = P.W + off;
    float *__restrict__ C = P.Q + off;
    const long NAPT = (long)P.NA * PBS_PT;
    __shared__ float As[16][132];
    __shared__ float Bs[16][132];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int wm = wid >> 1, wn = wid & 1;
    floatx16 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    const int nk = P.Kp / 16;
    float4 ra[2], rb[2];
    auto gload = [&](int kt) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int idx = tid + 256 * i;
            const int k = idx >> 5, q4 = idx & 31;
            ra[i] = *reinterpret_cast<const float4 *>(P2p + (long)(kt * 16 + k) * P.Mp + mt * 128 + q4 * 4);
            const int pb = nt * 4 + (q4 >> 3), pt = (q4 & 7) * 4;
            const int gk = kt * 16 + k;
            if (gk < P.NA && pb < P.NPB)
                rb[i] = *reinterpret_cast<const float4 *>(B + pb * NAPT + (long)gk * PBS_PT + pt);
            else
                rb[i] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
    };
    auto sstore = [&]() {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int idx = tid + 256 * i;
            const int k = idx >> 5, q4 = idx & 31;
            *reinterpret_cast<float4 *>(&As[k][q4 * 4]) = ra[i];
            *reinterpret_cast<float4 *>(&Bs[k][q4 * 4]) = rb[i];
        }
    };
    gload(0);
    sstore();
    __syncthreads();
    for (int kt = 0; kt < nk; ++kt) {
        if (kt + 1 < nk) gload(kt + 1);
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) {
            const int kr = 2 * kk + (lane >> 5);
            float a[2], b[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) a[i] = As[kr][wm * 64 + i * 32 + (lane & 31)];
#pragma unroll
            for (int j = 0; j < 2; ++j) b[j] = Bs[kr][wn * 64 + j * 32 + (lane & 31)];
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], b[j], acc[i][j], 0, 0, 0);
        }
        __syncthreads();
        if (kt + 1 < nk) {
            sstore();
            __syncthreads();
        }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int pb = nt * 4 + wn * 2 + j;
            if (pb >= P.NPB) continue;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = mt * 128 + wm * 64 + i * 32 + (r & 3) + 8 * (r >> 2) + 4 * (lane >> 5);
                if (row < P.NA) C[pb * NAPT + (long)row * PBS_PT + (lane & 31)] = acc[i][j][r];
            }
        }
}

// Split-BF16 version on v_mfma_f32_32x32x16_bf16: each FP32 operand is written as hi + lo
// (hi = bf16(x), lo = bf16(x - hi), |x - hi - lo| <= 2^-16 |x|) and the product is accumulated in
// FP32 as A_lo B_hi + A_hi B_lo + A_hi B_hi (the A_lo B_lo term, O(2^-16), is dropped).
// Block tile 128 destination nodes x 256 columns (8 lateral tiles), BK = 32; 8 waves in 2 x 4,
// each 64 x 64 = 2 x 2 MFMA tiles.  A = P2 split on the host, row-major [Mp][Kp] (k contiguous);
// B arrives split from the energy pass, 8 consecutive source nodes contiguous per lateral cell.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));

// a float moved between the lanes of each quad by the DPP quad permutation CTRL
template <int CTRL>
__device__ __forceinline__ float dpp_quad(float x)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), CTRL, 0xF, 0xF, false));
}

// Stores one 32 x 32 accumulator tile of v_mfma_f32_32x32x16 (rows row0 .. row0 + 31 of lateral tile pb)
// into the source Q [pb][row][32 cells].  Lane l holds column l % 32 of rows (r % 4) + 8 (r / 4) + 4 (l / 32):
// for each group r / 4 a 4 x 4 transpose inside every quad of lanes (two DPP butterfly stages) leaves
// lane t of the quad with row t of the group for the quad's 4 columns, written as one 16-byte store, so a
// wave writes 1 KB contiguous (8 rows of 32 cells) per instruction.  Non-temporal: the source is read
// once, by the next generation's energy pass, and is kept out of the caches the product streams through.
__device__ __forceinline__ void store_source_tile(float *__restrict__ C, long NAPT, int pb, int row0,
                                                  const floatx16 &a, int lane, int NA, int NPB)
{
    const int t4 = lane & 3;
    const bool up1 = (t4 & 1) != 0, up2 = (t4 & 2) != 0;
    // one butterfly: lanes with `up` send x and take the partner's y into x; the others send y and take
    // the partner's x into y (quad_perm [1,0,3,2] for the first stage, [2,3,0,1] for the second)
    auto b1 = [&](float &x, float &y) {
        const float r = dpp_quad<0xB1>(up1 ? x : y);
        if (up1) x = r; else y = r;
    };
    auto b2 = [&](float &x, float &y) {
        const float r = dpp_quad<0x4E>(up2 ? x : y);
        if (up2) x = r; else y = r;
    };
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        float v0 = a[4 * q], v1 = a[4 * q + 1], v2 = a[4 * q + 2], v3 = a[4 * q + 3];
        b1(v0, v1);
        b1(v2, v3);
        b2(v0, v2);
        b2(v1, v3);
        const int row = row0 + 8 * q + 4 * (lane >> 5) + t4;
        if (pb < NPB && row < NA)
            __builtin_nontemporal_store(
                floatx4{v0, v1, v2, v3},
                reinterpret_cast<floatx4 *>(&C[pb * NAPT + (long)row * PBS_PT + ((lane & 31) & ~3)]));
    }
}

// The same tile into the BF16 source [pb][row / 4][32 cells][4] (Qb): lane l holds column l % 32 of rows
// 8 q + 4 (l / 32) + 0..3, i.e. one 4-row group of one cell, which leaves as one 8-byte store (each wave
// instruction writes 2 x 256 B contiguous) with no exchange between lanes.  Rows NA .. NAq - 1 come from
// the zero-padded rows of the transfer matrix.
__device__ __forceinline__ void store_source_tile_bf16(unsigned short *__restrict__ Cb, int NAq, int pb, int row0,
                                                       const floatx16 &a, int lane, int NPB)
{
    typedef unsigned short u16x4 __attribute__((ext_vector_type(4)));
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int row = row0 + 8 * q + 4 * (lane >> 5);
        if (pb < NPB && row < NAq) {
            u16x4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = __builtin_bit_cast(unsigned short, (__bf16)a[4 * q + e]);
            __builtin_nontemporal_store(v, reinterpret_cast<u16x4 *>(&Cb[((long)pb * NAq + row) * PBS_PT + (lane & 31) * 4]));
        }
    }
}

template <int BN, int NPROD>
__device__ __forceinline__ void qgemm_bf16s_body(const QParams<float> &P, const unsigned short *__restrict__ Ahi,
                                                  const unsigned short *__restrict__ Alo, int Kp, int nmt, int nnt,
                                                  long nlogical, long per_xcd, long bid)
{
    constexpr int BK = 32, LD = BK + 8;   // LDS row stride in bf16 elements (80 B)
    constexpr int NPBT = BN / 32;         // lateral tiles per block
    constexpr int WN = BN / 64;           // waves along N (2 along M)
    constexpr int NT = 128 * WN;          // threads
    constexpr bool BLO = NPROD == 3;      // the lo part of the scanned fluence takes part
    constexpr bool ALO = NPROD >= 2;      // the lo part of the transfer matrix takes part
    __shared__ unsigned short sAh[128 * LD], sAl[ALO ? 128 * LD : 8], sBh[BN * LD], sBl[BLO ? BN * LD : 8];
    const long logical = (bid & 7) * per_xcd + (bid >> 3);
    if (logical >= nlogical) return;
    const int mt = (int)(logical % nmt);
    const long rest = logical / nmt;
    const int nt = (int)(rest % nnt);
    const long batch = rest / nnt;
    const int s = P.s0 + (int)(batch / P.G), g = (int)(batch % P.G);
    if (P.band) {   // the transfer matrix of the destination group's band
        const long bo = (long)P.band[g] * 3 * P.Mp * Kp;
        Ahi += bo;
        Alo += bo;
    }
    const long off = ((long)s * P.G + g) * P.NLINE;
    float *__restrict__ C = P.Q + off;
    const int NAq = (P.NA + 3) & ~3;
    unsigned short *__restrict__ Cb = P.Qb ? P.Qb + ((long)s * P.G + g) * P.NPB * NAq * PBS_PT : nullptr;
    const long NAPT = (long)P.NA * PBS_PT;
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int wm = wid / WN, wn = wid % WN;
    floatx16 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    const int nk = Kp / BK;
    // staging: A chunks (row, 8 k) c = tid + NT*i over 128 x 4; B items column tid % BN, octets tid / BN and +2
    constexpr int NA_CH = 512 / NT;
    const int bcol = tid % BN, boct = tid / BN;
    const int bpb = nt * NPBT + (bcol >> 5), bpt = bcol & 31;
    const bool bok = bpb < P.NPB;
    const long bbase = (((long)s * P.G + g) * P.NPB + (bok ? bpb : 0)) * P.NOCT * (PBS_PT * 8) + bpt * 8;
    u16x8 rah[NA_CH], ral[NA_CH];
    u16x8 rbh[2], rbl[2];
    auto gload = [&](int kt) {
#pragma unroll
        for (int c = 0; c < NA_CH; ++c) {
            const int ch = tid + NT * c, arow = ch >> 2, akq = ch & 3;
            const long ao = (long)(mt * 128 + arow) * Kp + kt * BK + akq * 8;
            rah[c] = *reinterpret_cast<const u16x8 *>(Ahi + ao);
            if constexpr (ALO) ral[c] = *reinterpret_cast<const u16x8 *>(Alo + ao);
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int oc = kt * (BK / 8) + boct + 2 * h;
            if (bok && oc < P.NOCT) {
                rbh[h] = *reinterpret_cast<const u16x8 *>(P.Bh + bbase + (long)oc * (PBS_PT * 8));
                if constexpr (BLO) rbl[h] = *reinterpret_cast<const u16x8 *>(P.Bl + bbase + (long)oc * (PBS_PT * 8));
            } else {
                rbh[h] = u16x8{0, 0, 0, 0, 0, 0, 0, 0};
                if constexpr (BLO) rbl[h] = rbh[h];
            }
        }
    };
    auto sstore = [&]() {
#pragma unroll
        for (int c = 0; c < NA_CH; ++c) {
            const int ch = tid + NT * c, arow = ch >> 2, akq = ch & 3;
            *reinterpret_cast<u16x8 *>(&sAh[arow * LD + akq * 8]) = rah[c];
            if constexpr (ALO) *reinterpret_cast<u16x8 *>(&sAl[arow * LD + akq * 8]) = ral[c];
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            *reinterpret_cast<u16x8 *>(&sBh[bcol * LD + (boct + 2 * h) * 8]) = rbh[h];
            if constexpr (BLO) *reinterpret_cast<u16x8 *>(&sBl[bcol * LD + (boct + 2 * h) * 8]) = rbl[h];
        }
    };
    gload(0);
    sstore();
    __syncthreads();
    for (int kt = 0; kt < nk; ++kt) {
        if (kt + 1 < nk) gload(kt + 1);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const int ko = ks * 16 + 8 * (lane >> 5);
            bf16x8 ah[2], al[2], bh[2], bl[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int r = wm * 64 + i * 32 + (lane & 31);
                ah[i] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u16x8 *>(&sAh[r * LD + ko]));
                if constexpr (ALO)
                    al[i] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u16x8 *>(&sAl[r * LD + ko]));
            }
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int cidx = wn * 64 + j * 32 + (lane & 31);
                bh[j] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u16x8 *>(&sBh[cidx * LD + ko]));
                if constexpr (BLO)
                    bl[j] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u16x8 *>(&sBl[cidx * LD + ko]));
            }
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    if constexpr (ALO)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al[i], bh[j], acc[i][j], 0, 0, 0);
                    if constexpr (BLO)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah[i], bl[j], acc[i][j], 0, 0, 0);
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah[i], bh[j], acc[i][j], 0, 0, 0);
                }
        }
        __syncthreads();
        if (kt + 1 < nk) {
            sstore();
            __syncthreads();
        }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
            if (Cb)
                store_source_tile_bf16(Cb, NAq, nt * NPBT + wn * 2 + j, mt * 128 + wm * 64 + i * 32, acc[i][j], lane,
                                       P.NPB);
            else
                store_source_tile(C, NAPT, nt * NPBT + wn * 2 + j, mt * 128 + wm * 64 + i * 32, acc[i][j], lane, P.NA,
                                  P.NPB);
}

// Source product with the energy-scanned fluence read straight from global memory: its split
// layout [g][pb][oct][cell][8] is the register layout of the v_mfma_f32_32x32x16_bf16 B operand
// (lane l: cell l % 32, source nodes 8 (2 kk + l / 32) + 0..7 of the 16-node step kk), so one 16-byte
// buffer load per lane fetches a whole fragment, 1 KB contiguous per wave.  Only the transfer-matrix
// tile (128 destination rows x 64 source nodes, hi and lo) is staged in LDS and shared by the 4 waves.
// Block = 128 rows x 256 cells (8 lateral tiles of 32 cells).  With QG_WM = 1 each wave owns all 128
// rows of 2 lateral tiles (4 x 2 tiles of 32 x 32), so every B fragment is fetched by one wave only;
// with QG_WM = 2 a wave owns 64 rows x 4 lateral tiles.  B fragments of the next QG_PFD 16-node steps
// are in flight while a step computes.
// Tuning knobs (compile-time): B prefetch depth in 16-node steps (single-beam and batched kernels),
// minimum waves per SIMD for the one-product kernels, waves along rows, and two LDS buffers for the
// transfer-matrix stage (one barrier per stage instead of two).
#ifndef QG_PFD
#define QG_PFD 3
#endif
#ifndef QG_PFD_BATCH
#define QG_PFD_BATCH 1
#endif
#ifndef QG_WPE
#define QG_WPE 2
#endif
#ifndef QG_WM
#define QG_WM 1
#endif
#ifndef QG_DB
#define QG_DB 1
#endif

template <int NPROD, int PFD_ = QG_PFD>
__device__ __forceinline__ void qgemm_bf16g_body(const QParams<float> &P, const unsigned short *__restrict__ Ahi,
                                                 const unsigned short *__restrict__ Alo, int Kp, int nmt, int nnt,
                                                 long nlogical, long per_xcd, long bid)
{
    constexpr int BK = 64, LD = BK + 8;   // 64-node stages (the split table is padded to 64); LDS row stride
    constexpr int KS = BK / 16;                  // 16-node steps per stage
    constexpr int NCH = 128 * (BK / 8) / 256;    // A chunks of 8 nodes per thread
    constexpr int NT = 256;
    constexpr bool BLO = NPROD == 3;
    constexpr bool ALO = NPROD >= 2;
    constexpr int WM = QG_WM, WN = 4 / WM;       // waves along rows / along lateral tiles
    constexpr int TI = 4 / WM, TJ = 8 / WN;      // 32-row tiles and lateral tiles per wave
    constexpr int NBUF = QG_DB ? 2 : 1;   // A stages in LDS (2: the next stage is written during this one)
    __shared__ unsigned short sAh[NBUF][128 * LD], sAl[NBUF][ALO ? 128 * LD : 8];
    const long logical = (bid & 7) * per_xcd + (bid >> 3);
    if (logical >= nlogical) return;
    const int mt = (int)(logical % nmt);
    const long rest = logical / nmt;
    const int nt = (int)(rest % nnt);
    const long batch = rest / nnt;
    const int s = P.s0 + (int)(batch / P.G), g = (int)(batch % P.G);
    if (P.band) {   // the transfer matrix of the destination group's band
        const long bo = (long)P.band[g] * 3 * P.Mp * Kp;
        Ahi += bo;
        Alo += bo;
    }
    const long off = ((long)s * P.G + g) * P.NLINE;
    float *__restrict__ C = P.Q + off;
    const int NAq = (P.NA + 3) & ~3;
    unsigned short *__restrict__ Cb = P.Qb ? P.Qb + ((long)s * P.G + g) * P.NPB * NAq * PBS_PT : nullptr;
    const long NAPT = (long)P.NA * PBS_PT;
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int wm = wid / WN, wn = wid % WN;
    floatx16 acc[TI][TJ];
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TJ; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    const int nk = Kp / BK;
    // B fragments through buffer loads on the (s, g) slab of the split fluence: tile j of this wave
    // is lateral tile nt*8 + wn*TJ + j, and this lane's octet at 16-node step kk is 2 kk + lane / 32.
    // An octet past the last one of a tile reads the next tile (finite values that meet the zero
    // columns of the padded transfer matrix); anything past the slab, including lateral tiles past
    // the last one (never stored), reads zero through the buffer range check.  No lane branches, so
    // the waits before the products count exactly the loads in flight.
    const long slab = ((long)s * P.G + g) * P.NPB * P.NOCT * (PBS_PT * 8);
    const int tile_bytes = P.NOCT * (PBS_PT * 8) * 2;
    const int slab_bytes = P.NPB * tile_bytes;
    const __amdgpu_buffer_rsrc_t rbh =
        __builtin_amdgcn_make_buffer_rsrc((void *)(P.Bh + slab), (short)0, slab_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rbl =
        __builtin_amdgcn_make_buffer_rsrc((void *)((BLO ? P.Bl : P.Bh) + slab), (short)0, slab_bytes, 0x00020000);
    const int vb = (nt * 8 + wn * TJ) * tile_bytes + (lane & 31) * 16 + (lane >> 5) * (PBS_PT * 8 * 2);
    auto bload = [&](int kk, u16x8 (&bh)[TJ], u16x8 (&bl)[TJ]) {
#pragma unroll
        for (int j = 0; j < TJ; ++j) {
            const int o = vb + j * tile_bytes + kk * (2 * PBS_PT * 8 * 2);
            bh[j] = __builtin_bit_cast(u16x8, __builtin_amdgcn_raw_buffer_load_b128(rbh, o, 0, 0));
            if constexpr (BLO) bl[j] = __builtin_bit_cast(u16x8, __builtin_amdgcn_raw_buffer_load_b128(rbl, o, 0, 0));
        }
    };
    // A staging: 128 rows x 8 chunks of 8 source nodes, hi and lo, 4 chunks per thread
    u16x8 rah[NCH], ral[NCH];
    auto aload = [&](int kt) {
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            const int ch = tid + NT * c, arow = ch / (BK / 8), akq = ch % (BK / 8);
            const long ao = (long)(mt * 128 + arow) * Kp + kt * BK + akq * 8;
            rah[c] = *reinterpret_cast<const u16x8 *>(Ahi + ao);
            if constexpr (ALO) ral[c] = *reinterpret_cast<const u16x8 *>(Alo + ao);
        }
    };
    auto astore = [&](int buf) {
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            const int ch = tid + NT * c, arow = ch / (BK / 8), akq = ch % (BK / 8);
            *reinterpret_cast<u16x8 *>(&sAh[buf][arow * LD + akq * 8]) = rah[c];
            if constexpr (ALO) *reinterpret_cast<u16x8 *>(&sAl[buf][arow * LD + akq * 8]) = ral[c];
        }
    };
    // ring of B fragments: step kk lives in slot kk % NR; steps kk + 1 .. kk + PFD are in flight.
    // Every load is unconditional (past the end they re-read the last stage or step).
    constexpr int PFD = NPROD == 1 ? PFD_ : 1;
    constexpr int NR = PFD == 1 ? 2 : KS;
    static_assert(PFD < NR && KS % NR == 0, "B ring");
    u16x8 bbh[NR][TJ], bbl[NR][TJ];
    aload(0);
    astore(0);
#pragma unroll
    for (int d = 0; d < PFD; ++d) bload(min(d, KS * nk - 1), bbh[d], bbl[d]);
    __syncthreads();
    for (int kt = 0; kt < nk; ++kt) {
        const int cur = NBUF == 2 ? (kt & 1) : 0;
        aload(min(kt + 1, nk - 1));
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const int kk = KS * kt + ks;
            bload(min(kk + PFD, KS * nk - 1), bbh[(ks + PFD) % NR], bbl[(ks + PFD) % NR]);
            // keep the prefetch ahead of this step's products (the scheduler would sink it to its use)
            __builtin_amdgcn_sched_barrier(0);
            u16x8(&cbh)[TJ] = bbh[ks % NR];
            u16x8(&cbl)[TJ] = bbl[ks % NR];
            const int ko = ks * 16 + 8 * (lane >> 5);
            bf16x8 ah[TI], al[TI];
#pragma unroll
            for (int i = 0; i < TI; ++i) {
                const int r = wm * (32 * TI) + i * 32 + (lane & 31);
                ah[i] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u16x8 *>(&sAh[cur][r * LD + ko]));
                if constexpr (ALO)
                    al[i] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u16x8 *>(&sAl[cur][r * LD + ko]));
            }
#pragma unroll
            for (int j = 0; j < TJ; ++j) {
                const bf16x8 bh = __builtin_bit_cast(bf16x8, cbh[j]);
#pragma unroll
                for (int i = 0; i < TI; ++i) {
                    if constexpr (ALO)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al[i], bh, acc[i][j], 0, 0, 0);
                    if constexpr (BLO)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah[i], __builtin_bit_cast(bf16x8, cbl[j]),
                                                                             acc[i][j], 0, 0, 0);
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah[i], bh, acc[i][j], 0, 0, 0);
                }
            }
        }
        if constexpr (NBUF == 2) {
            // the other buffer was last read in the previous stage, which every wave has left
            if (kt + 1 < nk) astore(cur ^ 1);
            __syncthreads();
        } else {
            __syncthreads();
            if (kt + 1 < nk) {
                astore(0);
                __syncthreads();
            }
        }
    }
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TJ; ++j)
            if (Cb)
                store_source_tile_bf16(Cb, NAq, nt * 8 + wn * TJ + j, mt * 128 + wm * (32 * TI) + i * 32, acc[i][j],
                                       lane, P.NPB);
            else
                store_source_tile(C, NAPT, nt * 8 + wn * TJ + j, mt * 128 + wm * (32 * TI) + i * 32, acc[i][j], lane,
                                  P.NA, P.NPB);
}

template <int NPROD>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(NPROD <= 2 ? QG_WPE : 1))) void qgemm_bf16g_kernel(QParams<float> P, const unsigned short *__restrict__ Ahi,
                                                          const unsigned short *__restrict__ Alo, int Kp, int nmt,
                                                          int nnt, long nlogical, long per_xcd)
{
    qgemm_bf16g_body<NPROD>(P, Ahi, Alo, Kp, nmt, nnt, nlogical, per_xcd, blockIdx.x);
}

template <int BN, int NPROD>
__global__ __launch_bounds__(2 * BN) void qgemm_bf16s_kernel(QParams<float> P, const unsigned short *__restrict__ Ahi,
                                                             const unsigned short *__restrict__ Alo, int Kp, int nmt,
                                                             int nnt, long nlogical, long per_xcd)
{
    qgemm_bf16s_body<BN, NPROD>(P, Ahi, Alo, Kp, nmt, nnt, nlogical, per_xcd, blockIdx.x);
}

// The global-B kernel addresses a (half, g) slab of the split scans with 32-bit buffer offsets; larger
// slabs take the LDS-staged kernel (bitwise the same products: the same accumulation order per output).
static inline bool qgemm_global_b_fits(long NPB, int NOCT)
{
    return (NPB + 9) * NOCT * (long)(PBS_PT * 8 * 2) < (1L << 31);   // tiles up to a block past the end
}

hipError_t launch_qgemm_bf16s(const QParams<float> &P, const unsigned short *Ahi, const unsigned short *Alo, int Kp,
                              int nprod, hipStream_t st, int kind)
{
    if (kind == QGEMM_GLOBAL_B && !qgemm_global_b_fits(P.NPB, P.NOCT)) kind = QGEMM_LDS_256;
    const int bn = kind == QGEMM_LDS_128 ? 128 : 256;
    const int nmt = P.Mp / 128, nnt = (P.NPB + bn / 32 - 1) / (bn / 32);
    const long nlog = (long)P.ns * P.G * nnt * nmt;
    const long per = (nlog + 7) / 8;
    if (kind == QGEMM_GLOBAL_B) {
        const int nmt2 = P.Mp / 128, nnt2 = (P.NPB + 7) / 8;
        const long nlog2 = (long)P.ns * P.G * nnt2 * nmt2;
        const long per2 = (nlog2 + 7) / 8;
        const dim3 g2((unsigned)(per2 * 8));
        if (nprod == 3)
            hipLaunchKernelGGL(qgemm_bf16g_kernel<3>, g2, dim3(256), 0, st, P, Ahi, Alo, Kp, nmt2, nnt2, nlog2, per2);
        else if (nprod == 2)
            hipLaunchKernelGGL(qgemm_bf16g_kernel<2>, g2, dim3(256), 0, st, P, Ahi, Alo, Kp, nmt2, nnt2, nlog2, per2);
        else
            hipLaunchKernelGGL(qgemm_bf16g_kernel<1>, g2, dim3(256), 0, st, P, Ahi, Alo, Kp, nmt2, nnt2, nlog2, per2);
        return hipGetLastError();
    }
    const dim3 grid((unsigned)(per * 8));
#define PBS_QG(BN_, NP_) \
    hipLaunchKernelGGL((qgemm_bf16s_kernel<BN_, NP_>), grid, dim3(2 * BN_), 0, st, P, Ahi, Alo, Kp, nmt, nnt, nlog, per)
    if (bn == 128) {
        if (nprod == 3) PBS_QG(128, 3); else if (nprod == 2) PBS_QG(128, 2); else PBS_QG(128, 1);
    } else {
        if (nprod == 3) PBS_QG(256, 3); else if (nprod == 2) PBS_QG(256, 2); else PBS_QG(256, 1);
    }
#undef PBS_QG
    return hipGetLastError();
}

// FP64, and FP32 below 128 angular unknowns (up to 12 nodes per axis): v_mfma_f64_16x16x4 / v_mfma_f32_16x16x4.
// What bounded the vector kernel it replaces: its LDS staging (a barrier pair per 32 source nodes) on small
// grids, two LDS reads per multiply on large ones.  Here both operands go from global memory straight into MFMA
// registers: P2 (rows Mp apart, resident in L2) and the scan, whose row of 32 cells
// a lane reads as one pair, cell 2 c + h being column c of column tile h.  Block = up to 4 waves of 32 destination
// rows each (blockIdx.y: the next 128 rows) over NTL lateral tiles of one (half, group); loads run QS_PF 4-node steps ahead.  NTL = 1 where the
// grid has few tiles (latency), else as many as the registers hold, for each P2 load to feed more products.
// Measured, us per product, before -> after: 4 x 4 cells, 11 x 11 angles, 60 groups 21 -> 10; 24 x 24, 9 x 9, 60 73 ->
// 22 (FP64 121 -> 32); 48 x 128, 11 x 11, 60 1104 -> 321; 90 x 96, 7 x 7, 80 in FP64 845 -> 244.
// In FP64 it also beats a 128 x 128 block tile staged in LDS at every size (64 x 64 cells, 15 x 15 angles, 64 groups 1472 ->
// 1200, 44 TFLOP/s; 32 x 32, 31 x 31, 32 2688 -> 2390); in FP32 that kernel (qgemm_mfma_f32_kernel) wins from 128
// unknowns on (685 against 788, 4678 against 6297 at 64 x 64, 31 x 31, 32 groups): a matrix step there takes half the
// time and the operand loads no longer hide behind it.  The last node has a step of its own, loaded first, with a zero
// scan beside it, so that the matrix needs no rows of zeros below 128 unknowns (us with them and without: 4 x 4 cells,
// 11 x 11, 60 9.4 | 9.5; 64 x 64, 7 x 7, 100 89 | 90; FP64 32 x 32, 11 x 11, 60 94 | 98; 64 x 64, 15 x 15, 64 1315 | 1253).
constexpr int QS_PF = 4;

template <typename T, int NTL>
__global__ __launch_bounds__(256) void qgemm_direct_kernel(QParams<T> P, int nnt)
{
    typedef T T2 __attribute__((ext_vector_type(2)));
    typedef T T4 __attribute__((ext_vector_type(4)));
    const int nt = (int)(blockIdx.x % nnt);
    const long sg = blockIdx.x / nnt;
    const int g = (int)(sg % P.G), s = P.s0 + (int)(sg / P.G);
    const long off = ((long)s * P.G + g) * P.NLINE, NAPT = (long)P.NA * PBS_PT;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, c = lane & 15, kq = lane >> 4;
    const int row0 = 128 * (int)blockIdx.y + 32 * w;   // this wave's destination rows
    const T *A = P.P2p + (P.band ? (long)P.band[g] * P.Kp * P.Mp : 0L) + (long)kq * P.Mp + row0 + c;
    const T *B[NTL];
#pragma unroll
    for (int j = 0; j < NTL; ++j) B[j] = P.W + off + (long)min(nt * NTL + j, P.NPB - 1) * NAPT + 2 * c;
    const int KF = P.NA / 4;   // whole steps; one node is left (NA is odd squared)
    T4 acc[2][NTL][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < NTL; ++j) acc[i][j][0] = acc[i][j][1] = T4{0, 0, 0, 0};
    T ra[QS_PF][2], la[2];
    T2 rb[QS_PF][NTL], lb[NTL];
    // operands of step k: P2's rows of 4 source nodes (whole tiles of it: rows past the last node are dropped at the end,
    // columns past it meet a zero scan) and the scan of one of them per lane group
    auto load = [&](int k, int node, T (&a)[2], T2 (&b)[NTL]) {
        const T *p = A + (long)k * 4 * P.Mp;
        a[0] = p[0];
        a[1] = p[16];
#pragma unroll
        for (int j = 0; j < NTL; ++j) b[j] = *reinterpret_cast<const T2 *>(B[j] + (long)node * PBS_PT);
    };
    auto fetch = [&](int k, int u) {
        const int kc = min(k, KF - 1);
        load(kc, 4 * kc + kq, ra[u], rb[u]);
    };
    auto mac = [&](const T (&a)[2], const T2 (&b)[NTL]) {
#pragma unroll
        for (int j = 0; j < NTL; ++j)
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int h = 0; h < 2; ++h) acc[i][j][h] = mfma16(a[i], b[j][h], acc[i][j][h]);
    };
    auto step = [&](int k, int u) {
        const T a[2] = {ra[u][0], ra[u][1]};
        T2 b[NTL];
#pragma unroll
        for (int j = 0; j < NTL; ++j) b[j] = rb[u][j];
        fetch(k + QS_PF, u);
        mac(a, b);
    };
#pragma unroll
    for (int u = 0; u < QS_PF; ++u) fetch(u, u);
    load(KF, P.NA - 1, la, lb);
    int k0 = 0;
    for (; k0 + QS_PF <= KF; k0 += QS_PF) {
#pragma unroll
        for (int u = 0; u < QS_PF; ++u) step(k0 + u, u);
    }
#pragma unroll
    for (int u = 0; u < QS_PF - 1; ++u)
        if (k0 + u < KF) step(k0 + u, u);
    // the last node, beside three that do not exist
#pragma unroll
    for (int j = 0; j < NTL; ++j) lb[j] = kq == 0 ? lb[j] : T2{0, 0};
    mac(la, lb);
#pragma unroll
    for (int j = 0; j < NTL; ++j) {
        const int pb = nt * NTL + j;
        if (pb >= P.NPB) continue;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                // result rows of a lane: FP32 4 (lane / 16) + q, FP64 lane / 16 + 4 q
                const int row = row0 + 16 * i + (sizeof(T) == 4 ? 4 * kq + q : kq + 4 * q);
                if (row < P.NA)
                    *reinterpret_cast<T2 *>(P.Q + off + pb * NAPT + (long)row * PBS_PT + 2 * c) =
                        T2{acc[i][j][0][q], acc[i][j][1][q]};
            }
    }
}

// Up to 8192 (half, group, tile) items a tile per block; more tiles per block above, where it pays: 48 x 60 cells,
// 11 x 11 angles, 60 groups, FP64 (10800 items) 254 us against 271, 64 x 64, 9 x 9, 100 (25600) 189 against 200; but
// 32 x 32, 11 x 11, 60 (3840) 58 against 55 and 4 x 4 (120) 15.5 against 9.7.
constexpr long QS_WIDE_ITEMS = 8192;
template <typename T>
static hipError_t launch_qgemm_direct(const QParams<T> &P, hipStream_t st)
{
    constexpr int WIDE = sizeof(T) == 4 ? 4 : 2;
    const dim3 block(P.NA > 96 ? 256 : 64 * ((P.NA + 31) / 32));
    const unsigned nmt = (unsigned)((P.NA + 127) / 128);
    const long items = (long)P.ns * P.G * P.NPB;
    if (items > QS_WIDE_ITEMS) {
        const int nnt = (P.NPB + WIDE - 1) / WIDE;
        hipLaunchKernelGGL((qgemm_direct_kernel<T, WIDE>), dim3((unsigned)((long)P.ns * P.G * nnt), nmt), block, 0, st, P, nnt);
    } else {
        hipLaunchKernelGGL((qgemm_direct_kernel<T, 1>), dim3((unsigned)items, nmt), block, 0, st, P, P.NPB);
    }
    return hipGetLastError();
}

template <typename T>
hipError_t launch_qgemm(const QParams<T> &P, hipStream_t st)
{
    if (P.P2p == nullptr) return hipErrorInvalidValue;
    if constexpr (sizeof(T) == 4) {
        if (P.NA >= 128) {
            const int nmt = P.Mp / 128, nnt = (P.NPB + 3) / 4;
            const long nlog = (long)P.ns * P.G * nnt * nmt;
            const long per = (nlog + 7) / 8;
            hipLaunchKernelGGL(qgemm_mfma_f32_kernel, dim3((unsigned)(per * 8)), dim3(256), 0, st, P, nmt, nnt, nlog,
                               per);
            return hipGetLastError();
        }
    }
    return launch_qgemm_direct(P, st);
}

// ----------------------------------------------------------------------------------- misc
template <typename T>
__global__ void fill_kernel(T *p, T v, long n)
{
    for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < n; i += (long)gridDim.x * 256) p[i] = v;
}

template <typename T>
hipError_t launch_fill(T *p, T v, long n, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    long nb = (n + 255) / 256;
    if (nb > 65536) nb = 65536;
    hipLaunchKernelGGL((fill_kernel<T>), dim3((unsigned)nb), dim3(256), 0, st, p, v, n);
    return hipGetLastError();
}

template <typename T>
__global__ void combine_kernel(T *y, const T *x, T a, T b, long n)
{
    for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < n; i += (long)gridDim.x * 256) y[i] = a * y[i] + b * x[i];
}

template <typename T>
hipError_t launch_combine(T *y, const T *x, T a, T b, long n, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    long nb = (n + 255) / 256;
    if (nb > 65536) nb = 65536;
    hipLaunchKernelGGL((combine_kernel<T>), dim3((unsigned)nb), dim3(256), 0, st, y, x, a, b, n);
    return hipGetLastError();
}
template hipError_t launch_combine<float>(float *, const float *, float, float, long, hipStream_t);
template hipError_t launch_combine<double>(double *, const double *, double, double, long, hipStream_t);

// edep[pq] += sum over generations and angles of dep[k][line(pq, a)], fixed order: one block of four waves per
// lateral tile; lane (pt, h) of wave w sums the slots a = 2 w + h, + 8, ... of every generation in turn, then the
// eight partials of a cell are added in the order of (w, h).  What bounds it is the latency of its loads (a
// few hundred KB): four waves and eight loads in flight per lane took a launch at 4 x 4 cells, 11 x 11
// angles, two generations from 17 to 9 us, one at 45 x 70, 19 x 19, three from 35 to 13.  Sixteen-wave blocks lose that
// again where the reduction runs beside the transport and angular passes (they wait for a whole CU to drain); one wave
// that takes all four shares is quicker there by itself (114 -> 45 us) but no batch is (48 to 128 beams: the same).
__device__ __forceinline__ void dose_reduce_body(double *edep, const double *dep, int ngen, int NA, int nslot,
                                                 long NLINE, int NP, int pb)
{
    __shared__ double part[4][32];
    const int tid = threadIdx.x, pt = tid & 31, h = (tid >> 5) & 1, w = tid >> 6;
    const long base = (long)pb * NA * PBS_PT + pt;
    const bool adds = w < 4;   // further waves of a larger block only meet the barriers
    double s = 0.0;
    if (adds) {
        for (int k = 0; k < ngen; ++k) {
            const double *d = dep + (long)k * NLINE + base;
#pragma unroll 8
            for (int a = 2 * w + h; a < nslot; a += 8) s += d[(long)a * PBS_PT];
        }
    }
    s += __shfl_xor(s, 32);
    __syncthreads();   // a second reduction of the same block: the first one's partials have been read
    if (adds && h == 0) part[w][pt] = s;
    __syncthreads();
    const int pq = pb * PBS_PT + pt;
    if (tid < 32 && pq < NP) edep[pq] += ((part[0][pt] + part[1][pt]) + part[2][pt]) + part[3][pt];
}

// blockIdx.y picks the reduction: rows that differ, so that the blocks of one launch never meet
__global__ __launch_bounds__(256) void dose_reduce_kernel(DoseJobs J, int NA, long NLINE, int NP)
{
    const int j = blockIdx.y;
    dose_reduce_body(J.row[j], J.dep[j], J.ngen[j], NA, J.nslot, NLINE, NP, blockIdx.x);
}

hipError_t launch_dose_reduce(const DoseJobs &J, int NA, long NLINE, int NP, hipStream_t st)
{
    if (J.n <= 0) return hipSuccess;
    for (int i = 0; i < J.n; ++i)
        for (int j = i + 1; j < J.n; ++j)
            if (J.row[i] == J.row[j]) {
                // one row twice (both halves of an extrapolated step's inner pair): one launch after the other
                DoseJobs A = J, B = J;
                A.n = j;
                B.n = J.n - j;
                for (int q = 0; q < B.n; ++q) B.row[q] = J.row[j + q], B.dep[q] = J.dep[j + q], B.ngen[q] = J.ngen[j + q];
                const hipError_t e = launch_dose_reduce(A, NA, NLINE, NP, st);
                return e != hipSuccess ? e : launch_dose_reduce(B, NA, NLINE, NP, st);
            }
    const int npb = (NP + PBS_PT - 1) / PBS_PT;
    hipLaunchKernelGGL(dose_reduce_kernel, dim3(npb, J.n), dim3(256), 0, st, J, NA, NLINE, NP);
    return hipGetLastError();
}

__global__ void dose_finalize_kernel(double *out, const double *edep, const double *rho, double vol, long n)
{
    const long i = (long)blockIdx.x * 256 + threadIdx.x;
    if (i < n) out[i] = edep[i] / (rho[i] * vol);
}

hipError_t launch_dose_finalize(double *out, const double *edep, const double *rho, double vol, long n,
                                hipStream_t st)
{
    hipLaunchKernelGGL(dose_finalize_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, out, edep, rho,
                       vol, n);
    return hipGetLastError();
}

// initial fluence on the theta = 0 node: psi[g][l][pb][center][pt] = E_l[g] * lat[pq]
template <typename T>
__global__ void initial_kernel(T *psi0, const double *E1, const double *E2, const double *lat, long center_a,
                               int G, int NA, int NPB, int NP)
{
    const long i = (long)blockIdx.x * 256 + threadIdx.x;
    if (i >= (long)G * NP) return;
    const int g = (int)(i / NP), pq = (int)(i % NP);
    const long NLINE = (long)NPB * NA * PBS_PT;
    const long line = ((long)(pq / PBS_PT) * NA + center_a) * PBS_PT + (pq % PBS_PT);
    psi0[(2L * g) * NLINE + line] = (T)(E1[g] * lat[pq]);
    psi0[(2L * g + 1) * NLINE + line] = (T)(E2[g] * lat[pq]);
}

template <typename T>
hipError_t launch_initial(T *psi0, const double *E1, const double *E2, const double *lat, long center_a, int G,
                          int NA, int NPB, int NP, hipStream_t st)
{
    const long n = (long)G * NP;
    hipLaunchKernelGGL((initial_kernel<T>), dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, psi0, E1, E2, lat,
                       center_a, G, NA, NPB, NP);
    return hipGetLastError();
}

// ------------------------------------------------------------------------- batched wrappers
// Every launch covers all beams of a resident wave (grid y or z = beam); each block reads its beam's
// descriptor, derives the sub-step of step s for that beam (open at s = 0, fused pair for
// 0 < s < nz, close at s = nz) and exits when the beam has nothing to do.
__device__ __forceinline__ int beam_mode(int s, int nz)
{
    if (s > nz) return 0;
    if (s == 0) return MODE_OPEN;
    if (s == nz) return MODE_CLOSE;
    return MODE_PAIR;
}

template <bool LO, int RING, bool HASQ>
__global__ __launch_bounds__(256) void epass_batched_kernel(
    const BeamDev *__restrict__ beams, BatchShape Sh, int k, int s)
{
    const BeamDev &B = beams[blockIdx.y];
    const int mode = beam_mode(s, B.nz);
    if (mode == 0) return;
    EParams<float> P;
    const int G = B.G;
    P.psi = B.psi + (long)k * G * 2 * Sh.NLINE;
    P.Q = k > 0 ? B.Q : nullptr;
    P.Qb = (k > 0 && Sh.nprod == 1) ? reinterpret_cast<const unsigned short *>(B.Q) : nullptr;
    P.W = nullptr;
    const bool w = k + 1 < Sh.ngen;
    P.Wh = w ? B.Wh : nullptr;
    P.Wl = w ? B.Wl : nullptr;
    P.NOCT = Sh.NOCT;
    P.rho_c = (mode & MODE_CLOSE) ? B.rho + (long)(s - 1) * Sh.NPB * PBS_PT : nullptr;
    P.rho_o = (mode & MODE_OPEN) ? B.rho + (long)s * Sh.NPB * PBS_PT : nullptr;
    P.dep_c = B.dep + (long)k * Sh.NLINE;
    P.dep_o = B.dep + ((long)Sh.ngen + k) * Sh.NLINE;
    P.Sm = B.tabf;
    P.Sp = B.tabf + G;
    P.kap = B.tabf + 2 * G;
    P.wc = B.tabf + 3 * G;
    P.wdec = B.tabf + 4 * G;
    P.invdE = B.tabf + 5 * G;
    P.dA = B.tabd;
    P.dB = B.tabd + G;
    P.dInj = B.tabd + 2 * G;
    P.dBot = B.dBot;
    P.scale = Sh.scale;
    P.h = 0.5f * B.dz;
    P.G = G;
    P.NLINE = Sh.NLINE;
    P.NAPT = (long)Sh.NA * PBS_PT;
    const long gid = (long)blockIdx.x * 256 + threadIdx.x;
    if (mode == MODE_PAIR)
        epass8_body<MODE_PAIR, false, LO, false, RING, HASQ>(P, gid);
    else if (mode == MODE_OPEN)
        epass8_body<MODE_OPEN, false, LO, false, RING, HASQ>(P, gid);
    else
        epass8_body<MODE_CLOSE, false, LO, false, RING, HASQ>(P, gid);
}

// BN = 128 / 256: LDS-staged kernel with BN-column blocks; BN = 0: global-B kernel (256 columns)
template <int BN, int NPROD>
__global__ __launch_bounds__(BN == 0 ? 256 : 2 * BN)
__attribute__((amdgpu_waves_per_eu(BN == 0 && NPROD == 1 ? QG_WPE : 1))) void qgemm_batched_kernel(
    const BeamDev *__restrict__ beams, BatchShape Sh, int s)
{
    const BeamDev &B = beams[blockIdx.y];
    const int mode = beam_mode(s, B.nz);
    if (mode == 0) return;
    QParams<float> P;
    P.W = nullptr;
    P.Q = B.Q;
    P.Qb = NPROD == 1 ? reinterpret_cast<unsigned short *>(B.Q) : nullptr;   // single product: BF16 source
    P.P2p = nullptr;
    P.Kp = Sh.Kpb;
    P.Mp = Sh.Mp;
    P.Bh = B.Wh;
    P.Bl = B.Wl;
    P.NOCT = Sh.NOCT;
    P.NA = Sh.NA;
    P.NPB = Sh.NPB;
    P.G = B.G;
    P.s0 = (mode == MODE_OPEN) ? 1 : 0;
    P.ns = (mode == MODE_PAIR) ? 2 : 1;
    P.NLINE = Sh.NLINE;
    constexpr int BW = BN == 0 ? 256 : BN;
    const int nmt = Sh.Mp / 128, nnt = (Sh.NPB + BW / 32 - 1) / (BW / 32);
    const long nlog = (long)P.ns * P.G * nnt * nmt;
    const long per = (nlog + 7) / 8;
    if ((long)blockIdx.x >= per * 8) return;
    if constexpr (BN == 0)
        qgemm_bf16g_body<NPROD, QG_PFD_BATCH>(P, Sh.Ahi, Sh.Alo, Sh.Kpb, nmt, nnt, nlog, per, blockIdx.x);
    else
        qgemm_bf16s_body<BN, NPROD>(P, Sh.Ahi, Sh.Alo, Sh.Kpb, nmt, nnt, nlog, per, blockIdx.x);
}

// the transport record of one beam of the batch (generation k, or all for k < 0)
__device__ __forceinline__ TParams<float> batch_tparams(const BeamDev &B, const BatchShape &Sh, int k)
{
    TParams<float> P;
    P.psi = k < 0 ? B.psi : B.psi + (long)k * B.G * 2 * Sh.NLINE;
    P.theta = Sh.theta;
    P.h_half_over_dx = B.thx;
    P.h_half_over_dy = B.thy;
    P.nx = Sh.nx;
    P.ny = Sh.ny;
    P.m = Sh.m;
    P.NA = Sh.NA;
    P.NLINE = Sh.NLINE;
    P.nplanes = (long)(k < 0 ? Sh.ngen : 1) * B.G * 2 * Sh.NA;
    return P;
}

template <int V, bool NT>
__global__ __launch_bounds__(256) void tpass_batched_packed_kernel(const BeamDev *__restrict__ beams, BatchShape Sh,
                                                                    int s, int k)
{
    const BeamDev &B = beams[blockIdx.y];
    if (s >= B.nz) return;
    tpass_packed_body<float, V, NT>(batch_tparams(B, Sh, k), blockIdx.x * 4 + (threadIdx.x >> 6));
}

__global__ __launch_bounds__(256) void tpass_batched_far_kernel(const BeamDev *__restrict__ beams, BatchShape Sh, int s, int k)
{
    const BeamDev &B = beams[blockIdx.y];
    if (s >= B.nz) return;
    tpass_far_body(batch_tparams(B, Sh, k), blockIdx.x * 4 + (threadIdx.x >> 6));
}

template <int NSEG, int WPB>
__global__ __launch_bounds__(64 * WPB) void tpass_batched_kernel(const BeamDev *__restrict__ beams, BatchShape Sh,
                                                                 int s, int k)
{
    const BeamDev &B = beams[blockIdx.y];
    if (s >= B.nz) return;
    const TParams<float> P = batch_tparams(B, Sh, k);
    tpass_body<float, NSEG>(P, (long)blockIdx.x * WPB + (threadIdx.x >> 6));
}

template <int NY, int WPB>
__global__ __launch_bounds__(64 * WPB) void tpass_batched_affine_kernel(const BeamDev *__restrict__ beams,
                                                                        BatchShape Sh, int s, int k)
{
    const BeamDev &B = beams[blockIdx.y];
    if (s >= B.nz) return;
    const TParams<float> P = batch_tparams(B, Sh, k);
    tpass_affine_body<NY>(P, (long)blockIdx.x * WPB + (threadIdx.x >> 6));
}

template <int NY, int WPB>
__global__ __launch_bounds__(64 * WPB) void tpass_batched_wide_kernel(const BeamDev *__restrict__ beams,
                                                                      BatchShape Sh, int s, int k)
{
    const BeamDev &B = beams[blockIdx.y];
    if (s >= B.nz) return;
    const TParams<float> P = batch_tparams(B, Sh, k);
    tpass_wide_body<NY>(P, (long)blockIdx.x * WPB + (threadIdx.x >> 6));
}

template <int WPB>
__global__ __launch_bounds__(64 * WPB) void tpass_batched_pair_kernel(const BeamDev *__restrict__ beams,
                                                                      BatchShape Sh, int s, int k)
{
    const BeamDev &B = beams[blockIdx.y];
    if (s >= B.nz) return;
    const TParams<float> P = batch_tparams(B, Sh, k);
    tpass_pair_body(P, (long)blockIdx.x * WPB + (threadIdx.x >> 6));
}

// angular record of one beam of the batch at step s (generation k, or all for k < 0)
__device__ __forceinline__ AParams<float> batch_aparams(const BeamDev &B, const BatchShape &Sh, int s, int k)
{
    AParams<float> P;
    P.psi = k < 0 ? B.psi : B.psi + (long)k * B.G * 2 * Sh.NLINE;
    P.rho = B.rho + (long)s * Sh.NPB * PBS_PT;
    P.sig = B.tabf + 6 * B.G;
    P.S = Sh.S;
    P.lam = Sh.lam;
    P.h = B.dz;
    P.G = B.G;
    P.NA = Sh.NA;
    P.NPB = Sh.NPB;
    P.NLINE = Sh.NLINE;
    return P;
}

// Held to eight waves per SIMD: the registers then do without the accumulation file, and the pass, which shares the chip
// with the energy passes, leaves them more of it (20 beams of 16 x 32 cells, 15 x 15 angles 66.5 -> 66.0 ms, 24 of
// 32 x 32 with three generations 273.2 -> 271.9).
template <int N>
__global__ __launch_bounds__((AngMfma<float, N>::NT)) __attribute__((amdgpu_waves_per_eu(8)))
void apass_batched_kernel(const BeamDev *__restrict__ beams, BatchShape Sh, int s, int k)
{
    const BeamDev &B = beams[blockIdx.z];
    if (s >= B.nz || blockIdx.y >= (unsigned)((k < 0 ? Sh.ngen : 1) * B.G * 2)) return;
    apass_mfma_block<float, N>(batch_aparams(B, Sh, s, k), Sh.K, blockIdx.x, blockIdx.y, Sh.NPB);
}

// the 32-node FP32 pass, beam = blockIdx.z
__global__ __launch_bounds__(APASS32_NT) __attribute__((amdgpu_waves_per_eu(8)))
void apass_mfma32_batched_kernel(const BeamDev *__restrict__ beams, BatchShape Sh, int s, int k)
{
    const BeamDev &B = beams[blockIdx.z];
    if (s >= B.nz || blockIdx.y >= (unsigned)((k < 0 ? Sh.ngen : 1) * B.G * 2)) return;
    int pb, half;
    apass_half_tile(blockIdx.x, Sh.NPB, pb, half);
    if (pb >= Sh.NPB) return;
    apass_mfma32_body(batch_aparams(B, Sh, s, k), Sh.K, blockIdx.y, pb, half);
}

__global__ __launch_bounds__(256) void dose_batched_kernel(const BeamDev *__restrict__ beams, BatchShape Sh, int s)
{
    const BeamDev &B = beams[blockIdx.y];
    const int mode = beam_mode(s, B.nz);
    const int NP = Sh.nx * Sh.ny;
    if (mode & MODE_CLOSE)
        dose_reduce_body(B.edep + (long)(s - 1) * NP, B.dep, Sh.ngen, Sh.NA, epass8_slots(Sh.NOCT), Sh.NLINE, NP,
                         blockIdx.x);
    if (mode & MODE_OPEN)
        dose_reduce_body(B.edep + (long)s * NP, B.dep + (long)Sh.ngen * Sh.NLINE, Sh.ngen, Sh.NA,
                         epass8_slots(Sh.NOCT), Sh.NLINE, NP, blockIdx.x);
}

// the sizes that the rules of the packed sweeps look at
static TParams<float> batch_tsize(const BatchShape &Sh, long planes)
{
    TParams<float> P;
    P.ny = Sh.ny;
    P.NLINE = Sh.NLINE;
    P.nplanes = planes;
    return P;
}

// the sweeps that take BatchTuning::tpass_wpb waves per block: the aligned widths, and the shuffle sweep
static bool batch_tpass_aligned(const BatchShape &Sh)
{
    return Sh.nx % TPASS_PF == 0 && (Sh.ny == 32 || Sh.ny == 64 || Sh.ny == 96 || Sh.ny == 128);
}
bool batch_tpass_tunes(const BatchShape &Sh, int maxG)
{
    const TParams<float> size = batch_tsize(Sh, (long)Sh.ngen * maxG * 2 * Sh.NA);
    return batch_tpass_aligned(Sh) || (!tpass_packed_fits(size) && !tpass_far_fits(size));
}

hipError_t launch_batch_step(const BeamDev *beams, int nbeam, const BatchShape &Sh, int s, int maxG,
                             const BatchTuning &tu, hipStream_t st, const BatchSide *sd)
{
    // T(dz/2) A(dz) T(dz/2) of generation k (all generations for k < 0) on stream q
    auto tat = [&](int k, hipStream_t q) {
        const long planes = (long)(k < 0 ? Sh.ngen : 1) * maxG * 2 * Sh.NA;
        const int nstack = (k < 0 ? Sh.ngen : 1) * maxG * 2;
        const int nseg = (Sh.ny + 63) / 64;
        auto tpass = [&]() {
            const int w = tu.tpass_wpb;
            const unsigned nb = (unsigned)((planes + w - 1) / w);
#define PBS_TB(NS, W) hipLaunchKernelGGL((tpass_batched_kernel<NS, W>), dim3(nb, nbeam), dim3(64 * W), 0, q, beams, Sh, s, k)
#define PBS_TW(NS) do { if (w == 1) PBS_TB(NS, 1); else if (w == 2) PBS_TB(NS, 2); else PBS_TB(NS, 4); } while (0)
#define PBS_TA(NY, W) hipLaunchKernelGGL((tpass_batched_affine_kernel<NY, W>), dim3(nb, nbeam), dim3(64 * W), 0, q, beams, Sh, s, k)
#define PBS_TAW(NY) do { if (w == 1) PBS_TA(NY, 1); else if (w == 2) PBS_TA(NY, 2); else PBS_TA(NY, 4); } while (0)
#define PBS_TD(NY, W) hipLaunchKernelGGL((tpass_batched_wide_kernel<NY, W>), dim3(nb, nbeam), dim3(64 * W), 0, q, beams, Sh, s, k)
#define PBS_TWW(NY) do { if (w == 1) PBS_TD(NY, 1); else if (w == 2) PBS_TD(NY, 2); else PBS_TD(NY, 4); } while (0)
            if (Sh.nx % TPASS_PF == 0 && Sh.ny == 64) {
                PBS_TAW(64);
                return;
            }
            if (Sh.nx % TPASS_PF == 0 && Sh.ny == 32) {
                // two planes per wave
                const unsigned nbp = (unsigned)(((planes + 1) / 2 + w - 1) / w);
                if (w == 1)
                    hipLaunchKernelGGL((tpass_batched_pair_kernel<1>), dim3(nbp, nbeam), dim3(64), 0, q, beams, Sh, s, k);
                else if (w == 2)
                    hipLaunchKernelGGL((tpass_batched_pair_kernel<2>), dim3(nbp, nbeam), dim3(128), 0, q, beams, Sh, s, k);
                else
                    hipLaunchKernelGGL((tpass_batched_pair_kernel<4>), dim3(nbp, nbeam), dim3(256), 0, q, beams, Sh, s, k);
                return;
            }
            if (Sh.nx % TPASS_PF == 0 && Sh.ny == 96) {
                PBS_TWW(96);
                return;
            }
            if (Sh.nx % TPASS_PF == 0 && Sh.ny == 128) {
                PBS_TWW(128);
                return;
            }
            const TParams<float> size = batch_tsize(Sh, planes);   // of the largest beam
            if (tpass_packed_fits(size)) {
                const int np = tpass_packed_planes(Sh.ny);
                const dim3 g((unsigned)(((planes + np - 1) / np + 3) / 4), nbeam);
                tpass_packed_select(Sh.ny, [&](auto v, auto nt) {
                    hipLaunchKernelGGL((tpass_batched_packed_kernel<decltype(v)::value, decltype(nt)::value>), g,
                                       dim3(256), 0, q, beams, Sh, s, k);
                });
                return;
            }
            if (tpass_far_fits(size)) {
                hipLaunchKernelGGL(tpass_batched_far_kernel, dim3((unsigned)((planes + 3) / 4), nbeam), dim3(256), 0, q,
                                   beams, Sh, s, k);
                return;
            }
            switch (nseg) {
            case 1: PBS_TW(1); break;
            case 2: PBS_TW(2); break;
            case 3: PBS_TW(3); break;
            default: PBS_TW(4); break;
            }
#undef PBS_TW
#undef PBS_TB
#undef PBS_TAW
#undef PBS_TA
#undef PBS_TWW
#undef PBS_TD
        };
        tpass();
        const dim3 grid((unsigned)apass_half_blocks(Sh.NPB), (unsigned)nstack, nbeam);
#define PBS_AB(N) \
    hipLaunchKernelGGL((apass_batched_kernel<N>), grid, dim3(AngMfma<float, N>::NT), 0, q, beams, Sh, s, k)
        switch (Sh.nth) {
        case 16: PBS_AB(16); break;
        case 20: PBS_AB(20); break;
        case 24: PBS_AB(24); break;
        case 32:
            hipLaunchKernelGGL(apass_mfma32_batched_kernel, grid, dim3(APASS32_NT), 0, q, beams, Sh, s, k);
            break;
        default: return hipErrorInvalidValue;
        }
#undef PBS_AB
        tpass();
        return hipGetLastError();
    };
    const bool march = s < tu.max_nz;
    for (int k = 0; k < Sh.ngen; ++k) {
        if (sd && sd->pend[k]) {
            // this generation's T A T of the previous step
            if (hipStreamWaitEvent(st, sd->ev_tat[k], 0) != hipSuccess) return hipErrorUnknown;
            sd->pend[k] = 0;
        }
        const unsigned nbe = (unsigned)(((long)Sh.NPB * Sh.NOCT * (8 / PBS_EPASS_LPT) * PBS_PT + 255) / 256);
        const bool ring = 4L * nbe * nbeam <= EP8_RING_WAVES && Sh.nprod == 1;
        if (Sh.nprod == 3)
            hipLaunchKernelGGL((epass_batched_kernel<true, 0, false>), dim3(nbe, nbeam), dim3(256), 0, st, beams, Sh, k, s);
        else if (!ring)
            hipLaunchKernelGGL((epass_batched_kernel<false, 0, false>), dim3(nbe, nbeam), dim3(256), 0, st, beams, Sh, k, s);
        else if (k > 0)
            hipLaunchKernelGGL((epass_batched_kernel<false, EP8_RING, true>), dim3(nbe, nbeam), dim3(256), 0, st, beams, Sh, k, s);
        else
            hipLaunchKernelGGL((epass_batched_kernel<false, EP8_RING, false>), dim3(nbe, nbeam), dim3(256), 0, st, beams, Sh, k, s);
        if (sd && march) {
            // generation k's T A T beside the source product and the later generations' energy passes
            hipError_t e = hipEventRecord(sd->ev_e[k], st);
            if (e == hipSuccess) e = hipStreamWaitEvent(sd->side, sd->ev_e[k], 0);
            if (e == hipSuccess) e = tat(k, sd->side);
            if (e == hipSuccess) e = hipEventRecord(sd->ev_tat[k], sd->side);
            if (e != hipSuccess) return e;
            sd->pend[k] = 1;
        }
        if (k + 1 < Sh.ngen) {
            const int kind = tu.gemm_kind == QGEMM_GLOBAL_B && !qgemm_global_b_fits(Sh.NPB, Sh.NOCT) ? QGEMM_LDS_256
                                                                                                  : tu.gemm_kind;
            const int bn = kind == QGEMM_LDS_128 ? 128 : 256;
            const int nmt = Sh.Mp / 128, nnt = (Sh.NPB + bn / 32 - 1) / (bn / 32);
            const long per = ((long)2 * maxG * nnt * nmt + 7) / 8;
            const dim3 grid((unsigned)(per * 8), nbeam);
#define PBS_QB(BN_, NP_) hipLaunchKernelGGL((qgemm_batched_kernel<BN_, NP_>), grid, dim3(2 * BN_), 0, st, beams, Sh, s)
#define PBS_QG(NP_) hipLaunchKernelGGL((qgemm_batched_kernel<0, NP_>), grid, dim3(256), 0, st, beams, Sh, s)
            if (kind == QGEMM_GLOBAL_B) {
                if (Sh.nprod == 3) PBS_QG(3); else if (Sh.nprod == 2) PBS_QG(2); else PBS_QG(1);
            } else if (bn == 128) {
                if (Sh.nprod == 3) PBS_QB(128, 3); else if (Sh.nprod == 2) PBS_QB(128, 2); else PBS_QB(128, 1);
            } else {
                if (Sh.nprod == 3) PBS_QB(256, 3); else if (Sh.nprod == 2) PBS_QB(256, 2); else PBS_QB(256, 1);
            }
#undef PBS_QB
#undef PBS_QG
        }
    }
    hipLaunchKernelGGL(dose_batched_kernel, dim3(Sh.NPB, nbeam), dim3(256), 0, st, beams, Sh, s);
    if (!sd && march) {
        const hipError_t e = tat(-1, st);
        if (e != hipSuccess) return e;
    }
    return hipGetLastError();
}

#define PBS_INSTANTIATE(T)                                                                                    \
    template hipError_t launch_epass<T>(const EParams<T> &, int, hipStream_t);                                \
    template hipError_t launch_tpass<T>(const TParams<T> &, hipStream_t);                                     \
    template hipError_t launch_apass<T>(const AParams<T> &, const T *, int, long, hipStream_t);                        \
    template bool tat_fits<T>(int, int, long, long, int, bool);                                                     \
    template hipError_t launch_tat<T>(const TParams<T> &, const AParams<T> &, int, long, const DoseJobs &, hipStream_t); \
    template hipError_t launch_qgemm<T>(const QParams<T> &, hipStream_t);                                     \
    template hipError_t launch_fill<T>(T *, T, long, hipStream_t);                                            \
    template hipError_t launch_initial<T>(T *, const double *, const double *, const double *, long, int, int, \
                                          int, int, hipStream_t);
PBS_INSTANTIATE(float)
PBS_INSTANTIATE(double)

}  // namespace pbs
