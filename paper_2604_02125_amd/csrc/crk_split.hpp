// crk_split.hpp -- local stages of the GLM-MHD step with two lanes per node.
//
// The one-lane form (local_tile) keeps nine conserved variables, up to four
// pending stage sums, the update, two face shares and two nodes' fields per
// lane: 392 registers in FP64 at degree 4, one wavefront per SIMD, and every
// dependency and LDS wait exposed.  Here a node has one lane per direction,
// in different wavefronts: the lanes of the first half of the workgroup
// evaluate the x pairs, those of the second half the y pairs.
//   - Pairs, the diagonal and non-conservative terms, the face terms and the
//     element's share P_d of its direction's faces belong to the direction's
//     lane.
//   - u^n, the pending stage sums and the summed residual R are split by
//     variable: the x lane owns 0..4 (density, momentum, energy), the y lane
//     5..8 (B, psi).  Each lane hands the other the part of its direction's
//     residual that the other owns, and reads the mirrored fluxes of both
//     directions for its own variables (the same number of LDS reads as both
//     directions for all variables in half the lanes).
//   - The stage state is put together from the two halves through LDS.
// That is at most 256 registers, two wavefronts per SIMD, for three workgroup
// barriers per stage.  Orszag-Tang 192^2, degree 4, FP64, when written: local
// phase 345 -> 300 us (372 -> 346 us per step against the one-lane kernel
// with the same pair flux and logarithm), bound by vector issue (62 % busy)
// and LDS (53 %) together, the rest waiting at barriers.  With the series for
// the logarithmic means the phase took 262 us, the step 301; with far means in
// one uniform branch 253 and 292.
#pragma once
#include "crk_kernels.hpp"

namespace crk {

template <typename real, int N, int FLUX>
struct SplitShape {
    using Phys = MhdP<real, FLUX>;
    static constexpr int n1 = N + 1, NP = n1 * n1;
    static constexpr int HALF = tile_block<NP>();          // lanes per direction
    static constexpr int EPB = HALF / NP;
    static constexpr int M = Phys::M, NF = Phys::NF, NL = Phys::NL;
    static constexpr int OWN0 = 5;                          // variables of the x lane
    static constexpr bool SYM = N >= 2;
    static constexpr int NPRIM = SYM ? (n1 - 1) / 2 : 0;
    static constexpr int KSELF = (SYM && n1 % 2 == 0) ? n1 / 2 : 0;
    static constexpr int MX = Phys::MX;                     // variables with pair fluxes
    __device__ __forceinline__ static constexpr int xslot(int dd, int k, int v)
    {
        return (dd * NPRIM + (k - 1)) * MX + Phys::xidx(dd, v);
    }
    static constexpr int X = 2 * NPRIM * MX;                // mirrored fluxes of both directions
    // fields, fluxes, handed-over values; u^n and the coefficients 2 D/dx
    // (in LDS instead of 34 registers)
    static constexpr int slots = NL + X + M + M + 1;
    static_assert(Phys::LEAN, "written for the reduced exchange");
    static_assert(2 * n1 * n1 <= HALF, "the coefficient table fits one slot");
};

// The lane of direction ROLE of a node: everything between the loads and the
// stores of one tile.
template <typename real, int N, int FLUX, int S, int TAB, bool NCS, int ROLE>
__device__ __forceinline__ void split_lane(const Tables &t, const StepPtrs &a, long e0, real *smem, int lane)
{
    using Sh = SplitShape<real, N, FLUX>;
    using Phys = typename Sh::Phys;
    constexpr int n1 = Sh::n1, NP = Sh::NP, H = Sh::HALF, M = Sh::M, NF = Sh::NF;
    constexpr int NPRIM = Sh::NPRIM, KSELF = Sh::KSELF;
    constexpr bool SYM = Sh::SYM;
    constexpr int d = ROLE;
    constexpr int V0 = ROLE == 0 ? 0 : Sh::OWN0, V1 = ROLE == 0 ? Sh::OWN0 : M, NV = V1 - V0;   // owned variables
    using FD = FaceData<EQ_MHD, M>;
    real *lf = smem;                  // [NL][H] node fields
    real *lx = lf + Sh::NL * H;           // [2][NPRIM][M][H] fluxes whose mirror a line neighbour takes
    // [M][H] what a node's lanes hand each other: variable v of the residual
    // from the lane that does not own v, then of the stage state from the one
    // that does (each reads before it writes)
    real *lh = lx + Sh::X * H;
    real *ln = lh + M * H;            // [M][H] u^n
    real *lt = ln + M * H;            // [2][n1][n1] 2 D_{r,(r+k) mod n1} / dx_d

    int le = lane / NP;
    const int node = lane - le * NP;
    const long e = e0 + le;
    const bool valid = le < Sh::EPB && e < t.nelem;
    if (le >= Sh::EPB) le = 0;        // spare lanes read element 0's fields
    const long es = valid ? e : 0;
    const int base = le * NP;
    const int pd[2] = {node % n1, node / n1};
    const int r = pd[d];
    const long E = t.nelem;
    const Ctx<real> ctx = make_ctx<real>(t, a.dt);
    const real rdt = real(a.dt[0]);

    const real *uin = (const real *)a.u_in;
    real us[M];
#pragma unroll
    for (int v = 0; v < M; ++v) us[v] = uin[((long)v * E + es) * NP + node];
#pragma unroll
    for (int v = V0; v < V1; ++v) ln[v * H + lane] = us[v];
    auto un = [&](int o) -> real { return ln[(V0 + o) * H + lane]; };

    // 2 D/dx of the own direction's rotations (k = 0: the diagonal); half of
    // it is the coefficient of the non-conservative term; of the other
    // direction only the mirrored rotations n1 - k are used.  (Each
    // direction's lanes write their own half of the table.)
    if (lane < n1 * n1) lt[d * n1 * n1 + lane] = Tab<real>::dk(t, d, lane / n1, lane % n1);
    auto Dk = [&](int k) -> real { return lt[(d * n1 + r) * n1 + k]; };
    auto Do = [&](int k) -> real { return lt[((1 - d) * n1 + pd[1 - d]) * n1 + n1 - k]; };

    // Rusanov speed of the face through this node in the own direction
    const bool onface = r == 0 || r == N;
    const int side = r == N ? 1 : 0;
    const int kk = pd[1 - d];
    const int face = 2 * d + side;
    real lam;
    {
        const Nbrs nb = neighbours<2, false>(t, es);
        const real *ts = (const real *)a.traces;
        const real so = ts[((long)(face * FD::NCT + FD::SPEED) * E + es) * n1 + kk];
        const real sn = ts[((long)((2 * d + 1 - side) * FD::NCT + FD::SPEED) * E + (side ? nb.n[d][1] : nb.n[d][0])) * n1 + kk];
        lam = dmax(dmax(so, sn), ctx.ch);
    }
    const real invw = Tab<real>::invw(t, d, r);
    const real sw = onface ? (side ? -invw : invw) : real(0);
    const real hl = onface ? (side ? real(0.5) : real(-0.5)) * lam : real(0);
    const real cF = sw * real(-0.5);       // s/(w dx) (1/2 - 1)
    const real cU = sw * hl;

    // Wf: face terms of the own direction, all variables; W: the owned
    // variables' sum_i b_i R^(i); P: the element's share of the own faces
    real Z[S][NV], W[NV], Wf[M], P[M], UB = real(0), Upsi = real(0);
#pragma unroll
    for (int v = 0; v < M; ++v) Wf[v] = P[v] = real(0);
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        W[v] = real(0);
#pragma unroll
        for (int k = 0; k < S; ++k) Z[k][v] = real(0);
    }

    // neighbours on the lines, as LDS offsets
    int q[n1], m[2][NPRIM > 0 ? NPRIM : 1];
#pragma unroll
    for (int k = 1; k <= N; ++k) q[k] = base + line_node<N, 2>(pd, d, r + k < n1 ? r + k : r + k - n1);
    q[0] = lane;
#pragma unroll
    for (int dd = 0; dd < 2; ++dd)
#pragma unroll
        for (int k = 1; k <= NPRIM; ++k)
            m[dd][k - 1] = base + line_node<N, 2>(pd, dd, pd[dd] - k < 0 ? pd[dd] - k + n1 : pd[dd] - k);

#pragma unroll
    for (int i = 0; i < S; ++i) {
        if (i > 0) {
            // the stage state: own half to LDS, all of it back
            const real cz = TAB == 1 ? rdt * Tab<real>::A(t, i, i - 1) : rdt;
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                us[V0 + v] = un(v) - cz * Z[i][v];
                lh[(V0 + v) * H + lane] = us[V0 + v];
            }
            __syncthreads();
#pragma unroll
            for (int v = 0; v < M; ++v)
                if (v < V0 || v >= V1) us[v] = lh[v * H + lane];
        }
        const real bi = Tab<real>::b(t, i);
        {
            const real g = bi * hl, c = bi * cU;
#pragma unroll
            for (int v = 0; v < M; ++v) {
                P[v] += g * us[v];
                Wf[v] -= c * us[v];
            }
            UB += bi * us[5 + d];
            Upsi += bi * us[8];
        }
        if constexpr (NCS) {
            // stage-wise interface flux: this stage's state at the face nodes
            if (valid && onface) {
                real *st = (real *)a.stage_tr;
#pragma unroll
                for (int v = 0; v < M; ++v) st[(((long)(face * S + i) * M + v) * E + e) * n1 + kk] = us[v];
            }
        }
        real nd[NF];
        Phys::node(us, nd, ctx);
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            const bool mine = ROLE == 0 ? (f < 5 || f >= 12) : (f >= 5 && f < 12);
            if (mine && Phys::paired(f)) lf[Phys::lidx(f) * H + lane] = nd[f];
        }
        __syncthreads();
        // own direction: directly evaluated rotations, diagonal, non-conservative term
        real R[M];
#pragma unroll
        for (int v = 0; v < M; ++v) R[v] = real(0);
        // sum_q D_pq g_d(u_q), twice
        real gB = Dk(0) * nd[5 + d], gpsi = Dk(0) * nd[8];
#pragma unroll
        for (int k = 1; k <= N; ++k) {
            const bool direct = !SYM || k <= NPRIM || k == KSELF;
            if (!direct) {
                gB += Dk(k) * lf[Phys::lidx(5 + d) * H + q[k]];
                gpsi += Dk(k) * lf[Phys::lidx(8) * H + q[k]];
                continue;
            }
            real ndq[NF], fs[M];
#pragma unroll
            for (int f = 0; f < NF; ++f)
                if (Phys::paired(f)) ndq[f] = lf[Phys::lidx(f) * H + q[k]];
            Phys::pair(d, nd, ndq, fs, ctx);
#pragma unroll
            for (int v = 0; v < M; ++v)
                if (Phys::pairs(d, v)) R[v] += Dk(k) * fs[v];
            gB += Dk(k) * ndq[5 + d];
            gpsi += Dk(k) * ndq[8];
            if constexpr (SYM) {
                if (k <= NPRIM) {
#pragma unroll
                    for (int v = 0; v < M; ++v)
                        if (Phys::pairs(d, v)) lx[Sh::xslot(d, k, v) * H + lane] = fs[v];
                }
            }
        }
        if (onface) {
            real fp[M], o[M];
            Phys::phys(d, nd, fp, ctx);
            Phys::btimes(d, nd, nd[5 + d], nd[8], o);
            const real c0 = Dk(0), gp = bi * real(0.5), gw = bi * cF, go = NCS ? real(0.5) * bi * sw : bi * sw;
#pragma unroll
            for (int v = 0; v < M; ++v) {
                if (Phys::pairs(d, v)) R[v] += c0 * fp[v];
                P[v] += gp * fp[v];
                Wf[v] += go * o[v] - gw * fp[v];
            }
        }
        {
            // sum_q D_pq B_d(u_p) g_d(u_q) = B_d(u_p) (sum_q D_pq g_d(u_q))
            real o[M];
            Phys::btimes(d, nd, real(0.5) * gB, real(0.5) * gpsi, o);
#pragma unroll
            for (int v = 0; v < M; ++v) R[v] += o[v];
            R[8] += real(0.5) * ctx.ch * gB;
            R[5 + d] += real(0.5) * ctx.ch * gpsi;
        }
#pragma unroll
        for (int v = 0; v < M; ++v)
            if (v < V0 || v >= V1) lh[v * H + lane] = R[v];
        __syncthreads();
        // the owned variables' whole residual
#pragma unroll
        for (int v = V0; v < V1; ++v) {
            real Rv = R[v] + lh[v * H + lane];
            if constexpr (SYM) {
#pragma unroll
                for (int dd = 0; dd < 2; ++dd)
#pragma unroll
                    for (int k = 1; k <= NPRIM; ++k)
                        if (Phys::pairs(dd, v))
                            Rv += (dd == d ? Dk(n1 - k) : Do(k)) * lx[Sh::xslot(dd, k, v) * H + m[dd][k - 1]];
            }
            const int o = v - V0;
            if constexpr (TAB == 1) {
                if (i + 1 < S) Z[i + 1][o] = Rv;
            } else {
#pragma unroll
                for (int k = i + 1; k < S; ++k)
                    if (stage_coupled<TAB>(k, i)) Z[k][o] += Tab<real>::A(t, k, i) * Rv;
            }
            W[o] += bi * Rv;
        }
    }

    if constexpr (!NCS) {
        // own half of 1/2 B(u^n)(g(U^-) + g(U^+))
        if (onface) {
            real uo[M], ndo[NF], o[M];
#pragma unroll
            for (int v = 0; v < M; ++v) uo[v] = uin[((long)v * E + es) * NP + node];
            Phys::node_basic(uo, ndo, ctx);
            Phys::btimes(d, ndo, real(0.5) * UB, real(0.5) * Upsi, o);
#pragma unroll
            for (int v = 0; v < M; ++v) Wf[v] -= sw * o[v];
        }
    }
    // the face terms of the variables the other lane owns (into the fields'
    // slots, which no lane reads any more)
#pragma unroll
    for (int v = 0; v < M; ++v)
        if (v < V0 || v >= V1) lf[v * H + lane] = Wf[v];
    __syncthreads();
    if (!valid) return;
    real *uout = (real *)a.u_out;
#pragma unroll
    for (int v = V0; v < V1; ++v)
        uout[((long)v * E + e) * NP + node] = un(v - V0) - rdt * (W[v - V0] + (Wf[v] + lf[v * H + lane]));
    if (onface) {
        real *tb = (real *)a.traces + ((long)face * FD::NCT * E + e) * n1 + kk;
#pragma unroll
        for (int v = 0; v < M; ++v) tb[((long)v * E) * n1] = P[v];
        tb[((long)M * E) * n1] = UB;
        tb[((long)(M + 1) * E) * n1] = Upsi;
    }
}

template <typename real, int N, int FLUX, int S, int TAB, bool NCS>
__global__ void __launch_bounds__(2 * tile_block<(N + 1) * (N + 1)>()) __attribute__((amdgpu_waves_per_eu(2)))
k_local_split(const Tables t, const StepPtrs a)
{
    using Sh = SplitShape<real, N, FLUX>;
    __shared__ real smem[Sh::slots * Sh::HALF];
    const long e0 = (long)xcd_chunk_tile(blockIdx.x, gridDim.x) * Sh::EPB;
    const int lane = threadIdx.x % Sh::HALF;
    if (__builtin_amdgcn_readfirstlane(threadIdx.x / Sh::HALF) == 0)
        split_lane<real, N, FLUX, S, TAB, NCS, 0>(t, a, e0, smem, lane);
    else
        split_lane<real, N, FLUX, S, TAB, NCS, 1>(t, a, e0, smem, lane);
}

template <typename real, int N, int FLUX>
hipError_t launch_local_split(const Tables &t, const StepPtrs &p, hipStream_t s)
{
    using Sh = SplitShape<real, N, FLUX>;
    const dim3 g((t.nelem + Sh::EPB - 1) / Sh::EPB), b(2 * Sh::HALF);
    // (one launch; with phases issued separately it belongs to the instance without the blending code)
    if (!(p.instances == 0 || (p.instances & 1))) return hipSuccess;
#define CRK_SPLIT(SS, TT, NC) hipLaunchKernelGGL((k_local_split<real, N, FLUX, SS, TT, NC>), g, b, 0, s, t, p)
    if (p.stage_tr != nullptr) {
        // stage-wise non-conservative interface flux: the default tableaus only
        if (t.stages == 4 && t.tableau == 1) CRK_SPLIT(4, 1, true);
        else if (t.stages == 6 && t.tableau == 2) CRK_SPLIT(6, 2, true);
        else return hipErrorInvalidValue;
        return hipGetLastError();
    }
    switch (t.stages) {
    case 1: CRK_SPLIT(1, 0, false); break;
    case 2: CRK_SPLIT(2, 0, false); break;
    case 3: CRK_SPLIT(3, 0, false); break;
    case 4: if (t.tableau == 1) CRK_SPLIT(4, 1, false); else CRK_SPLIT(4, 0, false); break;
    case 5: CRK_SPLIT(5, 0, false); break;
    case 6: if (t.tableau == 2) CRK_SPLIT(6, 2, false); else CRK_SPLIT(6, 0, false); break;
    default: return hipErrorInvalidValue;
    }
#undef CRK_SPLIT
    return hipGetLastError();
}

} // namespace crk
