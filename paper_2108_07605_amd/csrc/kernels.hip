// HIP kernels of the reactive-mixture lattice Boltzmann step for gfx950.
//
// One time step is three launches over a (possibly batched) work list:
//   k_boundary   interface nodes: advection + wall / inlet / outlet
//                reconstruction (section 4) into the planes' interface slots;
//   k_species    every node: advection, moments, temperature (eq.
//                temperature), relaxation rates, Stefan-Maxwell diffusion
//                velocities (eq. transform1), the reaction increment by l
//                forward-Euler sub-steps (eq. R3) and the collision of the
//                species lattices, whose populations stay in registers from
//                the moments to the collision; publishes T, Phi_a and the
//                enthalpy moments for the neighbours and the record that
//                k_flow reads;
//   k_flow       every node: the same-time gradients of Phi_a and
//                sum_b H_b Y_b and the collisions of the momentum and energy
//                lattices.
// Lattices with the linearly implicit reaction update, whose Jacobian takes
// the registers that would hold the populations, run
//   k_local (moments, diffusion), k_chem_implicit (its sub-steps, then the
//   gradients) and k_update (advection again, every collision)
// in place of the last two.
// Populations are structure-of-arrays [L][27][P] (x fastest), pulled from the
// source buffer, so every load and store of a wavefront is coalesced.  The
// storage type S is double (FP64) or float (FP32 deviation from a reference
// population per lattice and velocity, decoded to FP64 on load).

#include <hip/hip_runtime.h>

#include <mutex>
#include <type_traits>

#include "launch.hpp"
#include "physics.hpp"

namespace rlbm {

// ---------------------------------------------------------------------------
// storage references
// ---------------------------------------------------------------------------
// FP32 deviation storage: population (l, i) is stored as its deviation from
// s_l(y) G_li, where G_li is the zero-velocity equilibrium shape of lattice l
// at the domain-mean initial state normalised to unit zeroth moment, and
// s_l(y) a zeroth moment of lattice l (rho_a, rho or rho E) at the node y
// that reads the population, rounded to FP32.
// Both factors hold FP32 values, so their product is exact in FP64: every
// writer and reader forms the same reference however the compiler fuses it.
__device__ __forceinline__ double ref_of(float s, double G) { return (double)s * G; }

// The energy lattice's reference: at zero velocity its equilibrium is
// rho U W_i(theta) + rho K_i(theta) (eq. geq_i with u = 0: K carries the
// theta^2 terms and has zero sum), so its reference is s_g W_i + s_f K_i with
// s_g = rho E and s_f = rho of the reading node (both products exact).
__device__ __forceinline__ double ref_g(float sg, float sf, double W, double K) {
    return (double)sg * W + (double)sf * K;
}

// Stored lattices: the species lattices (M - 1 of them when one species is
// slaved, eq. strongest; all M in the weakly coupled storage, W = 1), then
// the momentum lattice f at LF and the energy lattice g at LG.
template <int M, int W>
struct Lat {
    static constexpr int NSP = M - 1 + W;
    static constexpr int LF = NSP;
    static constexpr int LG = NSP + 1;
    static constexpr int NL = NSP + 2;
    // linearly implicit update, FP32 storage: the scales of f and g fill up the
    // species' row
    static constexpr bool ROW = (NL + 3) / 4 == (NSP + 3) / 4;
};

// Layout of the reference table for NL stored lattices: shapes G[NL][Q] (the
// energy lattice's row is W), the zeroth moments sum_i G_li [NL],
// sum_i G_fi c_ix^2, the energy lattice's K[Q] and sum_i K_i.
template <int NL> constexpr int REF_M0 = NL * Q;
template <int NL> constexpr int REF_M2 = NL * Q + NL;
template <int NL> constexpr int REF_K = NL * Q + NL + 1;
template <int NL> constexpr int REF_K0 = NL * Q + NL + 1 + Q;
// then the shapes again, velocity by velocity: [Q][NL] (one wide scalar load
// per velocity where a kernel walks the lattices)
template <int NL> constexpr int REF_T = NL * Q + NL + 2 + Q;

// Scales s_l of node n in buffer q: the stored species (rss floats per node),
// and rho, rho E (fss floats per node).  Buffer par decodes the step's source
// populations, buffer par ^ 1 encodes what it writes.
//   Linearly implicit update: k_local writes the step's own moments to buffer
// par ^ 1, for k_update.  Where the species leave two floats of their row free
// (Lat::ROW), f and g take them (rss = fss).
//   Explicit update: a species population written in a step is encoded with the
// zeroth moment its reader had one step earlier, which is known before the
// step's moments (the species collide in the kernel that forms them); the
// step's own moments then replace buffer par, for the step after.  f and g,
// which collide a kernel later, take the moment of the step itself (fss = 2).
__device__ __forceinline__ const RLBM_GLOBAL float* scale_at(const LatDev& L, int q, long long n) {
    return as_global(L.rscale[q]) + (size_t)n * L.rss;
}
__device__ __forceinline__ const RLBM_GLOBAL float* fscale_at(const LatDev& L, int q, long long n) {
    return as_global(L.fscale[q]) + (size_t)n * L.fss;
}
// the scale of lattice l (wave-uniform; LF: the momentum lattice)
__device__ __forceinline__ float scale_l(const LatDev& L, int q, long long n, int l, int LF) {
    return l < LF ? scale_at(L, q, n)[l] : fscale_at(L, q, n)[l - LF];
}

// Block index -> work tile, XCD-aware.  Workgroups are dispatched to the
// eight XCDs round-robin (block b on XCD b mod 8), and each XCD has its own
// L2.  Remapping gives every XCD one contiguous range of tiles, so tiles that
// share cache lines (x-neighbours of the pull advection, the rows of a
// gradient stencil) are processed by the same L2 at about the same time.
// A bijection on [0, gridDim.x) for any grid size.
__device__ __forceinline__ int xcd_block() {
    const int nb = gridDim.x, b = blockIdx.x;
    const int q = nb >> 3, r = nb & 7, j = b & 7, i = b >> 3;
    return j * q + (j < r ? j : r) + i;
}

// Byte-offset addressing: a uniform base plus a 32-bit per-lane offset keeps
// every population access in the scalar-base form (no 64-bit address math).
template <typename S>
__device__ __forceinline__ S ld_at(const RLBM_GLOBAL S* base, int idx) {
    return *(const RLBM_GLOBAL S*)((const RLBM_GLOBAL char*)base + (unsigned)(idx * (int)sizeof(S)));
}
template <typename S>
__device__ __forceinline__ void st_at(RLBM_GLOBAL S* base, int idx, S v) {
    *(RLBM_GLOBAL S*)((RLBM_GLOBAL char*)base + (unsigned)(idx * (int)sizeof(S))) = v;
}

template <typename S>
__device__ __forceinline__ void st_off(RLBM_GLOBAL S* base, unsigned off, S v) {
    *(RLBM_GLOBAL S*)((RLBM_GLOBAL char*)base + off) = v;
}

// A correction row of the per-node record: FP32 (rounded to nearest even)
// when F32, else FP64.
template <bool F32>
__device__ __forceinline__ void st_corr(RLBM_GLOBAL double* prm, int row, size_t N, int node, double v) {
    if constexpr (F32) st_at(reinterpret_cast<RLBM_GLOBAL float*>(prm + (size_t)row * N), node, (float)v);
    else st_at(prm + (size_t)row * N, node, v);
}
template <bool F32>
__device__ __forceinline__ double ld_corr(const RLBM_GLOBAL double* prm, int row, size_t N, int node) {
    if constexpr (F32) return (double)ld_at(reinterpret_cast<const RLBM_GLOBAL float*>(prm + (size_t)row * N), node);
    else return ld_at(prm + (size_t)row * N, node);
}

// ---------------------------------------------------------------------------
// work-list helpers
// ---------------------------------------------------------------------------
// Step counter of a launch: a device counter (batched steps replayed from a
// captured graph advance it with k_advance_time) plus the launch's offset.
__device__ __forceinline__ long long step_time(const long long* tp, long long toff) {
    return (tp ? *tp : 0) + toff;
}
__device__ __forceinline__ int find_lattice(const int* blk, int n_lat, int b) {
    int lo = 0, hi = n_lat - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (blk[mid] <= b) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// ---------------------------------------------------------------------------
// pull-advection addressing for the hot kernels
// ---------------------------------------------------------------------------
// Node offsets of the source x - c for c = -1, 0, +1 along each axis, with
// periodic wrap.  Along non-periodic axes only interface nodes would leave
// the box, and those read the boundary buffer instead, so the wrapped value
// is only ever an in-bounds placeholder.
struct PullOff {
    int x[3], y[3], z[3];   // index c + 1
};

__device__ __forceinline__ void pull_offsets(const LatDev& L, int x, int y, int z, PullOff& o) {
    const int nx = L.nx, ny = L.ny, nz = L.nz, sxy = nx * ny;
    o.x[0] = x == nx - 1 ? -(nx - 1) : 1;   // c = -1: source x + 1
    o.x[1] = 0;
    o.x[2] = x == 0 ? nx - 1 : -1;          // c = +1: source x - 1
    o.y[0] = y == ny - 1 ? -(ny - 1) * nx : nx;
    o.y[1] = 0;
    o.y[2] = y == 0 ? (ny - 1) * nx : -nx;
    o.z[0] = z == nz - 1 ? -(nz - 1) * sxy : sxy;
    o.z[1] = 0;
    o.z[2] = z == 0 ? (nz - 1) * sxy : -sxy;
}

__device__ __forceinline__ int sel3(int c, int m, int z, int p) { return c < 0 ? m : (c == 0 ? z : p); }
__device__ __forceinline__ double sel3d(int c, double m, double z, double p) { return c < 0 ? m : (c == 0 ? z : p); }

// Node that pulls the population stored at slot (node, i): node + c_i,
// wrapped on every axis (the placeholder rule of the pull offsets o).
__device__ __forceinline__ int reader_at(int node, const PullOff& o, int c0, int c1, int c2) {
    return node + sel3(c0, o.x[2], 0, o.x[0]) + sel3(c1, o.y[2], 0, o.y[0]) + sel3(c2, o.z[2], 0, o.z[0]);
}

// The first NSP scales of node n's row in buffer q (FP32 storage), as whole
// 16-byte loads (rss is a multiple of four floats).
template <int NSP>
__device__ __forceinline__ void species_scales(const LatDev& L, int q, int n, float* out) {
    typedef float f4 __attribute__((ext_vector_type(4)));
    const RLBM_GLOBAL f4* p4 = reinterpret_cast<const RLBM_GLOBAL f4*>(scale_at(L, q, n));
#pragma unroll
    for (int v = 0; v < (NSP + 3) / 4; ++v) {
        const f4 w = p4[v];
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (4 * v + e < NSP) out[4 * v + e] = w[e];
    }
}
// rho and rho E scales of node n in buffer q, in rows of two floats.
__device__ __forceinline__ void flow_scales(const LatDev& L, int q, int n, float* out) {
    typedef float f2 __attribute__((ext_vector_type(2)));
    const f2 v = *(reinterpret_cast<const RLBM_GLOBAL f2*>(as_global(L.fscale[q])) + n);
    out[0] = v.x;
    out[1] = v.y;
}
// all NL of them, stored lattices in order, of either update
template <int NL>
__device__ __forceinline__ void scales_of(const LatDev& L, int q, int n, float (&out)[NL]) {
    species_scales<NL - 2>(L, q, n, out);
    const RLBM_GLOBAL float* f = fscale_at(L, q, n);
    out[NL - 2] = f[0];
    out[NL - 1] = f[1];
}

// Stored lattice of species a; a slaved index of M (the weakly coupled
// storage) stores every species at its own index.
__device__ __forceinline__ int lat_of(int a, int slaved) { return a - (a > slaved ? 1 : 0); }

// Per-thread LDS columns of k_local (stride LOC_T doubles between rows): the
// species densities rho_a [M] and velocity differences u_a - u [3 M], handed
// from the streaming part to the Stefan-Maxwell step without a trip to memory.
struct LocalLds {
    double* ra;   // &rho_a[0][tid]
    double* dv;   // &(u_a - u)[0][tid], row 3 a + d
};
constexpr int LOC_T = NODE_TILE;   // k_local threads per block

// ---------------------------------------------------------------------------
// Stefan-Maxwell diffusion velocities (section 2.3, eq. transform1)
// ---------------------------------------------------------------------------
// The system (dt = 1)
//   (1 + 1/(2 tau_a)) V_a - 1/2 sum_{b != a} Y_b V_b / tau_ab = u_a - u
// with 1/tau_ab = common K_ab and 1/tau_a = sum_{b != a} Y_b / tau_ab, for
// the three components at once.  Its matrix is strictly row diagonally
// dominant with margin 1 (the off-diagonal row sums are -1/(2 tau_a)), so
// Doolittle LU without pivoting is stable.  Rows are generated on the fly
// from cY_b = -common Y_b / 2 (A_ab = K_ab cY_b) and the forward substitution
// runs with the factorisation.  The velocity differences u_a - u and the
// densities rho_a come from k_local's LDS columns, the node's scalars from
// its registers; writes V_a and the energy flux base Qb plus
// omega1 sum_a H_a rho_a V_a to the per-node record.
template <int M, int W, bool F32>
__device__ __forceinline__ void stefan_maxwell(const LatDev& L, int node, const LocalLds& ls, double T, double rho,
                                               double common, double omega1, const double* Y, const double* Qb,
                                               double rho_over_rhoY) {
    MechC mc0 = *as_const(L.mech);
    const size_t N = (size_t)L.N;
    RLBM_GLOBAL double* prm = as_global(L.prm);
    double cY[M], V[M][3];
#pragma unroll
    for (int a = 0; a < M; ++a) {
        cY[a] = -0.5 * common * Y[a];
#pragma unroll
        for (int d = 0; d < 3; ++d) V[a][d] = ls.dv[(3 * a + d) * LOC_T];
    }
    double Uu[M][M];
    double inv_diag[M];
#pragma unroll
    for (int i = 0; i < M; ++i) {
        reload_barrier();
        MechC mc = in_loop(mc0);   // this row's K_ab as scalar loads, not hoisted
        double st = 0.0;
#pragma unroll
        for (int c = 0; c < M; ++c)
            if (c != i) st += mc.Kab[i][c] * cY[c];
        const double inv_tau = -2.0 * st;
        double lrow[M];
#pragma unroll
        for (int j = 0; j < i; ++j) {
            double a = mc.Kab[i][j] * cY[j];
#pragma unroll
            for (int kk = 0; kk < j; ++kk) a -= lrow[kk] * Uu[kk][j];
            lrow[j] = a * inv_diag[j];
        }
#pragma unroll
        for (int j = i; j < M; ++j) {
            double a = (i == j) ? 1.0 + 0.5 * inv_tau : mc.Kab[i][j] * cY[j];
#pragma unroll
            for (int kk = 0; kk < i; ++kk) a -= lrow[kk] * Uu[kk][j];
            Uu[i][j] = a;
        }
        inv_diag[i] = 1.0 / Uu[i][i];
#pragma unroll
        for (int dd = 0; dd < 3; ++dd) {
            double yv = V[i][dd];
#pragma unroll
            for (int kk = 0; kk < i; ++kk) yv -= lrow[kk] * V[kk][dd];
            V[i][dd] = yv;
        }
    }
#pragma unroll
    for (int i = M - 1; i >= 0; --i) {
#pragma unroll
        for (int dd = 0; dd < 3; ++dd) {
            double sm = V[i][dd];
#pragma unroll
            for (int j = i + 1; j < M; ++j) sm -= Uu[i][j] * V[j][dd];
            V[i][dd] = sm * inv_diag[i];
            st_corr<F32>(prm, PRM_SP + 6 * i + 1 + dd, N, node, V[i][dd]);
        }
    }
    // energy flux: Qb + omega1 sum_a H_a rho_a V_a
    MechC mc = mc0;
    double diff[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int a = 0; a < M; ++a) {
        const double hy = (species_U(mc, a, T) + mc.Ra[a] * T) * ls.ra[a * LOC_T];
#pragma unroll
        for (int dd = 0; dd < 3; ++dd) diff[dd] += hy * V[a][dd];
    }
    (void)rho;
    // rho Y_a = rho_a, except in the weakly coupled storage where Y_a is
    // normalised by sum_b rho_b
    if constexpr (W) {
#pragma unroll
        for (int dd = 0; dd < 3; ++dd) diff[dd] *= rho_over_rhoY;
    } else {
        (void)rho_over_rhoY;
    }
#pragma unroll
    for (int dd = 0; dd < 3; ++dd) st_corr<F32>(prm, PRM_QB + dd, N, node, Qb[dd] + omega1 * diff[dd]);
}

// Relaxation rates of a node (sections 2.3 and 3.4) from its temperature,
// pressure and mixture gas constant Rmix = R_univ sum_a Y_a / m_a: the
// factor `common` of 1/tau_ab = common K_ab (eqs. betaa, taua), and omega,
// omega_1 of the momentum and energy lattices.
__device__ __forceinline__ void relax_rates(MechC mc, double T, double P, double Rmix, double& common,
                                            double& omega, double& omega1) {
    const double lnr = ln(T * mc.inv_T_ref);
    common = mc.R_univ * mc.R_univ * T * recip(Rmix) * P * mc.inv_P_ref * expo(mc.ec, -mc.D_exp * lnr);
    const double muP = mc.mu_ref * expo(mc.ec, mc.mu_exp * lnr) * recip(P);
    omega = recip(muP + 0.5);
    omega1 = recip(fma(muP, mc.inv_Pr, 0.5));
}

// ---------------------------------------------------------------------------
// k_local: moments and everything else a node needs from its own populations
// (lattices with the linearly implicit reaction update)
// ---------------------------------------------------------------------------
// Moments of the node's post-advection, post-boundary populations (eqs.
// density1, momentum1, fdensity, f1momMomentum, g0momTotalEnergy), the
// slaved species by difference (eq. strongest), then the temperature (eq.
// temperature), the relaxation rates and the local part of the energy flux.
// The momentum and energy lattices are summed first so the mixture velocity
// is known when each species lattice is summed: its velocity difference
// u_a - u is written out at once and only rho_a stays in registers.  In FP32
// deviation storage the sums run over the stored deviations and the
// reference's own moments are added in closed form (zeroth s_l sum_i G_li,
// second s_f sum_i G_fi c c, first zero by symmetry); the stored species'
// rho_a, rho and rho E become the scales of the populations written this step,
// in whole 16-byte stores.
// The Stefan-Maxwell solve comes last, once the streaming part no longer holds
// registers.
template <int M>
struct LocalMoments {
    double rho, rhoE, j[3], q[3], Pd[3], Po[3];   // Pd: xx yy zz, Po: xy xz yz
    double u[3];
    double rho_a[M];
};

// Bytes of a population plane.
__device__ __forceinline__ unsigned plane_bytes(long long N, int s) {
    const unsigned long long b = (unsigned long long)N * (unsigned)s;
    return b > 0xffffffffull ? 0xffffffffu : (unsigned)b;
}

// Population loads through one resource per window of nine planes (the nine
// velocities of one c_z layer of one lattice): the plane within the window is
// a scalar offset, the node a per-lane offset.  Few resources stay live, so
// the scalar registers do not run out.  The host keeps nine planes below 2^32
// bytes.
template <typename S>
__device__ __forceinline__ S ld_win(const RLBM_GLOBAL S* win, unsigned plane, int iw, int idx) {
    const __amdgpu_buffer_rsrc_t r =
        __builtin_amdgcn_make_buffer_rsrc((void*)(unsigned long long)win, 0, (int)(9u * plane), 0x00020000);
    if constexpr (sizeof(S) == 4)
        return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, (unsigned)idx * 4u, iw * plane, 0));
    else
        return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, (unsigned)idx * 8u, iw * plane, 0));
}

// Scales of what is written for f and g this step: the node's rho and rho E
// (rows of two floats).
__device__ __forceinline__ void store_fscale(const LatDev& L, int q, int node, double rho, double rhoE) {
    typedef float f2 __attribute__((ext_vector_type(2)));
    f2 v;
    v.x = __double2float_rn(rho);
    v.y = __double2float_rn(rhoE);
    *(reinterpret_cast<RLBM_GLOBAL f2*>(as_global(L.fscale[q])) + node) = v;
}

// The moment sums of k_local.  IF = false: no lane of the wave is an
// interface node and every population is pulled from the source buffer;
// IF = true: interface lanes read their reconstructed populations from the
// planes' interface slots instead.
template <int M, typename S, int W, bool IF>
__device__ __forceinline__ void local_moments(const LatDev& L, int par, int k, int node, const PullOff& o,
                                              const LocalLds& ls, LocalMoments<M>& m) {
    constexpr int NSP = Lat<M, W>::NSP, LF = Lat<M, W>::LF, LG = Lat<M, W>::LG, NL = Lat<M, W>::NL;
    const size_t N = (size_t)L.N;
    const int s = W ? M : L.slaved;
    const RLBM_GLOBAL S* src = as_global(static_cast<const S*>(L.pop[par]));
    RLBM_GLOBAL double* prm = as_global(L.prm);
    auto off_of = [&](int i) { return node + o.x[cx_of(i) + 1] + o.y[cy_of(i) + 1] + o.z[cz_of(i) + 1]; };
    const size_t P = (size_t)L.P;
    const unsigned nb = plane_bytes(L.P, sizeof(S));
    // an interface lane reads its post-boundary population from the plane's
    // interface slot N + k instead of its pull source: the same load with
    // another index
    auto ld = [&](int l, int i) -> S {
        const int idx = IF ? (k >= 0 ? (int)N + k : off_of(i)) : off_of(i);
        return ld_win(src + (size_t)(l * Q + 9 * (i / 9)) * P, nb, i % 9, idx);
    };
    const RLBM_GLOBAL float *sc = nullptr, *fs = nullptr;
    if constexpr (sizeof(S) == 4) {
        sc = scale_at(L, par, node);
        fs = fscale_at(L, par, node);
    }

    // the first species lattice's loads go out with the momentum and energy
    // lattices' (FP32 storage), so its sum does not wait for a round trip of
    // its own
    constexpr bool PF = sizeof(S) == 4;
    S cur[Q];
    if constexpr (PF) {
#pragma unroll
        for (int i = 0; i < Q; ++i) cur[i] = ld(0, i);
    }
    // momentum and energy lattices
    double rho = 0.0, rhoE = 0.0, j[3] = {0.0, 0.0, 0.0}, q[3] = {0.0, 0.0, 0.0};
    double Pd[3] = {0.0, 0.0, 0.0}, Po[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        const int cx = cx_of(i), cy = cy_of(i), cz = cz_of(i);
        const double f = (double)ld(LF, i);
        const double g = (double)ld(LG, i);
        rho += f;
        rhoE += g;
        if (cx) { j[0] += cx > 0 ? f : -f; Pd[0] += f; q[0] += cx > 0 ? g : -g; }
        if (cy) { j[1] += cy > 0 ? f : -f; Pd[1] += f; q[1] += cy > 0 ? g : -g; }
        if (cz) { j[2] += cz > 0 ? f : -f; Pd[2] += f; q[2] += cz > 0 ? g : -g; }
        if (cx * cy) Po[0] += cx * cy > 0 ? f : -f;
        if (cx * cz) Po[1] += cx * cz > 0 ? f : -f;
        if (cy * cz) Po[2] += cy * cz > 0 ? f : -f;
    }
    if constexpr (sizeof(S) == 4) {
        const RLBM_CONST double* G = as_const(L.ref);
        const double sf = (double)fs[0];
        rho += sf * G[REF_M0<NL> + LF];
        rhoE += (double)fs[1] * G[REF_M0<NL> + LG] + sf * G[REF_K0<NL>];
        const double p2 = sf * G[REF_M2<NL>];
        Pd[0] += p2; Pd[1] += p2; Pd[2] += p2;
    }
    const double inv_rho = 1.0 / rho;
    const double u[3] = {j[0] * inv_rho, j[1] * inv_rho, j[2] * inv_rho};

    // species lattices, one at a time, the next one's loads in flight while
    // the current one is summed; rho_a goes to the record row PRM_SP + 6 a and
    // with u_a - u (zero for an absent species, u_a := u) to LDS
    double rs = rho, js[3] = {j[0], j[1], j[2]};
    auto put_species = [&](int a, double ra, double jx, double jy, double jz) {
        const bool small = ra <= 1e-14 * rho;
        const double inv = small ? 0.0 : 1.0 / ra;
        st_at(prm + (size_t)(PRM_SP + 6 * a) * N, node, ra);
        ls.ra[a * LOC_T] = ra;
        ls.dv[(3 * a + 0) * LOC_T] = small ? 0.0 : jx * inv - u[0];
        ls.dv[(3 * a + 1) * LOC_T] = small ? 0.0 : jy * inv - u[1];
        ls.dv[(3 * a + 2) * LOC_T] = small ? 0.0 : jz * inv - u[2];
    };
    // FP32 storage double-buffers the species loads (the first lattice's
    // were issued above); FP64 has no registers to spare for it
#pragma unroll 1
    for (int l = 0; l < NSP; ++l) {
        reload_barrier();
        S nxt[Q];
        if constexpr (PF) {
            if (l + 1 < NSP) {
#pragma unroll
                for (int i = 0; i < Q; ++i) nxt[i] = ld(l + 1, i);
            }
        } else {
#pragma unroll
            for (int i = 0; i < Q; ++i) cur[i] = ld(l, i);
        }
        double ra = 0.0, jx = 0.0, jy = 0.0, jz = 0.0;
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            const int cx = cx_of(i), cy = cy_of(i), cz = cz_of(i);
            const double v = (double)cur[i];
            ra += v;
            if (cx) jx += cx > 0 ? v : -v;
            if (cy) jy += cy > 0 ? v : -v;
            if (cz) jz += cz > 0 ? v : -v;
        }
        if constexpr (sizeof(S) == 4) {
            const RLBM_CONST double* rm = as_const(L.ref) + REF_M0<NL> + opaque_zero();
            ra += (double)sc[l] * rm[l];
        }
        const int a = W ? l : l + (l >= s ? 1 : 0);
        put_species(a, ra, jx, jy, jz);
        rs -= ra; js[0] -= jx; js[1] -= jy; js[2] -= jz;
        if constexpr (PF) {
#pragma unroll
            for (int i = 0; i < Q; ++i) cur[i] = nxt[i];
        }
    }
    if constexpr (!W) put_species(s, rs, js[0], js[1], js[2]);
    // the species densities come back from LDS rather than being held in
    // registers through the loop
#pragma unroll
    for (int c = 0; c < M; ++c) m.rho_a[c] = ls.ra[c * LOC_T];
    if constexpr (sizeof(S) == 4) {
        typedef float f4 __attribute__((ext_vector_type(4)));
        RLBM_GLOBAL f4* so = reinterpret_cast<RLBM_GLOBAL f4*>(as_global(L.rscale[par ^ 1]) + (size_t)node * L.rss);
#pragma unroll
        for (int v = 0; v < (NSP + 3) / 4; ++v) {
            f4 w = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int l = 4 * v + e;
                if (l < NSP) w[e] = __double2float_rn(ls.ra[(l + (!W && l >= s ? 1 : 0)) * LOC_T]);
                else if (Lat<M, W>::ROW && l < NL) w[e] = __double2float_rn(l == LF ? rho : rhoE);
            }
            so[v] = w;
        }
        if constexpr (!Lat<M, W>::ROW) store_fscale(L, par ^ 1, node, rho, rhoE);
    }
    m.rho = rho;
    m.rhoE = rhoE;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        m.j[d] = j[d]; m.q[d] = q[d]; m.Pd[d] = Pd[d]; m.Po[d] = Po[d]; m.u[d] = u[d];
    }
}

template <int M, typename S, int W>
__global__ __launch_bounds__(NODE_TILE) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_local(const LatDev* __restrict__ lats, const int* __restrict__ blk,
                                               int n_lat, const long long* __restrict__ tp, long long toff) {
    const long long t = step_time(tp, toff);
    const int b = xcd_block();
    const int lj = find_lattice(blk, n_lat, b);
    const LatDev& L = lats[lj];
    if (t >= L.t_end || L.reaction == RLBM_REACTION_EXPLICIT) return;
    const int node = (b - blk[lj]) * NODE_TILE + threadIdx.x;
    if (node >= L.N) return;
    MechC mc = *as_const(L.mech);
    const int par = (L.parity0 + t) & 1;
    const int x = node % L.nx, r = node / L.nx, y = r % L.ny, z = r / L.ny;
    PullOff o;
    pull_offsets(L, x, y, z, o);
    const int k = L.n_if ? L.if_index[node] : -1;
    double* aux = L.aux;
    double* prm = L.prm;
    const size_t N = (size_t)L.N;

    __shared__ double s_ra[M][LOC_T], s_dv[3 * M][LOC_T];
    const LocalLds ls{&s_ra[0][threadIdx.x], &s_dv[0][threadIdx.x]};
    LocalMoments<M> m;
    if (__builtin_amdgcn_ballot_w64(k >= 0) != 0) local_moments<M, S, W, true>(L, par, k, node, o, ls, m);
    else local_moments<M, S, W, false>(L, par, k, node, o, ls, m);
    const double rho = m.rho, inv_rho = 1.0 / rho;
    const double u[3] = {m.u[0], m.u[1], m.u[2]};
    const double rhoE = m.rhoE;
    const double* rho_a = m.rho_a;
    const double* q = m.q;
    const double* Pd = m.Pd;
    const double* Po = m.Po;

    const double usq = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
    // composition: Y_a = rho_a / rho, or rho_a / sum_b rho_b in the weakly
    // coupled storage, where the species supply the composition and the
    // momentum lattice rho
    double rhoY = rho;
    if constexpr (W) {
        rhoY = 0.0;
#pragma unroll
        for (int a = 0; a < M; ++a) rhoY += rho_a[a];
    }
    const double inv_rhoY = W ? 1.0 / rhoY : inv_rho;
    double Y[M];
#pragma unroll
    for (int a = 0; a < M; ++a) Y[a] = rho_a[a] * inv_rhoY;
    const double U = rhoE * inv_rho - 0.5 * usq;
    int fail = 0;
    // temperature (eq. temperature), Newton from the previous step's value
    const double T = solve_T<M>(mc, Y, U, aux[AUX_T * N + node], &fail);
    if (fail) atomicOr(L.flag, 1);
    const double Rmix = mc.R_univ * mix_inv_m<M>(mc, Y);
    const double th = Rmix * T;
    const double P = rho * th;

    // relaxation rates (sections 2.3 and 3.4); k_update derives the same
    // values again from the record rather than reading them
    double common, omega, omega1;
    relax_rates(mc, T, P, Rmix, common, omega, omega1);

    // enthalpy-weighted composition moments sum_a H_a(T') Y_a = sum_kk T'^kk Pk
    double Pk[6];
#pragma unroll
    for (int kk = 0; kk < 6; ++kk) {
        double pk = 0.0;
#pragma unroll
        for (int a = 0; a < M; ++a) pk += mc.hc[a][kk] * Y[a];
        Pk[kk] = pk;
    }
    // local part of the energy-lattice flux
    //   Qb = (omega - omega1)(q - u.(P - P^eq) - q^eq); the Stefan-Maxwell step adds
    //   omega1 rho sum_a H_a Y_a V_a
    double Qb[3];
    {
        const double H = Pk[0] + T * (Pk[1] + T * (Pk[2] + T * (Pk[3] + T * (Pk[4] + T * Pk[5]))));
        const double hq = rho * (H + 0.5 * usq);
        const double Pt[3][3] = {{Pd[0], Po[0], Po[1]}, {Po[0], Pd[1], Po[2]}, {Po[1], Po[2], Pd[2]}};
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            double uP = 0.0;
#pragma unroll
            for (int c = 0; c < 3; ++c) uP += u[c] * (Pt[c][a] - rho * ((a == c ? th : 0.0) + u[c] * u[a]));
            Qb[a] = (omega - omega1) * (q[a] - uP - hq * u[a]);
        }
    }

    // neighbour-facing fields: Phi and the enthalpy moments for the gradient
    // stencil, T for the next step's Newton start; rho, u and Y only where
    // an outlet reads them (the first interior node of the x+ face)
#pragma unroll
    for (int d = 0; d < 3; ++d)
        aux[(AUX_PHI + d) * N + node] = rho * u[d] * (1.0 - 3.0 * th) - rho * u[d] * u[d] * u[d];
    aux[AUX_T * N + node] = T;
#pragma unroll
    for (int kk = 0; kk < 6; ++kk) aux[(AUX_Y + M + kk) * N + node] = Pk[kk];
    if (L.n_out > 0 && x == L.nx - 2) {
        aux[AUX_RHO * N + node] = rho;
#pragma unroll
        for (int d = 0; d < 3; ++d) aux[(AUX_U + d) * N + node] = u[d];
#pragma unroll
        for (int a = 0; a < M; ++a) aux[(AUX_Y + a) * N + node] = Y[a];
    }

    prm[PRM_RHO * N + node] = rho;
#pragma unroll
    for (int d = 0; d < 3; ++d) prm[(PRM_U + d) * N + node] = u[d];
    prm[PRM_T * N + node] = T;
    prm[PRM_UINT * N + node] = U;
    stefan_maxwell<M, W, sizeof(S) == 4>(L, node, ls, T, rho, common, omega1, Y, Qb, rho * inv_rhoY);
}

// ---------------------------------------------------------------------------
// same-time gradients with the isotropic D3Q27 stencil
//   d phi/dx_a = 3 sum_i w_i c_ia phi(x + c_i)
// of Phi_a (extension, eqs. Pex, qex) and of sum_b H_b Y_b with H_b at this
// node's temperature (Fourier correction, eq. corrFourier), from the fields
// k_local published.  Ghost values beyond a non-periodic face repeat the
// nearest node.  Writes rows PRM_GRAD..PRM_GRAD+5 of the per-node record.
// ---------------------------------------------------------------------------
template <int M>
__device__ __forceinline__ void store_gradients(const LatDev& L, int node, const double (&acc)[6]) {
    const size_t N = (size_t)L.N;
    if (L.storage == RLBM_STORAGE_F32_DEV) {
#pragma unroll
        for (int q = 0; q < 6; ++q) st_corr<true>(as_global(L.prm), prm_grad(M) + q, N, node, acc[q]);
    } else {
#pragma unroll
        for (int q = 0; q < 6; ++q) st_corr<false>(as_global(L.prm), prm_grad(M) + q, N, node, acc[q]);
    }
}

// Any node: the 26 neighbours' fields, each at its own offset.
template <int M>
__device__ __forceinline__ void node_gradients(const LatDev& L, int node, double (&acc)[6]) {
    const int nx = L.nx, ny = L.ny, nz = L.nz;
    const int x = node % nx, r = node / nx, y = r % ny, z = r / ny;
    const size_t N = (size_t)L.N;
    const double* aux = L.aux;
    const double T = aux[AUX_T * N + node];
    const double T2 = T * T, T3 = T2 * T, T4 = T3 * T, T5 = T4 * T;
    const bool px = L.per[0], py = L.per[1], pz = L.per[2];
    const int gx[3] = {x == 0 ? (px ? nx - 1 : 0) : x - 1, x, x == nx - 1 ? (px ? 0 : x) : x + 1};
    const int gy[3] = {y == 0 ? (py ? ny - 1 : 0) : y - 1, y, y == ny - 1 ? (py ? 0 : y) : y + 1};
    const int gz[3] = {z == 0 ? (pz ? nz - 1 : 0) : z - 1, z, z == nz - 1 ? (pz ? 0 : z) : z + 1};
    const double* Pk = aux + (size_t)(AUX_Y + M) * N;
#pragma unroll
    for (int k = 0; k < 6; ++k) acc[k] = 0.0;
#pragma unroll 1
    for (int czi = 0; czi < 3; ++czi) {
        const int cz = czi - 1;
        const size_t zrow = (size_t)sel3(cz, gz[0], gz[1], gz[2]) * ny;
        const double wz = cz ? 1.0 / 6.0 : 2.0 / 3.0;
#pragma unroll
        for (int j = 0; j < 9; ++j) {
            const int cx = j % 3 - 1, cy = j / 3 - 1;
            if (cx == 0 && cy == 0 && cz == 0) continue;
            const double w = 3.0 * (cx ? 1.0 / 6.0 : 2.0 / 3.0) * (cy ? 1.0 / 6.0 : 2.0 / 3.0) * wz;
            const size_t nb = (zrow + gy[cy + 1]) * nx + gx[cx + 1];
            const double hy = Pk[nb] + T * Pk[N + nb] + T2 * Pk[2 * N + nb] + T3 * Pk[3 * N + nb] +
                              T4 * Pk[4 * N + nb] + T5 * Pk[5 * N + nb];
            if (cx) { acc[0] += (cx * w) * aux[(AUX_PHI + 0) * N + nb]; acc[3] += (cx * w) * hy; }
            if (cy) { acc[1] += (cy * w) * aux[(AUX_PHI + 1) * N + nb]; acc[4] += (cy * w) * hy; }
            if (cz) { acc[2] += (cz * w) * aux[(AUX_PHI + 2) * N + nb]; acc[5] += (cz * w) * hy; }
        }
    }
}

// The weights factor per direction, w_i = w(c_ix) w(c_iy) w(c_iz) with
// w(0) = 2/3 and w(+-1) = 1/6.  With the sums over the 3x3 (y, z)
// neighbourhood of one column x
//   A(x) = sum w(cy) w(cz) phi,  B(x) = sum cy w(cz) phi,  C(x) = sum cz w(cy) phi
// the stencil is
//   d_x phi = (A(x+1) - A(x-1)) / 2,  d_y phi = sum_cx w(cx) B(x+cx) / 2,
//   d_z phi = sum_cx w(cx) C(x+cx) / 2.
// Column sums of one x: the six enthalpy coefficients (A, B, C each) and
// A of Phi_x, B of Phi_y, C of Phi_z.
struct ColSums {
    double a[6], b[6], c[6];
    double ax, by, cz;
};
template <int M>
__device__ __forceinline__ void column_sums(const LatDev& L, int xc, const int (&gy)[3], const int (&gz)[3],
                                            ColSums& o) {
    const size_t N = (size_t)L.N;
    const int nx = L.nx, ny = L.ny;
    const double* aux = L.aux;
    const double* Pk = aux + (size_t)(AUX_Y + M) * N;
#pragma unroll
    for (int k = 0; k < 6; ++k) o.a[k] = o.b[k] = o.c[k] = 0.0;
    o.ax = o.by = o.cz = 0.0;
#pragma unroll
    for (int j = 0; j < 9; ++j) {
        const int cy = j % 3 - 1, cz = j / 3 - 1;
        const double wy = cy ? 1.0 / 6.0 : 2.0 / 3.0, wz = cz ? 1.0 / 6.0 : 2.0 / 3.0;
        const size_t nb = ((size_t)gz[cz + 1] * ny + gy[cy + 1]) * nx + xc;
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            const double f = Pk[k * N + nb];
            o.a[k] += (wy * wz) * f;
            if (cy) o.b[k] += (cy * wz) * f;
            if (cz) o.c[k] += (cz * wy) * f;
        }
        o.ax += (wy * wz) * aux[(AUX_PHI + 0) * N + nb];
        if (cy) o.by += (cy * wz) * aux[(AUX_PHI + 1) * N + nb];
        if (cz) o.cz += (cz * wy) * aux[(AUX_PHI + 2) * N + nb];
    }
}

__device__ __forceinline__ double poly5(double t, const double (&v)[6]) {
    return v[0] + t * (v[1] + t * (v[2] + t * (v[3] + t * (v[4] + t * v[5]))));
}

// A wave whose 64 lanes are the consecutive nodes x0..x0+63 of one x-row
// (lane = x - x0): each lane loads its own column's 9 (y, z) neighbours and
// takes the column sums of x-1 and x+1 from the adjacent lanes; lane 0 and
// lane 63 load the ghost-aware column beyond the tile themselves.  The sum
// of H_b Y_b at this node's temperature is formed from the neighbour's
// coefficient sums, so a lane evaluates its sums at the temperature of the
// lane that receives them (the adjacent lane's T).  Every lane of the wave
// must reach this function.
template <int M>
__device__ __forceinline__ void row_tile_gradients(const LatDev& L, int node, int lane, double (&acc)[6]) {
    const int nx = L.nx, ny = L.ny, nz = L.nz;
    const int x = node % nx, r = node / nx, y = r % ny, z = r / ny;
    const size_t N = (size_t)L.N;
    const double T = L.aux[AUX_T * N + node];
    const bool px = L.per[0], py = L.per[1], pz = L.per[2];
    const int gy[3] = {y == 0 ? (py ? ny - 1 : 0) : y - 1, y, y == ny - 1 ? (py ? 0 : y) : y + 1};
    const int gz[3] = {z == 0 ? (pz ? nz - 1 : 0) : z - 1, z, z == nz - 1 ? (pz ? 0 : z) : z + 1};
    // the adjacent lanes' temperatures (lane 0 and lane 63 keep their own;
    // what they would send across the tile edge is not used)
    const double Tl = __shfl_up(T, 1u), Tr = __shfl_down(T, 1u);
    // from x+1 (sums at this lane's T), from x-1, and this column's own
    double hp_a, hp_b, hp_c, hm_a, hm_b, hm_c, h0_b, h0_c, fp_ax, fp_by, fp_cz, fm_ax, fm_by, fm_cz, f0_by, f0_cz;
    {
        ColSums s;
        column_sums<M>(L, x, gy, gz, s);
        h0_b = poly5(T, s.b);
        h0_c = poly5(T, s.c);
        f0_by = s.by;
        f0_cz = s.cz;
        hp_a = __shfl_down(poly5(Tl, s.a), 1u);
        hp_b = __shfl_down(poly5(Tl, s.b), 1u);
        hp_c = __shfl_down(poly5(Tl, s.c), 1u);
        hm_a = __shfl_up(poly5(Tr, s.a), 1u);
        hm_b = __shfl_up(poly5(Tr, s.b), 1u);
        hm_c = __shfl_up(poly5(Tr, s.c), 1u);
        fp_ax = __shfl_down(s.ax, 1u);
        fp_by = __shfl_down(s.by, 1u);
        fp_cz = __shfl_down(s.cz, 1u);
        fm_ax = __shfl_up(s.ax, 1u);
        fm_by = __shfl_up(s.by, 1u);
        fm_cz = __shfl_up(s.cz, 1u);
    }
    if (lane == 0 || lane == NODE_TILE - 1) {
        const int xg = lane == 0 ? (x == 0 ? (px ? nx - 1 : 0) : x - 1) : (x == nx - 1 ? (px ? 0 : x) : x + 1);
        ColSums s;
        column_sums<M>(L, xg, gy, gz, s);
        const double ga = poly5(T, s.a), gb = poly5(T, s.b), gc = poly5(T, s.c);
        if (lane == 0) {
            hm_a = ga; hm_b = gb; hm_c = gc; fm_ax = s.ax; fm_by = s.by; fm_cz = s.cz;
        } else {
            hp_a = ga; hp_b = gb; hp_c = gc; fp_ax = s.ax; fp_by = s.by; fp_cz = s.cz;
        }
    }
    constexpr double w0 = 2.0 / 3.0, w1 = 1.0 / 6.0;
    acc[0] = 0.5 * (fp_ax - fm_ax);
    acc[1] = 0.5 * (w1 * fm_by + w0 * f0_by + w1 * fp_by);
    acc[2] = 0.5 * (w1 * fm_cz + w0 * f0_cz + w1 * fp_cz);
    acc[3] = 0.5 * (hp_a - hm_a);
    acc[4] = 0.5 * (w1 * hm_b + w0 * h0_b + w1 * hp_b);
    acc[5] = 0.5 * (w1 * hm_c + w0 * h0_c + w1 * hp_c);
}

// The gradients at `node`, lane `lane` of its tile: a tile inside one x-row
// (wave-uniform) passes column sums between its lanes.
template <int M>
__device__ __forceinline__ void tile_gradients(const LatDev& L, int node, int lane, double (&acc)[6]) {
    const int x0 = __builtin_amdgcn_readfirstlane((node - lane) % L.nx);
    if (x0 + NODE_TILE <= L.nx) row_tile_gradients<M>(L, node, lane, acc);
    else node_gradients<M>(L, node, acc);
}

// ---------------------------------------------------------------------------
// k_chem_implicit: for lattices with the linearly implicit reaction update,
// that increment (reading rho_a, rho, U, T from the per-node record and
// writing Delta rho_a into it), then the gradients.  The stencil's neighbour
// loads are latency-bound and the chemistry arithmetic-bound, so the two
// share one launch.  Holds an (M-1)^2 matrix in registers.  150x31x29, two
// sub-steps: 144 -> 140 us with this file's ln, exp and reciprocals in the rates
// and the pivots' reciprocals kept, 135 us with the derivatives of the factors a
// reaction has instead of all its slots.
// ---------------------------------------------------------------------------
static_assert(NODE_TILE == 64, "one wave per tile");
template <int M>
__global__ __launch_bounds__(NODE_TILE) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_chem_implicit(
    const LatDev* __restrict__ lats, const int* __restrict__ blk, int n_lat, const long long* __restrict__ tp, long long toff) {
    const long long t = step_time(tp, toff);
    const int b = xcd_block(), tid = (int)threadIdx.x;
    const int lj = find_lattice(blk, n_lat, b);
    const LatDev& L = lats[lj];
    if (t >= L.t_end || L.reaction != RLBM_REACTION_LINEARLY_IMPLICIT) return;
    const int node = (b - blk[lj]) * NODE_TILE + tid;
    if (node >= L.N) return;
    MechC mc = *as_const(L.mech);
    double* prm = L.prm;
    const size_t N = (size_t)L.N;
    // one row more than species: the unused factor slots name it (masked)
    __shared__ double s_c[M + 1][NODE_TILE], s_g[M + 1][NODE_TILE], s_q[M + 1][NODE_TILE];
    const ChemLds<NODE_TILE> ls{&s_c[0][tid], &s_g[0][tid], &s_q[0][tid]};
    s_c[M][tid] = 1.0;
    s_g[M][tid] = 0.0;
    s_q[M][tid] = 0.0;
    double rho_a[M], fin[M];
#pragma unroll
    for (int a = 0; a < M; ++a) rho_a[a] = prm[(PRM_SP + 6 * a) * N + node];
    // the density that normalises the composition (sum_a rho_a in the
    // weakly coupled storage)
    double rho = prm[PRM_RHO * N + node];
    if (L.weak) {
        rho = 0.0;
#pragma unroll
        for (int a = 0; a < M; ++a) rho += rho_a[a];
    }
    const double U = prm[PRM_UINT * N + node];
    const double T = prm[PRM_T * N + node];
    int fail = 0;
    reaction_increment<M, NODE_TILE>(mc, rho_a, rho, U, T, L.substeps, ls, fin, &fail);
    if (fail) atomicOr(L.flag, 1);
    // Delta rho_a against the densities read again, so that they need not
    // stay in registers through the sub-steps
    reload_barrier();
    if (L.storage == RLBM_STORAGE_F32_DEV) {
#pragma unroll
        for (int a = 0; a < M; ++a)
            st_corr<true>(as_global(prm), PRM_SP + 6 * a + 5, N, node, fin[a] - prm[(PRM_SP + 6 * a) * N + node]);
    } else {
#pragma unroll
        for (int a = 0; a < M; ++a)
            st_corr<false>(as_global(prm), PRM_SP + 6 * a + 5, N, node, fin[a] - prm[(PRM_SP + 6 * a) * N + node]);
    }
    double acc[6];
    tile_gradients<M>(L, node, tid, acc);
    store_gradients<M>(L, node, acc);
}

// ---------------------------------------------------------------------------
// k_update: the collision of every stored lattice (section 2.3 eq.
// finalNumericalEquationsReactive, section 3.2 eq. f, section 3.3 eq. g) of the
// lattices with the linearly implicit reaction update.
// A block of three waves covers 64 consecutive nodes; wave w takes the nine
// velocities with c_z = w - 1, one node per lane.  The per-node record is
// staged once in LDS with the species in slot order (the stored species in
// lattice order, then the slaved one), so every per-species quantity sits at
// a compile-time index.  Product-form factors along y and z are formed once
// per row of three velocities (fixed c_y, c_z); the x factor per velocity.
// ---------------------------------------------------------------------------
// Record rows k_update reads: rho, u, T, U (0..5), the energy-flux base
// (9..11), per species slot rho_a, V_a and Delta rho_a (c = 0..3, 5), and the
// six gradient rows.  theta, omega, the diffusion factor, omega - omega_1,
// (2 - omega_1) P / 2 and beta_a are derived in the kernel instead.
__host__ __device__ constexpr int upd_loaded_rows(int M) { return 9 + 5 * M + 6; }
__host__ __device__ constexpr int upd_loaded_row(int M, int idx) {
    return idx < 6 ? idx
                   : idx < 9 ? idx + 3
                             : idx < 9 + 5 * M ? PRM_SP + 6 * ((idx - 9) / 5) + ((idx - 9) % 5 < 4 ? (idx - 9) % 5 : 5)
                                               : prm_grad(M) + (idx - 9 - 5 * M);
}

constexpr int UPD_NODES = 64;
constexpr int UPD_WAVES = 3;
constexpr int UPD_THREADS = UPD_WAVES * UPD_NODES;

// Product-form factor with a compile-time velocity component C.
template <int C>
__device__ __forceinline__ double psi_c(double xi, double P) {
    if constexpr (C == 0) return 1.0 - P;
    else if constexpr (C > 0) return 0.5 * (P + xi);
    else return 0.5 * (P - xi);
}

// Product-form factor with a wave-uniform component c, as a + b xi + d P.
struct PsiCoef {
    double a, b, d;
};
__device__ __forceinline__ PsiCoef psi_coef(int c) {
    PsiCoef r;
    r.a = c == 0 ? 1.0 : 0.0;
    r.b = 0.5 * (double)c;
    r.d = c == 0 ? -1.0 : 0.5;
    return r;
}
__device__ __forceinline__ double psi_u(const PsiCoef& k, double xi, double P) {
    return fma(k.b, xi, fma(k.d, P, k.a));
}
// Energy-equilibrium axis factors (W, k) of eq. geq_i for a uniform c.
__device__ __forceinline__ void geq_wk(int c, double u, double th, double& W, double& k) {
    const double u2 = u * u;
    const double P = th + u2;
    const double o1 = th * u + 0.5 * u2 * u;
    const double o2 = th * th + 2.5 * th * u2 + 0.5 * u2 * u2;
    const PsiCoef pc = psi_coef(c);
    W = psi_u(pc, u, P);
    // k_0 = u^2/2 - o2, k_{+-1} = (o2 +- o1)/2
    k = c == 0 ? 0.5 * u2 - o2 : 0.5 * (o2 + (double)c * o1);
}


// The weakly coupled storage's extra lattice would otherwise take the
// kernel just past three waves per SIMD (the LDS allows three).
template <int M, typename S, int W>
__global__ __launch_bounds__(UPD_THREADS) __attribute__((amdgpu_waves_per_eu(W ? 3 : 1))) void k_update(const LatDev* __restrict__ lats, const int* __restrict__ blk,
                                                        int n_lat, const long long* __restrict__ tp, long long toff) {
    const long long t = step_time(tp, toff);
    constexpr int NR = prm_rows(M);
    constexpr int NSP = Lat<M, W>::NSP, LF = Lat<M, W>::LF, LG = Lat<M, W>::LG;
    constexpr int NL = Lat<M, W>::NL;   // stored lattices
    constexpr int NS = sizeof(S) == 4 ? NL : 1;
    __shared__ double sp[NR][UPD_NODES];
    __shared__ float ssc[NS][UPD_NODES];     // FP32 storage: this node's reference scales
    const int b = xcd_block();
    const int lj = find_lattice(blk, n_lat, b);
    const LatDev& L = lats[lj];
    if (t >= L.t_end || L.reaction == RLBM_REACTION_EXPLICIT) return;
    const int node0 = (b - blk[lj]) * UPD_NODES;
    const int lane = threadIdx.x % UPD_NODES;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / UPD_NODES);
    const int c2 = wave - 1;
    const int node = node0 + lane;
    const int N = (int)L.N;
    const bool valid = node < N;
    const int s = W ? M : L.slaved;
    const int par = (L.parity0 + t) & 1;
    const RLBM_GLOBAL S* src = as_global(static_cast<const S*>(L.pop[par]));
    RLBM_GLOBAL S* dst = as_global(static_cast<S*>(L.pop[par ^ 1]));
    const size_t P = (size_t)L.P;
    const RLBM_GLOBAL double* prm = as_global(L.prm);

    // stage the record's stored rows (species rows in slot order) and (FP32
    // storage) this node's reference scales: wave w takes stored rows w,
    // w + 3, ..., one node per lane; every load is in flight before the first
    // LDS write.  The rows derived below are not read.
    {
        constexpr int NLD = upd_loaded_rows(M);
        constexpr int RPW = (NLD + UPD_WAVES - 1) / UPD_WAVES;
        constexpr int LPW = (NS + UPD_WAVES - 1) / UPD_WAVES;
        const int nd = node0 + lane < N ? node0 + lane : 0;   // beyond the end: a placeholder node
        // one copy per wave, so that each load's row, and with it its width
        // (the correction rows are FP32 in FP32 storage), is a compile-time
        // constant: no branches between the loads
        auto stage = [&](auto wave_c) {
            constexpr int WV = decltype(wave_c)::value;
            double v[RPW];
            float vf[RPW];
            float w[LPW];
#pragma unroll
            for (int q = 0; q < RPW; ++q) {
                const int idx = WV + UPD_WAVES * q;
                const int row = upd_loaded_row(M, idx < NLD ? idx : 0);
                int srow = row;
                if (row >= PRM_SP && row < prm_grad(M)) {
                    const int slot = (row - PRM_SP) / 6, c = (row - PRM_SP) % 6;
                    const int a = W ? slot : (slot < M - 1 ? slot + (slot >= s ? 1 : 0) : s);
                    srow = PRM_SP + 6 * a + c;
                }
                // unconditional: no waits between
                if (sizeof(S) == 4 && prm_is_corr(M, row))
                    vf[q] = ld_at(reinterpret_cast<const RLBM_GLOBAL float*>(prm + (size_t)srow * L.N), nd);
                else
                    v[q] = ld_at(prm + (size_t)srow * L.N, nd);
            }
            if constexpr (sizeof(S) == 4) {
#pragma unroll
                for (int q = 0; q < LPW; ++q) {
                    const int l = WV + UPD_WAVES * q;
                    w[q] = scale_l(L, par, nd, l < NS ? l : 0, LF);
                }
            }
#pragma unroll
            for (int q = 0; q < RPW; ++q) {
                const int idx = WV + UPD_WAVES * q;
                if (idx < NLD) {
                    const int row = upd_loaded_row(M, idx);
                    sp[row][lane] = (sizeof(S) == 4 && prm_is_corr(M, row)) ? (double)vf[q] : v[q];
                }
            }
            if constexpr (sizeof(S) == 4) {
#pragma unroll
                for (int q = 0; q < LPW; ++q) {
                    const int l = WV + UPD_WAVES * q;
                    if (l < NS) ssc[l][lane] = w[q];
                }
            }
        };
        static_assert(UPD_WAVES == 3, "one staging copy per wave");
        if (wave == 0) stage(std::integral_constant<int, 0>{});
        else if (wave == 1) stage(std::integral_constant<int, 1>{});
        else stage(std::integral_constant<int, 2>{});
    }

    int x = 0, y = 0, z = 0;
    if (valid) { x = node % L.nx; const int r = node / L.nx; y = r % L.ny; z = r / L.ny; }
    const int k = (L.n_if && valid) ? as_global(L.if_index)[node] : -1;
    const bool wave_if = __builtin_amdgcn_ballot_w64(k >= 0) != 0;   // uniform
    PullOff o;
    pull_offsets(L, x, y, z, o);
    const int offz = node + sel3(c2, o.z[0], 0, o.z[2]);

    // populations of velocity i at node offset off (after advection and
    // boundary reconstruction: an interface lane reads the plane's interface
    // slot N + k)
    auto load = [&](int i, int off, S* out) {
        const int idx = wave_if && k >= 0 ? N + k : off;
#pragma unroll
        for (int l = 0; l < NL; ++l) out[l] = ld_at(src + (size_t)(l * Q + i) * P, idx);
    };
    // FP32 deviation storage: reference scales of this node (decode) and of
    // the node that reads what is written for velocity (c0, c1, c2) (encode)
    S fin[NL];
    const int i_first = 9 * (c2 + 1);
    if (valid) load(i_first, offz + o.y[0] + o.x[0], fin);
    __syncthreads();
    // the derived rows, once per node by the first wave: theta, the
    // relaxation rates (as k_local computes them) and beta_a =
    // 1/(2 tau_a + 1) with 1/tau_a = common sum_{b != a} K_ab Y_b (eqs.
    // betaa, taua), Y in slot order
    if (wave == 0) {
        MechC mc = *as_const(L.mech);
        const RLBM_CONST double* slotc = as_const(L.slotc);
        const double T = sp[PRM_T][lane], rho = sp[PRM_RHO][lane];
        double ry = rho;   // Y_a = rho_a / rho, or rho_a / sum_b rho_b (weakly coupled)
        if constexpr (W) {
            ry = 0.0;
#pragma unroll
            for (int q = 0; q < M; ++q) ry += sp[PRM_SP + 6 * q][lane];
        }
        const double iry = 1.0 / ry;
        double Y[M];
        double Rmix = 0.0;
#pragma unroll
        for (int q = 0; q < M; ++q) {
            Y[q] = sp[PRM_SP + 6 * q][lane] * iry;
            Rmix = fma(Y[q], slotc[q], Rmix);
        }
        const double th = Rmix * T, P = rho * th;
        double common, omega, omega1;
        relax_rates(mc, T, P, Rmix, common, omega, omega1);
        sp[PRM_TH][lane] = th;
        sp[PRM_OMEGA][lane] = omega;
        sp[PRM_COMMON][lane] = common;
        sp[PRM_WQ][lane] = omega - omega1;
        sp[PRM_CC][lane] = 0.5 * (2.0 - omega1) * P;
        const RLBM_CONST double* Ks = slotc + M;
#pragma unroll
        for (int j = 0; j < NSP; ++j) {
            double st = 0.0;
#pragma unroll
            for (int q = 0; q < M; ++q)
                if (q != j) st = fma(Ks[j * M + q], Y[q], st);
            const double inv_tau = common * st;
            sp[PRM_SP + 6 * j + 4][lane] = inv_tau / (2.0 + inv_tau);
        }
    }
    __syncthreads();
    if (!valid) return;

    const int GR = prm_grad(M);
    // per-node values used by every velocity are re-read from LDS where they
    // are needed; only the few derived ones stay in registers
    const double exf = [&] {
        const double w = sp[PRM_OMEGA][lane];
        return (2.0 - w) / (2.0 * sp[PRM_RHO][lane] * w);
    }();
    // F_ai = common Y_a sum_b K_ab D_bi with Y_a = rho_a / rho, or
    // rho_a / sum_b rho_b in the weakly coupled storage
    const double fcm = [&] {
        double ry = sp[PRM_RHO][lane];
        if constexpr (W) {
            ry = 0.0;
#pragma unroll
            for (int q = 0; q < M; ++q) ry += sp[PRM_SP + 6 * q][lane];
        }
        return sp[PRM_COMMON][lane] / ry;
    }();
    const PsiCoef pz = psi_coef(c2);

#pragma unroll 1
    for (int c1 = -1; c1 <= 1; ++c1) {
        reload_barrier();
        const RLBM_CONST double* Ra = as_const(L.slotc) + opaque_zero();   // [M] gas constants, slot order
        const PsiCoef py = psi_coef(c1);
        const int offyz = offz + sel3(c1, o.y[0], 0, o.y[2]);
        const double T = sp[PRM_T][lane], th = sp[PRM_TH][lane];
        const double uy = sp[PRM_U + 1][lane], uz = sp[PRM_U + 2][lane];
        // y/z factors of the species equilibria (xi = u) and quasi-equilibria
        // (xi = u + V_b, eq. xiPstar2)
        double YZe[M], YZs[M];
#pragma unroll
        for (int q = 0; q < M; ++q) {
            const double tq = Ra[q] * T;
            const double vy = uy + sp[PRM_SP + 6 * q + 2][lane], vz = uz + sp[PRM_SP + 6 * q + 3][lane];
            YZe[q] = psi_u(py, uy, fma(uy, uy, tq)) * psi_u(pz, uz, fma(uz, uz, tq));
            YZs[q] = psi_u(py, vy, fma(vy, vy, tq)) * psi_u(pz, vz, fma(vz, vz, tq));
        }
        // momentum lattice: y/z factors of the extended equilibrium (eq. Pex)
        const double Fyz = psi_u(py, uy, th + uy * uy + exf * sp[GR + 1][lane]) *
                           psi_u(pz, uz, th + uz * uz + exf * sp[GR + 2][lane]);
        // energy lattice: y/z factors of eq. geq_i
        double Wy, ky, Wz, kz;
        geq_wk(c1, uy, th, Wy, ky);
        geq_wk(c2, uz, th, Wz, kz);
        const double Wyz = Wy * Wz, kyz = ky * Wz + Wy * kz;
        const int cyz2 = c1 * c1 + c2 * c2;

        auto body = [&](auto c0t) {
            constexpr int c0 = decltype(c0t)::value;
            const int i = 9 * (c2 + 1) + 3 * (c1 + 1) + (c0 + 1);
            // per-velocity re-reads of LDS and constants (cheap) instead of
            // keeping them live across the three velocities
            reload_barrier();
            const RLBM_CONST double* slotc = as_const(L.slotc) + opaque_zero();
            const RLBM_CONST double* Ra = slotc;
            const RLBM_CONST double* Ks = slotc + M;
            const RLBM_CONST double* ref = as_const(L.ref) + opaque_zero();
            // scales of the node that reads what this velocity writes (L2 hits,
            // consumed after the species work below), issued before the
            // prefetch so that waiting for them leaves the prefetch in flight
            float srd[NS];
            if constexpr (sizeof(S) == 4) {
                const int rd = reader_at(node, o, c0, c1, c2);
                if constexpr (Lat<M, W>::ROW) species_scales<NL>(L, par ^ 1, rd, srd);
                else {
                    species_scales<NSP>(L, par ^ 1, rd, srd);
                    flow_scales(L, par ^ 1, rd, srd + NSP);
                }
            }
            // prefetch the next velocity of this thread
            S fnx[NL];
            if constexpr (c0 < 1) {
                load(i + 1, offyz + o.x[c0 + 2], fnx);
            } else {
                if (c1 < 1) load(i + 1, offyz + sel3(c1 + 1, o.y[0], 0, o.y[2]) - sel3(c1, o.y[0], 0, o.y[2]) + o.x[0], fnx);
            }
            const double T = sp[PRM_T][lane], ux = sp[PRM_U][lane];
            double D[M];
#pragma unroll
            for (int q = 0; q < M; ++q) {
                reload_barrier();   // keep each species' LDS reads next to their use
                const double tq = Ra[q] * T;
                const double vx = ux + sp[PRM_SP + 6 * q + 1][lane];
                const double Xe = psi_c<c0>(ux, fma(ux, ux, tq));
                const double Xs = psi_c<c0>(vx, fma(vx, vx, tq));
                D[q] = sp[PRM_SP + 6 * q][lane] * (Xe * YZe[q] - Xs * YZs[q]);
            }
            // species (eq. finalNumericalEquationsReactive with eq. fStar)
#pragma unroll
            for (int j = 0; j < NSP; ++j) {
                reload_barrier();
                double F = 0.0;
#pragma unroll
                for (int q = 0; q < M; ++q)
                    if (q != j) F = fma(Ks[j * M + q], D[q], F);
                const double ra = sp[PRM_SP + 6 * j][lane], be = sp[PRM_SP + 6 * j + 4][lane],
                             dr = sp[PRM_SP + 6 * j + 5][lane];
                const double Wj = psi_c<c0>(ux, fma(ux, ux, Ra[j] * T)) * YZe[j];   // W_ji, recomputed
                const int li = j * Q + i;
                double f = (double)fin[j];
                if constexpr (sizeof(S) == 4) f += ref_of(ssc[j][lane], ref[li]);
                const double out = f + 2.0 * be * (ra * Wj - f) + (be - 1.0) * (fcm * ra * F) + Wj * dr;
                if constexpr (sizeof(S) == 4)
                    st_at(dst + (size_t)li * P, node, __double2float_rn(out - ref_of(srd[j], ref[li])));
                else st_at(dst + (size_t)li * P, node, out);
            }
            const double rho = sp[PRM_RHO][lane], th = sp[PRM_TH][lane], omega = sp[PRM_OMEGA][lane];
            // momentum lattice, extended equilibrium (eqs. f, feqmix, Pex)
            {
                const int li = LF * Q + i;
                double f = (double)fin[LF];
                if constexpr (sizeof(S) == 4) f += ref_of(ssc[LF][lane], ref[li]);
                const double fe = rho * psi_c<c0>(ux, th + ux * ux + exf * sp[GR][lane]) * Fyz;
                const double out = f + omega * (fe - f);
                if constexpr (sizeof(S) == 4)
                    st_at(dst + (size_t)li * P, node, __double2float_rn(out - ref_of(srd[LF], ref[li])));
                else st_at(dst + (size_t)li * P, node, out);
            }
            // energy lattice (eqs. g, geq_i, gstar)
            {
                const int li = LG * Q + i;
                double g = (double)fin[LG];
                if constexpr (sizeof(S) == 4)
                    g += ref_g(ssc[LG][lane], ssc[LF][lane], ref[li], ref[REF_K<NL> + i]);
                const double ux2 = ux * ux;
                const double Wx = psi_c<c0>(ux, th + ux2);
                double kx;
                if constexpr (c0 == 0) {
                    kx = 0.5 * ux2 - (th * th + 2.5 * th * ux2 + 0.5 * ux2 * ux2);
                } else {
                    const double o1 = th * ux + 0.5 * ux2 * ux;
                    const double o2 = th * th + 2.5 * th * ux2 + 0.5 * ux2 * ux2;
                    kx = 0.5 * (o2 + (double)c0 * o1);
                }
                const double geq = rho * (Wyz * (sp[PRM_UINT][lane] * Wx + kx) + Wx * kyz);
                double out = g + omega * (geq - g);
                // the singularity-free flux term on the six |c| = 1 velocities
                const double wq = sp[PRM_WQ][lane], cc = sp[PRM_CC][lane];
                if constexpr (c0 != 0) {
                    if (cyz2 == 0)
                        out += 0.5 * (double)c0 *
                               (sp[PRM_QB][lane] - 0.5 * wq * ux * sp[GR][lane] + cc * sp[GR + 3][lane]);
                } else {
                    if (cyz2 == 1) {
                        const int ax = c1 != 0 ? 1 : 2;   // uniform
                        const double ua = sp[PRM_U + ax][lane];
                        const double Qa = sp[PRM_QB + ax][lane] - 0.5 * wq * ua * sp[GR + ax][lane] +
                                          cc * sp[GR + 3 + ax][lane];
                        out += 0.5 * (double)(c1 + c2) * Qa;
                    }
                }
                if constexpr (sizeof(S) == 4)
                    st_at(dst + (size_t)li * P, node,
                          __double2float_rn(out - ref_g(srd[LG], srd[LF], ref[li], ref[REF_K<NL> + i])));
                else st_at(dst + (size_t)li * P, node, out);
            }
#pragma unroll
            for (int l = 0; l < NL; ++l) fin[l] = fnx[l];
        };
        body(std::integral_constant<int, -1>{});
        body(std::integral_constant<int, 0>{});
        body(std::integral_constant<int, 1>{});
    }
}

// ---------------------------------------------------------------------------
// k_species: everything a node does with the species (sections 2.2, 2.3, 3.1,
// 3.5), in one pass over their populations.  A block takes 64 nodes with four
// waves.  Waves 0..2 hold one c_z layer each, nine velocities of every species
// lattice in registers, from the pull to the collision; the fourth wave reads
// the momentum and energy lattices (for their moments only) and solves the
// node: temperature, relaxation rates, Stefan-Maxwell system.  The reactions
// are dealt to the first three waves.
//   Bound: FP64 issue and its latency (two waves per SIMD; about 15,000 vector
// instructions per tile, which keep the SIMDs issuing 49% of the time at 2.4
// GHz) in FP32 storage, those and the traffic in FP64: 2.1 and 4.1 KB per node, against
// 4.0 and 7.5 for a moments pass and a collision that each read every
// population.  Three waves hold what one cannot, 216 registers of populations
// per node (FP32) beside the collision's working set, and they divide the
// node's serial chain, which is what a lattice too small to fill the chip
// waits for.  With k_flow against the passes it replaced (moments, gradients,
// collision of all lattices), 512x64x64: 1.65 + 0.36 against 0.93 + 0.18 + 1.28
// ms in FP32 storage, 2.00 + 0.50 against 1.19 + 0.18 + 2.00 in FP64; 1024
// nodes: 21 + 6 against 38 + 9 + 23 us.
//   Scalar loads return after about 200 cycles, more than the arithmetic of one
// species, and out of order, so a wait for one is a wait for all, LDS loads
// included: the rows of the collision and of the solve ask for the next
// species' constants once this one's have arrived, and the stores' operands
// come in one batch.  Each loaded where it is used: 1.79 and 2.05 ms.
//   The order of the barriers is the same on both sides of the role branch:
// partial sums written, partial sums read, node state, per sub-step
// (concentrations, rates), collision coefficients.
// ---------------------------------------------------------------------------
constexpr int SPC_NODES = 64;
constexpr int SPC_THREADS = 4 * SPC_NODES;

// Rows (64 doubles each) of the block's LDS.  Species quantities are in slot
// order (the stored species in lattice order, then the slaved one) except the
// chemistry's, which are in species order.
template <int M, int W>
struct SpcRows {
    static constexpr int NSP = Lat<M, W>::NSP;
    // slot q: 4 q + {0: rho_q, 1..3: j_q - rho_q u, then u + V_q}
    static constexpr int ST = 0;
    static constexpr int CG = 4 * M;                 // concentration and Gibbs function of species a: CG + 2 a, CG + 2 a + 1
    static constexpr int WD = CG + 2 * (M + 1);      // three waves' partial rates [3][M]
    static constexpr int U = WD + 3 * M, T = U + 3, RHO = U + 4, RHOY = U + 5, UINT = U + 6;
    static constexpr int A = U + 7, K = A + NSP;     // collision coefficients
    static constexpr int B = WD;                     // the last of them, once the chemistry is done
    // the fourth wave's own, during its solve: q - u.(P - P^eq) - rho u^2/2 u, theta, omega, omega_1
    static constexpr int AX = K + NSP;
    static constexpr int SC = AX + 6;                // FP32 storage: A times this node's scales
    // partial sums of lattice l, layer w: row PS + 9 l + 3 k + w, k = {zeroth, x, y}; read before the rows above are written
    static constexpr int PS = 0;
    static_assert(PS + 9 * NSP <= U, "the node's velocity is written beside the partial sums");
    static constexpr int N = SC + NSP;
};

// Interface slot of a node, or -1.  The index is loaded only by waves with a
// node on a non-periodic face (wave-uniform), so the loads of the others do
// not wait for it.
__device__ __forceinline__ int interface_slot(const LatDev& L, int node, int x, int y, int z) {
    const bool on = (!L.per[0] && (x == 0 || x == L.nx - 1)) || (!L.per[1] && (y == 0 || y == L.ny - 1)) ||
                    (!L.per[2] && (z == 0 || z == L.nz - 1));
    if (__builtin_amdgcn_ballot_w64(on) == 0) return -1;
    return as_global(L.if_index)[node];
}

// Has a scalar load and an LDS load, and all before them, waited for here: loads
// that follow then are on their way while what arrived is used.
__device__ __forceinline__ void arrived(double s, double v) { asm volatile("" : : "s"(s), "v"(v) : "memory"); }

// Waves 0..2: partial moments, reactions, collision.
template <int M, typename S, int W>
__device__ __forceinline__ void species_layer(const LatDev& L, int par, int layer, int lane, int node, bool valid,
                                              double (&sp)[SpcRows<M, W>::N][SPC_NODES]) {
    using R = SpcRows<M, W>;
    constexpr int NSP = Lat<M, W>::NSP, NL = Lat<M, W>::NL;
    constexpr bool F32 = sizeof(S) == 4;
    const int s = W ? M : L.slaved;
    const int c2 = layer - 1;
    const size_t N = (size_t)L.N, P = (size_t)L.P;
    const RLBM_GLOBAL S* src = as_global(static_cast<const S*>(L.pop[par]));
    RLBM_GLOBAL S* dst = as_global(static_cast<S*>(L.pop[par ^ 1]));
    MechC mc0 = *as_const(L.mech);
    const int x = node % L.nx, r = node / L.nx, y = r % L.ny, z = r / L.ny;
    PullOff o;
    pull_offsets(L, x, y, z, o);
    S raw[NSP][9];
    const unsigned nb = plane_bytes(L.P, sizeof(S));
    {
        const int k = interface_slot(L, node, x, y, z);
        const int nz = node + sel3(c2, o.z[0], 0, o.z[2]);
        int idx[9];
#pragma unroll
        for (int j = 0; j < 9; ++j) idx[j] = k >= 0 ? (int)N + k : nz + o.x[j % 3] + o.y[j / 3];
        const RLBM_GLOBAL S* win = src + (size_t)(9 * layer) * P;
#pragma unroll
        for (int l = 0; l < NSP; ++l) {
#pragma unroll
            for (int j = 0; j < 9; ++j) raw[l][j] = ld_win(win, nb, j, idx[j]);
            win += (size_t)Q * P;
            opaque(win);
        }
    }
#pragma unroll
    for (int l = 0; l < NSP; ++l) {
        double v[9];
#pragma unroll
        for (int j = 0; j < 9; ++j) v[j] = (double)raw[l][j];
        const double lo = v[0] + v[1] + v[2], mid = v[3] + v[4] + v[5], hi = v[6] + v[7] + v[8];
        double* ps = &sp[R::PS + 9 * l + layer][lane];
        ps[0] = lo + mid + hi;
        ps[3 * SPC_NODES] = (v[2] + v[5] + v[8]) - (v[0] + v[3] + v[6]);
        ps[6 * SPC_NODES] = hi - lo;
    }
    __syncthreads();   // partial sums
    // densities and j_a - rho_a u (eqs. density1, momentum1) of a third of the
    // species each, while the fourth wave solves for T
    {
        constexpr int NT = (NSP + 2) / 3;
        const double ux = sp[R::U][lane], uy = sp[R::U + 1][lane], uz = sp[R::U + 2][lane];
        double ra[NT], X[NT][3];
#pragma unroll
        for (int e = 0; e < NT; ++e) {
            const int l = 3 * e + layer;
            if (l < NSP) {
                const double* ps = &sp[R::PS + 9 * l][lane];
                const double m0 = ps[0], m1 = ps[SPC_NODES], m2 = ps[2 * SPC_NODES];
                ra[e] = m0 + m1 + m2;
                if constexpr (F32) ra[e] += (double)scale_at(L, par, node)[l] * as_const(L.ref)[REF_M0<NL> + l];
                X[e][0] = fma(-ra[e], ux, ps[3 * SPC_NODES] + ps[4 * SPC_NODES] + ps[5 * SPC_NODES]);
                X[e][1] = fma(-ra[e], uy, ps[6 * SPC_NODES] + ps[7 * SPC_NODES] + ps[8 * SPC_NODES]);
                X[e][2] = fma(-ra[e], uz, m2 - m0);
            }
        }
        __syncthreads();   // partial sums read
#pragma unroll
        for (int e = 0; e < NT; ++e) {
            const int l = 3 * e + layer;
            if (l < NSP) {
                sp[R::ST + 4 * l][lane] = ra[e];
#pragma unroll
                for (int d = 0; d < 3; ++d) sp[R::ST + 4 * l + 1 + d][lane] = X[e][d];
            }
        }
    }
    __syncthreads();   // node state

    // reaction increment (section 2.3, eq. R3): forward Euler sub-steps at
    // frozen U; every wave follows the densities, and takes a third of the
    // reactions and of the species' concentrations and Gibbs functions
    double cur[M];
#pragma unroll
    for (int a = 0; a < M; ++a) cur[a] = sp[R::ST + 4 * (W ? a : (a == s ? M - 1 : a - (a > s ? 1 : 0)))][lane];
    if (mc0.R > 0) {
        const double inv_rho = recip(sp[R::RHOY][lane]), U = sp[R::UINT][lane];
        double T = sp[R::T][lane];
        const double inv_l = 1.0 / (double)L.substeps;
        int fail = 0;
        for (int st = 0;; ++st) {
            reload_barrier();
            MechC mc = in_loop(mc0);
            const double lnT = ln(T), invT = recip(T);
#pragma unroll
            for (int a = 0; a < M; ++a)
                if (a % 3 == layer) {
                    sp[R::CG + 2 * a][lane] = fmax(cur[a], 0.0) * mc.inv_m[a];
                    sp[R::CG + 2 * a + 1][lane] = gibbs_RT(mc, a, T, lnT, invT);
                }
            if (layer == 0) {
                sp[R::CG + 2 * M][lane] = 1.0;
                sp[R::CG + 2 * M + 1][lane] = 0.0;
            }
            __syncthreads();   // concentrations
            double w[M];
#pragma unroll
            for (int a = 0; a < M; ++a) w[a] = 0.0;
            reaction_rates<M, SPC_NODES>(mc0, &sp[R::CG][lane], lnT, invT, layer, 3, w);
#pragma unroll
            for (int a = 0; a < M; ++a) sp[R::WD + layer * M + a][lane] = w[a];
            __syncthreads();   // rates
            if (st + 1 == L.substeps && layer != 0) break;
#pragma unroll
            for (int a = 0; a < M; ++a)
                cur[a] = fma(sp[R::WD + a][lane] + sp[R::WD + M + a][lane] + sp[R::WD + 2 * M + a][lane],
                             mc.m[a] * inv_l, cur[a]);
            if (st + 1 == L.substeps) break;
            double Y[M];
#pragma unroll
            for (int a = 0; a < M; ++a) Y[a] = cur[a] * inv_rho;
            T = solve_T<M>(mc, Y, U, T, &fail);
        }
        if (layer == 0 && fail && valid) atomicOr(L.flag, 1);
    } else {
        __syncthreads();   // concentrations
        __syncthreads();   // rates
    }
    if (layer == 0) {
        // half of 2 beta rho + Delta rho, with 2 beta = 1 - A
#pragma unroll
        for (int a = 0; a < M; ++a)
            if (W || a != s) {
                const int q = W ? a : a - (a > s ? 1 : 0);
                const double rq = sp[R::ST + 4 * q][lane];
                sp[R::B + q][lane] = 0.5 * fma(1.0 - sp[R::A + q][lane], rq, cur[a] - rq);
            }
    }
    if constexpr (F32) {
        if (layer == 2) {
            float sc[NSP];
            species_scales<NSP>(L, par, node, sc);
#pragma unroll
            for (int j = 0; j < NSP; ++j) sp[R::SC + j][lane] = sp[R::A + j][lane] * (double)sc[j];
        }
    }
    __syncthreads();   // collision coefficients
    if (!valid) return;

    // Collision, a row of three velocities (fixed c_y, c_z) at a time.  With
    // Psi_0 = 1 - P and Psi_{+-1} = (P +- xi)/2 a product form over the row is
    // given by z = Y Z, s = Y Z P_x and o = Y Z xi_x: its values are z - s and
    // (s +- o)/2.  The sums over the species are linear, so they run over
    // (z, s, o) of D_b = f_b^eq - f_b^* and the row is formed once per species:
    //   f' = A f + (2 beta rho + Delta rho) W + 2 K sum_b K_ab D_b,
    // A = 1 - 2 beta, 2 K = (beta - 1) common Y (eqs. betaa, taua).
    const double T = sp[R::T][lane];
    const double ux = sp[R::U][lane], uy = sp[R::U + 1][lane], uz = sp[R::U + 2][lane];
    const PsiCoef pz = psi_coef(c2);
    // one copy of the row's code (three would not fit the instruction cache
    // beside the rest): the next row's populations move down after each
    RLBM_GLOBAL S* win0 = dst + (size_t)(9 * layer) * P;
    unsigned off = (unsigned)node * (unsigned)sizeof(S);
    asm volatile("" : "+v"(off));   // a 32-bit offset, not folded into 64-bit addresses
    const RLBM_CONST double* ref0 = F32 ? as_const(L.ref) + REF_T<NL> + 9 * layer * NL : nullptr;
    const RLBM_CONST double* slot0 = as_const(L.slotc);   // not loaded again behind every barrier
#pragma unroll 1
    for (int c1 = -1; c1 <= 1; ++c1) {
        const PsiCoef py = psi_coef(c1);
        float rd[F32 ? 3 : 1][NSP];   // scales of the nodes that pull the row from here
        if constexpr (F32) {
#pragma unroll
            for (int c0 = 0; c0 < 3; ++c0) species_scales<NSP>(L, par ^ 1, reader_at(node, o, c0 - 1, c1, c2), rd[c0]);
        }
        double Fz[NSP], Fs[NSP], Fo[NSP], yz[NSP];
        // a species' constants and state are asked for one species ahead: the
        // wait for a scalar load is longer than a species' arithmetic
        double Kn[NSP], sn[4], Rn;
        auto ask = [&](int q) {
            const RLBM_CONST double* slotc = slot0 + opaque_zero();
#pragma unroll
            for (int j = 0; j < NSP; ++j) Kn[j] = slotc[M + q * M + j];   // symmetric
            Rn = slotc[q];
#pragma unroll
            for (int k = 0; k < 4; ++k) sn[k] = sp[R::ST + 4 * q + k][lane];
        };
        ask(0);
#pragma unroll
        for (int q = 0; q < M; ++q) {
            double Kq[NSP];
            arrived(Kn[0], sn[0]);
#pragma unroll
            for (int j = 0; j < NSP; ++j) Kq[j] = Kn[j];
            const double rq = sn[0], vx = sn[1], vy = sn[2], vz = sn[3], tq = Rn * T;
            if (q + 1 < M) ask(q + 1);
            reload_barrier();
            const double e = psi_u(py, uy, fma(uy, uy, tq)) * psi_u(pz, uz, fma(uz, uz, tq));
            const double v = psi_u(py, vy, fma(vy, vy, tq)) * psi_u(pz, vz, fma(vz, vz, tq));
            if (q < NSP) yz[q] = e;
            const double re = rq * e, rv = rq * v;
            const double dz = re - rv;
            const double ds = fma(re, fma(ux, ux, tq), -(rv * fma(vx, vx, tq)));
            const double d_o = fma(re, ux, -(rv * vx));
#pragma unroll
            for (int j = 0; j < NSP; ++j)
                if (j != q) {
                    const bool first = q == 0 || (q == 1 && j == 0);
                    Fz[j] = first ? Kq[j] * dz : fma(Kq[j], dz, Fz[j]);
                    Fs[j] = first ? Kq[j] * ds : fma(Kq[j], ds, Fs[j]);
                    Fo[j] = first ? Kq[j] * d_o : fma(Kq[j], d_o, Fo[j]);
                }
        }
        reload_barrier();
        // the row's values without the old populations, in place: Fz = the
        // value at c_x = 0, (Fs, Fo) = those at c_x = -1, +1
#pragma unroll
        for (int j0 = 0; j0 < NSP; j0 += 4) {
            double K[4], B[4], Rj[4];
            const RLBM_CONST double* slotc = slot0 + opaque_zero();
#pragma unroll
            for (int e = 0; e < 4 && j0 + e < NSP; ++e) {
                K[e] = sp[R::K + j0 + e][lane];
                B[e] = sp[R::B + j0 + e][lane];
                Rj[e] = slotc[j0 + e];
            }
            reload_barrier();
#pragma unroll
            for (int e = 0; e < 4 && j0 + e < NSP; ++e) {
                const int j = j0 + e;
                const double g = B[e] * yz[j];
                const double hs = fma(K[e], Fs[j], g * fma(ux, ux, Rj[e] * T));
                const double ho = fma(K[e], Fo[j], g * ux);
                Fz[j] = 2.0 * (fma(K[e], Fz[j], g) - hs);
                Fs[j] = hs - ho;
                Fo[j] = hs + ho;
            }
        }
        double A[NSP], SC[F32 ? NSP : 1], G[F32 ? 3 : 1][NSP];
        if constexpr (F32) {
            const RLBM_CONST double* g = ref0 + opaque_zero();
#pragma unroll
            for (int c0 = 0; c0 < 3; ++c0)
#pragma unroll
                for (int j = 0; j < NSP; ++j) G[c0][j] = g[c0 * NL + j];
        }
#pragma unroll
        for (int j = 0; j < NSP; ++j) {
            A[j] = sp[R::A + j][lane];
            if constexpr (F32) SC[j] = sp[R::SC + j][lane];
        }
        reload_barrier();
        auto put = [&](auto c0t, const double (&eq)[NSP]) {
            constexpr int c0 = decltype(c0t)::value;
            const float(&srd)[NSP] = rd[F32 ? c0 + 1 : 0];
            RLBM_GLOBAL S* win = win0 + (size_t)(c0 + 1) * P;
#pragma unroll
            for (int j = 0; j < NSP; ++j) {
                const double f = (double)raw[j][c0 + 1];
                opaque(win);
                if constexpr (F32)
                    // A (f + s G) + eq - s_reader G
                    st_off(win, off, __double2float_rn(fma(A[j], f, fma(SC[j] - (double)srd[j], G[c0 + 1][j], eq[j]))));
                else
                    st_off(win, off, fma(A[j], f, eq[j]));
                win += (size_t)Q * P;
            }
        };
        put(std::integral_constant<int, -1>{}, Fs);
        put(std::integral_constant<int, 0>{}, Fz);
        put(std::integral_constant<int, 1>{}, Fo);
        win0 += 3 * P;
        if constexpr (F32) ref0 += 3 * NL;
#pragma unroll
        for (int j = 0; j < NSP; ++j)
#pragma unroll
            for (int k = 0; k < 6; ++k) raw[j][k] = raw[j][k + 3];
    }
}

// The rest of the fourth wave's work, after its solve: the energy flux, the
// neighbour-facing fields (Phi and the enthalpy moments for the gradient
// stencil, T for the next step's Newton start; rho, u and Y only where an
// outlet reads them, at the first interior node of the x+ face) and k_flow's
// record.  flux = sum_a H_a Y_a V_a.
template <int M, typename S, int W>
__device__ __forceinline__ void write_record(const LatDev& L, int lane, int node, int x, bool valid, const double (&Y)[M],
                                             const double (&flux)[3], const double (&sp)[SpcRows<M, W>::N][SPC_NODES]) {
    using R = SpcRows<M, W>;
    if (!valid) return;
    reload_barrier();
    const int s = W ? M : L.slaved;
    const size_t N = (size_t)L.N;
    RLBM_GLOBAL double* prm = as_global(L.prm);
    RLBM_GLOBAL double* aux = as_global(L.aux);
    MechC mc = in_loop(*as_const(L.mech));
    auto sp_of = [&](int q) { return W ? q : (q < M - 1 ? q + (q >= s ? 1 : 0) : s); };
    const double u[3] = {sp[R::U][lane], sp[R::U + 1][lane], sp[R::U + 2][lane]};
    const double T = sp[R::T][lane], rho = sp[R::RHO][lane], U = sp[R::UINT][lane];
    const double th = sp[R::AX + 3][lane], omega = sp[R::AX + 4][lane], omega1 = sp[R::AX + 5][lane];
    // enthalpy-weighted composition moments sum_a H_a(T') Y_a = sum_kk T'^kk Pk
    double Pk[6];
#pragma unroll
    for (int kk = 0; kk < 6; ++kk) Pk[kk] = 0.0;
#pragma unroll
    for (int sl = 0; sl < M; ++sl) {
        const RLBM_CONST double* h = mc.hc[sp_of(sl)];
#pragma unroll
        for (int kk = 0; kk < 6; ++kk) Pk[kk] = fma(h[kk], Y[sl], Pk[kk]);
    }
    // local part of the energy flux, Qb = (omega - omega1)(q - u.(P - P^eq) - q^eq),
    // with the diffusion term omega1 rho sum_a H_a Y_a V_a
    const double hr = rho * poly5(T, Pk);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const double Qb = (omega - omega1) * fma(-hr, u[a], sp[R::AX + a][lane]);
        st_corr<sizeof(S) == 4>(prm, PRM_QB + a, N, node, fma(omega1 * rho, flux[a], Qb));
    }
#pragma unroll
    for (int d = 0; d < 3; ++d)
        st_at(aux + (AUX_PHI + d) * N, node, rho * u[d] * (1.0 - 3.0 * th) - rho * u[d] * u[d] * u[d]);
    st_at(aux + AUX_T * N, node, T);
#pragma unroll
    for (int kk = 0; kk < 6; ++kk) st_at(aux + (AUX_Y + M + kk) * N, node, Pk[kk]);
    if (L.n_out > 0 && x == L.nx - 2) {
        st_at(aux + AUX_RHO * N, node, rho);
#pragma unroll
        for (int d = 0; d < 3; ++d) st_at(aux + (AUX_U + d) * N, node, u[d]);
#pragma unroll
        for (int sl = 0; sl < M; ++sl) st_at(aux + (size_t)(AUX_Y + sp_of(sl)) * N, node, Y[sl]);
    }
    st_at(prm + PRM_RHO * N, node, rho);
#pragma unroll
    for (int d = 0; d < 3; ++d) st_at(prm + (PRM_U + d) * N, node, u[d]);
    st_at(prm + PRM_UINT * N, node, U);
    st_at(prm + PRM_TH * N, node, th);
    st_at(prm + PRM_OMEGA * N, node, omega);
    st_at(prm + PRM_OMEGA1 * N, node, omega1);
}

// Wave 3: the momentum and energy lattices' moments and the node's solve.
template <int M, typename S, int W>
__device__ __forceinline__ void node_solve(const LatDev& L, int par, int lane, int node, bool valid,
                                           double (&sp)[SpcRows<M, W>::N][SPC_NODES]) {
    using R = SpcRows<M, W>;
    constexpr int NSP = Lat<M, W>::NSP, LF = Lat<M, W>::LF, LG = Lat<M, W>::LG, NL = Lat<M, W>::NL;
    constexpr bool F32 = sizeof(S) == 4;
    const int s = W ? M : L.slaved;
    const size_t N = (size_t)L.N, P = (size_t)L.P;
    const RLBM_GLOBAL S* src = as_global(static_cast<const S*>(L.pop[par]));
    RLBM_GLOBAL double* prm = as_global(L.prm);
    RLBM_GLOBAL double* aux = as_global(L.aux);
    MechC mc0 = *as_const(L.mech);
    const RLBM_CONST double* slotc = as_const(L.slotc);
    const int x = node % L.nx, r = node / L.nx, y = r % L.ny, z = r / L.ny;
    auto sp_of = [&](int q) { return W ? q : (q < M - 1 ? q + (q >= s ? 1 : 0) : s); };
    double rho = 0.0, rhoE = 0.0, j[3] = {0.0, 0.0, 0.0}, q[3] = {0.0, 0.0, 0.0};
    double Pd[3] = {0.0, 0.0, 0.0}, Po[3] = {0.0, 0.0, 0.0};
    float fs[2] = {0.0f, 0.0f}, sc[NSP];
    double T_prev;
    {
        PullOff o;
        pull_offsets(L, x, y, z, o);
        const int k = interface_slot(L, node, x, y, z);
        const unsigned nb = plane_bytes(L.P, sizeof(S));
        S f[Q], g[Q];
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            const int idx = k >= 0 ? (int)N + k : node + o.x[cx_of(i) + 1] + o.y[cy_of(i) + 1] + o.z[cz_of(i) + 1];
            f[i] = ld_win(src + (size_t)(LF * Q + 9 * (i / 9)) * P, nb, i % 9, idx);
            g[i] = ld_win(src + (size_t)(LG * Q + 9 * (i / 9)) * P, nb, i % 9, idx);
        }
        if constexpr (F32) {
            flow_scales(L, par, node, fs);
            species_scales<NSP>(L, par, node, sc);
        }
        T_prev = ld_at(aux + AUX_T * N, node);
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            const int cx = cx_of(i), cy = cy_of(i), cz = cz_of(i);
            const double a = (double)f[i], b = (double)g[i];
            rho += a;
            rhoE += b;
            if (cx) { j[0] += cx > 0 ? a : -a; Pd[0] += a; q[0] += cx > 0 ? b : -b; }
            if (cy) { j[1] += cy > 0 ? a : -a; Pd[1] += a; q[1] += cy > 0 ? b : -b; }
            if (cz) { j[2] += cz > 0 ? a : -a; Pd[2] += a; q[2] += cz > 0 ? b : -b; }
            if (cx * cy) Po[0] += cx * cy > 0 ? a : -a;
            if (cx * cz) Po[1] += cx * cz > 0 ? a : -a;
            if (cy * cz) Po[2] += cy * cz > 0 ? a : -a;
        }
    }
    if constexpr (F32) {
        const RLBM_CONST double* G = as_const(L.ref);
        const double sf = (double)fs[0];
        rho += sf * G[REF_M0<NL> + LF];
        rhoE += (double)fs[1] * G[REF_M0<NL> + LG] + sf * G[REF_K0<NL>];
        const double p2 = sf * G[REF_M2<NL>];
        Pd[0] += p2; Pd[1] += p2; Pd[2] += p2;
        if (valid) store_fscale(L, par ^ 1, node, rho, rhoE);
    }
    const double inv_rho = recip(rho);
    const double u[3] = {j[0] * inv_rho, j[1] * inv_rho, j[2] * inv_rho};
#pragma unroll
    for (int d = 0; d < 3; ++d) sp[R::U + d][lane] = u[d];
    sp[R::RHO][lane] = rho;
    __syncthreads();   // partial sums

    // composition (eq. density1; the slaved species by difference, eq.
    // strongest) and temperature (eq. temperature; Newton from the previous
    // step's value)
    double Y[M], rY = 0.0;
    {
        double rs = rho;
#pragma unroll
        for (int l = 0; l < NSP; ++l) {
            const double* ps = &sp[R::PS + 9 * l][lane];
            double ra = ps[0] + ps[SPC_NODES] + ps[2 * SPC_NODES];
            if constexpr (F32) ra += (double)sc[l] * as_const(L.ref)[REF_M0<NL> + l];
            Y[l] = ra;
            rY += ra;
            rs -= ra;
        }
        if constexpr (!W) Y[M - 1] = rs;
    }
    __syncthreads();   // partial sums read
    if constexpr (!W) {
        sp[R::ST + 4 * (M - 1)][lane] = Y[M - 1];
        rY = rho;
    }
    const double inv_rY = W ? recip(rY) : inv_rho;
#pragma unroll
    for (int sl = 0; sl < M; ++sl) Y[sl] *= inv_rY;
    const double usq = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
    const double U = rhoE * inv_rho - 0.5 * usq;
    int fail = 0;
    const double T = solve_T<M>(mc0, sp_of, Y, U, T_prev, &fail);
    if (fail && valid) atomicOr(L.flag, 1);
    sp[R::T][lane] = T;
    sp[R::RHOY][lane] = rY;
    sp[R::UINT][lane] = U;
    __syncthreads();   // node state

    // relaxation rates
    double Rmix = 0.0;
#pragma unroll
    for (int sl = 0; sl < M; ++sl) Rmix = fma(Y[sl], slotc[sl], Rmix);
    const double th = Rmix * T, Pr = rho * th;
    double common, omega, omega1;
    relax_rates(mc0, T, Pr, Rmix, common, omega, omega1);
    // what only the energy flux and the record need waits in LDS while the
    // solve takes the registers
    {
        const double Pt[3][3] = {{Pd[0], Po[0], Po[1]}, {Po[0], Pd[1], Po[2]}, {Po[1], Po[2], Pd[2]}};
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            double uP = 0.5 * rho * usq * u[a];
#pragma unroll
            for (int c = 0; c < 3; ++c) uP += u[c] * (Pt[c][a] - rho * ((a == c ? th : 0.0) + u[c] * u[a]));
            sp[R::AX + a][lane] = q[a] - uP;
        }
    }
    sp[R::AX + 3][lane] = th;
    sp[R::AX + 4][lane] = omega;
    sp[R::AX + 5][lane] = omega1;

    __syncthreads();   // concentrations

    // Stefan-Maxwell system (section 2.3, eq. transform1; dt = 1)
    //   (1 + 1/(2 tau_a)) V_a - 1/2 sum_{b != a} Y_b V_b / tau_ab = u_a - u,
    // 1/tau_ab = common K_ab, for the three components.  Off the diagonal the
    // matrix is -m_ab Y_b with m symmetric, and elimination keeps that form
    // (m_ij += m_ik m_kj Y_k / d_k), so only the upper triangle of m is formed:
    // half the products of a general elimination and no division by Y.  The
    // matrix is strictly row diagonally dominant with margin 1, so no pivoting.
    double flux[3] = {0.0, 0.0, 0.0};   // sum_a H_a Y_a V_a
    {
        const RLBM_CONST double* Ks = slotc + M;
        const double h = 0.5 * common;
        double m[M][M], t[M], idg[M], V[M][3];   // m: upper triangle; t = Y_k / d_k
        double js[3] = {0.0, 0.0, 0.0};
        double Kn[M], sn[4] = {0.0, 0.0, 0.0, 0.0};   // the next row's couplings and state, asked for one row ahead
        auto ask = [&](int i) {
            const RLBM_CONST double* k = Ks + i * M + opaque_zero();
#pragma unroll
            for (int c = 0; c < M; ++c) Kn[c] = k[c];
#pragma unroll
            for (int k4 = 0; k4 < (W || i < M - 1 ? 4 : 1); ++k4) sn[k4] = sp[R::ST + 4 * i + k4][lane];
        };
        ask(0);
#pragma unroll
        for (int i = 0; i < M; ++i) {
            arrived(Kn[0], sn[0]);
            double Ki[M];
#pragma unroll
            for (int c = 0; c < M; ++c) Ki[c] = Kn[c];
            const double ra = sn[0], X3[3] = {sn[1], sn[2], sn[3]};
            if (i + 1 < M) ask(i + 1);
            reload_barrier();
            double dg = 0.0;
#pragma unroll
            for (int c = 0; c < M; ++c)
                if (c != i) dg = fma(Ki[c], Y[c], dg);
            dg = fma(h, dg, 1.0);   // 1 + 1/(2 tau_i)
            if (i < NSP) {
                // the collision's coefficients, with beta = 1 / (2 tau + 1) = 1 - 1 / dg
                const double b1 = recip(dg);   // 1 - beta
                sp[R::A + i][lane] = fma(2.0, b1, -1.0);
                sp[R::K + i][lane] = -0.5 * b1 * (common * Y[i]);
            }
#pragma unroll
            for (int c = i + 1; c < M; ++c) m[i][c] = h * Ki[c];
            // u_a - u (u_a := u for an absent species); the slaved one's from
            // sum_a (j_a - rho_a u) = 0 (eq. strongest)
            const double inv = ra <= 1e-14 * rho ? 0.0 : recip(ra);
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                double X;
                if (W || i < M - 1) {
                    X = X3[d];
                    js[d] -= X;
                } else {
                    X = js[d];
                }
                V[i][d] = X * inv;
            }
#pragma unroll
            for (int k = 0; k < i; ++k) {
                const double e = m[k][i] * t[k];
                dg = fma(-e * m[k][i], Y[i], dg);
#pragma unroll
                for (int c = i + 1; c < M; ++c) m[i][c] = fma(e, m[k][c], m[i][c]);
#pragma unroll
                for (int d = 0; d < 3; ++d) V[i][d] = fma(e, V[k][d], V[i][d]);
            }
            idg[i] = recip(dg);
            t[i] = Y[i] * idg[i];
        }
        const double u3[3] = {sp[R::U][lane], sp[R::U + 1][lane], sp[R::U + 2][lane]};
#pragma unroll
        for (int i = M - 1; i >= 0; --i) {
            reload_barrier();
            MechC mc = in_loop(mc0);
            const double hy = species_U(mc, sp_of(i), T) + slotc[i] * T;   // H_a
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                double v = V[i][d];
#pragma unroll
                for (int c = i + 1; c < M; ++c) v = fma(m[i][c], V[c][d], v);   // V_c holds Y_c V_c here
                v *= idg[i];
                sp[R::ST + 4 * i + 1 + d][lane] = u3[d] + v;
                V[i][d] = Y[i] * v;
                flux[d] = fma(hy, V[i][d], flux[d]);
            }
        }
    }
    __syncthreads();   // rates
    write_record<M, S, W>(L, lane, node, x, valid, Y, flux, sp);
    if (mc0.R > 0) {
        for (int st = 1; st < L.substeps; ++st) {
            __syncthreads();
            __syncthreads();
        }
    }
    __syncthreads();   // collision coefficients (the node's scales have been read)
    if constexpr (F32) {
        if (!valid) return;
        typedef float f4 __attribute__((ext_vector_type(4)));
        RLBM_GLOBAL f4* so = reinterpret_cast<RLBM_GLOBAL f4*>(as_global(L.rscale[par]) + (size_t)node * L.rss);
#pragma unroll
        for (int v = 0; v < (NSP + 3) / 4; ++v) {
            f4 w = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (4 * v + e < NSP) w[e] = __double2float_rn(sp[R::ST + 4 * (4 * v + e)][lane]);
            so[v] = w;
        }
    }
}

template <int M, typename S, int W>
__global__ __launch_bounds__(SPC_THREADS) __attribute__((amdgpu_waves_per_eu(2))) void k_species(
    const LatDev* __restrict__ lats, const int* __restrict__ blk, int n_lat, const long long* __restrict__ tp, long long toff) {
    __shared__ double sp[SpcRows<M, W>::N][SPC_NODES];
    const long long t = step_time(tp, toff);
    const int b = xcd_block();
    const int lj = find_lattice(blk, n_lat, b);
    const LatDev& L = lats[lj];
    if (t >= L.t_end || L.reaction != RLBM_REACTION_EXPLICIT) return;   // the whole block
    const int lane = (int)threadIdx.x % SPC_NODES;
    // the roles rotate with the block, so that the lighter fourth one does not
    // always fall to the same SIMD
    const int role = (__builtin_amdgcn_readfirstlane((int)threadIdx.x / SPC_NODES) + (int)blockIdx.x) & 3;
    const int n = (b - blk[lj]) * SPC_NODES + lane;
    const bool valid = n < (int)L.N;
    const int node = valid ? n : (int)L.N - 1;   // beyond the end: a placeholder that writes nothing
    const int par = (int)((L.parity0 + t) & 1);
    if (role == 3) node_solve<M, S, W>(L, par, lane, node, valid, sp);
    else species_layer<M, S, W>(L, par, role, lane, node, valid, sp);
}

// ---------------------------------------------------------------------------
// k_flow: the same-time gradients, then the collisions of the momentum and the
// energy lattice (section 3.2 eq. f, section 3.3 eq. g).  Three waves per 64
// nodes, one c_z layer each: a wave's share of the stencil is the layer's nine
// neighbours, the partial gradients meet in LDS, then it collides the layer's
// nine velocities.  Populations and the readers' scales are asked for ahead of
// the barrier.  Bound by its traffic on large lattices (54 populations in and
// out, the record, nine fields for the stencil: 512x64x64 moves 1.3 GB in FP32
// storage, 0.35 ms) and by one tile's latency on small ones.  Against one wave
// per 64 nodes: 1024 nodes 14.4 -> 6.3 us, 203x53x37 (weak coupling) 105 -> 88,
// 512x64x64 419 -> 354 (FP32) and 530 -> 493 (FP64).  Three waves per SIMD: at
// four the registers spill (423 and 582 us at 512x64x64 without the early
// scales).
// ---------------------------------------------------------------------------
constexpr int FLOW_THREADS = 3 * NODE_TILE;

// What this wave's lanes wrote to LDS before is seen by all of them after.  A
// wave's LDS operations run in order, so this costs no instruction; it keeps
// the compiler from moving one lane's reads above another's writes.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Sums over c_y of one column of a layer: the enthalpy coefficients and
// Phi_x, Phi_z with the weights w(c_y), and the coefficients and Phi_y with
// c_y.
struct LayerCol {
    double a[6], b[6], ax, by, az;
};
__device__ __forceinline__ void layer_sums_y(const double (&v)[3][9], LayerCol& o) {
    constexpr double w0 = 2.0 / 3.0, w1 = 1.0 / 6.0;
    auto even = [&](int k) { return fma(w1, v[0][k] + v[2][k], w0 * v[1][k]); };
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        o.a[k] = even(k);
        o.b[k] = v[2][k] - v[0][k];
    }
    o.ax = even(6);
    o.by = v[2][7] - v[0][7];
    o.az = even(8);
}
template <int M>
__device__ __forceinline__ void layer_column(const RLBM_GLOBAL double* aux, size_t N, int nx, int zr, const int (&gy)[3],
                                             int xc, LayerCol& o) {
    double v[3][9];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        const int nb = (zr + gy[j]) * nx + xc;
#pragma unroll
        for (int k = 0; k < 6; ++k) v[j][k] = ld_at(aux + (AUX_Y + M + k) * N, nb);
#pragma unroll
        for (int k = 0; k < 3; ++k) v[j][6 + k] = ld_at(aux + (AUX_PHI + k) * N, nb);
    }
    layer_sums_y(v, o);
}

// One layer's part of the gradients (see the factored weights above
// column_sums): d_x and d_z from the even sums A, d_y from the odd ones B.
// A tile inside one x-row (wave-uniform, all its nodes exist) takes the
// columns beside its own from the adjacent lanes, which evaluate them at this
// lane's temperature, and the two columns beyond the tile with one load of
// 54 lanes (nine fields, three y, two sides) through LDS: loads by the first
// and the last lane alone would double the stencil's load instructions, and
// those bound the kernel.  Other tiles load all three columns.
constexpr int EDGE = 27;   // values of one column of a layer
template <int M>
__device__ __forceinline__ void layer_gradients(const LatDev& L, int n0, int lane, int x, int y, int z, int node, int c2,
                                                double (&edges)[2 * EDGE], double (&part)[6]) {
    const int nx = L.nx, ny = L.ny, nz = L.nz;
    const size_t N = (size_t)L.N;
    const RLBM_GLOBAL double* aux = as_global(L.aux);
    const bool px = L.per[0], py = L.per[1], pz = L.per[2];
    const int gy[3] = {y == 0 ? (py ? ny - 1 : 0) : y - 1, y, y == ny - 1 ? (py ? 0 : y) : y + 1};
    const int zc = c2 < 0 ? (z == 0 ? (pz ? nz - 1 : 0) : z - 1) : (c2 > 0 ? (z == nz - 1 ? (pz ? 0 : z) : z + 1) : z);
    const int xm = x == 0 ? (px ? nx - 1 : 0) : x - 1, xp = x == nx - 1 ? (px ? 0 : x) : x + 1;
    const int zr = zc * ny;
    const double T = ld_at(aux + AUX_T * N, node);
    constexpr double w0 = 2.0 / 3.0, w1 = 1.0 / 6.0;
    const double hz = c2 ? 0.5 * w1 : 0.5 * w0, hc = 0.5 * (double)c2;
    struct Column {   // the sums at a lane's temperature
        double A, B, ax, by, az;
    };
    auto at = [](double t, const LayerCol& s) { return Column{poly5(t, s.a), poly5(t, s.b), s.ax, s.by, s.az}; };
    // column x + c
    auto add = [&](int c, const Column& v) {
        const double w = c ? w1 : w0;
        if (c) {
            part[0] = c < 0 ? -v.ax : part[0] + v.ax;
            part[3] = c < 0 ? -v.A : part[3] + v.A;
        }
        part[1] = c < 0 ? w * v.by : fma(w, v.by, part[1]);
        part[2] = c < 0 ? w * v.az : fma(w, v.az, part[2]);
        part[4] = c < 0 ? w * v.B : fma(w, v.B, part[4]);
        part[5] = c < 0 ? w * v.A : fma(w, v.A, part[5]);
    };
    if (n0 % nx + NODE_TILE <= nx) {
        double outer = 0.0;
        {
            const int side = lane >= EDGE ? 1 : 0, q = lane - side * EDGE, j = q / 9, k = q - 9 * j;
            const int x0 = n0 % nx, x1 = x0 + NODE_TILE - 1;
            const int xg = side ? (x1 == nx - 1 ? (px ? 0 : x1) : x1 + 1) : (x0 == 0 ? (px ? nx - 1 : 0) : x0 - 1);
            if (lane < 2 * EDGE)
                outer = aux[(k < 6 ? AUX_Y + M + k : AUX_PHI + k - 6) * N + (size_t)((zr + sel3(j - 1, gy[0], gy[1], gy[2])) * nx + xg)];
        }
        LayerCol s;
        layer_column<M>(aux, N, nx, zr, gy, x, s);
        // written only now, so that the wait below leaves the columns' loads in flight
        if (lane < 2 * EDGE) edges[lane] = outer;
        wave_sync();
        Column edge = {0.0, 0.0, 0.0, 0.0, 0.0};
        if (lane == 0 || lane == NODE_TILE - 1) {
            const double* from = &edges[lane == 0 ? 0 : EDGE];
            LayerCol g;
            constexpr double w0 = 2.0 / 3.0, w1 = 1.0 / 6.0;
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                const double* e = from + 9 * j;
                const double w = j == 1 ? w0 : w1;
#pragma unroll
                for (int k = 0; k < 6; ++k) {
                    g.a[k] = j ? fma(w, e[k], g.a[k]) : w * e[k];
                    g.b[k] = j == 2 ? g.b[k] + e[k] : (j ? g.b[k] : -e[k]);
                }
                g.ax = j ? fma(w, e[6], g.ax) : w * e[6];
                g.by = j == 2 ? g.by + e[7] : (j ? g.by : -e[7]);
                g.az = j ? fma(w, e[8], g.az) : w * e[8];
                reload_barrier();
            }
            edge = at(T, g);
        }
        Column v = at(__shfl_down(T, 1u), s);
        auto pass = [&](int c, double e, double w) {   // from lane - 1 or lane + 1, or the column beyond the tile
            const double r = c < 0 ? __shfl_up(w, 1u) : __shfl_down(w, 1u);
            return (c < 0 ? lane == 0 : lane == NODE_TILE - 1) ? e : r;
        };
        add(-1, Column{pass(-1, edge.A, v.A), pass(-1, edge.B, v.B), pass(-1, edge.ax, v.ax), pass(-1, edge.by, v.by),
                       pass(-1, edge.az, v.az)});
        add(0, at(T, s));
        v = at(__shfl_up(T, 1u), s);
        add(1, Column{pass(1, edge.A, v.A), pass(1, edge.B, v.B), pass(1, edge.ax, v.ax), pass(1, edge.by, v.by),
                      pass(1, edge.az, v.az)});
    } else {
#pragma unroll
        for (int c = -1; c <= 1; ++c) {
            reload_barrier();   // one column's loads at a time
            LayerCol s;
            layer_column<M>(aux, N, nx, zr, gy, c < 0 ? xm : (c > 0 ? xp : x), s);
            add(c, at(T, s));
        }
    }
    part[0] *= hz;
    part[1] *= hz;
    part[2] *= hc;
    part[3] *= hz;
    part[4] *= hz;
    part[5] *= hc;
}

// The tile that takes the place `q` of a lattice's order.  Whole planes in
// order have each XCD fetch the stencil's nine fields once per c_z once three
// planes exceed its L2; strips of 64 tiles (0.9 MB for three planes), all z of
// a strip after another, keep them there: 512x64x64 437 -> 419 us (FP32), 562
// -> 547 us (FP64).  Planes that are no whole number of tiles stay in order.
__device__ __forceinline__ int strip_tile(const LatDev& L, int q) {
    constexpr int SW = 64;
    const int plane = L.nx * L.ny, tp = plane / NODE_TILE;
    if (plane % NODE_TILE || tp <= SW || L.nz == 1) return q;
    const int s = q / (SW * L.nz), r = q - s * SW * L.nz;
    const int w = min(SW, tp - s * SW), z = r / w;
    return z * tp + s * SW + (r - z * w);
}

template <int M, typename S, int W>
__global__ __launch_bounds__(FLOW_THREADS) __attribute__((amdgpu_waves_per_eu(3))) void k_flow(const LatDev* __restrict__ lats, const int* __restrict__ blk, int n_lat,
                                                       const long long* __restrict__ tp, long long toff) {
    constexpr int LF = Lat<M, W>::LF, LG = Lat<M, W>::LG, NL = Lat<M, W>::NL;
    constexpr bool F32 = sizeof(S) == 4;
    __shared__ double part[3][6][NODE_TILE], edges[3][2 * EDGE];
    // k_flow's record, a third of its rows loaded by each wave
    enum { R_RHO, R_U = 1, R_UINT = 4, R_TH, R_OMEGA, R_OMEGA1, R_QB, R_N = 11 };
    __shared__ double rec[R_N][NODE_TILE];
    const long long t = step_time(tp, toff);
    const int b = xcd_block();
    const int lj = find_lattice(blk, n_lat, b);
    const LatDev& L = lats[lj];
    if (t >= L.t_end || L.reaction != RLBM_REACTION_EXPLICIT) return;   // the whole block
    const int lane = (int)threadIdx.x % NODE_TILE;
    const int layer = __builtin_amdgcn_readfirstlane((int)threadIdx.x / NODE_TILE), c2 = layer - 1;
    const int n0 = strip_tile(L, b - blk[lj]) * NODE_TILE;
    const bool valid = n0 + lane < (int)L.N;
    const int node = valid ? n0 + lane : (int)L.N - 1;   // beyond the end: a placeholder that writes nothing
    const size_t N = (size_t)L.N, P = (size_t)L.P;
    const int par = (int)((L.parity0 + t) & 1);
    const RLBM_GLOBAL S* src = as_global(static_cast<const S*>(L.pop[par]));
    RLBM_GLOBAL S* dst = as_global(static_cast<S*>(L.pop[par ^ 1]));
    const RLBM_GLOBAL double* prm = as_global(L.prm);
    const int x = node % L.nx, r = node / L.nx, y = r % L.ny, z = r / L.ny;
    PullOff o;
    pull_offsets(L, x, y, z, o);
    S fi[9], gi[9];
    {
        const int k = interface_slot(L, node, x, y, z);
        const unsigned nb = plane_bytes(L.P, sizeof(S));
        const int nz = node + sel3(c2, o.z[0], 0, o.z[2]);
#pragma unroll
        for (int j = 0; j < 9; ++j) {
            const int idx = k >= 0 ? (int)N + k : nz + o.x[j % 3] + o.y[j / 3];
            fi[j] = ld_win(src + (size_t)(LF * Q + 9 * layer) * P, nb, j, idx);
            gi[j] = ld_win(src + (size_t)(LG * Q + 9 * layer) * P, nb, j, idx);
        }
    }
    float fs[2] = {0.0f, 0.0f};
    if constexpr (F32) flow_scales(L, par, node, fs);
    double row[4];
    if (layer == 0) {
        row[0] = ld_at(prm + PRM_RHO * N, node);
#pragma unroll
        for (int d = 0; d < 3; ++d) row[1 + d] = ld_at(prm + (PRM_U + d) * N, node);
    } else if (layer == 1) {
        row[0] = ld_at(prm + PRM_UINT * N, node);
        row[1] = ld_at(prm + PRM_TH * N, node);
        row[2] = ld_at(prm + PRM_OMEGA * N, node);
        row[3] = ld_at(prm + PRM_OMEGA1 * N, node);
    } else {
#pragma unroll
        for (int d = 0; d < 3; ++d) row[d] = ld_corr<F32>(prm, PRM_QB + d, N, node);
        row[3] = 0.0;
    }
    double gr[6];
    layer_gradients<M>(L, n0, lane, x, y, z, node, c2, edges[layer], gr);
#pragma unroll
    for (int k = 0; k < 4; ++k)
        if (4 * layer + k < R_N) rec[4 * layer + k][lane] = row[k];
#pragma unroll
    for (int k = 0; k < 6; ++k) part[layer][k][lane] = gr[k];
    // the scales of the nodes that pull from here
    float srd[9][2];
    if constexpr (F32) {
#pragma unroll
        for (int j = 0; j < 9; ++j) flow_scales(L, par ^ 1, reader_at(node, o, j % 3 - 1, j / 3 - 1, c2), srd[j]);
    }
    __syncthreads();
    if (!valid) return;
    const double rho = rec[R_RHO][lane], U = rec[R_UINT][lane], th = rec[R_TH][lane];
    const double omega = rec[R_OMEGA][lane], omega1 = rec[R_OMEGA1][lane];
    double u[3], Qb[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        u[d] = rec[R_U + d][lane];
        Qb[d] = rec[R_QB + d][lane];
    }
#pragma unroll
    for (int k = 0; k < 6; ++k) gr[k] = part[0][k][lane] + part[1][k][lane] + part[2][k][lane];

    const double exf = (2.0 - omega) / (2.0 * rho * omega);
    const double cc = 0.5 * (2.0 - omega1) * (rho * th), wq = 0.5 * (omega - omega1);
    double E[3][3], Wa[3][3], ka[3][3];   // per axis and c + 1: eq. Pex, eq. geq_i
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        Qb[d] = 0.5 * (Qb[d] - wq * u[d] * gr[d] + cc * gr[3 + d]);
        const double P0 = fma(u[d], u[d], th), Px = fma(exf, gr[d], P0);
        E[d][0] = 0.5 * (Px - u[d]);
        E[d][1] = 1.0 - Px;
        E[d][2] = 0.5 * (Px + u[d]);
        GeqAxis g;
        geq_axis(u[d], th, g);
#pragma unroll
        for (int c = 0; c < 3; ++c) { Wa[d][c] = g.W[c]; ka[d][c] = g.k[c]; }
    }
    const double Ez = rho * sel3d(c2, E[2][0], E[2][1], E[2][2]);
    const double Wz = sel3d(c2, Wa[2][0], Wa[2][1], Wa[2][2]), kz = sel3d(c2, ka[2][0], ka[2][1], ka[2][2]);
#pragma unroll
    for (int c1 = 0; c1 < 3; ++c1) {
        const double Eyz = Ez * E[1][c1], Wyz = Wa[1][c1] * Wz, kyz = ka[1][c1] * Wz + Wa[1][c1] * kz;
#pragma unroll
        for (int c0 = 0; c0 < 3; ++c0) {
            const int j = 3 * c1 + c0, i = 9 * layer + j;
            double f = (double)fi[j], g = (double)gi[j];
            const RLBM_CONST double* ref = as_const(L.ref) + opaque_zero();
            if constexpr (F32) {
                f += ref_of(fs[0], ref[LF * Q + i]);
                g += ref_g(fs[1], fs[0], ref[LG * Q + i], ref[REF_K<NL> + i]);
            }
            const double fo = f + omega * (E[0][c0] * Eyz - f);
            const double geq = rho * (Wyz * (U * Wa[0][c0] + ka[0][c0]) + Wa[0][c0] * kyz);
            double go = g + omega * (geq - g);
            // the singularity-free flux term on the six |c| = 1 velocities
            if (c0 == 1 && c1 == 1) {
                if (c2 != 0) go += c2 > 0 ? Qb[2] : -Qb[2];
            } else if ((c0 == 1 || c1 == 1) && c2 == 0) {
                const double q = c0 != 1 ? Qb[0] : Qb[1];
                go += c0 + c1 > 2 ? q : -q;
            }
            if constexpr (F32) {
                st_at(dst + (size_t)(LF * Q + i) * P, node, __double2float_rn(fo - ref_of(srd[j][0], ref[LF * Q + i])));
                st_at(dst + (size_t)(LG * Q + i) * P, node,
                      __double2float_rn(go - ref_g(srd[j][1], srd[j][0], ref[LG * Q + i], ref[REF_K<NL> + i])));
            } else {
                st_at(dst + (size_t)(LF * Q + i) * P, node, fo);
                st_at(dst + (size_t)(LG * Q + i) * P, node, go);
            }
        }
    }
}

// ---------------------------------------------------------------------------
// k_boundary: reconstruction at interface nodes (section 4).  A block takes
// up to 64 consecutive entries of the interface list (grouped by boundary type
// and ordered by node within a type, so mostly a run of a wall row or plane),
// one lane per node, and one wave per stored lattice (the energy lattice's
// layers are dealt to two or three): every population load
// and store of a wave is coalesced and its lattice, with the lattice's
// constants, is the same for the whole wave.  Each wave loads its lattice's
// populations once, in one pass with all 27 loads in flight, and keeps them
// in LDS for the moments and the reconstruction (the pull reads of the
// interface list are scattered over the lattice, so a second pass over them
// costs as much as the first); lattices beyond what the LDS holds beside the
// node states read them again per pass.  The output goes to the interface
// slots N + k of the planes of the buffer the step reads.  The node's state
// goes between the waves through LDS: the lattices' moments, and the imposed
// and local states that the first wave forms from them (temperature by the
// bounded Newton iteration, the LODI outlet state).  All barriers are at the
// top level of the kernel, so every wave meets all of them.
//   Two passes walk the three layers of nine velocities in a loop: unrolled over
// all 27 velocities the kernel was 75 KB of code (FP32 storage), more than the
// instruction cache, and a launch with few blocks spent its time fetching it.
//   Bound by latency: four dependent phases of one block per CU, and for inlet
// and outlet planes by the cache lines their scattered nodes touch (see the
// block rule in the host library).  Unrolled with 64-node blocks throughout
// against this form: two nodes of a 1024-node tube 35 -> 20 us, a 1024x64
// channel in FP64 storage 48 -> 23 us, 512x64x64 285 -> 224 us (FP32) and 250
// -> 227 us (FP64).
// ---------------------------------------------------------------------------
static_assert(BC_NODES == 64, "one lane per node in a wave");

// An equilibrium of one lattice, s (U Wx Wy Wz + kx Wy Wz + Wx (ky Wz + Wy kz)),
// with W the product-form factors of the axes.  The species and momentum
// lattices have U = 1 and k = 0; the energy lattice has the factors of eq.
// geq_i (section 3.3) and U the internal energy.  The x and y factors are kept
// for c + 1; layer() forms the z factors of c_z (wave-uniform), s included.
struct LatEq {
    double s, U, th, uz;
    double Wx[3], kx[3], Wy[3], ky[3];
    double Wz, kz;
    __device__ __forceinline__ void layer(bool energy, int c2) {
        if (energy) {
            geq_wk(c2, uz, th, Wz, kz);
            Wz *= s;
            kz *= s;
        } else {
            Wz = s * psi_u(psi_coef(c2), uz, fma(uz, uz, th));
        }
    }
    // values at c_x + 1 = 0, 1, 2 of the layer's row c_y + 1 = j
    __device__ __forceinline__ void row(bool energy, int j, double (&v)[3]) const {
        const double w = Wy[j] * Wz;
        if (energy) {
            const double q = fma(ky[j], Wz, Wy[j] * kz);
#pragma unroll
            for (int c = 0; c < 3; ++c) v[c] = fma(w, fma(U, Wx[c], kx[c]), Wx[c] * q);
        } else {
#pragma unroll
            for (int c = 0; c < 3; ++c) v[c] = w * Wx[c];
        }
    }
};

// Node state of an equilibrium (sections 4.1-4.4), one LDS column per node:
// density, temperature, mixture theta, internal energy, velocity, mass
// fractions.
constexpr int ST_RHO = 0, ST_T = 1, ST_TH = 2, ST_U = 3, ST_V = 4, ST_Y = 7;

template <int M>
__device__ __forceinline__ void state_store(MechC mc0, double (*st)[BC_NODES], int lane, double rho, const double* u,
                                            const double* Y, double T) {
    reload_barrier();
    MechC mc = in_loop(mc0);
    st[ST_RHO][lane] = rho;
    st[ST_T][lane] = T;
    st[ST_TH][lane] = mc.R_univ * mix_inv_m<M>(mc, Y) * T;
    st[ST_U][lane] = mix_U<M>(mc, Y, T);
#pragma unroll
    for (int d = 0; d < 3; ++d) st[ST_V + d][lane] = u[d];
#pragma unroll
    for (int c = 0; c < M; ++c) st[ST_Y + c][lane] = Y[c];
}

// Equilibrium of stored lattice l (the wave's) for the density and composition
// in column `lane` of st and the given T, theta, U and velocity.
template <int M, int W>
__device__ __forceinline__ void lat_prepare(MechC mc0, const double (*st)[BC_NODES], int lane, int l, int slaved, double T,
                                            double thm, double U, double u0, double u1, double u2, LatEq& q) {
    constexpr int LF = Lat<M, W>::LF, LG = Lat<M, W>::LG;
    reload_barrier();
    MechC mc = in_loop(mc0);
    const bool sp = l < LF;
    const int a = sp ? (W ? l : l + (l >= slaved ? 1 : 0)) : 0;
    const double rho = st[ST_RHO][lane];
    q.th = sp ? mc.Ra[a] * T : thm;
    q.s = sp ? rho * st[ST_Y + a][lane] : rho;
    q.U = l == LG ? U : 1.0;
    q.uz = u2;
    GeqAxis gx, gy;
    geq_axis(u0, q.th, gx);
    geq_axis(u1, q.th, gy);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        q.Wx[c] = gx.W[c];
        q.kx[c] = gx.k[c];
        q.Wy[c] = gy.W[c];
        q.ky[c] = gy.k[c];
    }
}

// Compile-time loop over the 27 velocities.
template <int I, typename F>
__device__ __forceinline__ void for_q(F&& f) {
    if constexpr (I < Q) {
        f(std::integral_constant<int, I>{});
        for_q<I + 1>(f);
    }
}

// Waves that share the energy lattice, whose equilibrium is the dearest: three
// (one c_z layer each) where a block then still has at most twelve waves, the
// most that leaves each 168 registers, else two.
template <int M, int W>
constexpr int bc_energy_waves() { return Lat<M, W>::NL + 2 <= 12 ? 3 : 2; }
template <int M, int W>
constexpr int bc_threads() { return BC_NODES * (Lat<M, W>::NL - 1 + bc_energy_waves<M, W>()); }

// How many of a block's lattices keep their advected populations (27 * 64
// stored values each) in LDS beside the node states and moments, within the
// 160 KB of LDS per CU on gfx950.
template <int M, typename S, int W>
constexpr int bc_stash() {
    constexpr int NL = Lat<M, W>::NL;
    constexpr long state = (long)(NL * 4 + 2 * (ST_Y + M) + 2) * BC_NODES * (long)sizeof(double) + BC_NODES * 4L;
    constexpr long n = (160L * 1024 - state) / ((long)Q * BC_NODES * (long)sizeof(S));
    return n < 0 ? 0 : (n < NL ? (int)n : NL);
}

template <int M, typename S, int W>
__global__ __launch_bounds__((bc_threads<M, W>())) void k_boundary(
    const LatDev* __restrict__ lats, const int* __restrict__ blk, int n_lat, const long long* __restrict__ tp,
    long long toff) {
    constexpr int LF = Lat<M, W>::LF, LG = Lat<M, W>::LG, NL = Lat<M, W>::NL;
    constexpr bool F32 = sizeof(S) == 4;
    __shared__ double mom[NL][4][BC_NODES];             // moments per lattice and node
    __shared__ double stA[ST_Y + M][BC_NODES];          // imposed state
    __shared__ double stL[ST_Y + M][BC_NODES];          // local state
    __shared__ double stT[2][BC_NODES];                 // theta and U of the full inlet's target
    __shared__ int flg[BC_NODES];
    // the advected populations of the first NS lattices as stored, loaded
    // once and read by all passes (NS = NL where they fit beside the state;
    // one block per CU runs anyway, as the kernel's registers allow no second
    // one)
    constexpr int NS = bc_stash<M, S, W>();
    __shared__ S stash[NS > 0 ? NS : 1][Q][BC_NODES];
    const long long t = step_time(tp, toff);
    // tiles in reverse list order, without the XCD remap: the list is sorted
    // by boundary type and starts with the TMS walls (the cheapest entries),
    // so the costlier inlet, outlet and bounce-back tiles start first and
    // wall tiles fill the tail; and consecutive tiles go to different XCDs,
    // so every XCD gets a share of each kind (L2 sharing between neighbouring
    // tiles matters little here)
    const int b = (int)(gridDim.x - 1 - blockIdx.x);
    const int lj = find_lattice(blk, n_lat, b);
    const LatDev& L = lats[lj];
    if (t >= L.t_end) return;                       // the whole block
    const int lane = (int)threadIdx.x % BC_NODES;
    constexpr int EW = bc_energy_waves<M, W>();
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / BC_NODES);
    const int l = wave < LG ? wave : LG;            // this wave's lattice
    const int ew = wave - l;                        // and its share of the c_z layers
    const int lay0 = l < LG ? 0 : (EW == 3 ? ew : 2 * ew), lay1 = l < LG ? 3 : (EW == 3 ? ew + 1 : 2 + ew);
    // the block's run of the interface list
    const int k0 = as_global(L.if_blk)[b - blk[lj]], k1 = as_global(L.if_blk)[b - blk[lj] + 1];
    const int k = k0 + lane;
    const bool live = k < k1;
    const int kk = live ? k : k0;                   // lanes past the end mirror the first node and write nothing
    MechC mc0 = *as_const(L.mech);
    const int par = (L.parity0 + t) & 1;
    const RLBM_GLOBAL S* src = as_global(static_cast<const S*>(L.pop[par]));
    // the output: interface slot N + k of every plane of the same buffer,
    // disjoint from the node slots the pull reads
    RLBM_GLOBAL S* bc = as_global(static_cast<S*>(L.pop[par])) + L.N;
    const size_t N = (size_t)L.N;
    const size_t P = (size_t)L.P;
    const int node = as_global(L.if_node)[kk];
    const unsigned Dm = as_global(L.if_mask)[kk];
    const int type = as_global(L.if_type)[kk];
    const int s = W ? M : L.slaved;
    const int x = node % L.nx, r = node / L.nx, y = r % L.ny, z = r / L.ny;
    PullOff o;
    pull_offsets(L, x, y, z, o);
    const bool wall = type == RLBM_FACE_WALL;
    const bool bback = type == RLBM_FACE_BOUNCEBACK;
    const bool outlet = type == RLBM_FACE_OUTLET;
    const bool inlet_full = type == RLBM_FACE_INLET;
    const bool energy = l == LG;
    const RLBM_CONST double* G = as_const(L.ref);
    if (l == 0) flg[lane] = 0;

    // FP32 deviation storage: references belong to the node that reads a
    // value, this node for an advected value and for what is written to the
    // interface slots, the pull source x - c_i (wrapped) for a bounce-back
    // source f'_{opp(i)}(x)
    float sl = 0.0f, sf = 0.0f;
    // this wave's lattice' scale of node n: sbase[n * sstep]
    const RLBM_GLOBAL float* sbase = nullptr;
    int sstep = 0;
    if constexpr (F32) {
        sbase = l < LF ? as_global(L.rscale[par]) + l : as_global(L.fscale[par]) + (l - LF);
        sstep = l < LF ? L.rss : L.fss;
        sl = sbase[(size_t)node * sstep];
        sf = fscale_at(L, par, node)[0];
    }
    auto ref = [&](int i, float sc, float scf) -> double {   // reference of (l, i) with the given scales
        if constexpr (!F32) return 0.0;
        else if (energy) return ref_g(sc, scf, G[LG * Q + i], G[REF_K<NL> + i]);
        else return ref_of(sc, G[l * Q + i]);
    };
    const bool stashed = NS == NL || l < NS;   // wave-uniform
    // the advected population (l, i) as stored, i uniform
    auto adv = [&](int i, int c0, int c1, int c2) -> double {
        if (NS > 0 && stashed) return (double)stash[NS > 0 ? l : 0][i][lane];
        const int off = node + sel3(c0, o.x[0], 0, o.x[2]) + sel3(c1, o.y[0], 0, o.y[2]) + sel3(c2, o.z[0], 0, o.z[2]);
        return (double)ld_at(src + (size_t)(l * Q + i) * P, off);
    };

    // step 1: one pass of loads, all in flight together: the advected
    // populations of outgoing links and, at a bounce-back wall (section 4.2.1,
    // eq. bb; every lattice) or a TMS wall (section 4.2.2; species and
    // momentum), the bounce-back sources of incoming ones; any other incoming
    // link loads the plane's first value, a stand-in that no pass reads (the
    // same cache line for every lane: the nodes of an inlet or outlet plane
    // have a line each)
    const bool bbs = bback || (wall && l <= LF);
    {
        S raw[Q];
        for_q<0>([&](auto ic) {
            constexpr int i = decltype(ic)::value, io = Q - 1 - i;
            constexpr int c0 = cx_of(i), c1 = cy_of(i), c2 = cz_of(i);
            raw[i] = S(0);
            if (i / 9 < lay0 || i / 9 >= lay1) return;   // wave-uniform
            const bool in = (Dm >> i) & 1u;
            const int off = node + sel3(c0, o.x[0], 0, o.x[2]) + sel3(c1, o.y[0], 0, o.y[2]) + sel3(c2, o.z[0], 0, o.z[2]);
            raw[i] = ld_at(src + (size_t)(l * Q + i) * P + (bbs && in ? (long long)(io - i) * (long long)P : 0LL),
                           in ? (bbs ? node : 0) : off);
        });
        // the sources, decoded: their sum gives the TMS wall's bounce-back
        // densities (eqs. BBrho, BBY); a bounce-back wall's output is them
        if (__builtin_amdgcn_ballot_w64(bbs) != 0) {
            float sb[F32 ? Q : 1], sbf[F32 ? Q : 1];
            if constexpr (F32) {
                auto readers = [&](float own, const RLBM_GLOBAL float* base, int step, float* out) {
                    for_q<0>([&](auto ic) {
                        constexpr int i = decltype(ic)::value;
                        constexpr int c0 = cx_of(i), c1 = cy_of(i), c2 = cz_of(i);
                        const int off = node + sel3(c0, o.x[0], 0, o.x[2]) + sel3(c1, o.y[0], 0, o.y[2]) +
                                        sel3(c2, o.z[0], 0, o.z[2]);
                        out[i] = own;
                        if (bbs && ((Dm >> i) & 1u)) out[i] = base[(size_t)off * step];
                    });
                };
                readers(sl, sbase, sstep, sb);
                if (energy) readers(sf, as_global(L.fscale[par]), L.fss, sbf);
            }
            double m0 = 0.0;
            for_q<0>([&](auto ic) {
                constexpr int i = decltype(ic)::value, io = Q - 1 - i;
                double v = (double)raw[i];
                if constexpr (F32) {
                    const bool in = (Dm >> i) & 1u;
                    v += in ? ref(io, sb[i], sbf[i]) : ref(i, sl, sf);
                    if (bback && in) raw[i] = __double2float_rn(v - ref(i, sl, sf));
                }
                m0 += v;
            });
            if (wall && l <= LF) mom[l][0][lane] = m0;
        }
        if (NS > 0 && stashed) {
            for_q<0>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                if (i / 9 < lay0 || i / 9 >= lay1) return;
                stash[NS > 0 ? l : 0][i][lane] = raw[i];
            });
        }
        if (bback && live) {
            for_q<0>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                if (i / 9 < lay0 || i / 9 >= lay1) return;
                st_at(bc + (size_t)(l * Q + i) * P, k, raw[i]);
            });
        }
    }
    __syncthreads();
    // step 2: the imposed state, formed by the first wave: the TMS target
    // (u = 0, T_w(x)), the LODI outlet state (section 4.4, from the previous
    // outlet state and the previous post-boundary moments of the first
    // interior node), or the inlet equilibrium (section 4.3, eqs. in_f, in_g,
    // in_fa)
    if (l == 0 && !bback) {
        double Y[M], u[3] = {0.0, 0.0, 0.0}, rho, T;
        if (wall) {
            double rs = 0.0;
            const double rb = mom[LF][0][lane];
#pragma unroll
            for (int c = 0; c < M; ++c) {
                const bool slv = !W && c == s;
                const double v = slv ? 0.0 : mom[slv ? 0 : (W ? c : c - (c > s ? 1 : 0))][0][lane];
                Y[c] = v;
                rs += v;
            }
            if constexpr (!W) {
#pragma unroll
                for (int c = 0; c < M; ++c)
                    if (c == s) Y[c] = rb - rs;
            }
            const double iry = 1.0 / (W ? rs : rb);   // the weakly coupled storage normalises Y by sum_a rho_a
#pragma unroll
            for (int c = 0; c < M; ++c) Y[c] *= iry;
            rho = rb;
            T = L.if_T[kk];
        } else if (outlet) {
            reload_barrier();
            MechC mc = in_loop(mc0);
            const int ko = L.if_out[kk];
            const size_t No = (size_t)L.n_out;
            double* os = L.out_state;
            const double rho0 = os[0 * No + ko];
            const double u0[3] = {os[1 * No + ko], os[2 * No + ko], os[3 * No + ko]};
            const double T0 = os[4 * No + ko];
            double Y0[M], Y1[M];
            const size_t inn = (size_t)node - 1;
#pragma unroll
            for (int c = 0; c < M; ++c) {
                Y0[c] = os[(5 + c) * No + ko];
                Y1[c] = L.aux[(AUX_Y + c) * N + inn];
            }
            const double rho1 = L.aux[AUX_RHO * N + inn];
            const double u1[3] = {L.aux[(AUX_U + 0) * N + inn], L.aux[(AUX_U + 1) * N + inn],
                                  L.aux[(AUX_U + 2) * N + inn]};
            const double T1 = L.aux[AUX_T * N + inn];
            const double R0 = mc.R_univ * mix_inv_m<M>(mc, Y0);
            const double P0 = rho0 * R0 * T0;
            const double P1 = rho1 * mc.R_univ * mix_inv_m<M>(mc, Y1) * T1;
            double Cv = 0.0;
#pragma unroll
            for (int c = 0; c < M; ++c) Cv += Y0[c] * species_cv(mc, c, T0);
            const double gam = (Cv + R0) / Cv;
            const double cs = sqrt(gam * P0 / rho0);
            const double un = u0[0];
            const double Ma = un / cs;
            const double L1 = L.sigma * (1.0 - Ma * Ma) * cs / (double)L.nx * (P0 - L.P_inf);
            const double L2 = un * (cs * cs * (rho0 - rho1) - (P0 - P1));
            const double L3 = un * (u0[1] - u1[1]);
            const double L4 = un * (u0[2] - u1[2]);
            const double L5 = (un + cs) * ((P0 - P1) + rho0 * cs * (u0[0] - u1[0]));
            rho = rho0 - (L2 + 0.5 * (L5 + L1)) / (cs * cs);
            const double P_o = P0 - 0.5 * (L5 + L1);
            u[0] = un - (L5 - L1) / (2.0 * rho0 * cs);
            u[1] = u0[1] - L3;
            u[2] = u0[2] - L4;
#pragma unroll
            for (int c = 0; c < M; ++c) Y[c] = Y0[c] - un * (Y0[c] - Y1[c]);   // eq. convectiveBC
            T = P_o / (rho * mc.R_univ * mix_inv_m<M>(mc, Y));
            if (live) {
                os[0 * No + ko] = rho;
                os[1 * No + ko] = u[0]; os[2 * No + ko] = u[1]; os[3 * No + ko] = u[2];
                os[4 * No + ko] = T;
#pragma unroll
                for (int c = 0; c < M; ++c) os[(5 + c) * No + ko] = Y[c];
            }
        } else {
            rho = L.rho_in;
            u[0] = L.u_in;
#pragma unroll
            for (int c = 0; c < M; ++c) Y[c] = L.Y_in[c];
            T = L.T_in;
        }
        state_store<M>(mc0, stA, lane, rho, u, Y, T);
    }
    __syncthreads();
    // step 3: moments of the mixed set, incoming links at the imposed
    // equilibria and outgoing ones advected (eqs. locRho .. locT and their
    // inlet and outlet counterparts)
    LatEq eA;
    if (!bback) {
        lat_prepare<M, W>(mc0, stA, lane, l, s, stA[ST_T][lane], stA[ST_TH][lane], stA[ST_U][lane], stA[ST_V][lane],
                          stA[ST_V + 1][lane], stA[ST_V + 2][lane], eA);
        double m0 = 0.0, m1 = 0.0, m2 = 0.0, m3 = 0.0;
#pragma unroll 1
        for (int lay = lay0; lay < lay1; ++lay) {
            const int c2 = lay - 1, i0 = 9 * lay;
            const unsigned in = Dm >> i0;
            eA.layer(energy, c2);
            double f[9], sum = 0.0;
#pragma unroll
            for (int j = 0; j < 9; ++j) f[j] = adv(i0 + j, j % 3 - 1, j / 3 - 1, c2) + ref(i0 + j, sl, sf);
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                double v[3];
                eA.row(energy, j, v);
#pragma unroll
                for (int c = 0; c < 3; ++c) v[c] = (in >> (3 * j + c)) & 1u ? v[c] : f[3 * j + c];
                const double rs = v[0] + v[1] + v[2];
                sum += rs;
                m1 += v[2] - v[0];
                if (j != 1) m2 += j ? rs : -rs;
            }
            m0 += sum;
            m3 = fma((double)c2, sum, m3);
        }
        if (energy) {
            mom[LG][ew][lane] = m0;   // its waves' shares of rho E
        } else {
            mom[l][0][lane] = m0; mom[l][1][lane] = m1; mom[l][2][lane] = m2; mom[l][3][lane] = m3;
        }
    }
    __syncthreads();
    // the local state (first wave): rho and u from the momentum lattice, the
    // species densities (the slaved one by difference, eq. strongest), T by
    // Newton on the energy lattice's internal energy from the imposed T; and
    // the full inlet's target, the local density and composition at the
    // imposed u^in and T^in (eqs. in_tgt_*)
    if (l == 0 && !bback) {
        double Y[M], u[3];
        const double rl = mom[LF][0][lane];
        double rs = rl, ry = 0.0;
#pragma unroll
        for (int c = 0; c < M; ++c) {
            const bool slv = !W && c == s;
            const double v = slv ? 0.0 : mom[slv ? 0 : (W ? c : c - (c > s ? 1 : 0))][0][lane];
            Y[c] = v;
            rs -= v;
            ry += v;
        }
        if constexpr (!W) {
#pragma unroll
            for (int c = 0; c < M; ++c)
                if (c == s) Y[c] = rs;
        }
        const double iry = 1.0 / (W ? ry : rl), irl = 1.0 / rl;   // weakly coupled: Y by sum_a rho_a
#pragma unroll
        for (int c = 0; c < M; ++c) Y[c] *= iry;
#pragma unroll
        for (int d = 0; d < 3; ++d) u[d] = mom[LF][1 + d][lane] * irl;
        double rE = mom[LG][0][lane];
#pragma unroll
        for (int e = 1; e < EW; ++e) rE += mom[LG][e][lane];
        const double Ul = rE * irl - 0.5 * (u[0] * u[0] + u[1] * u[1] + u[2] * u[2]);
        int fail = 0;
        reload_barrier();
        const double Tl = solve_T<M>(in_loop(mc0), Y, Ul, stA[ST_T][lane], &fail);
        flg[lane] = fail;
        state_store<M>(mc0, stL, lane, rl, u, Y, Tl);
        if (inlet_full) {
            reload_barrier();
            MechC mc = in_loop(mc0);
            stT[0][lane] = mc.R_univ * mix_inv_m<M>(mc, Y) * L.T_in;
            stT[1][lane] = mix_U<M>(mc, Y, L.T_in);
        }
    }
    __syncthreads();
    // step 4: reconstruction of this wave's lattice.  The wall's local species
    // equilibria take the species' own velocity u_a = j_a / rho_a (u where
    // rho_a <= 1e-14 rho, eq. locua).
    //   TMS wall (eqs. ftms, gtms, fatms) and outlet (eqs. f_outlet, g_outlet,
    // fa_outlet): 2 A - loc on incoming links, A + f - loc on outgoing ones;
    //   full inlet (eqs. f_inlet, g_inlet, fa_inlet): tgt + A - loc and
    // tgt + f - loc;
    //   simplified inlet (eqs. in_loc_*): loc on every link.
    // An advected value's reference is that of the slot it goes to.
    if (!bback) {
        double w[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) w[d] = stL[ST_V + d][lane];
        if (wall && l < LF) {
            const double ra = mom[l][0][lane];
            if (!(ra <= 1e-14 * stL[ST_RHO][lane])) {
                const double ir = 1.0 / ra;
#pragma unroll
                for (int d = 0; d < 3; ++d) w[d] = mom[l][1 + d][lane] * ir;
            }
        }
        LatEq eL, eT;
        lat_prepare<M, W>(mc0, stL, lane, l, s, stL[ST_T][lane], stL[ST_TH][lane], stL[ST_U][lane], w[0], w[1], w[2], eL);
        const bool any_inlet = __builtin_amdgcn_ballot_w64(inlet_full) != 0;
        if (any_inlet)
            lat_prepare<M, W>(mc0, stL, lane, l, s, L.T_in, stT[0][lane], stT[1][lane], L.u_in, 0.0, 0.0, eT);
        const bool local = type == RLBM_FACE_INLET_LOCAL;
#pragma unroll 1
        for (int lay = lay0; lay < lay1; ++lay) {
            const int c2 = lay - 1, i0 = 9 * lay;
            const unsigned in = Dm >> i0;
            eA.layer(energy, c2);
            eL.layer(energy, c2);
            if (any_inlet) eT.layer(energy, c2);
            double f[9];
#pragma unroll
            for (int j = 0; j < 9; ++j) f[j] = adv(i0 + j, j % 3 - 1, j / 3 - 1, c2);
            RLBM_GLOBAL S* pl = bc + (size_t)(l * Q + i0) * P;
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                double va[3], vl[3], vt[3];
                eA.row(energy, j, va);
                eL.row(energy, j, vl);
#pragma unroll
                for (int c = 0; c < 3; ++c) vt[c] = va[c];
                if (any_inlet) {
                    double e[3];
                    eT.row(energy, j, e);
#pragma unroll
                    for (int c = 0; c < 3; ++c) vt[c] = inlet_full ? e[c] : vt[c];
                }
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    const double rf = ref(i0 + 3 * j + c, sl, sf);
                    const double d = vt[c] - vl[c];
                    double v = (in >> (3 * j + c)) & 1u ? d + (va[c] - rf) : d + f[3 * j + c];
                    if (local) v = vl[c] - rf;
                    if (live) st_at(pl + (size_t)(3 * j + c) * P, k, (S)v);
                }
            }
        }
    }
    if (l == 0 && live && flg[lane]) atomicOr(L.flag, 1);
}

// ---------------------------------------------------------------------------
// initial state, read-out, populations I/O, invariants
// ---------------------------------------------------------------------------
// The read-out kernels take k_update's split: three waves per 64 nodes, wave w
// the nine velocities with c_z = w - 1.
constexpr int IO_NODES = 64;
constexpr int IO_THREADS = 3 * IO_NODES;

// Moments of the stored populations of one node over the c_z = c2 layer: rho,
// rho u, rho E and the stored species' rho_a.  Every load of a row of three
// velocities is in flight together (NL populations and the reader's scales as
// 16-byte loads), where a loop over single velocities waited for each.
template <int M, int W>
struct LayerSums {
    static constexpr int N = 5 + Lat<M, W>::NSP;   // rho, j[3], rho E, rho_a
    double v[N];
};
template <int M, typename S, int W, bool CHECK>
__device__ __forceinline__ void layer_sums(const LatDev& L, int q, int node, int c2, LayerSums<M, W>& t, bool& bad) {
    constexpr int NSP = Lat<M, W>::NSP, LF = Lat<M, W>::LF, LG = Lat<M, W>::LG, NL = Lat<M, W>::NL;
    const RLBM_GLOBAL S* src = as_global(static_cast<const S*>(L.pop[q]));
    const size_t P = (size_t)L.P;
    const int x = node % L.nx, r = node / L.nx, y = r % L.ny, z = r / L.ny;
    PullOff o;
    pull_offsets(L, x, y, z, o);
#pragma unroll
    for (int a = 0; a < LayerSums<M, W>::N; ++a) t.v[a] = 0.0;
#pragma unroll 1
    for (int c1 = -1; c1 <= 1; ++c1) {
        const int i0 = 9 * (c2 + 1) + 3 * (c1 + 1);
        S raw[3][NL];
        float sc[3][NL];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
#pragma unroll
            for (int l = 0; l < NL; ++l) raw[c][l] = ld_at(src + (size_t)(l * Q + i0 + c) * P, node);
            if constexpr (sizeof(S) == 4) scales_of<NL>(L, q, reader_at(node, o, c - 1, c1, c2), sc[c]);
        }
        double m[NL], jx = 0.0;
#pragma unroll
        for (int l = 0; l < NL; ++l) m[l] = 0.0;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
#pragma unroll
            for (int l = 0; l < NL; ++l) {
                double v = (double)raw[c][l];
                if constexpr (sizeof(S) == 4) {
                    const RLBM_CONST double* G = as_const(L.ref) + opaque_zero();
                    const int i = i0 + c;
                    v += l == LG ? ref_g(sc[c][LG], sc[c][LF], G[LG * Q + i], G[REF_K<NL> + i]) : ref_of(sc[c][l], G[l * Q + i]);
                }
                if constexpr (CHECK) bad |= !isfinite(v);
                m[l] += v;
                if (l == LF) jx += c == 2 ? v : (c == 0 ? -v : 0.0);
            }
        }
        t.v[0] += m[LF];
        t.v[1] += jx;
        t.v[2] += (double)c1 * m[LF];
        t.v[3] += (double)c2 * m[LF];
        t.v[4] += m[LG];
#pragma unroll
        for (int l = 0; l < NSP; ++l) t.v[5 + l] += m[l];
    }
}

// The species densities of a node in species order from its layer sums (the
// slaved one by difference, eq. strongest).
template <int M, int W>
__device__ __forceinline__ void species_of_sums(const LayerSums<M, W>& t, int s, double (&ra)[M]) {
    double rs = t.v[0];
#pragma unroll
    for (int l = 0; l < Lat<M, W>::NSP; ++l) rs -= t.v[5 + l];
#pragma unroll
    for (int a = 0; a < M; ++a) {
        if constexpr (W) ra[a] = t.v[5 + a];
        else {
            double v = rs;
#pragma unroll
            for (int l = 0; l < Lat<M, W>::NSP; ++l)
                if (a != s && l == lat_of(a, s)) v = t.v[5 + l];
            ra[a] = v;
        }
    }
}

// Reference scales of the initial populations: the zeroth moments rho_a of
// the stored species, rho and rho E.
template <int M, int W>
__global__ __launch_bounds__(256) void k_scale_init(const LatDev* __restrict__ lat, const double* __restrict__ rho_in,
                                                    const double* __restrict__ u_in, const double* __restrict__ T_in,
                                                    const double* __restrict__ Y_in) {
    const LatDev& L = *lat;
    const long long node = (long long)blockIdx.x * 256 + threadIdx.x;
    if (node >= L.N) return;
    MechC mc = *as_const(L.mech);
    const size_t N = (size_t)L.N;
    constexpr int NSP = Lat<M, W>::NSP;
    const int s = W ? M : L.slaved;
    const double rho = rho_in[node];
    double Y[M];
#pragma unroll
    for (int a = 0; a < M; ++a) Y[a] = Y_in[a * N + node];
    for (int l = 0; l < NSP; ++l) {
        const int a = W ? l : l + (l >= s ? 1 : 0);
        // both buffers: the populations' own, and what the first explicit step
        // encodes with
        const float v = __double2float_rn(rho * Y_in[a * N + node]);
        L.rscale[0][(size_t)node * L.rss + l] = v;
        L.rscale[1][(size_t)node * L.rss + l] = v;
    }
    double usq = 0.0;
#pragma unroll
    for (int dd = 0; dd < 3; ++dd) usq += u_in[dd * N + node] * u_in[dd * N + node];
    float* f = L.fscale[L.parity0] + (size_t)node * L.fss;
    f[0] = __double2float_rn(rho);
    f[1] = __double2float_rn(rho * (mix_U<M>(mc, Y, T_in[node]) + 0.5 * usq));
}

// Initial populations: the equilibria of the given state, k_update's split
// (three waves per 64 nodes, one c_z layer each).  A lattice's axis factors
// are formed once and multiplied out over the layer's nine velocities; the
// kernel is bound by its stores.  512x64x64, FP32 storage: 2.38 -> 1.43 ms
// against one thread per node that evaluated every velocity from the state.
template <int M, typename S, int W>
__global__ __launch_bounds__(IO_THREADS) void k_init(const LatDev* __restrict__ lat, const double* __restrict__ rho_in,
                                                     const double* __restrict__ u_in, const double* __restrict__ T_in,
                                                     const double* __restrict__ Y_in) {
    constexpr int NSP = Lat<M, W>::NSP, LF = Lat<M, W>::LF, LG = Lat<M, W>::LG, NL = Lat<M, W>::NL;
    const LatDev& L = *lat;
    const int node = (int)blockIdx.x * IO_NODES + (int)threadIdx.x % IO_NODES;
    const int c2 = __builtin_amdgcn_readfirstlane((int)threadIdx.x / IO_NODES) - 1;
    if (node >= (int)L.N) return;
    MechC mc = *as_const(L.mech);
    const size_t N = (size_t)L.N, P = (size_t)L.P;
    const int s = W ? M : L.slaved;
    RLBM_GLOBAL S* dst = as_global(static_cast<S*>(L.pop[L.parity0]));
    const double rho = rho_in[node], T = T_in[node];
    double u[3], Y[M];
#pragma unroll
    for (int d = 0; d < 3; ++d) u[d] = u_in[d * N + node];
#pragma unroll
    for (int a = 0; a < M; ++a) Y[a] = Y_in[a * N + node];
    const double th = mc.R_univ * mix_inv_m<M>(mc, Y) * T;
    const int x = node % L.nx, r = node / L.nx, y = r % L.ny, z = r / L.ny;
    PullOff o;
    pull_offsets(L, x, y, z, o);
#pragma unroll 1
    for (int l = 0; l < NL; ++l) {
        double X[3], Yf[3], kx[3] = {0.0, 0.0, 0.0}, ky[3] = {0.0, 0.0, 0.0}, Zf, kz = 0.0, amp = rho, U = 1.0;
        if (l == LG) {
            GeqAxis gx, gy, gz;
            geq_axis(u[0], th, gx);
            geq_axis(u[1], th, gy);
            geq_axis(u[2], th, gz);
#pragma unroll
            for (int c = 0; c < 3; ++c) { X[c] = gx.W[c]; kx[c] = gx.k[c]; Yf[c] = gy.W[c]; ky[c] = gy.k[c]; }
            Zf = sel3d(c2, gz.W[0], gz.W[1], gz.W[2]);
            kz = sel3d(c2, gz.k[0], gz.k[1], gz.k[2]);
            U = mix_U<M>(mc, Y, T);
        } else {
            double tl = th;
            if (l < NSP) {
                const int a = W ? l : l + (l >= s ? 1 : 0);
                tl = mc.Ra[a] * T;
                amp = rho * Y_in[a * N + node];
            }
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                X[c] = psi(c - 1, u[0], u[0] * u[0] + tl);
                Yf[c] = psi(c - 1, u[1], u[1] * u[1] + tl);
            }
            Zf = psi(c2, u[2], u[2] * u[2] + tl);
        }
        const RLBM_CONST double* G = as_const(L.ref);
#pragma unroll
        for (int j = 0; j < 9; ++j) {
            const int c0 = j % 3, c1 = j / 3, i = 9 * (c2 + 1) + j;
            const double wyz = Yf[c1] * Zf;
            const double v = amp * (U * X[c0] * wyz + kx[c0] * wyz + X[c0] * (ky[c1] * Zf + Yf[c1] * kz));
            RLBM_GLOBAL S* pl = dst + (size_t)(l * Q + i) * P;
            if constexpr (sizeof(S) == 4) {
                const int rd = reader_at(node, o, c0 - 1, c1 - 1, c2);
                const float sl = scale_l(L, L.parity0, rd, l, LF), sf = fscale_at(L, L.parity0, rd)[0];
                const double ref = l == LG ? ref_g(sl, sf, G[l * Q + i], G[REF_K<NL> + i]) : ref_of(sl, G[l * Q + i]);
                st_at(pl, node, __double2float_rn(v - ref));
            } else {
                st_at(pl, node, v);
            }
        }
    }
    if (c2 != 0) return;
    double* aux = L.aux;
    aux[AUX_RHO * N + node] = rho;
#pragma unroll
    for (int dd = 0; dd < 3; ++dd) {
        aux[(AUX_U + dd) * N + node] = u[dd];
        aux[(AUX_PHI + dd) * N + node] = rho * u[dd] * (1.0 - 3.0 * th) - rho * u[dd] * u[dd] * u[dd];
    }
    aux[AUX_T * N + node] = T;
#pragma unroll
    for (int a = 0; a < M; ++a) aux[(AUX_Y + a) * N + node] = Y[a];
    if (L.n_if) {
        const int k = L.if_index[node];
        if (k >= 0 && L.if_out[k] >= 0) {
            const int ko = L.if_out[k];
            const size_t No = (size_t)L.n_out;
            L.out_state[0 * No + ko] = rho;
#pragma unroll
            for (int dd = 0; dd < 3; ++dd) L.out_state[(1 + dd) * No + ko] = u[dd];
            L.out_state[4 * No + ko] = T;
#pragma unroll
            for (int a = 0; a < M; ++a) L.out_state[(5 + a) * No + ko] = Y[a];
        }
    }
}

// Reference shapes for FP32 deviation storage (one block): for the stored
// species, the momentum lattice and the energy lattice's internal-energy part
// the zero-velocity equilibrium shape (unit zeroth moment) at the
// domain-mean temperature and composition, and the energy lattice's theta^2
// part K (eq. geq_i at u = 0 with rho = 1, U = 0); then the zeroth moments,
// the momentum shape's sum_i G c_x^2 and sum_i K_i.
template <int M, int W>
__global__ __launch_bounds__(512) void k_refs(const LatDev* __restrict__ lat, double* __restrict__ ref, double rho,
                                              double T, const double* __restrict__ Y) {
    constexpr int NSP = Lat<M, W>::NSP, LF = Lat<M, W>::LF, LG = Lat<M, W>::LG, NL = Lat<M, W>::NL;
    static_assert(NL * Q <= 512, "one thread per reference shape value");
    (void)rho;
    const LatDev& L = *lat;
    const int li = threadIdx.x;
    MechC mc = *as_const(L.mech);
    const double th_mix = mc.R_univ * mix_inv_m<M>(mc, Y) * T;
    if (li < NL * Q) {
        const int l = li / Q, i = li % Q;
        const int c0 = cx_of(i), c1 = cy_of(i), c2 = cz_of(i);
        double th = th_mix;
        if (l < NSP) th = mc.Ra[W ? l : l + (l >= L.slaved ? 1 : 0)] * T;
        // shapes are rounded to FP32 values (see ref_of)
        ref[li] = (double)(float)(psi(c0, 0.0, th) * psi(c1, 0.0, th) * psi(c2, 0.0, th));
        ref[REF_T<NL> + i * NL + l] = ref[li];
        if (l == LG) {
            const double Wx = psi(c0, 0.0, th), Wy = psi(c1, 0.0, th), Wz = psi(c2, 0.0, th);
            const double k0 = -th * th, k1 = 0.5 * th * th;
            const double kx = c0 ? k1 : k0, ky = c1 ? k1 : k0, kz = c2 ? k1 : k0;
            ref[REF_K<NL> + i] = (double)(float)(kx * Wy * Wz + Wx * (ky * Wz + Wy * kz));
        }
    }
    __syncthreads();
    if (li < NL) {
        double m0 = 0.0;
        for (int i = 0; i < Q; ++i) m0 += ref[li * Q + i];
        ref[REF_M0<NL> + li] = m0;
    } else if (li == NL) {
        double m2 = 0.0;
        for (int i = 0; i < Q; ++i) m2 += ref[LF * Q + i] * (double)(cx_of(i) * cx_of(i));
        ref[REF_M2<NL>] = m2;
    } else if (li == NL + 1) {
        double k0 = 0.0;
        for (int i = 0; i < Q; ++i) k0 += ref[REF_K<NL> + i];
        ref[REF_K0<NL>] = k0;
    }
}

// Macroscopic fields of the stored populations.  Bound by the populations'
// read; the layers' sums meet in LDS and the first wave solves for T.
// 512x64x64, FP32 storage: 2.41 -> 0.53 ms against one thread per node
// looping over single velocities; 1024 nodes: 106 -> 8 us.  status[0] takes
// the failure flag as the steps left it, status[1] this kernel's own, in
// pinned host memory: a copy of the flag after the kernel takes 11 us.
template <int M, typename S, int W>
__global__ __launch_bounds__(IO_THREADS) void k_fields(const LatDev* __restrict__ lat, long long t, double* rho_o,
                                                       double* u_o, double* T_o, double* Y_o, double* P_o,
                                                       int* __restrict__ status) {
    constexpr int NV = LayerSums<M, W>::N;
    __shared__ double part[2][NV][IO_NODES];
    const LatDev& L = *lat;
    const int lane = (int)threadIdx.x % IO_NODES;
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / IO_NODES);
    const int n = (int)blockIdx.x * IO_NODES + lane;
    const size_t N = (size_t)L.N;
    const bool live = n < (int)N;
    const int node = live ? n : 0;
    if (blockIdx.x == 0 && threadIdx.x == 0) status[0] = *(const volatile int*)L.flag;
    LayerSums<M, W> m;
    bool bad = false;
    layer_sums<M, S, W, false>(L, (int)((L.parity0 + t) & 1), node, w - 1, m, bad);
    if (w) {
#pragma unroll
        for (int k = 0; k < NV; ++k) part[w - 1][k][lane] = m.v[k];
    }
    __syncthreads();
    if (w || !live) return;
#pragma unroll
    for (int k = 0; k < NV; ++k) m.v[k] += part[0][k][lane] + part[1][k][lane];
    MechC mc = *as_const(L.mech);
    double Y[M];
    species_of_sums<M, W>(m, W ? M : L.slaved, Y);
    const double rho = m.v[0];
    double ry = rho;   // the weakly coupled storage normalises Y by sum_a rho_a
    if constexpr (W) {
        ry = 0.0;
#pragma unroll
        for (int a = 0; a < M; ++a) ry += Y[a];
    }
#pragma unroll
    for (int a = 0; a < M; ++a) Y[a] /= ry;
    const double u[3] = {m.v[1] / rho, m.v[2] / rho, m.v[3] / rho};
    const double U = m.v[4] / rho - 0.5 * (u[0] * u[0] + u[1] * u[1] + u[2] * u[2]);
    int fail = 0;
    const double T = solve_T<M>(mc, Y, U, L.aux[AUX_T * N + node], &fail);
    if (fail) {
        atomicOr(L.flag, 1);
        status[1] = 1;
    }
    if (rho_o) rho_o[node] = rho;
    if (u_o)
#pragma unroll
        for (int dd = 0; dd < 3; ++dd) u_o[dd * N + node] = u[dd];
    if (T_o) T_o[node] = T;
    if (Y_o)
#pragma unroll
        for (int a = 0; a < M; ++a) Y_o[a * N + node] = Y[a];
    if (P_o) P_o[node] = rho * mc.R_univ * mix_inv_m<M>(mc, Y) * T;
}

// References of the row's three velocities of lattice l at `node` (FP32 storage).
template <int M, int W>
__device__ __forceinline__ void row_refs(const LatDev& L, int q, int node, int l, int row, double (&ref)[3]) {
    constexpr int LF = Lat<M, W>::LF, LG = Lat<M, W>::LG, NL = Lat<M, W>::NL;
    const int x = node % L.nx, r = node / L.nx, y = r % L.ny, z = r / L.ny;
    PullOff o;
    pull_offsets(L, x, y, z, o);
    const RLBM_CONST double* G = as_const(L.ref);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const int i = 3 * row + c, rd = reader_at(node, o, c - 1, row % 3 - 1, row / 3 - 1);
        const float sl = scale_l(L, q, rd, l, LF), sf = fscale_at(L, q, rd)[0];
        ref[c] = l == LG ? ref_g(sl, sf, G[l * Q + i], G[REF_K<NL> + i]) : ref_of(sl, G[l * Q + i]);
    }
}

// FP64 copies of the stored lattices l0 .. l0 + nl - 1 from (write = 0) or, FP64
// storage, into (write = 1) the current population buffer; buf holds
// [nl][27][N].  One thread per node and three velocities of one row
// (blockIdx.y the row, z the lattice): the plane is uniform, where one thread
// per value divided 64-bit indices.  256x64x16, all lattices: 433 -> 288 us
// (FP32 storage), 236 -> 204 us (FP64).
template <int M, typename S, int W>
__global__ __launch_bounds__(256) void k_pops(const LatDev* __restrict__ lat, long long t, int l0, double* buf, int write) {
    const LatDev& L = *lat;
    const int node = (int)blockIdx.x * 256 + (int)threadIdx.x;
    if (node >= (int)L.N) return;
    const int l = l0 + (int)blockIdx.z, i0 = 3 * (int)blockIdx.y;
    const size_t N = (size_t)L.N, P = (size_t)L.P;
    const int q = (int)((L.parity0 + t) & 1);
    RLBM_GLOBAL S* pop = as_global(static_cast<S*>(L.pop[q])) + (size_t)(l * Q + i0) * P;
    RLBM_GLOBAL double* out = as_global(buf) + ((size_t)blockIdx.z * Q + i0) * N;
    if constexpr (sizeof(S) == 4) {
        S v[3];
        double ref[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) v[c] = ld_at(pop + c * P, node);
        row_refs<M, W>(L, q, node, l, (int)blockIdx.y, ref);
#pragma unroll
        for (int c = 0; c < 3; ++c) out[c * N + node] = (double)v[c] + ref[c];
    } else {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            if (write) st_at(pop + c * P, node, (S)out[c * N + node]);
            else out[c * N + node] = ld_at(pop + c * P, node);
        }
    }
}

// The writing of FP32 storage: a block takes 64 nodes of a lattice, one wave
// per row of three velocities.  An explicit step encodes a species with the
// scales of the other buffer; they become the zeroth moments of what is
// written here, so that populations of another state than the lattice's own
// are not rounded a second time, as coarsely, in the step after (with the old
// scales kept the error after it was 1.4 times as large).
constexpr int WRITE_NODES = 64;
template <int M, int W>
__global__ __launch_bounds__(9 * WRITE_NODES) void k_write_pops(const LatDev* __restrict__ lat, long long t, int l0,
                                                               const double* buf) {
    constexpr int LF = Lat<M, W>::LF;
    __shared__ double part[9][WRITE_NODES];
    const LatDev& L = *lat;
    const int lane = (int)threadIdx.x % WRITE_NODES;
    const int row = __builtin_amdgcn_readfirstlane((int)threadIdx.x / WRITE_NODES);
    const int n = (int)blockIdx.x * WRITE_NODES + lane;
    const bool live = n < (int)L.N;
    const int node = live ? n : (int)L.N - 1;
    const int l = l0 + (int)blockIdx.y, i0 = 3 * row;
    const size_t N = (size_t)L.N, P = (size_t)L.P;
    const int q = (int)((L.parity0 + t) & 1);
    RLBM_GLOBAL float* pop = as_global(static_cast<float*>(L.pop[q])) + (size_t)(l * Q + i0) * P;
    const RLBM_GLOBAL double* in = as_global(buf) + ((size_t)blockIdx.y * Q + i0) * N;
    double v[3], ref[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) v[c] = in[c * N + node];
    row_refs<M, W>(L, q, node, l, row, ref);
    if (live) {
#pragma unroll
        for (int c = 0; c < 3; ++c) st_at(pop + c * P, node, __double2float_rn(v[c] - ref[c]));
    }
    if (L.reaction != RLBM_REACTION_EXPLICIT || l >= LF) return;   // the whole block
    part[row][lane] = v[0] + v[1] + v[2];
    __syncthreads();
    if (row || !live) return;
    double m = 0.0;
#pragma unroll
    for (int k = 0; k < 9; ++k) m += part[k][lane];
    as_global(L.rscale[q ^ 1])[(size_t)node * L.rss + l] = __double2float_rn(m);
}

// Per-block partial sums of the invariants over INV_NODES nodes; nv = 6 + E
// values per block.  Every sum has a fixed order: over a lane's nodes, over
// the lanes of a wave (a butterfly), over the three waves.  256x64x64, FP32
// storage: 1.25 -> 0.25 ms.
constexpr int INV_NODES = 256;
template <int M, typename S, int W>
__global__ __launch_bounds__(IO_THREADS) void k_invariants(const LatDev* __restrict__ lat, long long t,
                                                           double* __restrict__ partial, int nv) {
    constexpr int NV = LayerSums<M, W>::N;
    __shared__ double red[3][NV + 1];
    const LatDev& L = *lat;
    const int lane = (int)threadIdx.x % IO_NODES;
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / IO_NODES);
    LayerSums<M, W> acc;
#pragma unroll
    for (int k = 0; k < NV; ++k) acc.v[k] = 0.0;
    bool bad = false;
    for (int c = 0; c < INV_NODES; c += IO_NODES) {
        const int node = (int)blockIdx.x * INV_NODES + c + lane;
        if (node < (int)L.N) {
            LayerSums<M, W> m;
            layer_sums<M, S, W, true>(L, (int)((L.parity0 + t) & 1), node, w - 1, m, bad);
#pragma unroll
            for (int k = 0; k < NV; ++k) acc.v[k] += m.v[k];
        }
    }
#pragma unroll
    for (int k = 0; k < NV; ++k) {
#pragma unroll
        for (int d = 1; d < IO_NODES; d <<= 1) acc.v[k] += __shfl_xor(acc.v[k], d);
        if (lane == 0) red[w][k] = acc.v[k];
    }
    const bool any = __builtin_amdgcn_ballot_w64(bad) != 0;
    if (lane == 0) red[w][NV] = any ? 1.0 : 0.0;
    __syncthreads();
    if (threadIdx.x) return;
#pragma unroll
    for (int k = 0; k < NV; ++k) acc.v[k] = red[0][k] + red[1][k] + red[2][k];
    MechC mc = *as_const(L.mech);
    double ra[M];
    species_of_sums<M, W>(acc, W ? M : L.slaved, ra);
    double* out = partial + (size_t)blockIdx.x * nv;
#pragma unroll
    for (int k = 0; k < 5; ++k) out[k] = acc.v[k];
    for (int e = 0; e < mc.E; ++e) {
        double sum = 0.0;
#pragma unroll
        for (int a = 0; a < M; ++a) sum += ra[a] * mc.inv_m[a] * mc.comp[a][e];
        out[5 + e] = sum;
    }
    out[5 + mc.E] = fmax(fmax(red[0][NV], red[1][NV]), red[2][NV]);
}

// One block per value, every partial read once by 256 threads and summed in a
// fixed order.  One thread per value took 943 us for 4,096 blocks (a chain of
// dependent loads), one block per value takes 9 us.
__global__ __launch_bounds__(256) void k_reduce_partials(const double* __restrict__ partial, int nblocks, int nv,
                                                         double* __restrict__ out) {
    __shared__ double red[4];
    const int q = blockIdx.x;
    const bool largest = q == nv - 1;
    double acc = 0.0;
    for (int b = threadIdx.x; b < nblocks; b += 256) {
        const double x = partial[(size_t)b * nv + q];
        acc = largest ? fmax(acc, x) : acc + x;
    }
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const double x = __shfl_xor(acc, d);
        acc = largest ? fmax(acc, x) : acc + x;
    }
    if (threadIdx.x % 64 == 0) red[threadIdx.x / 64] = acc;
    __syncthreads();
    if (threadIdx.x) return;
    out[q] = largest ? fmax(fmax(red[0], red[1]), fmax(red[2], red[3])) : (red[0] + red[1]) + (red[2] + red[3]);
}

// The small sections of a snapshot, to or from one piece of memory: one launch
// in place of a copy each, of which the runtime takes four in 3 us apiece and
// every further one in 8.
__global__ __launch_bounds__(256) void k_pack(Pack p) {
    const PackSeg g = p.seg[blockIdx.y];
    const RLBM_GLOBAL unsigned* src = as_global(static_cast<const unsigned*>(g.src));
    RLBM_GLOBAL unsigned* dst = as_global(static_cast<unsigned*>(g.dst));
    const unsigned n = g.rows * g.words;
    for (unsigned w = blockIdx.x * 256u + threadIdx.x; w < n; w += gridDim.x * 256u) {
        const unsigned r = w / g.words, c = w - r * g.words;
        dst[(size_t)r * g.dst_step + c] = src[(size_t)r * g.src_step + c];
    }
}

// Advances the device step counter of a launch series by n (the last node
// of a captured chunk of batched steps).
__global__ void k_advance_time(long long* __restrict__ tp, long long n) {
    if (threadIdx.x == 0 && blockIdx.x == 0) *tp += n;
}

// Reads and clears the failure flags of k lattices: out[j] = *flags[j].
__global__ __launch_bounds__(256) void k_gather_flags(int* const* __restrict__ flags, int k, int* __restrict__ out) {
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j < k) out[j] = atomicExch(flags[j], 0);
}

hipError_t launch_pack(const Pack& p, hipStream_t st) {
    (void)hipGetLastError();   // report this launch's error only
    if (p.n <= 0) return hipSuccess;
    unsigned most = 1;
    for (int k = 0; k < p.n; ++k) most = p.seg[k].rows * p.seg[k].words > most ? p.seg[k].rows * p.seg[k].words : most;
    const unsigned blocks = most / 1024u + 1u;
    hipLaunchKernelGGL(k_pack, dim3(blocks < 2048u ? blocks : 2048u, p.n), dim3(256), 0, st, p);
    return hipGetLastError();
}

hipError_t launch_advance_time(long long* tp, long long n, hipStream_t st) {
    (void)hipGetLastError();   // report this launch's error only
    hipLaunchKernelGGL(k_advance_time, dim3(1), dim3(64), 0, st, tp, n);
    return hipGetLastError();
}

hipError_t launch_gather_flags(int* const* flags, int k, int* out, hipStream_t st) {
    (void)hipGetLastError();   // report this launch's error only
    if (k <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_gather_flags, dim3((k + 255) / 256), dim3(256), 0, st, flags, k, out);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// allocation-free group steps: tables in a file-scope device array
// ---------------------------------------------------------------------------
// Each GPU holds its own copy until the process ends.  Host code never
// names it: it uses the device address that group_scratch() returns.
static __device__ __align__(256) unsigned char scratch[GROUP_SCRATCH_BYTES];

hipError_t group_scratch(int device, char** ptr) {
    // one address per device, looked up once with that device current
    static std::mutex mu;
    static char* addr[64] = {};
    if (device < 0 || device >= 64) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[device]) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        addr[device] = (char*)p;
    }
    *ptr = addr[device];
    return hipSuccess;
}

// Entries base .. base + n - 1 of the group table: block j copies lattice
// j's device entry word by word, then sets its buffer parity and step
// count; block 0 writes the block prefixes of those entries (and of the
// entry after the last), and resets the step counter on the first chunk.
__global__ __launch_bounds__(64) void k_group_gather(char* __restrict__ sc, GroupChunk c) {
    const int j = blockIdx.x;
    LatDev* table = (LatDev*)(sc + GROUP_OFF_TABLE);
    int* blk = (int*)(sc + GROUP_OFF_BLK);
    static_assert(sizeof(LatDev) % 8 == 0, "the entry is copied in 8-byte words");
    const unsigned long long* src = (const unsigned long long*)c.src[j];
    unsigned long long* dst = (unsigned long long*)&table[c.base + j];
    for (int w = threadIdx.x; w < (int)(sizeof(LatDev) / 8); w += 64) dst[w] = src[w];
    __syncthreads();
    if (threadIdx.x == 0) {
        table[c.base + j].parity0 = c.parity[j];
        table[c.base + j].t_end = c.t_end[j];
    }
    if (j == 0) {
        for (int q = threadIdx.x; q < 3 * (c.n + 1); q += 64) {
            const int a = q / (c.n + 1), e = q % (c.n + 1);
            blk[a * (c.k + 1) + c.base + e] = c.blk[a][e];
        }
        if (c.base == 0 && threadIdx.x == 0) *(long long*)sc = 0;
    }
}

hipError_t launch_group_gather(char* sc, const GroupChunk& c, hipStream_t st) {
    (void)hipGetLastError();   // report this launch's error only
    if (c.n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_group_gather, dim3(c.n), dim3(64), 0, st, sc, c);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// dispatch
// ---------------------------------------------------------------------------
#define RLBM_DISPATCH(M_, ...)                            \
    switch (M_) {                                         \
        case 2: { constexpr int MM = 2; __VA_ARGS__; break; } \
        case 3: { constexpr int MM = 3; __VA_ARGS__; break; } \
        case 4: { constexpr int MM = 4; __VA_ARGS__; break; } \
        case 9: { constexpr int MM = 9; __VA_ARGS__; break; } \
        default: return hipErrorInvalidValue;             \
    }
// species count and storage coupling (WW = 1: weakly coupled, all M species stored)
#define RLBM_DISPATCH_W(M_, W_, ...)                                                   \
    if (W_) {                                                                          \
        constexpr int WW = 1;                                                          \
        RLBM_DISPATCH(M_, __VA_ARGS__)                                                 \
    } else {                                                                           \
        constexpr int WW = 0;                                                          \
        RLBM_DISPATCH(M_, __VA_ARGS__)                                                 \
    }

template <typename S>
static hipError_t launch_step_phase(int phase, int M, int weak, const StepLaunch& a) {
    if (a.blocks <= 0) return hipSuccess;
    (void)hipGetLastError();   // report this launch's error only
    const bool explicit_ = a.schemes & (1u << RLBM_REACTION_EXPLICIT);
    const bool implicit_ = a.schemes & (1u << RLBM_REACTION_LINEARLY_IMPLICIT);
    if (phase == 0) {
        RLBM_DISPATCH_W(M, weak, hipLaunchKernelGGL((k_boundary<MM, S, WW>), dim3(a.blocks), dim3(bc_threads<MM, WW>()), 0,
                                                    a.stream, a.lats, a.blk, a.n_lat, a.tp, a.toff))
    } else if (phase == 1) {
        if (explicit_)
            RLBM_DISPATCH_W(M, weak, hipLaunchKernelGGL((k_species<MM, S, WW>), dim3(a.blocks), dim3(SPC_THREADS), 0, a.stream,
                                                        a.lats, a.blk, a.n_lat, a.tp, a.toff))
        if (implicit_)
            RLBM_DISPATCH_W(M, weak, hipLaunchKernelGGL((k_local<MM, S, WW>), dim3(a.blocks), dim3(NODE_TILE), 0, a.stream,
                                                        a.lats, a.blk, a.n_lat, a.tp, a.toff))
    } else if (phase == 2) {
        if (implicit_)
            RLBM_DISPATCH(M, hipLaunchKernelGGL((k_chem_implicit<MM>), dim3(a.blocks), dim3(NODE_TILE), 0, a.stream, a.lats,
                                                a.blk, a.n_lat, a.tp, a.toff))
    } else {
        if (explicit_)
            RLBM_DISPATCH_W(M, weak, hipLaunchKernelGGL((k_flow<MM, S, WW>), dim3(a.blocks), dim3(FLOW_THREADS), 0, a.stream,
                                                        a.lats, a.blk, a.n_lat, a.tp, a.toff))
        if (implicit_)
            RLBM_DISPATCH_W(M, weak, hipLaunchKernelGGL((k_update<MM, S, WW>), dim3(a.blocks), dim3(UPD_THREADS), 0,
                                                        a.stream, a.lats, a.blk, a.n_lat, a.tp, a.toff))
    }
    return hipGetLastError();
}

hipError_t launch_phase(int phase, int M, int storage, int weak, const StepLaunch& a) {
    return storage == RLBM_STORAGE_F32_DEV ? launch_step_phase<float>(phase, M, weak, a)
                                           : launch_step_phase<double>(phase, M, weak, a);
}

static int io_blocks(long long N) { return (int)((N + IO_NODES - 1) / IO_NODES); }

template <typename S>
static hipError_t launch_init_t(int M, int weak, const LatDev* lat, long long N, const double* rho,
                                const double* u, const double* T, const double* Y, hipStream_t st) {
    (void)hipGetLastError();   // report this launch's error only
    if constexpr (sizeof(S) == 4) {
        RLBM_DISPATCH_W(M, weak, hipLaunchKernelGGL((k_scale_init<MM, WW>), dim3((int)((N + 255) / 256)), dim3(256), 0, st,
                                                    lat, rho, u, T, Y))
    }
    RLBM_DISPATCH_W(M, weak, hipLaunchKernelGGL((k_init<MM, S, WW>), dim3(io_blocks(N)), dim3(IO_THREADS), 0, st, lat, rho,
                                                u, T, Y))
    return hipGetLastError();
}

hipError_t launch_init(int M, int storage, int weak, const LatDev* lat, long long N, const double* rho,
                       const double* u, const double* T, const double* Y, hipStream_t st) {
    return storage == RLBM_STORAGE_F32_DEV ? launch_init_t<float>(M, weak, lat, N, rho, u, T, Y, st)
                                           : launch_init_t<double>(M, weak, lat, N, rho, u, T, Y, st);
}

hipError_t launch_refs(int M, int weak, const LatDev* lat, double* ref, double rho, double T, const double* Y,
                       hipStream_t st) {
    (void)hipGetLastError();   // report this launch's error only
    RLBM_DISPATCH_W(M, weak, hipLaunchKernelGGL((k_refs<MM, WW>), dim3(1), dim3(512), 0, st, lat, ref, rho, T, Y))
    return hipGetLastError();
}

template <typename S>
static hipError_t launch_fields_t(int M, int weak, const LatDev* lat, long long N, long long t, double* rho,
                                  double* u, double* T, double* Y, double* P, int* status, hipStream_t st) {
    (void)hipGetLastError();   // report this launch's error only
    RLBM_DISPATCH_W(M, weak, hipLaunchKernelGGL((k_fields<MM, S, WW>), dim3(io_blocks(N)), dim3(IO_THREADS), 0, st, lat, t,
                                                rho, u, T, Y, P, status))
    return hipGetLastError();
}

hipError_t launch_fields(int M, int storage, int weak, const LatDev* lat, long long N, long long t, double* rho,
                         double* u, double* T, double* Y, double* P, int* status, hipStream_t st) {
    return storage == RLBM_STORAGE_F32_DEV ? launch_fields_t<float>(M, weak, lat, N, t, rho, u, T, Y, P, status, st)
                                           : launch_fields_t<double>(M, weak, lat, N, t, rho, u, T, Y, P, status, st);
}

hipError_t launch_pops(int M, int storage, int weak, const LatDev* lat, long long N, int l0, int nl, long long t,
                       double* buf, int write, hipStream_t st) {
    (void)hipGetLastError();   // report this launch's error only
    const dim3 grid((unsigned)((N + 255) / 256), Q / 3, nl), tiles((unsigned)((N + WRITE_NODES - 1) / WRITE_NODES), nl);
    if (storage != RLBM_STORAGE_F32_DEV)
        RLBM_DISPATCH_W(M, weak, hipLaunchKernelGGL((k_pops<MM, double, WW>), grid, dim3(256), 0, st, lat, t, l0, buf, write))
    else if (write)
        RLBM_DISPATCH_W(M, weak, hipLaunchKernelGGL((k_write_pops<MM, WW>), tiles, dim3(9 * WRITE_NODES), 0, st, lat, t, l0, buf))
    else
        RLBM_DISPATCH_W(M, weak, hipLaunchKernelGGL((k_pops<MM, float, WW>), grid, dim3(256), 0, st, lat, t, l0, buf, 0))
    return hipGetLastError();
}

template <typename S>
static hipError_t launch_inv_t(int M, int weak, const LatDev* lat, long long N, long long t, double* partial,
                               int nv, double* out, hipStream_t st) {
    (void)hipGetLastError();   // report this launch's error only
    const int blocks = (int)((N + INV_NODES - 1) / INV_NODES);
    RLBM_DISPATCH_W(M, weak, hipLaunchKernelGGL((k_invariants<MM, S, WW>), dim3(blocks), dim3(IO_THREADS), 0, st, lat, t,
                                                partial, nv))
    hipLaunchKernelGGL(k_reduce_partials, dim3(nv), dim3(256), 0, st, partial, blocks, nv, out);
    return hipGetLastError();
}

hipError_t launch_invariants(int M, int storage, int weak, const LatDev* lat, long long N, long long t,
                             double* partial, int nv, double* out, hipStream_t st) {
    return storage == RLBM_STORAGE_F32_DEV ? launch_inv_t<float>(M, weak, lat, N, t, partial, nv, out, st)
                                           : launch_inv_t<double>(M, weak, lat, N, t, partial, nv, out, st);
}

bool species_supported(int M) { return M == 2 || M == 3 || M == 4 || M == 9; }

}  // namespace rlbm
