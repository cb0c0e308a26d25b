// HIP kernels of the fluctuating D3Q19 LB step with a dissipatively coupled
// bead-spring chain, for gfx950 (MI355X).
//
//   k_couple      chains of up to 256 beads, one workgroup per chain (T lanes
//                 per bead, T a function of N only): velocity-Verlet
//                 substeps in the fluid velocity field frozen at the
//                 pre-collision state, trilinear interpolation, friction +
//                 Langevin force, and the impulse handed back to the stencil
//                 nodes (Sec. II.B, coupling paragraph; potentials of
//                 Sec. II.A).  Impulses go into a dense fixed-point field by
//                 atomic adds that nothing waits on (order-independent, hence
//                 bitwise reproducible); each bead lists the nodes it touched.
//   k_collide     fused stream + collide of every node, no impulse
//                 (Sec. II.B, LB equation), thread per node; populations in
//                 1024-node tiles of 19 planes each (pop_at).
//                 Pull form: a buffer holds post-collision populations p,
//                 the pre-collision population of node r is n_i(r) =
//                 p_i(r - c_i); reads are gathered, writes aligned and
//                 non-temporal.
//   k_near_nodes, k_chain_wg, k_spread
//                 the same coupling stage for chains of 257..1024 beads: node
//                 velocities around each bead, all substeps in one
//                 1024-thread workgroup writing per-substep records, and the
//                 records turned into node impulses
//   k_fixup       re-collides the nodes the beads touched, with their
//                 impulse, and overwrites their outputs
//   k_step        a batched step of chains of up to 256 beads in one kernel:
//                 the first workgroups do k_couple's work and collide the
//                 beads' nodes, which the tiles of the others skip
//   k_collide_deferred, k_overflow
//                 batched steps with chains of 257..1024 beads in sparse
//                 boxes: the tiles holding the beads' node tables skip the
//                 plain collide and are collided with their impulses beside
//                 it, after the coupling; nodes outside them that got an
//                 impulse are fixed up after the collide
//   k_node_field, k_collide_forced
//                 boxes whose beads cover much of the box: node velocities
//                 once per step for the beads' tables, and a collide after
//                 the coupling that takes the node impulses itself
//   k_stats*      FP64 conserved sums, mode variances, negative-population
//                 count; k_obs: these per box, and the chain's centre of mass,
//                 R_g^2, R_e^2 (Sec. III.A)
#include "lbmd_device.hpp"
#include "lbmd_kernels.hpp"

namespace lbd {

__device__ __forceinline__ uint32_t div_L(uint32_t r, int L, double inv_L, uint32_t* rem)
{
    uint32_t q = (uint32_t)((double)r * inv_L);
    int32_t rr = (int32_t)(r - q * (uint32_t)L);
    if (rr < 0) { q -= 1; rr += L; }
    else if (rr >= L) { q += 1; rr -= L; }
    *rem = (uint32_t)rr;
    return q;
}

// Index of the node r - c_i for every direction i (periodic), from the node's
// coordinates: the source of the population that arrives at r.
struct Upwind {
    uint32_t X[3], Y[3], Z[3];
    __device__ __forceinline__ Upwind(uint32_t x, uint32_t y, uint32_t z, uint32_t L)
    {
        const uint32_t LL = L * L;
        X[0] = x + 1 == L ? 0 : x + 1; X[1] = x; X[2] = x == 0 ? L - 1 : x - 1;
        Y[0] = (y + 1 == L ? 0 : y + 1) * L; Y[1] = y * L; Y[2] = (y == 0 ? L - 1 : y - 1) * L;
        Z[0] = (z + 1 == L ? 0 : z + 1) * LL; Z[1] = z * LL; Z[2] = (z == 0 ? L - 1 : z - 1) * LL;
    }
    // slot 0 holds coordinate + 1, slot 2 coordinate - 1: r - c_i uses slot c_i + 1
    __device__ __forceinline__ uint32_t src(int i) const { return X[cxv(i) + 1] + Y[cyv(i) + 1] + Z[czv(i) + 1]; }
};

template <typename R, bool NT>
__device__ __forceinline__ void gather_pre(const R* __restrict__ a, const Upwind& up, R d[19])
{
#pragma unroll
    for (int i = 0; i < 19; ++i) {
        const uint64_t q = pop_at(i, up.src(i));
        d[i] = NT ? __builtin_nontemporal_load(a + q) : a[q];
    }
}

// the pre-collision populations of node `up` with 32-bit offsets from the
// box's array (valid while that array is under 4 GiB): a uniform base and one
// 32-bit offset per load instead of 64-bit address arithmetic
template <typename R>
__device__ __forceinline__ void gather_pre32(const R* __restrict__ a, const Upwind& up, R d[19])
{
    const char* base = (const char*)a;
#pragma unroll
    for (int i = 0; i < 19; ++i) {
        const uint32_t s = up.src(i);
        const uint32_t e = ((s >> PTILE_LOG) * 19u + (uint32_t)i) * PTILE + (s & (PTILE - 1u));
        d[i] = *(const R*)(base + (uint64_t)(e * (uint32_t)sizeof(R)));
    }
}

__device__ __forceinline__ Upwind upwind_of(uint32_t r, int L, double inv_L)
{
    uint32_t x, y;
    const uint32_t q = div_L(r, L, inv_L, &x);
    const uint32_t z = div_L(q, L, inv_L, &y);
    return Upwind(x, y, z, (uint32_t)L);
}

// deferral segment of node `node` of box bx (its stamps sit at 2 * segment
// and 2 * segment + 1)
__device__ __forceinline__ uint32_t dseg_of(const BoxDev& bx, uint32_t node)
{
    return DSEG_PER_TILE * bx.tile_begin + node / DSEG;
}

// -------------------------------------------------------------- collide
// One tile of 256 nodes: gather the pre-collision populations (pull), collide
// with no impulse, write post-collision values aligned and non-temporal.
template <typename R>
__device__ __forceinline__ void collide_tile(const BoxDev* __restrict__ boxes, const CollideConst<R>* __restrict__ ccs,
                                             const uint32_t* __restrict__ tile_box, int fixed_box, uint32_t tile,
                                             const R* __restrict__ A, R* __restrict__ B, Ctrl* __restrict__ ctrl,
                                             uint32_t t, const uint32_t* __restrict__ defer, uint32_t lane)
{
    int bi;
    if (defer) {   // batched steps (every tile's box from tile_box)
        // a deferred segment (this wavefront's nodes) is collided after the
        // coupling, with its impulses (k_collide_deferred); the stamp load
        // goes out beside the box load
        const uint32_t w = __builtin_amdgcn_readfirstlane(lane / DSEG);   // wavefront-uniform: a scalar load
        const uint32_t st = defer[2u * (DSEG_PER_TILE * tile + w) + (t & 1u)];
        bi = (int)tile_box[tile];
        if (st == defer_stamp(t)) return;
    } else {
        bi = fixed_box >= 0 ? fixed_box : (int)tile_box[tile];
    }
    const BoxDev& bx = boxes[bi];
    const int L = bx.L;
    const uint32_t V = (uint32_t)L * L * L;
    const uint32_t r = (tile - bx.tile_begin) * 256u + lane;
    if (r >= V) return;
    const CollideConst<R> cc = ccs[bi];
    const Upwind up = upwind_of(r, L, bx.inv_L);
    R d[19];
    gather_pre<R, false>(A + bx.pop_off, up, d);
    R o[19];
    const uint32_t h = collide<R>(d, o, (R)0, (R)0, (R)0, cc, r, t, bx.seed, bx.box_id);
    R* b = B + bx.pop_off;
#pragma unroll
    for (int i = 0; i < 19; ++i) __builtin_nontemporal_store(o[i], b + pop_at(i, r));
    if (h) atomicOr(&ctrl->health, h);
}

// Launch shapes the autotuner chooses from: W caps the waves per SIMD (4..8);
// BT threads per block collide BT / 256 consecutive 256-node tiles (256, 512
// or 1024 nodes per block); PERSIST selects a grid of a few blocks per CU
// that strides over the tiles instead of one block per tile group.  Every
// node gets the same per-node arithmetic, so all shapes compute the same bits.
template <typename R, int W, bool PERSIST, int BT = 256>
__global__ __launch_bounds__(BT) __attribute__((amdgpu_waves_per_eu(1, W))) void k_collide(
    const BoxDev* __restrict__ boxes, const CollideConst<R>* __restrict__ ccs, const uint32_t* __restrict__ tile_box,
    int fixed_box, uint32_t tile0, uint32_t n_tiles, const R* __restrict__ A, R* __restrict__ B,
    Ctrl* __restrict__ ctrl, uint32_t s_off, const uint32_t* __restrict__ defer)
{
    constexpr uint32_t M = BT / 256;   // 256-node tiles per block
    const uint32_t t = ctrl->step + s_off;
    if constexpr (M == 1) {
        if (PERSIST) {
            for (uint32_t k = blockIdx.x; k < n_tiles; k += gridDim.x)
                collide_tile<R>(boxes, ccs, tile_box, fixed_box, tile0 + k, A, B, ctrl, t, defer, threadIdx.x);
        } else {
            collide_tile<R>(boxes, ccs, tile_box, fixed_box, tile0 + blockIdx.x, A, B, ctrl, t, defer, threadIdx.x);
        }
    } else {
        const uint32_t sub = threadIdx.x / 256u, lane = threadIdx.x % 256u;
        if (PERSIST) {
            for (uint32_t k = blockIdx.x * M + sub; k < n_tiles; k += gridDim.x * M)
                collide_tile<R>(boxes, ccs, tile_box, fixed_box, tile0 + k, A, B, ctrl, t, defer, lane);
        } else {
            const uint32_t k = blockIdx.x * M + sub;
            if (k < n_tiles) collide_tile<R>(boxes, ccs, tile_box, fixed_box, tile0 + k, A, B, ctrl, t, defer, lane);
        }
    }
}

// --------------------------------------------------------------- couple
struct ChainArgs {
    double* x; double* v; double* f; double* fc;   // [total beads][3]
    int32_t* nl_cnt; uint16_t* nl_idx; double* nl_x0; int nl_cap;
    unsigned long long* imp;   // dense impulse field, 3 per node (global node index), fixed point
    uint32_t* touched;         // per bead: local nodes it handed impulse to this step
    int32_t* touched_cnt;
    int touch_cap;             // slots per bead: 8 x (substeps + 1), one stencil change per substep at most
    uint32_t* nl_rebuilds;     // per box: neighbour-list builds so far (diagnostic)
    double* vhist; int hist_len; uint64_t total_beads;
    double* tape;              // non-null while replaying a window segment: per substep and bead,
                               // TAPE_REC doubles (see k_couple)
    double* tape_x0;           // with tape: the step's starting x, v (at tape_vo), f (at tape_fo)
    uint64_t tape_vo, tape_fo;
    uint32_t* defer;           // non-null when the step defers tiles: per collide tile, the stamp of
                               // the last step that deferred it
    uint32_t* dclaim;          // per collide tile: stamp of the last step that listed it
    uint32_t* defer_list; uint32_t defer_cap;
    uint32_t* ovf; uint32_t ovf_cap;   // (bead, local node) pairs outside the deferred tiles
    uint32_t* ovm;             // per global node: stamp of the last step that listed it in ovf
};

// node velocities (MD units) of the 8 stencil nodes from the frozen populations;
// the loads of NB nodes are issued before any of them is used (NB = 8: one
// round trip to memory, for register-rich callers)
template <typename R, typename U, int NB>
__device__ __forceinline__ void stencil_velocities(const R* __restrict__ a, const int i0[3], int L,
                                                   double rho0, double inv_tau, U u[8][3])
{
    static_assert(NB == 1 || NB == 2 || NB == 4 || NB == 8, "NB divides 8");
#pragma unroll
    for (int k0 = 0; k0 < 8; k0 += NB) {
        R d[NB][19];
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            const int kk = k0 + k;
            const int ix = i0[0] + (kk & 1), iy = i0[1] + ((kk >> 1) & 1), iz = i0[2] + ((kk >> 2) & 1);
            const Upwind up((uint32_t)(ix >= L ? ix - L : ix), (uint32_t)(iy >= L ? iy - L : iy),
                            (uint32_t)(iz >= L ? iz - L : iz), (uint32_t)L);
            gather_pre<R, false>(a, up, d[k]);
        }
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            double rho = 0.0, jx = 0.0, jy = 0.0, jz = 0.0;
#pragma unroll
            for (int i = 0; i < 19; ++i) {
                const double di = (double)d[k][i];
                rho += di;
                if (cxv(i)) jx += cxv(i) * di;
                if (cyv(i)) jy += cyv(i) * di;
                if (czv(i)) jz += czv(i) * di;
            }
            rho += rho0;
            u[k0 + k][0] = (U)(jx / rho * inv_tau);
            u[k0 + k][1] = (U)(jy / rho * inv_tau);
            u[k0 + k][2] = (U)(jz / rho * inv_tau);
        }
    }
}

// node at (ix, iy, iz), each at most one box edge outside
__device__ __forceinline__ uint32_t node_of(int ix, int iy, int iz, int L)
{
    ix = ix >= L ? ix - L : (ix < 0 ? ix + L : ix);
    iy = iy >= L ? iy - L : (iy < 0 ? iy + L : iy);
    iz = iz >= L ? iz - L : (iz < 0 ? iz + L : iz);
    return (uint32_t)ix + (uint32_t)L * ((uint32_t)iy + (uint32_t)L * (uint32_t)iz);
}

// fluid velocity of one node in MD units (u = j / rho / tau_lb) from its
// gathered pre-collision deviations
template <typename R>
__device__ __forceinline__ void node_velocity(const R d[19], double rho0, double inv_tau, R u[3])
{
    double rho = 0.0, jx = 0.0, jy = 0.0, jz = 0.0;
#pragma unroll
    for (int i = 0; i < 19; ++i) {
        const double di = (double)d[i];
        rho += di;
        if (cxv(i)) jx += cxv(i) * di;
        if (cyv(i)) jy += cyv(i) * di;
        if (czv(i)) jz += czv(i) * di;
    }
    rho += rho0;
    u[0] = (R)(jx / rho * inv_tau);
    u[1] = (R)(jy / rho * inv_tau);
    u[2] = (R)(jz / rho * inv_tau);
}

constexpr int MAXB = 1024;
constexpr double NL_SKIN = 0.5;

// first and last bead of bead b's chain: a box's beads form chains of
// chain_len consecutive indices (one chain, or the several chains of a
// semidilute solution, Sec. III.C)
struct ChainSpan { int lo, hi; };
__device__ __forceinline__ ChainSpan chain_span(const BoxDev& bx, int b)
{
    const int n = bx.chain_len;
    const int lo = b - b % n;
    return ChainSpan{lo, lo + n - 1};
}

// FENE force on bead b from its bonded neighbours, b - 1 and b + 1 when they
// are on its chain (Sec. II.A), unwrapped separations
__device__ __forceinline__ uint32_t fene_force(const BoxDev& bx, int b, ChainSpan sp, const double x[3],
                                               const double* xs, double F[3])
{
    uint32_t hb = 0;
#pragma unroll
    for (int side = 0; side < 2; ++side) {
        const int j = side ? b + 1 : b - 1;
        if (j < sp.lo || j > sp.hi) continue;
        const double d0 = x[0] - xs[3 * j], d1 = x[1] - xs[3 * j + 1], d2 = x[2] - xs[3 * j + 2];
        const double r2 = d0 * d0 + d1 * d1 + d2 * d2;
        double den = 1.0 - r2 * bx.inv_r0sq;
        if (!(den > 0.0)) { hb |= H_FENE; den = 1e-12; }
        const double gf = -bx.k_fene / den;
        F[0] += gf * d0; F[1] += gf * d1; F[2] += gf * d2;
    }
    return hb;
}

// purely repulsive LJ on bead b from beads j0, j0+T, j0+2T, j0+3T (those < N
// and != b): the four separations are independent, so their latencies overlap;
// the forces are added in ascending j.
template <typename IDX>
__device__ __forceinline__ void wca_add4(const double x[3], const double* xs, IDX jof, int k0, int kend, int step,
                                         int b, double Ld, double iL, double rc2, double sigsq, double eps24,
                                         double F[3])
{
    double d[4][3], r2[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int k = k0 + u * step;
        const int j = k < kend ? jof(k) : b;
        d[u][0] = x[0] - xs[3 * j]; d[u][1] = x[1] - xs[3 * j + 1]; d[u][2] = x[2] - xs[3 * j + 2];
        d[u][0] -= Ld * rint(d[u][0] * iL); d[u][1] -= Ld * rint(d[u][1] * iL); d[u][2] -= Ld * rint(d[u][2] * iL);
        r2[u] = j == b ? rc2 : d[u][0] * d[u][0] + d[u][1] * d[u][1] + d[u][2] * d[u][2];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        if (r2[u] < rc2) {
            const double ir2 = 1.0 / r2[u];
            const double s2 = sigsq * ir2;
            const double s6 = s2 * s2 * s2;
            const double gf = eps24 * s6 * (2.0 * s6 - 1.0) * ir2;
            F[0] += gf * d[u][0]; F[1] += gf * d[u][1]; F[2] += gf * d[u][2];
        }
    }
}

// purely repulsive LJ on bead b from bead j (minimum image), cut at 2^(1/6) sigma
__device__ __forceinline__ void wca_add(const double x[3], const double* xs, int j, double Ld, double iL,
                                        double rc2, double sigsq, double eps24, double F[3])
{
    double d0 = x[0] - xs[3 * j], d1 = x[1] - xs[3 * j + 1], d2 = x[2] - xs[3 * j + 2];
    d0 -= Ld * rint(d0 * iL); d1 -= Ld * rint(d1 * iL); d2 -= Ld * rint(d2 * iL);
    const double r2 = d0 * d0 + d1 * d1 + d2 * d2;
    if (r2 < rc2) {
        const double ir2 = 1.0 / r2;
        const double s2 = sigsq * ir2;
        const double s6 = s2 * s2 * s2;
        const double gf = eps24 * s6 * (2.0 * s6 - 1.0) * ir2;
        F[0] += gf * d0; F[1] += gf * d1; F[2] += gf * d2;
    }
}

// initial last-force of every bead: the conservative force at the start positions
__global__ __launch_bounds__(1024) void k_init_forces(const BoxDev* __restrict__ boxes,
                                                      const int32_t* __restrict__ couple_list,
                                                      double* __restrict__ xg, double* __restrict__ fg,
                                                      Ctrl* __restrict__ ctrl)
{
    __shared__ double xs[3 * MAXB];
    const BoxDev& bx = boxes[couple_list[blockIdx.x]];
    const int N = bx.N, b = threadIdx.x;
    const uint64_t g = bx.bead_off + b;
    double x[3] = {0, 0, 0};
    if (b < N)
        for (int c = 0; c < 3; ++c) { x[c] = xg[3 * g + c]; xs[3 * b + c] = x[c]; }
    __syncthreads();
    if (b < N) {
        double F[3] = {0, 0, 0};
        uint32_t hb = fene_force(bx, b, chain_span(bx, b), x, xs, F);
        double W[3] = {0, 0, 0};
        for (int j = 0; j < N; ++j)
            if (j != b) wca_add(x, xs, j, (double)bx.L, bx.inv_L, bx.rc2, bx.sigsq, 24.0 * bx.eps, W);
        for (int c = 0; c < 3; ++c) fg[3 * g + c] = F[c] + W[c];
        if (hb) atomicOr(&ctrl->health, hb);
    }
}

// value of v in another lane of the same 16-lane row, by a DPP lane move of
// both 32-bit halves (CTRL: a gfx9 DPP control; every source lane is active)
template <int CTRL>
__device__ __forceinline__ double dpp_from(double v)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xF, 0xF, false);
    return __hiloint2double(hi, lo);
}

// value of component c's lane (c = 0, 1, 2) of the quad
template <int C>
__device__ __forceinline__ double quad_value(double v) { return dpp_from<C * 0x55>(v); }

// Repulsive LJ on a bead at x from up to U of its partners j[u] (those with
// ok[u]): the separations and the two divisions of all U run side by side,
// without a branch each; the forces are added in order of u.
template <int U>
__device__ __forceinline__ void wca_add(const double x[3], const double* xs, const int j[U], const bool ok[U],
                                        double Ld, double iL, double rc2, double sigsq, double eps24, double F[3])
{
#pragma clang fp contract(on)
    double d[U][3], r2[U];
    bool hit[U], any = false;
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            d[u][c] = x[c] - xs[3 * j[u] + c];
            d[u][c] -= Ld * rint(d[u][c] * iL);
        }
        r2[u] = d[u][0] * d[u][0] + d[u][1] * d[u][1] + d[u][2] * d[u][2];
        hit[u] = ok[u] && r2[u] < rc2;
        any |= hit[u];
    }
    if (any) {
        double gf[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const double ir2 = 1.0 / (hit[u] ? r2[u] : 1.0);
            const double s2 = sigsq * ir2;
            const double s6 = s2 * s2 * s2;
            gf[u] = eps24 * s6 * (2.0 * s6 - 1.0) * ir2;
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (hit[u]) {
#pragma unroll
                for (int c = 0; c < 3; ++c) F[c] += gf[u] * d[u][c];
            }
    }
}

// The substeps of one LB step for a chain of at most BIG_CHAIN beads, by one
// workgroup: T lanes per bead (a function of N only), bead b = thread / T.
// What bounds it is the serial chain of a substep (drift, positions to LDS,
// barrier, pair forces, interpolation, kick) at one or a few wavefronts per
// SIMD, so the lanes share a bead's work:
//   - lane l holds component c = l mod 4 of the bead (position, velocity,
//     force, the eight stencil velocities and impulses); the fourth lane of a
//     quad repeats the third, further quads the first;
//   - the partners of the pair forces are split over `cls` lanes (the 16, 8,
//     4, 2 or 1 lanes that 256 threads hold per bead): lane l sums those with
//     j = l (mod cls), ascending, then a butterfly adds the lanes' sums.
//     Chains above 64 beads have 4 lanes each and cls = 2 or 1: lanes repeat
//     a class rather than split it further, which would change the sums;
//   - lanes 0 and 1 take the bonds to b - 1 and b + 1;
//   - the noise: lane l draws the words of substeps l, l + T, ..., handed
//     over by a shuffle ahead of the barrier;
//   - a new stencil's populations are gathered by corner: lane l takes corners
//     l mod T8, + T8, ... (T8 = min(T, 8)).
// Lanes exchange values by DPP moves within the quad (a few cycles, where a
// shuffle through LDS takes ~60 per stage).  Positions alternate between two
// LDS buffers, so a substep has one barrier.
// Pair lists (chains above 16 beads): the partners of a lane's class within
// the list radius (cut-off plus NL_SKIN) are bits of one 64-bit word (four
// words for cls = 1), set at the first substep and again whenever a coordinate
// of some bead has moved more than half the skin / sqrt(3); the exact cut-off
// decides, so the list's age does not show in the bits.
// Measured per substep in a one-kernel step (24^3, kT = 0.01, dt = 0.005, list
// builds and new stencils included): 16 beads 0.83 us, 32 1.34, 64 1.9, 128 2.8,
// 256 6.5.  Near rest, where those are rare: 16 beads 0.84 us, 32 1.15, 64 1.5;
// lanes that each repeated the whole bead but its pair forces took 2.1, 1.9 and
// 2.0 us there (alone).

// the same value, unknown to the compiler: keeps the addresses of rare paths
// from being computed ahead of the substep loop and held through it
__device__ __forceinline__ int here(int v)
{
    asm volatile("" : "+v"(v));
    return v;
}
__device__ __forceinline__ double here(double uniform)
{
    asm volatile("" : "+s"(uniform));
    return uniform;
}

template <int MB>   // most beads
struct ChainLds {
    union {
        struct {
            double xs[2][3 * MB];   // positions of this and the previous substep
        };
        uint32_t hash[MB > 64 ? 4096 : 1024];   // after the substeps: nodes set aside for the next step
    };
    int moved[3];                  // per substep mod 3: a bead moved past half the skin
    uint32_t n_ovf, n_next;        // one-kernel steps: impulses outside the set-aside nodes, next step's such nodes
};
// ONE: the step is one kernel (k_step): `mask` holds this step's set-aside
// nodes, impulses on other nodes are listed in the box's touched slots,
// sh.n_ovf of them; xe, ve return the bead's end position and velocity.
template <typename R, int T, bool ONE, int MB>
__device__ __forceinline__ uint32_t chain_substeps(const BoxDev& bx, const R* __restrict__ A, const ChainArgs& ca,
                                                   uint32_t t, ChainLds<MB>& sh,
                                                   const unsigned long long* __restrict__ mask, double xe[3],
                                                   double ve[3])
{
#pragma clang fp contract(on)
    constexpr int T8 = T < 8 ? T : 8, NC = 8 / T8;   // corners gathered per lane
    constexpr bool LISTS = T < 16;                   // T = 16: one partner per lane at most
    constexpr int U = T == 4 ? 2 : 1;                // partners tested side by side
    constexpr int NW = MB > 64 && T == 4 ? 4 : 1;    // list words per lane
    constexpr int NQ = T / 4;                        // quads per bead
    const int N = bx.N, L = bx.L;
    const int cls = T > 4 || MB <= 64 ? T : (N <= 64 ? 4 : (N <= 128 ? 2 : 1));
    const int b = (int)threadIdx.x / T, lane = (int)threadIdx.x % T;
    const bool act = b < N;
    const int c = (lane & 3) < 3 ? lane & 3 : 2;   // this lane's component
    const bool own = lane < 3;                     // the lanes that store the bead
    const uint64_t g = bx.bead_off + (uint64_t)(act ? b : 0);
    const ChainSpan sp = chain_span(bx, act ? b : 0);
    const double Ld = (double)L, iL = bx.inv_L;
    const double dt = bx.dt, hdt_m = 0.5 * dt / bx.mass;
    const double eps24 = 24.0 * bx.eps;
    const R* a = A + bx.pop_off;
    const bool off32 = pop_elems_of((uint64_t)L * L * L) * sizeof(R) < (1ull << 32);
    // bonded partners (the bead itself, a zero separation, where there is none)
    const int jb0 = act && b > sp.lo ? b - 1 : (act ? b : 0), jb1 = act && b < sp.hi ? b + 1 : (act ? b : 0);
    const int jb = lane & 1 ? jb1 : jb0;
    if (threadIdx.x < 3) sh.moved[threadIdx.x] = 0;

    double x = 0.0, v = 0.0, f = 0.0, fc = 0.0;
    if (act) {
        x = ca.x[3 * g + c]; v = ca.v[3 * g + c]; f = ca.f[3 * g + c];
        if (ca.tape_x0 && own) {   // the step's starting beads, for the adjoint
            ca.tape_x0[3 * g + c] = x;
            ca.tape_x0[ca.tape_vo + 3 * g + c] = v;
            ca.tape_x0[ca.tape_fo + 3 * g + c] = f;
        }
    }
    int cb = -1;                  // base cell of the cached stencil, this component
    uint32_t base = 0;            // its base node, all components
    // component c of the stencil's node velocities (MD units), kept in the
    // storage precision: FP32 storage carries no more digits than that
    R cu[8];
    double acc[8];                // impulse accumulated on them (MD units)
    uint32_t aside = 0;           // ONE: bit k: corner k's node is set aside
    uint32_t hbits = 0;
    int tcnt = 0;
    double x0 = 0.0;              // position at the last list build
    unsigned long long nl[NW] = {};   // partners of the lane's class within the list radius
    U4 pw{0, 0, 0, 0};            // noise words of this lane's substep

    // hand the accumulated impulses over, quad by quad: fixed-point adds that
    // nothing waits on; the bead lists the nodes
    auto flush = [&]() __attribute__((always_inline)) {
        const int lane = here((int)threadIdx.x % T), c = (lane & 3) < 3 ? lane & 3 : 2;
        const uint64_t g = bx.bead_off + (uint64_t)here(b);
        const double tau = here(bx.tau_lb);
        const uint32_t LL = (uint32_t)L * (uint32_t)L;
        const uint32_t bz = base / LL, rem = base - bz * LL, by = rem / (uint32_t)L, bx_ = rem - by * (uint32_t)L;
        const int q = lane >> 2;
#pragma unroll
        for (int kk = 0; kk < 8 / NQ; ++kk) {
            // quad q takes corners q, q + NQ, ...
            const double a0 = acc[NQ * kk], a1 = acc[NQ * kk + (NQ > 1 ? 1 : 0)], a2 = acc[NQ * kk + (NQ > 2 ? 2 : 0)],
                         a3 = acc[NQ * kk + (NQ > 2 ? 3 : 0)];
            const double ak = q == 0 ? a0 : (q == 1 ? a1 : (q == 2 ? a2 : a3));
            const int k = NQ * kk + q;
            const uint32_t node = node_of((int)bx_ + (k & 1), (int)by + ((k >> 1) & 1), (int)bz + (k >> 2), L);
            if ((lane & 3) < 3) {
                double m = ak * tau;      // lattice momentum units
                if (!(fabs(m) < IMP_MAX)) { hbits |= H_FIXED; m = 0.0; }
                atomicAdd(ca.imp + 3 * (bx.node_off + node) + c, (unsigned long long)(long long)llrint(m * IMP_SCALE));
            } else if (ONE) {
                // at most 8 per bead and stencil, so the box's slots hold them
                if (!((aside >> k) & 1u)) ca.touched[bx.bead_off * ca.touch_cap + atomicAdd(&sh.n_ovf, 1u)] = node;
            } else {
                const int slot = tcnt + k;
                if (slot < ca.touch_cap) ca.touched[g * ca.touch_cap + slot] = node;
                else hbits |= H_TABLE;
            }
        }
        tcnt += 8;
    };

    for (int s = 0; s < bx.substeps; ++s) {
        double* xs = sh.xs[s & 1];
        double fr = 0.0, nz = 0.0;
        int ii = 0;
        if (act) {
            v += f * hdt_m;
            x += v * dt;
            if (own) {
                xs[3 * b + c] = x;
                if (LISTS && s > 0 && fabs(x - x0) > 0.5 * NL_SKIN * 0.577) sh.moved[s % 3] = 1;
            }
            // ahead of the barrier: what depends on the bead alone
            if (s % T == 0) pw = philox10(U4{(uint32_t)b, t, (1u << 16) | (uint32_t)(s + lane), 0u}, bx.seed, bx.box_id);
            const uint32_t w0 = __shfl(pw.x, s % T, T), w1 = __shfl(pw.y, s % T, T), w2 = __shfl(pw.z, s % T, T);
            nz = unit_noise<double>(c == 0 ? w0 : (c == 1 ? w1 : w2));
            // stencil of the bead: nodes at integer coordinates, periodic
            const double xt = x - Ld * floor(x * iL);
            const double fl = floor(xt);
            fr = xt - fl;
            ii = on_edge((int)fl, L);
        }
        __syncthreads();
        // the same for every thread; flag s + 2 (mod 3) was last read a
        // substep ago and is next set after the next barrier
        const bool rebuild = LISTS && (s == 0 || sh.moved[s % 3] != 0);
        if (LISTS && threadIdx.x == 0) sh.moved[(s + 2) % 3] = 0;
        if (act) {
            const double xb[3] = {quad_value<0>(x), quad_value<1>(x), quad_value<2>(x)};
            // bond of lanes 0 and 1 (FENE, unwrapped separations), then both
            // bonds' component c in each lane
            double Ff;
            {
                const double d0 = xb[0] - xs[3 * jb], d1 = xb[1] - xs[3 * jb + 1], d2 = xb[2] - xs[3 * jb + 2];
                const double r2 = d0 * d0 + d1 * d1 + d2 * d2;
                double den = 1.0 - r2 * bx.inv_r0sq;
                if (!(den > 0.0)) { hbits |= H_FENE; den = 1e-12; }
                const double gf = -bx.k_fene / den;
                const double e0 = x - xs[3 * jb0 + c], e1 = x - xs[3 * jb1 + c];
                Ff = quad_value<0>(gf) * e0;
                Ff += quad_value<1>(gf) * e1;
            }
            // repulsive LJ over the partners of this lane's class
            double W[3] = {0, 0, 0};
            if (LISTS) {
                if (rebuild) {
                    x0 = x;
                    // list radius, a hair above cut-off plus skin so that rounding cannot
                    // drop a partner that comes within the cut-off
                    const double rl = sqrt(here(bx.rc2)) + NL_SKIN + 1e-6;
                    const double rl2 = rl * rl;
                    // cls = T: bit m is partner lane + T m; cls = 2: (lane mod 2) + 2 m, half of the
                    // word by each of two lanes; cls = 1: word l is partners 64 l .. 64 l + 63, by lane l
                    const int j0 = cls == 1 ? 64 * lane : (cls == 2 ? (lane & 1) + 64 * (lane >> 1) : lane);
                    const int nj = cls == 1 ? 64 : (cls == 2 ? 32 : (N - lane + T - 1) / T);
                    unsigned long long found = 0ull;
#pragma unroll 2
                    for (int m = 0; m < nj; ++m) {
                        const int j = j0 + cls * m < N ? j0 + cls * m : b;
                        double d0 = xb[0] - xs[3 * j], d1 = xb[1] - xs[3 * j + 1], d2 = xb[2] - xs[3 * j + 2];
                        d0 -= Ld * rint(d0 * iL); d1 -= Ld * rint(d1 * iL); d2 -= Ld * rint(d2 * iL);
                        if (j != b && d0 * d0 + d1 * d1 + d2 * d2 < rl2) found |= 1ull << m;
                    }
                    if (cls == T) {
                        nl[0] = found;
                    } else if (cls == 2) {
                        const unsigned long long lo = __shfl(found, lane & 1, T), hi = __shfl(found, (lane & 1) + 2, T);
                        nl[0] = lo | (hi << 32);
                    } else {
#pragma unroll
                        for (int w = 0; w < NW; ++w) nl[w] = __shfl(found, w, T);
                    }
                }
                const int jl = cls == 1 ? 0 : lane & (cls - 1);
                auto pairs = [&](unsigned long long m, int j0) __attribute__((always_inline)) {
                    while (m) {
                        int j[U];
                        bool ok[U];
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            ok[u] = m != 0ull;
                            j[u] = ok[u] ? j0 + cls * (__ffsll((long long)m) - 1) : b;
                            m &= m - 1ull;
                        }
                        wca_add<U>(xb, xs, j, ok, Ld, iL, bx.rc2, bx.sigsq, eps24, W);
                    }
                };
                pairs(nl[0], jl);
                if (NW > 1 && cls == 1) {
                    pairs(nl[NW > 1 ? 1 : 0], 64);
                    pairs(nl[NW > 2 ? 2 : 0], 128);
                    pairs(nl[NW > 3 ? 3 : 0], 192);
                }
            } else {
                const int j[U] = {lane < N ? lane : b};
                const bool ok[U] = {j[0] != b};
                wca_add<U>(xb, xs, j, ok, Ld, iL, bx.rc2, bx.sigsq, eps24, W);
            }
            // the class sums: each stage adds the same two values in either
            // order, so every lane gets the same bits
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                if (T > 4 || cls >= 2) W[d] += dpp_from<0xB1>(W[d]);                  // quad_perm [1,0,3,2]
                if (T > 4 || cls >= 4) W[d] += dpp_from<0x4E>(W[d]);                  // quad_perm [2,3,0,1]
                if (T >= 8) W[d] += dpp_from<0x141>(W[d]);                   // row_half_mirror
                if (T >= 16) W[d] += dpp_from<0x140>(W[d]);                  // row_mirror
            }
            const double F = Ff + (c == 0 ? W[0] : (c == 1 ? W[1] : W[2]));
            // a change in any of the quad's components
            const int chg = ii != cb ? 1 : 0;
            if (__builtin_amdgcn_update_dpp(0, chg, 0x00, 0xF, 0xF, false) |
                __builtin_amdgcn_update_dpp(0, chg, 0x55, 0xF, 0xF, false) |
                __builtin_amdgcn_update_dpp(0, chg, 0xAA, 0xF, 0xF, false)) {
                if (s > 0) flush();
                const int i0[3] = {__builtin_amdgcn_update_dpp(0, ii, 0x00, 0xF, 0xF, false),
                                   __builtin_amdgcn_update_dpp(0, ii, 0x55, 0xF, 0xF, false),
                                   __builtin_amdgcn_update_dpp(0, ii, 0xAA, 0xF, 0xF, false)};
                base = (uint32_t)i0[0] + (uint32_t)L * ((uint32_t)i0[1] + (uint32_t)L * (uint32_t)i0[2]);
                cb = ii;
                const int kc = lane & (T8 - 1);
                const double inv_tau = 1.0 / here(bx.tau_lb);
                R u[NC][3];
                uint32_t in = 0;
                auto at_corner = [&](int k) __attribute__((always_inline)) {
                    const int ix = i0[0] + (k & 1), iy = i0[1] + ((k >> 1) & 1), iz = i0[2] + (k >> 2);
                    const uint32_t nx = ix >= L ? ix - L : ix, ny = iy >= L ? iy - L : iy, nz_ = iz >= L ? iz - L : iz;
                    if (ONE) {
                        const uint32_t node = nx + (uint32_t)L * (ny + (uint32_t)L * nz_);
                        in |= (uint32_t)((mask[dseg_of(bx, node)] >> (node % DSEG)) & 1ull) << k;
                    }
                    return Upwind(nx, ny, nz_, (uint32_t)L);
                };
                // one corner's loads at a time: those of two (T = 4) would
                // cost the loop its registers
#pragma unroll
                for (int kk = 0; kk < NC; ++kk) {
                    R d[19];
                    const Upwind up = at_corner(kc + kk * T8);
                    if (off32) gather_pre32<R>(a, up, d);
                    else gather_pre<R, false>(a, up, d);
                    node_velocity<R>(d, bx.rho0, inv_tau, u[kk]);
                    __builtin_amdgcn_sched_barrier(0);
                }
                // corner k sits in slot k / T8 of lane k mod T8
                aside = 0;
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const R u0 = __shfl(u[k / T8][0], k % T8, T), u1 = __shfl(u[k / T8][1], k % T8, T),
                            u2 = __shfl(u[k / T8][2], k % T8, T);
                    cu[k] = c == 0 ? u0 : (c == 1 ? u1 : u2);
                    acc[k] = 0.0;
                    if (ONE) aside |= __shfl(in, k % T8, T) & (1u << k);
                }
            }
            const double fx = quad_value<0>(fr), fy = quad_value<1>(fr), fz = quad_value<2>(fr);
            double wt[8], ub = 0.0;
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                wt[k] = ((k & 1) ? fx : 1.0 - fx) * (((k >> 1) & 1) ? fy : 1.0 - fy) * ((k >> 2) ? fz : 1.0 - fz);
                ub += wt[k] * (double)cu[k];
            }
            const double fric = bx.zeta * (v - ub);
            fc = fma(bx.bead_noise, nz, -fric);
            if (ca.tape && own) {   // substep record for the adjoint: x1, v1, fc, base cell, fractions, node velocities
                double* tp = ca.tape + ((uint64_t)s * ca.total_beads + bx.bead_off + (uint64_t)here(b)) * TAPE_REC;
                tp[c] = x; tp[3 + c] = v; tp[6 + c] = fc; tp[9 + c] = (double)ii; tp[12 + c] = fr;
#pragma unroll
                for (int k = 0; k < 8; ++k) tp[15 + 3 * k + c] = (double)cu[k];
            }
            f = F + fc;
            v += f * hdt_m;
#pragma unroll
            for (int k = 0; k < 8; ++k) acc[k] -= wt[k] * fc * dt;
        }
    }
    if (act) {
        flush();
        if (own) {
            const uint64_t g = bx.bead_off + (uint64_t)here(b);
            if (!ONE && lane == 0) ca.touched_cnt[g] = tcnt < ca.touch_cap ? tcnt : ca.touch_cap;
            ca.x[3 * g + c] = x; ca.v[3 * g + c] = v; ca.f[3 * g + c] = f; ca.fc[3 * g + c] = fc;
            if (ca.vhist) ca.vhist[((uint64_t)(t % (uint32_t)ca.hist_len) * ca.total_beads + g) * 3 + c] = v;
        }
    }
    if (ONE) {
        xe[0] = quad_value<0>(x); xe[1] = quad_value<1>(x); xe[2] = quad_value<2>(x);
        ve[0] = quad_value<0>(v); ve[1] = quad_value<1>(v); ve[2] = quad_value<2>(v);
    }
    return act ? hbits : 0u;
}

// the coupling stage of one box per workgroup: couple_T lanes per bead
template <typename R, int MAXT>
__global__ __launch_bounds__(MAXT) void k_couple(const BoxDev* __restrict__ boxes,
                                                 const int32_t* __restrict__ couple_list,
                                                 const R* __restrict__ A, ChainArgs ca,
                                                 Ctrl* __restrict__ ctrl, uint32_t s_off)
{
    __shared__ ChainLds<MAXT / 4> sh;
    __builtin_amdgcn_s_setprio(3);   // latency-bound chain beside the bandwidth-bound collide
    const BoxDev bx = boxes[couple_list[blockIdx.x]];   // a copy: its fields stay in registers across the substeps
    const uint32_t t = ctrl->step + s_off;
    uint32_t hbits;
    double xe[3], ve[3];
    if (bx.couple_T == 4) hbits = chain_substeps<R, 4, false>(bx, A, ca, t, sh, nullptr, xe, ve);
    else if (bx.couple_T == 8) hbits = chain_substeps<R, 8, false>(bx, A, ca, t, sh, nullptr, xe, ve);
    else hbits = chain_substeps<R, 16, false>(bx, A, ca, t, sh, nullptr, xe, ve);
    if (hbits) atomicOr(&ctrl->health, hbits);
}

// ------------------------------------------------- couple, large chains
// Chains above 256 beads take three launches per LB step, on one stream:
//   k_near_nodes  every bead's 3x3x3 nodes around its nearest node: the node
//                 velocities (MD units), one thread per (bead, node), so all
//                 the population loads of the stage go out in one wave;
//   k_chain_wg    one workgroup of up to 1024 threads per box, one thread
//                 per bead, every MD substep in one launch.  Positions,
//                 neighbour lists, the positions they were built at and the
//                 cell buckets of the list build live in LDS (156 KB for 1024
//                 beads, 90 KB for 512); each
//                 bead's stencil velocities in
//                 registers, refilled from the 3x3x3 table when the bead
//                 changes cell.  Per substep each bead writes one record
//                 (fractions, coupling force, base cell) instead of handing
//                 impulses over, so no atomic traffic sits in the barrier-
//                 synchronised substep loop;
//   k_spread      one thread per (bead, stencil corner) turns the records into
//                 node impulses: the same accumulation per stencil as the
//                 one-workgroup path of small chains, then one fixed-point
//                 atomic per component and stencil.
constexpr int WG_MAXB = 1024;
constexpr int NEAR = 27;    // nodes in the table of one bead

// Neighbour-list build over cells: nc cells per axis, each at least the list
// radius wide (plus a margin far above rounding), so every partner within the
// radius lies in the 3x3x3 cells around a bead's own.  A cell's bucket is its
// coordinates mod 16 (4096 buckets): the 27 cells around any cell land in 27
// distinct buckets when nc <= 16, or when nc mod 16 is neither 1 nor 2, which
// list_cells ensures (it keeps nc mod 8 off 1 and 2 above 8 by taking fewer,
// wider cells).  Beads of other cells that share a bucket fail the distance
// test.  The test runs in FP32 on positions wrapped into the box, against a
// radius 1e-3 above the list radius: an FP32 rounding of the coordinates
// (under 2.5e-4 for L <= 1625) cannot drop a partner, and the few extra
// partners are skipped by the force loop's exact cut-off test.
constexpr int NBK = 4096;
constexpr int SORT_REGS = 16;   // lists up to this long are sorted in registers
constexpr double NL_FP32_MARGIN = 1e-3;
__device__ __forceinline__ int list_cells(int L, double rl)
{
    int nc = (int)floor((double)L / (rl + 1e-6));
    if (nc > 8 && (nc % 8 == 1 || nc % 8 == 2)) nc -= nc % 8;
    return nc;
}
__device__ __forceinline__ int wrap_cell(int q, int nc) { return q < 0 ? q + nc : (q >= nc ? q - nc : q); }
__device__ __forceinline__ int bucket_of(int cx, int cy, int cz) { return (cx & 15) | ((cy & 15) << 4) | ((cz & 15) << 8); }

// dense boxes: the velocity of every node, once per LB step, so that their
// beads' tables read 3 values per node instead of gathering 19 populations
// (the tables of a dense box cover it several times over)
template <typename R>
__global__ __launch_bounds__(256) void k_node_field(const BoxDev* __restrict__ boxes,
                                                    const int32_t* __restrict__ list, const R* __restrict__ A,
                                                    R* __restrict__ field)
{
    const BoxDev& bx = boxes[list[blockIdx.y]];
    if (!bx.dense) return;
    const int L = bx.L;
    const uint32_t V = (uint32_t)L * L * L;
    const uint32_t r = blockIdx.x * 256u + threadIdx.x;
    if (r >= V) return;
    const Upwind up = upwind_of(r, L, bx.inv_L);
    R d[19];
    gather_pre<R, false>(A + bx.pop_off, up, d);
    R u[3];
    node_velocity<R>(d, bx.rho0, 1.0 / bx.tau_lb, u);
    R* o = field + 3 * (bx.field_off + r);
    o[0] = u[0]; o[1] = u[1]; o[2] = u[2];
}

// the box fields a fix-up uses, read once
struct FixBox {
    int L;
    uint32_t seed, box_id;
    uint64_t pop_off, node_off;
    double inv_L;
};
__device__ __forceinline__ FixBox fix_box(const BoxDev& bx)
{
    return FixBox{bx.L, bx.seed, bx.box_id, bx.pop_off, bx.node_off, bx.inv_L};
}

// fix-up of one node after the plain collide: defined with the fix-up kernels
template <typename R>
__device__ __forceinline__ void fixup_node(const FixBox& bx, const CollideConst<R>& cc, uint32_t r,
                                           unsigned long long* __restrict__ imp, uint32_t* __restrict__ claim,
                                           const R* __restrict__ A, R* __restrict__ B, Ctrl* __restrict__ ctrl,
                                           uint32_t t, int keep_imp);

// the same fix-up (impulses left in the field), the node claimed before its
// populations are read: fewer live registers, for a rare path inside a
// bandwidth-bound kernel
template <typename R>
__device__ __forceinline__ void fixup_node_claim_first(const BoxDev& bx, const CollideConst<R>* __restrict__ ccs,
                                                       int bi, uint32_t r, const unsigned long long* __restrict__ imp,
                                                       uint32_t* __restrict__ claim, const R* __restrict__ A,
                                                       R* __restrict__ B, Ctrl* __restrict__ ctrl, uint32_t t)
{
    const uint64_t node = bx.node_off + r;
    if (atomicExch(&claim[node], t + 1u) == t + 1u) return;   // another caller took this node
    R d[19];
    gather_pre<R, false>(A + bx.pop_off, upwind_of(r, bx.L, bx.inv_L), d);
    const unsigned long long* q = imp + 3 * node;
    const R fx = (R)((double)(long long)q[0] * IMP_INV_SCALE), fy = (R)((double)(long long)q[1] * IMP_INV_SCALE),
            fz = (R)((double)(long long)q[2] * IMP_INV_SCALE);
    R o[19];
    const uint32_t h = collide<R>(d, o, fx, fy, fz, ccs[bi], r, t, bx.seed, bx.box_id);
    R* b = B + bx.pop_off;
#pragma unroll
    for (int i = 0; i < 19; ++i) b[pop_at(i, r)] = o[i];
    if (h) atomicOr(&ctrl->health, h);
}

// The node table of the step, one (bead, table node) item per thread: item
// `item` of list entry `li`.  With Aprev (batched steps that defer tiles,
// from the second step of a run of steps on) it also finishes the previous
// step first: the impulses that landed outside that step's deferred tiles are
// collided again (Aprev -> A, the previous step's number), their impulses
// left in the field for the chain kernel to clear; this thread takes entries
// fix_e0, fix_e0 + fix_n, ...  A table node whose population comes from such
// a node takes the fixed value computed here instead of reading it, so no
// thread reads what another writes.  With `stamp` the item also stamps its
// node's collide tile as deferred in step t.
template <typename R>
__device__ __forceinline__ void near_work(const BoxDev* __restrict__ boxes, const int32_t* __restrict__ list,
                                          R* A, const ChainArgs& ca, R* __restrict__ near_u,
                                          int4* __restrict__ near_c, Ctrl* ctrl,
                                          uint32_t t, const CollideConst<R>* __restrict__ ccs,
                                          const int32_t* __restrict__ bead_box, uint32_t* __restrict__ claim,
                                          const R* __restrict__ Aprev, int one_box, const BoxDev& one, int li,
                                          int item, uint32_t fix_e0, uint32_t fix_n, bool stamp)
{
    uint32_t n_pend = 0;
    if (Aprev) {
        n_pend = min(ctrl->ovf_cnt, ca.ovf_cap);
        for (uint32_t e = fix_e0; e < n_pend; e += fix_n) {
            const uint64_t g = ca.ovf[2 * (uint64_t)e];
            const uint32_t r = ca.ovf[2 * (uint64_t)e + 1];
            const int bi = bead_box[g];
            fixup_node<R>(fix_box(boxes[bi]), ccs[bi], r, ca.imp, claim, Aprev, A, ctrl, t - 1u, 1);
        }
    }
    // one_box >= 0: the launch covers that box alone, its descriptor passed by
    // value (no dependent loads of the box list and table before the beads')
    const int bi = one_box >= 0 ? one_box : list[li];
    const BoxDev bx = one_box >= 0 ? one : boxes[bi];   // a copy: its fields stay in registers
    const int N = bx.N, L = bx.L;
    if (item >= N * NEAR || bx.dense) return;   // the beads of a dense box read the node field
    const int b = item / NEAR, q = item - b * NEAR;
    const uint64_t g = bx.bead_off + (uint64_t)b;
    const double Ld = (double)L, iL = bx.inv_L;
    const int n0 = nearest_of(ca.x[3 * g], L, Ld, iL), n1 = nearest_of(ca.x[3 * g + 1], L, Ld, iL),
              n2 = nearest_of(ca.x[3 * g + 2], L, Ld, iL);
    if (q == 0) near_c[g] = make_int4(n0, n1, n2, 0);
    const int ix = n0 - 1 + q % 3, iy = n1 - 1 + (q / 3) % 3, iz = n2 - 1 + q / 9;
    const uint32_t node = node_of(ix, iy, iz, L);
    R* o = near_u + (g * NEAR + (uint64_t)q) * 3;
    const uint32_t nz = node / ((uint32_t)L * (uint32_t)L), rem = node - nz * (uint32_t)L * (uint32_t)L;
    const uint32_t ny = rem / (uint32_t)L, nx = rem - ny * (uint32_t)L;
    const Upwind up(nx, ny, nz, (uint32_t)L);
    R d[19];
    gather_pre<R, false>(A + bx.pop_off, up, d);
    if (n_pend) {
        // directions whose source node the previous step listed; every array
        // index below is a compile-time constant, so d and oo stay in registers
        const uint32_t pst = defer_stamp(t - 1u);
        uint32_t need = 0;
#pragma unroll
        for (int i = 0; i < 19; ++i)
            if (ca.ovm[bx.node_off + up.src(i)] == pst) need |= 1u << i;
        while (need) {
            const int ik = __builtin_ctz(need);
            need &= need - 1u;
            uint32_t src = 0;
#pragma unroll
            for (int j = 0; j < 19; ++j)
                if (j == ik) src = up.src(j);
            R dd[19], oo[19];
            gather_pre<R, false>(Aprev + bx.pop_off, upwind_of(src, L, bx.inv_L), dd);
            const unsigned long long* qi = ca.imp + 3 * (bx.node_off + src);
            const R fx = (R)((double)(long long)qi[0] * IMP_INV_SCALE),
                    fy = (R)((double)(long long)qi[1] * IMP_INV_SCALE),
                    fz = (R)((double)(long long)qi[2] * IMP_INV_SCALE);
            (void)collide<R>(dd, oo, fx, fy, fz, ccs[bi], src, t - 1u, bx.seed, bx.box_id);
#pragma unroll
            for (int j = 0; j < 19; ++j)
                if (j == ik) d[j] = oo[j];
        }
    }
    if (stamp && ca.defer)   // the bead's stencil stays on its table's nodes while it moves
                             // less than half a cell from its nearest node: their tiles wait
                             // for the impulses (a plain store: every writer stores the same stamp)
        ca.defer[2u * dseg_of(bx, node) + (t & 1u)] = defer_stamp(t);
    R u[3];
    node_velocity<R>(d, bx.rho0, 1.0 / bx.tau_lb, u);
    o[0] = u[0]; o[1] = u[1]; o[2] = u[2];
}

// The node-table kernel: grid (items of the largest chain / 256, list
// entries).  zero_head: a run of steps starts here; its later collides count
// their node-table workgroups from zero.
template <typename R>
__global__ __launch_bounds__(256) void k_near_nodes(const BoxDev* __restrict__ boxes,
                                                    const int32_t* __restrict__ list, R* A,
                                                    ChainArgs ca, R* __restrict__ near_u, int4* __restrict__ near_c,
                                                    Ctrl* __restrict__ ctrl,
                                                    uint32_t s_off, const CollideConst<R>* __restrict__ ccs,
                                                    const int32_t* __restrict__ bead_box,
                                                    uint32_t* __restrict__ claim, const R* __restrict__ Aprev,
                                                    int one_box, BoxDev one, int zero_head)
{
    const uint32_t t = ctrl->step + s_off;
    if (zero_head && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x < 2) {
        ctrl->head_done[threadIdx.x] = 0u;
        ctrl->head_fix[threadIdx.x] = 0u;
    }
    const uint32_t nth = gridDim.x * gridDim.y * blockDim.x;
    const uint32_t e0 = (blockIdx.y * gridDim.x + blockIdx.x) * blockDim.x + threadIdx.x;
    near_work<R>(boxes, list, A, ca, near_u, near_c, ctrl, t, ccs, bead_box, claim, Aprev, one_box, one,
                 (int)blockIdx.y, (int)(blockIdx.x * blockDim.x + threadIdx.x), e0, nth, true);
}

// Step t's collide in a run of batched steps that carries its own node
// tables: workgroups 0..n_head-1 do the node-table kernel's work (step t's
// tables; the tiles were stamped by the previous step's chain kernel) and
// count themselves done in head_done[t & 1]; the chain kernel, already
// resident on another queue, waits for that count.  The other workgroups
// collide one tile each, like k_collide.  When the previous step listed
// impulses outside its deferred tiles, the node-table workgroups first fix
// those nodes up and wait for each other (head_fix), so that the tables read
// the fixed values; and every tile waits for the node-table workgroups, whose
// fix-up rewrites populations that the tiles read, from inputs the tiles
// overwrite.  The node-table workgroups come first in the grid, are
// dispatched first and fit on the GPU at once (n_head <= CUs), so no
// workgroup waits for one that is not running.  The table code here has no
// in-register re-collision, so the kernel keeps the plain collide's
// register count and occupancy.
constexpr uint32_t SPIN_LIMIT = 1u << 19;   // polls of a bounded wait (~0.1 s)

// thread 0 polls *cnt (relaxed, so a poll invalidates no cache) until it
// reaches target, then acquires; the workgroup waits at the barrier
__device__ __forceinline__ void wait_count(Ctrl* __restrict__ ctrl, uint32_t* cnt, uint32_t target)
{
    if (threadIdx.x == 0) {
        uint32_t it = 0;
        while (__hip_atomic_load(cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) {
            if (++it > SPIN_LIMIT) { atomicOr(&ctrl->health, H_SYNC); break; }
            __builtin_amdgcn_s_sleep(8);
        }
        __atomic_thread_fence(__ATOMIC_ACQUIRE);
    }
    __syncthreads();
}

// Every thread of the workgroup has written what another agent will read:
// wait at the barrier with each wavefront's stores in L2.  The barrier alone
// does not wait for them (the compiler drains LDS there, not global stores),
// and a fence after it drains the fencing wavefront's only; with this, one
// thread's release fence behind it covers the whole workgroup.
__device__ __forceinline__ void all_stored()
{
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
}

// count the workgroup, whose threads are done, in *cnt, visibly for the other
// agents' acquire
__device__ __forceinline__ void count_done(uint32_t* cnt)
{
    all_stored();
    if (threadIdx.x == 0) {
        __threadfence();
        atomicAdd(cnt, 1u);
    }
}

// one (bead, table node) item of a sparse box: the node's fluid velocity from
// the current populations
template <typename R>
__device__ __forceinline__ void table_item(const BoxDev* __restrict__ boxes, const int32_t* __restrict__ list,
                                           const R* A, const ChainArgs& ca, R* __restrict__ near_u,
                                           int4* __restrict__ near_c, int one_box, const BoxDev& one, int li,
                                           int item)
{
    const int bi = one_box >= 0 ? one_box : list[li];
    const BoxDev bx = one_box >= 0 ? one : boxes[bi];
    const int N = bx.N, L = bx.L;
    if (item >= N * NEAR) return;
    const int b = item / NEAR, q = item - b * NEAR;
    const uint64_t g = bx.bead_off + (uint64_t)b;
    const double Ld = (double)L, iL = bx.inv_L;
    const int n0 = nearest_of(ca.x[3 * g], L, Ld, iL), n1 = nearest_of(ca.x[3 * g + 1], L, Ld, iL),
              n2 = nearest_of(ca.x[3 * g + 2], L, Ld, iL);
    if (q == 0) near_c[g] = make_int4(n0, n1, n2, 0);
    const uint32_t node = node_of(n0 - 1 + q % 3, n1 - 1 + (q / 3) % 3, n2 - 1 + q / 9, L);
    const uint32_t nz = node / ((uint32_t)L * (uint32_t)L), rem = node - nz * (uint32_t)L * (uint32_t)L;
    const uint32_t ny = rem / (uint32_t)L, nx = rem - ny * (uint32_t)L;
    R d[19];
    gather_pre<R, false>(A + bx.pop_off, Upwind(nx, ny, nz, (uint32_t)L), d);
    R u[3];
    node_velocity<R>(d, bx.rho0, 1.0 / bx.tau_lb, u);
    R* o = near_u + (g * NEAR + (uint64_t)q) * 3;
    o[0] = u[0]; o[1] = u[1]; o[2] = u[2];
}

template <typename R, int W>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, W))) void k_collide_headed(
    const BoxDev* __restrict__ boxes, const CollideConst<R>* __restrict__ ccs, const uint32_t* __restrict__ tile_box,
    R* A, R* B, Ctrl* __restrict__ ctrl, uint32_t s_off, const uint32_t* __restrict__ defer, uint32_t n_head,
    uint32_t head_x, const int32_t* __restrict__ list, ChainArgs ca, R* __restrict__ near_u,
    int4* __restrict__ near_c, const int32_t* __restrict__ bead_box, uint32_t* __restrict__ claim,
    const R* Aprev, int one_box, BoxDev one)   // Aprev and B are one buffer: the fix-up reads it, the tiles write it
{
    const uint32_t t = ctrl->step + s_off;
    const bool pend = ctrl->ovf_flag[(t - 1u) & 1u] == defer_stamp(t - 1u);
    if (blockIdx.x < n_head) {
        const uint32_t li = blockIdx.x / head_x, bx_ = blockIdx.x - li * head_x;
        if (pend) {
            // the workgroups of list entry li fix the listed nodes of its box:
            // the box and its constants stay uniform (scalar registers)
            const int bi = __builtin_amdgcn_readfirstlane(one_box >= 0 ? one_box : list[li]);
            const BoxDev& bx = boxes[bi];
            const uint32_t n_pend = min(ctrl->ovf_cnt, ca.ovf_cap);
            for (uint32_t e = bx_ * 256u + threadIdx.x; e < n_pend; e += head_x * 256u) {
                const uint64_t g = ca.ovf[2 * (uint64_t)e];
                const uint32_t r = ca.ovf[2 * (uint64_t)e + 1];
                if (bead_box[g] == bi)
                    fixup_node_claim_first<R>(bx, ccs, bi, r, ca.imp, claim, Aprev, A, ctrl, t - 1u);
            }
            count_done(&ctrl->head_fix[t & 1u]);
            wait_count(ctrl, &ctrl->head_fix[t & 1u], n_head);
        }
        table_item<R>(boxes, list, A, ca, near_u, near_c, one_box, one, (int)li, (int)(bx_ * 256u + threadIdx.x));
        count_done(&ctrl->head_done[t & 1u]);
        return;
    }
    if (pend) wait_count(ctrl, &ctrl->head_done[t & 1u], n_head);
    collide_tile<R>(boxes, ccs, tile_box, -1, blockIdx.x - n_head, A, B, ctrl, t, defer, threadIdx.x);
}

// one substep of one bead, as k_spread reads it
constexpr int REC = 8;   // doubles: fraction x3, coupling force x3, base cell (packed), unused
// a base cell as one number: its coordinates, 11 bits each (L <= 1625)
__device__ __forceinline__ double pack_cell(int x, int y, int z)
{
    return __longlong_as_double((long long)((unsigned long long)x | (unsigned long long)y << 11 | (unsigned long long)z << 22));
}
struct Cell { int x, y, z; };
__device__ __forceinline__ Cell cell_of_packed(unsigned long long c)
{
    return Cell{(int)(c & 2047u), (int)((c >> 11) & 2047u), (int)(c >> 22)};
}

// NT: threads, and the most beads; chains up to 512 beads take 512 threads,
// which leaves each twice the registers (none spilled) at the same waves per bead.
template <typename R, int NT>
__global__ __launch_bounds__(NT) void k_chain_wg(const BoxDev* __restrict__ boxes,
                                                      const int32_t* __restrict__ list,
                                                      const R* __restrict__ A, ChainArgs ca,
                                                      const R* __restrict__ near_u,
                                                      const int4* __restrict__ near_c, const R* __restrict__ field,
                                                      double* __restrict__ rec, Ctrl* __restrict__ ctrl,
                                                      uint32_t s_off, const int32_t* __restrict__ ca_bead_box,
                                                      int clear_ovf, uint32_t wait_head, int stamp_next)
{
    __shared__ double xs[3 * NT];           // current positions
    __shared__ double x0s[3 * NT];          // positions at the last list build
    __shared__ uint16_t nls[NL_SLOTS * NT];  // neighbour k of bead b at [k * NT + b]
    __shared__ uint32_t bk_cnt[NBK];             // list build: beads per cell bucket,
    __shared__ uint32_t bk_wsum[NT / 64];   //   per-wave totals of the scan,
    __shared__ uint16_t bk_start[NBK + 1];       //   first slot of each bucket,
    __shared__ float4 bk_pos[NT];           //   beads ordered by bucket: position wrapped into the box, index
    __builtin_amdgcn_s_setprio(3);   // latency-bound chain beside the bandwidth-bound collide
    const int bi = list[blockIdx.x];
    const BoxDev& bx = boxes[bi];
    const int N = bx.N;
    const int b = (int)threadIdx.x;
    const bool act = b < N;
    const uint64_t g = bx.bead_off + (uint64_t)(act ? b : 0);
    const ChainSpan sp = chain_span(bx, act ? b : 0);
    const uint32_t t = ctrl->step + s_off;
    const int L = bx.L;
    const double Ld = (double)L, iL = bx.inv_L;
    const double dt = bx.dt, hdt_m = 0.5 * dt / bx.mass;
    const double eps24 = 24.0 * bx.eps;
    const double rl = sqrt(bx.rc2) + NL_SKIN;
    const double rl2 = rl * rl;
    const int nl_cap = ca.nl_cap < NL_SLOTS ? ca.nl_cap : NL_SLOTS;

    double x[3] = {0, 0, 0}, v[3] = {0, 0, 0}, f[3] = {0, 0, 0};
    int nl_n = -2;
    int4 nc = make_int4(0, 0, 0, 0);
    // the beads and their lists, ahead of the wait: the previous chain kernel
    // left them
    if (act) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            x[c] = ca.x[3 * g + c]; v[c] = ca.v[3 * g + c]; f[c] = ca.f[3 * g + c];
            x0s[3 * b + c] = ca.nl_x0[3 * g + c];
        }
        nl_n = ca.nl_cnt[g];
        // the list, eight entries per load
        const uint4* row = (const uint4*)(ca.nl_idx + g * NL_SLOTS);
#pragma unroll
        for (int q = 0; q < NL_SLOTS / 8; ++q)
            if (nl_n > 8 * q) {
                const uint4 e = row[q];
                const uint32_t w[4] = {e.x, e.y, e.z, e.w};
#pragma unroll
                for (int k = 0; k < 8; ++k)
                    nls[(8 * q + k) * NT + b] = (uint16_t)(w[k / 2] >> (16 * (k & 1)));
            }
    }
    if (wait_head) {
        // the node tables come from the first workgroups of this step's
        // collide, which starts once the previous collide is done
        wait_count(ctrl, &ctrl->head_done[t & 1u], wait_head);
        if (b == 0) {   // the previous step's readers of its counts are done
            ctrl->head_done[(t + 1u) & 1u] = 0u;
            ctrl->head_fix[(t + 1u) & 1u] = 0u;
        }
    }
    if (clear_ovf) {
        // the previous step's impulses outside its deferred tiles were fixed
        // up by the node-table work, which left them in the field: clear
        // them before this step's spread, then reset both list counts
        const uint32_t n_ovf = min(ctrl->ovf_cnt, ca.ovf_cap);
        for (uint32_t e = (uint32_t)b; e < n_ovf; e += NT) {
            const uint64_t gg = ca.ovf[2 * (uint64_t)e];
            const uint32_t r = ca.ovf[2 * (uint64_t)e + 1];
            unsigned long long* q = ca.imp + 3 * (boxes[ca_bead_box[gg]].node_off + r);
            q[0] = 0ull; q[1] = 0ull; q[2] = 0ull;
        }
        __syncthreads();   // every thread has read the count
        if (b == 0) { ctrl->ovf_cnt = 0u; ctrl->defer_cnt = 0u; }
    }

    if (act && !bx.dense) nc = near_c[g];
    int rebuilds = 0;
    int cb0 = -1, cb1 = -1, cb2 = -1;   // base cell of the cached stencil
    R cu[8][3];                          // its node velocities (MD units), storage precision
    uint32_t hbits = 0;
    int tcnt = 0;
    // the fix-up's node list: not for dense boxes and deferred tiles, whose
    // nodes no fix-up visits
    const bool list_touched = !bx.dense && !ca.defer;

    for (int s = 0; s < bx.substeps; ++s) {
        if (act) {
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                v[c] += f[c] * hdt_m;
                x[c] += v[c] * dt;
            }
        }
        __syncthreads();   // every read of xs by the previous substep is done
        bool rebuild = false;
        if (act) {
            xs[3 * b] = x[0]; xs[3 * b + 1] = x[1]; xs[3 * b + 2] = x[2];
            const double e0 = x[0] - x0s[3 * b], e1 = x[1] - x0s[3 * b + 1], e2 = x[2] - x0s[3 * b + 2];
            rebuild = nl_n == -2 || e0 * e0 + e1 * e1 + e2 * e2 > 0.25 * NL_SKIN * NL_SKIN;
        }
        // one bead past half the skin rebuilds every list; also publishes xs
        rebuild = __syncthreads_or(rebuild);
        if (rebuild) {
            ++rebuilds;
            int cnt = 0;
            bool stored = false;
            // scan over every bead (boxes under three list radii across):
            // partner j joins the list when its minimum-image distance is
            // below the list radius
            auto consider = [&](int j) {
                double d0 = x[0] - xs[3 * j], d1 = x[1] - xs[3 * j + 1], d2 = x[2] - xs[3 * j + 2];
                d0 -= Ld * rint(d0 * iL); d1 -= Ld * rint(d1 * iL); d2 -= Ld * rint(d2 * iL);
                if (d0 * d0 + d1 * d1 + d2 * d2 < rl2) {
                    if (cnt < nl_cap) nls[cnt * NT + b] = (uint16_t)j;
                    ++cnt;
                }
            };
            const int nc = list_cells(L, rl);
            if (nc >= 3) {
                // beads binned by cell bucket (counting sort in LDS), then each
                // bead visits the 27 buckets around its own cell
                int cc[3] = {0, 0, 0}, slot = 0, hb = 0;
                float pb[3] = {0.f, 0.f, 0.f};   // own position wrapped into [0, L)
                if (act) {
                    const double scl = (double)nc / Ld;
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        double xt = x[c] - Ld * floor(x[c] * iL);
                        if (xt < 0.0) xt += Ld;
                        if (xt >= Ld) xt -= Ld;
                        const int q = (int)(xt * scl);
                        cc[c] = q < 0 ? 0 : (q >= nc ? nc - 1 : q);
                        pb[c] = (float)xt;
                    }
                    hb = bucket_of(cc[0], cc[1], cc[2]);
                }
                for (int i = b; i < NBK; i += NT) bk_cnt[i] = 0u;
                __syncthreads();
                if (act) slot = (int)atomicAdd(&bk_cnt[hb], 1u);
                __syncthreads();
                // exclusive prefix sum of the bucket counts, NBK / NT per thread: a
                // scan per wave, then the totals of the waves before
                constexpr int BPT = NBK / NT;
                uint32_t vb[BPT], vs = 0;
#pragma unroll
                for (int u = 0; u < BPT; ++u) { vb[u] = bk_cnt[BPT * b + u]; vs += vb[u]; }
                uint32_t inc = vs;
                for (int o = 1; o < 64; o <<= 1) {
                    const uint32_t t = __shfl_up(inc, o, 64);
                    if ((b & 63) >= o) inc += t;
                }
                if ((b & 63) == 63) bk_wsum[b >> 6] = inc;
                __syncthreads();
                {
                    uint32_t base = 0;
                    for (int w = 0; w < (b >> 6); ++w) base += bk_wsum[w];
                    uint32_t ex = base + inc - vs;
#pragma unroll
                    for (int u = 0; u < BPT; ++u) { bk_start[BPT * b + u] = (uint16_t)ex; ex += vb[u]; }
                    if (b == NT - 1) bk_start[NBK] = (uint16_t)ex;
                }
                __syncthreads();
                if (act) {
                    const int sl = bk_start[hb] + slot;
                    bk_pos[sl] = make_float4(pb[0], pb[1], pb[2], __int_as_float(b));
                }
                __syncthreads();
                if (act) {
                    const float Lf = (float)Ld;
                    const float rlf2 = (float)((rl + NL_FP32_MARGIN) * (rl + NL_FP32_MARGIN));
                    // candidates in bucket slots k0..k1-1, seen with this
                    // bead at (ox, oy, oz); two per pass (a row of three cells
                    // holds about two beads), one load each
                    auto visit = [&](int k0, int k1, float ox, float oy, float oz) __attribute__((always_inline)) {
#pragma unroll 1
                        for (int k = k0; k < k1; k += 2) {
                            int jj[2];
                            float r2[2];
#pragma unroll
                            for (int u = 0; u < 2; ++u) {
                                const bool ok = k + u < k1;
                                const float4 e = bk_pos[ok ? k + u : k];
                                jj[u] = ok ? __float_as_int(e.w) : b;
                                const float d0 = e.x - ox, d1 = e.y - oy, d2 = e.z - oz;
                                r2[u] = jj[u] == b ? rlf2 : d0 * d0 + d1 * d1 + d2 * d2;
                            }
#pragma unroll
                            for (int u = 0; u < 2; ++u)
                                if (r2[u] < rlf2) {
                                    if (cnt < nl_cap) nls[cnt * NT + b] = (uint16_t)jj[u];
                                    ++cnt;
                                }
                        }
                    };
                    // a row of cells along x lies in consecutive buckets (cells
                    // lo..hi; where it passes a multiple of 16, from there on in
                    // the row's first buckets), but for its image across the
                    // box edge: one or two visits per row instead of three
                    const int lo = cc[0] > 0 ? cc[0] - 1 : 0, hi = cc[0] + 1 < nc ? cc[0] + 1 : nc - 1;
                    const int cut = (hi & 15) < (lo & 15) ? hi & ~15 : hi + 1;   // first cell of the second part
#pragma unroll 1
                    for (int dz = -1; dz <= 1; ++dz) {
                        const int rz = cc[2] + dz, qz = wrap_cell(rz, nc);
                        // the neighbour cell's image next to this bead
                        const float oz = pb[2] + (rz < 0 ? Lf : (rz >= nc ? -Lf : 0.f));
#pragma unroll 1
                        for (int dy = -1; dy <= 1; ++dy) {
                            const int ry = cc[1] + dy, qy = wrap_cell(ry, nc);
                            const float oy = pb[1] + (ry < 0 ? Lf : (ry >= nc ? -Lf : 0.f));
                            const int row = bucket_of(0, qy, qz);
                            visit(bk_start[row + (lo & 15)], bk_start[row + ((cut - 1) & 15) + 1], pb[0], oy, oz);
                            if (cut <= hi) visit(bk_start[row], bk_start[row + (hi & 15) + 1], pb[0], oy, oz);
                            if (cc[0] == 0) {
                                const int q = row + ((nc - 1) & 15);
                                visit(bk_start[q], bk_start[q + 1], pb[0] + Lf, oy, oz);
                            } else if (cc[0] == nc - 1) {
                                visit(bk_start[row], bk_start[row + 1], pb[0] - Lf, oy, oz);
                            }
                        }
                    }
                    // ascending partner order, as a scan over all beads gives,
                    // and the list stored for the next step
                    if (cnt <= SORT_REGS) {   // an odd-even merge network in registers
                        uint32_t key[SORT_REGS];
#pragma unroll
                        for (int i = 0; i < SORT_REGS; ++i) key[i] = i < cnt ? (uint32_t)nls[i * NT + b] : 0xffffu;
#pragma unroll
                        for (int p = 1; p < SORT_REGS; p *= 2)
#pragma unroll
                            for (int k = p; k >= 1; k /= 2)
#pragma unroll
                                for (int j = k % p; j + k < SORT_REGS; j += 2 * k)
#pragma unroll
                                    for (int i = 0; i < k; ++i)
                                        if (i + j + k < SORT_REGS && (i + j) / (2 * p) == (i + j + k) / (2 * p)) {
                                            const uint32_t x1 = key[i + j], x2 = key[i + j + k];
                                            key[i + j] = min(x1, x2);
                                            key[i + j + k] = max(x1, x2);
                                        }
#pragma unroll
                        for (int i = 0; i < SORT_REGS; ++i)
                            if (i < cnt) nls[i * NT + b] = (uint16_t)key[i];
                        uint4* row = (uint4*)(ca.nl_idx + g * NL_SLOTS);
#pragma unroll
                        for (int q = 0; q < SORT_REGS / 8; ++q)
                            if (cnt > 8 * q)
                                row[q] = make_uint4(key[8 * q] | key[8 * q + 1] << 16, key[8 * q + 2] | key[8 * q + 3] << 16,
                                                    key[8 * q + 4] | key[8 * q + 5] << 16,
                                                    key[8 * q + 6] | key[8 * q + 7] << 16);
                        stored = true;
                    } else if (cnt <= nl_cap)
                        for (int i = 1; i < cnt; ++i) {
                            const uint16_t key = nls[i * NT + b];
                            int k = i - 1;
                            while (k >= 0 && nls[k * NT + b] > key) {
                                nls[(k + 1) * NT + b] = nls[k * NT + b];
                                --k;
                            }
                            nls[(k + 1) * NT + b] = key;
                        }
                }
            } else if (act) {   // boxes under three list radii across: every bead
                for (int j = 0; j < N; ++j)
                    if (j != b) consider(j);
            }
            if (act) {
                const int kept = cnt < nl_cap ? cnt : nl_cap;
                if (!stored)
                    for (int k = 0; k < kept; ++k) ca.nl_idx[g * ca.nl_cap + k] = nls[k * NT + b];
                nl_n = cnt > nl_cap ? -1 : cnt;   // -1: overflow, the full loop is used
                ca.nl_cnt[g] = nl_n;
#pragma unroll
                for (int c = 0; c < 3; ++c) { x0s[3 * b + c] = x[c]; ca.nl_x0[3 * g + c] = x[c]; }
            }
        }
        if (act) {
            // stencil first: the last force is dead after the drift
            double fr[3];
            const int i0 = cell_of(x[0], L, Ld, iL, fr[0]), i1 = cell_of(x[1], L, Ld, iL, fr[1]),
                      i2 = cell_of(x[2], L, Ld, iL, fr[2]);
            if (i0 != cb0 || i1 != cb1 || i2 != cb2) {
                cb0 = i0; cb1 = i1; cb2 = i2;
#pragma unroll
                for (int k = 0; k < (list_touched ? 8 : 0); ++k) {
                    const uint32_t node = node_of(cb0 + (k & 1), cb1 + ((k >> 1) & 1), cb2 + ((k >> 2) & 1), L);
                    if (tcnt < ca.touch_cap) ca.touched[g * ca.touch_cap + tcnt] = node;
                    else hbits |= H_TABLE;
                    ++tcnt;
                }
                // offset of the base cell in the bead's 3x3x3 table: the
                // stencil lies inside it when the base cell is the nearest
                // node or the one below, on every axis
                int d0 = cb0 - nc.x + 1, d1 = cb1 - nc.y + 1, d2 = cb2 - nc.z + 1;
                d0 = d0 < 0 ? d0 + L : (d0 >= L ? d0 - L : d0);
                d1 = d1 < 0 ? d1 + L : (d1 >= L ? d1 - L : d1);
                d2 = d2 < 0 ? d2 + L : (d2 >= L ? d2 - L : d2);
                if (bx.dense) {   // every node's velocity
#pragma unroll
                    for (int k = 0; k < 8; ++k) {
                        const R* fu = field + 3 * (bx.field_off + node_of(cb0 + (k & 1), cb1 + ((k >> 1) & 1),
                                                                          cb2 + ((k >> 2) & 1), L));
                        cu[k][0] = fu[0]; cu[k][1] = fu[1]; cu[k][2] = fu[2];
                    }
                } else if (d0 <= 1 && d1 <= 1 && d2 <= 1) {
                    const R* tb = near_u + g * NEAR * 3;
#pragma unroll
                    for (int k = 0; k < 8; ++k) {
                        const int q = (d0 + (k & 1)) + 3 * (d1 + ((k >> 1) & 1)) + 9 * (d2 + ((k >> 2) & 1));
                        cu[k][0] = tb[3 * q]; cu[k][1] = tb[3 * q + 1]; cu[k][2] = tb[3 * q + 2];
                    }
                } else {   // moved past the table within this LB step: read the populations
                    const int i0v[3] = {cb0, cb1, cb2};
                    stencil_velocities<R, R, 1>(A + bx.pop_off, i0v, L, bx.rho0, 1.0 / bx.tau_lb, cu);
                }
            }
            double F[3] = {0, 0, 0};
            if (nl_n >= 0) {
                auto jof = [&](int k) { return (int)nls[k * NT + b]; };
                for (int k = 0; k < nl_n; k += 4) wca_add4(x, xs, jof, k, nl_n, 1, b, Ld, iL, bx.rc2, bx.sigsq, eps24, F);
            } else {
                auto jof = [](int k) { return k; };
                for (int j = 0; j < N; j += 4) wca_add4(x, xs, jof, j, N, 1, b, Ld, iL, bx.rc2, bx.sigsq, eps24, F);
            }
            double Ff[3] = {0, 0, 0};
            hbits |= fene_force(bx, b, sp, x, xs, Ff);
            F[0] = Ff[0] + F[0]; F[1] = Ff[1] + F[1]; F[2] = Ff[2] + F[2];
            double ub[3] = {0, 0, 0};
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const double wk = ((k & 1) ? fr[0] : 1.0 - fr[0]) * (((k >> 1) & 1) ? fr[1] : 1.0 - fr[1]) *
                                  (((k >> 2) & 1) ? fr[2] : 1.0 - fr[2]);
                ub[0] += wk * (double)cu[k][0]; ub[1] += wk * (double)cu[k][1]; ub[2] += wk * (double)cu[k][2];
            }
            const U4 w = philox10(U4{(uint32_t)b, t, (1u << 16) | (uint32_t)s, 0u}, bx.seed, bx.box_id);
            const uint32_t ws[3] = {w.x, w.y, w.z};
            double fcl[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const double ffr = -bx.zeta * (v[c] - ub[c]);
                const double frn = bx.bead_noise * unit_noise<double>(ws[c]);
                fcl[c] = ffr + frn;
                f[c] = F[c] + fcl[c];
                v[c] += f[c] * hdt_m;
            }
            double* r = rec + ((uint64_t)s * ca.total_beads + g) * REC;
            r[0] = fr[0]; r[1] = fr[1]; r[2] = fr[2];
            r[3] = fcl[0]; r[4] = fcl[1]; r[5] = fcl[2];
            r[6] = pack_cell(cb0, cb1, cb2);
            if (s + 1 == bx.substeps) {
#pragma unroll
                for (int c = 0; c < 3; ++c) ca.fc[3 * g + c] = fcl[c];
            }
        }
    }
    if (act) {
        if (list_touched) ca.touched_cnt[g] = tcnt < ca.touch_cap ? tcnt : ca.touch_cap;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            ca.x[3 * g + c] = x[c]; ca.v[3 * g + c] = v[c]; ca.f[3 * g + c] = f[c];
        }
        if (stamp_next && ca.defer) {
            // the next step's deferred tiles: those of the table around the
            // nearest node of the end position (what its node-table work uses)
            const int m0 = nearest_of(x[0], L, Ld, iL), m1 = nearest_of(x[1], L, Ld, iL),
                      m2 = nearest_of(x[2], L, Ld, iL);
            const uint32_t sn = defer_stamp(t + 1u);
            for (int q = 0; q < NEAR; ++q) {
                const uint32_t node = node_of(m0 - 1 + q % 3, m1 - 1 + (q / 3) % 3, m2 - 1 + q / 9, L);
                ca.defer[2u * dseg_of(bx, node) + (sn & 1u)] = sn;
            }
        }
        if (ca.vhist) {
            double* hv = ca.vhist + ((uint64_t)(t % (uint32_t)ca.hist_len) * ca.total_beads + g) * 3;
            hv[0] = v[0]; hv[1] = v[1]; hv[2] = v[2];
        }
        if (hbits) atomicOr(&ctrl->health, hbits);
    }
    if (b == 0 && rebuilds) atomicAdd(&ca.nl_rebuilds[bi], (uint32_t)rebuilds);
}

// an impulse on a node whose tile is not deferred (the bead left its table):
// listed for the end-of-step fix-up
__device__ __forceinline__ uint32_t list_overflow(const ChainArgs& ca, uint64_t g, uint64_t node_at, uint32_t node,
                                                  Ctrl* __restrict__ ctrl, uint32_t stamp)
{
    ca.ovm[node_at] = stamp;              // read by the next step's node-table work
    ctrl->ovf_flag[stamp & 1u] = stamp;   // the next step's collide waits for that work
    const uint32_t k = atomicAdd(&ctrl->ovf_cnt, 1u);
    if (k >= ca.ovf_cap) return H_TABLE;
    ca.ovf[2 * (uint64_t)k] = (uint32_t)g;
    ca.ovf[2 * (uint64_t)k + 1] = node;
    return 0u;
}

// The deferred tiles of a step as a list, built after the coupling on the
// chain's stream: thread (bead, table node) of a sparse box claims the node's
// tile for this step; each wave appends its new tiles with one atomic.
__device__ __forceinline__ void list_deferred(const BoxDev& bx, const ChainArgs& ca, const int4* __restrict__ near_c,
                                              Ctrl* __restrict__ ctrl, uint32_t s_off, int tid)
{
    const uint32_t stamp = defer_stamp(ctrl->step + s_off);
    bool win = false;
    uint32_t seg = 0;
    if (tid < bx.N * NEAR) {
        const int b = tid / NEAR, q = tid - b * NEAR;
        const int4 nc = near_c[bx.bead_off + (uint64_t)b];
        const uint32_t node = node_of(nc.x - 1 + q % 3, nc.y - 1 + (q / 3) % 3, nc.z - 1 + q / 9, bx.L);
        seg = dseg_of(bx, node);
        win = ca.dclaim[seg] != stamp && atomicExch(&ca.dclaim[seg], stamp) != stamp;
    }
    const unsigned long long m = __ballot(win);
    if (m == 0ull) return;
    const int lane = (int)(threadIdx.x & 63u);
    const int lead = __ffsll((long long)m) - 1;
    uint32_t base = 0;
    if (lane == lead) base = atomicAdd(&ctrl->defer_cnt, (uint32_t)__popcll(m));
    base = __shfl(base, lead);
    if (win) {
        const uint32_t k = base + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
        if (k < ca.defer_cap) ca.defer_list[k] = seg;
        else atomicOr(&ctrl->health, H_TABLE);
    }
}

// node impulses from the substep records: thread (bead, corner k) accumulates
// -w_k (F_fric + F_rand) dt over the substeps that share a stencil, in MD
// units and in substep order, and hands each stencil's sum over when the
// stencil changes and after the last substep (lattice units, fixed point)
// The workgroups from n_spread on build the list of the step's deferred
// tiles, which needs nothing of the impulses.
// Bounds: latency (16 to 32 workgroups for one chain).  The records of
// REC_AHEAD substeps are read together, and the segment's stamp when a stencil
// begins: a load per substep, each behind the one before, took 13.1 us for 512
// beads and 10 substeps, this form 9.7 us.
constexpr int REC_AHEAD = 5;
__global__ __launch_bounds__(256) void k_spread(const BoxDev* __restrict__ boxes, const int32_t* __restrict__ list,
                                                ChainArgs ca, const double* __restrict__ rec,
                                                const int4* __restrict__ near_c, Ctrl* __restrict__ ctrl,
                                                uint32_t s_off, uint32_t n_spread)
{
    const BoxDev& bx = boxes[list[blockIdx.y]];
    if (bx.dense) return;   // k_dense_impulse
    if (blockIdx.x >= n_spread) {
        list_deferred(bx, ca, near_c, ctrl, s_off, (int)((blockIdx.x - n_spread) * blockDim.x + threadIdx.x));
        return;
    }
    const int N = bx.N, L = bx.L;
    const int tid = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (tid >= N * 8) return;
    const int b = tid >> 3, k = tid & 7;
    const uint64_t g = bx.bead_off + (uint64_t)b;
    const double dt = bx.dt, tau = bx.tau_lb;
    const uint32_t stamp = defer_stamp(ctrl->step + s_off);
    unsigned long long* imp = ca.imp + 3 * bx.node_off;
    uint32_t hb = 0;
    double acc[3] = {0, 0, 0};
    uint32_t cur = 0xffffffffu, cur_stamp = 0;
    auto hand_over = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            double q = acc[c] * tau;
            if (!(fabs(q) < IMP_MAX)) { hb |= H_FIXED; q = 0.0; }
            atomicAdd(imp + 3 * (uint64_t)cur + c, (unsigned long long)(long long)llrint(q * IMP_SCALE));
        }
        if (cur_stamp != stamp) hb |= list_overflow(ca, g, bx.node_off + cur, cur, ctrl, stamp);
    };
    const int S = bx.substeps;
    for (int s0 = 0; s0 < S; s0 += REC_AHEAD) {
        double2 r[REC_AHEAD][3];
        unsigned long long cell[REC_AHEAD];
#pragma unroll
        for (int u = 0; u < REC_AHEAD; ++u) {
            const double2* q = (const double2*)(rec + ((uint64_t)min(s0 + u, S - 1) * ca.total_beads + g) * REC);
            r[u][0] = q[0]; r[u][1] = q[1]; r[u][2] = q[2];
            cell[u] = ((const unsigned long long*)q)[6];
        }
#pragma unroll
        for (int u = 0; u < REC_AHEAD; ++u) {
            if (s0 + u >= S) break;
            const Cell cl = cell_of_packed(cell[u]);
            const uint32_t node = node_of(cl.x + (k & 1), cl.y + ((k >> 1) & 1), cl.z + ((k >> 2) & 1), L);
            if (node != cur) {
                if (cur != 0xffffffffu) hand_over();
                cur = node;
                // read here, used at the hand-over
                cur_stamp = ca.defer ? ca.defer[2u * dseg_of(bx, node) + (stamp & 1u)] : stamp;
                acc[0] = acc[1] = acc[2] = 0.0;
            }
            const double wk = ((k & 1) ? r[u][0].x : 1.0 - r[u][0].x) * (((k >> 1) & 1) ? r[u][0].y : 1.0 - r[u][0].y) *
                              (((k >> 2) & 1) ? r[u][1].x : 1.0 - r[u][1].x);
            acc[0] -= wk * r[u][1].y * dt;
            acc[1] -= wk * r[u][2].x * dt;
            acc[2] -= wk * r[u][2].y * dt;
        }
    }
    if (cur != 0xffffffffu) hand_over();
    if (hb) atomicOr(&ctrl->health, hb);
}

// Dense boxes hand their impulses over in LDS: grid (node ranges of the
// largest box, list), one workgroup holds the fixed-point sums of DENSE_NODES
// consecutive nodes of a box (64 KB: two workgroups per CU), adds every
// (bead, corner) impulse that falls into them, accumulated over the substeps
// that share a stencil and rounded once as in k_spread, and writes the range
// out.  Integer sums do not depend on order.  Bounds: the latency of the
// records' reads (each range reads every bead's base node) and of the LDS
// atomics.  A counting sort of the stencils by node, their values and a
// gather per node, three kernels, took 31 us on 64 boxes of 20^3 with 1024
// beads; this takes 15.
constexpr uint32_t DENSE_NODES = 2720;
__global__ __launch_bounds__(1024) void k_dense_impulse(const BoxDev* __restrict__ boxes,
                                                        const int32_t* __restrict__ list, ChainArgs ca,
                                                        const double* __restrict__ rec, Ctrl* __restrict__ ctrl)
{
    __shared__ unsigned long long sum[3 * DENSE_NODES];
    const BoxDev& bx = boxes[list[blockIdx.y]];
    if (!bx.dense) return;
    const int N = bx.N, S = bx.substeps, L = bx.L;
    const uint32_t V = (uint32_t)L * L * L, r0 = blockIdx.x * DENSE_NODES;
    if (r0 >= V) return;
    const uint32_t nr = min(DENSE_NODES, V - r0);
    for (uint32_t i = threadIdx.x; i < 3 * nr; i += 1024) sum[i] = 0ull;
    __syncthreads();
    const double dt = bx.dt, tau = bx.tau_lb;
    uint32_t hb = 0;
    // four (bead, corner) items at a time, their records' loads in flight
    // together; k is the same for all of a thread's items
    const int k = (int)threadIdx.x & 7;
    for (int e0 = (int)threadIdx.x; e0 < 8 * N; e0 += 4 * 1024) {
        double acc[4][3];
        unsigned long long cur[4];   // base cell of the stencil
        uint32_t at[4];              // its corner's node in the range (nr: outside)
        uint64_t g[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int e = e0 + 1024 * u;
            g[u] = bx.bead_off + (uint64_t)((e < 8 * N ? e : e0) >> 3);
            cur[u] = ~0ull;
            at[u] = nr;
            acc[u][0] = acc[u][1] = acc[u][2] = 0.0;
        }
        auto hand_over = [&](uint32_t i, const double q3[3]) __attribute__((always_inline)) {
            if (i >= nr) return;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                double q = q3[c] * tau;
                if (!(fabs(q) < IMP_MAX)) { hb |= H_FIXED; q = 0.0; }
                atomicAdd(&sum[3 * i + c], (unsigned long long)(long long)llrint(q * IMP_SCALE));
            }
        };
        for (int s = 0; s < S; ++s) {
            // the base nodes first: the beads of a wavefront are neighbours
            // on a chain, so it often has nothing in the range
            const double* p[4];
            double r[4][6], bd[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                p[u] = rec + ((uint64_t)s * ca.total_beads + g[u]) * REC;
                bd[u] = p[u][6];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const unsigned long long cell = (unsigned long long)__double_as_longlong(bd[u]);
                if (cell != cur[u]) {
                    hand_over(at[u], acc[u]);
                    cur[u] = cell;
                    acc[u][0] = acc[u][1] = acc[u][2] = 0.0;
                    const Cell cl = cell_of_packed(cell);
                    const uint32_t node = node_of(cl.x + (k & 1), cl.y + ((k >> 1) & 1), cl.z + (k >> 2), L);
                    at[u] = node - r0 < nr && e0 + 1024 * u < 8 * N ? node - r0 : nr;
                }
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (at[u] < nr) {
#pragma unroll
                    for (int c = 0; c < 6; ++c) r[u][c] = p[u][c];
                }
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (at[u] < nr) {
                    const double wk = ((k & 1) ? r[u][0] : 1.0 - r[u][0]) * (((k >> 1) & 1) ? r[u][1] : 1.0 - r[u][1]) *
                                      (((k >> 2) & 1) ? r[u][2] : 1.0 - r[u][2]);
#pragma unroll
                    for (int c = 0; c < 3; ++c) acc[u][c] -= wk * r[u][3 + c] * dt;
                }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) hand_over(at[u], acc[u]);
    }
    __syncthreads();
    unsigned long long* imp = ca.imp + 3 * (bx.node_off + r0);
    for (uint32_t i = threadIdx.x; i < 3 * nr; i += 1024) imp[i] = sum[i];
    if (hb) atomicOr(&ctrl->health, hb);
}

// ---------------------------------------------------------------- fixup
// Collide node r of box bi with its impulse from the dense field and
// overwrite its streamed outputs.  The claim stamp makes one caller per node
// and step do it: the populations and the impulse are loaded before the
// claim returns, so the three latencies overlap.
template <typename R>
__device__ __forceinline__ void fixup_node(const FixBox& bx, const CollideConst<R>& cc, uint32_t r,
                                           unsigned long long* __restrict__ imp, uint32_t* __restrict__ claim,
                                           const R* __restrict__ A, R* __restrict__ B, Ctrl* __restrict__ ctrl,
                                           uint32_t t, int keep_imp)
{
    const uint64_t node = bx.node_off + r;
    const Upwind up = upwind_of(r, bx.L, bx.inv_L);
    R d[19];
    gather_pre<R, false>(A + bx.pop_off, up, d);
    unsigned long long* q = imp + 3 * node;
    const unsigned long long q0 = q[0], q1 = q[1], q2 = q[2];
    if (atomicExch(&claim[node], t + 1u) == t + 1u) return;   // another caller took this node
    if (!keep_imp) { q[0] = 0ull; q[1] = 0ull; q[2] = 0ull; }
    const R fx = (R)((double)(long long)q0 * IMP_INV_SCALE), fy = (R)((double)(long long)q1 * IMP_INV_SCALE),
            fz = (R)((double)(long long)q2 * IMP_INV_SCALE);
    R o[19];
    const uint32_t h = collide<R>(d, o, fx, fy, fz, cc, r, t, bx.seed, bx.box_id);
    R* b = B + bx.pop_off;
#pragma unroll
    for (int i = 0; i < 19; ++i) b[pop_at(i, r)] = o[i];
    if (h) atomicOr(&ctrl->health, h);
}

// FIX_LANES threads per launched bead; thread j fixes the bead's touched-node
// slots j, j + FIX_LANES, ... (a bead that keeps its cell fills 8 slots, so
// one pass is the rule).  A node touched by several beads is fixed once
// (claim stamp).  skip_big: the beads of chains above BIG_CHAIN have their
// nodes in deferred tiles or in the overflow list.
constexpr int FIX_LANES = 16;   // <= touch_cap = 8 (substeps + 1)
template <typename R>
__global__ __launch_bounds__(256) void k_fixup(const BoxDev* __restrict__ boxes,
                                               const CollideConst<R>* __restrict__ ccs,
                                               const int32_t* __restrict__ bead_box, uint64_t bead0,
                                               uint32_t n_entries, ChainArgs ca, uint32_t* __restrict__ claim,
                                               const R* __restrict__ A, R* __restrict__ B,
                                               Ctrl* __restrict__ ctrl, uint32_t s_off, int keep_imp, int skip_big)
{
    const uint32_t e = blockIdx.x * 256u + threadIdx.x;
    if (e >= n_entries) return;
    const uint64_t g = bead0 + e / (uint32_t)FIX_LANES;
    const int j = (int)(e % (uint32_t)FIX_LANES);
    // independent loads together: the slot count, the box, the first slot
    // (read for every thread, used below the count) and the step; then, in
    // one more round, every field of the box and its collision constants
    const int cnt = ca.touched_cnt[g];
    const int bi = bead_box[g];
    const uint32_t r0 = ca.touched[g * ca.touch_cap + j];
    const uint32_t t = ctrl->step + s_off;
    const BoxDev& bx = boxes[bi];
    const FixBox fb = fix_box(bx);
    const int dense = bx.dense, nb = bx.N;
    const CollideConst<R> cc = ccs[bi];
    // a dense box's collide takes the impulses itself
    // (one test, so that no load waits for another's branch; the empty asm
    // keeps the box fields' loads above it, beside the tested ones)
    asm volatile("" ::"v"(fb.L), "v"(fb.pop_off), "v"(fb.node_off), "v"(fb.inv_L), "v"(fb.seed), "v"(fb.box_id));
    if ((j >= cnt) | (dense != 0) | ((skip_big != 0) & (nb > BIG_CHAIN))) return;
    fixup_node<R>(fb, cc, r0, ca.imp, claim, A, B, ctrl, t, keep_imp);
    for (int k = j + FIX_LANES; k < cnt; k += FIX_LANES)
        fixup_node<R>(fb, cc, ca.touched[g * ca.touch_cap + k], ca.imp, claim, A, B, ctrl, t, keep_imp);
}

// ------------------------------------------------ one kernel per step
// Batched steps whose chains all have at most BIG_CHAIN beads.  The first
// n_chain workgroups run one box's coupling each, the others collide the
// tiles.  The nodes a chain will hand impulses to are set aside beforehand:
// their bits are set in a node mask (one 64-bit word per wavefront of a
// tile), the tiles' lanes skip them, and the chain's workgroup collides them
// itself, with their impulses, once its substeps are done.  Both sides read
// A and write disjoint nodes of B, so nothing waits within the kernel, and a
// step is max(chain + its nodes, tiles) and one kernel boundary.  Bounds: the
// chain's serial substeps for small boxes, HBM for large ones.
//   - Set aside at the end of each step for the next: the stencil of the
//     bead's end position, one node wider on a side the bead may reach within
//     a step (set_aside); two masks and lists, by step parity.
//   - A bead that leaves them all the same hands its impulse to nodes that
//     the tiles have collided without it: those are listed, and the next
//     step's chain workgroup re-collides them (Aprev -> A) before anything
//     reads them; the box's tiles wait for that (a bounded wait; the chain
//     workgroups come first in the grid and wait for nothing).
// Every node gets the same collide call with the same impulse as in the
// fix-up form (k_couple, k_collide, k_fixup), so the bits are the same.
// Measured against that form, its coupling on a second queue (us per step):
// 16^3, 16 beads, FP64 20 against 40; 64^3, 64 beads 40 against 48; 128 boxes
// of 15^3, 32 beads 28 against 41; 256 boxes of 16^3..64^3 543 against 569 (the
// tiles alone: 545).

// the nodes (range per axis) that a bead at x with velocity v may touch in
// the next step: its stencil, wider by one node on a side whose distance to
// the cell's face is under twice the bead's ballistic path plus four thermal
// ones (or half a cell)
struct NodeRange { int lo[3], n[3]; };
__device__ __forceinline__ NodeRange set_aside(const BoxDev& bx, const double x[3], const double v[3])
{
    NodeRange r;
    const double th = 4.0 * sqrt(bx.mu / (3.0 * bx.mass));
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        double fr;
        const int i = cell_of(x[c], bx.L, (double)bx.L, bx.inv_L, fr);
        double m = 2.0 * fabs(v[c]) * bx.tau_lb + th;
        m = m < 0.5 ? m : 0.5;
        const int below = fr < m ? 1 : 0, above = fr > 1.0 - m ? 1 : 0;
        r.lo[c] = i - below;
        r.n[c] = 2 + below + above;
    }
    return r;
}

// set aside a bead's nodes, shared by the `step` threads of which this is the
// `first`: each node once, its mask bit set and appended to `list`.  Who
// comes first is decided by a hash table in LDS (linear probing; a returning
// atomic on the mask takes a microsecond or more, and each thread has two or
// three nodes), or without one (hash null), and for a node that finds no
// slot, by the mask bit's old value.
template <int HASH_BITS>
__device__ __forceinline__ void set_aside_nodes(const BoxDev& bx, const double x[3], const double v[3], int first,
                                                int step, unsigned long long* mask, uint32_t* list, uint32_t* n,
                                                uint32_t* hash)
{
    const NodeRange r = set_aside(bx, x, v);
    const int cnt = r.n[0] * r.n[1] * r.n[2];
    for (int q = first; q < cnt; q += step) {
        const int qyz = r.n[0] == 2 ? q >> 1 : q / 3, qx = q - qyz * r.n[0];
        const int qz = r.n[1] == 2 ? qyz >> 1 : qyz / 3, qy = qyz - qz * r.n[1];
        const uint32_t node = node_of(r.lo[0] + qx, r.lo[1] + qy, r.lo[2] + qz, bx.L);
        const unsigned long long bit = 1ull << (node % DSEG);
        int won = -1;
        if (HASH_BITS > 0) {
            uint32_t h = (node * 2654435761u) >> (32 - (HASH_BITS > 0 ? HASH_BITS : 1));
            for (int k = 0; k < 32 && won < 0; ++k) {
                const uint32_t old = atomicCAS(hash + h, 0u, node + 1u);
                if (old == 0u) won = 1;
                else if (old == node + 1u) won = 0;
                h = (h + 1u) & ((1u << HASH_BITS) - 1u);
            }
            if (won == 1) atomicOr(mask + dseg_of(bx, node), bit);
        }
        if (won < 0) won = !(atomicOr(mask + dseg_of(bx, node), bit) & bit);
        if (won) list[atomicAdd(n, 1u)] = node;
    }
}

// one tile, its set-aside lanes left out
template <typename R>
__device__ __forceinline__ void step_tile(const BoxDev* __restrict__ boxes, const CollideConst<R>* __restrict__ ccs,
                                          const uint32_t* __restrict__ tile_box, const StepArgs& sa, uint32_t tile,
                                          uint32_t lane, const R* A, R* B, Ctrl* __restrict__ ctrl, uint32_t t)
{
    const uint32_t p = t & 1u;
    const uint32_t w = __builtin_amdgcn_readfirstlane(lane / DSEG);   // wavefront-uniform: scalar loads
    const unsigned long long aside = sa.mask[p][DSEG_PER_TILE * tile + w];
    const int bi = (int)tile_box[tile];
    if (ctrl->step_pend[p ^ 1u] == defer_stamp(t - 1u) && sa.rec[bi].pend[p ^ 1u] == defer_stamp(t - 1u)) {
        uint32_t it = 0;
        while (__hip_atomic_load(&sa.rec[bi].fixed[p], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != defer_stamp(t)) {
            if (++it > SPIN_LIMIT) { atomicOr(&ctrl->health, H_SYNC); break; }
            __builtin_amdgcn_s_sleep(8);
        }
        __atomic_thread_fence(__ATOMIC_ACQUIRE);
    }
    if ((aside >> (lane % DSEG)) & 1ull) return;
    collide_tile<R>(boxes, ccs, tile_box, bi, tile, A, B, ctrl, t, nullptr, lane);
}

// BT threads per workgroup, at least W waves per SIMD, chains of at most MB
// beads.  A chain's workgroup needs couple_T lanes per bead; further threads clear the old mask and take
// the first of its nodes while the bead's lanes set the next step's nodes
// aside.
template <typename R, int BT, int W, int MB>
__global__ __launch_bounds__(BT) __attribute__((amdgpu_waves_per_eu(W))) void k_step(
    const BoxDev* __restrict__ boxes, const CollideConst<R>* __restrict__ ccs, const uint32_t* __restrict__ tile_box,
    const int32_t* __restrict__ list, uint32_t n_chain, uint32_t n_tiles, R* A, R* B, const R* Aprev, ChainArgs ca,
    unsigned long long* imp_prev, StepArgs sa, uint32_t* __restrict__ claim, Ctrl* __restrict__ ctrl, uint32_t s_off,
    int keep_imp)   // Aprev and B may be one buffer: the fix-up reads it, the tiles write it
{
    const uint32_t t = ctrl->step + s_off, p = t & 1u;
    if (blockIdx.x >= n_chain) {
        const uint32_t sub = BT == 256 ? 0u : __builtin_amdgcn_readfirstlane(threadIdx.x / 256u);
        const uint32_t lane = BT == 256 ? threadIdx.x : threadIdx.x % 256u;
        const uint32_t tile = (blockIdx.x - n_chain) * (BT / 256) + sub;
        if (BT == 256 || tile < n_tiles) step_tile<R>(boxes, ccs, tile_box, sa, tile, lane, A, B, ctrl, t);
        return;
    }
    __shared__ ChainLds<MB> sh;
    __builtin_amdgcn_s_setprio(3);   // latency-bound chain beside the bandwidth-bound tiles
    const int bi = list[blockIdx.x];
    const BoxDev bx = boxes[bi];   // a copy: its fields stay in registers across the substeps
    StepRec& rec = sa.rec[bi];
    const uint32_t n_def = rec.n[p], n_old = rec.n[p ^ 1u];
    const uint32_t from_top = (uint32_t)BT - 1u - threadIdx.x;   // threads without a bead come first
    const uint64_t l0 = (uint64_t)NODES_PER_BEAD * bx.bead_off;
    if (rec.pend[p ^ 1u] == defer_stamp(t - 1u)) {
        const FixBox fb = fix_box(bx);
        const uint32_t n_ovf = rec.n_ovf;
        for (uint32_t e = threadIdx.x; e < n_ovf; e += BT)
            fixup_node<R>(fb, ccs[bi], ca.touched[bx.bead_off * ca.touch_cap + e], imp_prev, claim, Aprev, A, ctrl,
                          t - 1u, keep_imp);
        all_stored();
        if (threadIdx.x == 0) {
            __threadfence();
            __hip_atomic_store(&rec.fixed[p], defer_stamp(t), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    // the other parity's mask held the previous step's nodes and takes the next step's
    for (uint32_t i = from_top; i < n_old; i += BT)
        atomicExch(&sa.mask[p ^ 1u][dseg_of(bx, sa.list[p ^ 1u][l0 + i])], 0ull);
    if (threadIdx.x == 0) { sh.n_ovf = 0u; sh.n_next = 0u; }
    uint32_t hbits;
    double xe[3], ve[3];
    const int T = bx.couple_T;
    if (T == 4) hbits = chain_substeps<R, 4, true>(bx, A, ca, t, sh, sa.mask[p], xe, ve);
    else if (T == 8) hbits = chain_substeps<R, 8, true>(bx, A, ca, t, sh, sa.mask[p], xe, ve);
    else hbits = chain_substeps<R, 16, true>(bx, A, ca, t, sh, sa.mask[p], xe, ve);
    constexpr int HASH = sizeof(sh.hash) / sizeof(uint32_t);
    __syncthreads();   // every impulse of the box is in the field, the positions in LDS are done with
    for (int i = (int)threadIdx.x; i < HASH; i += BT) sh.hash[i] = 0u;
    __syncthreads();
    if ((int)threadIdx.x / T < bx.N)
        set_aside_nodes<HASH == 1024 ? 10 : 12>(bx, xe, ve, (int)threadIdx.x % T, T, sa.mask[p ^ 1u],
                                                sa.list[p ^ 1u] + l0, &sh.n_next, sh.hash);
    const CollideConst<R> cc = ccs[bi];
    for (uint32_t i = from_top; i < n_def; i += BT) {
        const uint32_t r = sa.list[p][l0 + i];
        R d[19];
        gather_pre<R, false>(A + bx.pop_off, upwind_of(r, bx.L, bx.inv_L), d);
        unsigned long long* q = ca.imp + 3 * (bx.node_off + r);
        unsigned long long qc[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) qc[c] = __hip_atomic_load(q + c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (!keep_imp && (qc[0] | qc[1] | qc[2])) { q[0] = 0ull; q[1] = 0ull; q[2] = 0ull; }
        const R fx = (R)((double)(long long)qc[0] * IMP_INV_SCALE), fy = (R)((double)(long long)qc[1] * IMP_INV_SCALE),
                fz = (R)((double)(long long)qc[2] * IMP_INV_SCALE);
        R o[19];
        hbits |= collide<R>(d, o, fx, fy, fz, cc, r, t, bx.seed, bx.box_id);
        R* b = B + bx.pop_off;
#pragma unroll
        for (int k = 0; k < 19; ++k) b[pop_at(k, r)] = o[k];
    }
    __syncthreads();   // the next step's nodes are counted
    if (threadIdx.x == 0) {
        rec.n[p ^ 1u] = sh.n_next;
        rec.n_ovf = sh.n_ovf;
        rec.pend[p] = sh.n_ovf ? defer_stamp(t) : 0u;
        if (sh.n_ovf) ctrl->step_pend[p] = defer_stamp(t);   // every writer stores the same
        rec.t = t;
    }
    if (hbits) atomicOr(&ctrl->health, hbits);
}

// start of a run of one-kernel steps: every chain's nodes for step s_off
// (both masks are clear between runs)
__global__ __launch_bounds__(256) void k_step_begin(const BoxDev* __restrict__ boxes, const int32_t* __restrict__ list,
                                                    ChainArgs ca, StepArgs sa, const Ctrl* __restrict__ ctrl,
                                                    uint32_t s_off)
{
    __shared__ uint32_t n;
    const int bi = list[blockIdx.x];
    const BoxDev& bx = boxes[bi];
    const uint32_t p = (ctrl->step + s_off) & 1u;
    if (threadIdx.x == 0) n = 0u;
    __syncthreads();
    for (int e = (int)threadIdx.x; e < 4 * bx.N; e += 256) {
        const uint64_t g = bx.bead_off + (uint64_t)(e / 4);
        const double x[3] = {ca.x[3 * g], ca.x[3 * g + 1], ca.x[3 * g + 2]};
        const double v[3] = {ca.v[3 * g], ca.v[3 * g + 1], ca.v[3 * g + 2]};
        set_aside_nodes<0>(bx, x, v, e % 4, 4, sa.mask[p], sa.list[p] + NODES_PER_BEAD * bx.bead_off, &n, nullptr);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        StepRec& rec = sa.rec[bi];
        rec.n[p] = n;
        rec.n[p ^ 1u] = 0u;
        rec.pend[0] = rec.pend[1] = 0u;
        rec.fixed[0] = rec.fixed[1] = 0u;
        rec.n_ovf = 0u;
    }
}

// end of a run of one-kernel steps: the last step's impulses outside its
// set-aside nodes, both node masks cleared, and the step counter advanced (no workgroup reads it here: the
// step number comes from the box's record)
template <typename R>
__global__ __launch_bounds__(256) void k_step_end(const BoxDev* __restrict__ boxes,
                                                  const CollideConst<R>* __restrict__ ccs,
                                                  const int32_t* __restrict__ list, ChainArgs ca, StepArgs sa,
                                                  uint32_t* __restrict__ claim, const R* __restrict__ A,
                                                  R* __restrict__ B, Ctrl* __restrict__ ctrl, uint32_t advance,
                                                  int keep_imp)
{
    const int bi = list[blockIdx.x];
    const BoxDev& bx = boxes[bi];
    const StepRec& rec = sa.rec[bi];
    const uint32_t t = rec.t, p = t & 1u;
    if (rec.pend[p] == defer_stamp(t))
        for (uint32_t e = threadIdx.x; e < rec.n_ovf; e += 256)
            fixup_node<R>(fix_box(bx), ccs[bi], ca.touched[bx.bead_off * ca.touch_cap + e], ca.imp, claim, A, B, ctrl,
                          t, keep_imp);
    for (int q = 0; q < 2; ++q)
        for (uint32_t i = threadIdx.x; i < rec.n[q]; i += 256)
            sa.mask[q][dseg_of(bx, sa.list[q][NODES_PER_BEAD * bx.bead_off + i])] = 0ull;
    if (blockIdx.x == 0 && threadIdx.x == 0) ctrl->step += advance;
}

// End of a step that deferred tiles (one workgroup): fix the listed nodes
// outside the deferred tiles, then reset both list counts for the next step
// (the per-tile stamps need no clearing).  Runs after the plain collide, the
// deferred tiles' collide and the coupling.
template <typename R>
__global__ __launch_bounds__(256) void k_overflow(const BoxDev* __restrict__ boxes,
                                                   const CollideConst<R>* __restrict__ ccs,
                                                   const int32_t* __restrict__ bead_box, ChainArgs ca,
                                                   uint32_t* __restrict__ claim, const R* __restrict__ A,
                                                   R* __restrict__ B, Ctrl* __restrict__ ctrl, uint32_t s_off,
                                                   uint32_t advance)
{
    const uint32_t t = ctrl->step + s_off;
    const uint32_t n_ovf = min(ctrl->ovf_cnt, ca.ovf_cap);
    for (uint32_t e = threadIdx.x; e < n_ovf; e += blockDim.x) {
        const uint64_t g = ca.ovf[2 * (uint64_t)e];
        const uint32_t r = ca.ovf[2 * (uint64_t)e + 1];
        const int bi = bead_box[g];
        fixup_node<R>(fix_box(boxes[bi]), ccs[bi], r, ca.imp, claim, A, B, ctrl, t, 0);
    }
    __syncthreads();   // every thread has read the count and the step
    if (threadIdx.x == 0) {
        ctrl->defer_cnt = 0u;
        ctrl->ovf_cnt = 0u;
        ctrl->step += advance;   // the run's steps, when this kernel ends it (else 0)
    }
}

// Collide and stream one 256-node tile after the coupling stage: each node's
// impulse comes straight from the fixed-point field, which is cleared where
// it was set.  Same arithmetic as the fix-up, over a whole tile.
template <typename R>
__device__ __forceinline__ void collide_forced_tile(const BoxDev* __restrict__ boxes,
                                                    const CollideConst<R>* __restrict__ ccs,
                                                    const uint32_t* __restrict__ tile_box, int fixed_box,
                                                    uint32_t tile, unsigned long long* __restrict__ imp,
                                                    const R* __restrict__ A, R* __restrict__ B,
                                                    Ctrl* __restrict__ ctrl, uint32_t t, uint32_t lane)
{
    const int bi = fixed_box >= 0 ? fixed_box : (int)tile_box[tile];
    const BoxDev& bx = boxes[bi];
    const int L = bx.L;
    const uint32_t V = (uint32_t)L * L * L;
    const uint32_t r = (tile - bx.tile_begin) * 256u + lane;
    if (r >= V) return;
    const CollideConst<R> cc = ccs[bi];
    const Upwind up = upwind_of(r, L, bx.inv_L);
    R d[19];
    gather_pre<R, false>(A + bx.pop_off, up, d);
    unsigned long long* q = imp + 3 * (bx.node_off + r);
    const unsigned long long q0 = q[0], q1 = q[1], q2 = q[2];
    if (q0 | q1 | q2) { q[0] = 0ull; q[1] = 0ull; q[2] = 0ull; }
    const R fx = (R)((double)(long long)q0 * IMP_INV_SCALE), fy = (R)((double)(long long)q1 * IMP_INV_SCALE),
            fz = (R)((double)(long long)q2 * IMP_INV_SCALE);
    R o[19];
    const uint32_t h = collide<R>(d, o, fx, fy, fz, cc, r, t, bx.seed, bx.box_id);
    R* b = B + bx.pop_off;
#pragma unroll
    for (int i = 0; i < 19; ++i) __builtin_nontemporal_store(o[i], b + pop_at(i, r));
    if (h) atomicOr(&ctrl->health, h);
}

// every node of a dense box, after its coupling stage
template <typename R>
__global__ __launch_bounds__(256) void k_collide_forced(const BoxDev* __restrict__ boxes,
                                                        const CollideConst<R>* __restrict__ ccs,
                                                        const uint32_t* __restrict__ tile_box, int fixed_box,
                                                        uint32_t tile0, unsigned long long* __restrict__ imp,
                                                        const R* __restrict__ A, R* __restrict__ B,
                                                        Ctrl* __restrict__ ctrl, uint32_t s_off)
{
    collide_forced_tile<R>(boxes, ccs, tile_box, fixed_box, tile0 + blockIdx.x, imp, A, B, ctrl,
                           ctrl->step + s_off, threadIdx.x);
}

// the deferred tiles of a step, after its coupling stage, beside the plain
// collide of the other tiles (both only read the current state and write
// disjoint nodes)
template <typename R>
__global__ __launch_bounds__(256) void k_collide_deferred(const BoxDev* __restrict__ boxes,
                                                          const CollideConst<R>* __restrict__ ccs,
                                                          const uint32_t* __restrict__ tile_box,
                                                          const uint32_t* __restrict__ defer_list, uint32_t cap,
                                                          unsigned long long* __restrict__ imp,
                                                          const R* __restrict__ A, R* __restrict__ B,
                                                          Ctrl* __restrict__ ctrl, uint32_t s_off)
{
    // one wavefront per listed segment
    const uint32_t t = ctrl->step + s_off;
    const uint32_t n = min(ctrl->defer_cnt, cap);
    // the wavefront index made uniform: the segment, its tile and box, and the
    // box constants then sit in scalar registers
    const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x / DSEG), lane = threadIdx.x % DSEG;
    for (uint32_t k = blockIdx.x * DSEG_PER_TILE + w; k < n; k += gridDim.x * DSEG_PER_TILE) {
        const uint32_t seg = defer_list[k];
        collide_forced_tile<R>(boxes, ccs, tile_box, -1, seg / DSEG_PER_TILE, imp, A, B, ctrl, t,
                               (seg % DSEG_PER_TILE) * DSEG + lane);
    }
}

// --------------------------------------------------------------- advance
__global__ void k_advance(Ctrl* ctrl, uint32_t n)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) ctrl->step += n;
}

// ---------------------------------------------------------- queue probe
// Do two streams run on hardware queues of their own?  k_probe_wait on one of
// them waits for the flag that k_probe_set, launched after it on the other,
// sets; on one queue the second starts when the first has ended, at its limit.
constexpr uint64_t PROBE_TICKS = 20000;   // of the 100 MHz clock: 200 us
__global__ void k_probe_wait(uint32_t* probe)
{
    const uint64_t t0 = wall_clock64();
    bool set = false;
    while (!set && wall_clock64() - t0 < PROBE_TICKS) {
        set = __hip_atomic_load(probe, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u;
        __builtin_amdgcn_s_sleep(8);
    }
    probe[1] = set ? 1u : 0u;
}
__global__ void k_probe_set(uint32_t* probe, uint32_t value)
{
    __hip_atomic_store(probe, value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ----------------------------------------------------------------- stats
// Per tile of 256 nodes: FP64 sums of mass deviation, momentum, squared modes,
// negative population count.  Layout of a record: [0] sum drho, [1..3] j,
// [4] neg count, [5..23] sum m_k^2 (m of the deviations; m_0 = drho).
// Every sum is a fixed tree (butterfly within each wavefront, then the four
// wavefronts in order, then fixed chunks of a box's tiles, then the chunks in
// order), so a state gives the same bits on every call and in any batch.
constexpr int NSTAT = NSTAT_REC;

__device__ __forceinline__ double lane_value(double v, int lane)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                            __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// Sum of v[k] over the 64 lanes of a wavefront for k < NV, with every lane of
// the wavefront active: within each 16-lane row by DPP moves (neighbour in the
// pair, the other pair of the quad, the mirrored quad, the mirrored half-row;
// each stage adds the same two values in either order, so all 16 lanes hold
// the same row sum), then the four row sums in row order.  The NV sums are
// advanced stage by stage so that their moves issue back to back.  Every lane
// returns the same bits.
template <int NV>
__device__ __forceinline__ void wave_sums(double v[NV])
{
#pragma unroll
    for (int k = 0; k < NV; ++k) v[k] += dpp_from<0xB1>(v[k]);    // quad_perm [1,0,3,2]
#pragma unroll
    for (int k = 0; k < NV; ++k) v[k] += dpp_from<0x4E>(v[k]);    // quad_perm [2,3,0,1]
#pragma unroll
    for (int k = 0; k < NV; ++k) v[k] += dpp_from<0x141>(v[k]);   // row_half_mirror
#pragma unroll
    for (int k = 0; k < NV; ++k) v[k] += dpp_from<0x140>(v[k]);   // row_mirror
#pragma unroll
    for (int k = 0; k < NV; ++k)
        v[k] = ((lane_value(v[k], 0) + lane_value(v[k], 16)) + lane_value(v[k], 32)) + lane_value(v[k], 48);
}

// sum of acc[0..NV-1] over a 256-thread block (all threads active): per
// wavefront, then wavefronts 0..3 in order; the result is valid in threads
// 0..NV-1 (thread k holds sum k).  acc is consumed.
template <int NV>
__device__ __forceinline__ double block_sum256(double acc[NV], double (*lds)[NV])
{
    const int wv_ = threadIdx.x >> 6, ln = threadIdx.x & 63;
    wave_sums<NV>(acc);
    if (ln == 0) {
#pragma unroll
        for (int k = 0; k < NV; ++k) lds[wv_][k] = acc[k];
    }
    __syncthreads();
    double r = 0.0;
    if ((int)threadIdx.x < NV) r = ((lds[0][threadIdx.x] + lds[1][threadIdx.x]) + lds[2][threadIdx.x]) + lds[3][threadIdx.x];
    return r;
}

// Sums of v[0..23] over the 64 lanes of a wavefront (all active), written to
// dst[0..23] by the first 16: at each stage a lane keeps half of its values
// and hands the other half to its partner (mirrored row, mirrored half-row,
// mirrored quad, neighbour: the partner differs in the bit that says which
// half is kept and agrees in those before), so 24 values cost ~170
// instructions where a full butterfly of each costs ~550; then the four rows.
__device__ __forceinline__ void wave_sums24(const double v[24], double* dst)
{
    const int lane = (int)(threadIdx.x & 63u);
    const bool b3 = lane & 8, b2 = lane & 4, b1 = lane & 2, b0 = lane & 1;
    double a[12], c[6], d[3];
#pragma unroll
    for (int i = 0; i < 12; ++i) a[i] = (b3 ? v[i + 12] : v[i]) + dpp_from<0x140>(b3 ? v[i] : v[i + 12]);
#pragma unroll
    for (int i = 0; i < 6; ++i) c[i] = (b2 ? a[i + 6] : a[i]) + dpp_from<0x141>(b2 ? a[i] : a[i + 6]);
#pragma unroll
    for (int i = 0; i < 3; ++i) d[i] = (b1 ? c[i + 3] : c[i]) + dpp_from<0x1B>(b1 ? c[i] : c[i + 3]);
    double r0 = (b0 ? d[2] : d[0]) + dpp_from<0xB1>(b0 ? d[0] : d[2]);
    double r1 = d[1] + dpp_from<0xB1>(d[1]);
#pragma unroll
    for (int o = 16; o < 64; o <<= 1) { r0 += __shfl_xor(r0, o, 64); r1 += __shfl_xor(r1, o, 64); }
    if (lane < 16) {
        const int i = (b3 ? 12 : 0) + (b2 ? 6 : 0) + (b1 ? 3 : 0);
        dst[i + (b0 ? 2 : 0)] = r0;
        if (!b0) dst[i + 1] = r1;
    }
}

// grid (records of the largest box, boxes): block (c, box) sums the
// stat_tpb(n_tiles) tiles from c * stat_tpb on, one node per thread and four
// tiles, into record stat_off + c.  Bound by HBM on large boxes (one read of
// each population); on small ones by how many wavefronts share the nodes (a
// 64^3 box's 64 blocks of 256 threads took 27 us).  The whole call, with one
// copy to the host instead of four: 64^3 106 -> 39 us, 128 boxes of 15^3 178
// -> 61, 256^3 304 -> 267 (1.275 GB).
__device__ __forceinline__ float uniform_value(float v)
{
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}
__device__ __forceinline__ double uniform_value(double v)
{
    return __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(v)),
                            __builtin_amdgcn_readfirstlane(__double2loint(v)));
}

constexpr int STAT_BLOCK = 1024;
template <typename R, bool O32>
__global__ __launch_bounds__(STAT_BLOCK) void k_stats(const BoxDev* __restrict__ boxes, const R* __restrict__ A,
                                                      double* __restrict__ part)
{
    __shared__ double red[STAT_BLOCK / 64][NSTAT];
    const BoxDev& bx = boxes[blockIdx.y];
    const uint32_t c = blockIdx.x, tpb = stat_tpb(bx.n_tiles);
    if (c >= stat_recs_of(bx.n_tiles)) return;
    const uint32_t V = (uint32_t)bx.L * bx.L * bx.L;
    const R* a = A + bx.pop_off;
    // n_i = fl(w_i rho0) + delta_i (FP64) is negative exactly when delta_i
    // lies below -fl(w_i rho0): the rounded sum of two doubles keeps the sign
    // of the exact one.  For FP32 storage the test compares delta_i with the
    // smallest float not below that double, which decides the same; the
    // count is an integer.
    R thr[19];
#pragma unroll
    for (int i = 0; i < 19; ++i) {
        const double cth = -(wv(i) * bx.rho0);
        R f = (R)cth;
        if ((double)f < cth) f = nextafter(f, (R)INFINITY);
        thr[i] = uniform_value(f);   // the same in every lane: kept in scalar registers
    }
    double acc[NSTAT];
#pragma unroll
    for (int k = 0; k < NSTAT; ++k) acc[k] = 0.0;
    uint32_t neg = 0;
    for (uint32_t k = threadIdx.x; k < 256u * tpb; k += STAT_BLOCK) {
        const uint32_t r = c * tpb * 256u + k;
        if (r >= V) break;
        const Upwind up = upwind_of(r, bx.L, bx.inv_L);
        R dr[19];
        if (O32) gather_pre32<R>(a, up, dr);
        else gather_pre<R, false>(a, up, dr);
        double d[19], m[19];
#pragma unroll
        for (int i = 0; i < 19; ++i) {
            d[i] = (double)dr[i];
            neg += dr[i] < thr[i] ? 1u : 0u;
        }
        to_modes<double>(d, m);
        acc[0] += m[0]; acc[1] += m[1]; acc[2] += m[2]; acc[3] += m[3];
#pragma unroll
        for (int q = 0; q < 19; ++q) acc[5 + q] += m[q] * m[q];
    }
    acc[4] = (double)neg;   // what adding 1.0 per negative population gives, exactly
    wave_sums24(acc, red[threadIdx.x / 64]);
    __syncthreads();
    if (threadIdx.x < NSTAT) {
        double s = 0.0;
        for (int w = 0; w < STAT_BLOCK / 64; ++w) s += red[w][threadIdx.x];
        part[(uint64_t)(bx.stat_off + c) * NSTAT + threadIdx.x] = s;
    }
}

// sum of records rec[0..n-1], by a block of 256 threads: ten ranges of every
// tenth record, then the ranges in order; the result in threads 0..NSTAT-1
__device__ __forceinline__ double sum_records(const double* __restrict__ rec, uint32_t n, double (*red)[NSTAT])
{
    const uint32_t g = threadIdx.x / NSTAT, k = threadIdx.x % NSTAT;
    if (g < 10) {
        double s = 0.0;
#pragma unroll 8
        for (uint32_t i = g; i < n; i += 10) s += rec[(uint64_t)i * NSTAT + k];
        red[g][k] = s;
    }
    __syncthreads();
    double s = 0.0;
    if (threadIdx.x < NSTAT)
        for (int w = 0; w < 10; ++w) s += red[w][threadIdx.x];
    return s;
}

// boxes of more than STAT_DIRECT records: grid (STAT_CHUNKS, boxes), block
// (c, box) sums range c of the box's records, into slot c behind them
__global__ __launch_bounds__(256) void k_stats_mid(const BoxDev* __restrict__ boxes, double* part)
{
    __shared__ double red[10][NSTAT];
    const BoxDev& bx = boxes[blockIdx.y];
    const uint32_t nrec = stat_recs_of(bx.n_tiles);
    if (nrec <= STAT_DIRECT) return;
    const uint32_t per = (nrec + STAT_CHUNKS - 1) / STAT_CHUNKS;
    const uint32_t t0 = min(nrec, blockIdx.x * per), t1 = min(nrec, t0 + per);
    const double s = sum_records(part + (uint64_t)(bx.stat_off + t0) * NSTAT, t1 - t0, red);
    if (threadIdx.x < NSTAT) part[(uint64_t)(bx.stat_off + nrec + blockIdx.x) * NSTAT + threadIdx.x] = s;
}

// one block per box: the box's record of OBS_REC doubles, [0..23] the fluid
// sums, then the chain sums, [35] the neighbour-list builds; block 0 also
// writes the health bits and the step behind the last record, so that one
// copy brings everything to the host.  Chain sums: [0..2] sum x, [3..5] sum m v,
// [6..8] sum fc, [9] sum over the chains of R_e^2, then after the second pass
// [10] sum over beads of |x - com of the bead's chain|^2.
constexpr int NCHAIN = NCHAIN_REC;

__global__ __launch_bounds__(256) void k_obs(const BoxDev* __restrict__ boxes, ChainArgs ca,
                                             const double* __restrict__ part, const Ctrl* __restrict__ ctrl,
                                             double* __restrict__ out)
{
    __shared__ double red10[10][NSTAT];
    {
        const BoxDev& bx = boxes[blockIdx.x];
        const uint32_t nrec = stat_recs_of(bx.n_tiles);
        const double s = nrec <= STAT_DIRECT
                             ? sum_records(part + (uint64_t)bx.stat_off * NSTAT, nrec, red10)
                             : sum_records(part + (uint64_t)(bx.stat_off + nrec) * NSTAT, STAT_CHUNKS, red10);
        if (threadIdx.x < NSTAT) out[(uint64_t)blockIdx.x * OBS_REC + threadIdx.x] = s;
        if (threadIdx.x == 0) {
            out[(uint64_t)blockIdx.x * OBS_REC + NSTAT + NCHAIN] = (double)ca.nl_rebuilds[blockIdx.x];
            if (blockIdx.x == 0) {
                out[(uint64_t)gridDim.x * OBS_REC] = (double)ctrl->health;
                out[(uint64_t)gridDim.x * OBS_REC + 1] = (double)ctrl->step;
            }
        }
    }
    __shared__ double red[4][9];
    __shared__ double red1[4][1];
    __shared__ double sums[9];
    __shared__ double ccom[3 * MAXB];   // per-chain centres of mass (several chains)
    const BoxDev& bx = boxes[blockIdx.x];
    const int N = bx.N;
    const int n = bx.chain_len, M = N > 0 ? N / n : 0;
    double acc[9];
    for (int k = 0; k < 9; ++k) acc[k] = 0.0;
    for (int b = threadIdx.x; b < N; b += 256) {
        const uint64_t g = bx.bead_off + b;
        for (int c = 0; c < 3; ++c) {
            acc[c] += ca.x[3 * g + c];
            acc[3 + c] += bx.mass * ca.v[3 * g + c];
            acc[6 + c] += ca.fc[3 * g + c];
        }
    }
    const double s9 = block_sum256<9>(acc, red);
    if (threadIdx.x < 9) sums[threadIdx.x] = s9;
    // several chains: each chain's centre of mass, in bead order
    if (M > 1)
        for (int ch = threadIdx.x; ch < M; ch += 256) {
            double cm[3] = {0, 0, 0};
            for (int k = 0; k < n; ++k) {
                const uint64_t g = bx.bead_off + (uint64_t)ch * n + k;
                for (int c = 0; c < 3; ++c) cm[c] += ca.x[3 * g + c];
            }
            for (int c = 0; c < 3; ++c) ccom[3 * ch + c] = cm[c] / n;
        }
    __syncthreads();
    double s = 0.0;
    for (int b = threadIdx.x; b < N; b += 256) {
        const uint64_t g = bx.bead_off + b;
        for (int c = 0; c < 3; ++c) {
            const double d = ca.x[3 * g + c] - (M > 1 ? ccom[3 * (b / n) + c] : sums[c] / N);
            s += d * d;
        }
    }
    double s1[1] = {s};
    const double sg = block_sum256<1>(s1, red1);
    if (threadIdx.x == 0) {
        double* o = out + (uint64_t)blockIdx.x * OBS_REC + NSTAT;
        for (int k = 0; k < 9; ++k) o[k] = sums[k];
        o[10] = sg;
        double e2 = 0.0;
        for (int ch = 0; ch < M; ++ch) {
            const uint64_t g0 = bx.bead_off + (uint64_t)ch * n, g1 = g0 + n - 1;
            for (int c = 0; c < 3; ++c) {
                const double d = ca.x[3 * g1 + c] - ca.x[3 * g0 + c];
                e2 += d * d;
            }
        }
        o[9] = e2;
    }
}

// ---------------------------------------------------------- checkpoints
// Planes q0 .. q0 + nq - 1 of a box between the pull layout and the canonical
// one, FP64 full populations n_q(r), node r fastest: n_q(r) = w_q rho0 +
// p_q(r - c_q).  Bound by the copy over PCIe that follows or precedes; the
// host loops that did this took 33 ms for a 64^3 box, out and back.
template <typename R>
__global__ __launch_bounds__(256) void k_export(const BoxDev* __restrict__ boxes, int bi, const R* __restrict__ A,
                                                double* __restrict__ n, int q0, int nq)
{
#pragma clang fp contract(off)   // w_q rho0 rounded first: an import takes the same value off again
    const BoxDev& bx = boxes[bi];
    const uint32_t V = (uint32_t)bx.L * bx.L * bx.L, r = blockIdx.x * 256u + threadIdx.x;
    if (r >= V) return;
    const Upwind up = upwind_of(r, bx.L, bx.inv_L);
    const R* a = A + bx.pop_off;
#pragma unroll
    for (int q = 0; q < 19; ++q)
        if (q >= q0 && q < q0 + nq) n[(uint64_t)(q - q0) * V + r] = wv(q) * bx.rho0 + (double)a[pop_at(q, up.src(q))];
}
template <typename R>
__global__ __launch_bounds__(256) void k_import(const BoxDev* __restrict__ boxes, int bi, const double* __restrict__ n,
                                                R* __restrict__ A, int q0, int nq)
{
#pragma clang fp contract(off)
    const BoxDev& bx = boxes[bi];
    const uint32_t V = (uint32_t)bx.L * bx.L * bx.L, r = blockIdx.x * 256u + threadIdx.x;
    if (r >= V) return;
    const Upwind up = upwind_of(r, bx.L, bx.inv_L);
    R* a = A + bx.pop_off;
#pragma unroll
    for (int q = 0; q < 19; ++q)
        if (q >= q0 && q < q0 + nq) a[pop_at(q, up.src(q))] = (R)(n[(uint64_t)(q - q0) * V + r] - wv(q) * bx.rho0);
}
// zeros behind each box's last node (the buffer served as staging space)
template <typename R>
__global__ __launch_bounds__(256) void k_clear_tails(const BoxDev* __restrict__ boxes, R* __restrict__ A)
{
    const BoxDev& bx = boxes[blockIdx.x];
    const uint32_t V = (uint32_t)bx.L * bx.L * bx.L, end = (V + PTILE - 1) / PTILE * PTILE;
    for (uint32_t e = threadIdx.x; e < 19u * (end - V); e += 256)
        A[bx.pop_off + pop_at((int)(e / (end - V)), V + e % (end - V))] = (R)0;
}

// --------------------------------------------------------------- launchers
static ChainArgs chain_args(const LaunchCtx& c)
{
    return ChainArgs{c.x, c.v, c.f, c.fc, c.nl_cnt, c.nl_idx, c.nl_x0, c.nl_cap, c.imp, c.touched,
                     c.touched_cnt, c.touch_cap, c.nl_rebuilds, c.vhist, c.hist_len, c.total_beads, c.tape,
                     c.tape_x0, c.tape_vo, c.tape_fo,
                     c.defer_on ? c.defer : nullptr, c.dclaim, c.defer_list, c.defer_cap, c.ovf, c.ovf_cap, c.ovm};
}

template <typename R, int W, bool PERSIST, int BT = 256>
static void launch_collide_v(const LaunchCtx& c, const void* A, void* B, int fixed_box, uint32_t tile0,
                             uint32_t n_tiles, uint32_t s_off)
{
    constexpr uint32_t M = BT / 256;
    const uint32_t groups = (n_tiles + M - 1) / M;
    const uint32_t grid = PERSIST ? std::min<uint32_t>(groups, (uint32_t)(c.n_cu * W)) : groups;
    hipLaunchKernelGGL((k_collide<R, W, PERSIST, BT>), dim3(grid), dim3(BT), 0, c.stream, c.boxes,
                       (const CollideConst<R>*)c.ccs, c.tile_box, fixed_box, tile0, n_tiles, (const R*)A, (R*)B,
                       c.ctrl, s_off, c.defer_on ? (const uint32_t*)c.defer : nullptr);
}

template <typename R>
hipError_t launch_collide(const LaunchCtx& c, const void* A, void* B, int fixed_box, uint32_t tile0,
                          uint32_t n_tiles, uint32_t s_off)
{
    if (n_tiles == 0) return hipSuccess;
    switch (c.collide_variant) {
    case 0: launch_collide_v<R, 4, false>(c, A, B, fixed_box, tile0, n_tiles, s_off); break;
    case 1: launch_collide_v<R, 5, false>(c, A, B, fixed_box, tile0, n_tiles, s_off); break;
    case 2: launch_collide_v<R, 6, false>(c, A, B, fixed_box, tile0, n_tiles, s_off); break;
    case 3: launch_collide_v<R, 7, false>(c, A, B, fixed_box, tile0, n_tiles, s_off); break;
    case 4: launch_collide_v<R, 8, false>(c, A, B, fixed_box, tile0, n_tiles, s_off); break;
    case 5: launch_collide_v<R, 4, true>(c, A, B, fixed_box, tile0, n_tiles, s_off); break;
    case 6: launch_collide_v<R, 5, true>(c, A, B, fixed_box, tile0, n_tiles, s_off); break;
    case 7: launch_collide_v<R, 6, true>(c, A, B, fixed_box, tile0, n_tiles, s_off); break;
    case 8: launch_collide_v<R, 7, true>(c, A, B, fixed_box, tile0, n_tiles, s_off); break;
    case 9: launch_collide_v<R, 8, true>(c, A, B, fixed_box, tile0, n_tiles, s_off); break;
    case 10: launch_collide_v<R, 4, false, 512>(c, A, B, fixed_box, tile0, n_tiles, s_off); break;
    case 11: launch_collide_v<R, 6, false, 512>(c, A, B, fixed_box, tile0, n_tiles, s_off); break;
    default: launch_collide_v<R, 4, false, 1024>(c, A, B, fixed_box, tile0, n_tiles, s_off); break;
    }
    return hipGetLastError();
}

template <typename R>
hipError_t launch_fixup(const LaunchCtx& c, const void* A, void* B, uint64_t bead0, uint64_t n_beads,
                        uint32_t s_off)
{
    if (n_beads == 0) return hipSuccess;
    if (c.touch_cap < FIX_LANES) return hipErrorInvalidValue;
    const uint32_t n = (uint32_t)(n_beads * (uint64_t)FIX_LANES);
    hipLaunchKernelGGL(k_fixup<R>, dim3((n + 255) / 256), dim3(256), 0, c.stream, c.boxes,
                       (const CollideConst<R>*)c.ccs, c.bead_box, bead0, n, chain_args(c), c.claim,
                       (const R*)A, (R*)B, c.ctrl, s_off, c.keep_imp, c.defer_on);
    return hipGetLastError();
}

template <typename R>
hipError_t launch_collide_deferred(const LaunchCtx& c, const void* A, void* B, uint32_t s_off)
{
    if (!c.defer_on || c.defer_cap == 0) return hipErrorInvalidValue;
    // a grid of a few blocks per CU strides over the list (its length is
    // known on the device only)
    const uint32_t grid = std::min<uint32_t>((c.defer_cap + DSEG_PER_TILE - 1) / DSEG_PER_TILE, (uint32_t)(4 * c.n_cu));
    hipLaunchKernelGGL(k_collide_deferred<R>, dim3(grid), dim3(256), 0, c.stream, c.boxes,
                       (const CollideConst<R>*)c.ccs, c.tile_box, (const uint32_t*)c.defer_list, c.defer_cap, c.imp,
                       (const R*)A, (R*)B, c.ctrl, s_off);
    return hipGetLastError();
}

template <typename R>
hipError_t launch_overflow(const LaunchCtx& c, const void* A, void* B, uint32_t s_off, uint32_t advance)
{
    if (!c.defer_on) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_overflow<R>, dim3(1), dim3(256), 0, c.stream, c.boxes, (const CollideConst<R>*)c.ccs,
                       c.bead_box, chain_args(c), c.claim, (const R*)A, (R*)B, c.ctrl, s_off, advance);
    return hipGetLastError();
}

template <typename R>
hipError_t launch_collide_forced(const LaunchCtx& c, const void* A, void* B, int fixed_box, uint32_t tile0,
                                 uint32_t n_tiles, uint32_t s_off)
{
    if (n_tiles == 0) return hipSuccess;
    hipLaunchKernelGGL(k_collide_forced<R>, dim3(n_tiles), dim3(256), 0, c.stream, c.boxes,
                       (const CollideConst<R>*)c.ccs, c.tile_box, fixed_box, tile0, c.imp, (const R*)A, (R*)B,
                       c.ctrl, s_off);
    return hipGetLastError();
}

template <typename R>
hipError_t launch_couple(const LaunchCtx& c, const void* A, const int32_t* list, int n_list, int block,
                         uint32_t s_off)
{
    if (n_list == 0) return hipSuccess;
    if (block > 1024) return hipErrorInvalidValue;   // larger chains take the one-workgroup-per-chain kernel
    if (block > 256)
        hipLaunchKernelGGL((k_couple<R, 1024>), dim3(n_list), dim3(block), 0, c.stream, c.boxes, list, (const R*)A,
                           chain_args(c), c.ctrl, s_off);
    else
        hipLaunchKernelGGL((k_couple<R, 256>), dim3(n_list), dim3(block), 0, c.stream, c.boxes, list, (const R*)A,
                           chain_args(c), c.ctrl, s_off);
    return hipGetLastError();
}

static StepArgs step_args(const LaunchCtx& c) { return StepArgs{{c.nmask[0], c.nmask[1]}, {c.nlist[0], c.nlist[1]}, c.step_rec}; }

// Launch shapes of k_step (threads, waves per SIMD it is held to), us per step:
//   - Chains to 64 beads, few tiles: 512 threads, whose spare ones take set-aside
//     nodes and shorten the chain's end; many: 256, where the tiles set the
//     time.  The line at 16 tiles per CU lies between the chains' lengths (256
//     against 512 threads, FP32): 4 per CU, 16 beads 23.0 and 22.4, 64 beads
//     48.4 and 44.7; 16 per CU, 16 beads 43.0 and 47.5, 64 beads 81.0 and 79.6;
//     62 per CU, 64 beads 113 and 120.
//   - Held to four waves per SIMD (128 VGPRs), as the tiles want it, the coupling
//     code spills 55 VGPRs in FP32 and 85 in FP64 (free it takes 170 and 196).
//     In FP64 that traffic shows with many chains of more than 32 beads at
//     once: 128 boxes of 15^3, 64 beads 91.6, with three waves (170 VGPRs) 67.0;
//     256 boxes of 12^3 101 and 78.  Above one chain per CU the fewer waves
//     cost more (500 boxes of 10^3 126.5 and 128.3), as they do below 33 beads.
//   - Chains of 65 to 128 beads: 512 threads, three waves; in FP32 four where
//     the tiles set the time or chains fill the CUs.  1024 threads, three and
//     four waves: FP64 32 boxes of 32^3, 100 beads 114, 91, 122; FP32 128^3,
//     128 beads 88.9, 79.7, 91.5; 900 boxes of 16^3 426, 403, 348.
//   - Longer chains need 1024 threads, and with them four waves.
constexpr int STEP_FEW_TILES_PER_CU = 16;

template <typename R, int BT, int W, int MB>
static void launch_step_v(const LaunchCtx& c, const int32_t* list, int n_list, void* A, void* B, const void* Aprev,
                          unsigned long long* imp_prev, uint32_t n_tiles, uint32_t s_off)
{
    constexpr uint32_t M = BT / 256;
    hipLaunchKernelGGL((k_step<R, BT, W, MB>), dim3((uint32_t)n_list + (n_tiles + M - 1) / M), dim3(BT), 0, c.stream,
                       c.boxes, (const CollideConst<R>*)c.ccs, c.tile_box, list, (uint32_t)n_list, n_tiles, (R*)A,
                       (R*)B, (const R*)Aprev, chain_args(c), imp_prev, step_args(c), c.claim, c.ctrl, s_off,
                       c.keep_imp);
}

template <typename R>
hipError_t launch_step(const LaunchCtx& c, const int32_t* list, int n_list, int block, int max_n, void* A, void* B,
                       const void* Aprev, unsigned long long* imp_prev, uint32_t n_tiles, uint32_t s_off)
{
    if (n_list <= 0 || n_tiles == 0 || block > 1024 || block < 4 * max_n || !c.step_rec) return hipErrorInvalidValue;
    const bool few = n_tiles <= (uint32_t)(STEP_FEW_TILES_PER_CU * c.n_cu);
    if (block > 512) {
        launch_step_v<R, 1024, 4, 256>(c, list, n_list, A, B, Aprev, imp_prev, n_tiles, s_off);
    } else if (block > 256) {
        const bool tiles_bound = n_tiles > (uint32_t)(2 * STEP_FEW_TILES_PER_CU * c.n_cu) || n_list > c.n_cu / 2;
        if (sizeof(R) == 4 && tiles_bound)
            launch_step_v<R, 512, 4, 128>(c, list, n_list, A, B, Aprev, imp_prev, n_tiles, s_off);
        else
            launch_step_v<R, 512, 3, 128>(c, list, n_list, A, B, Aprev, imp_prev, n_tiles, s_off);
    } else if (few) {
        if (sizeof(R) == 8 && max_n > 32 && n_list <= c.n_cu)
            launch_step_v<R, 512, 3, 64>(c, list, n_list, A, B, Aprev, imp_prev, n_tiles, s_off);
        else
            launch_step_v<R, 512, 4, 64>(c, list, n_list, A, B, Aprev, imp_prev, n_tiles, s_off);
    } else {
        launch_step_v<R, 256, 4, 64>(c, list, n_list, A, B, Aprev, imp_prev, n_tiles, s_off);
    }
    return hipGetLastError();
}

hipError_t launch_step_begin(const LaunchCtx& c, const int32_t* list, int n_list, uint32_t s_off)
{
    if (n_list <= 0 || !c.step_rec) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_step_begin, dim3(n_list), dim3(256), 0, c.stream, c.boxes, list, chain_args(c), step_args(c),
                       c.ctrl, s_off);
    return hipGetLastError();
}

template <typename R>
hipError_t launch_step_end(const LaunchCtx& c, const int32_t* list, int n_list, const void* A, void* B,
                           uint32_t advance)
{
    if (n_list <= 0 || !c.step_rec) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_step_end<R>, dim3(n_list), dim3(256), 0, c.stream, c.boxes, (const CollideConst<R>*)c.ccs,
                       list, chain_args(c), step_args(c), c.claim, (const R*)A, (R*)B, c.ctrl, advance, c.keep_imp);
    return hipGetLastError();
}

template <typename R>
hipError_t launch_couple_big(const LaunchCtx& c, const void* A, const int32_t* list, int n_list, int max_n,
                             uint32_t s_off, hipEvent_t after_table, const void* Aprev, int single_box,
                             uint32_t wait_head, int zero_head, int stamp_next)
{
    if (n_list == 0) return hipSuccess;
    if (c.nl_cap > NL_SLOTS || max_n > WG_MAXB || max_n <= 0) return hipErrorInvalidValue;
    if ((Aprev || wait_head || stamp_next) && (c.dense_max_tiles || !c.defer_on)) return hipErrorInvalidValue;
    if (wait_head && (Aprev || after_table)) return hipErrorInvalidValue;
    const ChainArgs ca = chain_args(c);
    if (c.dense_max_tiles)
        hipLaunchKernelGGL(k_node_field<R>, dim3(c.dense_max_tiles, n_list), dim3(256), 0, c.stream, c.boxes, list,
                           (const R*)A, (R*)c.field);
    if (!wait_head && c.big_sparse)   // a dense box's beads read the node field
        hipLaunchKernelGGL(k_near_nodes<R>, dim3((max_n * NEAR + 255) / 256, n_list), dim3(256), 0, c.stream,
                           c.boxes, list, (R*)A, ca, (R*)c.near_u, c.near_c, c.ctrl, s_off,
                           (const CollideConst<R>*)c.ccs, c.bead_box, c.claim, (const R*)Aprev,
                           n_list == 1 && single_box >= 0 ? single_box : -1,
                           n_list == 1 && single_box >= 0 ? c.boxes_host[single_box] : BoxDev{}, zero_head);
    if (after_table) {
        const hipError_t e = hipEventRecord(after_table, c.stream);
        if (e != hipSuccess) return e;
    }
    if (max_n <= 512)
        hipLaunchKernelGGL((k_chain_wg<R, 512>), dim3(n_list), dim3(512), 0, c.stream, c.boxes, list, (const R*)A, ca,
                       (const R*)c.near_u, (const int4*)c.near_c, (const R*)c.field, c.sub_rec, c.ctrl, s_off,
                       c.bead_box,
                       (Aprev || wait_head) ? 1 : 0, wait_head, stamp_next);
    else
        hipLaunchKernelGGL((k_chain_wg<R, WG_MAXB>), dim3(n_list), dim3(WG_MAXB), 0, c.stream, c.boxes, list, (const R*)A, ca,
                       (const R*)c.near_u, (const int4*)c.near_c, (const R*)c.field, c.sub_rec, c.ctrl, s_off,
                       c.bead_box,
                       (Aprev || wait_head) ? 1 : 0, wait_head, stamp_next);
    if (c.big_sparse) {
        const uint32_t n_spread = (uint32_t)(max_n * 8 + 255) / 256;
        const uint32_t n_defer = c.defer_on ? (uint32_t)(max_n * NEAR + 255) / 256 : 0u;
        hipLaunchKernelGGL(k_spread, dim3(n_spread + n_defer, n_list), dim3(256), 0, c.stream, c.boxes, list, ca,
                           (const double*)c.sub_rec, (const int4*)c.near_c, c.ctrl, s_off, n_spread);
    }
    if (c.dense_max_tiles) {
        hipLaunchKernelGGL(k_dense_impulse, dim3((c.dense_max_tiles * 256 + DENSE_NODES - 1) / DENSE_NODES, n_list),
                           dim3(1024), 0, c.stream, c.boxes, list, ca, (const double*)c.sub_rec, c.ctrl);
    }
    return hipGetLastError();
}

template <typename R, int W>
static void launch_collide_headed_w(const LaunchCtx& c, const void* A, void* B, uint32_t n_tiles, uint32_t s_off,
                                    const int32_t* list, int n_list, int max_n, const void* Aprev, int single_box)
{
    const uint32_t head_x = (uint32_t)((max_n * NEAR + 255) / 256);
    const uint32_t n_head = head_blocks(n_list, max_n);
    hipLaunchKernelGGL((k_collide_headed<R, W>), dim3(n_head + n_tiles), dim3(256), 0, c.stream, c.boxes,
                       (const CollideConst<R>*)c.ccs, c.tile_box, (R*)A, (R*)B, c.ctrl, s_off,
                       (const uint32_t*)c.defer, n_head, head_x, list, chain_args(c), (R*)c.near_u, c.near_c,
                       c.bead_box, c.claim, (const R*)Aprev, n_list == 1 && single_box >= 0 ? single_box : -1,
                       n_list == 1 && single_box >= 0 ? c.boxes_host[single_box] : BoxDev{});
}

template <typename R>
hipError_t launch_collide_headed(const LaunchCtx& c, const void* A, void* B, uint32_t n_tiles, uint32_t s_off,
                                 const int32_t* list, int n_list, int max_n, const void* Aprev, int single_box)
{
    static_assert(NEAR == NEAR_ITEMS, "one table size");
    if (n_list == 0 || n_tiles == 0 || !Aprev || !c.defer_on || c.dense_max_tiles) return hipErrorInvalidValue;
    if (max_n > WG_MAXB || max_n <= 0) return hipErrorInvalidValue;
    // the node-table code caps the occupancy at 5 waves per SIMD, so the
    // launch shape keeps only the autotuned cap of 4
    if (c.collide_variant == 0)
        launch_collide_headed_w<R, 4>(c, A, B, n_tiles, s_off, list, n_list, max_n, Aprev, single_box);
    else
        launch_collide_headed_w<R, 5>(c, A, B, n_tiles, s_off, list, n_list, max_n, Aprev, single_box);
    return hipGetLastError();
}

template <typename R>
hipError_t launch_export(const LaunchCtx& c, int box, const void* A, double* n, int q0, int nq)
{
    const uint32_t tiles = c.boxes_host[box].n_tiles;
    hipLaunchKernelGGL(k_export<R>, dim3(tiles), dim3(256), 0, c.stream, c.boxes, box, (const R*)A, n, q0, nq);
    return hipGetLastError();
}
template <typename R>
hipError_t launch_import(const LaunchCtx& c, int box, const double* n, void* A, int q0, int nq)
{
    const uint32_t tiles = c.boxes_host[box].n_tiles;
    hipLaunchKernelGGL(k_import<R>, dim3(tiles), dim3(256), 0, c.stream, c.boxes, box, n, (R*)A, q0, nq);
    return hipGetLastError();
}
template <typename R>
hipError_t launch_clear_tails(const LaunchCtx& c, void* A)
{
    hipLaunchKernelGGL(k_clear_tails<R>, dim3(c.n_boxes), dim3(256), 0, c.stream, c.boxes, (R*)A);
    return hipGetLastError();
}
template hipError_t launch_export<float>(const LaunchCtx&, int, const void*, double*, int, int);
template hipError_t launch_export<double>(const LaunchCtx&, int, const void*, double*, int, int);
template hipError_t launch_import<float>(const LaunchCtx&, int, const double*, void*, int, int);
template hipError_t launch_import<double>(const LaunchCtx&, int, const double*, void*, int, int);
template hipError_t launch_clear_tails<float>(const LaunchCtx&, void*);
template hipError_t launch_clear_tails<double>(const LaunchCtx&, void*);

hipError_t launch_init_forces(const LaunchCtx& c, const int32_t* list, int n_list, int block)
{
    if (n_list == 0) return hipSuccess;
    hipLaunchKernelGGL(k_init_forces, dim3(n_list), dim3(block), 0, c.stream, c.boxes, list, c.x, c.f, c.ctrl);
    return hipGetLastError();
}

hipError_t launch_advance(const LaunchCtx& c, uint32_t n)
{
    hipLaunchKernelGGL(k_advance, dim3(1), dim3(64), 0, c.stream, c.ctrl, n);
    return hipGetLastError();
}

hipError_t launch_probe_wait(hipStream_t stream, uint32_t* probe)
{
    hipLaunchKernelGGL(k_probe_wait, dim3(1), dim3(1), 0, stream, probe);
    return hipGetLastError();
}

hipError_t launch_probe_set(hipStream_t stream, uint32_t* probe, uint32_t value)
{
    hipLaunchKernelGGL(k_probe_set, dim3(1), dim3(1), 0, stream, probe, value);
    return hipGetLastError();
}

template <typename R>
hipError_t launch_observables(const LaunchCtx& c, const void* A, uint32_t max_recs, double* part, double* out)
{
    // every box's population array under 4 GiB: 32-bit offsets
    bool o32 = true;
    for (int b = 0; b < c.n_boxes; ++b)
        o32 = o32 && pop_elems_of((uint64_t)c.boxes_host[b].L * c.boxes_host[b].L * c.boxes_host[b].L) * sizeof(R) <
                         ((uint64_t)1 << 32);
    if (o32)
        hipLaunchKernelGGL((k_stats<R, true>), dim3(max_recs, c.n_boxes), dim3(STAT_BLOCK), 0, c.stream, c.boxes,
                           (const R*)A, part);
    else
        hipLaunchKernelGGL((k_stats<R, false>), dim3(max_recs, c.n_boxes), dim3(STAT_BLOCK), 0, c.stream, c.boxes,
                           (const R*)A, part);
    if (max_recs > STAT_DIRECT)
        hipLaunchKernelGGL(k_stats_mid, dim3(STAT_CHUNKS, c.n_boxes), dim3(256), 0, c.stream, c.boxes, part);
    hipLaunchKernelGGL(k_obs, dim3(c.n_boxes), dim3(256), 0, c.stream, c.boxes, chain_args(c), (const double*)part,
                       (const Ctrl*)c.ctrl, out);
    return hipGetLastError();
}


// =================================================================== adjoint
// Reverse sweep of one LB step for the gradient of a loss of the bead
// velocities with respect to (omega_shear, omega_bulk, zeta).  The forward
// state of the step (pre-collision populations in the stored pull layout, the
// node impulses, the substep tape of the chain) comes from replaying the
// window segment; noise words are regenerated from Philox.  Adjoints are FP64.
//   lam_n[i * nodes + node]   adjoint of the pre-collision population n_i
//   lam_dp[c * nodes + node]  adjoint of the lattice impulse handed to a node

// VJP of one node's collision: given lam_o = dJ/d(post-collision d*), return
// lam_d = dJ/d(pre-collision d), lam_f = dJ/d(impulse), and the contributions
// to dJ/d(omega_s), dJ/d(omega_b).
__device__ __forceinline__ void collide_vjp(const double d[19], const double f[3], const CollideConst<double>& cc,
                                            uint32_t node, uint32_t step, uint32_t k0, uint32_t k1,
                                            const double lam_o[19], double lam_d[19], double lam_f[3],
                                            double& g_ws, double& g_wb)
{
    double m[19];
    to_modes<double>(d, m);
    const double rho = cc.rho0 + m[0], irho = 1.0 / rho;
    const double u[3] = {(m[1] + 0.5 * f[0]) * irho, (m[2] + 0.5 * f[1]) * irho, (m[3] + 0.5 * f[2]) * irho};
    const double e[10] = {0, 0, 0, 0, rho * (u[0] * u[0] + u[1] * u[1] + u[2] * u[2]),
                          rho * (2 * u[0] * u[0] - u[1] * u[1] - u[2] * u[2]), rho * (u[1] * u[1] - u[2] * u[2]),
                          rho * u[0] * u[1], rho * u[1] * u[2], rho * u[0] * u[2]};
    const double uf[3] = {u[0] * f[0], u[1] * f[1], u[2] * f[2]};
    const double sv[10] = {0, 0, 0, 0, 2 * (uf[0] + uf[1] + uf[2]), 2 * (2 * uf[0] - uf[1] - uf[2]), 2 * (uf[1] - uf[2]),
                           u[0] * f[1] + u[1] * f[0], u[1] * f[2] + u[2] * f[1], u[0] * f[2] + u[2] * f[0]};
    double r[19];
#pragma unroll
    for (int k = 0; k < 19; ++k) r[k] = 0.0;
    const double a = cc.therm > 0 ? sqrt(cc.mu * rho) : 0.0;
    if (cc.therm > 0) {
        const U4 w0 = philox10(U4{node, step, 0u, 0u}, k0, k1), w1 = philox10(U4{node, step, 0u, 1u}, k0, k1);
        r[4] = unit_noise<double>(w0.x); r[5] = unit_noise<double>(w0.y); r[6] = unit_noise<double>(w0.z);
        r[7] = unit_noise<double>(w0.w); r[8] = unit_noise<double>(w1.x); r[9] = unit_noise<double>(w1.y);
        if (cc.therm > 1) {
            const U4 w2 = philox10(U4{node, step, 0u, 2u}, k0, k1), w3 = philox10(U4{node, step, 0u, 3u}, k0, k1);
            r[10] = unit_noise<double>(w1.z); r[11] = unit_noise<double>(w1.w);
            r[12] = unit_noise<double>(w2.x); r[13] = unit_noise<double>(w2.y); r[14] = unit_noise<double>(w2.z);
            r[15] = unit_noise<double>(w2.w); r[16] = unit_noise<double>(w3.x); r[17] = unit_noise<double>(w3.y);
            r[18] = unit_noise<double>(w3.z);
        }
    }
    // d* = w_i sum_k e_ki M_k  ->  lam_M = E (w o lam_o)
    double wl[19], lM[19];
#pragma unroll
    for (int i = 0; i < 19; ++i) wl[i] = wv(i) * lam_o[i];
    to_modes<double>(wl, lM);
    double lm[19];
#pragma unroll
    for (int k = 0; k < 19; ++k) lm[k] = 0.0;
    double lu[3] = {0, 0, 0}, lrho = 0.0, la = 0.0, lgs = 0.0, lgb = 0.0;
    lam_f[0] = lam_f[1] = lam_f[2] = 0.0;
    lm[0] += lM[0];
#pragma unroll
    for (int c = 0; c < 3; ++c) { lm[1 + c] += 3.0 * lM[1 + c]; lam_f[c] += 3.0 * lM[1 + c]; }
    double le[10], ls[10];
#pragma unroll
    for (int k = 4; k <= 9; ++k) {
        const double gam = k == 4 ? cc.gb : cc.gs, h = k == 4 ? cc.hb : cc.hs;
        const double lP = lM[k] * inv_b<double>(k);
        lm[k] += gam * lP;
        le[k] = (1.0 - gam) * lP;
        ls[k] = h * lP;
        double lg = (m[k] - e[k]) * lP + 0.5 * sv[k] * lP;
        if (cc.therm > 0 && cc.q[k] > 0.0) lg += a * r[k] * (-gam * inv_b<double>(k) / cc.q[k]) * lM[k];
        la += cc.q[k] * r[k] * lM[k];
        if (k == 4) lgb += lg; else lgs += lg;
    }
#pragma unroll
    for (int k = 10; k < 19; ++k) {
        lm[k] += cc.gg * inv_b<double>(k) * lM[k];
        la += cc.q[k] * r[k] * lM[k];
    }
    // equilibrium stress modes e_k(rho, u)
    lrho += (le[4] * e[4] + le[5] * e[5] + le[6] * e[6] + le[7] * e[7] + le[8] * e[8] + le[9] * e[9]) * irho;
    lu[0] += rho * (2 * u[0] * le[4] + 4 * u[0] * le[5] + u[1] * le[7] + u[2] * le[9]);
    lu[1] += rho * (2 * u[1] * le[4] - 2 * u[1] * le[5] + 2 * u[1] * le[6] + u[0] * le[7] + u[2] * le[8]);
    lu[2] += rho * (2 * u[2] * le[4] - 2 * u[2] * le[5] - 2 * u[2] * le[6] + u[1] * le[8] + u[0] * le[9]);
    // source terms s_k(u, f)
    lu[0] += 2 * f[0] * ls[4] + 4 * f[0] * ls[5] + f[1] * ls[7] + f[2] * ls[9];
    lu[1] += 2 * f[1] * ls[4] - 2 * f[1] * ls[5] + 2 * f[1] * ls[6] + f[0] * ls[7] + f[2] * ls[8];
    lu[2] += 2 * f[2] * ls[4] - 2 * f[2] * ls[5] - 2 * f[2] * ls[6] + f[1] * ls[8] + f[0] * ls[9];
    lam_f[0] += 2 * u[0] * ls[4] + 4 * u[0] * ls[5] + u[1] * ls[7] + u[2] * ls[9];
    lam_f[1] += 2 * u[1] * ls[4] - 2 * u[1] * ls[5] + 2 * u[1] * ls[6] + u[0] * ls[7] + u[2] * ls[8];
    lam_f[2] += 2 * u[2] * ls[4] - 2 * u[2] * ls[5] - 2 * u[2] * ls[6] + u[1] * ls[8] + u[0] * ls[9];
    // a = sqrt(mu rho)
    if (a > 0.0) lrho += la * a * 0.5 * irho;
    // u = (j + f/2) / rho
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        lm[1 + c] += lu[c] * irho;
        lam_f[c] += 0.5 * lu[c] * irho;
    }
    lrho -= (u[0] * lu[0] + u[1] * lu[1] + u[2] * lu[2]) * irho;
    lm[0] += lrho;
    // m = E d  ->  lam_d = E^T lam_m
    from_scaled_modes<double>(lm, lam_d);
#pragma unroll
    for (int i = 0; i < 19; ++i) lam_d[i] /= wv(i);
    // gamma = 1 - omega
    g_ws = -lgs;
    g_wb = -lgb;
}

// One thread per node: lam_d*(r) is gathered from lam_n_next at the nodes the
// populations stream to (r + c_i); the forward state is the replayed
// pre-collision state.  Writes lam_n_cur and lam_dp; adds the tile's rate
// gradient to gpart[tile][2].
template <typename R>
__global__ __launch_bounds__(256) void k_adj_collide(const BoxDev* __restrict__ boxes,
                                                     const CollideConst<double>* __restrict__ ccd,
                                                     const uint32_t* __restrict__ tile_box,
                                                     const R* __restrict__ P, const unsigned long long* __restrict__ imp,
                                                     const double* __restrict__ lam_next, double* __restrict__ lam_cur,
                                                     double* __restrict__ lam_dp, double* __restrict__ gpart,
                                                     uint64_t nodes, uint32_t step)
{
    __shared__ double red[4][2];
    const uint32_t tile = blockIdx.x;
    const int bi = (int)tile_box[tile];
    const BoxDev& bx = boxes[bi];
    const int L = bx.L;
    const uint32_t V = (uint32_t)L * L * L;
    const uint32_t r = (tile - bx.tile_begin) * 256u + threadIdx.x;
    double gws = 0.0, gwb = 0.0;
    if (r < V) {
        const Upwind up = upwind_of(r, L, bx.inv_L);
        R dr[19];
        gather_pre<R, false>(P + bx.pop_off, up, dr);
        double d[19], f[3] = {0, 0, 0};
#pragma unroll
        for (int i = 0; i < 19; ++i) d[i] = (double)dr[i];
        const uint64_t gn = bx.node_off + r;
        if (bx.N > 0)
#pragma unroll
            for (int c = 0; c < 3; ++c) f[c] = (double)(long long)imp[3 * gn + c] * IMP_INV_SCALE;
        // the population leaving r along c_i arrives at r + c_i
        uint32_t x, y;
        const uint32_t q = div_L(r, L, bx.inv_L, &x);
        const uint32_t z = div_L(q, L, bx.inv_L, &y);
        const uint32_t Xd[3] = {x == 0 ? L - 1 : x - 1, x, x + 1 == (uint32_t)L ? 0 : x + 1};
        const uint32_t Yd[3] = {y == 0 ? L - 1 : y - 1, y, y + 1 == (uint32_t)L ? 0 : y + 1};
        const uint32_t Zd[3] = {z == 0 ? L - 1 : z - 1, z, z + 1 == (uint32_t)L ? 0 : z + 1};
        double lo[19];
#pragma unroll
        for (int i = 0; i < 19; ++i) {
            const uint32_t dn = Xd[cxv(i) + 1] + (uint32_t)L * (Yd[cyv(i) + 1] + (uint32_t)L * Zd[czv(i) + 1]);
            lo[i] = lam_next[i * nodes + bx.node_off + dn];
        }
        double ld[19], lf[3];
        collide_vjp(d, f, ccd[bi], r, step, bx.seed, bx.box_id, lo, ld, lf, gws, gwb);
#pragma unroll
        for (int i = 0; i < 19; ++i) lam_cur[i * nodes + gn] = ld[i];
#pragma unroll
        for (int c = 0; c < 3; ++c) lam_dp[c * nodes + gn] = lf[c];
    }
    // the tile's sums: nothing waits for the old value
    double g2[2] = {gws, gwb};
    const double gs = block_sum256<2>(g2, red);
    if (threadIdx.x < 2) atomicAdd(&gpart[2 * (uint64_t)tile + threadIdx.x], gs);
}

// add dJ/dv(end of step) and reverse the chain's substeps of one LB step; one
// workgroup per chain (at most 256 beads), thread per bead.
struct AdjChainArgs {
    const double* x0; const double* v0; const double* f0;   // bead state at the step start (replayed)
    const double* tape;                                     // [substep][total beads][TAPE_REC]
    const double* dj;                                       // dJ/dv at the step end [total beads][3]
    double* lx; double* lv; double* lf;                     // bead adjoints, in: step end, out: step start
    double* lam_n;                                          // pre-collision population adjoint (accumulated)
    const double* lam_dp;
    double* gz;                                             // per box dJ/dzeta
    uint64_t nodes, total_beads;
};

__device__ __forceinline__ void pair_kernel(const double d[3], double g, double gp, const double v[3], double out[3])
{
    // (g I + 2 g' d d^T) v
    const double dv = 2.0 * gp * (d[0] * v[0] + d[1] * v[1] + d[2] * v[2]);
    out[0] += g * v[0] + dv * d[0];
    out[1] += g * v[1] + dv * d[1];
    out[2] += g * v[2] + dv * d[2];
}

// sum of v over the T lanes of a bead (all active), the same bits in each
template <int T>
__device__ __forceinline__ double bead_sum(double v)
{
    v += dpp_from<0xB1>(v);                 // quad_perm [1,0,3,2]
    v += dpp_from<0x4E>(v);                 // quad_perm [2,3,0,1]
    if (T >= 8) v += dpp_from<0x141>(v);    // row_half_mirror
    if (T >= 16) v += dpp_from<0x140>(v);   // row_mirror
    return v;
}

// Reverse sweep of one LB step's substeps for chains of at most 256 beads, T
// lanes per bead as in the forward kernel (a function of N only).  Bound, like
// it, by the serial chain of a substep; the lanes of a bead share its work:
// each holds 8 / T corners of the stencil (velocities, densities, impulse and
// velocity adjoints) and hands their adjoints over itself, takes every T-th
// partner of the force Hessian from a list (bits of one word, as in the
// forward kernel) and, lanes 0 and 1, one bond each; the noise words of T
// substeps are drawn at once.  Sums over the lanes are DPP butterflies, so
// every lane carries the same bead adjoint.  Positions and force adjoints
// alternate between two LDS buffers: one barrier per substep.  32 beads, ten
// substeps: 26.5 us, where lanes that each held all eight corners, with
// lane 0 handing over and every partner tested, took 43 us.
template <int MB>
struct AdjLds {
    double xs[2][3 * MB], lF[2][3 * MB];
    int moved[3];
    double red[16];
};
template <typename R, int T, int MB>
__device__ __forceinline__ double adj_substeps(const BoxDev& bx, const R* __restrict__ P, const AdjChainArgs& aa,
                                               uint32_t step, AdjLds<MB>& sh)
{
    constexpr int T8 = T < 8 ? T : 8, NC = 8 / T8;
    constexpr int NB = MB <= 128 ? NC : 1;   // corners whose loads are in flight together
    const int N = bx.N, S = bx.substeps, L = bx.L;
    const int b = (int)threadIdx.x / T, lane = (int)threadIdx.x % T;
    const bool act = b < N;
    const uint64_t g = bx.bead_off + (uint64_t)(act ? b : 0);
    const ChainSpan sp = chain_span(bx, act ? b : 0);
    const double dt = bx.dt, h = 0.5 * dt / bx.mass, tau = bx.tau_lb, Ld = (double)L, iL = bx.inv_L;
    const double eps24 = 24.0 * bx.eps, s6c = bx.sigsq * bx.sigsq * bx.sigsq, s12c = s6c * s6c;
    const int kc = lane & (T8 - 1);
    const double half = T == 16 && lane >= 8 ? 0.0 : 1.0;   // T = 16: the upper lanes repeat the corners
    const bool bonded = act && ((lane == 0 && b > sp.lo) || (lane == 1 && b < sp.hi));
    const int jb = lane == 0 ? b - 1 : b + 1;
    if (threadIdx.x < 3) sh.moved[threadIdx.x] = 0;
    double lx[3] = {0, 0, 0}, lv[3] = {0, 0, 0}, lf[3] = {0, 0, 0}, x0[3] = {0, 0, 0};
    if (act)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            lx[c] = aa.lx[3 * g + c]; lv[c] = aa.lv[3 * g + c] + aa.dj[3 * g + c]; lf[c] = aa.lf[3 * g + c];
        }
    double gz = 0.0;
    int cb[3] = {-1, -1, -1};
    double lcu[NC][3];         // accumulated adjoint of the stencil's node velocities
    double rho_k[NC], cuk[NC][3];
    double la[NC][3];          // tau * lam_dp at the stencil's nodes
    uint32_t cnode[NC];
    unsigned long long nl = 0ull;   // partners lane + T m within the list radius
    U4 pw{0, 0, 0, 0};
    const R* pb = P + bx.pop_off;
    auto flush = [&]() __attribute__((always_inline)) {   // node velocity adjoint -> population adjoint at the stencil nodes
        if (lane >= T8) return;
#pragma unroll
        for (int kk = 0; kk < NC; ++kk) {
            const double ir = 1.0 / (rho_k[kk] * tau);
            const double lsum = lcu[kk][0] * (cuk[kk][0] * tau) + lcu[kk][1] * (cuk[kk][1] * tau) + lcu[kk][2] * (cuk[kk][2] * tau);
            double* dst = aa.lam_n + bx.node_off + cnode[kk];
#pragma unroll
            for (int i = 0; i < 19; ++i) {
                const double cc = (double)cxv(i) * lcu[kk][0] + (double)cyv(i) * lcu[kk][1] + (double)czv(i) * lcu[kk][2];
                atomicAdd(dst + i * aa.nodes, (cc - lsum) * ir);
            }
        }
    };
    // tape record of substep s, loaded one substep ahead where the registers
    // allow it
    constexpr bool AHEAD = MB <= 128;
    double nx1[3] = {0, 0, 0}, nv1[3] = {0, 0, 0}, nfc[3] = {0, 0, 0}, nfr[3] = {0, 0, 0}, ni0[3] = {0, 0, 0};
    auto load_rec = [&](int s) __attribute__((always_inline)) {
        const double* tq = aa.tape + ((uint64_t)s * aa.total_beads + g) * TAPE_REC;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            nx1[c] = tq[c]; nv1[c] = tq[3 + c]; nfc[c] = tq[6 + c]; ni0[c] = tq[9 + c]; nfr[c] = tq[12 + c];
        }
    };
    if (AHEAD && act) load_rec(S - 1);
    for (int s = S - 1, it = 0; s >= 0; --s, ++it) {
        if (!AHEAD && act) load_rec(s);
        double* xs = sh.xs[s & 1];
        double* lF = sh.lF[s & 1];
        double x1[3], v1[3], fc[3], fr[3], rn[3] = {0, 0, 0};
        int i0[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) { x1[c] = nx1[c]; v1[c] = nv1[c]; fc[c] = nfc[c]; i0[c] = (int)ni0[c]; fr[c] = nfr[c]; }
        // v' = v1 + f' h and f' = F_c + fc
        double lft[3], lv1[3], lfc[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) { lft[c] = lf[c] + h * lv[c]; lv1[c] = lv[c]; lfc[c] = lft[c]; }
        if (act) {
            if (lane == 0) {
                bool far = false;
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    xs[3 * b + c] = x1[c];
                    lF[3 * b + c] = lft[c];
                    far |= fabs(x1[c] - x0[c]) > 0.5 * NL_SKIN * 0.577;
                }
                if (it > 0 && far) sh.moved[it % 3] = 1;
            }
            if (AHEAD && s > 0) load_rec(s - 1);
            if (it == 0 || s % T == T - 1)
                pw = philox10(U4{(uint32_t)b, step, (1u << 16) | (uint32_t)(s - s % T + lane), 0u}, bx.seed, bx.box_id);
            rn[0] = unit_noise<double>(__shfl(pw.x, s % T, T));
            rn[1] = unit_noise<double>(__shfl(pw.y, s % T, T));
            rn[2] = unit_noise<double>(__shfl(pw.z, s % T, T));
        }
        __syncthreads();
        const bool rebuild = it == 0 || sh.moved[it % 3] != 0;
        if (threadIdx.x == 0) sh.moved[(it + 2) % 3] = 0;
        double lx1[3] = {lx[0], lx[1], lx[2]};
        if (act) {
            // stencil of this substep
            if (i0[0] != cb[0] || i0[1] != cb[1] || i0[2] != cb[2]) {
                if (it > 0) flush();
                const double* tp = aa.tape + ((uint64_t)s * aa.total_beads + g) * TAPE_REC + 15;
#pragma unroll
                for (int k0 = 0; k0 < NC; k0 += NB) {
                    R d[NB][19];
#pragma unroll
                    for (int kk = k0; kk < k0 + NB; ++kk) {
                        const int k = kc + kk * T8;
                        const int ix = i0[0] + (k & 1), iy = i0[1] + ((k >> 1) & 1), iz = i0[2] + (k >> 2);
                        const uint32_t nx = ix >= L ? ix - L : ix, ny = iy >= L ? iy - L : iy, nz = iz >= L ? iz - L : iz;
                        cnode[kk] = nx + (uint32_t)L * (ny + (uint32_t)L * nz);
                        gather_pre<R, false>(pb, Upwind(nx, ny, nz, (uint32_t)L), d[kk - k0]);
#pragma unroll
                        for (int c = 0; c < 3; ++c) {
                            cuk[kk][c] = tp[3 * k + c];
                            lcu[kk][c] = 0.0;
                            la[kk][c] = tau * aa.lam_dp[c * aa.nodes + bx.node_off + cnode[kk]];
                        }
                    }
#pragma unroll
                    for (int kk = k0; kk < k0 + NB; ++kk) {
                        double rho = 0.0;
#pragma unroll
                        for (int i = 0; i < 19; ++i) rho += (double)d[kk - k0][i];
                        rho_k[kk] = rho + bx.rho0;
                    }
                }
                cb[0] = i0[0]; cb[1] = i0[1]; cb[2] = i0[2];
            }
            double wt[NC], gx[NC], gy[NC], gw3[NC], ub[3] = {0, 0, 0}, sl[3] = {0, 0, 0};
#pragma unroll
            for (int kk = 0; kk < NC; ++kk) {
                const int k = kc + kk * T8;
                gx[kk] = (k & 1) ? fr[0] : 1.0 - fr[0];
                gy[kk] = ((k >> 1) & 1) ? fr[1] : 1.0 - fr[1];
                gw3[kk] = (k >> 2) ? fr[2] : 1.0 - fr[2];
                wt[kk] = gx[kk] * gy[kk] * gw3[kk];
#pragma unroll
                for (int c = 0; c < 3; ++c) { ub[c] += wt[kk] * cuk[kk][c]; sl[c] += wt[kk] * la[kk][c]; }
            }
#pragma unroll
            for (int c = 0; c < 3; ++c) { ub[c] = bead_sum<T8>(ub[c]); sl[c] = bead_sum<T8>(sl[c]); }
            // impulse spread: acc_k -= w_k fc dt, handed over as tau * acc;
            // fc = -zeta (v1 - u_b) + A(zeta) r
            double lub[3], part[3] = {0, 0, 0};
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                lfc[c] -= dt * sl[c];
                if (bx.zeta > 0.0) gz += 0.5 * bx.bead_noise / bx.zeta * rn[c] * lfc[c];
                gz -= (v1[c] - ub[c]) * lfc[c];
                lub[c] = bx.zeta * lfc[c];
                lv1[c] -= lub[c];
            }
            // u_b = sum_k w_k cu_k, and the trilinear weights w_k(fractions of x1)
#pragma unroll
            for (int kk = 0; kk < NC; ++kk) {
                const int k = kc + kk * T8;
                double lw = -dt * (fc[0] * la[kk][0] + fc[1] * la[kk][1] + fc[2] * la[kk][2]);
                lw += cuk[kk][0] * lub[0] + cuk[kk][1] * lub[1] + cuk[kk][2] * lub[2];
                lw *= half;
#pragma unroll
                for (int c = 0; c < 3; ++c) lcu[kk][c] += wt[kk] * lub[c];
                part[0] += lw * ((k & 1) ? 1.0 : -1.0) * gy[kk] * gw3[kk];
                part[1] += lw * (((k >> 1) & 1) ? 1.0 : -1.0) * gx[kk] * gw3[kk];
                part[2] += lw * ((k >> 2) ? 1.0 : -1.0) * gx[kk] * gy[kk];
            }
            // conservative forces at x1: lam_x1_b += sum_j K_bj (lam_F_b - lam_F_j).
            // This lane's bond (FENE) ...
            {
                const int j = bonded ? jb : b;
                const double dl[3] = {lft[0] - lF[3 * j], lft[1] - lF[3 * j + 1], lft[2] - lF[3 * j + 2]};
                const double d[3] = {x1[0] - xs[3 * j], x1[1] - xs[3 * j + 1], x1[2] - xs[3 * j + 2]};
                const double r2 = d[0] * d[0] + d[1] * d[1] + d[2] * d[2];
                const double iden = 1.0 / (1.0 - r2 * bx.inv_r0sq);
                const double gfe = -bx.k_fene * iden;
                pair_kernel(d, gfe, gfe * bx.inv_r0sq * iden, dl, part);   // a zero separation adds nothing
            }
            // ... and its share of the repulsive LJ partners
            if (rebuild) {
                const double rl = sqrt(bx.rc2) + NL_SKIN + 1e-6, rl2 = rl * rl;
#pragma unroll
                for (int c = 0; c < 3; ++c) x0[c] = x1[c];
                nl = 0ull;
#pragma unroll 2
                for (int j = lane, m = 0; j < N; j += T, ++m) {
                    double d0 = x1[0] - xs[3 * j], d1 = x1[1] - xs[3 * j + 1], d2 = x1[2] - xs[3 * j + 2];
                    d0 -= Ld * rint(d0 * iL); d1 -= Ld * rint(d1 * iL); d2 -= Ld * rint(d2 * iL);
                    if (j != b && d0 * d0 + d1 * d1 + d2 * d2 < rl2) nl |= 1ull << m;
                }
            }
            for (unsigned long long m = nl; m; m &= m - 1ull) {
                const int j = lane + T * (__ffsll((long long)m) - 1);
                double d[3], dl[3];
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    dl[c] = lft[c] - lF[3 * j + c];
                    d[c] = x1[c] - xs[3 * j + c];
                    d[c] -= Ld * rint(d[c] * iL);
                }
                const double q = d[0] * d[0] + d[1] * d[1] + d[2] * d[2];
                if (q < bx.rc2) {
                    const double iq = 1.0 / q, iq4 = iq * iq * iq * iq, iq7 = iq4 * iq * iq * iq;
                    pair_kernel(d, eps24 * (2.0 * s12c * iq7 - s6c * iq4),
                                eps24 * (-14.0 * s12c * iq7 * iq + 4.0 * s6c * iq4 * iq), dl, part);
                }
            }
#pragma unroll
            for (int c = 0; c < 3; ++c) lx1[c] += bead_sum<T>(part[c]);
        }
        // x1 = x + v1 dt,  v1 = v + f h
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            lv1[c] += dt * lx1[c];
            lx[c] = lx1[c];
            lv[c] = lv1[c];
            lf[c] = h * lv1[c];
        }
    }
    if (act) {
        flush();
        if (lane == 0) {
#pragma unroll
            for (int c = 0; c < 3; ++c) { aa.lx[3 * g + c] = lx[c]; aa.lv[3 * g + c] = lv[c]; aa.lf[3 * g + c] = lf[c]; }
        }
    }
    return act && lane == 0 ? gz : 0.0;   // one copy per bead
}

template <typename R, int MAXT>
__global__ __launch_bounds__(MAXT) void k_adj_couple(const BoxDev* __restrict__ boxes,
                                                     const int32_t* __restrict__ couple_list, const R* __restrict__ P,
                                                     AdjChainArgs aa, uint32_t step)
{
    __shared__ AdjLds<MAXT / 4> sh;
    const int bi = couple_list[blockIdx.x];
    const BoxDev bx = boxes[bi];   // a copy: its fields stay in registers across the substeps
    double gz;
    if (bx.couple_T == 4) gz = adj_substeps<R, 4>(bx, P, aa, step, sh);
    else if (bx.couple_T == 8) gz = adj_substeps<R, 8>(bx, P, aa, step, sh);
    else gz = adj_substeps<R, 16>(bx, P, aa, step, sh);
    // dJ/dzeta of the box: over each wavefront, then the wavefronts in order
    for (int o = 1; o < 64; o <<= 1) gz += __shfl_xor(gz, o, 64);
    if ((threadIdx.x & 63u) == 0u) sh.red[threadIdx.x / 64u] = gz;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (uint32_t w = 0; w < blockDim.x / 64u; ++w) t += sh.red[w];
        aa.gz[bi] += t;
    }
}

template <typename R>
hipError_t launch_adj_collide(const LaunchCtx& c, const void* ccd, const void* P, const unsigned long long* imp,
                              const double* lam_next, double* lam_cur, double* lam_dp, double* gpart,
                              uint64_t nodes, uint32_t total_tiles, uint32_t step)
{
    hipLaunchKernelGGL(k_adj_collide<R>, dim3(total_tiles), dim3(256), 0, c.stream, c.boxes,
                       (const CollideConst<double>*)ccd, c.tile_box, (const R*)P, imp, lam_next, lam_cur, lam_dp,
                       gpart, nodes, step);
    return hipGetLastError();
}

template <typename R>
hipError_t launch_adj_couple(const LaunchCtx& c, const int32_t* list, int n_list, int block, const void* P,
                             const AdjArgsHost& a, uint32_t step)
{
    if (n_list == 0) return hipSuccess;
    if (block < 64 || block > 1024) return hipErrorInvalidValue;
    AdjChainArgs aa{a.x0, a.v0, a.f0, a.tape, a.dj, a.lx, a.lv, a.lf, a.lam_n, a.lam_dp, a.gz, a.nodes,
                    c.total_beads};
    if (block > 512)
        hipLaunchKernelGGL((k_adj_couple<R, 1024>), dim3(n_list), dim3(block), 0, c.stream, c.boxes, list, (const R*)P,
                           aa, step);
    else if (block > 256)
        hipLaunchKernelGGL((k_adj_couple<R, 512>), dim3(n_list), dim3(block), 0, c.stream, c.boxes, list, (const R*)P,
                           aa, step);
    else
        hipLaunchKernelGGL((k_adj_couple<R, 256>), dim3(n_list), dim3(block), 0, c.stream, c.boxes, list, (const R*)P,
                           aa, step);
    return hipGetLastError();
}

template hipError_t launch_adj_collide<float>(const LaunchCtx&, const void*, const void*, const unsigned long long*,
                                              const double*, double*, double*, double*, uint64_t, uint32_t, uint32_t);
template hipError_t launch_adj_collide<double>(const LaunchCtx&, const void*, const void*, const unsigned long long*,
                                               const double*, double*, double*, double*, uint64_t, uint32_t, uint32_t);
template hipError_t launch_adj_couple<float>(const LaunchCtx&, const int32_t*, int, int, const void*,
                                             const AdjArgsHost&, uint32_t);
template hipError_t launch_adj_couple<double>(const LaunchCtx&, const int32_t*, int, int, const void*,
                                              const AdjArgsHost&, uint32_t);

template hipError_t launch_collide<float>(const LaunchCtx&, const void*, void*, int, uint32_t, uint32_t, uint32_t);
template hipError_t launch_collide<double>(const LaunchCtx&, const void*, void*, int, uint32_t, uint32_t, uint32_t);
template hipError_t launch_fixup<float>(const LaunchCtx&, const void*, void*, uint64_t, uint64_t, uint32_t);
template hipError_t launch_fixup<double>(const LaunchCtx&, const void*, void*, uint64_t, uint64_t, uint32_t);
template hipError_t launch_collide_deferred<float>(const LaunchCtx&, const void*, void*, uint32_t);
template hipError_t launch_collide_deferred<double>(const LaunchCtx&, const void*, void*, uint32_t);
template hipError_t launch_overflow<float>(const LaunchCtx&, const void*, void*, uint32_t, uint32_t);
template hipError_t launch_overflow<double>(const LaunchCtx&, const void*, void*, uint32_t, uint32_t);
template hipError_t launch_collide_forced<float>(const LaunchCtx&, const void*, void*, int, uint32_t, uint32_t,
                                                 uint32_t);
template hipError_t launch_collide_forced<double>(const LaunchCtx&, const void*, void*, int, uint32_t, uint32_t,
                                                  uint32_t);
template hipError_t launch_couple<float>(const LaunchCtx&, const void*, const int32_t*, int, int, uint32_t);
template hipError_t launch_couple<double>(const LaunchCtx&, const void*, const int32_t*, int, int, uint32_t);
template hipError_t launch_step<float>(const LaunchCtx&, const int32_t*, int, int, int, void*, void*, const void*,
                                       unsigned long long*, uint32_t, uint32_t);
template hipError_t launch_step<double>(const LaunchCtx&, const int32_t*, int, int, int, void*, void*, const void*,
                                        unsigned long long*, uint32_t, uint32_t);
template hipError_t launch_step_end<float>(const LaunchCtx&, const int32_t*, int, const void*, void*, uint32_t);
template hipError_t launch_step_end<double>(const LaunchCtx&, const int32_t*, int, const void*, void*, uint32_t);
template hipError_t launch_couple_big<float>(const LaunchCtx&, const void*, const int32_t*, int, int, uint32_t,
                                            hipEvent_t, const void*, int, uint32_t, int, int);
template hipError_t launch_couple_big<double>(const LaunchCtx&, const void*, const int32_t*, int, int, uint32_t,
                                             hipEvent_t, const void*, int, uint32_t, int, int);
template hipError_t launch_collide_headed<float>(const LaunchCtx&, const void*, void*, uint32_t, uint32_t,
                                                 const int32_t*, int, int, const void*, int);
template hipError_t launch_collide_headed<double>(const LaunchCtx&, const void*, void*, uint32_t, uint32_t,
                                                  const int32_t*, int, int, const void*, int);
template hipError_t launch_observables<float>(const LaunchCtx&, const void*, uint32_t, double*, double*);
template hipError_t launch_observables<double>(const LaunchCtx&, const void*, uint32_t, double*, double*);

}  // namespace lbd
