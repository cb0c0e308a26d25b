// Launch interface between the host runtime and the HIP kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "lbmd_device.hpp"

namespace lbd {

// One-kernel steps (k_step): per box, the nodes set aside for its chain's
// workgroup (count by step parity), and the impulses outside them.
struct alignas(128) StepRec {
    uint32_t n[2];       // set-aside nodes of the steps of either parity
    uint32_t pend[2];    // by parity: the step's deferral stamp if it listed impulses outside them
    uint32_t fixed[2];   // by parity: stamp of the step whose start re-collided the previous step's
    uint32_t n_ovf;      // impulses the last step listed
    uint32_t t;          // the last step
};
struct StepArgs {
    unsigned long long* mask[2];   // by step parity: one bit per node, a word per DSEG nodes
    uint32_t* list[2];             // by step parity: the set-aside nodes, NODES_PER_BEAD slots per bead
    StepRec* rec;
};
constexpr int NODES_PER_BEAD = 27;   // a bead's stencil, at most one node wider on one side per axis

// Device pointers and sizes every launcher needs; filled by the runtime.
struct LaunchCtx {
    hipStream_t stream;
    int n_cu;                      // compute units of the device
    int collide_variant;           // launch shape of the collide kernel (0..N_COLLIDE_VARIANTS-1)
    const BoxDev* boxes;
    const BoxDev* boxes_host;      // host copy of the box table
    int n_boxes;
    const void* ccs;               // CollideConst<R>[n_boxes]
    const uint32_t* tile_box;      // box index of every collide tile
    Ctrl* ctrl;
    unsigned long long* imp;       // dense node impulses, 3 per global node, fixed point 2^-52
    uint32_t* claim;               // per global node: step stamp of the last fix-up
    uint32_t* touched;             // per bead: touch_cap slots of local node ids
    int32_t* touched_cnt;          // per bead
    int touch_cap;                 // touched slots per bead
    uint32_t* nl_rebuilds;         // per box: neighbour-list builds (diagnostic)
    const int32_t* bead_box;       // box index of every bead
    double *x, *v, *f, *fc;        // beads [total][3]
    int32_t* nl_cnt; uint16_t* nl_idx; double* nl_x0; int nl_cap;
    double* vhist; int hist_len; uint64_t total_beads;
    double* tape;                  // substep tape while replaying an adjoint window segment (else null)
    double* tape_x0;               // with tape: the step's starting bead x; v and f follow at tape_vo, tape_fo
    uint64_t tape_vo, tape_fo;     // (in doubles), the state's own layout
    int keep_imp;                  // 1: the fix-up leaves the node impulses in place (adjoint replay records them)
    // chains above BIG_CHAIN beads
    void* near_u;                  // [total beads][27][3] node velocities around each bead (storage precision)
    int4* near_c;                  // [total beads] nearest node the table is centred on
    double* sub_rec;               // [most substeps][total beads][8] per-substep records
    void* field;                   // dense boxes: node velocities (MD units, storage precision) [nodes][3]
    uint32_t dense_max_tiles;      // collide tiles of the largest dense box (0: none)
    int big_sparse;                // boxes on the 1024-thread path that are not dense (k_spread's boxes)
    // deferred segments: in a batched step the 64-node segments (wavefronts
    // of the collide tiles) that hold a node of any table of a sparse box's
    // large chain are left out of the plain collide and collided with their
    // impulses beside it, once the coupling is done; impulses that land
    // outside them are listed for a fix-up
    int defer_on;                  // this launch defers (the pointers below are always set)
    uint32_t* defer;               // per segment and step parity: stamp of the last step that deferred it
    uint32_t* dclaim;              // per segment: stamp of the last step that listed it
    uint32_t* defer_list;          // the deferred segments, Ctrl::defer_cnt of them
    uint32_t defer_cap;
    uint32_t* ovf;                 // (bead, local node) pairs, Ctrl::ovf_cnt of them
    uint32_t ovf_cap;
    uint32_t* ovm;                 // per global node: stamp of the last step that listed it in ovf
    unsigned long long* nmask[2];  // one-kernel steps (StepArgs)
    uint32_t* nlist[2];
    StepRec* step_rec;             // null: no such steps
};

template <typename R>
hipError_t launch_collide(const LaunchCtx& c, const void* A, void* B, int fixed_box, uint32_t tile0,
                          uint32_t n_tiles, uint32_t s_off);
template <typename R>
hipError_t launch_fixup(const LaunchCtx& c, const void* A, void* B, uint64_t bead0, uint64_t n_beads,
                        uint32_t s_off);
// the deferred tiles' collide (after the coupling, beside the plain
// collide) and the end-of-step pass: fix-up of the listed impulses outside
// them, then the deferral cleared
template <typename R>
hipError_t launch_collide_deferred(const LaunchCtx& c, const void* A, void* B, uint32_t s_off);
// advance: added to the device step counter once the fix-up is done (0: none)
template <typename R>
hipError_t launch_overflow(const LaunchCtx& c, const void* A, void* B, uint32_t s_off, uint32_t advance = 0);
template <typename R>
hipError_t launch_collide_forced(const LaunchCtx& c, const void* A, void* B, int fixed_box, uint32_t tile0,
                                 uint32_t n_tiles, uint32_t s_off);
template <typename R>
hipError_t launch_couple(const LaunchCtx& c, const void* A, const int32_t* list, int n_list, int block,
                         uint32_t s_off);
// one whole step of boxes whose chains (those in `list`) have at most
// BIG_CHAIN beads, from A into B; Aprev, imp_prev: the previous step's input
// and impulse field (unused by the first step after launch_step_begin).
// block: threads of the widest chain workgroup, max_n: beads of the longest
// chain.  A run of steps starts with
// launch_step_begin and ends with launch_step_end on the last step's buffers.
template <typename R>
hipError_t launch_step(const LaunchCtx& c, const int32_t* list, int n_list, int block, int max_n, void* A, void* B,
                       const void* Aprev, unsigned long long* imp_prev, uint32_t n_tiles, uint32_t s_off);
hipError_t launch_step_begin(const LaunchCtx& c, const int32_t* list, int n_list, uint32_t s_off);
template <typename R>
hipError_t launch_step_end(const LaunchCtx& c, const int32_t* list, int n_list, const void* A, void* B,
                           uint32_t advance);
// chains of BIG_CHAIN+1..1024 beads (at most max_n): one 1024-thread workgroup
// per box in `list`, with its node-table and impulse-spreading launches.
// after_table (may be null) is recorded on c.stream between the node-table
// kernel and the chain kernel.  Aprev (batched steps that defer tiles, sparse
// boxes only): the previous step's input buffer; the node-table kernel then
// fixes up the previous step's impulses outside its deferred tiles and the
// chain kernel clears them and resets the list counts (instead of the
// end-of-step kernel of launch_overflow).
// single_box: the box `list` holds when n_list == 1 (its descriptor is then
// passed to the node-table kernel by value), or -1.
// wait_head > 0: no node-table kernel; the step's collide carries the node
// tables (launch_collide_headed) and the chain kernel waits for its wait_head
// node-table workgroups, then clears the previous step's impulses outside its
// deferred tiles.  zero_head: the node-table kernel starts a run of such
// steps (zeroes the workgroup counts).  stamp_next: the chain kernel stamps
// the next step's deferred tiles from its end positions.
template <typename R>
hipError_t launch_couple_big(const LaunchCtx& c, const void* A, const int32_t* list, int n_list, int max_n,
                             uint32_t s_off, hipEvent_t after_table, const void* Aprev = nullptr,
                             int single_box = -1, uint32_t wait_head = 0, int zero_head = 0, int stamp_next = 0);
// step s_off's plain collide over tiles 0..n_tiles-1 with the node-table work
// of the big chains in `list` in its first workgroups (their count is
// head_blocks(n_list, max_n)); Aprev: the previous step's input buffer
template <typename R>
hipError_t launch_collide_headed(const LaunchCtx& c, const void* A, void* B, uint32_t n_tiles, uint32_t s_off,
                                 const int32_t* list, int n_list, int max_n, const void* Aprev, int single_box);
constexpr int BIG_CHAIN = 256;   // chains above this many beads take the one-workgroup-per-chain kernel
constexpr int NEAR_ITEMS = 27;   // table nodes per bead
inline uint32_t head_blocks(int n_list, int max_n)
{
    return (uint32_t)n_list * (uint32_t)((max_n * NEAR_ITEMS + 255) / 256);
}
hipError_t launch_advance(const LaunchCtx& c, uint32_t n);
// probe[0] set to value; probe[1] = whether probe[0] was set within 200 us
hipError_t launch_probe_set(hipStream_t stream, uint32_t* probe, uint32_t value);
hipError_t launch_probe_wait(hipStream_t stream, uint32_t* probe);
hipError_t launch_init_forces(const LaunchCtx& c, const int32_t* list, int n_list, int block);
// planes q0 .. q0 + nq - 1 of one box as canonical FP64 populations in n
// [nq][L^3], from or into the stored populations A; zeros behind every box's
// last node in a buffer that held other data
template <typename R>
hipError_t launch_export(const LaunchCtx& c, int box, const void* A, double* n, int q0, int nq);
template <typename R>
hipError_t launch_import(const LaunchCtx& c, int box, const double* n, void* A, int q0, int nq);
template <typename R>
hipError_t launch_clear_tails(const LaunchCtx& c, void* A);
// observables of the state A: per-block records in part [sum of stat_slots_of(n_tiles)][NSTAT_REC]
// (box b's from BoxDev::stat_off, sums of ranges of them behind, in boxes of more than STAT_DIRECT
// records), per-box records in out [n_boxes][OBS_REC], then the health bits and the step; max_recs: the
// most records of any box
template <typename R>
hipError_t launch_observables(const LaunchCtx& c, const void* A, uint32_t max_recs, double* part, double* out);

// device pointers of one reverse step of the adjoint window
struct AdjArgsHost {
    const double *x0, *v0, *f0, *tape, *dj;
    double *lx, *lv, *lf, *lam_n;
    const double* lam_dp;
    double* gz;
    uint64_t nodes;
};
template <typename R>
hipError_t launch_adj_collide(const LaunchCtx& c, const void* ccd, const void* P, const unsigned long long* imp,
                              const double* lam_next, double* lam_cur, double* lam_dp, double* gpart,
                              uint64_t nodes, uint32_t total_tiles, uint32_t step);
template <typename R>
hipError_t launch_adj_couple(const LaunchCtx& c, const int32_t* list, int n_list, int block, const void* P,
                             const AdjArgsHost& a, uint32_t step);

constexpr int N_COLLIDE_VARIANTS = 13;
constexpr int DEFAULT_COLLIDE_VARIANT = 3;   // one block per tile, at most 7 waves per SIMD
constexpr int NSTAT_REC = 24;
constexpr uint32_t STAT_CHUNKS = 64;    // ranges of a box's block records that are summed first,
constexpr uint32_t STAT_DIRECT = 256;   // where it has more than these
// Collide tiles per block of the observables pass, a function of the box
// alone: few for a small box, so that its blocks fill the GPU, as far as its
// records and their ranges fit 64 + n_tiles / 16 of them (what
// lb_observables_static counts per box).  Above 12000 tiles, where a CU holds
// one block (1024 threads, four waves per SIMD) and a block's sums weigh more
// than an uneven share: up to 64, in whole rounds of 256 blocks.  The whole
// call with 16 against this, us: 150^3 85 and 76, 160^3 93 and 84, 192^3 148
// and 131, 256^3 300 and 267; 128^3 and 144^3 are no faster with 32 to 64.
__host__ __device__ inline uint32_t stat_tpb(uint32_t n_tiles)
{
    if (n_tiles > 12000) {
        const uint32_t blocks = 256u * ((n_tiles + 256u * 64u - 1) / (256u * 64u));
        return ((n_tiles + blocks - 1) / blocks + 3u) & ~3u;
    }
    return n_tiles <= 320 ? 4u : (n_tiles <= 960 ? 8u : (n_tiles <= 2880 ? 12u : 16u));
}
__host__ __device__ inline uint32_t stat_recs_of(uint32_t n_tiles)
{
    return (n_tiles + stat_tpb(n_tiles) - 1) / stat_tpb(n_tiles);
}
// records of a box with the ranges behind them: at most 64 + n_tiles / 16 (rounded up)
__host__ __device__ inline uint32_t stat_slots_of(uint32_t n_tiles)
{
    const uint32_t n = stat_recs_of(n_tiles);
    return n > STAT_DIRECT ? n + STAT_CHUNKS : n;
}
constexpr int NCHAIN_REC = 11;
constexpr int OBS_REC = NSTAT_REC + NCHAIN_REC + 1;
constexpr int NL_SLOTS = 32;
constexpr int TAPE_REC = 40;     // doubles per bead and substep in the adjoint tape

}  // namespace lbd
