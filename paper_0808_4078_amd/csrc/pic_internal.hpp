// Internal layout shared by the HIP kernels and the host runtime of libpic.
//
// Everything the kernels need lives in one device-resident KParams block
// written once at initialisation, so a step is a fixed sequence of launches
// with pointer-only arguments (replayable as a graph).  Per-step mutable
// state (step counter, particle-set parity, overflow flags) is in DevState,
// also in device memory, and is advanced by the last kernel of each step.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/pic.h"

namespace pic {

constexpr int kMaxSpecies = PIC_MAX_SPECIES;
// Launch shapes of the particle kernel: threads per workgroup and the
// particles each lane keeps in flight (their loads issued ahead of the one it
// processes).  Shape 0 is the default and the only one of the FP64 kernels;
// mixed-precision runs take any (pic_grid_desc.shape, chosen by the tuner).
constexpr int kShapes = PIC_PARTICLE_SHAPES;
constexpr int kShapeBlock[kShapes] = {256, 256, 256, 512, 128};
constexpr int kShapeInflight[kShapes] = {2, 1, 3, 2, 2};
// Threads per workgroup of the particle kernel.  A 3D tile in FP64 takes 80 KB
// of LDS for its fields and current, so only one workgroup fits a CU: it has
// 512 threads, two waves per SIMD instead of one (64x64x128 cells, 8 + 8 per cell:
// particle kernel 590 -> 440 us).
constexpr int shape_threads(bool fp64, int ndim, int shape)
{
    return fp64 && ndim == 3 && shape == 0 ? 512 : kShapeBlock[shape];
}
constexpr int kRing = 4096;          // diagnostic records kept on the device
constexpr int kTileDiag = 6;         // per tile and species: KE, px, py, pz, count, collisions
constexpr int kFieldDiag = 10;       // per block: W[6], p_field[3], unused
constexpr int kFieldDiagBlocks = 512;
constexpr int64_t kSplitGroups = 1024;             // workgroups that a grid with few tiles is split into
constexpr int64_t kSplitMin = 512;                 // particles that a workgroup of a split tile takes at least
constexpr int64_t kSplitBytes = int64_t(24) << 20; // bound of the split tiles' partial currents
constexpr int kSplitLine = 32;                     // words per counter of a split tile: a cache line
constexpr int kBinAlign = 64;        // particle-store bins start at multiples of this many slots
constexpr int kMomentBlocks = 1024;  // loader reductions
constexpr int kMomentVals = 6;

// Philox counter word 2 tags the purpose of a draw.
constexpr uint32_t kPurposeCollide = 1u;
constexpr uint32_t kPurposeLoad = 2u;
constexpr uint32_t kPurposeCoulomb = 3u;
constexpr uint32_t kPurposeBinaryKey = 4u;     // pairing order of the binary collisions
constexpr uint32_t kPurposeBinaryPair = 5u;    // one pair's deflection

struct DevState {
    int64_t step;        // index n of the step about to run
    int32_t par;         // particle set holding the current particles (0/1)
    int32_t rebin;       // an incoming-mover reserve overflowed during this step
    int32_t fatal;       // sticky: 1 overflow list exhausted, 2 particle off the grid, 4 store reserve
                         // exhausted, 8 particle outside its bin, 16 binary collisions: a cell above the
                         // participant limit
    int32_t pad;
    int64_t rebins;      // re-layouts performed so far
    int64_t ring_head;   // diagnostic records written so far
    uint32_t ovf_count[kMaxSpecies];
};

// Particle arrays of one species.  Sets 0 and 1 alternate as source and
// destination from step to step; set 2 is the overflow list.
//  mixed: sets 0, 1: cell within the tile of the particle's bin, 16 bits
//         (lx | ly << ts | lz << 2 ts, ts = log2 T); set 2: global packed
//         cell (ix | iy << sh1 | iz << sh2); pos = FP32 in-cell offset
//  fp64 : no cell array, pos = absolute FP64 position in cell units
struct SpeciesDev {
    uint16_t *cell[2];
    uint32_t *ovf_cell;
    void *pos[3][3];     // [set][axis]
    void *u[3][3];       // [set][component]
    uint32_t *id[3];
    int32_t *start;      // [tiles] first slot of each tile's bin
    int32_t *cap;        // [tiles] bin capacity
    uint32_t *cnt_front; // [2][tiles] particles written from the bin's front
    uint32_t *cnt_back;  // [2][tiles] movers written from the bin's back
    int64_t ncap;        // slots per set
    int64_t nominal;     // ppc * cells
    uint32_t ovf_cap;
    uint32_t coll_thr;   // scatter when the 32-bit draw is below this (isotropic model)
    int32_t collide;
    int32_t coll_model;  // PIC_COLL_ISOTROPIC or PIC_COLL_COULOMB
    double coll_sig2;    // Coulomb model: variance of tan(theta/2) = coll_sig2 / v^3
    int32_t track_id;    // carry ids (collisional species, or all in test mode)
    double q, m, w;
    double qmdt2;        // q dt / (2 m)
    double qw;           // q w
    int32_t ppc;
    int32_t id_base;
    double drift[3];     // loader: mean momentum
    double uth;          // loader: Gaussian spread per component
    int32_t binary;      // takes part in the binary (pairwise) collisions
};

struct Geometry {
    int ndim;
    int n[3];
    double d[3];
    double dt;
    int tile[3];
    int nt[3];           // tiles per axis
    int ntiles;
    int tshift[3];       // log2(tile)
    int csh[3];          // cell packing shifts (mixed)
    uint32_t cmask[3];
    int64_t cells;
};

struct KParams {
    Geometry g;
    int nspecies;
    int precision;       // PIC_PREC_*
    int diag_every;
    unsigned flags;
    uint64_t seed;
    uint32_t run;
    SpeciesDev sp[kMaxSpecies];
    void *F;             // 6 planes Ex Ey Ez Bx By Bz (float or double)
    double *J;           // 3 planes
    void *Jtile;         // [tiles][3][nj^ndim] per-tile partial currents
    int nj;              // tile edge + 3
    double *tile_diag;   // [tiles][nspecies][kTileDiag]
    double *field_diag;  // [kFieldDiagBlocks][kFieldDiag]
    double *moments;     // [kMomentBlocks][kMomentVals]
    DevState *state;
    pic_diag *ring;      // [kRing]
    int32_t *rb_count;   // [nspecies][tiles]
    int32_t *rb_start;   // [nspecies][tiles]
    int32_t *rb_cap;     // [nspecies][tiles]
    int32_t *rb_fill;    // [nspecies][tiles]
    int64_t *ex_off;     // [tiles + 1] read-out: first particle of each tile, total
    int32_t *rl_ovf;     // [nspecies][tiles] overflowed particles per new tile (zero between steps)
    int32_t *rl_ticket;  // [2] workgroups that have ended a re-layout phase (zero between steps)
    void *Ft;            // 6 planes: E^{n+1} and B^{n+1/2} between the field passes (null: unfused passes)
    int fd_blocks;       // blocks (and partial records) of the field-diagnostic reduction
    int32_t split;       // workgroups per tile of the particle kernel (1, or more where the grid has few tiles)
    void *Jsplit;        // split > 1: [tiles][split][3][nj^ndim] FP64 partial currents
    uint32_t *split_cnt;    // split > 1: [nspecies][tiles][2][kSplitLine] particles written to the bin's front
                            // and back so far this step
    double *split_diag;  // split > 1: [tiles][split][nspecies][kTileDiag]
    int32_t *order;      // [tiles] particle-kernel work order (XCD class, then decreasing load)
    uint8_t *tile_bucket;   // [tiles] load bucket of each tile, written by the particle kernel
    double order_scale;  // bucket = round(particles in the tile * order_scale): 16 per nominal load
    int32_t coulomb;     // 1 if a species scatters with the Coulomb model (selects the particle kernel)
    int32_t shape;       // particle-kernel launch shape (index into kShapeBlock / kShapeInflight)
    double nu_ee;        // binary collisions: rate at relative speed ee_vref (0 = off)
    double ee_vref;
    int32_t binary;      // 1 if the binary-collision kernel runs (nu_ee > 0 and a species takes part)
    uint32_t *ee_ent;    // binary collisions: each tile's participants (slot | species << 29) by block of cells,
                         // the tile's list at the sum over participating species of its bin starts
    uint32_t *ee_off;    // [tiles][blocks] end of each block's part of the tile's list
    uint32_t *ee_part;   // [ee_nparts] pairs scattered this step by each workgroup of the binary-collision kernel
    int32_t ee_nparts;
    // Gauss-law and continuity checks (PIC_FLAG_GAUSS_RESIDUAL only; null otherwise)
    double *rho_tile;    // [tiles][(T+1)^ndim] per-tile charge partials
    double *rho0;        // [cells] charge on the nodes at step 0
    double *rho_n;       // [cells] charge on the nodes at the start of the current check step
    double *gauss_part;  // [ceil(cells / 256)][2] per-block maxima of the residual and of |rho - rho0|
    double *cont_part;   // [ceil(cells / 256)][2] per-block maxima of the continuity residual and |rho' - rho|
};

// An ensemble of runs stepped together: every launch of a step covers all
// runs.  Runs share precision and dimension; in 2D each run has its own tile
// edge, and the particle kernel is launched once per edge (group g: edge
// 8 << g; 3D runs use group 0).  The work items (run, k) -- the k-th tile of
// the run's work order, whose tile index is k mod 8 -- are split by XCD
// class k mod 8 into one list and one queue per class.
constexpr int kBatchXcds = 8;
struct BatchGroup {
    int n_items;                   // work items of the runs with this edge
    const int2 *items;             // [n_items] (run, k), class-major; in a class,
                                   // runs with the most particles per tile first
    int cls_start[kBatchXcds];     // first item of each class
    int cls_len[kBatchXcds];       // items of each class
    int *queue;                    // [kBatchXcds] work counters of the persistent particle kernel
    int shape;                     // particle-kernel launch shape of the runs with this edge
};
constexpr int kBatchGroups = 3;
struct BatchTable {
    int nruns;
    int n_cell_blocks;    // 256-cell blocks over all runs
    int fused;            // 1: fused field passes (every run has KParams::Ft, up to kFusedCells in all)
    int max_fd_blocks;    // max over runs of KParams::fd_blocks
    int coulomb;          // 1 if any run has a species on the Coulomb scattering model
    const KParams *const *kp;   // [nruns] device parameter blocks
    const int2 *cell_blocks;    // [n_cell_blocks] (run, block of that run)
    BatchGroup grp[kBatchGroups];
};
// Steps of a single run that one graph replay enqueues, while as many are asked
// for (the rest are replays of one step): consecutive replays lie 5 us further
// apart than the nodes of one graph (10 steps of 64x64, FP64: 380 -> 351 us; of
// 160x160, mixed: 864 -> 833 us).  Eight would save half as much again of that
// for twice the nodes; four cost 60 us more when the run is made.
constexpr int kChainSteps = 4;
// Cells up to which a 2D run, or an ensemble in all, takes the fused field
// passes.  On larger grids they lose what they save: mostly to the registers
// that the re-layout's copies give the second pass (three or four waves per
// SIMD; with the copies in a launch of their own 4096^2 takes 1.478 ms fused,
// 1.476 one by one, 1.665 with them, 2048^2 0.654, 0.637, 0.679), which small
// grids pay for with a launch less (512^2: 0.060 against 0.066).  ms per step, one by one / fused, ensembles of 1.1M cells
// 1.103 / 1.100, 2.2M 2.384 / 2.382, 4.6M 4.72 / 4.79, 21M 20.40 / 20.87; runs of
// 1M cells 0.515 / 0.493, 2.1M 1.160 / 1.150, 4.2M 1.795 / 1.807, 17M 2.69 / 2.78.
constexpr int64_t kFusedCells = 1ll << 21;
// workgroups per run of an ensemble for the two phases of its re-layout
constexpr int kBatchCountBlocks = 32;
constexpr int kBatchRebinBlocks = 256;

// Host-callable launchers (defined in the .hip translation units).
// Groups of a step's kernels: field record and checks (0), particle and binary
// collisions (1), re-layout launched apart (2), current reduction / first field
// pass (3), Yee / second field pass (4), end of step (5).  step_kernel_groups
// fills groups[] with each launch's group and returns the number of launches
// (at most kMaxStepKernels).
constexpr int kNumGroups = 6;
constexpr int kMaxStepKernels = 16;
int step_kernel_groups(const KParams &hp, int *groups);
// Workgroups per tile of the binary-collision kernel, and the cells each
// takes, for ppc participants per cell.
int binary_blocks(bool mixed, int64_t tile_cells, int64_t ppc, int *width);
// Room for the parameter block in the part of the scratch that a checkpoint
// holds (the block itself lies behind that part).
constexpr size_t kCkptParamBytes = 3256;
// ev: NULL, or two events (start/stop) per launch
hipError_t launch_step(const KParams &hp, const KParams *dp, hipStream_t s, hipEvent_t *ev = nullptr);
// Batch step: batch_kernel_groups fills groups[] as step_kernel_groups does.
// pblocks[g]: persistent workgroups of group g's particle launch.
int batch_kernel_groups(int precision, int ndim, const BatchTable &ht, int *groups);
hipError_t launch_batch_step(int precision, int ndim, const BatchTable &ht, const BatchTable *dt,
                             const int pblocks[kBatchGroups], hipStream_t s, hipEvent_t *ev = nullptr);
// Workgroups of the batch particle kernel of tile group g that fit on one
// compute unit at once.
hipError_t batch_particle_occupancy(int precision, int ndim, int g, bool coulomb, int shape, int *blocks_per_cu);
// Initialisation shared by pic_init (static_device = -1, the caller's
// scratch) and pic_init_static_scratch (the library's scratch of that
// device, already claimed; pic_destroy releases it).
// static_scratch_needed: bytes of that scratch that count against
// PIC_STATIC_SCRATCH_BYTES; parts of the scratch that a run can do without are
// left out where the whole does not fit.
size_t static_scratch_needed(const pic_grid_desc *grid, const pic_species_desc *species, int nspecies);
int init_run(const pic_grid_desc *grid, const pic_species_desc *species, int nspecies,
             const pic_buffers *buffers, void *hip_stream, pic_run **out, int static_device);
// The library's scratch: what a caller may count on, and room for what lies
// behind the part of the scratch that a checkpoint holds (parameter block,
// read-out places, re-layout and binary-collision counts).  That is at most
// 8 + 4 nspecies bytes per tile, 48 with 8 species and collisions, where the
// part itself is at least 1452 (8^2 tiles, FP32 currents) + 64 nspecies: at the
// most 1.4 MiB for a run whose part fits PIC_STATIC_SCRATCH_BYTES.
constexpr size_t kStaticScratch = PIC_STATIC_SCRATCH_BYTES + ((size_t)2 << 20);
// One run at a time per device may hold the library's scratch of that device.
constexpr int kMaxDevices = 64;
bool claim_static_scratch(int device);     // false if held
void release_static_scratch(int device);
// Records a message for pic_last_error(NULL, ...) and returns code.
int fail_global(int code, const char *fmt, ...);

// Read-out of species s: the tiles' first places (ex_off), then the particles
// in places [k0, k0 + n) as FP64 x [ndim][n] and u [3][n] and ids [n] to `out`.
hipError_t launch_export_scan(const KParams &hp, const KParams *dp, int s, hipStream_t st);
hipError_t launch_export(const KParams &hp, const KParams *dp, int s, int64_t k0, int64_t n, void *out, hipStream_t st);
hipError_t launch_load_species(const KParams &hp, const KParams *dp, int s, hipStream_t st);
hipError_t launch_moments(const KParams &hp, const KParams *dp, int s, double delta_uz, hipStream_t st);
hipError_t launch_shift_u(const KParams &hp, const KParams *dp, int s, double dux, double duy,
                          double duz, hipStream_t st);

}  // namespace pic
