// Kernel launchers (C++ linkage, internal to the library).
#pragma once

#include "lbm_common.h"

// One work item of the fused D2Q9 kernel: a 60-column strip of a simulation
// starting at column x0, output rows [y0, y0 + rows).  sim < 0: padding.
struct FusedItem {
    int32_t sim, x0, y0, rows;
};

// Per-simulation pointers for the fused kernel.  The source buffer of a
// launch is buf[parity ^ flip], the destination the other one.
struct FusedSim {
    const SimConst *c;
    void *buf[2];
    uint32_t *status;
    int32_t parity;
    int32_t nx, ny;
    int32_t pad;
};

// What a fused step is launched over: items of at most `rows` rows, nsims
// simulations.
struct FusedTable {
    const FusedItem *items;
    int nitems;
    const FusedSim *sims;
    int nsims;
    int rows;
};

constexpr int FUSED_LANES = 64;
constexpr int FUSED_OUT = 60;  // output columns per strip (2-column halo each side)

hipError_t launch_init(int lattice, bool fp32, const SimConst *c, int64_t ns, const double *rho,
                       void *g, hipStream_t st);
// keep_old: tau != 1, the collision reads the old populations
hipError_t launch_step_generic(int lattice, bool fp32, const SimConst *c, int ncomp, int nx, int ny,
                               int nz, const void *gs, void *gd, double *rho_f, double *psi_f,
                               double *s_f, double *j_f, double *u_f, uint32_t *status,
                               bool keep_old, hipStream_t st);
// Planes [p0, p0 + n) of a state's populations in host order (plane i Q + a:
// population a of component i, [sites] FP64) <-> a population buffer:
// out, buffer to planes; else planes to buffer (FP32 storage rounds).
hipError_t launch_planes(int lattice, bool fp32, bool out, int ncomp, int nx, int ny, int nz,
                         int p0, int n, void *buf, void *planes, hipStream_t st);
// na doubles of a and nb of b behind each other at `to`, and the status word
// to `word` (pinned host memory both), in one launch.
hipError_t launch_to_host(const double *a, int64_t na, const double *b, int64_t nb,
                          const uint32_t *status, double *to, uint32_t *word, hipStream_t st);
// One member of a batched multi-pass step (fuglbm_step_many for simulations
// on the multi-pass kernels).  A launch reads buf[parity ^ flip] and writes
// the other buffer.  end[p]: work units of pass p through this member,
// cumulative over the table (p = 0: TPB-site blocks of the moments and
// interface passes, 1: velocity tiles, 2: collision (tile, component) units).
struct GenMember {
    const SimConst *c;
    void *buf[2];
    double *rho_f, *psi_f, *s_f, *j_f, *u_f;
    uint32_t *status;
    int64_t end[3];
    int32_t parity;
    int32_t pad;
};
// Work units of one simulation for the three kinds of GenMember::end.
void generic_units(int lattice, int ncomp, int nx, int ny, int nz, int64_t units[3]);
// One step of every member (same lattice, storage precision and keep_old);
// total[p] = members[nmembers - 1].end[p].
hipError_t launch_step_generic_batch(int lattice, bool fp32, bool keep_old,
                                     const GenMember *members, int nmembers,
                                     const int64_t total[3], int flip, hipStream_t st);
// Macroscopic fields of a state: rho_i, RT ln f_i (in psi_f), s, j and (u_f
// non-null) psi_i and the force-corrected velocity.
hipError_t launch_fields(int lattice, bool fp32, const SimConst *c, int nx, int ny, int nz,
                         const void *g, double *rho_f, double *psi_f, double *s_f, double *j_f,
                         double *u_f, uint32_t *status, hipStream_t st);
// Diagnostic sums over the fields (rho_i, j, u): per-block partials in
// part[(ncomp + 1) * nblk * DIAG_QUANT], final sums in out[(ncomp + 1) * DIAG_QUANT]:
// out[i] = {mass_i, sum |rho_i - snap_i|, 0...} for i < ncomp (snap_i <- rho_i),
// out[ncomp] = {sum j (3), sum rho u (3)}.
constexpr int DIAG_QUANT = 6;
hipError_t launch_diag(int dim, int ncomp, int64_t ns, const double *rho_f, const double *j_f,
                       const double *u_f, double *snap, double *part, int nblk, double *out,
                       int use_snap, hipStream_t st);
int diag_blocks(int64_t ns);

// Fused one-pass D2Q9 step over a table of work items (any mix of
// simulations with the same component count and storage precision).
// Resident workgroups of the fused kernel per CU (occupancy query).
int fused_blocks_per_cu(int ncomp, bool fp32);

hipError_t launch_fused_d2q9(int ncomp, bool fp32, const FusedItem *items, int nitems,
                             const FusedSim *sims, int flip, hipStream_t st);

// The same step for tables whose items have at most `rows` (1 or 2) rows,
// built for ncomp <= 10 (fused2d_block.h).
constexpr int FUSED_BLOCK_ROWS = 2;
constexpr int FUSED_BLOCK_COMP = 10;
hipError_t launch_fused_block(int ncomp, bool fp32, const FusedTable &t, int flip, hipStream_t st);

// Store-wave variant of the fused D2Q9 step (component waves only load;
// two extra waves per workgroup store; rows requested three ahead).  Same
// items, same results bit for bit.  Built for ncomp <= fused_ws_max_comp().
int fused_ws_max_comp();
bool fused_ws_fits(int ncomp, bool fp32);
int fused_ws_blocks_per_cu(int ncomp, bool fp32);
hipError_t launch_fused_d2q9_ws(int ncomp, bool fp32, const FusedItem *items, int nitems,
                                const FusedSim *sims, int flip, hipStream_t st);

// ---- D2Q9 steps at tau = 1 in field form (fields2d.h) -----------
// One simulation: its population buffers (the run reads buf[parity ^ flip]
// and writes its last state there again; the other buffer holds fields
// between the steps) and workspace fields.  ld: elements from one component
// of a field to the next; wide: every field lies in the spare population
// buffer (else set 0 and psi in the workspace, components ld = sites apart).
// end: blocks of 256 sites through this member, cumulative over a table.
struct FieldSim {
    const SimConst *c;
    void *buf[2];
    double *rho, *psi, *s, *j, *u;
    uint32_t *status;
    int64_t end, ld;
    int32_t parity, wide;
    int32_t nx, ny;
};
// What the steps of a run are launched over: one simulation (tab null; work
// items follow from strips and rows, nitems of them) or a table of nm
// members with a work-item table.
struct FieldRun {
    const FieldSim *tab;
    int nm;
    FieldSim one;
    const FusedItem *items;
    int nitems, strips, rows;
    int64_t blocks;
    int flip;
    bool single;          // steps (but the last) by single wavefronts
};
int field_max_comp();   // built for ncomp <= this
int field_single_comp();  // `single` for ncomp <= this
int field_blocks_per_cu2d(int ncomp, bool single);
// populations -> set 0
hipError_t launch_field_moments2d(const FieldRun &q, bool fp32, hipStream_t st);
// psi and 1/rho of set `set`
hipError_t launch_field_eos2d(const FieldRun &q, int ncomp, int set, hipStream_t st);
// one step from set `set` to the other one, or (last) to the populations
hipError_t launch_field_step2d(const FieldRun &q, int ncomp, bool fp32, bool last, int set,
                               hipStream_t st);

// ---- D3Q19 steps at tau = 1 in field form (fields3d.h) --------------------
// Tiles of the stream kernel: W - 4 columns, (threads / W) - 2 rows, zc planes;
// how many of them there are along x, y, z.
struct Tiles3 {
    int32_t W, zc, tx, ty, tz;
};
// What the steps of a run are launched over: the two sets of fields.
struct FieldRun3 {
    GenMember f[2];
    int64_t ns;
    int nitems;           // workgroups of the stream kernel
    int waves;            // wavefronts of one (FP32 storage: at most 12, else 8)
    Tiles3 tiles;
    int64_t total[3];     // work units as of GenMember::end
};
// Resident workgroups of the stream kernel per CU (occupancy query).
int field3_blocks_per_cu(bool fp32, int waves);
// populations -> set 0 with its psi
hipError_t launch_field_moments3(const FieldRun3 &q, bool fp32, hipStream_t st);
// one step from set `set` to the other one with its psi
hipError_t launch_field_step3(const FieldRun3 &q, int ncomp, bool fp32, int set, hipStream_t st);
// the last step: from set `set` to the populations
hipError_t launch_field_last3(const FieldRun3 &q, bool fp32, int set, hipStream_t st);
