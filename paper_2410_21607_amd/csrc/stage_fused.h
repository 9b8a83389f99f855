// Fused Runge-Kutta stage: one pass over the columns of every refinement
// level computes q_out = a q^n + b q_s + c M^-1 Z^T (m_L R_L(Z q_s)).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <vector>

#include "devmesh.h"
#include "sem.h"

namespace sem {

struct HostMesh;

// Host-built tables of the fused path (device pointers).
//
// Columns are coloured so that no two columns of one colour contribute to a
// common unique node or hanging point; each colour is one launch.  For every
// (column, position) `first` says whether this column is the lowest-coloured
// contributor of its node: the first contributor writes the node, later ones
// add to it (plain read-modify-write, ordered by the launches).
struct FusedTables {
    const int32_t* col_order;   // columns sorted by colour; inside a colour by
                                // decreasing work (hanging positions), then Morton
    const int32_t* color_ptr;   // n_color + 1 offsets into col_order (host copy below)
    int n_color;
    const uint8_t* first;       // per (column, position)
    double* cH;                 // hanging-point contributions [F][n_hh][nzn]
    int layers_per_chunk;       // layers handled together by one workgroup step
    int thread_order;           // FP64 thread order: 0 = nodes of the planes between
                                // elements first, 1 = vertical index fastest,
                                // 2 = split element
    // Position map and interpolation rows the kernel reads (the mesh's own,
    // extended when the plan has side columns).  Side columns (the columns
    // of the small colour classes of an uneven mesh, and those that are their
    // own neighbour across a periodic side) run in the launches of
    // the other colours, spread to even them out; every position of theirs
    // maps to a pseudo hanging
    // point past the mesh's n_hh, whose row is the unit row of its node (or a
    // copy of its hanging row), so that the kernel stores the position's
    // contribution in cH unchanged; the tail launch assembles them.
    const int32_t* gmap;
    const int32_t *hang_ptr, *hang_src;
    const double* hang_w;
    const int32_t* hreal;       // per (pseudo) hanging point: index into the
                                // surface and reference rows ([0, n_h + n_hh))
    int64_t fsh;                // field stride of cH: (hanging + pseudo points) * ldz
};

// Tail launch: the unique nodes that receive side-slot or hanging-point
// contributions, each summing them in a fixed order and finishing the node.
struct TailTables {
    const int32_t* h;           // n: unique horizontal node
    const uint8_t* first;       // n: no column launch writes the node first
    // per node a flat list of contribution rows (hanging or pseudo hanging
    // points of cH) in groups: the node's side slots (weight 1), then per
    // hanging point of its Z^T row that point (when a column launch writes
    // it) and its side slots (weight w of the row); estart marks a group's
    // first entry and carries its weight; row -1 adds nothing
    const int32_t *eptr, *erow;
    const double* ew;
    const uint8_t* estart;
    const double* cH;           // hanging and pseudo hanging points
    int n;
    int64_t fsh;                // field stride of cH
};

// Block layout: the work unit is a 2 x 2 block of columns of one level (a
// sibling family, or four level-0 columns), split vertically into segments of
// `Ls` layers.  Blocks are coloured so that blocks of one colour share no
// node; a segment's planes are its own except the plane it shares with the
// segment above or below, whose first writer is the even segment (launches
// run colour by colour, even segments before odd ones).  Columns in no block
// run through the column kernel in their colour's turn.
struct BlockTables {
    const int32_t* order;       // blocks sorted by colour
    const int32_t* pos_g;       // n_blk * (2N+1)^2: unique node or -(hh+1) per block position
    const uint8_t* pos_first;   // n_blk * (2N+1)^2: first contributor of its node
    const int32_t* blk_col;     // n_blk: a member column (all four share the geometry)
    double* cH;                 // hanging-point contributions (the column layout's buffer)
    int64_t fsh;                // its field stride
    int n_seg, Ls;              // vertical segments, layers per segment
};

// Owner kernel: regular nodes, each computed whole by one column.  A node is
// regular when every column sharing it has the same level and the columns
// surround it completely (one inside a column, two at a face, four at a
// corner) and no hanging point takes its value from it; its owner is the
// column that has it at a position i < N, j < N.  `map` lists per column the
// positions the kernel loads (row_offset of each, rows.h): the owned N x N
// (i + N j), the upper faces (N, j) and (i, N), then the halo lines, N
// positions each: per j the left neighbour's (i, j), per i the lower
// neighbour's (i, j).  The nodes that are not regular are left to the side
// columns and the tail.
constexpr int own_owned(int N) { return N * N; }
constexpr int own_positions(int N) { return 3 * N * N + 2 * N; }
struct OwnTables {
    const uint32_t* map;        // n * own_positions(N)
    const double* sxy;          // n * (2/dx, 2/dy)
    const uint64_t* mask;       // n: bit i + N j, the node is regular
    const uint8_t* hang;        // n: some position of `map` hangs
    int n;
};

// Owns the device memory of the tables.
struct FusedPlan {
    FusedTables t{};                      // column layout (every column)
    std::vector<int32_t> color_ptr_host;
    TailTables tail{};                    // column layout with side columns
    bool has_tail = false;
    bool own = false;                     // tables of the owner kernel (own_used: whether a stage runs it)
    bool by_default = false;              // column layout at param = 0
    OwnTables ot{};
    FusedTables to{};                     // its side columns (one launch) and their tail
    TailTables own_tail{};
    int n_side = 0;
    int layout = 0;                       // SEM_LAYOUT_COLUMNS, _COLUMNS_KZ, _COLUMNS_SPLIT or _BLOCKS
    BlockTables bt{};                     // block layout
    FusedTables ts{};                     // block layout: the columns in no block
    std::vector<int32_t> blk_ptr_host, single_ptr_host;   // per colour
    int n_unit_color = 0;
    bool blk_wrap = false;                // fused_blocks_wrap: the stage runs the column layout
    std::vector<void*> allocs;
    int64_t bytes = 0;
};
// layout SEM_LAYOUT_COLUMNS / _COLUMNS_KZ / _COLUMNS_SPLIT: param = layers per
// chunk (0 = default);
// SEM_LAYOUT_BLOCKS: param = vertical segments (0 = default).  owner: with the
// owner kernel's tables where it applies.
int fused_plan_build(const HostMesh& H, int layout, int param, FusedPlan& plan, bool owner);
// Another layout of the same kind, or another param, on the tables that a plan
// has (none of them depends on these).
int fused_plan_set(const HostMesh& H, int layout, int param, FusedPlan& plan);
// Whether stages of a layout take the owner kernel where it applies: a program
// that names a thread order or a chunk gets the coloured launches it names.
inline bool fused_plan_owner(int layout, int param) { return layout == SEM_LAYOUT_COLUMNS && param == 0; }
void fused_plan_free(FusedPlan& plan);
bool fused_lpc_supported(int N, int layers_per_chunk);
// whether the split-element thread order applies (two or more layers per
// chunk, every pair of threads of a plane node in one wave)
bool fused_split_supported(int N, int layers_per_chunk);
bool fused_blocks_supported(const HostMesh& H);
// whether a block, or a column in no block, touches itself across a periodic
// side: two of its positions are then one node
bool fused_blocks_wrap(const HostMesh& H);

// Whether sem_stage evaluates the optional dissipation inside the column
// kernel (FP64, box elements, column layout) instead of a pre-pass.
bool fused_dissipation_inline(const DevMesh& m, const FusedPlan& plan, int precision);

// The owner kernel: whether it has an instance of order N; whether a state is
// within its limits (32-bit offsets, the level table in LDS); whether plans of a
// mesh hold its tables (an instance, the limits, and where it is the faster
// one, by the mesh and by its side columns); whether a default-layout stage on
// such a mesh takes it; its launch over the plan's regular nodes.
bool own_supported(int N);
bool own_fits(int64_t n_h, int ldz, int nzn);
bool own_applies(const HostMesh& H);
bool own_with_sides(const HostMesh& H, int n_side);
bool own_used(const DevMesh& m, int precision);
int own_launch(const DevMesh& m, const OwnTables& ot, double a, double b, double c, const double* qn,
               const double* qs, double* qout, hipStream_t stream);

// Launches the column kernel and the shared-node kernel on `stream`.
int fused_stage_launch(const DevMesh& m, const FusedPlan& plan, double a, double b, double c,
                       const double* qn, const double* qs, double* qout, int precision,
                       hipStream_t stream);

}  // namespace sem
