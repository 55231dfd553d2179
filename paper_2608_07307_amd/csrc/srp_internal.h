// Internal data layout shared by the host runtime and the gfx950 kernels.
//
// Device memory of a scene (built once, Sec. 4.4.1: one rigid node = one
// bottom-level hierarchy in rest-pose coordinates):
//   TriRec  tris[T]   triangles in leaf order, 48 B each (3 corners + ids)
//   BNode4  blas[..]  4-wide hierarchy nodes of all tree nodes, 128 B each
//   float2  mats[M]   (rho_s, rho_d)
//   WPoint  wpts[..]  distinct (vertex, tree node) pairs, for the window pass
// Device memory of an articulation slot (one per distinct hinge-angle vector,
// Sec. 4.4.2 steps 1, 4, 5 as rigid instance transforms; built by the host for
// a scene's current angles, by k_articulate for a batch's angle vectors):
//   Inst    inst[K]   local->world transform + bottom-level root, 64 B each
//   BNode4  tlas[..]  the scene's top-level topology refitted to the instances'
//                     world boxes
//   double  xf[K][12] FP64 transforms (window pass)
//   double  axw[J][3] world-frame hinge axes (gradient)
//   int32   dof_node[J]
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace srp {

// ---- references stored in hierarchy nodes and on the traversal stack ----
// bits 31..30 type; BLAS leaf payload = (first_tri << 3) | (count - 1).
constexpr uint32_t REF_BLAS_NODE = 0u;
constexpr uint32_t REF_BLAS_LEAF = 1u;
constexpr uint32_t REF_TLAS_NODE = 2u;
constexpr uint32_t REF_TLAS_LEAF = 3u;
constexpr uint32_t REF_NONE = 0xFFFFFFFFu;
constexpr int LEAF_MAX = 8;
#ifndef SRP_STACK_DEPTH
#define SRP_STACK_DEPTH 64                  // (a host build of the traversal may lower it to check overflow reporting)
#endif
constexpr int STACK_DEPTH = SRP_STACK_DEPTH;   // per-lane traversal stack entries (the build checks each hierarchy's worst case)
#ifndef SRP_STACK_LDS
#define SRP_STACK_LDS 16                    // (a host build may shrink it to exercise the spill path)
#endif
constexpr int STACK_LDS = SRP_STACK_LDS;    // of which the newest live in LDS (a ring)
constexpr int STACK_SPILL = STACK_DEPTH - STACK_LDS;   // older ones: per-lane global spill area
static_assert((STACK_LDS & (STACK_LDS - 1)) == 0, "the LDS ring size is a power of two");
constexpr int BLAS_MAX_DEPTH = 24;          // binary internal nodes on any root-to-leaf path (build)
constexpr int TLAS_MAX_DEPTH = 7;           // <= 128 instances, median split (build)
constexpr int BLOCK = 256;                  // threads per block of the trace kernel (4 waves)
constexpr int PATCH = 8;                    // a patch is PATCH x PATCH pixels: one ray per lane of a wave
constexpr int TILE = 16;                    // patches are numbered by 16x16 tile (row-major), 4 per tile
constexpr int MAX_PPC = 64;                 // patches per chunk or gradient group (one wave's work item) at most
constexpr int GROUP_PART = 8;               // patches of a gradient group per wave of the adjoint kernel
constexpr int MAX_GRAD_SLOTS = 960;         // doubles per wave for gradient partials (LDS <= 64 KB)

#define SRP_HD __host__ __device__
// Memory that nothing writes during the kernel: its uniform reads are scalar loads.
#define SRP_CONST __attribute__((address_space(4)))

SRP_HD inline uint32_t make_ref(uint32_t type, uint32_t idx) { return (type << 30) | idx; }
SRP_HD inline uint32_t ref_type(uint32_t r) { return r >> 30; }
SRP_HD inline uint32_t ref_index(uint32_t r) { return r & 0x3FFFFFFFu; }

// 4-wide hierarchy node: the boxes of up to four children as structure of
// arrays inside the node (one 16-byte load gives one bound of all four), their
// references, 128 B.  An empty slot has reference REF_NONE and a box with
// every coordinate +inf, which no ray enters.
struct alignas(128) BNode4 {
    float lox[4], loy[4], loz[4];
    float hix[4], hiy[4], hiz[4];
    uint32_t ref[4];
    uint32_t pad[4];
};
static_assert(sizeof(BNode4) == 128, "BNode4 is 128 bytes");

struct alignas(16) TriRec {
    float v0[3];
    int32_t id;     // original triangle index
    float v1[3];
    int32_t mat;
    float v2[3];
    int32_t node;
};
static_assert(sizeof(TriRec) == 48, "TriRec is 48 bytes");

struct alignas(64) Inst {
    float R[9];       // local -> world rotation, row-major
    float t[3];       // local -> world translation
    uint32_t root;    // bottom-level root reference
    int32_t node;
    float pad[2];
};
static_assert(sizeof(Inst) == 64, "Inst is 64 bytes");

struct alignas(32) WPoint {
    double x, y, z;
    int32_t node;
    int32_t pad;
};

// Per-patch partial sums (unscaled: multiply by P * A_pix).
struct alignas(64) PatchOut {
    double f[6];        // force (3), torque (3)
    uint32_t hits, sec, sec_hits, flags;
};

// A fan emitter (a chain hit that emits diffuse rays), written by the trace
// kernel at slot gen * 64 + lane of its patch's region and read by the fan
// kernel: hit point, weight w rho_d / K of each diffuse ray, oriented normal,
// original index of the hit triangle (excluded from the fan's rays).
struct alignas(16) FanRec {
    float x[3];
    float wd;
    float n[3];
    int32_t id;
};
static_assert(sizeof(FanRec) == 32, "FanRec is 32 bytes");

// Diffuse rays per fan task: the fan kernel's lane task is one emitter times
// one slice of FAN_SLICE consecutive fan-ray indices.
constexpr int FAN_SLICE = 2;   // (4 and 1 measured: 2 gives single evaluations at the paper's
                                //  setting 3 % with batches unchanged; 1 costs batches 2 %)
static_assert(SRP_MAX_BOUNCES == 4, "fan emitter masks: four generations");
// Most range sums per evaluation in the reduction's first stage (separate
// blocks, added in order by the second).
constexpr int MAX_SLICES = 16;

// A range sum of an evaluation's patch (and fan) partials: force and torque
// (FP64, before scaling), hit and test counts, status flags.
struct alignas(16) SliceOut {
    double f[6];
    uint64_t cnt[5];   // primary hits, secondary rays, secondary hits, box tests, triangle tests
    uint32_t flags;
    uint32_t pad_;
};
static_assert(sizeof(SliceOut) == 96, "SliceOut is 96 bytes");

// One kinematic-tree node as the articulation kernel reads it (built once per
// scene): the edge label (pivot, axes as given and renormalised for the
// rotation), the padded rest-pose box of the node's triangles and its
// bottom-level root.
struct alignas(16) ArtNode {
    double pivot[3];
    double axis[3][3];
    double unit[3][3];
    double blo[3], bhi[3];
    int32_t parent, n_axes, dof_offset;
    uint32_t blas_root;
    int32_t depth;      // edges from the root
    int32_t pad_;
};
static_assert(sizeof(ArtNode) == 240, "ArtNode layout");

// One articulation slot to build on the device: the scene's nodes and top-level
// topology (each node's height, the most inner-node levels below it, in
// pad[0]), the cosine and sine of each clamped hinge angle (2 per degree of
// freedom), and where the slot's arrays go.
struct alignas(16) ArtJob {
    const ArtNode *nodes;
    const BNode4 *topo;
    const double *cs;
    Inst *inst;
    BNode4 *tlas;
    double *xf;
    double *axw;
    int32_t *dof_node;
    double pad;
    int32_t n_nodes, n_tlas;
    int32_t max_depth, max_height;
    int32_t pad_[2];
};
static_assert(sizeof(ArtJob) == 96, "ArtJob layout");

// An evaluation's primary rays and, per instance, the map of its rest-pose
// points to image coordinates (column X = u . p + uc, row Y = v . p + vc; pixel k's
// ray at k), its frame of the photon direction and its image rectangle:
// written by k_primary_setup, read by k_primary.
struct alignas(64) PrimaryEval {
    float o0[3], su[3], sv[3];   // ray (px, py) starts at fma(py, sv, fma(px, su, o0))
    float mx, my;                // pixel margin: twice the hierarchy's box padding
    int32_t empty;               // nothing to trace
    int32_t traced;              // a sliver of a window: the trace kernel traces the primary rays
    int32_t pad_[3];
};
static_assert(sizeof(PrimaryEval) == 64, "PrimaryEval layout");
struct alignas(64) PrimaryInst {
    float rect[4];               // x0, x1, y0, y1 of the node's padded box, widened by the margin
    float u[3], uc, v[3], vc;
    float R[9], t[3];            // the instance's transform
    float mx[3], my[3], mz[3];   // its frame (trace.h)
    uint32_t root;               // bottom-level root
    uint32_t pad_[14];
};
static_assert(sizeof(PrimaryInst) == 192, "PrimaryInst layout");

constexpr uint32_t VIS_UNKNOWN = 0xFFFFFFFFu;

// One evaluation, as the kernels see it.
struct alignas(64) EvalDesc {
    // scene
    const TriRec *tris;
    const BNode4 *blas;
    const float *mats;       // 2 floats per material
    const WPoint *wpts;
    int64_t n_wpts;
    // articulation slot
    const Inst *inst;
    const BNode4 *tlas;
    const double *xf;        // K x 12
    const double *axw;       // J x 3
    const int32_t *dof_node; // J
    const int32_t *parent;   // K (device copy of the tree)
    uint32_t root_ref;
    int32_t n_nodes, n_mats, n_dof;
    // parameters (basis in FP64 from the host)
    double u[3], v[3], d[3];
    double pressure;
    double ref[3];
    int32_t n, bounces;
    uint32_t flags;
    int32_t tiles_x;        // 16-pixel tile columns
    int32_t ppc;            // patches per chunk
    int32_t grad_n;         // doubles per group gradient partial (0 = no gradient)
    uint32_t *chain;        // adjoint: the pixels' hit chains, n_patches x (bounces + 1) x 64 words, or null
    int64_t n_groups;       // adjoint: gradient groups
    int64_t patch_base;     // first patch of this evaluation (partial sums are per patch)
    int64_t n_patches;      // 4 * tiles_x * tiles_y (of a piece: the patch after its last)
    int32_t tiles_y;        // 16-pixel tile rows
    int32_t n_diffuse;      // diffuse rays per emitting hit (0 = none)
    // optional outputs
    int32_t *hit_ids;       // N*N*R (R = B+1 + B*n_diffuse) or null
    float *hit_t;
    double *grad_part;      // n_groups x grad_n (gradient partials)
    double *grad_out;       // 3*(2M+J) final gradient or null
    const float *dset;      // n_diffuse > 0: the diffuse set, 4 floats per ray (x, y, z, 0), then its mean
    FanRec *emit;           // n_diffuse > 0, forward: emitter records, n_patches x bounces x 64, then as
                            // many bytes: the planar instance each record's rays leave, or -1
    uint64_t *emit_mask;    // which of them are filled: n_patches x bounces masks of 64 lanes
    int32_t n_slices;       // reduction: contiguous ranges summed by separate blocks (1..MAX_SLICES)
    int64_t fan_base;       // first fan partial slot (n_patches x bounces x ceil(n_diffuse / FAN_SLICE))
    double *gslice;         // gradient: n_slices x grad_n range sums
    SliceOut *pslice;       // n_slices range sums of the patch (and fan) partials
    int64_t slice_base;     // the batch's number of this evaluation's first range sum
    int32_t n_clamped;      // hinge angles of this evaluation clamped to their intervals
    float box_pad;          // padding of the hierarchies' boxes (metres)
    uint64_t planar[2];     // bit k: every triangle of node k lies in one plane (rays leaving it skip it)
    // primary hits by k_primary (null: the trace kernel traces the primary rays)
    uint2 *vis;             // n_patches x 64: distance bits, leaf-order triangle (where the mask is set), or
                            // VIS_UNKNOWN for the triangle: the trace kernel traces the primary ray
    uint64_t *vis_mask;     // n_patches: the patch's pixels that hit, or that are not known to miss
    const int32_t *leaf_of; // T: leaf-order index of an original triangle index
    const ArtNode *art;     // K tree nodes
    PrimaryEval *prim;      // the image of this evaluation's instances: a PrimaryEval, then K PrimaryInst
    int32_t group;          // patches per gradient group
    int32_t patch0;         // first patch: 0, or that of a piece of an evaluation whose hit chains do not
                            // fit at once (whole groups; chain, grad_part and n_groups are then the piece's)
};

// The host writes these records and the kernels read them: both compilation
// passes (host and gfx950) must agree on every offset.
static_assert(sizeof(EvalDesc) == 448, "EvalDesc layout");
static_assert(offsetof(EvalDesc, tris) == 0, "EvalDesc layout");
static_assert(offsetof(EvalDesc, blas) == 8, "EvalDesc layout");
static_assert(offsetof(EvalDesc, mats) == 16, "EvalDesc layout");
static_assert(offsetof(EvalDesc, wpts) == 24, "EvalDesc layout");
static_assert(offsetof(EvalDesc, n_wpts) == 32, "EvalDesc layout");
static_assert(offsetof(EvalDesc, inst) == 40, "EvalDesc layout");
static_assert(offsetof(EvalDesc, tlas) == 48, "EvalDesc layout");
static_assert(offsetof(EvalDesc, xf) == 56, "EvalDesc layout");
static_assert(offsetof(EvalDesc, axw) == 64, "EvalDesc layout");
static_assert(offsetof(EvalDesc, dof_node) == 72, "EvalDesc layout");
static_assert(offsetof(EvalDesc, parent) == 80, "EvalDesc layout");
static_assert(offsetof(EvalDesc, root_ref) == 88, "EvalDesc layout");
static_assert(offsetof(EvalDesc, n_nodes) == 92, "EvalDesc layout");
static_assert(offsetof(EvalDesc, n_mats) == 96, "EvalDesc layout");
static_assert(offsetof(EvalDesc, n_dof) == 100, "EvalDesc layout");
static_assert(offsetof(EvalDesc, u) == 104, "EvalDesc layout");
static_assert(offsetof(EvalDesc, v) == 128, "EvalDesc layout");
static_assert(offsetof(EvalDesc, d) == 152, "EvalDesc layout");
static_assert(offsetof(EvalDesc, pressure) == 176, "EvalDesc layout");
static_assert(offsetof(EvalDesc, ref) == 184, "EvalDesc layout");
static_assert(offsetof(EvalDesc, n) == 208, "EvalDesc layout");
static_assert(offsetof(EvalDesc, bounces) == 212, "EvalDesc layout");
static_assert(offsetof(EvalDesc, flags) == 216, "EvalDesc layout");
static_assert(offsetof(EvalDesc, tiles_x) == 220, "EvalDesc layout");
static_assert(offsetof(EvalDesc, ppc) == 224, "EvalDesc layout");
static_assert(offsetof(EvalDesc, grad_n) == 228, "EvalDesc layout");
static_assert(offsetof(EvalDesc, chain) == 232, "EvalDesc layout");
static_assert(offsetof(EvalDesc, n_groups) == 240, "EvalDesc layout");
static_assert(offsetof(EvalDesc, patch_base) == 248, "EvalDesc layout");
static_assert(offsetof(EvalDesc, n_patches) == 256, "EvalDesc layout");
static_assert(offsetof(EvalDesc, tiles_y) == 264, "EvalDesc layout");
static_assert(offsetof(EvalDesc, n_diffuse) == 268, "EvalDesc layout");
static_assert(offsetof(EvalDesc, hit_ids) == 272, "EvalDesc layout");
static_assert(offsetof(EvalDesc, hit_t) == 280, "EvalDesc layout");
static_assert(offsetof(EvalDesc, grad_part) == 288, "EvalDesc layout");
static_assert(offsetof(EvalDesc, grad_out) == 296, "EvalDesc layout");
static_assert(offsetof(EvalDesc, dset) == 304, "EvalDesc layout");
static_assert(offsetof(EvalDesc, emit) == 312, "EvalDesc layout");
static_assert(offsetof(EvalDesc, emit_mask) == 320, "EvalDesc layout");
static_assert(offsetof(EvalDesc, n_slices) == 328, "EvalDesc layout");
static_assert(offsetof(EvalDesc, fan_base) == 336, "EvalDesc layout");
static_assert(offsetof(EvalDesc, gslice) == 344, "EvalDesc layout");
static_assert(offsetof(EvalDesc, pslice) == 352, "EvalDesc layout");
static_assert(offsetof(EvalDesc, slice_base) == 360, "EvalDesc layout");
static_assert(offsetof(EvalDesc, n_clamped) == 368, "EvalDesc layout");
static_assert(offsetof(EvalDesc, planar) == 376, "EvalDesc layout");
static_assert(offsetof(EvalDesc, vis) == 392, "EvalDesc layout");
static_assert(offsetof(EvalDesc, leaf_of) == 408, "EvalDesc layout");
static_assert(offsetof(EvalDesc, patch0) == 436, "EvalDesc layout");
static_assert(sizeof(EvalDesc) == 448, "EvalDesc layout");
static_assert(sizeof(PatchOut) == 64, "PatchOut layout");
static_assert(offsetof(PatchOut, f) == 0, "PatchOut layout");
static_assert(offsetof(PatchOut, hits) == 48, "PatchOut layout");
static_assert(offsetof(PatchOut, flags) == 60, "PatchOut layout");
static_assert(sizeof(WPoint) == 32, "WPoint layout");
static_assert(offsetof(WPoint, node) == 24, "WPoint layout");
static_assert(offsetof(Inst, t) == 36, "Inst layout");
static_assert(offsetof(Inst, root) == 48, "Inst layout");
static_assert(offsetof(BNode4, ref) == 96, "BNode4 layout");
static_assert(offsetof(TriRec, id) == 12, "TriRec layout");
static_assert(offsetof(TriRec, mat) == 28, "TriRec layout");
static_assert(offsetof(TriRec, node) == 44, "TriRec layout");

// Order-preserving map of doubles to unsigned 64-bit integers (for
// atomic min/max of the window bounds).
SRP_HD inline uint64_t enc_f64(double x) {
    union { double d; uint64_t u; } c;
    c.d = x;
    return (c.u >> 63) ? ~c.u : (c.u | 0x8000000000000000ull);
}
SRP_HD inline double dec_f64(uint64_t e) {
    union { double d; uint64_t u; } c;
    c.u = (e >> 63) ? (e & 0x7FFFFFFFFFFFFFFFull) : ~e;
    return c.d;
}

// window slots per evaluation: enc(umin), enc(-umax), enc(vmin), enc(-vmax), enc(hmin)
constexpr int WIN_STRIDE = 8;

// Kernel launchers (kernels.hip)
// Work queues of the trace kernel (and, after them, of the fan kernel): N_QUEUES
// counters QUEUE_STRIDE words apart; after both sets, the count of fan units
// the trace kernel listed (FAN_UNITS_AT)
// (launch_window zeroes them).
constexpr int N_QUEUES = 64;      // (one lane per counter when a wave looks at all of them)
constexpr int QUEUE_STRIDE = 8;   // (128-byte spacing measured the same)
constexpr int FAN_UNITS_AT = 2 * N_QUEUES * QUEUE_STRIDE;
constexpr int QUEUE_WORDS = FAN_UNITS_AT + 64;
// The items of queue r: one of every N_QUEUES consecutive ones, a different one at
// every position i, so that a run of positions samples the whole image (a fixed one
// would follow one image column wherever a row of the image holds a multiple of
// N_QUEUES items: 8.1 ms in place of 3.5), and of the rest item r, so that the number of
// positions is plain.  (Exact, for a wave asks every queue that seems to hold
// items: with a position for every queue in the rest, a launch of 4 chunks asked up
// to 60 empty queues one by one, 20 us of a 77 us call.)
SRP_HD inline uint32_t queue_positions(uint32_t total, uint32_t r) { return (total + N_QUEUES - 1 - r) / N_QUEUES; }
SRP_HD inline uint32_t queue_item(uint32_t i, uint32_t r, uint32_t total) {
    const uint32_t skew = i < total / N_QUEUES ? i * 37u : 0u;
    return i * N_QUEUES + ((r + skew) & (N_QUEUES - 1));
}
// The items that one request takes when a queue has `left`: about a fourth of a wave's
// share of them (so that the 32-bit counters do not overflow), one at a time at the
// end; one at a time throughout where an item is long beside a request (`single`: chunks
// that trace the diffuse fans of a craft, of up to 1.7 ms; in runs, 24 images at 400^2 of the
// 8k craft, B = 2, K = 16, took 2,196 us, so 1,924).
SRP_HD inline uint32_t queue_run(uint32_t left, uint32_t blocks, bool single) {
    const uint32_t waves = blocks * (BLOCK / 64) / N_QUEUES;   // of one counter
    const int share = 33 - __builtin_clz(waves > 1u ? waves : 1u);
    const uint32_t n = single ? 0u : left >> share;
    return n > 1u ? n : 1u;
}
// Whether each of `total` items belongs to a wave of its own, and which: the waves
// suffice, and there is a block for every compute unit.  (A smaller launch ends on the
// compute unit that holds most of its long patches, which a queue spreads: the 36
// patches of one 33^2 image of the 50k craft 69 us by queues, 71-75 us so; a batch of eight
// 128^2 images 140 us by queues, 128 so.)  Neighbouring items, and the heaviest ones of an
// ordered launch's evaluations, go to different blocks: the blocks' first waves take the
// first items, their second waves the next ones, from another block on (from the same
// block on, a captured batch of eight 128^2 images of 200k triangles took 240 us, by
// queues 220, so 211).
constexpr uint32_t OWN_ITEM_BLOCKS = 256;   // the MI355X's compute units
SRP_HD inline bool own_items(uint32_t total, uint32_t blocks) {
    return blocks >= OWN_ITEM_BLOCKS && total <= blocks * (BLOCK / 64);
}
SRP_HD inline uint32_t own_item(uint32_t block, uint32_t wave, uint32_t blocks) {
    return wave * blocks + (block + wave * 101u) % blocks;
}
// Copies bytes (a multiple of 16) of pinned host memory to the device by a kernel.
int launch_upload(char *dst, const char *src, size_t bytes, void *stream);
int launch_window(const EvalDesc *d_desc, int n_evals, int blocks_x, uint64_t *d_win, uint32_t *d_queue,
                  void *stream);
// Builds n_jobs articulation slots, one thread each (articulate.hip); the
// window kernel reads them, so it runs first on the same stream.
int launch_articulate(const ArtJob *d_jobs, int n_jobs, void *stream);
// Primary hits of the evaluations whose descriptor has vis, on tiles of tile x
// tile pixels (16 or 8).  d_tile_base: the tiles before each evaluation (none of
// one without vis), n_tiles in all, max_tiles of one evaluation at most.  Runs
// after the window kernel and before the trace kernel (primary.hip).
int launch_primary(const EvalDesc *d_desc, int n_evals, const uint64_t *d_win, int tile, const uint32_t *d_tile_base,
                   uint32_t n_tiles, uint32_t max_tiles, void *stream);
// d_spill: grid_blocks * BLOCK * STACK_SPILL words; chunk counts below 2^31.
// d_fan_out, d_fan_counts (forward, diffuse rays on): the fan pass partial
// slots.  With fans_inline the trace kernel also traces every patch's diffuse
// fans into them (no fan launch follows; long_chunks: its waves take one chunk at
// a time, queue_run); otherwise it lists each patch's
// non-empty passes in d_fan_units (capacity: one entry per pass slot; their
// number at d_queue[FAN_UNITS_AT]) for the fan launch and writes the empty
// passes' zero partials itself.  blocks_per_cu <= 2 (grid_blocks = that times the CU count) launches the
// kernel compiled for 2 waves per SIMD.  d_order, d_cost (such forward
// launches of one patch per chunk, else null; other launches ignore them):
// one word per patch of the batch (at each evaluation's patch_base); chunk c
// of an evaluation traces its patch d_order[c], and d_cost receives every
// patch's trace time (constant-rate clock ticks).
int launch_trace(const EvalDesc *d_desc, const int64_t *d_chunk_base, int n_evals,
                 const uint64_t *d_win, int64_t total_chunks, uint32_t *d_queue, uint32_t *d_spill,
                 PatchOut *d_patches, uint64_t *d_counts, bool count, int grid_blocks, PatchOut *d_fan_out,
                 uint64_t *d_fan_counts, bool fans_inline, bool long_chunks, int4 *d_fan_units, int blocks_per_cu,
                 const uint32_t *d_order, uint32_t *d_cost, void *stream);
// Gradient partials of every group from the chains and hit counts that the
// trace kernel wrote, in blocks of block_waves = max group / GROUP_PART waves.
// d_block_base: the blocks before each evaluation (adjoint_blocks of each),
// n_blocks in all, max_blocks of one evaluation at most.  lds_grad_doubles: the
// largest grad_n.
int launch_adjoint(const EvalDesc *d_desc, int n_evals, const uint32_t *d_block_base, uint32_t n_blocks,
                   uint32_t max_blocks, int block_waves, const PatchOut *d_patches, bool dir, int lds_grad_doubles,
                   void *stream);
SRP_HD inline int64_t adjoint_blocks(int64_t n_groups, int group, int block_waves) {
    return (n_groups * (group / GROUP_PART) + block_waves - 1) / block_waves;
}
// Blocks of such a launch per kernel launch at most (a dispatch counts its
// work-items with 32 bits).
constexpr uint32_t MAX_LAUNCH_BLOCKS = (uint32_t)1 << 22;

// The evaluation that owns block b of a launch numbered through its batch, and its first
// block: base[k] blocks before evaluation k, base[n] > b in all.  per_most: 2^32 over the
// most blocks of one (launch_share), so that no evaluation before b / most can own b:
// evaluations of one size need no search (nor a division, 2 % of the rasteriser on
// 8-pixel tiles).
struct BlockOwner {
    int eval;
    uint32_t first;
};
inline uint32_t launch_share(uint32_t most) { return most > 1 ? (uint32_t)(((uint64_t)1 << 32) / most) : 0xFFFFFFFFu; }
template <class P>
SRP_HD inline BlockOwner block_owner(P base, int n, uint32_t b, uint32_t per_most) {
    int lo = (int)(((uint64_t)b * per_most) >> 32);   // b / most, or one less
    if (lo > n - 1) lo = n - 1;
    uint32_t first = base[lo], next = base[lo + 1];
    if (b >= next && lo < n - 1) {
        first = next;
        next = base[++lo + 1];
    }
    if (b < next) return {lo, first};
    int hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (base[mid] <= b) lo = mid; else hi = mid - 1;
    }
    return {lo, base[lo]};
}
// Diffuse fans of the recorded emitters: one work unit per non-empty fan pass,
// as the trace kernel listed them in d_fan_units (at most max_units); uses the
// second set of queue counters and the same spill area as the trace kernel.
int launch_fans(const EvalDesc *d_desc, const uint64_t *d_win, int64_t max_units, uint32_t *d_queue,
                uint32_t *d_spill, PatchOut *d_fan_out, uint64_t *d_fan_counts, const int4 *d_fan_units, bool count,
                int grid_blocks, void *stream);
// d_slice_eval: the evaluation of each of the batch's total_slices range sums
// (one block each; an evaluation's are consecutive, from its slice_base).
// With d_order and d_cost (as for launch_trace) the second stage also
// rewrites every evaluation's patch order from the costs, heaviest first, for
// the next launches, on every eighth launch as counted in *d_order_launch.
int launch_reduce(const EvalDesc *d_desc, int n_evals, const uint64_t *d_win, const PatchOut *d_patches,
                  const uint64_t *d_counts, const PatchOut *d_fan_out, const uint64_t *d_fan_counts, bool count,
                  bool grad, const uint32_t *d_slice_eval, int64_t total_slices, void *d_out, uint32_t *d_order,
                  const uint32_t *d_cost, uint32_t *d_order_launch, void *stream);
// Resident blocks per compute unit of the trace kernel variant.
int trace_blocks_per_cu(bool count);
// Resident blocks per compute unit of the fan kernel variant.
int fan_blocks_per_cu(bool count);

// Fixed device workspace of the entry point that allocates nothing: a
// file-scope static device array in kernels.hip, NOALLOC_SCRATCH_BYTES per
// GPU, held until the process ends.  noalloc_scratch_init looks up its address
// on the current device (once per device; the library's init calls it);
// noalloc_scratch returns that address (nullptr before the lookup).
constexpr size_t NOALLOC_SCRATCH_BYTES = (size_t)64 << 20;
constexpr int NOALLOC_MAX_DEVICES = 64;
int noalloc_scratch_init();
char *noalloc_scratch(int device);

}  // namespace srp
