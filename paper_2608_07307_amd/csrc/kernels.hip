// gfx950 kernels of the ray-traced SRP library.
//
//   k_window  per evaluation, the tight projected window of the articulated
//             mesh (FP64 bounds of every (vertex, node) point on the image
//             axes u, v and the photon direction d), merged across blocks with
//             order-preserving 64-bit atomic min.
//   k_trace   persistent: every wave takes chunks (runs of 8x8-pixel patches
//             of one evaluation) from 64 work queues until none is left,
//             (or, in a launch of few chunks, its own one) with no block
//             barrier; one ray per lane; primary hits of large
//             images read from k_primary's records; two-level traversal (top level over
//             the kinematic-tree nodes, rigid instance transform, bottom level
//             in rest-pose coordinates) with a per-lane stack (LDS ring, global
//             spill); watertight FP32 triangle test; momentum law at each hit;
//             specular secondary rays iteratively; FP64 per-lane sums, a wave
//             reduction, one partial per patch (no floating-point atomics, so
//             results do not depend on scheduling).  With diffuse rays a chain
//             hit that emits a fan writes an emitter record; for big batches
//             the kernel then traces the patch's fan passes itself.  For the
//             adjoint it also records each pixel's hit chain.
//   k_adjoint per group of patches, differentiates the recorded chains at
//             fixed visibility.
//   k_fans    the patches' fan passes as a separate persistent launch, each
//             patch split into several work units, where the batch is small or
//             its fans are dear (many directions through a large mesh).
//   k_upload  copies a small staging image from pinned memory.
//   k_slices  one block per range sum (up to 16 per evaluation, numbered
//             through the batch), summing a contiguous range of its evaluation's
//             patch, fan-pass and gradient partials in a fixed order.
//   k_reduce  per evaluation, adds the ranges in order, scales by P * A_pix and
//             writes the srp_result (and assembles the gradients).
//   k_sums    k_slices and k_reduce in one, where every evaluation is one range.
//
// The per-pixel structure, the iterative secondary rays and the GPU-side
// reduction follow Sec. 4.3 of the paper; the articulation follows Sec. 4.4.
#include <float.h>

#include <algorithm>

#include "srp.h"
#include "srp_internal.h"
#include "trace.h"

namespace srp {

namespace {

constexpr int WAVE = 64;
constexpr int HWREG_XCC_ID = 20;   // hardware register holding the wave's XCD (accelerator complex die)

// Occupancy targets of the trace kernels (waves per SIMD): the register
// budget the compiler keeps to.
#ifndef SRP_WPE_FWD
#define SRP_WPE_FWD 4
#endif
constexpr size_t GRID_LDS = (BLOCK / 64) * 4 * sizeof(float4);   // the waves' ray grids (k_trace)

// x from another lane of the same 16-lane row (data-parallel primitive move,
// one per 32-bit half).  Every lane of the wave must be active.
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double x) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, 0xF, 0xF, false);
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double readlane_f64(double x, int lane) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), lane),
                            __builtin_amdgcn_readlane(__double2loint(x), lane));
}

// Wave-wide sum and maximum of 32-bit integers, returned to every lane
// (quads, then rows by rotation, then the rows' first lanes).  Every lane of
// the wave must be active.
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xF, 0xF, false);
}
__device__ __forceinline__ uint32_t rows_u32(uint32_t x, int k) {
    return (uint32_t)__builtin_amdgcn_readlane((int)x, k);
}
__device__ __forceinline__ uint32_t wave_add_u32(uint32_t x) {
    x += dpp_u32<0xB1>(x);
    x += dpp_u32<0x4E>(x);
    x += dpp_u32<0x124>(x);
    x += dpp_u32<0x128>(x);
    return rows_u32(x, 0) + rows_u32(x, 16) + rows_u32(x, 32) + rows_u32(x, 48);
}
__device__ __forceinline__ int wave_max_i32(int x) {
    x = max(x, (int)dpp_u32<0xB1>((uint32_t)x));
    x = max(x, (int)dpp_u32<0x4E>((uint32_t)x));
    x = max(x, (int)dpp_u32<0x124>((uint32_t)x));
    x = max(x, (int)dpp_u32<0x128>((uint32_t)x));
    return max(max((int)rows_u32((uint32_t)x, 0), (int)rows_u32((uint32_t)x, 16)),
               max((int)rows_u32((uint32_t)x, 32), (int)rows_u32((uint32_t)x, 48)));
}

// Orders this wave's earlier LDS accesses before its later ones across lanes
// (one wave's LDS operations execute in issue order; this keeps the compiler
// from reordering them).
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// The six sums over the wave's 64 lanes of the lanes' LDS accumulators (lane
// 0's at acc, component k at acc[k * BLOCK + lane]), in a fixed order: quads
// ((0 + 1) + (2 + 3)), the four quads of each 16 lanes ((0 + 3) + (2 + 1)), the
// four of those ((0 + 1) + (2 + 3)).  Eight lanes share a component and add
// eight accumulators each, so lane 8 k (and the seven after it) returns the
// sum of component k: about 30 instructions, against 170 for six butterflies
// over all 64 lanes (with the ray grid in LDS, below: 64 x 1024^2 forward 3.30 -> 3.11 ms,
// with the adjoint 4.26 -> 3.98).  Lanes 48..63 return nothing of use.  Every lane of the
// wave must be active; the accumulators' last writes come first.
__device__ __forceinline__ double wave_sums6(const double *acc, int lane) {
    wave_lds_fence();
    const double2 *p = reinterpret_cast<const double2 *>(acc + min(lane >> 3, 5) * BLOCK + (lane & 7) * 8);
    const double2 a = p[0], b = p[1], c = p[2], d = p[3];
    const double q0 = (a.x + a.y) + (b.x + b.y), q1 = (c.x + c.y) + (d.x + d.y);
    double x = q0 + dpp_f64<0xB1>(q1);   // even lanes: quads 0 + 3, odd ones: 2 + 1 (quad_perm (1, 0, 3, 2))
    x += dpp_f64<0xB1>(x);
    x += dpp_f64<0x4E>(x);               // (quad_perm (2, 3, 0, 1))
    x += dpp_f64<0x141>(x);              // the other quad of the eight lanes (row_half_mirror)
    return x;
}

// The sum of x over the wave's 64 lanes, returned to every lane, in the same
// order as wave_sums6.  Every lane of the wave must be active.
__device__ __forceinline__ double wave_sum(double x) {
    x += dpp_f64<0xB1>(x);    // quad_perm (1, 0, 3, 2)
    x += dpp_f64<0x4E>(x);    // quad_perm (2, 3, 0, 1)
    x += dpp_f64<0x124>(x);   // row_ror 4
    x += dpp_f64<0x128>(x);   // row_ror 8
    return (readlane_f64(x, 0) + readlane_f64(x, 16)) + (readlane_f64(x, 32) + readlane_f64(x, 48));
}

// The adjoint's record of a pixel's chain is one word per hit: the triangle's
// leaf-order index (below 2^27), with the top bit set when the geometric normal
// was flipped to face the incoming ray; CHAIN_END after the last hit when it
// is not the longest possible chain.  The sweep recomputes the normals from it
// bit for bit and recovers each incoming direction and weight backwards from
// the last ones (a mirror reflection is its own inverse).
constexpr uint32_t CHAIN_END = 0xFFFFFFFFu;
constexpr uint32_t CHAIN_FLIP = 0x80000000u;

// *p += v as one LDS add, for accumulators that only this wave adds to (its
// adds execute in program order)
__device__ __forceinline__ void lds_add(double *p, double v) {
    (void)__hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// x from the row pairs' and the half-waves' partners, added: rows 0 + 1 and 2 + 3,
// then both (permlane swaps: of two copies of x, the first ends with rows 0, 0,
// 2, 2 and the second with rows 1, 1, 3, 3; halves likewise).
__device__ __forceinline__ float add_rows_f32(float x) {
    const uint32_t u = __float_as_uint(x);
    const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    const uint32_t h = __float_as_uint(__uint_as_float(r[0]) + __uint_as_float(r[1]));
    const auto q = __builtin_amdgcn_permlane32_swap(h, h, false, false);
    return __uint_as_float(q[0]) + __uint_as_float(q[1]);
}
template <int CTRL>
__device__ __forceinline__ float dpp_f32(float x) {
    return __uint_as_float(dpp_u32<CTRL>(__float_as_uint(x)));
}

// Adds per-lane vectors of N values into per-wave FP64 LDS accumulators
// acc[key * stride + 0..N), one wave-wide sum per distinct key (keys processed
// lowest lane first).  The wave sum of the (at most 64) FP32 terms is taken in
// FP32 (relative rounding below 64 ulp of FP32, far under the adjoint's 1e-4
// tolerance), the accumulation across a chunk's patches in FP64.  The sums of
// four values share their first two steps: a lane hands the half it does not
// keep to its neighbour, so lane j of a quad ends with values j, 4 + j, ...; about
// 65 instructions for 9 values, against 170 for 9 butterflies with the same order
// of additions (quads, the four quads of a row, the rows); adjoint batch 64 x
// 1024^2: 3.39 -> 3.23 ms, 1M triangles 2.80 -> 2.59.
template <int N>
__device__ __forceinline__ void wave_scatter_add(double *acc, int key, bool active, const float *vals, int stride) {
    constexpr int P = (N + 3) / 4;
    const int lane = threadIdx.x & (WAVE - 1);
    const bool odd = lane & 1, high = lane & 2;
    uint64_t pending = __ballot(active);
    while (pending) {
        const int leader = __ffsll((unsigned long long)pending) - 1;
        const int k = __builtin_amdgcn_readlane(key, leader);
        const bool sel = active && key == k;
        pending &= ~__ballot(sel);
        float b[P];
#pragma unroll
        for (int p = 0; p < P; ++p) {
            float v[4], a[2];
            for (int c = 0; c < 4; ++c) v[c] = (4 * p + c < N && sel) ? vals[4 * p + c < N ? 4 * p + c : 0] : 0.0f;
            for (int h = 0; h < 2; ++h)
                a[h] = (odd ? v[2 * h + 1] : v[2 * h]) + dpp_f32<0xB1>(odd ? v[2 * h] : v[2 * h + 1]);
            b[p] = (high ? a[1] : a[0]) + dpp_f32<0x4E>(high ? a[0] : a[1]);
            b[p] += dpp_f32<0x124>(b[p]);
            b[p] += dpp_f32<0x128>(b[p]);
            b[p] = add_rows_f32(b[p]);
        }
        if (lane < 4)
#pragma unroll
            for (int p = 0; p < P; ++p)
                if (4 * p + lane < N) lds_add(acc + k * stride + 4 * p + lane, (double)b[p]);
    }
}

// 3x3 helpers (row-major)
__device__ __forceinline__ void m3_zero(float *M) {
#pragma unroll
    for (int i = 0; i < 9; ++i) M[i] = 0.0f;
}

// A wave-uniform float held in a scalar register.
__device__ __forceinline__ float uniform_f32(float x) {
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x)));
}

// Whether every triangle of node k lies in one plane (a ray leaving one of
// them cannot meet the node again, so its traversal skips the node).
__device__ __forceinline__ bool planar_node(const EvalDesc &D, int k) {
    const uint64_t m = k < 64 ? D.planar[0] : D.planar[1];
    return ((m >> (k & 63)) & 1ull) != 0;
}

// The byte per emitter record that follows an evaluation's records: the
// planar instance the record's diffuse rays leave, or -1.
__device__ __forceinline__ int8_t SRP_GLOBAL *emit_skip(const EvalDesc &D) {
    return (int8_t SRP_GLOBAL *)(D.emit + (size_t)D.n_patches * D.bounces * WAVE);
}

// Hit record -> unit normal n facing the incoming direction d, c = -n.d, the
// material's (rho_s, rho_d) and the original triangle index; returns whether
// the geometric normal was flipped.
__device__ __forceinline__ bool hit_normal(const TraceCtx &TC, const EvalDesc &D, const Hit &h, const float d[3],
                                           float n[3], float &c, float &rs, float &rd, int32_t &id) {
    // the instance's rotation does not depend on the triangle: read it first
    const Inst SRP_GLOBAL &I = TC.inst[h.inst];
    const float4 Ra = *(const float4 SRP_GLOBAL *)&I.R[0], Rb = *(const float4 SRP_GLOBAL *)&I.R[4];
    const float R8 = I.R[8];
    const float IR[9] = {Ra.x, Ra.y, Ra.z, Ra.w, Rb.x, Rb.y, Rb.z, Rb.w, R8};
    const TriRec SRP_GLOBAL &T = TC.tris[h.tri];
    float e1[3] = {T.v1[0] - T.v0[0], T.v1[1] - T.v0[1], T.v1[2] - T.v0[2]};
    float e2[3] = {T.v2[0] - T.v0[0], T.v2[1] - T.v0[1], T.v2[2] - T.v0[2]};
    float nl[3] = {e1[1] * e2[2] - e1[2] * e2[1], e1[2] * e2[0] - e1[0] * e2[2], e1[0] * e2[1] - e1[1] * e2[0]};
    for (int k = 0; k < 3; ++k) n[k] = IR[3 * k] * nl[0] + IR[3 * k + 1] * nl[1] + IR[3 * k + 2] * nl[2];
    float inv = rsqrtf(n[0] * n[0] + n[1] * n[1] + n[2] * n[2]);
    const float nd = (n[0] * d[0] + n[1] * d[1] + n[2] * d[2]) * inv;
    const bool flip = nd > 0.0f;
    if (flip) inv = -inv;
    for (int k = 0; k < 3; ++k) n[k] *= inv;
    c = -(n[0] * d[0] + n[1] * d[1] + n[2] * d[2]);
    const float SRP_GLOBAL *mats = (const float SRP_GLOBAL *)D.mats;
    rs = mats[2 * T.mat];
    rd = mats[2 * T.mat + 1];
    id = T.id;
    return flip;
}

// The first hits' words of a lane's recorded chain (of B + 1 at most), read
// together; later ones stay in memory.
struct ChainWords {
    uint32_t w0, w1, w2;
    __device__ __forceinline__ uint32_t at(const uint32_t SRP_GLOBAL *chain, int k) const {
        return k == 0 ? w0 : k == 1 ? w1 : k == 2 ? w2 : chain[k * WAVE];
    }
};
__device__ __forceinline__ ChainWords chain_words(const uint32_t SRP_GLOBAL *chain, int B) {
    return {chain[0], chain[min(1, B) * WAVE], chain[min(2, B) * WAVE]};
}

// A recorded chain hit: its normal bit for bit as hit_normal formed it, its
// material and node.  The triangle's record in one round trip, then its
// instance's rotation and its material together.
struct ChainHit {
    float n[3], rs, rd;
    int node, mat;
};
__device__ __forceinline__ ChainHit chain_hit(const TraceCtx &TC, const EvalDesc &D, uint32_t ew) {
    ChainHit C;
    const float4 SRP_GLOBAL *tq = (const float4 SRP_GLOBAL *)(TC.tris + (ew & ~CHAIN_FLIP));
    const float4 T0 = tq[0], T1 = tq[1], T2 = tq[2];
    C.node = f2i(T2.w);
    C.mat = f2i(T1.w);
    const Inst SRP_GLOBAL &I = TC.inst[C.node];
    const float4 Ra = *(const float4 SRP_GLOBAL *)&I.R[0], Rb = *(const float4 SRP_GLOBAL *)&I.R[4];
    const float R8 = I.R[8];
    const float2 rm = ((const float2 SRP_GLOBAL *)D.mats)[C.mat];
    const float IR[9] = {Ra.x, Ra.y, Ra.z, Ra.w, Rb.x, Rb.y, Rb.z, Rb.w, R8};
    const float e1[3] = {T1.x - T0.x, T1.y - T0.y, T1.z - T0.z};
    const float e2[3] = {T2.x - T0.x, T2.y - T0.y, T2.z - T0.z};
    const float nl[3] = {e1[1] * e2[2] - e1[2] * e2[1], e1[2] * e2[0] - e1[0] * e2[2], e1[0] * e2[1] - e1[1] * e2[0]};
    for (int i = 0; i < 3; ++i) C.n[i] = IR[3 * i] * nl[0] + IR[3 * i + 1] * nl[1] + IR[3 * i + 2] * nl[2];
    float inv = rsqrtf(C.n[0] * C.n[0] + C.n[1] * C.n[1] + C.n[2] * C.n[2]);
    if (ew & CHAIN_FLIP) inv = -inv;
    for (int i = 0; i < 3; ++i) C.n[i] *= inv;
    C.rs = rm.x;
    C.rd = rm.y;
    return C;
}

// Adds force f at point x (and its torque about ref) to the lane's FP64 sums.
__device__ __forceinline__ void deposit(double *lacc, const float f[3], const float x[3], const double ref[3]) {
    float rr[3];
    for (int k = 0; k < 3; ++k) rr[k] = x[k] - (float)ref[k];
    lds_add(lacc, (double)f[0]);
    lds_add(lacc + BLOCK, (double)f[1]);
    lds_add(lacc + 2 * BLOCK, (double)f[2]);
    lds_add(lacc + 3 * BLOCK, (double)(rr[1] * f[2] - rr[2] * f[1]));
    lds_add(lacc + 4 * BLOCK, (double)(rr[2] * f[0] - rr[0] * f[2]));
    lds_add(lacc + 5 * BLOCK, (double)(rr[0] * f[1] - rr[1] * f[0]));
}

// Tangent frame of a diffuse fan about unit normal n: t = normalize(h x n)
// with the fixed helper h = (1, 2, 3) (e_x when h x n vanishes), b = n x t.
// A generic helper keeps the frame smooth for every normal but +-h.
__device__ __forceinline__ void fan_frame(const float n[3], float t[3], float b[3]) {
    float c0 = 2.0f * n[2] - 3.0f * n[1], c1 = 3.0f * n[0] - n[2], c2 = n[1] - 2.0f * n[0];
    float l2 = c0 * c0 + c1 * c1 + c2 * c2;
    if (!(l2 > 0.0f)) {
        c0 = 0.0f;
        c1 = -n[2];
        c2 = n[1];
        l2 = c1 * c1 + c2 * c2;
    }
    const float il = rsqrtf(l2);
    t[0] = c0 * il;
    t[1] = c1 * il;
    t[2] = c2 * il;
    b[0] = n[1] * t[2] - n[2] * t[1];
    b[1] = n[2] * t[0] - n[0] * t[2];
    b[2] = n[0] * t[1] - n[1] * t[0];
}

// World direction of the fan ray with local direction l about normal n.
__device__ __forceinline__ void fan_dir(const float n[3], const float4 l, float d[3]) {
    float t[3], b[3];
    fan_frame(n, t, b);
    for (int k = 0; k < 3; ++k) d[k] = l.x * t[k] + l.y * b[k] + l.z * n[k];
}

// The work queues of a persistent launch, as one wave sees them: N_QUEUES
// counters, N_QUEUES / 8 of them per XCD.  What bounds a counter is the rate of
// atomics on one address, about 90 ns each: with one counter per XCD and one
// atomic (and one load) per chunk, 64 evaluations at 1024^2 spent 3.0 ms of the
// forward trace kernel's 4.2 ms on 262,144 requests.  So a wave shares its
// counter with 64 waves of the batch grid instead of 512, takes a run of
// remaining / (4 waves of the counter) items per atomic while much is left and
// single ones at the end, and looks at all counters in one load when its own
// is drained.  Measured on one box (forward batch of 64 at 1024^2, 50k
// triangles, B = 2): 4.45 -> 3.29 ms; 1,024 box-wing evaluations at 128^2: 0.95 ->
// 0.59 ms; runs half, a quarter and an eighth as long changed nothing more.
// (Item numbers stay below 2^31 and are 32-bit here: the scalar unit has no
// 64-bit order compare, and 64-bit ones cost the batch kernels 14 spilled
// registers and 6 % of the forward launch.)
// A trace launch of one item per wave at most asks no counter (own_items): 32 waves of
// each counter took 10 us of a launch over 2,048 patches of the box-wing (28 us, now 18).
struct WorkQueue {
    uint32_t r;          // the queue (N_QUEUES: none, the wave has item `at` only)
    uint32_t at, seen;   // its next position of this wave; its counter as last known (the run's end)
};
constexpr uint32_t NO_ITEM = 0xFFFFFFFFu;

__device__ __forceinline__ uint32_t uniform_u32(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)x);
}

__device__ __forceinline__ WorkQueue work_queue(int wv) {
    const uint32_t xcd = __builtin_amdgcn_s_getreg((HWREG_XCC_ID << 0) | (0 << 6) | (3 << 11)) & 7u;
    WorkQueue q;
    q.r = uniform_u32(xcd | ((((blockIdx.x >> 3) * (BLOCK / WAVE) + (uint32_t)wv) & (N_QUEUES / 8 - 1)) << 3));
    q.at = q.seen = 0;
    return q;
}

// The same for a launch of `total` items, each of them its wave's own where own_items says so.
__device__ __forceinline__ WorkQueue work_queue(int wv, uint32_t total, int grid_blocks) {
    WorkQueue q = work_queue(wv);
    if (own_items(total, (uint32_t)grid_blocks)) {
        q.r = N_QUEUES;
        q.at = uniform_u32(own_item(blockIdx.x, (uint32_t)wv, (uint32_t)grid_blocks));
    }
    return q;
}

// The next of `total` work items, or NO_ITEM once every queue is drained.
// Lane 0 talks to the queue's counter and broadcasts, so the result is
// wave-uniform.
__device__ __forceinline__ uint32_t take_work(WorkQueue &q, uint32_t *counters, uint32_t total, int grid_blocks,
                                              bool single, int lane) {
    if (q.r == N_QUEUES) {
        const uint32_t c = q.at < total ? q.at : NO_ITEM;
        q.at = NO_ITEM;
        return c;
    }
    #pragma unroll 1
    for (;;) {
        const uint32_t n_r = queue_positions(total, q.r);
        if (q.at < q.seen && q.at < n_r) return queue_item(q.at++, q.r, total);
        if (q.seen < n_r) {
            const uint32_t n = queue_run(n_r - q.seen, (uint32_t)grid_blocks, single);
            uint32_t v = 0;
            if (lane == 0) v = atomicAdd(counters + q.r * QUEUE_STRIDE, n);
            q.at = uniform_u32(v);
            q.seen = q.at + n;
            continue;
        }
        // drained: look at every queue's counter at once, one per lane
        const uint32_t c = __hip_atomic_load(counters + lane * QUEUE_STRIDE, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint32_t have = queue_positions(total, (uint32_t)lane), left = c < have ? have - c : 0u;
        const uint32_t most = (uint32_t)wave_max_i32((int)left);
        if (most == 0) return NO_ITEM;
        // one of those with at least half as much left as the fullest, every wave from
        // another start: with the next open one after r, all waves whose queues were
        // drained met at the same counter, 90 ns each (one evaluation of a 5,120-triangle
        // sphere at 776^2: k_trace 143 to 220 us by the order of its patches, now 142 to 180;
        // 64 x 1024^2 of the 50k craft, B = 2, 2,784 -> 2,723 for the call)
        const uint64_t full = __ballot(left > 0 && 2 * left >= most);
        const uint32_t from = ((blockIdx.x * (BLOCK / WAVE) + (threadIdx.x >> 6)) * 11u + q.r * 5u + 1u) & (N_QUEUES - 1);
        const uint64_t above = full & (~0ull << uniform_u32(from));
        q.r = (uint32_t)(__ffsll((unsigned long long)(above ? above : full)) - 1);
        q.at = q.seen = (uint32_t)__builtin_amdgcn_readlane((int)c, (int)q.r);
    }
}

// Writes a wave's partial sums: the sum of component k from lane 8 k.
__device__ __forceinline__ void store_partial(PatchOut *out, double tot, uint32_t hits, uint32_t sec, uint32_t sec_hits,
                                              uint32_t flags, int lane) {
    PatchOut SRP_GLOBAL *o = (PatchOut SRP_GLOBAL *)out;
    if ((lane & 7) == 0 && lane < 48) o->f[lane >> 3] = tot;
    if (lane == 48) *(uint4 SRP_GLOBAL *)&o->hits = make_uint4(hits, sec, sec_hits, flags);
}

// Position of the (j+1)-th set bit of m (j < popcount(m)).
__device__ __forceinline__ int nth_set_bit(uint64_t m, int j) {
    int pos = 0;
    #pragma unroll
    for (int w = 32; w >= 1; w >>= 1) {
        const uint64_t low = m & ((1ull << w) - 1ull);
        const int c = __popcll(low);
        if (j >= c) {
            j -= c;
            m >>= w;
            pos += w;
        } else {
            m = low;
        }
    }
    return pos;
}

// The diffuse fans of one patch's recorded emitters.  The patch's fan work is
// split into tasks (emitter, slice of FAN_SLICE consecutive fan-ray indices),
// slice-major, packed 64 to a pass, so lanes idle only in the patch's last
// pass.  Every pass writes its own partial sums (force, torque, diffuse rays
// and hits) to its slot of the patch's B * ceil(K / FAN_SLICE) slots (passes
// past the patch's tasks write zeros), so the result depends neither on the
// schedule nor on which kernel, or how many work units, traced the passes.
// This call traces passes pass0, pass0 + step, ...; m[g] = the patch's
// emitters of generation g (bit = lane of the trace kernel's patch).
template <bool COUNT>
__device__ __forceinline__ void fan_passes(const EvalDesc &D, const TraceCtx &TC, int64_t p, uint64_t m0, uint64_t m1,
                                           uint64_t m2, uint64_t m3, int pass0, int step, float tmin2,
                                           LaneStack &stack, double *lacc, int lane, PatchOut *fan_out,
                                           uint64_t *fan_counts) {
    const int KD = D.n_diffuse, B = D.bounces, N = D.n;
    const int S = (KD + FAN_SLICE - 1) / FAN_SLICE;
    const int PM = B * S;               // pass slots per patch
    const int R = B + 1 + B * KD;
    const float4 SRP_GLOBAL *dset = (const float4 SRP_GLOBAL *)D.dset;
    // emitters packed in generation-then-lane order
    const int c0 = __popcll(m0), c1 = c0 + __popcll(m1), c2 = c1 + __popcll(m2), total = c2 + __popcll(m3);
    const int tasks = total * S;
    const int tile = (int)(p >> 2), q = (int)(p & 3);
    #pragma unroll 1
    for (int pass = pass0; pass < PM; pass += step) {
        const int64_t slot_out = D.fan_base + p * PM + pass;
        uint32_t rays = 0, hits = 0, nbox = 0, ntri = 0, status = 0;
        double tot = 0.0;   // lane 8 k: component k
        if (pass * WAVE < tasks) {
            for (int k = 0; k < 6; ++k) lacc[k * BLOCK] = 0.0;
            const int t = pass * WAVE + lane;
            if (t < tasks) {
                const int sl = t / total;
                const int j = t - sl * total;
                const int k0 = sl * FAN_SLICE, k1 = min(k0 + FAN_SLICE, KD);
                const int g = j >= c0 ? (j >= c1 ? (j >= c2 ? 3 : 2) : 1) : 0;
                const uint64_t mg = g == 0 ? m0 : g == 1 ? m1 : g == 2 ? m2 : m3;
                const int base = g == 0 ? 0 : g == 1 ? c0 : g == 2 ? c1 : c2;
                const int bl = nth_set_bit(mg, j - base);   // the emitting lane of the trace kernel's patch
                const float4 SRP_GLOBAL *er =
                    (const float4 SRP_GLOBAL *)(D.emit + ((size_t)(p * B + g) * WAVE + bl));
                const float4 ea = er[0], eb = er[1];
                const int32_t skip = emit_skip(D)[(size_t)(p * B + g) * WAVE + bl];
                const float x[3] = {ea.x, ea.y, ea.z}, n[3] = {eb.x, eb.y, eb.z};
                const float wd = ea.w;
                const int32_t excl = __float_as_int(eb.w);
                const int px = (tile % D.tiles_x) * TILE + (q & 1) * PATCH + (bl & 7);
                const int py = (tile / D.tiles_x) * TILE + (q >> 1) * PATCH + (bl >> 3);
                const int64_t pix = (int64_t)py * N + px;
                #pragma unroll 1
                for (int k = k0; k < k1; ++k) {
                    float d[3];
                    fan_dir(n, dset[k], d);
                    Hit h;
                    if (!trace_closest<COUNT>(TC, x, d, tmin2, excl, skip, stack, h, nbox, ntri)) {
                        status |= SRP_STATUS_STACK;
                        break;
                    }
                    ++rays;
                    if (D.hit_ids) {
                        const int64_t slot = pix * R + (B + 1 + g * KD + k);
                        ((int32_t SRP_GLOBAL *)D.hit_ids)[slot] = h.tri >= 0 ? h.id : -1;
                        ((float SRP_GLOBAL *)D.hit_t)[slot] = h.tri >= 0 ? h.t : 0.0f;
                    }
                    if (h.tri >= 0) {
                        ++hits;
                        float nh[3], ch, rs, rd;
                        int32_t id;
                        hit_normal(TC, D, h, d, nh, ch, rs, rd, id);
                        const float a = wd * (1.0f - rs), bb = -2.0f * wd * (rs * ch + rd * (1.0f / 3.0f));
                        float f[3], y[3];
                        for (int i = 0; i < 3; ++i) {
                            f[i] = a * d[i] + bb * nh[i];
                            y[i] = fmaf(h.t, d[i], x[i]);
                        }
                        deposit(lacc, f, y, D.ref);
                    }
                }
            }
            tot = wave_sums6(lacc - lane, lane);
            rays = wave_add_u32(rays);
            hits = wave_add_u32(hits);
            status = __ballot(status != 0) ? SRP_STATUS_STACK : 0u;
            if (COUNT) {
                nbox = wave_add_u32(nbox);
                ntri = wave_add_u32(ntri);
            }
        }
        store_partial(fan_out + slot_out, tot, 0, rays, hits, status, lane);
        if (lane == 0) {
            if (COUNT) {
                fan_counts[2 * slot_out] = nbox;
                fan_counts[2 * slot_out + 1] = ntri;
            }
        }
    }
}

// WPE = 0: registers for the occupancy targets above (batches); WPE = 2: for
// launches of at most 2 blocks per CU (single evaluations), which lose no
// occupancy by it and keep every value in registers.
template <bool COUNT, int WPE = 0>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(WPE ? WPE : SRP_WPE_FWD))) void k_trace(
    const EvalDesc *__restrict__ descs, const int64_t *__restrict__ chunk_base, int n_evals,
    const uint64_t *__restrict__ win, int grid_blocks, int64_t total_chunks, uint32_t *queue, uint32_t *spill,
    PatchOut *__restrict__ patches, uint64_t *__restrict__ counts, int fans_inline,
    PatchOut *__restrict__ fan_out, uint64_t *__restrict__ fan_counts, int4 *__restrict__ fan_units,
    const uint32_t *__restrict__ order, uint32_t *__restrict__ cost) {
    extern __shared__ char smem[];
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), wv = tid >> 6;
    LaneStack stack;
    stack.ring = reinterpret_cast<uint32_t *>(smem) + tid;   // slot k at [k * BLOCK]
    stack.stride = BLOCK;
    stack.spill = (uint32_t SRP_GLOBAL *)spill + (size_t)blockIdx.x * BLOCK + tid;
    stack.sstride = grid_blocks * BLOCK;
    // per-lane FP64 force/torque sums of the current patch (component k at [k * BLOCK]):
    // kept in LDS and updated with LDS adds, out of the traversal's registers
    double *lacc = reinterpret_cast<double *>(smem + sizeof(uint32_t) * STACK_LDS * BLOCK) + tid;
    // Every wave is persistent on its own and takes chunks from the work queues
    // until all are drained, with no block barrier.  Every queue walks the whole
    // batch in order, so expensive image regions spread over the grid and over
    // time.
    WorkQueue wq = work_queue(wv, (uint32_t)total_chunks, grid_blocks);
    int cur = -1;                          // evaluation of the previous chunk
    uint32_t cur_begin = 0, cur_end = 0;   // its chunk range
    // its ray grid: origin o0, steps su and sv, direction dd (3 floats each, a float4
    // apart) in LDS, read per patch (in registers they were spilled and reloaded)
    float4 *grid = reinterpret_cast<float4 *>(smem + sizeof(uint32_t) * STACK_LDS * BLOCK + sizeof(double) * 6 * BLOCK) +
                   4 * wv;
    float tmin2 = 0.0f;
    bool empty = true;
    #pragma unroll 1
    for (;;) {
        const uint32_t c = take_work(wq, queue, (uint32_t)total_chunks, grid_blocks, fans_inline == 2, lane);
        if (c == NO_ITEM) break;

        if (c < cur_begin || c >= cur_end) {
            // evaluation owning chunk c (chunk_base is increasing; chunk_base[n_evals] = total)
            int lo = (cur >= 0 && c >= cur_end) ? cur : 0, hi = n_evals - 1;
            while (lo < hi) {
                int mid = (lo + hi + 1) >> 1;
                if ((uint32_t)chunk_base[mid] <= c) lo = mid; else hi = mid - 1;
            }
            cur = lo;
            cur_begin = (uint32_t)chunk_base[lo];
            cur_end = (uint32_t)chunk_base[lo + 1];
            const EvalDesc &D = descs[lo];
            // window -> ray grid (FP64 -> FP32 constants)
            const RayGrid G = ray_grid(D, win + (size_t)lo * WIN_STRIDE);
            if (lane == 0) {
                grid[0] = make_float4(G.o0[0], G.o0[1], G.o0[2], 0.0f);
                grid[1] = make_float4(G.su[0], G.su[1], G.su[2], 0.0f);
                grid[2] = make_float4(G.sv[0], G.sv[1], G.sv[2], 0.0f);
                grid[3] = make_float4(G.dd[0], G.dd[1], G.dd[2], 0.0f);
            }
            wave_lds_fence();
            tmin2 = uniform_f32(G.tmin2);
            empty = __builtin_amdgcn_readfirstlane((int)G.empty) != 0;
        }
        const EvalDesc &D = descs[cur];
        const int64_t kc = c - cur_begin;
        const int N = D.n;

        int64_t p0 = D.patch0 + kc * D.ppc, p1 = min(p0 + D.ppc, D.n_patches);
        // (patch order and costs: only in the 2-wave build, which the ordered
        // launches use, so the batch builds keep their registers)
        constexpr bool ORDERED = WPE == 2;
        if (ORDERED && order) {
            // a captured forward plan of one patch per chunk hands out its patches
            // heaviest first, in the order its previous launch measured; any order
            // gives the same result, since every patch writes its own partial slot
            p0 = ((const uint32_t SRP_GLOBAL *)order)[D.patch_base + kc];
            p1 = p0 < D.n_patches ? p0 + 1 : p0;
        }
        const int B = D.bounces;
        const int KD = D.n_diffuse;                     // diffuse rays per emitting hit
        const int R = B + 1 + B * KD;                   // recorded rays per pixel
        const float4 SRP_GLOBAL *dset = (const float4 SRP_GLOBAL *)D.dset;   // KD directions, then their mean
        const TraceCtx TC = trace_ctx(D);

        // Rasterised evaluations: the hit masks of the chunk's patches (lane i: patch
        // p0 + i); patches without a hit get their zero sums here, one per lane,
        // and are not visited (half of a spacecraft's image is empty), unless every
        // ray is to be recorded
        const bool seen = D.vis != nullptr && !((const PrimaryEval SRP_CONST *)D.prim)->traced;
        uint64_t hits = 0, visit = ~0ull;
        if (seen) {
            const int64_t mp = p0 + lane;
            if (mp < p1) hits = ((const uint64_t SRP_GLOBAL *)D.vis_mask)[mp];
            if (KD == 0 && !D.hit_ids) {
                visit = __ballot(hits != 0);
                if (mp < p1 && hits == 0) {
                    const PatchOut none = {};
                    patches[D.patch_base + mp] = none;
                    if (ORDERED && cost) ((uint32_t SRP_GLOBAL *)cost)[D.patch_base + mp] = 0u;
                }
            }
        }

        if (p1 - p0 < 64) visit &= (1ull << (int)(p1 - p0)) - 1ull;   // (p0 < p1 <= p0 + MAX_PPC)
        uint2 next = make_uint2(0, 0);   // the next visited patch's first hits, read one patch ahead
        if (seen && visit)
            next = ((const uint2 SRP_GLOBAL *)D.vis)[(p0 + __ffsll((unsigned long long)visit) - 1) * WAVE + lane];
        #pragma unroll 1
        while (visit) {
            // one 8x8 patch per iteration, one ray per lane; its sums go to the
            // patch's own slot, so the forward result does not depend on the
            // chunking or on which wave runs it
            const int64_t pt = p0 + __ffsll((unsigned long long)visit) - 1;
            visit &= visit - 1;
            const uint2 first = next;
            if (seen && visit)
                next = ((const uint2 SRP_GLOBAL *)D.vis)[(p0 + __ffsll((unsigned long long)visit) - 1) * WAVE + lane];
            const int tile = (int)(pt >> 2), q = (int)(pt & 3);
            const int px = (tile % D.tiles_x) * TILE + (q & 1) * PATCH + (lane & 7);
            const int py = (tile / D.tiles_x) * TILE + (q >> 1) * PATCH + (lane >> 3);
            const uint64_t clock0 = (ORDERED && cost) ? wall_clock64() : 0;
            for (int k = 0; k < 6; ++k) lacc[k * BLOCK] = 0.0;
            // hit counts packed in 10-bit fields (primary hits, specular secondary rays and
            // their hits; a patch sums at most 64 * SRP_MAX_BOUNCES of each), the status
            // separately (the diffuse rays are counted by the fan kernel)
            uint32_t hcnt = 0, nbox = 0, ntri = 0, status = 0;
            uint64_t em[SRP_MAX_BOUNCES] = {};   // the patch's fan emitters per generation
            {
                const bool inside = px < N && py < N;
                const uint64_t hm =
                    (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)hits, (int)(pt - p0)) |
                    (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(hits >> 32), (int)(pt - p0)) << 32;
                const bool valid = seen ? ((hm >> lane) & 1ull) != 0 : !empty && inside;
                const int64_t pix = (int64_t)py * N + px;
                int K = 0;
                const float4 g3 = grid[3];
                float d[3] = {g3.x, g3.y, g3.z}, w = 1.0f;   // the current ray's direction and weight
                uint32_t emitted = 0;                           // generations whose hit emitted a fan
                if (inside && D.hit_ids) {   // rays that are not traced or miss stay "no hit"
                    for (int s = 0; s < R; ++s) {
                        ((int32_t SRP_GLOBAL *)D.hit_ids)[pix * R + s] = -1;
                        ((float SRP_GLOBAL *)D.hit_t)[pix * R + s] = 0.0f;
                    }
                }
                if (valid) {
                    float o[3];
                    const float4 g0 = grid[0], g1 = grid[1], g2 = grid[2];
                    o[0] = fmaf((float)py, g2.x, fmaf((float)px, g1.x, g0.x));
                    o[1] = fmaf((float)py, g2.y, fmaf((float)px, g1.y, g0.y));
                    o[2] = fmaf((float)py, g2.z, fmaf((float)px, g1.z, g0.z));
                    float tmin = 0.0f;
                    int32_t excl = -1, skip = -1;   // the triangle and the planar instance the ray leaves
                    int gen = 0;   // chain generation
                    #pragma unroll 1
                    for (;;) {
                        Hit h;
                        if (seen && gen == 0 && first.y != VIS_UNKNOWN) {
                            h.t = __uint_as_float(first.x);
                            h.tri = (int32_t)first.y;
                            const TriRec SRP_GLOBAL &T = TC.tris[h.tri];
                            h.inst = T.node;
                            h.id = T.id;
                        } else if (!trace_closest<COUNT>(TC, o, d, tmin, excl, skip, stack, h, nbox, ntri)) {
                            status |= SRP_STATUS_STACK;
                            break;
                        }
                        if (D.hit_ids) {
                            ((int32_t SRP_GLOBAL *)D.hit_ids)[pix * R + gen] = h.tri >= 0 ? h.id : -1;
                            ((float SRP_GLOBAL *)D.hit_t)[pix * R + gen] = h.tri >= 0 ? h.t : 0.0f;
                        }
                        if (h.tri < 0) break;
                        hcnt += gen == 0 ? 1u : (1u << 20);
                        float n[3], cth, rs, rd;
                        int32_t id;
                        const bool flip = hit_normal(TC, D, h, d, n, cth, rs, rd, id);
                        const bool emit = KD > 0 && gen < B && rd > 0.0f;
                        const bool spec = gen < B && rs > 0.0f;
                        const float a = w * (1.0f - rs);
                        float f[3], x[3];
                        if (emit) {
                            // the fan's exact mean direction replaces the Lambertian 2/3 n recoil
                            float ft[3], fb[3];
                            fan_frame(n, ft, fb);
                            const float4 m = dset[KD];
                            const float b = -2.0f * w * rs * cth - w * rd * m.z, e = -w * rd;
                            for (int k = 0; k < 3; ++k) f[k] = a * d[k] + b * n[k] + e * (m.x * ft[k] + m.y * fb[k]);
                        } else {
                            const float b = -2.0f * w * (rs * cth + rd * (1.0f / 3.0f));
                            for (int k = 0; k < 3; ++k) f[k] = a * d[k] + b * n[k];
                        }
                        for (int k = 0; k < 3; ++k) x[k] = fmaf(h.t, d[k], o[k]);
                        deposit(lacc, f, x, D.ref);
                        if (emit) {
                            // the fan kernel traces this hit's diffuse rays from its record
                            // (slot gen * 64 + lane of the patch's region)
                            float4 SRP_GLOBAL *er = (float4 SRP_GLOBAL *)(D.emit + ((size_t)(pt * B + gen) * WAVE + lane));
                            er[0] = make_float4(x[0], x[1], x[2], w * rd / (float)KD);
                            er[1] = make_float4(n[0], n[1], n[2], __int_as_float(id));
                            emit_skip(D)[(size_t)(pt * B + gen) * WAVE + lane] =
                                (int8_t)(planar_node(D, h.inst) ? h.inst : -1);
                            emitted |= 1u << gen;
                        }
                        if (D.chain)   // (hit number gen of the chain)
                            ((uint32_t SRP_GLOBAL *)D.chain)[(pt * (B + 1) + gen) * WAVE + lane] =
                                (uint32_t)h.tri | (flip ? CHAIN_FLIP : 0u);
                        K = gen + 1;
                        if (!spec) break;
                        for (int k = 0; k < 3; ++k) {
                            o[k] = x[k];
                            d[k] = fmaf(2.0f * cth, n[k], d[k]);   // the specular direction
                        }
                        w *= rs;
                        tmin = tmin2;
                        excl = id;
                        skip = planar_node(D, h.inst) ? h.inst : -1;
                        ++gen;
                        hcnt += 1u << 10;
                    }
                }
                if (D.chain && K <= B)   // ends the pixel's chain
                    ((uint32_t SRP_GLOBAL *)D.chain)[(pt * (B + 1) + K) * WAVE + lane] = CHAIN_END;
                if (KD > 0) {
                    // which slots of the patch's emitter region hold records, per generation
                    #pragma unroll
                    for (int g = 0; g < SRP_MAX_BOUNCES; ++g) {
                        if (g >= B) break;
                        em[g] = __ballot((emitted >> g) & 1u);
                        if (lane == 0) ((uint64_t SRP_GLOBAL *)D.emit_mask)[(size_t)pt * B + g] = em[g];
                    }
                }
            }

            // the patch's sums; a patch without a hit has zero sums (secondary hits need a primary)
            double tot = 0.0;   // lane 8 k: component k
            if (__ballot((hcnt & 1023u) != 0)) tot = wave_sums6(lacc - lane, lane);
            hcnt = wave_add_u32(hcnt);
            status = __ballot(status != 0) ? SRP_STATUS_STACK : 0u;
            const int64_t t = D.patch_base + pt;
            store_partial(patches + t, tot, hcnt & 1023u, (hcnt >> 10) & 1023u, hcnt >> 20, status, lane);
            if (COUNT) {
                nbox = wave_add_u32(nbox);
                ntri = wave_add_u32(ntri);
                if (lane == 0) {
                    counts[2 * t] = nbox;
                    counts[2 * t + 1] = ntri;
                }
            }
            if (KD > 0 && fans_inline) {
                // the patch's fans right away, from the records its lanes just wrote
                __threadfence_block();
                fan_passes<COUNT>(D, TC, pt, em[0], em[1], em[2], em[3], 0, 1, tmin2, stack, lacc, lane, fan_out,
                                  fan_counts);
            } else if (KD > 0 && fan_units) {
                // a fan launch follows: list the patch's non-empty fan passes as its
                // work units (one pass each), and write the empty passes' zero
                // partials here, as a pass with no task writes them
                const int S = (KD + FAN_SLICE - 1) / FAN_SLICE, PM = B * S;
                int ne = 0;
                for (int g = 0; g < B; ++g) ne += __popcll(em[g]);
                const int np = (ne * S + WAVE - 1) / WAVE;
                uint32_t ubase = 0;
                if (lane == 0 && np > 0) ubase = atomicAdd(queue + FAN_UNITS_AT, (uint32_t)np);
                ubase = (uint32_t)__builtin_amdgcn_readfirstlane((int)ubase);
                for (int l = lane; l < PM; l += WAVE) {
                    if (l < np) {
                        ((int4 SRP_GLOBAL *)fan_units)[ubase + l] = make_int4(cur, (int)pt, l, 0);
                    } else {
                        const int64_t slot = D.fan_base + pt * PM + l;
                        PatchOut co = {};
                        fan_out[slot] = co;
                        if (COUNT) {
                            fan_counts[2 * slot] = 0;
                            fan_counts[2 * slot + 1] = 0;
                        }
                    }
                }
            }
            if (ORDERED && cost && lane == 0) {
                const uint64_t dt = wall_clock64() - clock0;
                ((uint32_t SRP_GLOBAL *)cost)[D.patch_base + pt] = dt < 0xFFFFFFFFull ? (uint32_t)dt : 0xFFFFFFFFu;
            }
        }
    }
}

// The adjoint of the traced hit chains.  One wave per gradient group (a fixed
// run of an evaluation's patches), one lane per pixel: each lane walks its
// chain forward to the last ray, then back at fixed visibility, and the wave
// adds the lanes' terms into its FP64 sums per node and material.  It traces
// nothing, so its groups cost alike, while a launch that traced and
// differentiated a group in one wave ended on a few groups of expensive rays
// (12 % of its wave slots filled over an adjoint batch of the 1M-triangle
// craft, 11 % over eight evaluations at 512^2).  Measured, both in one kernel
// and now: 8 x 2048^2 of 1M triangles 2.62 -> 1.48 ms, the autograd step of 8 x 512^2 1.21 ->
// 0.83, 64 x 1024^2 of 50k (many groups per wave) 3.23 -> 3.29.
// A group of more than GROUP_PART patches is shared by as many waves of the
// block, each summing GROUP_PART of them, and their sums are added in order: a
// wave of 64 patches with hits took 390 us, the whole launch for the 1M-triangle
// craft (393 -> 251 us before the chains' words were read ahead).  A block holds blockDim.x / 64 such parts, one when every
// group is a single part; blocks are numbered through the batch (block_owner), since
// evaluations differ in size: with the largest one's groups x all evaluations, one
// 1024^2 image beside 512 box-wing evaluations at 64^2 took 2.29 ms, now 0.35.
template <bool DIR>
__global__ __launch_bounds__(WAVE * (MAX_PPC / GROUP_PART)) void k_adjoint(
    const EvalDesc *__restrict__ descs, int n_evals, const uint32_t *__restrict__ block_base, uint32_t first_block,
    uint32_t per_most, int block_waves, const PatchOut *__restrict__ patches, int lds_grad_doubles) {
    extern __shared__ char smem[];
    const int lane = threadIdx.x & (WAVE - 1), wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    double *gw = reinterpret_cast<double *>(smem) + (size_t)wv * lds_grad_doubles;
    const uint32_t SRP_CONST *base = (const uint32_t SRP_CONST *)block_base;
    const uint32_t block = first_block + blockIdx.x;
    const BlockOwner own = block_owner(base, n_evals, block, per_most);
    const EvalDesc &D = descs[own.eval];
    const int parts = D.group / GROUP_PART, part = wv % parts;   // (powers of two; parts <= block_waves)
    const int64_t kc = ((int64_t)(block - own.first) * block_waves + wv) / parts;
    const bool mine = kc < D.n_groups;
    for (int i = lane; i < D.grad_n; i += WAVE) gw[i] = 0.0;
    wave_lds_fence();
    const TraceCtx TC = trace_ctx(D);
    const int B = D.bounces, gK = D.n_nodes;
    const int64_t p0 = D.patch0 + kc * D.group + part * GROUP_PART, p1 = min(p0 + GROUP_PART, D.n_patches);
    // the part's patches with hits (lane i looks at patch p0 + i)
    uint64_t visit = __ballot(mine && p0 + lane < p1 &&
                              patches[D.patch_base + max((int64_t)0, min(p0 + lane, D.n_patches - 1))].hits != 0);
    // The first words of a patch's chains, read together and while the patch before
    // is swept (a word past the chain's end is not used): one round trip in place of
    // one per hit took the launch over 64 x 1024^2 at B = 2 from 629 to 572 us, 8 x
    // 2048^2 at B = 1 from 254 to 236.  (Keeping the first two hits as well costs two
    // of seven waves per SIMD: 611 and 284.)
    const auto chain_of_first = [&](uint64_t patches_left) {
        return (const uint32_t SRP_GLOBAL *)D.chain +
               (p0 + __ffsll((unsigned long long)patches_left) - 1) * (B + 1) * WAVE + lane;
    };
    ChainWords next = {};
    if (visit) next = chain_words(chain_of_first(visit), B);
    #pragma unroll 1
    while (visit) {
        const ChainWords cw = next;
        const uint32_t SRP_GLOBAL *chain = chain_of_first(visit);
        visit &= visit - 1;
        if (visit) next = chain_words(chain_of_first(visit), B);
        int K = 0;
        for (; K <= B; ++K)
            if (cw.at(chain, K) == CHAIN_END) break;
        const int Kmax = wave_max_i32(K);
        // the ray after the last hit, as the trace kernel formed it
        float d[3] = {(float)D.d[0], (float)D.d[1], (float)D.d[2]}, w = 1.0f;
        bool cont = false;   // the last chain hit spawned a specular ray
        ChainHit last = {};
        for (int k = 0; k < K; ++k) {
            last = chain_hit(TC, D, cw.at(chain, k));
            const float cth = -(last.n[0] * d[0] + last.n[1] * d[1] + last.n[2] * d[2]);
            cont = k < B && last.rs > 0.0f;
            if (!cont) break;
            for (int i = 0; i < 3; ++i) d[i] = fmaf(2.0f * cth, last.n[i], d[i]);
            w *= last.rs;
        }
        // Reverse sweep over the chain at fixed visibility.
        //   A  = d(sum of later contributions)/d(incoming direction)   (3x3)
        //   Tn = later contributions divided by the weight after this hit
        float A[9], Tn[3] = {0, 0, 0};
        float n0[3] = {0, 0, 0}, c0 = 1.0f;   // the primary hit's normal and cosine (DIR)
        m3_zero(A);
        for (int k = Kmax - 1; k >= 0; --k) {
            const bool act = k < K;
            float Hm[9], gmat[6];
            int node = 0, mat = 0;
            if (act) {
                // hit k's normal exactly as the forward pass computed it
                ChainHit C = last;
                if (k < K - 1) C = chain_hit(TC, D, cw.at(chain, k));
                const int tnode = C.node, tmat = C.mat;
                const float n[3] = {C.n[0], C.n[1], C.n[2]}, rs = C.rs, rd = C.rd;
                // (d, w) hold the ray after hit k when hit k spawned one: undo the
                // reflection and the weight factor to get hit k's incoming ray
                if (k < K - 1 || cont) {
                    const float dn = n[0] * d[0] + n[1] * d[1] + n[2] * d[2];
                    for (int i = 0; i < 3; ++i) d[i] = fmaf(-2.0f * dn, n[i], d[i]);
                    w = w / rs;
                }
                const float cc = -(n[0] * d[0] + n[1] * d[1] + n[2] * d[2]);
                const float sc = rs * cc + rd * (1.0f / 3.0f);
                if (DIR && k == 0) {
                    for (int i = 0; i < 3; ++i) n0[i] = n[i];
                    c0 = cc;
                }
                // material terms
                for (int i = 0; i < 3; ++i) {
                    gmat[i] = w * (-d[i] - 2.0f * cc * n[i] + Tn[i]);
                    gmat[3 + i] = w * (-2.0f / 3.0f) * n[i];
                }
                // G = dF/dn (explicit) + A (2c I - 2 n d^T)
                float G[9];
                for (int i = 0; i < 3; ++i)
                    for (int j = 0; j < 3; ++j) {
                        float e = w * (2.0f * rs * n[i] * d[j] - (i == j ? 2.0f * sc : 0.0f));
                        float an = A[3 * i] * n[0] + A[3 * i + 1] * n[1] + A[3 * i + 2] * n[2];
                        e += 2.0f * cc * A[3 * i + j] - 2.0f * an * d[j];
                        G[3 * i + j] = e;
                    }
                if (k == 0) {
                    // the primary ray keeps its share of the triangle's visible surface,
                    // whose projected area scales with c0 = -n0.d: the whole chain's
                    // contribution S (per unit weight) adds dF/dn0 = -S d^T / c0
                    float S[3];
                    for (int i = 0; i < 3; ++i) S[i] = (1.0f - rs) * d[i] - 2.0f * sc * n[i] + rs * Tn[i];
                    const float ws = w / cc;
                    for (int i = 0; i < 3; ++i)
                        for (int j = 0; j < 3; ++j) G[3 * i + j] -= ws * S[i] * d[j];
                }
                // H = -G [n]x
                for (int i = 0; i < 3; ++i) {
                    const float g0 = G[3 * i], g1 = G[3 * i + 1], g2 = G[3 * i + 2];
                    Hm[3 * i + 0] = -(g1 * n[2] - g2 * n[1]);
                    Hm[3 * i + 1] = -(g2 * n[0] - g0 * n[2]);
                    Hm[3 * i + 2] = -(g0 * n[1] - g1 * n[0]);
                }
                // A <- dF_k/dd + A (I - 2 n n^T);  Tn <- f_k + rs Tn
                float An[3];
                for (int i = 0; i < 3; ++i) An[i] = A[3 * i] * n[0] + A[3 * i + 1] * n[1] + A[3 * i + 2] * n[2];
                for (int i = 0; i < 3; ++i)
                    for (int j = 0; j < 3; ++j)
                        A[3 * i + j] = A[3 * i + j] - 2.0f * An[i] * n[j] +
                                       w * ((i == j ? 1.0f - rs : 0.0f) + 2.0f * rs * n[i] * n[j]);
                for (int i = 0; i < 3; ++i) Tn[i] = (1.0f - rs) * d[i] - 2.0f * sc * n[i] + rs * Tn[i];
                node = tnode;
                mat = tmat;
            }
            wave_scatter_add<9>(gw, node, act, Hm, 9);
            wave_scatter_add<6>(gw + 9 * gK, mat, act, gmat, 6);
        }
        // Photon-direction Jacobian of the ray's whole chain, each primary ray
        // keeping its triangle and its share of that triangle's visible area
        // (the share's projected area scales with c = -n0.d):
        //   dF/dd = A - S n0^T / c0,  S = chain contribution per unit weight (Tn)
        if (DIR && (D.flags & SRP_F_GRAD_DIR)) {
            float Jd[9];
            for (int i = 0; i < 3; ++i)
                for (int j = 0; j < 3; ++j) Jd[3 * i + j] = A[3 * i + j] - Tn[i] * n0[j] / c0;
            wave_scatter_add<9>(gw + 9 * gK + 6 * D.n_mats, 0, K > 0, Jd, 9);
        }
    }
    if (parts > 1) __syncthreads();   // (the same for the whole block)
    else wave_lds_fence();
    if (!mine || part != 0) return;
    double SRP_GLOBAL *dst = (double SRP_GLOBAL *)(D.grad_part + (size_t)kc * D.grad_n);
    for (int i = lane; i < D.grad_n; i += WAVE) {
        double t = gw[i];
        for (int k = 1; k < parts; ++k) t += gw[(size_t)k * lds_grad_doubles + i];
        dst[i] = t;
    }
}

// Fan work of the trace kernel's recorded emitters as a separate launch, for
// batches too small to fill the GPU with whole patches and for many fan rays through
// large meshes (the rule is in the host code's layout): one unit per non-empty fan
// pass, as the trace kernel listed them (evaluation, patch, pass), so that one heavy
// patch's passes run side by side on as many waves and no wave claims an empty pass.
// Persistent waves and work queues as in k_trace.
template <bool COUNT>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(SRP_WPE_FWD))) void k_fans(
    const EvalDesc *__restrict__ descs, const uint64_t *__restrict__ win, int grid_blocks,
    const int4 *__restrict__ units, int64_t max_units, uint32_t *queue, uint32_t *spill,
    PatchOut *__restrict__ fan_out, uint64_t *__restrict__ fan_counts) {
    extern __shared__ char smem[];
    const int tid = threadIdx.x, lane = tid & (WAVE - 1);
    LaneStack stack;
    stack.ring = reinterpret_cast<uint32_t *>(smem) + tid;
    stack.stride = BLOCK;
    stack.spill = (uint32_t SRP_GLOBAL *)spill + (size_t)blockIdx.x * BLOCK + tid;
    stack.sstride = grid_blocks * BLOCK;
    double *lacc = reinterpret_cast<double *>(smem + sizeof(uint32_t) * STACK_LDS * BLOCK) + tid;

    // the units the trace kernel listed (it finished before this launch)
    const int64_t listed = (int64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)queue[FAN_UNITS_AT]);
    const uint32_t total = (uint32_t)min(listed, max_units);
    WorkQueue wq = work_queue(tid >> 6);
    int cur = -1;
    float tmin2 = 0.0f;
    #pragma unroll 1
    for (;;) {
        // (the fan kernel's own counters)
        const uint32_t c = take_work(wq, queue + N_QUEUES * QUEUE_STRIDE, total, grid_blocks, false, lane);
        if (c == NO_ITEM) break;
        const int4 U = ((const int4 SRP_GLOBAL *)units)[c];
        if (U.x != cur) {
            cur = U.x;
            const uint64_t *W = win + (size_t)cur * WIN_STRIDE;
            const double wu = -dec_f64(W[1]) - dec_f64(W[0]), wv_ = -dec_f64(W[3]) - dec_f64(W[2]);
            tmin2 = uniform_f32((float)(1e-6 * fmax(wu, wv_)));
        }
        const EvalDesc &D = descs[cur];
        const int B = D.bounces, PM = B * ((D.n_diffuse + FAN_SLICE - 1) / FAN_SLICE);
        const int64_t p = U.y;   // the patch
        const uint64_t SRP_GLOBAL *em = (const uint64_t SRP_GLOBAL *)(D.emit_mask + (size_t)p * B);
        const uint64_t m0 = em[0], m1 = B > 1 ? em[1] : 0ull, m2 = B > 2 ? em[2] : 0ull, m3 = B > 3 ? em[3] : 0ull;
        // exactly pass U.z (a step of PM ends the pass loop after it)
        fan_passes<COUNT>(D, trace_ctx(D), p, m0, m1, m2, m3, U.z, PM, tmin2, stack, lacc, lane, fan_out, fan_counts);
    }
}

constexpr int WBLOCK = 256;   // threads per block of the window kernel

// Copies a small staging image from pinned host memory.  A copy command of a
// few kilobytes waits about 10 us for the copy engine and its signals, this one for
// one read over the bus (one box-wing evaluation at 64^2 with its result written
// straight to pinned memory: 60 -> 57 us).
__global__ __launch_bounds__(WBLOCK) void k_upload(uint4 *__restrict__ dst, const uint4 *__restrict__ src, uint32_t n) {
    const uint32_t i = blockIdx.x * WBLOCK + threadIdx.x;
    if (i < n) dst[i] = src[i];
}

// Loop strides use compile-time block sizes and an explicit grid-width
// argument, so termination never depends on runtime-filled dispatch values.
__global__ __launch_bounds__(WBLOCK) void k_window(const EvalDesc *__restrict__ descs, uint64_t *win, int blocks_x,
                                                  uint32_t *queue) {
    const EvalDesc &D = descs[blockIdx.y];
    // the trace and fan kernels' work counters and the count of listed fan
    // units start at zero
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x <= 2 * N_QUEUES) queue[threadIdx.x * QUEUE_STRIDE] = 0u;
    double mn[5] = {INFINITY, INFINITY, INFINITY, INFINITY, INFINITY};
    const int64_t stride = (int64_t)blocks_x * WBLOCK;
    for (int64_t i = (int64_t)blockIdx.x * WBLOCK + threadIdx.x; i < D.n_wpts; i += stride) {
        const WPoint p = D.wpts[i];
        const double *X = D.xf + 12 * p.node;
        double x = X[0] * p.x + X[1] * p.y + X[2] * p.z + X[9];
        double y = X[3] * p.x + X[4] * p.y + X[5] * p.z + X[10];
        double z = X[6] * p.x + X[7] * p.y + X[8] * p.z + X[11];
        double a = x * D.u[0] + y * D.u[1] + z * D.u[2];
        double b = x * D.v[0] + y * D.v[1] + z * D.v[2];
        double h = x * D.d[0] + y * D.d[1] + z * D.d[2];
        mn[0] = fmin(mn[0], a);
        mn[1] = fmin(mn[1], -a);
        mn[2] = fmin(mn[2], b);
        mn[3] = fmin(mn[3], -b);
        mn[4] = fmin(mn[4], h);
    }
    __shared__ double s[WBLOCK / WAVE][5];
    const int lane = threadIdx.x & (WAVE - 1), wv = threadIdx.x >> 6;
    for (int k = 0; k < 5; ++k) {
        double x = mn[k];
        for (int m = 32; m >= 1; m >>= 1) x = fmin(x, __shfl_xor(x, m, WAVE));
        if (lane == 0) s[wv][k] = x;
    }
    __syncthreads();
    if (threadIdx.x < 5) {
        double x = s[0][threadIdx.x];
        for (int w = 1; w < WBLOCK / WAVE; ++w) x = fmin(x, s[w][threadIdx.x]);
        if (x != INFINITY) atomicMin((unsigned long long *)(win + (size_t)blockIdx.y * WIN_STRIDE + threadIdx.x),
                                     (unsigned long long)enc_f64(x));
    }
}

constexpr int RBLOCK = 1024;   // threads per block of the reduction kernels
constexpr uint32_t ORDER_EVERY = 8;   // launches of a plan per rebuild of its patch order

// Reduction, first stage: block (q, e) sums the q-th of n_slices contiguous
// ranges of evaluation e's patch partials (patches np q / Q .. np (q + 1) / Q),
// then the same range of its fan pass slots, with per-thread strided sums,
// wave butterflies and the waves in order; with GRAD also the q-th range of its
// gradient partials, one per gradient group (the range split again into P
// contiguous slices, P threads per component when the components fit the block
// several times, each summed with eight interleaved accumulators, the slices
// added in order).  Q and the groups depend only on the evaluation's own size, so
// every result depends only on the evaluation, not on the schedule or the batch
// around it.
template <bool COUNT, bool GRAD>
__device__ __forceinline__ void slice_sum_block(const EvalDesc &D, int q, const PatchOut *__restrict__ patches,
                                                const uint64_t *__restrict__ counts,
                                                const PatchOut *__restrict__ fan_out,
                                                const uint64_t *__restrict__ fan_counts) {
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), wid = tid >> 6;
    const int Q = D.n_slices;
    double f[6] = {0, 0, 0, 0, 0, 0};
    unsigned long long cn[5] = {0, 0, 0, 0, 0};
    uint32_t st = 0;
    {
        const int64_t np = D.n_patches;
        const int64_t c0 = D.patch_base + np * q / Q, c1 = D.patch_base + np * (q + 1) / Q;
        for (int64_t c = c0 + tid; c < c1; c += RBLOCK) {
            const PatchOut &co = patches[c];
            for (int k = 0; k < 6; ++k) f[k] += co.f[k];
            cn[0] += co.hits;
            cn[1] += co.sec;
            cn[2] += co.sec_hits;
            st |= co.flags;
            if (COUNT) { cn[3] += counts[2 * c]; cn[4] += counts[2 * c + 1]; }
        }
    }
    if (!GRAD && D.emit) {
        // the fan pass slots (diffuse rays): B ceil(K / FAN_SLICE) per patch
        const int64_t nf = D.n_patches * D.bounces * ((D.n_diffuse + FAN_SLICE - 1) / FAN_SLICE);
        const int64_t u0 = D.fan_base + nf * q / Q, u1 = D.fan_base + nf * (q + 1) / Q;
        for (int64_t c = u0 + tid; c < u1; c += RBLOCK) {
            const PatchOut &co = fan_out[c];
            for (int k = 0; k < 6; ++k) f[k] += co.f[k];
            cn[1] += co.sec;
            cn[2] += co.sec_hits;
            st |= co.flags;
            if (COUNT) { cn[3] += fan_counts[2 * c]; cn[4] += fan_counts[2 * c + 1]; }
        }
    }
    for (int k = 0; k < 6; ++k) f[k] = wave_sum(f[k]);
    for (int m = 32; m >= 1; m >>= 1) {
        for (int k = 0; k < 5; ++k) cn[k] += __shfl_xor(cn[k], m, WAVE);
        st |= __shfl_xor(st, m, WAVE);
    }
    __shared__ double sf[RBLOCK / WAVE][6];
    __shared__ unsigned long long sc[RBLOCK / WAVE][5];
    __shared__ uint32_t ss[RBLOCK / WAVE];
    if (lane == 0) {
        for (int k = 0; k < 6; ++k) sf[wid][k] = f[k];
        for (int k = 0; k < 5; ++k) sc[wid][k] = cn[k];
        ss[wid] = st;
    }
    __syncthreads();
    if (tid == 0) {
        SliceOut o = {};
        for (int w = 0; w < RBLOCK / WAVE; ++w) {
            for (int k = 0; k < 6; ++k) o.f[k] += sf[w][k];
            for (int k = 0; k < 5; ++k) o.cnt[k] += sc[w][k];
            o.flags |= ss[w];
        }
        D.pslice[q] = o;
    }
    if (GRAD) {
        const int G = D.grad_n;
        const double *gp = D.grad_part;
        const int64_t NC = D.n_groups, r0 = NC * q / Q, r1 = NC * (q + 1) / Q;
        const int P = (G > 0 && G <= RBLOCK) ? RBLOCK / G : 1;
        __shared__ double sl[RBLOCK];
        auto slice_sum = [&](int i, int64_t a0, int64_t a1) {
            double a[8] = {0, 0, 0, 0, 0, 0, 0, 0};
            int64_t c = a0;
            for (; c + 8 <= a1; c += 8)
                for (int u = 0; u < 8; ++u) a[u] += gp[(size_t)(c + u) * G + i];
            for (; c < a1; ++c) a[0] += gp[(size_t)c * G + i];
            return ((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7]));
        };
        double *gs = D.gslice + (size_t)q * G;
        if (P > 1) {
            const int i = tid % G, p = tid / G;
            if (p < P) sl[p * G + i] = slice_sum(i, r0 + (r1 - r0) * p / P, r0 + (r1 - r0) * (p + 1) / P);
            __syncthreads();
            for (int j = tid; j < G; j += RBLOCK) {
                double t = 0.0;
                for (int k = 0; k < P; ++k) t += sl[k * G + j];
                gs[j] = t;
            }
        } else {
            for (int j = tid; j < G; j += RBLOCK) gs[j] = slice_sum(j, r0, r1);
        }
    }
}

template <bool COUNT, bool GRAD>
__global__ __launch_bounds__(RBLOCK) void k_slices(const EvalDesc *__restrict__ descs,
                                                const uint32_t *__restrict__ slice_eval,
                                                const PatchOut *__restrict__ patches,
                                                const uint64_t *__restrict__ counts,
                                                const PatchOut *__restrict__ fan_out,
                                                const uint64_t *__restrict__ fan_counts) {
    const EvalDesc &D = descs[slice_eval[blockIdx.x]];
    const int q = (int)((int64_t)blockIdx.x - D.slice_base);
    if (q < 0 || q >= D.n_slices) return;
    slice_sum_block<COUNT, GRAD>(D, q, patches, counts, fan_out, fan_counts);
}

// Heaviest-first patch order for the next launch of a captured forward plan
// (run by the reduction's block of the evaluation, all RBLOCK threads): the
// patches grouped by the bit length of their measured cost (trace time on
// the constant-rate clock, so groups differ by factors of two), groups in
// decreasing cost.  Positions inside a group come from LDS atomics and may
// differ between launches; that changes which wave traces a patch and when,
// never the result.  Every count is exact, so the positions form a
// permutation of the evaluation's patches.
__device__ void patch_order(const EvalDesc &D, uint32_t *order_all, const uint32_t *cost_all, int tid) {
    uint32_t SRP_GLOBAL *ord = (uint32_t SRP_GLOBAL *)order_all + D.patch_base;
    const uint32_t SRP_GLOBAL *cost = (const uint32_t SRP_GLOBAL *)cost_all + D.patch_base;
    const int64_t n = D.n_patches;
    constexpr int NG = 33;   // bit lengths 0..32
    __shared__ uint32_t cnt[NG];
    if (tid < NG) cnt[tid] = 0;
    __syncthreads();
    for (int64_t i = tid; i < n; i += RBLOCK) atomicAdd(&cnt[32 - __clz(cost[i])], 1u);
    __syncthreads();
    if (tid == 0) {
        uint32_t run = 0;
        for (int g = NG - 1; g >= 0; --g) {
            const uint32_t c = cnt[g];
            cnt[g] = run;
            run += c;
        }
    }
    __syncthreads();
    for (int64_t i = tid; i < n; i += RBLOCK) ord[atomicAdd(&cnt[32 - __clz(cost[i])], 1u)] = (uint32_t)i;
}

// Reduction, second stage (one block per evaluation): the first stage's
// range sums added in order, scaled to newtons; with GRAD the gradient range
// sums likewise, then assembled per material and hinge DOF.  A captured
// forward plan's block also orders the patches for the plan's next launch.
template <bool COUNT, bool GRAD>
__device__ __forceinline__ void reduce_block(const EvalDesc &D, int e, const uint64_t *W, srp_result *out,
                                             uint32_t *order, const uint32_t *cost, uint32_t *order_launch) {
    const int tid = threadIdx.x;
    const int Q = D.n_slices;
    const double umin = dec_f64(W[0]), umax = -dec_f64(W[1]);
    const double vmin = dec_f64(W[2]), vmax = -dec_f64(W[3]);
    const double wu = umax - umin, wv = vmax - vmin;
    const bool empty = !(wu * wv > 0.0) || !(wu < INFINITY) || !(wv < INFINITY) || D.root_ref == REF_NONE;
    const double scale = empty ? 0.0 : D.pressure * (wu * wv / ((double)D.n * (double)D.n));
    if (tid == 0) {
        double F[6] = {0, 0, 0, 0, 0, 0};
        unsigned long long N[5] = {0, 0, 0, 0, 0};
        uint32_t S = 0;
        for (int q = 0; q < Q; ++q) {
            const SliceOut &o = D.pslice[q];
            for (int k = 0; k < 6; ++k) F[k] += o.f[k];
            for (int k = 0; k < 5; ++k) N[k] += o.cnt[k];
            S |= o.flags;
        }
        srp_result r;
        for (int k = 0; k < 3; ++k) {
            r.force[k] = scale * F[k];
            r.torque[k] = scale * F[3 + k];
        }
        r.n_rays = (int64_t)D.n * D.n;
        r.n_hits = (int64_t)N[0];
        r.n_secondary = (int64_t)N[1];
        r.n_secondary_hits = (int64_t)N[2];
        r.n_box_tests = COUNT ? (int64_t)N[3] : 0;
        r.n_tri_tests = COUNT ? (int64_t)N[4] : 0;
        r.status = S;
        r.n_clamped = (uint32_t)D.n_clamped;
        out[e] = r;
    }
    if (!GRAD && order && cost) {   // (the same for the whole block)
        // rebuilt on every ORDER_EVERY-th launch of the plan: the order stays
        // useful while consecutive launches see similar images, and the pass
        // costs as much as the reduction itself (its LDS counters are hot)
        __shared__ uint32_t s_launch;
        if (tid == 0) s_launch = *order_launch;
        __syncthreads();
        const uint32_t launch = s_launch;
        if (launch % ORDER_EVERY == 0) patch_order(D, order, cost, tid);
        // (one increment per launch; another evaluation's block may read either
        // value, which only moves the launch its order is rebuilt on)
        if (e == 0 && tid == 0) *order_launch = launch + 1;
    }
    if (GRAD) {
        const int G = D.grad_n, K = D.n_nodes, M = D.n_mats, J = D.n_dof;
        __shared__ double sg[MAX_GRAD_SLOTS];
        __shared__ int spar[SRP_MAX_NODES];   // the tree, for the subtree walks below
        for (int j = tid; j < G; j += RBLOCK) {
            double t = 0.0;
            for (int q = 0; q < Q; ++q) t += D.gslice[(size_t)q * G + j];
            sg[j] = t;
        }
        for (int q = tid; q < K; q += RBLOCK) spar[q] = D.parent[q];
        __syncthreads();
        double *g = D.grad_out;
        if (g) {
            // rho_s (M x 3), rho_d (M x 3)
            for (int i = tid; i < 6 * M; i += RBLOCK) {
                int m = i / 6, k = i % 6;
                double v = scale * sg[9 * K + i];
                if (k < 3) g[3 * m + k] = v;
                else g[3 * M + 3 * m + (k - 3)] = v;
            }
            // theta: (sum of S_q over the subtree of the joint's node) * world axis
            for (int j = tid; j < J; j += RBLOCK) {
                const int p = D.dof_node[j];
                double S[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
                for (int q = 0; q < K; ++q) {
                    int a = q;
                    while (a > p) a = spar[a];
                    if (a != p) continue;
                    for (int i = 0; i < 9; ++i) S[i] += sg[9 * q + i];
                }
                const double *ax = D.axw + 3 * j;
                for (int i = 0; i < 3; ++i)
                    g[6 * M + 3 * j + i] = scale * (S[3 * i] * ax[0] + S[3 * i + 1] * ax[1] + S[3 * i + 2] * ax[2]);
            }
            // photon-direction Jacobian dF_i/dd_j (row-major); zeros when the item
            // did not ask for it (its partials then have no direction slots)
            const bool has_dir = G >= 9 * K + 6 * M + 9;
            for (int i = tid; i < 9; i += RBLOCK) g[6 * M + 3 * J + i] = has_dir ? scale * sg[9 * K + 6 * M + i] : 0.0;
        }
    }
}

template <bool COUNT, bool GRAD>
__global__ __launch_bounds__(RBLOCK) void k_reduce(const EvalDesc *__restrict__ descs,
                                                const uint64_t *__restrict__ win, srp_result *out,
                                                uint32_t *order, const uint32_t *cost, uint32_t *order_launch) {
    const int e = blockIdx.x;
    reduce_block<COUNT, GRAD>(descs[e], e, win + (size_t)e * WIN_STRIDE, out, order, cost, order_launch);
}

// Both stages in one launch where every evaluation has a single range (below
// 2,048 partials): one launch less, which is what bounds them (one box-wing
// evaluation at 64^2 56.2 -> 54.6 us whole).  With several ranges the last block
// to finish could add them, but the fence before it writes back the L2: 512^2
// propagation stages 1.90 -> 1.95 ms, 900^2 187 -> 196 us.
template <bool COUNT, bool GRAD>
__global__ __launch_bounds__(RBLOCK) void k_sums(const EvalDesc *__restrict__ descs,
                                              const PatchOut *__restrict__ patches,
                                              const uint64_t *__restrict__ counts,
                                              const PatchOut *__restrict__ fan_out,
                                              const uint64_t *__restrict__ fan_counts, const uint64_t *__restrict__ win,
                                              srp_result *out, uint32_t *order, const uint32_t *cost,
                                              uint32_t *order_launch) {
    const int e = blockIdx.x;
    slice_sum_block<COUNT, GRAD>(descs[e], 0, patches, counts, fan_out, fan_counts);
    __syncthreads();
    reduce_block<COUNT, GRAD>(descs[e], e, win + (size_t)e * WIN_STRIDE, out, order, cost, order_launch);
}

int check(hipError_t e) { return e == hipSuccess ? 0 : (int)e; }

}  // namespace

// The device workspace of srp_eval_batch_noalloc.  Its name is a host-side
// stand-in in host code: only the address looked up on each device is passed
// to kernels and copies.
static __device__ __align__(256) char scratch[NOALLOC_SCRATCH_BYTES];

static char *g_scratch_ptr[NOALLOC_MAX_DEVICES] = {};

int noalloc_scratch_init() {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return (int)e;
    if (dev < 0 || dev >= NOALLOC_MAX_DEVICES) return (int)hipErrorInvalidDevice;
    if (g_scratch_ptr[dev]) return 0;
    void *p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return (int)e;
    g_scratch_ptr[dev] = static_cast<char *>(p);
    return 0;
}

char *noalloc_scratch(int device) {
    return (device >= 0 && device < NOALLOC_MAX_DEVICES) ? g_scratch_ptr[device] : nullptr;
}

int launch_upload(char *dst, const char *src, size_t bytes, void *stream) {
    const uint32_t n = (uint32_t)(bytes / sizeof(uint4));
    if (n == 0) return 0;
    hipLaunchKernelGGL(k_upload, dim3((n + WBLOCK - 1) / WBLOCK), dim3(WBLOCK), 0, (hipStream_t)stream,
                       reinterpret_cast<uint4 *>(dst), reinterpret_cast<const uint4 *>(src), n);
    return check(hipGetLastError());
}

int launch_window(const EvalDesc *d_desc, int n_evals, int blocks_x, uint64_t *d_win, uint32_t *d_queue,
                  void *stream) {
    if (n_evals <= 0) return 0;
    hipLaunchKernelGGL(k_window, dim3(blocks_x, n_evals), dim3(WBLOCK), 0, (hipStream_t)stream, d_desc, d_win, blocks_x,
                       d_queue);
    return check(hipGetLastError());
}

size_t trace_lds_bytes() { return sizeof(uint32_t) * STACK_LDS * BLOCK + sizeof(double) * 6 * BLOCK + GRID_LDS; }

int launch_trace(const EvalDesc *d_desc, const int64_t *d_chunk_base, int n_evals, const uint64_t *d_win,
                 int64_t total_chunks, uint32_t *d_queue, uint32_t *d_spill, PatchOut *d_chunks,
                 uint64_t *d_counts, bool count, int grid_blocks, PatchOut *d_fan_out, uint64_t *d_fan_counts,
                 bool fans_inline_, bool long_chunks, int4 *d_fan_units, int blocks_per_cu, const uint32_t *d_order, uint32_t *d_cost,
                 void *stream) {
    if (total_chunks <= 0) return 0;
    const size_t lds = trace_lds_bytes();
    const int fans_inline = (d_fan_out && fans_inline_) ? (long_chunks ? 2 : 1) : 0;
    int4 *fan_units = (d_fan_out && !fans_inline_) ? d_fan_units : nullptr;
    hipStream_t s = (hipStream_t)stream;
#define SRP_LAUNCH_TRACE(C, W)                                                                                    \
    hipLaunchKernelGGL((k_trace<C, W>), dim3(grid_blocks), dim3(BLOCK), lds, s, d_desc, d_chunk_base, n_evals,     \
                       d_win, grid_blocks, total_chunks, d_queue, d_spill, d_chunks, d_counts, fans_inline,       \
                       d_fan_out, d_fan_counts, fan_units, d_order, d_cost)
    // (the counting variant serves tests and the benchmark's work counts: one
    // instantiation; both instantiations compute the same bits)
    if (count) SRP_LAUNCH_TRACE(true, 0);
    else if (blocks_per_cu <= 2) SRP_LAUNCH_TRACE(false, 2);
    else SRP_LAUNCH_TRACE(false, 0);
#undef SRP_LAUNCH_TRACE
    return check(hipGetLastError());
}

int launch_adjoint(const EvalDesc *d_desc, int n_evals, const uint32_t *d_block_base, uint32_t n_blocks,
                   uint32_t max_blocks, int block_waves, const PatchOut *d_patches, bool dir, int lds_grad_doubles,
                   void *stream) {
    if (n_evals <= 0 || n_blocks == 0) return 0;
    if (block_waves < 1 || block_waves > MAX_PPC / GROUP_PART || (block_waves & (block_waves - 1)) || max_blocks == 0)
        return (int)hipErrorInvalidValue;
    const size_t lds = sizeof(double) * block_waves * lds_grad_doubles;
    const dim3 block(WAVE * block_waves);
    for (uint32_t b = 0; b < n_blocks; b += MAX_LAUNCH_BLOCKS) {
        const dim3 grid(std::min(n_blocks - b, MAX_LAUNCH_BLOCKS));
        if (dir)
            hipLaunchKernelGGL((k_adjoint<true>), grid, block, lds, (hipStream_t)stream, d_desc, n_evals, d_block_base,
                               b, launch_share(max_blocks), block_waves, d_patches, lds_grad_doubles);
        else
            hipLaunchKernelGGL((k_adjoint<false>), grid, block, lds, (hipStream_t)stream, d_desc, n_evals, d_block_base,
                               b, launch_share(max_blocks), block_waves, d_patches, lds_grad_doubles);
        const hipError_t err = hipGetLastError();
        if (err != hipSuccess) return (int)err;
    }
    return 0;
}

int launch_fans(const EvalDesc *d_desc, const uint64_t *d_win, int64_t max_units, uint32_t *d_queue,
                uint32_t *d_spill, PatchOut *d_fan_out, uint64_t *d_fan_counts, const int4 *d_fan_units, bool count,
                int grid_blocks, void *stream) {
    if (max_units <= 0) return 0;
    const size_t lds = trace_lds_bytes();   // the same ring and accumulators as the forward trace
    hipStream_t s = (hipStream_t)stream;
    if (count)
        hipLaunchKernelGGL((k_fans<true>), dim3(grid_blocks), dim3(BLOCK), lds, s, d_desc, d_win, grid_blocks,
                           d_fan_units, max_units, d_queue, d_spill, d_fan_out, d_fan_counts);
    else
        hipLaunchKernelGGL((k_fans<false>), dim3(grid_blocks), dim3(BLOCK), lds, s, d_desc, d_win, grid_blocks,
                           d_fan_units, max_units, d_queue, d_spill, d_fan_out, d_fan_counts);
    return check(hipGetLastError());
}

int launch_reduce(const EvalDesc *d_desc, int n_evals, const uint64_t *d_win, const PatchOut *d_patches,
                  const uint64_t *d_counts, const PatchOut *d_fan_out, const uint64_t *d_fan_counts, bool count,
                  bool grad, const uint32_t *d_slice_eval, int64_t total_slices, void *d_out, uint32_t *d_order,
                  const uint32_t *d_cost, uint32_t *d_order_launch, void *stream) {
    if (n_evals <= 0) return 0;
    if (total_slices < n_evals || total_slices > INT32_MAX) return (int)hipErrorInvalidValue;
    hipStream_t s = (hipStream_t)stream;
    srp_result *out = (srp_result *)d_out;
#define SRP_LAUNCH_REDUCE(C, G)                                                                                 \
    do {                                                                                                        \
        if (total_slices == n_evals) {                                                                          \
            hipLaunchKernelGGL((k_sums<C, G>), dim3(n_evals), dim3(RBLOCK), 0, s, d_desc, d_patches, d_counts,  \
                               d_fan_out, d_fan_counts, d_win, out, d_order, d_cost, d_order_launch);           \
            break;                                                                                              \
        }                                                                                                       \
        hipLaunchKernelGGL((k_slices<C, G>), dim3((uint32_t)total_slices), dim3(RBLOCK), 0, s, d_desc,          \
                           d_slice_eval, d_patches, d_counts, d_fan_out, d_fan_counts);                         \
        hipLaunchKernelGGL((k_reduce<C, G>), dim3(n_evals), dim3(RBLOCK), 0, s, d_desc, d_win, out, d_order,    \
                           d_cost, d_order_launch);                                                             \
    } while (0)
    if (count && grad) SRP_LAUNCH_REDUCE(true, true);
    else if (count) SRP_LAUNCH_REDUCE(true, false);
    else if (grad) SRP_LAUNCH_REDUCE(false, true);
    else SRP_LAUNCH_REDUCE(false, false);
#undef SRP_LAUNCH_REDUCE
    return check(hipGetLastError());
}

int trace_blocks_per_cu(bool count) {
    const size_t lds = trace_lds_bytes();
    int nb = 0;
    hipError_t e = count ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_trace<true, 0>, BLOCK, lds)
                         : hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_trace<false, 0>, BLOCK, lds);
    if (e != hipSuccess || nb < 1) nb = 1;
    return nb;
}

int fan_blocks_per_cu(bool count) {
    const size_t lds = trace_lds_bytes();
    int nb = 0;
    hipError_t e = count ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_fans<true>, BLOCK, lds)
                         : hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_fans<false>, BLOCK, lds);
    if (e != hipSuccess || nb < 1) nb = 1;
    return nb;
}

}  // namespace srp
