// Primary visibility of an evaluation by rasterisation.
//
//   k_primary  one wave per square tile of the ray grid (TW x TW pixels): walks
//              every instance's bottom-level hierarchy for the tile (four
//              children of up to 16 nodes per step, one per lane), gathers the
//              triangles whose leaves meet it, and tests (triangle, pixel) pairs
//              of their pixel rectangles, 64 pairs per step, against the tile's
//              depth buffer in LDS.
//
// The primary rays of an evaluation are one parallel bundle, so their first
// hits need no per-ray traversal: box and triangle bounds in image coordinates
// select the pairs (conservatively), and each selected pair is decided by the
// ray tracer's own arithmetic (the instance frame and the watertight test of
// trace.h, on the same FP32 ray), with its tie rule (smaller distance, then
// smaller original index).  The trace kernel therefore sees the hits that its
// own traversal would find, and starts at the shading of the first hit.  (A ray
// that lies in a triangle's plane to FP32 rounding has no meaningful distance
// to it; a window so thin that its pixels are below that rounding, a body seen
// edge-on, is left to the traversal, and so is a tile of very many layers.)
#include <float.h>

#include "srp.h"
#include "srp_internal.h"
#include "trace.h"

namespace srp {

namespace {

constexpr int WAVE = 64;
constexpr int NODES_PER_STEP = WAVE / 4;
constexpr int STACK_CAP = 384;
// A step takes fewer nodes as the stack fills, down to one: depth first from
// there, at most 3 more entries per level of the hierarchy.
constexpr int STACK_SLACK = 3 * (BLAS_MAX_DEPTH + 1) + 4;
constexpr int LIST_CAP = WAVE + WAVE * LEAF_MAX;   // a step adds at most 64 leaves to fewer than 64 triangles
static_assert(STACK_CAP > STACK_SLACK + 4 * NODES_PER_STEP, "the stack holds a full step and the slack");

// A tile that has been hit this many times over is left to the traversal, whose rays
// stop near their first hit while the tile tests every layer behind it.  (us per
// call at B = 1, by traversal / all layers tested / now: 200 plates a tenth of the image
// wide beside a sphere, 512^2 x 64 1,261 / 1,673 / 1,233, 1024^2 x 64 4,038 / 3,674 / 2,871; 50
// plates three tenths wide, 1024^2 x 64 4,289 / 3,469 / 3,667.  With 16 layers the first two
// are 1,201 and 2,852, but eight 2048^2 images of a million triangles 1,356 in place of
// 1,284; 8 layers cost the 50k craft 5 to 12 %.  Counting the hits takes 15 of 837 us
// over 64 x 1024^2.)
constexpr int MAX_LAYERS = 24;

__device__ __forceinline__ int rank_below(uint64_t m, int lane) {
    return __popcll(m & ((1ull << lane) - 1ull));
}

// Inclusive prefix sum over the wave's 64 lanes (rows by shifts, then the rows' totals).
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_add(uint32_t x) {
    return x + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, ROWS, 0xF, false);
}
__device__ __forceinline__ uint32_t wave_scan(uint32_t x) {
    x = dpp_add<0x111, 0xF>(x);   // row_shr 1, 2, 4, 8
    x = dpp_add<0x112, 0xF>(x);
    x = dpp_add<0x114, 0xF>(x);
    x = dpp_add<0x118, 0xF>(x);
    x = dpp_add<0x142, 0xA>(x);   // row_bcast 15 into rows 1 and 3
    x = dpp_add<0x143, 0xC>(x);   // row_bcast 31 into rows 2 and 3
    return x;
}

// Per evaluation (one wave each), what every tile needs of it and of its
// instances.
__global__ __launch_bounds__(WAVE) void k_primary_setup(const EvalDesc *__restrict__ descs,
                                                        const uint64_t *__restrict__ win) {
    const EvalDesc &D = descs[blockIdx.x];
    if (!D.prim) return;
    const int tid = threadIdx.x;
    const RayGrid G = ray_grid(D, win + (size_t)blockIdx.x * WIN_STRIDE);
    const double iu = 1.0 / G.du, iv = 1.0 / G.dv;
    // Margin: twice the hierarchy's box padding (4e-6 of the mesh's scale), which
    // exceeds every FP32 rounding of the projected points and of the rays.
    const float mx = (float)(2.0 * D.box_pad * iu), my = (float)(2.0 * D.box_pad * iv);
    if (tid == 0) {
        PrimaryEval E = {};
        for (int k = 0; k < 3; ++k) {
            E.o0[k] = G.o0[k];
            E.su[k] = G.su[k];
            E.sv[k] = G.sv[k];
        }
        E.mx = mx;
        E.my = my;
        E.empty = G.empty;
        E.traced = !(mx < 0.5f) || !(my < 0.5f);
        *D.prim = E;
    }
    PrimaryInst *out = reinterpret_cast<PrimaryInst *>(D.prim + 1);
    for (int i = tid; i < D.n_nodes; i += WAVE) {
        const Inst &I = D.inst[i];
        const ArtNode &A = D.art[i];
        PrimaryInst P = {};
        float ld[3];
        for (int k = 0; k < 3; ++k) {
            P.u[k] = (float)(((double)I.R[k] * D.u[0] + (double)I.R[3 + k] * D.u[1] + (double)I.R[6 + k] * D.u[2]) * iu);
            P.v[k] = (float)(((double)I.R[k] * D.v[0] + (double)I.R[3 + k] * D.v[1] + (double)I.R[6 + k] * D.v[2]) * iv);
            ld[k] = dot3(I.R[k], I.R[3 + k], I.R[6 + k], G.dd[0], G.dd[1], G.dd[2]);
            P.t[k] = I.t[k];
        }
        P.uc = (float)(((double)I.t[0] * D.u[0] + (double)I.t[1] * D.u[1] + (double)I.t[2] * D.u[2] - G.umin) * iu - 0.5);
        P.vc = (float)(((double)I.t[0] * D.v[0] + (double)I.t[1] * D.v[1] + (double)I.t[2] * D.v[2] - G.vmin) * iv - 0.5);
        for (int k = 0; k < 9; ++k) P.R[k] = I.R[k];
        onb(ld, P.mx, P.my);
        for (int k = 0; k < 3; ++k) P.mz[k] = ld[k];
        P.root = I.root;
        float r[4] = {P.uc - mx, P.uc + mx, P.vc - my, P.vc + my};
        for (int k = 0; k < 3; ++k) {
            const float a = P.u[k] * (float)A.blo[k], b = P.u[k] * (float)A.bhi[k];
            const float c = P.v[k] * (float)A.blo[k], d = P.v[k] * (float)A.bhi[k];
            r[0] += fminf(a, b);
            r[1] += fmaxf(a, b);
            r[2] += fminf(c, d);
            r[3] += fmaxf(c, d);
        }
        for (int k = 0; k < 4; ++k) P.rect[k] = r[k];
        out[i] = P;
    }
}

// Whether a padded box of the instance can meet pixel centres [x0, x1] x [y0, y1]
// (bounds already widened by the margin; a NaN bound counts as meeting).
__device__ __forceinline__ bool box_meets(const PrimaryInst SRP_CONST &M, const float lo[3], const float hi[3], float x0, float x1,
                                          float y0, float y1) {
    float xa = M.uc, xb = M.uc, ya = M.vc, yb = M.vc;
    for (int k = 0; k < 3; ++k) {
        const float p = M.u[k] * lo[k], q = M.u[k] * hi[k];
        xa += fminf(p, q);
        xb += fmaxf(p, q);
        const float r = M.v[k] * lo[k], s = M.v[k] * hi[k];
        ya += fminf(r, s);
        yb += fmaxf(r, s);
    }
    return !(xb < x0) && !(xa > x1) && !(yb < y0) && !(ya > y1);
}

// Blocks are numbered through the batch's rasterised evaluations (block_owner).
// Laid out as the largest evaluation's tiles x all evaluations, one 1024^2 image
// beside 4,096 box-wing evaluations at 64^2 launched 67 million blocks: 14.9 ms for
// the call, now 0.84 (2048^2: 57.3 and 1.06 ms).
template <int TW>
__global__ __launch_bounds__(WAVE) void k_primary(const EvalDesc *__restrict__ descs, int n_evals,
                                                  const uint32_t *__restrict__ tile_base, uint32_t first_tile,
                                                  uint32_t per_most) {
    __shared__ uint64_t zb[TW * TW];   // patch-major: (patch of the tile) * 64 + pixel of the patch
    __shared__ uint32_t stk[STACK_CAP];
    __shared__ uint32_t lst[LIST_CAP];
    __shared__ float4 ta[WAVE], tb[WAVE], tc[WAVE];   // a batch's triangles with pairs: corners (and the index)
    __shared__ uint4 info[WAVE];       // first pair, x0 | y0 << 8 | width << 16, 1 / width
    __shared__ uint32_t mark[WAVE];
    constexpr int PW = TW / PATCH;

    const int lane = threadIdx.x;
    const uint32_t SRP_CONST *base = (const uint32_t SRP_CONST *)tile_base;
    const uint32_t block = first_tile + blockIdx.x;
    const BlockOwner own = block_owner(base, n_evals, block, per_most);
    const int e = own.eval;
    const EvalDesc SRP_CONST &D = ((const EvalDesc SRP_CONST *)descs)[e];
    const int N = D.n, gp = 2 * D.tiles_x;             // patches per row of the image
    const int nt = (gp + PW - 1) / PW;                 // tiles per row
    const int tile = (int)(block - own.first);
    const int tx = tile % nt, ty = tile / nt;
    const int X0 = tx * TW, Y0 = ty * TW;
    const int X1 = min(X0 + TW, N) - 1, Y1 = min(Y0 + TW, N) - 1;

    const PrimaryEval SRP_CONST &E = *(const PrimaryEval SRP_CONST *)D.prim;
    const PrimaryInst SRP_CONST *PI = (const PrimaryInst SRP_CONST *)(&E + 1);
    if (E.traced) return;
    const float mx = E.mx, my = E.my;
    const float bx0 = (float)X0 - mx, bx1 = (float)X1 + mx, by0 = (float)Y0 - my, by1 = (float)Y1 + my;
    const BNode4 SRP_GLOBAL *blas = (const BNode4 SRP_GLOBAL *)D.blas;
    const TriRec SRP_GLOBAL *tris = (const TriRec SRP_GLOBAL *)D.tris;
    const int K = D.n_nodes;
    bool any = false;   // the depth buffer is set up
    bool left = false;  // the tile is left to the traversal
    int steps = 0;      // pair steps so far
    uint32_t hits = 0;  // this lane's pairs that met

    if (!E.empty && X1 >= X0 && Y1 >= Y0) {
        for (int i0 = 0; i0 < K && !left; i0 += WAVE) {
            // the instances whose image rectangle meets the tile
            bool meets = false;
            if (i0 + lane < K) {
                const PrimaryInst SRP_GLOBAL *pl = (const PrimaryInst SRP_GLOBAL *)(D.prim + 1) + i0 + lane;
                const float4 r = *(const float4 SRP_GLOBAL *)pl->rect;
                meets = pl->root != REF_NONE && !(r.y < (float)X0) && !(r.x > (float)X1) &&
                        !(r.w < (float)Y0) && !(r.z > (float)Y1);
            }
            uint64_t todo = __ballot(meets);
            if (todo && !any) {
                any = true;
                for (int i = lane; i < TW * TW; i += WAVE) zb[i] = ~0ull;
                __syncthreads();
            }
            while (todo && !left) {
                const int inst = i0 + __ffsll((unsigned long long)todo) - 1;
                todo &= todo - 1;
                const PrimaryInst SRP_CONST &M = PI[inst];
                Frame F;
                for (int k = 0; k < 3; ++k) {
                    F.mx[k] = M.mx[k];
                    F.my[k] = M.my[k];
                    F.mz[k] = M.mz[k];
                }
                // child c of node q: its reference (REF_NONE when its box misses the tile)
                auto child = [&](uint32_t q, int c) -> uint32_t {
                    const float SRP_GLOBAL *b = (const float SRP_GLOBAL *)(blas + q);
                    const uint32_t ref = ((const uint32_t SRP_GLOBAL *)b)[24 + c];
                    const float lo[3] = {b[c], b[4 + c], b[8 + c]}, hi[3] = {b[12 + c], b[16 + c], b[20 + c]};
                    return ref != REF_NONE && box_meets(M, lo, hi, bx0, bx1, by0, by1) ? ref : REF_NONE;
                };

                int sp = 0, nl = 0;
                // inner children onto the stack, the triangles of leaves onto the list
                auto emit = [&](uint32_t ref) {
                    const bool any = ref != REF_NONE;
                    const bool leaf = any && ref_type(ref) == REF_BLAS_LEAF;
                    const uint64_t mi = __ballot(any && !leaf);
                    if (any && !leaf) stk[sp + rank_below(mi, lane)] = ref_index(ref);
                    sp += __popcll(mi);
                    if (__ballot(leaf)) {
                        const uint32_t p = ref_index(ref);
                        const uint32_t cnt = leaf ? (p & 7u) + 1u : 0u;
                        const uint32_t inc = wave_scan(cnt);
                        for (uint32_t k = 0; k < cnt; ++k) lst[nl + inc - cnt + k] = (p >> 3) + k;
                        nl += __builtin_amdgcn_readlane((int)inc, 63);
                    }
                };
                const uint32_t root = M.root;
                if (ref_type(root) == REF_BLAS_LEAF) emit(lane == 0 ? root : REF_NONE);
                else emit(lane < 4 ? child(ref_index(root), lane) : REF_NONE);
                __syncthreads();
                while ((sp > 0 || nl > 0) && !left) {
                    if (sp > 0 && nl < WAVE) {
                        const int room = (STACK_CAP - STACK_SLACK - sp) / 3;
                        const int take = max(1, min(min(NODES_PER_STEP, sp), room));
                        uint32_t ref = REF_NONE;
                        if ((lane >> 2) < take) ref = child(stk[sp - 1 - (lane >> 2)], lane & 3);
                        sp -= take;
                        __syncthreads();
                        emit(ref);
                        __syncthreads();
                        continue;
                    }
                    // up to 64 triangles: pixel rectangles, then their pairs
                    const int m = min(nl, WAVE);
                    nl -= m;
                    uint32_t cnt = 0, packed = 0;
                    float4 A, B, C;
                    float w = 1.0f;
                    if (lane < m) {
                        const float4 SRP_GLOBAL *q = (const float4 SRP_GLOBAL *)(tris + lst[nl + lane]);
                        A = q[0];
                        B = q[1];
                        C = q[2];
                        const float xa = fmaf(M.u[0], A.x, fmaf(M.u[1], A.y, fmaf(M.u[2], A.z, M.uc)));
                        const float xb = fmaf(M.u[0], B.x, fmaf(M.u[1], B.y, fmaf(M.u[2], B.z, M.uc)));
                        const float xc = fmaf(M.u[0], C.x, fmaf(M.u[1], C.y, fmaf(M.u[2], C.z, M.uc)));
                        const float ya = fmaf(M.v[0], A.x, fmaf(M.v[1], A.y, fmaf(M.v[2], A.z, M.vc)));
                        const float yb = fmaf(M.v[0], B.x, fmaf(M.v[1], B.y, fmaf(M.v[2], B.z, M.vc)));
                        const float yc = fmaf(M.v[0], C.x, fmaf(M.v[1], C.y, fmaf(M.v[2], C.z, M.vc)));
                        // (max and min drop a NaN bound for the tile's own)
                        const float fx0 = fmaxf(ceilf(fminf(fminf(xa, xb), xc) - mx), (float)X0);
                        const float fx1 = fminf(floorf(fmaxf(fmaxf(xa, xb), xc) + mx), (float)X1);
                        const float fy0 = fmaxf(ceilf(fminf(fminf(ya, yb), yc) - my), (float)Y0);
                        const float fy1 = fminf(floorf(fmaxf(fmaxf(ya, yb), yc) + my), (float)Y1);
                        if (fx0 <= fx1 && fy0 <= fy1) {
                            const int x0 = (int)fx0 - X0, y0 = (int)fy0 - Y0;
                            const int wi = (int)(fx1 - fx0) + 1, hi = (int)(fy1 - fy0) + 1;
                            cnt = (uint32_t)(wi * hi);
                            packed = (uint32_t)x0 | ((uint32_t)y0 << 8) | ((uint32_t)wi << 16);
                            w = 1.0f / (float)wi;
                        }
                    }
                    const uint32_t inc = wave_scan(cnt), start = inc - cnt;
                    const int total = __builtin_amdgcn_readlane((int)inc, 63);
                    const uint64_t has = __ballot(cnt > 0);
                    if (cnt > 0) {
                        const int s = rank_below(has, lane);
                        ta[s] = A;
                        tb[s] = B;
                        tc[s] = C;
                        info[s] = make_uint4(start, packed, __float_as_uint(w), 0u);
                    }
                    int run = 0;
                    for (int base = 0; base < total; base += WAVE) {
                        // the triangles whose first pair lies in this step, as a lane mask
                        mark[lane] = 0;
                        __syncthreads();
                        const uint32_t rel = start - (uint32_t)base;
                        if (cnt > 0 && rel < (uint32_t)WAVE) mark[rel] = 1;
                        __syncthreads();
                        const uint64_t starts = __ballot(mark[lane] != 0);
                        const int p = base + lane;
                        if (p < total) {
                            const int s = run + __popcll(starts & ((2ull << lane) - 1ull)) - 1;
                            const uint4 in = info[s];
                            const float4 a = ta[s], b = tb[s], c = tc[s];
                            const int q = p - (int)in.x, wi = (int)(in.y >> 16);
                            const int row = (int)(((float)q + 0.5f) * __uint_as_float(in.z));
                            const int lx = (int)(in.y & 255u) + q - row * wi, ly = (int)((in.y >> 8) & 255u) + row;
                            const float fx = (float)(X0 + lx), fy = (float)(Y0 + ly);
                            float r[3], lo[3];
                            for (int k = 0; k < 3; ++k) r[k] = fmaf(fy, E.sv[k], fmaf(fx, E.su[k], E.o0[k])) - M.t[k];
                            for (int k = 0; k < 3; ++k) lo[k] = dot3(M.R[k], M.R[3 + k], M.R[6 + k], r[0], r[1], r[2]);
                            frame_offsets(lo, F);
                            const float va[3] = {a.x, a.y, a.z}, vb[3] = {b.x, b.y, b.z}, vc[3] = {c.x, c.y, c.z};
                            const float th = tri_hit(F, va, vb, vc);
                            if (th > 0.0f && th <= T_INF) {
                                ++hits;
                                const uint64_t key = ((uint64_t)__float_as_uint(th) << 32) | (uint32_t)f2i(a.w);
                                const int idx = (((ly >> 3) * PW + (lx >> 3)) << 6) | ((ly & 7) << 3) | (lx & 7);
                                (void)__hip_atomic_fetch_min(&zb[idx], key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                            }
                        }
                        run += __popcll(starts);
                        __syncthreads();
                    }
                    steps += (total + WAVE - 1) / WAVE;
                    if (steps > MAX_LAYERS * TW * TW / WAVE)
                        left = __builtin_amdgcn_readlane((int)wave_scan(hits), 63) > MAX_LAYERS * TW * TW;
                }
            }
        }
    }
    __syncthreads();

    // the tile's hit masks and hits, patch by patch
    uint64_t SRP_GLOBAL *vmask = (uint64_t SRP_GLOBAL *)D.vis_mask;
    uint2 SRP_GLOBAL *vis = (uint2 SRP_GLOBAL *)D.vis;
    const int32_t SRP_GLOBAL *leaf_of = (const int32_t SRP_GLOBAL *)D.leaf_of;
    for (int q = 0; q < PW * PW; ++q) {
        const int gx = tx * PW + q % PW, gy = ty * PW + q / PW;
        if (gx >= gp || gy >= gp) continue;
        const int64_t pt = 4 * ((int64_t)(gy >> 1) * D.tiles_x + (gx >> 1)) + 2 * (gy & 1) + (gx & 1);
        const uint64_t key = any ? zb[q * WAVE + lane] : ~0ull;
        const bool hit = !left && key != ~0ull;
        const bool unknown = left && gx * PATCH + (lane & 7) < N && gy * PATCH + (lane >> 3) < N;
        const uint64_t m = __ballot(hit || unknown);
        if (hit) vis[pt * WAVE + lane] = make_uint2((uint32_t)(key >> 32), (uint32_t)leaf_of[(uint32_t)key]);
        if (unknown) vis[pt * WAVE + lane] = make_uint2(0u, VIS_UNKNOWN);
        if (lane == 0) vmask[pt] = m;
    }
}

}  // namespace

int launch_primary(const EvalDesc *d_desc, int n_evals, const uint64_t *d_win, int tile, const uint32_t *d_tile_base,
                   uint32_t n_tiles, uint32_t max_tiles, void *stream) {
    if (n_evals <= 0 || n_tiles == 0) return 0;
    if ((tile != 16 && tile != 8) || max_tiles == 0) return (int)hipErrorInvalidValue;
    hipLaunchKernelGGL(k_primary_setup, dim3((uint32_t)n_evals), dim3(WAVE), 0, (hipStream_t)stream, d_desc, d_win);
    for (uint32_t b = 0; b < n_tiles; b += MAX_LAUNCH_BLOCKS) {
        const dim3 grid(n_tiles - b < MAX_LAUNCH_BLOCKS ? n_tiles - b : MAX_LAUNCH_BLOCKS);
        if (tile == 16)
            hipLaunchKernelGGL((k_primary<16>), grid, dim3(WAVE), 0, (hipStream_t)stream, d_desc, n_evals, d_tile_base,
                               b, launch_share(max_tiles));
        else
            hipLaunchKernelGGL((k_primary<8>), grid, dim3(WAVE), 0, (hipStream_t)stream, d_desc, n_evals, d_tile_base,
                               b, launch_share(max_tiles));
        const hipError_t err = hipGetLastError();
        if (err != hipSuccess) return (int)err;
    }
    return 0;
}

}  // namespace srp
