// dock_device.hip -- gfx950 kernels of the geometric-docking hot path.
//
// Method: Alg. 1 of arXiv:2209.05069 (Application Description).  One
// wavefront docks one (ligand, restart): Generate_Starting_Pose, the A*A rigid
// alignment and the greedy torsion sweep (Optimize Pose).  A second kernel does
// Select Poses and the final rigid step per ligand.  Mapping choices for CDNA4:
//  * lanes hold atoms (atom i = lane + 64*slot) for every per-atom update, so a
//    pose lives in registers; a wave-uniform atom is fetched with readlane;
//  * the alignment spreads the A*A orientations over the 64 lanes, and the
//    torsion step spreads the T candidates over the lanes (T/64 per lane); each
//    lane scores its candidates over the moving atoms, whose rotation frames
//    sit once per wave in LDS (broadcast reads);
//  * only the moving fragment's score changes with the torsion angle, so the
//    candidates are ranked by that partial sum (same argmax as the full score);
//  * bump check in closed form: turning a moving atom about the bond axis makes
//    its squared distance to a static atom C + A cos(theta) + B sin(theta), so
//    pairs whose closest approach stays above the bump distance are dropped
//    (ballot), and the few remaining pairs are tested against the candidates they
//    can reach with two FMAs; one 64-bit key max
//    (order-preserving score bits, then the lower index) over the bump-free
//    candidates picks the step;
//  * grid gathers are raw buffer loads of cell cubes (a cell's trilinear
//    coefficients in one 32-byte record): two 16-byte loads from one cache line
//    per sample, a 32-bit voffset for the cell and the atom type as scalar offset,
//    with the range checked by hardware;
//  * a persistent grid pops (ligand, restart-group) items from a per-bin queue;
//    the ligand's coordinates, bump-pair rows and masks are staged once per
//    item in LDS and shared by the workgroup's waves.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <cmath>

#include "dock_internal.h"

namespace dockgpu {

typedef unsigned long long u64;

// ---------------------------------------------------------------------------
// wavefront helpers
__device__ __forceinline__ int lane_id() { return (int)__lane_id(); }

// Whole-wave reductions with DPP: row_shr 1, 2, 4, 8 leave in lane 15 of every
// 16-lane row the reduction of its row; row_bcast 15 and 31 carry the rows into
// lane 63, whose value is then read by every lane.  Lanes outside a shift read 0,
// the identity of the sum, the max of unsigned keys and the or.  Call with the
// whole wave active.
template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp_read(int v) {
    return __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xF, true);
}

template <int CTRL, int ROWS>
__device__ __forceinline__ u64 dpp_read64(u64 v) {
    const uint32_t lo = (uint32_t)dpp_read<CTRL, ROWS>((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)dpp_read<CTRL, ROWS>((int)(uint32_t)(v >> 32));
    return ((u64)hi << 32) | lo;
}

__device__ __forceinline__ u64 read_lane64(u64 v, int lane) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), lane);
    return ((u64)hi << 32) | lo;
}

#define DOCK_DPP_STEPS(STEP) \
    STEP(0x111, 0xF) STEP(0x112, 0xF) STEP(0x114, 0xF) STEP(0x118, 0xF) STEP(0x142, 0xA) STEP(0x143, 0xC)

__device__ __forceinline__ float wave_sum(float v) {
#define DOCK_SUM_STEP(C, R) v += __int_as_float(dpp_read<C, R>(__float_as_int(v)));
    DOCK_DPP_STEPS(DOCK_SUM_STEP)
#undef DOCK_SUM_STEP
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
    v = max(v, (uint32_t)dpp_read<0x111, 0xF>((int)v));
    v = max(v, (uint32_t)dpp_read<0x112, 0xF>((int)v));
    v = max(v, (uint32_t)dpp_read<0x114, 0xF>((int)v));
    v = max(v, (uint32_t)dpp_read<0x118, 0xF>((int)v));
    v = max(v, (uint32_t)dpp_read<0x142, 0xA>((int)v));
    v = max(v, (uint32_t)dpp_read<0x143, 0xC>((int)v));
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// Largest key of the wave in two 32-bit steps: the largest upper half, then the
// largest lower half among its lanes (most often one lane).
__device__ __forceinline__ u64 wave_max_key(u64 v) {
    const uint32_t hi = (uint32_t)(v >> 32), top = wave_max_u32(hi);
    const u64 at = __builtin_amdgcn_ballot_w64(hi == top);
    uint32_t lo;
    if ((at & (at - 1ull)) == 0ull)
        lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, __ffsll((long long)at) - 1);
    else
        lo = wave_max_u32(hi == top ? (uint32_t)v : 0u);
    return ((u64)top << 32) | lo;
}

__device__ __forceinline__ u64 wave_or_u64(u64 v) {
#define DOCK_OR_STEP(C, R) v |= dpp_read64<C, R>(v);
    DOCK_DPP_STEPS(DOCK_OR_STEP)
#undef DOCK_OR_STEP
    return read_lane64(v, 63);
}
#undef DOCK_DPP_STEPS

__device__ __forceinline__ int uniform_int(int v) { return __builtin_amdgcn_readfirstlane(v); }

// A wave-uniform value read from memory or LDS, as a scalar: masks, counts and loop
// bounds derived from it then stay in scalar registers.
__device__ __forceinline__ u64 uniform_u64(u64 v) {
    const uint32_t lo = (uint32_t)uniform_int((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)uniform_int((int)(uint32_t)(v >> 32));
    return ((u64)hi << 32) | lo;
}

__device__ __forceinline__ float read_lane(float v, int lane) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}

// Order-preserving map of a float to uint32 (larger float -> larger integer).
__device__ __forceinline__ uint32_t ord_f32(float f) {
    uint32_t u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float unord_f32(uint32_t u) {
    return __uint_as_float((u & 0x80000000u) ? (u & 0x7fffffffu) : ~u);
}
// Key of (score, index): the max key has the best score, then the lowest index.
__device__ __forceinline__ u64 make_key(float s, uint32_t idx) {
    return ((u64)ord_f32(s) << 32) | (u64)(0xFFFFFFFFu - idx);
}
__device__ __forceinline__ uint32_t key_index(u64 k) { return 0xFFFFFFFFu - (uint32_t)k; }
__device__ __forceinline__ float key_score(u64 k) { return unord_f32((uint32_t)(k >> 32)); }

// Make LDS writes of this wave visible to its own later LDS reads by other lanes.
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---------------------------------------------------------------------------
// Trilinear interpolation.  (gx,gy,gz) are grid coordinates ((p - origin)/h);
// each is clamped to [0, n-1], the cell corner is min(floor, n-2).  The pocket
// is stored as cell cubes (see GridArgs): the two x-vertex columns of a cell,
// each as the bilinear coefficients of its (y,z) face, are one 32-byte record,
// read as two 16-byte loads from the same cache line.
// toff is the byte offset of the atom type's block.
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

struct Tri {
    __amdgpu_buffer_rsrc_t rs;
    float mx, my, mz, m2x, m2y, m2z, fnx, fslab;
    uint32_t nx, slab;  // cells per row and per slab
};

__device__ __forceinline__ Tri make_tri(const GridArgs &g) {
    Tri t;
    t.rs = __builtin_amdgcn_make_buffer_rsrc((void *)g.cubes, (short)0,
                                             (int)(g.ncells * 32u), 0x00020000);
    t.mx = g.mx; t.my = g.my; t.mz = g.mz;
    t.m2x = g.m2x; t.m2y = g.m2y; t.m2z = g.m2z;
    t.fnx = g.fnx; t.fslab = g.fslab;
    t.nx = (uint32_t)g.nx;
    t.slab = (uint32_t)g.nx * (uint32_t)g.ny;
    return t;
}

// byte offset of the cell record within the type block, and the fractions
__device__ __forceinline__ uint32_t tri_cell(const Tri &t, float gx, float gy, float gz, float &fx,
                                             float &fy, float &fz) {
    const float cx = __builtin_amdgcn_fmed3f(gx, 0.0f, t.mx);
    const float cy = __builtin_amdgcn_fmed3f(gy, 0.0f, t.my);
    const float cz = __builtin_amdgcn_fmed3f(gz, 0.0f, t.mz);
    const float ix = floorf(__builtin_amdgcn_fmed3f(gx, 0.0f, t.m2x));
    const float iy = floorf(__builtin_amdgcn_fmed3f(gy, 0.0f, t.m2y));
    const float iz = floorf(__builtin_amdgcn_fmed3f(gz, 0.0f, t.m2z));
    fx = cx - ix;
    fy = cy - iy;
    fz = cz - iz;
    // element index < 2^24: exact in float
    const float e = fmaf(iz, t.fslab, fmaf(iy, t.fnx, ix));
    return ((uint32_t)e) << 5;
}

// 16-byte raw buffer load; the builtin returns the bits as integers.
__device__ __forceinline__ float4 ldq(__amdgpu_buffer_rsrc_t rs, uint32_t voff, int soff) {
    const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)voff, soff, 0);
    return make_float4(__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z),
                       __uint_as_float(v.w));
}

// Bilinear (y,z) form of one x-vertex column: q = (a, b, c, d) with
// v(fy,fz) = a + b*fy + c*fz + d*fy*fz.
__device__ __forceinline__ float col_bilin(const float4 q, float fy, float fz) {
    return fmaf(fz, fmaf(fy, q.w, q.z), fmaf(fy, q.y, q.x));
}

// q0, q1: the columns at x vertices i and i+1; the x interpolation comes last.
__device__ __forceinline__ float tri_blend(const float4 q0, const float4 q1, float fx, float fy,
                                           float fz) {
    const float b0 = col_bilin(q0, fy, fz), b1 = col_bilin(q1, fy, fz);
    return fmaf(fx, b1 - b0, b0);
}

// wave-uniform type offset (scalar offsets)
__device__ __forceinline__ float tri_u(const Tri &t, float gx, float gy, float gz, int toff) {
    float fx, fy, fz;
    const uint32_t off = tri_cell(t, gx, gy, gz, fx, fy, fz);
    const float4 q0 = ldq(t.rs, off, toff);
    const float4 q1 = ldq(t.rs, off, toff + 16);
    return tri_blend(q0, q1, fx, fy, fz);
}

// per-lane type offset
__device__ __forceinline__ float tri_v(const Tri &t, float gx, float gy, float gz, uint32_t toff) {
    float fx, fy, fz;
    const uint32_t off = tri_cell(t, gx, gy, gz, fx, fy, fz) + toff;
    const float4 q0 = ldq(t.rs, off, 0);
    const float4 q1 = ldq(t.rs, off, 16);
    return tri_blend(q0, q1, fx, fy, fz);
}

// Samples known to lie in [0, n-2] on every axis: the clamps of tri_u are then
// the identity, floor is truncation and the fraction is exact as v_fract, so
// this returns the same value with fewer instructions.
// Byte offset of the cube of a sample in [0, n-2] on every axis: truncation is
// floor there, and cell indices and sizes fit the 24-bit multipliers.
__device__ __forceinline__ uint32_t in_cell(const Tri &t, float gx, float gy, float gz) {
    return (__umul24((uint32_t)gz, t.slab) + __umul24((uint32_t)gy, t.nx) + (uint32_t)gx) << 5;
}
constexpr float kInsideMargin = 0.5f;  // grid cells, far above FP32 rounding of coordinates
__device__ __forceinline__ float tri_in(const Tri &t, float gx, float gy, float gz, int toff) {
    const float fx = __builtin_amdgcn_fractf(gx), fy = __builtin_amdgcn_fractf(gy),
                fz = __builtin_amdgcn_fractf(gz);
    const uint32_t off = in_cell(t, gx, gy, gz);
    const float4 q0 = ldq(t.rs, off, toff);
    const float4 q1 = ldq(t.rs, off, toff + 16);
    return tri_blend(q0, q1, fx, fy, fz);
}

// Flag of a listed torsion candidate that bumps (see score_free).
constexpr int kCandBumped = 0x8000;

// Radius for ball_inside from its square: the hardware square root (about one
// ulp).  Only the choice between tri_in and tri_u depends on it, the two give the
// same value inside [0, n-2], and kInsideMargin dwarfs the error.
__device__ __forceinline__ float ball_radius(float r2) { return __builtin_amdgcn_sqrtf(r2); }

// Whether the ball of radius rad (grid units) about (cx,cy,cz), widened by
// kInsideMargin, stays inside [0, n-2] on every axis.
template <class G>  // Tri or GridArgs
__device__ __forceinline__ bool ball_inside(const G &t, float cx, float cy, float cz, float rad) {
    const float r = rad + kInsideMargin;
    // (all six at once, no branches)
    return (cx - r >= 0.0f) & (cy - r >= 0.0f) & (cz - r >= 0.0f) & (cx + r <= t.m2x) &
           (cy + r <= t.m2y) & (cz + r <= t.m2z);
}

// Bilinear coefficients of the (y,z) face at x vertex i of cell (j,k): from
// its corners v00 = v(i,j,k), v10 = v(i,j+1,k), v01 = v(i,j,k+1),
// v11 = v(i,j+1,k+1), (a, b, c, d) = (v00, v10 - v00, v01 - v00,
// (v11 - v10) - (v01 - v00)).
__device__ __forceinline__ float4 face_coeffs(const float *b0, const float *b1, long long r0,
                                              long long r1, int i) {
    const float v00 = b0[r0 + i], v10 = b0[r1 + i], v01 = b1[r0 + i], v11 = b1[r1 + i];
    return make_float4(v00, v10 - v00, v01 - v00, (v11 - v10) - (v01 - v00));
}

// Cell cubes from the plain grid (one thread per cell).  Cells at i = nx-1,
// j = ny-1 or k = nz-1 are never read (the cell corner is at most n-2); they
// repeat the edge values.
__global__ void k_build_cubes(const float *__restrict__ v, float4 *__restrict__ q, int ntypes,
                              int nx, int ny, int nz) {
    const long long cells = (long long)nx * ny * nz;
    const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= cells * ntypes) return;
    const long long t = e / cells;
    long long r = e - t * cells;
    const int k = (int)(r / ((long long)nx * ny));
    r -= (long long)k * nx * ny;
    const int j = (int)(r / nx), i = (int)(r - (long long)j * nx);
    const int i1 = i + 1 < nx ? i + 1 : i, j1 = j + 1 < ny ? j + 1 : j, k1 = k + 1 < nz ? k + 1 : k;
    const float *b0 = v + t * cells + (long long)k * nx * ny;
    const float *b1 = v + t * cells + (long long)k1 * nx * ny;
    const long long r0 = (long long)j * nx, r1 = (long long)j1 * nx;
    q[2 * e] = face_coeffs(b0, b1, r0, r1, i);
    q[2 * e + 1] = face_coeffs(b0, b1, r0, r1, i1);
}

// ---------------------------------------------------------------------------
// Pose held across lanes: atom i = lane + 64*s in slot s.
template <int NS>
struct Pose {
    float x[NS], y[NS], z[NS];
};

template <int NS>
__device__ __forceinline__ void pick_atom(const Pose<NS> &Y, int i, float &px, float &py,
                                          float &pz) {
    const int l = i & 63, s = i >> 6;
    px = read_lane(Y.x[0], l);
    py = read_lane(Y.y[0], l);
    pz = read_lane(Y.z[0], l);
#pragma unroll
    for (int q = 1; q < NS; ++q) {
        if (s == q) {
            px = read_lane(Y.x[q], l);
            py = read_lane(Y.y[q], l);
            pz = read_lane(Y.z[q], l);
        }
    }
}

template <int NS>
__device__ __forceinline__ void centroid(const Pose<NS> &Y, int n, float &cx, float &cy,
                                         float &cz) {
    float sx = 0.f, sy = 0.f, sz = 0.f;
    const int lane = lane_id();
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        if (lane + 64 * s < n) {
            sx += Y.x[s];
            sy += Y.y[s];
            sz += Y.z[s];
        }
    }
    const float inv = 1.0f / (float)n;
    cx = wave_sum(sx) * inv;
    cy = wave_sum(sy) * inv;
    cz = wave_sum(sz) * inv;
}

// Generate_Starting_Pose: Y = S_r (X - c0) + grid centre.  X rows in LDS (x,y,z,toff).
template <int NS>
__device__ __forceinline__ void start_pose(Pose<NS> &Y, const float4 *xyzt, int n, int r,
                                           const GridArgs &g, const SearchArgs &sa) {
    const int lane = lane_id();
    Pose<NS> X;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const int i = lane + 64 * s;
        const float4 v = i < n ? xyzt[i] : make_float4(0.f, 0.f, 0.f, 0.f);
        X.x[s] = v.x;
        X.y[s] = v.y;
        X.z[s] = v.z;
    }
    float c0x, c0y, c0z;
    centroid(X, n, c0x, c0y, c0z);
    const float4 m0 = sa.smat[3 * r + 0], m1 = sa.smat[3 * r + 1], m2 = sa.smat[3 * r + 2];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const float dx = X.x[s] - c0x, dy = X.y[s] - c0y, dz = X.z[s] - c0z;
        Y.x[s] = fmaf(m0.x, dx, fmaf(m0.y, dy, fmaf(m0.z, dz, g.cx)));
        Y.y[s] = fmaf(m1.x, dx, fmaf(m1.y, dy, fmaf(m1.z, dz, g.cy)));
        Y.z[s] = fmaf(m2.x, dx, fmaf(m2.y, dy, fmaf(m2.z, dz, g.cz)));
    }
}

// Apply alignment orientation o about the pose centroid.
template <int NS>
__device__ __forceinline__ void apply_align(Pose<NS> &Y, int n, int o, const SearchArgs &sa) {
    float cx, cy, cz;
    centroid(Y, n, cx, cy, cz);
    const float4 m0 = sa.amat[3 * o + 0], m1 = sa.amat[3 * o + 1], m2 = sa.amat[3 * o + 2];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const float dx = Y.x[s] - cx, dy = Y.y[s] - cy, dz = Y.z[s] - cz;
        Y.x[s] = fmaf(m0.x, dx, fmaf(m0.y, dy, fmaf(m0.z, dz, cx)));
        Y.y[s] = fmaf(m1.x, dx, fmaf(m1.y, dy, fmaf(m1.z, dz, cy)));
        Y.z[s] = fmaf(m2.x, dx, fmaf(m2.y, dy, fmaf(m2.z, dz, cz)));
    }
}

// How the candidates of one decision (alignment orientations, torsion steps) are
// spread and reduced.  WaveSplit: one wavefront holds them all (batched form).
// BlockSplit: the waves of a workgroup hold interleaved slices and the argmax
// goes through LDS with workgroup barriers (plain form; every wave keeps the
// same pose).
struct WaveSplit {
    __device__ __forceinline__ int first() const { return 0; }
    __device__ __forceinline__ int stride() const { return 64; }
    __device__ __forceinline__ u64 reduce(u64 k) const { return wave_max_key(k); }
};

struct BlockSplit {
    int wave, waves;
    u64 *slots;  // LDS, [waves]
    __device__ __forceinline__ int first() const { return 64 * wave; }
    __device__ __forceinline__ int stride() const { return 64 * waves; }
    __device__ __forceinline__ u64 reduce(u64 k) const {
        k = wave_max_key(k);
        if (lane_id() == 0) slots[wave] = k;
        __syncthreads();
        u64 r = slots[0];
        for (int w = 1; w < waves; ++w) r = slots[w] > r ? slots[w] : r;
        __syncthreads();
        return r;
    }
};

// Read-only (cos, sin) table in the constant address space: wave-uniform
// indices load through the scalar cache into SGPRs.
typedef const __attribute__((address_space(4))) float *cfloat2_p;
__device__ __forceinline__ float2 ld_cs(cfloat2_p p, int k) {
    return make_float2(p[2 * k], p[2 * k + 1]);
}

// Alignment orientation o = i*A + j is R_y(2 pi j / A) R_x(2 pi i / A) about the
// pose centroid, applied in two stages to the centred grid-unit offset r of an
// atom.  The x rotation (per atom and i) gives the final y coordinate and the
// rotated z; the y rotation (per j) the final x and z.  (cos, sin) of 2 pi k / A
// come from the acs table; e is the centroid in grid units.
struct XStage {
    float rx, qz, gy;
};
__device__ __forceinline__ XStage align_x(float rx, float ry, float rz, float2 ci, float ey) {
    XStage s;
    s.rx = rx;
    s.qz = fmaf(ci.y, ry, ci.x * rz);
    s.gy = fmaf(ci.x, ry, fmaf(-ci.y, rz, ey));
    return s;
}
__device__ __forceinline__ float align_gx(const XStage &s, float2 cj, float ex) {
    return fmaf(cj.x, s.rx, fmaf(cj.y, s.qz, ex));
}
__device__ __forceinline__ float align_gz(const XStage &s, float2 cj, float ez) {
    return fmaf(-cj.y, s.rx, fmaf(cj.x, s.qz, ez));
}

// Alignment (Rigid Rotation): lanes over the A*A orientations, loop over atoms.
// rec: per-wave LDS, >= n float4.  toff[s]: type byte offset of this lane's atoms.
// Applies and returns the best orientation; *best_out = its score.
template <int NS, class Split>
__device__ int align_pose(Pose<NS> &Y, int n, const int (&toff)[NS], float4 *rec, const Tri &tr,
                          const GridArgs &g, const SearchArgs &sa, float *best_out,
                          const Split &sp) {
    const int lane = lane_id();
    float cx, cy, cz;
    centroid(Y, n, cx, cy, cz);
    const float ex = (cx - g.ox) * g.inv_h, ey = (cy - g.oy) * g.inv_h, ez = (cz - g.oz) * g.inv_h;
    // record: centred grid-unit offset and type offset; all_in: every orientation
    // of every atom samples inside the grid (spheres about the centroid)
    bool out_any = false;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const int i = lane + 64 * s;
        if (i < n) {
            const float rx = (Y.x[s] - cx) * g.inv_h, ry = (Y.y[s] - cy) * g.inv_h,
                        rz = (Y.z[s] - cz) * g.inv_h;
            out_any = out_any ||
                      !ball_inside(tr, ex, ey, ez, ball_radius(fmaf(rx, rx, fmaf(ry, ry, rz * rz))));
            rec[i] = make_float4(rx, ry, rz, __int_as_float(toff[s]));
        }
    }
    const bool all_in = __ballot(out_any) == 0ull;
    wave_lds_sync();
    const int NO = sa.A * sa.A;
    u64 best = 0;
    for (int base = sp.first(); base < NO; base += sp.stride()) {
        const int o = base + lane;
        const bool ov = o < NO;
        const int oo = ov ? o : 0;
        const int oi = oo / sa.A;
        const float2 ci = sa.acs[oi], cj = sa.acs[oo - oi * sa.A];
        float acc = 0.f;
        if (all_in) {
            for (int a = 0; a < n; ++a) {
                const float4 r = rec[a];
                const int to = uniform_int(__float_as_int(r.w));
                const XStage xs = align_x(r.x, r.y, r.z, ci, ey);
                acc += tri_in(tr, align_gx(xs, cj, ex), xs.gy, align_gz(xs, cj, ez), to);
            }
        } else {
            for (int a = 0; a < n; ++a) {
                const float4 r = rec[a];
                const int to = uniform_int(__float_as_int(r.w));
                const XStage xs = align_x(r.x, r.y, r.z, ci, ey);
                acc += tri_u(tr, align_gx(xs, cj, ex), xs.gy, align_gz(xs, cj, ez), to);
            }
        }
        const u64 key = ov ? make_key(acc, (uint32_t)o) : 0ull;
        best = key > best ? key : best;
    }
    best = sp.reduce(best);
    const int ob = (int)key_index(best);
    if (best_out) *best_out = key_score(best);
    wave_lds_sync();  // rec is rewritten by the caller next
    apply_align(Y, n, ob, sa);
    return ob;
}

// Rotation frame of bond (a,b) for this lane's atoms: p = a + u(u.v),
// vp = v - u(u.v), w = u x v, with v = Y_i - a; a rotation by theta sends Y_i to
// p + cos(theta) vp + sin(theta) w.
struct Axis {
    float ax, ay, az, ux, uy, uz;
};

template <int NS>
__device__ __forceinline__ Axis bond_axis(const Pose<NS> &Y, int a, int b) {
    Axis A;
    float bx, by, bz;
    pick_atom(Y, a, A.ax, A.ay, A.az);
    pick_atom(Y, b, bx, by, bz);
    const float dx = bx - A.ax, dy = by - A.ay, dz = bz - A.az;
    // unit axis from the hardware reciprocal square root (about one ulp, as
    // against two roundings for a square root and a divide)
    const float inv = __builtin_amdgcn_rsqf(dx * dx + dy * dy + dz * dz);
    A.ux = dx * inv;
    A.uy = dy * inv;
    A.uz = dz * inv;
    return A;
}

__device__ __forceinline__ void torsion_frame(const Axis &A, float x, float y, float z, float &px,
                                              float &py, float &pz, float &vx, float &vy,
                                              float &vz, float &wx, float &wy, float &wz) {
    const float dx = x - A.ax, dy = y - A.ay, dz = z - A.az;
    const float ud = A.ux * dx + A.uy * dy + A.uz * dz;
    px = fmaf(A.ux, ud, A.ax);
    py = fmaf(A.uy, ud, A.ay);
    pz = fmaf(A.uz, ud, A.az);
    vx = fmaf(-A.ux, ud, dx);
    vy = fmaf(-A.uy, ud, dy);
    vz = fmaf(-A.uz, ud, dz);
    wx = A.uy * dz - A.uz * dy;
    wy = A.uz * dx - A.ux * dz;
    wz = A.ux * dy - A.uy * dx;
}

// Turn the moving atoms (mask row mrow) by (c, sn) = (cos, sin) about axis A.
template <int NS>
__device__ __forceinline__ void apply_torsion(Pose<NS> &Y, const u64 *mrow, const Axis &A,
                                              float c, float sn) {
    const int lane = lane_id();
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const bool mv = (mrow[s] >> lane) & 1ull;
        if (mv) {
            float px, py, pz, vx, vy, vz, wx, wy, wz;
            torsion_frame(A, Y.x[s], Y.y[s], Y.z[s], px, py, pz, vx, vy, vz, wx, wy, wz);
            Y.x[s] = fmaf(sn, wx, fmaf(c, vx, px));
            Y.y[s] = fmaf(sn, wy, fmaf(c, vy, py));
            Y.z[s] = fmaf(sn, wz, fmaf(c, vz, pz));
        }
    }
}

// One torsion decision (Optimize Pose, inner angle loop) for rotatable bond with
// moving-mask row mrow (NS words), axis atoms (a,b).  cs[c] = (cos,sin) of this
// lane's candidates k = lane + 64c.  Returns the applied step or kTraceNone.
// Best key (score, candidate) among the nfree candidates of a torsion step
// listed in cand, scored on the moving fragment (frames of m moving atoms in
// rec): lanes take the listed candidates in P passes of 64, each candidate's sum
// runs over the atoms in order, as when every candidate is scored in place.  An
// entry is the step index, with kCandBumped set when the candidate is listed
// although it bumps (no-pruning mode): it is scored but cannot win.
// Inside: every candidate position lies in [0, n-2] on every axis.
template <int P, bool Inside>
__device__ __forceinline__ u64 score_free(int nfree, const uint16_t *cand, const float4 *rec,
                                          int m, const float2 *tors, const Tri &tr) {
    const int lane = lane_id();
    int kp[P];
    bool ok[P];
    float2 csp[P];
    float acc[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const int idx = lane + 64 * p;
        const int e = cand[idx < nfree ? idx : 0];
        kp[p] = e & (kCandBumped - 1);
        ok[p] = idx < nfree && !(e & kCandBumped);
        csp[p] = tors[kp[p]];
        acc[p] = 0.f;
    }
    int q = 0;
    // U atoms at a time (up to four (atom, pass) cube loads): their loads are in
    // flight together; the sums still take the atoms in order
    constexpr int U = P == 1 ? 4 : (P == 2 ? 2 : 1);
    if (Inside && U > 1) {
        for (; q + U - 1 < m; q += U) {
            float f[U][P][3];
            float4 c0[U][P], c1[U][P];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const float4 r0 = rec[3 * (q + u) + 0], r1 = rec[3 * (q + u) + 1],
                             r2 = rec[3 * (q + u) + 2];
                const int to = uniform_int(__float_as_int(r0.w));
#pragma unroll
                for (int p = 0; p < P; ++p) {
                    const float gx = fmaf(csp[p].y, r2.x, fmaf(csp[p].x, r1.x, r0.x));
                    const float gy = fmaf(csp[p].y, r2.y, fmaf(csp[p].x, r1.y, r0.y));
                    const float gz = fmaf(csp[p].y, r2.z, fmaf(csp[p].x, r1.z, r0.z));
                    f[u][p][0] = __builtin_amdgcn_fractf(gx);
                    f[u][p][1] = __builtin_amdgcn_fractf(gy);
                    f[u][p][2] = __builtin_amdgcn_fractf(gz);
                    const uint32_t off = in_cell(tr, gx, gy, gz);
                    c0[u][p] = ldq(tr.rs, off, to);
                    c1[u][p] = ldq(tr.rs, off, to + 16);
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int p = 0; p < P; ++p)
                    acc[p] += tri_blend(c0[u][p], c1[u][p], f[u][p][0], f[u][p][1], f[u][p][2]);
        }
    }
    for (; q < m; ++q) {
        const float4 r0 = rec[3 * q + 0], r1 = rec[3 * q + 1], r2 = rec[3 * q + 2];
        const int to = uniform_int(__float_as_int(r0.w));
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const float gx = fmaf(csp[p].y, r2.x, fmaf(csp[p].x, r1.x, r0.x));
            const float gy = fmaf(csp[p].y, r2.y, fmaf(csp[p].x, r1.y, r0.y));
            const float gz = fmaf(csp[p].y, r2.z, fmaf(csp[p].x, r1.z, r0.z));
            acc[p] += Inside ? tri_in(tr, gx, gy, gz, to) : tri_u(tr, gx, gy, gz, to);
        }
    }
    u64 best = 0ull;
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const u64 key = ok[p] ? make_key(acc[p], (uint32_t)kp[p]) : 0ull;
        best = key > best ? key : best;
    }
    return best;
}

// score_free with the pass count rounded up to a quarter of C (uniform branch).
template <int C, bool Inside>
__device__ __forceinline__ u64 score_free_any(int nfree, const uint16_t *cand, const float4 *rec,
                                              int m, const float2 *tors, const Tri &tr) {
    constexpr int Q = C >= 4 ? C / 4 : 1;
    constexpr int P2 = 2 * Q <= C ? 2 * Q : C, P3 = 3 * Q <= C ? 3 * Q : C;
    const int np = (nfree + 63) >> 6;
    if (np <= Q) return score_free<Q, Inside>(nfree, cand, rec, m, tors, tr);
    if (np <= P2) return score_free<P2, Inside>(nfree, cand, rec, m, tors, tr);
    if (np <= P3) return score_free<P3, Inside>(nfree, cand, rec, m, tors, tr);
    return score_free<C, Inside>(nfree, cand, rec, m, tors, tr);
}

// The kernel's arguments, to be loaded again: read through this reference a value
// is live from its first to its last use in the phase that took the reference.
// (Kept from the kernel's start, the arguments of all phases together overflow the
// scalar registers and are spilled to vector lanes, a VALU instruction each way.)
__device__ __forceinline__ const DockArgs &fresh_args() {
    auto p = (const __attribute__((address_space(4))) DockArgs *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return *(const DockArgs *)p;
}

__device__ __forceinline__ u64 ballot(bool v) { return __builtin_amdgcn_ballot_w64(v); }
// The lane's bit of a wave-uniform mask, and the number of lower lanes set in it.
__device__ __forceinline__ bool inverse_ballot(u64 m) {
    return __builtin_amdgcn_inverse_ballot_w64(m);
}
__device__ __forceinline__ int mbcnt(u64 m) {
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                          __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Moving atoms up to which a decision tests each row's pairs as they are found.  More
// rows are listed first: finding a pair then costs less (10 VALU a row instead of 25),
// a list costs about 120 more.  Torsion sweep of 2,500 ligands of 20-80 atoms and of
// 6,000 of 16 atoms: 22.8 and 11.4 ms with every decision direct, 22.0 and 12.2 ms with
// every decision listed, 21.3 and 11.4 ms with the line at 4 (21.5 and 11.8 ms at 2,
// 21.3 and 11.4 ms at 8).
constexpr int kBumpDirect = 4;
// Scratch of the bump check, in the LDS of the candidate list that follows it.
struct BumpLds {
    float4 coef[64];                // (Cq, Aq, Bq, 0) of pairs
    uint16_t pair[64 + kMaxAtoms];  // pairs: moving row << 8 | static atom
};
static_assert(sizeof(BumpLds) <= kMaxTorsionSteps * 2, "bump scratch fits the candidate list");

// Tests up to 64 listed pairs (lane p: pair p of np) against the candidates.  For
// moving atom i (frame P0, V, W) and static atom j, the squared distance after a
// turn by theta is
//   d2(theta) = Cq + Aq cos(theta) + Bq sin(theta),
//   Cq = |P0 - Y_j|^2 + |V|^2, Aq = 2 (P0 - Y_j).V, Bq = 2 (P0 - Y_j).W
// (V and W are orthogonal with |V| = |W|).  Its minimum over theta is
// Cq - sqrt(Aq^2 + Bq^2); pairs that cannot come closer than the bump distance are
// dropped.  Over a slot's arc the extremes of Aq cos + Bq sin are +-sqrt(Aq^2 +
// Bq^2) inside the arc or the values at its ends: a slot that some pair bumps from
// end to end is done, and only pairs that reach into a slot are tested against its
// candidates, with two FMAs each.  (mg: above the roundings of both.)  On random trees
// of 20-100 atoms 18 pairs a decision are listed and 21 (pair, slot) tests are left of
// 73, 0.46 slots being done without one.  Sweep of 16,000 such ligands: 225 ms with
// every pair tested against every candidate, 198 ms so; bound by issue (VALU 0.8 busy,
// SALU 0.5).  Without pruning (300 ligands of 64 atoms): 38.2 -> 22.0 ms, since a pair's
// terms are read through LDS (no VALU) instead of lane by lane.
template <int NS, int C>
__device__ __forceinline__ void bump_pairs(int np, const uint16_t *pair, BumpLds *bl,
                                           const float4 *rec,
                                           const float (&sgx)[NS], const float (&sgy)[NS],
                                           const float (&sgz)[NS], const float2 (&cs)[C],
                                           int first, int stride, const TorsionArgs &k,
                                           u64 (&bumped)[C]) {
    const float lim = k.lim;
    const int lane = lane_id();
    const int e = pair[lane < np ? lane : 0];
    const int q = e >> 8, j = e & 255;
    const float4 r0 = rec[3 * q + 0], r1 = rec[3 * q + 1], r2 = rec[3 * q + 2];
    auto pick = [&](const float (&v)[NS]) -> float {
        float x = __int_as_float(__builtin_amdgcn_ds_bpermute(4 * (j & 63), __float_as_int(v[0])));
#pragma unroll
        for (int s = 1; s < NS; ++s) {
            const float y =
                __int_as_float(__builtin_amdgcn_ds_bpermute(4 * (j & 63), __float_as_int(v[s])));
            x = (j >> 6) == s ? y : x;
        }
        return x;
    };
    const float dx = r0.x - pick(sgx), dy = r0.y - pick(sgy), dz = r0.z - pick(sgz);
    const float vv = fmaf(r1.x, r1.x, fmaf(r1.y, r1.y, r1.z * r1.z));
    const float cq = fmaf(dx, dx, fmaf(dy, dy, fmaf(dz, dz, vv)));
    const float aq = 2.0f * fmaf(dx, r1.x, fmaf(dy, r1.y, dz * r1.z));
    const float bq = 2.0f * fmaf(dx, r2.x, fmaf(dy, r2.y, dz * r2.z));
    const u64 live = np >= 64 ? ~0ull : (1ull << np) - 1ull;
    if (!k.prune) {
        bl->coef[lane] = make_float4(cq, aq, bq, 0.0f);
        wave_lds_sync();
        for (int p = 0; p < np; p += 4) {  // (lanes past np hold the first pair again)
            const float4 *t = bl->coef + p;
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int c = 0; c < C; ++c)
                    bumped[c] |= ballot(fmaf(t[u].z, cs[c].y, fmaf(t[u].y, cs[c].x, t[u].x)) < lim);
        }
        wave_lds_sync();
        return;
    }
    const float lim_in = lim * (1.0f + 1e-4f);  // filter margin: keeps borderline pairs
    const float d = cq - lim_in;
    const u64 in = live & (ballot(d < 0.0f) | ballot(d * d < fmaf(aq, aq, bq * bq)));
    const float mg = 4e-6f * (cq + fabsf(aq) + fabsf(bq));
    const float room = cq - lim;  // d2 < lim where Aq cos + Bq sin < -room
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const float2 mid = k.mid[(first + stride * c) >> 6];
        const float v = fmaf(aq, mid.x, bq * mid.y);            // at the middle
        const float s = fabsf(fmaf(bq, mid.x, -(aq * mid.y)));  // |slope| there
        const float vt = v * k.tw, ends = fmaf(v, k.cw, room), lift = fmaf(s, k.sw, k.sb);
        const u64 peak = ballot(s <= vt), dip = ballot(s <= -vt);  // inside the arc
        const u64 whole = in & ~peak & ballot(ends + lift < -mg);
        const u64 hit = in & (dip | ballot(ends - lift < mg));
        if (whole != 0ull) bumped[c] = ~0ull;
        if (bumped[c] == ~0ull) continue;
        // the pairs that reach into the slot first, the others' places with one that
        // bumps nothing; then four at a time
        const int cnt = __popcll(hit);
        const bool mine = inverse_ballot(hit);
        const int at = mine ? mbcnt(hit) : cnt + mbcnt(~hit);
        bl->coef[at] = make_float4(mine ? cq : 3e38f, mine ? aq : 0.0f, mine ? bq : 0.0f, 0.0f);
        wave_lds_sync();
        for (int p = 0; p < cnt; p += 4) {
            const float4 *t = bl->coef + p;
#pragma unroll
            for (int u = 0; u < 4; ++u)
                bumped[c] |= ballot(fmaf(t[u].z, cs[c].y, fmaf(t[u].y, cs[c].x, t[u].x)) < lim);
        }
        wave_lds_sync();
    }
}

template <int NS, int C, class Split>
__device__ int torsion_decide(Pose<NS> &Y, int n, const u64 *mrow, int a, int b,
                              const u64 *far, const int (&toff)[NS], float4 *rec,
                              uint16_t *cand, const float2 (&cs)[C], const Split &sp,
                              long long &nscored) {
    const int lane = lane_id();
    const TorsionArgs &g = fresh_args().t;
    const Axis A = bond_axis(Y, a, b);
    u64 mw[NS];
    int m = 0;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        mw[s] = uniform_u64(mrow[s]);
        m += __popcll(mw[s]);
    }
    // moving-atom frames -> LDS (grid units), static atoms -> registers
    float sgx[NS], sgy[NS], sgz[NS];
    float hgt[NS], rad[NS];  // height along the axis and distance from it, grid units
    u64 stm[NS];             // static atoms of each slot as wave masks (bit = lane)
    bool out_any = false;    // a moving atom's circle leaves [0, n-2]
    int before = 0;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const int i = lane + 64 * s;
        const bool mv = inverse_ballot(mw[s]);
        const int left = n - 64 * s;  // atoms of this slot
        stm[s] = ~mw[s] & (left >= 64 ? ~0ull : left > 0 ? (1ull << left) - 1ull : 0ull);
        sgx[s] = (Y.x[s] - g.ox) * g.inv_h;
        sgy[s] = (Y.y[s] - g.oy) * g.inv_h;
        sgz[s] = (Y.z[s] - g.oz) * g.inv_h;
        float px, py, pz, vx, vy, vz, wx, wy, wz;
        torsion_frame(A, Y.x[s], Y.y[s], Y.z[s], px, py, pz, vx, vy, vz, wx, wy, wz);
        rad[s] = ball_radius(fmaf(vx, vx, fmaf(vy, vy, vz * vz))) * g.inv_h;
        hgt[s] = fmaf(A.ux, Y.x[s] - A.ax, fmaf(A.uy, Y.y[s] - A.ay, A.uz * (Y.z[s] - A.az))) * g.inv_h;
        const int q = before + mbcnt(mw[s]);
        if (mv) {
            rec[3 * q + 0] = make_float4((px - g.ox) * g.inv_h, (py - g.oy) * g.inv_h,
                                         (pz - g.oz) * g.inv_h, __int_as_float(toff[s]));
            rec[3 * q + 1] = make_float4(vx * g.inv_h, vy * g.inv_h, vz * g.inv_h,
                                         __int_as_float(i));
            // every candidate of this atom lies on the circle of radius |V| about P0
            const bool in = ball_inside(g, (px - g.ox) * g.inv_h, (py - g.oy) * g.inv_h,
                                        (pz - g.oz) * g.inv_h, rad[s]);
            rec[3 * q + 2] = make_float4(wx * g.inv_h, wy * g.inv_h, wz * g.inv_h, 0.f);
            out_any = out_any || !in;
        }
        before += __popcll(mw[s]);
    }
    const bool all_in = ballot(out_any) == 0ull;

    // Bump Check of every candidate at once: bumped candidates as wave masks (bit =
    // lane) per candidate slot c.  A moving and a static atom come closest to
    // each other at (height difference, radius difference) about the axis; pairs that
    // may come within the bump distance are listed, and the list is tested 64 pairs
    // at a time, a lane per pair (bump_pairs).  The filter's limit is above what
    // the roundings of both forms of the distance can differ by: Cq is up to about
    // (2 |V|)^2, its terms round at 2^-24 of that; and P0 rounds at the coordinates' own
    // magnitude, which the axial form does not (see torsion_args).
    u64 bumped[C];
#pragma unroll
    for (int c = 0; c < C; ++c) bumped[c] = 0ull;
    const float lim = g.lim;
    const u64 every = g.prune ? 0ull : ~0ull;
    BumpLds *bl = (BumpLds *)cand;
    // (a moving atom within the bump distance of the lane's is at most twice as far
    // from the axis atom, and a bump distance)
    float reach[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s)
        reach[s] = fmaf(fmaf(rad[s], rad[s], hgt[s] * hgt[s]), 1e-4f, g.reach);
    wave_lds_sync();  // the frames
    // the moving atoms in order: their bits, and each one's far row a step ahead
    int q = 0, sw = 0;
    u64 bits = mw[0];
    auto next_atom = [&]() -> int {
#pragma unroll
        for (int s = 1; s < NS; ++s)
            if (bits == 0ull && sw < s) {
                sw = s;
                bits = mw[s];
            }
        const int l = bits != 0ull ? __ffsll((long long)bits) - 1 : 0;
        bits &= bits - 1ull;
        return l + 64 * sw;
    };
    int i = next_atom();
    u64 fw[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) fw[s] = far[i * NS + s];
    if (m <= kBumpDirect && every == 0ull) {
        for (; q < m; ++q) {
            const float4 r0 = rec[3 * q + 0], r1 = rec[3 * q + 1], r2 = rec[3 * q + 2];
            u64 fi[NS];
            i = next_atom();
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                fi[s] = fw[s];
                fw[s] = far[i * NS + s];
            }
            const float vv = fmaf(r1.x, r1.x, fmaf(r1.y, r1.y, r1.z * r1.z));
            const float lim_in = lim * (1.0f + 1e-4f);
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                const u64 elm = uniform_u64(fi[s]) & stm[s];
                if (elm == 0ull) continue;
                const float dx = r0.x - sgx[s], dy = r0.y - sgy[s], dz = r0.z - sgz[s];
                const float cq = fmaf(dx, dx, fmaf(dy, dy, fmaf(dz, dz, vv)));
                const float aq = 2.0f * fmaf(dx, r1.x, fmaf(dy, r1.y, dz * r1.z));
                const float bq = 2.0f * fmaf(dx, r2.x, fmaf(dy, r2.y, dz * r2.z));
                const float e = cq - lim_in;
                u64 bal = elm & (ballot(e < 0.0f) | ballot(e * e < fmaf(aq, aq, bq * bq)));
                while (bal != 0ull) {
                    const int p = __ffsll((long long)bal) - 1;
                    bal &= bal - 1ull;
                    const float c0 = read_lane(cq, p), a0 = read_lane(aq, p), b0 = read_lane(bq, p);
#pragma unroll
                    for (int c = 0; c < C; ++c)
                        bumped[c] |= ballot(fmaf(b0, cs[c].y, fmaf(a0, cs[c].x, c0)) < lim);
                }
            }
        }
    }
    int np = 0;
    while (q < m || np > 0) {
        while (q < m && np < 64) {
            float hi = read_lane(hgt[0], i & 63), ri = read_lane(rad[0], i & 63);
#pragma unroll
            for (int s = 1; s < NS; ++s)
                if ((i >> 6) == s) {
                    hi = read_lane(hgt[s], i & 63);
                    ri = read_lane(rad[s], i & 63);
                }
            u64 fi[NS];
            i = next_atom();
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                fi[s] = fw[s];
                fw[s] = far[i * NS + s];
            }
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                // static atoms of slot s at least bmin bonds from the moving atom
                const float dh = hgt[s] - hi, dr = rad[s] - ri;
                const u64 near = every | ballot(fmaf(dh, dh, dr * dr) < reach[s]);
                const u64 bal = uniform_u64(fi[s]) & stm[s] & near;
                if (bal == 0ull) continue;
                if (inverse_ballot(bal))
                    bl->pair[np + mbcnt(bal)] = (uint16_t)((q << 8) | (lane + 64 * s));
                np += __popcll(bal);
            }
            ++q;
        }
        if (np > 0) {
            const int cnt = np < 64 ? np : 64;
            np -= cnt;
            wave_lds_sync();
            bump_pairs<NS, C>(cnt, bl->pair + np, bl, rec, sgx, sgy, sgz, cs, sp.first(),
                              sp.stride(), g, bumped);
        }
    }
    // Only the bump-free candidates are scored (on the paper's workloads more than
    // half are bumped): list them for this wave, then score the list.  Without
    // pruning every candidate is listed and scored, the bumped ones flagged.
    const DockArgs &ks = fresh_args();
    const TorsionArgs &sa = ks.t;
    const Tri tr = make_tri(ks.g);
    int nfree = 0;
    const u64 flagged = sa.prune ? 0ull : ~0ull;
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const int k0 = sp.first() + sp.stride() * c, left = sa.T - k0;
        const u64 real = left >= 64 ? ~0ull : left > 0 ? (1ull << left) - 1ull : 0ull;
        const u64 bm = real & (~bumped[c] | flagged);
        if (inverse_ballot(bm))
            cand[nfree + mbcnt(bm)] =
                (uint16_t)(k0 + lane + (inverse_ballot(bumped[c]) ? kCandBumped : 0));
        nfree += __popcll(bm);
    }
    wave_lds_sync();
    nscored += (long long)nfree * m;
    u64 best = 0ull;
    if (nfree > 0)
        best = all_in ? score_free_any<C, true>(nfree, cand, rec, m, sa.tors, tr)
                      : score_free_any<C, false>(nfree, cand, rec, m, sa.tors, tr);
    best = sp.reduce(best);
    const int kstar = best == 0ull ? (int)kTraceNone : (int)key_index(best);
    wave_lds_sync();  // rec is rewritten next
    if (kstar != (int)kTraceNone) {
        const float2 t = ld_cs((cfloat2_p)sa.tors, uniform_int(kstar));
        apply_torsion(Y, mrow, A, t.x, t.y);  // the pose is unchanged since A was taken
    }
    return kstar;
}

// Score of the pose: sum over atoms of the grid of the atom's type.
template <int NS>
__device__ __forceinline__ float pose_score(const Pose<NS> &Y, int n, const int (&toff)[NS],
                                            const Tri &tr, const GridArgs &g) {
    const int lane = lane_id();
    float s = 0.f;
#pragma unroll
    for (int q = 0; q < NS; ++q) {
        if (lane + 64 * q < n)
            s += tri_v(tr, (Y.x[q] - g.ox) * g.inv_h, (Y.y[q] - g.oy) * g.inv_h,
                       (Y.z[q] - g.oz) * g.inv_h, (uint32_t)toff[q]);
    }
    return wave_sum(s);
}

// ---------------------------------------------------------------------------
// Shared-memory layout (bytes), identical for host and device.
struct Lds {
    static __host__ __device__ size_t xyzt(int nmax) { return 0; }
    static __host__ __device__ size_t far(int nmax) { return (size_t)nmax * 16; }
    static __host__ __device__ size_t mask(int nmax, int nw) {
        return far(nmax) + (size_t)nmax * nw * 8;
    }
    static __host__ __device__ size_t rot(int nmax, int nw) {
        return mask(nmax, nw) + (size_t)kMaxRot * nw * 8;
    }
    static __host__ __device__ size_t misc(int nmax, int nw) {
        return rot(nmax, nw) + (size_t)kMaxRot * 8;
    }
    static __host__ __device__ size_t rec(int nmax, int nw) { return misc(nmax, nw) + 16; }
    // per wave: moving-atom frames (3 float4 per atom), then the list of
    // bump-free torsion candidates (u16, up to kMaxTorsionSteps)
    static __host__ __device__ size_t rec_stride(int nmax) {
        return (size_t)nmax * 48 + (size_t)kMaxTorsionSteps * 2;
    }
    static __host__ __device__ size_t cand(int nmax) { return (size_t)nmax * 48; }
};

static inline __host__ __device__ int bin_nmax(int bin) { return 32 * (bin + 1); }
static inline __host__ __device__ int bin_slots(int bin) { return (bin_nmax(bin) + 63) / 64; }

size_t dock_lds_bytes(int nmax, int waves) {
    const int nw = (nmax + 63) / 64;
    return Lds::rec(nmax, nw) + (size_t)waves * Lds::rec_stride(nmax);
}

// Stage ligand l into LDS (whole workgroup).
template <int NS>
__device__ void stage_ligand(unsigned char *smem, int nmax, int l, const LibArgs &lib,
                             const WorkArgs &ws, const GridArgs &g, bool with_far) {
    float4 *xyzt = (float4 *)(smem + Lds::xyzt(nmax));
    u64 *far = (u64 *)(smem + Lds::far(nmax));
    u64 *mask = (u64 *)(smem + Lds::mask(nmax, NS));
    int2 *rot = (int2 *)(smem + Lds::rot(nmax, NS));
    int *misc = (int *)(smem + Lds::misc(nmax, NS));
    const int a0 = lib.atom_off[l], n = lib.atom_off[l + 1] - a0;
    const int r0 = lib.rot_off[l], B = lib.rot_off[l + 1] - r0;
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
        const float *p = lib.xyz + 3 * (size_t)(a0 + i);
        const uint32_t toff = (uint32_t)lib.type[a0 + i] * g.type_bytes;
        xyzt[i] = make_float4(p[0], p[1], p[2], __uint_as_float(toff));
    }
    if (with_far) {
        for (int e = threadIdx.x; e < n * NS; e += blockDim.x) {
            const int i = e / NS, w = e - i * NS;
            far[e] = ws.far[(size_t)(a0 + i) * kFarWords + w];
        }
    }
    for (int e = threadIdx.x; e < B * NS; e += blockDim.x) {
        const int b = e / NS, w = e - b * NS;
        mask[e] = w < lib.mask_words ? lib.rot_mask[(size_t)(r0 + b) * lib.mask_words + w] : 0ull;
    }
    for (int b = threadIdx.x; b < B; b += blockDim.x)
        rot[b] = make_int2(lib.rot_bond[2 * (size_t)(r0 + b)], lib.rot_bond[2 * (size_t)(r0 + b) + 1]);
    if (threadIdx.x == 0) {
        misc[1] = n;
        misc[2] = B;
    }
}

template <int NS>
__device__ __forceinline__ void lane_toff(const float4 *xyzt, int n, int (&toff)[NS]) {
    const int lane = lane_id();
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const int i = lane + 64 * s;
        toff[s] = i < n ? __float_as_int(xyzt[i].w) : 0;
    }
}

static __device__ __forceinline__ size_t trace_base(const LibArgs &lib, const SearchArgs &sa, int l) {
    return (size_t)sa.R * ((size_t)l + (size_t)sa.P * (size_t)lib.rot_off[l]);
}

// ---------------------------------------------------------------------------
// Docking kernel: persistent workgroups pop (ligand, restart-group) items of one
// size bin; each wave docks one restart from the orientation k_align chose.
template <int NS, int C>
__global__ __launch_bounds__(512, C <= 4 ? (NS == 1 ? 5 : 4) : 2) void k_dock(DockArgs args) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int nmax = bin_nmax(args.bin), lst = args.lst;
    const int W = blockDim.x >> 6, wave = threadIdx.x >> 6, lane = lane_id();
    float4 *xyzt = (float4 *)(smem + Lds::xyzt(nmax));
    const u64 *far = (const u64 *)(smem + Lds::far(nmax));
    const u64 *mask = (const u64 *)(smem + Lds::mask(nmax, NS));
    const int2 *rot = (const int2 *)(smem + Lds::rot(nmax, NS));
    int *misc = (int *)(smem + Lds::misc(nmax, NS));
    float4 *rec = (float4 *)(smem + Lds::rec(nmax, NS) + (size_t)wave * Lds::rec_stride(nmax));
    uint16_t *cand = (uint16_t *)((unsigned char *)rec + Lds::cand(nmax));
    float2 cs[C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const int k = lane + 64 * c;
        cs[c] = k < args.sa.T ? args.sa.tors[k] : make_float2(1.f, 0.f);
    }
    const int groups = (args.sa.R + W - 1) / W;
    const long long total = (long long)args.ws.counters[lst] * groups;
    int cur = -1;
    for (;;) {
        const DockArgs &k = fresh_args();
        const GridArgs &g = k.g;
        const SearchArgs &sa = k.sa;
        const LibArgs &lib = k.lib;
        const WorkArgs &ws = k.ws;
        if (threadIdx.x == 0) misc[0] = atomicAdd(&ws.counters[kMaxLists + lst], 1);
        __syncthreads();
        const int item = uniform_int(misc[0]);
        if ((long long)item >= total) break;
        const int li = item / groups, grp = item - li * groups;
        const int l = ws.bin_list[li];
        if (l != cur) {
            stage_ligand<NS>(smem, nmax, l, lib, ws, g, true);
            cur = l;
        }
        __syncthreads();
        const int r = grp * W + uniform_int(wave);
        if (r < sa.R) {
            const int n = uniform_int(misc[1]), B = uniform_int(misc[2]);
            int toff[NS];
            lane_toff(xyzt, n, toff);
            Pose<NS> Y;
            start_pose(Y, xyzt, n, r, g, sa);
            uint16_t *tr_out = ws.rtrace + trace_base(lib, sa, l) + (size_t)r * (1 + sa.P * B);
            // the alignment step was taken by k_align (first trace entry)
            const int o = uniform_int((int)tr_out[0]);
            apply_align(Y, n, o < sa.A * sa.A ? o : 0, sa);
            int d = 1;
            long long nsc = 0;
            for (int p = 0; p < sa.P; ++p) {
                for (int b = 0; b < B; ++b, ++d) {
                    const int2 ab = rot[b];
                    const int k = torsion_decide<NS, C>(Y, n, mask + b * NS, uniform_int(ab.x),
                                                        uniform_int(ab.y), far, toff, rec,
                                                        cand, cs, WaveSplit(), nsc);
                    if (lane == 0) tr_out[d] = (uint16_t)k;
                }
            }
            const DockArgs &ke = fresh_args();
            if (ke.ws.scored && lane == 0) atomicAdd(ke.ws.scored, (unsigned long long)nsc);
            const float sc = pose_score(Y, n, toff, make_tri(ke.g), ke.g);
            if (lane == 0) ke.ws.rscore[(size_t)l * ke.sa.R + r] = sc;
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// Batched rigid alignment (Rigid Rotation of Alg. 1) from sphere shells in LDS.
//
// Every alignment sample of atom a lies on the sphere of radius |Y_a - c| about
// the pose centroid c, and Generate_Starting_Pose puts c at the grid centre for
// every restart and every ligand.  So the grid cells a sample can fall in
// depend only on the atom type and that radius.  At pocket load the shell
// atlas stores, per type and per radius band of kBandWidth cells (thickened by
// kShellPad on both sides), the cells the band crosses as face columns: for
// vertex x-position i of cell row (j,k) the bilinear coefficients of the face
// with corners v(i,j,k), v(i,j+1,k), v(i,j,k+1), v(i,j+1,k+1) (the first half
// of cube (i,j,k)); cell (i,j,k) is the two consecutive columns i and i+1.  A
// row table indexed by (j,k) gives each row's cell range on the low-x and the
// high-x side of the centre.  A workgroup of k_align aligns GR restarts of one
// ligand: per atom one wave streams that atom's band into LDS while the others
// sample the previous one, and all GR * A * A samples of the atom read LDS.  A
// sample whose cell is not in the band reads its cube from global memory; both
// give the same values, and the transform, blend and atom-order sum are those
// of align_pose, so the scores are bit-identical.
// The pad covers the rounding of a sample's distance from the grid centre (the turn
// keeps |r| up to a few ulps: ~1e-4 cells, and pockets whose coordinates round by more
// have no atlas) and the pose centroid's own distance from it: ~1e-5 cells for ligands
// near their frame's origin, more for coordinates far from it; beyond kShellOffset the
// ligand's samples read global memory.
constexpr float kShellPad = 0.02f;
constexpr float kShellOffset = 0.008f;
constexpr float kBandWidth = 0.125f;
constexpr int kShellRowsPerThread = 4;  // atlas kernels: rows per thread of 1024
#ifndef DOCK_SHELL_BATCH
#define DOCK_SHELL_BATCH 2
#endif
constexpr int kShellBatch = DOCK_SHELL_BATCH;  // samples scheduled together

// Of the JM y-rotation slots of a k_align lane, align_global_count(JM) take
// their samples from the cubes in global memory (through L1/L2) instead of the
// LDS band: the value is the same, and the two paths run on separate hardware
// (the LDS versus the vector-memory pipeline), so their sample rates add.  The
// global slots are spread evenly over the JM (is_global_slot).
#ifndef DOCK_ALIGN_GLOBAL_32THS
#define DOCK_ALIGN_GLOBAL_32THS 0
#endif
__host__ __device__ constexpr int align_global_count(int G) {
    return G * DOCK_ALIGN_GLOBAL_32THS / 32;
}
__host__ __device__ constexpr bool is_global_slot(int G, int gg) {
    return (gg + 1) * align_global_count(G) / G != gg * align_global_count(G) / G;
}

// Side entry of a row: bits 0-15 first column (relative to the band's columns)
// minus the first cell x plus kEntryBias, so that cell ix of the segment is
// column (e & 0xFFFF) - kEntryBias + ix; bits 16-23 first cell x, 24-31 number
// of cells (0: empty side).
constexpr int kEntryBias = 512;
__device__ __forceinline__ int seg_entry(int base, int lo, int len) {
    return len > 0 ? ((base - lo + kEntryBias) | (lo << 16) | (len << 24)) : kEntryBias;
}

struct RowShell {
    int nlo, nhi, plo, phi;  // cell x ranges, low and high side; empty: lo > hi
    bool merged;             // one segment serves both sides
    __device__ int cols_n() const { return nhi >= nlo ? nhi - nlo + 2 : 0; }
    __device__ int cols_p() const { return (!merged && phi >= plo) ? phi - plo + 2 : 0; }
};

// Cells of row (iy, iz) crossed by the shell rlo <= |p - ec| <= rhi (grid units).
__device__ RowShell shell_row(int iy, int iz, float ecx, float ecy, float ecz, float rlo2,
                              float rhi2, const GridArgs &g) {
    RowShell r{1, 0, 1, 0, false};
    if (iy < 0 || iy > g.ny - 2 || iz < 0 || iz > g.nz - 2) return r;
    const float ya = (float)iy - ecy, yb = ya + 1.0f;
    const float za = (float)iz - ecz, zb = za + 1.0f;
    const float dy0 = ya > 0.0f ? ya : (yb < 0.0f ? -yb : 0.0f);
    const float dz0 = za > 0.0f ? za : (zb < 0.0f ? -zb : 0.0f);
    const float dy1 = fmaxf(fabsf(ya), fabsf(yb)), dz1 = fmaxf(fabsf(za), fabsf(zb));
    const float dmin2 = dy0 * dy0 + dz0 * dz0, dmax2 = dy1 * dy1 + dz1 * dz1;
    if (dmin2 > rhi2) return r;
    const float xa = sqrtf(fmaxf(rlo2 - dmax2, 0.0f)), xb = sqrtf(rhi2 - dmin2);
    r.nlo = max((int)floorf(ecx - xb), 0);
    r.nhi = min((int)floorf(ecx - xa), g.nx - 2);
    r.plo = max((int)floorf(ecx + xa), 0);
    r.phi = min((int)floorf(ecx + xb), g.nx - 2);
    if (r.nlo > r.nhi) {  // only the high side: keep it as the segment of both sides
        r.nlo = r.plo;
        r.nhi = r.phi;
        r.merged = true;
    } else if (r.plo > r.phi) {
        r.merged = true;
    } else if (r.nhi + 1 >= r.plo) {
        r.nhi = max(r.nhi, r.phi);
        r.merged = true;
    }
    return r;
}

// Whether a pose turns about the grid centre: its centroid (grid units) is within
// `limit` of it.
__device__ __forceinline__ bool centred(const GridArgs &g, float ex, float ey, float ez,
                                        float limit) {
    const float x = ex - g.acx, y = ey - g.acy, z = ez - g.acz;
    return fmaf(x, x, fmaf(y, y, z * z)) <= limit * limit;
}

struct BandGeom {
    int y0, z0, thy, thz;
    float rlo2, rhi2;
};

__device__ __forceinline__ BandGeom band_geom(int b, float ecy, float ecz) {
    BandGeom q;
    const float rlo = fmaxf((float)b * kBandWidth - kShellPad, 0.0f);
    const float rhi = (float)(b + 1) * kBandWidth + kShellPad;
    q.rlo2 = rlo * rlo;
    q.rhi2 = rhi * rhi;
    q.y0 = (int)floorf(ecy - rhi) - 1;
    q.z0 = (int)floorf(ecz - rhi) - 1;
    q.thy = (int)floorf(ecy + rhi) + 1 - q.y0 + 1;
    q.thz = (int)floorf(ecz + rhi) + 1 - q.z0 + 1;
    return q;
}

// Atlas pass 1 (one workgroup of 1024 per band): band geometry and column count.
// info[2b] = (y0, z0, thy, thz), info[2b+1] = (rows, ncols or -1, table bytes, 0);
// pass 2 sets info[2b+1].w to the band's row split (see k_atlas_fill).
__global__ __launch_bounds__(1024) void k_atlas_count(GridArgs g, int4 *info) {
    __shared__ int wsum[16];
    const int b = blockIdx.x, tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
    const BandGeom q = band_geom(b, g.acy, g.acz);
    const int rows = q.thy * q.thz;
    const int per = (rows + (int)blockDim.x - 1) / (int)blockDim.x;
    int local = 0;
    if (per <= kShellRowsPerThread) {
        for (int k = 0; k < per; ++k) {
            const int t = tid * per + k;
            if (t < rows) {
                const RowShell r = shell_row(q.y0 + t / q.thz, q.z0 + t % q.thz, g.acx, g.acy,
                                             g.acz, q.rlo2, q.rhi2, g);
                local += r.cols_n() + r.cols_p();
            }
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) local += __shfl_xor(local, o, 64);
    if (lane == 0) wsum[wave] = local;
    __syncthreads();
    if (tid == 0) {
        int total = 0;
        for (int w = 0; w < (int)(blockDim.x >> 6); ++w) total += wsum[w];
        // entries hold (first column - first cell + kEntryBias) in 16 bits
        const bool ok = per <= kShellRowsPerThread && total < (1 << 15);
        info[2 * b] = make_int4(q.y0, q.z0, q.thy, q.thz);
        info[2 * b + 1] = make_int4(rows, ok ? total : -1, (rows * 8 + 15) & ~15, 0);
    }
}

// Atlas pass 2 (one workgroup of 1024 per (type, band)): the row table and the
// face columns of the band, from the cell cubes.  blob16[t*nb + b] is the
// band's offset in float4 units.  The columns are stored row by row, so the
// column index C1 at which the first row starts whose columns begin at or past
// half the band splits it into two chunks, each a run of whole rows (both
// columns of every cell in one chunk); the type-0 workgroup writes C1 into
// info[2b+1].w (k_align streams a band larger than its LDS region in two
// chunks of the same table).
__global__ __launch_bounds__(1024) void k_atlas_fill(GridArgs g, int4 *info,
                                                     const int *blob16, float4 *atlas, int nb) {
    __shared__ int pre[kShellRowsPerThread * 1024 + 1];
    __shared__ int wsum[16];
    const int t = blockIdx.x / nb, b = blockIdx.x - t * nb;
    const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6, BD = blockDim.x;
    const int4 i1 = info[2 * b + 1];
    if (i1.y < 0) return;
    const BandGeom q = band_geom(b, g.acy, g.acz);
    const int rows = i1.x, per = (rows + BD - 1) / BD;
    int2 *table = (int2 *)(atlas + blob16[blockIdx.x]);
    float4 *col = atlas + blob16[blockIdx.x] + i1.z / 16;
    int cnt[kShellRowsPerThread];
    int local = 0;
#pragma unroll
    for (int k = 0; k < kShellRowsPerThread; ++k) {
        cnt[k] = 0;
        const int r = tid * per + k;
        if (k < per && r < rows) {
            const RowShell s = shell_row(q.y0 + r / q.thz, q.z0 + r % q.thz, g.acx, g.acy, g.acz,
                                         q.rlo2, q.rhi2, g);
            cnt[k] = s.cols_n() + s.cols_p();
        }
        local += cnt[k];
    }
    int incl = local;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_up(incl, o, 64);
        if (lane >= o) incl += v;
    }
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    int run = incl - local;
    for (int w = 0; w < wave; ++w) run += wsum[w];
#pragma unroll
    for (int k = 0; k < kShellRowsPerThread; ++k) {
        const int r = tid * per + k;
        if (k < per && r < rows) {
            pre[r] = run;
            const RowShell s = shell_row(q.y0 + r / q.thz, q.z0 + r % q.thz, g.acx, g.acy, g.acz,
                                         q.rlo2, q.rhi2, g);
            const int cn = s.cols_n();
            const int en = seg_entry(run, s.nlo, cn > 0 ? s.nhi - s.nlo + 1 : 0);
            const int ep = s.merged ? en
                                    : seg_entry(run + cn, s.plo, s.phi >= s.plo ? s.phi - s.plo + 1 : 0);
            table[r] = make_int2(en, ep);
            run += cnt[k];
        }
    }
    __syncthreads();
    if (t == 0) {
        // C1 = pre[r] for the first row r with pre[r] >= ncols / 2 (a row boundary)
        for (int r = tid; r < rows; r += BD) {
            const bool first = pre[r] >= i1.y / 2 && (r == 0 || pre[r - 1] < i1.y / 2);
            if (first) info[2 * b + 1].w = pre[r];
        }
    }
    for (int v = tid; v < i1.y; v += BD) {
        int lo = 0, hi = rows - 1;  // last row whose first column is <= v
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (pre[mid] <= v) lo = mid;
            else hi = mid - 1;
        }
        const int iy = q.y0 + lo / q.thz, iz = q.z0 + lo % q.thz;
        const RowShell s = shell_row(iy, iz, g.acx, g.acy, g.acz, q.rlo2, q.rhi2, g);
        const int u = v - pre[lo], cn = s.cols_n();
        const int i = u < cn ? s.nlo + u : s.plo + (u - cn);
        const size_t e = ((size_t)t * g.nz * g.ny + (size_t)iz * g.ny + iy) * g.nx + i;
        col[v] = g.cubes[2 * e];
    }
}

// Shared-memory layout of k_align (bytes); GR restarts per item.
struct AlignLds {
    static __host__ __device__ size_t xyzt() { return 0; }                  // [nmax] x,y,z,toff
    static __host__ __device__ size_t dxyz(int nmax) { return (size_t)nmax * 16; }  // X - c0, toff
    static __host__ __device__ size_t ectr(int nmax) { return dxyz(nmax) + (size_t)nmax * 16; }
    static __host__ __device__ size_t ainf(int nmax, int GR) {
        return ectr(nmax) + (size_t)GR * 32;  // [GR] centroid (world), centroid (grid units)
    }
    static __host__ __device__ size_t misc(int nmax, int GR) { return ainf(nmax, GR) + (size_t)nmax * 32; }
    static __host__ __device__ size_t best(int nmax, int GR) { return misc(nmax, GR) + 128; }
    static __host__ __device__ size_t region(int nmax, int GR) {
        return (best(nmax, GR) + (size_t)GR * 8 + 15) & ~(size_t)15;
    }
};

struct Shell {
    int y0, z0, thy, thz, rows, maxcol;
    float cx;             // centre x (grid units): side of a sample
    unsigned koff;        // absolute row index y0*thz + z0 of the first row
    const int2 *table;    // [thy*thz] (low-side entry, high-side entry)
    const float4 *col;    // face columns
    const float4 *zero;   // two zero columns: a miss blends to +0
    // The same band as LDS byte addresses, for the in-grid sample paths (unsigned
    // arithmetic, so an address below the region start wraps and wraps back):
    uint32_t t0b;         // absolute row 0 (the table's first row less koff rows)
    uint32_t tlob, thib;  // the table's first and last rows
    uint32_t colb;        // column c at colb + 16 (c + kEntryBias)
    uint32_t cmaxb;       // maxcol + kEntryBias
    uint32_t zerob;       // the zero pair
};

// LDS byte address of a pointer into shared memory, and loads from one.
typedef int lds_i32x2 __attribute__((ext_vector_type(2)));
typedef float lds_f32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint32_t lds_addr(const void *p) {
    return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void *)p;
}
__device__ __forceinline__ int2 lds_ld_int2(uint32_t a) {
    const lds_i32x2 v = *(const __attribute__((address_space(3))) lds_i32x2 *)a;
    return make_int2(v.x, v.y);
}
__device__ __forceinline__ float4 lds_ld_float4(uint32_t a) {
    const lds_f32x4 v = *(const __attribute__((address_space(3))) lds_f32x4 *)a;
    return make_float4(v.x, v.y, v.z, v.w);
}

// Byte-address fields of a shell whose table starts at LDS address table_b and
// whose column c lies at col_b + 16 c (rows, koff, maxcol already set).
__device__ __forceinline__ void shell_bytes(Shell &s, uint32_t table_b, uint32_t col_b) {
    s.tlob = table_b;
    s.thib = table_b + 8u * (uint32_t)(s.rows - 1);
    s.t0b = table_b - 8u * s.koff;
    // wave-uniform and opaque, so that a column address stays one shift-and-add
    // of the index
    s.colb = (uint32_t)uniform_int((int)(col_b - 16u * (uint32_t)kEntryBias));
    asm volatile("" : "+s"(s.colb));
    s.cmaxb = (uint32_t)(s.maxcol + kEntryBias);
}

// x clamped to [lo, hi] in one instruction (lo <= hi).
__device__ __forceinline__ uint32_t med3_u32(uint32_t x, uint32_t lo, uint32_t hi) {
    uint32_t r;
    asm("v_med3_u32 %0, %1, %2, %3" : "=v"(r) : "v"(x), "v"(lo), "v"(hi));
    return r;
}

// Low 16 bits of a row entry pair's entry on the sample's side of the centre
// (e.x when gx < cx, else e.y; cx wave-uniform): the compare, then one
// sub-dword select that takes the low halves of both operands.
__device__ __forceinline__ uint32_t side_lo16(int2 e, float gx, float cx) {
    uint32_t r;
    asm("v_cmp_gt_f32 vcc, %3, %4\n\t"
        "v_cndmask_b32_sdwa %0, %2, %1, vcc dst_sel:DWORD dst_unused:UNUSED_PAD "
        "src0_sel:WORD_0 src1_sel:WORD_0"
        : "=v"(r)
        : "v"(e.x), "v"(e.y), "s"(cx), "v"(gx)
        : "vcc");
    return r;
}

__device__ __forceinline__ float lerp_cell(const float4 *p, float fx, float fy, float fz) {
    return tri_blend(p[0], p[1], fx, fy, fz);
}

// Column pair of cell x index ix in row entry pair e2 (side by gx), or the zero
// pair when the cell is not in the shell.
__device__ __forceinline__ const float4 *shell_cols(const Shell &s, int2 e2, float gx, int ix,
                                                    bool &hit) {
    const unsigned e = (unsigned)(gx < s.cx ? e2.x : e2.y);
    const int d = ix - (int)((e >> 16) & 255u);
    hit = (unsigned)d < (e >> 24);
    return hit ? s.col + ((int)(e & 0xFFFFu) - kEntryBias + ix) : s.zero;
}

// Trilinear sample of grid coordinates (gx,gy,gz) from the shell, for an atom
// whose sphere may leave the grid: the clamps of tri_u, the row range and the
// segment are checked, and a cell not in the shell gives +0 and hit = false.
// Same arithmetic as tri_u.
__device__ __forceinline__ float shell_sample(const Shell &s, const Tri &t, float gx, float gy,
                                              float gz, bool &hit) {
    const float cx = __builtin_amdgcn_fmed3f(gx, 0.0f, t.mx);
    const float cy = __builtin_amdgcn_fmed3f(gy, 0.0f, t.my);
    const float cz = __builtin_amdgcn_fmed3f(gz, 0.0f, t.mz);
    const float ix = floorf(__builtin_amdgcn_fmed3f(gx, 0.0f, t.m2x));
    const float iy = floorf(__builtin_amdgcn_fmed3f(gy, 0.0f, t.m2y));
    const float iz = floorf(__builtin_amdgcn_fmed3f(gz, 0.0f, t.m2z));
    const int jy = (int)iy - s.y0, kz = (int)iz - s.z0;
    const bool rin = (unsigned)jy < (unsigned)s.thy && (unsigned)kz < (unsigned)s.thz;
    const unsigned ri = min((unsigned)(__mul24(jy, s.thz) + kz), (unsigned)s.rows - 1u);
    int2 e2 = s.table[ri];
    e2.x &= 0 - (int)rin;
    e2.y &= 0 - (int)rin;
    return lerp_cell(shell_cols(s, e2, gx, (int)ix, hit), cx - ix, cy - iy, cz - iz);
}

// One batch of kShellBatch samples (y slots j0..) of a sphere inside the grid,
// in phases so that a wave keeps every sample's reads in flight together:
// fractions and row entries, then the cell columns (LDS band, or the cube in
// global memory for the slots is_global_slot picks), then the blends.  Each
// value is the one tri_in gives.  Every sample lies in [0, n-2] on each axis, so
// the clamps of tri_u are the identity, floor is truncation and the fraction is
// exact as v_fract.  A sample's distance to the grid centre differs from the
// atom's radius by FP32 rounding only (~1e-4 cells, against kShellPad), so by
// construction of the band its row lies in the table and its cell in the row's
// segment on its side of the centre (two separate segments are more than a cell
// apart): the row and column indices are only clamped, to keep reads in bounds.
// fy is the fraction of gy and rowy the byte address of row (int) gy * thz of
// the table (both per atom); the indices are LDS byte addresses.
template <int JM>
__device__ __forceinline__ void shell_batch_in(float (&v)[kShellBatch], int j0, const Shell &s,
                                               const Tri &t, const float (&gx)[kShellBatch],
                                               float gy, float fy, uint32_t rowy,
                                               const float (&gz)[kShellBatch], int to) {
    float fx[kShellBatch], fz[kShellBatch];
    uint32_t off[kShellBatch];
    int2 e2[kShellBatch];
#pragma unroll
    for (int k = 0; k < kShellBatch; ++k) {
        fx[k] = __builtin_amdgcn_fractf(gx[k]);
        fz[k] = __builtin_amdgcn_fractf(gz[k]);
        if (is_global_slot(JM, j0 + k)) {
            off[k] = in_cell(t, gx[k], gy, gz[k]);
        } else {
            // absolute row iy*thz + iz, clamped to the table's rows
            e2[k] = lds_ld_int2(med3_u32(rowy + ((uint32_t)(int)gz[k] << 3), s.tlob, s.thib));
        }
    }
    // every row read is issued before the first column address waits for one
    __builtin_amdgcn_sched_barrier(0);
    float4 q0[kShellBatch], q1[kShellBatch];
#pragma unroll
    for (int k = 0; k < kShellBatch; ++k) {
        if (is_global_slot(JM, j0 + k)) {
            q0[k] = ldq(t.rs, off[k], to);
            q1[k] = ldq(t.rs, off[k], to + 16);
        } else {
            const uint32_t c = min(side_lo16(e2[k], gx[k], s.cx) + (uint32_t)(int)gx[k], s.cmaxb);
            const uint32_t a = s.colb + (c << 4);
            q0[k] = lds_ld_float4(a);
            q1[k] = lds_ld_float4(a + 16u);
        }
    }
    // every column read is issued before the first blend waits for one
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < kShellBatch; ++k) v[k] = tri_blend(q0[k], q1[k], fx[k], fy, fz[k]);
}

// Per-atom inputs of shell_batch_in / shell_batch_part: the fraction of gy and
// the byte address of table row (int) gy * thz.
__device__ __forceinline__ uint32_t shell_rowy(const Shell &s, float gy) {
    return s.t0b + (__umul24((uint32_t)(int)gy, (uint32_t)s.thz) << 3);
}

// The JM samples of one atom for one lane's strip (restart, x-rotation i, y
// rotations j0 .. j0+JM-1; cj = the (cos, sin) entries from j0), added to acc in
// slot order.  Slots from jw on are past A for every lane of the wave and are
// skipped in whole batches.  A sample whose cell is not in the shell adds +0
// (the exact identity: a sum that starts at +0 never becomes -0) and is redone
// from global memory before any later addition to its accumulator, so every sum
// keeps atom order.
template <int JM, bool Inside>
__device__ __forceinline__ void shell_atom(float (&acc)[JM], const Shell &sh, const Tri &tr,
                                           const XStage &xs, cfloat2_p cj, int jw, float ex,
                                           float ez, int to) {
    if constexpr (Inside) {
        const float fy = __builtin_amdgcn_fractf(xs.gy);
        const uint32_t rowy = shell_rowy(sh, xs.gy);
        // (cos, sin) of the next batch's y rotations, loaded one batch ahead
        float2 cn[kShellBatch];
#pragma unroll
        for (int k = 0; k < kShellBatch; ++k) cn[k] = ld_cs(cj, k);
#pragma unroll
        for (int j0 = 0; j0 < JM; j0 += kShellBatch) {
            if (j0 < jw) {
                float gx[kShellBatch], gz[kShellBatch], v[kShellBatch];
                float2 cc[kShellBatch];
#pragma unroll
                for (int k = 0; k < kShellBatch; ++k) cc[k] = cn[k];
                if (j0 + kShellBatch < JM) {
#pragma unroll
                    for (int k = 0; k < kShellBatch; ++k) cn[k] = ld_cs(cj, j0 + kShellBatch + k);
                }
#pragma unroll
                for (int k = 0; k < kShellBatch; ++k) {
                    gx[k] = align_gx(xs, cc[k], ex);
                    gz[k] = align_gz(xs, cc[k], ez);
                }
                shell_batch_in<JM>(v, j0, sh, tr, gx, xs.gy, fy, rowy, gz, to);
#pragma unroll
                for (int k = 0; k < kShellBatch; ++k) acc[j0 + k] += v[k];
            }
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int jj = 0; jj < JM; ++jj) asm volatile("" : "+v"(acc[jj]));
        return;
    } else {
    bool miss = false;
#pragma unroll
    for (int j0 = 0; j0 < JM; j0 += kShellBatch) {
        if (j0 < jw) {
#pragma unroll
            for (int jj = j0; jj < j0 + kShellBatch; ++jj) {
                const float2 c = ld_cs(cj, jj);
                const float gx = align_gx(xs, c, ex), gz = align_gz(xs, c, ez);
                if (is_global_slot(JM, jj)) {
                    acc[jj] += tri_u(tr, gx, xs.gy, gz, to);
                } else {
                    bool hit;
                    acc[jj] += shell_sample(sh, tr, gx, xs.gy, gz, hit);
                    miss = miss || !hit;
                }
            }
        }
        // keep the scheduler from hoisting every sample's loads (register spills)
        __builtin_amdgcn_sched_barrier(0);
    }
    // materialise the sums here (else the compiler defers them past the branch
    // below and keeps every sample's inputs live)
#pragma unroll
    for (int jj = 0; jj < JM; ++jj) asm volatile("" : "+v"(acc[jj]));
    if (__ballot(miss) != 0ull) {
        // recompute rather than keep the first pass's coordinates live across it
        // (an opaque zero offset stops the compiler merging the two passes)
        int z = 0;
        asm volatile("" : "+v"(z));
#pragma unroll
        for (int jj = 0; jj < JM; ++jj) {
            if (is_global_slot(JM, jj) || jj >= jw) continue;
            const float2 c = ld_cs(cj, jj + z);
            const float gx = align_gx(xs, c, ex), gz = align_gz(xs, c, ez);
            bool hit;
            (void)shell_sample(sh, tr, gx, xs.gy, gz, hit);
            if (!hit) acc[jj] += tri_u(tr, gx, xs.gy, gz, to);
        }
    }
    }
}

// shell_batch_in for a band of which only columns [lo, hi) are resident (a band
// streamed in two chunks of whole rows): a sample whose column lies in the
// resident chunk reads it, the others read the zero pair and add +0.  Each
// sample's column lies in exactly one chunk and the two passes of an atom run
// before the next atom, so every accumulator gets each sample once, in atom
// order, and +0 never changes a sum (sums start at +0 and never become -0).
// plo = lo + kEntryBias and pn = hi - lo: the chunk in biased column indices;
// the chunk test replaces the column clamp of shell_batch_in.
template <int JM>
__device__ __forceinline__ void shell_batch_part(float (&v)[kShellBatch], const Shell &s,
                                                 const float (&gx)[kShellBatch], float fy,
                                                 uint32_t rowy, const float (&gz)[kShellBatch],
                                                 uint32_t plo, uint32_t pn) {
    static_assert(align_global_count(JM) == 0, "no global slots in a chunked band");
    float fx[kShellBatch], fz[kShellBatch];
    int2 e2[kShellBatch];
#pragma unroll
    for (int k = 0; k < kShellBatch; ++k) {
        fx[k] = __builtin_amdgcn_fractf(gx[k]);
        fz[k] = __builtin_amdgcn_fractf(gz[k]);
        e2[k] = lds_ld_int2(med3_u32(rowy + ((uint32_t)(int)gz[k] << 3), s.tlob, s.thib));
    }
    float4 q0[kShellBatch], q1[kShellBatch];
#pragma unroll
    for (int k = 0; k < kShellBatch; ++k) {
        const uint32_t c = side_lo16(e2[k], gx[k], s.cx) + (uint32_t)(int)gx[k];
        const uint32_t a = c - plo < pn ? s.colb + (c << 4) : s.zerob;
        q0[k] = lds_ld_float4(a);
        q1[k] = lds_ld_float4(a + 16u);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < kShellBatch; ++k) v[k] = tri_blend(q0[k], q1[k], fx[k], fy, fz[k]);
}

// shell_atom<JM, true> over the resident chunk [lo, hi) of the atom's band.
template <int JM>
__device__ __forceinline__ void shell_atom_part(float (&acc)[JM], const Shell &sh,
                                                const XStage &xs, cfloat2_p cj, int jw, float ex,
                                                float ez, int lo, int hi) {
    const float fy = __builtin_amdgcn_fractf(xs.gy);
    const uint32_t rowy = shell_rowy(sh, xs.gy);
    const uint32_t plo = (uint32_t)(lo + kEntryBias), pn = (uint32_t)(hi - lo);
#pragma unroll
    for (int j0 = 0; j0 < JM; j0 += kShellBatch) {
        if (j0 < jw) {
            float gx[kShellBatch], gz[kShellBatch], v[kShellBatch];
#pragma unroll
            for (int k = 0; k < kShellBatch; ++k) {
                const float2 c = ld_cs(cj, j0 + k);
                gx[k] = align_gx(xs, c, ex);
                gz[k] = align_gz(xs, c, ez);
            }
            shell_batch_part<JM>(v, sh, gx, fy, rowy, gz, plo, pn);
#pragma unroll
            for (int k = 0; k < kShellBatch; ++k) acc[j0 + k] += v[k];
        }
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int jj = 0; jj < JM; ++jj) asm volatile("" : "+v"(acc[jj]));
}

// Copy by every wave of the workgroup (wave: its wave-uniform index of W): n16
// float4 (a whole number of 64-float4 instructions) from src in global memory to
// dst in LDS with direct global-to-LDS loads, all in flight before one wait; the
// caller's barrier then publishes them.
__device__ __forceinline__ void lds_fill(float4 *dst, const float4 *src, int n16, int wave, int W) {
    const float4 *sl = src + lane_id();
    for (int c = 64 * wave; c < n16; c += 64 * W)
        __builtin_amdgcn_global_load_lds((const void *)(sl + c),
                                         (__attribute__((address_space(3))) void *)(dst + c), 16, 0,
                                         0);
    __builtin_amdgcn_s_waitcnt(0);
}

// Float4 count of the first copy of an atom's band (c0, c1 from k_align's ainf):
// the whole band, or for a band in two chunks its table and first chunk.
__device__ __forceinline__ int band_copy16(const int4 &c0, const int4 &c1) {
    const int C1 = c1.w >> 1;
    return C1 > 0 ? band_padded(c1.z + C1) : band_padded(c0.y);
}

// Persistent workgroups pop (ligand, group of GR restarts) items of one size bin
// and write each restart's best orientation as the first entry of its decision
// trace; k_dock then starts from it.  A lane holds a strip: one restart, one x
// rotation i and JM consecutive y rotations, with JM score accumulators; strips
// are ordered (part of the y range, restart, i).  Per atom a lane rebuilds its
// restart's start-pose offset from the ligand-centred coordinates (the same
// arithmetic as start_pose), applies the x rotation once and then samples the JM
// y rotations.  The last wave streams the next atom's band into LDS.
template <int NS, int JM>
__global__ __launch_bounds__(1024) void k_align(GridArgs g, SearchArgs sa, LibArgs lib, WorkArgs ws,
                                                int bin, int lst, int arena, int GR) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int nmax = bin_nmax(bin);
    const int BD = blockDim.x, W = BD >> 6, tid = threadIdx.x, wave = tid >> 6, lane = lane_id();
    const int A = sa.A, parts = (A + JM - 1) / JM;
    float4 *xyzt = (float4 *)(smem + AlignLds::xyzt());
    float4 *dxyz = (float4 *)(smem + AlignLds::dxyz(nmax));
    float4 *ectr = (float4 *)(smem + AlignLds::ectr(nmax));
    int4 *ainf = (int4 *)(smem + AlignLds::ainf(nmax, GR));  // per atom: band copy, band rows
    int *misc = (int *)(smem + AlignLds::misc(nmax, GR));    // [0] item, bytes 64..95 zero pair
    float4 *zero2 = (float4 *)(smem + AlignLds::misc(nmax, GR) + 64);
    u64 *bestk = (u64 *)(smem + AlignLds::best(nmax, GR));
    float4 *region = (float4 *)(smem + AlignLds::region(nmax, GR));
    const int region16 = (arena - (int)AlignLds::region(nmax, GR)) / 16;
    const uint32_t region_b = lds_addr(region), zero_b = lds_addr(zero2);
    const int wave_u = uniform_int(wave);
    const Tri tr = make_tri(g);
    const int groups = (sa.R + GR - 1) / GR;
    const int Ws = W - 1;  // sampling waves; wave Ws copies bands
    const bool sampler = wave < Ws;
    // strips of one part padded to whole waves, so that j0 is wave-uniform
    const int spp = (GR * A + 63) & ~63, strips = parts * spp;
    if (tid < 2) zero2[tid] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    // Items (ligand of the list, group of GR restarts), one queue per XCD: XCD x
    // (workgroup b runs on XCD b % kXcds, the round-robin dispatch) takes the
    // x-th contiguous share of the list's ligands with all their restart groups,
    // so the groups of a ligand, which copy the same bands, read them through one
    // L2.  A workgroup whose queue is empty takes items from the next queues.
    const long long nl = ws.counters[lst];
    int *qc = ws.counters + 4 * kMaxLists + lst * kXcds;
    int qcur = (int)(blockIdx.x % kXcds), qleft = kXcds;  // thread 0's cursor
    for (;;) {
        if (tid == 0) {
            int qli = -1, qgrp = 0;
            while (qleft > 0) {
                const long long l0 = nl * qcur / kXcds, l1 = nl * (qcur + 1) / kXcds;
                const int got = atomicAdd(&qc[qcur], 1);
                if ((long long)got < (l1 - l0) * groups) {
                    qli = (int)(l0 + got / groups);
                    qgrp = got % groups;
                    break;
                }
                qcur = qcur + 1 == kXcds ? 0 : qcur + 1;
                --qleft;
            }
            misc[0] = qli;
            misc[1] = qgrp;
        }
        __syncthreads();
        const int li = misc[0], grp = misc[1];
        if (li < 0) break;
        const int l = ws.bin_list[li];
        const int a0 = lib.atom_off[l], n = lib.atom_off[l + 1] - a0;
        const int B = lib.rot_off[l + 1] - lib.rot_off[l];
        const int rbase = grp * GR;
        for (int i = tid; i < n; i += BD) {
            const float *p = lib.xyz + 3 * (size_t)(a0 + i);
            const uint32_t toff = (uint32_t)lib.type[a0 + i] * g.type_bytes;
            xyzt[i] = make_float4(p[0], p[1], p[2], __uint_as_float(toff));
        }
        if (tid < GR) bestk[tid] = 0ull;
        __syncthreads();
        if (wave == W - 1) {
            // ligand-centred coordinates X - c0, with the c0 of start_pose
            Pose<NS> X;
#pragma unroll
            for (int q = 0; q < NS; ++q) {
                const int i = lane + 64 * q;
                const float4 v = i < n ? xyzt[i] : make_float4(0.f, 0.f, 0.f, 0.f);
                X.x[q] = v.x;
                X.y[q] = v.y;
                X.z[q] = v.z;
            }
            float c0x, c0y, c0z;
            centroid(X, n, c0x, c0y, c0z);
#pragma unroll
            for (int q = 0; q < NS; ++q) {
                const int i = lane + 64 * q;
                if (i < n)
                    dxyz[i] = make_float4(X.x[q] - c0x, X.y[q] - c0y, X.z[q] - c0z, xyzt[i].w);
            }
        }
        for (int gg = wave; gg < GR; gg += W) {
            // restarts past R (last group) repeat the group's first restart
            const int r = rbase + gg < sa.R ? rbase + gg : rbase;
            Pose<NS> Y;
            start_pose(Y, xyzt, n, r, g, sa);
            float cx, cy, cz;
            centroid(Y, n, cx, cy, cz);
            const float ex = (cx - g.ox) * g.inv_h, ey = (cy - g.oy) * g.inv_h,
                        ez = (cz - g.oz) * g.inv_h;
            if (lane == 0) {
                ectr[2 * gg] = make_float4(cx, cy, cz, 0.0f);
                ectr[2 * gg + 1] = make_float4(ex, ey, ez, 0.0f);
            }
            if (gg != 0) continue;
            // each atom's band in the atlas (radius from the group's first restart); none
            // where the restarts turn about a point so far off the grid centre (by a
            // rotated offset each) that samples may leave the padded band
            const bool on_centre = centred(g, ex, ey, ez, kShellOffset);
#pragma unroll
            for (int q = 0; q < NS; ++q) {
                const int a = lane + 64 * q;
                if (a >= n) continue;
                const float rx = (Y.x[q] - cx) * g.inv_h, ry = (Y.y[q] - cy) * g.inv_h,
                            rz = (Y.z[q] - cz) * g.inv_h;
                const float rg = sqrtf(fmaf(rx, rx, fmaf(ry, ry, rz * rz)));
                const int b = (int)(rg * (1.0f / kBandWidth));
                // clamps are the identity when the sphere stays inside [0, n-2]
                const bool inside = ball_inside(tr, ex, ey, ez, rg);
                int4 c0 = make_int4(-1, 0, 0, 0), c1 = make_int4(0, 0, 0, inside ? 1 : 0);
                if (b < g.nbands && on_centre) {
                    const int4 gi = g.bands[2 * b], gj = g.bands[2 * b + 1];
                    const int size16 = gj.z / 16 + gj.y;
                    const int t = (int)(lib.type[a0 + a]);
                    if (gj.y >= 0 && band_padded(size16) <= region16) {
                        c0 = make_int4(g.blob16[t * g.nbands + b], size16, gi.x, gi.y);
                        c1 = make_int4(gi.z, gi.w, gj.z / 16, inside ? 1 : 0);
                    } else if (gj.y >= 0 && inside && gj.w > 0 &&
                               band_padded(gj.z / 16 + gj.w) <= region16 &&
                               gj.z / 16 + band_padded(gj.y - gj.w) <= region16) {
                        // too large for the region: two chunks of whole rows, columns
                        // [0, C1) and [C1, ncols), each resident with the table
                        // (c1.w: bit 0 inside, bits 1.. C1)
                        c0 = make_int4(g.blob16[t * g.nbands + b], size16, gi.x, gi.y);
                        c1 = make_int4(gi.z, gi.w, gj.z / 16, 1 | (gj.w << 1));
                    }
                }
                ainf[2 * a] = c0;
                ainf[2 * a + 1] = c1;
            }
        }
        __syncthreads();
        for (int sbase = 0; sbase < strips; sbase += Ws * 64) {
            const int wbase = __builtin_amdgcn_readfirstlane(sbase + 64 * wave);
            const int part = wbase / spp, rem = sbase + tid - part * spp;
            const bool sv = sampler && wbase < strips && rem < GR * A;
            const int rr = sv ? rem : 0;  // padding lanes repeat the part's first strip
            const int gg = rr / A, i = rr - gg * A, j0 = part * JM;
            const bool won = sampler && wbase < strips;
            const int jw_part = min(JM, A - j0);
            const int r = rbase + gg < sa.R ? rbase + gg : rbase;
            const float4 m0 = sa.smat[3 * r + 0], m1 = sa.smat[3 * r + 1], m2 = sa.smat[3 * r + 2];
            const float4 cw = ectr[2 * gg], ce = ectr[2 * gg + 1];
            const float2 ci = sa.acs[i];
            const cfloat2_p cj = (cfloat2_p)sa.acs + 2 * j0;
            float acc[JM];
#pragma unroll
            for (int jj = 0; jj < JM; ++jj) acc[jj] = 0.0f;
            // the first atom's band, at the start of the region
            int offA = 0;
            {
                const int4 c0 = ainf[0];
                if (c0.x >= 0) {
                    const int sz = band_copy16(c0, ainf[1]);
                    lds_fill(region, g.atlas + c0.x, sz, wave_u, W);
                }
            }
            __syncthreads();
            for (int a = 0; a < n; ++a) {
                const int4 cn = a + 1 < n ? ainf[2 * (a + 1)] : make_int4(-1, 0, 0, 0);
                const int4 cn1 = a + 1 < n ? ainf[2 * (a + 1) + 1] : make_int4(0, 0, 0, 0);
                const int4 c0 = ainf[2 * a], c1 = ainf[2 * a + 1];
                // A band in two chunks fills the region (its first chunk and table at
                // the start, the second chunk after the table) and is never double
                // buffered.  Where the next band (or first chunk) goes: when both fit,
                // at the other end of the region, streamed by the copier wave while
                // this atom is sampled; else at the start, copied by everyone after the
                // barrier.
                const int C1 = c1.w >> 1;
                const bool two = c0.x >= 0 && C1 > 0;
                const bool next_two = cn.x >= 0 && (cn1.w >> 1) > 0;
                const int sa_ = c0.x >= 0 ? band_padded(c0.y) : 0;
                const int sn = cn.x >= 0 ? band_copy16(cn, cn1) : 0;
                const bool dbl = cn.x >= 0 && !two && !next_two && sa_ + sn <= region16;
                const int offN = dbl ? (offA == 0 ? region16 - sn : 0) : 0;
                if (won) {
                    const float4 d = dxyz[a];
                    const int to = uniform_int(__float_as_int(d.w));
                    // the batch tests j0 < jw are made here, per atom, in scalar
                    // registers (hoisted out of the atom loop they are spilled)
                    int jw = jw_part;
                    asm volatile("" : "+s"(jw));
                    // start-pose offset of this atom for the lane's restart
                    const float yx = fmaf(m0.x, d.x, fmaf(m0.y, d.y, fmaf(m0.z, d.z, g.cx)));
                    const float yy = fmaf(m1.x, d.x, fmaf(m1.y, d.y, fmaf(m1.z, d.z, g.cy)));
                    const float yz = fmaf(m2.x, d.x, fmaf(m2.y, d.y, fmaf(m2.z, d.z, g.cz)));
                    const XStage xs = align_x((yx - cw.x) * g.inv_h, (yy - cw.y) * g.inv_h,
                                              (yz - cw.z) * g.inv_h, ci, ce.y);
                    if (c0.x >= 0) {
                        Shell sh;
                        sh.y0 = c0.z;
                        sh.z0 = c0.w;
                        sh.thy = c1.x;
                        sh.thz = c1.y;
                        sh.rows = c1.x * c1.y;
                        sh.maxcol = c0.y - c1.z - 2;  // last column pair of the band
                        sh.cx = g.acx;
                        sh.koff = (unsigned)(c0.z * c1.y + c0.w);
                        sh.table = (const int2 *)(region + offA);
                        sh.col = region + offA + c1.z;
                        sh.zero = zero2;
                        sh.zerob = zero_b;
                        shell_bytes(sh, region_b + 16u * (uint32_t)offA,
                                    region_b + 16u * (uint32_t)(offA + c1.z));
                        if (two) shell_atom_part<JM>(acc, sh, xs, cj, jw, ce.x, ce.z, 0, C1);
                        else if (c1.w) shell_atom<JM, true>(acc, sh, tr, xs, cj, jw, ce.x, ce.z, to);
                        else shell_atom<JM, false>(acc, sh, tr, xs, cj, jw, ce.x, ce.z, to);
                    } else if (c1.w) {
#pragma unroll
                        for (int jj = 0; jj < JM; ++jj) {
                            if (jj >= jw) break;
                            const float2 c = ld_cs(cj, jj);
                            acc[jj] += tri_in(tr, align_gx(xs, c, ce.x), xs.gy,
                                              align_gz(xs, c, ce.z), to);
                        }
                    } else {
#pragma unroll
                        for (int jj = 0; jj < JM; ++jj) {
                            if (jj >= jw) break;
                            const float2 c = ld_cs(cj, jj);
                            acc[jj] += tri_u(tr, align_gx(xs, c, ce.x), xs.gy,
                                             align_gz(xs, c, ce.z), to);
                        }
                    }
                } else if (wave == Ws && dbl) {
                    // copier wave: global -> LDS loads, 64 float4 per instruction (band
                    // sizes are padded to whole instructions, so every lane stays in
                    // the band's slot), then wait for them before the barrier
                    const float4 *src = g.atlas + cn.x + lane;
                    for (int c = 0; c < sn; c += 64)
                        __builtin_amdgcn_global_load_lds(
                            (const void *)(src + c),
                            (__attribute__((address_space(3))) void *)(region + offN + c), 16, 0, 0);
                    __builtin_amdgcn_s_waitcnt(0);
                }
                __syncthreads();  // every sample of atom a has read the region
                if (two) {
                    // second chunk: columns [C1, ncols) after the table, then the
                    // samples whose columns lie there
                    const int nB = band_padded(c0.y - c1.z - C1);
                    lds_fill(region + c1.z, g.atlas + c0.x + c1.z + C1, nB, wave_u, W);
                    __syncthreads();
                    if (won) {
                        const float4 d = dxyz[a];
                        int jw = jw_part;
                        asm volatile("" : "+s"(jw));
                        const float yx = fmaf(m0.x, d.x, fmaf(m0.y, d.y, fmaf(m0.z, d.z, g.cx)));
                        const float yy = fmaf(m1.x, d.x, fmaf(m1.y, d.y, fmaf(m1.z, d.z, g.cy)));
                        const float yz = fmaf(m2.x, d.x, fmaf(m2.y, d.y, fmaf(m2.z, d.z, g.cz)));
                        const XStage xs = align_x((yx - cw.x) * g.inv_h, (yy - cw.y) * g.inv_h,
                                                  (yz - cw.z) * g.inv_h, ci, ce.y);
                        Shell sh;
                        sh.y0 = c0.z;
                        sh.z0 = c0.w;
                        sh.thy = c1.x;
                        sh.thz = c1.y;
                        sh.rows = c1.x * c1.y;
                        sh.maxcol = c0.y - c1.z - 2;
                        sh.cx = g.acx;
                        sh.koff = (unsigned)(c0.z * c1.y + c0.w);
                        sh.table = (const int2 *)region;
                        sh.col = region + c1.z - C1;  // column c >= C1 at region + c1.z + (c - C1)
                        sh.zero = zero2;
                        sh.zerob = zero_b;
                        shell_bytes(sh, region_b, region_b + 16u * (uint32_t)(c1.z - C1));
                        shell_atom_part<JM>(acc, sh, xs, cj, jw, ce.x, ce.z, C1, c0.y - c1.z);
                    }
                    __syncthreads();
                }
                if (cn.x >= 0 && !dbl) {  // the next atom's band, at the start
                    lds_fill(region, g.atlas + cn.x, sn, wave_u, W);
                    __syncthreads();
                }
                offA = offN;
            }
            if (sv) {
                // best (score, then lowest index) of the strip, into its restart's slot
                u64 best = 0ull;
#pragma unroll
                for (int jj = 0; jj < JM; ++jj) {
                    const int j = j0 + jj;
                    const u64 key = j < A ? make_key(acc[jj], (uint32_t)(i * A + j)) : 0ull;
                    best = key > best ? key : best;
                }
                atomicMax(&bestk[gg], best);
            }
        }
        __syncthreads();
        if (tid < GR && rbase + tid < sa.R) {
            const int r = rbase + tid;
            ws.rtrace[trace_base(lib, sa, l) + (size_t)r * (1 + sa.P * B)] =
                (uint16_t)key_index(bestk[tid]);
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// Batched rigid alignment by score bounds.
//
// As for the shells, every alignment sample of an atom lies on the sphere of its
// radius r about the grid centre, up to roundings and to twice the distance of the
// start pose's centroid from that centre: zero but for the rounding of the ligand's own
// centroid, which grows with its coordinates.  The bins are padded for kBoundOffset of
// it; restarts farther off score every orientation.  On that sphere a sample is (polar position,
// azimuth phi about the y axis), and the y rotations of a strip (restart, x
// rotation i) only turn phi by 12 degrees each: its 30 samples share the polar
// position and take phi0 + 12 j degrees.  At pocket load k_bounds stores, per
// atom type and radius band, an upper bound of the interpolated grid over each
// (band, polar row, azimuth sub-bin of a 12 degree sector), the 30 sectors of a
// sub-bin side by side: a strip then reads the bounds of all its samples of an
// atom as one run of 30 16-bit integers.
//
// Their sum over the atoms bounds an orientation's score from above.  The
// orientation of the largest bound is scored first; every orientation whose
// bound does not reach that score (less a margin above all roundings) cannot be
// the best one, and the others -- about 2% with bins of a quarter cell -- are
// scored in FP32 as in align_pose: same transform, samples and atom order, so
// the chosen orientation is the same one.
//
// Bound by the texture unit (busy 0.90): reading a record costs its cache line, and a
// line from L2 takes about 2 CU-clocks whatever part of it is used; records and the
// exact scores' cubes are half of it each.  Alignment of 2,500 ligands of 20-80 atoms
// (256 restarts): 13.1 ms, from 30.9 ms in k_align, which samples every orientation
// from LDS.  16,000 ligands of 20-100 atoms: 118 ms from 234 ms.
struct BoundRow {
    float ylo, yhi, rlo, rhi;  // |y| range and range of the distance to the y axis
};

__device__ __forceinline__ float band_top(const BoundArgs &bd, int b) { return bd.edge[b + 1]; }

// Rows are uniform in t = sqrt(1 - |y|/r), which is near the polar angle over the
// whole half sphere (dtheta/dt in [sqrt 2, 2]).  kBoundRowPad covers t's rounding,
// largest at the pole, where 1 - |y|/r cancels.
constexpr float kBoundRowPad = 2e-3f;
constexpr float kBoundPhiPad = 4e-5f;  // turns: bound_sector's error (2e-6) and roundings

__device__ __forceinline__ BoundRow bound_row(float r0, float r1, int row, int rows, float pad) {
    BoundRow q;
    const float t0 = fmaxf((float)row / (float)rows - kBoundRowPad, 0.0f);
    const float t1 = fminf((float)(row + 1) / (float)rows + kBoundRowPad, 1.0f);
    const float u1 = 1.0f - t0 * t0, u0 = 1.0f - t1 * t1;  // |y|/r in [u0, u1]
    const float ra = fmaxf(r0 - pad, 0.0f), rb = r1 + pad;
    q.ylo = u0 * ra - pad;
    q.yhi = u1 * rb + pad;
    q.rlo = fmaxf(ra * sqrtf(fmaxf(1.0f - u1 * u1, 0.0f)) - pad, 0.0f);
    q.rhi = rb * sqrtf(fmaxf(1.0f - u0 * u0, 0.0f)) + pad;
    return q;
}

// Ranges of the sine and the cosine over [a, b] turns (b - a below half a turn, both in
// [-1, 3]), from the hardware sine, whose error is below kBoundSinPad (1.3e-7 at most
// against 64 bits, over 2^24 arguments there).  The sine has its peak in between where the cosine falls
// through zero, its trough where it rises, and so on.
constexpr float kBoundSinPad = 4e-6f;
__device__ __forceinline__ void sin_cos_range(float a, float b, float (&s)[2], float (&c)[2]) {
    const float sa = __builtin_amdgcn_sinf(__builtin_amdgcn_fractf(a)),
                sb = __builtin_amdgcn_sinf(__builtin_amdgcn_fractf(b)),
                ca = __builtin_amdgcn_cosf(__builtin_amdgcn_fractf(a)),
                cb = __builtin_amdgcn_cosf(__builtin_amdgcn_fractf(b));
    s[0] = ca < 0.0f && cb >= 0.0f ? -1.0f : fminf(sa, sb);
    s[1] = ca >= 0.0f && cb < 0.0f ? 1.0f : fmaxf(sa, sb);
    c[0] = sa >= 0.0f && sb < 0.0f ? -1.0f : fminf(ca, cb);
    c[1] = sa < 0.0f && sb >= 0.0f ? 1.0f : fmaxf(ca, cb);
}

// Largest value of the interpolated grid (edge values beyond the box, as the
// clamps of tri_u give) over the box [lo, hi] in grid units, plus the rounding of
// a sample there.  In a cell the interpolant is linear along each axis, so its
// largest value over the box's part of the cell is at one of that part's corners.
// A box of at most a cell's edges (the bins') meets at most one grid plane on each axis:
// the corners of its parts are the 27 points at either end and on that plane, from 27
// values, the same instructions in every lane (cell by cell a wave takes all 8 whenever
// each plane is met in some lane).
// (vals: the type's grid, of fewer than 2^24 values)
__device__ __forceinline__ float box_max(const GridArgs &g, const float *__restrict__ vals,
                                         const float (&lo)[3], const float (&hi)[3]) {
    const int dim[3] = {g.nx, g.ny, g.nz};
    float a[3], b[3], wa[3][3], wb[3][3];
    int c[3];
    bool in[3], small = true;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const float top = (float)(dim[k] - 1);
        a[k] = __builtin_amdgcn_fmed3f(lo[k], 0.0f, top);
        b[k] = __builtin_amdgcn_fmed3f(hi[k], 0.0f, top);
        c[k] = max(min((int)a[k], dim[k] - 3), 0);
        const float ta = a[k] - (float)c[k], tb = b[k] - (float)c[k];
        small = small && dim[k] >= 3 && tb <= 2.0f;
        in[k] = ta < 1.0f && tb > 1.0f;  // meets the plane c + 1
        wa[k][0] = fmaxf(1.0f - ta, 0.0f);
        wa[k][2] = fmaxf(ta - 1.0f, 0.0f);
        wa[k][1] = 1.0f - wa[k][0] - wa[k][2];
        wb[k][0] = fmaxf(1.0f - tb, 0.0f);
        wb[k][2] = fmaxf(tb - 1.0f, 0.0f);
        wb[k][1] = 1.0f - wb[k][0] - wb[k][2];
    }
    float best = -3.4e38f, big = 0.0f;
    if (small) {
        struct Three {
            float v0, v1, v2;
        };
        const uint32_t nx = 4 * (uint32_t)g.nx, slab = nx * (uint32_t)g.ny;  // bytes
        uint32_t row = (uint32_t)c[2] * slab + (uint32_t)c[1] * nx + 4 * (uint32_t)c[0];
        float za[9], zb[9];
#pragma unroll
        for (int e = 0; e < 9; ++e) za[e] = zb[e] = 0.0f;
#pragma unroll
        for (int dz = 0; dz < 3; ++dz) {
            float ya[3], ym[3], yb[3];  // per x point: rows y folded to the three y points
#pragma unroll
            for (int e = 0; e < 3; ++e) ya[e] = ym[e] = yb[e] = 0.0f;
#pragma unroll
            for (int dy = 0; dy < 3; ++dy) {
                const uint32_t at = row + (dy == 0 ? 0u : dy == 1 ? nx : 2 * nx);
                const Three r = *(const Three *)((const char *)vals + at);
                const float v0 = r.v0, v1 = r.v1, v2 = r.v2;
                big = fmaxf(fmaxf(big, fabsf(v0)), fmaxf(fabsf(v1), fabsf(v2)));
                const float xa = fmaf(wa[0][2], v2, fmaf(wa[0][1], v1, wa[0][0] * v0));
                const float xb = fmaf(wb[0][2], v2, fmaf(wb[0][1], v1, wb[0][0] * v0));
                const float x[3] = {xa, in[0] ? v1 : xa, xb};
#pragma unroll
                for (int e = 0; e < 3; ++e) {
                    ya[e] = fmaf(wa[1][dy], x[e], ya[e]);
                    yb[e] = fmaf(wb[1][dy], x[e], yb[e]);
                    if (dy == 1) ym[e] = x[e];
                }
            }
#pragma unroll
            for (int e = 0; e < 3; ++e) {
                const float y[3] = {ya[e], in[1] ? ym[e] : ya[e], yb[e]};
#pragma unroll
                for (int f = 0; f < 3; ++f) {
                    za[3 * e + f] = fmaf(wa[2][dz], y[f], za[3 * e + f]);
                    zb[3 * e + f] = fmaf(wb[2][dz], y[f], zb[3 * e + f]);
                    if (dz == 1 && in[2]) best = fmaxf(best, y[f]);
                }
            }
            row += slab;
        }
#pragma unroll
        for (int e = 0; e < 9; ++e) best = fmaxf(best, fmaxf(za[e], zb[e]));
    } else {
        // any box: the values of all cells it meets bound it
        for (int z = (int)a[2]; z <= min((int)b[2] + 1, dim[2] - 1); ++z)
            for (int y = (int)a[1]; y <= min((int)b[1] + 1, dim[1] - 1); ++y)
                for (int x = (int)a[0]; x <= min((int)b[0] + 1, dim[0] - 1); ++x) {
                    const float v = vals[(z * g.ny + y) * g.nx + x];
                    best = fmaxf(best, v);
                    big = fmaxf(big, fabsf(v));
                }
    }
    // a sample's blend adds terms of up to 9 times the cell's largest value, each
    // rounding at 2^-24, as do the sums above
    return fmaf(big, 2e-5f, best);
}

// One workgroup column per (type, band); a thread per record, its 30 sectors in turn, so
// that the lanes of a wave read neighbouring cells; the records are written from LDS in
// one run.  Bound by the texture unit (9 loads of 3 values an entry): 0.72 ms for the 55
// million entries of 4 types of 96^3 values, 0.89 cell by cell with a thread per entry.
__global__ __launch_bounds__(256) void k_bounds(GridArgs g, BoundArgs bd,
                                                const float *__restrict__ vals,
                                                const uint32_t *__restrict__ mm,
                                                unsigned short *__restrict__ tab) {
    __shared__ __align__(16) unsigned short tile[256 * kBoundRec];
    const int t = blockIdx.y / bd.nb, b = blockIdx.y - t * bd.nb;
    const int4 q = bd.band[b];
    const int rows = q.x, m = q.y, recs = 2 * rows * m;
    uint32_t *out = (uint32_t *)(tab + ((size_t)t * bd.type_bytes + (size_t)q.z) / 2);
    const bool last = b == bd.nb - 1;
    const float r0 = bd.edge[b], r1 = last ? r0 : band_top(bd, b);
    const float sector = 1.0f / (float)kBoundSteps;
    float vlow, step, mag;
    bound_scale(unord_f32(mm[0]), unord_f32(~mm[1]), vlow, step, mag);
    const float inv_step = 1.0f / step;
    vals += (size_t)t * g.nz * g.ny * g.nx;
    for (int base = blockIdx.x * 256; base < recs; base += gridDim.x * 256) {
        const int rec = base + (int)threadIdx.x;
        if (rec < recs) {
            const int row2 = rec / m, f = rec - row2 * m;
            const bool south = row2 >= rows;
            const BoundRow br = bound_row(r0, r1, south ? row2 - rows : row2, rows, bd.pad);
            const float f0 = sector * ((float)f / (float)m) - kBoundPhiPad;
            const float f1 = sector * ((float)(f + 1) / (float)m) + kBoundPhiPad;
            const float side = fmaf(br.rhi, kBoundSinPad, bd.pad);
            unsigned short *at = tile + threadIdx.x * kBoundRec;
            for (int k = 0; k < kBoundSteps; ++k) {
                int v = kBoundMax;
                if (!last) {
                    const float p0 = fmaf(sector, (float)k, f0), p1 = fmaf(sector, (float)k, f1);
                    float sn[2], cs[2];
                    sin_cos_range(p0, p1, sn, cs);
                    const float lo[3] = {g.acx + fminf(br.rlo * sn[0], br.rhi * sn[0]) - side,
                                         g.acy + (south ? -br.yhi : br.ylo),
                                         g.acz + fminf(br.rlo * cs[0], br.rhi * cs[0]) - side};
                    const float hi[3] = {g.acx + fmaxf(br.rlo * sn[1], br.rhi * sn[1]) + side,
                                         g.acy + (south ? -br.ylo : br.yhi),
                                         g.acz + fmaxf(br.rlo * cs[1], br.rhi * cs[1]) + side};
                    const float u = (box_max(g, vals, lo, hi) - vlow) * inv_step;
                    // the integer above u, so that vlow + step * v is not below the maximum
                    v = u > 0.0f ? (u < (float)kBoundMax ? (int)u + 1 : kBoundMax) : 1;
                }
                at[k] = (unsigned short)v;
                if (k < kBoundRec - kBoundSteps) at[k + kBoundSteps] = (unsigned short)v;
            }
        }
        __syncthreads();
        // (an even number of records: whole 32-bit words)
        const int words = min(recs - base, 256) * kBoundRec / 2;
        for (int e = threadIdx.x; e < words; e += 256)
            out[(size_t)base * kBoundRec / 2 + e] = ((const uint32_t *)tile)[e];
        __syncthreads();
    }
}

// Bound by the atomics on three words (14 ns each): a workgroup adds its own once.
__global__ __launch_bounds__(1024) void k_value_range(const float *__restrict__ v, long long n,
                                                      uint32_t *mm) {
    __shared__ uint32_t part[16][3];
    uint32_t hi = 0u, nlo = 0u, bad = 0u;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x) {
        const float x = v[i];
        const uint32_t o = ord_f32(x);
        hi = max(hi, o);
        nlo = max(nlo, ~o);
        bad |= !(fabsf(x) <= 1e30f);
    }
    hi = wave_max_u32(hi);
    nlo = wave_max_u32(nlo);
    bad = wave_max_u32(bad);
    if (lane_id() == 0) {
        part[threadIdx.x >> 6][0] = hi;
        part[threadIdx.x >> 6][1] = nlo;
        part[threadIdx.x >> 6][2] = bad;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        uint32_t m = 0u;
        for (int w = 0; w < (int)(blockDim.x >> 6); ++w) m = max(m, part[w][threadIdx.x]);
        if (m != 0u) atomicMax(&mm[threadIdx.x], m);
    }
}

// Azimuth of (x, z) = rho (sin phi, cos phi) in sectors of 12 degrees, in [0, 30).
// The arc tangent is the polynomial of Abramowitz and Stegun 4.4.47 (1e-5
// radians); the scale is a few ulps short of a full turn so that the sector
// index stays below 30.
__device__ __forceinline__ float bound_sector(float x, float z) {
    constexpr float kTurn = (float)kBoundSteps * (1.0f - 1e-6f);
    constexpr float kRad = kTurn / 6.28318530717959f;
    const float ax = fabsf(x), az = fabsf(z);
    const float mn = fminf(ax, az), mx = fmaxf(fmaxf(ax, az), 1e-20f);
    const float a = mn * __builtin_amdgcn_rcpf(mx), s = a * a;
    float p = fmaf(s, 0.0208351f * kRad, -0.0851330f * kRad);
    p = fmaf(s, p, 0.1801410f * kRad);
    p = fmaf(s, p, -0.3302995f * kRad);
    p = fmaf(s, p, 0.9998660f * kRad);
    p *= a;
    p = ax > az ? 0.25f * kTurn - p : p;
    p = z < 0.0f ? 0.5f * kTurn - p : p;
    return x < 0.0f ? kTurn - p : p;
}

// Record in a band (rows per half sphere, azimuth sub-bins m) of a sample whose place on
// the sphere, before its y rotation, is (rx, gy, qz); k0: its sector.
__device__ __forceinline__ float bound_record(float rx, float gy, float qz, float inv_r,
                                              float rows, float m, float &k0) {
    // t and the sector fraction are below 1 by an ulp at least, so their rows and
    // sub-bins are in range
    const float t = __builtin_amdgcn_sqrtf(fmaxf(fmaf(-fabsf(gy), inv_r, 0.99999988f), 0.0f));
    const float row = floorf(t * rows) + (gy < 0.0f ? rows : 0.0f);
    const float p = bound_sector(rx, qz);
    k0 = floorf(p);
    return fmaf(row, m, floorf((p - k0) * m));
}

// Last band whose lower radius is not above rad.
__device__ __forceinline__ int bound_band(const BoundArgs &bd, float rad) {
    int lo = 0, hi = bd.nb - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (bd.edge[mid] <= rad) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// The smallest bound (an integer) that can be the best score of n atoms, given that some
// orientation scores `got`.  Roundings of the two sums of n terms: their magnitudes add up
// to at most 3 n mag where `got` is not below n vlow (a term is at most mag, and so the
// negative ones at most 2 n mag together), n^2 2^-24 times 3 mag each; below that, every
// orientation's bound is higher.  And of the bound's quantisation.
__device__ __forceinline__ uint32_t bound_least(float got, int n, float vlow, float step,
                                                float mag) {
    const float nf = (float)n;
    const float low = got - fabsf(got) * 1e-5f - nf * nf * 5e-7f * mag - nf * 2e-3f * step;
    const float x = (low - nf * vlow) / step;
    // not above 2, or NaN: every orientation stays
    return x > 2.0f ? (uint32_t)fminf(x, 1e9f) - 1u : 1u;
}

// Orientations that stay, of 900, in alignments of made-up ligands: block (bin, probe) takes
// 32 bin + 24 atoms of random types in a ball of 1.1 n^0.4 A, as wide as molecules of
// n heavy atoms are, and adds their number to stay[bin].
__global__ __launch_bounds__(960) void k_bound_probe(GridArgs g, BoundArgs bd,
                                                     const uint32_t *__restrict__ mm,
                                                     int *__restrict__ stay) {
    __shared__ float4 unit[kMaxAtoms], band[kMaxAtoms];  // as k_align_bound; band.w: cubes' type
    __shared__ u64 key[15];
    __shared__ float part[15];
    const int bin = blockIdx.x / kBoundProbes, n = 32 * bin + 24;
    const int tid = threadIdx.x, wave = tid >> 6;
    float vlow, step, mag;
    bound_scale(unord_f32(mm[0]), unord_f32(~mm[1]), vlow, step, mag);
    if (tid < n) {
        uint32_t h = ((uint32_t)blockIdx.x * kMaxAtoms + (uint32_t)tid) * 2654435761u + 12345u;
        auto next = [&]() -> float {  // in [0, 1)
            h ^= h >> 16;
            h *= 0x7feb352du;
            h ^= h >> 15;
            h *= 0x846ca68bu;
            h ^= h >> 16;
            return (float)(h >> 8) * (1.0f / 16777216.0f);
        };
        const float rad = 1.1f * powf((float)n, 0.4f) * g.inv_h * cbrtf(next());
        const float z = 2.0f * next() - 1.0f, w = sqrtf(fmaxf(1.0f - z * z, 0.0f)), phi = next();
        const int type = min((int)(next() * (float)g.ntypes), g.ntypes - 1);
        const int4 bq = bd.band[bound_band(bd, rad)];
        unit[tid] = make_float4(rad * w * __builtin_amdgcn_cosf(phi), rad * w * __builtin_amdgcn_sinf(phi),
                                rad * z, rad > 1e-6f ? 1.0f / rad : 0.0f);
        band[tid] = make_float4((float)bq.x, (float)bq.y,
                                __uint_as_float((uint32_t)type * bd.type_bytes + (uint32_t)bq.z),
                                __uint_as_float((uint32_t)type * g.type_bytes));
    }
    __syncthreads();
    const bool real = tid < kBoundSteps * kBoundSteps;
    const int ii = tid / kBoundSteps, j = tid - ii * kBoundSteps, i = min(ii, kBoundSteps - 1);
    const float turn = 1.0f / (float)kBoundSteps;
    const float ci = __builtin_amdgcn_cosf((float)i * turn), si = __builtin_amdgcn_sinf((float)i * turn);
    uint32_t sum = 0u;
#pragma unroll 8
    for (int a = 0; a < n; ++a) {  // (n is a multiple of 8)
        const float4 u = unit[a], b = band[a];
        float k0;
        const float rec = bound_record(u.x, fmaf(ci, u.y, -si * u.z), fmaf(si, u.y, ci * u.z), u.w,
                                       b.x, b.y, k0);
        const int s0 = (int)k0 + j, at = (int)rec * kBoundRec + (s0 < kBoundSteps ? s0 : s0 - kBoundSteps);
        sum += bd.tab[__float_as_uint(b.z) / 2 + (uint32_t)at];
    }
    u64 top = wave_max_key(real ? ((u64)sum << 32) | (uint32_t)tid : 0ull);
    if (lane_id() == 0) key[wave] = top;
    __syncthreads();
    for (int w = 0; w < 15; ++w) top = key[w] > top ? key[w] : top;
    // the score of the orientation of the largest bound
    const int best = (int)(uint32_t)top, bi = best / kBoundSteps, bj = best - bi * kBoundSteps;
    float v = 0.0f;
    if (tid < n) {
        const float4 u = unit[tid];
        const float2 x = make_float2(__builtin_amdgcn_cosf((float)bi * turn), __builtin_amdgcn_sinf((float)bi * turn));
        const float2 y = make_float2(__builtin_amdgcn_cosf((float)bj * turn), __builtin_amdgcn_sinf((float)bj * turn));
        const XStage xs = align_x(u.x, u.y, u.z, x, g.acy);
        v = tri_v(make_tri(g), align_gx(xs, y, g.acx), xs.gy, align_gz(xs, y, g.acz),
                  __float_as_uint(band[tid].w));
    }
    v = wave_sum(v);
    if (lane_id() == 0) part[wave] = v;
    __syncthreads();
    float got = 0.0f;
    for (int w = 0; w < 15; ++w) got += part[w];
    const u64 bm = __ballot(real && sum >= bound_least(got, n, vlow, step, mag));
    if (lane_id() == 0 && bm != 0ull) atomicAdd(&stay[bin], __popcll(bm));
}

// Low 24 bits of x, plus c.
__device__ __forceinline__ uint32_t add_low24(uint32_t x, int c) {
    uint32_t r;
    asm("v_mad_u32_u24 %0, %1, 1, %2" : "=v"(r) : "v"(x), "v"(c));
    return r;
}

// Shared memory of k_align_bound (bytes).
constexpr int kBoundWaves = 4;                     // waves per workgroup
constexpr int kBoundPerWave = 2;                   // restarts per wave: 60 strips in 64 lanes
constexpr int kBoundCand = kBoundPerWave * kBoundSteps * kBoundSteps;
struct BoundLds {
    static __host__ __device__ size_t xyzt() { return 0; }                     // [nmax] x,y,z,toff
    static __host__ __device__ size_t dxyz(int nmax) { return (size_t)nmax * 16; }  // X - c0, toff
    static __host__ __device__ size_t unit(int nmax) { return (size_t)nmax * 32; }  // grid units, 1/r
    static __host__ __device__ size_t band(int nmax) { return (size_t)nmax * 48; }  // rows, sub-bins, offset
    static __host__ __device__ size_t misc(int nmax) { return (size_t)nmax * 64; }
    static __host__ __device__ size_t cand(int nmax) { return misc(nmax) + 16; }
    static __host__ __device__ size_t total(int nmax) {
        return cand(nmax) + (size_t)kBoundWaves * kBoundCand * 2;
    }
};

typedef unsigned short us2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

// Restart slot, x and y rotation of a bound's place e = lane << 5 | 4 s + c in the
// wave: strip (lane & ~7) + s, y rotation 4 (lane & 7) + c.
__device__ __forceinline__ int bound_slot(uint32_t e, int &oi, int &oj) {
    const int strip = (int)((e >> 5) & 56u) + (int)((e >> 2) & 7u);
    oj = 4 * (int)((e >> 5) & 7u) + (int)(e & 3u);
    const int k = strip >= kBoundSteps ? 1 : 0;
    oi = strip - k * kBoundSteps;
    return k;
}

// Exact scores of the listed orientations (see bound_slot), 64 at a time, a lane per
// orientation: align_pose's samples in its atom order.  best[k] is raised to the best key
// of restart slot k.
template <bool Inside>
__device__ __forceinline__ void score_listed(const uint16_t *cand, int nc, const float4 *dxyz, int n,
                                             const int (&r)[kBoundPerWave],
                                             const float4 (&cw)[kBoundPerWave],
                                             const float4 (&ce)[kBoundPerWave], const Tri &tr,
                                             const GridArgs &g, const SearchArgs &sa,
                                             u64 (&best)[kBoundPerWave]) {
    const int lane = lane_id();
    // lanes past the list leave the loop: a load costs by its active lanes
    for (int c = lane; c < nc; c += 64) {
        int oi, oj;
        const int k = bound_slot(cand[c], oi, oj);
        const int rr = k ? r[1] : r[0];
        const float cwx = k ? cw[1].x : cw[0].x, cwy = k ? cw[1].y : cw[0].y,
                    cwz = k ? cw[1].z : cw[0].z;
        const float ex = k ? ce[1].x : ce[0].x, ey = k ? ce[1].y : ce[0].y,
                    ez = k ? ce[1].z : ce[0].z;
        const float4 m0 = sa.smat[3 * rr + 0], m1 = sa.smat[3 * rr + 1], m2 = sa.smat[3 * rr + 2];
        const float2 ci = sa.acs[oi], cj = sa.acs[oj];
        float acc = 0.0f;
        auto place = [&](const float4 d, float &gx, float &gy, float &gz) {
            const float yx = fmaf(m0.x, d.x, fmaf(m0.y, d.y, fmaf(m0.z, d.z, g.cx)));
            const float yy = fmaf(m1.x, d.x, fmaf(m1.y, d.y, fmaf(m1.z, d.z, g.cy)));
            const float yz = fmaf(m2.x, d.x, fmaf(m2.y, d.y, fmaf(m2.z, d.z, g.cz)));
            const XStage xs = align_x((yx - cwx) * g.inv_h, (yy - cwy) * g.inv_h,
                                      (yz - cwz) * g.inv_h, ci, ey);
            gx = align_gx(xs, cj, ex);
            gy = xs.gy;
            gz = align_gz(xs, cj, ez);
        };
        constexpr int U = 4;  // atoms whose cube loads are in flight together
        int a = 0;
        for (; a + U - 1 < n; a += U) {
            float fx[U], fy[U], fz[U];
            float4 q0[U], q1[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const float4 d = dxyz[a + u];
                const int to = uniform_int(__float_as_int(d.w));
                float gx, gy, gz;
                place(d, gx, gy, gz);
                uint32_t off;
                if (Inside) {
                    fx[u] = __builtin_amdgcn_fractf(gx);
                    fy[u] = __builtin_amdgcn_fractf(gy);
                    fz[u] = __builtin_amdgcn_fractf(gz);
                    off = in_cell(tr, gx, gy, gz);
                } else {
                    off = tri_cell(tr, gx, gy, gz, fx[u], fy[u], fz[u]);
                }
                q0[u] = ldq(tr.rs, off, to);
                q1[u] = ldq(tr.rs, off, to + 16);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < U; ++u) acc += tri_blend(q0[u], q1[u], fx[u], fy[u], fz[u]);
        }
        for (; a < n; ++a) {
            const float4 d = dxyz[a];
            const int to = uniform_int(__float_as_int(d.w));
            float gx, gy, gz;
            place(d, gx, gy, gz);
            acc += Inside ? tri_in(tr, gx, gy, gz, to) : tri_u(tr, gx, gy, gz, to);
        }
        const u64 key = make_key(acc, (uint32_t)(oi * kBoundSteps + oj));
        if (k == 0) best[0] = key > best[0] ? key : best[0];
        else best[1] = key > best[1] ? key : best[1];
    }
}

// Persistent workgroups pop (ligand, group of kBoundWaves * kBoundPerWave restarts)
// items (queues as in k_align).  A wave holds two restarts' 60 strips, one per
// lane.  Per atom each lane finds its strip's record; then eight lanes at a time
// read one record (a lane 4 of its 32 entries, 8 bytes), so a load covers eight
// strips with 64 contiguous bytes each, and add them as packed 16-bit integers
// (ligands of more than kBoundRun atoms: every kBoundRun into 32 bits).
template <int NS>
__global__ __launch_bounds__(64 * kBoundWaves, 4) void k_align_bound(GridArgs g, SearchArgs sa,
                                                                     LibArgs lib, WorkArgs ws,
                                                                     BoundArgs bd, int bin, int lst) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int nmax = bin_nmax(bin);
    const int tid = threadIdx.x, wave = uniform_int(tid >> 6), lane = lane_id();
    float4 *xyzt = (float4 *)(smem + BoundLds::xyzt());
    float4 *dxyz = (float4 *)(smem + BoundLds::dxyz(nmax));
    float4 *unit = (float4 *)(smem + BoundLds::unit(nmax));
    float4 *band = (float4 *)(smem + BoundLds::band(nmax));
    int *misc = (int *)(smem + BoundLds::misc(nmax));
    uint16_t *cand = (uint16_t *)(smem + BoundLds::cand(nmax)) + (size_t)wave * kBoundCand;
    const Tri tr = make_tri(g);
    const __amdgpu_buffer_rsrc_t brs =
        __builtin_amdgcn_make_buffer_rsrc((void *)bd.tab, (short)0, (int)bd.bytes, 0x00020000);
    constexpr int GR = kBoundWaves * kBoundPerWave;
    const int groups = (sa.R + GR - 1) / GR;
    // the lane's strip, its 8-lane group and place in it
    const int q8 = lane & 7;
    const int slot = lane >= kBoundSteps && lane < 2 * kBoundSteps ? 1 : 0;
    const int si = lane < 2 * kBoundSteps ? lane - kBoundSteps * slot : 0;
    const float2 ci = sa.acs[si];
    const uint32_t wrap_at = (uint32_t)(q8 + 1) << 24;
    const int c_in = 8 * q8, c_wrap = 8 * q8 - 2 * kBoundSteps;
    const long long nl = ws.counters[lst];
    int *qc = ws.counters + 4 * kMaxLists + lst * kXcds;
    int qcur = (int)(blockIdx.x % kXcds), qleft = kXcds;
    for (;;) {
        if (tid == 0) {
            int qli = -1, qgrp = 0;
            while (qleft > 0) {
                const long long l0 = nl * qcur / kXcds, l1 = nl * (qcur + 1) / kXcds;
                const long long items = (l1 - l0) * groups;
                const int got = items > 0 ? atomicAdd(&qc[qcur], 1) : 0;
                if ((long long)got < items) {
                    qli = (int)(l0 + got / groups);
                    qgrp = got % groups;
                    break;
                }
                qcur = qcur + 1 == kXcds ? 0 : qcur + 1;
                --qleft;
            }
            misc[0] = qli;
            misc[1] = qgrp;
        }
        __syncthreads();
        const int li = uniform_int(misc[0]), grp = uniform_int(misc[1]);
        if (li < 0) break;
        const int l = ws.bin_list[li];
        const int a0 = lib.atom_off[l], n = lib.atom_off[l + 1] - a0;
        const int B = lib.rot_off[l + 1] - lib.rot_off[l];
        for (int i = tid; i < n; i += 64 * kBoundWaves) {
            const float *p = lib.xyz + 3 * (size_t)(a0 + i);
            const uint32_t toff = (uint32_t)lib.type[a0 + i] * g.type_bytes;
            xyzt[i] = make_float4(p[0], p[1], p[2], __uint_as_float(toff));
        }
        __syncthreads();
        if (wave == 0) {
            // ligand-centred coordinates X - c0, with the c0 of start_pose, and each
            // atom's radius band
            Pose<NS> X;
#pragma unroll
            for (int q = 0; q < NS; ++q) {
                const int i = lane + 64 * q;
                const float4 v = i < n ? xyzt[i] : make_float4(0.f, 0.f, 0.f, 0.f);
                X.x[q] = v.x;
                X.y[q] = v.y;
                X.z[q] = v.z;
            }
            float c0x, c0y, c0z;
            centroid(X, n, c0x, c0y, c0z);
#pragma unroll
            for (int q = 0; q < NS; ++q) {
                const int i = lane + 64 * q;
                if (i >= n) continue;
                const float dx = X.x[q] - c0x, dy = X.y[q] - c0y, dz = X.z[q] - c0z;
                const float ux = dx * g.inv_h, uy = dy * g.inv_h, uz = dz * g.inv_h;
                const float rad = sqrtf(fmaf(ux, ux, fmaf(uy, uy, uz * uz)));
                const int4 bq = bd.band[bound_band(bd, rad)];
                const uint32_t off = (uint32_t)lib.type[a0 + i] * bd.type_bytes + (uint32_t)bq.z;
                dxyz[i] = make_float4(dx, dy, dz, xyzt[i].w);
                unit[i] = make_float4(ux, uy, uz, rad > 1e-6f ? 1.0f / rad : 0.0f);
                band[i] = make_float4((float)bq.x, (float)bq.y, __uint_as_float(off), 0.0f);
            }
        }
        int r[kBoundPerWave];
        float4 cw[kBoundPerWave], ce[kBoundPerWave];
        bool off[kBoundPerWave];  // turns about a point too far off the grid centre
        bool out_any = false;
        const int rbase = grp * GR + wave * kBoundPerWave;
#pragma unroll
        for (int k = 0; k < kBoundPerWave; ++k) {
            r[k] = min(rbase + k, sa.R - 1);  // restarts past R repeat the last one
            Pose<NS> Y;
            start_pose(Y, xyzt, n, r[k], g, sa);
            float cx, cy, cz;
            centroid(Y, n, cx, cy, cz);
            cw[k] = make_float4(cx, cy, cz, 0.f);
            ce[k] = make_float4((cx - g.ox) * g.inv_h, (cy - g.oy) * g.inv_h,
                                (cz - g.oz) * g.inv_h, 0.f);
            off[k] = !centred(g, ce[k].x, ce[k].y, ce[k].z, kBoundOffset);
#pragma unroll
            for (int q = 0; q < NS; ++q) {
                const float rx = (Y.x[q] - cx) * g.inv_h, ry = (Y.y[q] - cy) * g.inv_h,
                            rz = (Y.z[q] - cz) * g.inv_h;
                if (lane + 64 * q < n)
                    out_any = out_any ||
                              !ball_inside(tr, ce[k].x, ce[k].y, ce[k].z,
                                           ball_radius(fmaf(rx, rx, fmaf(ry, ry, rz * rz))));
            }
        }
        const bool all_in = __ballot(out_any) == 0ull;
        __syncthreads();
        if (rbase < sa.R) {
            // rows of R_x(i) S_r of the lane's strip
            const int rs = slot ? r[1] : r[0];
            const float4 s0 = sa.smat[3 * rs + 0], s1 = sa.smat[3 * rs + 1], s2 = sa.smat[3 * rs + 2];
            const float ax = fmaf(ci.x, s1.x, -ci.y * s2.x), ay = fmaf(ci.x, s1.y, -ci.y * s2.y),
                        az = fmaf(ci.x, s1.z, -ci.y * s2.z);
            const float bx = fmaf(ci.y, s1.x, ci.x * s2.x), by = fmaf(ci.y, s1.y, ci.x * s2.y),
                        bz = fmaf(ci.y, s1.z, ci.x * s2.z);
            us2 acc[8][2];
            constexpr bool kWide = NS * 64 > kBoundRun;
            uint32_t sum[kWide ? 8 : 1][4];
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                acc[s][0] = acc[s][1] = (us2)(0);
                if constexpr (kWide) sum[s][0] = sum[s][1] = sum[s][2] = sum[s][3] = 0u;
            }
            // The record of the lane's strip for atom a: byte offset of its entry k0 in the
            // band (below 2^24) and, in the top byte, the first lane of an 8-lane group
            // whose 4 entries start past the turn.
            auto record = [&](int a, int &soff) -> uint32_t {
                const float4 u = unit[a], bq = band[a];
                const float rx = fmaf(s0.x, u.x, fmaf(s0.y, u.y, s0.z * u.z));
                const float gy = fmaf(ax, u.x, fmaf(ay, u.y, az * u.z));
                const float qz = fmaf(bx, u.x, fmaf(by, u.y, bz * u.z));
                float k0;
                const float rec = bound_record(rx, gy, qz, u.w, bq.x, bq.y, k0);
                const uint32_t ki = (uint32_t)k0;
                const uint32_t at = (uint32_t)(rec * (2.0f * (float)kBoundRec)) + 2u * ki;
                soff = uniform_int(__float_as_int(bq.z));
                return at | ((((uint32_t)(kBoundSteps + 3) << 22) - (ki << 22)) & 0xFF000000u);
            };
            int soff;
            uint32_t v = record(0, soff);
            for (int a = 0; a < n; ++a) {
                u32x2 w[8];
#define DOCK_BOUND_LOAD(S)                                                                      \
    {                                                                                           \
        const uint32_t x = (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, (S << 5) | 0x18);      \
        w[S] = __builtin_amdgcn_raw_buffer_load_b64(                                            \
            brs, (int)add_low24(x, x < wrap_at ? c_wrap : c_in), soff, 0);                      \
    }
                DOCK_BOUND_LOAD(0) DOCK_BOUND_LOAD(1) DOCK_BOUND_LOAD(2) DOCK_BOUND_LOAD(3)
                DOCK_BOUND_LOAD(4) DOCK_BOUND_LOAD(5) DOCK_BOUND_LOAD(6) DOCK_BOUND_LOAD(7)
#undef DOCK_BOUND_LOAD
                // the next atom's record while the loads are in flight
                v = record(a + 1 < n ? a + 1 : a, soff);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int s = 0; s < 8; ++s) {
                    acc[s][0] += __builtin_bit_cast(us2, (uint32_t)w[s].x);
                    acc[s][1] += __builtin_bit_cast(us2, (uint32_t)w[s].y);
                }
                if constexpr (kWide) {
                    if ((a & (kBoundRun - 1)) == kBoundRun - 1) {
#pragma unroll
                        for (int s = 0; s < 8; ++s) {
#pragma unroll
                            for (int c = 0; c < 4; ++c) sum[s][c] += acc[s][c >> 1][c & 1];
                            acc[s][0] = acc[s][1] = (us2)(0);
                        }
                    }
                }
            }
            // no bound for strips past the second restart's and y rotations past the turn
            // (every real one is at least 1 per atom)
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                const bool no_strip = s >= 4 && lane >= 56;
                if (no_strip) acc[s][0] = (us2)(0);
                if (no_strip || q8 == 7) acc[s][1] = (us2)(0);
                if constexpr (kWide) {
                    if (no_strip) sum[s][0] = sum[s][1] = 0u;
                    if (no_strip || q8 == 7) sum[s][2] = sum[s][3] = 0u;
                }
            }
            auto bound = [&](int s, int c) -> uint32_t {
                uint32_t v = acc[s][c >> 1][c & 1];
                if constexpr (kWide) v += sum[s][c];
                return v;
            };
            const bool second = lane >= 32;  // strips of lane & ~7 + s >= 30: or lanes 24..31, s >= 6
            const bool split = lane >= 24 && lane < 32;
            // slot of the largest bound of each restart: key = bound << 11 | lane << 5 | 4 s + c
            uint32_t top[kBoundPerWave] = {0u, 0u};
            {
                uint32_t lo = 0u, hi = 0u;  // slots s < 6 and s >= 6
#pragma unroll
                for (int s = 0; s < 8; ++s)
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const uint32_t key = (bound(s, c) << 11) | (uint32_t)(4 * s + c);
                        if (s < 6) lo = max(lo, key);
                        else hi = max(hi, key);
                    }
                const uint32_t at = (uint32_t)lane << 5;
                lo |= at;
                hi |= at;
                top[0] = second ? 0u : (split ? lo : max(lo, hi));
                top[1] = second ? max(lo, hi) : (split ? hi : 0u);
            }
            // (the bounds again below: keeping all 32 unpacked would fill the registers)
#pragma unroll
            for (int s = 0; s < 8; ++s)
                asm volatile("" : "+v"(acc[s][0]), "+v"(acc[s][1]));
            uint32_t least[kBoundPerWave];  // smallest bound that can be the best score
#pragma unroll
            for (int k = 0; k < kBoundPerWave; ++k) {
                int oi, oj;
                bound_slot(wave_max_u32(top[k]) & 2047u, oi, oj);
                const float2 xi = sa.acs[oi], xj = sa.acs[oj];
                const float4 m0 = sa.smat[3 * r[k] + 0], m1 = sa.smat[3 * r[k] + 1],
                             m2 = sa.smat[3 * r[k] + 2];
                float v = 0.0f;
#pragma unroll
                for (int q = 0; q < NS; ++q) {
                    const int i = lane + 64 * q;
                    if (i < n) {
                        const float4 d = dxyz[i];
                        const float yx = fmaf(m0.x, d.x, fmaf(m0.y, d.y, fmaf(m0.z, d.z, g.cx)));
                        const float yy = fmaf(m1.x, d.x, fmaf(m1.y, d.y, fmaf(m1.z, d.z, g.cy)));
                        const float yz = fmaf(m2.x, d.x, fmaf(m2.y, d.y, fmaf(m2.z, d.z, g.cz)));
                        const XStage xs = align_x((yx - cw[k].x) * g.inv_h, (yy - cw[k].y) * g.inv_h,
                                                  (yz - cw[k].z) * g.inv_h, xi, ce[k].y);
                        v += tri_v(tr, align_gx(xs, xj, ce[k].x), xs.gy, align_gz(xs, xj, ce[k].z),
                                   (uint32_t)__float_as_int(d.w));
                    }
                }
                const float got = wave_sum(v);
                least[k] = off[k] ? 1u : bound_least(got, n, bd.vlow, bd.step, bd.mag);
            }
            // the orientations that stay
            int nc = 0;
            const uint32_t lim_lo = second ? least[1] : least[0];
            const uint32_t lim_hi = second || split ? least[1] : least[0];
#pragma unroll
            for (int s = 0; s < 8; ++s) {
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const bool ok = bound(s, c) >= (s < 6 ? lim_lo : lim_hi);
                    const u64 bm = __ballot(ok);
                    if (bm == 0ull) continue;
                    if (ok)
                        cand[nc + (int)__builtin_amdgcn_mbcnt_hi(
                                      (uint32_t)(bm >> 32),
                                      __builtin_amdgcn_mbcnt_lo((uint32_t)bm, 0u))] =
                            (uint16_t)((lane << 5) | (4 * s + c));
                    nc += __popcll(bm);
                }
            }
            wave_lds_sync();
            u64 best[kBoundPerWave] = {0ull, 0ull};
            if (all_in) score_listed<true>(cand, nc, dxyz, n, r, cw, ce, tr, g, sa, best);
            else score_listed<false>(cand, nc, dxyz, n, r, cw, ce, tr, g, sa, best);
#pragma unroll
            for (int k = 0; k < kBoundPerWave; ++k) {
                const u64 bk = wave_max_key(best[k]);
                if (lane == 0 && rbase + k < sa.R)
                    ws.rtrace[trace_base(lib, sa, l) + (size_t)(rbase + k) * (1 + sa.P * B)] =
                        (uint16_t)key_index(bk);
            }
        }
        __syncthreads();
    }
}

// Plain (latency) form: one ligand per launch sequence.  Workgroup r docks
// restart r; its waves split the orientations and the torsion candidates and
// agree on every decision through LDS and workgroup barriers.
template <int NS, int C>
__global__ __launch_bounds__(256) void k_plain(DockArgs args) {
    extern __shared__ __align__(16) unsigned char smem[];
    const GridArgs &g = args.g;
    const SearchArgs &sa = args.sa;
    const LibArgs &lib = args.lib;
    const WorkArgs &ws = args.ws;
    const int l = args.lig, nmax = bin_nmax(args.bin);
    const int W = blockDim.x >> 6, wave = uniform_int((int)(threadIdx.x >> 6)), lane = lane_id();
    if (args.status[l] != 0) return;
    float4 *xyzt = (float4 *)(smem + Lds::xyzt(nmax));
    const u64 *far = (const u64 *)(smem + Lds::far(nmax));
    const u64 *mask = (const u64 *)(smem + Lds::mask(nmax, NS));
    const int2 *rot = (const int2 *)(smem + Lds::rot(nmax, NS));
    int *misc = (int *)(smem + Lds::misc(nmax, NS));
    float4 *rec = (float4 *)(smem + Lds::rec(nmax, NS) + (size_t)wave * Lds::rec_stride(nmax));
    uint16_t *cand = (uint16_t *)((unsigned char *)rec + Lds::cand(nmax));
    u64 *slots = (u64 *)(smem + Lds::rec(nmax, NS) + (size_t)W * Lds::rec_stride(nmax));
    const Tri tr = make_tri(g);
    const BlockSplit sp{wave, W, slots};
    float2 cs[C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const int k = sp.first() + lane + sp.stride() * c;
        cs[c] = k < sa.T ? sa.tors[k] : make_float2(1.f, 0.f);
    }
    stage_ligand<NS>(smem, nmax, l, lib, ws, g, true);
    __syncthreads();
    const int r = blockIdx.x;
    const int n = uniform_int(misc[1]), B = uniform_int(misc[2]);
    int toff[NS];
    lane_toff(xyzt, n, toff);
    Pose<NS> Y;
    start_pose(Y, xyzt, n, r, g, sa);
    uint16_t *tr_out = ws.rtrace + trace_base(lib, sa, l) + (size_t)r * (1 + sa.P * B);
    const bool writer = threadIdx.x == 0;
    const int o = align_pose(Y, n, toff, rec, tr, g, sa, nullptr, sp);
    if (writer) tr_out[0] = (uint16_t)o;
    int d = 1;
    long long nsc = 0;  // this wave's share of the scored torsion samples
    for (int p = 0; p < sa.P; ++p) {
        for (int b = 0; b < B; ++b, ++d) {
            const int2 ab = rot[b];
            const int k = torsion_decide<NS, C>(Y, n, mask + b * NS, uniform_int(ab.x),
                                                uniform_int(ab.y), far, toff, rec, cand, cs,
                                                sp, nsc);
            if (writer) tr_out[d] = (uint16_t)k;
        }
    }
    if (ws.scored && lane == 0) atomicAdd(ws.scored, (unsigned long long)nsc);
    if (ws.rpose && wave == 0) {
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int i = lane + 64 * s;
            float *P = ws.rpose + ((size_t)r * n + i) * 3;
            if (i < n) {
                P[0] = Y.x[s];
                P[1] = Y.y[s];
                P[2] = Y.z[s];
            }
        }
    }
    const float sc = pose_score(Y, n, toff, tr, g);
    if (writer) ws.rscore[(size_t)l * sa.R + r] = sc;
}

// Replay restart r of ligand l from its decision trace (same arithmetic as k_dock).
template <int NS>
__device__ void replay_pose(Pose<NS> &Y, const float4 *xyzt, const u64 *mask, const int2 *rot,
                            int n, int B, int r, const uint16_t *trace, const GridArgs &g,
                            const SearchArgs &sa) {
    const int lane = lane_id();
    start_pose(Y, xyzt, n, r, g, sa);
    // The trace and each step's (cos, sin) are loaded 64 entries at a time, one
    // entry per lane, so the replay waits for one round of loads per 64 steps
    // instead of one per step; entry 0 is the alignment, entry 1 + p*B + b the
    // step of bond b in pass p.
    const int D = 1 + sa.P * B;
    for (int base = 0; base < D; base += 64) {
        const int e = base + lane;
        const int kl = e < D ? (int)trace[e] : (int)kTraceNone;
        const float2 tl = e > 0 && kl < sa.T ? sa.tors[kl] : make_float2(1.f, 0.f);
        const int cnt = D - base < 64 ? D - base : 64;
        for (int u = 0; u < cnt; ++u) {
            const int d = base + u;
            const int k = __builtin_amdgcn_readlane(kl, u);
            if (d == 0) {
                apply_align(Y, n, k < sa.A * sa.A ? k : 0, sa);  // from k_dock; bound anyway
            } else if (k < sa.T) {
                const int b = (d - 1) % B;
                const float c = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(tl.x), u));
                const float sn = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(tl.y), u));
                const int2 ab = rot[b];
                apply_torsion(Y, mask + b * NS, bond_axis(Y, uniform_int(ab.x), uniform_int(ab.y)),
                              c, sn);
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Final stage (Select Poses, then the final rigid step and score of every kept
// pose, then the outputs), as three kernels per size bin:
//   k_select: one workgroup per ligand (persistent over the bin list): ranks the
//     restarts, rebuilds candidates from their traces and keeps them greedily;
//     writes the kept poses (workspace acc_pose), their restarts and count;
//   k_falign: one wave per (ligand, pair of kept poses) item (the grid's waves take the
//     bin's items from a queue or in turn), or in the plain form one workgroup per kept pose
//     with the orientations split over its waves: alignment again about the
//     pose centroid, final score and orientation;
//   k_out: one workgroup per ligand: output order (final score desc, restart
//     asc), scores, restarts, final-step indices, and the kept poses turned by
//     their final-step orientation.
// k_select's shared memory: staged ligand, restart keys and order, selection
// scratch, then (sel_lds) the batch of candidate poses and the kept poses.

static __host__ __device__ size_t select_sel_offset(int nmax, int waves, int R, int K) {
    const int nw = (nmax + 63) / 64;
    const size_t b = Lds::rec(nmax, nw) + (size_t)R * 12 + (size_t)K * 4 + 4 +
                     (size_t)(2 * waves + 1) * 4;
    return (b + 15) & ~(size_t)15;
}

size_t select_lds_bytes(int nmax, int waves, int R, int K, int sel_lds) {
    return select_sel_offset(nmax, waves, R, K) +
           (sel_lds ? (size_t)(waves + K) * ((size_t)nmax * 12 + (sel_lds == 2 ? 4 : 0)) : 0);
}

int select_sel_lds(int nmax, int waves, int R, int K) {
    return select_lds_bytes(nmax, waves, R, K, 1) <= (size_t)160 * 1024 ? 1 : 0;
}

// Whether the poses are kept in LDS, and the waves: the batched form decides by what
// fits with kSelectGroup waves, whatever the tile, and a tile that needs more LDS than
// there is loses waves (the path over global memory sums distances in another order).
// 2: with room for an odd number of words a pose, so that lanes that each read one are on
// different banks.
static int select_shape(int nmax, int R, int K, bool plain, int *waves) {
    const int sel = select_sel_lds(nmax, plain ? *waves : kSelectGroup, R, K);
    while (sel && !select_sel_lds(nmax, *waves, R, K)) --*waves;
    return sel && select_lds_bytes(nmax, *waves, R, K, 2) <= (size_t)160 * 1024 ? 2 : sel;
}

// Given: the restarts' poses are in ws.rpose (the plain form, with sel_lds); without the
// replay its 16 waves need fewer registers and start beside the next ligand's k_plain (40
// ligands of 200-240 atoms, 1,000 restarts of 5 steps: 9.3 -> 8.5 ms, at 20 steps
// 27.5 -> 25.7).  With the replay at most 64 registers up to 64 atoms (65 otherwise), which leaves
// more room beside another third's sweep: 2,500 ligands of 20-80 atoms 42.8 -> 42.5 ms; with
// as many up to 128 atoms, 42.1, but 4,096 of 12-150 atoms 63.6 -> 65.1.
template <int NS, bool Given>
__global__ __launch_bounds__(1024, NS == 1 && !Given ? 8 : 4) void k_select(GridArgs g, SearchArgs sa, LibArgs lib,
                                                WorkArgs ws, OutArgs out, int bin, int lst, int single,
                                                int sel_lds) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int nmax = bin_nmax(bin);
    const int W = blockDim.x >> 6, wave = uniform_int((int)(threadIdx.x >> 6)), lane = lane_id();
    const int R = sa.R, K = sa.K;
    float4 *xyzt = (float4 *)(smem + Lds::xyzt(nmax));
    const u64 *mask = (const u64 *)(smem + Lds::mask(nmax, NS));
    const int2 *rot = (const int2 *)(smem + Lds::rot(nmax, NS));
    int *misc = (int *)(smem + Lds::misc(nmax, NS));
    unsigned char *p = smem + Lds::rec(nmax, NS);
    u64 *rkey = (u64 *)p;                     // [R]
    int *order = (int *)(p + (size_t)R * 8);  // [R]
    int *sel = (int *)(p + (size_t)R * 12);   // [K] restart, and its rank << 16
    int *nsel = sel + K;                      // [1]
    int *cflag = nsel + 1;                    // [W] candidate conflicts
    int *kinfo = cflag + W;                   // [1 + W] kept count, slot of each wave's candidate
    const int pad = sel_lds == 2 ? 1 : 0;
    float *candL = (float *)(smem + select_sel_offset(nmax, W, R, K));  // [W][ps] poses [n][3]
    float *keptL = candL + (size_t)W * (nmax * 3 + pad);                 // [K][ps]

    if (single >= 0 && out.status[single] != 0) return;
    for (int pass = 0;; ++pass) {
        int l;
        if (single >= 0) {
            // plain form: exactly one ligand, given by the launch
            if (pass > 0) break;
            l = single;
        } else {
            if (threadIdx.x == 0) misc[0] = atomicAdd(&ws.counters[2 * kMaxLists + lst], 1);
            __syncthreads();
            const int li = misc[0];
            if (li >= ws.counters[lst]) break;
            l = ws.bin_list[li];
        }
        stage_ligand<NS>(smem, nmax, l, lib, ws, g, false);
        for (int r = threadIdx.x; r < R; r += blockDim.x) {
            const float s = ws.rscore[(size_t)l * R + r];
            rkey[r] = make_key(s, (uint32_t)r);
            if (out.rscore_user) out.rscore_user[(size_t)l * R + r] = s;
        }
        __syncthreads();
        // order restarts by (score desc, restart asc): rank = number of larger keys
        for (int r = threadIdx.x; r < R; r += blockDim.x) {
            const u64 kr = rkey[r];
            int rk = 0;
            for (int q = 0; q < R; ++q) rk += rkey[q] > kr;
            order[rk] = r;
        }
        __syncthreads();
        const int n = uniform_int(misc[1]), B = uniform_int(misc[2]);
        const int a0 = lib.atom_off[l];
        float *accp = ws.acc_pose + (size_t)a0 * K * 3;
        const uint16_t *trl = ws.rtrace + trace_base(lib, sa, l);
        const int D = 1 + sa.P * B;
        if (sel_lds) {
            // Select Poses with every wave: per round, wave w replays the restart
            // ranked t0 + w and tests it against the poses kept so far and against the
            // round's earlier candidates; one thread then takes the round's candidates
            // in rank order, which is the greedy rule.  How a distance is summed depends
            // on the two ranks alone, so that the number of waves changes no rounding:
            // of two in the same group of G ranks over lanes, else over the atoms in
            // order (a lane per earlier pose).
            const float lim = sa.dedup2 * (float)n;
            const int G = single >= 0 ? kPlainSelectGroup : kSelectGroup;
            const int ps = pad ? (3 * n) | 1 : 3 * n;  // words a pose
            int ns = 0;
            for (int t0 = 0; t0 < R && ns < K; t0 += W) {
                const int t = t0 + wave, g0 = t - t % G;  // g0: first rank of its group
                float *cp = candL + (size_t)wave * ps;
                int flag = 1;  // bit 0: conflicts with a kept pose (or no candidate)
                // over the atoms in order / over lanes, to pose vp
                auto in_order = [&](const float *vp) -> float {
                    float ssd = 0.f;
#pragma unroll 4
                    for (int i = 0; i < n; ++i) {
                        const float dx = cp[3 * i + 0] - vp[3 * i + 0];
                        const float dy = cp[3 * i + 1] - vp[3 * i + 1];
                        const float dz = cp[3 * i + 2] - vp[3 * i + 2];
                        ssd = fmaf(dx, dx, fmaf(dy, dy, fmaf(dz, dz, ssd)));
                    }
                    return ssd;
                };
                auto over_lanes = [&](const float *vp) -> float {
                    float ssd = 0.f;
#pragma unroll
                    for (int q = 0; q < NS; ++q) {
                        const int i = lane + 64 * q;
                        if (i < n) {
                            const float dx = cp[3 * i + 0] - vp[3 * i + 0];
                            const float dy = cp[3 * i + 1] - vp[3 * i + 1];
                            const float dz = cp[3 * i + 2] - vp[3 * i + 2];
                            ssd = fmaf(dx, dx, fmaf(dy, dy, fmaf(dz, dz, ssd)));
                        }
                    }
                    return wave_sum(ssd);
                };
                if (t < R) {
                    const int r = uniform_int(order[t]);
                    if constexpr (Given) {
                        const float *P = ws.rpose + (size_t)r * n * 3;
                        for (int e = lane; e < 3 * n; e += 64) cp[e] = P[e];
                    } else {
                        Pose<NS> Y;
                        replay_pose(Y, xyzt, mask, rot, n, B, r, trl + (size_t)r * D, g, sa);
#pragma unroll
                        for (int q = 0; q < NS; ++q) {
                            const int i = lane + 64 * q;
                            if (i < n) {
                                cp[3 * i + 0] = Y.x[q];
                                cp[3 * i + 1] = Y.y[q];
                                cp[3 * i + 2] = Y.z[q];
                            }
                        }
                    }
                    wave_lds_sync();
                    flag = 0;
                }
                // of other groups: kept poses (all but the last ones, those with W not a
                // multiple of G) and the round's earlier candidates, a lane each
                int na = ns;
                while (na > 0 && (uniform_int(sel[na - 1]) >> 16) >= g0) --na;
                const int ve = g0 > t0 ? g0 - t0 : 0;
                auto others = [&]() {
                    u64 kept = 0ull, cand = 0ull;  // (na < 64)
                    for (int e0 = 0; e0 < na + ve; e0 += 64) {
                        const int e = e0 + lane;
                        const bool on = e < na + ve;
                        const float ssd = in_order(e < na ? keptL + (size_t)e * ps
                                                          : candL + (size_t)(on ? e - na : 0) * ps);
                        const u64 hit = __ballot(on && ssd < lim);
                        if (e0 == 0) {
                            kept = hit & ((1ull << na) - 1ull);
                            cand = hit >> na;
                        } else {
                            cand |= hit << (64 - na);
                        }
                    }
                    flag = (kept != 0ull ? 1 : 0) | (int)(uint32_t)cand << 1;
                    for (int k = na; k < ns; ++k)
                        if (over_lanes(keptL + (size_t)k * ps) < lim) flag |= 1;
                };
                const bool test = t < R && sa.dedup2 > 0.f;
                const bool alone = G % W == 0;  // no earlier candidates of other groups
                if (test && alone) others();
                __syncthreads();  // the round's candidates are in LDS
                if (test && !alone) others();
                if (test) {
#pragma unroll 4
                    for (int v = ve; v < wave; ++v)
                        if (over_lanes(candL + (size_t)v * ps) < lim) flag |= 2 << v;
                }
                if (lane == 0) cflag[wave] = flag;
                __syncthreads();
                if (threadIdx.x == 0) {
                    int nn = ns, kept = 0;
                    for (int w = 0; w < W; ++w) {
                        kinfo[1 + w] = -1;
                        const int f = cflag[w];
                        if (nn >= K || (f & 1) || ((f >> 1) & kept)) continue;
                        kept |= 1 << w;
                        kinfo[1 + w] = nn;
                        sel[nn++] = order[t0 + w] | (t0 + w) << 16;
                    }
                    kinfo[0] = nn;
                }
                __syncthreads();
                const int slot = kinfo[1 + wave];
                if (slot >= 0) {
                    float *kd = keptL + (size_t)slot * ps;
                    for (int e = lane; e < 3 * n; e += 64) kd[e] = cp[e];
                }
                ns = kinfo[0];
                __syncthreads();
            }
            if (threadIdx.x == 0) *nsel = ns;
            // kept poses to the workspace, for k_falign
            for (int k = 0; k < ns; ++k)
                for (int e = threadIdx.x; e < 3 * n; e += blockDim.x)
                    accp[(size_t)k * 3 * n + e] = keptL[(size_t)k * ps + e];
        } else if (!Given && wave == 0) {
            // greedy selection with plain-RMSD dedup; poses rebuilt from traces
            int ns = 0;
            const float lim = sa.dedup2 * (float)n;
            for (int t = 0; t < R && ns < K; ++t) {
                const int r = order[t];
                Pose<NS> Y;
                replay_pose(Y, xyzt, mask, rot, n, B, r, trl + (size_t)r * D, g, sa);
                bool keep = true;
                if (sa.dedup2 > 0.f) {
                    for (int s = 0; s < ns && keep; ++s) {
                        float ssd = 0.f;
#pragma unroll
                        for (int q = 0; q < NS; ++q) {
                            const int i = lane + 64 * q;
                            if (i < n) {
                                const float *P = accp + ((size_t)s * n + i) * 3;
                                const float dx = Y.x[q] - P[0], dy = Y.y[q] - P[1],
                                            dz = Y.z[q] - P[2];
                                ssd += dx * dx + dy * dy + dz * dz;
                            }
                        }
                        ssd = wave_sum(ssd);
                        if (ssd < lim) keep = false;
                    }
                }
                if (keep) {
#pragma unroll
                    for (int q = 0; q < NS; ++q) {
                        const int i = lane + 64 * q;
                        if (i < n) {
                            float *P = accp + ((size_t)ns * n + i) * 3;
                            P[0] = Y.x[q];
                            P[1] = Y.y[q];
                            P[2] = Y.z[q];
                        }
                    }
                    if (lane == 0) sel[ns] = r;
                    ++ns;
                }
            }
            if (lane == 0) *nsel = ns;
        }
        __syncthreads();
        const int ns = *nsel;
        for (int s = threadIdx.x; s < ns; s += blockDim.x) ws.sel[(size_t)l * K + s] = sel[s] & 0xFFFF;
        if (threadIdx.x == 0) ws.nsel[l] = ns;
        __syncthreads();
    }
}

// Final rigid step and score of kept pose s of ligand l (Rescore Pose stand-in):
// the alignment about the pose centroid (if final_align), then the grid score,
// written to fscore / fo by the lead wave.  The kept pose itself is left as it
// is (k_out applies the chosen orientation), so the kernel can be run again on
// the same inputs.  rec: LDS for >= n float4.
template <int NS, class Split>
__device__ void final_item(int l, int s, float4 *rec, const Tri &tr, const GridArgs &g,
                           const SearchArgs &sa, const LibArgs &lib, const WorkArgs &ws,
                           const Split &sp, bool lead_wave) {
    const int lane = lane_id();
    const int a0 = lib.atom_off[l], n = lib.atom_off[l + 1] - a0;
    const float *P = ws.acc_pose + ((size_t)a0 * sa.K + (size_t)s * n) * 3;
    Pose<NS> Y;
    int toff[NS];
#pragma unroll
    for (int q = 0; q < NS; ++q) {
        const int i = lane + 64 * q;
        const int ii = i < n ? i : 0;
        Y.x[q] = P[3 * ii + 0];
        Y.y[q] = P[3 * ii + 1];
        Y.z[q] = P[3 * ii + 2];
        toff[q] = i < n ? (int)((uint32_t)lib.type[a0 + i] * g.type_bytes) : 0;
    }
    int o = 0;
    if (sa.final_align) o = align_pose(Y, n, toff, rec, tr, g, sa, nullptr, sp);
    const float sc = pose_score(Y, n, toff, tr, g);
    if (lead_wave && lane == 0) {
        ws.fscore[(size_t)l * sa.K + s] = sc;
        ws.fo[(size_t)l * sa.K + s] = o;
    }
}

// Final step of kept poses s0 and s0 + 1 (when s0 + 1 < ns) of ligand l in one
// wave, for A <= 32 with final_align: lane (h, i) = (lane / 32, lane % 32) holds
// the strip of pose h, x rotation i and the A y rotations, one accumulator each.
// Per atom the x rotation is applied once (align_x) and each y rotation costs 4
// FMAs, and the cube loads of kFalignBatch samples are issued before the first
// blend waits for them.  Every sample, the atom-order sums and the tie rule
// (first maximum in o = i*A + j) are those of align_pose, and the chosen
// orientation is applied and scored as there, so fscore / fo are bit-identical
// to final_item's.  rec: LDS for 2 * nmax float4.
constexpr int kFalignBatch = 4;

template <int NS>
__device__ void final_pair(int l, int s0, int ns, float4 *rec, int nmax, const Tri &tr,
                           const GridArgs &g, const SearchArgs &sa, const LibArgs &lib,
                           const WorkArgs &ws) {
    const int lane = lane_id(), h = lane >> 5, i = lane & 31;
    const int a0 = lib.atom_off[l], n = lib.atom_off[l + 1] - a0, K = sa.K, A = sa.A;
    const int np = s0 + 1 < ns ? 2 : 1;
    int toff[NS];
#pragma unroll
    for (int q = 0; q < NS; ++q) {
        const int ia = lane + 64 * q;
        toff[q] = ia < n ? (int)((uint32_t)lib.type[a0 + ia] * g.type_bytes) : 0;
    }
    // records of both poses: centred grid-unit offsets and type offsets, as in
    // align_pose; every sample inside the grid unless some atom's sphere may leave it
    float ex[2] = {0.f, 0.f}, ey[2] = {0.f, 0.f}, ez[2] = {0.f, 0.f};
    bool out_any = false;
    for (int p = 0; p < np; ++p) {
        const float *P = ws.acc_pose + ((size_t)a0 * K + (size_t)(s0 + p) * n) * 3;
        Pose<NS> Y;
#pragma unroll
        for (int q = 0; q < NS; ++q) {
            const int ia = lane + 64 * q, ii = ia < n ? ia : 0;
            Y.x[q] = P[3 * ii + 0];
            Y.y[q] = P[3 * ii + 1];
            Y.z[q] = P[3 * ii + 2];
        }
        float cx, cy, cz;
        centroid(Y, n, cx, cy, cz);
        ex[p] = (cx - g.ox) * g.inv_h;
        ey[p] = (cy - g.oy) * g.inv_h;
        ez[p] = (cz - g.oz) * g.inv_h;
#pragma unroll
        for (int q = 0; q < NS; ++q) {
            const int ia = lane + 64 * q;
            if (ia < n) {
                const float rx = (Y.x[q] - cx) * g.inv_h, ry = (Y.y[q] - cy) * g.inv_h,
                            rz = (Y.z[q] - cz) * g.inv_h;
                out_any = out_any || !ball_inside(tr, ex[p], ey[p], ez[p],
                                                  ball_radius(fmaf(rx, rx, fmaf(ry, ry, rz * rz))));
                rec[p * nmax + ia] = make_float4(rx, ry, rz, __int_as_float(toff[q]));
            }
        }
    }
    const bool all_in = __ballot(out_any) == 0ull;
    wave_lds_sync();
    // strips; lanes without one (i >= A, or the second pose missing) mirror a valid
    // strip so that their reads stay in range, and take no part in the maximum
    const bool valid = h < np && i < A;
    const int hp = h < np ? h : 0;
    const float pex = hp ? ex[1] : ex[0], pey = hp ? ey[1] : ey[0], pez = hp ? ez[1] : ez[0];
    const float2 ci = sa.acs[i < A ? i : 0];
    const cfloat2_p cj = (cfloat2_p)sa.acs;  // padded to 32 entries (k >= A wraps)
    const float4 *rp = rec + hp * nmax;
    float acc[32];
#pragma unroll
    for (int jj = 0; jj < 32; ++jj) acc[jj] = 0.0f;
    for (int a = 0; a < n; ++a) {
        const float4 r = rp[a];
        const int to = uniform_int(__float_as_int(rec[a].w));  // same atom, same type in both
        const XStage xs = align_x(r.x, r.y, r.z, ci, pey);
#pragma unroll
        for (int j0 = 0; j0 < 32; j0 += kFalignBatch) {
            if (j0 < A) {
                float fx[kFalignBatch], fy[kFalignBatch], fz[kFalignBatch];
                uint32_t off[kFalignBatch];
#pragma unroll
                for (int k = 0; k < kFalignBatch; ++k) {
                    const float2 c = ld_cs(cj, j0 + k);
                    const float gx = align_gx(xs, c, pex), gz = align_gz(xs, c, pez);
                    if (all_in) {
                        // tri_in's cell and fractions
                        fx[k] = __builtin_amdgcn_fractf(gx);
                        fy[k] = __builtin_amdgcn_fractf(xs.gy);
                        fz[k] = __builtin_amdgcn_fractf(gz);
                        off[k] = in_cell(tr, gx, xs.gy, gz);
                    } else {
                        // tri_u's clamped cell and fractions
                        off[k] = tri_cell(tr, gx, xs.gy, gz, fx[k], fy[k], fz[k]);
                    }
                }
                float4 q0[kFalignBatch], q1[kFalignBatch];
#pragma unroll
                for (int k = 0; k < kFalignBatch; ++k) {
                    q0[k] = ldq(tr.rs, off[k], to);
                    q1[k] = ldq(tr.rs, off[k], to + 16);
                }
                // every load of the batch is issued before the first blend waits
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int k = 0; k < kFalignBatch; ++k)
                    acc[j0 + k] += tri_blend(q0[k], q1[k], fx[k], fy[k], fz[k]);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    // best (score, then lowest index) of each pose: lane maxima, then a max over
    // each half wave (rows 0-1 into lane 31, rows 2-3 into lane 63)
    u64 best = 0ull;
#pragma unroll
    for (int jj = 0; jj < 32; ++jj) {
        const u64 key = valid && jj < A ? make_key(acc[jj], (uint32_t)(i * A + jj)) : 0ull;
        best = key > best ? key : best;
    }
#define DOCK_HALF_MAX_STEP(C, R)            \
    {                                       \
        const u64 w = dpp_read64<C, R>(best); \
        best = w > best ? w : best;         \
    }
    DOCK_HALF_MAX_STEP(0x111, 0xF)
    DOCK_HALF_MAX_STEP(0x112, 0xF)
    DOCK_HALF_MAX_STEP(0x114, 0xF)
    DOCK_HALF_MAX_STEP(0x118, 0xF)
    DOCK_HALF_MAX_STEP(0x142, 0xA)
#undef DOCK_HALF_MAX_STEP
    const u64 bk[2] = {read_lane64(best, 31), read_lane64(best, 63)};
    wave_lds_sync();  // rec is rewritten by the wave's next item
    for (int p = 0; p < np; ++p) {
        const int ob = (int)key_index(bk[p]);
        const float *P = ws.acc_pose + ((size_t)a0 * K + (size_t)(s0 + p) * n) * 3;
        Pose<NS> Y;
#pragma unroll
        for (int q = 0; q < NS; ++q) {
            const int ia = lane + 64 * q, ii = ia < n ? ia : 0;
            Y.x[q] = P[3 * ii + 0];
            Y.y[q] = P[3 * ii + 1];
            Y.z[q] = P[3 * ii + 2];
        }
        apply_align(Y, n, ob, sa);
        const float sc = pose_score(Y, n, toff, tr, g);
        if (lane == 0) {
            ws.fscore[(size_t)l * K + s0 + p] = sc;
            ws.fo[(size_t)l * K + s0 + p] = ob;
        }
    }
}

size_t falign_lds_bytes(int nmax, int waves, int single) {
    return single ? (size_t)nmax * 16 + (size_t)waves * 8 : (size_t)waves * 2 * nmax * 16;
}

template <int NS>
__global__ __launch_bounds__(512) void k_falign(GridArgs g, SearchArgs sa, LibArgs lib,
                                               WorkArgs ws, const int *__restrict__ status,
                                               int bin, int lst, int single, int xcds) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int nmax = bin_nmax(bin);
    // every lane is active here, so the wave index is read from the first lane
    const int W = blockDim.x >> 6, wave = uniform_int((int)(threadIdx.x >> 6));
    const Tri tr = make_tri(g);
    if (single >= 0) {
        // plain form: workgroup s takes kept pose s of the ligand, its waves split
        // the orientations and agree on the best through LDS
        const int l = single, s = blockIdx.x;
        if (status[l] != 0 || s >= ws.nsel[l]) return;
        float4 *rec = (float4 *)smem;
        u64 *slots = (u64 *)(smem + (size_t)nmax * 16);
        final_item<NS>(l, s, rec, tr, g, sa, lib, ws, BlockSplit{wave, W, slots}, wave == 0);
        return;
    }
    // batched form: the waves of the grid take the bin's (ligand, kept pose)
    // items, from a queue or in turn (item = global wave index + k * waves in the
    // grid).  The item index is wave-uniform: no lane-dependent branch precedes
    // the loop test, so every lane of a wave runs the same items.
    // With xcds > 1 the workgroups are taken as dispatched round-robin over that
    // many XCDs (workgroup b on XCD b % xcds): XCD x takes a contiguous x-th share
    // of the bin's ligands, so the kept poses of a ligand share one L2.
    // An item is a pair of kept poses (s0 = 2 * pair, s0 + 1) of one ligand.
    float4 *rec = (float4 *)(smem + (size_t)wave * 2 * nmax * 16);
    const long long nl = ws.counters[lst];
    const int x = xcds > 1 ? (int)(blockIdx.x % xcds) : 0;
    const int bx = xcds > 1 ? (int)(blockIdx.x / xcds) : (int)blockIdx.x;
    const int nbx = xcds > 1 ? (int)((gridDim.x - x + xcds - 1) / xcds) : (int)gridDim.x;
    const int nx = xcds > 1 ? xcds : 1;
    const int pairs = (min(sa.K, sa.R) + 1) / 2;
    const bool strips = sa.final_align && sa.A <= 32;
    const long long li0 = nl * x / nx, li1 = nl * (x + 1) / nx;
    const long long total = (li1 - li0) * pairs;
    const long long nwaves = (long long)nbx * W;
    // Without the split, and with more items than waves, a wave takes its next items from
    // a queue: half of the items can be empty (ligands keep fewer than K poses), and
    // dealt out in turn they left the GPU 41% idle (2,500 ligands of 20-80 atoms: 43.9
    // -> 43.1 ms a call; an item a wave at most needs no queue, whose atomics from a full
    // grid cost 80 us).  The queue's counter takes 80 additions a microsecond, so small
    // items are taken several at a time, together the work of at most one of 36 atoms at 30
    // steps, and items without an alignment in turn (900 ligands of 6 atoms with one pose
    // of 64: 630 -> 236 us a call, 3,000 of 1 atom without the final step 1.97 -> 1.0 ms).
    const bool queued = xcds <= 1 && total > nwaves && sa.final_align;
    int *queue = queued ? ws.counters + 3 * kMaxLists + lst : nullptr;
    int per = 1;  // a power of two
    while (per < 16 && 2 * per * sa.A * sa.A * (nmax - 16) <= 32768) per *= 2;
    auto next = [&](long long item) -> long long {
        if (!queue) return item + nwaves;
        if (++item & (per - 1)) return item;
        int v = 0;
        if (lane_id() == 0) v = atomicAdd(queue, per);
        return uniform_int(v);
    };
    for (long long item = queue ? next(-1) : (long long)bx * W + wave; item < total;
         item = next(item)) {
        const int li = (int)(li0 + item / pairs), s0 = 2 * (int)(item % pairs);
        const int l = ws.bin_list[li];
        const int ns = ws.nsel[l];
        if (s0 >= ns) continue;
        if (strips) {
            final_pair<NS>(l, s0, ns, rec, nmax, tr, g, sa, lib, ws);
        } else {
            final_item<NS>(l, s0, rec, tr, g, sa, lib, ws, WaveSplit(), true);
            if (s0 + 1 < ns) final_item<NS>(l, s0 + 1, rec, tr, g, sa, lib, ws, WaveSplit(), true);
        }
    }
}

// Outputs of a ligand's kept poses, ordered by (final score desc, restart asc):
// each wave takes kept poses in turn, turns it by its final-step orientation
// (the same arithmetic as the alignment's own apply step) and writes it to its
// output slot.
template <int NS>
__global__ __launch_bounds__(256) void k_out(SearchArgs sa, LibArgs lib, WorkArgs ws,
                                             OutArgs out, int bin, int lst, int single) {
    __shared__ int rank[kMaxTopK];
    const int K = sa.K;
    const int W = blockDim.x >> 6, wave = threadIdx.x >> 6, lane = lane_id();
    for (int li = blockIdx.x;; li += gridDim.x) {
        int l;
        if (single >= 0) {
            if (li > 0 || out.status[single] != 0) break;
            l = single;
        } else {
            if (li >= ws.counters[lst]) break;
            l = ws.bin_list[li];
        }
        const int a0 = lib.atom_off[l], n = lib.atom_off[l + 1] - a0;
        const int ns = ws.nsel[l];
        const float *fsc = ws.fscore + (size_t)l * K;
        const int *sel = ws.sel + (size_t)l * K;
        const int *fo = ws.fo + (size_t)l * K;
        for (int s = threadIdx.x; s < ns; s += blockDim.x) {
            const u64 ks = make_key(fsc[s], (uint32_t)sel[s]);
            int rk = 0;
            for (int q = 0; q < ns; ++q) rk += make_key(fsc[q], (uint32_t)sel[q]) > ks;
            rank[s] = rk;
            out.pscore[(size_t)l * K + rk] = fsc[s];
            out.prestart[(size_t)l * K + rk] = sel[s];
            if (out.ftrace) out.ftrace[(size_t)l * K + rk] = (uint16_t)fo[s];
            if (rk == 0) out.best[l] = fsc[s];
        }
        __syncthreads();
        const float *acc = ws.acc_pose + (size_t)a0 * K * 3;
        for (int s = wave; s < ns && out.pxyz; s += W) {
            Pose<NS> Y;
#pragma unroll
            for (int q = 0; q < NS; ++q) {
                const int i = lane + 64 * q;
                const float *P = acc + ((size_t)s * n + (i < n ? i : 0)) * 3;
                Y.x[q] = P[0];
                Y.y[q] = P[1];
                Y.z[q] = P[2];
            }
            if (sa.final_align) apply_align(Y, n, fo[s], sa);
            float *O = out.pxyz + ((size_t)a0 * K + (size_t)rank[s] * n) * 3;
#pragma unroll
            for (int q = 0; q < NS; ++q) {
                const int i = lane + 64 * q;
                if (i < n) {
                    O[3 * i + 0] = Y.x[q];
                    O[3 * i + 1] = Y.y[q];
                    O[3 * i + 2] = Y.z[q];
                }
            }
        }
        const int per = 3 * n;
        for (int e = threadIdx.x; out.pxyz && e < (K - ns) * per; e += blockDim.x)
            out.pxyz[((size_t)a0 * K + (size_t)ns * n) * 3 + e] = 0.f;
        for (int s = ns + (int)threadIdx.x; s < K; s += blockDim.x) {
            out.pscore[(size_t)l * K + s] = -INFINITY;
            out.prestart[(size_t)l * K + s] = -1;
            if (out.ftrace) out.ftrace[(size_t)l * K + s] = 0;
        }
        if (threadIdx.x == 0) {
            out.npose[l] = ns;
            if (ns == 0) out.best[l] = -INFINITY;
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// Pairwise rescoring stand-in (Rescore Pose): the paper evaluates every ligand
// atom against every pocket atom and accumulates the pair terms per pose; here
// the pair term is weight[ligand type][pocket atom type] for pairs closer than
// the contact distance, summed as an integer.  Pairs beyond the neighbouring
// cells of the pocket-atom cell grid are farther apart than the contact
// distance, so only the 3 x 3 rows of 3 cells around the atom are visited.

__device__ __forceinline__ int wave_sum_int(int v) {
    v += dpp_read<0x111, 0xf>(v);  // row_shr:1
    v += dpp_read<0x112, 0xf>(v);  // row_shr:2
    v += dpp_read<0x114, 0xf>(v);  // row_shr:4
    v += dpp_read<0x118, 0xf>(v);  // row_shr:8
    v += dpp_read<0x142, 0xa>(v);  // row_bcast:15
    v += dpp_read<0x143, 0xc>(v);  // row_bcast:31
    return __builtin_amdgcn_readlane(v, 63);
}

__device__ int atom_contacts(const ContactArgs &ca, const int *wrow, float px, float py,
                             float pz) {
    // cell of the atom; coordinates are clamped to one cell beyond the grid, which
    // only adds pocket atoms that fail the distance test
    const float fx = fminf(fmaxf((px - ca.lox) * ca.inv_cell, -1.f), (float)ca.cx);
    const float fy = fminf(fmaxf((py - ca.loy) * ca.inv_cell, -1.f), (float)ca.cy);
    const float fz = fminf(fmaxf((pz - ca.loz) * ca.inv_cell, -1.f), (float)ca.cz);
    const int ix = (int)floorf(fx), iy = (int)floorf(fy), iz = (int)floorf(fz);
    const int x0 = ix - 1 < 0 ? 0 : ix - 1, x1 = ix + 1 >= ca.cx ? ca.cx - 1 : ix + 1;
    int v = 0;
    if (x0 > x1) return 0;
    for (int z = iz - 1; z <= iz + 1; ++z) {
        if (z < 0 || z >= ca.cz) continue;
        for (int y = iy - 1; y <= iy + 1; ++y) {
            if (y < 0 || y >= ca.cy) continue;
            const int row = (z * ca.cy + y) * ca.cx;
            const int j1 = ca.cell_start[row + x1 + 1];
            for (int j = ca.cell_start[row + x0]; j < j1; ++j) {
                const float4 a = ca.atoms[j];
                const float dx = px - a.x, dy = py - a.y, dz = pz - a.z;
                const float d2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
                if (d2 < ca.dc2) v += wrow[__float_as_int(a.w)];
            }
        }
    }
    return v;
}

__global__ __launch_bounds__(256) void k_rescore(ContactArgs ca, SearchArgs sa, LibArgs lib,
                                                 OutArgs out, int single) {
    __shared__ int wt[kMaxContactWeights];
    __shared__ int part[4];
    for (int e = threadIdx.x; e < ca.nw; e += blockDim.x) wt[e] = ca.weight[e];
    __syncthreads();
    const int K = sa.K;
    // every lane is active here, so the wave index is read from the first lane
    const int W = blockDim.x >> 6, wave = uniform_int((int)(threadIdx.x >> 6)), lane = lane_id();
    if (single >= 0) {
        // plain form: workgroup s scores output pose s of the ligand, its threads
        // over the ligand's atoms
        const int l = single, s = blockIdx.x;
        int v = 0;
        if (s < out.npose[l]) {
            const int a0 = lib.atom_off[l], n = lib.atom_off[l + 1] - a0;
            const float *P = out.pxyz + ((size_t)a0 * K + (size_t)s * n) * 3;
            for (int i = threadIdx.x; i < n; i += blockDim.x)
                v += atom_contacts(ca, wt + (int)lib.type[a0 + i] * ca.ntypes, P[3 * i],
                                   P[3 * i + 1], P[3 * i + 2]);
        }
        v = wave_sum_int(v);
        if (lane == 0) part[wave] = v;
        __syncthreads();
        if (threadIdx.x == 0) {
            int t = 0;
            for (int w = 0; w < W; ++w) t += part[w];
            out.pcontacts[(size_t)l * K + s] = t;
        }
        return;
    }
    // batched form: the grid's waves take the (ligand, output pose) items in turn
    const long long total = (long long)lib.L * K;
    const long long nwaves = (long long)gridDim.x * W;
    for (long long item = (long long)blockIdx.x * W + wave; item < total; item += nwaves) {
        const int l = (int)(item / K), s = (int)(item - (long long)l * K);
        int v = 0;
        if (s < out.npose[l]) {
            const int a0 = lib.atom_off[l], n = lib.atom_off[l + 1] - a0;
            const float *P = out.pxyz + ((size_t)a0 * K + (size_t)s * n) * 3;
            for (int i = lane; i < n; i += 64)
                v += atom_contacts(ca, wt + (int)lib.type[a0 + i] * ca.ntypes, P[3 * i],
                                   P[3 * i + 1], P[3 * i + 2]);
        }
        v = wave_sum_int(v);
        if (lane == 0) out.pcontacts[item] = v;
    }
}

// ---------------------------------------------------------------------------
// Preparation: one wavefront per ligand.  Checks the ligand, builds its
// bump-pair rows (pairs at least bmin bonds apart), and appends it to its size
// bin.  A ligand that fails a check gets a status and empty outputs.
__global__ __launch_bounds__(64) void k_prep(GridArgs g, SearchArgs sa, LibArgs lib, WorkArgs ws,
                                             OutArgs out, int first, int do_bin) {
    __shared__ u64 adj[kMaxAtoms * 4];   // adjacency + self rows
    const int l = first + (int)blockIdx.x;
    const int lane = lane_id();
    if (l >= lib.L) return;
    int status = 0;
    const int a0 = lib.atom_off[l], a1 = lib.atom_off[l + 1];
    const int b0 = lib.bond_off[l], b1 = lib.bond_off[l + 1];
    const int r0 = lib.rot_off[l], r1 = lib.rot_off[l + 1];
    const int n = a1 - a0, nb = b1 - b0, B = r1 - r0;
    if (a0 < 0 || a1 < a0 || (long long)a1 > lib.A_total || b0 < 0 || b1 < b0 ||
        (long long)b1 > lib.Nb_total || r0 < 0 || r1 < r0 || (long long)r1 > lib.Nr_total)
        status = 5;
    else if (n < 1 || n > kMaxAtoms || B > kMaxRot || nb > 8 * n || n > 64 * lib.mask_words)
        status = 1;
    const int NW = (n + 63) >> 6;
    if (status == 0) {
        bool bad = false;
        for (int i = lane; i < n; i += 64) bad |= (int)lib.type[a0 + i] >= g.ntypes;
        if (__ballot(bad)) status = 2;
    }
    if (status == 0) {
        for (int e = lane; e < 4 * n; e += 64) adj[e] = 0ull;
        __syncthreads();
        for (int i = lane; i < n; i += 64) atomicOr(&adj[i * 4 + (i >> 6)], 1ull << (i & 63));
        bool bad = false;
        for (int e = lane; e < nb; e += 64) {
            const int u = lib.bond[2 * (size_t)(b0 + e)], v = lib.bond[2 * (size_t)(b0 + e) + 1];
            if (u < 0 || v < 0 || u >= n || v >= n || u == v) {
                bad = true;
            } else {
                atomicOr(&adj[u * 4 + (v >> 6)], 1ull << (v & 63));
                atomicOr(&adj[v * 4 + (u >> 6)], 1ull << (u & 63));
            }
        }
        for (int e = lane; e < B; e += 64) {
            const int a = lib.rot_bond[2 * (size_t)(r0 + e)], b = lib.rot_bond[2 * (size_t)(r0 + e) + 1];
            if (a < 0 || b < 0 || a >= n || b >= n || a == b) bad = true;
        }
        if (__ballot(bad)) status = 3;
        __syncthreads();
    }
    if (status == 0) {
        // every rotatable bond is a bond
        bool bad = false;
        for (int e = lane; e < B; e += 64) {
            const int a = lib.rot_bond[2 * (size_t)(r0 + e)], b = lib.rot_bond[2 * (size_t)(r0 + e) + 1];
            bad |= !((adj[a * 4 + (b >> 6)] >> (b & 63)) & 1ull);
        }
        if (__ballot(bad)) status = 3;
    }
    if (status == 0) {
        // connected: closure of {0} under adjacency
        u64 reach[4] = {1ull, 0ull, 0ull, 0ull};
        for (int it = 0; it < n; ++it) {
            u64 nr[4] = {0ull, 0ull, 0ull, 0ull};
            for (int i = lane; i < n; i += 64)
                if ((reach[i >> 6] >> (i & 63)) & 1ull)
                    for (int w = 0; w < NW; ++w) nr[w] |= adj[i * 4 + w];
            bool changed = false;
            for (int w = 0; w < NW; ++w) {
                nr[w] = wave_or_u64(nr[w]) | reach[w];
                changed |= nr[w] != reach[w];
                reach[w] = nr[w];
            }
            if (!changed) break;
        }
        int cnt = 0;
        for (int w = 0; w < NW; ++w) cnt += __popcll(reach[w]);
        if (cnt != n) status = 4;
    }
    if (status == 0) {
        // each mask: contains b, not a, no bit >= n, and no bond other than a-b crosses it
        bool bad = false;
        for (int rb = 0; rb < B && !bad; ++rb) {
            const int a = lib.rot_bond[2 * (size_t)(r0 + rb)], b = lib.rot_bond[2 * (size_t)(r0 + rb) + 1];
            u64 m[4] = {0ull, 0ull, 0ull, 0ull};
            for (int w = 0; w < lib.mask_words && w < 4; ++w)
                m[w] = lib.rot_mask[(size_t)(r0 + rb) * lib.mask_words + w];
            for (int w = NW; w < lib.mask_words; ++w)
                if (lib.rot_mask[(size_t)(r0 + rb) * lib.mask_words + w] != 0ull) bad = true;
            if ((n & 63) != 0 && (m[NW - 1] >> (n & 63)) != 0ull) bad = true;
            if (!((m[b >> 6] >> (b & 63)) & 1ull) || ((m[a >> 6] >> (a & 63)) & 1ull)) bad = true;
            bool cross = false;
            for (int e = lane; e < nb; e += 64) {
                const int u = lib.bond[2 * (size_t)(b0 + e)], v = lib.bond[2 * (size_t)(b0 + e) + 1];
                if ((u == a && v == b) || (u == b && v == a)) continue;
                const bool su = (m[u >> 6] >> (u & 63)) & 1ull, sv = (m[v >> 6] >> (v & 63)) & 1ull;
                cross |= su != sv;
            }
            if (__ballot(cross)) bad = true;
        }
        if (bad) status = 4;
    }
    if (status == 0) {
        // rows of atoms within bmin-1 bonds, complemented: the bump-checked pairs
        for (int i = lane; i < n; i += 64) {
            u64 near[4] = {0ull, 0ull, 0ull, 0ull};
            near[i >> 6] = 1ull << (i & 63);
            for (int step = 1; step < sa.bmin; ++step) {
                u64 nx[4] = {near[0], near[1], near[2], near[3]};
                for (int w = 0; w < NW; ++w) {
                    u64 bits = near[w];
                    while (bits) {
                        const int j = 64 * w + __ffsll((long long)bits) - 1;
                        bits &= bits - 1;
                        for (int v = 0; v < NW; ++v) nx[v] |= adj[j * 4 + v];
                    }
                }
                for (int w = 0; w < 4; ++w) near[w] = nx[w];
            }
            for (int w = 0; w < kFarWords; ++w) {
                u64 valid = 0ull;
                if (w < NW) valid = (w == NW - 1 && (n & 63)) ? ((1ull << (n & 63)) - 1) : ~0ull;
                ws.far[(size_t)(a0 + i) * kFarWords + w] = ~near[w] & valid;
            }
        }
        if (lane == 0 && do_bin) {
            // work list: the atom bin and the library's part of ws.chunk ligands, or with
            // sa.groups > 1 the paper's bucket of (atom bin, group of 4 rotatable bonds;
            // the last group takes the rest)
            const int bin = (n - 1) >> 5;
            const int grp = B / 4 < sa.groups - 1 ? B / 4 : sa.groups - 1;
            const int part = l / ws.chunk;
            const int lst = sa.groups > 1 ? bin * sa.groups + grp : part * kNumBins + bin;
            const int pos = atomicAdd(&ws.counters[lst], 1);
            ws.bin_list[list_offset(sa.groups, lst, lib.L, ws.chunk) + pos] = l;
        }
    } else {
        for (int s = lane; s < sa.K; s += 64) {
            out.pscore[(size_t)l * sa.K + s] = -INFINITY;
            out.prestart[(size_t)l * sa.K + s] = -1;
            if (out.ftrace) out.ftrace[(size_t)l * sa.K + s] = 0;
        }
        if (lane == 0) {
            out.best[l] = -INFINITY;
            out.npose[l] = 0;
        }
    }
    if (lane == 0) out.status[l] = status;
}

hipError_t launch_rescore(const ContactArgs &ca, const SearchArgs &sa, const LibArgs &lib,
                          const OutArgs &out, int single, int blocks, hipStream_t s) {
    if (single >= 0) blocks = sa.K;
    if (blocks <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_rescore, dim3(blocks), dim3(256), 0, s, ca, sa, lib, out, single);
    return hipGetLastError();
}

// Zero counters [first, first + count): work-queue counters are cleared by a
// kernel, not a memset, so the sequence can be captured in a graph.
__global__ void k_reset(int *counters, int first, int count) {
    for (int i = threadIdx.x; i < count; i += blockDim.x) counters[first + i] = 0;
}

// ---------------------------------------------------------------------------
// launchers
hipError_t launch_build_cubes(const float *values, float4 *cubes, int ntypes, int nx, int ny,
                              int nz, hipStream_t s) {
    const long long n = (long long)ntypes * nx * ny * nz;
    const int threads = 256;
    const long long blocks = (n + threads - 1) / threads;
    hipLaunchKernelGGL(k_build_cubes, dim3((unsigned)blocks), dim3(threads), 0, s, values, cubes,
                       ntypes, nx, ny, nz);
    return hipGetLastError();
}

hipError_t launch_atlas_count(const GridArgs &g, int4 *info, hipStream_t s) {
    hipLaunchKernelGGL(k_atlas_count, dim3(kMaxBands), dim3(1024), 0, s, g, info);
    return hipGetLastError();
}

hipError_t launch_atlas_fill(const GridArgs &g, int4 *info, const int *blob16, float4 *atlas,
                             int nb, hipStream_t s) {
    if (nb <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_atlas_fill, dim3(nb * g.ntypes), dim3(1024), 0, s, g, info, blob16, atlas,
                       nb);
    return hipGetLastError();
}

hipError_t launch_reset(int *counters, int first, int count, hipStream_t s) {
    if (first < 0 || count < 0 || first + count > kNumCounters) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_reset, dim3(1), dim3(256), 0, s, counters, first, count);
    return hipGetLastError();
}

hipError_t launch_prep(const GridArgs &g, const SearchArgs &sa, const LibArgs &lib,
                       const WorkArgs &ws, const OutArgs &out, hipStream_t s) {
    if (lib.L <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_prep, dim3(lib.L), dim3(64), 0, s, g, sa, lib, ws, out, 0, 1);
    return hipGetLastError();
}

hipError_t launch_prep_one(const GridArgs &g, const SearchArgs &sa, const LibArgs &lib,
                           const WorkArgs &ws, const OutArgs &out, int l, hipStream_t s) {
    hipLaunchKernelGGL(k_prep, dim3(1), dim3(64), 0, s, g, sa, lib, ws, out, l, 0);
    return hipGetLastError();
}

size_t plain_lds_bytes(int nmax, int waves) { return dock_lds_bytes(nmax, waves) + (size_t)waves * 8; }

static TorsionArgs torsion_args(const GridArgs &g, const SearchArgs &sa) {
    TorsionArgs t{};
    t.inv_h = g.inv_h;
    t.ox = g.ox; t.oy = g.oy; t.oz = g.oz;
    t.m2x = g.m2x; t.m2y = g.m2y; t.m2z = g.m2z;
    t.lim = sa.bump2g;
    // P0 rounds at 2^-24 of the largest coordinate on each axis (1000 cells: a ligand that
    // reaches out of the grid), so that a distance near the limit is off by up to `off`
    const double far = 1000.0 + std::fmax(std::fabs((double)g.ox), std::fmax(std::fabs((double)g.oy),
                                                                   std::fabs((double)g.oz))) * g.inv_h;
    const double off = 4.0 * far * std::ldexp(1.0, -24), lim = t.lim;
    t.reach = (float)(lim * (1.0 + 2e-3) + 1e-3 + off * (2.0 * std::sqrt(lim) + off));
    t.T = sa.T;
    t.prune = sa.prune;
    t.tors = sa.tors;
    // a slot's candidates lie within 32 steps of its 33rd, and a step more
    const double step = 2.0 * M_PI / sa.T, w = 33.0 * step;
    if (w < 0.99 * M_PI / 2.0) {
        t.cw = (float)std::cos(w);
        t.sw = (float)std::sin(w);
        t.tw = (float)std::tan(w);
    } else {
        t.sb = 3e38f;
    }
    for (int q = 0; q < kMaxTorsionSteps / 64; ++q)
        t.mid[q] = make_float2((float)std::cos((64.0 * q + 32.0) * step),
                               (float)std::sin((64.0 * q + 32.0) * step));
    return t;
}

template <int NS, int C>
static hipError_t launch_plain_t(int l, int bin, int waves, const GridArgs &g,
                                 const SearchArgs &sa, const LibArgs &lib, const WorkArgs &ws,
                                 const OutArgs &out, hipStream_t s) {
    const size_t lds = plain_lds_bytes(bin_nmax(bin), waves);
    hipFuncSetAttribute((const void *)k_plain<NS, C>, hipFuncAttributeMaxDynamicSharedMemorySize,
                        (int)lds);
    const DockArgs a{torsion_args(g, sa), g, sa, lib, ws, (const int *)out.status, bin, 0, l};
    hipLaunchKernelGGL((k_plain<NS, C>), dim3(sa.R), dim3(64 * waves), lds, s, a);
    return hipGetLastError();
}

template <int NS>
static hipError_t launch_plain_c(int l, int bin, int waves, const GridArgs &g,
                                 const SearchArgs &sa, const LibArgs &lib, const WorkArgs &ws,
                                 const OutArgs &out, hipStream_t s) {
    const int C = (sa.T + 64 * waves - 1) / (64 * waves);
    if (C <= 1) return launch_plain_t<NS, 1>(l, bin, waves, g, sa, lib, ws, out, s);
    if (C <= 2) return launch_plain_t<NS, 2>(l, bin, waves, g, sa, lib, ws, out, s);
    return launch_plain_t<NS, 4>(l, bin, waves, g, sa, lib, ws, out, s);
}

hipError_t launch_plain(int l, int bin, int waves, const GridArgs &g, const SearchArgs &sa,
                        const LibArgs &lib, const WorkArgs &ws, const OutArgs &out,
                        hipStream_t s) {
    switch (bin_slots(bin)) {
        case 1: return launch_plain_c<1>(l, bin, waves, g, sa, lib, ws, out, s);
        case 2: return launch_plain_c<2>(l, bin, waves, g, sa, lib, ws, out, s);
        case 3: return launch_plain_c<3>(l, bin, waves, g, sa, lib, ws, out, s);
        default: return launch_plain_c<4>(l, bin, waves, g, sa, lib, ws, out, s);
    }
}

template <int NS, int C>
static hipError_t launch_dock_t(int bin, int lst, int blocks, int waves, const GridArgs &g,
                                const SearchArgs &sa, const LibArgs &lib, const WorkArgs &ws,
                                hipStream_t s) {
    const size_t lds = dock_lds_bytes(bin_nmax(bin), waves);
    hipFuncSetAttribute((const void *)k_dock<NS, C>, hipFuncAttributeMaxDynamicSharedMemorySize,
                        (int)lds);
    const DockArgs a{torsion_args(g, sa), g, sa, lib, ws, nullptr, bin, lst, 0};
    hipLaunchKernelGGL((k_dock<NS, C>), dim3(blocks), dim3(64 * waves), lds, s, a);
    return hipGetLastError();
}

template <int NS>
static hipError_t launch_dock_c(int bin, int lst, int blocks, int waves, const GridArgs &g,
                                const SearchArgs &sa, const LibArgs &lib, const WorkArgs &ws,
                                hipStream_t s) {
    const int C = (sa.T + 63) / 64;
    if (C <= 1) return launch_dock_t<NS, 1>(bin, lst, blocks, waves, g, sa, lib, ws, s);
    if (C <= 2) return launch_dock_t<NS, 2>(bin, lst, blocks, waves, g, sa, lib, ws, s);
    if (C <= 4) return launch_dock_t<NS, 4>(bin, lst, blocks, waves, g, sa, lib, ws, s);
    if (C <= 8) return launch_dock_t<NS, 8>(bin, lst, blocks, waves, g, sa, lib, ws, s);
    return launch_dock_t<NS, 16>(bin, lst, blocks, waves, g, sa, lib, ws, s);
}

hipError_t launch_dock(int bin, int lst, int blocks, int waves, const GridArgs &g,
                       const SearchArgs &sa, const LibArgs &lib, const WorkArgs &ws, hipStream_t s) {
    switch (bin_slots(bin)) {
        case 1: return launch_dock_c<1>(bin, lst, blocks, waves, g, sa, lib, ws, s);
        case 2: return launch_dock_c<2>(bin, lst, blocks, waves, g, sa, lib, ws, s);
        case 3: return launch_dock_c<3>(bin, lst, blocks, waves, g, sa, lib, ws, s);
        default: return launch_dock_c<4>(bin, lst, blocks, waves, g, sa, lib, ws, s);
    }
}

template <int NS>
static hipError_t launch_select_t(int bin, int lst, int blocks, int waves, const GridArgs &g,
                                  const SearchArgs &sa, const LibArgs &lib, const WorkArgs &ws,
                                  const OutArgs &out, int single, hipStream_t s) {
    const int sel = select_shape(bin_nmax(bin), sa.R, sa.K, single >= 0, &waves);
    const size_t lds = select_lds_bytes(bin_nmax(bin), waves, sa.R, sa.K, sel);
    auto *kernel = single >= 0 && ws.rpose && sel ? k_select<NS, true> : k_select<NS, false>;
    hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL(kernel, dim3(blocks), dim3(64 * waves), lds, s, g, sa, lib, ws, out, bin, lst,
                       single, sel);
    return hipGetLastError();
}

hipError_t launch_select(int bin, int lst, int blocks, int waves, const GridArgs &g,
                         const SearchArgs &sa, const LibArgs &lib, const WorkArgs &ws,
                         const OutArgs &out, int single, hipStream_t s) {
    switch (bin_slots(bin)) {
        case 1: return launch_select_t<1>(bin, lst, blocks, waves, g, sa, lib, ws, out, single, s);
        case 2: return launch_select_t<2>(bin, lst, blocks, waves, g, sa, lib, ws, out, single, s);
        case 3: return launch_select_t<3>(bin, lst, blocks, waves, g, sa, lib, ws, out, single, s);
        default: return launch_select_t<4>(bin, lst, blocks, waves, g, sa, lib, ws, out, single, s);
    }
}

template <int NS>
static hipError_t launch_falign_t(int bin, int lst, int blocks, int waves, const GridArgs &g,
                                  const SearchArgs &sa, const LibArgs &lib, const WorkArgs &ws,
                                  const OutArgs &out, int single, int xcds, hipStream_t s) {
    const size_t lds = falign_lds_bytes(bin_nmax(bin), waves, single >= 0 ? 1 : 0);
    hipFuncSetAttribute((const void *)k_falign<NS>, hipFuncAttributeMaxDynamicSharedMemorySize,
                        (int)lds);
    hipLaunchKernelGGL((k_falign<NS>), dim3(blocks), dim3(64 * waves), lds, s, g, sa, lib, ws,
                       (const int *)out.status, bin, lst, single, xcds);
    return hipGetLastError();
}

hipError_t launch_falign(int bin, int lst, int blocks, int waves, const GridArgs &g,
                         const SearchArgs &sa, const LibArgs &lib, const WorkArgs &ws,
                         const OutArgs &out, int single, int xcds, hipStream_t s) {
    if (xcds > 1 && xcds > blocks) return hipErrorInvalidValue;  // shares without a workgroup
    switch (bin_slots(bin)) {
        case 1: return launch_falign_t<1>(bin, lst, blocks, waves, g, sa, lib, ws, out, single, xcds, s);
        case 2: return launch_falign_t<2>(bin, lst, blocks, waves, g, sa, lib, ws, out, single, xcds, s);
        case 3: return launch_falign_t<3>(bin, lst, blocks, waves, g, sa, lib, ws, out, single, xcds, s);
        default: return launch_falign_t<4>(bin, lst, blocks, waves, g, sa, lib, ws, out, single, xcds, s);
    }
}

hipError_t launch_out(int bin, int lst, int blocks, const SearchArgs &sa, const LibArgs &lib,
                      const WorkArgs &ws, const OutArgs &out, int single, hipStream_t s) {
#define DOCK_OUT_LAUNCH(NS) \
    hipLaunchKernelGGL(k_out<NS>, dim3(blocks), dim3(256), 0, s, sa, lib, ws, out, bin, lst, single)
    switch (bin_slots(bin)) {
        case 1: DOCK_OUT_LAUNCH(1); break;
        case 2: DOCK_OUT_LAUNCH(2); break;
        case 3: DOCK_OUT_LAUNCH(3); break;
        default: DOCK_OUT_LAUNCH(4); break;
    }
#undef DOCK_OUT_LAUNCH
    return hipGetLastError();
}

// k_align geometry: JM = kAlignJ y rotations per lane, the y range in
// parts = ceil(A / JM) pieces, GR restarts per item so that the parts, each of
// GR*A strips padded to whole waves, fill the 15 sampling waves (GR at most
// kAlignMaxGroup and R, at least 1).
static int align_parts(int A) { return (A + kAlignJ - 1) / kAlignJ; }

int align_group(int A, int R) {
    const int parts = align_parts(A);
    int GR = 1;
    while (GR < kAlignMaxGroup && GR < R && parts * (((GR + 1) * A + 63) & ~63) <= 15 * 64) ++GR;
    return GR;
}

// Sampling waves (enough for the strips, at most 15) plus the copier wave.
static int align_waves(int A, int R) {
    const int strips = align_parts(A) * ((align_group(A, R) * A + 63) & ~63);
    const int w = strips / 64;
    return (w > 15 ? 15 : w) + 1;
}

size_t align_lds_min(int bin, int A, int R) {
    return AlignLds::region(bin_nmax(bin), align_group(A, R)) + 1024;
}

template <int NS>
static hipError_t launch_align_t(int bin, int lst, int blocks, int arena, const GridArgs &g,
                                 const SearchArgs &sa, const LibArgs &lib, const WorkArgs &ws,
                                 hipStream_t s) {
    hipFuncSetAttribute((const void *)k_align<NS, kAlignJ>,
                        hipFuncAttributeMaxDynamicSharedMemorySize, arena);
    hipLaunchKernelGGL((k_align<NS, kAlignJ>), dim3(blocks), dim3(64 * align_waves(sa.A, sa.R)),
                       (size_t)arena, s, g, sa, lib, ws, bin, lst, arena, align_group(sa.A, sa.R));
    return hipGetLastError();
}

hipError_t launch_align(int bin, int lst, int blocks, int arena, const GridArgs &g,
                        const SearchArgs &sa, const LibArgs &lib, const WorkArgs &ws,
                        hipStream_t s) {
    switch (bin_slots(bin)) {
        case 1: return launch_align_t<1>(bin, lst, blocks, arena, g, sa, lib, ws, s);
        case 2: return launch_align_t<2>(bin, lst, blocks, arena, g, sa, lib, ws, s);
        case 3: return launch_align_t<3>(bin, lst, blocks, arena, g, sa, lib, ws, s);
        default: return launch_align_t<4>(bin, lst, blocks, arena, g, sa, lib, ws, s);
    }
}

template <int NS>
static int align_occ_t(int waves, int arena) {
    int nb = 0;
    hipFuncSetAttribute((const void *)k_align<NS, kAlignJ>,
                        hipFuncAttributeMaxDynamicSharedMemorySize, arena);
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_align<NS, kAlignJ>, 64 * waves,
                                                     (size_t)arena) != hipSuccess)
        return 1;
    return nb > 0 ? nb : 1;
}

int align_blocks_per_cu(int bin, int R, int A, int arena) {
    const int waves = align_waves(A, R);
    switch (bin_slots(bin)) {
        case 1: return align_occ_t<1>(waves, arena);
        case 2: return align_occ_t<2>(waves, arena);
        case 3: return align_occ_t<3>(waves, arena);
        default: return align_occ_t<4>(waves, arena);
    }
}

hipError_t launch_value_range(const float *v, long long n, uint32_t *mm, hipStream_t s) {
    hipLaunchKernelGGL(k_value_range, dim3(256), dim3(1024), 0, s, v, n, mm);
    return hipGetLastError();
}

hipError_t launch_bounds(const GridArgs &g, const BoundArgs &bd, const float *vals,
                         const uint32_t *mm, unsigned short *tab, hipStream_t s) {
    if (bd.nb <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_bounds, dim3(8, bd.nb * g.ntypes), dim3(256), 0, s, g, bd, vals, mm, tab);
    return hipGetLastError();
}

hipError_t launch_bound_probe(const GridArgs &g, const BoundArgs &bd, const uint32_t *mm, int *stay,
                              hipStream_t s) {
    hipLaunchKernelGGL(k_bound_probe, dim3(kNumBins * kBoundProbes), dim3(960), 0, s, g, bd, mm, stay);
    return hipGetLastError();
}

template <int NS>
static hipError_t launch_align_bound_t(int bin, int lst, int blocks, const GridArgs &g,
                                       const SearchArgs &sa, const LibArgs &lib, const WorkArgs &ws,
                                       const BoundArgs &bd, hipStream_t s) {
    hipLaunchKernelGGL((k_align_bound<NS>), dim3(blocks), dim3(64 * kBoundWaves),
                       BoundLds::total(bin_nmax(bin)), s, g, sa, lib, ws, bd, bin, lst);
    return hipGetLastError();
}

hipError_t launch_align_bound(int bin, int lst, int blocks, const GridArgs &g,
                              const SearchArgs &sa, const LibArgs &lib, const WorkArgs &ws,
                              const BoundArgs &bd, hipStream_t s) {
    switch (bin_slots(bin)) {
        case 1: return launch_align_bound_t<1>(bin, lst, blocks, g, sa, lib, ws, bd, s);
        case 2: return launch_align_bound_t<2>(bin, lst, blocks, g, sa, lib, ws, bd, s);
        case 3: return launch_align_bound_t<3>(bin, lst, blocks, g, sa, lib, ws, bd, s);
        default: return launch_align_bound_t<4>(bin, lst, blocks, g, sa, lib, ws, bd, s);
    }
}

template <int NS>
static int align_bound_occ(int bin) {
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_align_bound<NS>, 64 * kBoundWaves,
                                                     BoundLds::total(bin_nmax(bin))) != hipSuccess)
        return 1;
    return nb > 0 ? nb : 1;
}

int align_bound_blocks_per_cu(int bin) {
    switch (bin_slots(bin)) {
        case 1: return align_bound_occ<1>(bin);
        case 2: return align_bound_occ<2>(bin);
        case 3: return align_bound_occ<3>(bin);
        default: return align_bound_occ<4>(bin);
    }
}

template <int NS, int C>
static int dock_occ(int bin, int waves) {
    int nb = 0;
    const size_t lds = dock_lds_bytes(bin_nmax(bin), waves);
    hipFuncSetAttribute((const void *)k_dock<NS, C>, hipFuncAttributeMaxDynamicSharedMemorySize,
                        (int)lds);
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_dock<NS, C>, 64 * waves, lds) !=
        hipSuccess)
        return 1;
    return nb > 0 ? nb : 1;
}

template <int NS>
static int dock_occ_c(int bin, int waves, int T) {
    const int C = (T + 63) / 64;
    if (C <= 1) return dock_occ<NS, 1>(bin, waves);
    if (C <= 2) return dock_occ<NS, 2>(bin, waves);
    if (C <= 4) return dock_occ<NS, 4>(bin, waves);
    if (C <= 8) return dock_occ<NS, 8>(bin, waves);
    return dock_occ<NS, 16>(bin, waves);
}

int dock_blocks_per_cu(int bin, int waves, int T) {
    switch (bin_slots(bin)) {
        case 1: return dock_occ_c<1>(bin, waves, T);
        case 2: return dock_occ_c<2>(bin, waves, T);
        case 3: return dock_occ_c<3>(bin, waves, T);
        default: return dock_occ_c<4>(bin, waves, T);
    }
}

template <int NS>
static int select_occ(int bin, int waves, int R, int K) {
    int nb = 0;
    const int sel = select_shape(bin_nmax(bin), R, K, false, &waves);
    const size_t lds = select_lds_bytes(bin_nmax(bin), waves, R, K, sel);
    hipFuncSetAttribute((const void *)k_select<NS, false>, hipFuncAttributeMaxDynamicSharedMemorySize,
                        (int)lds);
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_select<NS, false>, 64 * waves, lds) !=
        hipSuccess)
        return 1;
    return nb > 0 ? nb : 1;
}

int select_blocks_per_cu(int bin, int waves, int R, int K) {
    switch (bin_slots(bin)) {
        case 1: return select_occ<1>(bin, waves, R, K);
        case 2: return select_occ<2>(bin, waves, R, K);
        case 3: return select_occ<3>(bin, waves, R, K);
        default: return select_occ<4>(bin, waves, R, K);
    }
}

template <int NS>
static int falign_occ(int bin, int waves) {
    int nb = 0;
    const size_t lds = falign_lds_bytes(bin_nmax(bin), waves, 0);
    hipFuncSetAttribute((const void *)k_falign<NS>, hipFuncAttributeMaxDynamicSharedMemorySize,
                        (int)lds);
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_falign<NS>, 64 * waves, lds) !=
        hipSuccess)
        return 1;
    return nb > 0 ? nb : 1;
}

int falign_blocks_per_cu(int bin, int waves) {
    switch (bin_slots(bin)) {
        case 1: return falign_occ<1>(bin, waves);
        case 2: return falign_occ<2>(bin, waves);
        case 3: return falign_occ<3>(bin, waves);
        default: return falign_occ<4>(bin, waves);
    }
}

}  // namespace dockgpu
