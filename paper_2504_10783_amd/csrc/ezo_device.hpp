// ezo_device.hpp -- device-side building blocks of the EI-ZO hot path on
// gfx950: Philox4x32-10, DH forward kinematics into LDS, and the workgroup
// "tile check" that decides collision for a tile of configurations.
//
// Two tiles: flags mode (FlagTile below) holds the link frames of a tile's
// configurations and skips every pair it can prove separated; signed-distance
// mode (TileSmem) holds every sphere centre as [sphere][config] float4, lane l
// of every wave working on configuration l % T, and the W waves split the
// obstacles into contiguous slices, whose records are wave-uniform and come
// through scalar loads.  Centres are kept in a frame whose origin is the
// centre of the obstacle cloud.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ezo {

// LDS (address space 3) views of generic pointers that point into the
// workgroup's LDS.  Through a generic pointer -- one that may also point to
// global memory, or any volatile access, which the compiler's address-space
// inference leaves alone -- every access is a flat instruction followed by a
// wait on both memory counters; through these it is a ds_* instruction.
template <class T>
using lds_ptr = __attribute__((address_space(3))) T*;
template <class T>
__device__ __forceinline__ lds_ptr<T> to_lds(T* p) { return (lds_ptr<T>)p; }

// Element i of an LDS array of int4 / int2 / float4, read as the compiler's
// native vectors (HIP's vector classes cannot be copied out of another
// address space).
typedef int lds_i4_t __attribute__((ext_vector_type(4)));
typedef int lds_i2_t __attribute__((ext_vector_type(2)));
typedef float lds_f4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ int4 lds_load(lds_ptr<const int4> p, int i) {
    const lds_i4_t v = ((lds_ptr<const lds_i4_t>)p)[i];
    return make_int4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ int2 lds_load(lds_ptr<const int2> p, int i) {
    const lds_i2_t v = ((lds_ptr<const lds_i2_t>)p)[i];
    return make_int2(v.x, v.y);
}
__device__ __forceinline__ float4 lds_load(lds_ptr<const float4> p, int i) {
    const lds_f4_t v = ((lds_ptr<const lds_f4_t>)p)[i];
    return make_float4(v.x, v.y, v.z, v.w);
}

constexpr int kMaxDof = 8;
constexpr float kHuge = 3.0e38f;

// ---------------------------------------------------------------------------
// Robot and obstacles as seen by kernels
// ---------------------------------------------------------------------------
struct RobotView {
    int dof;
    unsigned prismatic;        // bit j: joint j is prismatic (theta = 0, offset d_j + q_j)
    int n_spheres;
    int n_self;
    int n_blocks;
    int rec_bytes;             // of a configuration's record in a flags tile (16 rec_rows)
    int item_shift;            // lanes of a part pair there (item_lanes_log2)
    int deal_blocks;           // its part pairs when they are dealt out over the waves (see tile_self_pairs)
    const float4* dh;          // [kMaxDof] (a, d, cos alpha, sin alpha), zero past dof
    const int* link_begin;     // [dof + 1] spheres of link i: [link_begin[i], link_begin[i+1])
    const float4* sph;         // [S] local (x, y, z), r -- sorted by link
    const int2* pairs;         // [P] self pairs, indices into the sorted order, grouped by block, the sphere
                               // of the block's part a first
    const float4* lbound;      // [kPartsPerLink dof] bounding sphere of each part of a link (part
                               // p of link l = index kPartsPerLink l + p, a consecutive run of the
                               // link's spheres): centre in the link frame, radius
    const int4* blocks;        // [n_blocks] per part pair: (part a, part b, first pair, pair count)
    // boxes on links, sorted by link: box k = four float4 in the link frame,
    // (centre, h_x), (rotation row 0, h_y), (row 1, h_z), (row 2, bounding
    // radius |h|); the rotation's columns are the box axes
    int n_boxes;
    int n_box_pairs;
    const float4* box;         // [B][4]
    const int* box_begin;      // [dof + 1] boxes of link i: [box_begin[i], box_begin[i+1])
    const int2* box_pairs;     // [Q] box self pairs (sorted indices)
    const int* box_link;       // [B] link of each box (sorted order)
    const float4* image;       // the tables that a flags check copies into LDS (robot_stage_bytes)
};

// LDS rows of a tile's pose array: one per sphere, four per box.
__host__ __device__ inline int tile_slots(int n_spheres, int n_boxes) { return n_spheres + 4 * n_boxes; }

// Self-pair broad phase: each link's spheres split into kPartsPerLink parts
// (consecutive runs of its sphere list), each with its own bounding sphere;
// a work item (configuration, part pair) is taken by 16 lanes, by 8 or 4 when that
// is all the sphere pairs that a part pair has on average (16 left most lanes of an
// arm of 30 spheres and 267 pairs idle: 262 144 checks among 40 obstacles 106 and
// 84 us).
constexpr int kPartsPerLink = 2;
__host__ __device__ inline int item_lanes_log2(int n_self, int n_blocks) {
    return n_self > 8 * n_blocks ? 4 : (n_self > 4 * n_blocks ? 3 : 2);
}
constexpr int kMaxParts = kPartsPerLink * kMaxDof;
constexpr int kMaxPartPairs = kMaxParts * (kMaxParts + 1) / 2;   // part pairs, same-part pairs included

// Robot tables of a flags check, copied into LDS by each workgroup from one
// block of memory with the same layout (RobotView::image): part bounding
// spheres, self-pair blocks, spheres, the spheres' links; then the self pairs,
// which a workgroup with many dependent checks (the bisection) copies too, up
// to kStagePairs of them.
constexpr int kStagePairs = 2048;

__host__ __device__ inline int robot_staged_pairs(int n_self) { return n_self <= kStagePairs ? n_self : 0; }

__host__ __device__ inline size_t robot_image_off_sph(int n_blocks) { return 16 * (size_t)(kMaxParts + n_blocks); }
__host__ __device__ inline size_t robot_image_off_link(int S, int n_blocks) {
    return robot_image_off_sph(n_blocks) + 16 * (size_t)S;
}
__host__ __device__ inline size_t robot_image_off_pairs(int S, int n_blocks) {
    return robot_image_off_link(S, n_blocks) + 16 * (((size_t)S + 3) / 4);
}
// Bytes of the copy (a multiple of 16), with or without the pairs.
__host__ __device__ inline size_t robot_stage_bytes(int S, int n_blocks, int n_self, bool pairs) {
    return robot_image_off_pairs(S, n_blocks) + (pairs ? 16 * (((size_t)robot_staged_pairs(n_self) + 1) / 2) : 0);
}

// Uniform grid over the obstacle cloud (shifted frame).  Cell k lists every
// obstacle that a robot sphere centred anywhere in cell k could touch: the
// distance from o to the cell's box is below r_o + r_sphere_max + slack (a
// sphere centre c in the box has |c - o| >= that distance).  A sphere centre
// outside the grid box is farther than r_sphere_max + r_o_max from every
// obstacle.  count[k] > cap marks an overflowing cell (scan all).
// state holds two bits per cell, what a sweep asks first: bit 0, the list is not
// empty; bit 1, some obstacle collides with every robot sphere centred anywhere
// in the cell (the farthest point of the cell's box is nearer to o than r_o +
// r_sphere_min - slack), so that no list is needed.
__host__ __device__ inline int state_words(int G) { return G * G * G / 16; }

struct GridGeom {
    float ox, oy, oz;          // origin (min corner)
    float hx, hy, hz;          // cell size
    float ihx, ihy, ihz;       // 1 / cell size
    float reach;               // r_sphere_max + slack
    float hit_reach;           // r_sphere_min - slack (hugely negative for a robot without spheres)
    float r_max;               // largest obstacle radius
    // distance field only: magnitude of the coordinates (for rounding), how far
    // from the robot's base a sphere centre may lie along an axis, the least
    // distance from there to a far obstacle, the largest radius of the others
    float extent, limit, far, r_near;
};

// Grid geometry through scalar loads (wave-uniform, written by earlier kernels).
__device__ __forceinline__ GridGeom load_geom(const GridGeom* p) {
    const __attribute__((address_space(4))) float* s = (const __attribute__((address_space(4))) float*)p;
    return GridGeom{s[0], s[1], s[2], s[3], s[4], s[5], s[6], s[7], s[8], s[9], s[10], s[11],
                    s[12], s[13], s[14], s[15]};
}

struct GridView {
    int G;                     // cells per axis
    int cap;                   // list capacity per cell
    const GridGeom* geom;
    const int* count;          // [G^3]
    const unsigned* state;     // [G^3 / 16] two bits per cell
    const unsigned short* list;  // [G^3][cap] obstacle indices
    unsigned long long* tests;   // optional [kTestSlots] counters of sphere-sphere tests performed
};

// Read-only global memory viewed through the constant address space: loads
// with a wave-uniform address then become scalar (s_load) loads.
typedef __attribute__((address_space(4))) const float cfloat;

__device__ __forceinline__ float4 cload4(const cfloat* p) { return make_float4(p[0], p[1], p[2], p[3]); }

struct ObsView {
    int n;
    int lds_n;                 // > 0: the workgroup stages the n records (x, y, z, r) in LDS
    const float4* rec;         // [n] (ox, oy, oz, ro), shifted frame
    const float4* centre;      // [1] shift applied to world coordinates (x' = x - centre)
    int n_ebox;                // obstacle boxes (world frame, packed like robot boxes)
    const float4* ebox;        // [n_ebox][4]
};

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon et al., SC'11)
// ---------------------------------------------------------------------------
struct U4 { uint32_t x, y, z, w; };

__device__ __forceinline__ U4 philox4x32_10(U4 c, uint32_t k0, uint32_t k1) {
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        // one 32 x 32 -> 64-bit multiply (v_mad_u64_u32) gives both halves
        const uint64_t p0 = (uint64_t)0xD2511F53u * c.x, p1 = (uint64_t)0xCD9E8D57u * c.z;
        const uint32_t lo0 = (uint32_t)p0, hi0 = (uint32_t)(p0 >> 32);
        const uint32_t lo1 = (uint32_t)p1, hi1 = (uint32_t)(p1 >> 32);
        U4 n;
        n.x = hi1 ^ c.y ^ k0;
        n.y = lo1;
        n.z = hi0 ^ c.w ^ k1;
        n.w = lo0;
        c = n;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return c;
}

// word -> (0, 1): ((x >> 9) + 1/2) * 2^-23, exact in FP32
__device__ __forceinline__ float u01(uint32_t x) {
    return ((float)(x >> 9) + 0.5f) * (1.0f / 8388608.0f);
}

__device__ __forceinline__ uint32_t word_of(const U4& v, int i) {
    return i == 0 ? v.x : (i == 1 ? v.y : (i == 2 ? v.z : v.w));
}

// ---------------------------------------------------------------------------
// Forward kinematics: compose T <- T * A_l with the standard DH matrix
//   A = [[ct, -st ca,  st sa, a ct],
//        [st,  ct ca, -ct sa, a st],
//        [0,   sa,     ca,    d   ]]
// R is row-major 3x3, p the translation.
// ---------------------------------------------------------------------------
// dh_compose_row: one row (r0, r1, r2 | p).
__device__ __forceinline__ void dh_compose_row(float& r0, float& r1, float& r2, float& p, float ct, float st,
                                               float4 dh) {
    const float a = dh.x, d = dh.y, ca = dh.z, sa = dh.w;
    const float u = fmaf(r0, ct, r1 * st);        // new column 0
    const float w = fmaf(r1, ct, -r0 * st);       // R * (-st, ct, 0)
    p = fmaf(a, u, fmaf(d, r2, p));
    r0 = u;
    r1 = fmaf(w, ca, r2 * sa);
    r2 = fmaf(r2, ca, -w * sa);
}

__device__ __forceinline__ void dh_compose(float R[9], float p[3], float ct, float st, float4 dh) {
#pragma unroll
    for (int r = 0; r < 3; ++r) dh_compose_row(R[3 * r], R[3 * r + 1], R[3 * r + 2], p[r], ct, st, dh);
}

// ---------------------------------------------------------------------------
// Tile shared-memory carve-up (dynamic LDS)
// ---------------------------------------------------------------------------
struct TileSmem {
    float* q;          // [T][kMaxDof] configurations of the tile
    float2* trig;      // [kMaxDof][T] (cos, sin) of each joint
    float4* cen;       // [S + 4B][T] sphere centres (shifted frame) and radius, then each
                       // box's world pose as four rows (packed like RobotView::box)
    float4* lb;        // [kMaxParts][T] part bounding spheres (shifted frame)
    int* hit;          // [T] collision flag (flags mode) / validity
    float* red;        // [2][W][T] partial minima (signed-distance mode)
};

__host__ __device__ inline size_t tile_smem_bytes(int T, int S, int W) {
    size_t b = 0;
    b += sizeof(float) * (size_t)T * kMaxDof;
    b += sizeof(float2) * (size_t)kMaxDof * T;
    b += sizeof(float4) * (size_t)(S > 0 ? S : 1) * T;
    b += sizeof(float4) * (size_t)kMaxParts * T;
    b += sizeof(int) * (size_t)T;
    b += sizeof(float) * 2 * (size_t)W * T;
    return (b + 15) & ~(size_t)15;
}

__device__ inline TileSmem carve_tile(char* base, int T, int S, int W) {
    TileSmem t;
    char* p = base;
    t.cen = reinterpret_cast<float4*>(p);   p += sizeof(float4) * (size_t)(S > 0 ? S : 1) * T;
    t.lb = reinterpret_cast<float4*>(p);    p += sizeof(float4) * (size_t)kMaxParts * T;
    t.trig = reinterpret_cast<float2*>(p);  p += sizeof(float2) * (size_t)kMaxDof * T;
    t.q = reinterpret_cast<float*>(p);      p += sizeof(float) * (size_t)T * kMaxDof;
    t.red = reinterpret_cast<float*>(p);    p += sizeof(float) * 2 * (size_t)W * T;
    t.hit = reinterpret_cast<int*>(p);
    return t;
}

// Work items (c, k), c < n, k < K, item index k n + c, spread over the
// workgroup's threads: one division per loop instead of one per item.
struct ItemWalk {
    int c, k, dc, dk;
    __device__ ItemWalk(int n) : ItemWalk(n, threadIdx.x) {}
    __device__ ItemWalk(int n, int tid) {
        const int nt = blockDim.x;
        if ((n & (n - 1)) == 0) {                  // a power of two: shifts
            const int sh = __builtin_ctz(n);
            k = tid >> sh;
            dk = nt >> sh;
        } else {
            k = tid / n;
            dk = nt / n;
        }
        c = tid - k * n;
        dc = nt - dk * n;
    }
    __device__ void next(int n) {
        c += dc;
        k += dk;
        if (c >= n) {
            c -= n;
            ++k;
        }
    }
};

struct Frame { float4 r0, r1, r2; };     // rows (R | p) of a link's frame

// A box's world pose, four rows at dst, dst + T, ...: centre and rotation
// through the link's frame f.
__device__ __forceinline__ void place_box(const Frame& f, float4 b0, float4 b1, float4 b2, float4 b3, float4* dst,
                                          int T) {
    const float R[9] = {f.r0.x, f.r0.y, f.r0.z, f.r1.x, f.r1.y, f.r1.z, f.r2.x, f.r2.y, f.r2.z};
    const float L[9] = {b1.x, b1.y, b1.z, b2.x, b2.y, b2.z, b3.x, b3.y, b3.z};
    float W[9];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j)
            W[3 * i + j] = fmaf(R[3 * i], L[j], fmaf(R[3 * i + 1], L[3 + j], R[3 * i + 2] * L[6 + j]));
    dst[0] = make_float4(fmaf(R[0], b0.x, fmaf(R[1], b0.y, fmaf(R[2], b0.z, f.r0.w))),
                         fmaf(R[3], b0.x, fmaf(R[4], b0.y, fmaf(R[5], b0.z, f.r1.w))),
                         fmaf(R[6], b0.x, fmaf(R[7], b0.y, fmaf(R[8], b0.z, f.r2.w))), b0.w);
    dst[T] = make_float4(W[0], W[1], W[2], b1.w);
    dst[2 * T] = make_float4(W[3], W[4], W[5], b2.w);
    dst[3 * T] = make_float4(W[6], W[7], W[8], b3.w);
}

// FK phase: t.q[c][j] (c < n_valid) -> t.cen[s][c].  Ends with a barrier.
// Only the n_valid >= 1 configurations of the tile are computed.
// BOX = false compiles the sphere-only path (no box code, fewer registers);
// BOX = true adds the boxes of RobotView and ObsView.
template <bool BOX>
__device__ inline void tile_fk(const RobotView& rb, const ObsView& ob, const TileSmem& t, int T, int n_valid) {
    const int dof = rb.dof;
    for (ItemWalk w(n_valid); w.k < dof; w.next(n_valid)) {
        const int c = w.c, j = w.k;
        float s = 0.f, co = 1.f;
        if (!((rb.prismatic >> j) & 1u)) {
            // v_sin_f32 / v_cos_f32 take revolutions: q / (2 pi), rounded once
            const float rev = t.q[c * kMaxDof + j] * 0.15915494309189535f;
            s = __builtin_amdgcn_sinf(rev);
            co = __builtin_amdgcn_cosf(rev);
        }
        t.trig[j * T + c] = make_float2(co, s);
    }
    __syncthreads();
    const float4 sh = ob.centre[0];
    // P lanes per (configuration, link), P the largest power of two (<= 16)
    // with n_valid dof P items in one pass of the workgroup: each composes the
    // link's frame and places every P-th sphere (and box) of the link, so a
    // long link is spread over idle lanes instead of being placed by one
    int lp = 0;
    while (lp < 4 && n_valid * dof * (2 << lp) <= (int)blockDim.x) ++lp;
    const int P = 1 << lp;
    for (ItemWalk w(n_valid); w.k < dof * P; w.next(n_valid)) {
        const int c = w.c, link = w.k >> lp, part = w.k & (P - 1);
        float R[9] = {1.f, 0.f, 0.f, 0.f, 1.f, 0.f, 0.f, 0.f, 1.f};
        float p[3] = {-sh.x, -sh.y, -sh.z};
        for (int l = 0; l <= link; ++l) {
            const float2 cs = t.trig[l * T + c];
            float4 dh = rb.dh[l];
            if ((rb.prismatic >> l) & 1u) dh.y += t.q[c * kMaxDof + l];
            dh_compose(R, p, cs.x, cs.y, dh);
        }
        if (part < kPartsPerLink) {       // the link's part bounds, spread over its P lanes
            for (int pp = part; pp < kPartsPerLink; pp += P) {
                const float4 lc = rb.lbound[kPartsPerLink * link + pp];
                float4 o;
                o.x = fmaf(R[0], lc.x, fmaf(R[1], lc.y, fmaf(R[2], lc.z, p[0])));
                o.y = fmaf(R[3], lc.x, fmaf(R[4], lc.y, fmaf(R[5], lc.z, p[1])));
                o.z = fmaf(R[6], lc.x, fmaf(R[7], lc.y, fmaf(R[8], lc.z, p[2])));
                o.w = lc.w;
                t.lb[(kPartsPerLink * link + pp) * T + c] = o;
            }
        }
        const int s1 = rb.link_begin[link + 1];
        for (int s = rb.link_begin[link] + part; s < s1; s += P) {
            const float4 ps = rb.sph[s];
            float4 o;
            o.x = fmaf(R[0], ps.x, fmaf(R[1], ps.y, fmaf(R[2], ps.z, p[0])));
            o.y = fmaf(R[3], ps.x, fmaf(R[4], ps.y, fmaf(R[5], ps.z, p[1])));
            o.z = fmaf(R[6], ps.x, fmaf(R[7], ps.y, fmaf(R[8], ps.z, p[2])));
            o.w = ps.w;
            t.cen[s * T + c] = o;
        }
        if (BOX && rb.n_boxes > 0) {
            const int S = rb.n_spheres;
            const int k1 = rb.box_begin[link + 1];
            for (int k = rb.box_begin[link] + part; k < k1; k += P) {
                const float4 b0 = rb.box[4 * k], b1 = rb.box[4 * k + 1], b2 = rb.box[4 * k + 2], b3 = rb.box[4 * k + 3];
                place_box(Frame{make_float4(R[0], R[1], R[2], p[0]), make_float4(R[3], R[4], R[5], p[1]),
                                make_float4(R[6], R[7], R[8], p[2])},
                          b0, b1, b2, b3, t.cen + (size_t)(S + 4 * k) * T + c, T);
            }
        }
    }
    __syncthreads();
}

// ---------------------------------------------------------------------------
// Box geometry (FP32).  A box: centre c, rotation R (row-major, columns = the
// box axes), half extents h, bounding radius |h|.
// ---------------------------------------------------------------------------
struct DBox {
    float c[3];
    float R[9];
    float h[3];
    float rb;
};

// Row i of a box's four packed float4 (c, h_x), (R row 0, h_y), (R row 1, h_z),
// (R row 2, bounding radius); the centre shifted by -sh.
__device__ __forceinline__ DBox unpack_box(float4 b0, float4 b1, float4 b2, float4 b3, float3 sh) {
    DBox x;
    x.c[0] = b0.x - sh.x;
    x.c[1] = b0.y - sh.y;
    x.c[2] = b0.z - sh.z;
    x.R[0] = b1.x; x.R[1] = b1.y; x.R[2] = b1.z;
    x.R[3] = b2.x; x.R[4] = b2.y; x.R[5] = b2.z;
    x.R[6] = b3.x; x.R[7] = b3.y; x.R[8] = b3.z;
    x.h[0] = b0.w;
    x.h[1] = b1.w;
    x.h[2] = b2.w;
    x.rb = b3.w;
    return x;
}

__device__ __forceinline__ DBox tile_box(const TileSmem& t, int S, int T, int k, int c) {
    const float4* p = t.cen + (size_t)(S + 4 * k) * T + c;
    return unpack_box(p[0], p[T], p[2 * T], p[3 * T], make_float3(0.f, 0.f, 0.f));
}

// Per-axis excess of a point over the box, e_k = |p_k| - h_k with p the
// point in box coordinates; returns max_k e_k and sum_k max(e_k, 0)^2.
__device__ __forceinline__ void box_excess(const DBox& B, float x, float y, float z, float* emax, float* out2) {
    const float dx = x - B.c[0], dy = y - B.c[1], dz = z - B.c[2];
    float m = -INFINITY, o = 0.f;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const float pk = fmaf(B.R[k], dx, fmaf(B.R[3 + k], dy, B.R[6 + k] * dz));
        const float e = fabsf(pk) - B.h[k];
        m = fmaxf(m, e);
        const float ep = fmaxf(e, 0.f);
        o = fmaf(ep, ep, o);
    }
    *emax = m;
    *out2 = o;
}

// Signed distance sphere (x, r) - box: outside sqrt(sum max(e,0)^2) - r, inside
// max_k e_k - r (minus the distance to the nearest face, minus r).
__device__ __forceinline__ float sd_sphere_box(const DBox& B, float x, float y, float z, float r) {
    float m, o;
    box_excess(B, x, y, z, &m, &o);
    return (m <= 0.f ? m : sqrtf(o)) - r;
}

// Collision test of the same pair: signed distance < 0.
__device__ __forceinline__ bool hit_sphere_box(const DBox& B, float x, float y, float z, float r) {
    float m, o;
    box_excess(B, x, y, z, &m, &o);
    return m <= 0.f ? (m < r) : (o < r * r);
}

// Separating-axis value of two boxes: with C_ij = A_i . B_j and t_i = A_i . t
// (t = c_B - c_A, A_i and B_j the box axes), the face axes give
// |t_i| - h_Ai - sum_j h_Bj |C_ij| and |sum_i C_ij t_i| - sum_i h_Ai |C_ij| - h_Bj.
// A cross axis n = A_i x B_j is taken in A's frame, where it is
// (n_i, n_i1, n_i2) = (0, -C_i2,j, C_i1,j) (i1 = i+1, i2 = i+2 mod 3): its
// length is sqrt(C_i1,j^2 + C_i2,j^2) (a sum of squares, so nearly parallel
// edges keep their length to full relative precision; skipped below 1e-6),
// and every term of the unnormalised value
//   |t . n| - sum_k h_Ak |n_k| - sum_k h_Bk |B_k . n|,
//   B_k . n = C_i1,j C_i2,k - C_i2,j C_i1,k   (a cofactor of C; 0 for k = j)
// is a product of n's components, so its rounding error scales with |n| and
// the normalised value is as accurate as that of a well separated axis.
// Returns the largest value (exact: all axes).  With early = true it returns
// as soon as an axis has a value >= 0 (the boxes do not collide) and the
// result is then only that value.
template <bool EARLY>
__device__ inline float sat_value(const DBox& A, const DBox& B) {
    const float tx = B.c[0] - A.c[0], ty = B.c[1] - A.c[1], tz = B.c[2] - A.c[2];
    float C[3][3], aC[3][3], t[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        t[i] = fmaf(A.R[i], tx, fmaf(A.R[3 + i], ty, A.R[6 + i] * tz));
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            C[i][j] = fmaf(A.R[i], B.R[j], fmaf(A.R[3 + i], B.R[3 + j], A.R[6 + i] * B.R[6 + j]));
            aC[i][j] = fabsf(C[i][j]);
        }
    }
    float best = -INFINITY;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const float v = fabsf(t[i]) - A.h[i] - fmaf(B.h[0], aC[i][0], fmaf(B.h[1], aC[i][1], B.h[2] * aC[i][2]));
        best = fmaxf(best, v);
        if (EARLY && v >= 0.f) return v;
    }
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        const float tb = fmaf(C[0][j], t[0], fmaf(C[1][j], t[1], C[2][j] * t[2]));
        const float v = fabsf(tb) - fmaf(A.h[0], aC[0][j], fmaf(A.h[1], aC[1][j], A.h[2] * aC[2][j])) - B.h[j];
        best = fmaxf(best, v);
        if (EARLY && v >= 0.f) return v;
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const int i1 = (i + 1) % 3, i2 = (i + 2) % 3;
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const int j1 = (j + 1) % 3, j2 = (j + 2) % 3;
            const float n2 = fmaf(C[i1][j], C[i1][j], C[i2][j] * C[i2][j]);
            if (n2 < 1e-12f) continue;
            const float bj1 = fmaf(C[i1][j], C[i2][j1], -C[i2][j] * C[i1][j1]);
            const float bj2 = fmaf(C[i1][j], C[i2][j2], -C[i2][j] * C[i1][j2]);
            const float u = fabsf(fmaf(t[i2], C[i1][j], -t[i1] * C[i2][j])) -
                            fmaf(A.h[i1], aC[i2][j], fmaf(A.h[i2], aC[i1][j],
                                 fmaf(B.h[j1], fabsf(bj1), B.h[j2] * fabsf(bj2))));
            const float v = u * rsqrtf(n2);
            best = fmaxf(best, v);
            if (EARLY && u >= 0.f) return v;
        }
    }
    return best;
}

__device__ __forceinline__ int wave_id() {
    return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
}

__device__ __forceinline__ bool wave_all(bool p) {
    return __ballot(p) == __ballot(true);
}

// Signed-distance pair sweep.  Results: t.red[0][0][c] = overall minimum,
// t.red[1][0][c] = self minimum; t.hit[c] = (overall < 0).  Barrier at exit.
// Distances by v_sqrt_f32 (one instruction, within about 1 ulp; the
// correctly rounded sqrtf takes several more per pair).
template <int T, bool BOX>
__device__ inline void tile_pairs_sd(const RobotView& rb, const ObsView& ob, const TileSmem& t, int n_valid) {
    const int tid = threadIdx.x;
    const int W = blockDim.x >> 6;
    const int w = wave_id();
    const int lane = tid & 63;
    const int c = lane % T;
    constexpr int nsub = 64 / T;
    const int j = lane / T;
    const int S = rb.n_spheres;
    float env = INFINITY, self = INFINITY;
    {
        const int P = rb.n_self;
        for (int p = w * nsub + j; p < P; p += W * nsub) {
            const int2 pr = rb.pairs[p];
            const float4 a = t.cen[pr.x * T + c];
            const float4 b = t.cen[pr.y * T + c];
            const float dx = a.x - b.x, dy = a.y - b.y, dz = a.z - b.z;
            const float d = __builtin_amdgcn_sqrtf(fmaf(dx, dx, fmaf(dy, dy, dz * dz)));
            self = fminf(self, d - a.w - b.w);
        }
    }
    const int o0 = (int)(((long)ob.n * w) / W);
    const int o1 = (int)(((long)ob.n * (w + 1)) / W);
    if (o1 > o0) {
        for (int s0 = 0; s0 < S; s0 += 2 * nsub) {
            const int sa = s0 + j, sb = s0 + nsub + j;
            const float4 A = sa < S ? t.cen[sa * T + c] : make_float4(kHuge, kHuge, kHuge, 0.f);
            const float4 B = sb < S ? t.cen[sb * T + c] : make_float4(kHuge, kHuge, kHuge, 0.f);
            float bestA = INFINITY, bestB = INFINITY;
            const cfloat* rec = (const cfloat*)ob.rec;
#pragma unroll 4
            for (int o = o0; o < o1; ++o) {
                const float4 P0 = cload4(rec + 4 * o);
                const float ax = A.x - P0.x, ay = A.y - P0.y, az = A.z - P0.z;
                const float bx = B.x - P0.x, by = B.y - P0.y, bz = B.z - P0.z;
                const float dA = __builtin_amdgcn_sqrtf(fmaf(ax, ax, fmaf(ay, ay, az * az)));
                const float dB = __builtin_amdgcn_sqrtf(fmaf(bx, bx, fmaf(by, by, bz * bz)));
                bestA = fminf(bestA, dA - P0.w);
                bestB = fminf(bestB, dB - P0.w);
            }
            if (sa < S) env = fminf(env, bestA - A.w);
            if (sb < S) env = fminf(env, bestB - B.w);
        }
    }
    if (BOX && (rb.n_boxes > 0 || ob.n_ebox > 0)) {
        const float4 shv = ob.centre[0];
        const float3 sh = make_float3(shv.x, shv.y, shv.z);
        const int B = rb.n_boxes;
        const bool ok = c < n_valid;
        for (int p = w * nsub + j; ok && p < rb.n_box_pairs; p += W * nsub) {
            const int2 pr = rb.box_pairs[p];
            self = fminf(self, sat_value<false>(tile_box(t, S, T, pr.x, c), tile_box(t, S, T, pr.y, c)));
        }
        for (int k = w * nsub + j; ok && k < B; k += W * nsub) {
            const DBox X = tile_box(t, S, T, k, c);
            for (int o = 0; o < ob.n; ++o) {
                const float4 O = ob.rec[o];
                env = fminf(env, sd_sphere_box(X, O.x, O.y, O.z, O.w));
            }
            for (int e = 0; e < ob.n_ebox; ++e)
                env = fminf(env, sat_value<false>(X, unpack_box(ob.ebox[4 * e], ob.ebox[4 * e + 1], ob.ebox[4 * e + 2],
                                                                ob.ebox[4 * e + 3], sh)));
        }
        for (int s2 = w * nsub + j; ok && ob.n_ebox > 0 && s2 < S; s2 += W * nsub) {
            const float4 C = t.cen[s2 * T + c];
            for (int e = 0; e < ob.n_ebox; ++e)
                env = fminf(env, sd_sphere_box(unpack_box(ob.ebox[4 * e], ob.ebox[4 * e + 1], ob.ebox[4 * e + 2],
                                                          ob.ebox[4 * e + 3], sh), C.x, C.y, C.z, C.w));
        }
    }
    // reduce over the lanes of one configuration, then over waves
    for (int off = T; off < 64; off <<= 1) {
        env = fminf(env, __shfl_xor(env, off));
        self = fminf(self, __shfl_xor(self, off));
    }
    if (j == 0) {
        t.red[(0 * W + w) * T + c] = fminf(env, self);
        t.red[(1 * W + w) * T + c] = self;
    }
    __syncthreads();
    if (tid < T) {
        float m = INFINITY, s = INFINITY;
        for (int k = 0; k < W; ++k) {
            m = fminf(m, t.red[(0 * W + k) * T + tid]);
            s = fminf(s, t.red[(1 * W + k) * T + tid]);
        }
        t.red[tid] = m;
        t.red[W * T + tid] = s;
        t.hit[tid] = (m < 0.f) ? 1 : 0;
    }
    __syncthreads();
}

// ---------------------------------------------------------------------------
// Flags mode: the tile of a collision check that only asks whether a
// configuration collides.  Per configuration the LDS holds the link frames
// (48 bytes a link), not the spheres: a sphere's centre is nine multiply-adds
// from its link's frame, placed by the lane that tests it, and a
// configuration takes 0.7 KB instead of the 1.9 KB that the 70 centres of a
// 7-DOF arm made it, so that more than twice as many waves fit a CU.
//
// One check:
//   1. eight lanes per configuration, lane j joint j: cosine and sine to LDS;
//      three of them compose the frames, one row each (row r of [R | p]
//      depends on row r of the previous link's only); all eight place the
//      link parts' bounding spheres                                    | barrier
//   2. obstacles: a lane per (configuration, sphere), two a step, places its
//      spheres and looks their grid cells up in the workgroup's copy of the
//      cell states (8 KB of LDS for 32^3 cells): nothing near, certain hit, or
//      a list.  Listed spheres go to the wave's own LDS list and are tested
//      from there with full lanes (one to eight a sphere).  Then self pairs: a lane per
//      (configuration, part pair) tests the parts' bounding spheres;
//      overlapping ones go to the wave's list, and up to 16 lanes each test
//      the sphere pairs of one.  (Boxes: placed, a barrier, their pairs) | barrier
// Configurations found colliding drop out of everything that follows.  Every
// pair not tested is provably separated (or its configuration already hit),
// so the flag equals that of the all-pairs test; the pair test is
// |c - o|^2 < (r_c + r_o)^2 on centres computed by the same FP32 operations
// wherever they are placed.
//
// Bound by VALU issue when there are many configurations (199 instructions of a
// wave per configuration of the 7-DOF arm among 1024 spheres, 90 % of what the chip
// issues, 68 % of their lanes active; the former tile, with the centres in LDS and
// every sphere in the grid looking its list up, issued 259, 87 % and 60 %), by
// latency when there are few.  Measured: 4 M
// configurations 2.24 -> 1.55 ms; the check of an inflation's 10 000 samples
// 10.2 -> 9.8 us, of 96 edges 33.3 -> 27.5 us a launch.
// ---------------------------------------------------------------------------
// Native vectors (HIP's vector classes cannot live in another address space).
typedef lds_f4_t f4;
typedef lds_i4_t i4;
typedef float f2 __attribute__((ext_vector_type(2)));
typedef int i2 __attribute__((ext_vector_type(2)));

// A configuration's record in the tile, in 16-byte rows: the parts' bounding
// spheres, (collision flag, 1 = the learned screen cleared its self pairs), each
// link's offset d (plus q for a prismatic joint), each joint's (cos, sin), and the
// links' frames (three rows (R | p) each, shifted frame).  The rows of a record are
// at fixed offsets (no address arithmetic or registers for them); a robot keeps its
// own links' frames only, and without self pairs of spheres no bounds (the record
// then starts kMaxParts rows in: more waves fit a CU: 2 M point-robot checks among
// 15 discs 64 us, 134 with all 47 rows).  The rows of a tile's records lie on distinct
// LDS banks when their number is odd, and neighbouring records' frames collide least
// when it is 1 or 7 modulo 8 (4 M configurations of seven joints: 47 rows 1573 us,
// 45 rows 1587).
constexpr int kRecLb = 0, kRecHit = kMaxParts, kRecD = kRecHit + 1, kRecTrig = kRecD + kMaxDof / 4,
              kRecFrame = kRecTrig + kMaxDof / 2, kRecRows = kRecFrame + 3 * kMaxDof;
__host__ __device__ constexpr int rec_rows(int dof, int n_blocks) {
    const int r = (kRecFrame + 3 * dof - (n_blocks > 0 ? 0 : kMaxParts)) | 1;
    return r % 8 == 3 || r % 8 == 5 ? r | 7 : r;
}
static_assert(rec_rows(kMaxDof, 1) == kRecRows, "the distance kernel's records are the largest robot's");

struct FlagTile {
    lds_ptr<f4> rec;        // [T][rows], kMaxParts rows before the first record that holds no bounds
    int stride;             // bytes of a record
    bool bounds;            // records hold the parts' bounding spheres
    int item_shift;
    lds_ptr<f4> box;        // [4 B][T] each box's world pose as four rows (packed like RobotView::box)
    int T;
    lds_ptr<unsigned> wl;   // [W][kWaveList] each wave's list
    lds_ptr<unsigned> state;   // [state_words] the grid's cell states (a robot without boxes)
    lds_ptr<f4> obs;        // [lds_n] staged obstacle records (x, y, z, r)
    // the robot's tables
    lds_ptr<f4> lbound, sph;
    lds_ptr<i4> blocks;
    lds_ptr<int> link;
    lds_ptr<i2> pairs;

    __device__ __forceinline__ lds_ptr<f4> row(int c) const {
        return (lds_ptr<f4>)((lds_ptr<char>)rec + __umul24(c, stride));
    }
    __device__ __forceinline__ lds_ptr<volatile int> hit(int c) const {
        return (lds_ptr<volatile int>)(row(c) + kRecHit);
    }
    __device__ __forceinline__ lds_ptr<int> scr(int c) const { return (lds_ptr<int>)(row(c) + kRecHit) + 1; }
};

// Entries of a wave's list: a step adds at most 128 (two spheres a lane) to at
// most 63 left by the step before.
constexpr int kWaveList = 192;

// A robot of boxes only keeps no lists.
__host__ __device__ inline bool boxes_only(int n_spheres, int n_boxes) { return n_spheres == 0 && n_boxes > 0; }

// The waves' lists lie first (a record without bounds is addressed from kMaxParts
// rows before it: at least that much lies there).
__host__ __device__ inline size_t flag_lists_bytes(bool lists, int W) {
    return lists ? sizeof(unsigned) * (size_t)kWaveList * W : sizeof(float4) * kMaxParts;
}
static_assert(sizeof(unsigned) * kWaveList >= sizeof(float4) * kMaxParts, "room before the first record");

__host__ __device__ inline size_t flag_tile_bytes(int T, bool lists, int rec_bytes, int n_boxes, int W) {
    return (size_t)T * (rec_bytes + sizeof(float4) * 4 * n_boxes) + flag_lists_bytes(lists, W);
}

// The cell states and the staged obstacles follow the tile region, then the
// robot's tables.  A robot with boxes reads the states from global memory: its box
// pairs take most of the time and more waves serve them (300 001 of a 7-DOF arm of
// 70 spheres and 11 boxes among 512 spheres: 1.64 ms with the states in LDS, 1.31
// without; 194 spheres 664 and 647 us).
__host__ __device__ inline size_t flag_grid_bytes(bool states, int n_obs, int G, int lds_n) {
    return (states && n_obs > 0 ? sizeof(unsigned) * (size_t)state_words(G) : 0) + sizeof(float4) * (size_t)lds_n;
}

// base: the workgroup's LDS (16-byte aligned); *end receives the first byte
// after the robot's tables.
template <bool BOX>
__device__ inline FlagTile carve_flag_tile(char* base, int T, int W, const RobotView& rb, bool pairs, const ObsView& ob,
                                           int lds_n, int G, char** end) {
    FlagTile t;
    const int n_boxes = BOX ? rb.n_boxes : 0;
    const bool lists = !BOX || !boxes_only(rb.n_spheres, n_boxes);
    const size_t tile = flag_tile_bytes(T, lists, rb.rec_bytes, n_boxes, W);
    lds_ptr<char> p = to_lds(base);
    t.T = T;
    t.stride = rb.rec_bytes;
    t.bounds = rb.n_blocks > 0;
    t.item_shift = rb.item_shift;
    t.wl = (lds_ptr<unsigned>)p;    p += (int)flag_lists_bytes(lists, W);
    t.rec = (lds_ptr<f4>)p - (t.bounds ? 0 : kMaxParts);
    p += t.stride * T;
    t.box = (lds_ptr<f4>)p;         p += (int)sizeof(f4) * 4 * n_boxes * T;
    p = to_lds(base) + (int)tile;
    t.state = (lds_ptr<unsigned>)p; p += (int)flag_grid_bytes(n_boxes == 0, ob.n, G, 0);
    t.obs = (lds_ptr<f4>)p;         p += sizeof(f4) * lds_n;
    t.lbound = (lds_ptr<f4>)p;
    t.blocks = (lds_ptr<i4>)(t.lbound + kMaxParts);
    t.sph = (lds_ptr<f4>)(p + (int)robot_image_off_sph(rb.n_blocks));
    t.link = (lds_ptr<int>)(p + (int)robot_image_off_link(rb.n_spheres, rb.n_blocks));
    t.pairs = (lds_ptr<i2>)(p + (int)robot_image_off_pairs(rb.n_spheres, rb.n_blocks));
    if (end)
        *end = base + tile + flag_grid_bytes(n_boxes == 0, ob.n, G, lds_n) +
               robot_stage_bytes(rb.n_spheres, rb.n_blocks, rb.n_self, pairs);
    return t;
}

// Copies n 16-byte words into LDS, four loads in flight a thread.
__device__ __forceinline__ void copy_to_lds(lds_ptr<f4> dst, const float4* src, int n) {
    const f4* s = reinterpret_cast<const f4*>(src);
    const int nt = blockDim.x;
    for (int i = threadIdx.x; i < n; i += 4 * nt) {
        f4 v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = s[min(i + k * nt, n - 1)];
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (i + k * nt < n) dst[i + k * nt] = v[k];
    }
}

// The workgroup's copies of the cell states, (OST) the obstacle records and
// the robot's tables; the caller places a barrier before their first use.
template <bool BOX, bool OST>
__device__ inline void stage_tables(const RobotView& rb, bool pairs, const ObsView& ob, const GridView& gv,
                                    const FlagTile& t) {
    if (ob.n > 0) {
        if (!BOX || rb.n_boxes == 0)
            copy_to_lds((lds_ptr<f4>)t.state, reinterpret_cast<const float4*>(gv.state), state_words(gv.G) / 4);
        if constexpr (OST) copy_to_lds(t.obs, ob.rec, ob.n);
    }
    copy_to_lds(t.lbound, rb.image, (int)(robot_stage_bytes(rb.n_spheres, rb.n_blocks, rb.n_self, pairs) / 16));
}

// LDS written by some lanes of a wave and read by others of the same wave: a
// wave's LDS accesses complete in order, so only the compiler is held.
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

struct LFrame { f4 r0, r1, r2; };

__device__ __forceinline__ LFrame tile_frame(const FlagTile& t, int c, int link) {
    const lds_ptr<f4> f = t.row(c) + kRecFrame + 3 * link;
    return LFrame{f[0], f[1], f[2]};
}

// Point (x, y, z) of the link's frame in the (shifted) world, w kept.
__device__ __forceinline__ f4 place(const LFrame& f, f4 v) {
    f4 o;
    o.x = fmaf(f.r0.x, v.x, fmaf(f.r0.y, v.y, fmaf(f.r0.z, v.z, f.r0.w)));
    o.y = fmaf(f.r1.x, v.x, fmaf(f.r1.y, v.y, fmaf(f.r1.z, v.z, f.r1.w)));
    o.z = fmaf(f.r2.x, v.x, fmaf(f.r2.y, v.y, fmaf(f.r2.z, v.z, f.r2.w)));
    o.w = v.w;
    return o;
}

// Configuration x's pose by its eight lanes (of one wave), lane j with joint j's
// value qj and link offset dj: the joint's cosine and sine, the link frames
// (three lanes, one row each), the link parts' bounding spheres.  Straight-line
// code: a taken branch costs a lone wave over 100 cycles, more than the
// instructions it skips (lanes past the last joint or part write slots that
// nothing reads).
__device__ __forceinline__ void tile_pose(const RobotView& rb, float4 sh, const FlagTile& t, int x, int j, float qj,
                                          float dj) {
    const lds_ptr<f4> rec = t.row(x);
    const bool prism = ((rb.prismatic >> j) & 1u) != 0;
    // v_sin_f32 / v_cos_f32 take revolutions: q / (2 pi), rounded once
    const float rev = qj * 0.15915494309189535f;
    const float sn = __builtin_amdgcn_sinf(rev), cn = __builtin_amdgcn_cosf(rev);
    f2 cs;
    cs.x = prism ? 1.f : cn;
    cs.y = prism ? 0.f : sn;
    ((lds_ptr<f2>)(rec + kRecTrig))[j] = cs;
    ((lds_ptr<float>)(rec + kRecD))[j] = prism ? dj + qj : dj;
    wave_lds_sync();
    if (j < 3) {
        f4 c[4], d[2];
#pragma unroll
        for (int l = 0; l < 4; ++l) c[l] = rec[kRecTrig + l];
        d[0] = rec[kRecD];
        d[1] = rec[kRecD + 1];
        float r0 = j == 0 ? 1.f : 0.f, r1 = j == 1 ? 1.f : 0.f, r2 = j == 2 ? 1.f : 0.f;
        float p = -(j == 0 ? sh.x : (j == 1 ? sh.y : sh.z));
        const lds_ptr<f4> out = rec + kRecFrame + j;
#pragma unroll
        for (int l = 0; l < kMaxDof; ++l) {
            if (l >= rb.dof) break;
            float4 dh = cload4((const cfloat*)rb.dh + 4 * l);
            dh.y = d[l / 4][l % 4];
            dh_compose_row(r0, r1, r2, p, c[l / 2][2 * (l % 2)], c[l / 2][2 * (l % 2) + 1], dh);
            f4 row;
            row.x = r0; row.y = r1; row.z = r2; row.w = p;
            out[3 * l] = row;
        }
    }
    if (!t.bounds) return;
    wave_lds_sync();
    static_assert(kMaxParts == 16 && kPartsPerLink == 2, "two parts a lane");
    const LFrame f0 = tile_frame(t, x, j / kPartsPerLink), f1 = tile_frame(t, x, j / kPartsPerLink + 4);
    rec[kRecLb + j] = place(f0, t.lbound[j]);
    rec[kRecLb + j + 8] = place(f1, t.lbound[j + 8]);
}

// The wave's list: entries appended by the lanes with a true predicate,
// taken off its end.  n is wave-uniform.
struct WaveList {
    lds_ptr<unsigned> e;
    int n;
    __device__ WaveList(const FlagTile& t) : e(t.wl + kWaveList * wave_id()), n(0) {}
    __device__ void push(bool p, unsigned v) {
        const unsigned long long b = __ballot(p);
        if (p) e[n + __popcll(b & ((1ull << (threadIdx.x & 63)) - 1ull))] = v;
        n += __popcll(b);
    }
};

// Grid cell of a sphere centre; in = false outside the grid (or not a number),
// where the cell returned is some cell of the grid.
__device__ __forceinline__ int grid_cell(const GridGeom& g, int G, f4 C, bool* in) {
    const float fx = (C.x - g.ox) * g.ihx, fy = (C.y - g.oy) * g.ihy, fz = (C.z - g.oz) * g.ihz;
    // IEEE 754-2019 minimum / maximum: a NaN coordinate stays NaN and is outside
    const float lo = __builtin_elementwise_minimum(__builtin_elementwise_minimum(fx, fy), fz);
    const float hi = __builtin_elementwise_maximum(__builtin_elementwise_maximum(fx, fy), fz);
    *in = lo >= 0.f && hi < (float)G;
    const int cx = (int)fx & (G - 1), cy = (int)fy & (G - 1), cz = (int)fz & (G - 1);    // G a power of two
    return (cz * G + cy) * G + cx;
}

// Tests the last m <= 64 listed spheres (configuration | sphere << 6) against
// the obstacles of their cells; with few entries several lanes share one, each
// taking every so many groups of four list entries (records from LDS when
// staged, else from global memory; the four records of a group are fetched
// together and tested branch-free).
template <class RecF>
__device__ __forceinline__ void drain_spheres(WaveList& wl, int m, RecF rec, const ObsView& ob, const GridView& gv,
                                              const GridGeom& g, const FlagTile& t, unsigned& ntest) {
    wave_lds_sync();
    const int lane = threadIdx.x & 63;
    const int sh = m > 32 ? 0 : (m > 16 ? 1 : (m > 8 ? 2 : 3));       // lanes per entry, as a shift
    const int i = lane >> sh, sub = lane & ((1 << sh) - 1);
    const unsigned e = wl.e[wl.n - m + min(i, m - 1)];
    const int c = e & 63, s = e >> 6;
    if (i < m && *t.hit(c) == 0) {
        const f4 C = place(tile_frame(t, c, t.link[s]), t.sph[s]);
        bool in;
        const int cell = grid_cell(g, gv.G, C, &in);
        // the cell's count and this lane's first four list entries together
        // (cell lists are 8-byte aligned, cap >= 32)
        const ushort4* lst4 = reinterpret_cast<const ushort4*>(gv.list + (size_t)cell * gv.cap);
        const int cnt = gv.count[cell];
        ushort4 v = lst4[sub];
        const bool full = cnt > gv.cap;
        const int n = full ? ob.n : cnt;
        bool found = false;
        for (int k0 = 4 * sub; k0 < n && !found; k0 += 4 << sh) {
            int oi[4];
            if (full) {
                oi[0] = k0; oi[1] = k0 + 1; oi[2] = k0 + 2; oi[3] = k0 + 3;
            } else {
                if (k0 != 4 * sub) v = lst4[k0 >> 2];
                oi[0] = v.x; oi[1] = v.y; oi[2] = v.z; oi[3] = v.w;
            }
            ntest += (unsigned)min(4, n - k0);
            float4 O[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) O[k] = rec((k0 + k < n) ? oi[k] : oi[0]);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const bool ok = k0 + k < n;
                const float ex = C.x - O[k].x, ey = C.y - O[k].y, ez = C.z - O[k].z;
                const float Rr = C.w + O[k].w;
                found |= ok && fmaf(ex, ex, fmaf(ey, ey, ez * ez)) < Rr * Rr;
            }
        }
        if (found) *t.hit(c) = 1;
    }
    wl.n -= m;
    wave_lds_sync();
}

// The spheres against the obstacles: a lane per (configuration, sphere), two a
// step.
template <class StateF, class RecF>
__device__ __forceinline__ void tile_obstacles(StateF state, RecF rec, const RobotView& rb, const ObsView& ob, const GridView& gv,
                                               const FlagTile& t, int n_valid, unsigned& ntest) {
    const int S = rb.n_spheres;
    const GridGeom g = load_geom(gv.geom);
    const int G = gv.G;
    WaveList wl(t);
    ItemWalk w(n_valid);
    // one step adds to the list or takes from it (each once in the code: the
    // kernels of an inflation's iteration share 64 KB of instruction cache)
    while (true) {
        if (wl.n < 64 && __any(w.k < S)) {
            const bool a0 = w.k < S;
            const int c0 = w.c, s0 = a0 ? w.k : 0;
            w.next(n_valid);
            const bool a1 = w.k < S;
            const int c1 = w.c, s1 = a1 ? w.k : 0;
            w.next(n_valid);
            const LFrame f0 = tile_frame(t, c0, t.link[s0]), f1 = tile_frame(t, c1, t.link[s1]);
            const f4 C0 = place(f0, t.sph[s0]), C1 = place(f1, t.sph[s1]);
            bool i0, i1;
            const int k0 = grid_cell(g, G, C0, &i0), k1 = grid_cell(g, G, C1, &i1);
            const unsigned n0 = a0 && i0 ? state(k0 >> 4) >> (2 * (k0 & 15)) : 0u;
            const unsigned n1 = a1 && i1 ? state(k1 >> 4) >> (2 * (k1 & 15)) : 0u;
            if (n0 & 2u) *t.hit(c0) = 1;
            if (n1 & 2u) *t.hit(c1) = 1;
            wl.push((n0 & 3u) == 1u && *t.hit(c0) == 0, (unsigned)c0 | (unsigned)s0 << 6);
            wl.push((n1 & 3u) == 1u && *t.hit(c1) == 0, (unsigned)c1 | (unsigned)s1 << 6);
        } else if (wl.n > 0) {
            drain_spheres(wl, min(wl.n, 64), rec, ob, gv, g, t, ntest);
        } else {
            break;
        }
    }
}

// Tests the sphere pairs of the last m listed (configuration, part pair)
// items: 2^item_shift lanes each, 32 or 64 when there are at most two.
template <class PairF>
__device__ __forceinline__ void drain_parts(WaveList& wl, int m, PairF pair, const FlagTile& t,
                                            unsigned& ntest) {
    wave_lds_sync();
    const int lane = threadIdx.x & 63;
    const int sh = m > 2 ? t.item_shift : (m > 1 ? 5 : 6), L = 1 << sh;       // lanes an item
    const int sub = lane >> sh, li = lane & (L - 1);
    for (int it0 = 0; it0 < m; it0 += 64 >> sh) {
        const int it = it0 + sub;
        const unsigned e = wl.e[wl.n - m + min(it, m - 1)];
        const int c = e & 63;
        if (it < m && *t.hit(c) == 0) {                   // uniform in the lane group
            const i4 blk = t.blocks[e >> 6];
            const LFrame fa = tile_frame(t, c, blk.x / kPartsPerLink), fb = tile_frame(t, c, blk.y / kPartsPerLink);
            bool found = false;
            for (int p = li; p < blk.w; p += L) {
                const int2 pr = pair(blk.z + p);
                const f4 a = place(fa, t.sph[pr.x]), b = place(fb, t.sph[pr.y]);
                const float ex = a.x - b.x, ey = a.y - b.y, ez = a.z - b.z;
                const float Rr = a.w + b.w;
                ++ntest;
                found |= fmaf(ex, ex, fmaf(ey, ey, ez * ez)) < Rr * Rr;
            }
            if (found) *t.hit(c) = 1;
        }
    }
    wl.n -= m;
    wave_lds_sync();
}

// The self pairs: a lane per (configuration, part pair).
template <class PairF>
__device__ __forceinline__ void tile_self_pairs(PairF pair, const RobotView& rb, const FlagTile& t, int n_valid,
                                                unsigned& ntest) {
    WaveList wl(t);
    // part pairs of many sphere pairs that would fill half the waves or fewer are dealt
    // out over all of them (an arm of 200 spheres and 4000 pairs, 1000 configurations
    // among 40 obstacles: 25.0 us a call in order, 19.5 dealt out; with the 25 sphere
    // pairs a part pair of the 7-DOF arm it costs 2 %)
    const bool deal = 2 * n_valid * rb.deal_blocks <= (int)blockDim.x;
    ItemWalk w(n_valid, deal ? (int)(threadIdx.x & 63) * (int)(blockDim.x >> 6) + wave_id() : (int)threadIdx.x);
    while (true) {
        if (wl.n < 64 && __any(w.k < rb.n_blocks)) {
            const bool on = w.k < rb.n_blocks;
            const int c = w.c, bk = on ? w.k : 0;
            w.next(n_valid);
            const i4 blk = t.blocks[bk];
            const lds_ptr<f4> part = t.row(c) + kRecLb;
            const f4 A = part[blk.x], B = part[blk.y];
            const float dx = A.x - B.x, dy = A.y - B.y, dz = A.z - B.z;
            const float R = A.w + B.w;
            const bool test = on && (*t.hit(c) | *t.scr(c)) == 0;
            ntest += test ? 1u : 0u;
            wl.push(test && fmaf(dx, dx, fmaf(dy, dy, dz * dz)) < R * R, (unsigned)c | (unsigned)bk << 6);
        } else if (wl.n > 0) {
            drain_parts(wl, min(wl.n, 64), pair, t, ntest);
        } else {
            break;
        }
    }
}

// The boxes' world poses: a lane per (configuration, box).  Row i of a box of
// neighbouring configurations, which neighbouring lanes read, is contiguous (a
// configuration's boxes side by side: 300 001 checks of 11 boxes among 194 spheres
// 948 us, four lanes to a bank).
__device__ inline void tile_place_boxes(const RobotView& rb, const FlagTile& t, int n_valid) {
    for (ItemWalk w(n_valid); w.k < rb.n_boxes; w.next(n_valid)) {
        const int c = w.c, k = w.k;
        const LFrame f = tile_frame(t, c, rb.box_link[k]);
        const float4 b0 = rb.box[4 * k], b1 = rb.box[4 * k + 1], b2 = rb.box[4 * k + 2], b3 = rb.box[4 * k + 3];
        float4 o[4];
        place_box(Frame{make_float4(f.r0.x, f.r0.y, f.r0.z, f.r0.w), make_float4(f.r1.x, f.r1.y, f.r1.z, f.r1.w),
                        make_float4(f.r2.x, f.r2.y, f.r2.z, f.r2.w)},
                  b0, b1, b2, b3, o, 1);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            f4 r;
            r.x = o[i].x; r.y = o[i].y; r.z = o[i].z; r.w = o[i].w;
            t.box[(4 * k + i) * t.T + c] = r;
        }
    }
}

__device__ __forceinline__ DBox flag_box(const FlagTile& t, int k, int c) {
    float4 b[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) b[i] = lds_load((lds_ptr<const float4>)t.box, (4 * k + i) * t.T + c);
    return unpack_box(b[0], b[1], b[2], b[3], make_float3(0.f, 0.f, 0.f));
}

// Box pairs of a tile, flags mode (after the sphere passes; configurations
// already hit are skipped): the box self pairs, every robot box against every
// obstacle sphere and obstacle box, every robot sphere against every obstacle
// box.  Each pair is first bounded by the two bounding spheres (a pair they
// prove apart cannot collide), then tested exactly.
template <bool OST>
__device__ inline void tile_boxes_flags(const RobotView& rb, const ObsView& ob, const FlagTile& t,
                                        int n_valid) {
    const int S = rb.n_spheres, B = rb.n_boxes;
    const float4 shv = ob.centre[0];
    const float3 sh = make_float3(shv.x, shv.y, shv.z);
    for (ItemWalk w(n_valid); w.k < rb.n_box_pairs; w.next(n_valid)) {
        const int c = w.c;
        if (*t.hit(c)) continue;
        const int2 pr = rb.box_pairs[w.k];
        const DBox X = flag_box(t, pr.x, c), Y = flag_box(t, pr.y, c);
        const float dx = X.c[0] - Y.c[0], dy = X.c[1] - Y.c[1], dz = X.c[2] - Y.c[2];
        const float Rr = X.rb + Y.rb;
        if (fmaf(dx, dx, fmaf(dy, dy, dz * dz)) >= Rr * Rr) continue;
        if (sat_value<true>(X, Y) < 0.f) *t.hit(c) = 1;
    }
    for (ItemWalk w(n_valid); w.k < B; w.next(n_valid)) {
        const int c = w.c;
        if (*t.hit(c)) continue;
        const DBox X = flag_box(t, w.k, c);
        bool found = false;
        for (int o = 0; o < ob.n && !found; ++o) {
            const float4 O = OST ? lds_load((lds_ptr<const float4>)t.obs, o) : ob.rec[o];
            const float dx = O.x - X.c[0], dy = O.y - X.c[1], dz = O.z - X.c[2];
            const float Rr = X.rb + O.w;
            if (fmaf(dx, dx, fmaf(dy, dy, dz * dz)) < Rr * Rr && hit_sphere_box(X, O.x, O.y, O.z, O.w)) found = true;
        }
        for (int e = 0; e < ob.n_ebox && !found; ++e) {
            const DBox E = unpack_box(ob.ebox[4 * e], ob.ebox[4 * e + 1], ob.ebox[4 * e + 2], ob.ebox[4 * e + 3], sh);
            const float dx = E.c[0] - X.c[0], dy = E.c[1] - X.c[1], dz = E.c[2] - X.c[2];
            const float Rr = X.rb + E.rb;
            if (fmaf(dx, dx, fmaf(dy, dy, dz * dz)) < Rr * Rr && sat_value<true>(X, E) < 0.f) found = true;
        }
        if (found) *t.hit(c) = 1;
    }
    if (ob.n_ebox > 0) {
        for (ItemWalk w(n_valid); w.k < S; w.next(n_valid)) {
            const int c = w.c;
            if (*t.hit(c)) continue;
            const f4 C = place(tile_frame(t, c, t.link[w.k]), t.sph[w.k]);
            bool found = false;
            for (int e = 0; e < ob.n_ebox && !found; ++e) {
                const DBox E = unpack_box(ob.ebox[4 * e], ob.ebox[4 * e + 1], ob.ebox[4 * e + 2], ob.ebox[4 * e + 3], sh);
                const float dx = E.c[0] - C.x, dy = E.c[1] - C.y, dz = E.c[2] - C.z;
                const float Rr = E.rb + C.w;
                if (fmaf(dx, dx, fmaf(dy, dy, dz * dz)) < Rr * Rr && hit_sphere_box(E, C.x, C.y, C.z, C.w)) found = true;
            }
            if (found) *t.hit(c) = 1;
        }
    }
}

// Adds the wave's test counts to one of kTestSlots counters (spread by
// workgroup, so that the atomics of many small workgroups do not queue on
// one address).  Every lane of the wave must call it.
constexpr int kTestSlots = 256;

__device__ inline void flush_tests(unsigned long long* tests, unsigned n) {
    unsigned long long v = n;
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    if ((threadIdx.x & 63) == 0) atomicAdd(tests + (blockIdx.x + 97u * blockIdx.y) % kTestSlots, v);
}

// Step 2 on the frames and part bounds of t (written, and t.hit and t.scr set,
// by the caller): fills t.hit.  Starts and ends with a barrier.  Returns the
// thread's count of pair tests.  PST: the self pairs lie in LDS when they are
// few enough; OST: the obstacle records do.
template <bool BOX, bool PST, bool OST>
__device__ inline unsigned tile_flags(const RobotView& rb, const ObsView& ob, const GridView& gv, const FlagTile& t,
                                      int n_valid) {
    unsigned ntest = 0;
    __syncthreads();
    if (ob.n > 0 && rb.n_spheres > 0) {
        const lds_ptr<const unsigned> sl = t.state;
        const unsigned* sg = gv.state;
        const bool lds_state = !BOX || rb.n_boxes == 0;
        const auto state = [=](int i) { return lds_state ? sl[i] : sg[i]; };
        if constexpr (OST) {
            const lds_ptr<const float4> rl = (lds_ptr<const float4>)t.obs;
            tile_obstacles(state, [=](int o) { return lds_load(rl, o); }, rb, ob, gv, t, n_valid, ntest);
        } else {
            const float4* rg = ob.rec;
            tile_obstacles(state, [=](int o) { return rg[o]; }, rb, ob, gv, t, n_valid, ntest);
        }
    }
    if (rb.n_blocks > 0) {
        const lds_ptr<const int2> pl = (lds_ptr<const int2>)t.pairs;
        const int2* pg = rb.pairs;
        const bool in_lds = PST && rb.n_self <= kStagePairs;
        tile_self_pairs([=](int i) { return in_lds ? lds_load(pl, i) : pg[i]; }, rb, t, n_valid, ntest);
    }
    if (BOX && (rb.n_boxes > 0 || ob.n_ebox > 0)) {
        tile_place_boxes(rb, t, n_valid);
        __syncthreads();
        tile_boxes_flags<OST>(rb, ob, t, n_valid);
    }
    __syncthreads();
    return ntest;
}

// Whole tile check in signed-distance mode on t.q[0..n_valid): fills t.hit,
// t.red[c] (overall) and t.red[W*T + c] (self).
template <int T, bool BOX>
__device__ inline void tile_check_sd(const RobotView& rb, const ObsView& ob, const TileSmem& t, int n_valid) {
    tile_fk<BOX>(rb, ob, t, T, n_valid);
    tile_pairs_sd<T, BOX>(rb, ob, t, n_valid);
}

}  // namespace ezo
