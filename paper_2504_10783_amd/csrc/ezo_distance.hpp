// ezo_distance.hpp -- signed distances of large batches: the minimum over all
// pairs of a configuration without testing all pairs.
//
// The minimum of the pairs' FP32 values is the same number whichever pairs are
// left out, as long as each of them is known to be no smaller than one that is
// kept.  So every configuration first takes the exact value of one likely
// nearest pair per sphere (the obstacle nearest to the centre of the sphere's
// grid cell), which bounds its minimum from above within a few millimetres, and
// then tests exactly only the spheres whose lower bound (the distance field at
// the cell's centre, which moves by at most the distance to that centre) is
// below, each against the obstacles that can be nearest from anywhere in its
// cell.  Self pairs: link parts by their bounding spheres in the same way.
//
// k_check_sd (all pairs) stays for batches too small to pay
// for the field and for boxes: the same scheme with box bounding spheres and
// face normals as bounds took 735 us where all pairs take 654 (300 001
// configurations of the 11-box arm among 194 spheres; a long box's bounds are
// too wide).
#pragma once
#include "ezo_device.hpp"

namespace ezo {

constexpr int kNearG = 32;               // cells per axis of the distance field
constexpr int kNearCells = kNearG * kNearG * kNearG;
constexpr int kNearCap = 128;            // obstacles listed per cell
constexpr int kNearBlock = 4;            // cells per axis of a build workgroup
constexpr int kNearBlockList = 2048;     // obstacles a build workgroup holds for its block
constexpr unsigned kNearFull = 0xFFFFu;  // list length of a cell that did not fit: scan all
constexpr float kNearGrow = 0.35f;       // the field reaches this share of the cloud's largest extent beyond it
constexpr int kAllSpheres = 8;           // spheres that an obstacle record is read for at once where no list serves

// Field entry: distance of the cell's centre to the nearest obstacle surface
// (-inf: unknown), nearest obstacle | list length << 16.
struct NearView {
    const GridGeom* geom;
    const uint2* near;                   // [kNearCells]
    const unsigned short* list;          // [kNearCells][kNearCap]
};

// FP32 values as signed integers in the same order.
__device__ __forceinline__ int fkey(float f) {
    const int b = __float_as_int(f);
    return b ^ ((b >> 31) & 0x7fffffff);
}
__device__ __forceinline__ float fval(int k) { return __int_as_float(k ^ ((k >> 31) & 0x7fffffff)); }

// Minimum over the 16 lanes of a row (quad permutations, half-row and row
// mirror), over the wave.  NaN operands are ignored.
__device__ __forceinline__ float row_min(float v) {
    v = fminf(v, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0xB1, 0xF, 0xF, true)));
    v = fminf(v, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x4E, 0xF, 0xF, true)));
    v = fminf(v, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x141, 0xF, 0xF, true)));
    return fminf(v, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x140, 0xF, 0xF, true)));
}
__device__ __forceinline__ float wave_min(float v) {
    const int r = __float_as_int(row_min(v));
    return fminf(fminf(__int_as_float(__builtin_amdgcn_readlane(r, 0)), __int_as_float(__builtin_amdgcn_readlane(r, 16))),
                 fminf(__int_as_float(__builtin_amdgcn_readlane(r, 32)), __int_as_float(__builtin_amdgcn_readlane(r, 48))));
}

// Distances from o to the nearest and the farthest point of the box [l, u].
__device__ __forceinline__ float box_near(float4 o, const float (&l)[3], const float (&u)[3]) {
    const float x = fmaxf(fmaxf(l[0] - o.x, o.x - u[0]), 0.f), y = fmaxf(fmaxf(l[1] - o.y, o.y - u[1]), 0.f),
                z = fmaxf(fmaxf(l[2] - o.z, o.z - u[2]), 0.f);
    return __builtin_amdgcn_sqrtf(fmaf(x, x, fmaf(y, y, z * z)));
}
__device__ __forceinline__ float box_far(float4 o, const float (&l)[3], const float (&u)[3]) {
    const float x = fmaxf(o.x - l[0], u[0] - o.x), y = fmaxf(o.y - l[1], u[1] - o.y), z = fmaxf(o.z - l[2], u[2] - o.z);
    return __builtin_amdgcn_sqrtf(fmaf(x, x, fmaf(y, y, z * z)));
}

// Rounding slack of the field's bounds: coordinates of magnitude up to ext.
__device__ __forceinline__ float near_slack(float ext) { return 1e-5f + 4e-6f * ext; }

// The field, one workgroup per block of kNearBlock^3 cells: the obstacles that
// can be nearest from anywhere in the block are copied to LDS (those no farther
// from the block's box than the least farthest distance of any), and each cell
// then looks at those only, a wave per cell.  Bound by load latency: 4096
// obstacles take 73 us with the records in LDS and eight waves, 199 us
// with four waves reading them from L2.  A block with more obstacles than it holds
// takes the nearest of all for each cell and keeps no lists (4096 heaped up: 80 us,
// 290 with lists over all of them, which hardly ever fit).
__global__ void __launch_bounds__(512) k_near_build(const float4* __restrict__ rec, int n,
                                                    const GridGeom* __restrict__ geom, uint2* __restrict__ near,
                                                    unsigned short* __restrict__ list) {
    __shared__ float4 crec[kNearBlockList];
    __shared__ unsigned short cand[kNearBlockList];
    __shared__ int s_n;
    __shared__ float s_min[8];
    constexpr int NB = kNearG / kNearBlock;
    const GridGeom g = load_geom(geom);
    const int tid = threadIdx.x, lane = tid & 63, w = wave_id();
    const int bx = blockIdx.x % NB, by = (blockIdx.x / NB) % NB, bz = blockIdx.x / (NB * NB);
    const float sl = near_slack(g.extent);
    const float org[3] = {g.ox, g.oy, g.oz}, h[3] = {g.hx, g.hy, g.hz};
    // a cell's (a block's) box, widened by the rounding of the cell assignment
    auto box = [&](int x, int y, int z, int cells, float (&l)[3], float (&u)[3]) {
        const int i[3] = {x, y, z};
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            l[a] = org[a] + (float)i[a] * h[a] - sl - 1e-5f * h[a];
            u[a] = org[a] + (float)(i[a] + cells) * h[a] + sl + 1e-5f * h[a];
        }
    };
    float l[3], u[3];
    box(bx * kNearBlock, by * kNearBlock, bz * kNearBlock, kNearBlock, l, u);
    float best = INFINITY;
    // four records in flight a thread (a repeated last one changes nothing)
    for (int o = tid; o < n; o += 4 * 512) {
        float4 O[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) O[k] = rec[min(o + 512 * k, n - 1)];
#pragma unroll
        for (int k = 0; k < 4; ++k) best = fminf(best, box_far(O[k], l, u) - O[k].w);
    }
    best = wave_min(best);
    if (lane == 0) s_min[w] = best;
    if (tid == 0) s_n = 0;
    __syncthreads();
    float bound = s_min[0];
#pragma unroll
    for (int k = 1; k < 8; ++k) bound = fminf(bound, s_min[k]);
    for (int o = tid; o < n; o += 4 * 512) {
        float4 O[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) O[k] = rec[min(o + 512 * k, n - 1)];
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (o + 512 * k < n && box_near(O[k], l, u) - O[k].w <= bound + sl) {
                const int i = atomicAdd(&s_n, 1);
                if (i < kNearBlockList) {
                    cand[i] = (unsigned short)(o + 512 * k);
                    crec[i] = O[k];
                }
            }
    }
    __syncthreads();
    // too many: the cells look for the nearest of all obstacles and keep no lists
    // (which would not fit)
    const bool all = s_n > kNearBlockList;
    const int m = all ? n : s_n;
    for (int c = w; c < kNearBlock * kNearBlock * kNearBlock; c += 8) {
        const int x = bx * kNearBlock + c % kNearBlock, y = by * kNearBlock + (c / kNearBlock) % kNearBlock,
                  z = bz * kNearBlock + c / (kNearBlock * kNearBlock);
        const int cell = (z * kNearG + y) * kNearG + x;
        box(x, y, z, 1, l, u);
        const float mx = g.ox + ((float)x + 0.5f) * g.hx, my = g.oy + ((float)y + 0.5f) * g.hy,
                    mz = g.oz + ((float)z + 0.5f) * g.hz;
        float d = INFINITY, far = INFINITY;
        int at = 0;
        auto nearest = [&](float4 O, int k) {
            const float ex = O.x - mx, ey = O.y - my, ez = O.z - mz;
            const float v = __builtin_amdgcn_sqrtf(fmaf(ex, ex, fmaf(ey, ey, ez * ez))) - O.w;
            at = v < d ? k : at;
            d = v < d ? v : d;
        };
        if (all) {
#pragma unroll 4
            for (int k = lane; k < n; k += 64) nearest(rec[k], k);
        } else {
#pragma unroll 2
            for (int k = lane; k < m; k += 64) {
                nearest(crec[k], k);
                far = fminf(far, box_far(crec[k], l, u) - crec[k].w);
            }
        }
        const float dm = wave_min(d);
        far = wave_min(far);
        const unsigned long long who = __ballot(d == dm);
        int near_o = 0;
        if (m > 0 && who) {
            const int k = __builtin_amdgcn_readlane(at, __builtin_ctzll(who));
            near_o = all ? k : cand[k];
        }
        int cnt = 0;
#pragma unroll 2
        for (int k0 = 0; !all && k0 < m && cnt <= kNearCap; k0 += 64) {
            const int k = k0 + lane, kk = min(k, m - 1);
            const float4 O = crec[kk];
            const bool keep = k < m && box_near(O, l, u) - O.w <= far + sl;
            const unsigned long long b = __ballot(keep);
            const int pos = cnt + __popcll(b & ((1ull << lane) - 1ull));
            if (keep && pos < kNearCap) list[(size_t)cell * kNearCap + pos] = cand[kk];
            cnt += __popcll(b);
        }
        if (lane == 0) {
            // a distance past FP32 says nothing: scan all
            const bool known = dm < 3e38f && !all && cnt <= kNearCap;
            const unsigned len = known ? (unsigned)cnt : kNearFull;
            near[cell] = make_uint2(__float_as_uint(dm < 3e38f ? dm : -INFINITY), (unsigned)near_o | len << 16);
        }
    }
}

// A wave's share of LDS: CW configurations' records, the running
// minima (as fkey: overall without self pairs, self pairs, the first self item
// to test) and the list of items still to test (item, lower bound, cell, length
// of the cell's list).
constexpr int kSdList = 128;
__host__ __device__ inline size_t sd_wave_bytes(int CW) {
    return sizeof(float4) * ((size_t)CW * kRecRows + kSdList) + 4 * sizeof(int) * 8;
}

struct SdWave {
    lds_ptr<int> env, self, pick;        // [CW]
    lds_ptr<i4> e;                       // [kSdList] items
    int n;                               // wave-uniform
    __device__ void push(bool p, int item, float lb, int cell = 0, int len = 0) {
        const unsigned long long b = __ballot(p);
        if (p) {
            i4 v;
            v.x = item;
            v.y = __float_as_int(lb);
            v.z = cell;
            v.w = len;
            e[n + __popcll(b & ((1ull << (threadIdx.x & 63)) - 1ull))] = v;
        }
        n += __popcll(b);
    }
};

__device__ __forceinline__ void lds_min(lds_ptr<int> p, float v) {
    __hip_atomic_fetch_min(p, fkey(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ float lds_val(lds_ptr<int> p) { return fval(*(lds_ptr<volatile int>)p); }

// Items (c, k), c < n, k < K, over the lanes of a wave.
struct WaveWalk {
    int c, k, dc, dk;
    __device__ WaveWalk(int n) {
        const int lane = threadIdx.x & 63;
        k = lane / n;
        dk = 64 / n;
        c = lane - k * n;
        dc = 64 - dk * n;
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

// Where a point lies in the field: its cell, the nearest obstacle of the
// cell's centre, and a lower bound of the point's distance to every obstacle's
// surface.  Outside the field's box the point's projection onto the box is
// looked up: along the axes where it differs the centres of the obstacles about the
// robot lie within the box, so |c - o|^2 >= |c - pc|^2 + |pc - o|^2 for them; the
// far ones are no nearer than g.far.  A point past the robot's reach (a prismatic
// joint beyond its limits) keeps every pair.  base: the frame's origin, -base
// the robot's.
struct NearAt {
    int cell, o, len;
    float lb;
};
__device__ __forceinline__ NearAt near_at(const GridGeom& g, const NearView& nv, float4 base, float x, float y, float z) {
    const float top = (float)kNearG - 0.5f;
    const float fx = fminf(fmaxf((x - g.ox) * g.ihx, 0.f), top + 0.49f), fy = fminf(fmaxf((y - g.oy) * g.ihy, 0.f), top + 0.49f),
                fz = fminf(fmaxf((z - g.oz) * g.ihz, 0.f), top + 0.49f);
    const int ix = (int)fx, iy = (int)fy, iz = (int)fz;
    NearAt r;
    r.cell = (iz * kNearG + iy) * kNearG + ix;
    const uint2 e = nv.near[r.cell];
    r.o = e.y & 0xFFFFu;
    r.len = e.y >> 16;
    const float px = fminf(fmaxf(x, g.ox), g.ox + kNearG * g.hx), py = fminf(fmaxf(y, g.oy), g.oy + kNearG * g.hy),
                pz = fminf(fmaxf(z, g.oz), g.oz + kNearG * g.hz);
    const float ex = x - px, ey = y - py, ez = z - pz;
    const float e2 = fmaf(ex, ex, fmaf(ey, ey, ez * ez));
    const float mx = px - (g.ox + ((float)ix + 0.5f) * g.hx), my = py - (g.oy + ((float)iy + 0.5f) * g.hy),
                mz = pz - (g.oz + ((float)iz + 0.5f) * g.hz);
    const float d = __uint_as_float(e.x) - __builtin_amdgcn_sqrtf(fmaf(mx, mx, fmaf(my, my, mz * mz)));
    const bool inside = e2 == 0.f;
    if (!inside) r.len = (int)kNearFull;               // (a NaN coordinate too)
    const float t = fmaxf(d + g.r_near, 0.f);
    const float lb = inside ? d : fminf(__builtin_amdgcn_sqrtf(fmaf(t, t, e2)) - g.r_near, g.far);
    r.lb = lb - near_slack(fabsf(x) + fabsf(y) + fabsf(z) + g.extent) - 4e-6f * fabsf(lb);
    const bool past = fmaxf(fmaxf(fabsf(x + base.x), fabsf(y + base.y)), fabsf(z + base.z)) > g.limit;
    // not a number: keeps every pair (their values are ignored)
    if (past || x != x || y != y || z != z) r.lb = -INFINITY;
    return r;
}

__device__ __forceinline__ float sd_pair(f4 C, float4 O) {
    const float ax = C.x - O.x, ay = C.y - O.y, az = C.z - O.z;
    return __builtin_amdgcn_sqrtf(fmaf(ax, ax, fmaf(ay, ay, az * az))) - O.w - C.w;
}

// Minimum signed distances of n configurations; a wave takes CW <= 8 of them at
// a time, eight lanes each for the pose, all lanes over (configuration, sphere)
// and (configuration, part pair) items after that.
//
// Bound by latency of the list and record gathers, which is why a row of lanes
// takes four spheres (two part pairs) at a time.  256 k configurations of the
// 7-DOF arm (70 spheres, 1500 self pairs) among 4096 spheres: all pairs 15.7 ms;
// one sphere per row at a time 484 us, four 414, in 127 registers (four waves a
// SIMD; five with spills 516).  With the field's build the call takes 0.46 ms.
__global__ void __launch_bounds__(256, 4) k_distances(RobotView rb, ObsView ob, NearView nv, int CW,
                                                   const float* __restrict__ q, int64_t n, int64_t stride_n,
                                                   int64_t stride_d, uint8_t* __restrict__ flags,
                                                   float* __restrict__ min_sd, float* __restrict__ min_sd_self) {
    extern __shared__ __align__(16) char smem[];
    const int lane = threadIdx.x & 63, w = wave_id(), W = blockDim.x >> 6;
    // the workgroup's tables, then each wave's share
    FlagTile t;
    {
        const lds_ptr<char> p = to_lds(smem);
        t.lbound = (lds_ptr<f4>)p;
        t.blocks = (lds_ptr<i4>)(t.lbound + kMaxParts);
        t.sph = (lds_ptr<f4>)(p + (int)robot_image_off_sph(rb.n_blocks));
        t.link = (lds_ptr<int>)(p + (int)robot_image_off_link(rb.n_spheres, rb.n_blocks));
        const int tb = (int)robot_stage_bytes(rb.n_spheres, rb.n_blocks, rb.n_self, false);
        const lds_ptr<char> m = p + tb + w * (int)sd_wave_bytes(CW);
        t.rec = (lds_ptr<f4>)m;
        t.stride = (int)sizeof(f4) * kRecRows;
        t.bounds = true;
        copy_to_lds(t.lbound, rb.image, tb / 16);
    }
    SdWave sw;
    sw.env = (lds_ptr<int>)(t.rec + CW * kRecRows);
    sw.self = sw.env + 8;
    sw.pick = sw.self + 8;
    sw.e = (lds_ptr<i4>)(sw.pick + 16);
    sw.n = 0;
    const float4 sh = cload4((const cfloat*)ob.centre);
    GridGeom g{};
    if (ob.n > 0) g = load_geom(nv.geom);
    const int j = lane & 7;
    const float dj = rb.dh[j].y;
    const int S = rb.n_spheres;
    __syncthreads();
    for (int64_t base = ((int64_t)blockIdx.x * W + w) * CW; base < n; base += (int64_t)gridDim.x * W * CW) {
        const int nc = (int)((n - base) < CW ? (n - base) : CW);
        if ((lane >> 3) < nc) {
            const float qj = q[(base + (lane >> 3)) * stride_n + (j < rb.dof ? j : 0) * stride_d];
            tile_pose(rb, sh, t, lane >> 3, j, qj, dj);
        }
        if (lane < nc) {
            sw.env[lane] = fkey(INFINITY);
            sw.self[lane] = fkey(INFINITY);
            sw.pick[lane] = 0x7fffffff;
        }
        wave_lds_sync();
        if (ob.n > 0 && S > 0) {
            // the exact value of a likely nearest pair of every sphere, three
            // spheres a lane in flight; then the spheres that may be nearer
            for (WaveWalk k(nc); __any(k.k < S);) {
                int c[3];
                f4 C[3];
                NearAt a[3];
                bool on[3];
#pragma unroll
                for (int u = 0; u < 3; ++u) {
                    on[u] = k.k < S;
                    c[u] = k.c;
                    const int s = on[u] ? k.k : 0;
                    k.next(nc);
                    C[u] = place(tile_frame(t, c[u], t.link[s]), t.sph[s]);
                    a[u] = near_at(g, nv, sh, C[u].x, C[u].y, C[u].z);
                }
#pragma unroll
                for (int u = 0; u < 3; ++u) {
                    const float v = sd_pair(C[u], ob.rec[a[u].o]);
                    if (on[u] && v == v) lds_min(sw.env + c[u], v);
                }
            }
            wave_lds_sync();
            WaveWalk k(nc);
            while (true) {
                if (sw.n < 64 && __any(k.k < S)) {
                    const bool on = k.k < S;
                    const int c = k.c, s = on ? k.k : 0;
                    k.next(nc);
                    const f4 C = place(tile_frame(t, c, t.link[s]), t.sph[s]);
                    const NearAt a = near_at(g, nv, sh, C.x, C.y, C.z);
                    const float lb = a.lb - C.w;
                    sw.push(on && !(lb >= lds_val(sw.env + c)), c | s << 6, lb, a.cell, a.len);
                } else if (sw.n > 0) {
                    wave_lds_sync();
                    const int m = min(sw.n, 64), sub = lane >> 4, li = lane & 15;
                    // spheres that no list serves: the wave's lanes over all
                    // obstacles, kAllSpheres of them to a record (their cost is
                    // that of the all-pairs kernel's pairs)
                    {
                        const i4 e = sw.e[sw.n - m + min(lane, m - 1)];
                        const int c = e.x & 63, s = e.x >> 6;
                        const f4 C = place(tile_frame(t, c, t.link[s]), t.sph[s]);
                        unsigned long long left = __ballot(lane < m && e.w == (int)kNearFull);
                        while (left) {
                            left &= __ballot(!(__int_as_float(e.y) >= lds_val(sw.env + c)));
                            if (!left) break;
                            f4 D[kAllSpheres];
                            int at[kAllSpheres];
                            float best[kAllSpheres];
#pragma unroll
                            for (int u = 0; u < kAllSpheres; ++u) {
                                at[u] = left ? __builtin_ctzll(left) : at[u > 0 ? u - 1 : 0];     // (a repeated one changes nothing)
                                left &= left - 1ull;
#pragma unroll
                                for (int k = 0; k < 4; ++k)
                                    D[u][k] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(C[k]), at[u]));
                                best[u] = INFINITY;
                            }
                            for (int o = lane; o < ob.n; o += 64) {
                                const float4 O = ob.rec[o];
#pragma unroll
                                for (int u = 0; u < kAllSpheres; ++u) best[u] = fminf(best[u], sd_pair(D[u], O));
                            }
#pragma unroll
                            for (int u = 0; u < kAllSpheres; ++u) {
                                const float v = wave_min(best[u]);
                                if (lane == 0) lds_min(sw.env + __builtin_amdgcn_readlane(c, at[u]), v);
                            }
                            wave_lds_sync();
                        }
                    }
                    // the others sixteen at a time, four to a row of 16 lanes, each
                    // over its cell's list
                    for (int i0 = 0; i0 < m; i0 += 16) {
                        f4 C[4];
                        int c[4], len[4];
                        const unsigned short* lst[4];
                        float best[4];
                        int most = 0;
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            const int i = i0 + 4 * u + sub;
                            const i4 e = sw.e[sw.n - m + min(i, m - 1)];
                            c[u] = e.x & 63;
                            const int s = e.x >> 6;
                            C[u] = place(tile_frame(t, c[u], t.link[s]), t.sph[s]);
                            lst[u] = nv.list + (size_t)e.z * kNearCap;
                            len[u] = e.w;
                            if (i >= m || e.w == (int)kNearFull || __int_as_float(e.y) >= lds_val(sw.env + c[u])) len[u] = 0;
                            most = max(most, len[u]);
                            best[u] = INFINITY;
                        }
                        for (int k2 = li; __any(k2 < most); k2 += 16) {
                            int o[4];
#pragma unroll
                            for (int u = 0; u < 4; ++u)
                                o[u] = k2 < len[u] ? (int)lst[u][k2] : -1;
                            float4 O[4];
#pragma unroll
                            for (int u = 0; u < 4; ++u) O[u] = ob.rec[max(o[u], 0)];
#pragma unroll
                            for (int u = 0; u < 4; ++u) best[u] = fminf(best[u], o[u] >= 0 ? sd_pair(C[u], O[u]) : INFINITY);
                        }
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            const float v = row_min(best[u]);
                            if (li == 0) lds_min(sw.env + c[u], v);
                        }
                    }
                    sw.n -= m;
                    wave_lds_sync();
                } else {
                    break;
                }
            }
        }
        // self pairs; when their own minimum is not asked for, the minimum so
        // far bounds them
        if (!min_sd_self && lane < nc) sw.self[lane] = sw.env[lane];
        wave_lds_sync();
        if (rb.n_blocks > 0) {
            // lower bound of a part pair's values
            auto part_lb = [&](int c, int bk) {
                const i4 blk = t.blocks[bk];
                const f4 A = t.row(c)[kRecLb + blk.x], B = t.row(c)[kRecLb + blk.y];
                const float dx = A.x - B.x, dy = A.y - B.y, dz = A.z - B.z;
                const float d = __builtin_amdgcn_sqrtf(fmaf(dx, dx, fmaf(dy, dy, dz * dz)));
                return d - A.w - B.w - near_slack(fabsf(A.x) + fabsf(A.y) + fabsf(A.z) + d);
            };
            if (lane < nc) sw.pick[lane] = 0x7fffffff;
            wave_lds_sync();
            for (WaveWalk k(nc); __any(k.k < rb.n_blocks); k.next(nc))
                if (k.k < rb.n_blocks)
                    __hip_atomic_fetch_min(sw.pick + k.c, (fkey(part_lb(k.c, k.k)) & ~255) | k.k, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_WORKGROUP);
            wave_lds_sync();
            const int own = sw.pick[lane < nc ? lane : 0] & 255;
            sw.push(lane < nc, lane | min(own, rb.n_blocks - 1) << 6, -INFINITY);
            WaveWalk k(nc);
            bool picked = false;
            while (true) {
                if (picked && sw.n < 64 && __any(k.k < rb.n_blocks)) {
                    const bool on = k.k < rb.n_blocks;
                    const int c = k.c, bk = on ? k.k : 0;
                    k.next(nc);
                    const float lb = part_lb(c, bk);
                    sw.push(on && bk != (sw.pick[c] & 255) && !(lb >= lds_val(sw.self + c)), c | bk << 6, lb);
                } else if (sw.n > 0) {
                    wave_lds_sync();
                    picked = true;
                    const int m = min(sw.n, 64), sub = lane >> 4, li = lane & 15;
                    for (int i0 = 0; i0 < m; i0 += 8) {
                        int c[2], p0[2], len[2], most = 0;
                        LFrame fa[2], fb[2];
                        float best[2];
#pragma unroll
                        for (int u = 0; u < 2; ++u) {
                            const int i = i0 + 4 * u + sub;
                            const i4 e = sw.e[sw.n - m + min(i, m - 1)];
                            c[u] = e.x & 63;
                            const i4 blk = t.blocks[e.x >> 6];
                            fa[u] = tile_frame(t, c[u], blk.x / kPartsPerLink);
                            fb[u] = tile_frame(t, c[u], blk.y / kPartsPerLink);
                            p0[u] = blk.z;
                            len[u] = i >= m || __int_as_float(e.y) >= lds_val(sw.self + c[u]) ? 0 : blk.w;
                            most = max(most, len[u]);
                            best[u] = INFINITY;
                        }
                        for (int p = li; __any(p < most); p += 16) {
                            int2 pr[2];
#pragma unroll
                            for (int u = 0; u < 2; ++u) pr[u] = rb.pairs[p0[u] + min(p, max(len[u] - 1, 0))];
#pragma unroll
                            for (int u = 0; u < 2; ++u) {
                                const f4 a = place(fa[u], t.sph[pr[u].x]), b = place(fb[u], t.sph[pr[u].y]);
                                const float dx = a.x - b.x, dy = a.y - b.y, dz = a.z - b.z;
                                const float v = __builtin_amdgcn_sqrtf(fmaf(dx, dx, fmaf(dy, dy, dz * dz))) - a.w - b.w;
                                best[u] = fminf(best[u], p < len[u] ? v : INFINITY);
                            }
                        }
#pragma unroll
                        for (int u = 0; u < 2; ++u) {
                            const float v = row_min(best[u]);
                            if (li == 0) lds_min(sw.self + c[u], v);
                        }
                    }
                    sw.n -= m;
                    wave_lds_sync();
                } else {
                    break;
                }
            }
        }
        wave_lds_sync();
        if (lane < nc) {
            const float self = lds_val(sw.self + lane), m = fminf(lds_val(sw.env + lane), self);
            const int64_t i = base + lane;
            flags[i] = m < 0.f ? 1 : 0;
            if (min_sd) min_sd[i] = m;
            if (min_sd_self) min_sd_self[i] = self;
        }
        wave_lds_sync();
    }
}

}  // namespace ezo
