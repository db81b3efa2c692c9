// nc_device.hpp -- device building blocks of the null-collision tracer (gfx950).
//
// Counter-based random numbers, ordered crossing of the hierarchical
// majorant grid, collision sampling with null/real rejection, and the
// scattering laws.  Everything here is FP32 except the merge criterion of the
// grid build (FP64).  The whole library is compiled with -ffp-contract=off so
// that every expression below rounds exactly as written: the traversal relies
// on each face parameter being the same function of the face index wherever
// it is evaluated.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <cmath>

#include "nctrace.h"

namespace nc {

constexpr float kPi = 3.14159265358979f;
constexpr float kInv4Pi = 0.0795774715459477f;

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon et al., SC'11): ten rounds of two 32x32->64-bit
// multiplies mixed with the key, the key bumped by Weyl constants.
// ---------------------------------------------------------------------------
struct U4 {
    uint32_t x, y, z, w;
};

__host__ __device__ inline U4 philox4x32_10(U4 c, uint32_t k0, uint32_t k1)
{
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        // one 32x32->64-bit product per multiplier (a single v_mad_u64_u32)
        const uint64_t p0 = (uint64_t)0xD2511F53u * (uint64_t)c.x;
        const uint64_t p1 = (uint64_t)0xCD9E8D57u * (uint64_t)c.z;
        const uint32_t hi0 = (uint32_t)(p0 >> 32), lo0 = (uint32_t)p0;
        const uint32_t hi1 = (uint32_t)(p1 >> 32), lo1 = (uint32_t)p1;
        c = U4{hi1 ^ c.y ^ k0, lo1, hi0 ^ c.w ^ k1, lo0};
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return c;
}

// The same with a key that is uniform over the wave (a kernel argument): the
// empty asm makes the key a fresh scalar at every call, so the round keys are
// formed by scalar adds inside the rounds instead of being hoisted out of
// the tracing loop as 18 loop invariants that take scalar registers from the
// loop (and are spilled).  Never call it with a key that differs across lanes.
__device__ inline U4 philox4x32_10_uk(U4 c, uint32_t k0, uint32_t k1)
{
    k0 = __builtin_amdgcn_readfirstlane(k0);   // uniform by contract: scalar registers
    k1 = __builtin_amdgcn_readfirstlane(k1);
    asm volatile("" : "+s"(k0), "+s"(k1));
    return philox4x32_10(c, k0, k1);
}

// -ln(w) for w in (0, 1] that is a multiple of 2^-24: the hardware's log2 times
// ln 2 in two floats (no subnormal, infinite or NaN argument to care for; the
// value of -__logf for all 2^24 arguments, up to the sign of -ln(1) = 0).
__device__ inline float neg_log_unit(float w)
{
    const float y = -__builtin_amdgcn_logf(w);   // (log2)
    const float p = y * 0x1.62e42ep-1f;
    const float e = __builtin_fmaf(y, 0x1.62e42ep-1f, -p);
    return p + __builtin_fmaf(y, 0x1.efa39ep-25f, e);
}

// A path's random stream: counter = (a, b, draw, stream), key = seed.  Each
// Philox call yields four uniforms, consumed in order.
// The counter words a, b and stream are supplied by the caller at each refill
// (the renderer rebuilds them from its pixel, sample and job), so a lane keeps
// only the draw index and the four buffered words.
struct RngBuf {
    uint32_t draw;
    uint32_t q0, q1, q2, q3;
    int left;

    __device__ void reset()
    {
        draw = 0;
        left = 0;
    }
    __device__ void need(int k, uint32_t a, uint32_t b, uint32_t stream, uint32_t k0, uint32_t k1)
    {
        if (left < k) {
            U4 r = philox4x32_10_uk(U4{a, b, draw, stream}, k0, k1);
            ++draw;
            q0 = r.x; q1 = r.y; q2 = r.z; q3 = r.w;
            left = 4;
        }
    }
    // drop a block that holds fewer than k numbers, as need(k) does; the next
    // one is computed when it is first needed
    __device__ void skip(int k) { left = left < k ? 0 : left; }
    __device__ float take()
    {
        const uint32_t v = q0;
        q0 = q1; q1 = q2; q2 = q3;
        --left;
        return (float)(v >> 8) * 5.9604644775390625e-08f;
    }
    __device__ float take_exp1() { return neg_log_unit(1.0f - take()); }
};

// A path's random stream kept per lane as a ring of four Philox blocks in LDS,
// for a kernel whose phases take several numbers at once without dropping any:
// before a phase that takes up to k numbers (k <= 12) the caller fills the ring
// where it holds fewer, and since a block costs a wave the same for one lane as
// for all, every lane with a free slot then computes its next block.  The
// numbers and their order are the stream's.  Layout [block % 4][word][lane]: a lane
// always falls on its own bank.
struct RngRing {
    static constexpr uint32_t kBlocks = 4;
    static constexpr int kWordsPerWave = kBlocks * 4 * 64;
    uint32_t *q;      // the lane's column of the wave's ring
    uint32_t head;    // next number of the stream (4 block + word)
    uint32_t gen;     // blocks computed so far

    __device__ void reset() { head = gen = 0; }
    __device__ bool holds(uint32_t k) const { return head + k <= 4u * gen; }
    __device__ bool space() const { return gen < (head >> 2) + kBlocks; }
    __device__ void fill(uint32_t a, uint32_t b, uint32_t stream, uint32_t k0, uint32_t k1)
    {
        const U4 r = philox4x32_10_uk(U4{a, b, gen, stream}, k0, k1);
        uint32_t *w = q + (gen & (kBlocks - 1u)) * 256u;
        w[0] = r.x;
        w[64] = r.y;
        w[128] = r.z;
        w[192] = r.w;
        ++gen;
    }
    __device__ float take()
    {
        const uint32_t v = q[(head & (4u * kBlocks - 1u)) * 64u];
        ++head;
        return (float)(v >> 8) * 5.9604644775390625e-08f;
    }
    __device__ float take_exp1() { return neg_log_unit(1.0f - take()); }
};

// ---------------------------------------------------------------------------
// Grid as seen by the kernels.
// Nodes of levels 1..L are stored level after level, each level [z][y][x]
// with ceil(n/2^l) nodes per axis; a node is float2(kmin_c, kmax_c) with the
// merged flag in the sign bit of kmin_c (k_c >= 0, so the bit is free).
// ---------------------------------------------------------------------------
struct GridView {
    int n[3];
    int L;
    float lo[3];
    float h[3];
    float inv_h[3];
    float hi[3];         // the box's far faces, (float)n h + lo rounded as the crossing rounds a face position
    float k_gas;
    float kscale;        // droplet extinction is kscale * kc (the grid holds kc's min and max)
    const float *kc;
    const float2 *nodes;
    const int *off;      // device array: node offset of level l at index l, off[L+1] = total
    const uint16_t *mask;  // per level-1 node [z][y][x]: bit l (1..L) set if the level-l ancestor is merged
    // nx ny < 2^24 and fewer than 2^30 cells: element numbers by full-rate
    // 24-bit multiply-adds and byte offsets in 32 bits (the general form takes
    // quarter-rate 32-bit products and 64-bit address adds)
    int narrow = 0;
};

__host__ __device__ inline int level_dim(int n, int l) { return (n + (1 << l) - 1) >> l; }

__host__ __device__ inline bool node_merged(float2 v) { return (__builtin_bit_cast(uint32_t, v.x) >> 31) != 0; }
__host__ __device__ inline float node_kmin(float2 v)
{
    return __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, v.x) & 0x7fffffffu);
}

// Node access with the top levels (l >= lds_first) staged in LDS.
struct NodeSrc {
    const float2 *glob;
    const float2 *lds;   // nodes of levels lds_first..L, same order
    const int *off;      // per-level offsets (LDS copy)
    int lds_first;
    int lds_base;        // off[lds_first]
    int n0, n1;
    const int4 *rows = nullptr;   // per level (LDS): node offset (within the staged block for a staged level),
                                  // nodes per row, nodes per slice, 0
};

// a b + c for a, b < 2^24 (one full-rate instruction on the GPU)
__host__ __device__ inline uint32_t mad24(uint32_t a, uint32_t b, uint32_t c)
{
    return (a & 0xffffffu) * (b & 0xffffffu) + c;
}

// (int)floorf(x) in one instruction (finite x; saturates like the conversion)
__host__ __device__ inline int floor_int(float x)
{
#ifdef __HIP_DEVICE_COMPILE__
    int j;
    asm("v_cvt_flr_i32_f32 %0, %1" : "=v"(j) : "v"(x));
    return j;
#else
    return (int)floorf(x);
#endif
}

__host__ __device__ inline int clamp_int(int j, int lo, int hi)   // lo <= hi
{
    return j < lo ? lo : (j > hi ? hi : j);
}

__host__ __device__ inline float2 fetch_node(const NodeSrc &s, int l, int c0, int c1, int c2, uint32_t &gcount)
{
    const int d0 = level_dim(s.n0, l), d1 = level_dim(s.n1, l);
    const int idx = s.off[l] + ((c2 >> l) * d1 + (c1 >> l)) * d0 + (c0 >> l);
    if (l >= s.lds_first) return s.lds[idx - s.lds_base];
    ++gcount;
    return s.glob[idx];
}

// ---------------------------------------------------------------------------
// Ray state for the ordered crossing of the grid (Section 3.1.3).
//
// Face j of axis a lies at lo[a] + j h[a]; the ray meets it at
//   tf(a, j) = ((float)j * h[a] + lo[a] - o[a]) * inv[a],
// monotone in j.  A voxel's exit parameter is the smallest tf over its faces
// (clipped to the box), and every axis whose face attains it is stepped
// across exactly; the other axes keep a cell inside the voxel's slab (the
// floor of the position, clamped).  Only the voxel matters to the walk, the
// exit axes always move forward and no axis steps back across a voxel face,
// so the walk visits each voxel at most once and ends after at most
// nx + ny + nz voxels.  The cell past the exit face is found together with
// the exit parameter (both need the voxel's two faces per axis): the crossing
// itself is then a copy.
//
// The crossing functions are compiled for the host as well (a bit-exact
// FP32 twin for testing the walk on every ray): they use only IEEE
// operations that round the same on both sides (the GPU's short reciprocal is
// correctly rounded; the library is built without FP contraction).
// ---------------------------------------------------------------------------
struct Ray {
    float o[3], d[3], inv[3];
    float t, tend;       // current parameter, exit from the box
    int c[3];            // current cell
    int lev;             // current voxel: level and node indices (c >> lev)
    float khat;          // voxel majorant m (kscale kmax_c + k_gas)
    float kmin;          // voxel minimum of k_c (for a level-0 voxel: k_c of the cell)
    float texit;         // voxel exit parameter
    int cn[3];           // first cell past the exit face (set with texit)
    int xmask;           // axes whose voxel face is met at texit (bit a)
};

// Per axis 1 / d rounded to nearest, NaN for d = 0.  v_rcp_f32 and one Newton
// step in FMAs give the correctly rounded reciprocal of every normal
// |d| < 2^126 (checked over all mantissas and exponents) in 3 instructions
// where the IEEE division takes 10; a direction with a subnormal component or
// one of 2^126 or more takes the division.
__host__ __device__ inline void ray_inverse(const float d[3], float inv[3])
{
#ifdef __HIP_DEVICE_COMPILE__
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const float y = __builtin_amdgcn_rcpf(d[a]);
        inv[a] = __builtin_fmaf(__builtin_fmaf(-d[a], y, 1.0f), y, y);
    }
    const float m = fmaxf(fmaxf(fabsf(d[0]), fabsf(d[1])), fabsf(d[2]));
    if (!(__builtin_amdgcn_classf(d[0], 0x90) | __builtin_amdgcn_classf(d[1], 0x90) |
          __builtin_amdgcn_classf(d[2], 0x90) | (m >= 0x1p126f)))
        return;
#endif
#pragma unroll
    for (int a = 0; a < 3; ++a) inv[a] = d[a] == 0.0f ? __builtin_nanf("") : 1.0f / d[a];
}

__host__ __device__ inline float face_t(const GridView &g, const Ray &r, int a, int j)
{
    return ((float)j * g.h[a] + g.lo[a] - r.o[a]) * r.inv[a];
}

// Clip o + t d (t >= tmin) to the box; false if it misses.
// An axis the ray is parallel to (d = 0) has inv = NaN: its face parameters
// are NaN, which min, max and the comparisons below pass over.
__host__ __device__ inline bool ray_setup(const GridView &g, Ray &r, const float o[3], const float d[3], float tmin)
{
    float tin = tmin, tout = INFINITY;
    bool miss = false;
    float tlo[3];
    ray_inverse(d, r.inv);
    // per axis, as selects (lanes that disagree would run both sides of a branch)
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        r.o[a] = o[a];
        r.d[a] = d[a];
        // (both faces straight from the grid view, not through face_t: the
        // compiler cannot fold 0 h, and the hoisted per-axis values held through a
        // persistent loop cost registers)
        const float b0 = g.lo[a], b1 = g.hi[a];
        miss |= (d[a] == 0.0f) & ((o[a] < b0) | (o[a] > b1));   // parallel to the axis' faces and outside their slab
        const float t0 = (b0 - r.o[a]) * r.inv[a], t1 = (b1 - r.o[a]) * r.inv[a];
        tlo[a] = t0 > t1 ? t1 : t0;
        tin = fmaxf(tin, tlo[a]);
        tout = fminf(tout, t0 > t1 ? t0 : t1);
    }
    if (miss | !(tin < tout)) return false;
    r.t = tin;
    r.tend = tout;
    // starting cell: exact on the axis through whose face the ray enters the
    // box, the floor of the position (clamped) on the others; only the voxel
    // matters for the walk, and the walk never steps back across a face
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const int j = floor_int((o[a] + tin * d[a] - g.lo[a]) * g.inv_h[a]);
        const bool entered = (tin > tmin) & (tlo[a] == tin);   // entered through this axis' face
        // (the far end by the clamp: the sign bit spread over the word, less its top bit)
        const int end = (int)((uint32_t)(__builtin_bit_cast(int, d[a]) >> 31) >> 1);
        r.c[a] = clamp_int(entered ? end : j, 0, g.n[a] - 1);
    }
    return true;
}

__host__ __device__ inline void leaf_exit(const GridView &g, Ray &r);

// Voxel of the current cell: its coarsest merged ancestor (the cell itself
// when no ancestor is merged), with its majorant and minimum.  The ancestry
// mask of the cell's level-1 node gives the level in one read (highest set
// bit); the cell's own value is read at the same time, so a level-0 voxel
// costs one round trip to memory and a coarser one at most two (none when
// its level is staged in LDS).
// kUnit: the grid view's kscale is 1.
template <bool kUnit = false>
__host__ __device__ inline void locate_voxel(const GridView &g, const NodeSrc &ns, Ray &r, float mscale,
                                             uint32_t &node_reads)
{
    float kmin, kmax;
    int l = 0;
    // cell indices are >= 0; the row index fits 32 bits (n1, n2 <= 2^15)
    if (g.narrow && ns.rows) {
        const uint32_t x = (uint32_t)r.c[0], y = (uint32_t)r.c[1], z = (uint32_t)r.c[2];
        const uint32_t cell = mad24(z, (uint32_t)(g.n[0] * g.n[1]), mad24(y, (uint32_t)g.n[0], x));
        const float kcell = *(const float *)((const char *)g.kc + (cell << 2));
        const uint32_t d0 = (uint32_t)level_dim(g.n[0], 1), d1 = (uint32_t)level_dim(g.n[1], 1);
        const uint32_t mi = mad24(z >> 1, d0 * d1, mad24(y >> 1, d0, x >> 1));
        const uint32_t m = *(const uint16_t *)((const char *)g.mask + (mi << 1));   // (L >= 1: a narrow grid has a mask)
        node_reads += 2;
        l = 31 - __builtin_clz(m | 1u);
        kmin = kmax = kcell;
        if (l != 0) {
            const int4 row = ns.rows[l];
            const uint32_t idx = mad24(z >> l, (uint32_t)row.z, mad24(y >> l, (uint32_t)row.y, (x >> l) + (uint32_t)row.x));
            float2 nd;
            // two loads on two paths (not one flat load through a selected
            // address, which waits for both memories)
            if (l >= ns.lds_first) {
                nd = ns.lds[idx];
#ifdef __HIP_DEVICE_COMPILE__
                asm volatile("" : "+v"(nd.x), "+v"(nd.y));
#endif
            } else {
                ++node_reads;
                nd = *(const float2 *)((const char *)ns.glob + (idx << 3));
            }
            kmin = node_kmin(nd);
            kmax = nd.y;
        }
    } else {
        const uint32_t row = (uint32_t)r.c[2] * (uint32_t)g.n[1] + (uint32_t)r.c[1];
        const uint64_t cell = (uint64_t)row * (uint32_t)g.n[0] + (uint32_t)r.c[0];
        const float kcell = g.kc[cell];
        ++node_reads;
        if (g.L >= 1) {
            const int d0 = level_dim(g.n[0], 1), d1 = level_dim(g.n[1], 1);
            const uint32_t mrow = (uint32_t)(r.c[2] >> 1) * (uint32_t)d1 + (uint32_t)(r.c[1] >> 1);
            const uint32_t m = g.mask[(uint64_t)mrow * (uint32_t)d0 + (uint32_t)(r.c[0] >> 1)];
            ++node_reads;
            l = m ? 31 - __builtin_clz(m) : 0;
        }
        if (l == 0) {
            kmin = kmax = kcell;
        } else {
            const float2 nd = fetch_node(ns, l, r.c[0], r.c[1], r.c[2], node_reads);
            kmin = node_kmin(nd);
            kmax = nd.y;
        }
    }
    r.lev = l;
    r.khat = mscale * ((kUnit ? kmax : g.kscale * kmax) + g.k_gas);
    r.kmin = kmin;
}

__host__ __device__ inline void find_leaf(const GridView &g, const NodeSrc &ns, Ray &r, float mscale,
                                          uint32_t &node_reads)
{
    locate_voxel(g, ns, r, mscale, node_reads);
    leaf_exit(g, r);
}

// Exit parameter of the current voxel (its faces clipped to the field) and
// the first cell past the exit face.  A face on the box's side needs no
// exception: its parameter is the one tend was taken from, bit for bit, or
// beyond it, and at tend the ray ends without using the next cell.
__host__ __device__ inline void leaf_exit(const GridView &g, Ray &r)
{
    const int l = r.lev;
    float tf[3];
    int lo[3], hi[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        lo[a] = (r.c[a] >> l) << l;
        hi[a] = min(lo[a] + (1 << l), g.n[a]);
        tf[a] = face_t(g, r, a, r.d[a] > 0.0f ? hi[a] : lo[a]);
    }
    float te = fminf(fminf(fminf(r.tend, tf[0]), tf[1]), tf[2]);
    const float tx = te < r.t ? r.t : te;
    r.xmask = (tf[0] == te ? 1 : 0) | (tf[1] == te ? 2 : 0) | (tf[2] == te ? 4 : 0);
    r.texit = tx;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        // the exit axes step across their face, the others stay inside the voxel's slab
        const int j = clamp_int(floor_int((r.o[a] + tx * r.d[a] - g.lo[a]) * g.inv_h[a]), lo[a], hi[a] - 1);
        r.cn[a] = tf[a] == te ? (r.d[a] > 0.0f ? hi[a] : lo[a] - 1) : j;
    }
}

// Cross the current voxel's exit face: the ray moves to its exit parameter
// and its cell to the first one past the face (false when the ray leaves the
// box).  The voxel there is not located.
__host__ __device__ inline bool step_cell(const GridView &g, Ray &r)
{
    (void)g;
    r.t = r.texit;
    if (!(r.t < r.tend)) return false;
#pragma unroll
    for (int a = 0; a < 3; ++a) r.c[a] = r.cn[a];
    return true;
}

// Move to the voxel after the current one; false when the ray leaves the box.
__host__ __device__ inline bool next_leaf(const GridView &g, const NodeSrc &ns, Ray &r, float mscale,
                                          uint32_t &node_reads)
{
    if (!step_cell(g, r)) return false;
    find_leaf(g, ns, r, mscale, node_reads);
    return true;
}

// k_c of a cell
__device__ inline float cell_k(const GridView &g, const int cc[3])
{
    if (g.narrow) {
        const uint32_t cell = mad24((uint32_t)cc[2], (uint32_t)(g.n[0] * g.n[1]),
                                    mad24((uint32_t)cc[1], (uint32_t)g.n[0], (uint32_t)cc[0]));
        return *(const float *)((const char *)g.kc + (cell << 2));
    }
    const uint32_t row = (uint32_t)cc[2] * (uint32_t)g.n[1] + (uint32_t)cc[1];
    return g.kc[(uint64_t)row * (uint32_t)g.n[0] + (uint32_t)cc[0]];
}

// k_c of the cell holding the point at parameter t, kept inside the current voxel
// so that it never exceeds the voxel's majorant.  The voxel is found
// from the next cell (which lies in its slab on every axis but those of the
// exit face, one cell past it there), so that no register holds the current
// cell between the crossing and a collision.
__device__ inline float collision_k(const GridView &g, const Ray &r, float t)
{
    const int l = r.lev;
    int cc[3];
    // (a level-0 voxel clamps to its own cell)
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const int past = (r.xmask & (1 << a)) ? (r.d[a] > 0.0f ? 1 : -1) : 0;
        const int base = ((r.cn[a] - past) >> l) << l;
        const int top = min(base + (1 << l), g.n[a]) - 1;
        cc[a] = clamp_int(floor_int((r.o[a] + t * r.d[a] - g.lo[a]) * g.inv_h[a]), base, top);
    }
    return cell_k(g, cc);
}

// ---------------------------------------------------------------------------
// Scattering
// ---------------------------------------------------------------------------
// (reciprocals by v_rcp/v_rsq: a relative error of ~1e-7 in a Monte Carlo
// weight is far below the statistical error)
//
// The constants of one asymmetry g are formed once on the host and reach the
// kernels as arguments (scalar registers), so that no vector register holds
// them through the persistent loop.
struct HGc {
    float a;     // 1 + g^2
    float b;     // 2 g
    float c;     // (1 - g^2) / (4 pi)
    float e;     // 1 - g^2
    float d;     // 1 - g
    float r2g;   // 1 / (2 g); 0 when |g| < 1e-4 (then the cosine is uniform)
};

inline HGc make_hg(double g)
{
    HGc h;
    h.a = (float)(1.0 + g * g);
    h.b = (float)(2.0 * g);
    h.c = (float)((1.0 - g * g) / (4.0 * 3.14159265358979323846));
    h.e = (float)(1.0 - g * g);
    h.d = (float)(1.0 - g);
    h.r2g = std::fabs(g) < 1e-4 ? 0.0f : (float)(1.0 / (2.0 * g));
    return h;
}

__device__ inline float hg_phase(const HGc &h, float mu)
{
    const float den = h.a - h.b * mu;
    return h.c * __builtin_amdgcn_rsqf(den) * __builtin_amdgcn_rcpf(den);
}

// Inverse-CDF sample of the HG cosine.
__device__ inline float hg_sample_mu(const HGc &h, float xi)
{
    if (h.r2g == 0.0f) return 2.0f * xi - 1.0f;
    const float s = h.e * __builtin_amdgcn_rcpf(h.d + h.b * xi);
    const float mu = (h.a - s * s) * h.r2g;
    return fminf(1.0f, fmaxf(-1.0f, mu));
}

// A tabulated phase function: values p at cosines mu (n nodes, -1 .. 1),
// linear in between, normalised per steradian; cdf[i] = 2 pi times its
// integral up to mu[i].
struct PhaseView {
    const float *mu, *p, *cdf;
    int n;
};

// the node interval [mu[i], mu[i+1]] holding x of a sorted array (i in 0..n-2)
__device__ inline int tab_interval(const float *a, int n, float x)
{
    int lo = 0, hi = n - 1;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (a[mid] <= x) lo = mid;
        else hi = mid;
    }
    return lo;
}

__device__ inline float tab_phase(const PhaseView &t, float m)
{
    const int i = tab_interval(t.mu, t.n, m);
    const float f = (m - t.mu[i]) * __builtin_amdgcn_rcpf(t.mu[i + 1] - t.mu[i]);
    return t.p[i] + f * (t.p[i + 1] - t.p[i]);
}

// Inverse CDF: in the interval holding xi the CDF is 2 pi (p_i x + s x^2 / 2)
// above cdf[i], x = m - mu[i], s the slope; x is the positive root, in the
// form without cancellation.
__device__ inline float tab_sample(const PhaseView &t, float xi)
{
    const int i = tab_interval(t.cdf, t.n, xi);
    const float m0 = t.mu[i], dm = t.mu[i + 1] - m0, p0 = t.p[i];
    const float s = (t.p[i + 1] - p0) * __builtin_amdgcn_rcpf(dm);
    const float r = fmaxf(xi - t.cdf[i], 0.0f) * (1.0f / (2.0f * kPi));
    const float den = p0 + sqrtf(fmaxf(p0 * p0 + 2.0f * s * r, 0.0f));
    const float x = den > 0.0f ? 2.0f * r * __builtin_amdgcn_rcpf(den) : 0.0f;
    return fminf(m0 + fminf(x, dm), 1.0f);
}

// The medium's phase function: the table when there is one, else HG.
__device__ inline float phase_eval(const HGc &h, const PhaseView &t, float mu)
{
    return t.n ? tab_phase(t, mu) : hg_phase(h, mu);
}

__device__ inline float phase_sample_mu(const HGc &h, const PhaseView &t, float xi)
{
    return t.n ? tab_sample(t, xi) : hg_sample_mu(h, xi);
}

// Orthonormal basis around unit n (Duff et al., "Building an orthonormal
// basis, revisited", JCGT 2017), then the direction at cosine mu, azimuth
// 2 pi u about n.
// (sp, cp: sine and cosine of the azimuth; the final normalisation absorbs the
// rounding of the basis.)
__device__ inline void turn_sc(float d[3], float mu, float sp, float cp)
{
    const float sgn = copysignf(1.0f, d[2]);
    const float a = -__builtin_amdgcn_rcpf(sgn + d[2]);
    const float b = d[0] * d[1] * a;
    const float b1[3] = {1.0f + sgn * d[0] * d[0] * a, sgn * b, -sgn * d[0]};
    const float b2[3] = {b, sgn + d[1] * d[1] * a, -d[1]};
    const float st = __builtin_amdgcn_sqrtf(fmaxf(0.0f, 1.0f - mu * mu));
    float n[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) n[k] = mu * d[k] + st * (cp * b1[k] + sp * b2[k]);
    const float inv = __builtin_amdgcn_rsqf(n[0] * n[0] + n[1] * n[1] + n[2] * n[2]);   // (|n|^2 is about 1)
#pragma unroll
    for (int k = 0; k < 3; ++k) d[k] = n[k] * inv;
}

__device__ inline void turn(float d[3], float mu, float u)
{
    turn_sc(d, mu, __builtin_amdgcn_sinf(u), __builtin_amdgcn_cosf(u));   // sin, cos of 2 pi u
}

// Cosine-weighted direction about +z (Lambertian reflection).
__device__ inline void lambert(float d[3], float u1, float u2)
{
    const float sp = __builtin_amdgcn_sinf(u2), cp = __builtin_amdgcn_cosf(u2);   // sin, cos of 2 pi u2
    const float r = __builtin_amdgcn_sqrtf(u1);
    d[0] = r * cp;
    d[1] = r * sp;
    d[2] = __builtin_amdgcn_sqrtf(fmaxf(0.0f, 1.0f - u1));
}

// ---------------------------------------------------------------------------
// Per-lane event counters, reduced once per wave at the end of a launch.
// ---------------------------------------------------------------------------
struct Counters {
    uint32_t paths, segments, tentative, nulls, reals, leaf_visits, gathers, node_reads, nee_rays, truncated;
};

__device__ inline unsigned long long wave_sum(uint32_t v)
{
    unsigned long long s = v;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off);
    return s;
}

__device__ inline void flush_counters(const Counters &c, nc_counters *out)
{
    if (!out) return;
    const unsigned long long v[10] = {wave_sum(c.paths), wave_sum(c.segments), wave_sum(c.tentative),
                                      wave_sum(c.nulls), wave_sum(c.reals), wave_sum(c.leaf_visits),
                                      wave_sum(c.gathers), wave_sum(c.node_reads), wave_sum(c.nee_rays),
                                      wave_sum(c.truncated)};
    if (__lane_id() == 0) {
        unsigned long long *o = reinterpret_cast<unsigned long long *>(out);
#pragma unroll
        for (int k = 0; k < 10; ++k)
            if (v[k]) atomicAdd(o + k, v[k]);
    }
}

// Lanes for which pred holds.  (The scalar count by hand: the compiler keeps
// __popcll's result, and every comparison with it, in 64 bits, which the
// scalar unit does not compare.)
__device__ inline int lane_count(bool pred)
{
    const unsigned long long m = __ballot(pred);
    int n;
    asm("s_bcnt1_i32_b64 %0, %1" : "=s"(n) : "s"(m) : "scc");
    return n;
}

__device__ inline unsigned int lanes_below(unsigned long long mask)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// Lane phases of the phase-scheduled kernels.  Each loop trip the wave runs the
// phase that the most lanes are waiting in (ballot counts); the other lanes
// wait.  Expensive code (events, ray starts, new samples) thus runs for many
// lanes at once instead of diverging inside every traversal step.
enum Phase { kPhCross = 0, kPhCollide = 1, kPhEvent = 2, kPhRay = 3, kPhSample = 4, kPhGuide = 5, kPhIdle = 6 };
static_assert(kPhGuide == 5 && kPhIdle == 6, "six running phases, one counter slot each");
// Queue items a wave takes per global atomic: one per lane, so that the last
// chunks are short (paths differ a lot in cost and the launch ends with the
// slowest wave).
constexpr int kChunk = 64;
static_assert(kChunk >= 64, "a chunk must cover every lane of a wave that needs an item");

// After the optical thickness tau has been drawn or carried: a tentative
// collision inside the current voxel, or a move to the next voxel.
__device__ inline int voxel_phase(const Ray &r, float tau)
{
    return (r.khat > 0.0f && tau < r.khat * (r.texit - r.t)) ? kPhCollide : kPhCross;
}

// block-level event counters in LDS (same order as nc_counters)
enum BlockCounter {
    kCPaths = 0, kCSegments, kCTentative, kCNulls, kCReals, kCLeaf, kCGathers, kCReads, kCNee, kCTrunc,
    kCTrips0, kCLanes0 = kCTrips0 + 6, kCCycles0 = kCLanes0 + 6, kCDeep = kCCycles0 + 6,
    kNumBlockCounters = kCDeep + 1
};

__device__ inline void wave_count(unsigned long long *s_cnt, int k, bool pred)
{
    if (!s_cnt) return;   // no counters asked for
    const unsigned long long m = __ballot(pred);
    if (m && __lane_id() == 0) atomicAdd(s_cnt + k, (unsigned long long)__popcll(m));
}

// How a ray's step ended.
enum StepResult { kContinue = 0, kReal = 1, kExit = 2 };

// Start a ray; a ray that misses the box is set up to exit on its first step.
__device__ inline void start_ray(const GridView &g, const NodeSrc &ns, Ray &r, const float o[3], const float d[3],
                                 float mscale, Counters &cnt)
{
    if (ray_setup(g, r, o, d, 0.0f)) {
        find_leaf(g, ns, r, mscale, cnt.node_reads);
        ++cnt.leaf_visits;
    } else {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            r.o[a] = o[a];
            r.d[a] = d[a];
        }
        r.t = r.tend = r.texit = 0.0f;
        r.khat = 0.0f;
        r.kmin = 0.0f;
        r.lev = g.L;
    }
}

// The level offsets and the staged levels' nodes into LDS; rows (may be
// null): the level table of locate_voxel.  Ends with a block barrier.
__device__ inline void stage_levels(const GridView &g, int lds_first, int lds_nodes, float2 *s_nodes, int *s_off,
                                    int4 *rows = nullptr)
{
    for (int i = threadIdx.x; i < NC_MAX_LEVELS + 2; i += blockDim.x) {
        s_off[i] = i <= g.L + 1 ? g.off[i] : 0;
        if (rows) {
            const int d0 = level_dim(g.n[0], min(i, 30)), d1 = level_dim(g.n[1], min(i, 30));
            const int base = i >= lds_first && i <= g.L ? g.off[lds_first] : 0;
            rows[i] = make_int4(i <= g.L ? g.off[i] - base : 0, d0, d0 * d1, 0);
        }
    }
    if (lds_nodes > 0) {
        const int base = g.off[lds_first];
        for (int i = threadIdx.x; i < lds_nodes; i += blockDim.x) s_nodes[i] = g.nodes[base + i];
    }
    __syncthreads();
}

// ---------------------------------------------------------------------------
// A path on four lanes.  A wave that holds one path advances it by one
// instruction every 6 to 8 cycles whatever the instruction (measured: dependent
// FMAs 8.3 cycles, scalar adds 8, independent adds 6), so a lone path's speed is
// its instruction count.  Three of the four lanes of a quad therefore hold an
// axis each (the fourth repeats x), so what a ray does per axis is one
// instruction instead of three; minima and sums over the axes are two quad
// permutes; everything else is the same in the four lanes.  All branches are
// on values that are the same in the quad.  The arithmetic is the one-lane
// walk's, operation for operation (the order of a sum over the axes included),
// so a path may be handed from one form to the other at any point.  Narrow
// grids only (GridView::narrow).
// ---------------------------------------------------------------------------
template <int kCtrl>
__device__ inline int quad_perm(int x)
{
    return __builtin_amdgcn_mov_dpp(x, kCtrl, 0xf, 0xf, true);
}
template <int kCtrl>
__device__ inline float quad_perm(float x)
{
    return __int_as_float(quad_perm<kCtrl>(__float_as_int(x)));
}
constexpr int kQuadSwap1 = 0xb1, kQuadSwap2 = 0x4e;   // lane ^ 1, lane ^ 2
// the value of axis kAxis, in all four lanes
template <int kAxis, class T>
__device__ inline T quad_axis(T x)
{
    return quad_perm<kAxis * 0x55>(x);
}
__device__ inline float quad_min(float x)
{
    x = fminf(x, quad_perm<kQuadSwap1>(x));
    return fminf(x, quad_perm<kQuadSwap2>(x));
}
__device__ inline float quad_max(float x)
{
    x = fmaxf(x, quad_perm<kQuadSwap1>(x));
    return fmaxf(x, quad_perm<kQuadSwap2>(x));
}
__device__ inline int quad_add(int x)
{
    x += quad_perm<kQuadSwap1>(x);
    return x + quad_perm<kQuadSwap2>(x);
}
__device__ inline int quad_or(int x)
{
    x |= quad_perm<kQuadSwap1>(x);
    return x | quad_perm<kQuadSwap2>(x);
}
// x[0] + x[1] + x[2], summed in that order
__device__ inline float quad_sum(float x) { return quad_axis<0>(x) + quad_axis<1>(x) + quad_axis<2>(x); }

// The axis' value of three.  (By value: a choice between members of a record
// becomes an address into it, which puts the whole record in scratch memory.)
template <class T>
__device__ inline T quad_pick(int ax, T x, T y, T z)
{
    return ax == 0 ? x : ax == 1 ? y : z;
}

// The lane's axis of the grid.
struct QuadGrid {
    int ql, ax;          // lane of the quad, its axis (lane 3: x again)
    float lo, hi, h, inv_h;
    int n;
    int cell_stride, mask_stride;   // of the axis (lane 3: 0, it takes no part in the sums)
    const int4 *rows;    // LDS: per level nodes per row and slice, and the level's offset

    __device__ __attribute__((always_inline)) void init(const GridView &g, const int4 *rows_)
    {
        ql = (int)(threadIdx.x & 3u);
        ax = ql == 3 ? 0 : ql;
        lo = quad_pick(ax, g.lo[0], g.lo[1], g.lo[2]);
        hi = quad_pick(ax, g.hi[0], g.hi[1], g.hi[2]);
        h = quad_pick(ax, g.h[0], g.h[1], g.h[2]);
        inv_h = quad_pick(ax, g.inv_h[0], g.inv_h[1], g.inv_h[2]);
        n = quad_pick(ax, g.n[0], g.n[1], g.n[2]);
        const int d0 = level_dim(g.n[0], 1), d1 = level_dim(g.n[1], 1);
        cell_stride = ql == 0 ? 1 : ql == 1 ? g.n[0] : ql == 2 ? g.n[0] * g.n[1] : 0;
        mask_stride = ql == 0 ? 1 : ql == 1 ? d0 : ql == 2 ? d0 * d1 : 0;
        rows = rows_;
    }
};

// A ray on a quad: per axis o, d, inv, the cell and its voxel's faces; the rest as in Ray.
struct QuadRay {
    float o, d, inv, tf;
    int c, clo, chi;         // current cell; its voxel's first cell and the one past its last
    float t, tend, te, texit;
    float khat, kmin;
    int lev;
    // a cell of a voxel known before (an event's, or the one its sun ray started in)
    int vc, vlev;
    float vkmin, vkhat;

    // as ray_setup
    __device__ __attribute__((always_inline)) bool setup(const QuadGrid &g, float dir)
    {
        d = dir;
        {
            const float y = __builtin_amdgcn_rcpf(d);
            inv = __builtin_fmaf(__builtin_fmaf(-d, y, 1.0f), y, y);
            if (__builtin_amdgcn_classf(d, 0x90) | (fabsf(d) >= 0x1p126f)) {
                asm volatile("");   // (a branch: the division is not to be computed beside the short form)
                inv = 1.0f / d;
            }
        }
        const float t0 = (g.lo - o) * inv, t1 = (g.hi - o) * inv;
        float tlo = t0 > t1 ? t1 : t0;
        // parallel to the axis' faces and outside their slab: a miss
        const bool out = (d == 0.0f) & ((o < g.lo) | (o > g.hi));
        const float tin = fmaxf(0.0f, quad_max(out ? INFINITY : tlo));
        const float tout = quad_min(t0 > t1 ? t0 : t1);
        if (!(tin < tout)) return false;
        t = tin;
        tend = tout;
        const int j = floor_int((o + tin * d - g.lo) * g.inv_h);
        const bool entered = (tin > 0.0f) & (tlo == tin);
        const int end = (int)((uint32_t)(__float_as_int(d) >> 31) >> 1);
        c = clamp_int(entered ? end : j, 0, g.n - 1);
        return true;
    }
    // the current voxel's exit faces and parameter (as leaf_exit), from its level and a cell
    __device__ __attribute__((always_inline)) void faces(const QuadGrid &g)
    {
        clo = (c >> lev) << lev;
        chi = min(clo + (1 << lev), g.n);
        tf = ((float)(d > 0.0f ? chi : clo) * g.h + g.lo - o) * inv;
        te = fminf(tend, quad_min(tf));
    }
    __device__ __attribute__((always_inline)) void enter(const QuadGrid &g)
    {
        faces(g);
        texit = te < t ? t : te;
    }
    // across the exit face (t is there already): the next cell
    __device__ __attribute__((always_inline)) void next_cell(const QuadGrid &g)
    {
        const int j = clamp_int(floor_int((o + t * d - g.lo) * g.inv_h), clo, chi - 1);
        c = tf == te ? (d > 0.0f ? chi : clo - 1) : j;
    }
    // k_c of the cell at parameter t (as collision_k)
    __device__ __attribute__((always_inline)) float k_at(const GridView &gv, const QuadGrid &g) const
    {
        const int cc = clamp_int(floor_int((o + t * d - g.lo) * g.inv_h), clo, chi - 1);
        const uint32_t cell = (uint32_t)quad_add((int)mad24((uint32_t)cc, (uint32_t)g.cell_stride, 0u));
        return *(const float *)((const char *)gv.kc + (cell << 2));
    }
    // as locate_voxel
    __device__ __attribute__((always_inline)) void locate(const GridView &gv, const QuadGrid &g, const NodeSrc &ns,
                                                          float mscale)
    {
        const uint32_t cell = (uint32_t)quad_add((int)mad24((uint32_t)c, (uint32_t)g.cell_stride, 0u));
        const uint32_t mi = (uint32_t)quad_add((int)mad24((uint32_t)c >> 1, (uint32_t)g.mask_stride, 0u));
        const float kcell = *(const float *)((const char *)gv.kc + (cell << 2));
        const uint32_t m = *(const uint16_t *)((const char *)gv.mask + (mi << 1));
        lev = 31 - __builtin_clz(m | 1u);
        float kmax = kcell;
        kmin = kcell;
        if (lev != 0) {
            const int4 row = g.rows[lev];
            const int stride = g.ql == 3 ? 0 : quad_pick(g.ql, 1, row.y, row.z);
            const uint32_t idx =
                (uint32_t)row.x + (uint32_t)quad_add((int)mad24((uint32_t)(c >> lev), (uint32_t)stride, 0u));
            float2 nd;
            if (lev >= ns.lds_first) {
                nd = ns.lds[idx];
                asm volatile("" : "+v"(nd.x), "+v"(nd.y));   // (two loads, as in locate_voxel)
            } else {
                nd = *(const float2 *)((const char *)ns.glob + (idx << 3));
            }
            kmin = node_kmin(nd);
            kmax = nd.y;
        }
        khat = mscale * (gv.kscale * kmax + gv.k_gas);
    }
    // the voxel of the ray's first cell: the known one, if the cell lies in it (then nothing is read)
    __device__ __attribute__((always_inline)) void first_voxel(const GridView &gv, const QuadGrid &g,
                                                               const NodeSrc &ns, float mscale)
    {
        lev = vlev;
        kmin = vkmin;
        khat = vkhat;
        if ((quad_or(c ^ vc) >> vlev) != 0) locate(gv, g, ns, mscale);
        keep_voxel();
    }
    __device__ __attribute__((always_inline)) void keep_voxel()
    {
        vc = c;
        vlev = lev;
        vkmin = kmin;
        vkhat = khat;
    }
};

// A path's random numbers on a quad: its lanes compute four consecutive blocks
// at once (a quarter of the Philox instructions per block) into the quad's 16
// words of LDS, from where a block is read when its numbers are first needed.
// The same stream as RngBuf's.
struct RngQuad {
    uint32_t *buf;               // the quad's words
    uint32_t draw;               // next block
    uint32_t q0, q1, q2, q3;
    int left;

    __device__ __attribute__((always_inline)) void block(uint32_t a, uint32_t b, uint32_t stream, uint32_t k0,
                                                         uint32_t k1, bool fill)
    {
        if (fill) {
            const uint32_t ql = threadIdx.x & 3u;
            const U4 r = philox4x32_10_uk(U4{a, b, (draw & ~3u) + ql, stream}, k0, k1);
            *reinterpret_cast<uint4 *>(buf + 4u * ql) = make_uint4(r.x, r.y, r.z, r.w);
            // (lanes of one wave: LDS operations complete in order)
            __builtin_amdgcn_wave_barrier();
        }
        const uint4 v = *reinterpret_cast<const uint4 *>(buf + 4u * (draw & 3u));
        q0 = v.x;
        q1 = v.y;
        q2 = v.z;
        q3 = v.w;
        ++draw;
    }
    // continue a stream at block draw_ with left_ numbers of the block before it to come
    __device__ void resume(uint32_t draw_, int left_, uint32_t a, uint32_t b, uint32_t stream, uint32_t k0, uint32_t k1)
    {
        draw = draw_;
        left = left_;
        if (left_ > 0) --draw;
        if (left_ > 0 || (draw & 3u)) {
            const uint32_t at = draw;
            block(a, b, stream, k0, k1, true);
            draw = at + (left_ > 0 ? 1u : 0u);
            for (int k = left_ > 0 ? left_ : 4; k < 4; ++k) {
                q0 = q1;
                q1 = q2;
                q2 = q3;
            }
        }
    }
    __device__ __attribute__((always_inline)) void need(int k, uint32_t a, uint32_t b, uint32_t stream, uint32_t k0,
                                                        uint32_t k1)
    {
        if (left < k) {
            block(a, b, stream, k0, k1, (draw & 3u) == 0u);
            left = 4;
        }
    }
    __device__ void skip(int k) { left = left < k ? 0 : left; }
    __device__ float take()
    {
        const uint32_t v = q0;
        q0 = q1; q1 = q2; q2 = q3;
        --left;
        return (float)(v >> 8) * 5.9604644775390625e-08f;
    }
    __device__ float take_exp1() { return neg_log_unit(1.0f - take()); }
};

// ---------------------------------------------------------------------------
// Matrix-core fragments.  For v_mfma_f32_16x16x16_bf16, lane l (0..63) holds
//   A[m][k] for m = l % 16, k = 4 (l / 16) + i  (i = 0..3),
//   B[k][n] for n = l % 16, k = 4 (l / 16) + i,
//   D[m][n] for n = l % 16, m = 4 (l / 16) + i.
// ---------------------------------------------------------------------------
typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ inline short to_bf16(float x)
{
    // round to nearest even (v_cvt_pk_bf16_f32 on gfx950; the same bits as
    // adding 0x7fff plus the kept low bit, for every finite x)
    return __builtin_bit_cast(short, (__bf16)x);
}

__device__ inline float from_bf16(short h) { return __uint_as_float(((uint32_t)(uint16_t)h) << 16); }

__device__ inline f32x4 mfma16(bf16x4 a, bf16x4 b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}

// v_mfma_f32_16x16x32_bf16 (gfx950): as above with eight k values per lane,
// A[m][k] and B[k][n] from lane group l / 16 and element e alike, and the same
// D layout.  Callers only rely on A and B pairing lane group and element the
// same way (the order of k within a product is free).
typedef short bf16x8 __attribute__((ext_vector_type(8)));

__device__ inline f32x4 mfma32(bf16x8 a, bf16x8 b, f32x4 c)
{
    typedef __bf16 bf16v8 __attribute__((ext_vector_type(8)));
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16v8, a), __builtin_bit_cast(bf16v8, b), c, 0,
                                                   0, 0);
}

}  // namespace nc
