// nc_flux.hip -- forward photons: ground transmissivity under the field and
// its parametric sensitivities (Section 5.1), with the derivative-path
// (adjoint) replay.
//
// The sun lights the top of the box uniformly; photons start at a uniform
// point of the top face going along -omega_sun, are tracked by delta
// tracking in the grid's piecewise-constant majorant with analog absorption
// and HG scattering, and arrive at the ground, where an arrival inside the
// box's footprint is tallied in its ground pixel before a Lambertian
// reflection (probability rho) or absorption.
//
// Sensitivities follow the derivative of the integral formulation (Eq. 3):
// with k = s k_c + k_g and a majorant held fixed, every tentative collision
// multiplies the path density by k/k_hat (real) or 1 - k/k_hat (null), so a
// path carries the score
//   sigma_s = sum_real k_c/k - sum_null k_c/(k_hat - k) + sum_scatter k_g/(s k)
// (the last term is d ln ssa(x)/ds), every HG scattering of cosine mu adds
//   sigma_g += d ln p(mu)/dg = -2g/(1-g^2) - 3(g-mu)/(1+g^2-2g mu),
// and every scattering adds d ln ssa(x)/d alpha = -1/(1 - alpha) to the
// score of the droplets' absorptivity alpha = 1 - ssa (the sensitivity the
// paper computes in Section 5.1).  Absorbed photons arrive nowhere, so the
// absorption events need no term.
// The derivative of a tally is the mean of (tally) x sigma.  The adjoint
// replay re-runs the same photons (same counter-based random numbers) and
// accumulates grad[pixel] x sigma at each arrival.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "nc_internal.hpp"

namespace nc {

struct FluxArgs {
    GridView g;
    OptView op;
    int px_nx, px_ny;
    float x0, y0, Lx, Ly, ztop;
    unsigned long long n_photons;
    uint64_t seed, offset;
    double *tally;          // [9][px_ny][px_nx] (forward) or NULL
    double *glob;           // [4] (forward) or NULL
    const double *grad;     // [px_ny][px_nx] (adjoint) or NULL
    double *out;            // [3] (adjoint) or NULL
    double norm;            // factor of every arrival: 1, or px_nx px_ny / n_photons (normalised output)
    nc_counters *counters;
    unsigned long long *queue;   // 8 queue heads, 16 words apart (null: every wave has one chunk, its own)
    unsigned long long span;     // photons per queue
    int lds_first, lds_nodes, ring_lds;
    uint32_t *tail;              // photons handed to the tail kernel: word w of photon i at [w tail_cap + i] (null: none are)
    unsigned int *tail_count;
    uint32_t tail_cap;
    int tail_lanes;
};

__device__ inline float hg_dlng(float g, float mu)
{
    return -2.0f * g / (1.0f - g * g) - 3.0f * (g - mu) / (1.0f + g * g - 2.0f * g * mu);
}

// An arrival at ground pixel q: its tallies, or its term of the adjoint sums.
template <bool kAdjoint>
__device__ inline void tally_arrival(const FluxArgs &A, size_t np, size_t q, bool scattered, float sig_s, float sig_g,
                                     float sig_a, double &adj_s, double &adj_g, double &adj_a)
{
    if (kAdjoint) {
        const double w = A.grad[q] * A.norm;
        adj_s += w * (double)sig_s;
        adj_g += w * (double)sig_g;
        adj_a += w * (double)sig_a;
    } else {
        const double f = A.norm, f2 = f * f;
        unsafeAtomicAdd(A.tally + q, f);
        unsafeAtomicAdd(A.tally + np + q, f2);
        if (!scattered) unsafeAtomicAdd(A.tally + 2 * np + q, f);
        unsafeAtomicAdd(A.tally + 3 * np + q, f * (double)sig_s);
        unsafeAtomicAdd(A.tally + 4 * np + q, f2 * (double)sig_s * (double)sig_s);
        unsafeAtomicAdd(A.tally + 5 * np + q, f * (double)sig_g);
        unsafeAtomicAdd(A.tally + 6 * np + q, f2 * (double)sig_g * (double)sig_g);
        unsafeAtomicAdd(A.tally + 7 * np + q, f * (double)sig_a);
        unsafeAtomicAdd(A.tally + 8 * np + q, f2 * (double)sig_a * (double)sig_a);
    }
}

// A wave's totals: the photons that ended each way (wave-uniform), or the lanes' adjoint sums.
template <bool kAdjoint>
__device__ inline void flux_totals(const FluxArgs &A, int up, int gin, int gout, int vabs, double s, double t, double u)
{
    if (kAdjoint) {
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            s += __shfl_xor(s, off);
            t += __shfl_xor(t, off);
            u += __shfl_xor(u, off);
        }
        if (__lane_id() == 0) {
            unsafeAtomicAdd(A.out, s);
            unsafeAtomicAdd(A.out + 1, t);
            unsafeAtomicAdd(A.out + 2, u);
        }
    } else if (__lane_id() == 0) {
        if (up) unsafeAtomicAdd(A.glob, (double)up);
        if (gin) unsafeAtomicAdd(A.glob + 1, (double)gin);
        if (gout) unsafeAtomicAdd(A.glob + 2, (double)gout);
        if (vabs) unsafeAtomicAdd(A.glob + 3, (double)vabs);
    }
}

// Words of a photon handed to the tail kernel.
enum FluxWord { kFwFlags = 0, kFwHead, kFwId0, kFwId1, kFwSegs, kFwFloats = 5, kFwAxes = 15, kFwEnd = 24 };
static_assert(kFwEnd <= kTailWords, "a photon fits its words");

// Photons by phases, like the renderer's paths (render_kernel): a lane holds one
// photon and each trip the wave runs the phase most lanes wait in (a voxel
// crossing or a ray's first voxel, a tentative collision, an event, a new
// photon); lanes whose photon has ended take the next one of the queue.
// Bound by vector instruction issue at the lanes in use: a photon per thread,
// its loops nested, kept a wave until its longest photon ended.  10^7 photons
// over the 256^3 cylinder and 100 x 100 pixels, forward and adjoint: 62.0 ms
// that way, 9.4 ms here (with the tail kernel).
// At the end of the queue, and in small calls, what is left is the longest
// photon's serial chain: waves with few photons hand them to flux_tail_kernel.
template <bool kAdjoint>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(6))) void flux_kernel(FluxArgs A)
{
    extern __shared__ __align__(16) float2 s_nodes[];
    __shared__ int s_off[NC_MAX_LEVELS + 2];
    __shared__ int4 s_rows[NC_MAX_LEVELS + 2];
    __shared__ unsigned long long s_cnt[kNumBlockCounters];
    for (int i = threadIdx.x; i < kNumBlockCounters; i += blockDim.x) s_cnt[i] = 0ull;
    stage_levels(A.g, A.lds_first, A.lds_nodes, s_nodes, s_off, s_rows);
    const GridView &g = A.g;
    const NodeSrc ns{g.nodes, s_nodes, s_off, A.lds_first, s_off[A.lds_first <= g.L ? A.lds_first : 0], g.n[0],
                     g.n[1], s_rows};
    const size_t np = (size_t)A.px_nx * A.px_ny;
    const bool stats = A.counters != nullptr;
    unsigned long long *const cnt = stats ? s_cnt : nullptr;
    const float dln_alpha = A.op.ssa > 0.0f ? -1.0f / A.op.ssa : 0.0f;
    const uint32_t key0 = (uint32_t)A.seed, key1 = (uint32_t)(A.seed >> 32);

    int up = 0, gin = 0, gout = 0, vabs = 0;      // wave-uniform: photons that ended each way
    double adj_s = 0.0, adj_g = 0.0, adj_a = 0.0;
    int phase = kPhSample, res = kContinue, segs = 0;
    uint32_t id0 = 0, id1 = 0;                    // the lane's photon (its random stream)
    bool live = false, scattered = false;
    float sig_s = 0.0f, sig_g = 0.0f, sig_a = 0.0f;
    float kc_hit = 0.0f, tau = 0.0f;
    float pd[3] = {0.0f, 0.0f, 0.0f};             // direction of the next ray
    Ray r;                                        // at an event, r.o is the next ray's origin
    RngRing rng;
    rng.q = reinterpret_cast<uint32_t *>(reinterpret_cast<char *>(s_nodes) + A.ring_lds) +
            (threadIdx.x >> 6) * RngRing::kWordsPerWave + (threadIdx.x & 63u);
    rng.reset();
    // the wave's chunk of photons: without a queue its own 64, once
    const unsigned long long wave = blockIdx.x * (unsigned long long)(blockDim.x >> 6) + (threadIdx.x >> 6);
    unsigned long long chunk_base = wave * kChunk;
    int chunk_left = A.queue ? 0 : kChunk;
    bool drained = !A.queue;
    int q_seen = 0;

    for (;;) {
        const int n_step = lane_count((phase == kPhCross) | (phase == kPhRay));
        const int n_coll = lane_count(phase == kPhCollide);
        const int n_event = lane_count(phase == kPhEvent);
        const int n_sample = lane_count(phase == kPhSample);
        const int n_all = n_step + n_coll + n_event + n_sample;
        if (n_all == 0) break;
        int run = kPhCross, best = n_step;
        if (n_coll >= best) { run = kPhCollide; best = n_coll; }
        if (n_event >= best) { run = kPhEvent; best = n_event; }
        if (n_sample > best) { run = kPhSample; best = n_sample; }
        if (A.tail && drained && n_all <= A.tail_lanes) {
            // the last photons of the wave go to the tail kernel
            const bool going = phase < kPhSample;
            const unsigned long long m = __ballot(going);
            if (m) {
                unsigned int base = 0;
                if (__lane_id() == 0) base = atomicAdd(A.tail_count, (unsigned int)__popcll(m));
                base = __shfl(base, 0);
                if (going) {
                    uint32_t *p = A.tail + base + lanes_below(m);
                    auto put = [&](uint32_t v) {
                        *p = v;
                        p += A.tail_cap;
                    };
                    // (before a photon's first voxel its mask and level hold anything: masked)
                    put((uint32_t)(phase | (scattered ? 8 : 0) | (res << 4) | ((r.xmask & 7) << 8) | ((r.lev & 0xff) << 12)));
                    put(rng.head);
                    put(id0);
                    put(id1);
                    put((uint32_t)segs);
                    const float f[] = {sig_s, sig_g, sig_a, tau, kc_hit, r.t, r.tend, r.texit, r.khat, r.kmin};
#pragma unroll
                    for (int k = 0; k < 10; ++k) put(__float_as_uint(f[k]));
#pragma unroll
                    for (int a = 0; a < 3; ++a) {
                        put(__float_as_uint(r.o[a]));
                        put(__float_as_uint(r.d[a]));
                        // a ray's first cell, later the cell past its voxel: only one of them is live
                        put((uint32_t)(phase == kPhRay ? r.c[a] : r.cn[a]));
                    }
                    phase = kPhIdle;
                    live = false;
                }
                continue;
            }
        }
        const bool run_step = run == kPhCross, run_coll = run == kPhCollide;
        const bool run_event = run == kPhEvent, run_sample = run == kPhSample;
        bool start = false;   // the lane starts a ray from r.o along pd at the end of this trip

        if (run_sample) {
            // ---- the next photon, if any is left
            if (stats) wave_count(cnt, kCPaths, phase == kPhSample && live);
            const bool want = phase == kPhSample;
            const unsigned long long need = __ballot(want);
            const int n_need = __popcll(need);
            const int rank = (int)lanes_below(need);
            const int more = n_need - chunk_left;
            unsigned long long nb = A.n_photons;
            if (more > 0 && !drained) {
                // the XCD's own queue first, then the others
                const int leader = __ffsll((unsigned long long)need) - 1;
                if ((int)__lane_id() == leader) {
                    for (;;) {
                        const int q = (int)((blockIdx.x + (unsigned)q_seen) & 7u);
                        const unsigned long long lo = (unsigned long long)q * A.span;
                        const unsigned long long hi = lo + A.span < A.n_photons ? lo + A.span : A.n_photons;
                        const unsigned long long b = lo + atomicAdd(A.queue + 16 * q, (unsigned long long)kChunk);
                        if (b < hi) { nb = b; break; }
                        if (++q_seen == 8) break;
                    }
                }
                nb = __shfl(nb, leader);
                q_seen = __shfl(q_seen, leader);
                if (nb >= A.n_photons) drained = true;
            }
            if (want) {
                const unsigned long long p = rank < chunk_left ? chunk_base + (unsigned long long)rank
                                                               : nb + (unsigned long long)(rank - chunk_left);
                live = p < A.n_photons;
                phase = live ? kPhSample : kPhIdle;
                const unsigned long long id = A.offset + p;
                id0 = (uint32_t)id;
                id1 = (uint32_t)(id >> 32);
                rng.reset();
            }
            if (more > 0) {
                chunk_base = nb + (unsigned long long)more;
                chunk_left = nb < A.n_photons ? kChunk - more : 0;
            } else {
                chunk_base += (unsigned long long)n_need;
                chunk_left -= n_need;
            }
        }
        {
            // the phase's numbers: a collision takes two, a new photon or an event up to four
            const bool in_run = live & (phase == run);
            const uint32_t k = run == kPhCross ? 0u : run == kPhCollide ? 2u : 4u;
            while (__ballot(in_run && !rng.holds(k)))
                if (live && rng.space()) rng.fill(id0, id1, 2u, key0, key1);
        }
        if (run_sample && phase == kPhSample) {
            // ---- a photon enters through a uniform point of the top face
            r.o[0] = A.x0 + rng.take() * A.Lx;
            r.o[1] = A.y0 + rng.take() * A.Ly;
            r.o[2] = A.ztop;
#pragma unroll
            for (int a = 0; a < 3; ++a) pd[a] = -A.op.sun[a];
            sig_s = sig_g = sig_a = 0.0f;
            scattered = false;
            segs = 0;
            start = true;
        }
        if (run_event) {
            // ---- a real collision: absorption or scattering; the ray left the
            // box: at the ground a tally, then reflection or absorption
            bool e_up = false, e_in = false, e_out = false, e_abs = false;
            if (phase == kPhEvent) {
                phase = kPhSample;
                if (res == kReal) {
                    const float kd = g.kscale * kc_hit;
                    const float k = kd + g.k_gas;
                    const float ssa = A.op.ssa * kd / k;
                    e_abs = rng.take() >= ssa;
                    if (!e_abs) {
#pragma unroll
                        for (int a = 0; a < 3; ++a) {
                            pd[a] = r.d[a];
                            r.o[a] = r.o[a] + r.t * r.d[a];
                        }
                        if (g.k_gas > 0.0f) sig_s += g.k_gas / (g.kscale * k);
                        sig_a += dln_alpha;
                        const float mu = hg_sample_mu(A.op.hg, rng.take());
                        sig_g += hg_dlng(A.op.g, mu);
                        turn(pd, mu, rng.take());
                        start = true;
                    }
                } else if (r.d[2] < 0.0f) {
                    const float tg = -r.o[2] / r.d[2];
                    r.o[0] = r.o[0] + tg * r.d[0];
                    r.o[1] = r.o[1] + tg * r.d[1];
                    r.o[2] = 0.0f;
                    const float fx = (r.o[0] - A.x0) / A.Lx, fy = (r.o[1] - A.y0) / A.Ly;
                    const bool inside = fx >= 0.0f && fx < 1.0f && fy >= 0.0f && fy < 1.0f;
                    if (inside) {
                        const int i = min((int)(fx * (float)A.px_nx), A.px_nx - 1);
                        const int j = min((int)(fy * (float)A.px_ny), A.px_ny - 1);
                        tally_arrival<kAdjoint>(A, np, (size_t)j * A.px_nx + i, scattered, sig_s, sig_g, sig_a, adj_s, adj_g,
                                                adj_a);
                    }
                    if (rng.take() >= A.op.rho) {
                        e_in = inside;
                        e_out = !inside;
                    } else {
                        const float u1 = rng.take(), u2 = rng.take();
                        lambert(pd, u1, u2);
                        start = true;
                    }
                } else {
                    e_up = true;
                }
                scattered |= start;
            }
            if (!kAdjoint) {
                up += lane_count(e_up);
                gin += lane_count(e_in);
                gout += lane_count(e_out);
                vabs += lane_count(e_abs);
            }
        }
        if (run_sample || run_event) {
            // ---- rays started by this trip's photons and events
            if (start) {
                const float o[3] = {r.o[0], r.o[1], r.o[2]}, d[3] = {pd[0], pd[1], pd[2]};
                phase = kPhRay;
                if (!ray_setup(g, r, o, d, 0.0f)) {
                    // misses the box: the next step finds the ray outside
                    r.t = r.tend = r.texit = 0.0f;
                    r.khat = 0.0f;
                    r.kmin = 0.0f;
                    r.lev = g.L;
                    phase = kPhCross;
                }
                tau = rng.take_exp1();
            }
        }
        if (run_step) {
            // ---- across the voxel's exit face, or into a ray's first voxel
            const bool crossing = phase == kPhCross;
            bool locate = phase == kPhRay, trunc = false;
            if (crossing) {
                tau -= r.khat * (r.texit - r.t);
                ++segs;
                locate = step_cell(g, r);
                res = kExit;
                phase = locate ? phase : kPhEvent;
            }
            uint32_t nr = 0;
            if (locate) {
                locate_voxel(g, ns, r, A.op.mscale, nr);
                leaf_exit(g, r);
                phase = voxel_phase(r, tau);
                if (crossing && segs >= A.op.max_segments) {
                    trunc = true;
                    phase = kPhSample;      // stop the photon
                }
            }
            if (stats) {
                wave_count(cnt, kCReads, locate);
                if (g.L >= 1) wave_count(cnt, kCReads, locate);
                wave_count(cnt, kCReads, locate && r.lev >= 1 && r.lev < ns.lds_first);
                wave_count(cnt, kCSegments, crossing);
                wave_count(cnt, kCLeaf, locate);
                wave_count(cnt, kCTrunc, trunc);
            }
        }
        if (run_coll) {
            // ---- a tentative collision, with its term of the scale score
            const bool active = phase == kPhCollide;
            bool real = false, gathered = false, trunc = false;
            if (active) {
                r.t = fminf(r.t + tau / r.khat, r.texit);
                const float thr = rng.take() * r.khat;
                kc_hit = r.kmin;
                gathered = r.lev != 0;
                if (gathered) kc_hit = collision_k(g, r, r.t);
                const float k = g.kscale * kc_hit + g.k_gas;
                ++segs;
                real = thr < k;
                sig_s += real ? kc_hit / k : -(kc_hit / (r.khat - k));
                if (real) {
                    res = kReal;
                    phase = kPhEvent;
                } else {
                    tau = rng.take_exp1();
                    phase = voxel_phase(r, tau);
                    if (segs >= A.op.max_segments) {
                        trunc = true;
                        phase = kPhSample;
                    }
                }
            }
            if (stats) {
                wave_count(cnt, kCSegments, active);
                wave_count(cnt, kCTentative, active);
                wave_count(cnt, kCReals, real);
                wave_count(cnt, kCNulls, active && !real);
                wave_count(cnt, kCGathers, gathered);
                wave_count(cnt, kCTrunc, trunc);
            }
        }
    }
    flux_totals<kAdjoint>(A, up, gin, gout, vabs, adj_s, adj_g, adj_a);
    if (!stats) return;
    __syncthreads();
    if (threadIdx.x < 10) {
        unsigned long long *o = reinterpret_cast<unsigned long long *>(A.counters);
        if (s_cnt[threadIdx.x]) atomicAdd(o + threadIdx.x, s_cnt[threadIdx.x]);
    }
}

// The last photons of a flux call, each on four lanes (QuadRay), as in
// render_tail_kernel: bound by the instructions of the longest photon's chain.
// 200 k photons over 128 x 128 x 40 cells and a reflecting ground: 8.3 ms with a
// photon per thread, 10.3 ms by phases alone (all of them in each trip of a wave
// with few photons), 5.4 ms with this kernel.
template <bool kAdjoint>
__global__ __launch_bounds__(256) void flux_tail_kernel(FluxArgs A)
{
    extern __shared__ __align__(16) float2 s_nodes[];
    __shared__ int s_off[NC_MAX_LEVELS + 2];
    __shared__ int4 s_rows[NC_MAX_LEVELS + 2];
    __shared__ __align__(16) uint32_t s_rng[4 * 16 * 16];
    const unsigned int count = *A.tail_count;
    const unsigned int waves = gridDim.x * 4u, wave = blockIdx.x * 4u + (threadIdx.x >> 6);
    if (blockIdx.x * 4u >= count) return;   // (workgroup-uniform)
    stage_levels(A.g, A.lds_first, A.lds_nodes, s_nodes, s_off, s_rows);   // ends with a block barrier
    const NodeSrc ns{A.g.nodes, s_nodes, s_off, A.lds_first, 0, A.g.n[0], A.g.n[1], s_rows};
    QuadGrid G;
    G.init(A.g, s_rows);
    const int ax = G.ax, quad = (int)(__lane_id() >> 2);
    const bool first_lane = G.ql == 0;
    const size_t np = (size_t)A.px_nx * A.px_ny;
    const float dln_alpha = A.op.ssa > 0.0f ? -1.0f / A.op.ssa : 0.0f;
    const uint32_t key0 = (uint32_t)A.seed, key1 = (uint32_t)(A.seed >> 32);
    const HGc &hg = A.op.hg;
    int up = 0, gin = 0, gout = 0, vabs = 0;
    double adj_s = 0.0, adj_g = 0.0, adj_a = 0.0;
    // the wave's photons: wave, wave + waves, ...; a quad whose photon has ended takes its next one
    unsigned long long i = wave + (unsigned long long)quad * waves;
    {
        QuadRay r;
        RngQuad rng;
        rng.buf = s_rng + (threadIdx.x >> 2) * 16u;
        int phase = kPhSample, res = 0, segs = 0;
        uint32_t id0 = 0, id1 = 0;
        bool scattered = false, e_up = false, e_in = false, e_out = false, e_abs = false;
        float sig_s = 0.0f, sig_g = 0.0f, sig_a = 0.0f, tau = 0.0f, kc_hit = 0.0f;
        r.vc = -1;
        r.vlev = 0;
        r.vkmin = r.vkhat = 0.0f;
        auto u01 = [&]() __attribute__((always_inline)) {
            rng.need(1, id0, id1, 2u, key0, key1);
            return rng.take();
        };
        auto enter = [&]() __attribute__((always_inline)) {
            r.enter(G);
            phase = ((r.khat > 0.0f) & (tau < r.khat * (r.texit - r.t))) ? kPhCollide : kPhCross;
        };
        auto ray_start = [&](float dir) __attribute__((always_inline)) {
            const bool hit = r.setup(G, dir);
            tau = neg_log_unit(1.0f - u01());
            if (hit) {
                r.first_voxel(A.g, G, ns, A.op.mscale);
                enter();
            } else {
                // misses the box: the next step finds the ray outside
                r.t = r.tend = r.texit = 0.0f;
                r.khat = 0.0f;
                r.kmin = 0.0f;
                r.lev = 0;
                phase = kPhCross;
            }
        };
        auto take_photon = [&]() __attribute__((always_inline)) {
            const uint32_t *w = A.tail + i;
            i += 16ull * waves;
            r.vc = -1;
            r.vlev = 0;
            const size_t cap = A.tail_cap;
            auto get_u = [&](int k) { return w[(size_t)k * cap]; };
            auto get_f = [&](int k) { return __uint_as_float(w[(size_t)k * cap]); };
            const int fl = (int)get_u(kFwFlags);
            phase = fl & 7;
            scattered = (fl & 8) != 0;
            res = (fl >> 4) & 3;
            r.lev = (fl >> 12) & 0xff;
            id0 = get_u(kFwId0);
            id1 = get_u(kFwId1);
            segs = (int)get_u(kFwSegs);
            sig_s = get_f(kFwFloats);
            sig_g = get_f(kFwFloats + 1);
            sig_a = get_f(kFwFloats + 2);
            tau = get_f(kFwFloats + 3);
            kc_hit = get_f(kFwFloats + 4);
            r.t = get_f(kFwFloats + 5);
            r.tend = get_f(kFwFloats + 6);
            r.texit = get_f(kFwFloats + 7);
            r.khat = get_f(kFwFloats + 8);
            r.kmin = get_f(kFwFloats + 9);
            r.o = get_f(kFwAxes + 3 * ax);
            r.d = get_f(kFwAxes + 3 * ax + 1);
            r.c = (int)get_u(kFwAxes + 3 * ax + 2);
            {
                const float d3[3] = {r.d, r.d, r.d};
                float inv3[3];
                ray_inverse(d3, inv3);
                r.inv = inv3[0];
            }
            const uint32_t head = get_u(kFwHead);
            rng.resume((head + 3u) >> 2, (int)((0u - head) & 3u), id0, id1, 2u, key0, key1);
            if (phase == kPhRay) {
                r.locate(A.g, G, ns, A.op.mscale);
                enter();
            } else {
                // a cell of the current voxel from the one past it
                if ((fl >> (8 + ax)) & 1) r.c -= r.d > 0.0f ? 1 : -1;
                r.faces(G);
            }
        };
        // (one loop, in which every photon of the wave takes its next step)
        for (;;) {
            if (phase == kPhSample) {
                if (first_lane) {
                    up += e_up;
                    gin += e_in;
                    gout += e_out;
                    vabs += e_abs;
                }
                e_up = e_in = e_out = e_abs = false;
                phase = kPhIdle;
                if (i < count) take_photon();
            }
            if (!__ballot(phase < kPhSample)) break;
            if (phase == kPhEvent) {
                phase = kPhSample;
                if (res == kReal) {
                    const float kd = A.g.kscale * kc_hit;
                    const float k = kd + A.g.k_gas;
                    const float ssa = A.op.ssa * kd / k;
                    e_abs = u01() >= ssa;
                    if (!e_abs) {
                        r.keep_voxel();
                        r.o = r.o + r.t * r.d;
                        if (A.g.k_gas > 0.0f) sig_s += A.g.k_gas / (A.g.kscale * k);
                        sig_a += dln_alpha;
                        const float mu = hg_sample_mu(hg, u01());
                        sig_g += hg_dlng(A.op.g, mu);
                        float v[3] = {quad_axis<0>(r.d), quad_axis<1>(r.d), quad_axis<2>(r.d)};
                        turn(v, mu, u01());
                        scattered = true;
                        ray_start(quad_pick(ax, v[0], v[1], v[2]));
                    }
                } else {
                    const float dz = quad_axis<2>(r.d);
                    if (dz < 0.0f) {
                        const float tg = -quad_axis<2>(r.o) / dz;
                        r.o = ax == 2 ? 0.0f : r.o + tg * r.d;
                        const float x = quad_axis<0>(r.o), y = quad_axis<1>(r.o);
                        const float fx = (x - A.x0) / A.Lx, fy = (y - A.y0) / A.Ly;
                        const bool inside = fx >= 0.0f && fx < 1.0f && fy >= 0.0f && fy < 1.0f;
                        if (inside & first_lane) {
                            const int pi = min((int)(fx * (float)A.px_nx), A.px_nx - 1);
                            const int pj = min((int)(fy * (float)A.px_ny), A.px_ny - 1);
                            tally_arrival<kAdjoint>(A, np, (size_t)pj * A.px_nx + pi, scattered, sig_s, sig_g, sig_a, adj_s,
                                                    adj_g, adj_a);
                        }
                        if (u01() >= A.op.rho) {
                            e_in = inside;
                            e_out = !inside;
                        } else {
                            float v[3];
                            const float u1 = u01(), u2 = u01();
                            lambert(v, u1, u2);
                            scattered = true;
                            ray_start(quad_pick(ax, v[0], v[1], v[2]));
                        }
                    } else {
                        e_up = true;
                    }
                }
            }
            if (phase == kPhCross) {
                tau -= r.khat * (r.texit - r.t);
                ++segs;
                r.t = r.texit;
                res = kExit;
                phase = kPhEvent;
                if (r.t < r.tend) {
                    r.next_cell(G);
                    r.locate(A.g, G, ns, A.op.mscale);
                    enter();
                    if (segs >= A.op.max_segments) phase = kPhSample;      // stop the photon
                }
            }
            if (phase == kPhCollide) {
                r.t = fminf(r.t + tau / r.khat, r.texit);
                const float thr = u01() * r.khat;
                kc_hit = r.kmin;
                if (r.lev != 0) kc_hit = r.k_at(A.g, G);
                const float k = A.g.kscale * kc_hit + A.g.k_gas;
                ++segs;
                if (thr < k) {
                    sig_s += kc_hit / k;
                    res = kReal;
                    phase = kPhEvent;
                } else {
                    sig_s -= kc_hit / (r.khat - k);
                    tau = neg_log_unit(1.0f - u01());
                    phase = ((r.khat > 0.0f) & (tau < r.khat * (r.texit - r.t))) ? kPhCollide : kPhCross;
                    if (segs >= A.op.max_segments) phase = kPhSample;
                }
            }
        }
    }
    if (!kAdjoint) {
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            up += __shfl_xor(up, off);
            gin += __shfl_xor(gin, off);
            gout += __shfl_xor(gout, off);
            vabs += __shfl_xor(vabs, off);
        }
    }
    flux_totals<kAdjoint>(A, up, gin, gout, vabs, adj_s, adj_g, adj_a);
}

hipError_t launch_flux(const nc_ctx *ctx, const nc_grid *g, const float *d_kc, const OptView &op, float kscale,
                       int px_nx, int px_ny, unsigned long long n_photons, const nc_sampling &s, double *tally,
                       double *glob, const double *grad, double *out, nc_counters *counters)
{
    const size_t ring_bytes = sizeof(uint32_t) * 4 * RngRing::kWordsPerWave;   // 4 waves per workgroup
    Shape sh = choose_shape(ctx, g, 256, ring_bytes);
    FluxArgs A;
    A.g = grid_view(g, d_kc);
    A.g.kscale = kscale;
    A.op = op;
    A.px_nx = px_nx;
    A.px_ny = px_ny;
    A.x0 = (float)g->lo[0];
    A.y0 = (float)g->lo[1];
    A.Lx = (float)(g->n[0] * g->h[0]);
    A.Ly = (float)(g->n[1] * g->h[1]);
    A.ztop = (float)(g->lo[2] + g->n[2] * g->h[2]);
    A.n_photons = n_photons;
    A.seed = s.seed;
    A.offset = s.sample_offset;
    A.tally = tally;
    A.glob = glob;
    A.grad = grad;
    A.out = out;
    A.norm = (s.flags & NC_FLUX_NORMALISE) ? (double)px_nx * (double)px_ny / (double)n_photons : 1.0;
    A.counters = counters;
    A.lds_first = sh.lds_first;
    A.lds_nodes = sh.lds_nodes;
    const size_t node_bytes = ((size_t)sh.lds_nodes * sizeof(float2) + 15) & ~(size_t)15;
    A.ring_lds = (int)node_bytes;
    const size_t lds = node_bytes + ring_bytes;
    const void *fn = grad ? (const void *)flux_kernel<true> : (const void *)flux_kernel<false>;
    int resident = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&resident, fn, 256, lds) == hipSuccess && resident > 0)
        sh.wgs = ctx->num_cus * resident;
    const unsigned long long blocks = (n_photons + 255) / 256;
    const int wgs = (int)std::max<unsigned long long>(1, std::min<unsigned long long>(blocks, (unsigned long long)sh.wgs));
    // a photon per lane needs no queue
    unsigned long long *const heads = ctx->d_scratch + kScratchQueues;
    A.queue = nullptr;
    A.span = 0;
    if (blocks > (unsigned long long)wgs) {
        A.queue = heads;
        A.span = (n_photons + 8 * kChunk - 1) / (8 * kChunk) * kChunk;
    }
    // the last photons (not where statistics are kept or on a grid too large for the tail kernel's arithmetic)
    const TailShape ts = tail_shape(n_photons, (long long)wgs * 4, kTailPhotons);
    A.tail_lanes = ts.lanes;
    A.tail = !counters && A.g.narrow && ts.lanes > 0
                 ? reinterpret_cast<uint32_t *>(ctx->d_scratch + kScratchWords)
                 : nullptr;
    A.tail_count = reinterpret_cast<unsigned int *>(heads + 8);   // in the first queue head's line, zeroed with it
    A.tail_cap = kTailCap;
    if (A.queue || A.tail) launch_zero_u64(ctx, heads, 128);
    void *args[] = {&A};
    const hipError_t e = hipLaunchKernel(fn, dim3(wgs), dim3(256), args, lds, ctx->stream);
    if (e != hipSuccess || !A.tail) return e;
    return hipLaunchKernel(grad ? (const void *)flux_tail_kernel<true> : (const void *)flux_tail_kernel<false>,
                           dim3((ts.waves + 3) / 4), dim3(256), args, node_bytes, ctx->stream);
}

}  // namespace nc
