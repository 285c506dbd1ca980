// Ray traversal kernels for gfx950: camera rays (closest hit into the G-buffer) and shadow
// rays (any hit) towards point lights or rectangular-light samples.
//
// Persistent waves: each 64-lane wave keeps its lanes busy from a device work counter.
// A lane owns one work item (a camera sample, or a shaded point with its list of shadow
// rays); when enough lanes of a wave have finished, the idle lanes are refilled together
// (ballot of idle lanes, one atomicAdd for the wave, prefix count for the lane's slot),
// which regroups live rays into full waves without moving ray state.
//
// Traversal: 4-wide BVH, all child boxes of a node in one 128-byte record; ray/box slab
// tests with the octant-selected near/far planes and a conservative far distance; ordered
// descent (nearest child first) for closest hits; per-lane stack of (node, entry distance)
// in LDS with a lane-interleaved global overflow area.  Triangles: Moller-Trumbore in FP32.
#include <algorithm>
#include <cmath>

#include "rc_wave.h"

namespace {

constexpr int BLOCK = RC_TRACE_BLOCK;
constexpr int SL = RC_STACK_LDS;
constexpr int REFILL_AT = 40;    // refill once a wave has at most this many busy lanes
constexpr uint32_t ITEM_CHUNK = 256;
constexpr uint32_t RECT_CHUNK = 64;   // packets per chunk dealt to one XCD

enum { MODE_PRIMARY = 0, MODE_POINT = 1, MODE_RECT = 2 };

struct KParams {
    DevScene sc;
    DevCamera cam;
    DevLights L;
    float nL[3];              // unit normal of the rect light (emitting side)
    uint4* gbuf_out;
    const uint4* gbuf_in;
    uint32_t* mask;
    float* vis;
    const float4* setup;      // shadow rays: per sample (origin, 1 | 0 without a hit) and (normal, 0), k_shadow_setup
    TraceWork w;
    uint32_t n_items;
    uint32_t slot;
    uint32_t claim;           // work positions a wave claims with one atomic (set by the launcher)
    uint32_t light_groups;    // k_trace<point>: work units per sample (1: all lights in turn; n_point: one each)
};

// Positions per claim: large enough that the atomics stay few, small enough that every wave makes about
// `per_wave` claims, so that the last claims of the waves end close together.
inline uint32_t claim_size(uint64_t n_work, int grid, uint32_t per_wave, uint32_t lo, uint32_t hi)
{
    uint64_t waves = (uint64_t)grid * (BLOCK / 64);
    uint64_t c = n_work / (waves * per_wave);
    return (uint32_t)std::min<uint64_t>(hi, std::max<uint64_t>(lo, c));
}

// Waves per SIMD: 6 for flat-tree camera rays (80 registers; 3% faster than 5), 5 for two-level structures (96; their
// camera rays at 720p 0.265 ms against 0.283 at the natural 4 and 0.293 at 6, on 1.1M triangles; their point-light shadow
// rays at 5 / 4 within 3% of each other from 0.5M samples on and 3 to 7% slower at 0.23M, which go four lanes to a ray
// by default: 1.1M triangles, 4 lights, 640x360 0.39 / 0.40, 960x540 0.61 / 0.63, 1080p 1.56 / 1.58 ms; 7.3M 0.51 / 0.50, 0.70 /
// 0.70, 1.85 / 1.88), the compiler's choice elsewhere (flat shadow rays at 6: 2 to 5% slower).
template <int MODE, bool TWO, bool WT, bool COUNT>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(WT ? 1 : TWO ? 5 : MODE == MODE_PRIMARY ? 6 : 1))) void k_trace(KParams P)
{
    constexpr bool ANY = MODE != MODE_PRIMARY;

    const int tid = threadIdx.x;
    const uint32_t lane = __lane_id();
    const uint32_t glane = blockIdx.x * BLOCK + tid;
    const DevScene sc = P.sc;
    const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    TravStack<SL, BLOCK, !ANY> st{tid, reinterpret_cast<uint2*>(P.w.overflow), P.w.overflow_depth, P.w.n_lanes,
                                   glane, P.w.error_flag};

    int state = 0;                    // 0 idle, 1 tracing
    uint32_t px = 0, pk = 0;          // pixel and sample of the current item
    uint32_t j = 0, acc = 0;          // shadow: current light, mask so far
    uint32_t n_rays = 0;
    float os[3] = {0, 0, 0}, nf[3] = {0, 0, 0};
    TravRay ray;
    TravState ts;
    TravWorld tw;
    TravWorld* twp = TWO ? &tw : nullptr;
    const uint32_t root = TWO ? sc.tlas_root : 0u;
    bool queue_empty = false;
    // point lights: a unit is 64 consecutive samples x one light group, so that the lanes of a refill trace
    // neighbouring samples towards one light
    const uint32_t groups = ANY ? P.light_groups : 1u;
    const uint32_t n_units = P.n_items * groups;
    const XcdQueue<ITEM_CHUNK> queue(P.w.counters, P.slot, n_units);
    uint32_t pool_next = 0, pool_end = 0;   // wave-uniform range of claimed, not yet started positions
    uint32_t rays_cast = 0, node_visits = 0, tri_tests = 0;

    // shadow items: set up the next ray that is cast, or return false
    auto next_shadow_ray = [&]() -> bool {
        while (j < n_rays) {
            if (rc_shadow_ray(P.L.point[j], P.L.rect, P.nL, false, px, j, P.L.area_stream, P.cam.seed, P.cam.frame, os, nf,
                              ray)) {
                trav_begin(ray, ts, root, twp);
                if constexpr (COUNT) ++rays_cast;
                return true;
            }
            j += groups;
        }
        return false;
    };

    auto finish_item = [&]() {
        if (MODE == MODE_POINT) {
            uint32_t* m = P.mask + (size_t)px * (P.cam.ssaa * P.cam.ssaa) + pk;
            if (groups == 1u) *m = acc;
            else if (acc != 0u) atomicOr(m, acc);   // cleared by the setup pass
        }
    };

    auto start_item = [&](uint32_t unit) -> bool {
        uint32_t item = unit, group = 0;
        if (ANY && groups > 1u) {
            const uint32_t tile = (unit >> 6) / groups;
            group = (unit >> 6) - tile * groups;
            item = tile * 64u + (unit & 63u);
        }
        if (!rc_item_to_sample(P.cam, item, px, pk)) return false;
        if (MODE == MODE_PRIMARY) {
            rc_camera_ray(P.cam, px, pk, ray.o, ray.d);
            trav_begin(ray, ts, root, twp);
            if constexpr (COUNT) ++rays_cast;
            return true;
        } else {
            // origin and normal from the setup pass (the FP64 reconstruction stays out of this kernel)
            size_t s = (size_t)px * (P.cam.ssaa * P.cam.ssaa) + pk;
            const float4 a = P.setup[2 * s];
            acc = 0;
            j = group;
            n_rays = (uint32_t)P.L.n_point;
            if (a.w == 0.0f) { finish_item(); return false; }
            const float4 b = P.setup[2 * s + 1];
            os[0] = a.x; os[1] = a.y; os[2] = a.z;
            nf[0] = b.x; nf[1] = b.y; nf[2] = b.z;
            if (next_shadow_ray()) return true;
            finish_item();
            return false;
        }
    };

    // a ray ended: record it; returns true when the lane continues with another ray of its item
    auto end_ray = [&](bool occluded) -> bool {
        if (MODE == MODE_PRIMARY) {
            P.gbuf_out[(size_t)px * (P.cam.ssaa * P.cam.ssaa) + pk] =
                make_uint4(ts.best_id, __float_as_uint(ts.best_t), __float_as_uint(ts.best_u), __float_as_uint(ts.best_v));
            return false;
        } else {
            if (!occluded) acc |= 1u << j;
            j += groups;
            if (next_shadow_ray()) return true;
            finish_item();
            return false;
        }
    };

    for (;;) {
        // ---- refill idle lanes from the work counter
        for (;;) {
            uint64_t need = __ballot(state == 0);
            if (need == 0 || queue_empty) break;
            if (pool_next == pool_end) {   // the wave's pool is used up: claim the next POOL positions
                pool_next = queue.claim(P.claim);
                pool_end = pool_next + P.claim;
                if (queue.exhausted(pool_next)) { queue_empty = true; break; }
            }
            const uint32_t cnt = min((uint32_t)__popcll(need), pool_end - pool_next);
            const uint32_t base = pool_next;
            pool_next += cnt;
            if (state == 0) {
                uint32_t rank = (uint32_t)__popcll(need & below);
                uint64_t my = queue.at(base + rank);
                if (rank < cnt && my < n_units && start_item((uint32_t)my)) state = 1;
            }
            if (queue.exhausted(pool_next)) queue_empty = true;
        }
        if (__ballot(state == 1) == 0) break;

        // ---- traversal: node phase then leaf phase for all busy lanes, until enough lanes are idle
        for (;;) {
            uint32_t occluded = 0u;
            trav_advance<TWO, WT, 3, 1, COUNT>(sc, ray, ts, st, state == 1, ANY, occluded, node_visits, tri_tests, twp);
            if (state == 1 && ts.cur == RC_STACK_EMPTY) {
                if (!end_ray(occluded != 0u)) state = 0;
            }
            uint32_t n_act = (uint32_t)__popcll(__ballot(state == 1));
            if (n_act == 0) break;
            if (!queue_empty && n_act <= (uint32_t)REFILL_AT) break;
        }
    }

    if constexpr (COUNT) {
        unsigned long long cnt[3] = {rays_cast, node_visits, tri_tests};
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            unsigned long long v = cnt[q];
            for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
            if (lane == 0) atomicAdd(P.w.ray_count + 2 * q, v);
        }
    }
}

// Rect-light visibility with one ray per lane.  The N light samples of a pixel occupy N consecutive
// ray slots, so a wave traces the samples of one pixel (N >= 64) or of 64/N neighbouring pixels
// together: its lanes start from the same point towards nearby targets and mostly fetch the same
// nodes.  A wave claims 64 ray slots at a time, advances them to completion, and adds the visible
// count of each pixel segment (ballot + popcount) to a per-pixel counter.
template <bool TWO, bool WT, bool COUNT>
__global__ __launch_bounds__(BLOCK) void k_rect_packets(KParams P, uint32_t* counts)
{
    const int tid = threadIdx.x;
    const uint32_t lane = __lane_id();
    const uint32_t glane = blockIdx.x * BLOCK + tid;
    const DevScene sc = P.sc;
    TravStack<SL, BLOCK, false> st{tid, reinterpret_cast<uint2*>(P.w.overflow), P.w.overflow_depth, P.w.n_lanes,
                                   glane, P.w.error_flag};
    const uint64_t N = (uint64_t)P.L.area_samples;
    const uint64_t total = (uint64_t)P.n_items * N;
    const uint64_t n_blocks = (total + 63) / 64;
    uint32_t rays_cast = 0, node_visits = 0, tri_tests = 0;
    TravRay ray;
    TravState ts;
    TravWorld tw;
    TravWorld* twp = TWO ? &tw : nullptr;
    const XcdQueue<RECT_CHUNK> queue(P.w.counters, P.slot, n_blocks);
    uint32_t pos = 0, pos_end = 0;   // wave-uniform range of claimed positions
    for (;;) {
        if (pos == pos_end) {
            pos = queue.claim(P.claim);
            pos_end = pos + P.claim;
        }
        const uint32_t j = pos++;
        if (queue.exhausted(j)) break;
        const uint64_t blk = queue.at(j);
        if (blk >= n_blocks) continue;
        const uint64_t r = (uint64_t)blk * 64 + lane;
        const uint32_t item = (uint32_t)(r / N), k = (uint32_t)(r % N);
        uint32_t px = 0, pk = 0;
        const bool in_image = r < total && rc_item_to_sample(P.cam, item, px, pk);
        bool busy = false;
        if (in_image) {
            const float4 a = P.setup[2 * (size_t)px];   // one sample per pixel: setup entry px
            if (a.w != 0.0f) {
                const float4 b = P.setup[2 * (size_t)px + 1];
                float os[3] = {a.x, a.y, a.z};
                float nf[3] = {b.x, b.y, b.z};
                busy = rc_shadow_ray(P.L.point[0], P.L.rect, P.nL, true, px, k, P.L.area_stream, P.cam.seed,
                                     P.cam.frame, os, nf, ray);
                if (busy) {
                    trav_begin(ray, ts, TWO ? sc.tlas_root : 0u, twp);
                    if constexpr (COUNT) ++rays_cast;
                }
            }
        }
        uint32_t occluded = 0u;
        while (__ballot(busy && ts.cur != RC_STACK_EMPTY) != 0)
            trav_advance<TWO, WT, 3, 1, COUNT>(sc, ray, ts, st, busy, true, occluded, node_visits, tri_tests, twp);
        const uint64_t vis = __ballot(busy && occluded == 0u);
        if (in_image && (lane == 0 || k == 0)) {
            uint32_t end = (uint32_t)min<uint64_t>(64, lane + (N - k));
            uint64_t seg = (end >= 64 ? ~0ull : ((1ull << end) - 1)) & ~((1ull << lane) - 1);
            uint32_t c = (uint32_t)__popcll(vis & seg);
            if (c) atomicAdd(counts + px, c);
        }
    }
    if constexpr (COUNT) {
        unsigned long long cnt[3] = {rays_cast, node_visits, tri_tests};
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            unsigned long long v = cnt[q];
            for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
            if (lane == 0) atomicAdd(P.w.ray_count + 2 * q, v);
        }
    }
}

// Per-sample shadow-ray setup of the shadow passes: (origin, 1) and (unit normal, 0) in FP32 from the
// FP64 surface reconstruction, or (0, 0, 0, 0) for samples without a primary hit.  Keeps the FP64 code
// (and its registers) out of the traversal kernels, wave-uniform and per-lane alike.  mask: where the point-light
// kernels add one light's bit at a time, each sample's mask is cleared here (NULL otherwise).
__global__ __launch_bounds__(256) void k_shadow_setup(DevScene sc, DevCamera cam, const uint4* gbuf, uint32_t n_samples,
                                                      float4* setup, uint32_t* mask)
{
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_samples) return;
    const uint32_t spp = (uint32_t)(cam.ssaa * cam.ssaa);
    const uint4 h = gbuf[i];
    float4 a = make_float4(0.0f, 0.0f, 0.0f, 0.0f), b = a;
    if (h.x != RC_NO_HIT) {
        Surface S = rc_surface(sc, cam, i / spp, i % spp, h.x);
        D3 O = rc_shadow_origin(S);
        a = make_float4((float)O.x, (float)O.y, (float)O.z, 1.0f);
        b = make_float4((float)S.n.x, (float)S.n.y, (float)S.n.z, 0.0f);
    }
    setup[2 * (size_t)i] = a;
    setup[2 * (size_t)i + 1] = b;
    if (mask) mask[i] = 0u;
}

// Rect-light visibility, wave-uniform traversal.  The 64 ray slots of a wave (the samples of one
// pixel, or the N samples of each of 64 / N neighbouring pixels) walk the BVH together: the wave visits a node
// when any of its live rays hits one of its boxes, so node and triangle records are read once per wave
// through the scalar cache, and the traversal stack is wave-uniform, held one entry per lane in one
// register (64 entries) or two (128; the host picks the smallest that holds 3 x depth + 1 entries).  Each lane still
// tests its own ray against every box and triangle the wave visits, with the same FP32 arithmetic as
// the per-lane traversal; a triangle that a lane's own boxes would not have led to can only report a
// true crossing, so the occlusion result of every ray is the one the per-lane traversal finds.
// Children that some live ray enters are visited nearest first by lane 0's entry distance.  The
// distances are non-negative, so their bit patterns order like the values; the two lowest bits carry the
// child's slot instead (children whose keys differ only there are ordered by slot), so the keys sort with
// plain minima and maxima on the scalar unit and the child word is then taken by slot.  When all live
// rays share a direction octant (the usual case for a small light), the near and far plane blocks of the
// node are loaded at byte offsets picked by the octant; otherwise each lane picks its own planes.
template <bool TWO, bool WT, bool BIG, bool COUNT>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(TWO || WT ? 1 : 8))) void k_rect_wave(KParams P, uint32_t* counts, const float4* setup)
{
    const uint32_t lane = __lane_id();
    const DevScene sc = P.sc;
    const uint64_t N = (uint64_t)P.L.area_samples;
    const uint64_t total = (uint64_t)P.n_items * N;
    const uint64_t n_blocks = (total + 63) / 64;
    uint32_t rays_cast = 0, node_visits = 0, tri_tests = 0;
    const char* nodes_b = (const char*)(const void*)sc.nodes;
    const char* tris_b = (const char*)(const void*)sc.tris;
    const XcdQueue<RECT_CHUNK> queue(P.w.counters, P.slot, n_blocks);
    uint32_t pos = 0, pos_end = 0;   // wave-uniform range of claimed positions
    for (;;) {
        if (pos == pos_end) {
            pos = queue.claim(P.claim);
            pos_end = pos + P.claim;
        }
        const uint32_t j = pos++;
        if (queue.exhausted(j)) break;
        const uint64_t blk = queue.at(j);
        if (blk >= n_blocks) continue;
        const uint64_t r = (uint64_t)blk * 64 + lane;
        const uint32_t item = (uint32_t)(r / N), k = (uint32_t)(r % N);
        uint32_t px = 0, pk = 0;
        const bool in_image = r < total && rc_item_to_sample(P.cam, item, px, pk);
        TravRay ray;
        bool busy = false;
        if (in_image) {
            const float4 a = setup[2 * (size_t)px], b = setup[2 * (size_t)px + 1];
            if (a.w != 0.0f) {
                float os[3] = {a.x, a.y, a.z}, nf[3] = {b.x, b.y, b.z};
                busy = rc_shadow_ray(P.L.point[0], P.L.rect, P.nL, true, px, k, P.L.area_stream, P.cam.seed,
                                     P.cam.frame, os, nf, ray);
                if (busy) {
                    rc_ray_inv<!TWO && !WT>(ray);   // the flat Moller-Trumbore walk takes the clamped slab test
                    ++rays_cast;
                }
            }
        }
        const uint32_t occ = wave_occluded<TWO, WT, BIG, COUNT>(sc, nodes_b, tris_b, ray, busy, node_visits, tri_tests,
                                                         P.w.error_flag);
        const uint64_t vis = __ballot(busy && occ == 0u);
        if (in_image && (lane == 0 || k == 0)) {
            uint32_t end = (uint32_t)min<uint64_t>(64, lane + (N - k));
            uint64_t seg = (end >= 64 ? ~0ull : ((1ull << end) - 1)) & ~((1ull << lane) - 1);
            uint32_t c = (uint32_t)__popcll(vis & seg);
            if (c) atomicAdd(counts + px, c);
        }
    }
    if (P.w.ray_count) {
        unsigned long long cnt[3] = {rays_cast, node_visits, tri_tests};
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            unsigned long long v = cnt[q];
            for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
            if (lane == 0) atomicAdd(P.w.ray_count + 2 * q, v);
        }
    }
}

// Point-light shadow rays, wave-uniform traversal.  A unit of work is 64 consecutive samples (neighbouring
// pixels) and one light, or with TURN and all lights: the wave walks the tree once per light, each lane casting its
// sample's segment to the light where that lies above the surface, with the same tests and results as the per-lane
// kernel.  Mask bit l of a sample (cleared by the setup pass unless TURN): the ray to light l is cast and not occluded.  The pass cannot end before its longest unit, so the lights of a packet are units
// of their own (4 lights: the 64 samples that diverge most take a quarter of the time) unless the pass is so long that
// the number of claims and the repeated set-up cost more (point_lights_in_turn).  An instance for each: with the loop
// over the lights the watertight kernel takes 66 registers instead of 60, 7 waves per SIMD instead of 8 (8% slower).
template <bool TWO, bool WT, bool BIG, bool COUNT, bool TURN>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(TWO || WT ? 1 : 8))) void k_point_wave(KParams P, const float4* setup)
{
    const uint32_t lane = __lane_id();
    const DevScene sc = P.sc;
    const uint32_t spp = (uint32_t)(P.cam.ssaa * P.cam.ssaa);
    const uint32_t n_l = (uint32_t)P.L.n_point;
    const uint64_t n_units = (uint64_t)((P.n_items + 63u) / 64u) * (TURN ? 1u : n_l);
    uint32_t rays_cast = 0, node_visits = 0, tri_tests = 0;
    const char* nodes_b = (const char*)(const void*)sc.nodes;
    const char* tris_b = (const char*)(const void*)sc.tris;
    const XcdQueue<RECT_CHUNK> queue(P.w.counters, P.slot, n_units);
    uint32_t pos = 0, pos_end = 0;   // wave-uniform range of claimed positions
    for (;;) {
        if (pos == pos_end) {
            pos = queue.claim(P.claim);
            pos_end = pos + P.claim;
        }
        const uint32_t j = pos++;
        if (queue.exhausted(j)) break;
        const uint64_t unit = queue.at(j);
        if (unit >= n_units) continue;
        const uint32_t blk = TURN ? (uint32_t)unit : (uint32_t)unit / n_l, l0 = TURN ? 0u : (uint32_t)unit - blk * n_l;
        const uint32_t item = blk * 64u + lane;
        uint32_t px = 0, pk = 0;
        const bool in_image = item < P.n_items && rc_item_to_sample(P.cam, item, px, pk);
        const size_t smp = (size_t)px * spp + pk;
        if constexpr (!TURN) {
            TravRay ray;
            bool busy = false;
            if (in_image) {
                const float4 a = setup[2 * smp], b = setup[2 * smp + 1];
                if (a.w != 0.0f) {
                    float os[3] = {a.x, a.y, a.z}, nf[3] = {b.x, b.y, b.z};
                    busy = rc_shadow_ray(P.L.point[l0], P.L.rect, P.nL, false, px, l0, P.L.area_stream, P.cam.seed,
                                         P.cam.frame, os, nf, ray);
                    if (busy) {
                        rc_ray_inv<!TWO && !WT>(ray);   // the flat Moller-Trumbore walk takes the clamped slab test
                        ++rays_cast;
                    }
                }
            }
            const uint32_t occ = wave_occluded<TWO, WT, BIG, COUNT>(sc, nodes_b, tris_b, ray, busy, node_visits, tri_tests,
                                                             P.w.error_flag);
            if (busy && occ == 0u) atomicOr(P.mask + smp, 1u << l0);
            continue;
        }
        float4 a = make_float4(0.0f, 0.0f, 0.0f, 0.0f), b = a;
        if (in_image) {
            a = setup[2 * smp];
            b = setup[2 * smp + 1];
        }
        const float os[3] = {a.x, a.y, a.z}, nf[3] = {b.x, b.y, b.z};
        uint32_t mask = 0;
        for (uint32_t l = 0; l < n_l; ++l) {
            TravRay ray;
            bool busy = false;
            if (a.w != 0.0f) {
                busy = rc_shadow_ray(P.L.point[l], P.L.rect, P.nL, false, px, l, P.L.area_stream, P.cam.seed,
                                     P.cam.frame, os, nf, ray);
                if (busy) {
                    rc_ray_inv<!TWO && !WT>(ray);
                    ++rays_cast;
                }
            }
            const uint32_t occ = wave_occluded<TWO, WT, BIG, COUNT>(sc, nodes_b, tris_b, ray, busy, node_visits, tri_tests,
                                                             P.w.error_flag);
            if (busy && occ == 0u) mask |= 1u << l;
        }
        if (in_image) P.mask[smp] = mask;
    }
    if (P.w.ray_count) {
        unsigned long long cnt[3] = {rays_cast, node_visits, tri_tests};
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            unsigned long long v = cnt[q];
            for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
            if (lane == 0) atomicAdd(P.w.ray_count + 2 * q, v);
        }
    }
}

// Camera rays, wave-uniform closest-hit traversal.  The 64 samples of a packet (an 8x8-pixel tile, or 4x4
// pixels x 4 samples) share the eye point and walk the BVH together, reading nodes and triangles once per
// wave through the scalar cache; every lane keeps its own closest hit (t, then the smaller id) and tests
// only what its own bound allows.  A child that any lane's box test accepts is pushed with a bound shared
// by all lanes: the squared distance from the eye to its box, a lower bound on every lane's entry distance.
// A popped entry is skipped when that bound exceeds the largest closest-hit distance of the wave (with a
// relative margin of 1e-5 that covers the FP32 rounding of the slab tests and of |d| = 1).  Results equal
// the per-lane traversal's: extra triangle tests can only report true crossings.
template <bool WT>
__global__ __launch_bounds__(BLOCK) void k_primary_wave(KParams P)
{
    const uint32_t lane = __lane_id();
    const DevScene sc = P.sc;
    const uint32_t n_packets = (P.n_items + 63) / 64;
    const uint32_t KEY_MISS = 0x7F800000u;
    const float ex = P.cam.eye[0], ey = P.cam.eye[1], ez = P.cam.eye[2];
    uint32_t rays_cast = 0, node_visits = 0, tri_tests = 0;
    const XcdQueue<RECT_CHUNK> queue(P.w.counters, P.slot, n_packets);
    uint32_t pos = 0, pos_end = 0;
    for (;;) {
        if (pos == pos_end) {
            pos = queue.claim(P.claim);
            pos_end = pos + P.claim;
        }
        const uint32_t j = pos++;
        if (queue.exhausted(j)) break;
        const uint64_t blk = queue.at(j);
        if (blk >= n_packets) continue;
        const uint32_t item = (uint32_t)blk * 64 + lane;
        uint32_t px = 0, pk = 0;
        const bool valid = item < P.n_items && rc_item_to_sample(P.cam, item, px, pk);
        TravRay ray;
        ray.o[0] = ex; ray.o[1] = ey; ray.o[2] = ez;
        ray.d[0] = 1.0f; ray.d[1] = 0.0f; ray.d[2] = 0.0f;
        float best_t = -INFINITY, best_u = 0.0f, best_v = 0.0f;   // invalid lanes accept nothing
        uint32_t best_id = RC_NO_HIT;
        if (valid) {
            rc_camera_ray(P.cam, px, pk, ray.o, ray.d);
            best_t = INFINITY;
            ++rays_cast;
        }
        rc_ray_inv(ray);
        float wmax = INFINITY;                                    // largest closest-hit distance of the wave
        uint32_t cur = __ballot(valid) != 0 ? 0u : RC_STACK_EMPTY;
        int sp = 0;
        uint32_t stk0 = 0, stk1 = 0, lbs0 = 0, lbs1 = 0;         // entry e: lane e % 64 of {stk,lbs}{e / 64}
        auto pop = [&]() -> uint32_t {
            const float lim = wmax * 1.00001f;
            const float lim2 = lim * lim;
            while (sp > 0) {
                --sp;
                const uint32_t w = (uint32_t)__builtin_amdgcn_readlane((int)(sp < 64 ? stk0 : stk1), sp & 63);
                const float lb = __uint_as_float(
                    (uint32_t)__builtin_amdgcn_readlane((int)(sp < 64 ? lbs0 : lbs1), sp & 63));
                if (!(lb > lim2)) return w;
            }
            return RC_STACK_EMPTY;
        };
        while (cur != RC_STACK_EMPTY) {
            if (!rc_is_leaf(cur)) {
                rc_const_v4f* np = (rc_const_v4f*)(const void*)(sc.nodes + cur);
                const rc_v4f lx = np[0], hx = np[1], ly = np[2], hy = np[3], lz = np[4], hz = np[5];
                const rc_v4f chf = np[6];
                uint32_t key[4], cw[4];
                float lb[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    float nx = ray.inv[0] >= 0.0f ? lx[c] : hx[c], fx = ray.inv[0] >= 0.0f ? hx[c] : lx[c];
                    float ny = ray.inv[1] >= 0.0f ? ly[c] : hy[c], fy = ray.inv[1] >= 0.0f ? hy[c] : ly[c];
                    float nz = ray.inv[2] >= 0.0f ? lz[c] : hz[c], fz = ray.inv[2] >= 0.0f ? hz[c] : lz[c];
                    float t0;
                    const bool hit = rc_slab(ray, ray.invf, nx, ny, nz, fx, fy, fz, best_t, t0);
                    uint64_t m = __ballot(hit);
                    uint32_t k = KEY_MISS;
                    if (m != 0) {
                        int first = __builtin_ctzll(m);
                        k = (uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(t0), first) & 0x7FFFFFFFu;
                    }
                    key[c] = k;
                    cw[c] = __float_as_uint(chf[c]);
                    // squared distance from the eye to the child box (uniform)
                    float qx = fmaxf(fmaxf(lx[c] - ex, ex - hx[c]), 0.0f);
                    float qy = fmaxf(fmaxf(ly[c] - ey, ey - hy[c]), 0.0f);
                    float qz = fmaxf(fmaxf(lz[c] - ez, ez - hz[c]), 0.0f);
                    float q2 = qx * qx + qy * qy;
                    lb[c] = q2 + qz * qz;
                }
                if (valid) ++node_visits;
#define RC_CS(a, b)                                                                   \
    {                                                                                 \
        bool sw = key[b] < key[a];                                                    \
        uint32_t ka = sw ? key[b] : key[a], kb = sw ? key[a] : key[b];                \
        uint32_t ca = sw ? cw[b] : cw[a], cb = sw ? cw[a] : cw[b];                    \
        float la = sw ? lb[b] : lb[a], lbb = sw ? lb[a] : lb[b];                      \
        key[a] = ka; key[b] = kb; cw[a] = ca; cw[b] = cb; lb[a] = la; lb[b] = lbb;    \
    }
                RC_CS(0, 1) RC_CS(2, 3) RC_CS(0, 2) RC_CS(1, 3) RC_CS(1, 2)
#undef RC_CS
#pragma unroll
                for (int c = 3; c >= 1; --c) {
                    if (key[c] < KEY_MISS) {
                        if (sp < 64) {
                            stk0 = (int)lane == sp ? cw[c] : stk0;
                            lbs0 = (int)lane == sp ? __float_as_uint(lb[c]) : lbs0;
                            ++sp;
                        } else if (sp < 128) {
                            stk1 = (int)lane == sp - 64 ? cw[c] : stk1;
                            lbs1 = (int)lane == sp - 64 ? __float_as_uint(lb[c]) : lbs1;
                            ++sp;
                        } else if (lane == 0) {
                            *P.w.error_flag = 1u;   // beyond the bound the host checked: entry dropped, reported
                        }
                    }
                }
                cur = key[0] < KEY_MISS ? cw[0] : pop();
            } else {
                const uint32_t first = rc_leaf_first(cur), cnt = rc_leaf_count(cur);
                for (uint32_t i = 0; i < cnt; ++i) {
                    rc_const_v4f* tp = (rc_const_v4f*)(const void*)(sc.tris + 3 * (size_t)(first + i));
                    const rc_v4f A = tp[0], B = tp[1], C = tp[2];
                    if (valid) {
                        ++tri_tests;
                        float t, u, v;
                        bool hit = WT ? rc_wt(ray, A.x, A.y, A.z, B.x, B.y, B.z, C.x, C.y, C.z, t, u, v)
                                      : rc_mt(ray, A.x, A.y, A.z, B.x, B.y, B.z, C.x, C.y, C.z, t, u, v);
                        const uint32_t id = __float_as_uint(A.w);
                        if (hit && (t < best_t || (t == best_t && id < best_id))) {
                            best_t = t; best_u = u; best_v = v; best_id = id;
                        }
                    }
                }
                // largest closest-hit distance over the wave's valid lanes (non-negative floats order like
                // their bit patterns; invalid lanes, at -inf, count as 0), reduced in registers
                wmax = __uint_as_float(__ockl_wfred_max_u32(__float_as_uint(fmaxf(best_t, 0.0f))));
                cur = pop();
            }
            cur = __builtin_amdgcn_readfirstlane(cur);
        }
        if (valid)
            P.gbuf_out[(size_t)px * (P.cam.ssaa * P.cam.ssaa) + pk] =
                make_uint4(best_id, __float_as_uint(best_t), __float_as_uint(best_u), __float_as_uint(best_v));
    }
    if (P.w.ray_count) {
        unsigned long long cnt[3] = {rays_cast, node_visits, tri_tests};
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            unsigned long long v = cnt[q];
            for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
            if (lane == 0) atomicAdd(P.w.ray_count + 2 * q, v);
        }
    }
}

// value of the quad's lane (own lane ^ X)
template <int X>
__device__ inline uint32_t quad_xor(uint32_t v)
{
    constexpr int ctrl = (0 ^ X) | (1 ^ X) << 2 | (2 ^ X) << 4 | (3 ^ X) << 6;   // quad_perm
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, ctrl, 0xF, 0xF, true);
}

// Camera and shadow rays of small passes: four lanes to a ray, which test the four children of a node and up to four
// triangles of a leaf at once.  A pass that leaves the chip idle lasts as long as its longest wave, a serial chain
// of node visits whose time is half latency, half the wave's own instructions (four cycles each); here a visit
// takes about 45 of them instead of 90, a leaf one round of loads instead of one per triangle, and a wave waits for
// 16 rays instead of 64.  No queue and no refill: one wave per 16 rays, the workgroups of an XCD on neighbouring
// tiles.  The tests are those of the per-lane walk (rc_slab, rc_tri), hits are kept per lane and reduced by (t, id).
// 128x128 on 1.1M triangles: camera rays 0.093 to 0.051 ms, one point light 0.113 to 0.056; figures by size at quad_ok.
template <int MODE, bool TWO, bool WT>
__global__ __launch_bounds__(64) void k_quad(KParams P, uint32_t* counts)
{
    constexpr bool ANY = MODE != MODE_PRIMARY;
    const uint32_t lane = threadIdx.x, q = lane >> 2, c = lane & 3u;
    const DevScene& sc = P.sc;
    // block b of XCD b % 8 takes the b / 8-th block of that XCD's contiguous share
    const uint32_t share = (gridDim.x + RC_XCDS - 1) / RC_XCDS;
    const uint32_t blk = (blockIdx.x % RC_XCDS) * share + blockIdx.x / RC_XCDS;
    uint32_t px = 0, k = 0, light = 0;
    bool on;
    if (MODE == MODE_RECT) {
        const uint64_t r = (uint64_t)blk * 16u + q;
        const uint32_t N = (uint32_t)P.L.area_samples;
        uint32_t none = 0;
        on = r < (uint64_t)P.n_items * N && rc_item_to_sample(P.cam, (uint32_t)r / N, px, none);
        k = (uint32_t)r % N;
    } else {
        const uint32_t groups = ANY ? (uint32_t)P.L.n_point : 1u;
        const uint32_t part = blk / groups;
        light = blk - part * groups;
        const uint32_t item = part * 16u + q;
        on = item < P.n_items && rc_item_to_sample(P.cam, item, px, k);
    }
    TravRay ray;
    TravState ts;
    TravWorld tw;
    const size_t smp = MODE == MODE_RECT ? (size_t)px : (size_t)px * (P.cam.ssaa * P.cam.ssaa) + k;
    if (on) {
        if constexpr (MODE == MODE_PRIMARY) {
            rc_camera_ray(P.cam, px, k, ray.o, ray.d);
        } else {
            const float4 a = P.setup[2 * smp], b = P.setup[2 * smp + 1];
            const float os[3] = {a.x, a.y, a.z}, nf[3] = {b.x, b.y, b.z};
            on = a.w != 0.0f && rc_shadow_ray(P.L.point[light], P.L.rect, P.nL, MODE == MODE_RECT, px, k, P.L.area_stream,
                                              P.cam.seed, P.cam.frame, os, nf, ray);
        }
    }
    const bool cast = on;
    uint32_t occluded = 0u;
    if (on) {
        trav_begin(ray, ts, TWO ? sc.tlas_root : 0u, TWO ? &tw : nullptr);
        const char* nb = reinterpret_cast<const char*>(sc.nodes);
        uint32_t ofs[3];   // this child's near planes within a node
        auto set_ofs = [&]() {
#pragma unroll
            for (int a = 0; a < 3; ++a) ofs[a] = 32u * a + 4u * c + ((__float_as_uint(ray.inv[a]) >> 31) << 4);
        };
        set_ofs();
        uint2* stk = reinterpret_cast<uint2*>(rc_lds) + q;   // entry e of the quad's ray: stk[16 e]
        float bound = ANY ? 1.0f : INFINITY;                 // closest hit of the quad so far
        while (ts.cur != RC_STACK_EMPTY) {
            if (!rc_is_leaf(ts.cur)) {
                const uint32_t np = ts.cur << 7;
                float n[3], f[3];
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    n[a] = *reinterpret_cast<const float*>(nb + (np | ofs[a]));
                    f[a] = *reinterpret_cast<const float*>(nb + ((np | ofs[a]) ^ 16u));
                }
                const uint32_t ch = *reinterpret_cast<const uint32_t*>(nb + (np | (4u * c)) + 96);
                float t0;
                const bool hit = rc_slab(ray, ray.invf, n[0], n[1], n[2], f[0], f[1], f[2], bound, t0);
                asm volatile("" : : "v"(ch));   // loaded with the planes, not after the test
                const uint32_t key = hit ? __float_as_uint(fabsf(t0)) : 0xFFFFFFF0u;
                // this child's place among the four: by entry distance, then by slot
                const uint32_t rank = (quad_xor<1>(key) < key + (c & 1u) ? 1u : 0u) +
                                      (quad_xor<2>(key) < key + (c >> 1) ? 1u : 0u) +
                                      (quad_xor<3>(key) < key + (c >> 1) ? 1u : 0u);
                uint32_t hits = hit ? 1u : 0u;
                hits += quad_xor<1>(hits);
                hits += quad_xor<2>(hits);
                if (hits != 0u) {
                    // read by the quad's other lanes: the compiler may not move the stack's accesses past this
                    if (hit && rank != 0u) stk[16 * (ts.sp + (int)(hits - 1u - rank))] = make_uint2(ch, key);
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                    ts.sp += (int)hits - 1;
                    uint32_t first = rank == 0u ? ch : 0u;
                    first |= quad_xor<1>(first);
                    ts.cur = first | quad_xor<2>(first);
                    continue;
                }
            } else if (TWO && tw.in_blas == 0u) {
                // top-level leaf: enter the instance, its return point on the stack
                const DevInst& I = sc.inst[rc_leaf_first(ts.cur)];
                rc_map_ray(I.w2o, tw.o, tw.d, ray);
                set_ofs();
                if (c == 0u) stk[16 * ts.sp] = make_uint2(RC_INST_RETURN, 0u);
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                ++ts.sp;
                tw.in_blas = 1u;
                ts.cur = I.root;
                continue;
            } else {
                const uint32_t first = rc_leaf_first(ts.cur), cnt = rc_leaf_count(ts.cur);
                for (uint32_t i = c; i < cnt; i += 4u) {
                    const float4* tp = sc.tris + 3 * (size_t)(first + i);
                    const float4 A = tp[0], B = tp[1], C = tp[2];
                    float t, u, v;
                    const bool hit = rc_tri<WT>(ray, A, B, C, t, u, v);
                    if (ANY) {
                        if (hit && t < 1.0f) occluded = 1u;
                    } else {
                        const uint32_t id = __float_as_uint(A.w);
                        if (hit && (t < ts.best_t || (t == ts.best_t && id < ts.best_id))) {
                            ts.best_t = t; ts.best_u = u; ts.best_v = v; ts.best_id = id;
                        }
                    }
                }
                if (ANY) {
                    occluded |= quad_xor<1>(occluded);
                    occluded |= quad_xor<2>(occluded);
                    if (occluded != 0u) break;
                } else {
                    bound = fminf(bound, ts.best_t);
                    bound = fminf(bound, __uint_as_float(quad_xor<1>(__float_as_uint(bound))));
                    bound = fminf(bound, __uint_as_float(quad_xor<2>(__float_as_uint(bound))));
                }
            }
            // next entry; closest-hit rays skip those that start beyond the current hit
            ts.cur = RC_STACK_EMPTY;
            while (ts.sp > 0) {
                --ts.sp;
                const uint2 e = stk[16 * ts.sp];
                if (TWO && e.x == RC_INST_RETURN) {   // back in world space
#pragma unroll
                    for (int a = 0; a < 3; ++a) { ray.o[a] = tw.o[a]; ray.d[a] = tw.d[a]; }
                    rc_ray_inv(ray);
                    set_ofs();
                    tw.in_blas = 0u;
                    continue;
                }
                if (ANY || __uint_as_float(e.y) <= bound) {
                    ts.cur = e.x;
                    break;
                }
            }
        }
        if constexpr (!ANY) {
            auto take = [&](uint32_t id, float t, float u, float v) {
                if (t < ts.best_t || (t == ts.best_t && id < ts.best_id)) {
                    ts.best_t = t; ts.best_u = u; ts.best_v = v; ts.best_id = id;
                }
            };
#define RC_TAKE(X)                                                                                              \
    take(quad_xor<X>(ts.best_id), __uint_as_float(quad_xor<X>(__float_as_uint(ts.best_t))),                     \
         __uint_as_float(quad_xor<X>(__float_as_uint(ts.best_u))), __uint_as_float(quad_xor<X>(__float_as_uint(ts.best_v))))
            RC_TAKE(1);
            RC_TAKE(2);
#undef RC_TAKE
        }
    }
    if (c != 0u || !cast) return;
    if (MODE == MODE_PRIMARY)
        P.gbuf_out[smp] = make_uint4(ts.best_id, __float_as_uint(ts.best_t), __float_as_uint(ts.best_u), __float_as_uint(ts.best_v));
    else if (occluded == 0u) {
        if (MODE == MODE_RECT) atomicAdd(counts + px, 1u);
        else atomicOr(P.mask + smp, 1u << light);   // cleared by the setup pass
    }
}

__global__ void k_rect_finish(const uint32_t* counts, uint32_t n_pix, uint32_t N, float* vis)
{
    uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n_pix) vis[i] = (float)counts[i] / (float)N;
}

template <int MODE>
constexpr size_t lds_bytes() { return TravStack<SL, BLOCK, MODE == MODE_PRIMARY>::lds_bytes(); }

// Small passes go four lanes to a ray (k_quad): stacks up to 128 entries in LDS, nodes at 32-bit offsets, nothing
// counted.  The limits lie where the chip is full and the quad's extra instructions per ray begin to cost: later in
// small trees, whose nodes stay in the L2, and early for camera rays of large two-level structures, whose rays go
// through many bodies.  Time four lanes to a ray over one lane to a ray:
//   flat, 1.1M triangles (7.3M): camera rays 0.20M 0.65 (0.62), 0.39M 0.82 (0.81), 0.58M 0.87 (0.86), 0.92M 1.00 (1.01), of an
//       LBVH 0.58M 1.08 (0.91); point lights 0.31M 0.69 (0.76), 0.61M 0.92 (0.97), LBVH 1.04 (0.97); rect light 0.61M
//       0.68 (0.98), 0.77M 0.71 (1.12), 0.92M 0.76 to 1.05 (1.03 to 1.22)
//   flat, 20K triangles (200K): camera rays 0.92M 0.51 (0.63); point lights 0.58M 0.47 (0.63); rect light 0.92M 0.68 (0.70)
//   two-level, 1.1M (7.3M): camera rays 0.12M 0.88 (1.03), 0.15M 0.99 (0.97), 0.20M 1.07 (1.08), 0.31M 1.42 (1.39); point lights
//       0.31M 0.88 to 1.07 (0.96 to 1.02), 0.39M 1.00 (1.16); rect light 0.31M 0.74 to 0.86 (0.94 to 1.02), 0.46M 0.90 (1.07)
//   two-level, 20K (200K): camera rays 0.31M 0.63 (0.73); point lights 0.31M 0.61 (0.83); rect light 0.31M 0.71 (0.66)
// Stacks that leave LDS for fewer than 20 waves on a CU, as of two-level structures: in proportion to the waves that fit
// (330K rays at 11).
constexpr uint64_t QUAD_RAYS = 600000;
uint64_t quad_limit(const DevScene& sc, int mode)
{
    if (mode == MODE_PRIMARY && sc.inst && sc.n_tris >= 600000u) return 180000;
    if (mode == MODE_RECT) return sc.n_tris >= 3000000u ? 620000 : 950000;
    return QUAD_RAYS;
}
constexpr uint64_t PRIMARY_WAVE = 5000000;   // 2x2 samples: camera rays wave-uniform above (rc_launch_primary)
size_t quad_lds(const DevScene& sc) { return (size_t)sc.max_stack * 16 * sizeof(uint2); }
bool quad_ok(const DevScene& sc, const TraceWork& w, uint64_t rays, int mode)
{
    if (w.ray_count || sc.max_stack > 128 || sc.n_nodes >= (1u << 25)) return false;
    const uint64_t waves = 163840 / quad_lds(sc), limit = quad_limit(sc, mode);
    return rays <= (waves >= 20 ? limit : std::min(limit, QUAD_RAYS * waves / 20));
}
// waves of 16 rays for `rays` rays in each of `groups`, a whole share for every XCD
uint32_t quad_grid(uint64_t rays, uint32_t groups)
{
    const uint64_t waves = (rays + 15) / 16 * groups;
    return (uint32_t)((waves + RC_XCDS - 1) / RC_XCDS * RC_XCDS);
}

// compute units of the device and resident blocks of a kernel per compute unit (1 if a query fails)
int cu_count(int device)
{
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess || n < 1) n = 1;
    return n;
}

int blocks_per_cu(const void* kernel, size_t lds)
{
    int b = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&b, kernel, BLOCK, lds) != hipSuccess || b < 1) b = 1;
    return b;
}

}  // namespace

// Launch the instance of KERNEL (written with RC_TWO and RC_WT in its template arguments) that matches the
// scene: flat or two-level structure, Moller-Trumbore or watertight triangle test (`two`, `wt` in scope).
#define RC_LAUNCH_ONE(TWO_, WT_, KERNEL, ...)                   \
    do {                                                         \
        constexpr bool RC_TWO = TWO_, RC_WT = WT_;               \
        hipLaunchKernelGGL(KERNEL, __VA_ARGS__);                 \
    } while (0)
#define RC_LAUNCH_TW(KERNEL, ...)                                                  \
    do {                                                                           \
        if (two) {                                                                 \
            if (wt) RC_LAUNCH_ONE(true, true, KERNEL, __VA_ARGS__);                \
            else RC_LAUNCH_ONE(true, false, KERNEL, __VA_ARGS__);                  \
        } else {                                                                   \
            if (wt) RC_LAUNCH_ONE(false, true, KERNEL, __VA_ARGS__);               \
            else RC_LAUNCH_ONE(false, false, KERNEL, __VA_ARGS__);                 \
        }                                                                          \
    } while (0)

// persistent grid of the traversal kernels: compute units x the largest resident block count among them
int rc_trace_grid(int device)
{
    const int blocks[] = {
        blocks_per_cu(reinterpret_cast<const void*>(&k_trace<MODE_PRIMARY, false, false, false>), lds_bytes<MODE_PRIMARY>()),
        blocks_per_cu(reinterpret_cast<const void*>(&k_trace<MODE_POINT, false, false, false>), lds_bytes<MODE_POINT>()),
        blocks_per_cu(reinterpret_cast<const void*>(&k_rect_packets<false, false, false>), TravStack<SL, BLOCK, false>::lds_bytes()),
        blocks_per_cu(reinterpret_cast<const void*>(&k_rect_wave<false, false, false, false>), 0),
        blocks_per_cu(reinterpret_cast<const void*>(&k_primary_wave<false>), 0),
        blocks_per_cu(reinterpret_cast<const void*>(&k_point_wave<false, false, false, false, false>), 0)};
    int b = 1;
    for (int x : blocks) b = std::max(b, x);
    return cu_count(device) * b;
}

void rc_launch_primary(const DevScene& sc, const DevCamera& cam, uint4* gbuf, const TraceWork& w, int grid,
                       bool per_lane, hipStream_t st)
{
    KParams P = {};
    P.sc = sc;
    P.cam = cam;
    P.gbuf_out = gbuf;
    P.w = w;
    P.n_items = rc_n_items(cam.width, cam.height, cam.ssaa);
    P.slot = 0;
    // with one sample per pixel, a wave's 8x8-pixel tile diverges too much for the wave-uniform traversal; with 2x2 (4
    // samples of each of 16 neighbouring pixels) it pays off where there are enough waves to hide the longest walks.
    // Wave / per lane (ms), 1.1M triangles (7.3M): 2.07M samples 0.37 / 0.26 (0.51 / 0.38), 3.7M 0.45 / 0.36 (0.63 /
    // 0.52), 8.3M 0.68 / 0.68 (0.93 / 0.96), 33M 1.65 / 2.02 (2.26 / 2.95).  Counted frames keep the wave kernel at
    // any size, two-level structures the per-lane one.
    const bool two = sc.inst != nullptr, wt = sc.watertight != 0u;
    if (!per_lane && quad_ok(sc, w, P.n_items, MODE_PRIMARY)) {
        const dim3 g(quad_grid(P.n_items, 1));
        RC_LAUNCH_TW((k_quad<MODE_PRIMARY, RC_TWO, RC_WT>), g, dim3(64), quad_lds(sc), st, P, (uint32_t*)nullptr);
    } else if (sc.max_stack <= 128 && !per_lane && cam.ssaa > 1 && !two && (P.n_items > PRIMARY_WAVE || w.ray_count)) {
        P.claim = claim_size((P.n_items + 63) / 64, grid, 64, 1, 4);
        if (wt)
            hipLaunchKernelGGL(k_primary_wave<true>, dim3(grid), dim3(BLOCK), 0, st, P);
        else
            hipLaunchKernelGGL(k_primary_wave<false>, dim3(grid), dim3(BLOCK), 0, st, P);
    } else {
        P.claim = claim_size(P.n_items, grid, 16, 32, 128);
        if (w.ray_count)
            RC_LAUNCH_TW((k_trace<MODE_PRIMARY, RC_TWO, RC_WT, true>), dim3(grid), dim3(BLOCK), lds_bytes<MODE_PRIMARY>(), st, P);
        else
            RC_LAUNCH_TW((k_trace<MODE_PRIMARY, RC_TWO, RC_WT, false>), dim3(grid), dim3(BLOCK), lds_bytes<MODE_PRIMARY>(), st, P);
    }
}

// Whether a packet's lights are walked in turn by one wave, one claim and one set-up for all of them, instead of as units
// of their own.  A claim is an atomic on one of eight counters, and these pass about 0.5 claims per ns: a pass of U
// units takes at least 2 U ns, which short walks (small trees) do not.  Against that stands the tail, a packet's
// walks one after another.  Separate units / in turn (ms), 2, 4 and 8 lights:
//     20K triangles  2.07M samples 0.19 / 0.21, 0.28 / 0.35, 0.51 / 0.59; 3.7M 0.27 / 0.25, 0.46 / 0.33, 0.86 / 0.53
//    200K            2.07M 0.75, 0.66, 0.52 of in turn; 3.7M 1.05, 1.02, 0.87; 5.0M 1.11, 1.12, 1.08; 8.3M 1.22, 1.43, 1.56
//    500K            3.7M 0.79, 0.84, 0.75; 6.5M 0.82, 1.01, 1.04; 8.3M 1.04, 1.11, 1.11; 14.7M 1.18, 1.40, 1.01
//    1.1M            5.0M 0.87, 0.87, 0.86; 6.5M 0.95, 0.92, 0.94; 8.3M 0.82, 1.02, 1.08; 14.7M 1.08, 1.24, 1.04
//    7.3M            8.3M 1.03, 0.94, 0.88; 14.7M 1.05, 1.08, 0.98
// so the line lies at 2.5M samples for 20K triangles and moves out with the fourth root of their number (watertight
// tests and two-level structures cross within a tenth of the same places).
static bool point_lights_in_turn(const DevScene& sc, uint64_t n_samples)
{
    return (double)n_samples >= 2.5e6 * std::sqrt(std::sqrt((double)sc.n_tris / 20000.0));
}

void rc_launch_shadow(const DevScene& sc, const DevCamera& cam, const DevLights& L, const uint4* gbuf,
                      uint32_t* mask, float* visibility, uint32_t* counts, float4* setup, const TraceWork& w,
                      int grid, RcKernels kernels, hipStream_t st)
{
    KParams P = {};
    P.sc = sc;
    P.cam = cam;
    P.L = L;
    P.gbuf_in = gbuf;
    P.mask = mask;
    P.vis = visibility;
    P.w = w;
    P.n_items = rc_n_items(cam.width, cam.height, cam.ssaa);
    const bool two = sc.inst != nullptr, wt = sc.watertight != 0u;
    const bool count = w.ray_count != nullptr;   // visits are counted only when asked
    // the wave-uniform kernels address nodes and triangles by 32-bit byte offsets and hold at most 128 stack
    // entries; they read each sample's shadow-ray origin and normal from `setup`
    const bool wave_ok = kernels != RC_KERNELS_LANE && rc_wave_ok(sc);
    // By default they serve the passes with many rays.  A wave-uniform pass cannot end before its slowest
    // wave, whose 64 rays (an 8x8-pixel tile at one sample per pixel) may diverge over detailed geometry and
    // walk the union of their paths, some hundreds of dependent node steps.  With few rays that walk sets the
    // pass's duration and the per-lane kernels finish first; with many, the wave kernels' shared node loads
    // win.  Shadow pass, per-lane / wave (ms), on 7.2M triangles (1.1M in brackets):
    //   1 light   0.52M samples 0.29 / 0.43 (0.22 / 0.32), 2.07M 0.49 / 0.47 (0.38 / 0.32), 8.3M 1.33 / 0.67
    //   4 lights  0.13M samples 0.33 / 0.62 (0.26 / 0.39), 0.52M 0.50 / 0.62 (0.45 / 0.46), 2.07M 1.28 / 0.88
    //             (1.15 / 0.61), 8.3M 4.2 / 1.8 (3.5 / 1.5); with a packet's lights walked in turn by one wave, and
    //             a sample's by one lane: 0.52M 0.84 / 1.36 (0.61 / 1.01), 2.07M 1.54 / 1.33 (1.28 / 0.88)
    //   rect light, 1 sample per pixel at 1080p 0.56 / 0.58 (0.34 / 0.40), 2 samples 0.71 / 0.58 (0.48 / 0.45), 1
    //             sample at 2160p 1.17 / 0.88 (0.88 / 0.69)
    // Two-level structures cross somewhat earlier; the same lines serve them (per-lane / wave on 1.1M triangles, 200K in
    // brackets):
    //   1 light   0.92M samples 0.35 / 0.35 (0.25 / 0.25), 2.07M 0.51 / 0.32 (0.35 / 0.29)
    //   2 lights  0.52M 0.42 / 0.37 (0.26 / 0.31), 0.92M 0.52 / 0.44 (0.32 / 0.30), 2.07M 0.82 / 0.46 (0.50 / 0.35)
    //   4 lights  0.23M 0.40 / 0.45 (0.23 / 0.32), 0.52M 0.60 / 0.48 (0.33 / 0.32), 0.92M 0.87 / 0.55 (0.45 / 0.34)
    //   rect light, 1.8M rays 0.36 / 0.40 (0.21 / 0.27), 3.7M 0.57 / 0.46 (0.28 / 0.31), 8.3M 0.90 / 0.61 (0.42 / 0.40), 16.6M
    //             1.69 / 1.13 (0.73 / 0.60), 133M 9.76 / 5.47 (3.31 / 2.24)
    const uint64_t n_samples_img = (uint64_t)cam.width * cam.height * cam.ssaa * cam.ssaa;
    const bool big_point = rc_wave_work(n_samples_img, (uint64_t)L.n_point) >= RC_WAVE_WORK;
    const bool big_rect = n_samples_img * (uint64_t)(L.has_rect ? L.area_samples : 0) >= 3000000u;
    const bool wave_point = wave_ok && (kernels == RC_KERNELS_WAVE || big_point);
    const bool wave_rect = wave_ok && (kernels == RC_KERNELS_WAVE || big_rect);
    // one unit of work per sample and light in the per-lane kernel too, where the unit count fits 32 bits; but two lights
    // of a small tree in turn, whose walks are too short for a second claim and set-up to pay (units / in turn, ms, 2
    // lights: 1.3K triangles 0.3M samples 0.095 / 0.085, 1.15M 0.195 / 0.166; 20K 0.77M 0.172 / 0.151, 1.15M 0.197 / 0.164; 60K
    // 1.15M 0.202 / 0.173; 3 lights within 4%, 200K triangles faster as units)
    const bool split = (L.n_point > 2 || (L.n_point == 2 && sc.n_tris >= 100000u)) &&
                       (uint64_t)P.n_items * (uint64_t)L.n_point < (1ull << 31);
    P.light_groups = split ? (uint32_t)L.n_point : 1u;
    const bool turn = L.n_point > 1 && point_lights_in_turn(sc, n_samples_img);   // wave-uniform
    const bool quad_point = kernels == RC_KERNELS_AUTO && quad_ok(sc, w, (uint64_t)P.n_items * (uint64_t)L.n_point, MODE_POINT);
    const bool quad_rect = kernels == RC_KERNELS_AUTO && L.has_rect &&
                           quad_ok(sc, w, (uint64_t)P.n_items * (uint64_t)L.area_samples, MODE_RECT);
    P.setup = setup;
    if (L.n_point > 0 || L.has_rect) {
        // one setup entry per sample of the image (the item count is padded to whole tiles); every shadow kernel
        // reads its rays' origins and normals from there
        const uint32_t n_samples = (uint32_t)(cam.width * cam.height * cam.ssaa * cam.ssaa);
        hipLaunchKernelGGL(k_shadow_setup, dim3((n_samples + 255) / 256), dim3(256), 0, st, sc, cam, gbuf, n_samples,
                           setup, L.n_point > 0 && (quad_point || (wave_point ? !turn : split)) ? mask : nullptr);
    }
    if (L.n_point > 0) {
        P.slot = 1;
        if (quad_point) {
            const dim3 g(quad_grid(P.n_items, (uint32_t)L.n_point));
            RC_LAUNCH_TW((k_quad<MODE_POINT, RC_TWO, RC_WT>), g, dim3(64), quad_lds(sc), st, P, (uint32_t*)nullptr);
        } else if (wave_point) {
            P.claim = claim_size((uint64_t)((P.n_items + 63) / 64) * (turn ? 1u : (uint64_t)L.n_point), grid, 64, 1, 4);
#define RC_POINT_WAVE(BIG_, COUNT_)                                                                                        \
    do {                                                                                                               \
        if (turn)                                                                                                      \
            RC_LAUNCH_TW((k_point_wave<RC_TWO, RC_WT, BIG_, COUNT_, true>), dim3(grid), dim3(BLOCK), 0, st, P,         \
                         (const float4*)setup);                                                                        \
        else                                                                                                           \
            RC_LAUNCH_TW((k_point_wave<RC_TWO, RC_WT, BIG_, COUNT_, false>), dim3(grid), dim3(BLOCK), 0, st, P,        \
                         (const float4*)setup);                                                                        \
    } while (0)
            if (sc.max_stack <= 64) {
                if (count) RC_POINT_WAVE(false, true);
                else RC_POINT_WAVE(false, false);
            } else {
                if (count) RC_POINT_WAVE(true, true);
                else RC_POINT_WAVE(true, false);
            }
#undef RC_POINT_WAVE
        } else {
            P.claim = claim_size((uint64_t)P.n_items * P.light_groups, grid, 16, 32, 128);
            if (count)
                RC_LAUNCH_TW((k_trace<MODE_POINT, RC_TWO, RC_WT, true>), dim3(grid), dim3(BLOCK), lds_bytes<MODE_POINT>(), st, P);
            else
                RC_LAUNCH_TW((k_trace<MODE_POINT, RC_TWO, RC_WT, false>), dim3(grid), dim3(BLOCK), lds_bytes<MODE_POINT>(), st, P);
        }
    }
    if (L.has_rect) {
        // unit normal of the emitting side, from FP64 and rounded once
        double eu[3] = {L.rect[3], L.rect[4], L.rect[5]}, ev[3] = {L.rect[6], L.rect[7], L.rect[8]};
        double n[3] = {eu[1] * ev[2] - eu[2] * ev[1], eu[2] * ev[0] - eu[0] * ev[2], eu[0] * ev[1] - eu[1] * ev[0]};
        double len = sqrt(n[0] * n[0] + n[1] * n[1] + n[2] * n[2]);
        for (int a = 0; a < 3; ++a) P.nL[a] = (float)(n[a] / len);
        P.slot = 2;
        const uint64_t n_packets = ((uint64_t)P.n_items * (uint64_t)L.area_samples + 63) / 64;
        P.claim = claim_size(n_packets, grid, 64, 1, 4);
        uint32_t n_pix = (uint32_t)(cam.width * cam.height);
        rc_launch_fill_u32(counts, 0u, n_pix, st);
        // the wave-uniform traversal: a wave holds the samples of one pixel, or of 64 / N neighbouring
        // pixels, whose rays start close together
        if (quad_rect) {
            const dim3 g(quad_grid((uint64_t)P.n_items * (uint64_t)L.area_samples, 1));
            RC_LAUNCH_TW((k_quad<MODE_RECT, RC_TWO, RC_WT>), g, dim3(64), quad_lds(sc), st, P, counts);
        } else if (wave_rect) {
            if (sc.max_stack <= 64) {
                if (count)
                    RC_LAUNCH_TW((k_rect_wave<RC_TWO, RC_WT, false, true>), dim3(grid), dim3(BLOCK), 0, st, P, counts,
                                 (const float4*)setup);
                else
                    RC_LAUNCH_TW((k_rect_wave<RC_TWO, RC_WT, false, false>), dim3(grid), dim3(BLOCK), 0, st, P, counts,
                                 (const float4*)setup);
            } else {
                if (count)
                    RC_LAUNCH_TW((k_rect_wave<RC_TWO, RC_WT, true, true>), dim3(grid), dim3(BLOCK), 0, st, P, counts,
                                 (const float4*)setup);
                else
                    RC_LAUNCH_TW((k_rect_wave<RC_TWO, RC_WT, true, false>), dim3(grid), dim3(BLOCK), 0, st, P, counts,
                                 (const float4*)setup);
            }
        } else {
            const size_t lds = TravStack<SL, BLOCK, false>::lds_bytes();
            if (count)
                RC_LAUNCH_TW((k_rect_packets<RC_TWO, RC_WT, true>), dim3(grid), dim3(BLOCK), lds, st, P, counts);
            else
                RC_LAUNCH_TW((k_rect_packets<RC_TWO, RC_WT, false>), dim3(grid), dim3(BLOCK), lds, st, P, counts);
        }
        hipLaunchKernelGGL(k_rect_finish, dim3((n_pix + 255) / 256), dim3(256), 0, st, counts, n_pix,
                           (uint32_t)L.area_samples, visibility);
    }
}
