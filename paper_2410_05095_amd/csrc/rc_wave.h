// Wave-uniform any-hit traversal of the 4-wide BVH: the 64 rays of a wave walk the tree together, node and triangle
// records read once per wave through the scalar cache, the stack held one entry per lane in registers.  Shared by
// the single-view shadow kernels and the batched ones.
#pragma once

#include "rc_trav.h"

#ifndef RC_SKIP_EMPTY
#define RC_SKIP_EMPTY 1   // the wave walk skips the slab tests of empty child slots 2 and 3
#endif

namespace {

typedef float rc_v4f __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(4))) rc_v4f rc_const_v4f;
typedef float rc_v8f __attribute__((ext_vector_type(8)));
typedef const __attribute__((address_space(4))) rc_v8f rc_const_v8f;
typedef uint32_t rc_v4u __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(4))) rc_v4u rc_const_v4u;

extern "C" __device__ uint32_t __ockl_wfred_max_u32(uint32_t);   // ROCm device library: wavefront maximum
// the compiler intrinsic behind v_writelane_b32 (no clang builtin in this toolchain): returns `old` with lane
// `lane` (wave-uniform) replaced by the wave-uniform `value`
extern "C" __device__ int rc_writelane(int value, int lane, int old) __asm("llvm.amdgcn.writelane.i32");

#define RC_KEY_MISS 0x7F800000u   // keys >= this: no live ray enters the child

// The child's key when any lane enters it: lane 0's entry distance (every lane computes one, hit or not, and
// the rays of a wave start at or near one point, so it orders the children about as any hitting lane's would),
// clamped below the miss key; otherwise a miss key.  The entry distance is >= 0, so its bits order like the
// value, and the two low bits carry the slot.  This replaces a select per lane and a find-first-hitting-lane
// by scalar operations (the wave kernel is bound by vector issue), and measured slightly fewer node visits.
__device__ inline uint32_t wave_key(bool hit, float t0, uint32_t slot)
{
    const uint64_t m = __ballot(hit);
    const uint32_t k0 = min((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(t0), 0) & 0x7FFFFFFCu, 0x7F7FFFFCu);
    return m != 0 ? (k0 | slot) : (RC_KEY_MISS | slot);
}

// Slab test of the wave kernels for a segment 0 < t < 1: entry and exit distance each clamped to [0, 1] (the
// clamp modifiers of v_max3 and v_min3, no instruction) and compared strictly, so that a box left before t = 0
// (exit 0) or entered after t = 1 (entry 1) fails: 6 FMAs, v_max3, v_min3 and a compare.  A box that the segment
// enters passes: its entry is computed below 1 (rc_ray_inv<true>), its exit is above 0 and, by the outward far
// constants, above its entry.  (Clamping the entry alone, entry <= exit, had accepted every box whose exit lies
// beyond t = 1, met or missed: towards a light amid the geometry, one walk could visit the whole tree.  4 point
// lights, 1080p, 2x2 samples, 1.1M triangles: shadow pass 154.7 ms then, 1.42 ms now.)  Finished and idle lanes carry far-plane
// addends of -inf (wave_mute), so their exit is 0 (NaN clamps to 0 as well) and no box accepts them.
__device__ inline bool rc_slab_seg(const TravRay& r, float nx, float ny, float nz, float fx, float fy, float fz,
                                   float& t0)
{
    const float u = fmaxf(fmaxf(fmaf(nx, r.inv[0], r.cn[0]), fmaf(ny, r.inv[1], r.cn[1])), fmaf(nz, r.inv[2], r.cn[2]));
    t0 = __builtin_amdgcn_fmed3f(u, 0.0f, 1.0f);
    const float v = fminf(fminf(fmaf(fx, r.invf[0], r.cf[0]), fmaf(fy, r.invf[1], r.cf[1])), fmaf(fz, r.invf[2], r.cf[2]));
    const float t1 = __builtin_amdgcn_fmed3f(v, 0.0f, 1.0f);
    return t0 < t1;
}

// A lane whose ray is finished (live == 0) takes part in no slab test: its far-plane addends become -inf.  An
// idle lane's traversal constants were never set (set == false): they become 0 first, so that every far
// distance is -inf (or NaN for an infinite plane) and the exit clamps to 0.
__device__ inline void wave_mute(TravRay& r, uint32_t live, bool set)
{
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        if (!set) {
            r.inv[a] = 0.0f;
            r.cn[a] = 0.0f;
            r.invf[a] = 0.0f;
        }
        r.cf[a] = live != 0u ? r.cf[a] : -INFINITY;
    }
}

// CLAMP: rc_slab_seg (finished lanes muted); otherwise rc_slab with bound, 1 for live rays and -1 for finished
// ones, which then never hit (t0 >= 0)
template <bool CLAMP>
__device__ inline void wave_keys_uniform(const rc_v4f& nx, const rc_v4f& fx, const rc_v4f& ny, const rc_v4f& fy,
                                         const rc_v4f& nz, const rc_v4f& fz, const TravRay& ray, float bound,
                                         uint32_t key[4])
{
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        float t0;
        const bool hit = CLAMP ? rc_slab_seg(ray, nx[c], ny[c], nz[c], fx[c], fy[c], fz[c], t0)
                                 : rc_slab(ray, ray.invf, nx[c], ny[c], nz[c], fx[c], fy[c], fz[c], bound, t0);
        key[c] = wave_key(hit, t0, (uint32_t)c);
    }
}

// As wave_keys_uniform, for a node whose child words `chw` (wave-uniform) are known: slots 2 and 3 that hold no
// child get a miss key without their slab tests (a uniform branch), since an empty slot's box never hits.
template <bool CLAMP>
__device__ inline void wave_keys_uniform_skip(const rc_v4f& nx, const rc_v4f& fx, const rc_v4f& ny, const rc_v4f& fy,
                                              const rc_v4f& nz, const rc_v4f& fz, const TravRay& ray, float bound,
                                              const uint32_t chw[4], uint32_t key[4])
{
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        if (RC_SKIP_EMPTY && c >= 2 && chw[c] == RC_EMPTY_CHILD) {
            key[c] = RC_KEY_MISS | (uint32_t)c;
            continue;
        }
        float t0;
        const bool hit = CLAMP ? rc_slab_seg(ray, nx[c], ny[c], nz[c], fx[c], fy[c], fz[c], t0)
                                 : rc_slab(ray, ray.invf, nx[c], ny[c], nz[c], fx[c], fy[c], fz[c], bound, t0);
        key[c] = wave_key(hit, t0, (uint32_t)c);
    }
}

template <bool CLAMP>
__device__ inline void wave_keys_mixed(const rc_v4f& lx, const rc_v4f& hx, const rc_v4f& ly, const rc_v4f& hy,
                                       const rc_v4f& lz, const rc_v4f& hz, const TravRay& ray, float bound,
                                       uint32_t key[4])
{
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const float nx = ray.inv[0] >= 0.0f ? lx[c] : hx[c], fx = ray.inv[0] >= 0.0f ? hx[c] : lx[c];
        const float ny = ray.inv[1] >= 0.0f ? ly[c] : hy[c], fy = ray.inv[1] >= 0.0f ? hy[c] : ly[c];
        const float nz = ray.inv[2] >= 0.0f ? lz[c] : hz[c], fz = ray.inv[2] >= 0.0f ? hz[c] : lz[c];
        float t0;
        const bool hit = CLAMP ? rc_slab_seg(ray, nx, ny, nz, fx, fy, fz, t0) : rc_slab(ray, ray.invf, nx, ny, nz, fx, fy, fz, bound, t0);
        key[c] = wave_key(hit, t0, (uint32_t)c);
    }
}

// EXACT walks return the per-lane walk's answer for every ray, not only outside the FP32 band.  The per-lane walk
// tests exactly the triangles of the leaves whose own box rc_slab accepts: the boxes nest, an FMA with a fixed factor
// and addend is monotone in the plane, so rc_slab accepts every box around one that it accepts.  A wave also tests
// triangles of leaves that only other lanes enter, and an FP32 triangle test can report a hit a little outside
// the box.  So
//  - the walk enters every box that rc_slab accepts: wave_ray_exact doubles the margins of rc_slab_seg's constants,
//    which lie within 14 ulp of it otherwise (its entry is then at most rc_slab's, and below it when that is
//    above 0; its exit is above rc_slab's);
//  - a triangle hit counts once rc_slab, with its own constants, has accepted the leaf's box (rc_enters): a few
//    leaves per walk, found through the node that each stack entry came from.
__device__ inline void wave_ray_exact(TravRay& r)
{
    rc_ray_inv<true>(r);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        r.cn[a] -= fabsf(r.cn[a]) * 0x1p-21f + 0x1p-120f;
        r.cf[a] += fabsf(r.cf[a]) * 0x1p-21f + 0x1p-120f;
    }
}

// Whether the per-lane walk's box test (rc_slab, segment 0 <= t <= 1) lets the ray into the child `w` of a node.
__device__ inline bool rc_enters(const char* node, uint32_t w, const TravRay& ray)
{
    typedef const __attribute__((address_space(4))) float c_float;
    const rc_v4u ch = *(rc_const_v4u*)(const void*)(node + 96);
    const char* lo = node + (ch[0] == w ? 0u : ch[1] == w ? 4u : ch[2] == w ? 8u : 12u);
    TravRay q;
    float n[3], f[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) { q.o[a] = ray.o[a]; q.d[a] = ray.d[a]; }
    rc_ray_inv(q);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const float l = *(c_float*)(const void*)(lo + 32 * a), h = *(c_float*)(const void*)(lo + 32 * a + 16);
        n[a] = q.inv[a] >= 0.0f ? l : h;
        f[a] = q.inv[a] >= 0.0f ? h : l;
    }
    float t0;
    return rc_slab(q, q.invf, n[0], n[1], n[2], f[0], f[1], f[2], 1.0f, t0);
}

// Two-level structures: at a top-level leaf every lane maps its ray into the instance (rc_map_ray), the
// wave pushes an end marker and descends into the instance's tree; popping the marker restores the world
// rays (and the wave's octant).
// The walk of wave_occluded.  BIG: the stack spans two registers (128 entries); otherwise one (64 entries,
// when 3 x depth + 1 <= 64).
// OCT: 0..7, every busy ray in that direction octant (fixed for the whole walk, as in flat trees): the node's
// plane blocks come with three 32-byte loads at constant offsets and the near/far choice is made when
// compiling; 8: mixed octants (each lane picks its planes); -1: decided at run time, per instance for
// two-level structures (the mapped rays' octant changes at each instance).
template <bool WT, bool BIG, bool CLAMP, bool COUNT, bool EXACT = false>
__device__ __attribute__((always_inline)) inline uint32_t wave_walk_flat(const DevScene& sc, const char* nodes_b,
                                                                       const char* tris_b, TravRay& ray, bool busy,
                                                                       uint32_t& node_visits, uint32_t& tri_tests,
                                                                       uint32_t* error_flag, uint32_t root);

// CLAMP: the slab test rc_slab_seg with muted lanes (flat trees, Moller-Trumbore: 10 vector operations per child
// instead of 12); otherwise rc_slab with a bound per lane (two-level structures and the watertight test, whose
// walks hold more registers and measured slower with the muting)
// COUNT: the walk counts node visits and triangle tests of live lanes (frames timed by stage report them)
// EXACT: the per-lane walk's decisions (see wave_ray_exact; flat trees)
template <bool TWO, bool WT, bool BIG, int OCT, bool CLAMP, bool COUNT, bool EXACT = false>
__device__ __attribute__((always_inline)) inline uint32_t wave_walk(const DevScene& sc, const char* nodes_b,
                                                                  const char* tris_b, TravRay& ray, bool busy,
                                                                  uint32_t& node_visits, uint32_t& tri_tests,
                                                                  uint32_t* error_flag, uint32_t root)
{
    const uint32_t lane = __lane_id();
    const uint64_t busy_mask = __ballot(busy);
    uint32_t oct = 0, on0 = 0, on1 = 32, on2 = 64, of0 = 16, of1 = 48, of2 = 80;
    bool uniform_oct = false;
    auto set_octant = [&]() {
        const uint32_t my_oct = (ray.inv[0] < 0.0f ? 1u : 0u) | (ray.inv[1] < 0.0f ? 2u : 0u) |
                                (ray.inv[2] < 0.0f ? 4u : 0u);
        oct = 0;
        if (busy_mask != 0) oct = (uint32_t)__builtin_amdgcn_readlane((int)my_oct, __builtin_ctzll(busy_mask));
        uniform_oct = __ballot(busy && my_oct != oct) == 0;
        // byte offsets of the near- and far-plane blocks (axis a: lo at 32 a, hi at 32 a + 16)
        on0 = (oct & 1u) ? 16u : 0u;
        on1 = (oct & 2u) ? 48u : 32u;
        on2 = (oct & 4u) ? 80u : 64u;
        of0 = on0 ^ 16u;
        of1 = on1 ^ 16u;
        of2 = on2 ^ 16u;
        // opaque to the compiler (no instruction): keeps node + offset in the scalar-offset form of the loads
        asm volatile("" : "+s"(on0), "+s"(on1), "+s"(on2), "+s"(of0), "+s"(of1), "+s"(of2));
    };
    if constexpr (OCT < 0) set_octant();
    float wo[3] = {ray.o[0], ray.o[1], ray.o[2]}, wd[3] = {ray.d[0], ray.d[1], ray.d[2]};   // world ray
    // per-lane state as 32-bit words: occ (an occluder found) and live (busy and not occluded); lanes that
    // are not live take part in no slab test (muted, or bound = -1)
    uint32_t occ = 0u, live = busy ? 1u : 0u;
    float bound = busy ? 1.0f : -1.0f;
    if constexpr (CLAMP) wave_mute(ray, live, busy);
    uint32_t cur = busy_mask != 0 ? (TWO ? sc.tlas_root : root) : RC_STACK_EMPTY;
    int sp = 0;
    uint32_t stk0 = 0, stk1 = 0;   // entry e of the wave's stack lives in lane e % 64 of stk{e / 64}
    uint32_t up0 = 0, up1 = 0;     // EXACT: the node that holds each entry's child word
    uint32_t up = 0;               // EXACT: the node that holds `cur`, or ~0 if it was popped (then entry sp's)
    // next entry of the wave's stack
    auto pop_next = [&]() -> uint32_t {
        if (sp == 0) return RC_STACK_EMPTY;
        --sp;
        if constexpr (EXACT) up = 0xFFFFFFFFu;
        return BIG ? (uint32_t)__builtin_amdgcn_readlane((int)(sp < 64 ? stk0 : stk1), sp & 63)
                   : (uint32_t)__builtin_amdgcn_readlane((int)stk0, sp);
    };
    auto push_entry = [&](uint32_t w) {
        if (sp < 64) {
            stk0 = (uint32_t)rc_writelane((int)w, sp, (int)stk0);
            if constexpr (EXACT) up0 = (uint32_t)rc_writelane((int)cur, sp, (int)up0);
            ++sp;
        } else if (BIG && sp < 128) {
            stk1 = (uint32_t)rc_writelane((int)w, sp - 64, (int)stk1);
            if constexpr (EXACT) up1 = (uint32_t)rc_writelane((int)cur, sp - 64, (int)up1);
            ++sp;
        } else if (lane == 0) {
            *error_flag = 1u;   // beyond the bound the host checked: entry dropped, reported
        }
    };
    while (cur != RC_STACK_EMPTY) {
        if (!rc_is_leaf(cur)) {
            // 32-bit byte offsets into the node array (the host keeps it below 4 GiB for this kernel), so
            // that each block load takes its offset in a scalar register
            const uint32_t nofs = cur << 7;
            auto blk = [&](uint32_t off) { return *(rc_const_v4f*)(const void*)(nodes_b + (uint32_t)(nofs + off)); };
            uint32_t key[4];
            if constexpr (OCT >= 0) {
                // axis a: lo[4] then hi[4] in one 32-byte block at 32 a
                const char* np = nodes_b + nofs;
                const rc_v8f X = *(rc_const_v8f*)(const void*)np, Y = *(rc_const_v8f*)(const void*)(np + 32),
                             Z = *(rc_const_v8f*)(const void*)(np + 64);
                const rc_v4f lx = X.lo, hx = X.hi, ly = Y.lo, hy = Y.hi, lz = Z.lo, hz = Z.hi;
                if constexpr (OCT < 8) {
                    const rc_v4u cw = *(rc_const_v4u*)(const void*)(np + 96);
                    const uint32_t cws[4] = {cw[0], cw[1], cw[2], cw[3]};
                    wave_keys_uniform_skip<CLAMP>((OCT & 1) ? hx : lx, (OCT & 1) ? lx : hx, (OCT & 2) ? hy : ly,
                                           (OCT & 2) ? ly : hy, (OCT & 4) ? hz : lz, (OCT & 4) ? lz : hz, ray, bound,
                                           cws, key);
                } else
                    wave_keys_mixed<CLAMP>(lx, hx, ly, hy, lz, hz, ray, bound, key);
            } else if (uniform_oct) {
                wave_keys_uniform<CLAMP>(blk(on0), blk(of0), blk(on1), blk(of1), blk(on2), blk(of2), ray, bound, key);
            } else {
                wave_keys_mixed<CLAMP>(blk(0), blk(16), blk(32), blk(48), blk(64), blk(80), ray, bound, key);
            }
            if constexpr (COUNT) node_visits += live;
#define RC_CS(a, b)                                                                   \
{                                                                                 \
    const uint32_t lo = min(key[a], key[b]), hi = max(key[a], key[b]);            \
    key[a] = lo; key[b] = hi;                                                     \
}
            RC_CS(0, 1) RC_CS(2, 3) RC_CS(0, 2) RC_CS(1, 3) RC_CS(1, 2)
#undef RC_CS
            const rc_v4u chw = OCT >= 0 ? *(rc_const_v4u*)(const void*)(nodes_b + nofs + 96u)
                                        : *(rc_const_v4u*)(const void*)(nodes_b + (uint32_t)(nofs + 96u));
            const uint64_t c01 = ((uint64_t)chw[1] << 32) | chw[0], c23 = ((uint64_t)chw[3] << 32) | chw[2];
            auto child = [&](uint32_t k) {
                const uint64_t pr = (k & 2u) ? c23 : c01;
                return (k & 1u) ? (uint32_t)(pr >> 32) : (uint32_t)pr;
            };
            if (sp <= 61) {
                // room for the (at most 3) pushes of this node in the first stack register
#pragma unroll
                for (int c = 3; c >= 1; --c)
                    if (key[c] < RC_KEY_MISS) {
                        stk0 = (uint32_t)rc_writelane((int)child(key[c]), sp, (int)stk0);
                        if constexpr (EXACT) up0 = (uint32_t)rc_writelane((int)cur, sp, (int)up0);
                        ++sp;
                    }
            } else {
#pragma unroll
                for (int c = 3; c >= 1; --c)
                    if (key[c] < RC_KEY_MISS) push_entry(child(key[c]));
            }
            if constexpr (EXACT) up = cur;
            cur = key[0] < RC_KEY_MISS ? child(key[0]) : pop_next();
        } else if (TWO) {
            // top-level leaf: every ray mapped into the instance, whose tree the flat walk takes (compiled for
            // the mapped rays' octant, with a stack of its own) for the rays still live; then back to world
            // space
            rc_const_v4f* ip = (rc_const_v4f*)(const void*)(sc.inst + rc_leaf_first(cur));
            const rc_v4f q0 = ip[0], q1 = ip[1], q2 = ip[2], q3 = ip[3];
            const float W[12] = {q0[0], q0[1], q0[2], q0[3], q1[0], q1[1], q1[2], q1[3],
                                 q2[0], q2[1], q2[2], q2[3]};
            rc_map_ray(W, wo, wd, ray);
            const uint32_t ob = wave_walk_flat<WT, false, false, COUNT>(sc, nodes_b, tris_b, ray, live != 0u, node_visits,
                                                          tri_tests, error_flag, __float_as_uint(q3[0]));
            occ |= ob;
            live &= ob ^ 1u;
#pragma unroll
            for (int a = 0; a < 3; ++a) { ray.o[a] = wo[a]; ray.d[a] = wd[a]; }
            rc_ray_inv(ray);
            bound = live != 0u ? bound : -1.0f;
            cur = __ballot(live != 0u) == 0 ? RC_STACK_EMPTY : pop_next();
        } else {
            // every lane tests every triangle of the leaf, without lane branches: a finished lane only
            // repeats work (its flag stays set; idle lanes' flags are never read), and the counter
            // takes the tests of live lanes
            const uint32_t first = rc_leaf_first(cur), cnt = rc_leaf_count(cur);
            const uint32_t tofs = first * 48u;   // 32-bit byte offset (the host keeps the array below 4 GiB)
            uint32_t o = occ;
            for (uint32_t i = 0; i < cnt; ++i) {
                rc_const_v4f* tp = (rc_const_v4f*)(const void*)(tris_b + (uint32_t)(tofs + 48u * i));
                const rc_v4f A = tp[0], B = tp[1], C = tp[2];
                if constexpr (COUNT) tri_tests += live & (o ^ 1u);
                const bool hit = WT ? rc_wt_segment(ray, A.x, A.y, A.z, B.x, B.y, B.z, C.x, C.y, C.z)
                                    : rc_mt_segment(ray, A.x, A.y, A.z, B.x, B.y, B.z, C.x, C.y, C.z);
                o |= hit ? 1u : 0u;
            }
            if constexpr (EXACT) {
                const uint32_t fresh = o ^ occ;
                if (__ballot(fresh != 0u) != 0) {
                    const uint32_t e = BIG && sp >= 64 ? (uint32_t)__builtin_amdgcn_readlane((int)up1, sp - 64)
                                                       : (uint32_t)__builtin_amdgcn_readlane((int)up0, sp & 63);
                    const char* node = nodes_b + ((up != 0xFFFFFFFFu ? up : e) << 7);
                    o = occ | (rc_enters(node, cur, ray) ? fresh : 0u);
                }
            }
            occ = o;
            live &= o ^ 1u;
            if constexpr (CLAMP) wave_mute(ray, live, true);
            else bound = live != 0u ? bound : -1.0f;
            cur = __ballot(live != 0u) == 0 ? RC_STACK_EMPTY : pop_next();
        }
        cur = __builtin_amdgcn_readfirstlane(cur);
    }
    return occ;
}

// Any-hit traversal of the segments o + t d, 0 <= t <= 1, of a wave's rays (called by all 64 lanes; busy
// lanes hold a ray whose traversal constants rc_ray_inv set): returns 1 in the lanes whose segment is
// occluded.  Flat trees: one walk specialised for the wave's octant, or for mixed octants.  EXACT: constants
// set by wave_ray_exact, the per-lane walk's answers.
template <bool TWO, bool WT, bool BIG, bool COUNT, bool EXACT = false>
__device__ __attribute__((always_inline)) inline uint32_t wave_occluded(const DevScene& sc, const char* nodes_b,
                                                                      const char* tris_b, TravRay& ray, bool busy,
                                                                      uint32_t& node_visits, uint32_t& tri_tests,
                                                                      uint32_t* error_flag)
{
    if constexpr (TWO)
        return wave_walk<TWO, WT, BIG, -1, false, COUNT>(sc, nodes_b, tris_b, ray, busy, node_visits, tri_tests, error_flag,
                                                        0u);
    else
        return wave_walk_flat<WT, BIG, !WT, COUNT, EXACT>(sc, nodes_b, tris_b, ray, busy, node_visits, tri_tests, error_flag, 0u);
}

// The flat walk from node `root`, compiled once per direction octant of the busy rays and once for mixed
// octants.  For two-level structures it walks an instance's tree with a one-register stack: the host takes
// the wave kernels only when 3 x (deepest instance tree + 24) + 2 <= 128, so an instance tree is at most 18
// levels deep and its walk needs at most 55 stack entries.
template <bool WT, bool BIG, bool CLAMP, bool COUNT, bool EXACT>
__device__ __attribute__((always_inline)) inline uint32_t wave_walk_flat(const DevScene& sc, const char* nodes_b,
                                                                       const char* tris_b, TravRay& ray, bool busy,
                                                                       uint32_t& node_visits, uint32_t& tri_tests,
                                                                       uint32_t* error_flag, uint32_t root)
{
#define RC_WALK(o) \
    wave_walk<false, WT, BIG, o, CLAMP, COUNT, EXACT>(sc, nodes_b, tris_b, ray, busy, node_visits, tri_tests, error_flag, root)
    const uint64_t busy_mask = __ballot(busy);
    const uint32_t my_oct = (ray.inv[0] < 0.0f ? 1u : 0u) | (ray.inv[1] < 0.0f ? 2u : 0u) |
                            (ray.inv[2] < 0.0f ? 4u : 0u);
    const uint32_t oct = busy_mask != 0
                             ? (uint32_t)__builtin_amdgcn_readlane((int)my_oct, __builtin_ctzll(busy_mask))
                             : 0u;
    if (__ballot(busy && my_oct != oct) != 0) return RC_WALK(8);
    switch (oct) {
    case 0: return RC_WALK(0);
    case 1: return RC_WALK(1);
    case 2: return RC_WALK(2);
    case 3: return RC_WALK(3);
    case 4: return RC_WALK(4);
    case 5: return RC_WALK(5);
    case 6: return RC_WALK(6);
    default: return RC_WALK(7);
    }
#undef RC_WALK
}

}  // namespace
