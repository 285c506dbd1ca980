// U-Net shadow-denoiser kernels for gfx950: BF16 storage, FP32 accumulation.
//
// 3x3 convolutions are implicit GEMMs on the matrix cores (v_mfma_f32_16x16x32_bf16):
//   forward      out[p][co] = sum_{tap,ci} in[p + off(tap)][ci] * W[co][tap][ci]     (M = pixels, N = Cout)
//   input grad   gin[p][ci] = sum_{tap,co} g[p - off(tap)][co] * W[co][tap][ci]      = the forward kernel
//                with the flipped, transposed weights Wf[ci][8 - tap][co]
//   weight grad  dW[co][tap][ci] = sum_p g[p][co] * in[p + off(tap)][ci]            (K = pixels, split over
//                chunks; the per-chunk partials are summed in chunk order, so the result is deterministic)
// Tensors are NHWC; every reduction (bias, head, loss) is a fixed-order two-stage sum.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <stdint.h>

#include "rc_unet.h"

#ifndef RC_CONV_ROWS
#define RC_CONV_ROWS 8   // output rows per wave of the row-blocked convolution
#endif
// minimum waves per SIMD the compiler keeps the convolution kernels to (their register budget)
#ifndef RC_OCC_E1A
#define RC_OCC_E1A 4
#endif
#ifndef RC_OCC_ROWS
#define RC_OCC_ROWS 2
#endif
#ifndef RC_OCC_416
#define RC_OCC_416 3
#endif
#ifndef RC_OCC_816
#define RC_OCC_816 2
#endif

namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

__device__ inline uint16_t f2bf(float f)
{
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);   // round to nearest even
    return (uint16_t)(u >> 16);
}
__device__ inline float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

__device__ inline bf16x8 load8(const uint16_t* p) { return __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(p)); }

__device__ inline void unpack8(uint4 v, float f[8])
{
    uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        f[2 * e] = __uint_as_float(w[e] << 16);
        f[2 * e + 1] = __uint_as_float(w[e] & 0xFFFF0000u);
    }
}
__device__ inline uint4 pack8(const float f[8])
{
    uint32_t w[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) w[e] = (uint32_t)f2bf(f[2 * e]) | ((uint32_t)f2bf(f[2 * e + 1]) << 16);
    return make_uint4(w[0], w[1], w[2], w[3]);
}

// 2x2 average pool of four 8-channel groups: a = (2y, 2x), b = (2y, 2x + 1), c = (2y + 1, 2x),
// d = (2y + 1, 2x + 1), as ((a + b) + (c + d)) / 4 rounded to BF16
__device__ inline uint4 pool4(uint4 a, uint4 b, uint4 c, uint4 d)
{
    float fa[8], fb[8], fc[8], fd[8], r[8];
    unpack8(a, fa); unpack8(b, fb); unpack8(c, fc); unpack8(d, fd);
#pragma unroll
    for (int e = 0; e < 8; ++e) r[e] = ((fa[e] + fb[e]) + (fc[e] + fd[e])) * 0.25f;
    return pack8(r);
}

// the 1x1 head on one pixel's 32 BF16 channels (FP32, channels in order, weights rounded to BF16), then the
// sigmoid
__device__ inline float head_value(const float f[32], const float* wh, const float* bh)
{
    float s = 0.0f;
#pragma unroll
    for (int c = 0; c < 32; ++c) s = fmaf(f[c], bf2f(f2bf(wh[c])), s);
    s += bh[0];
    return 1.0f / (1.0f + expf(-s));
}

// ---------------------------------------------------------------- 3x3 convolution
// Each wave computes 32 pixels (two 16-row MFMA tiles) x 16*NT output channels; a block has 4 waves.
template <int NT>
__global__ __launch_bounds__(256) void k_conv3x3(ConvArgs a)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int P = a.N * a.H * a.W;
    const int p0 = (blockIdx.x * 4 + wave) * 32;
    if (p0 >= P) return;
    const int K = 9 * a.Cin;
    const int r = lane & 15, g = lane >> 4;
    int ny[2], yy[2], xx[2];
    bool pv[2];
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) {
        int p = p0 + 16 * mt + r;
        pv[mt] = p < P;
        int q = pv[mt] ? p : 0;
        xx[mt] = q % a.W;
        int t = q / a.W;
        yy[mt] = t % a.H;
        ny[mt] = t / a.H;
    }
    f32x4 acc[2][NT];
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
    const bf16x8 zero = {};
    for (int k0 = 0; k0 < K; k0 += 32) {
        const int kk = k0 + 8 * g;
        const bool kv = kk < K;
        const int tap = kv ? kk / a.Cin : 0;
        const int ci = kk - tap * a.Cin;
        const int dy = tap / 3 - 1, dx = tap % 3 - 1;
        bf16x8 A[2], B[NT];
#pragma unroll
        for (int mt = 0; mt < 2; ++mt) {
            int y = yy[mt] + dy, x = xx[mt] + dx;
            bool ok = pv[mt] && kv && y >= 0 && y < a.H && x >= 0 && x < a.W;
            A[mt] = ok ? load8(a.in + ((size_t)(ny[mt] * a.H + y) * a.W + x) * a.Cin + ci) : zero;
        }
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            int co = 16 * nt + r;
            B[nt] = (kv && co < a.Cout) ? load8(a.wt + (size_t)co * K + kk) : zero;
        }
#pragma unroll
        for (int mt = 0; mt < 2; ++mt)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
                acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[mt], B[nt], acc[mt][nt], 0, 0, 0);
    }
    // D layout: lane holds column (channel) 16 nt + (lane & 15), rows (pixels) 4 (lane >> 4) + i
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            int co = 16 * nt + r;
            if (co >= a.Cout) continue;
            float b = a.bias ? a.bias[co] : 0.0f;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                int p = p0 + 16 * mt + 4 * g + i;
                if (p >= P) continue;
                float v = acc[mt][nt][i] + b;
                if (a.relu) v = fmaxf(v, 0.0f);
                size_t o = (size_t)p * a.Cout + co;
                if (a.mask && !(bf2f(a.mask[o]) > 0.0f)) v = 0.0f;
                a.out[o] = f2bf(v);
            }
        }
}

// Tile of workgroup b among n: workgroups are dispatched to the 8 XCDs round-robin (b % 8), so XCD g is
// given the contiguous range of tiles [g q + min(g, r), ...) with q = n / 8, r = n % 8.  Tiles that share
// halo rows then run on the same XCD and meet in its L2.
__device__ inline int xcd_tile(int b, int n)
{
    const int g = b & 7, k = b >> 3, q = n >> 3, r = n & 7;
    return g * q + min(g, r) + k;
}

// One 16-byte group of a convolution's input halo: pixel (y, x) of image n, channels [ci, ci + 8), zero
// outside the image.  The address is formed from the clamped position, so the load is always in bounds and
// needs no branch, and the value is replaced by zero afterwards; a tile's loads can then all be in flight at
// once.  With a second source, channels below Ca come from the 2x nearest-upsampled `in`, the rest from in2.
__device__ inline const uint16_t* group_ptr(const ConvArgs& a, int n, int y, int x, int ci)
{
    if (a.in2 == nullptr) return a.in + ((size_t)(n * a.H + y) * a.W + x) * a.Cin + ci;
    const bool up = ci < a.Ca;
    const size_t ou = ((size_t)(n * (a.H >> 1) + (y >> 1)) * (a.W >> 1) + (x >> 1)) * a.Ca + ci;
    const size_t os = ((size_t)(n * a.H + y) * a.W + x) * (a.Cin - a.Ca) + (ci - a.Ca);
    return (up ? a.in : a.in2) + (up ? ou : os);
}
__device__ inline uint4 halo_group(const ConvArgs& a, int n, int y, int x, int ci)
{
    const bool inb = (unsigned)y < (unsigned)a.H && (unsigned)x < (unsigned)a.W;
    const int yc = min(max(y, 0), a.H - 1), xc = min(max(x, 0), a.W - 1);
    const uint4 v = *reinterpret_cast<const uint4*>(group_ptr(a, n, yc, xc, ci));
    return inb ? v : make_uint4(0u, 0u, 0u, 0u);
}

// 16 zero bytes in device memory: the source of halo groups outside the image for loads that write LDS
// directly
__device__ __align__(16) const uint4 g_zero_group = {0u, 0u, 0u, 0u};

// ---------------------------------------------------------------- 3x3 convolution, LDS-tiled
// Workgroup of 4 waves; output tile = 4 rows x TW = 16 MT columns of one image, wave w computes row w:
// MT 16-pixel M-tiles x NT 16-channel N-tiles.  For each chunk of CC input channels the input halo (6 rows
// x TW + 2 columns) is staged in LDS, zero outside the image, and the 9 taps read their shifted pixels
// from there (each input value is fetched from memory once per tile instead of once per tap).  With SW the
// chunk's weights are staged in LDS too, in MFMA fragment order, and read back with one conflict-free
// 16-byte LDS read per lane and N-tile: the 4 waves then fetch them from memory once per workgroup instead
// of once each per K-step, which pays from 4 N-tiles on; otherwise each wave streams its weight fragments
// through L1 one K-step ahead.  With a second source the halo loader reads channels [0, Ca) from the 2x
// nearest-upsampled low-resolution tensor and the rest from the skip tensor, so the decoder's upsample +
// concat is never materialised.
// SMALL (images that leave CUs idle): the workgroup takes the 16 NT output channels from 16 NT blockIdx.y on, and the
// next chunk's loads are in flight under this chunk's instructions (on large images the registers that they hold cost
// occupancy: 1080x1920 inference 714 against 743 us).
template <int MT, int NT, int CC, bool SW>
struct ConvLds {
    static constexpr int TW = 16 * MT, HW = TW + 2, HR = 6;
    static constexpr int PST = CC + 8;                         // LDS pixel stride in bf16 (bank padding)
    static constexpr int KS = (9 * CC + 31) / 32;              // K-steps of one chunk (zero-padded)
    static constexpr int HALO_U4 = (HR * HW * PST * 2 + 15) / 16;
    static constexpr int W_U4 = SW ? KS * NT * 64 : 0;         // weight fragments of one chunk
    static constexpr size_t bytes()
    {
        const size_t in = (size_t)(HALO_U4 + W_U4) * 16, out = (size_t)4 * TW * (16 * NT + 8) * 2;
        return in > out ? in : out;
    }
};

template <int MT, int NT, int CC, bool SW, int OCC, bool SMALL>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(OCC))) void k_conv_lds(ConvArgs a)
{
    extern __shared__ uint4 conv_lds[];
    using L = ConvLds<MT, NT, CC, SW>;
    constexpr int TW = L::TW, HW = L::HW, HR = L::HR, PST = L::PST, KS = L::KS;
    uint16_t* lds = reinterpret_cast<uint16_t*>(conv_lds);
    uint4* wfrag = conv_lds + L::HALO_U4;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int tiles_x = (a.W + TW - 1) / TW, tiles_y = (a.H + 3) / 4;
    int tt = xcd_tile(blockIdx.x, gridDim.x);
    const int tx = tt % tiles_x;
    tt /= tiles_x;
    const int ty = tt % tiles_y, n = tt / tiles_y;
    const int x0 = tx * TW, y0 = ty * 4;
    const int r = lane & 15, g = lane >> 4;
    const int K = 9 * a.Cin;
    const int co0 = SMALL ? 16 * NT * (int)blockIdx.y : 0;   // output channels [co0, co0 + cn)
    const int cn = SMALL ? min(a.Cout - co0, 16 * NT) : a.Cout;
    f32x4 acc[MT][NT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
    const bf16x8 zero = {};
    constexpr int GROUPS = CC / 8;
    constexpr int HALO_ITEMS = HR * HW * GROUPS;
    // item i of a chunk's halo: pixel i / GROUPS of the (HR x HW) halo, channel group i % GROUPS; item f of its
    // staged weights: lane f % 64 of fragment (K-step, N-tile) f / 64 (output channel 16 nt + (l & 15), the
    // 8 K values from 32 ks + 8 (l >> 4) on, tap = K / CC, input channel c0 + K % CC, zero from 9 CC on).
    // Every thread holds PF halo items and WPF weight items in registers: all of its loads are issued before
    // the first is waited for (loaded one by one, each load's latency would be paid in turn).
    constexpr int PF = (HALO_ITEMS + 255) / 256;
    constexpr int WPF = SW ? (L::W_U4 + 255) / 256 : 0;
    auto halo_item = [&](int c0, int i) -> uint4 {
        const int pix = i / GROUPS;
        return halo_group(a, n, y0 - 1 + pix / HW, x0 - 1 + pix % HW, c0 + 8 * (i % GROUPS));
    };
    auto w_item = [&](int c0, int f) -> uint4 {
        const int l = f & 63, q = f >> 6, nt = q % NT, ks = q / NT;
        const int co = co0 + 16 * nt + (l & 15), kk = 32 * ks + 8 * (l >> 4);
        uint4 v = make_uint4(0u, 0u, 0u, 0u);
        if (kk < 9 * CC && co < a.Cout) {
            const int tap = kk / CC, cl = kk - tap * CC;
            v = *reinterpret_cast<const uint4*>(a.wt + (size_t)co * K + tap * a.Cin + c0 + cl);
        }
        return v;
    };
    uint4 pf[PF];
    uint4 wpf[WPF > 0 ? WPF : 1];
    auto fetch = [&](int c0) {
#pragma unroll
        for (int k = 0; k < PF; ++k) {
            const int i = (int)threadIdx.x + 256 * k;
            pf[k] = (HALO_ITEMS % 256 == 0 || i < HALO_ITEMS) ? halo_item(c0, i) : make_uint4(0u, 0u, 0u, 0u);
        }
#pragma unroll
        for (int k = 0; k < WPF; ++k) {
            const int f = (int)threadIdx.x + 256 * k;
            wpf[k] = (L::W_U4 % 256 == 0 || f < L::W_U4) ? w_item(c0, f) : make_uint4(0u, 0u, 0u, 0u);
        }
    };
    if constexpr (SMALL) fetch(0);
    for (int c0 = 0; c0 < a.Cin; c0 += CC) {
        if constexpr (!SMALL) fetch(c0);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < PF; ++k) {
            const int i = (int)threadIdx.x + 256 * k;
            if (HALO_ITEMS % 256 == 0 || i < HALO_ITEMS)
                *reinterpret_cast<uint4*>(lds + (i / GROUPS) * PST + 8 * (i % GROUPS)) = pf[k];
        }
#pragma unroll
        for (int k = 0; k < WPF; ++k) {
            const int f = (int)threadIdx.x + 256 * k;
            if (L::W_U4 % 256 == 0 || f < L::W_U4) wfrag[f] = wpf[k];
        }
        __syncthreads();
        if (SMALL && c0 + CC < a.Cin) fetch(c0 + CC);   // in flight under this chunk's instructions
        // streamed weights: fragments of K-step ks loaded while the MFMAs of the step before run
        auto load_b = [&](int ks, bf16x8* Bd) {
            const int kk = 32 * ks + 8 * g;
            const bool kv = kk < 9 * CC;
            const int tap = kv ? kk / CC : 0;
            const int cl = kk - tap * CC;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const int co = co0 + 16 * nt + r;
                Bd[nt] = (kv && co < a.Cout) ? load8(a.wt + (size_t)co * K + tap * a.Cin + c0 + cl) : zero;
            }
        };
        bf16x8 B[NT], Bn[NT];
        if constexpr (!SW) load_b(0, B);
        for (int ks = 0; ks < KS; ++ks) {
            if constexpr (SW) {
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) B[nt] = __builtin_bit_cast(bf16x8, wfrag[(ks * NT + nt) * 64 + lane]);
            } else if (ks + 1 < KS) {
                load_b(ks + 1, Bn);
            }
            const int kk = 32 * ks + 8 * g;
            const bool kv = kk < 9 * CC;
            const int tap = kv ? kk / CC : 0;
            const int cl = kk - tap * CC;
            const int dy = tap / 3, dx = tap % 3;
            bf16x8 A[MT];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
                A[mt] = kv ? __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(
                                 lds + ((wave + dy) * HW + 16 * mt + r + dx) * PST + cl))
                           : zero;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
                    acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[mt], B[nt], acc[mt][nt], 0, 0, 0);
            if constexpr (!SW) {
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) B[nt] = Bn[nt];
            }
        }
    }
    // Epilogue through LDS: each wave writes its 16 MT pixels x 16 NT channels (bias, ReLU applied) as
    // bf16 rows of a [pixel][channel] tile, then the tile leaves in 16-byte chunks, consecutive pixels of
    // one image row being contiguous in NHWC.
    constexpr int TC = 16 * NT;                 // channels of the tile
    constexpr int TS = TC + 8;                  // tile row stride (padding spreads the 4 row groups over the banks)
    constexpr int TPX = 16 * MT;                // pixels per wave
    __syncthreads();                            // every wave is done with the halo
    uint16_t* tile = lds + (size_t)wave * TPX * TS;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int co = 16 * nt + r;
        const float b = (a.bias && co < cn) ? a.bias[co0 + co] : 0.0f;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float v = acc[mt][nt][i] + b;
                if (a.relu) v = fmaxf(v, 0.0f);
                tile[(16 * mt + 4 * g + i) * TS + co] = f2bf(v);
            }
    }
    __syncthreads();
    if (a.pool_out) {
        // 2x2 average pool of the tile (rows 0-1 and 2-3 of the 4 waves; tile origin and H, W even)
        const int Hp = a.H / 2, Wp = a.W / 2, c8p = cn / 8;
        for (int q = threadIdx.x; q < 2 * (TPX / 2) * c8p; q += 256) {
            const int pp = q / c8p, c8 = q - pp * c8p;
            const int po = pp / (TPX / 2), px2 = pp % (TPX / 2);
            const int y = y0 + 2 * po, x = x0 + 2 * px2;
            if (x >= a.W || y >= a.H) continue;
            const uint16_t* t0 = lds + (size_t)(2 * po) * TPX * TS + (2 * px2) * TS + 8 * c8;
            const uint4 v = pool4(*reinterpret_cast<const uint4*>(t0), *reinterpret_cast<const uint4*>(t0 + TS),
                                  *reinterpret_cast<const uint4*>(t0 + TPX * TS),
                                  *reinterpret_cast<const uint4*>(t0 + TPX * TS + TS));
            *reinterpret_cast<uint4*>(a.pool_out + ((size_t)(n * Hp + y / 2) * Wp + x / 2) * a.Cout + co0 + 8 * c8) = v;
        }
    }
    const int y = y0 + wave;
    if (y >= a.H) return;
    const int c8n = cn / 8;
    for (int q = lane; q < TPX * c8n; q += 64) {
        const int px = q / c8n, c8 = q - px * c8n;
        const int x = x0 + px;
        if (x >= a.W) continue;
        uint4 v = *reinterpret_cast<const uint4*>(tile + px * TS + 8 * c8);
        const size_t o = ((size_t)(n * a.H + y) * a.W + x) * a.Cout + co0 + 8 * c8;
        if (a.mask) {
            float f[8], mk[8];
            unpack8(v, f);
            unpack8(*reinterpret_cast<const uint4*>(a.mask + o), mk);
#pragma unroll
            for (int e = 0; e < 8; ++e) f[e] = mk[e] > 0.0f ? f[e] : 0.0f;
            v = pack8(f);
        }
        *reinterpret_cast<uint4*>(a.out + o) = v;
    }
}

// ---------------------------------------------------------------- 3x3 convolution, row-blocked
// For up to 32 output channels (NT <= 2) and Cin a multiple of 32.  With one row per wave (k_conv_lds) an
// A fragment read from LDS feeds only NT MFMAs, so these layers wait on LDS reads.  Here each wave owns R
// output rows x 16 pixels and walks the R + 2 halo rows: the fragment of halo row h and horizontal tap dx is
// read once and serves the vertical taps dy = 0, 1, 2 of output rows h - dy (up to 3 NT MFMAs per read).
// Workgroup: 4 waves side by side (tile R rows x 64 columns); the chunk's weights, 9 taps x NT fragments,
// stay in registers.  Each output row still sums its taps in the order tap = 3 dy + dx within a chunk, as
// k_conv_lds does with 32-channel chunks.
//
// Per chunk of 32 input channels the (R + 2) x 66-pixel halo is staged in LDS, 64 bytes per pixel with no
// padding: the four 16-byte channel groups of halo pixel hx sit in the slots g ^ ((hx >> 1) & 3), so that
// the A-fragment reads (16 consecutive pixels x 4 groups) hit distinct banks in every group of 8 lanes.
// The 64 interior pixels of a halo row are read from memory straight into LDS (global_load_lds_dwordx4: one
// instruction per wave and row, lane l landing at the wave's base + 16 l, so lane l fetches the channel
// group that the swizzle puts in its slot; pixels outside the image read g_zero_group); the two edge
// pixels of each row pass through registers.  No halo data occupies vector registers.
template <int R, int NT>
struct ConvRows {
    static constexpr int TW = 64, HW = TW + 2, HR = R + 2, CC = 32, PIX_BYTES = CC * 2;
    static constexpr int W_OFF = HR * HW * PIX_BYTES;   // then the chunk's 9 NT weight fragments, 1 KB each
    static constexpr size_t bytes()
    {
        const size_t in = (size_t)W_OFF + 9 * NT * 1024, out = (size_t)4 * R * 16 * (16 * NT + 8) * 2;
        return in > out ? in : out;
    }
};

__device__ inline int rows_slot_offset(int hx, int g) { return (g ^ ((hx >> 1) & 3)) << 4; }

// the 9 NT weight fragments of chunk c0 straight into LDS at `dst` (fragment f = NT tap + nt, 1 KB each; wave w
// issues every 4th); lane (r, g) of fragment (tap, nt) holds output channel 16 nt + r, input channels
// c0 + 8 g .. + 8 of that tap, zero beyond Cout
template <int NT>
__device__ __attribute__((always_inline)) inline void rows_weights_to_lds(const ConvArgs& a, int c0, char* dst, int wave,
                                                                          int r, int g)
{
    const int K = 9 * a.Cin;
    for (int f = wave; f < 9 * NT; f += 4) {
        const int tap = f / NT, co = 16 * (f % NT) + r;
        const void* src = co < a.Cout ? (const void*)(a.wt + (size_t)co * K + tap * a.Cin + c0 + 8 * g)
                                      : (const void*)&g_zero_group;
        __builtin_amdgcn_global_load_lds(src, dst + f * 1024, 16, 0, 0);
    }
}

template <int R, int NT, int OCC>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(OCC))) void k_conv_rows(ConvArgs a)
{
    extern __shared__ uint4 conv_lds[];
    using L = ConvRows<R, NT>;
    constexpr int TW = L::TW, HW = L::HW, HR = L::HR, CC = L::CC, PB = L::PIX_BYTES;
    static_assert(8 * HR <= 256, "edge items beyond one per thread");
    uint16_t* lds = reinterpret_cast<uint16_t*>(conv_lds);
    char* ldsb = reinterpret_cast<char*>(conv_lds);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int tiles_x = (a.W + TW - 1) / TW, tiles_y = (a.H + R - 1) / R;
    int tt = xcd_tile(blockIdx.x, gridDim.x);
    const int tx = tt % tiles_x;
    tt /= tiles_x;
    const int ty = tt % tiles_y, n = tt / tiles_y;
    const int x0 = tx * TW, y0 = ty * R;
    const int r = lane & 15, g = lane >> 4;
    const int K = 9 * a.Cin;
    // this lane's interior halo group: pixel hx = 1 + 16 wave + (lane >> 2) of every halo row, LDS slot lane & 3
    const int d_hx = 1 + 16 * wave + (lane >> 2);
    const int d_x = x0 - 1 + d_hx;
    const int d_g = (lane & 3) ^ ((d_hx >> 1) & 3);
    // this thread's edge group (threads below 8 HR): halo row t >> 3, pixel 0 or HW - 1, group t & 3
    const int t = threadIdx.x;
    const int e_hy = t >> 3, e_hx = ((t >> 2) & 1) ? HW - 1 : 0, e_g = t & 3;
    const int e_off = (e_hy * HW + e_hx) * PB + rows_slot_offset(e_hx, e_g);
    // byte offsets of this lane's A fragment (pixel 16 wave + r + dx, group g) within a halo row
    int a_off[3];
#pragma unroll
    for (int dx = 0; dx < 3; ++dx) {
        const int hx = 16 * wave + r + dx;
        a_off[dx] = hx * PB + rows_slot_offset(hx, g);
    }
    f32x4 acc[R][NT];
#pragma unroll
    for (int o = 0; o < R; ++o)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[o][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
    const bf16x8 zero = {};
    for (int c0 = 0; c0 < a.Cin; c0 += CC) {
        __syncthreads();   // every wave is done with the previous chunk's halo and weights
        // weight fragment f = NT tap + nt, read once per workgroup straight into LDS: lane l holds output
        // channel 16 nt + (l & 15), input channels c0 + 8 (l >> 4) .. + 8 of that tap
        rows_weights_to_lds<NT>(a, c0, ldsb + L::W_OFF, wave, r, g);
#pragma unroll
        for (int hy = 0; hy < HR; ++hy) {
            const int y = y0 - 1 + hy;
            const bool ok = (unsigned)y < (unsigned)a.H && d_x < a.W;
            const void* src = ok ? (const void*)group_ptr(a, n, y, d_x, c0 + 8 * d_g) : (const void*)&g_zero_group;
            __builtin_amdgcn_global_load_lds(src, ldsb + (hy * HW + 1 + 16 * wave) * PB, 16, 0, 0);
        }
        uint4 ev = make_uint4(0u, 0u, 0u, 0u);
        if (t < 8 * HR) ev = halo_group(a, n, y0 - 1 + e_hy, x0 - 1 + e_hx, c0 + 8 * e_g);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the direct-to-LDS loads have landed
        if (t < 8 * HR) *reinterpret_cast<uint4*>(ldsb + e_off) = ev;
        __syncthreads();
        bf16x8 B[9][NT];
#pragma unroll
        for (int tap = 0; tap < 9; ++tap)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
                B[tap][nt] = __builtin_bit_cast(
                    bf16x8, *reinterpret_cast<const uint4*>(ldsb + L::W_OFF + (tap * NT + nt) * 1024 + lane * 16));
#pragma unroll
        for (int h = 0; h < HR; ++h)
#pragma unroll
            for (int dx = 0; dx < 3; ++dx) {
                const bf16x8 A = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(ldsb + h * HW * PB + a_off[dx]));
#pragma unroll
                for (int dy = 0; dy < 3; ++dy) {
                    const int o = h - dy;
                    if (o >= 0 && o < R) {
#pragma unroll
                        for (int nt = 0; nt < NT; ++nt)
                            acc[o][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, B[3 * dy + dx][nt], acc[o][nt],
                                                                                  0, 0, 0);
                    }
                }
            }
    }
    // epilogue through LDS, as in k_conv_lds: per wave R rows of 16 pixels x 16 NT channels
    constexpr int TC = 16 * NT;
    constexpr int TS = TC + 8;                  // tile row stride (padding spreads the 4 row groups over the banks)
    __syncthreads();
    uint16_t* tile = lds + (size_t)wave * R * 16 * TS;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int co = 16 * nt + r;
        const float b = (a.bias && co < a.Cout) ? a.bias[co] : 0.0f;
#pragma unroll
        for (int o = 0; o < R; ++o)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float v = acc[o][nt][i] + b;
                if (a.relu) v = fmaxf(v, 0.0f);
                tile[(o * 16 + 4 * g + i) * TS + co] = f2bf(v);
            }
    }
    __syncthreads();
    const int c8n = a.Cout / 8;
    if (a.head_out) {
        // the network's head on each pixel of the tile, from the layer's BF16 values, stored (training) or not
        for (int px = lane; px < R * 16; px += 64) {
            const int o = px / 16, x = x0 + 16 * wave + (px % 16), y = y0 + o;
            if (x >= a.W || y >= a.H) continue;
            float f[32];
#pragma unroll
            for (int q = 0; q < 4; ++q) unpack8(*reinterpret_cast<const uint4*>(tile + px * TS + 8 * q), f + 8 * q);
            a.head_out[(size_t)(n * a.H + y) * a.W + x] = head_value(f, a.head_w, a.head_b);
        }
    }
    if (a.out) {
        for (int q = lane; q < R * 16 * c8n; q += 64) {
            const int px = q / c8n, c8 = q - px * c8n;
            const int o = px / 16, x = x0 + 16 * wave + (px % 16), y = y0 + o;
            if (x >= a.W || y >= a.H) continue;
            uint4 v = *reinterpret_cast<const uint4*>(tile + px * TS + 8 * c8);
            const size_t off = ((size_t)(n * a.H + y) * a.W + x) * a.Cout + 8 * c8;
            if (a.mask) {
                float f[8], mk[8];
                unpack8(v, f);
                unpack8(*reinterpret_cast<const uint4*>(a.mask + off), mk);
#pragma unroll
                for (int e = 0; e < 8; ++e) f[e] = mk[e] > 0.0f ? f[e] : 0.0f;
                v = pack8(f);
            }
            *reinterpret_cast<uint4*>(a.out + off) = v;
        }
    }
    if (a.pool_out) {
        // 2x2 average pool of the wave's R rows x 16 pixels (tile origin and H, W even)
        const int Hp = a.H / 2, Wp = a.W / 2;
        for (int q = lane; q < (R / 2) * 8 * c8n; q += 64) {
            const int pp = q / c8n, c8 = q - pp * c8n;
            const int po = pp / 8, px2 = pp % 8;
            const int y = y0 + 2 * po, x = x0 + 16 * wave + 2 * px2;
            if (x >= a.W || y >= a.H) continue;
            const uint16_t* t0 = tile + (2 * po * 16 + 2 * px2) * TS + 8 * c8;
            const uint4 v = pool4(*reinterpret_cast<const uint4*>(t0), *reinterpret_cast<const uint4*>(t0 + TS),
                                  *reinterpret_cast<const uint4*>(t0 + 16 * TS),
                                  *reinterpret_cast<const uint4*>(t0 + 17 * TS));
            *reinterpret_cast<uint4*>(a.pool_out + ((size_t)(n * Hp + y / 2) * Wp + x / 2) * a.Cout + 8 * c8) = v;
        }
    }
}

// ---------------------------------------------------------------- FP32 copy of the network
// 3x3 convolution in FP32 on v_mfma_f32_16x16x4_f32: FP32 activations and weights, FP32 accumulation.  Bound by the
// matrix cores (32 cycles per instruction), so the operands come in wide LDS reads that serve many instructions.
// Workgroup of 4 waves, tile of 4 rows x 16 MT columns x 16 NT output channels (blockIdx.y: the block of output
// channels), wave w computes row w as MT x NT tiles of 16 x 16.  Per chunk of CC input channels the halo and the
// chunk's weights are staged in LDS; of the chunk, lane group kq = lane / 16 holds the S = CC / 4 channels S kq ..
// S kq + S - 1, its K index 4 s + kq of instruction s standing for channel S kq + s on both sides, so that one
// 16-byte read per tile and tap feeds S instructions of each of its row or column of tiles.  The first layer reads the
// BF16 features; the decoder's upsample + concat is fused into the halo load as in the BF16 kernel.
// 540x960 inference: 2.43 ms when each instruction took one 4-byte LDS read and one 4-byte load from the weights in
// memory (48 TFLOP/s), 1.21 ms now (97; 1080x1920 4.4 ms, 106 TFLOP/s).  The next chunk's halo, or halo and weights, held
// in registers under this chunk's instructions measured 6% and 60% slower.
constexpr int F32_NB = 64;   // output channels of a block: 16 NT = min(Cout, F32_NB)

template <int S>
struct FVec;
template <>
struct FVec<4> { typedef float4 t; };
template <>
struct FVec<2> { typedef float2 t; };
__device__ inline float fvec_at(const float4& v, int s) { return s == 0 ? v.x : s == 1 ? v.y : s == 2 ? v.z : v.w; }
__device__ inline float fvec_at(const float2& v, int s) { return s == 0 ? v.x : v.y; }

template <int MT, int NT, int CC>
struct ConvF32 {
    static constexpr int TW = 16 * MT, HW = TW + 2, HR = 6, S = CC / 4;
    static constexpr int HALO_BYTES = 4 * HR * HW * S * 4, W_BYTES = 9 * 4 * 16 * NT * S * 4;
    static_assert(HALO_BYTES % 16 == 0 && W_BYTES % 1024 == 0, "LDS parts in 16-byte and wave-load units");
    static constexpr size_t bytes() { return (size_t)HALO_BYTES + W_BYTES; }
};

// W_BYTES of weights from src straight into LDS at dst, 1 KB per wave and instruction
template <int W_BYTES>
__device__ __attribute__((always_inline)) inline void f32_weights_to_lds(const char* src, char* dst, int wave, int lane)
{
    for (int f = wave; f < W_BYTES / 1024; f += 4)
        __builtin_amdgcn_global_load_lds(src + f * 1024 + lane * 16, dst + f * 1024, 16, 0, 0);
}

template <int MT, int NT, int CC>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_conv_f32(ConvArgsF32 a)
{
    extern __shared__ uint4 conv_lds[];
    using L = ConvF32<MT, NT, CC>;
    constexpr int HW = L::HW, HR = L::HR, S = L::S, HP = HR * HW;
    typedef typename FVec<S>::t vec;
    vec* halo = reinterpret_cast<vec*>(conv_lds);                                               // [4][HP]
    char* wl = reinterpret_cast<char*>(conv_lds) + L::HALO_BYTES;
    const vec* wt = reinterpret_cast<const vec*>(wl);                                           // [9][4][16 NT]
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int tiles_x = (a.W + L::TW - 1) / L::TW, tiles_y = (a.H + 3) / 4;
    int tt = xcd_tile(blockIdx.x, gridDim.x);
    const int tx = tt % tiles_x;
    tt /= tiles_x;
    const int ty = tt % tiles_y, n = tt / tiles_y;
    const int x0 = tx * L::TW, y0 = ty * 4;
    const int r = lane & 15, kq = lane >> 4;
    const int Cs = a.Cin - a.Ca, n_blocks = gridDim.y;
    f32x4 acc[MT][NT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
    // halo item i: the S channels of lane group i % 4 of halo pixel i / 4, zero outside the image (clamped address)
    constexpr int ITEMS = 4 * HP, PF = (ITEMS + 255) / 256;
    auto item = [&](int c0, int i) -> vec {
        const int pix = i >> 2, ci = c0 + S * (i & 3);
        const int y = y0 - 1 + pix / HW, x = x0 - 1 + pix % HW;
        const bool inb = (unsigned)y < (unsigned)a.H && (unsigned)x < (unsigned)a.W;
        const int yc = min(max(y, 0), a.H - 1), xc = min(max(x, 0), a.W - 1);
        vec v;
        if constexpr (S == 2) {   // 8-channel BF16 features
            const uint32_t q = *reinterpret_cast<const uint32_t*>(static_cast<const uint16_t*>(a.in) +
                                                                  ((size_t)(n * a.H + yc) * a.W + xc) * a.Cin + ci);
            v.x = inb ? __uint_as_float(q << 16) : 0.0f;
            v.y = inb ? __uint_as_float(q & 0xFFFF0000u) : 0.0f;
        } else {
            const float* src;
            if (a.in2 == nullptr)
                src = static_cast<const float*>(a.in) + ((size_t)(n * a.H + yc) * a.W + xc) * a.Cin + ci;
            else if (ci < a.Ca)
                src = static_cast<const float*>(a.in) +
                      ((size_t)(n * (a.H >> 1) + (yc >> 1)) * (a.W >> 1) + (xc >> 1)) * a.Ca + ci;
            else
                src = a.in2 + ((size_t)(n * a.H + yc) * a.W + xc) * Cs + (ci - a.Ca);
            const float4 q = *reinterpret_cast<const float4*>(src);
            v.x = inb ? q.x : 0.0f; v.y = inb ? q.y : 0.0f; v.z = inb ? q.z : 0.0f; v.w = inb ? q.w : 0.0f;
        }
        return v;
    };
    for (int c0 = 0; c0 < a.Cin; c0 += CC) {
        vec pf[PF];
#pragma unroll
        for (int k = 0; k < PF; ++k) {
            const int i = (int)threadIdx.x + 256 * k;
            if (ITEMS % 256 == 0 || i < ITEMS) pf[k] = item(c0, i);
        }
        __syncthreads();   // every wave is done with the previous chunk
        f32_weights_to_lds<L::W_BYTES>(reinterpret_cast<const char*>(a.wt) +
                                           ((size_t)(c0 / CC) * n_blocks + blockIdx.y) * L::W_BYTES,
                                       wl, wave, lane);
#pragma unroll
        for (int k = 0; k < PF; ++k) {
            const int i = (int)threadIdx.x + 256 * k;
            if (ITEMS % 256 == 0 || i < ITEMS) halo[(i & 3) * HP + (i >> 2)] = pf[k];
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the direct-to-LDS loads have landed
        __syncthreads();
#pragma unroll
        for (int tap = 0; tap < 9; ++tap) {
            const int dy = tap / 3, dx = tap % 3;
            vec A[MT], B[NT];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) A[mt] = halo[kq * HP + (wave + dy) * HW + 16 * mt + r + dx];
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) B[nt] = wt[(tap * 4 + kq) * 16 * NT + 16 * nt + r];
#pragma unroll
            for (int s = 0; s < S; ++s)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt)
                        acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(fvec_at(A[mt], s), fvec_at(B[nt], s),
                                                                           acc[mt][nt], 0, 0, 0);
        }
    }
    // D layout: lane holds column (channel) 16 nt + (lane & 15), rows (pixels) 4 (lane >> 4) + e
    const int y = y0 + wave;
    if (y >= a.H) return;
    const int co0 = blockIdx.y * 16 * NT;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int co = co0 + 16 * nt + r;
        const float b = a.bias[co];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int x = x0 + 16 * mt + 4 * kq + e;
                if (x >= a.W) continue;
                a.out[((size_t)(n * a.H + y) * a.W + x) * a.Cout + co] = fmaxf(acc[mt][nt][e] + b, 0.0f);
            }
    }
}

__global__ __launch_bounds__(256) void k_pool2_f32(const float* in, int N, int H, int W, int C, float* out)
{
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    int h = H / 2, w = W / 2, C4 = C / 4;
    size_t total = (size_t)N * h * w * C4;
    if (i >= total) return;
    int c = (int)(i % C4) * 4;
    size_t q = i / C4;
    int x = (int)(q % w), t = (int)(q / w), y = t % h, n = t / h;
    const float* b = in + (((size_t)n * H + 2 * y) * W + 2 * x) * C + c;
    float4 p0 = *reinterpret_cast<const float4*>(b), p1 = *reinterpret_cast<const float4*>(b + C);
    float4 p2 = *reinterpret_cast<const float4*>(b + (size_t)W * C), p3 = *reinterpret_cast<const float4*>(b + (size_t)W * C + C);
    float4 o;
    o.x = ((p0.x + p1.x) + (p2.x + p3.x)) * 0.25f;
    o.y = ((p0.y + p1.y) + (p2.y + p3.y)) * 0.25f;
    o.z = ((p0.z + p1.z) + (p2.z + p3.z)) * 0.25f;
    o.w = ((p0.w + p1.w) + (p2.w + p3.w)) * 0.25f;
    *reinterpret_cast<float4*>(out + q * C + c) = o;
}

// y = sigmoid(sum_c d1[p][c] wh[c] + bh) with the FP32 head weights
__global__ __launch_bounds__(256) void k_head_f32(const float* d1, const float* wh, const float* bh, int P, float* y)
{
    int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= P) return;
    float s = 0.0f;
    const float* row = d1 + (size_t)p * 32;
    for (int c = 0; c < 32; ++c) s += row[c] * wh[c];
    s += bh[0];
    y[p] = 1.0f / (1.0f + expf(-s));
}

// FP32 master [Cout][9][Cin] of every layer -> the order k_conv_f32 stages them in: [chunk of CC channels][block of
// output channels][tap][lane group kq][output channel of the block][S], CC = 16 (8 for the 8-channel first layer),
// channel CC chunk + S kq + s
__global__ __launch_bounds__(256) void k_weights_f32(UnetF32Weights u)
{
    const UnetF32Weights::Layer l = u.layer[blockIdx.y];
    const int cc = l.cin % 16 == 0 ? 16 : 8, S = cc / 4, cb = min(l.cout, F32_NB);
    for (int i = blockIdx.x * 256 + threadIdx.x; i < l.cout * 9 * l.cin; i += gridDim.x * 256) {
        const int ci = i % l.cin, tap = (i / l.cin) % 9, co = i / (9 * l.cin);
        const int chunk = ci / cc, kq = ci % cc / S, s = ci % S, blk = co / cb;
        const size_t o = ((((size_t)chunk * (l.cout / cb) + blk) * 9 + tap) * 4 + kq) * cb * S + (size_t)(co % cb) * S + s;
        u.out[l.out + o] = u.w[l.in + i];
    }
}

// ---------------------------------------------------------------- weight gradient
// dW[co][tap][ci] = sum_p g[p][co] x[p + off(tap)][ci] and db[co] = sum_p g[p][co] as MFMA GEMMs with K = pixels.
// Both operands need 8 consecutive pixels of one channel per lane, while memory holds the channels of a pixel together;
// ds_read_b64_tr_b16 transposes on the way out of LDS (of each 16 lanes, lane 4 q + c reads 4 channels of pixel q and
// lane i receives channel i of the 4 pixels), so tiles are staged as they lie in memory.
// Workgroup of 3 waves; wave w owns the taps of kernel row dy = w.  A pixel tile is 2 rows x 64 columns: its gradient (16
// CO_T channels) and its input halo (4 rows x 66 columns, 16 CI_T channels, zero outside the image); the next tile's
// groups are loaded into registers under this tile's instructions.  With a second source (the decoder's inputs)
// channels below Ca come from the 2x nearest-upsampled tensor, so the concatenation is never stored.  A workgroup
// accumulates a chunk of consecutive tiles for one group of output and one of input channels; chunks are then added
// in order, so the result is deterministic.  The bias gradient is one more product, with ones, in wave 0.
// Bound by memory for 32 channels (32 -> 32 at 8x512^2: 268 MB in 78 us, 3.4 TB/s) and by the matrix cores and the LDS
// reads that feed them beyond.  With tiles transposed in registers and stored to LDS in three shifted copies, all
// layers of the 8x512^2 step took 1.78 ms here, besides 0.21 ms of bias sums and 0.17 ms to store the
// concatenations; 0.97 ms now.  OCC, waves per SIMD: without the bound the compiler keeps copies of the sums in a
// second register class and one wave fits (96 -> 32 channels 334 us, 212 at 2 waves); 32 -> 32 at 2 instead of 3: 92 us.
constexpr int WG_TW = 64, WG_R = 2, WG_THREADS = 192;
template <int CO_T, int CI_T, bool SMALL>
struct Wgrad {
    static constexpr int HW = WG_TW + 2, HR = WG_R + 2;
    static constexpr int XC8 = SMALL ? 1 : 2 * CI_T, GC8 = 2 * CO_T;          // 16-byte groups per pixel
    static constexpr int X_ITEMS = HR * HW * XC8, G_ITEMS = WG_R * WG_TW * GC8;
    static constexpr int XPT = (X_ITEMS + WG_THREADS - 1) / WG_THREADS, GPT = (G_ITEMS + WG_THREADS - 1) / WG_THREADS;
    static constexpr int G_OFF = X_ITEMS + (SMALL ? 1 : 0);   // in groups; a read of 16 channels of the last 8-channel pixel
    static constexpr int GROUPS = G_OFF + G_ITEMS;
};
typedef __attribute__((__vector_size__(4 * sizeof(short)))) short s16x4;
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

// 8 K values (pixels) of one channel per lane: two transposed reads, `half` bytes apart
__device__ inline bf16x8 tr_frag(const char* p, int half)
{
    const s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)p);
    const s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + half));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
}

// v or zeros, by component (a conditional between two structs selects their addresses and keeps both in scratch memory)
__device__ inline uint4 keep_if(const uint4& v, uint32_t keep)
{
    return make_uint4(keep ? v.x : 0u, keep ? v.y : 0u, keep ? v.z : 0u, keep ? v.w : 0u);
}

// slot of channel group c8 in a staged gradient pixel px: with 64 channels, pixels lie 32 banks apart, so the 32-byte
// units of 4 neighbouring pixels are rotated against each other
template <int GC8>
__device__ inline int g_slot(int c8, int px) { return GC8 >= 8 ? c8 ^ ((px & 3) << 1) : c8; }

template <int CO_T, int CI_T, bool SMALL, bool CAT, int OCC>
__global__ __launch_bounds__(WG_THREADS) __attribute__((amdgpu_waves_per_eu(OCC))) void k_wgrad(WgradArgs a, int tiles_per_chunk, int ci_groups)
{
    using L = Wgrad<CO_T, CI_T, SMALL>;
    __shared__ uint4 lds[L::GROUPS];
    constexpr int XPB = L::XC8 * 16, GPB = L::GC8 * 16;   // bytes per staged pixel
    const char* xs = reinterpret_cast<const char*>(lds);
    const char* gs = reinterpret_cast<const char*>(lds + L::G_OFF);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r = lane & 15, g = lane >> 4;
    const int cig = blockIdx.y % ci_groups, cog = blockIdx.y / ci_groups;
    const int ci0 = cig * 16 * CI_T, co0 = cog * 16 * CO_T;
    const int tiles_x = (a.W + WG_TW - 1) / WG_TW, tiles_y = (a.H + WG_R - 1) / WG_R;
    const int n_tiles = a.N * tiles_x * tiles_y;
    const int t_begin = blockIdx.x * tiles_per_chunk, t_end = min(n_tiles, t_begin + tiles_per_chunk);
    f32x4 acc[3][CO_T][CI_T], accb[CO_T];
#pragma unroll
    for (int i = 0; i < CO_T; ++i) {
        accb[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int dx = 0; dx < 3; ++dx)
#pragma unroll
            for (int j = 0; j < CI_T; ++j) acc[dx][i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    const bf16x8 ones = __builtin_bit_cast(bf16x8, make_uint4(0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u));
    const bool bias = wave == 0 && cig == 0;
    // a tile's groups in registers, from clamped addresses so that all loads are in flight together; bit k of x_in / g_in
    // tells whether item k lies in the image (zeros are stored otherwise).  Item i of the halo is group i % XC8 of pixel
    // i / XC8, of the gradient the group that slot i % GC8 of pixel i / GC8 holds.
    uint4 xv[L::XPT], gv[L::GPT];
    uint32_t x_in = 0, g_in = 0;
    auto fetch = [&](int t) __attribute__((always_inline)) {
        const int tx = t % tiles_x, rest = t / tiles_x, ty = rest % tiles_y, n = rest / tiles_y;
        const int x0 = tx * WG_TW, y0 = ty * WG_R;
        x_in = g_in = 0;
#pragma unroll
        for (int k = 0; k < L::XPT; ++k) {
            const int i = min((int)threadIdx.x + WG_THREADS * k, L::X_ITEMS - 1);
            const int pix = i / L::XC8, ci = ci0 + 8 * (i - pix * L::XC8);
            const int row = pix / L::HW, y = y0 - 1 + row, x = x0 - 1 + pix - row * L::HW;
            const int yc = min(max(y, 0), a.H - 1), xc = min(max(x, 0), a.W - 1);
            const uint16_t* src;
            if constexpr (CAT) {
                const bool up = ci < a.Ca;
                const size_t ou = ((size_t)(n * (a.H >> 1) + (yc >> 1)) * (a.W >> 1) + (xc >> 1)) * a.Ca + ci;
                const size_t os = ((size_t)(n * a.H + yc) * a.W + xc) * (a.Cin - a.Ca) + (ci - a.Ca);
                src = (up ? a.x : a.x2) + (up ? ou : os);
            } else {
                src = a.x + ((size_t)(n * a.H + yc) * a.W + xc) * a.Cin + ci;
            }
            xv[k] = *reinterpret_cast<const uint4*>(src);
            x_in |= x == xc && y == yc ? 1u << k : 0u;
        }
#pragma unroll
        for (int k = 0; k < L::GPT; ++k) {
            const int i = min((int)threadIdx.x + WG_THREADS * k, L::G_ITEMS - 1);
            const int pix = i / L::GC8, slot = i - pix * L::GC8;
            const int row = pix / WG_TW, px = pix - row * WG_TW, y = y0 + row, x = x0 + px;
            const int co = co0 + 8 * g_slot<L::GC8>(slot, px);   // the rotation is its own inverse
            const int yc = min(y, a.H - 1), xc = min(x, a.W - 1);
            gv[k] = *reinterpret_cast<const uint4*>(a.g + ((size_t)(n * a.H + yc) * a.W + xc) * a.Cout + co);
            g_in |= x == xc && y == yc ? 1u << k : 0u;
        }
    };
    // this lane's pixel (of a group of 4) and 4 channels in a transposed read
    const int q = 4 * g + (r >> 2), c = r & 3;
    if (SMALL && threadIdx.x == 0) lds[L::X_ITEMS] = make_uint4(0u, 0u, 0u, 0u);
    if (t_begin < t_end) fetch(t_begin);
    for (int t = t_begin; t < t_end; ++t) {
        __syncthreads();   // every wave is done with the previous tile
#pragma unroll
        for (int k = 0; k < L::XPT; ++k) {
            const int i = (int)threadIdx.x + WG_THREADS * k;
            if (L::X_ITEMS % WG_THREADS == 0 || i < L::X_ITEMS) lds[i] = keep_if(xv[k], (x_in >> k) & 1u);
        }
#pragma unroll
        for (int k = 0; k < L::GPT; ++k) {
            const int i = (int)threadIdx.x + WG_THREADS * k;
            if (L::G_ITEMS % WG_THREADS == 0 || i < L::G_ITEMS) lds[L::G_OFF + i] = keep_if(gv[k], (g_in >> k) & 1u);
        }
        __syncthreads();
        if (t + 1 < t_end) fetch(t + 1);   // under this tile's instructions
#pragma unroll
        for (int s = 0; s < WG_R * WG_TW / 32; ++s) {
            const int row = s / (WG_TW / 32), c0 = 32 * (s % (WG_TW / 32));
            bf16x8 A[CO_T], B[3][CI_T];
#pragma unroll
            for (int i = 0; i < CO_T; ++i)
                A[i] = tr_frag(gs + (row * WG_TW + c0 + q) * GPB + 16 * g_slot<L::GC8>(2 * i + (c >> 1), q) + 8 * (c & 1), 16 * GPB);
#pragma unroll
            for (int dx = 0; dx < 3; ++dx)
#pragma unroll
                for (int j = 0; j < CI_T; ++j)
                    B[dx][j] = tr_frag(xs + ((row + wave) * L::HW + c0 + dx + q) * XPB + 32 * j + 8 * c, 16 * XPB);
            if (bias) {
#pragma unroll
                for (int i = 0; i < CO_T; ++i) accb[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[i], ones, accb[i], 0, 0, 0);
            }
#pragma unroll
            for (int dx = 0; dx < 3; ++dx)
#pragma unroll
                for (int i = 0; i < CO_T; ++i)
#pragma unroll
                    for (int j = 0; j < CI_T; ++j)
                        acc[dx][i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[i], B[dx][j], acc[dx][i][j], 0, 0, 0);
        }
    }
    // D[i = output channel][j = input channel]: lane holds j = lane & 15, rows 4 (lane >> 4) + e
    float* out = a.partial + (size_t)blockIdx.x * ((size_t)a.Cout * 9 * a.Cin + a.Cout);
#pragma unroll
    for (int dx = 0; dx < 3; ++dx)
#pragma unroll
        for (int i = 0; i < CO_T; ++i)
#pragma unroll
            for (int j = 0; j < CI_T; ++j) {
                const int ci = ci0 + 16 * j + r;
                if (ci >= a.Cin) continue;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    out[((size_t)(co0 + 16 * i + 4 * g + e) * 9 + 3 * wave + dx) * a.Cin + ci] = acc[dx][i][j][e];
            }
    if (bias && r == 0) {
#pragma unroll
        for (int i = 0; i < CO_T; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) out[(size_t)a.Cout * 9 * a.Cin + co0 + 16 * i + 4 * g + e] = accb[i][e];
    }
}

// out[i] = sum over chunks c of partial[c][i]: 64 outputs per workgroup (256-byte rows), 16 lanes per output summing
// chunks q, q + 16, q + 32, ... in order, then a fixed-order tree over the 16
__global__ __launch_bounds__(1024) void k_reduce_chunks(const float* partial, int n_chunks, int n, float* out)
{
    __shared__ float sm[16][64];
    const int o = threadIdx.x & 63, q = threadIdx.x >> 6;
    const int i = blockIdx.x * 64 + o;
    float s = 0.0f;
    if (i < n) {
#pragma unroll 8
        for (int c = q; c < n_chunks; c += 16) s += partial[(size_t)c * n + i];
    }
    sm[q][o] = s;
    __syncthreads();
    for (int h = 8; h > 0; h >>= 1) {
        if (q < h) sm[q][o] += sm[q + h][o];
        __syncthreads();
    }
    if (q == 0 && i < n) out[i] = sm[0][o];
}

// out[o] (+)= sum over blocks b of partial[b][o], o < n: one workgroup per output, fixed-order tree
__global__ __launch_bounds__(256) void k_reduce_blocks(const float* partial, int nb, int n, float* out, int add)
{
    __shared__ float sm[256];
    const int o = blockIdx.x, t = threadIdx.x;
    float s = 0.0f;
    for (int b = t; b < nb; b += 256) s += partial[(size_t)b * n + o];
    sm[t] = s;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if (t < h) sm[t] += sm[t + h];
        __syncthreads();
    }
    if (t == 0) out[o] = add ? out[o] + sm[0] : sm[0];
}

// ---------------------------------------------------------------- pooling / upsampling / concat
// All channel counts and offsets are multiples of 8: one thread handles 8 channels (16 bytes).
__device__ inline uint4 ld8(const uint16_t* p) { return *reinterpret_cast<const uint4*>(p); }
__device__ inline void st8(uint16_t* p, uint4 v) { *reinterpret_cast<uint4*>(p) = v; }

__global__ __launch_bounds__(256) void k_pool2(const uint16_t* in, int N, int H, int W, int C, uint16_t* out)
{
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    int h = H / 2, w = W / 2, C8 = C / 8;
    size_t total = (size_t)N * h * w * C8;
    if (i >= total) return;
    int c = (int)(i % C8) * 8;
    size_t q = i / C8;
    int x = (int)(q % w), t = (int)(q / w), y = t % h, n = t / h;
    const uint16_t* b = in + (((size_t)n * H + 2 * y) * W + 2 * x) * C + c;
    st8(out + q * C + c, pool4(ld8(b), ld8(b + C), ld8(b + (size_t)W * C), ld8(b + (size_t)W * C + C)));
}

// gradient of the upsampled part of a concat: out[n,y,x,c] = mask * sum_{2x2} g[n,2y+a,2x+b, c0 + c]
__global__ __launch_bounds__(256) void k_up_back_mask(const uint16_t* g, int N, int H2, int W2, int Ctot, int c0,
                                                      int C, const uint16_t* mask, uint16_t* out)
{
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    int h = H2 / 2, w = W2 / 2, C8 = C / 8;
    size_t total = (size_t)N * h * w * C8;
    if (i >= total) return;
    int c = (int)(i % C8) * 8;
    size_t q = i / C8;
    int x = (int)(q % w), t = (int)(q / w), y = t % h, n = t / h;
    const uint16_t* b = g + (((size_t)n * H2 + 2 * y) * W2 + 2 * x) * Ctot + c0 + c;
    float a[8], bb[8], cc[8], d[8], mk[8], r[8];
    unpack8(ld8(b), a); unpack8(ld8(b + Ctot), bb);
    unpack8(ld8(b + (size_t)W2 * Ctot), cc); unpack8(ld8(b + (size_t)W2 * Ctot + Ctot), d);
    unpack8(ld8(mask + q * C + c), mk);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        float s = (a[e] + bb[e]) + (cc[e] + d[e]);
        r[e] = mk[e] > 0.0f ? s : 0.0f;
    }
    st8(out + q * C + c, pack8(r));
}

// out[n,y,x,c] = mask * (gpool[n,y/2,x/2,c] / 4 + gcat[n,y,x,c0 + c])
__global__ __launch_bounds__(256) void k_pool_back_add_mask(const uint16_t* gpool, const uint16_t* gcat, int N, int H,
                                                            int W, int C, int Ctot, int c0, const uint16_t* mask,
                                                            uint16_t* out)
{
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    int C8 = C / 8;
    size_t total = (size_t)N * H * W * C8;
    if (i >= total) return;
    int c = (int)(i % C8) * 8;
    size_t q = i / C8;
    int x = (int)(q % W), t = (int)(q / W), y = t % H, n = t / H;
    float gp[8], gc[8], mk[8], r[8];
    unpack8(ld8(gpool + (((size_t)n * (H / 2) + y / 2) * (W / 2) + x / 2) * C + c), gp);
    unpack8(ld8(gcat + q * Ctot + c0 + c), gc);
    unpack8(ld8(mask + q * C + c), mk);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        float v = gp[e] * 0.25f;
        v = v + gc[e];
        r[e] = mk[e] > 0.0f ? v : 0.0f;
    }
    st8(out + q * C + c, pack8(r));
}

// ---------------------------------------------------------------- loss, head gradients
// per-chunk sums of mask and mask * (y - t)^2, chunks of LOSS_CHUNK pixels (8x512^2: 512 workgroups; with 64 of
// 32768 pixels the sums took 59 us, 14 now)
constexpr int LOSS_CHUNK = 4096;
__device__ inline void block_sum2(float& a, float& b, float* sm)   // of 256 threads, in thread 0
{
    for (int h = 32; h > 0; h >>= 1) {
        a += __shfl_xor(a, h);
        b += __shfl_xor(b, h);
    }
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) { sm[2 * wave] = a; sm[2 * wave + 1] = b; }
    __syncthreads();
    a = (sm[0] + sm[2]) + (sm[4] + sm[6]);
    b = (sm[1] + sm[3]) + (sm[5] + sm[7]);
}

__global__ __launch_bounds__(256) void k_loss_partials(const float* y, const float* t, const float* m, int P,
                                                       float* partial)
{
    __shared__ float sm[8];
    const int p0 = blockIdx.x * LOSS_CHUNK;
    float a = 0.0f, b = 0.0f;
#pragma unroll 4
    for (int k = 0; k < LOSS_CHUNK / 256; ++k) {
        const int p = p0 + 256 * k + (int)threadIdx.x;
        if (p >= P) break;
        const float d = y[p] - t[p], w = m[p];
        a += w;
        b += w * d * d;
    }
    block_sum2(a, b, sm);
    if (threadIdx.x == 0) { partial[2 * blockIdx.x] = a; partial[2 * blockIdx.x + 1] = b; }
}

// sums[0] = sum mask, sums[1] = loss = sum m (y-t)^2 / max(sum m, 1)
__global__ __launch_bounds__(256) void k_loss_final(const float* partial, int n, float* sums)
{
    __shared__ float sm[8];
    float a = 0.0f, b = 0.0f;
    for (int i = threadIdx.x; i < n; i += 256) { a += partial[2 * i]; b += partial[2 * i + 1]; }
    block_sum2(a, b, sm);
    if (threadIdx.x == 0) {
        sums[0] = a;
        sums[1] = b / fmaxf(a, 1.0f);
    }
}

// dlogit = 2 m (y - t) / max(sum m, 1) * y (1 - y); gpre_d1 = mask(d1 > 0) * dlogit * wh, and per block of HEAD_PX
// pixels the partial head gradients (32 weights, then the bias).  Memory-bound: 32 BF16 channels in, 32 out.  Four
// lanes to a pixel, 8 channels each, so that a wave's loads and stores are contiguous, the sums of 8 pixels in
// registers, then across the lanes in a fixed order.  8x512^2: 129 us with one pixel per thread, its 64 bytes apart
// from its neighbour's, and 33 sums per 256 pixels through LDS; 49 us now (294 MB, part of it from the last-level cache).
constexpr int HEAD_PX = 512;
__global__ __launch_bounds__(256) void k_head_back(const uint16_t* d1, const float* y, const float* t, const float* m,
                                                   const float* sums, const float* wh, int P, uint16_t* gpre,
                                                   float* partial)
{
    __shared__ float sm[4][36];
    const int tid = threadIdx.x, c4 = tid & 3;
    const float inv = 2.0f / fmaxf(sums[0], 1.0f);
    float wq[8], v[9];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        wq[e] = bf2f(f2bf(wh[8 * c4 + e]));
        v[e] = 0.0f;
    }
    v[8] = 0.0f;
#pragma unroll 2
    for (int k = 0; k < HEAD_PX / 64; ++k) {
        const int p = blockIdx.x * HEAD_PX + 64 * k + (tid >> 2);
        if (p >= P) break;
        const float yy = y[p];
        const float dl = m[p] * (yy - t[p]) * inv * yy * (1.0f - yy);
        const size_t o = (size_t)p * 32 + 8 * c4;
        float f[8], gr[8];
        unpack8(*reinterpret_cast<const uint4*>(d1 + o), f);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            v[e] += dl * f[e];
            gr[e] = f[e] > 0.0f ? dl * wq[e] : 0.0f;
        }
        v[8] += dl;
        *reinterpret_cast<uint4*>(gpre + o) = pack8(gr);
    }
#pragma unroll
    for (int e = 0; e < 9; ++e)
        for (int h = 4; h < 64; h <<= 1) v[e] += __shfl_xor(v[e], h);
    if ((tid & 63) < 4) {
#pragma unroll
        for (int e = 0; e < 9; ++e) sm[tid >> 6][9 * c4 + e] = v[e];
    }
    __syncthreads();
    if (tid < 33) {
        const int i = tid < 32 ? 9 * (tid >> 3) + (tid & 7) : 8;
        partial[(size_t)blockIdx.x * 33 + tid] = (sm[0][i] + sm[1][i]) + (sm[2][i] + sm[3][i]);
    }
}

// ---------------------------------------------------------------- weights, Adam, features
// FP32 master [Cout][9][Cin] of every layer -> BF16 copies: forward layout and flipped/transposed Wf[ci][8 - tap][co].
// One launch for all layers (one each took 54 us of a step; 9 now).
__global__ __launch_bounds__(256) void k_weights_bf16(UnetBf16Weights u)
{
    const UnetBf16Weights::Layer l = u.layer[blockIdx.y];
    for (int i = blockIdx.x * 256 + threadIdx.x; i < l.cout * 9 * l.cin; i += gridDim.x * 256) {
        const int ci = i % l.cin, tap = (i / l.cin) % 9, co = i / (9 * l.cin);
        const uint16_t v = f2bf(u.w[l.in + i]);
        u.wf[l.out + i] = v;
        u.wb[l.out + ((size_t)ci * 9 + (8 - tap)) * l.cout + co] = v;
    }
}

__global__ __launch_bounds__(256) void k_adam(float* w, const float* g, float* m, float* v, int n, float lr, float b1,
                                              float b2, float eps, float c1, float c2)
{
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    float gi = g[i];
    float mi = b1 * m[i] + (1.0f - b1) * gi;
    float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    float mh = mi / c1, vh = vi / c2;
    w[i] = w[i] - lr * mh / (sqrtf(vh) + eps);
}

__global__ void k_fill_f32(float* p, float v, size_t n)
{
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

inline unsigned nb(size_t n, unsigned b) { return (unsigned)((n + b - 1) / b); }

}  // namespace

size_t conv_tiles(const ConvArgs& a, int rows, int cols)
{
    return (size_t)a.N * ((a.H + rows - 1) / rows) * ((a.W + cols - 1) / cols);
}

template <int MT, int NT, int CC, bool SW, int OCC, bool SMALL = false>
void launch_conv_lds(const ConvArgs& a, hipStream_t st)
{
    const size_t lds = ConvLds<MT, NT, CC, SW>::bytes();
    hipLaunchKernelGGL((k_conv_lds<MT, NT, CC, SW, OCC, SMALL>),
                       dim3((unsigned)conv_tiles(a, 4, 16 * MT), SMALL ? (a.Cout + 16 * NT - 1) / (16 * NT) : 1), dim3(256),
                       lds, st, a);
}

template <int R, int NT, int OCC>
void launch_conv_rows(const ConvArgs& a, hipStream_t st)
{
    const size_t lds = ConvRows<R, NT>::bytes();
    hipLaunchKernelGGL((k_conv_rows<R, NT, OCC>), dim3((unsigned)conv_tiles(a, R, 64)), dim3(256), lds, st, a);
}

void unet_conv3x3(const ConvArgs& a, hipStream_t st)
{
    const int nt = (a.Cout + 15) / 16;
    // up to 2 N-tiles: row-blocked waves over 32-channel chunks with the weights in registers (8-channel
    // inputs: the one-row kernel with 8-channel chunks, weights streamed through L1); from 4 N-tiles on: weights
    // staged in LDS, with chunks small enough that halo and weights fit in 64 KB (16 channels up to 8
    // N-tiles, padding a chunk's 144 K values to 160; 8 channels beyond)
    int cfg = 0;
    if (nt <= 2)
        cfg = a.Cin % 64 == 0 ? 264 : (a.Cin % 32 == 0 ? 232 : 208);
    else if (a.Cin % 16 == 0)
        cfg = nt * 100 + (nt <= 8 ? 16 : 8);
    static_assert(ConvRows<RC_CONV_ROWS, 2>::bytes() <= 65536 && ConvLds<4, 4, 16, true>::bytes() <= 65536 &&
                      ConvLds<2, 6, 16, true>::bytes() <= 65536 && ConvLds<2, 8, 16, true>::bytes() <= 65536 &&
                      ConvLds<2, 12, 8, true>::bytes() <= 65536,
                  "convolution LDS beyond 64 KB");
    // Small images leave CUs idle, and a layer lasts as long as one workgroup's chain of chunks (load, stage, multiply):
    // smaller tiles, the output channels split over workgroups, and the next chunk loaded under this one's instructions
    // (k_conv_lds SMALL; rows of 2 instead of 8).  Same sums in the same order.  Inference, these kernels / the others
    // (us): 64^2 66 / 132, 256^2 74 / 142; 360x640 16- and 8-channel-chunk layers 90 / 119, row-blocked 51 / 44, first
    // layer 12 / 9; 540x960 171 / 171, 98 / 81, 22 / 15.  In workgroups of the smaller tiles (row-blocked: of the larger
    // ones) the layers cross over between 1100 and 2000, 128 and 450, and at about 1000.
    const size_t small_blocks = conv_tiles(a, 4, 32) * (size_t)((nt + 1) / 2);
    const bool small = nt <= 2 ? (cfg == 208 ? conv_tiles(a, 4, 16) <= 1024 : conv_tiles(a, RC_CONV_ROWS, 64) <= 256)
                               : small_blocks <= 1200;
    if (small) {
        switch (cfg) {
        case 208: launch_conv_lds<1, 2, 8, false, 4, true>(a, st); return;
        case 232:
        case 264:
            if (nt == 1) launch_conv_rows<2, 1, 4>(a, st);
            else launch_conv_rows<2, 2, 3>(a, st);
            return;
        case 416:
        case 616:
        case 816: launch_conv_lds<2, 2, 16, true, 3, true>(a, st); return;
        case 1208: launch_conv_lds<2, 2, 8, true, 3, true>(a, st); return;
        default: break;
        }
    }
    switch (cfg) {
    case 208: launch_conv_lds<4, 2, 8, false, RC_OCC_E1A>(a, st); return;
    case 232:
    case 264:
        if (nt == 1) launch_conv_rows<RC_CONV_ROWS, 1, RC_OCC_ROWS + 1>(a, st);
        else launch_conv_rows<RC_CONV_ROWS, 2, RC_OCC_ROWS>(a, st);
        return;
    case 416: launch_conv_lds<4, 4, 16, true, RC_OCC_416>(a, st); return;
    case 616: launch_conv_lds<2, 6, 16, true, RC_OCC_816>(a, st); return;
    case 816: launch_conv_lds<2, 8, 16, true, RC_OCC_816>(a, st); return;
    case 1208: launch_conv_lds<2, 12, 8, true, 1>(a, st); return;
    default: break;
    }
    unet_conv3x3_direct(a, st);
}

void unet_conv3x3_direct(const ConvArgs& a, hipStream_t st)
{
    size_t P = (size_t)a.N * a.H * a.W;
    dim3 grid(nb(P, 128)), block(256);
    int nt = (a.Cout + 15) / 16;
    switch (nt) {
    case 1: hipLaunchKernelGGL(k_conv3x3<1>, grid, block, 0, st, a); break;
    case 2: hipLaunchKernelGGL(k_conv3x3<2>, grid, block, 0, st, a); break;
    case 4: hipLaunchKernelGGL(k_conv3x3<4>, grid, block, 0, st, a); break;
    case 6: hipLaunchKernelGGL(k_conv3x3<6>, grid, block, 0, st, a); break;
    case 8: hipLaunchKernelGGL(k_conv3x3<8>, grid, block, 0, st, a); break;
    case 12: hipLaunchKernelGGL(k_conv3x3<12>, grid, block, 0, st, a); break;
    default: break;   // channel counts of this network only
    }
}

namespace {
// channels per workgroup: 32 x 32 (32 x 48 of the 96-channel input), 64 x 32 beyond; chunks so that the workgroups of all
// channel groups fill the 256 CUs once, at three (32 output channels) or two workgroups of 3 waves to a CU.  Registers
// hold that many at once, 12 and 8 waves (OCC 3 and 2; the 25 to 33 KB of LDS would admit 4 to 6); a second, partly
// filled round and more partial sums to add cost more than they balance.  Whole 8x512^2 step at 768 / 512 workgroups 3.08 ms;
// 512 / 512 3.07, 1024 / 512 3.12, 1280 / 512 3.13, 768 / 768 3.31, 768 / 384 3.28.
struct WgradShape {
    int co_t, ci_t, groups, ci_groups, tiles_per_chunk, chunks;
};
WgradShape wgrad_shape(const WgradArgs& a)
{
    WgradShape w;
    w.co_t = a.Cout >= 64 ? 4 : 2;
    w.ci_t = a.Cin <= 16 ? 1 : (w.co_t == 2 && a.Cin % 48 == 0 ? 3 : 2);
    w.ci_groups = (a.Cin + 16 * w.ci_t - 1) / (16 * w.ci_t);
    w.groups = w.ci_groups * (a.Cout / (16 * w.co_t));
    const int tiles = a.N * ((a.H + WG_R - 1) / WG_R) * ((a.W + WG_TW - 1) / WG_TW);
    const int target = std::max(1, (w.co_t == 2 && w.ci_t < 3 ? 768 : 512) / w.groups);
    w.tiles_per_chunk = std::max(1, (tiles + target - 1) / target);
    w.chunks = (tiles + w.tiles_per_chunk - 1) / w.tiles_per_chunk;
    return w;
}
template <int CO_T, int CI_T, bool SMALL, bool CAT, int OCC>
void launch_wgrad(const WgradArgs& a, const WgradShape& w, hipStream_t st)
{
    hipLaunchKernelGGL((k_wgrad<CO_T, CI_T, SMALL, CAT, OCC>), dim3(w.chunks, w.groups), dim3(WG_THREADS), 0, st, a,
                       w.tiles_per_chunk, w.ci_groups);
}
}  // namespace

int unet_wgrad_chunks(const WgradArgs& a) { return wgrad_shape(a).chunks; }

void unet_wgrad(const WgradArgs& a, hipStream_t st)
{
    const WgradShape w = wgrad_shape(a);
    const bool cat = a.x2 != nullptr;
    switch (w.co_t * 10 + w.ci_t) {
    case 21: launch_wgrad<2, 1, true, false, 4>(a, w, st); break;     // the 8-channel first layer
    case 22: launch_wgrad<2, 2, false, false, 3>(a, w, st); break;
    case 23: launch_wgrad<2, 3, false, true, 2>(a, w, st); break;      // the 96-channel concatenation
    case 42:
        if (cat) launch_wgrad<4, 2, false, true, 2>(a, w, st);
        else launch_wgrad<4, 2, false, false, 2>(a, w, st);
        break;
    default: break;   // channel counts of this network only
    }
}

void unet_reduce_chunks(const float* partial, int n_chunks, int n, float* out, hipStream_t st)
{
    hipLaunchKernelGGL(k_reduce_chunks, dim3(nb(n, 64)), dim3(1024), 0, st, partial, n_chunks, n, out);
}

void unet_reduce_blocks(const float* partial, int n_blocks, int n, float* out, int add, hipStream_t st)
{
    hipLaunchKernelGGL(k_reduce_blocks, dim3(n), dim3(256), 0, st, partial, n_blocks, n, out, add);
}

void unet_pool2(const uint16_t* in, int N, int H, int W, int C, uint16_t* out, hipStream_t st)
{
    size_t n = (size_t)N * (H / 2) * (W / 2) * (C / 8);
    hipLaunchKernelGGL(k_pool2, dim3(nb(n, 256)), dim3(256), 0, st, in, N, H, W, C, out);
}

void unet_up_back_mask(const uint16_t* g, int N, int H2, int W2, int Ctot, int c0, int C, const uint16_t* mask,
                       uint16_t* out, hipStream_t st)
{
    size_t n = (size_t)N * (H2 / 2) * (W2 / 2) * (C / 8);
    hipLaunchKernelGGL(k_up_back_mask, dim3(nb(n, 256)), dim3(256), 0, st, g, N, H2, W2, Ctot, c0, C, mask, out);
}

void unet_pool_back_add_mask(const uint16_t* gpool, const uint16_t* gcat, int N, int H, int W, int C, int Ctot, int c0,
                             const uint16_t* mask, uint16_t* out, hipStream_t st)
{
    size_t n = (size_t)N * H * W * (C / 8);
    hipLaunchKernelGGL(k_pool_back_add_mask, dim3(nb(n, 256)), dim3(256), 0, st, gpool, gcat, N, H, W, C, Ctot, c0,
                       mask, out);
}

int unet_loss_chunks(int P) { return (P + LOSS_CHUNK - 1) / LOSS_CHUNK; }

void unet_loss(const float* y, const float* t, const float* m, int P, float* partial, float* sums, hipStream_t st)
{
    const int chunks = unet_loss_chunks(P);
    hipLaunchKernelGGL(k_loss_partials, dim3(chunks), dim3(256), 0, st, y, t, m, P, partial);
    hipLaunchKernelGGL(k_loss_final, dim3(1), dim3(256), 0, st, partial, chunks, sums);
}

int unet_head_blocks(int P) { return (P + HEAD_PX - 1) / HEAD_PX; }

void unet_head_back(const uint16_t* d1, const float* y, const float* t, const float* m, const float* sums,
                    const float* wh, int P, uint16_t* gpre, float* partial, hipStream_t st)
{
    hipLaunchKernelGGL(k_head_back, dim3(unet_head_blocks(P)), dim3(256), 0, st, d1, y, t, m, sums, wh, P, gpre,
                       partial);
}

void unet_weights_bf16(const UnetBf16Weights& u, hipStream_t st)
{
    hipLaunchKernelGGL(k_weights_bf16, dim3(64, u.n_layers), dim3(256), 0, st, u);
}

void unet_adam(float* w, const float* g, float* m, float* v, int n, float lr, float b1, float b2, float eps, float c1,
               float c2, hipStream_t st)
{
    hipLaunchKernelGGL(k_adam, dim3(nb(n, 256)), dim3(256), 0, st, w, g, m, v, n, lr, b1, b2, eps, c1, c2);
}

namespace {
template <int MT, int NT, int CC>
void launch_conv_f32(const ConvArgsF32& a, hipStream_t st)
{
    static_assert(ConvF32<MT, NT, CC>::bytes() <= 65536, "LDS beyond 64 KB");
    const size_t tiles = (size_t)a.N * ((a.H + 3) / 4) * ((a.W + 16 * MT - 1) / (16 * MT));
    const size_t lds = ConvF32<MT, NT, CC>::bytes();
    hipLaunchKernelGGL((k_conv_f32<MT, NT, CC>), dim3((unsigned)tiles, a.Cout / (16 * NT)), dim3(256), lds, st, a);
}
}  // namespace

void unet_conv3x3_f32(const ConvArgsF32& a, hipStream_t st)
{
    // Narrow tiles hold little LDS and few registers, so more workgroups overlap one's staging with another's
    // instructions and the last round of workgroups is shorter; wide ones read and stage less per instruction, which
    // pays once there are many.  All convolutions of an inference, tiles of 16 / 32 / 64 columns: 256^2 224 / 318 /
    // 486 us, 540x960 1239 / 1318 / 1516 us, 1080x1920 4491 / 4326 / 4429 us (its 64-channel layers 1965 / 1903 / 1774).
    const int nt = std::min(a.Cout, F32_NB) / 16;
    auto blocks = [&](int mt) {
        return (size_t)a.N * ((a.H + 3) / 4) * ((a.W + 16 * mt - 1) / (16 * mt)) * (a.Cout / (16 * nt));
    };
    const int mt = nt == 4 && blocks(4) >= 2000 ? 4 : blocks(2) >= 4000 ? 2 : 1;
    switch ((a.Cin % 16 == 0 ? 100 : 0) + 10 * nt + mt) {
    case 22: launch_conv_f32<2, 2, 8>(a, st); break;
    case 21: launch_conv_f32<1, 2, 8>(a, st); break;
    case 122: launch_conv_f32<2, 2, 16>(a, st); break;
    case 121: launch_conv_f32<1, 2, 16>(a, st); break;
    case 144: launch_conv_f32<4, 4, 16>(a, st); break;
    case 142: launch_conv_f32<2, 4, 16>(a, st); break;
    case 141: launch_conv_f32<1, 4, 16>(a, st); break;
    default: break;   // channel counts of this network only
    }
}

void unet_pool2_f32(const float* in, int N, int H, int W, int C, float* out, hipStream_t st)
{
    size_t n = (size_t)N * (H / 2) * (W / 2) * (C / 4);
    hipLaunchKernelGGL(k_pool2_f32, dim3(nb(n, 256)), dim3(256), 0, st, in, N, H, W, C, out);
}

void unet_head_f32(const float* d1, const float* wh, const float* bh, int P, float* y, hipStream_t st)
{
    hipLaunchKernelGGL(k_head_f32, dim3(nb(P, 256)), dim3(256), 0, st, d1, wh, bh, P, y);
}

void unet_weights_f32(const UnetF32Weights& u, hipStream_t st)
{
    hipLaunchKernelGGL(k_weights_f32, dim3(64, u.n_layers), dim3(256), 0, st, u);
}

void unet_fill_f32(float* p, float v, size_t n, hipStream_t st)
{
    hipLaunchKernelGGL(k_fill_f32, dim3(nb(n, 256)), dim3(256), 0, st, p, v, n);
}
