// Display post pass of a rendered frame (the paper's main-pass tone mapping and gamma correction and its
// FXAA post-processing pass, Sec. IV-B): Reinhard tone map + sRGB8 encoding, then FXAA on the 8-bit image.
// The exact definition (integer luma, integer edge decisions, FP32 blend in a fixed order) is stated with
// rc_postprocess in include/raycast.h; both kernels are HBM-bound image passes.
#include "rc_internal.h"

#include <mutex>

namespace {

constexpr int EDGE_MIN = 2048;   // minimum local luma range (luma scale 0..65280)
constexpr int EDGE_REL_SHIFT = 3;
constexpr int SEARCH = 12;

// The transfer function and its rounding in FP64, as defined.
__device__ inline uint32_t srgb8_exact(float r)
{
    const double v = (double)r;
    const double s = v <= 0.0031308 ? 12.92 * v : 1.055 * pow(fmax(v, 0.0), 1.0 / 2.4) - 0.055;
    return (uint32_t)fmin(fmax(floor(s * 255.0 + 0.5), 0.0), 255.0);
}

// The same byte from FP32 where that decides it: with the hardware's log2 and exp2 (each within 2^-22 of its result on
// this range, log2 of at most 8.4), 255 s + 0.5 is within 255 x 1.055 x (8.4 / 2.4 + 2) x 2^-22 < 4e-4 of the exact
// value, so its floor is the exact one's unless it lies that close to an integer; those few (and what is no number of
// the range) take the FP64 path.  The FP64 power for every channel had taken 41 us of a 1080p image, 13 now.
constexpr float SRGB_GUARD = 5e-4f;
__device__ inline uint32_t srgb8(float v)
{
    const float s = v <= 0.0031308f ? 12.92f * v
                                    : fmaf(1.055f, __builtin_amdgcn_exp2f(__builtin_amdgcn_logf(v) * (1.0f / 2.4f)), -0.055f);
    const float y = fmaf(s, 255.0f, 0.5f), k = floorf(y), f = y - k;
    if (f > SRGB_GUARD && f < 1.0f - SRGB_GUARD) return (uint32_t)k;   // v in [0, 1]: k in 0 .. 255
    return srgb8_exact(v);
}

__global__ __launch_bounds__(256) void k_tonemap(const float4* rgba, uint32_t n, uchar4* out)
{
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float4 c = rgba[i];
    float v[3] = {fmaxf(c.x, 0.0f), fmaxf(c.y, 0.0f), fmaxf(c.z, 0.0f)};
    uint8_t q[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) q[k] = (uint8_t)srgb8(v[k] / (1.0f + v[k]));
    const double a = fmin(fmax((double)c.w, 0.0), 1.0);
    out[i] = make_uchar4(q[0], q[1], q[2], (uint8_t)floor(a * 255.0 + 0.5));
}

// Workgroup tile of 64 x FX_H pixels, staged in LDS with the 13 pixels around it that the edge search can reach (border
// clamped): the search reads one pixel after the other, up to 48 of them, each of which had waited for memory.  The tile's
// edge pixels are gathered first and blended by full waves: nearly every row of 64 pixels holds some, and a row's wave
// would walk the search for those alone.  1080p with 8% edge pixels, 16 rows: 39 us from memory, 35 from LDS, 19 gathered.
// 16 rows stage each pixel 3.7 times (4: 10.5 times), but an image of few such tiles lasts as long as one tile's rounds of
// edge pixels.  Whole post pass, one pixel per thread from memory / 16 rows / 4 rows: noise of 128x128 11.6 / 19.7 / 11.9 us,
// 480x640 18.7 / 23.1 / 15.9, 540x960 26.5 / 23.5 / 19.0, 720x1280 40.2 / 30.2 / 27.7, 1080p 72 / 42 / 50; hard-edged regions 12.7
// / 16.7 / 11.7, 21.1 / 19.0 / 14.6, 30.8 / 19.0 / 17.1, 46.8 / 24.3 / 24.4, 86 / 32 / 45.  So 4 rows up to FX_SMALL pixels (and 65535
// rows of tiles, the most that a grid takes).
constexpr int FX_W = 64, FX_B = SEARCH + 1, FX_P = FX_W + 2 * FX_B;
constexpr uint32_t FX_SMALL = 700000;

// 77 R + 150 G + 29 B
__device__ inline int luma(uint32_t p) { return (int)__builtin_amdgcn_udot4(p, 77u | (150u << 8) | (29u << 16), 0u, false); }

// the pixel at tile[at] (rows FX_P apart) and its four neighbours: the luma range, and whether it is an edge pixel
__device__ inline bool fxaa_edge(const uint32_t* tile, int at, int& Lc, int& Ln, int& Ls, int& Lw, int& Le, int& rng)
{
    Lc = luma(tile[at]);
    Ln = luma(tile[at - FX_P]);
    Ls = luma(tile[at + FX_P]);
    Lw = luma(tile[at - 1]);
    Le = luma(tile[at + 1]);
    const int lmax = max(max(max(Lc, Ln), max(Ls, Lw)), Le);
    const int lmin = min(min(min(Lc, Ln), min(Ls, Lw)), Le);
    rng = lmax - lmin;
    return rng >= EDGE_MIN && (rng << EDGE_REL_SHIFT) >= lmax;
}

// FXAA of the edge pixel at tile[at]
__device__ inline uchar4 fxaa_blend(const uint32_t* tile, int at)
{
    const uint32_t p = tile[at];
    int Lc, Ln, Ls, Lw, Le, rng;
    fxaa_edge(tile, at, Lc, Ln, Ls, Lw, Le, rng);
    const int Lnw = luma(tile[at - FX_P - 1]), Lne = luma(tile[at - FX_P + 1]);
    const int Lsw = luma(tile[at + FX_P - 1]), Lse = luma(tile[at + FX_P + 1]);
    // second differences across rows (large at an edge running along x) and across columns
    const int d_rows = abs(Lnw - 2 * Lw + Lsw) + 2 * abs(Ln - 2 * Lc + Ls) + abs(Lne - 2 * Le + Lse);
    const int d_cols = abs(Lnw - 2 * Ln + Lne) + 2 * abs(Lw - 2 * Lc + Le) + abs(Lsw - 2 * Ls + Lse);
    const bool horiz = d_rows >= d_cols;
    const int L1 = horiz ? Ln : Lw, L2 = horiz ? Ls : Le;
    const int g1 = abs(L1 - Lc), g2 = abs(L2 - Lc);
    const bool first = g1 >= g2;
    const int grad = max(g1, g2);
    const int S2 = Lc + (first ? L1 : L2);    // twice the mean luma of the pair straddling the edge
    const int side = horiz ? (first ? -FX_P : FX_P) : (first ? -1 : 1), along = horiz ? 1 : FX_P;
    int dist[2] = {SEARCH + 1, SEARCH + 1}, mend[2] = {0, 0};
#pragma unroll
    for (int d = 0; d < 2; ++d) {
        const int step = d == 0 ? along : -along;
        for (int i = 1; i <= SEARCH; ++i) {
            const int m = luma(tile[at + i * step]) + luma(tile[at + i * step + side]);
            if (2 * abs(m - S2) >= grad) {
                dist[d] = i;
                mend[d] = m;
                break;
            }
        }
    }
    const bool near_pos = dist[0] < dist[1];
    const int dmin = min(dist[0], dist[1]);
    const int me = near_pos ? mend[0] : mend[1];
    const bool found = (near_pos ? dist[0] : dist[1]) <= SEARCH;
    const bool blend_edge = found && ((me - S2 < 0) != (2 * Lc - S2 < 0));
    const float off_edge = blend_edge ? 0.5f - (float)dmin / (float)(dist[0] + dist[1]) : 0.0f;
    const int a12 = 2 * (Ln + Ls + Le + Lw) + (Lne + Lnw + Lse + Lsw);
    const float num = (float)abs(a12 - 12 * Lc), den = (float)max(12 * rng, 1);
    const float s1 = fminf(num / den, 1.0f);
    float t = -2.0f * s1;
    t = t + 3.0f;
    t = t * s1;
    t = t * s1;
    const float sub = (t * t) * 0.75f;
    const float w = fmaxf(off_edge, sub);
    const uint32_t q = tile[at + side];
    uint8_t r[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const float a = (float)((p >> (8 * k)) & 255u), b = (float)((q >> (8 * k)) & 255u);
        const float d = b - a;
        const float wd = w * d;
        const float v = a + wd;
        r[k] = (uint8_t)fminf(fmaxf(floorf(v + 0.5f), 0.0f), 255.0f);
    }
    return make_uchar4(r[0], r[1], r[2], p >> 24);
}

template <int FX_H>
__global__ __launch_bounds__(256) void k_fxaa(const uint32_t* in, int W, int H, uint32_t* out)
{
    __shared__ uint32_t tile[(FX_H + 2 * FX_B) * FX_P];
    __shared__ uint16_t edges[FX_W * FX_H];
    __shared__ uint32_t n_edges;
    const int x0 = blockIdx.x * FX_W, y0 = blockIdx.y * FX_H;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (threadIdx.x == 0) n_edges = 0;
    {   // a wave per row: 64 pixels, then the 26 left
        const int xa = min(max(x0 + lane - FX_B, 0), W - 1), xb = min(x0 + lane + 64 - FX_B, W - 1);
        for (int ty = wave; ty < FX_H + 2 * FX_B; ty += 4) {
            const uint32_t* row = in + (size_t)min(max(y0 + ty - FX_B, 0), H - 1) * W;
            tile[ty * FX_P + lane] = row[xa];
            if (lane < FX_P - 64) tile[ty * FX_P + 64 + lane] = row[xb];
        }
    }
    __syncthreads();
    const int x = x0 + lane;
    for (int ly = wave; ly < FX_H; ly += 4) {
        const int y = y0 + ly, at = (ly + FX_B) * FX_P + lane + FX_B;
        int Lc, Ln, Ls, Lw, Le, rng;
        const bool in_image = x < W && y < H;
        const bool edge = in_image && fxaa_edge(tile, at, Lc, Ln, Ls, Lw, Le, rng);
        if (in_image && !edge) out[(size_t)y * W + x] = tile[at];
        const uint64_t m = __ballot(edge);
        uint32_t base = 0;
        if (lane == 0 && m) base = atomicAdd(&n_edges, (uint32_t)__popcll(m));
        base = __builtin_amdgcn_readfirstlane(base);
        if (edge) edges[base + (uint32_t)__popcll(m & ((1ull << lane) - 1ull))] = (uint16_t)(ly * FX_W + lane);
    }
    __syncthreads();
    for (uint32_t k = threadIdx.x; k < n_edges; k += 256) {
        const int ly = edges[k] / FX_W, lx = edges[k] % FX_W;
        reinterpret_cast<uchar4*>(out)[(size_t)(y0 + ly) * W + x0 + lx] = fxaa_blend(tile, (ly + FX_B) * FX_P + lx + FX_B);
    }
}

}  // namespace

void rc_launch_postprocess(const float* rgba, uint32_t w, uint32_t h, bool fxaa, uint8_t* scratch, uint8_t* out,
                           hipStream_t st)
{
    const uint32_t n = w * h;
    uchar4* tm = reinterpret_cast<uchar4*>(fxaa ? scratch : out);
    hipLaunchKernelGGL(k_tonemap, dim3((n + 255) / 256), dim3(256), 0, st, reinterpret_cast<const float4*>(rgba), n,
                       tm);
    if (!fxaa) return;
    auto run = [&](auto kernel, uint32_t rows) {
        hipLaunchKernelGGL(kernel, dim3((w + FX_W - 1) / FX_W, (h + rows - 1) / rows), dim3(256), 0, st,
                           reinterpret_cast<const uint32_t*>(tm), (int)w, (int)h, reinterpret_cast<uint32_t*>(out));
    };
    if (n <= FX_SMALL && h <= 4u * 65535u) run(k_fxaa<4>, 4u);
    else run(k_fxaa<16>, 16u);
}

// Fixed scratch of rc_postprocess_noalloc: the tone-mapped 8-bit image that FXAA reads, for images of at most
// RC_POST_SCRATCH_PIXELS pixels (16 MiB).  Each GPU the library runs on holds its own copy until the
// process ends.  In host code this name is only a stand-in for the symbol: kernels receive the device address
// that rc_post_scratch_init obtained for the current device.
static __device__ __align__(256) uchar4 scratch[RC_POST_SCRATCH_PIXELS];

namespace {
constexpr int MAX_DEVICES = 64;
std::mutex g_scratch_mutex;
uint8_t* g_scratch_ptr[MAX_DEVICES] = {};
}  // namespace

hipError_t rc_post_scratch_init(int device)
{
    if (device < 0 || device >= MAX_DEVICES) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (g_scratch_ptr[device]) return hipSuccess;
    int prev = 0;
    hipError_t e = hipGetDevice(&prev);
    if (e != hipSuccess) return e;
    e = hipSetDevice(device);
    if (e != hipSuccess) return e;
    void* ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e == hipSuccess && ptr) g_scratch_ptr[device] = static_cast<uint8_t*>(ptr);
    else if (e == hipSuccess) e = hipErrorInvalidSymbol;
    hipError_t e2 = hipSetDevice(prev);
    return e != hipSuccess ? e : e2;
}

uint8_t* rc_post_scratch(int device)
{
    if (device < 0 || device >= MAX_DEVICES) return nullptr;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    return g_scratch_ptr[device];
}
