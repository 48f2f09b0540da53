// cost_volume.hip - truncated windowed SAD cost volume and contrast edge weights.
//
// Paper: the data term sampled at every label forms the unary cost vectors
// (Sec. 2.2 "Stereo"), precomputed for all labels before the discrete stage
// (Table tab:timing "Cost Vol.").  The paper's own data term is Census + Hamming
// (Sec. 3.1); this kernel provides a truncated windowed SAD in the same role.
// Edge strengths are image dependent, lower across image edges (Sec. 2.1).
//
// Layout: the volume is label-major ([y][x][d], d fastest).  Windows up to 7 of large frames
// are computed on strips of rows (sad_strip.h), others a row at a time.  Border handling:
// window positions are clamped to the image (clamp-to-edge), and a right-image column left
// of 0 costs `trunc`.
#include "common.h"
#include "sad_strip.h"

namespace dm {

// Small frames: a block owns one row and kSadTX pixels, its threads are the
// labels (K <= 256 -> 1..4 waves), so each pixel's K costs are one coalesced write.  Each
// thread sums the window vertically for the TX + 2R window columns of its label, then slides
// the horizontal sum: the same sums in the same order as the strips'.
constexpr int kSadTX = 16;  // pixels per block

template <typename OT, int R>
__global__ __launch_bounds__(256) void sad_tile_kernel(const float* __restrict__ IL, const float* __restrict__ IR, int W,
                                                       int H, int K, float trunc, float inv_area,
                                                       OT* __restrict__ out) {
    constexpr int TX = kSadTX;
    constexpr int NR = 2 * R + 1;   // window rows
    constexpr int NC = TX + 2 * R;  // window columns of the tile
    __shared__ float sL[NR][NC];
    __shared__ float sR[NR][NC + 255];
    const int y = blockIdx.y;
    const int x0 = blockIdx.x * TX;
    const int lr = x0 - R;            // image column of sL[.][0]
    const int rr = x0 - R - (K - 1);  // image column of sR[.][0]
    const int nrc = NC + K - 1;
    for (int e = threadIdx.x; e < NR * nrc; e += blockDim.x) {
        const int row = e / nrc, j = e - row * nrc;
        const int yy = min(max(y + row - R, 0), H - 1);
        const int xc = rr + j;
        sR[row][j] = (xc >= 0 && xc < W) ? IR[(long long)yy * W + xc] : 0.0f;
        if (j < NC) sL[row][j] = IL[(long long)yy * W + min(max(lr + j, 0), W - 1)];
    }
    __syncthreads();
    const int d = threadIdx.x;
    if (d >= K) return;
    // vertical window sums at the (clamped) columns lr + i
    float col[NC];
#pragma unroll
    for (int i = 0; i < NC; ++i) {
        const int xx = min(max(lr + i, 0), W - 1);  // clamped image column
        const int li = xx - lr;                     // its index in sL
        const int xr = xx - d;                      // matching right-image column
        const int ri = xr - rr;
        float acc = 0.0f;
#pragma unroll
        for (int row = 0; row < NR; ++row) acc += (xr >= 0) ? fabsf(sL[row][li] - sR[row][ri]) : trunc;
        col[i] = acc;
    }
#pragma unroll
    for (int xi = 0; xi < TX; ++xi) {
        const int x = x0 + xi;
        if (x >= W) break;
        float acc = 0.0f;
#pragma unroll
        for (int dx = 0; dx < NR; ++dx) acc += col[xi + dx];
        out[((long long)y * W + x) * K + d] = (OT)fminf(trunc, acc * inv_area);
    }
}

// Any odd window (the kernels above cover radii 1..3): one thread per (pixel, label).
template <typename OT>
__global__ __launch_bounds__(256) void sad_kernel(const float* __restrict__ IL, const float* __restrict__ IR, int W,
                                                  int H, int K, int r, float trunc, float inv_area,
                                                  OT* __restrict__ out) {
    const long long total = (long long)W * H * K;
    for (long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
         idx += (long long)gridDim.x * blockDim.x) {
        const int d = (int)(idx % K);
        const long long p = idx / K;
        const int x = (int)(p % W), y = (int)(p / W);
        float acc = 0.0f;
        for (int dx = -r; dx <= r; ++dx) {
            const int xx = min(max(x + dx, 0), W - 1);
            const int xr = xx - d;
            for (int dy = -r; dy <= r; ++dy) {
                const int yy = min(max(y + dy, 0), H - 1);
                acc += (xr >= 0) ? fabsf(IL[(long long)yy * W + xx] - IR[(long long)yy * W + xr]) : trunc;
            }
        }
        out[idx] = (OT)fminf(trunc, acc * inv_area);
    }
}

__global__ __launch_bounds__(256) void contrast_kernel(const float* __restrict__ IL, int W, int H, float lambda_pw,
                                                       float inv_sigma, float* __restrict__ w_h,
                                                       float* __restrict__ w_v) {
    const long long total = (long long)W * H;
    for (long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x; p < total;
         p += (long long)gridDim.x * blockDim.x) {
        const int x = (int)(p % W), y = (int)(p / W);
        const float c = IL[p];
        if (w_h != nullptr && x + 1 < W)
            w_h[(long long)y * (W - 1) + x] = contrast_weight(IL[p + 1], c, lambda_pw, inv_sigma);
        if (w_v != nullptr && y + 1 < H) w_v[p] = contrast_weight(IL[p + W], c, lambda_pw, inv_sigma);
    }
}

// Whether the strips serve a volume of `size`-byte costs (same values either way).  A strip's
// block does 64 x 4 pixels, so a frame needs 900 of them (3.5 per CU) to fill the chip: window
// 3, FP16, row kernel -> strips 640x240x192 35 -> 34, 640x360x192 47 -> 36, 1242x375x192 88 -> 56
// us, but 320x240x192 22 -> 29 and 96x72x192 11 -> 21 us.  Windows 5 and 7 share more of a row's
// differences and need fewer blocks for it: 320x240x201 44 -> 50 us at window 5, but 640x240x201
// 83 -> 56, x192 72 -> 41, x24 27 -> 14 us, and at window 7 144 -> 75, 119 -> 69, 44 -> 18 us.
// One label a thread (odd K) writes parts of lines: beyond the 256 MB that
// the last cache holds they no longer merge (1242x375, FP32, K = 135 81 -> 62, 201 112 -> 126 us).
// Window 1 replaces a thread per cost with 64-bit divisions, whose time is the volume's size:
// 320x240x32 11 -> 12, x64 14 -> 12 us.
bool strip_serves(int r, const dm_shape& s, size_t size) {
    const long long blocks = (long long)((s.W + kStripX - 1) / kStripX) * ((s.H + kStripY - 1) / kStripY);
    const long long labels = (long long)s.W * s.H * s.K;
    if (r == 0) return blocks >= 300 && labels >= 4000000;
    if (r > 1) return r <= 3 && blocks >= 600;
    return blocks >= 900 && (s.K % 2 == 0 || labels * (long long)size <= (256LL << 20));
}

hipError_t launch_contrast_weights(const float* I, int W, int H, float lambda_pw, float inv_sigma, float* w_h,
                                   float* w_v, hipStream_t stream) {
    const long long npx = (long long)W * H;
    const unsigned b2 = (unsigned)std::min<long long>((npx + 255) / 256, 65535LL);
    hipLaunchKernelGGL(contrast_kernel, dim3(b2), dim3(256), 0, stream, I, W, H, lambda_pw, inv_sigma, w_h, w_v);
    return hipGetLastError();
}

// ------------------------------------------------------------------ Census + Hamming
// The paper's data term (Sec. 3.1): each image's Census transform over a small patch,
// compared by the Hamming distance.  Readings: bit b of a pixel's code is
// [I(q_b) < I(centre)] for the b-th non-centre position q_b of the (2R+1)^2 window in
// raster order (dy outer, dx inner), coordinates clamped to the image; the cost is the
// number of differing bits over n = (2R+1)^2 - 1, truncated at `trunc`; a match outside
// the image costs `trunc`.  Left view: pixel x matches x - d of the right image; right
// view: pixel x of the right image matches x + d of the left image.
//
// What bounds it: the store of the volume, then the codes.  A block owns one image row and
// kCensusX pixels: the window rows of the reference image (kCensusX codes) and of the
// matched image (kCensusX + K - 1 codes) are staged in LDS and every code is computed once
// per block (in 32 bits for windows up to 5).  Then a thread owns LPT consecutive labels of
// kCensusTX pixels: the codes of the matched image that its labels and pixels meet are read
// once into registers, each output is an xor, a bit count and a look-up in a table of
// min(trunc, h / n), h = 0..n (each an IEEE division, so every value is the correctly rounded
// quotient; n + 1 words in as many LDS banks), and a pixel's LPT costs are one vector store.
// The block also writes the contrast weights of its pixels' edges.
//
// Measured, 1242 x 375 x 192 FP16, window 5, both views with their weights: 128 -> 95 us (64
// pixels a block and a pair of labels a thread before); 64, 128 and 256 pixels a block in one
// comparison: 95.5, 92.0, 96.4 us.
constexpr int kCensusX = 128, kCensusTX = 8;

template <int R>
struct CensusCode {
    using type = uint32_t;  // (2R+1)^2 - 1 = 8 or 24 bits
};
template <>
struct CensusCode<3> {
    using type = uint64_t;  // 48 bits
};
__device__ __forceinline__ int census_distance(uint32_t a, uint32_t b) { return __popc(a ^ b); }
__device__ __forceinline__ int census_distance(uint64_t a, uint64_t b) { return __popcll(a ^ b); }

// Code of the pixel at column c + R of the staged rows.
template <int R, int NC>
__device__ __forceinline__ typename CensusCode<R>::type census_code(const float (&rows)[2 * R + 1][NC], int c) {
    using code_t = typename CensusCode<R>::type;
    const float ctr = rows[R][c + R];
    code_t v = 0;
    int b = 0;
#pragma unroll
    for (int dy = 0; dy < 2 * R + 1; ++dy)
#pragma unroll
        for (int dx = 0; dx < 2 * R + 1; ++dx) {
            if (dy == R && dx == R) continue;
            v |= (code_t)(rows[dy][c + dx] < ctr) << b;
            ++b;
        }
    return v;
}

template <typename OT, int R, bool LEFT, int LPT>
__global__ __launch_bounds__(256) void census_tile_kernel(const float* __restrict__ IL, const float* __restrict__ IR,
                                                          int W, int H, int K, float trunc, OT* __restrict__ out,
                                                          StripWeights sw) {
    constexpr int TX = kCensusTX, NR = 2 * R + 1, n = NR * NR - 1;
    using code_t = typename CensusCode<R>::type;
    __shared__ float sA[NR][kCensusX + 2 * R];
    __shared__ float sB[NR][kCensusX + 255 + 2 * R];
    __shared__ code_t cA[kCensusX];
    __shared__ code_t cB[kCensusX + 255];
    __shared__ float lut[64];
    const float* __restrict__ A = LEFT ? IL : IR;  // reference image of the view
    const float* __restrict__ B = LEFT ? IR : IL;  // matched image
    const int y = blockIdx.y;
    const int x0 = blockIdx.x * kCensusX;
    const int nb = kCensusX + K - 1;          // codes of the matched image
    const int bB = LEFT ? x0 - (K - 1) : x0;  // image column of the first
#pragma unroll
    for (int row = 0; row < NR; ++row) {
        const long long yy = min(max(y + row - R, 0), H - 1);
        const float* __restrict__ Brow = B + yy * W;
        for (int j = threadIdx.x; j < nb + 2 * R; j += blockDim.x) sB[row][j] = Brow[min(max(bB - R + j, 0), W - 1)];
        const float* __restrict__ Arow = A + yy * W;
        for (int j = threadIdx.x; j < kCensusX + 2 * R; j += blockDim.x)
            sA[row][j] = Arow[min(max(x0 - R + j, 0), W - 1)];
    }
    if (threadIdx.x <= n) lut[threadIdx.x] = fminf(trunc, (float)threadIdx.x / (float)n);
    __syncthreads();
    for (int c = threadIdx.x; c < kCensusX; c += blockDim.x) {
        cA[c] = census_code<R>(sA, c);
        const int x = x0 + c;
        if (sw.w_h != nullptr && x + 1 < W)
            sw.w_h[(long long)y * (W - 1) + x] = contrast_weight(sA[R][c + R + 1], sA[R][c + R], sw.lambda_pw, sw.inv_sigma);
        if (sw.w_v != nullptr && x < W && y + 1 < H)
            sw.w_v[(long long)y * W + x] = contrast_weight(sA[R + 1][c + R], sA[R][c + R], sw.lambda_pw, sw.inv_sigma);
    }
    for (int c = threadIdx.x; c < nb; c += blockDim.x) cB[c] = census_code<R>(sB, c);
    __syncthreads();
    const int groups = K / LPT;  // LPT divides K
    const bool interior = bB >= 0 && bB + nb <= W && x0 + kCensusX <= W;
    for (int item = threadIdx.x; item < (kCensusX / TX) * groups; item += blockDim.x) {
        const int g = item / groups;
        const int i0 = (item - g * groups) * LPT;
        const int xa = x0 + g * TX;
        if (xa >= W) continue;
        // pixel q and label i0 + l meet code vb[q + LPT - 1 - l] (left) or vb[q + l] (right)
        const code_t* b = cB + g * TX + (LEFT ? K - LPT - i0 : i0);
        code_t va[TX], vb[TX + LPT - 1];
#pragma unroll
        for (int q = 0; q < TX; ++q) va[q] = cA[g * TX + q];
#pragma unroll
        for (int q = 0; q < TX + LPT - 1; ++q) vb[q] = b[q];
        OT* o = out + ((long long)y * W + xa) * K + i0;
#pragma unroll
        for (int q = 0; q < TX; ++q) {
            if (xa + q < W) {
                typedef OT vec_t __attribute__((ext_vector_type(LPT)));
                vec_t r;
#pragma unroll
                for (int l = 0; l < LPT; ++l) {
                    float c = lut[census_distance(va[q], vb[LEFT ? q + LPT - 1 - l : q + l])];
                    if (!interior) {
                        const int xo = LEFT ? xa + q - (i0 + l) : xa + q + (i0 + l);  // matched column
                        c = (xo >= 0 && xo < W) ? c : trunc;
                    }
                    r[l] = (OT)c;
                }
                *reinterpret_cast<vec_t*>(o + (long long)q * K) = r;
            }
        }
    }
}

// Left-right consistency check (Sec. 4.1): a left pixel keeps its disparity iff the
// right view's disparity at its match x - round(u) (round half up) differs by at most
// max_diff; otherwise it gets `invalid`.  The rounding is exact (floor plus the
// fraction's comparison with 1/2), the difference and its comparison are FP32.
__global__ __launch_bounds__(256) void lr_check_kernel(const float* __restrict__ uL, const float* __restrict__ uR,
                                                       int W, int H, float max_diff, float invalid,
                                                       float* __restrict__ out) {
    const long long total = (long long)W * H;
    for (long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x; p < total;
         p += (long long)gridDim.x * blockDim.x) {
        const int x = (int)(p % W);
        const float u = uL[p];
        const float fl = floorf(u);
        const float r = fl + ((u - fl) >= 0.5f ? 1.0f : 0.0f);
        const float xr = (float)x - r;
        float o = invalid;
        if (xr >= 0.0f && xr <= (float)(W - 1)) {
            const float v = uR[p - x + (long long)xr];
            if (fabsf(u - v) <= max_diff) o = u;
        }
        out[p] = o;
    }
}

}  // namespace dm

using namespace dm;

extern "C" int dm_build_cost_volume_census(const float* I_left, const float* I_right, dm_shape s,
                                           const dm_cost_params* p, int view, dm_dtype out_dtype, void* cost_out,
                                           float* w_h, float* w_v, void* hip_stream) {
    clear_error();
    int st = validate_shape(s);
    if (st != DM_OK) return st;
    DM_REQUIRE(p != nullptr, DM_ERR_NULL, "params is NULL");
    DM_REQUIRE(I_left != nullptr && I_right != nullptr && cost_out != nullptr, DM_ERR_NULL,
               "images and cost_out are required");
    DM_REQUIRE(out_dtype == DM_F32 || out_dtype == DM_F16, DM_ERR_DTYPE, "unknown dtype %d", (int)out_dtype);
    DM_REQUIRE(view == DM_VIEW_LEFT || view == DM_VIEW_RIGHT, DM_ERR_PARAM, "view=%d must be 0 (left) or 1 (right)",
               view);
    DM_REQUIRE(p->window == 3 || p->window == 5 || p->window == 7, DM_ERR_PARAM, "census window=%d must be 3, 5 or 7",
               p->window);
    DM_REQUIRE(p->trunc > 0.0f && p->trunc <= 1.0f, DM_ERR_PARAM, "census trunc must be in (0, 1]");
    DM_REQUIRE(p->lambda_pw >= 0.0f && p->contrast_sigma > 0.0f, DM_ERR_PARAM,
               "lambda_pw >= 0 and contrast_sigma > 0 required");
    {
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) {
            set_error("pending HIP error before dm_build_cost_volume_census: %s", hipGetErrorString(e));
            return DM_ERR_HIP;
        }
    }
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    const long long total = (long long)s.W * s.H * s.K;
    ProfScope ps(DM_PROF_CENSUS, (double)total * (out_dtype == DM_F16 ? 2 : 4) + 8.0 * s.W * s.H, stream);
    const dim3 grid((unsigned)((s.W + kCensusX - 1) / kCensusX), (unsigned)s.H);
    const bool left = view == DM_VIEW_LEFT;
    const StripWeights sw{w_h, w_v, p->lambda_pw, 1.0f / p->contrast_sigma};
    const size_t es = out_dtype == DM_F16 ? 2 : 4;
    // the widest vector that K and the volume's alignment allow; the items spread evenly
    const int lpt = (s.K % 4 == 0 && (uintptr_t)cost_out % (4 * es) == 0) ? 4
                    : (s.K % 2 == 0 && (uintptr_t)cost_out % (2 * es) == 0) ? 2 : 1;
    const int items = (kCensusX / kCensusTX) * (s.K / lpt), turns = (items + 255) / 256;
    const dim3 block((unsigned)(((items + turns - 1) / turns + 63) / 64 * 64));
#define DM_CENSUS_V(OT, RR, LF, LP)                                                                                 \
    hipLaunchKernelGGL((census_tile_kernel<OT, RR, LF, LP>), grid, block, 0, stream, I_left, I_right, s.W, s.H, s.K, \
                       p->trunc, static_cast<OT*>(cost_out), sw)
#define DM_CENSUS(OT, RR)                                     \
    do {                                                      \
        if (left) {                                           \
            if (lpt == 4) DM_CENSUS_V(OT, RR, true, 4);       \
            else if (lpt == 2) DM_CENSUS_V(OT, RR, true, 2);  \
            else DM_CENSUS_V(OT, RR, true, 1);                \
        } else {                                              \
            if (lpt == 4) DM_CENSUS_V(OT, RR, false, 4);      \
            else if (lpt == 2) DM_CENSUS_V(OT, RR, false, 2); \
            else DM_CENSUS_V(OT, RR, false, 1);               \
        }                                                     \
    } while (0)
    const int r = p->window / 2;
    if (out_dtype == DM_F16) {
        if (r == 1) DM_CENSUS(_Float16, 1);
        else if (r == 2) DM_CENSUS(_Float16, 2);
        else DM_CENSUS(_Float16, 3);
    } else {
        if (r == 1) DM_CENSUS(float, 1);
        else if (r == 2) DM_CENSUS(float, 2);
        else DM_CENSUS(float, 3);
    }
#undef DM_CENSUS
#undef DM_CENSUS_V
    ps.stop();
    DM_HIP_TRY(hipGetLastError(), "census launch");
    return DM_OK;
}

extern "C" int dm_lr_check(const float* u_left, const float* u_right, int W, int H, float max_diff, float invalid,
                           float* u_out, void* hip_stream) {
    clear_error();
    DM_REQUIRE(u_left != nullptr && u_right != nullptr && u_out != nullptr, DM_ERR_NULL,
               "u_left, u_right and u_out are required");
    DM_REQUIRE(W >= 1 && H >= 1 && (long long)W * H <= (1LL << 31), DM_ERR_SHAPE, "W=%d H=%d out of range", W, H);
    DM_REQUIRE(W <= (1 << 24), DM_ERR_SHAPE, "W=%d above 2^24", W);
    DM_REQUIRE(max_diff >= 0.0f, DM_ERR_PARAM, "max_diff must be >= 0");
    {
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) {
            set_error("pending HIP error before dm_lr_check: %s", hipGetErrorString(e));
            return DM_ERR_HIP;
        }
    }
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    const long long npx = (long long)W * H;
    ProfScope ps(DM_PROF_LR_CHECK, 12.0 * npx, stream);
    const unsigned blocks = (unsigned)std::min<long long>((npx + 255) / 256, 65535LL * 4);
    hipLaunchKernelGGL(lr_check_kernel, dim3(blocks), dim3(256), 0, stream, u_left, u_right, W, H, max_diff, invalid,
                       u_out);
    ps.stop();
    DM_HIP_TRY(hipGetLastError(), "lr check launch");
    return DM_OK;
}

extern "C" int dm_build_cost_volume(const float* I_left, const float* I_right, dm_shape s, const dm_cost_params* p,
                                    dm_dtype out_dtype, void* cost_out, float* w_h, float* w_v, void* hip_stream) {
    clear_error();
    int st = validate_shape(s);
    if (st != DM_OK) return st;
    DM_REQUIRE(p != nullptr, DM_ERR_NULL, "params is NULL");
    DM_REQUIRE(I_left != nullptr && I_right != nullptr && cost_out != nullptr, DM_ERR_NULL,
               "images and cost_out are required");
    DM_REQUIRE(out_dtype == DM_F32 || out_dtype == DM_F16, DM_ERR_DTYPE, "unknown dtype %d", (int)out_dtype);
    DM_REQUIRE(p->window >= 1 && p->window <= 15 && (p->window % 2) == 1, DM_ERR_PARAM,
               "window=%d must be odd in [1, 15]", p->window);
    DM_REQUIRE(p->trunc > 0.0f, DM_ERR_PARAM, "trunc must be > 0");
    DM_REQUIRE(p->lambda_pw >= 0.0f && p->contrast_sigma > 0.0f, DM_ERR_PARAM,
               "lambda_pw >= 0 and contrast_sigma > 0 required");
    {
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) {
            set_error("pending HIP error before dm_build_cost_volume: %s", hipGetErrorString(e));
            return DM_ERR_HIP;
        }
    }
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    const long long total = (long long)s.W * s.H * s.K;
    const unsigned blocks = (unsigned)std::min<long long>((total + 255) / 256, 65535LL * 8);
    const int r = p->window / 2;
    const float inv_area = 1.0f / (float)(p->window * p->window);
    // algorithmic bytes: the volume written once, the two images read once
    ProfScope ps(DM_PROF_COST_VOLUME, (double)total * (out_dtype == DM_F16 ? 2 : 4) + 8.0 * s.W * s.H, stream);
    hipError_t strip = hipSuccess;
    const StripWeights sw{w_h, w_v, p->lambda_pw, 1.0f / p->contrast_sigma};
    const bool strips = strip_serves(r, s, out_dtype == DM_F16 ? 2 : 4);
    const dim3 tgrid((unsigned)((s.W + kSadTX - 1) / kSadTX), (unsigned)s.H);
    const dim3 tblock((unsigned)((s.K + 63) / 64 * 64));
#define DM_SAD_STRIP(OT, RR)                                                                                        \
    strip = launch_sad_strip<OT, RR, -1>(I_left, I_right, s.W, s.H, s.K, 1, 0, 0, p->trunc, inv_area,               \
                                         static_cast<OT*>(cost_out), sw, stream)
#define DM_SAD(OT, RR)                                                                                              \
    if (strips)                                                                                                     \
        DM_SAD_STRIP(OT, RR);                                                                                       \
    else                                                                                                            \
        hipLaunchKernelGGL((sad_tile_kernel<OT, RR>), tgrid, tblock, 0, stream, I_left, I_right, s.W, s.H, s.K,     \
                           p->trunc, inv_area, static_cast<OT*>(cost_out))
    if (out_dtype == DM_F16) {
        if (r == 0 && strips) {
            DM_SAD_STRIP(_Float16, 0);
        } else if (r == 1) {
            DM_SAD(_Float16, 1);
        } else if (r == 2) {
            DM_SAD(_Float16, 2);
        } else if (r == 3) {
            DM_SAD(_Float16, 3);
        } else {
            hipLaunchKernelGGL(sad_kernel<_Float16>, dim3(blocks), dim3(256), 0, stream, I_left, I_right, s.W, s.H, s.K,
                               r, p->trunc, inv_area, static_cast<_Float16*>(cost_out));
        }
    } else {
        if (r == 0 && strips) {
            DM_SAD_STRIP(float, 0);
        } else if (r == 1) {
            DM_SAD(float, 1);
        } else if (r == 2) {
            DM_SAD(float, 2);
        } else if (r == 3) {
            DM_SAD(float, 3);
        } else {
            hipLaunchKernelGGL(sad_kernel<float>, dim3(blocks), dim3(256), 0, stream, I_left, I_right, s.W, s.H, s.K, r,
                               p->trunc, inv_area, static_cast<float*>(cost_out));
        }
    }
#undef DM_SAD
#undef DM_SAD_STRIP
    DM_HIP_TRY(strip, "sad strip launch");
    ps.stop();
    DM_HIP_TRY(hipGetLastError(), "sad launch");
    if (!strips && (w_h != nullptr || w_v != nullptr))  // the strips wrote them otherwise
        DM_HIP_TRY(launch_contrast_weights(I_left, s.W, s.H, p->lambda_pw, 1.0f / p->contrast_sigma, w_h, w_v, stream),
                   "contrast launch");
    return DM_OK;
}
