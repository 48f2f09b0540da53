// sad_strip.h - truncated windowed SAD costs on strips of pixels, shared by the stereo
// volume (cost_volume.hip) and the two-dimensional flow volume (flow.hip).
//
//   e(x, y, i)   = |A(x, y) - B(x + s(i), y + j - off2)|, trunc where B has no such pixel,
//                  s(i) = -i (stereo, DIR = -1) or i - off1 (flow, DIR = +1)
//   out(x, y, j, i) = min(trunc, mean of e over the window x.+-R, y.+-R clamped to the image)
//
// Layout of the output: [y][x][j][i], label i fastest (stereo: one j).
//
// What bounds it: the volume is written once and read never, so the floor is the store
// time; the rest is one absolute difference per (pixel, label, window row) and the window
// sums.  A block owns kStripX x kStripY pixels and up to kStripJ labels j, with the rows of
// both images that they reach in LDS.  A thread owns LPT consecutive labels of kStripTX
// pixels and walks down the strip: each image row's differences are formed once and stay in
// registers for the 2R + 1 output rows that use them, and each window column's sum is
// shared by the 2R + 1 outputs across.  The LPT labels share their reads of B (label i at
// column c reads what label i + 1 reads one column further) and leave as one vector store.
// The terms are added row by row within a column, then column by column.  The blocks of the
// first labels j also write the contrast weights of A's edges, whose pixels they hold in LDS.
//
// Measured: 1242 x 375 x 192 FP16, window 3: 107 -> 62 us with the weights (2.9 TB/s; a block
// of one row and 16 pixels with a label per thread before), window 5 203 -> 83 us; flow volume
// of 640 x 480 x 32 x 32 FP16, window 3 1214 -> 145 us (4.4 TB/s; a block per row and label j
// before), window 5 4887 -> 217 us (661 with the ring of differences in scratch memory).
// 8 rows a strip: that stereo volume 52 -> 48 us and the flow volumes 146 -> 140, 217 -> 186,
// but half as many blocks, so 1242 x 375 x 24 1.4 times and 320 x 240 x 17 x 15 1.3 times the
// time; 16 rows: the stereo volume 90 us.
#pragma once

#include <type_traits>
#include <utility>

#include "common.h"

namespace dm {

constexpr int kStripX = 64;  // pixels per block
constexpr int kStripTX = 8;  // pixels per thread
constexpr int kStripY = 4;   // rows per block
constexpr int kStripJ = 4;   // labels j per block

// LDS floats of a block (staged rows of A and B).
constexpr size_t strip_lds_floats(int R, int K, int nj) {
    return (size_t)(kStripY + 2 * R) * (kStripX + 2 * R) + (size_t)(kStripY + 2 * R + nj - 1) * (kStripX + 2 * R + K - 1);
}

// Contrast weights to write beside the volume (null: not wanted).
struct StripWeights {
    float *w_h, *w_v;
    float lambda_pw, inv_sigma;
};

// f(0), f(1), ... with constants, until one is false
template <class F, int... S>
__device__ __forceinline__ void strip_steps(F& f, std::integer_sequence<int, S...>) {
    (f(std::integral_constant<int, S>()) && ...);
}

template <typename OT, int R, int DIR, int LPT>
__global__ __launch_bounds__(256) void sad_strip_kernel(const float* __restrict__ A, const float* __restrict__ B, int W,
                                                        int H, int K, int K2, int off1, int off2, int nj, float trunc,
                                                        float inv_area, OT* __restrict__ out, StripWeights sw) {
    constexpr int TX = kStripTX, NR = 2 * R + 1, NC = TX + 2 * R, NS = kStripY + 2 * R;
    constexpr int colsA = kStripX + 2 * R;
    extern __shared__ float strip_lds[];
    float* sA = strip_lds;               // [NS][colsA]
    float* sB = strip_lds + NS * colsA;  // [NS + nj - 1][colsB]
    const int colsB = kStripX + 2 * R + K - 1;
    const int x0 = blockIdx.x * kStripX, y0 = blockIdx.y * kStripY, j0 = blockIdx.z * nj;
    const int cb0 = x0 - R + (DIR > 0 ? -off1 : -(K - 1));  // image column of sB[.][0]
    const int rb0 = y0 - R + j0 - off2;                                 // image row of sB[0]
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64, waves = blockDim.x / 64;
    for (int s = wave; s < NS; s += waves) {
        const float* row = A + (long long)min(max(y0 - R + s, 0), H - 1) * W;
        for (int t = lane; t < colsA; t += 64) sA[s * colsA + t] = row[min(max(x0 - R + t, 0), W - 1)];
    }
    for (int s = wave; s < NS + nj - 1; s += waves) {
        const float* row = B + (long long)min(max(rb0 + s, 0), H - 1) * W;  // clamped: validity is checked below
        for (int t = lane; t < colsB; t += 64) sB[s * colsB + t] = row[min(max(cb0 + t, 0), W - 1)];
    }
    __syncthreads();
    if constexpr (R >= 1) {
        if (blockIdx.z == 0) {
            for (int q = threadIdx.x; q < kStripX * kStripY; q += blockDim.x) {
                const int dx = q % kStripX, dy = q / kStripX, x = x0 + dx, y = y0 + dy;
                if (x >= W || y >= H) continue;
                const float* a = sA + (dy + R) * colsA + dx + R;
                if (sw.w_h != nullptr && x + 1 < W) sw.w_h[(long long)y * (W - 1) + x] = contrast_weight(a[1], a[0], sw.lambda_pw, sw.inv_sigma);
                if (sw.w_v != nullptr && y + 1 < H) sw.w_v[(long long)y * W + x] = contrast_weight(a[colsA], a[0], sw.lambda_pw, sw.inv_sigma);
            }
        }
    }
    const int groups = K / LPT;  // label groups of a pixel (LPT divides K)
    const int items = (kStripX / TX) * nj * groups;
    // every column of A and B that the block reaches lies in the image
    const bool interior = x0 - R >= 0 && x0 + kStripX + R <= W && cb0 >= 0 && cb0 + colsB <= W;
    for (int item = threadIdx.x; item < items; item += blockDim.x) {
        // (pixel group, label j, label group), the last fastest: a pixel's labels are contiguous
        const int gj = item / groups;
        const int i0 = (item - gj * groups) * LPT;
        const int g = gj / nj, jj = gj - g * nj;
        const int xa = x0 + g * TX;  // first output pixel
        const int j = j0 + jj, d2 = j - off2;
        if (xa >= W || j >= K2) continue;
        const float* a0 = sA + g * TX;
        // label i0 + l at window column c: b0[c + l] (flow) or b0[c + LPT - 1 - l] (stereo)
        const float* b0 = sB + g * TX + (DIR > 0 ? i0 : K - LPT - i0);
        // The ring of row differences: for R >= 2 a step's index into it is a compile-time constant
        // (indexed by a loop variable it stays in scratch memory); for R <= 1 the compiler resolves
        // the loop's and schedules it better (flow 160 x 120 x 17 x 15, window 3, 16.5 and 17.1 us).
        float e[NR][LPT][NC];
        auto step = [&](auto row) __attribute__((always_inline)) {
            const int s = row;
            const int cy = min(max(y0 - R + s, 0), H - 1);  // the window row's (clamped) image row
            const int my = cy + d2;
            float(&es)[LPT][NC] = e[s % NR];
            if (my >= 0 && my < H) {
                const float* a = a0 + s * colsA;
                const float* b = b0 + (cy - (y0 - R) + jj) * colsB;
                float v[NC + LPT - 1];
#pragma unroll
                for (int c = 0; c < NC + LPT - 1; ++c) v[c] = b[c];
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    const float ac = a[c];
#pragma unroll
                    for (int l = 0; l < LPT; ++l) es[l][c] = fabsf(ac - v[DIR > 0 ? c + l : c + LPT - 1 - l]);
                }
            } else {
#pragma unroll
                for (int l = 0; l < LPT; ++l)
#pragma unroll
                    for (int c = 0; c < NC; ++c) es[l][c] = trunc;
            }
            if (!interior) {
#pragma unroll
                for (int l = 0; l < LPT; ++l) {
                    const int d1 = DIR > 0 ? i0 + l - off1 : -(i0 + l);
#pragma unroll
                    for (int c = 0; c < NC; ++c) {
                        const int mx = xa - R + c + d1;
                        es[l][c] = (mx >= 0 && mx < W) ? es[l][c] : trunc;
                    }
                    // window columns outside the image repeat the border column's
#pragma unroll
                    for (int c = 1; c < NC; ++c) es[l][c] = xa - R + c > W - 1 ? es[l][c - 1] : es[l][c];
#pragma unroll
                    for (int c = R - 1; c >= 0; --c) es[l][c] = xa - R + c < 0 ? es[l][c + 1] : es[l][c];
                }
            }
            if (s >= 2 * R) {
                const int y = y0 + s - 2 * R;  // the output row that this window row completes
                if (y >= H) return false;
                float col[LPT][NC];
#pragma unroll
                for (int l = 0; l < LPT; ++l)
#pragma unroll
                    for (int c = 0; c < NC; ++c) {
                        float acc = e[(s - 2 * R) % NR][l][c];
#pragma unroll
                        for (int r = 1; r < NR; ++r) acc += e[(s - 2 * R + r) % NR][l][c];
                        col[l][c] = acc;
                    }
                OT* o = out + (((long long)y * W + xa) * K2 + j) * K + i0;
#pragma unroll
                for (int q = 0; q < TX; ++q) {
                    if (xa + q < W) {
                        typedef OT vec_t __attribute__((ext_vector_type(LPT)));
                        vec_t r;
#pragma unroll
                        for (int l = 0; l < LPT; ++l) {
                            float acc = col[l][q];
#pragma unroll
                            for (int dx = 1; dx < NR; ++dx) acc += col[l][q + dx];
                            r[l] = (OT)fminf(trunc, acc * inv_area);
                        }
                        *reinterpret_cast<vec_t*>(o + (long long)q * K2 * K) = r;
                    }
                }
            }
            return true;
        };
        if constexpr (R >= 2) {
            strip_steps(step, std::make_integer_sequence<int, NS>());
        } else {
#pragma unroll
            for (int s = 0; s < NS; ++s)
                if (!step(s)) break;
        }
    }
}

// LPT: the widest vector that K and the volume's alignment allow (8 or 16 bytes a lane; for
// windows above 3 half of that, as the differences of 2R + 1 rows live in registers).
template <typename OT, int R, int DIR>
hipError_t launch_sad_strip(const float* A, const float* B, int W, int H, int K, int K2, int off1, int off2,
                            float trunc, float inv_area, OT* out, StripWeights sw, hipStream_t st) {
    if (R == 0 && (sw.w_h != nullptr || sw.w_v != nullptr)) {  // no neighbours in LDS
        const hipError_t e = launch_contrast_weights(A, W, H, sw.lambda_pw, sw.inv_sigma, sw.w_h, sw.w_v, st);
        if (e != hipSuccess) return e;
    }
    const int gx = (W + kStripX - 1) / kStripX, gy = (H + kStripY - 1) / kStripY;
    auto items = [&](int lpt, int nj) { return (kStripX / kStripTX) * nj * (K / lpt); };
    // Labels j of a block: fewer where its threads would take several turns while CUs have no
    // block (64 x 48 x 64 x 5, window 5: 29 us with 4, 12 with 1; with one turn the blocks of 4
    // are no slower, 64 x 48 x 16 x 16 12.3 and 13.3 us).
    auto labels_j = [&](int lpt) {
        int nj = K2 < kStripJ ? K2 : kStripJ;
        while (nj > 1 && items(lpt, nj) > 256 && gx * gy * ((K2 + nj - 1) / nj) < 256) nj = (nj + 1) / 2;
        return nj;
    };
    auto fits = [&](int lpt) { return K % lpt == 0 && (uintptr_t)out % (lpt * sizeof(OT)) == 0; };
    // at most 256 threads, the items spread evenly over their turns
    auto block = [&](int n) {
        const int turns = (n + 255) / 256;
        return dim3((unsigned)(((n + turns - 1) / turns + 63) / 64 * 64));
    };
    auto launch = [&](auto lpt) {
        constexpr int LPT = decltype(lpt)::value;
        const int nj = labels_j(LPT);
        const dim3 grid((unsigned)gx, (unsigned)gy, (unsigned)((K2 + nj - 1) / nj));
        hipLaunchKernelGGL((sad_strip_kernel<OT, R, DIR, LPT>), grid, block(items(LPT, nj)),
                           strip_lds_floats(R, K, nj) * sizeof(float), st, A, B, W, H, K, K2, off1, off2, nj, trunc,
                           inv_area, out, sw);
    };
    if constexpr (R <= 1) {
        if (fits(4)) {
            launch(std::integral_constant<int, 4>());
            return hipGetLastError();
        }
    }
    if (fits(2)) launch(std::integral_constant<int, 2>());
    else launch(std::integral_constant<int, 1>());
    return hipGetLastError();
}

}  // namespace dm
