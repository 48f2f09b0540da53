// pdhg.h - one primal-dual iteration of the refinement on a tile (Sec. 2.4, eq. cont_iterates),
// shared by the stereo refinement (two-slope data model, Sec. 3.1) and the flow refinement
// (quadratic data model per component, Sec. 3.2): the iteration differs only in the prox
// of the data term, a template argument.
//
// With x = (u, q), y = (p, d = 1), per pixel / edge:
//     u+ = prox_{tau D~}( u - tau A^T (p - q) )
//     q+ = prox_{tau R_-^*}( q + tau A u )
//     p+ = prox_{sigma R_+^*}( p + sigma A (2 u+ - u) ),
// (Au)_e = u_i - u_j for the right / lower neighbour j of i.  Edge arrays are stored per
// pixel: ph/qh at (x, y) belong to the edge (x, y)-(x+1, y) (unused in the last column),
// pv/qv to (x, y)-(x, y+1) (unused in the last row).  State is double buffered between
// launches (every read of a launch sees the previous launch's iterate).  DataProx is the
// prox of tau D~ of a pixel around its model: load(p) reads the pixel's model once per
// launch, apply(uh, model, kmax, code) returns the prox and its branch code (4 bits).
#pragma once

#include "refine.h"

namespace dm {

// Branch codes of the conjugate prox (3 bits): 0 = identity slope in t, 1 / 2 = flat at
// +alpha*w / -alpha*w, 3 / 4 = clamped at +w / -w.
// Written with selects (every candidate computed, no divergent branches).
__device__ __forceinline__ rfloat prox_conj(rfloat t, rfloat w, rfloat alpha, rfloat beta, rfloat step, int& code) {
    const rfloat a = fabs(t);
    const rfloat aw = alpha * w;
    const rfloat sh = a - beta * step;
    const bool inner = a <= aw;
    const bool flat = !inner && sh < aw;
    rfloat r = inner ? t : copysign(flat ? aw : sh, t);
    const int c = flat ? (t > 0.0 ? 1 : 2) : 0;
    const bool lo = r < -w, hi = r > w;
    r = lo ? -w : (hi ? w : r);
    code = lo ? 4 : (hi ? 3 : c);
    return r;
}

// Mask layout (uint16 per pixel and iteration): [0,4) u-prox, [4,7) qh, [7,10) qv,
// [10,13) ph, [13,16) pv.
__device__ __forceinline__ int mfield(uint32_t m, int shift, int bits) { return (int)((m >> shift) & ((1u << bits) - 1u)); }

// n_iter <= S iterations in one launch (temporal tiling).  A block owns a TX x TY output
// tile and runs the iteration on the tile extended by S pixels on every side, one pixel per
// thread: values within s pixels of the region's border are wrong after s iterations (their
// neighbours outside the region are missing), but every dependency of the iteration reaches
// one pixel, so after n_iter <= S iterations the output tile is exact, and the arithmetic
// per pixel and iteration (the same expressions in the same order for every tile shape and
// S) does not depend on the tiling: the results equal one iteration per launch bit for bit.
//
// A pixel's state, model and weights stay in registers; LDS holds what neighbours read: the
// edges' p - q (phase A, from the right and lower neighbour), the old u and 2 u+ - u (phase
// B, from the left and upper one).  What bounds it: vector issue (65 % of a busy CU's cycles at
// 1242 x 375, counted; a sixth of those instructions are FP64 additions, multiplications and
// FMAs, the rest the compares and selects of the proxes and addresses), 47 % of it for the
// halo's pixels, against launches and the latency of an iteration (two barriers).  One pixel
// per thread (16 waves a block, two blocks a CU) hides that latency where 6 pixels per thread
// in 4 waves did not; rows that no output of the remaining iterations depends on are skipped
// (a wave is two rows).
// mask0: the branch-mask plane of the first iteration (nullptr: no tape), mask_stride the
// element distance between consecutive iterations' planes.
template <int TX, int TY, int S, class DataProx>
__device__ __forceinline__ void pdhg_fused_tile(const RefineState& in, const RefineState& out, const DataProx& prox,
                                                const float* __restrict__ w_h, const float* __restrict__ w_v, int W,
                                                int H, int K, const RefineScalars& sc, uint16_t* __restrict__ mask0,
                                                size_t mask_stride, int n_iter, int x0, int y0) {
    constexpr int RX = TX + 2 * S, RY = TY + 2 * S, NP = RX * RY;
    // one row and one pixel of padding in front: the first pixels' left and upper neighbours
    __shared__ rfloat s_zh[NP + RX + 1], s_zv[NP + RX + 1];
    // and behind: the last pixels' right and lower ones
    __shared__ rfloat s_u[2][NP + RX], s_b[NP + RX];
    const int idx = (int)threadIdx.x, zi = idx + RX + 1;
    const int rx = idx % RX, ry = idx / RX;
    const int x = x0 - S + rx, y = y0 - S + ry;
    const rfloat kmax = (rfloat)(K - 1);
    const bool inside = x >= 0 && x < W && y >= 0 && y < H;
    const bool edge_h = inside && x + 1 < W, edge_v = inside && y + 1 < H;
    // the left / upper edges exist; beyond the region they count as 0 (never used)
    const bool left = x > 0 && rx > 0, up = y > 0 && ry > 0;
    const bool central = rx >= S && rx < S + TX && ry >= S && ry < S + TY && inside;
    const long long p = (long long)y * W + x;
    typename DataProx::Px dm{};
    float wh = 0.0f, wv = 0.0f;
    rfloat u = 0.0, ph = 0.0, pv = 0.0, qh = 0.0, qv = 0.0;
    if (inside) {
        u = in.u[p];
        ph = in.ph[p];
        pv = in.pv[p];
        qh = in.qh[p];
        qv = in.qv[p];
        dm = prox.load(p);
        if (edge_h) wh = w_h[(long long)y * (W - 1) + x];
        if (edge_v) wv = w_v[p];
    }
    s_zh[zi] = ph - qh;
    s_zv[zi] = pv - qv;
    s_u[0][idx] = u;
    __syncthreads();
    int cur = 0;
    for (int it = 0; it < n_iter; ++it) {
        const int rem = n_iter - it;
        int code = 0;
        // Phase A: u+ and the extrapolated 2 u+ - u.
        rfloat un = 0.0;
        const bool rows_a = ry >= S - rem && ry <= S + TY - 1 + rem;
        if (inside && rows_a) {
            // (A^T z)_i = z_h(i) + z_v(i) - z_h(left) - z_v(up), z = p - q
            rfloat at = 0.0;
            if (edge_h) at += ph - qh;
            if (edge_v) at += pv - qv;
            if (x > 0) at -= left ? s_zh[zi - 1] : 0.0;
            if (y > 0) at -= up ? s_zv[zi - RX] : 0.0;
            un = prox.apply(u - sc.tau * at, dm, kmax, code);
        }
        const rfloat b = 2.0 * un - u;
        if (rows_a) s_b[idx] = b;
        __syncthreads();
        // Phase B: q+ (old u) and p+ (extrapolated) on the pixel's edges.
        if (inside && ry >= S - rem && ry <= S + TY - 2 + rem) {
            uint32_t m = (uint32_t)code;
            int c;
            if (edge_h) {  // (beyond the region's right border: values that are never used)
                const rfloat gq = u - s_u[cur][idx + 1];
                const rfloat w = (rfloat)wh;
                qh = prox_conj(qh + sc.tau * gq, w, 0.0, sc.beta_minus, sc.tau, c);
                m |= (uint32_t)c << 4;
                const rfloat gp = b - s_b[idx + 1];
                ph = prox_conj(ph + sc.sigma * gp, w, sc.eps, sc.delta, sc.sigma, c);
                m |= (uint32_t)c << 10;
                s_zh[zi] = ph - qh;
            }
            if (edge_v) {
                const rfloat gq = u - s_u[cur][idx + RX];
                const rfloat w = (rfloat)wv;
                qv = prox_conj(qv + sc.tau * gq, w, 0.0, sc.beta_minus, sc.tau, c);
                m |= (uint32_t)c << 7;
                const rfloat gp = b - s_b[idx + RX];
                pv = prox_conj(pv + sc.sigma * gp, w, sc.eps, sc.delta, sc.sigma, c);
                m |= (uint32_t)c << 13;
                s_zv[zi] = pv - qv;
            }
            if (mask0 != nullptr && central) mask0[(size_t)it * mask_stride + p] = (uint16_t)m;
        }
        u = un;
        cur ^= 1;
        s_u[cur][idx] = u;
        __syncthreads();
    }
    if (central) {
        out.u[p] = u;
        out.ph[p] = ph;
        out.pv[p] = pv;
        out.qh[p] = qh;
        out.qv[p] = qv;
    }
}

// Fused tile shapes, forward (stereo, batched and flow) and adjoint: 22 x 22 outputs, 5
// iterations per launch, a 32 x 32 region of 1024 threads in at most 64 registers, so two
// blocks share a CU; 40 iterations per warp take 8 launches.  Measured, 5 x 40 iterations at
// 1242 x 375 and 320 x 240: forward 2039 -> 1380 and 1508 -> 511 us, adjoint with the
// linearisations 2319 -> 1706 and 1178 -> 583 us (before: 40 x 24 x 4 with 6 pixels per thread
// and 32 x 16 x 4 with 4, the state in LDS).  Other regions, forward: 32 x 24 (24 x 16 x 4)
// 1434 and 493, 20 x 20 x 6 1381 and 469, 16 x 16 x 8 2324 and 657 us; one block per CU
// (more registers) 1759 us.
constexpr int kFTX = 22, kFTY = 22, kFS = 5;
constexpr int kFNT = (kFTX + 2 * kFS) * (kFTY + 2 * kFS);  // threads: one per pixel of the region
constexpr int kATX = 22, kATY = 22, kAS = 5;
constexpr int kANT = (kATX + 2 * kAS) * (kATY + 2 * kAS);

}  // namespace dm
