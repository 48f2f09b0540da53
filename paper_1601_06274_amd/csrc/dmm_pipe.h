// dmm_pipe.h - chain sweeps by pipelines of waves: one walks the chains, two move the data.
//
// The passes of chain_kernel (dmm_kernels.h: backward message pass, update passes, final
// min-marginal pass) with the work of a node split over the three waves of a workgroup:
//
//   loader   loads cost, dual, reverse message and edge weight through a register ring of
//            pipe_ahead() nodes, forms the unaries and stages them in LDS, two chunks of
//            C nodes ahead of the chain wave;
//   chain    per node: the sums of unary, carried and reverse message, the minimum of the
//            message input, the message.  Its inputs come from LDS, its results (the
//            min-marginals, the message) go back to LDS;
//   storer   one chunk behind: the minimum of the min-marginals, duals, labels, bounds, and
//            their stores.
//
// What bounds it: a chain's nodes are a serial dependence, so a sweep over few chains costs
// (nodes) x (issue and latency of one node on one SIMD); the one-wave kernel spends half of
// that on loads, stores, addresses, dual updates and the second minimum.  With those on two
// other SIMDs a node of the recursion is about 25 (1 label per lane) to 45 (3) instructions.
// C nodes between two barriers keep a barrier's cost to a few cycles per node; four staging
// buffers (being written, two ahead of the chain wave, read back for the dual update) and
// two result buffers leave room for several workgroups' LDS on a CU.
//
// Measured, half-step of 4 passes (one-wave kernel -> here): rows of 320x240, K = 64, FP16
// 198 -> 102 us (155 -> 80 ns a node), 128x96, K = 32 88 -> 55 us; with all of a large frame's
// traffic to HBM the gain is what bandwidth leaves: 640x480, K = 128, FP32 rows 534 -> 424 us
// (6.3 TB/s), 1242x375, K = 192, FP16 rows 1130 -> 1074 us.  The chain wave alone takes 72,
// 106, 128 ns a node at 1, 2, 3 labels per lane.  Messages by scans (T > 3), whole solve of
// 611x437, K = 100, T = 6: 5.91 -> 5.10 ms.
// A batched plan (a workgroup per chains of every frame, longest first), four iterations of 64
// uneven frames: 177 -> 164 ms.
// Whole-lane vectors where K is a multiple of the labels per lane, not only for a full tile
// (one access a label before): the T = 6 solve above 5.10 -> 4.30 ms, a plan of six
// frames up to 640x360, K = 128, with refinement 11.0 -> 10.1 ms.
//
// The arithmetic of every value is chain_kernel's, operation for operation, so the results
// are the same bit for bit, whatever tile (lanes, labels per lane) either uses.
#pragma once

#include "batched_kernels.h"
#include "dmm_kernels.h"
#include "pipe_rule.h"

namespace dm {

// Nodes in flight in the loader's register ring (fewer where their registers would pass 256:
// values moved to the accumulation registers would be waited for as they arrive).
constexpr int pipe_ahead(int lpl, bool theta) { return lpl <= 2 ? 16 : (lpl == 3 ? (theta ? 12 : 16) : (theta ? 8 : 12)); }

using lds_u32 = __attribute__((address_space(3))) uint32_t;
typedef uint32_t pipe_u4 __attribute__((ext_vector_type(4)));
typedef uint32_t pipe_u2 __attribute__((ext_vector_type(2)));
using lds_u4 = __attribute__((address_space(3))) pipe_u4;
using lds_u2 = __attribute__((address_space(3))) pipe_u2;

// Node records of NW words per lane in LDS: group k (words 4k .. 4k+3) of node slot s and
// lane l at base + k * 1024 * SLOTS + (s * 64 + l) * 16 bytes (a shorter last group: its size).
template <int NW, int SLOTS>
struct PipeRec {
    static constexpr int NP = pipe_padded(NW);
    lds_u32* base;
    template <int W>
    static constexpr int group_words() { return (NP - W / 4 * 4) < 4 ? (NP - W / 4 * 4) : 4; }
    template <int W>
    __device__ __forceinline__ lds_u32* at(int slot, int lane) const {  // the group that holds word W
        return base + W / 4 * (4 * 64 * SLOTS) + (slot * 64 + lane) * group_words<W>();
    }
    // words FIRST .. FIRST + N - 1 of w
    template <int FIRST, int N>
    __device__ __forceinline__ void put(int slot, int lane, const uint32_t* w) const {
        if constexpr (N > 0) {
            constexpr int in = FIRST % 4, take = (4 - in) < N ? (4 - in) : N;
            lds_u32* p = at<FIRST>(slot, lane);
            if constexpr (in == 0 && take >= 3 && group_words<FIRST>() == 4) {
                pipe_u4 v = {w[0], w[1], w[2], take == 4 ? w[3] : 0u};
                *(lds_u4*)p = v;
            } else if constexpr (in % 2 == 0 && take == 2) {
                pipe_u2 v = {w[0], w[1]};
                *(lds_u2*)(p + in) = v;
            } else {
#pragma unroll
                for (int i = 0; i < take; ++i) p[in + i] = w[i];
            }
            put<FIRST + take, N - take>(slot, lane, w + take);
        }
    }
    template <int FIRST, int N>
    __device__ __forceinline__ void get(int slot, int lane, uint32_t* w) const {
        if constexpr (N > 0) {
            constexpr int in = FIRST % 4, take = (4 - in) < N ? (4 - in) : N;
            const lds_u32* p = at<FIRST>(slot, lane);
            if constexpr (in == 0 && take >= 3 && group_words<FIRST>() == 4) {
                const pipe_u4 v = *(const lds_u4*)p;
#pragma unroll
                for (int i = 0; i < take; ++i) w[i] = v[i];
            } else if constexpr (in % 2 == 0 && take == 2) {
                const pipe_u2 v = *(const lds_u2*)(p + in);
                w[0] = v[0];
                w[1] = v[1];
            } else {
#pragma unroll
                for (int i = 0; i < take; ++i) w[i] = p[in + i];
            }
            get<FIRST + take, N - take>(slot, lane, w + take);
        }
    }
};

// Barrier of the workgroup's waves for LDS data only: global loads and stores stay in flight.
// Nothing is scheduled across it either: arithmetic on a later chunk's loads, moved up, would
// wait for them.
__device__ __forceinline__ void pipe_barrier() {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}
// The same, after every global access of this wave has completed: what one wave stored
// before it, another wave of the workgroup (same CU, same L1) may load after it.
__device__ __forceinline__ void pipe_barrier_global() {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

constexpr int kRowBcast15 = 0x142;  // DPP: rows 1..3 <- lane 15 of the row before
constexpr int kRowBcast31 = 0x143;  // DPP: rows 2, 3 <- lane 31

// Intervals (barrier to barrier) of a pass: every chunk staged, walked and stored.
constexpr int pipe_intervals(int n_chunks) { return n_chunks + 3; }

// ------------------------------------------------------------------ chain wave
// KIND as in Walker::pass: 0 message pass, 1 iterative update, 2 naive update, 3 final.
// MF: message form as there - 0 scans, 2 direct window, 3 direct window with T = 3.
template <int G, int LPL, int MF, bool HAS_THETA>
struct PipeChain {
    static constexpr int C = pipe_chunk(LPL);
    static constexpr int NIN = pipe_in_words(LPL, HAS_THETA), NOUT = pipe_out_words(LPL);
    PipeRec<NIN, kPipeBufs * C> in;
    PipeRec<NOUT, 2 * C> out;
    const lds_u32* wgt;  // this group's edge weights
    int lane, sub, T;
    int dt_steps;  // scans: lanes that the truncation reaches across
    bool lv[LPL];  // label exists
    // lane shifts: lanes without a source keep kBig
    float dl, dr, dl2, dr2, b15, b31;

    template <int CTRL>
    __device__ __forceinline__ static float shift(float x, float& keep) {
        keep = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, keep),
                                                                     __builtin_bit_cast(int, x), CTRL, 0xF, 0xF, false));
        return keep;
    }
    // Value of the lane `sub - 1` / `sub + 1` of the group, kBig at its ends.
    __device__ __forceinline__ float from_left(float x, float& keep) const {
        if constexpr (G == 64) return shift<kWaveShr1>(x, keep);
        if constexpr (G == 16) return shift<kRowShr1>(x, keep);
        const float c = dpp_fill<kWaveShr1>(x, kBig);
        return sub == 0 ? kBig : c;
    }
    __device__ __forceinline__ float from_right(float x, float& keep) const {
        if constexpr (G == 64) return shift<kWaveShl1>(x, keep);
        if constexpr (G == 16) return shift<kRowShl1>(x, keep);
        const float c = dpp_fill<kWaveShl1>(x, kBig);
        return sub == G - 1 ? kBig : c;
    }
    // Minimum over the group.  A whole wave's ends in a scalar register: two row broadcasts
    // (rows without a source keep kBig) gather it in lane 63, fewer steps than the swaps
    // that leave it in every lane.
    __device__ __forceinline__ float minimum(float x) {
        if constexpr (G == 64) {
            x = group_min<16>(x);
            x = fminf(x, shift<kRowBcast15>(x, b15));
            x = fminf(x, shift<kRowBcast31>(x, b31));
            return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), 63));
        }
        return group_min<G>(x);
    }

    // The message (Walker::message_direct, Walker::message) without the cap and the
    // normalisation, so that it does not wait for the minimum.  Labels that do not exist
    // hold kBig in v, so no window takes them, and what comes out at them is never used.
    __device__ __forceinline__ void window(const float (&v)[LPL], float wt, float (&e)[LPL]) {
        if constexpr (MF == 0) {
            float f[LPL], b[LPL];
            f[0] = v[0];
#pragma unroll
            for (int i = 1; i < LPL; ++i) f[i] = fminf(v[i], f[i - 1] + wt);
            b[LPL - 1] = v[LPL - 1];
#pragma unroll
            for (int i = LPL - 2; i >= 0; --i) b[i] = fminf(v[i], b[i + 1] + wt);
            for (int s = 0; s < dt_steps; ++s) {
                const float cl = from_left(f[LPL - 1], dl);
                const float cr = from_right(b[0], dr);
#pragma unroll
                for (int i = 0; i < LPL; ++i) {
                    f[i] = fminf(f[i], wdist(wt, i + 1, cl));
                    b[i] = fminf(b[i], wdist(wt, LPL - i, cr));
                }
            }
#pragma unroll
            for (int i = 0; i < LPL; ++i) e[i] = fminf(f[i], b[i]);
            return;
        }
        constexpr bool T3 = MF == 3;
        const float w1 = (T3 || T > 1) ? wt : kBig;
        const float w2 = T > 2 ? wt + wt : kBig;
        const float l1 = from_left(v[LPL - 1], dl);
        const float r1 = from_right(v[0], dr);
        const float l2 = LPL >= 2 ? from_left(v[LPL >= 2 ? LPL - 2 : 0], dl2) : from_left(l1, dl2);
        const float r2 = LPL >= 2 ? from_right(v[LPL >= 2 ? 1 : 0], dr2) : from_right(r1, dr2);
        auto val = [&](int a) -> float {
            return a < 0 ? (a == -1 ? l1 : l2) : (a >= LPL ? (a == LPL ? r1 : r2) : v[a]);
        };
#pragma unroll
        for (int i = 0; i < LPL; ++i) {
            const float cm1 = val(i - 1) + w1, cp1 = val(i + 1) + w1;
            const float cm2 = T3 ? __builtin_fmaf(wt, 2.0f, val(i - 2)) : val(i - 2) + w2;
            const float cp2 = T3 ? __builtin_fmaf(wt, 2.0f, val(i + 2)) : val(i + 2) + w2;
            e[i] = fminf(fminf(fminf(v[i], cm1), cp1), fminf(cm2, cp2));
        }
    }

    template <int KIND>
    __device__ __forceinline__ void node(const uint32_t* w, uint32_t wbits, float (&carry)[LPL],
                                         const float (&gam)[LPL], float Tv, int oslot) {
        const float wt = __builtin_bit_cast(float, wbits);
        float v[LPL], e[LPL];
        uint32_t o[NOUT];
#pragma unroll
        for (int i = 0; i < LPL; ++i) v[i] = __builtin_bit_cast(float, w[i]) + carry[i];
        if constexpr (KIND != 0) {
#pragma unroll
            for (int i = 0; i < LPL; ++i) {
                const float m = v[i] + __builtin_bit_cast(float, w[LPL + i]);
                o[i] = __builtin_bit_cast(uint32_t, m);
                if constexpr (KIND == 1) v[i] = __builtin_fmaf(-gam[i], m, v[i]);
            }
        }
        float lm = v[0];
#pragma unroll
        for (int i = 1; i < LPL; ++i) lm = fminf(lm, v[i]);
        const float vmin = minimum(lm);
        window(v, wt, e);
        const float cap = __builtin_fmaf(wt, Tv, vmin);
#pragma unroll
        for (int i = 0; i < LPL; ++i) {
            carry[i] = fminf(e[i], cap) - vmin;
            o[LPL + i] = __builtin_bit_cast(uint32_t, carry[i]);
        }
        if constexpr (KIND == 0) {
            o[LPL - 1] = __builtin_bit_cast(uint32_t, vmin);
            out.template put<LPL - 1, LPL + 1>(oslot, lane, o + LPL - 1);
        } else {
            out.template put<0, NOUT>(oslot, lane, o);
        }
    }

    // Chunks of one pass: interval i works on chunk i - 2 (staged during interval i - 2); the
    // records of the next R nodes are read ahead.
    template <int KIND>
    __device__ __forceinline__ void pass(int n_chunks, float gamma) {
        constexpr int R = 4;                           // nodes read ahead
        constexpr int NR = KIND == 0 ? LPL : 2 * LPL;  // words the recursion reads
        float carry[LPL], gam[LPL];
#pragma unroll
        for (int i = 0; i < LPL; ++i) {
            carry[i] = 0.0f;
            gam[i] = lv[i] ? gamma : 0.0f;  // a missing label's input stays kBig
        }
        dl = dr = dl2 = dr2 = b15 = b31 = kBig;
        float Tv = (float)T;
        asm volatile("" : "+v"(Tv));  // in a vector register: the cap's fma reads the minimum from a scalar one
        uint32_t ring[R][2 * LPL], wring[R];
        pipe_barrier();
        pipe_barrier();
        for (int c = 0; c < n_chunks; ++c) {
            const int b0 = (c % kPipeBufs) * C, b1 = ((c + 1) % kPipeBufs) * C, ob = (c & 1) * C;
            const lds_u32 *w0 = wgt + (c % kPipeBufs) * 64, *w1 = wgt + ((c + 1) % kPipeBufs) * 64;
            if (c == 0) {
#pragma unroll
                for (int q = 0; q < R; ++q) {
                    in.template get<0, NR>(b0 + q, lane, ring[q]);
                    wring[q] = w0[q];
                }
            }
#pragma unroll
            for (int q = 0; q < C; ++q) {
                node<KIND>(ring[q % R], wring[q % R], carry, gam, Tv, ob + q);
                in.template get<0, NR>(q + R < C ? b0 + q + R : b1 + q + R - C, lane, ring[q % R]);
                wring[q % R] = q + R < C ? w0[q + R] : w1[q + R - C];
            }
            pipe_barrier();
        }
        pipe_barrier();
    }
};

// ------------------------------------------------------------------ loader
// VEC: every lane's labels exist or none do (pipe_vec), so a lane's values move as one
// vector; else one access per label.
// Node offsets: a lane's offset in a volume is fixed (its label at node 0; out of range for
// labels and chains that do not exist), the node's offset is scalar and stays inside the
// chain.  Nodes beyond the end are loaded at an out-of-range lane offset: no traffic for
// values that are never used.  Lines that the storer writes may be loaded meanwhile for other
// nodes (the end of a row and the start of the next one); the waves of a workgroup share the
// CU's L1, and what one has stored another reads after both waited for their accesses
// (pipe_barrier_global).
template <int G, int LPL, typename TT, bool VEC, bool HAS_THETA>
struct PipeLane {
    static constexpr int ES = (int)sizeof(TT);
    unsigned f0, th0, w0, lab0;       // byte offsets at node 0: FP32 volumes, cost, edge weights, labels
    unsigned f[LPL], th[LPL];         // of each label (scalar accesses)
    unsigned f_step, th_step, w_step, lab_step;
    bool ok, lv[LPL];
    int sub, K;
    __device__ __forceinline__ PipeLane(const SweepArgs& a, int chain, int sub_) : sub(sub_), K(a.K) {
        ok = chain < a.n_chains;
        const unsigned long long cpx = (unsigned long long)(ok ? chain : 0) * (unsigned long long)a.chain_px;
        const unsigned long long e0 = cpx * (unsigned long long)a.K + (unsigned long long)(sub * LPL);
        const unsigned nk = (unsigned)(a.node_px * (long long)a.K);
        const bool any = ok && sub * LPL < K;
        f0 = any ? (unsigned)(e0 * 4ull) : kOOB;
        th0 = any ? (unsigned)(e0 * (unsigned long long)ES) : kOOB;
        w0 = ok ? (unsigned)((unsigned long long)chain * (unsigned long long)a.w_chain * 4ull) : kOOB;
        lab0 = ok && sub == 0 ? (unsigned)(cpx * 4ull) : kOOB;
        f_step = nk * 4u;
        th_step = nk * (unsigned)ES;
        w_step = (unsigned)(a.w_node * 4);
        lab_step = (unsigned)(a.node_px * 4);
#pragma unroll
        for (int i = 0; i < LPL; ++i) {
            lv[i] = ok && sub * LPL + i < K;
            f[i] = lv[i] ? f0 + 4u * i : kOOB;
            th[i] = lv[i] ? th0 + (unsigned)(ES * i) : kOOB;
        }
    }
};

// NW consecutive dwords at lane offset `off` + scalar offset `so`.
template <int NW>
__device__ __forceinline__ void load_words_s(__amdgpu_buffer_rsrc_t r, unsigned off, unsigned so, uint32_t* w) {
    if constexpr (NW == 4) {
        auto v = __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, (int)so, 0);
        w[0] = v[0]; w[1] = v[1]; w[2] = v[2]; w[3] = v[3];
    } else if constexpr (NW == 3) {
        auto v = __builtin_amdgcn_raw_buffer_load_b96(r, (int)off, (int)so, 0);
        w[0] = v[0]; w[1] = v[1]; w[2] = v[2];
    } else if constexpr (NW == 2) {
        auto v = __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, (int)so, 0);
        w[0] = v[0]; w[1] = v[1];
    } else {
        w[0] = __builtin_amdgcn_raw_buffer_load_b32(r, (int)off, (int)so, 0);
    }
}
template <int G, int LPL, typename TT, bool VEC, bool HAS_THETA>
struct PipeLoad {
    static constexpr int C = pipe_chunk(LPL);
    static constexpr int NIN = pipe_in_words(LPL, HAS_THETA);
    static constexpr int D = pipe_ahead(LPL, HAS_THETA), U = D / C;  // nodes in flight, intervals per turn of the ring
    // FP16 costs moved as vectors: a lane's labels packed in dwords; 3 labels start at 6 * sub
    // bytes, so the 8 bytes from the dword at or below hold them, shifted by a half for odd
    // lanes (the labels of a pixel end on a dword).
    static constexpr bool kPacked = sizeof(TT) == 2 && VEC && LPL > 1;
    static constexpr int TW = sizeof(TT) == 2 ? (kPacked ? (LPL + 1) / 2 : LPL) : LPL;
    using Lane = PipeLane<G, LPL, TT, VEC, HAS_THETA>;
    struct Node {
        uint32_t th[TW], lam[LPL], rev[LPL];
    };
    PipeRec<NIN, kPipeBufs * C> in;
    lds_u32* wgt;  // edge weights in LDS, this lane's word
    int lane, n;
    __amdgpu_buffer_rsrc_t r_theta, r_lam, r_msg, r_w;
    float one;  // 1.0 that the compiler cannot see: cost - dual as one (mixed-precision) FMA

    __device__ __forceinline__ static void load_f32(const Lane& ln, __amdgpu_buffer_rsrc_t r, bool live, unsigned so,
                                                    uint32_t* w) {
        if constexpr (VEC) {
            load_words_s<LPL>(r, live ? ln.f0 : kOOB, so, w);
        } else {
#pragma unroll
            for (int i = 0; i < LPL; ++i)
                w[i] = __builtin_amdgcn_raw_buffer_load_b32(r, (int)(live ? ln.f[i] : kOOB), (int)so, 0);
        }
    }
    __device__ __forceinline__ float cost(const Lane& ln, const Node& nd, int i) const {
        if constexpr (sizeof(TT) == 4) {
            return __builtin_bit_cast(float, nd.th[i]);
        } else if constexpr (kPacked && LPL == 3) {
            const uint32_t sh = (ln.sub & 1) ? 16u : 0u;
            if (i == 2) return f16_bits_to_f(nd.th[1] >> sh);
            const uint32_t lo = __builtin_amdgcn_alignbit(nd.th[1], nd.th[0], sh);
            return f16_bits_to_f(lo >> (16 * i));
        } else if constexpr (kPacked) {
            return f16_bits_to_f(nd.th[i >> 1] >> (16 * (i & 1)));
        } else {
            return f16_bits_to_f(nd.th[i]);
        }
    }
    // The node at walking position t of a pass in direction FWD.  IN: it is inside the chain.
    template <bool FWD, bool REV, bool IN>
    __device__ __forceinline__ void load(const Lane& ln, int t, Node& nd) const {
        const bool live = IN || t < n;
        const int tc = live ? t : n - 1;
        const int j = FWD ? tc : n - 1 - tc;
        const unsigned so = (unsigned)j * ln.f_step;
        if constexpr (REV) {
            // slot of the edge toward the unvisited side
            const int jr = FWD ? j : (j > 0 ? j - 1 : 0);
            load_f32(ln, r_msg, live, (unsigned)jr * ln.f_step, nd.rev);
        }
        load_f32(ln, r_lam, live, so, nd.lam);
        if constexpr (HAS_THETA) {
            const unsigned st = (unsigned)j * ln.th_step;
            if constexpr (sizeof(TT) == 2 && !kPacked) {
#pragma unroll
                for (int i = 0; i < LPL; ++i)
                    nd.th[i] = __builtin_amdgcn_raw_buffer_load_b16(r_theta, (int)(live ? ln.th[i] : kOOB), (int)st, 0);
            } else if constexpr (kPacked) {
                load_words_s<TW>(r_theta, live ? ln.th0 & ~3u : kOOB, st, nd.th);
            } else if constexpr (VEC) {
                load_words_s<LPL>(r_theta, live ? ln.th0 : kOOB, st, nd.th);
            } else {
#pragma unroll
                for (int i = 0; i < LPL; ++i)
                    nd.th[i] = __builtin_amdgcn_raw_buffer_load_b32(r_theta, (int)(live ? ln.th[i] : kOOB), (int)st, 0);
            }
        }
    }
    // weight of the chunk's node `sub`: the edge toward the next node in the walking direction
    template <bool FWD>
    __device__ __forceinline__ uint32_t load_w(const Lane& ln, int c) const {
        const int t = c * C + ln.sub;
        const unsigned off = ln.sub < C && t < n - 1 ? ln.w0 + (unsigned)(FWD ? t : n - 2 - t) * ln.w_step : kOOB;
        return __builtin_amdgcn_raw_buffer_load_b32(r_w, (int)off, 0, 0);
    }

    // Intervals i0 .. i0 + U - 1: stage their chunks, refill the ring with the nodes D further.
    template <bool FWD, int KIND, bool IN>
    __device__ __forceinline__ void turn(const Lane& ln, int i0, int n_chunks, Node (&ring)[D], uint32_t (&wring)[U]) {
        constexpr bool REV = KIND != 0;
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int i = i0 + k;
            if (!IN && i >= n_chunks) return;
            const int ib = (i % kPipeBufs) * C;
            wgt[(i % kPipeBufs) * 64] = wring[k];
            wring[k] = load_w<FWD>(ln, i + U);
#pragma unroll
            for (int q = 0; q < C; ++q) {
                Node& nd = ring[k * C + q];
                // Records of 3 labels cut across the loaded words: copies made here, not by the
                // register allocator where the loads are issued (they would wait there).
                if constexpr (LPL == 3) {
#pragma unroll
                    for (int l = 0; l < LPL; ++l) {
                        nd.lam[l] = opaque_copy(nd.lam[l]);
                        if constexpr (REV) nd.rev[l] = opaque_copy(nd.rev[l]);
                    }
                }
                uint32_t w[3 * LPL];
                const bool has_next = IN || i * C + q < n - 1;
#pragma unroll
                for (int l = 0; l < LPL; ++l) {
                    const float lam = __builtin_bit_cast(float, nd.lam[l]);
                    const float x = HAS_THETA ? __builtin_fmaf(cost(ln, nd, l), one, -lam) : lam;
                    w[l] = __builtin_bit_cast(uint32_t, ln.lv[l] ? x : kBig);
                    w[2 * LPL + l] = nd.lam[l];
                    if constexpr (REV) w[LPL + l] = has_next ? nd.rev[l] : 0u;  // no message beyond the end
                }
                if constexpr (REV) in.template put<0, NIN>(ib + q, lane, w);
                else in.template put<0, LPL>(ib + q, lane, w);
                load<FWD, REV, IN>(ln, (i + U) * C + q, nd);
                __builtin_amdgcn_sched_barrier(0);
            }
            pipe_barrier();
        }
    }

    template <bool FWD, int KIND>
    __device__ __forceinline__ void pass(const Lane& ln, int n_chunks) {
        constexpr bool REV = KIND != 0;
        static_assert(G >= C && D % C == 0, "a group's lanes hold a chunk's edge weights");
        const int n_int = pipe_intervals(n_chunks);
        Node ring[D];
        uint32_t wring[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            wring[k] = load_w<FWD>(ln, k);
#pragma unroll
            for (int q = 0; q < C; ++q) {
                load<FWD, REV, false>(ln, k * C + q, ring[k * C + q]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        // whole turns of the ring; in all but the last ones every node staged has a successor
        // and every node loaded exists
        int i0 = 0;
        for (; (i0 + 2 * U) * C <= n; i0 += U) turn<FWD, KIND, true>(ln, i0, n_chunks, ring, wring);
        for (; i0 < n_chunks; i0 += U) turn<FWD, KIND, false>(ln, i0, n_chunks, ring, wring);
        for (int i = n_chunks; i < n_int - 1; ++i) pipe_barrier();
        pipe_barrier_global();
    }
};

// ------------------------------------------------------------------ storer
template <int G, int LPL, typename TT, bool VEC, bool HAS_THETA>
struct PipeStore {
    static constexpr int C = pipe_chunk(LPL);
    static constexpr int NIN = pipe_in_words(LPL, HAS_THETA), NOUT = pipe_out_words(LPL);
    using Lane = PipeLane<G, LPL, TT, VEC, HAS_THETA>;
    PipeRec<NIN, kPipeBufs * C> in;
    PipeRec<NOUT, 2 * C> out;
    int lane, n;
    __amdgpu_buffer_rsrc_t r_lam, r_msg, r_mm, r_lab;
    float sign;
    static_assert(C % 4 == 0, "a chunk is whole groups of four nodes");

    // The node's offset is added in the vector register: a store of 3 or 4 dwords reads its
    // data a cycle after it issues, and the compiler keeps the next instruction from
    // overwriting that data only where the store has no scalar offset register.
    __device__ __forceinline__ static void store(const Lane& ln, __amdgpu_buffer_rsrc_t r, unsigned so, const float (&x)[LPL]) {
        unsigned os[LPL];
#pragma unroll
        for (int i = 0; i < LPL; ++i) os[i] = ln.lv[i] ? ln.f[i] + so : kOOB;
        store_f32<LPL, VEC>(r, ln.f0 != kOOB ? ln.f0 + so : kOOB, os, x);
    }

    // Group minima of N nodes' lane minima x.  A whole wave's four at a time: two permlane
    // swaps put one node into each row of 16 lanes on the way down, so the four share the
    // steps inside a row, and a read of each row's lane leaves them in scalar registers.
    template <int N>
    __device__ __forceinline__ static void minima(float (&x)[N]) {
        if constexpr (G == 64 && N == 4) {
            float c[2];
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                auto p = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, x[2 * k]),
                                                          __builtin_bit_cast(uint32_t, x[2 * k + 1]), false, false);
                c[k] = fminf(__builtin_bit_cast(float, (uint32_t)p[0]), __builtin_bit_cast(float, (uint32_t)p[1]));
            }
            auto p = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, c[0]),
                                                      __builtin_bit_cast(uint32_t, c[1]), false, false);
            // rows 0 .. 3: nodes 0, 2, 1, 3
            const float r = group_min<16>(
                fminf(__builtin_bit_cast(float, (uint32_t)p[0]), __builtin_bit_cast(float, (uint32_t)p[1])));
            const int b = __builtin_bit_cast(int, r);
            x[0] = __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 0));
            x[2] = __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 16));
            x[1] = __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 32));
            x[3] = __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 48));
        } else {
#pragma unroll
            for (int i = 0; i < N; ++i) x[i] = group_min<G>(x[i]);
        }
    }

    // Results of the N nodes from walking position t on (staged in slots fslot + i and
    // oslot + i).  LAST: they may include the chain's last node (it sends no message) and
    // positions beyond it.
    template <bool FWD, int KIND, int N, bool LAST>
    __device__ __forceinline__ void finish(const Lane& ln, int t, int fslot, int oslot, float g, __amdgpu_buffer_rsrc_t msg_st,
                                           double& opt) {
        uint32_t o[N][NOUT], lw[N][LPL];
#pragma unroll
        for (int i = 0; i < N; ++i) {
            if constexpr (KIND == 0) out.template get<LPL - 1, LPL + 1>(oslot + i, lane, o[i] + LPL - 1);
            else if constexpr (KIND == 3) out.template get<0, LPL>(oslot + i, lane, o[i]);
            else out.template get<0, NOUT>(oslot + i, lane, o[i]);
            if constexpr (KIND == 1) in.template get<HAS_THETA ? 2 * LPL : 0, LPL>(fslot + i, lane, lw[i]);
        }
        float mn[N];
        if constexpr (KIND != 0) {
#pragma unroll
            for (int i = 0; i < N; ++i) {
                mn[i] = __builtin_bit_cast(float, o[i][0]);
#pragma unroll
                for (int l = 1; l < LPL; ++l) mn[i] = fminf(mn[i], __builtin_bit_cast(float, o[i][l]));
            }
            minima<N>(mn);
        }
#pragma unroll
        for (int i = 0; i < N; ++i) {
            if (LAST && t + i >= n) return;
            const int j = FWD ? t + i : n - 1 - (t + i);
            const unsigned so = (unsigned)j * ln.f_step;
            if constexpr (KIND == 0) {
                opt += (double)__builtin_bit_cast(float, o[i][LPL - 1]);
            } else {
                float x[LPL];
                if constexpr (KIND == 3) {
                    int first = 0x7fffffff;
#pragma unroll
                    for (int l = LPL - 1; l >= 0; --l) {
                        const float m = __builtin_bit_cast(float, o[i][l]);
                        x[l] = m - mn[i];
                        if (ln.lv[l] && m == mn[i]) first = ln.sub * LPL + l;
                    }
                    int lab = group_min_i<G>(first);
                    lab = lab < ln.K ? lab : ln.K - 1;  // a label always exists for finite costs
                    store(ln, r_mm, so, x);
                    __builtin_amdgcn_raw_buffer_store_b32((uint32_t)lab, r_lab, (int)(ln.lab0 != kOOB ? ln.lab0 + (unsigned)j * ln.lab_step : kOOB), 0, 0);
                } else {
#pragma unroll
                    for (int l = 0; l < LPL; ++l) {
                        const float d = g * (__builtin_bit_cast(float, o[i][l]) - mn[i]);
                        x[l] = __builtin_fmaf(sign, d, __builtin_bit_cast(float, lw[i][l]));
                    }
                    store(ln, r_lam, so, x);
                }
            }
            if constexpr (KIND != 3) {
                if (!LAST || t + i < n - 1) {
                    float msg[LPL];
#pragma unroll
                    for (int l = 0; l < LPL; ++l) msg[l] = __builtin_bit_cast(float, o[i][LPL + l]);
                    store(ln, msg_st, FWD ? so : so - ln.f_step, msg);
                }
            }
        }
    }

    // opt: the message pass's normalisation constants, summed in node order
    template <bool FWD, int KIND>
    __device__ __forceinline__ void pass(const Lane& ln, int n_chunks, float g, bool store_msg, double& opt) {
        // a pass whose messages nobody reads stores them through an empty descriptor: no branch
        const __amdgpu_buffer_rsrc_t msg_st = store_msg ? r_msg : make_rsrc(nullptr, 0u);
        pipe_barrier();
        pipe_barrier();
        pipe_barrier();
        for (int c = 0; c < n_chunks; ++c) {
            const int fb = (c % kPipeBufs) * C, ob = (c & 1) * C;
            if (c * C + C < n) {
#pragma unroll
                for (int q = 0; q < C; q += 4) finish<FWD, KIND, 4, false>(ln, c * C + q, fb + q, ob + q, g, msg_st, opt);
            } else {
#pragma unroll 1
                for (int q = 0; q < C; q += 4) finish<FWD, KIND, 4, true>(ln, c * C + q, fb + q, ob + q, g, msg_st, opt);
            }
            if (c + 1 < n_chunks) pipe_barrier();
        }
        pipe_barrier_global();
    }
};

// All passes of one mode group for the chains chain0 .. chain0 + 64 / G - 1 of a, by the three
// waves of a workgroup.
template <int G, int LPL, typename TT, bool VEC, bool HAS_THETA, int MF, int MG>
__device__ __forceinline__ void pipe_run(const SweepArgs& a, int chain0, uint32_t* lds) {
    constexpr int C = pipe_chunk(LPL);
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64);
    const int lane = (int)threadIdx.x % 64;
    const int sub = lane % G, chain = chain0 + lane / G;
    const int n_chunks = (a.n + C - 1) / C;
    lds_u32* const base = (lds_u32*)lds;
    lds_u32* const obase = base + pipe_in_lds(LPL, HAS_THETA);
    lds_u32* const wbase = obase + pipe_out_lds(LPL);
    // R0, then the mode's passes; step s = 0 .. P-1 of a half-step walks forward first
    const bool iterative = MG == kGroupHalfStep && a.mode == kModeIterative;
    const int P = iterative ? a.n_pass : 1;
    auto gamma_of = [&](int s) {
        float g = a.gamma[0];  // selects: a dynamic index would put the arguments in scratch
#pragma unroll
        for (int i = 1; i < 8; ++i)
            if (s == i) g = a.gamma[i];
        return g;
    };
    if (wave == 0) {
        PipeChain<G, LPL, MF, HAS_THETA> ch;
        ch.in.base = base;
        ch.out.base = obase;
        ch.wgt = wbase + (lane - sub);
        ch.lane = lane;
        ch.sub = sub;
        ch.T = a.T;
        const int need = (a.T - 1 + LPL - 1) / LPL;
        ch.dt_steps = need < G - 1 ? need : G - 1;
#pragma unroll
        for (int i = 0; i < LPL; ++i) ch.lv[i] = chain < a.n_chains && sub * LPL + i < a.K;
        ch.template pass<0>(n_chunks, 0.0f);
        if constexpr (MG == kGroupFinal) {
            ch.template pass<3>(n_chunks, 0.0f);
        } else if constexpr (MG == kGroupHalfStep) {
            if (iterative)
                for (int s = 0; s < P; ++s) ch.template pass<1>(n_chunks, gamma_of(s));
            else
                ch.template pass<2>(n_chunks, 0.0f);
        }
    } else if (wave == 1) {
        using LD = PipeLoad<G, LPL, TT, VEC, HAS_THETA>;
        const typename LD::Lane ln(a, chain, sub);
        LD ld;
        ld.in.base = base;
        ld.wgt = wbase + lane;
        ld.lane = lane;
        ld.n = a.n;
        ld.one = a.sign * a.sign;
        ld.r_theta = make_rsrc(a.theta, HAS_THETA ? a.vol_bytes_theta : 0u);
        ld.r_lam = make_rsrc(a.lam_in != nullptr ? a.lam_in : a.lam, a.vol_bytes_f32);
        ld.r_msg = make_rsrc(a.msg, a.vol_bytes_f32);
        ld.r_w = make_rsrc(a.w, a.w_bytes);
        ld.template pass<false, 0>(ln, n_chunks);
        if constexpr (MG == kGroupFinal) {
            ld.template pass<true, 3>(ln, n_chunks);
        } else if constexpr (MG == kGroupHalfStep) {
            for (int s = 0; s < P; ++s) {
                if (s == 1) ld.r_lam = make_rsrc(a.lam, a.vol_bytes_f32);
                if ((s & 1) == 0) ld.template pass<true, 1>(ln, n_chunks);
                else ld.template pass<false, 1>(ln, n_chunks);
            }
        }
    } else {
        using ST = PipeStore<G, LPL, TT, VEC, HAS_THETA>;
        const typename ST::Lane ln(a, chain, sub);
        ST sr;
        sr.in.base = base;
        sr.out.base = obase;
        sr.lane = lane;
        sr.n = a.n;
        sr.sign = a.sign;
        sr.r_lam = make_rsrc(a.lam, a.vol_bytes_f32);
        sr.r_msg = make_rsrc(a.msg, a.vol_bytes_f32);
        sr.r_mm = make_rsrc(a.minmarg, a.minmarg != nullptr ? a.vol_bytes_f32 : 0u);
        sr.r_lab = make_rsrc(a.labels, a.labels != nullptr ? a.vol_bytes_f32 / (unsigned)a.K : 0u);
        double opt = 0.0;
        sr.template pass<false, 0>(ln, n_chunks, 0.0f, MG != kGroupOptimum, opt);
        if constexpr (MG == kGroupFinal) {
            sr.template pass<true, 3>(ln, n_chunks, 0.0f, false, opt);
        } else if constexpr (MG == kGroupHalfStep) {
            if (iterative) {
                for (int s = 0; s < P; ++s) {
                    if ((s & 1) == 0) sr.template pass<true, 1>(ln, n_chunks, gamma_of(s), s + 1 < P, opt);
                    else sr.template pass<false, 1>(ln, n_chunks, gamma_of(s), s + 1 < P, opt);
                }
            } else {
                sr.template pass<true, 1>(ln, n_chunks, a.inv_n, false, opt);
            }
        }
        if (a.opt != nullptr && ln.ok && sub == 0) a.opt[chain] = opt;
    }
}

template <int G, int LPL, typename TT, bool VEC, bool HAS_THETA, int MF, int MG>
__global__ __launch_bounds__(192) void pipe_kernel(SweepArgs a) {
    __shared__ __attribute__((aligned(16))) uint32_t lds[pipe_lds_words(LPL, HAS_THETA)];
    pipe_run<G, LPL, TT, VEC, HAS_THETA, MF, MG>(a, (int)blockIdx.x * (64 / G), lds);
}

// One workgroup per work item of a batched plan's table (longest chains first).
template <int G, int LPL, typename TT, bool VEC, bool HAS_THETA, int MF, int MG>
__global__ __launch_bounds__(192) void batched_pipe_kernel(BatchLaunch bl) {
    __shared__ __attribute__((aligned(16))) uint32_t lds[pipe_lds_words(LPL, HAS_THETA)];
    const BatchItem bi = bl.items[blockIdx.x];
    const SweepArgs a = batch_args(bl.insts[bi.inst], bl);
    pipe_run<G, LPL, TT, VEC, HAS_THETA, MF, MG>(a, bi.chain, lds);
}

// The kernels of a tile: half-steps (mode kModeIterative or kModeNaive), the final pass and
// the column optimum pass, for K <= G * LPL labels.  SCAN: messages by scans (any T), else
// the direct window (T <= 3).
template <int G, int LPL, bool SCAN, typename TT, bool VEC, bool HAS_THETA>
hipError_t launch_pipe_full(const SweepArgs& a, hipStream_t st) {
    constexpr int CPW = 64 / G;
    const dim3 grid((unsigned)((a.n_chains + CPW - 1) / CPW)), block(192);
#define DM_PIPE(MF, MG) hipLaunchKernelGGL((pipe_kernel<G, LPL, TT, VEC, HAS_THETA, MF, MG>), grid, block, 0, st, a)
    if (a.mode == kModeFinal) {
        DM_PIPE(SCAN ? 0 : 2, kGroupFinal);
    } else if (a.mode == kModeOptimum) {
        if constexpr (!HAS_THETA) DM_PIPE(SCAN ? 0 : 2, kGroupOptimum);
        else return hipErrorInvalidValue;
    } else if (SCAN || a.T == 3) {
        DM_PIPE(SCAN ? 0 : 3, kGroupHalfStep);
    } else {
        DM_PIPE(SCAN ? 0 : 2, kGroupHalfStep);
    }
#undef DM_PIPE
    return hipGetLastError();
}

template <int G, int LPL, bool SCAN, typename TT, bool HAS_THETA>
hipError_t launch_pipe_tt(const SweepArgs& a, hipStream_t st) {
    if constexpr (LPL > 1)
        if (!pipe_vec(a.K, LPL, HAS_THETA, sizeof(TT) == 2)) return launch_pipe_full<G, LPL, SCAN, TT, false, HAS_THETA>(a, st);
    return launch_pipe_full<G, LPL, SCAN, TT, true, HAS_THETA>(a, st);
}

template <int G, int LPL, bool SCAN>
hipError_t launch_pipe(const SweepArgs& a, dm_dtype dt, hipStream_t st) {
    if (a.theta == nullptr) return launch_pipe_tt<G, LPL, SCAN, float, false>(a, st);
    if (dt == DM_F16) return launch_pipe_tt<G, LPL, SCAN, _Float16, true>(a, st);
    return launch_pipe_tt<G, LPL, SCAN, float, true>(a, st);
}

// Batched form (direct window): family 0 reads the cost; vec: see pipe_vec.
template <int G, int LPL, typename TT, bool VEC, bool HAS_THETA>
hipError_t launch_batched_pipe_full(const BatchLaunch& bl, hipStream_t st) {
#define DM_BPIPE(MF, MG)                                                                                        \
    hipLaunchKernelGGL((batched_pipe_kernel<G, LPL, TT, VEC, HAS_THETA, MF, MG>), dim3((unsigned)bl.n_items), \
                       dim3(192), 0, st, bl)
    if (bl.mode == kModeFinal) {
        if constexpr (HAS_THETA) DM_BPIPE(2, kGroupFinal);
        else return hipErrorInvalidValue;
    } else if (bl.mode == kModeOptimum) {
        if constexpr (!HAS_THETA) DM_BPIPE(2, kGroupOptimum);
        else return hipErrorInvalidValue;
    } else if (bl.T == 3) {
        DM_BPIPE(3, kGroupHalfStep);
    } else {
        DM_BPIPE(2, kGroupHalfStep);
    }
#undef DM_BPIPE
    return hipGetLastError();
}

template <int G, int LPL, typename TT, bool HAS_THETA>
hipError_t launch_batched_pipe_tt(const BatchLaunch& bl, bool vec, hipStream_t st) {
    if constexpr (LPL > 1)
        if (!vec) return launch_batched_pipe_full<G, LPL, TT, false, HAS_THETA>(bl, st);
    return launch_batched_pipe_full<G, LPL, TT, true, HAS_THETA>(bl, st);
}

template <int G, int LPL>
hipError_t launch_batched_pipe(const BatchLaunch& bl, bool vec, dm_dtype dt, hipStream_t st) {
    if (bl.family != 0) return launch_batched_pipe_tt<G, LPL, float, false>(bl, vec, st);
    if (dt == DM_F16) return launch_batched_pipe_tt<G, LPL, _Float16, true>(bl, vec, st);
    return launch_batched_pipe_tt<G, LPL, float, true>(bl, vec, st);
}

}  // namespace dm
