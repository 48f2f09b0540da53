// pipe_rule.h - the LDS of a pipelined sweep's workgroup and the rule that chooses between the
// pipelined sweeps (dmm_pipe.h) and the one-wave kernels (dmm_kernels.h).  Host code.
#pragma once

#include "tiles.h"

namespace dm {

// Nodes between two barriers, staging buffers (chunks)
constexpr int pipe_chunk(int lpl) { return lpl == 1 ? 8 : 4; }
constexpr int kPipeBufs = 4;
// staged words of a node and lane: unary[LPL], reverse message[LPL] and, for rows (the
// columns' unary is the dual itself), dual[LPL]
constexpr int pipe_in_words(int lpl, bool theta) { return (theta ? 3 : 2) * lpl; }
// result words: min-marginal[LPL], message[LPL]; of a message pass (which has no
// min-marginals) word LPL - 1 is the minimum
constexpr int pipe_out_words(int lpl) { return 2 * lpl; }
// Words are kept in groups of 4 (one 16-byte LDS access); a last group of 3 takes 4.
constexpr int pipe_padded(int w) { return w % 4 == 3 ? w + 1 : w; }
// LDS words of the staging records, the result records and the edge weights (of a chunk:
// word q of a group's lanes is the weight of its node q)
constexpr int pipe_in_lds(int lpl, bool theta) { return 64 * pipe_chunk(lpl) * kPipeBufs * pipe_padded(pipe_in_words(lpl, theta)); }
constexpr int pipe_out_lds(int lpl) { return 64 * pipe_chunk(lpl) * 2 * pipe_padded(pipe_out_words(lpl)); }
constexpr int pipe_lds_words(int lpl, bool theta) { return pipe_in_lds(lpl, theta) + pipe_out_lds(lpl) + 64 * kPipeBufs; }
// workgroups that a CU holds by their LDS (160 KB, given in units of 1280 bytes)
constexpr int pipe_lds_count(int lpl, bool theta) { return 163840 / ((4 * pipe_lds_words(lpl, theta) + 1279) / 1280 * 1280); }

// Whole-lane vectors: every lane's labels exist or none do, and FP16 costs, read as dwords, start
// on one.
inline bool pipe_vec(int K, int lpl, bool theta, bool f16) {
    return lpl == 1 || (K % lpl == 0 && !(theta && f16 && K % 2 != 0));
}

// Workgroups per CU up to which the pipelined sweep on tile d is taken for a launch that the
// one-wave kernel would run on tile t (0: never).  theta: the rows, which read the cost.
//
// What decides is how much of the one-wave kernel's time the pipeline can take over, and how many
// workgroups run at once.  Measured: time of a one-wave half-step (300 to 900 nodes) over that of
// the pipelined one.
//   * A one-wave kernel on a tile that K does not fill accesses label by label.  Where the pipeline
//     moves whole vectors it gains at every count (K = 48, 100, 150, 240, 250 .. 1500 chains: 1.15 ..
//     3.4): as many as LDS holds.
//   * Where the pipeline accesses label by label too, 3 labels a lane leave registers for two
//     workgroups a CU and 4 gain only with a CU each.  K = 130, 160, 191: 1.2 .. 1.6 up to 256
//     chains, 0.93 .. 1.2 up to 512, 0.7 .. 1.0 beyond; K = 193, 210: 1.2 .. 1.4, then 0.92 .. 1.0.
//     Scans: K = 160, T = 6 1.0 .. 1.3 up to 512, 0.63 at 520 columns; K = 126 (four labels, two
//     chains a wave) 1.2 .. 1.4 up to 512, 0.9 beyond.  Two labels a lane gain whatever the count
//     (K = 127 1.2 .. 2.4), but for columns whose one-wave tile has 3 (K = 65: 1.1 .. 1.9 up to
//     three a CU, 900 columns 0.87).
//   * On a tile that K fills both move whole vectors, and a large frame's half-step is HBM traffic
//     either way.  One label a lane (K = 64): rows 1.2 .. 2.0 up to three a CU, 0.85 .. 1.0 up to
//     1024, columns 1.0 .. 2.0 up to five, 0.93 beyond (K = 32, two chains a wave: four, then 0.91).
//     Two (K = 96, 128): FP16 rows 1.2 .. 1.7 up to two, 0.75 .. 1.0 beyond; FP32 rows and columns
//     0.9 .. 1.7 up to three, 0.85 .. 1.0 beyond.  Three and four (K = 192, 256): rows 0.95 .. 1.2
//     (FP32, K = 192, T = 1, 560 rows 0.93); columns 1.0 .. 1.15 with a CU each, then 0.89 .. 1.05, as the chain wave has no less to do
//     than the one wave.  Tiles of two labels a lane (K <= 8) are as the filled ones (6100 columns
//     of K = 6 0.83).  Scans on them never: 0.90.
//   * Scans of the widest tile, or that reach across more than 4 lanes, are most of a node and on
//     the chain wave: only with a CU each (T = 8, K = 210: 320 x 240 1.19, 640 x 480 0.95; T = 30,
//     K = 80: 1280 x 400 0.91).
inline int pipe_per_cu(Tile d, Tile t, bool scan, int T, int K, bool theta, bool f16) {
    const int lds = pipe_lds_count(d.LPL, theta);
    const bool full = t.G * t.LPL == K, vec = pipe_vec(K, d.LPL, theta, f16);
    if (scan) {
        if (full) return 0;
        if (t.G * t.LPL == 256 || T - 1 > 4 * t.LPL) return 1;
        return vec ? lds : (d.LPL == 3 ? 2 : 1);
    }
    if (full || t.LPL <= 2) {
        if (d.LPL == 1) return theta ? 3 : (d.G == 64 ? 5 : 4);
        if (d.LPL == 2) return theta && f16 ? 2 : 3;
        if (!theta) return 1;
        return d.LPL == 3 && !f16 ? 2 : lds;
    }
    if (vec) return lds;
    if (d.LPL >= 3) return d.LPL == 3 ? 2 : 1;
    return !theta && t.LPL == 3 ? 3 : lds;
}

// Whether a batched plan pipelines the chains of one label count and family (`blocks` workgroups,
// `bytes` in their FP32 dual volumes).  More workgroups than the chip holds follow each other and
// every chain still gains by its length, but on a filled tile of many chains a wave (t) whose
// volumes stay near the last cache (256 MB) the plan is bound by issue, and a wave for one or two
// chains issues more.  Measured, one-wave queue / pipelines, iterative and naive minorant:
// 96 frames of 96 x 72 K = 32 0.88 and 0.80, K = 64 0.86, 0.71, K = 96 0.88, 0.79 (71 .. 212 MB);
// 24 of 320 x 240 K = 32 0.98, 0.89 (236 MB), 48 of them 1.09, 1.03, K = 64 1.09, 1.03 (472 MB);
// with up to 8 workgroups a CU (two labels a lane: 12) 12 of 320 x 240 K = 32 1.13, 1.13, 24 of
// 160 x 120 K = 128 1.07, 1.03.
inline bool pipe_plan_serves(Tile d, Tile t, int K, long long blocks, long long bytes, int cus) {
    if (t.G * t.LPL != K || d.G < 32 || d.LPL > 2) return true;
    return blocks <= (long long)(d.LPL == 1 ? 8 : 12) * cus || bytes > (256LL << 20);
}

}  // namespace dm
