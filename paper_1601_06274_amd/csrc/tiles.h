// tiles.h - the chain tiles compiled into the library.
//
// A tile is (G lanes per chain, LPL labels per lane); a chain of K labels fits a tile
// with G*LPL >= K.  Every tile is instantiated in its own compilation unit (the build
// script reads this list), and the host dispatch tables below are generated from it.
#pragma once

#define DM_FOR_EACH_TILE(X) \
    X(4, 1)                 \
    X(4, 2)                 \
    X(8, 4)                 \
    X(16, 4)                \
    X(32, 3)                \
    X(32, 4)                \
    X(32, 6)                \
    X(64, 3)                \
    X(64, 4)

// Tiles of the pipelined sweeps (dmm_pipe.h), chosen by the library alone: with direct
// window messages, and (the chain tiles that a call may use, as results round by tile) with
// scan messages.
#define DM_FOR_EACH_PIPE_SCAN(Z) \
    Z(8, 4)                      \
    Z(16, 4)                     \
    Z(32, 3)                     \
    Z(32, 4)                     \
    Z(64, 3)                     \
    Z(64, 4)

#define DM_FOR_EACH_PIPE(Y) \
    Y(16, 1)               \
    Y(32, 1)               \
    Y(64, 1)               \
    Y(64, 2)               \
    Y(64, 3)               \
    Y(64, 4)

namespace dm {

struct Tile {
    int G, LPL;
};

// Tile of the pipelined sweeps with direct window messages: the fewest labels per lane.
inline Tile window_tile(int K) { return K <= 16 ? Tile{16, 1} : (K <= 32 ? Tile{32, 1} : Tile{64, (K + 63) / 64}); }

}  // namespace dm
