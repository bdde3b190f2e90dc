// The order in which a wave of the persistent launch (mq_linear.hip) fetches and multiplies the tiles of its workgroup's share, and what that
// order says about the age of a store.  No device code of its own, so that the CPU tests run what the kernel runs.
#pragma once
#include "mq_static_for.h"

namespace mq {

// The piece of a row block that a share has stored for others to add up, until it is counted.  A wave's transfers retire in the order in which
// they were issued: the stores have been acknowledged once no more transfers are in flight than were issued after them.
struct StoredPiece {
    int rb = 0, n = 0;   // row block, groups; n == 0: nothing is stored
    int fetched = 0;     // tiles whose loads were issued since
    bool counted = false;
    __device__ __forceinline__ void stored(int row_block, int groups) {
        rb = row_block;
        n = groups;
        fetched = 0;
    }
    __device__ __forceinline__ bool to_count() const { return n != 0 && !counted; }
    // The loads of the last D tiles may stay in flight when the piece is counted.  Tiles multiplied since do not say so: the last ones of a share
    // are multiplied without another fetch.
    template <int D> __device__ __forceinline__ bool behind_loads() const { return fetched >= D; }
};

// Tiles [u_begin, u_end) of a layer of G groups a row block; wave w of NW takes every NW-th.
struct ShareWalk {
    int G, u_begin, u_end;
    int rb, ga, seg_end;  // row block at work on, its first group in the share, the end of it or of the share
    __device__ __forceinline__ ShareWalk(int G_, int begin, int end) : G(G_), u_begin(begin), u_end(end) {
        rb = begin / G;
        ga = begin - rb * G;
        seg_end = end < (rb + 1) * G ? end : (rb + 1) * G;
    }
    // fetch(slot, u, g): tile u, group g, into slot of a ring of D + 1 (compile-time indices); past the end of the share the last tile is fetched again
    // instead of branching around the loads.  multiply(slot).  finish(gb): the row block, or the share, ends at group gb.  drain(): nothing is fetched
    // from here on; rotate(): slot j takes what slot j + 1 has.
    template <int D, int NW, class Fetch, class Multiply, class Finish, class Drain, class Rotate>
    __device__ __forceinline__ void run(int w, StoredPiece &piece, Fetch &&fetch, Multiply &&multiply, Finish &&finish, Drain &&drain, Rotate &&rotate) {
        constexpr int NB = D + 1;
        int u = u_begin + w;
        int u_pf = u < u_end ? u : u_end - 1, g_pf = u_pf % G;
        auto fetch_next = [&](auto slot) {
            fetch(slot, u_pf, g_pf);
            ++piece.fetched;
            if (u_pf + NW < u_end) {
                u_pf += NW;
                g_pf += NW;
                while (g_pf >= G) g_pf -= G;
            }
        };
        auto next_row_block = [&]() {
            finish(seg_end - rb * G);
            ++rb;
            ga = 0;
            seg_end = seg_end + G < u_end ? seg_end + G : u_end;
        };
        static_for<D>([&](auto j) { fetch_next(j); });
        // Whole rounds of the ring.  The loop has one way out, at its end: with one behind every tile the compiler joins those with the way back
        // and has every round begin with a wait for all but the last loads (32 Llama-2-7B blocks, mixed widths, M = 1 526 us, 487 so, M = 5 634 / 584).
        while (u + (NB - 1) * NW < u_end)
            static_for<NB>([&](auto j) {
                while (u >= seg_end) next_row_block();
                fetch_next(IntC<(decltype(j)::value + D) % NB>{});
                multiply(j);
                u += NW;
            });
        drain();
        while (u < u_end) {  // the last tiles, D at most, are on their way
            while (u >= seg_end) next_row_block();
            multiply(IntC<0>{});
            u += NW;
            rotate();
        }
        while (seg_end < u_end) next_row_block();
        finish(seg_end - rb * G);
    }
};

}  // namespace mq
