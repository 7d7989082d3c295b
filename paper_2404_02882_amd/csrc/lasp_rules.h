// Launch rules as plain arithmetic, without HIP, so that they can be checked on any machine.
#ifndef LASP_RULES_H
#define LASP_RULES_H

namespace lasp {

// Workgroups up to which every one has a CU (of 256) of its own: the target of the launches that want no more, and the line
// up to which the bfloat16 forward walk takes eight waves a workgroup.
constexpr int kOnePerCu = 256;

// Whether the workgroups of a walk compute their segments' start states themselves, `tiles` being what the last of them has
// in front of it (the first, backward, behind it): no local pass, no scan, one launch a pass. A tile taken through the state
// alone costs about 1.3 us (bfloat16, 64 tokens) or 3.5 us (float, 32), the local pass and its launch 6 - 9 us and a scan or
// the states carried over 5 more. Steps without / with, d=128: bfloat16 2 heads x 128 tokens 23.4 / 18.5 us, 16 x 256
// 38.0 / 24.9, 32 x 384 46.2 / 31.8, 2 x 512 42.3 / 33.8, 64 x 512 60.1 / 53.4; 16 x 768 51.7 / 51.9, 2 x 768 35.0 / 45.1;
// float 16 x 128 60.3 / 48.8, 2 x 256 51.4 / 67.9.
constexpr int kShortTiles = 8;
inline bool own_states(int tiles, bool two_byte) { return tiles < (two_byte ? kShortTiles : 4); }

// Whether the bfloat16 state cache holds the state of every tile, not of every second one, and the backward walk takes its
// tiles one by one (D: the larger dimension). Pairs halve the cache's bytes; but a sequence of an odd number of tiles has a
// pair of one, and cannot be cut below two tiles, which keeps a short sequence of few heads waiting; and at d=64, where a
// state is small, the walk by tiles leaves room for a second workgroup on its CU. Step by tiles / in pairs: d=128 2 heads x
// 448 tokens 34.3 / 42.3 us, 8 x 1088 (136 workgroups) 49.1 / 51.5, with a decay per token 16 x 448 46.8 / 53.8; d=64
// 16 x 5056 63.0 / 71.5, 100 x 8000 317 / 419, with a decay per token 362 / 562. The backward walk alone, d=128, from where
// one tile a segment no longer pays: 8 x 21 tiles 30.5 / 29.8, 16 x 16 34.9 / 32.6.
inline bool cache_every_tile(int ntiles, long long chains, int D) {
    return ntiles % 2 != 0 && (D == 64 || chains * ntiles <= kOnePerCu * 9 / 16);
}

// Tiles per segment of a bfloat16 pass that was asked for `want`: whole pairs where the cache has pairs. By tiles the
// backward pass takes what it was asked for. The forward walk, whose chain is shorter, takes single tiles up to 88 workgroups
// (d=128, 2 heads x 3 tiles 13.8 us / in pairs 15.2, 2 x 9 17.1 / 18.7, 4 x 17 19.9 / 20.5, 8 x 11 20.6 / 20.4 and with a
// decay per token 20.4 / 21.6, 16 x 9 23.0 / 22.2) or, at d=64, 208 (16 x 13 15.9 / 16.8), but not from five to eight tiles,
// where pairs make at most four segments and need no scan (16 x 7 21.1 / 18.0, 8 x 5 18.3 / 16.4); and other odd numbers at
// d=64 while three workgroups share a CU (16 heads x 79 tiles, three / four 27.0 / 29.3, 32 x 79, five / six 35.0 / 37.7).
// Both passes take single tiles, whatever the cache holds, where a short sequence goes through alone (own_states): steps with
// pairs / single tiles in the forward pass 16 x 384 33.6 / 30.7 us, 32 x 256 29.4 / 27.3, in the backward pass too 25.8 / 24.9
// (16 x 256), 41.1 / 36.9 (16 x 512); beside other sub-sequences, which are scanned together, pairs (4 x 16 x 512 46.1 / 49.6).
inline int segment_tiles(int want, int ntiles, long long chains, int D, bool every_tile, bool backward, bool alone) {
    if (alone && ntiles <= kShortTiles && chains * ntiles <= kOnePerCu) return 1;
    if (want % 2 == 0) return want;
    bool keep = every_tile;
    if (!backward) {
        const long long workgroups = chains * ((ntiles + want - 1) / want);
        keep = keep && (want == 1 ? workgroups <= (D == 64 ? 208 : 88) && (ntiles <= 4 || ntiles > 8) : D == 64 && workgroups <= 3 * kOnePerCu);
    }
    return keep ? want : want + 1;
}

// Whether a float forward call that keeps no cache (one lambda per head, outputs as they are) goes through k_short.
// Its work grows with the square of the tokens, and all of it is taken again by every head: while it leaves CUs idle it is
// faster than the walks (32 heads x 256 tokens d=64 17.7 -> 15.2 us, d=128 33.4 -> 28.6), but not for 128 heads (x 128 17.3 / 20.0; d=128
// 26.8 / 57.8), and at d=128 not for a single tile (9.4 / 11.5).
inline bool short_forward(int tokens, long long chains, int D) { return tokens > (D == 64 ? 12 : 32) && tokens <= 256 && chains <= 32; }

// Pieces that the local pass cuts a segment into. Where two segments (of a sequence, or of two sub-sequences) share a launch,
// only one of them is summed, and its workgroups are at most half as many as there are CUs: in two pieces they fill them.
// The walk then carries the boundary state over two pieces instead of one; two states are what the scratch holds anyway.
// The second state costs the walk 1.3 us, so only from 12 tiles a segment on. Steps of 128 heads, bf16 d=128, one piece / two:
// x 1024 tokens (8 tiles) 124.7 / 126.5 us, x 1536 181.1 / 177.7, x 2048 234.8 / 227.1, x 8192 880 / 831, x 16384 1737 / 1627 (a
// local pass 163 -> 100), decay per token x 8192 943 / 907, d=64 x 8192 457 / 441; 86 heads x 1536 150.8 / 146.0, x 3072 284.5 / 265.6; float
// d=128 86 x 768 (12 tiles) 310.3 / 301.7, 128 x 1536 599 / 590. (Other products are rounded then, a piece weighs its tokens from its
// own end: 128 x 2048, outputs 1.3e-3 apart, the error against 64 bits 2.828e-3 either way.)
inline int local_pieces(int segments, int tiles_per_seg, long long chains) {
    return segments == 2 && tiles_per_seg % 2 == 0 && tiles_per_seg >= 12 && chains <= kOnePerCu / 2 ? 2 : 1;
}

// Blocks of tiles per chain for `chains` independent rows of `ntiles` tiles where `slots` workgroups are resident at
// once. Two counts come into question, the share of the slots rounded down and up: the launch takes as many rounds as
// its workgroups fill the slots, each as long as the tiles of a block. The shorter is taken, and if both are as long the
// one with more workgroups, which leaves fewer slots empty. Steps of the bidirectional path (its products: 512 slots), bf16
// d=128, always down / always up / so: 16 heads x 32768 tokens 338 / 372 / 337 us, 32 x 768 49.4 / 46.5 / 45.9,
// 96 x 2560 210.8 / 196.4 / 194.4, 128 x 2560 231.4 / 219.8 / 221.0; float 96 x 512 181.3 / 167.5 / 167.5.
struct Blocks {
    int tiles, count;   // tiles per block (the last may be shorter), blocks per chain, none empty
};
inline Blocks blocks_for(int ntiles, long long chains, int slots) {
    Blocks best{};
    long long best_time = 0;
    for (long long n = slots / chains; n <= (slots + chains - 1) / chains; ++n) {
        const int want = n < 1 ? 1 : n > ntiles ? ntiles : (int)n;
        Blocks b;
        b.tiles = (ntiles + want - 1) / want;
        b.count = (ntiles + b.tiles - 1) / b.tiles;
        const long long rounds = (chains * b.count + slots - 1) / slots, time = rounds * b.tiles;
        if (best.count == 0 || time <= best_time) {
            best = b;
            best_time = time;
        }
    }
    return best;
}


// Rounds x tiles of a launch of blocks_for(): what it takes in tiles, one workgroup behind the other.
inline long long blocks_time(int ntiles, long long chains, int slots) {
    const Blocks b = blocks_for(ntiles, chains, slots);
    return (chains * b.count + slots - 1) / slots * b.tiles;
}

// Bidirectional backward: whether dQ = dO KV^T comes with the sum dKV = Q^T dO, which has dO on chip, or with the products for dK
// and dV. In the sum's launch (segments of tiles_per_seg tiles, chains x nseg workgroups, one a CU) a tile's product takes longer,
// by about a fifth of what a tile takes in the products' launch, which is `saved` (blocks_time) shorter with two products than
// with three. And the sum has to fill the CUs, else the product waits on few of them: from 13/16 of them on (float, whose products
// are longer, 3/4). At d = 64 and so many heads that a block of one head is more than half of the slots, three products fill the
// device as well as two: only bfloat16, and only long segments. Forward + backward, dQ apart / with the sum, us:
//   bf16 d=128 16 heads x 1024 tokens (one tile) 44.3 / 45.3, x 1152 (144 workgroups) 42.8 / 46.7, 32 x 636 (160) 43.4 / 46.1, 16 x 2048 (two
//   tiles) 51.2 / 49.5, 128 x 512 74.0 / 72.4, 3 x 16512 (258 workgroups) 68.0 / 72.2, 100 x 1920 (300, ten tiles) 166 / 146, 16 x 16384 (16)
//   187.6 / 180.6, 128 x 8192 657 / 602; d=64 16 x 2048 30.7 / 28.3, 128 x 768 44.1 / 46.6, 128 x 2048 87.2 / 85.9, 128 x 8192 346 / 328;
//   float d=64 32 x 384 (192 workgroups) 32.0 / 34.1, 64 x 256 39.9 / 35.6, 128 x 512 79.1 / 85.4; d=128 64 x 512 105.9 / 100.8.
inline bool dq_with_sum(bool two_byte, int D, long long chains, int tiles_per_seg, int nseg, long long saved) {
    const long long workgroups = chains * nseg, rounds = (workgroups + kOnePerCu - 1) / kOnePerCu;
    if (two_byte ? 16 * workgroups < 13 * kOnePerCu : 4 * workgroups <= 3 * kOnePerCu) return false;
    if (D == 64 && 3 * chains > kOnePerCu) return two_byte && tiles_per_seg >= 16;
    return 5 * saved >= rounds * tiles_per_seg + 3;
}

}  // namespace lasp
#endif
