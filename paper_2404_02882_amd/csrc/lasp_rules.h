// Launch rules as plain arithmetic, without HIP, so that they can be checked on any machine.
#ifndef LASP_RULES_H
#define LASP_RULES_H

namespace lasp {

// Workgroups up to which every one has a CU (of 256) of its own: the target of the launches that want no more, and the line
// up to which the bfloat16 forward walk takes eight waves a workgroup.
constexpr int kOnePerCu = 256;

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

}  // namespace lasp
#endif
