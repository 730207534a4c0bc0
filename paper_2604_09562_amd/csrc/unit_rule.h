// Which attention calls take a workgroup, or several, per unit (attn_unit.hip) instead of the plan and the streaming kernels, from what the host
// knows: the units (requests times KV heads), the width of the block table in tiles of 16 tokens, the bound of a unit's query rows, the
// cache's type and the compute units of the GPU.  Plain host code, so that it can be compiled and checked without a GPU.
#pragma once

namespace ss {

struct AttnUnitChoice {
    int splits, team;   // workgroups of a unit (0: the call is not one of them), wavefronts of a workgroup
};

constexpr int kUnitOne = 24, kUnitOne8 = 32;          // tiles that one workgroup walks as fast as several do (bf16, e4m3)
constexpr int kUnitStep = 8;                          // tiles of a step of four wavefronts
constexpr int kUnitTiles = 48, kUnitTilesFew = 80, kUnitTilesMany = 64, kShareTiles = 64, kMaxShares = 16, kUnitsPerCu = 6;

// Measured against the streaming kernels with a plan that is there already (stream and merge): the layers of a decode step reuse the plan of the
// first one, and a call must not give other bits for reusing a plan, so the rule cannot tell the two apart and goes by the dearer one.  (A
// call that makes its plan takes 4.5 to 10 us more on the streaming side and gains that much more.)  Captured graphs, layers with caches of
// their own in turn, tables as wide as the longest request, us, stream and merge / this path; 32 heads over 8 bf16 at depth 7 (two row
// blocks), then 64 heads over 8 e4m3 at depth 9 (five):
//   one workgroup a unit    8 units,  20 tiles  9.7 / 9.9    16.1 / 15.2      64 units, 20  12.3 / 10.3  21.1 / 16.1     128, 40  20.9 / 13.8
//   shares of a step        8 units,  39       10.6 / 10.3   16.3 / 13.7      16 units, 32  11.4 / 10.4  17.4 / 14.1     32, 40  12.8 / 11.8  19.7 / 16.4
//                           8 units,  63       12.3 / 10.8   16.0 / 14.0      32 units, 48  13.0 / 12.1  19.6 / 17.4
//   shares of two steps     8 units, 159       15.9 / 13.4   21.3 / 17.3      16 units, 159 17.0 / 14.2  22.1 / 19.4     64, 96  21.3 / 16.8
// With one workgroup up to 48 tiles (the rule before) 8 units of 39 tiles took 13.2 and 19.1, 16 of 32 11.6 and 15.6, 32 of 48 14.9 and 19.4.  Of 4080
// batches (1 to 1280 units, one to five row blocks, lengths uniform or uniform in the logarithm) it was more than 5 % behind the
// streaming kernels with a plan at hand in 786, by up to 40 %; this rule in 117, 16 % ahead in the mean.  Of 1100 with depths drawn per
// request (1 to 190 requests over 8 heads) 119 and 54, 15 % and 16 % ahead.  The worst, 0.78, are batches of one request much
// longer than the others, which nothing that the host knows tells from uniform ones.
//   - Up to 24 tiles (e4m3: 32, eight wavefronts from 25 on) a second workgroup costs more in the merge, 3 us, than it gains.
//   - Shares of one step of four wavefronts where there are compute units for them, up to eight of them: the merge reads every share.
//   - Else shares of sixteen tiles.  From four row blocks on a share is bound by its instructions, which the streaming kernels spread over the
//     whole chip: refused beyond 32 tiles a share (32 units, 320 tiles, five row blocks bf16 31.1 / 32.5) and, with bf16 and units on more than
//     an eighth of the compute units, beyond 64 tiles (8 requests of 160..1280, 64 heads, 19.9 / 23.4).
//   - More than a quarter of the chip's compute units: one workgroup or two, two up to 128 tiles (64 from four row blocks on).  What a uniform batch
//     gains there (16 requests of 160..1280, 32 heads bf16, 21.6 / 19.1) a batch of one long request among short ones loses (12 of 40..2000,
//     lengths uniform in the logarithm, 16.1 / 20.4).
//   - Half of them and more: one workgroup a unit.  A unit is walked by its workgroup alone, so a batch of very different lengths waits for the longest,
//     which the plan's spans share out: 80 tiles while all units are on the chip at once, 48 (from four row blocks on) with a second round that
//     is not full, else 64.  From six units to a compute unit on the workgroups that leave the plan take what the path gains (250 requests of
//     8..64 over 8 heads 39.7 / 39.3).
// Eight wavefronts or four: with four the chip holds two workgroups to a compute unit, and a unit of few tiles begins and ends sooner (32 requests of 64
// tokens 8.1 / 6.2, 64 12.7 / 7.2; 32 of 12..600, 32 heads bf16 at depths 0..8 15.9 / 12.4); eight walk a long unit faster where a step is bound
// by its instructions: four row blocks and more from 17 tiles on, e4m3 from 25 (8 units, 32 tiles, one row block 9.2 / 8.0), or from 49 where
// many units share the chip with the workgroups of the plan (32 requests of 50..400, 32 heads, 10.6 with four, 13.0 with eight).
inline AttnUnitChoice attn_unit_rule(long long units, int tiles, int rows, bool kv8, int cus)
{
    const bool deep = rows > 48, wide = kv8 || deep;   // four or five row blocks; steps bound by their instructions
    const AttnUnitChoice none = {0, 0};
    if (2 * units <= cus && tiles > (kv8 ? kUnitOne8 : kUnitOne)) {
        const int room = (int)(cus / units), top = room < kMaxShares ? room : kMaxShares;
        if (tiles <= kUnitStep * (top < 8 ? top : 8)) return {(tiles + kUnitStep - 1) / kUnitStep, 4};
        if (4 * units > cus) {
            if (tiles <= (kv8 ? kUnitTilesMany : kUnitTiles)) return {1, deep || (kv8 && tiles > kUnitTiles) ? 8 : 4};
            if (tiles > (deep ? kUnitTilesMany : 2 * kShareTiles)) return none;
            return {2, wide ? 8 : 4};
        }
        if (wide && tiles <= kUnitTiles) return {1, 8};
        const int by_tiles = (tiles + 15) / 16, splits = top < by_tiles ? top : by_tiles, share = (tiles + splits - 1) / splits;
        if (share > kShareTiles) return none;
        if (deep && (share > kShareTiles / 2 || (!kv8 && 8 * units > cus && tiles > kUnitTilesMany))) return none;
        return {splits, wide && share > kUnitStep ? 8 : 4};
    }
    if (tiles > (units <= cus ? kUnitTilesFew : deep && units < 2 * cus ? kUnitTiles : kUnitTilesMany)) return none;
    return {1, units <= cus && ((tiles > 16 && deep) || (kv8 && tiles > (4 * units <= cus ? kUnitOne : kUnitTiles))) ? 8 : 4};
}

}  // namespace ss
