// What a forward is launched as: the schedule of its work items and the number of waves that share a tile's keys.  Plain
// host code, no HIP in it.
#pragma once

#include <stdint.h>

namespace dma {

struct AttnArgs {
    const void* q;
    const void* k;
    const void* v;
    float* out;
    int B, Hq, Hkv, S, D;
    int tile;
    int band;
    int sink;        // leading key tiles in the high format
    int causal;
    int per_token;   // Alg. 2 Step 2 on queries and keys
    const float* q_amax;   // with per_token: group maxima per query row [B, Hq, S] instead of the row's own (or null)
    const float* k_amax;   // ... per key row [B, Hkv, S]
    int pv_mx;       // P V in MXFP8-E4M3 with blocks of 32 keys instead of 16-bit
    int hi_fmt, lo_fmt;
};

// The static schedule as the kernels see it: `blocks` workgroups; items ranked in blocks of head_block heads (see the kernel)
// of heads_x query heads, dealt to `workers` workgroups (those of one XCD when each keeps its own units).
struct Schedule {
    int64_t blocks;
    int workers, heads_x, head_block;
};
// NG items per query head or per heads_item query heads that share a kv head; slots: the workgroups the chip holds at once.
inline Schedule make_schedule(const AttnArgs& a, int NG, int heads_item, int64_t slots)
{
    Schedule s;
    const int64_t items = (int64_t)a.B * (a.Hq / heads_item) * NG;
    s.blocks = items < slots ? items : slots;
    // ranking blocks: the fewest heads that fill an even number of rounds, in whole
    // groups of query heads that share a kv head: the workers of a round then walk the SAME K/V stream with items of nearly
    // equal length (on the 32k GQA workload 17 % fewer bytes fetched than with single heads, 0.6 % less time)
    const int units = a.B * a.Hkv, group = a.Hq / a.Hkv / heads_item;
    const bool by_xcd = (units % 8 == 0) && (s.blocks % 8 == 0);
    s.workers = (int)(by_xcd ? s.blocks / 8 : s.blocks);
    s.heads_x = (by_xcd ? units / 8 : units) * group;
    s.head_block = s.heads_x;
    for (int hb = group; hb < s.heads_x; hb += group)
        if (s.heads_x % hb == 0 && ((int64_t)hb * NG) % (2 * s.workers) == 0) { s.head_block = hb; break; }
    return s;
}

// The query rows of an unsplit item: one logical tile, two in a row of a head, or the same tile of two heads that share a kv head.
enum class Item { ONE_TILE, TWO_TILES, TWO_HEADS };
// Two heads wherever the heads of a kv head divide into pairs: two tiles of one head leave half of the workgroup without work on
// the item's last key tile and an odd tile count half empty.  32 / 8 heads, us with two tiles of a head and with a tile of two
// heads: 64 x S = 100 67.0, 47.0; 64 x S = 300 199, 167; 16 x S = 1100 248, 222; S = 2500 61.9, 60.6; S = 8191 415, 407; S = 32768 5807,
// 5753; D = 64 64 x S = 700 281, 247.
// A single tile goes alone while every one has a compute unit to itself: a second head would only take half of the unit's
// issue slots (time alone over time in pairs, 2000 problems of up to cus query heads: D = 128 0.78 to 0.94, D = 64 0.89 to 0.99;
// with more heads than compute units 1.0 to 1.9 at D = 128).
// For the same reason two tiles of one head, where their count is odd, the mask makes the last one the longest item and every
// item has a unit: the last tile is then alone in its workgroup (D = 128, time with two tiles over two heads: 0.90 on
// average and 1.02 at most there, 1.2 with more items than units; even counts 1.02; without the mask 1.03; D = 64 0.99).
inline bool last_tile_alone(const AttnArgs& a, int64_t cus)
{
    const int N = (a.S + a.tile - 1) / a.tile;
    return a.D == 128 && a.causal && N % 2 == 1 && (int64_t)a.B * a.Hq * ((N + 1) / 2) <= cus;
}
inline Item unsplit_item(const AttnArgs& a, int64_t cus)
{
    const bool pairs = (a.Hq / a.Hkv) % 2 == 0;
    if (a.S <= a.tile) return pairs && (int64_t)a.B * a.Hq > cus ? Item::TWO_HEADS : Item::ONE_TILE;
    return pairs && !last_tile_alone(a, cus) ? Item::TWO_HEADS : Item::TWO_TILES;
}

// What a launch has its workgroups walk, in steps of the unsplit kernel (`step` per key tile and `item` per item: prologue,
// epilogue, band tiles): the longest list of items any of them is dealt, and the work of a compute unit.
struct Load {
    float longest, cu;
};
// Every ranking block is dealt the same way (it is an even number of rounds, or the only block), so the lists of one block are
// added up, a run of items of one length at a time: the workers of a run inside one round are consecutive, and a run costs
// two additions.  (Neither the first nor the last worker need have the longest list: 40 / 8 heads of S = 487 in items of 64
// rows, a worker in the middle has a key tile more than either.)
// resident: the workgroups a CU holds at once, as the launch has them.
constexpr int MAX_WORKERS = 2048;                    // 256 CUs with eight workgroups each
inline Load dealt_load(const AttnArgs& a, int rows, int heads_item, int64_t cus, int resident, float step, float item)
{
    const int N = (a.S + a.tile - 1) / a.tile, NG = (a.S + rows - 1) / rows;
    const Schedule s = make_schedule(a, NG, heads_item, cus * resident);
    auto tiles_of = [&](int grp) {
        const int last_tile = ((grp + 1) * rows - 1) / a.tile;                                    // of the item's rows
        return a.causal ? (last_tile + 1 < N ? last_tile + 1 : N) : N;
    };
    Load load;
    int64_t sum = 0;                                     // key tiles of all items of a head
    for (int grp = 0; grp < NG; ++grp) sum += tiles_of(grp);
    const float total = (float)((int64_t)a.B * (a.Hq / heads_item)) * (step * (float)sum + item * (float)NG);
    // The workgroups of a CU: with the causal mask lists of all lengths meet, so a CU has its share of the whole; without it
    // all lists are alike, and some CUs have a workgroup more than others.
    load.cu = a.causal ? total / (float)cus : total / (float)s.blocks * (float)((s.blocks + cus - 1) / cus);
    if ((int64_t)s.heads_x * NG <= s.workers) {                                                  // one item each
        load.longest = item + step * (float)N;
        return load;
    }
    int tiles[MAX_WORKERS + 1], count[MAX_WORKERS + 1];                          // by worker: change from the worker before
    for (int w = 0; w <= s.workers; ++w) tiles[w] = count[w] = 0;
    int round = 0, at = 0;                               // of the next item
    for (int grp = NG - 1; grp >= 0; --grp) {
        const int n = tiles_of(grp);
        for (int left = s.head_block; left > 0;) {
            const int len = left < s.workers - at ? left : s.workers - at;
            const int first = (round & 1) ? s.workers - at - len : at;
            tiles[first] += n, tiles[first + len] -= n;
            count[first] += 1, count[first + len] -= 1;
            left -= len, at += len;
            if (at == s.workers) at = 0, ++round;
        }
    }
    float longest = 0.f;
    for (int w = 0, t = 0, c = 0; w < s.workers; ++w) {
        t += tiles[w], c += count[w];
        const float of_w = step * (float)t + item * (float)c;
        longest = of_w > longest ? of_w : longest;
    }
    load.longest = longest * (float)(s.heads_x / s.head_block);
    return load;
}

// Waves per 32 query rows.  A split item takes the same number of steps for half (2) or a quarter (4) of the query rows, and
// a step does not get shorter in proportion, because every step still quantizes and stages a whole key tile: so the split
// pays exactly where the chip would otherwise wait for the longest list of items.  us per step of the unsplit, 2-way and
// 4-way kernel where nothing else limits it (4 heads, S = 900 to 3700):
//   D = 128  MXFP4 tiles 2.41, 1.76, 1.23; all MXFP8 2.96, 2.22, 1.59; unquantized 2.90, 2.01, 1.35; with the Step-2 scale
//            MXFP4 3.08, 2.22, 1.77, MXFP8 3.59, 2.67, 2.09
//   D = 64   MXFP4 tiles 0.83, 0.63; all MXFP8 0.94, 0.72; unquantized 0.85, 0.66; Step-2 scale 1.19, 0.87, MXFP8 1.35, 1.02
// A CU holds one workgroup at D = 128 and three or four at D = 64 (the occupancy that the launch uses): there a step
// takes longer the more of them share the CU, by CROWD of the work of the others.  us with 1 / 2 / 4 waves, D = 128: 4 / 1 heads
// S = 3700 78 / 57 / 41; 8 / 2 heads S = 7400 150 / 115 / 153, S = 10500 218 / 229 / 285; 16 / 8 heads S = 3700 79 / 64 / 87, S = 5200
// 114 / 125 / 157; 32 / 8 heads S = 640 20.3 / 17.8 / 15.5, S = 1800 45.2 / 41.5 / 55.7, S = 2600 62 / 77 / 94; all MXFP8, 32 / 8 heads,
// S = 2048 58 / 52 / 69, S = 3000 87 / 108 / 134.
// The costs below were fitted on problems timed with every split (2764 at D = 128, 6865 at D = 64; default, all MXFP8, all MXFP4 and
// unquantized, with and without the per-token scale and the mask; 2 to 500 heads over the batch, S up to 8200) on kernels whose
// waves each made their own query operands, as the ones whose choice loses least: less than by the ratios of the table, and
// unquantized problems at D = 128 lose more by ratios of their own.  On the present kernels (2 to 320 heads over the batch, S from a
// little over a tile to 9000, every pair of formats, of more than 9 us) the choice is from the best split of each, on average and
// at worst: D = 128 2486 problems 0.20 %, 13.7 % (one quantized format 0.29 %, 13.7 %; two 0.18 %, 10.8 %; unquantized 0.25 %, 10.5 %;
// Step-2 scale 0.06 %, 5.7 %); D = 64 985 problems 0.07 %, 8.4 %.  With 2.05 steps for every item of four waves, as it was fitted, the
// 873 of one quantized format at D = 128 lose 0.66 %, 21 %.
constexpr float CROWD = 0.3f;
inline int key_split(const AttnArgs& a, int64_t cus, int resident1, int resident2, int resident4)
{
    if (a.S <= a.tile) return 1;
    const bool d64 = a.D == 64;
    const int64_t items = (int64_t)a.B * a.Hq * ((a.S + 2 * a.tile - 1) / (2 * a.tile));
    if (items > 2 * cus) return 1;         // the lists are balanced: splitting only costs (it gained 1 % or more on 20 of 1585 such problems)
    const int most = resident1 > resident2 ? (resident1 > resident4 ? resident1 : resident4) : (resident2 > resident4 ? resident2 : resident4);
    if (cus * most > MAX_WORKERS) return 1;
    auto cost = [&](int rows, int heads_item, int resident, float step, float item) {
        const Load l = dealt_load(a, rows, heads_item, cus, resident, step, item);
        return l.longest + CROWD * (l.cu > l.longest ? l.cu - l.longest : 0.f);
    };
    const bool two_heads = unsplit_item(a, cus) == Item::TWO_HEADS;
    float whole = cost(two_heads ? a.tile : 2 * a.tile, two_heads ? 2 : 1, resident1, 1.f, d64 ? 2.f : 2.5f);
    if (last_tile_alone(a, cus)) whole *= 0.92f;
    if (d64) {
        // least for unquantized (FMT_BF16) keys and with the Step-2 scale, but not without the mask, where every list is long and
        // two workgroups or more share a CU throughout; 0.5: beside the lists of a split launch
        const float step = a.causal && (a.lo_fmt == 0 || a.per_token) ? 0.73f : 0.80f;
        return 0.5f + cost(a.tile, 1, resident2, step, 2.f * step) < whole ? 2 : 1;
    }
    const float two = cost(a.tile, 1, resident2, 0.70f, 2.2f);
    // One quantized format without the Step-2 scale: the four waves of an item share the making of its query operands.  On 70
    // problems between the two costs four waves take 0.91 of the time of two, 0.95 on the native FP8 MFMA (0.75 to 0.99; 1.01 to 1.08
    // on three of 5 heads with S = 7300).  Sharing them in two formats, four waves take 0.84 to 1.07 there, 0.99 on average (32 / 8
    // heads S = 822 20.5 us, two waves 20.1).  Where they are not shared: 40 / 8 heads S = 400 unquantized 15.3, 14.6, per token 18.8, 18.0.
    const bool shared = a.lo_fmt == a.hi_fmt && a.lo_fmt != 0 && !a.per_token;
    const float four = cost(a.tile / 2, 1, resident4, 0.51f, shared ? 1.9f : 2.05f);
    return four < two ? (four < whole ? 4 : 1) : two < whole ? 2 : 1;
}

}  // namespace dma
