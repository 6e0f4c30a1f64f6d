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

// Do the two logical tiles of a workgroup come from two query heads?  Wherever the heads of a kv head divide into pairs: two
// tiles of one head leave half of the workgroup without work on the item's last key tile and an odd tile count half empty.
// 32 / 8 heads, us with two tiles of a head and with a tile of two heads: 64 x S = 100 67.0, 47.0; 64 x S = 300 199, 167;
// 16 x S = 1100 248, 222; S = 2500 61.9, 60.6; S = 8191 415, 407; S = 32768 5807, 5753; D = 64 64 x S = 700 281, 247.
inline bool pair_heads(const AttnArgs& a) { return (a.Hq / a.Hkv) % 2 == 0; }

// The longest list of items any workgroup is dealt, in steps of the unsplit kernel: `step` per key tile and `item` per item
// (prologue, epilogue, band tiles).  Every ranking block is dealt the same way (it is an even number of rounds, or the only
// block), so the lists of one block are added up, a run of items of one length at a time: the workers of a run inside one
// round are consecutive, and a run costs two additions.  (Neither the first nor the last worker need have the longest list:
// 40 / 8 heads of S = 487 in items of 64 rows, a worker in the middle has a key tile more than either.)
constexpr int MAX_WORKERS = 2048;                    // 256 CUs with eight workgroups each
inline float longest_list(const AttnArgs& a, int rows, int heads_item, int64_t slots, float step, float item)
{
    const int N = (a.S + a.tile - 1) / a.tile, NG = (a.S + rows - 1) / rows;
    const Schedule s = make_schedule(a, NG, heads_item, slots);
    if ((int64_t)s.heads_x * NG <= s.workers) return item + step * (float)N;                   // one item each
    int tiles[MAX_WORKERS + 1], count[MAX_WORKERS + 1];                          // by worker: change from the worker before
    for (int w = 0; w <= s.workers; ++w) tiles[w] = count[w] = 0;
    int round = 0, at = 0;                               // of the next item
    for (int grp = NG - 1; grp >= 0; --grp) {
        const int last_tile = ((grp + 1) * rows - 1) / a.tile;                                    // of the item's rows
        const int n = a.causal ? (last_tile + 1 < N ? last_tile + 1 : N) : N;
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
        const float sum = step * (float)t + item * (float)c;
        longest = sum > longest ? sum : longest;
    }
    return longest * (float)(s.heads_x / s.head_block);
}

// Waves per 32 query rows.  A split item takes the same number of steps for half (2) or a quarter (4) of the query rows, and
// a step does not get shorter in proportion, because every step still quantizes and stages a whole key tile: so the split
// pays exactly where the chip would otherwise wait for the longest list of items.  us per step of the unsplit, 2-way and
// 4-way kernel where nothing else limits it (4 heads, S = 900 to 3700):
//   D = 128  MXFP4 tiles 2.40, 1.72, 1.27; all MXFP8 2.94, 2.14, 1.60; unquantized 2.85, 1.89, 1.32; with the Step-2 scale
//            MXFP4 3.27, 2.39, 1.91, MXFP8 3.81, 2.82, 2.23
//   D = 64   MXFP4 tiles 0.83, 0.59; all MXFP8 0.96, 0.71; unquantized 0.84, 0.61; Step-2 scale 1.23, 0.90
// and an item costs 2 to 2.5 unsplit steps (D = 128), 3.7 (D = 64, where two workgroups share a CU).  The choice and what it
// was made from (us with 1 / 2 / 4 waves): 4 / 1 heads S = 3700 80 / 57 / 44; 8 / 2 heads S = 7400 155 / 119 / 163, S = 10500
// 219 / 230 / 310; 16 / 8 heads S = 3700 82 / 66 / 97, S = 5200 115 / 127 / 176; 32 / 8 heads S = 640 21 / 18.3 / 18.7,
// S = 1800 47.5 / 43.9 / 64.8, S = 2600 65 / 79 / 110; all MXFP8, 32 / 8 heads, S = 2048 58 / 54 / 79, S = 3000 88 / 111 / 151.
inline int key_split(const AttnArgs& a, int64_t cus)
{
    if (a.S <= a.tile) return 1;
    const bool d64 = a.D == 64;
    const int64_t slots = d64 ? 2 * cus : cus;
    const int64_t items = (int64_t)a.B * a.Hq * ((a.S + 2 * a.tile - 1) / (2 * a.tile));
    if (items > 4 * slots || slots > MAX_WORKERS) return 1;      // the lists are balanced: splitting only costs
    const bool pair = pair_heads(a);
    const float whole = longest_list(a, pair ? a.tile : 2 * a.tile, pair ? 2 : 1, slots, 1.f, d64 ? 3.7f : 2.5f);
    const float two = longest_list(a, a.tile, 1, slots, 0.72f, d64 ? 3.7f : 2.1f);
    if (d64) return two < whole ? 2 : 1;
    const float four = longest_list(a, a.tile / 2, 1, slots, a.per_token ? 0.58f : 0.53f, 1.9f);
    return four < two ? (four < whole ? 4 : 1) : two < whole ? 2 : 1;
}

}  // namespace dma
