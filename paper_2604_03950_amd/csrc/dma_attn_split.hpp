// The forward of dma_attn_kernel.hpp for problems with few work items: the keys of a tile are split over waves.
//
// Work split.  A work item is 32 * NW / KS query rows of one logical tile (a whole tile or half of one); KS waves share 32
// query rows, and each computes the scores, probabilities and P V of 1 / KS of the keys of EVERY key tile, with its own
// partial O and l.  The row maximum of a tile is exchanged through LDS before the exponentials, so every wave uses the
// running maximum of the whole tile, as Alg. 1 does: the probabilities (and their rounding to bf16) are the ones the
// unsplit kernel forms; only the binary32 sums over the keys are taken in another order.  The partial sums meet in LDS at
// the end of the item.  Nothing but the output goes to memory.
//
// Pipeline.  One barrier per tile, in the middle of the step: before it K of tile jt + 1 is staged, the scores of tile jt
// are formed and each wave publishes its row maxima; behind it V of tile jt + 1 is staged, the maxima are read, and the
// exponentials and P V of tile jt follow.  K of buffer b is read before the barrier of a step only and V of buffer b
// behind it only, so the buffers of the step before are free at either place.
#pragma once

#include "dma_attn_kernel.hpp"

namespace dma {

// Sink window, non-causal variant and ragged lengths are all handled by this one instance (loads bounded by buffer
// resources, precision and mask decided per tile).
template <int D, int BT, int KS, int LO, int HI, bool PT>
__global__ void __launch_bounds__((BT / 32) * 2 * 64, 2)
dma_attn_split_kernel(const uint16_t* __restrict__ q, const uint16_t* __restrict__ k,
                      const uint16_t* __restrict__ v, float* __restrict__ out,
                      int B, int Hq, int Hkv, int S, int band, int sink, int causal, float c, int head_block,
                      const float* __restrict__ q_amax, const float* __restrict__ k_amax)
{
    using C = Cfg<D, BT, 1, KS>;
    constexpr bool TWO = (LO != HI);
    constexpr int RG = C::NW / KS;                       // groups of 32 query rows
    constexpr int ROWS = 32 * RG;                        // query rows of an item
    static_assert(BT % ROWS == 0, "an item lies inside one logical tile");
    constexpr int KLO = C::template kbytes<LO>();
    constexpr int KHI = TWO ? C::template kbytes<HI>() : 0;
    constexpr int KG = C::template kg<LO>(), KR = C::template kr<LO>();
    constexpr int QRLO = C::template qregs<LO>();
    constexpr int QRHI = TWO ? C::template qregs<HI>() : 1;
    // LDS map (bytes): the row maxima of the waves' shares (double-buffered), then V and K as in the unsplit kernel, all
    // double-buffered.  The partial sums of the epilogue reuse V and K.
    constexpr int MAXIMA = C::NW * 32 * 4;
    constexpr int OFF_V = 2 * MAXIMA;
    constexpr int OFF_KLO = OFF_V + 2 * C::VBYTES;
    constexpr int OFF_KSLO = OFF_KLO + 2 * KLO;
    constexpr int OFF_KHI = OFF_KSLO + 2 * C::KSC;
    constexpr bool HI_SCALES = TWO && !uses_bf16_mfma(HI);
    constexpr int OFF_KSHI = OFF_KHI + 2 * KHI;
    constexpr int OFF_KTS = OFF_KSHI + (HI_SCALES ? 2 * C::KSC : 0);
    constexpr int EPI_STRIDE = D * 4 + 16;               // bytes per row of a wave's partial O (padded against bank conflicts)
    constexpr int EPI_WAVE = 32 * EPI_STRIDE;
    constexpr int OFF_EPI = OFF_V;
    constexpr int LDS_TOTAL = cmax<OFF_KTS + (PT ? 2 * BT * 4 : 0), OFF_EPI + C::NW * EPI_WAVE>();
    static_assert(LDS_TOTAL <= 160 * 1024, "LDS budget of one CU");
    __shared__ __attribute__((aligned(1024))) uint8_t lds[LDS_TOTAL];
    const unsigned lds0 = (unsigned)(uintptr_t)(DMA_LDS uint8_t*)lds;
    auto v_at = [&](int buf) { return (unsigned)(buf * C::VBYTES); };              // as in the unsplit kernel
    auto klo_at = [&](int buf) { return (unsigned)(buf * KLO); };
    auto kslo_at = [&](int buf) { return (unsigned)(buf * C::KSC); };
    auto khi_at = [&](int buf) { return lds0 + OFF_KHI + buf * KHI; };
    auto kshi_at = [&](int buf) { return (unsigned)(OFF_KSHI - OFF_KSLO + (HI_SCALES ? buf * C::KSC : 0)); };
    auto kts_at = [&](int buf) { return lds0 + OFF_KTS + (PT ? buf * BT * 4 : 0); };

    const bool amax_given = PT && q_amax != nullptr;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;
    const int rg = wave % RG, kh = wave / RG;            // the wave's query rows and its share of the keys
    const int key0 = kh * C::NB * 32;
    LaneOffsets<C, LO> lofs;
    lofs.init(tid, lane, lds0 + OFF_KLO, lds0 + OFF_KSLO, lds0 + OFF_V);
    const unsigned mx_slot = pin((kh * RG + rg) * 128 + 4 * (lane & 31));      // the wave's maxima; the others' are a xor away

    // ---- static schedule: as in the unsplit kernel, with items of ROWS query rows
    const int N = (S + BT - 1) / BT;
    const int NG = (S + ROWS - 1) / ROWS;
    const int group = (unsigned)Hq / (unsigned)Hkv;
    const int units = B * Hkv;
    const bool by_xcd = (units % 8 == 0) && (gridDim.x % 8 == 0);
    const int xcd = by_xcd ? (int)(blockIdx.x & 7) : 0;
    const int slot = by_xcd ? (int)(blockIdx.x >> 3) : (int)blockIdx.x;
    const int workers = by_xcd ? (int)(gridDim.x >> 3) : (int)gridDim.x;
    const int heads_x = by_xcd ? (units / 8) * group : B * Hq;
    const int items = heads_x * NG;

    for (int round = 0;; ++round) {
        const int pos = round * workers + ((round & 1) ? workers - 1 - slot : slot);
        if (pos >= items) break;
        const unsigned blk = (unsigned)pos / (unsigned)(head_block * NG), within = (unsigned)pos % (unsigned)(head_block * NG);
        const int grp = NG - 1 - (int)(within / (unsigned)head_block);
        const unsigned hx = blk * head_block + within % (unsigned)head_block;
        const unsigned uh = hx / (unsigned)group, unit = by_xcd ? uh * 8 + xcd : uh;                  // unit: b * Hkv + kv head
        const unsigned hq = unit * group + hx % (unsigned)group;                                      // b * Hq + head
        const uint16_t* qhead = q + (int64_t)hq * S * D;
        const uint16_t* khead = k + (int64_t)unit * S * D;
        const uint16_t* vhead = v + (int64_t)unit * S * D;
        float* ohead = out + (int64_t)hq * S * D;
        const float* qam_head = amax_given ? q_amax + (int64_t)hq * S : nullptr;
        const float* kam_head = amax_given ? k_amax + (int64_t)unit * S : nullptr;

        const int row0 = grp * ROWS, it = row0 / BT;
        const int qrow = row0 + rg * 32, qrow_in_tile = qrow - it * BT;
        const int nt = causal ? it + 1 : N;
        auto tile_hi = [&](int jt) __attribute__((always_inline)) {
            if (!TWO) return false;
            if (jt < sink) return true;
            const int dist = (causal || it >= jt) ? it - jt : jt - it;
            return dist < band;
        };
        // main tiles (low format, unmasked) and band tiles [0, s1), [w0, w1) and a partial last tile without the causal mask
        int w0, w1, s1 = TWO ? min(sink, nt) : 0;
        if (causal) {
            w0 = (TWO && band > 0) ? max(0, it + 1 - band) : it;
            w1 = nt;
        } else if (TWO && band > 0) {
            w0 = max(0, it + 1 - band);
            w1 = min(N, it + band);
        } else {
            w0 = w1 = nt;
        }
        const bool ragged_tail = !causal && S % BT != 0;
        if (ragged_tail) w0 = min(w0, nt - 1);
        if (s1 > w0) { w1 = max(w1, s1); w0 = 0; s1 = 0; }

        float m = 0.f, mfloor = -INFINITY, l = 0.f;
        v16f o[C::NDB];
#pragma unroll
        for (int db = 0; db < C::NDB; ++db) o[db] = v16f{0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};

        v4i kreg[C::CPT], vreg[C::CPT];
        float kam[KR];
#pragma unroll
        for (int i = 0; i < KR; ++i) kam[i] = 0.f;
        auto load_k = [&](int jt) __attribute__((always_inline)) {
            load_tile<C, KG>(kreg, khead, jt * BT, S, tid);
            if constexpr (PT) {
                if (amax_given) load_key_amax<C, KG>(kam, kam_head, jt * BT, S, tid);
            }
        };
        auto load_v = [&](int jt) __attribute__((always_inline)) { load_tile<C>(vreg, vhead, jt * BT, S, tid); };
        auto stage_key = [&](int jt, bool lo_known) __attribute__((always_inline)) {                 // K tile jt from the registers into LDS
            const int buf = jt & 1;
            float inv_sk[KR], bam[KR];
#pragma unroll
            for (int i = 0; i < KR; ++i) inv_sk[i] = 1.f, bam[i] = 0.f;
            if constexpr (PT) key_token_scales<C, KG>(kreg, inv_sk, bam, kts_at(buf), tid, kam, amax_given);
            const bool h = !lo_known && tile_hi(jt);
            if (!h) stage_k<C, KG, LO, PT>(kreg, klo_at(buf), kslo_at(buf), lofs.stage_k, lofs.stage_s, inv_sk, bam);
            if constexpr (TWO) {
                if (h) stage_k<C, KG, HI, PT>(kreg, khi_at(buf), kshi_at(buf), stage_k_lane<C, KG, HI>(fresh(tid)), lofs.stage_s, inv_sk, bam);
            }
        };

        // ---- prologue: key tile 0 and the query operands, tile 0 into LDS buffer 0, tile 1 requested
        PTile<C, false> pb;
        v4i qr_lo[QRLO], qr_hi[QRHI];
        int qs_lo = 0, qs_hi = 0;
        float q_sq = 1.f;
        // Four waves that share query rows make a quarter of their operands each (one of the two blocks of a lane's row, in one of the
        // formats) and trade them through the V buffer that tile 1 is staged into behind the first barrier of the tile loop.
        // (All four read the same rows and quantized them to both formats before, 1.2 us of an item's 8 beyond its steps.)
        // 32 / 8 heads S = 300 11.9 -> 11.0 us, S = 613 17.2 -> 14.9, S = 700 19.0 -> 16.7; 4 / 1 heads S = 3700 all MXFP8 49.2 -> 47.4.
        // With the Step-2 scale a row's own maximum needs the whole row; unquantized rows are only copied.
        constexpr bool SHARE_Q = KS == 4 && !PT && LO != FMT_BF16;
        constexpr int NL = QRLO / C::NH, NHI = TWO ? QRHI / C::NH : 1;
        constexpr int SHARE_HI = RG * QRLO * 1024, SHARE_SLO = SHARE_HI + (TWO ? RG * QRHI * 1024 : 0), SHARE_SHI = SHARE_SLO + RG * 256;
        static_assert(!SHARE_Q || (C::NH == 2 && SHARE_SHI + RG * 256 <= C::VBYTES), "query operands of a workgroup in one V buffer");
        const unsigned share = lds0 + OFF_V + C::VBYTES;
        if constexpr (SHARE_Q) {
            const int h = kh & 1, ln = fresh(lane);
            v4i raw[4];
            const rsrc_t qmat = make_rsrc(qhead, (uint32_t)S * (D * 2));
            const unsigned off = (unsigned)(qrow + (ln & 31)) * (D * 2) + 64 * (ln >> 5) + 128 * h;
#pragma unroll
            for (int t = 0; t < 4; ++t) raw[t] = buffer_load16(qmat, off + 16 * t);
            load_k(0);
            load_v(0);
            __builtin_amdgcn_sched_barrier(0);
            const unsigned at = pin(share + ln * 16), sc = pin(share + SHARE_SLO + (rg * 64 + ln) * 4 + h);
            if (kh < 2) {
                v4i r[NL];
                const int code = make_q_block<LO, false>(r, raw, c, 1.f);
#pragma unroll
                for (int i = 0; i < NL; ++i) lds_write<v4i>(at + (rg * QRLO + h * NL + i) * 1024, r[i]);
                if constexpr (!uses_bf16_mfma(LO)) lds_write<uint8_t>(sc, (uint8_t)code);
            } else if constexpr (TWO) {
                v4i r[NHI];
                const int code = make_q_block<HI, false>(r, raw, c, 1.f);
#pragma unroll
                for (int i = 0; i < NHI; ++i) lds_write<v4i>(at + SHARE_HI + (rg * QRHI + h * NHI + i) * 1024, r[i]);
                if constexpr (!uses_bf16_mfma(HI)) lds_write<uint8_t>(sc + (SHARE_SHI - SHARE_SLO), (uint8_t)code);
            }
        } else {
            v4i qraw[C::NKK];
            load_q_raw<C>(qraw, make_rsrc(qhead, (uint32_t)S * (D * 2)), qrow, fresh(lane) & 31, fresh(lane) >> 5);
            load_k(0);
            load_v(0);
            __builtin_amdgcn_sched_barrier(0);
            float inv_sq = 1.f;
            if constexpr (PT) {
                float amax;
                if (amax_given) {
                    const int row = qrow + (fresh(lane) & 31);
                    amax = row < S ? qam_head[row] : 0.f;
                } else {
                    amax = q_row_amax<C>(qraw, c);
                }
                token_scale(amax, q_sq, inv_sq);
            }
            make_q<C, LO, PT>(qr_lo, qs_lo, qraw, c, inv_sq);
            if constexpr (TWO) {
                if (band > 0 || sink > 0) make_q<C, HI, PT>(qr_hi, qs_hi, qraw, c, inv_sq);
            }
        }
        stage_key(0, false);
        stage_v<C>(vreg, v_at(0), lofs.stage_v);
        load_k(1 < nt ? 1 : N);
        load_v(1 < nt ? 1 : N);
        __syncthreads();
        if constexpr (SHARE_Q) {
            const int ln = fresh(lane);
            const unsigned at = pin(share + ln * 16), sc = pin(share + SHARE_SLO + (rg * 64 + ln) * 4);
#pragma unroll
            for (int i = 0; i < QRLO; ++i) qr_lo[i] = lds_read<v4i>(at + (rg * QRLO + i) * 1024);
            if constexpr (!uses_bf16_mfma(LO)) qs_lo = lds_read<int>(sc);
            if constexpr (TWO) {
#pragma unroll
                for (int i = 0; i < QRHI; ++i) qr_hi[i] = lds_read<v4i>(at + SHARE_HI + (rg * QRHI + i) * 1024);
                if constexpr (!uses_bf16_mfma(HI)) qs_hi = lds_read<int>(sc + (SHARE_SHI - SHARE_SLO));
            }
        }

        // ---- tile loop.  MAIN: a main tile followed by another one, so that nothing of the step depends on jt.
        auto step = [&](int jt, auto MAIN) __attribute__((always_inline)) {
            constexpr bool main = decltype(MAIN)::value != 0;
            const int buf = jt & 1, ln = fresh(lane), g = ln >> 5;
            const unsigned kts = kts_at(buf) + 4 * key0;
            v16f s[C::NB];
            if (main || !tile_hi(jt)) {
                score_products<C, LO, PT>(s, qr_lo, qs_lo, klo_at(buf) + key0 * C::template kstride<LO>(), kslo_at(buf) + key0 * C::SPK, lofs.score_k, lofs.score_s, kts, q_sq, g, c, m);
            } else if constexpr (TWO) {
                score_products<C, HI, PT>(s, qr_hi, qs_hi, khi_at(buf) + key0 * C::template kstride<HI>(), kshi_at(buf) + key0 * C::SPK, score_k_lane<C, HI>(fresh(lane)), lofs.score_s, kts, q_sq, g, c, m);
            }
            // Where a wave has one 32-key block of the tile, its products are a chain of LDS reads and dependent MFMAs with nothing
            // else to issue: the next tile's staging fills it.  4 / 1 heads S = 8192 92.1 -> 89.8 us, 8 / 2 S = 4000 53.7 -> 52.4, D = 64
            // 16 / 8 S = 1500 19.4 -> 19.1, unquantized 4 / 1 S = 3700 43.2 -> 41.6.  Not with two blocks (32 / 8 S = 1000 22.3 -> 22.4),
            // nor with the Step-2 scale, whose staging is long (4 / 1 S = 3700 55.2 -> 57.7: it delays the row maxima).
            constexpr bool STAGE_EARLY = main && C::NB == 1 && !PT;
            if (STAGE_EARLY) stage_key(jt + 1, true);
            if (!main) mask_scores<C>(s, causal && jt == it, causal ? BT : min(BT, S - jt * BT), qrow_in_tile, key0, ln & 31, g);
            float mx = score_max<C>(s);
            const unsigned maxima = lds0 + buf * MAXIMA;
            lds_write<float>(maxima + mx_slot, mx);
            if (!STAGE_EARLY && (main || jt + 1 < nt)) stage_key(jt + 1, main);
            const int ahead = main || jt + 2 < nt ? jt + 2 : N;
            load_k(ahead);
            __syncthreads();
            float other[KS - 1];
#pragma unroll
            for (int i = 1; i < KS; ++i) other[i - 1] = lds_read<float>(maxima + (mx_slot ^ (i * RG * 128)));
            if (main || jt + 1 < nt) stage_v<C>(vreg, v_at(buf ^ 1), lofs.stage_v);
            if (D == 64) load_v(ahead);               // 16 / 8 heads S = 1500 19.1 us, behind the rescale 19.25
#pragma unroll
            for (int i = 1; i < KS; ++i) mx = fmaxf(mx, other[i - 1]);
            float alpha;
            move_max<C>(s, o, mx, m, mfloor, alpha);
            if (D != 64) {
                hold(vreg);
                load_v(ahead);
            }
            l = l * alpha + probabilities<C>(s, pb);
            value_part<C>(v_at(buf) + key0 * C::VS, lofs.value_v, o, pb);
        };
        const int mend = ragged_tail ? max(w1, nt - 1) : nt;
        for (int jt = 0; jt < nt; ++jt) {
            const int stop = jt < s1 ? jt : jt < w0 ? w0 - 1 : jt < w1 ? jt : mend - 1;      // main tiles up to here
            for (; jt < stop; ++jt) step(jt, IC<1>{});
            step(jt, IC<0>{});
        }

        // ---- epilogue: every wave parks its partial O row-major in LDS and its partial l beside the maxima; then the KS
        // waves of 32 query rows take 32 / KS of the rows each, add the partial sums in the order of the keys and store
        // whole rows.
        __syncthreads();
        {
            const int ln = fresh(lane);
            const int j = ln & 31, g = ln >> 5;
            lds_write<float>(lds0 + mx_slot, cross_half_sum(l));
            const unsigned wr = pin(lds0 + OFF_EPI + wave * EPI_WAVE + j * EPI_STRIDE + 16 * g);
#pragma unroll
            for (int db = 0; db < C::NDB; ++db)
#pragma unroll
                for (int r4 = 0; r4 < 4; ++r4)
                    lds_write<v4f>(wr + 128 * db + 32 * r4, v4f{o[db][4 * r4], o[db][4 * r4 + 1], o[db][4 * r4 + 2], o[db][4 * r4 + 3]});
        }
        __syncthreads();
        {
            constexpr int LPR = D / 4;                   // lanes per row, 16 bytes each
            constexpr int RPI = 64 / LPR;                // rows per store
            const int ln = fresh(lane);
            const int rsub = ln / LPR, piece = ln % LPR;
            const int first = kh * (32 / KS) + rsub;     // the lane's first row of the group
            const rsrc_t omat = make_rsrc(ohead, (uint32_t)S * (D * 4));
            const unsigned obase = (unsigned)(qrow + first) * (D * 4) + 16 * piece;
            const unsigned rd = pin(lds0 + OFF_EPI + rg * EPI_WAVE + first * EPI_STRIDE + 16 * piece);
            const unsigned rl = pin(lds0 + rg * 128 + 4 * first);
#pragma unroll
            for (int i = 0; i < 32 / KS / RPI; ++i) {
                v4f sum = lds_read<v4f>(rd + i * RPI * EPI_STRIDE);
                float lsum = lds_read<float>(rl + 4 * i * RPI);
#pragma unroll
                for (int p = 1; p < KS; ++p) {
                    sum += lds_read<v4f>(rd + i * RPI * EPI_STRIDE + p * RG * EPI_WAVE);
                    lsum += lds_read<float>(rl + 4 * i * RPI + p * RG * 128);
                }
                const float inv = 1.0f / lsum;
                buffer_store16(omat, obase + i * RPI * (D * 4), sum * inv);
            }
        }
        __syncthreads();                  // the next item's staging overwrites the partial sums
    }
}

// ---------------------------------------------------------------------------------------------
// Host side: launch (the number of waves that share a tile's keys comes from dma_plan.hpp)
// ---------------------------------------------------------------------------------------------
// f(PT) for the instance that serves the call.
template <int LO, int HI, typename F>
static int with_split(const AttnArgs& a, F&& f)
{
    if constexpr (takes_token_scale(LO, HI)) {
        if (a.per_token) return f(IC<1>{});
    }
    return f(IC<0>{});
}
template <int D, int BT, int KS, int LO, int HI>
static int launch_split(const AttnArgs& a, hipStream_t stream)
{
    using C = Cfg<D, BT, 1, KS>;
    constexpr int ROWS = 32 * C::NW / KS;
    return with_split<LO, HI>(a, [&](auto PT) {
        return launch_resident<dma_attn_split_kernel<D, BT, KS, LO, HI, PT != 0>>(C::T, (a.S + ROWS - 1) / ROWS, 1, a, stream);
    });
}
template <int D, int BT, int KS, int LO, int HI>
static int resident_split(const AttnArgs& a)
{
    return with_split<LO, HI>(a, [&](auto PT) { return resident_workgroups<dma_attn_split_kernel<D, BT, KS, LO, HI, PT != 0>>(Cfg<D, BT, 1, KS>::T); });
}

// Split, or unsplit items of one or two logical tiles per workgroup (of two, 256 query rows share each K/V tile; where two
// in a row of a head make up an item and their number is odd, the last pair is filled up with a tile past the end).
template <int D, int BT, int LO, int HI>
static int launch_tile(const AttnArgs& a, hipStream_t stream)
{
    constexpr bool FOUR = D == 128;
    const int cus = compute_units();
    if (cus <= 0) return DMA_ERR_HIP_;
    if (!a.pv_mx && a.S > BT) {
        const int r1 = resident_instance<D, BT, LO, HI>(a), r2 = resident_split<D, BT, 2, LO, HI>(a);
        int r4 = r2;
        if constexpr (FOUR) r4 = resident_split<D, BT, 4, LO, HI>(a);
        if (r1 <= 0 || r2 <= 0 || r4 <= 0) return DMA_ERR_HIP_;
        const int ks = key_split(a, cus, r1, r2, r4);
        if (ks == 2) return launch_split<D, BT, 2, LO, HI>(a, stream);
        if constexpr (FOUR) {
            if (ks == 4) return launch_split<D, BT, 4, LO, HI>(a, stream);
        }
    }
    return launch_instance<D, BT, LO, HI>(unsplit_item(a, cus), a, stream);
}

}  // namespace dma
