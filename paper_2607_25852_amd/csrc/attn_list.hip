// Verify attention over a paged KV cache, bf16, over a list of items: for calls of at least two
// (request, kv-head, row block) units per compute unit, for calls with a given split size, whose
// splits are each request's own, and for calls of short contexts (plan_attn).
//
// The same products as in attn.hip, over another division of the work: an item is one split of
// one (request, kv-head, row block), and persistent workgroups claim items, longest first, from a
// counter. With several items per workgroup the claims even out the end by themselves, whatever
// bounds an item. Below two units per compute unit the splits are too few or too short for that,
// and ranges of equal cost are faster. Measured, this kernel against the ranges of attn.hip
// (contexts lognormal, two runs of each):
//   256 units (32 requests, 8 kv-heads, pages of 64)   168 against 155 us
//   384 units (48 requests)                            228-238 against 215
//   512 units (64 requests)                            286-295 against 284-294
//   768 units (96 requests, 5 positions)               390-397 against 400-432
//   1024 units (128 requests, 5 positions)             273-278 against 276-291
//   512 and 768 units of 4 kv-heads                    164-167 against 159-164, 229 against 227-236
// On pages below 64 tokens, whose pages this kernel looks up per lane and the ranges per 1 KB
// segment, the ranges are still ahead there: 512 units on pages of 16 309-313 against 299-300 us, at
// head dim 64 166-168 against 155-158 us; 1024 units 310-314 against 311-313. The line is drawn by
// units alone.
// Bound by the K/V stream: at 64 requests of 512..32768 tokens and 16 positions 1.70 GB, 5.8 to 6.2
// TB/s over the call on several cards, of the 7.1 TB/s that a plain read reaches.
#include <algorithm>

#include "attn_list_plan.h"
#include "attn_tile.h"
#include "sv_internal.h"

namespace sv {
namespace {

template <int HD, int NBUF>
struct LdsRing {
    static constexpr int kTileBytes = kTile * HD * 2;  // one tensor
    static constexpr int kMaxSlots = 1024;              // page-table entries of one split
    uint16_t kv[NBUF][2][kTile * HD];                   // [buffer][K=0/V=1][token*HD + d]
    int32_t pid[kMaxSlots];
};

// One work item (request i, kv-head h, split s, up to (NW/HALVES)*32 query rows from row0
// of the kv-head group). NBUF-deep LDS ring:
// tile t is multiplied while tiles t+1 .. t+NBUF-1 stream in. HALVES == 2: wave w owns
// query rows 32*(w/2) .. +31 of the row block and token half w%2 of every tile (so a
// 64-row group keeps all four SIMDs busy, two waves each); the two halves of a row group
// merge their softmax states at the end. HALVES == 1: wave w owns rows 32*w .. +31 over
// the whole tile (256 rows per workgroup). Every early return is uniform over the
// workgroup.
template <int HD, int NW, int NBUF, bool ONEPAGE, int HALVES>
__device__ __forceinline__ void attn_item(const AttnArgs& a, LdsRing<HD, NBUF>& lds, int i, int h, int s, int row0) {
    constexpr int CPR = HD / 8;             // 16-byte chunks per token row
    constexpr int TPS = 1024 / (HD * 2);    // tokens per 1 KB DMA segment
    constexpr int NSEG = kTile / TPS;       // segments per tensor per tile
    constexpr int IPW = 2 * NSEG / NW;      // DMA instructions per wave per tile
    static_assert(IPW * NW == 2 * NSEG, "DMA split");
    constexpr int KK = HD / 16;             // MFMA k-steps over the head dim
    constexpr int DT = HD / 32;             // output d-tiles
    constexpr int PF = NBUF - 1;            // prefetch distance in tiles

    // The thread id passes through an empty asm statement, so the per-lane values derived
    // from it (LDS and DMA offsets) are recomputed per item instead of being hoisted out
    // of the persistent item loop, where the invariants of both wave mappings would stay
    // live together (252 VGPRs instead of about 220, leaving no room for the operand
    // prefetch in compute_tile).
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63, w = tid >> 6;
    const int q0 = a.qo[i];
    const int k_i = a.qo[i + 1] - q0;
    int kv_len = a.kv_lens[i];
    if (kv_len > a.max_kv_len) kv_len = a.max_kv_len;
    const int L = kv_len - k_i;
    // (bitwise or: both descriptor loads are issued before the test)
    if ((kv_len < k_i) | !rows_in_batch(q0, k_i, a.block, a.total_q)) return;
    const int tok_begin = s * a.split;
    if (tok_begin >= kv_len) return;
    const int tok_end = min(kv_len, tok_begin + a.split);
    const int nsplit = (kv_len + a.split - 1) / a.split;
    constexpr int RB = (NW / HALVES) * 32;    // query rows this mapping covers
    const int M = min(a.G * k_i - row0, RB);  // rows of this item
    if (M <= 0) return;

    // page ids of this split -> LDS (the host keeps a split within 1024 pages). The first
    // page id of each thread is loaded before the query fragments and stored after them,
    // so the two round trips overlap.
    const int slot0 = tok_begin >> a.log2P;
    const int nslots = ((tok_end - 1) >> a.log2P) - slot0 + 1;
    const int32_t* __restrict__ pt = a.page_table + (size_t)i * a.maxp;
    int pg0 = -1;
    if (tid < nslots && slot0 + tid < a.maxp) pg0 = pt[slot0 + tid];

    // this lane's query row (N index of the MFMA) and its half (K-slice selector)
    // row group; token half of each tile (HALVES == 2), else the whole tile
    const int rg = w / HALVES, th = HALVES == 2 ? (w & 1) : 0;
    const int r = rg * 32 + (lane & 31);
    const int half = lane >> 5;
    const bool row_ok = r < M;
    const int rr = row0 + (row_ok ? r : 0);  // row within the request's kv-head group
    const int jq = rr / a.G;
    const int head = h * a.G + rr % a.G;
    const int limit = L + jq;  // last visible key of this row (inclusive)
    const int last_key = min(limit, tok_end - 1);  // ... and of this split

    // Per-lane element offsets of the V^T transpose reads inside a tile's V buffer: read
    // (qh, d-tile t) of 16-token k-chunk c lies at 16c*HD + vofs[qh][t] (for half-tile waves
    // c counts from their own half, whose offset vofs includes). The swizzle sees only the
    // token's position mod 16, which c does not change, so these 2*DT values serve every
    // chunk of every tile and each read costs one add of the buffer base.
    int vofs[2][DT];
    {
        const int g = lane >> 4, jl = lane & 15;
#pragma unroll
        for (int qh = 0; qh < 2; qh++) {
            const int tl = 8 * qh + 4 * (g >> 1) + (jl >> 2);  // token mod 16
#pragma unroll
            for (int t = 0; t < DT; t++) {
                const int dd = 32 * t + 16 * (g & 1) + 4 * (jl & 3);
                vofs[qh][t] = (HALVES == 2 ? th * 32 * HD : 0) + tl * HD +
                              (((dd >> 3) ^ (swz(tl) & (CPR - 1))) << 3) + (dd & 7);
            }
        }
    }
    const uint16_t* __restrict__ qp = (const uint16_t*)a.q;
    const uint16_t* __restrict__ kcp = (const uint16_t*)a.kc;
    const uint16_t* __restrict__ vcp = (const uint16_t*)a.vc;
    bf16x8 qf[KK];
    {
        const uint16_t* src = qp + ((size_t)(q0 + jq) * a.Hq + head) * HD;
#pragma unroll
        for (int kk = 0; kk < KK; kk++) {
            u16x8 v = row_ok ? *(const u16x8*)(src + kk * 16 + half * 8) : u16x8{0, 0, 0, 0, 0, 0, 0, 0};
            qf[kk] = __builtin_bit_cast(bf16x8, v);
        }
    }
    if (tid < nslots) lds.pid[tid] = (pg0 >= 0 && pg0 < a.num_pages) ? pg0 : -1;
    for (int e = tid + NW * 64; e < nslots; e += NW * 64) {
        const int slot = slot0 + e;
        const int pg = slot < a.maxp ? pt[slot] : -1;
        lds.pid[e] = (pg >= 0 && pg < a.num_pages) ? pg : -1;
    }
    // the query fragments must have landed before the DMA ring starts: a wait the
    // compiler sees (vmcnt(0)) keeps it from re-checking them inside the loop, where
    // a vmcnt(0) would also drain the ring
    __builtin_amdgcn_s_waitcnt(0x0F70);
    f32x16 o[DT];
#pragma unroll
    for (int t = 0; t < DT; t++) o[t] = f32x16{};
    float m_run = -1e30f, l_run = 0.0f;

    const size_t head_off = (size_t)h << a.log2P;
    const int pmask = (1 << a.log2P) - 1;
    const uint32_t lds_ring = (uint32_t)(uintptr_t)&lds.kv[0][0][0];
    __syncthreads();  // page ids visible

    // DMA of one tile: wave w issues segments w*IPW .. w*IPW+IPW-1 of the 2*NSEG
    // (K segments first, then V). Lane l of a segment moves token row t = seg*TPS + l/CPR,
    // position l%CPR, fetching logical chunk (l%CPR) ^ swz(t); the per-lane byte offset of
    // that chunk inside the tile is loop-invariant.
    // ONEPAGE (page size >= 64): a 64-token tile lies inside one page, so each tile needs
    // one wave-uniform base address; an invalid page reads page 0 (always present).
    // Otherwise every lane looks its page up; tokens past the split end or on an invalid
    // page read the first element of the cache. Either way such tokens are masked out of
    // the scores and zeroed in the V operand.
    uint32_t voff[IPW], ldsoff[IPW];
    int tk[IPW];
#pragma unroll
    for (int k = 0; k < IPW; k++) {
        const int n = w * IPW + k;
        const int seg = n % NSEG;
        const int t = seg * TPS + lane / CPR;
        tk[k] = t;
        voff[k] = (uint32_t)(t * HD + (((lane % CPR) ^ (swz(t) & (CPR - 1))) << 3)) * 2u;
        ldsoff[k] = (uint32_t)__builtin_amdgcn_readfirstlane((n / NSEG) * LdsRing<HD, NBUF>::kTileBytes + seg * 1024);
    }
    const int my_tensor = __builtin_amdgcn_readfirstlane((w * IPW) / NSEG);  // a wave moves one tensor
    const uint16_t* cbase = my_tensor ? vcp : kcp;
    auto issue_tile = [&](int tile, int buf) {
        const int tb = tok_begin + tile * kTile;
        const uint32_t lbuf = lds_ring + (uint32_t)(buf * 2 * LdsRing<HD, NBUF>::kTileBytes);
        if constexpr (ONEPAGE) {
            const int pg = __builtin_amdgcn_readfirstlane(lds.pid[(tb >> a.log2P) - slot0]);
            const uint16_t* base = pg >= 0
                ? cbase + ((((size_t)pg * a.Hkv) << a.log2P) + head_off + (size_t)(tb & pmask)) * HD
                : cbase + (size_t)(tb & pmask) * HD;
#pragma unroll
            for (int k = 0; k < IPW; k++) dma16s(voff[k], base, lbuf + ldsoff[k]);
        } else {
#pragma unroll
            for (int k = 0; k < IPW; k++) {
                const int tok = tb + tk[k];
                const int pg = lds.pid[min((tok >> a.log2P) - slot0, nslots - 1)];
                const uint16_t* src = (tok < tok_end && pg >= 0)
                    ? cbase + ((((size_t)pg * a.Hkv) << a.log2P) + head_off + (size_t)(tok & pmask)) * HD
                          + (voff[k] / 2 - tk[k] * HD)
                    : cbase;
                dma16(src, lbuf + ldsoff[k]);
            }
        }
    };

    constexpr int NSB = 2 / HALVES;  // 32-token halves of a tile handled by this wave
    auto compute_tile = [&](int buf, int tb) {
        if (rg * 32 >= M) return;
        const uint16_t* kt = lds.kv[buf][0];
        const uint16_t* vt = lds.kv[buf][1];
        // S^T = K Q^T for each 32-token half this wave owns (unscaled), as two independent
        // accumulation chains: the two halves (whole-tile waves), or the even and odd
        // k-steps of one half. Each K fragment is read from LDS KPD MFMAs before the MFMA
        // that consumes it; the scheduling barriers keep that order, so the LDS latency
        // runs under the matrix pipe instead of stalling every MFMA.
        f32x16 sacc[NSB];
        {
            const int sw = swz(lane & 31) & (CPR - 1);  // swz depends on t % 16 only
            const uint16_t* krow0 = kt + ((HALVES == 2 ? th : 0) * 32 + (lane & 31)) * HD;
            constexpr int NF = NSB * KK;  // K fragments (= MFMAs) per tile
            constexpr int KPD = 4;
            // fragment j: whole-tile waves alternate the token halves (j % 2) at k-step j / 2;
            // half-tile waves take k-step j of their half
            auto kaddr = [&](int j) {
                if constexpr (NSB == 2) return krow0 + (j & 1) * 32 * HD + (((2 * (j >> 1) + half) ^ sw) << 3);
                else return krow0 + (((2 * j + half) ^ sw) << 3);
            };
            bf16x8 kb[KPD + 1];
            f32x16 c0 = f32x16{}, c1 = f32x16{};
#pragma unroll
            for (int j = 0; j < KPD; j++) kb[j] = __builtin_bit_cast(bf16x8, *(const u16x8*)kaddr(j));
#pragma unroll
            for (int j = 0; j < NF; j++) {
                if (j + KPD < NF) kb[(j + KPD) % (KPD + 1)] = __builtin_bit_cast(bf16x8, *(const u16x8*)kaddr(j + KPD));
                __builtin_amdgcn_sched_barrier(0);
                const bf16x8 bq = NSB == 2 ? qf[j >> 1] : qf[j];
                if (j & 1) c1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kb[j % (KPD + 1)], bq, c1, 0, 0, 0);
                else c0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kb[j % (KPD + 1)], bq, c0, 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (NSB == 2) {
                sacc[0] = c0;
                sacc[1] = c1;
            } else {
                sacc[0] = c0 + c1;
            }
        }
        if constexpr (NSB == 2) {
            // Causal/tail mask on the raw scores: register e of half hh holds token
            // tb + 32hh + 4*half + (8(e/4) + e%4), masked when that token is past the row's last
            // visible key or the split end. Only halves reaching past L (the first row's limit)
            // or the split end need it, a wave-uniform test. Padding rows (r >= M) are not
            // masked: their query is zero, and their output column is neither written nor
            // mixed into the other columns.
    #pragma unroll
            for (int sb = 0; sb < NSB; sb++) {
                const int tb_h = tb + (HALVES == 2 ? th : sb) * 32;
                if (tb_h + 31 > L || tb_h + 32 > tok_end) {
                    const int dlim = last_key - tb_h - 4 * half;  // mask where 8(e/4) + e%4 > dlim
    #pragma unroll
                    for (int e = 0; e < 16; e++)
                        if (8 * (e >> 2) + (e & 3) > dlim) sacc[sb][e] = -INFINITY;
                }
            }
            // One online-softmax step per tile over the owned halves: the row max (lane-local,
            // then across the lane halves: the row's other 16 scores sit in lane l ^ 32, and
            // v_permlane32_swap with both operands = mx returns the lower half's values in one
            // result and the upper half's in the other), then a lazy rescale: the running max
            // moves only when a score exceeds it by more than 8 (log2 units), so p = 2^(z - m)
            // <= 256 stays exact in fp32 and bf16, and most tiles skip the accumulator rescale.
            float mx = fmaxf(fmaxf(sacc[0][0], sacc[0][1]), sacc[0][2]);
    #pragma unroll
            for (int e = 3; e < 15; e += 2) mx = fmaxf(fmaxf(mx, sacc[0][e]), sacc[0][e + 1]);
            mx = fmaxf(mx, sacc[0][15]);
            if constexpr (NSB == 2) {
    #pragma unroll
                for (int e = 0; e < 16; e += 2) mx = fmaxf(fmaxf(mx, sacc[1][e]), sacc[1][e + 1]);
            }
            {
                const auto sw2 = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
                mx = fmaxf(__uint_as_float(sw2[0]), __uint_as_float(sw2[1]));
            }
            const float mxs = mx * a.scale_log2;  // max in scaled log2 units (-inf: all masked)
            if (__any(mxs > m_run + 8.0f)) {
                const float m_new = fmaxf(m_run, mxs);
                const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
                l_run *= alpha;
    #pragma unroll
                for (int t = 0; t < DT; t++) o[t] *= alpha;
                m_run = m_new;
            }
            const float nm = -m_run;

            // O^T += V^T P^T. MFMA J of the tile: half J / NJ (whole-tile waves; else this
            // wave's half), 16-token k-chunk (J % NJ) / DT of that half, d-tile J % DT. The V^T
            // operand comes from two transpose reads: in 16-lane group g = lane/16, input lane
            // jl addresses token 16c + 8q + 4(g/2) + jl/4 at dims 32t + 16(g%2) + 4(jl%4) .. +3,
            // and output lane jl receives dim 32t + 16(g%2) + jl of tokens 16c + 8q + 4(g/2) +
            // 0..3. The operands are read VPD MFMAs ahead; the first VPD are in flight while the
            // exponents of the first half are computed.
            constexpr int NJ = 2 * DT;    // PV MFMAs per 32-token half
            constexpr int NT = NSB * NJ;  // PV MFMAs per tile for this wave
            constexpr int VPD = 4;
            auto vread = [&](int J) {
                const int c = 2 * (J / NJ) + (J % NJ) / DT, t = J % DT;  // (whole-tile waves)
                i16x4 vq[2];
    #pragma unroll
                for (int qh = 0; qh < 2; qh++) {
                    const uint16_t* addr = vt + 16 * c * HD + vofs[qh][t];
                    vq[qh] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)addr);
                }
                return __builtin_shufflevector(vq[0], vq[1], 0, 1, 2, 3, 4, 5, 6, 7);
            };
            i16x8 vb[VPD + 1];
    #pragma unroll
            for (int j = 0; j < VPD; j++) vb[j] = vread(j);
            __builtin_amdgcn_sched_barrier(0);
            // p = 2^(z * scale * log2e - m) of the first half, its row sum, and the bf16 P^T
            // fragments (already in the B-operand layout)
            float ps0 = 0.0f, ps1 = 0.0f;
    #pragma unroll
            for (int e = 0; e < 16; e++) {
                sacc[0][e] = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[0][e], a.scale_log2, nm));
                ps0 += sacc[0][e];
            }
            bf16x8 pb[NSB][2];
    #pragma unroll
            for (int cc = 0; cc < 2; cc++)
    #pragma unroll
                for (int e = 0; e < 8; e++) pb[0][cc][e] = (__bf16)sacc[0][8 * cc + e];
            __builtin_amdgcn_sched_barrier(0);
            // PV MFMAs. Whole-tile waves compute the second half's exponents between the first
            // half's MFMAs (16 / NJ per MFMA), so the vector ALU works under the matrix pipe.
    #pragma unroll
            for (int J = 0; J < NT; J++) {
                if (J + VPD < NT) vb[(J + VPD) % (VPD + 1)] = vread(J + VPD);
                __builtin_amdgcn_sched_barrier(0);
                const int t = J % DT;
                o[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, vb[J % (VPD + 1)]),
                                                                pb[J / NJ][(J % NJ) / DT], o[t], 0, 0, 0);
                if constexpr (NSB == 2) {
                    if (J < NJ) {
                        constexpr int EPM = 16 / NJ;
    #pragma unroll
                        for (int x = 0; x < EPM; x++) {
                            const int e = EPM * J + x;
                            sacc[1][e] = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[1][e], a.scale_log2, nm));
                            ps1 += sacc[1][e];
                        }
                        if (J == NJ - 1) {
    #pragma unroll
                            for (int cc = 0; cc < 2; cc++)
    #pragma unroll
                                for (int e = 0; e < 8; e++) pb[1][cc][e] = (__bf16)sacc[1][8 * cc + e];
                        }
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            l_run += ps0 + ps1;
        } else {
            // Half-tile waves: one online-softmax step per tile on the wave's half.
            const int hh = th;
            const int tb_h = tb + hh * 32;
            if (tb_h + 31 > L || tb_h + 32 > tok_end) {
                const int dlim = last_key - tb_h - 4 * half;  // mask where 8(e/4) + e%4 > dlim
#pragma unroll
                for (int e = 0; e < 16; e++)
                    if (8 * (e >> 2) + (e & 3) > dlim) sacc[0][e] = -INFINITY;
            }
            float mx = fmaxf(fmaxf(sacc[0][0], sacc[0][1]), sacc[0][2]);
#pragma unroll
            for (int e = 3; e < 15; e += 2) mx = fmaxf(fmaxf(mx, sacc[0][e]), sacc[0][e + 1]);
            mx = fmaxf(mx, sacc[0][15]);
            {
                const auto sw2 = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
                mx = fmaxf(__uint_as_float(sw2[0]), __uint_as_float(sw2[1]));
            }
            const float mxs = mx * a.scale_log2;
            if (__any(mxs > m_run + 8.0f)) {
                const float m_new = fmaxf(m_run, mxs);
                const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
                l_run *= alpha;
#pragma unroll
                for (int t = 0; t < DT; t++) o[t] *= alpha;
                m_run = m_new;
            }
            constexpr int NJ = 2 * DT;
            constexpr int VPD = 4;
            auto vread = [&](int j) {
                const int c = j / DT, t = j % DT;  // chunk within the wave's half
                i16x4 vq[2];
#pragma unroll
                for (int qh = 0; qh < 2; qh++) {
                    const uint16_t* addr = vt + 16 * c * HD + vofs[qh][t];
                    vq[qh] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)addr);
                }
                return __builtin_shufflevector(vq[0], vq[1], 0, 1, 2, 3, 4, 5, 6, 7);
            };
            i16x8 vb[VPD + 1];
#pragma unroll
            for (int j = 0; j < VPD; j++) vb[j] = vread(j);
            __builtin_amdgcn_sched_barrier(0);
            const float nm = -m_run;
            float psum = 0.0f;
#pragma unroll
            for (int e = 0; e < 16; e++) {
                const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[0][e], a.scale_log2, nm));
                sacc[0][e] = p;
                psum += p;
            }
            l_run += psum;
            bf16x8 pb[2];
#pragma unroll
            for (int cc = 0; cc < 2; cc++)
#pragma unroll
                for (int e = 0; e < 8; e++) pb[cc][e] = (__bf16)sacc[0][8 * cc + e];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < NJ; j++) {
                if (j + VPD < NJ) vb[(j + VPD) % (VPD + 1)] = vread(j + VPD);
                __builtin_amdgcn_sched_barrier(0);
                const int t = j % DT;
                o[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, vb[j % (VPD + 1)]), pb[j / DT],
                                                                o[t], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };

    // pipeline: before multiplying tile t, wait until its DMA (and only its) is done,
    // barrier (tile t visible to all waves; tile t-1 no longer read), then refill the
    // buffer of tile t-1 with tile t+PF.
    const int ntiles = (tok_end - tok_begin + kTile - 1) / kTile;
#pragma unroll
    for (int t = 0; t < PF; t++)
        if (t < ntiles) issue_tile(t, t);
    for (int t = 0; t < ntiles; t++) {
        const int newer = min(PF - 1, ntiles - 1 - t);  // tiles issued after t
        if constexpr (PF >= 3) {
            if (newer >= 2) wait_vm<2 * IPW>();
            else if (newer == 1) wait_vm<IPW>();
            else wait_vm<0>();
        } else {
            if (newer >= 1) wait_vm<IPW>();
            else wait_vm<0>();
        }
        // the last tile may reach past the split end: the lanes that copied those V rows
        // (foreign data, possibly non-finite) zero them, so P = 0 there contributes exactly 0
        if (t == ntiles - 1 && tok_begin + (t + 1) * kTile > tok_end && my_tensor == 1) {
            const int tb = tok_begin + t * kTile;
            char* vbuf = (char*)&lds.kv[0][0][0] + (t % NBUF) * 2 * LdsRing<HD, NBUF>::kTileBytes;
#pragma unroll
            for (int k = 0; k < IPW; k++)
                if (tb + tk[k] >= tok_end) *(u16x8*)(vbuf + ldsoff[k] + 16 * lane) = u16x8{};
        }
        __syncthreads();
        if (t + PF < ntiles) issue_tile(t + PF, (t + PF) % NBUF);
        compute_tile(t % NBUF, tok_begin + t * kTile);
    }

    // HALVES == 2: merge the token halves of each row group. The odd wave parks O in the
    // ring and (m, l) in the page-id area (both free now), the even wave combines and
    // writes. Both waves hold the same (row, dim) elements in the same lanes and registers.
    float l_tot = l_run + __shfl_xor(l_run, 32, 64);
    const bool grp_ok = rg * 32 < M;
    if constexpr (HALVES == 2) {
        static_assert((NW / 2) * 64 * 16 * DT * sizeof(float) <= sizeof(lds.kv), "park O");
        static_assert((NW / 2) * 96 * sizeof(float) <= sizeof(lds.pid), "park m, l");
        __syncthreads();
        float* park = (float*)&lds.kv[0][0][0] + (size_t)rg * (64 * 16 * DT);
        float* park_ml = (float*)&lds.pid[0] + rg * 96;
        if (grp_ok && th == 1) {
#pragma unroll
            for (int t = 0; t < DT; t++)
#pragma unroll
                for (int e = 0; e < 16; e++) park[(t * 16 + e) * 64 + lane] = o[t][e];
            park_ml[lane] = m_run;
            if (lane < 32) park_ml[64 + lane] = l_tot;  // rows in lanes 0..31
        }
        __syncthreads();
        if (!grp_ok || th == 1 || !row_ok) return;
        const float m2 = park_ml[lane];
        const float l2 = park_ml[64 + (lane & 31)];
        const float mm = fmaxf(m_run, m2);
        const float a1 = __builtin_amdgcn_exp2f(m_run - mm), a2 = __builtin_amdgcn_exp2f(m2 - mm);
#pragma unroll
        for (int t = 0; t < DT; t++)
#pragma unroll
            for (int e = 0; e < 16; e++) o[t][e] = o[t][e] * a1 + park[(t * 16 + e) * 64 + lane] * a2;
        l_tot = l_tot * a1 + l2 * a2;
        m_run = mm;
    } else {
        if (!grp_ok || !row_ok) return;
    }
    const float inv = l_tot > 0.0f ? 1.0f / l_tot : 0.0f;
    const float lse2 = l_tot > 0.0f ? m_run + __log2f(l_tot) : -INFINITY;
    const size_t orow = (size_t)(q0 + jq) * a.Hq + head;
    if (nsplit == 1) {
        uint16_t* op = (uint16_t*)a.out + orow * HD;
#pragma unroll
        for (int t = 0; t < DT; t++)
#pragma unroll
            for (int g2 = 0; g2 < 4; g2++) {
                const int dd = t * 32 + 8 * g2 + 4 * half;
                uint64_t pk = 0;
#pragma unroll
                for (int e = 0; e < 4; e++) pk |= (uint64_t)f2bf(o[t][4 * g2 + e] * inv) << (16 * e);
                *(uint64_t*)(op + dd) = pk;
            }
        if (a.lse && half == 0) a.lse[orow] = lse2 * kLn2;
    } else {
        float* pp = a.part_o + ((size_t)s * a.total_q * a.Hq + orow) * HD;
#pragma unroll
        for (int t = 0; t < DT; t++)
#pragma unroll
            for (int g2 = 0; g2 < 4; g2++) {
                const int dd = t * 32 + 8 * g2 + 4 * half;
                f32x4 v = {o[t][4 * g2] * inv, o[t][4 * g2 + 1] * inv, o[t][4 * g2 + 2] * inv, o[t][4 * g2 + 3] * inv};
                *(f32x4*)(pp + dd) = v;
            }
        if (half == 0) a.part_lse[(size_t)s * a.total_q * a.Hq + orow] = lse2;
    }
}

// Work list of the persistent kernel (attn_plan.h), built by one workgroup.
__global__ __launch_bounds__(1024) void attn_list_plan_kernel(AttnArgs a, AttnListArgs pa) {
    __shared__ int cursor[kPlanBuckets];
    __shared__ int wsum[1024 / 64];
    build_attn_list<1024>(pa, [&](int i, int& q0, int& k_i, int& kv) {
        q0 = a.qo[i];
        k_i = a.qo[i + 1] - q0;
        kv = a.kv_lens[i];
    }, cursor, wsum);
}

template <int HD, int NW, int NBUF, bool ONEPAGE, bool WIDE>
__global__ __launch_bounds__(NW * 64, 1) void attn_list_kernel(AttnArgs a, const int32_t* __restrict__ groups,
                                                               int32_t* __restrict__ ctr) {
    __shared__ __attribute__((aligned(16))) LdsRing<HD, NBUF> lds;
    __shared__ int s_item;
    // A work list that was never built (a run on a workspace without a plan) holds arbitrary
    // values: its length is capped by the longest possible list, a negative claim ends the
    // loop and items naming a request or split that does not exist are skipped, so every
    // access stays in bounds (the results are then unspecified).
    const int nitems = min(ctr[0], a.max_items);
    const int per_group = a.Hkv * a.nrb;
    for (;;) {
        if (threadIdx.x == 0) s_item = atomicAdd(&ctr[1], 1);
        __syncthreads();
        const int item = s_item;
        __syncthreads();
        if (item < 0 || item >= nitems) break;
        const uint32_t gv = (uint32_t)groups[item / per_group];  // request << 16 | split
        const int within = item % per_group;
        const int i = (int)(gv >> 16), h = within / a.nrb, s = (int)(gv & 0xFFFFu);
        if (i >= a.R || s >= a.max_splits) continue;
        const int row0 = (within % a.nrb) * (WIDE ? 2 * NW * 16 : NW * 16);
        if (WIDE && a.G * (a.qo[i + 1] - a.qo[i]) - row0 > NW * 16)
            attn_item<HD, NW, NBUF, ONEPAGE, 1>(a, lds, i, h, s, row0);
        else
            attn_item<HD, NW, NBUF, ONEPAGE, 2>(a, lds, i, h, s, row0);
    }
    // the last workgroup to finish leaves the counters as the plan left them, so the
    // next call on the same plan (another layer of the round) starts clean: every
    // workgroup has made its last claim before it counts itself here
    if (threadIdx.x == 0 && atomicAdd(&ctr[2], 1) == (int)gridDim.x - 1) {
        ctr[1] = 0;
        ctr[2] = 0;
    }
}


// merge split partials: grid (row chunk, kv-head, request), one thread per (query row of
// the group, 4-dim slice); every split's lse and partial are loaded before any math (one
// round of loads for up to 8 splits). Requests with a single split were written
// directly by the main kernel and exit here.
template <int HD>
__global__ __launch_bounds__(256) void attn_list_merge_kernel(AttnArgs a) {
    constexpr int SL = HD / 4;  // 4-dim slices per row
    const int h = blockIdx.y, i = blockIdx.z;
    const int q0 = a.qo[i], k_i = a.qo[i + 1] - q0;
    int kv_len = a.kv_lens[i];
    if (kv_len > a.max_kv_len) kv_len = a.max_kv_len;
    if (!rows_in_batch(q0, k_i, a.block, a.total_q) || kv_len < k_i) return;
    const int nsplit = (kv_len + a.split - 1) / a.split;
    if (nsplit <= 1) return;
    const int u = blockIdx.x * 256 + threadIdx.x;
    if (u >= a.G * k_i * SL) return;
    const int r = u / SL, sl = u % SL;
    const size_t orow = (size_t)(q0 + r / a.G) * a.Hq + h * a.G + r % a.G;
    const size_t sstride = (size_t)a.total_q * a.Hq;
    float mx = -INFINITY, wsum = 0.0f;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int s0 = 0; s0 < nsplit; s0 += 8) {
        float lw[8];
        f32x4 v[8];
#pragma unroll
        for (int k = 0; k < 8; k++) {
            const bool ok = s0 + k < nsplit;
            lw[k] = ok ? a.part_lse[(s0 + k) * sstride + orow] : -INFINITY;
            v[k] = ok ? *(const f32x4*)(a.part_o + ((s0 + k) * sstride + orow) * HD + sl * 4) : f32x4{0.f, 0.f, 0.f, 0.f};
        }
        float bm = mx;
#pragma unroll
        for (int k = 0; k < 8; k++) bm = fmaxf(bm, lw[k]);
        if (bm == -INFINITY) continue;
        const float sc = mx == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(mx - bm);
        wsum *= sc;
        acc *= sc;
#pragma unroll
        for (int k = 0; k < 8; k++) {
            const float wgt = lw[k] == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(lw[k] - bm);
            wsum += wgt;
            acc += wgt * v[k];
        }
        mx = bm;
    }
    const float inv = wsum > 0.0f ? 1.0f / wsum : 0.0f;
    uint64_t pk = 0;
#pragma unroll
    for (int e = 0; e < 4; e++) pk |= (uint64_t)f2bf(acc[e] * inv) << (16 * e);
    *(uint64_t*)((uint16_t*)a.out + orow * HD + sl * 4) = pk;
    if (a.lse && sl == 0) a.lse[orow] = wsum > 0.0f ? (mx + __log2f(wsum)) * kLn2 : -INFINITY;
}

}  // namespace

hipError_t launch_attn_list(const AttnArgs& a, const AttnPlan& plan, int head_dim, int page_size, int ncu,
                            const AttnListArgs& list, hipStream_t stream, bool build, bool run) {
    if (build) hipLaunchKernelGGL(attn_list_plan_kernel, dim3(1), dim3(1024), 0, stream, a, list);
    if (!run) return hipGetLastError();
    const dim3 grid(ncu);
#define SV_LAUNCH_ATTN(HDV, ONEP, HALV) \
    hipLaunchKernelGGL((attn_list_kernel<HDV, 8, 4, ONEP, HALV == 1>), grid, dim3(8 * 64), 0, stream, a, \
                       list.groups, list.ctr)
    const bool onepage = page_size >= kTile;
    if (plan.halves == 2) {
        if (head_dim == 128) {
            if (onepage) SV_LAUNCH_ATTN(128, true, 2);
            else SV_LAUNCH_ATTN(128, false, 2);
        } else {
            if (onepage) SV_LAUNCH_ATTN(64, true, 2);
            else SV_LAUNCH_ATTN(64, false, 2);
        }
    } else {
        if (head_dim == 128) {
            if (onepage) SV_LAUNCH_ATTN(128, true, 1);
            else SV_LAUNCH_ATTN(128, false, 1);
        } else {
            if (onepage) SV_LAUNCH_ATTN(64, true, 1);
            else SV_LAUNCH_ATTN(64, false, 1);
        }
    }
#undef SV_LAUNCH_ATTN
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || plan.max_splits <= 1) return e;
    const dim3 mgrid((a.G * a.block * (head_dim / 4) + 255) / 256, a.Hkv, a.R);
    if (head_dim == 128)
        hipLaunchKernelGGL((attn_list_merge_kernel<128>), mgrid, dim3(256), 0, stream, a);
    else
        hipLaunchKernelGGL((attn_list_merge_kernel<64>), mgrid, dim3(256), 0, stream, a);
    return hipGetLastError();
}

}  // namespace sv
