// Verify attention over a paged KV cache (AngelSpec Sec. 4.1: every kept block
// position is evaluated by the target model; Sec. 4.2: one dense packed batch).
//
// bf16 path (MFMA), for the calls of few (request, kv-head, row block) units that the host does not
// give to the list of items in attn_list.hip (plan_attn, with what either side measured). The plan
// (attn_plan.h) cuts the line of all (request, row block) units of a kv-head into ranges by cost;
// a workgroup takes one range of one head at a time and processes its pieces: the query rows of a
// unit against a run of 64-token tiles of the request's context. Query rows go on the N side of
// the MFMA and KV tokens on the M side, so S^T = K Q^T puts all scores of one query row in one
// lane pair: the online-softmax max/sum is lane-local plus one cross-half swap. The P^T fragment
// is then already in the B-operand layout of O^T = V^T P^T; V is staged transposed in LDS to
// serve the A operand. K and V tiles of 64 tokens are gathered through the page table into an LDS
// ring while earlier tiles are multiplied. A unit that lies in one range is written directly; the
// pieces of a cut unit leave fp32 partials merged by a second kernel (log-sum-exp weights).
//
// Bound by the K/V stream up to 64 rows per kv-head group, and in whole-tile units (above 128 rows)
// by the chain of dependent steps in a tile (scores, maximum, exponents, PV), which keeps no unit
// busy: at 32 requests of 65536..131072 tokens the matrix cores work 41% of the time, the vector
// ALUs 40%, both at once 13%, neither 32%. The rest is the pieces' starts and, with a list of
// splits, the uneven end. Measured, the list of attn_list.hip against this: 4 requests of 5
// positions (188 MB) 44.7 and 40.1 us, 27 requests on pages of 16 tokens (256 MB) 65.1 and 53.4
// us, 32 requests of 65536..131072 tokens (6.45 GB) 1353 and 1248 us.
//
// fp32 path (vector ALU): one workgroup per (query row, head); its four waves take
// interleaved 64-key tiles and merge their softmax states at the end.
#include <algorithm>
#include <atomic>
#include <type_traits>

#include "attn_plan.h"
#include "attn_tile.h"
#include "sv_internal.h"

namespace sv {
namespace {

struct RangeArgs : AttnArgs {
    int ranges, slot_rows;  // most ranges per head, rows of a partial result
};
static_assert(kPlanGrid == kAttnItems && kPlanUnits == kAttnListUnits && sizeof(AttnRange) == 32, "the host sizes the plan");

// ---------------------------------------------------------------------------------
// bf16 MFMA kernel
// ---------------------------------------------------------------------------------
// How a tile's K/V addresses are found (by page size): one page holds the whole tile, one
// page holds each 1 KB DMA segment of it, or every lane looks its token's page up.
enum class PageMode { kTile, kSegment, kLane };

template <int HD, int NBUF>
struct LdsRing {
    static constexpr int kTileBytes = kTile * HD * 2;  // one tensor
    static constexpr int kMaxSlots = 1024;              // page-table entries of one split
    uint16_t k[NBUF][kTile * HD];                       // [buffer][token*HD + d]
    uint16_t v[NBUF][kTile * HD];
    int32_t pid[kMaxSlots];
};

// wait until at most min(newer, MAX) tiles of IPW loads each are outstanding
template <int MAX, int IPW>
__device__ inline void wait_tiles(int newer) {
    if constexpr (MAX == 0) {
        wait_vm<0>();
    } else {
        if (newer >= MAX) wait_vm<MAX * IPW>();
        else wait_tiles<MAX - 1, IPW>(newer);
    }
}

// One piece of a unit (request i, kv-head h, up to (NW/HALVES)*32 query rows from row0 of
// the kv-head group): tiles t0 .. t1-1 of the nt tiles of its context. slot: its partial
// result when the unit is cut (t1 - t0 < nt). NBUF-deep LDS ring:
// tile t is multiplied while tiles t+1 .. t+NBUF-1 stream in. HALVES == 2: wave w owns
// query rows 32*(w/2) .. +31 of the row block and token half w%2 of every tile (so a
// 64-row group keeps all four SIMDs busy, two waves each); the two halves of a row group
// merge their softmax states at the end. HALVES == 1: wave w owns rows 32*w .. +31 over
// the whole tile (256 rows per workgroup).
template <int HD, int NW, int NBUF, PageMode PM, int HALVES>
__device__ __forceinline__ void attn_item(const RangeArgs& a, LdsRing<HD, NBUF>& lds, int i, int h, int row0, int q0,
                                          int k_i, int kv_len, int t0, int t1, int nt, int slot) {
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
    const int L = kv_len - k_i;
    const int p_begin = t0 * kTile;                    // tokens of the piece
    const int p_end = min(kv_len, t1 * kTile);
    constexpr int RB = (NW / HALVES) * 32;    // query rows this mapping covers
    const int M = min(a.G * k_i - row0, RB);  // rows of this item (at least 1)

    // The page ids of at most kMaxSlots pages are staged in LDS at a time; a piece over more
    // pages is walked in chunks of whole tiles. The first page id of each thread is loaded
    // before the query fragments and stored after them, so the two round trips overlap.
    const int32_t* __restrict__ pt = a.page_table + (size_t)i * a.maxp;
    constexpr int kMaxSlots = LdsRing<HD, NBUF>::kMaxSlots;
    const int chunk_tiles = max(1, ((kMaxSlots - 2) << a.log2P) / kTile);
    int slot0 = p_begin >> a.log2P;
    int pg0 = -1;
    if (slot0 + tid < a.maxp) pg0 = pt[slot0 + tid];

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
    const int last_key = min(limit, p_end - 1);  // ... and of this piece

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
    // DMA of one tile: wave w issues segments w*IPW .. w*IPW+IPW-1 of the 2*NSEG
    // (K segments first, then V). Lane l of a segment moves token row t = seg*TPS + l/CPR,
    // position l%CPR, fetching logical chunk (l%CPR) ^ swz(t); the per-lane byte offset of
    // that chunk inside the tile (or segment) is loop-invariant.
    // Tile and segment pages need one wave-uniform base address each; an invalid page, or a
    // segment past the piece's end, reads page 0 (always present). Per-lane look-up: tokens
    // past the end or on an invalid page read the first element of the cache. Either way such
    // tokens are masked out of the scores and zeroed in the V operand.
    uint32_t voff[IPW], ldsoff[IPW];
    int tk[IPW], sg[IPW];
#pragma unroll
    for (int k = 0; k < IPW; k++) {
        const int n = w * IPW + k;
        const int seg = n % NSEG;
        const int t = seg * TPS + lane / CPR;
        tk[k] = t;
        sg[k] = __builtin_amdgcn_readfirstlane(seg * TPS);
        voff[k] = (uint32_t)((PM == PageMode::kSegment ? lane / CPR : t) * HD + (((lane % CPR) ^ (swz(t) & (CPR - 1))) << 3)) * 2u;
        ldsoff[k] = (uint32_t)__builtin_amdgcn_readfirstlane(seg * 1024);
    }
    constexpr int TB = LdsRing<HD, NBUF>::kTileBytes;
    const int my_tensor = __builtin_amdgcn_readfirstlane((w * IPW) / NSEG);  // a wave moves one tensor
    const uint16_t* cbase = my_tensor ? vcp : kcp;
    const uint32_t my_ring = (uint32_t)(uintptr_t)(my_tensor ? &lds.v[0][0] : &lds.k[0][0]);
    int ibuf = 0;  // the buffer of this wave's tensor that the next issued tile goes to
    // The page ids of a tile are read from LDS (find_pages) one step before its DMA is issued
    // (issue_tile), so the look-up's latency is off the path from barrier to barrier.
    constexpr int NPG = PM == PageMode::kTile ? 1 : IPW;
    int pgv[NPG];
    auto find_pages = [&](int tile) {
        const int tb = p_begin + tile * kTile;
#pragma unroll
        for (int k = 0; k < NPG; k++) {
            const int tok = PM == PageMode::kTile ? tb : tb + (PM == PageMode::kSegment ? sg[k] : tk[k]);
            pgv[k] = lds.pid[min((tok >> a.log2P) - slot0, kMaxSlots - 1)];
        }
    };
    auto issue_tile = [&](int tile) {
        const int tb = p_begin + tile * kTile;
        const uint32_t lbuf = my_ring + (uint32_t)(ibuf * TB);
        ibuf = ibuf + 1 == NBUF ? 0 : ibuf + 1;
        if constexpr (PM == PageMode::kTile) {
            const int pg = __builtin_amdgcn_readfirstlane(pgv[0]);
            const uint16_t* base = pg >= 0
                ? cbase + ((((size_t)pg * a.Hkv) << a.log2P) + head_off + (size_t)(tb & pmask)) * HD
                : cbase + (size_t)(tb & pmask) * HD;
#pragma unroll
            for (int k = 0; k < IPW; k++) dma16s(voff[k], base, lbuf + ldsoff[k]);
        } else if constexpr (PM == PageMode::kSegment) {
#pragma unroll
            for (int k = 0; k < IPW; k++) {
                const int tok = tb + sg[k];
                const int pg = __builtin_amdgcn_readfirstlane(pgv[k]);
                const uint16_t* base = pg >= 0 && tok < p_end
                    ? cbase + ((((size_t)pg * a.Hkv) << a.log2P) + head_off + (size_t)(tok & pmask)) * HD
                    : cbase + (size_t)(tok & pmask) * HD;
                dma16s(voff[k], base, lbuf + ldsoff[k]);
            }
        } else {
#pragma unroll
            for (int k = 0; k < IPW; k++) {
                const int tok = tb + tk[k];
                const uint16_t* src = (tok < p_end && pgv[k] >= 0)
                    ? cbase + ((((size_t)pgv[k] * a.Hkv) << a.log2P) + head_off + (size_t)(tok & pmask)) * HD
                          + (voff[k] / 2 - tk[k] * HD)
                    : cbase;
                dma16(src, lbuf + ldsoff[k]);
            }
        }
    };

    constexpr int NSB = 2 / HALVES;  // 32-token halves of a tile handled by this wave
    auto compute_tile = [&](const uint16_t* kt, const uint16_t* vt, int tb) {
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
                if (tb_h + 31 > L || tb_h + 32 > p_end) {
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
            if (tb_h + 31 > L || tb_h + 32 > p_end) {
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
    const bool active = __builtin_amdgcn_readfirstlane(rg) * 32 < M;
    const int ntiles = t1 - t0;
    for (int c0 = 0; c0 < ntiles; c0 += chunk_tiles) {
        const int c1 = min(ntiles, c0 + chunk_tiles);
        // (the ring is idle here: every earlier tile has been multiplied or is about to be by
        // waves that read no page id)
        const int tb0 = p_begin + c0 * kTile;
        slot0 = tb0 >> a.log2P;
        const int nslots = ((min(p_end, p_begin + c1 * kTile) - 1) >> a.log2P) - slot0 + 1;
        if (c0 > 0) pg0 = tid < nslots && slot0 + tid < a.maxp ? pt[slot0 + tid] : -1;
        if (tid < nslots) lds.pid[tid] = (pg0 >= 0 && pg0 < a.num_pages) ? pg0 : -1;
        for (int e = tid + NW * 64; e < nslots; e += NW * 64) {
            const int pslot = slot0 + e;
            const int pg = pslot < a.maxp ? pt[pslot] : -1;
            lds.pid[e] = (pg >= 0 && pg < a.num_pages) ? pg : -1;
        }
        __builtin_amdgcn_s_waitcnt(0x0F70);  // (as above: no load may be pending when the ring starts)
        __syncthreads();                     // page ids visible, the previous chunk's tiles read
#pragma unroll
        for (int t = 0; t < PF; t++)
            if (c0 + t < c1) {
                find_pages(c0 + t);
                issue_tile(c0 + t);
            }
        find_pages(c0 + PF);
        // Tile t: wait for its DMA (and only its), barrier (tile t visible to all waves; the
        // buffer that the next issue fills no longer read), issue tile t + PF, look the pages of
        // tile t + PF + 1 up, multiply. Waves without query rows only move data. (Both sides of
        // that wave-uniform branch run the same number of barriers.) The last PF tiles have
        // fewer loads behind them and, at the end of the context, a tail.
        int buf = c0 % NBUF;
        auto run = [&](auto with_rows) {
            int t = c0;
            for (; t + PF < c1; t++) {
                wait_vm<(PF - 1) * IPW>();
                __syncthreads();
                issue_tile(t + PF);
                find_pages(t + PF + 1);
                if constexpr (decltype(with_rows)::value) compute_tile(lds.k[buf], lds.v[buf], p_begin + t * kTile);
                buf = buf + 1 == NBUF ? 0 : buf + 1;
            }
            for (; t < c1; t++) {
                wait_tiles<PF - 1, IPW>(c1 - 1 - t);
                // the last tile may reach past the end: the lanes that copied those V rows (foreign
                // data, possibly non-finite) zero them, so P = 0 there contributes exactly 0
                if (t == ntiles - 1 && p_begin + (t + 1) * kTile > p_end && my_tensor == 1) {
                    const int tb = p_begin + t * kTile;
#pragma unroll
                    for (int k = 0; k < IPW; k++)
                        if (tb + tk[k] >= p_end) *(u16x8*)((char*)lds.v[buf] + ldsoff[k] + 16 * lane) = u16x8{};
                }
                __syncthreads();
                if constexpr (decltype(with_rows)::value) compute_tile(lds.k[buf], lds.v[buf], p_begin + t * kTile);
                buf = buf + 1 == NBUF ? 0 : buf + 1;
            }
        };
        if (active) run(std::true_type{});
        else run(std::false_type{});
    }

    // HALVES == 2: the two waves of a row group merge their token halves. Both hold the same
    // (row, dim) elements in the same lanes and registers; each parks the d-tiles the other
    // one finishes in the ring (free now), and (m, l) in the page-id area, then combines and
    // writes its own half of the d-tiles.
    float l_tot = l_run + __shfl_xor(l_run, 32, 64);
    constexpr int DO = HALVES == 2 ? DT / 2 : DT;  // d-tiles this wave writes, from d-tile th*DO
    f32x16 of[DO];
    if constexpr (HALVES == 2) {
        static_assert(NW * 64 * 16 * DO * sizeof(float) <= sizeof(lds.k) + sizeof(lds.v), "park O");
        static_assert(NW * 128 * sizeof(float) <= sizeof(lds.pid), "park m, l");
        __syncthreads();
        f32x4* park = (f32x4*)&lds.k[0][0] + lane;
        float* park_ml = (float*)&lds.pid[0] + lane;
        const bool odd = __builtin_amdgcn_readfirstlane(th);
        auto put = [&](int from) {
#pragma unroll
            for (int t = 0; t < DO; t++)
#pragma unroll
                for (int g = 0; g < 4; g++)
                    park[((w * DO + t) * 4 + g) * 64] = {o[from + t][4 * g], o[from + t][4 * g + 1], o[from + t][4 * g + 2],
                                                         o[from + t][4 * g + 3]};
        };
        if (active) {
            if (odd) put(0);
            else put(DO);
            park_ml[w * 128] = m_run;
            park_ml[w * 128 + 64] = l_tot;
        }
        __syncthreads();
        if (!active || !row_ok) return;
        const int ow = w ^ 1;
        const float m2 = park_ml[ow * 128], l2 = park_ml[ow * 128 + 64];
        const float mm = fmaxf(m_run, m2);
        const float a1 = __builtin_amdgcn_exp2f(m_run - mm), a2 = __builtin_amdgcn_exp2f(m2 - mm);
        auto get = [&](int from) {
#pragma unroll
            for (int t = 0; t < DO; t++)
#pragma unroll
                for (int g = 0; g < 4; g++) {
                    const f32x4 v = park[((ow * DO + t) * 4 + g) * 64];
#pragma unroll
                    for (int e = 0; e < 4; e++) of[t][4 * g + e] = o[from + t][4 * g + e] * a1 + v[e] * a2;
                }
        };
        if (odd) get(DO);
        else get(0);
        l_tot = l_tot * a1 + l2 * a2;
        m_run = mm;
    } else {
        if (!active || !row_ok) return;
#pragma unroll
        for (int t = 0; t < DO; t++) of[t] = o[t];
    }
    const float inv = l_tot > 0.0f ? 1.0f / l_tot : 0.0f;
    const float lse2 = l_tot > 0.0f ? m_run + __log2f(l_tot) : -INFINITY;
    const size_t orow = (size_t)(q0 + jq) * a.Hq + head;
    const int d0 = (HALVES == 2 ? th * DO * 32 : 0) + 4 * half;
    if (t1 - t0 == nt) {
        uint16_t* op = (uint16_t*)a.out + orow * HD + d0;
#pragma unroll
        for (int t = 0; t < DO; t++)
#pragma unroll
            for (int g = 0; g < 4; g++) {
                bf16x4 v;
#pragma unroll
                for (int e = 0; e < 4; e++) v[e] = (__bf16)(of[t][4 * g + e] * inv);
                *(bf16x4*)(op + t * 32 + 8 * g) = v;
            }
        if (a.lse && half == 0 && th == 0) a.lse[orow] = lse2 * kLn2;
    } else {
        const size_t prow = (size_t)slot * a.slot_rows + r;
        float* pp = a.part_o + prow * HD + d0;
#pragma unroll
        for (int t = 0; t < DO; t++)
#pragma unroll
            for (int g = 0; g < 4; g++) {
                f32x4 v;
#pragma unroll
                for (int e = 0; e < 4; e++) v[e] = of[t][4 * g + e] * inv;
                *(f32x4*)(pp + t * 32 + 8 * g) = v;
            }
        if (half == 0 && th == 0) a.part_lse[prow] = lse2;
    }
}

// The plan (attn_plan.h), built by one workgroup.
__global__ __launch_bounds__(1024) void attn_plan_kernel(RangeArgs a, AttnPlanArgs pa) {
    __shared__ uint32_t pre[kPlanUnits];  // (R units at least)
    __shared__ uint32_t wsum[1024 / 64];
    build_attn_plan<1024>(pa, [&](int i, int& q0, int& k_i, int& kv) {
        q0 = a.qo[i];
        k_i = a.qo[i + 1] - q0;
        kv = a.kv_lens[i];
    }, pre, wsum);
}

// Persistent kernel: a workgroup takes the item of its own index, then claims further ones
// from a counter when the grid does not take all items in one pass.
template <int HD, int NW, int NBUF, PageMode PM, bool WIDE>
__global__ __launch_bounds__(NW * 64, 1) void attn_bf16_kernel(RangeArgs a, const AttnRange* __restrict__ recs,
                                                               int32_t* __restrict__ ctr) {
    __shared__ __attribute__((aligned(16))) LdsRing<HD, NBUF> lds;
    __shared__ int s_item;
    // A plan that was never built (a run on a workspace without one) holds arbitrary values:
    // the number of ranges is clamped to what the workspace holds, a claim outside it ends the
    // loop, and walk_range passes existing pieces only, so every access stays in bounds and every
    // loop ends (the results are then unspecified).
    const int n = plan_ranges(ctr[0], a.ranges) * a.Hkv;  // (below 2^31: checked on the host)
    constexpr int RB = WIDE ? NW * 32 : NW * 16;
    const bool one_pass = plan_one_pass(n, gridDim.x);
    int index = blockIdx.x, claim = 0;
    for (;;) {
        // (opaque to the compiler, so that the claim stays at the head of the loop, in one
        // loop with its barriers)
        asm volatile("" : "+s"(claim));
        if (claim) {
            if (threadIdx.x == 0) s_item = (int)(gridDim.x + (unsigned)atomicAdd(&ctr[1], 1));
            __syncthreads();
            index = s_item;
            __syncthreads();
        }
        const int item = plan_item(index, n, one_pass);
        if (item < 0) break;
        const int rng = item / a.Hkv, h = item % a.Hkv;
        const AttnRange r0 = recs[rng], r1 = recs[rng + 1];
        walk_range(a, r0, r1, RB, [&](int i, int& q0, int& k_i, int& kv_len) {
            q0 = a.qo[i];
            k_i = a.qo[i + 1] - q0;
            kv_len = a.kv_lens[i];
        }, [&](int i, int row0, int q0, int k_i, int kv_len, int t0, int t1, int nt) {
            const int slot = 2 * (rng * a.Hkv + h) + (t0 == 0);
            if (WIDE && a.G * k_i - row0 > NW * 16)
                attn_item<HD, NW, NBUF, PM, 1>(a, lds, i, h, row0, q0, k_i, kv_len, t0, t1, nt, slot);
            else
                attn_item<HD, NW, NBUF, PM, 2>(a, lds, i, h, row0, q0, k_i, kv_len, t0, t1, nt, slot);
            __syncthreads();  // the LDS of this piece is free
        });
        if (one_pass) return;
        claim = 1;
    }
    // the last workgroup to finish leaves the counters as the plan left them, so the
    // next call on the same plan (another layer of the round) starts clean: every
    // workgroup has made its last claim before it counts itself here
    if (!one_pass && threadIdx.x == 0 && atomicAdd(&ctr[2], 1) == (int)gridDim.x - 1) {
        ctr[1] = 0;
        ctr[2] = 0;
    }
}

// merge of the cut units' partials: grid (row chunk, kv-head, cut). The workgroups of the
// first cut inside a unit merge its pieces: the one that starts it (the range before the cut)
// and one per cut. One thread per (query row, 4-dim slice); up to 8 pieces' lse and partials
// are loaded before any math.
template <int HD>
__global__ __launch_bounds__(256) void attn_merge_kernel(RangeArgs a, const AttnRange* __restrict__ recs,
                                                         const int32_t* __restrict__ ctr, int rb_rows) {
    constexpr int SL = HD / 4;  // 4-dim slices per row
    // one round of loads: the number of ranges, this cut, the one before and the 62 after
    const int c = blockIdx.z + 1, h = blockIdx.y, lane = threadIdx.x & 63;
    const int n = plan_ranges(ctr[0], a.ranges);
    const AttnRange mine = recs[min(c - 1 + lane, a.ranges)];
    if (c >= n) return;
    auto at = [&](int v, int l) { return __builtin_amdgcn_readlane(v, l); };
    const int i = at(mine.req, 1), block = at(mine.block, 1);
    if (at(mine.tile, 1) <= 0 || i < 0 || i >= a.R || block < 0 || block >= a.nrb) return;
    if (at(mine.req, 0) == i && at(mine.block, 0) == block && at(mine.tile, 0) > 0) return;  // not the unit's first cut
    const int q0 = at(mine.q0, 1), k_i = at(mine.k, 1);
    // the cuts of this unit follow each other
    uint64_t m = ~(__ballot(mine.req == i && mine.block == block && c - 1 + lane < n) | 1);
    int last = c - 1 + (m ? __builtin_ctzll(m) : 64) - 1;
    for (int b = c + 63; m == 0 && b < n; b += 64) {
        const AttnRange rn = recs[min(b + lane, a.ranges)];
        m = ~__ballot(rn.req == i && rn.block == block && b + lane < n);
        last += m ? __builtin_ctzll(m) : 64;
    }
    if (!rows_in_batch(q0, k_i, a.block, a.total_q)) return;  // (a plan of other inputs)
    const int row0 = block * rb_rows;
    const int M = min(a.G * k_i - row0, rb_rows);
    const int u = blockIdx.x * 256 + threadIdx.x;
    if (u >= M * SL) return;
    const int r = u / SL, sl = u % SL;
    const int rr = row0 + r;
    const size_t orow = (size_t)(q0 + rr / a.G) * a.Hq + h * a.G + rr % a.G;
    float mx = -INFINITY, wsum = 0.0f;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int s0 = c - 1; s0 <= last; s0 += 8) {
        float lw[8];
        f32x4 v[8];
#pragma unroll
        for (int k = 0; k < 8; k++) {
            const int s = s0 + k;
            const size_t prow = (2 * ((size_t)s * a.Hkv + h) + (s == c - 1)) * a.slot_rows + r;
            lw[k] = s <= last ? a.part_lse[prow] : -INFINITY;
            v[k] = s <= last ? *(const f32x4*)(a.part_o + prow * HD + sl * 4) : f32x4{0.f, 0.f, 0.f, 0.f};
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

// ---------------------------------------------------------------------------------
// fp32 vector kernel: one workgroup of four waves per (query row, head); HD <= 256, HD % 4 == 0
// ---------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void attn_f32_kernel(RangeArgs a, int HD) {
    // one workgroup per (row, head); wave wv takes the 64-key tiles wv, wv + 4, ... and the
    // four waves' softmax states are merged at the end
    __shared__ float s_o[4][4][64];
    __shared__ float s_ml[4][2];
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int unit = blockIdx.x;
    const int K = a.qo[a.R];
    if (K > a.total_q) return;
    const int row = unit / a.Hq, head = unit % a.Hq;
    if (row >= K) return;
    int lo = 0, hi = a.R - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (a.qo[mid] <= row) lo = mid; else hi = mid - 1;
    }
    const int i = lo;
    const int k_i = a.qo[i + 1] - a.qo[i];
    int kv_len = a.kv_lens[i];
    if (kv_len > a.max_kv_len) kv_len = a.max_kv_len;
    const int L = kv_len - k_i;
    if (L < 0 || k_i > a.block) return;
    const int limit = L + (row - a.qo[i]);
    const int kvh = head / a.G;
    const float* qp = (const float*)a.q + ((size_t)row * a.Hq + head) * HD;  // wave-uniform
    const float* kcp = (const float*)a.kc;
    const float* vcp = (const float*)a.vc;
    const int32_t* pt = a.page_table + (size_t)i * a.maxp;
    const int P = 1 << a.log2P;
    float o[4] = {0.f, 0.f, 0.f, 0.f};
    float m = -INFINITY, l = 0.0f;
    for (int base = 64 * wv; base <= limit; base += 256) {
        const int sk = base + lane;
        float z = -INFINITY;
        size_t off = 0;
        bool ok = false;
        if (sk <= limit) {
            const int slot = sk >> a.log2P;
            const int pg = slot < a.maxp ? pt[slot] : -1;
            if (pg >= 0 && pg < a.num_pages) {
                off = (((size_t)pg * a.Hkv + kvh) * P + (sk & (P - 1))) * HD;
                float dot = 0.0f;
#pragma unroll 4
                for (int e = 0; e < HD; e += 4) {
                    const f32x4 kv4 = *(const f32x4*)(kcp + off + e);
                    dot += qp[e] * kv4[0] + qp[e + 1] * kv4[1] + qp[e + 2] * kv4[2] + qp[e + 3] * kv4[3];
                }
                z = dot * a.scale;
                ok = true;
            }
        }
        float mx = z;
        for (int x = 32; x > 0; x >>= 1) mx = fmaxf(mx, __shfl_xor(mx, x, 64));
        const float m_new = fmaxf(m, mx);
        if (m_new == -INFINITY) continue;
        const float alpha = m == -INFINITY ? 0.0f : expf(m - m_new);
        const float p = ok ? expf(z - m_new) : 0.0f;
        float ps = p;
        for (int x = 32; x > 0; x >>= 1) ps += __shfl_xor(ps, x, 64);
        l = l * alpha + ps;
        m = m_new;
        for (int e = 0; e < 4; e++) o[e] *= alpha;
        // P V, keys in order for every output element. The key index is uniform, so each
        // key's p, mask bit and V row offset are broadcast with readlane (no LDS traffic), and
        // the V loads of 32 keys are issued before their products. Keys outside the mask or
        // on an invalid page are skipped, never multiplied.
        const int cnt = min(64, limit - base + 1);
        const uint32_t okmask_lo = (uint32_t)__ballot(ok), okmask_hi = (uint32_t)(__ballot(ok) >> 32);
        const uint32_t off_lo = (uint32_t)off, off_hi = (uint32_t)(off >> 32);
#pragma unroll
        for (int e = 0; e < 4; e++) {
            if (64 * e >= HD) break;
            const int dd = lane + 64 * e;
            const bool dok = dd < HD;
            for (int j0 = 0; j0 < cnt; j0 += 32) {
                float vv[32];
#pragma unroll
                for (int u = 0; u < 32; u++) {
                    const int jj = j0 + u;
                    const bool okj = jj < cnt && (((jj < 32 ? okmask_lo >> jj : okmask_hi >> (jj - 32)) & 1u) != 0);
                    const size_t offj = ((size_t)(uint32_t)__builtin_amdgcn_readlane((int)off_hi, jj & 63) << 32) |
                                        (uint32_t)__builtin_amdgcn_readlane((int)off_lo, jj & 63);
                    vv[u] = (okj && dok) ? vcp[offj + dd] : 0.0f;
                }
#pragma unroll
                for (int u = 0; u < 32; u++) {
                    const int jj = j0 + u;
                    const bool okj = jj < cnt && (((jj < 32 ? okmask_lo >> jj : okmask_hi >> (jj - 32)) & 1u) != 0);
                    if (okj) o[e] += __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, p), jj & 63)) * vv[u];
                }
            }
        }
    }
    // merge the four waves' (m, l, o): weights exp(m_w - M) over M = max m_w
#pragma unroll
    for (int e = 0; e < 4; e++) s_o[wv][e][lane] = o[e];
    if (lane == 0) {
        s_ml[wv][0] = m;
        s_ml[wv][1] = l;
    }
    __syncthreads();
    if (wv != 0) return;
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < 4; w++) M = fmaxf(M, s_ml[w][0]);
    float lt = 0.0f, ot[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < 4; w++) {
        const float mw = s_ml[w][0];
        const float wt = mw == -INFINITY ? 0.0f : expf(mw - M);
        lt += s_ml[w][1] * wt;
#pragma unroll
        for (int e = 0; e < 4; e++) ot[e] += s_o[w][e][lane] * wt;
    }
    float* op = (float*)a.out + ((size_t)row * a.Hq + head) * HD;
    const float inv = lt > 0.0f ? 1.0f / lt : 0.0f;
    for (int e = 0; e < 4; e++) {
        const int dd = lane + 64 * e;
        if (dd < HD) op[dd] = ot[e] * inv;
    }
    if (a.lse && lane == 0) a.lse[(size_t)row * a.Hq + head] = lt > 0.0f ? M + logf(lt) : -INFINITY;
}

int ilog2(int x) {
    int r = 0;
    while ((1 << r) < x) r++;
    return r;
}

}  // namespace

AttnPlanArgs attn_plan_args(const sv_attn_desc& d, const AttnPlan& p, void* ws) {
    char* w = (char*)ws;
    return AttnPlanArgs{d.num_reqs, d.block, d.total_q_max, d.max_kv_len, d.num_q_heads / d.num_kv_heads,
                        p.row_blocks, (p.waves / p.halves) * 32, p.ranges,
                        d.num_kv_heads, (AttnRange*)(w + p.off_groups),
                        (int32_t*)(w + p.off_ctr)};
}

AttnListArgs attn_list_args(const sv_attn_desc& d, const AttnPlan& p, void* ws) {
    char* w = (char*)ws;
    return AttnListArgs{d.num_reqs, d.block, d.total_q_max, d.max_kv_len, p.kv_split, d.num_kv_heads, p.row_blocks,
                        (int32_t*)(w + p.off_groups), (int32_t*)(w + p.off_ctr)};
}

hipError_t launch_attn(const sv_attn_desc& d, const AttnPlan& plan, const void* q,
                       const void* k_cache, const void* v_cache, const int32_t* page_table,
                       const int32_t* qo_indptr, const int32_t* kv_lens, void* out, float* lse,
                       void* ws, hipStream_t stream, int phases) {
    RangeArgs a{};
    a.q = q;
    a.kc = k_cache;
    a.vc = v_cache;
    a.page_table = page_table;
    a.qo = qo_indptr;
    a.kv_lens = kv_lens;
    a.out = out;
    a.lse = lse;
    a.part_o = plan.part_o_bytes ? (float*)ws : nullptr;
    a.part_lse = plan.part_o_bytes ? (float*)((char*)ws + plan.part_o_bytes) : nullptr;
    a.R = d.num_reqs;
    a.total_q = d.total_q_max;
    a.Hq = d.num_q_heads;
    a.Hkv = d.num_kv_heads;
    a.G = d.num_q_heads / d.num_kv_heads;
    a.block = d.block;
    a.log2P = ilog2(d.page_size);
    a.maxp = d.max_pages_per_req;
    a.num_pages = d.num_pages;
    a.max_kv_len = d.max_kv_len;
    a.ranges = plan.ranges;
    a.slot_rows = plan.slot_rows;
    a.split = plan.kv_split;
    a.max_splits = plan.max_splits;
    a.max_items = (int)std::min<long long>(
        (long long)d.num_reqs * plan.max_splits * d.num_kv_heads * plan.row_blocks, 0x7FFFFFFF);
    a.scale = d.sm_scale > 0.0f ? d.sm_scale : 1.0f / sqrtf((float)d.head_dim);
    a.scale_log2 = a.scale * kLog2e;

    if (d.dtype == SV_F32) {  // no work plan: one workgroup per (row, head)
        if (!(phases & kAttnRun)) return hipSuccess;
        const int units = d.total_q_max * d.num_q_heads;
        hipLaunchKernelGGL(attn_f32_kernel, dim3(units), dim3(256), 0, stream, a, d.head_dim);
        return hipGetLastError();
    }
    a.nrb = plan.row_blocks;
    // persistent grid: one workgroup per compute unit of the current device
    static std::atomic<int> cu_count[64];  // zero-initialised (static storage)
    int dev = 0;
    hipError_t e0 = hipGetDevice(&dev);
    if (e0 != hipSuccess) return e0;
    if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    int ncu = cu_count[dev].load(std::memory_order_relaxed);
    if (ncu == 0) {
        int n = 0;
        e0 = hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev);
        if (e0 != hipSuccess) return e0;
        ncu = n > 0 ? n : 1;
        cu_count[dev].store(ncu, std::memory_order_relaxed);
    }
    char* wsb = (char*)ws;
    if (plan.list)
        return launch_attn_list(a, plan, d.head_dim, d.page_size, ncu, attn_list_args(d, plan, ws), stream,
                                phases & kAttnPlan, phases & kAttnRun);
    const AttnPlanArgs pa = attn_plan_args(d, plan, ws);
    int32_t* ctr = (int32_t*)(wsb + plan.off_ctr);
    if (phases & kAttnPlan) hipLaunchKernelGGL(attn_plan_kernel, dim3(1), dim3(1024), 0, stream, a, pa);
    if (!(phases & kAttnRun)) return hipGetLastError();
    const dim3 grid(ncu);
#define SV_LAUNCH_ATTN(HDV, NB, PMODE, WIDE) \
    hipLaunchKernelGGL((attn_bf16_kernel<HDV, 8, NB, PageMode::PMODE, WIDE>), grid, dim3(8 * 64), 0, stream, a, \
                       pa.recs, ctr)
#define SV_LAUNCH_PAGES(HDV, NB, WIDE) \
    if (d.page_size >= kTile) SV_LAUNCH_ATTN(HDV, NB, kTile, WIDE); \
    else if (d.page_size >= 512 / HDV) SV_LAUNCH_ATTN(HDV, NB, kSegment, WIDE); \
    else SV_LAUNCH_ATTN(HDV, NB, kLane, WIDE)
    if (plan.halves == 2) {
        if (d.head_dim == 128) { SV_LAUNCH_PAGES(128, 4, false); }
        else { SV_LAUNCH_PAGES(64, 4, false); }
    } else {
        if (d.head_dim == 128) { SV_LAUNCH_PAGES(128, 4, true); }
        else { SV_LAUNCH_PAGES(64, 4, true); }
    }
#undef SV_LAUNCH_PAGES
#undef SV_LAUNCH_ATTN
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || plan.ranges <= 1) return e;
    const dim3 mgrid((plan.slot_rows * (d.head_dim / 4) + 255) / 256, d.num_kv_heads, plan.ranges - 1);
    if (d.head_dim == 128)
        hipLaunchKernelGGL((attn_merge_kernel<128>), mgrid, dim3(256), 0, stream, a, pa.recs, ctr, pa.rb_rows);
    else
        hipLaunchKernelGGL((attn_merge_kernel<64>), mgrid, dim3(256), 0, stream, a, pa.recs, ctr, pa.rb_rows);
    return hipGetLastError();
}

}  // namespace sv
