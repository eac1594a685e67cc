// What the two bf16 verify-attention kernels share (attn.hip: ranges of equal cost, attn_list.hip:
// a sorted work list): the call's arguments, the LDS tile layout and the copies into it.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "attn_list_plan.h"
#include "attn_plan.h"
#include "sv_host.h"

namespace sv {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint16_t u16x8 __attribute__((ext_vector_type(8)));

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr int kTile = 64;  // KV tokens per pipeline step
static_assert(kTile == kAttnTile, "the work plan counts tiles of the kernel's size");

struct AttnArgs {
    const void* q;
    const void* kc;
    const void* vc;
    const int32_t* page_table;
    const int32_t* qo;
    const int32_t* kv_lens;
    void* out;
    float* lse;
    // partial results, lse in the log2 domain. Ranges: [2 * items, slot_rows, d], slot 2x the
    // piece that continues a unit into item x, slot 2x + 1 the piece that starts one there.
    // List: [max_splits, total_q_max, Hq, d].
    float* part_o;
    float* part_lse;
    int R, total_q, Hq, Hkv, G, block;
    int log2P, maxp, num_pages, max_kv_len;
    // list: tokens per split, most per request; nrb: row blocks per (request, kv-head). (The order
    // of the fields matters to the compiler: with others the list kernels took 1% longer.)
    int split, max_splits, nrb;
    int max_items;               // list: R * max_splits * Hkv * nrb (capped at INT_MAX)
    float scale_log2;  // sm_scale * log2(e)
    float scale;       // sm_scale
};

// round-to-nearest-even fp32 -> bf16 bits
__device__ inline uint16_t f2bf(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7F800000u) == 0x7F800000u && (u & 0x7FFFFFu)) return 0x7FC0;
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// ---------------------------------------------------------------------------------
// LDS tile layout: a 64-token tile of K and of V, each [token][HD] bf16, rows of HD*2
// bytes with their 16-byte chunks XOR-swizzled: logical chunk c of token t sits at
// position c ^ swz(t). swz swaps the two 2-bit fields of t % 16 so that (a) the 16
// rows read together by one quarter-wave of the K-operand loads hit 16 different chunk
// positions and (b) the 4 rows x 4 chunks read by one half-wave of the transpose reads
// (two 16-lane groups) do too.
// ---------------------------------------------------------------------------------
__device__ __host__ inline int swz(int t) { return ((t & 3) << 2) | ((t >> 2) & 3); }

// Asynchronous 16-byte-per-lane copy global -> LDS: lane l's 16 bytes land at
// lds_base + 16*l. Issued from inline assembly so the compiler does not drain it
// before every LDS read; completion is awaited explicitly with wait_vm<N>(). The
// loads carry the non-temporal hint: every K/V byte is read by one workgroup once,
// so keeping it in L2 and the last-level cache only evicts lines that are reused.
__device__ inline void dma16(const void* gptr, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off nt" ::"v"(gptr), "s"(lds_base)
                 : "memory", "m0");
}
// Same copy with a wave-uniform 64-bit base in SGPRs and a 32-bit per-lane byte offset.
__device__ inline void dma16s(uint32_t voff, const void* sbase, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt" ::"v"(voff), "s"(sbase),
                 "s"(lds_base)
                 : "memory", "m0");
}
template <int N>
__device__ inline void wait_vm() {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef short i16x8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) i16x4 lds_i16x4;

// the bf16 attention over a work list (attn_list.hip); phases as launch_attn's
hipError_t launch_attn_list(const AttnArgs& a, const AttnPlan& plan, int head_dim, int page_size, int ncu,
                            const AttnListArgs& list, hipStream_t stream, bool build, bool run);

}  // namespace sv
