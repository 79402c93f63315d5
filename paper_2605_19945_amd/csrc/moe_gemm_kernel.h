// Grouped expert GEMMs on the gfx950 matrix cores -- the expert kernel the paper profiles in isolation
// (Sec. 3.3.2), whose latency over token count is the staircase GEM samples at tile boundaries.
//
//   GEMM1 + SwiGLU:  H[r, c] = silu(sum_i X[r,i] W1[e][i,c]) * (sum_i X[r,i] W3[e][i,c])
//   GEMM2:           Y[r, c] = sum_j H[r,j] W2[e][j,c]
// for the rows r of expert e (ragged, device-side counts), bf16 operands, fp32 accumulation.
// The router logits of large routers (E >= 32) run on the same kernel as one group.
//
// Design (CDNA4):
//   * work item = up to BM rows of ONE expert x 256 packed weight rows; the list of work items is
//     built on the device from the per-expert offsets (no host sync), experts with no rows get
//     none, row tiles have a run-time height (a multiple of 32 rows, the last one of an expert
//     possibly ragged: loads clamped, stores masked) -- no padding to the largest expert.
//   * v_mfma_f32_16x16x32_bf16 with the WEIGHT rows as the first operand and the TOKEN rows as the
//     second, so a lane's accumulator holds 4 consecutive output columns of one token row.  Under this
//     device's power limit the 16x16x32 shape sustains a higher clock than 32x32x16 (a quarter of the
//     accumulator registers read and written per flop): the same loop on 32x32x16 ran at 1.55 GHz and
//     1.28 PFLOP/s on the Mixtral shape, this one reaches 1.35.
//   * only the token rows go through LDS.  The weights are stored at load time in MFMA-fragment
//     order
//        Wf[e][n / 64][k / 64][4*q + a][lane][8],  lane l <-> packed weight row 64*(n/64) + 16*a + l % 16,
//                                                 reduction elements 64*(k/64) + 32*q + 8*(l/16) .. +8,
//     so a wavefront fetches one 16x32 operand fragment with ONE fully coalesced 1 KB load straight
//     into the registers the MFMA reads, two K steps ahead of its use (three register buffers), and the
//     eight fragments of its 64 weight rows for one K step are 8 KB in a row: one sequential stream per
//     wavefront (with a stream per row block the weight-streaming launches were 3 to 7 % slower).
//     The token rows are staged by global_load_lds into a ring of three LDS stages (XOR-swizzled 16-byte
//     chunks, see swz_of) and every wavefront multiplies ALL rows of the tile by its own 64 weight
//     rows (1 x 4 wave layout): no weight byte is loaded twice or touches LDS.
//   * weights and tokens are requested two K steps ahead, no further.  A compute unit gets no more than about
//     60 GB/s of what misses the L2 however much it has requested (read-only kernel, one wavefront per SIMD,
//     8 or 32 KB in flight for each), and where that is the limit the wavefronts never wait for data: they
//     stand at the next load, which is not accepted (time stamps around the waits: 56 cycles a K step at the
//     wait for the loads, which is what two stamps cost, of 1400 to 2500).  Requests further ahead only lengthen
//     the way to the first MFMA of a tile: with up to five K steps of weights in flight 1.9 -> 4.7 us for one
//     32-row block, 128 small experts, 8192 tokens 674 -> 717 us for the layer; a third token stage alone
//     687 -> 658, Mixtral shape, 4096 tokens 2156 -> 2101.
//   * every tile height has code of its own from the first load to the last store (tile_of): sharing the accumulators
//     and the epilogue between nine K loops keeps registers alive through all of them.  The last K steps
//     test once per sub-step whether they still request anything, not once per load; together with the scalar base
//     of the token loads this also compiles in a sixth of the time.
//     The 288-row kernel still spills 13 registers (second GEMM) and 15 (first), outside all loops: around the code of
//     the 8- and 9-block tiles, seven or eight stores and loads of a lane for a tile.
//   * one wavefront per SIMD (256 threads, up to 512 registers per lane, accumulators in AGPRs),
//     so all latency hiding is explicit: LDS fragment reads run one MFMA sub-step ahead, the
//     barrier that publishes stage kt+1 sits before the LAST sub-step of stage kt so that the first
//     fragments of the next stage are read under those MFMAs, and the loads of a K step are spread
//     one by one over its MFMA slots (bursts from four lockstep wavefronts overrun the compute
//     unit's single vector-memory pipe and stall MFMA issue).
//   * a K step of 64 is four sub-steps (K half q, token half th): the MFMAs of sub-step (q, th) multiply the
//     four 16-row weight blocks by the 16-row token blocks of half th, so the token fragments held in
//     registers at a time are those of half a tile.
//   * the tallest tile has 288 rows: 18 token blocks x 4 weight blocks of 4 accumulator registers: the 256
//     AGPRs hold sixteen token blocks, blocks 8 and 17 (the ninth of either half) accumulate in VGPRs.
//     Left to itself the compiler shuffles the 72 small accumulators between the two files inside the K
//     loop, so the tall tiles (256 and 288 rows) issue EVERY MFMA through inline asm with the register file
//     in the constraint (mfma_pinned_agpr / mfma_pinned_vgpr); what the compiler then no longer does for
//     these MFMAs -- keep writers of their operands and readers of their results at a distance -- the
//     kernel arranges itself and tests/test_isa_hazards.py checks on the compiled code.
//   * work items are ordered so that the workgroups running concurrently on one XCD share weight
//     panels through that XCD's L2, and so that each XCD's queue of work items is dense.
#pragma once
#include <stdlib.h>

#include <type_traits>
#include <utility>

#include "moe_internal.h"

// two floats rounded to nearest even and packed, a in the low half: one v_cvt_pk_bf16_f32
static __device__ inline uint32_t pack2_bf16(float a, float b) {
    typedef float f32x2_t __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
    const f32x2_t v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}
// g * sigmoid(g) with the hardware reciprocal (1 ulp): an IEEE division costs about ten more instructions
// per element, 144 elements per lane and tile, all of them after the last MFMA
static __device__ inline float silu_f32(float g) { return g * __builtin_amdgcn_rcpf(1.f + __expf(-g)); }

enum { EPI_PLAIN = 0, EPI_SWIGLU = 1, EPI_PAIR_SUM_F32 = 2, EPI_PARTIAL_F32 = 3 };

// Epilogues.  Accumulator element v of lane l in block (a, t) -- a: 16 packed weight rows, t: 16 token rows -- is
//   weight row  a*16 + 4*(l/16) + v,   token row  t*16 + l%16,
// so a lane owns 4 consecutive output columns of one token row per accumulator.  The wavefront's 64 packed
// weight rows are blocks a = 0..3; in the interleaved layouts (gate/up, high/low router term) rows 0..31 are
// the first and rows 32..63 the second member of the pair, i.e. block a pairs with block a + 2.
//
// Storage.  A tile of up to 256 rows keeps token block t in acc[.][t] (AGPRs).  The 288-row tile has 18 token
// blocks and 16 AGPR slots: when all nine 32-row blocks are valid (NINE), blocks 8 and 17 -- the last of either
// token half -- live in accv[.][0] and accv[.][1] (VGPRs) and the others close ranks; with fewer valid blocks
// everything fits the AGPR slots.  Every accumulator thus has ONE register file for the whole kernel: sharing
// a variable between an AGPR use in one case and a VGPR use in another makes the compiler keep it in one file
// and copy it around every MFMA of the other, right behind the MFMA that writes it.
template <int FT>
struct AccShape {
    static constexpr int NA = FT < 16 ? FT : 16;  // token blocks accumulating in AGPRs
    static constexpr int NV = FT > 16 ? FT - 16 : 1;  // in VGPRs (one unused slot keeps the type valid)
};
template <bool NINE, int FA, int NA, int NV>
static __device__ __forceinline__ const f32x4_t& acc_at(const f32x4_t (&acc)[FA][NA], const f32x4_t (&accv)[FA][NV],
                                                        int a, int t) {
    if (NINE) {
        if (t == 8) return accv[a][0];
        if (t == 17) return accv[a][NV - 1];
        return acc[a][t < 8 ? t : t - 1];
    }
    return acc[a][t < NA ? t : 0];  // (t >= NA is never reached at run time: fewer than nine valid blocks)
}

template <int FT, int FA, int TN, int EPI, bool NINE>
static __device__ inline void gemm_epilogue(const f32x4_t (&acc_)[FA][AccShape<FT>::NA],
                                            const f32x4_t (&accv_)[FA][AccShape<FT>::NV], const TileDesc& td, int Np,
                                            uint16_t* __restrict__ C, int ldc, int wn, int lane) {
    static_assert(FA == 4 && TN == 64, "wave tile");
    auto A = [&](int a, int t) -> const f32x4_t& {
        return acc_at<NINE, FA, AccShape<FT>::NA, AccShape<FT>::NV>(acc_, accv_, a, t);
    };
    const int frow = lane & 15, fq = lane >> 4;
#pragma unroll
    for (int t = 0; t < FT; ++t) {
        const int trow = t * 16 + frow;
        if (trow >= td.rows) continue;
        uint16_t* crow = C + (size_t)(td.row0 + trow) * ldc;
        const int prow = td.n0 + wn * TN;  // first packed weight row of this wavefront (Np is a multiple of 64)
        if (prow >= Np) continue;
        if constexpr (EPI == EPI_PAIR_SUM_F32) {
            // router logits: blocks 0, 1 hold the products with the high bf16 term of Wg, blocks 2, 3 those
            // with the low term of the same experts; their sum is stored as fp32 (C is a float matrix)
            float* frow_out = (float*)C + (size_t)(td.row0 + trow) * ldc;
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                f32x4_t o;
#pragma unroll
                for (int v = 0; v < 4; ++v) o[v] = A(a, t)[v] + A(a + 2, t)[v];
                *(f32x4_t*)(frow_out + prow / 2 + 16 * a + 4 * fq) = o;
            }
        } else if constexpr (EPI == EPI_PARTIAL_F32) {
            // partial sums of a reduction split, fp32 (C is a float matrix, one slab per split)
            float* frow_out = (float*)C + (size_t)(td.row0 + trow) * ldc;
#pragma unroll
            for (int a = 0; a < FA; ++a) *(f32x4_t*)(frow_out + prow + 16 * a + 4 * fq) = A(a, t);
        } else if constexpr (EPI == EPI_SWIGLU) {
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                float h[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) h[v] = silu_f32(A(a, t)[v]) * A(a + 2, t)[v];
                u32x2_t o;
                o.x = pack2_bf16(h[0], h[1]);
                o.y = pack2_bf16(h[2], h[3]);
                *(u32x2_t*)(crow + prow / 2 + 16 * a + 4 * fq) = o;
            }
        } else {
#pragma unroll
            for (int a = 0; a < FA; ++a) {
                u32x2_t o;
                o.x = pack2_bf16(A(a, t)[0], A(a, t)[1]);
                o.y = pack2_bf16(A(a, t)[2], A(a, t)[3]);
                *(u32x2_t*)(crow + prow + 16 * a + 4 * fq) = o;
            }
        }
    }
}

// A 16-byte store of device scope (sc1).  The compiler's builtin, not inline asm: a vector instruction that overwrites the
// data registers of a store of more than 64 bits has to stay two wait states behind it, which the compiler sees to for
// the stores it knows (tests/test_isa_hazards.py allows no others).
static __device__ inline void store_device_scope(char* p, const u32x4_t& v) {
    __builtin_amdgcn_global_store_b128((__attribute__((address_space(1))) u32x4_t*)p, v, "agent");
}

// bf16 epilogues (EPI_PLAIN, EPI_SWIGLU) through LDS.  Stored straight from the accumulators, a wave-level
// store would write 16 bytes to each of 32 rows; instead every wavefront parks its 64 output columns (32 after SwiGLU) of all rows in its own quarter of
// the token ring, which nobody reads any more, and writes them back out row-contiguously: 16 bytes per
// lane, whole 128-byte (64-byte) runs per row.  Rows are ROWB bytes apart in LDS with the 16-byte chunks
// XOR-swizzled by row so that both the 8-byte writes (32 rows at one column) and the 16-byte reads (8 or
// 16 rows at all columns) are spread over the banks.  Worth 0.2 % (Mixtral shape, 64 to 224 K steps per
// tile) to 1.8 % (f = 768: 12 K steps per tile) of the layer time; most of the cost of the scattered
// stores was their completion, which the wavefronts never waited for.
// The caller has made sure that no wavefront still reads the ring.
template <int FT, int FA, int BM, int TN, int EPI, bool NINE, bool MAY_SCOPE>
static __device__ inline void gemm_epilogue_staged(const f32x4_t (&acc_)[FA][AccShape<FT>::NA],
                                                   const f32x4_t (&accv_)[FA][AccShape<FT>::NV], const TileDesc& td,
                                                   int Np, uint16_t* __restrict__ C, int ldc, int wn, int lane,
                                                   char* lds_base, bool device_scope) {
    auto A = [&](int a, int t) -> const f32x4_t& {
        return acc_at<NINE, FA, AccShape<FT>::NA, AccShape<FT>::NV>(acc_, accv_, a, t);
    };
    static_assert(EPI == EPI_PLAIN || EPI == EPI_SWIGLU, "bf16 outputs");
    static_assert(FA == 4 && TN == 64, "wave tile");
    constexpr int OUTC = EPI == EPI_SWIGLU ? TN / 2 : TN;  // output columns of this wavefront per row
    constexpr int ROWB = OUTC * 2;                         // 128 or 64 bytes per row
    constexpr int NCH = ROWB / 16;                         // 16-byte chunks per row: 8 or 4
    char* stage = lds_base + wn * (BM * ROWB);
    const int frow = lane & 15, fq = lane >> 4;
    auto swz = [](int r) { return EPI == EPI_SWIGLU ? (r >> 2) & 3 : (r ^ (r >> 3)) & 7; };
#pragma unroll
    for (int t = 0; t < FT; ++t) {
        const int r = t * 16 + frow;
        // the lane's 4 columns of block a start at byte 32*a + 8*fq of the row: chunk 2*a + fq/2, half fq%2
        char* srow = stage + r * ROWB + 8 * (fq & 1);
        const int x = swz(r);
        if constexpr (EPI == EPI_SWIGLU) {
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                float h[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) h[v] = silu_f32(A(a, t)[v]) * A(a + 2, t)[v];
                u32x2_t o;
                o.x = pack2_bf16(h[0], h[1]);
                o.y = pack2_bf16(h[2], h[3]);
                *(u32x2_t*)(srow + (((2 * a + (fq >> 1)) ^ x) << 4)) = o;
            }
        } else {
#pragma unroll
            for (int a = 0; a < FA; ++a) {
                u32x2_t o;
                o.x = pack2_bf16(A(a, t)[0], A(a, t)[1]);
                o.y = pack2_bf16(A(a, t)[2], A(a, t)[3]);
                *(u32x2_t*)(srow + (((2 * a + (fq >> 1)) ^ x) << 4)) = o;
            }
        }
    }
    // The wavefront reads back only what it wrote itself, GRP wave-level stores at a time: the next group's LDS reads are
    // under way while this group is stored.  Read, wait and store one after the other cost a round trip to LDS for each of 36
    // (layer, us, that -> this: 64 medium experts 3862 -> 3845, 128 small experts, 8192 tokens, 671 -> 666, Mixtral shape, 4096
    // tokens, 2111 -> 2104).  What the stores themselves cost, expert GEMMs without those of GEMM2, us: 64 medium experts, 65536 rows,
    // 3397 -> 3307, 128 small experts 555 -> 517.  That is 44 and 37 ns for each of the 2048 and 1024 wave-level stores (1 KB) of a
    // compute unit; with all of them into 32 rows for each XCD (L2 hits) 32 and 26 ns of that go as well.
    const int prow = td.n0 + wn * TN;  // first packed weight row of this wavefront
    if (prow >= Np) return;            // Np is a multiple of 64
    constexpr int RPI = 64 / NCH;      // rows per wave-level store
    constexpr int NIT = FT * 16 / RPI, GRP = EPI == EPI_SWIGLU ? 2 : 4, NG = NIT / GRP;
    static_assert(NIT % GRP == 0, "whole groups");
    const int ch = lane % NCH, r0 = lane / NCH;
    char* const cbase = (char*)(C + (size_t)td.row0 * ldc + (EPI == EPI_SWIGLU ? prow / 2 : prow));  // wave-uniform
    const uint32_t voff = (uint32_t)r0 * (uint32_t)(ldc * 2) + (uint32_t)ch * 16u;
    const int lane_off = r0 * ROWB + ((ch ^ (EPI == EPI_SWIGLU ? (r0 >> 2) & 3 : r0)) << 4);
    auto copy_out = [&](auto full_c, auto scope_c) {
        constexpr bool FULL = decltype(full_c)::value;  // every row of the tile exists
        u32x4_t v[2][GRP];
        auto fetch = [&](int g, u32x4_t (&dst)[GRP]) {
#pragma unroll
            for (int i = 0; i < GRP; ++i) {
                const int it = g * GRP + i;  // rows it * RPI + r0; swz() of them as a fixed part and one of the place
                const int off = EPI == EPI_SWIGLU ? lane_off : lane_off ^ ((it & 7) << 4);
                dst[i] = *(const u32x4_t*)(stage + it * (RPI * ROWB) + off);
            }
        };
        fetch(0, v[0]);
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            if (g + 1 < NG) fetch(g + 1, v[(g + 1) & 1]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < GRP; ++i) {
                const int r = (g * GRP + i) * RPI;
                if (FULL || r + r0 < td.rows) {
                    char* const row = cbase + (size_t)r * (size_t)(ldc * 2);
                    if constexpr (decltype(scope_c)::value)
                        store_device_scope(row + voff, v[g & 1][i]);
                    else
                        *(u32x4_t*)(row + voff) = v[g & 1][i];
                }
            }
        }
    };
    const bool full = td.rows == FT * 16;
    if constexpr (MAY_SCOPE) {
        if (device_scope) {
            if (full) copy_out(std::true_type{}, std::true_type{});
            else copy_out(std::false_type{}, std::true_type{});
            return;
        }
    }
    if (full) copy_out(std::true_type{}, std::false_type{});
    else copy_out(std::false_type{}, std::false_type{});
}

template <int CH>
static __device__ inline int swz_of(int r) {
    // LDS: 64 banks x 4 B; a ds_read_b128 is served 16 lanes (256 B) per cycle.  The 16 rows a
    // lane group reads at one logical chunk must land in 16 distinct 16-byte slots of a 256-byte
    // bank line: rows sharing a bank-line position (r mod (16/CH)) get distinct XOR masks.
    static_assert(CH == 8, "128-byte staged rows");
    return (r >> 1) & 7;
}

// ---- explicitly scheduled LDS reads -------------------------------------------------------------
// The compiler's own placement of ds_read / s_waitcnt leaves every MFMA group waiting for the LDS
// reads issued just before it.  The reads of the software-pipelined K loop are issued through
// inline asm (invisible to the compiler's wait-count pass) and waited for explicitly.
template <int OFF>
static __device__ inline bf16x8_t lds_read_b128(uint32_t byte_addr) {
    u32x4_t v;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(byte_addr), "n"(OFF) : "memory");
    return __builtin_bit_cast(bf16x8_t, v);
}
template <int N>
static __device__ inline void wait_lgkmcnt() {
    asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(N) : "memory");
}
// makes the fragment "depend" on the preceding wait so that its consumers stay behind it
static __device__ inline void tie(bf16x8_t& f) { asm volatile("" : "+v"(f)); }
// the lane index, computed where it is asked for: the compiler can neither merge two of these nor move one
static __device__ inline int fresh_lane() {
    int lane;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=&v"(lane));
    return lane;
}

template <int N>
static __device__ inline void wait_vmcnt() {
    // s_waitcnt vmcnt(N) only: expcnt = 7, lgkmcnt = 15 are left unconstrained (gfx9 encoding)
    __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 0xF) | ((N >> 4) << 14));
}


template <int... I, class F>
static __device__ inline void static_for_impl(std::integer_sequence<int, I...>, F&& f) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
static __device__ inline void static_for(F&& f) {
    static_for_impl(std::make_integer_sequence<int, N>{}, f);
}

// Row tiles of more than 256 rows need more than the 256 accumulator registers (AGPRs) of a lane: two of
// the eighteen token blocks accumulate in ordinary VGPRs.  The MFMAs of the tall tiles are issued through
// inline asm that names the register file of the accumulator.  The asm is opaque to the compiler's hazard
// recogniser, which would otherwise keep a reader of an MFMA result, and a writer of an MFMA operand, the
// required wait states away: the caller places the VGPR ones first in a sub-step (the others follow before
// anything can read their result), reads accumulators only after the K loop, and claims the zeroed
// accumulators in their register file before the prologue (claim_agpr / claim_vgpr).
static __device__ inline void mfma_pinned_vgpr(f32x4_t& acc, const bf16x8_t& w, const bf16x8_t& x) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(w), "v"(x));
}
// the value exists in a register of that file from here on (see the use in gemm_tile)
static __device__ inline void claim_vgpr(f32x4_t& acc) { asm volatile("" : "+v"(acc)); }
static __device__ inline void claim_agpr(f32x4_t& acc) { asm volatile("" : "+a"(acc)); }
static __device__ inline void mfma_pinned_agpr(f32x4_t& acc, const bf16x8_t& w, const bf16x8_t& x) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(w), "v"(x));
}

// LDS of a workgroup: three stages of BM token rows of 128 bytes, or the staged output, BM rows of up to 128 bytes for
// each wavefront
static constexpr int gemm_lds_bytes(int bm, int nw) { return bm * 128 * (nw > 3 ? nw : 3); }

// Split K (gridDim.y > 1, used by the router-logit GEMM whose output is tiny next to its reduction
// length): workgroup (x, y) reduces over elements [y*K, (y+1)*K) of the K_total = gridDim.y * K long
// reduction dimension and writes its partial result c_split_bytes behind that of split y-1; the
// consumer adds the partial results in a fixed order.
// W_STREAM: the weight loads carry the non-temporal hint.  A launch in which every expert has a single row
// tile reads each weight once; plain loads then reach about 6.4 TB/s of the 8 TB/s HBM peak on this device and
// hinted ones about 7.2 TB/s (read-only streaming kernel, 1.9 GB).  Launches whose row tiles share weight
// panels through the L2 lose with the hint (Mixtral shape, 1024 rows per expert: +2.8 % time), so it is a
// variant picked per launch.
// gemm_tile: one work item (table entry bx) by one workgroup.
template <int BM, int EPI, int NW, bool W_STREAM>
static __device__ __forceinline__ void gemm_tile(int bx, const uint16_t* __restrict__ X, int ldx,
                                                 const int32_t* __restrict__ row_map,
                                                 const uint16_t* __restrict__ Wf, int Np, int K,
                                                 uint16_t* __restrict__ C, int ldc,
                                                 const TileDesc* __restrict__ table, size_t c_split_bytes,
                                                 bool device_scope) {
    constexpr int BN = 64 * NW, BK = 64, TN = BN / NW, FA = TN / 16, FM = BM / 32;
    constexpr int CH = BK / 8;   // 16-byte chunks per staged token row
    constexpr int RPL = 64 / CH; // rows covered by one wave-level load
    constexpr int XP = 32 / (NW * RPL);  // wave-level token loads of one wavefront per 32-row block
    constexpr int KQ = BK / 32;  // K halves of a K step: one v_mfma_f32_16x16x32_bf16 reduces over 32 elements
    constexpr int KK = 2 * KQ;   // MFMA sub-steps per K step: (K half q, token half th), kk = 2*q + th
    constexpr int WL = FA * KQ;  // weight loads per lane per K step
    constexpr int NB = 3, PF = NB - 1;  // weight register buffers and token ring stages; K steps both are requested ahead
    constexpr int SMEM = gemm_lds_bytes(BM, NW);
    constexpr int BLK = 16 * CH * 16;         // bytes between consecutive 16-row blocks in a stage
    static_assert(FA == 4 && KK == 4, "wave tile");
    static_assert(BM % 32 == 0 && FM >= 1 && FM <= 9, "row tile");
    static_assert(NW == 4 || NW == 2, "wavefronts per workgroup");

    extern __shared__ u32x4_t lds[];  // token ring: [stages][rows][CH]

    const TileDesc td = table[bx];
    if (td.rows <= 0) return;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lrow = lane / CH, lphys = lane % CH;
    const int KT = K / BK;
    const int fmv = (td.rows + 31) / 32;  // valid 32-row blocks: the same for all four wavefronts
    const int K_total = K * (int)gridDim.y;
    X += (size_t)blockIdx.y * K;
    C = (uint16_t*)((char*)C + (size_t)blockIdx.y * c_split_bytes);

    // token sources: pass p of a wavefront brings rows 8*(NW*p + wave) .. +8 of the tile (XP passes per
    // 32-row block), 32-bit byte offsets from the wave-uniform base X + kt*BK
    uint32_t xo[FM * XP];
#pragma unroll
    for (int p = 0; p < FM * XP; ++p) {
        const int r = (p * NW + wave) * RPL + lrow;
        xo[p] = (uint32_t)(td.row0 + (r < td.rows ? r : td.rows - 1));  // clamp: rows past the end are never stored
    }
    if (row_map != nullptr) {  // (one branch around all the look-ups: they are requested together)
#pragma unroll
        for (int p = 0; p < FM * XP; ++p) xo[p] = (uint32_t)row_map[xo[p]];
    }
#pragma unroll
    for (int p = 0; p < FM * XP; ++p) {
        const int r = (p * NW + wave) * RPL + lrow;
        // asm: the compiler would use a 64-bit multiply-add, whose result occupies a register pair through the K loop
        asm("v_mul_lo_u32 %0, %0, %1" : "+v"(xo[p]) : "s"(ldx * 2));
        xo[p] += (uint32_t)((lphys ^ swz_of<CH>(r)) * 16);
    }
    // weight source: the eight fragments a wavefront needs for one K step (4 row blocks x 2 K halves) are the
    // 8 KB at ((e*Np/64 + nb)*K/64 + kt)*8 KB, fragment j = 4*q + a at j KB: ONE sequential stream per
    // wavefront.  Wave-uniform base (scalar registers) plus the lane's 16 bytes.
    const int nbt = Np / 64;
    int nb = (td.n0 + wave * TN) / 64;
    if (nb >= nbt) nb = nbt - 1;  // past the last weight row: computed, never stored
    const char* wsrc = (const char*)(Wf + ((size_t)td.expert * nbt + nb) * ((size_t)K_total * 64) + (size_t)blockIdx.y * K * 64);
    // where this wavefront's 1 KB of a pass over a stage goes
    const uint32_t lds_wave = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds + (uint32_t)wave * (RPL * CH * 16);

    auto tile_of = [&](auto fmv_c) {
        constexpr int FMV = decltype(fmv_c)::value;  // valid 32-row blocks (compile time)
        constexpr int STAGE = FMV * 32 * CH;         // 16-byte chunks per token stage
        static_assert(NB * STAGE * 16 <= SMEM, "token ring");
        constexpr int NM = FMV * FA;                 // MFMAs per sub-step: FMV 16-row token blocks x 4 weight blocks
        constexpr int XV = FMV * XP;                 // token loads per lane per K step
        constexpr int NL = WL + XV;                  // loads per lane per K step

        // block (a, t): 16 packed weight rows x 16 token rows (storage: see AccShape)
        constexpr int FT = 2 * FMV, NA = AccShape<FT>::NA, NV = AccShape<FT>::NV;
        f32x4_t acc[FA][NA], accv[FA][NV];
#pragma unroll
        for (int a = 0; a < FA; ++a) {
#pragma unroll
            for (int t = 0; t < NA; ++t) acc[a][t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int t = 0; t < NV; ++t) accv[a][t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        }

        // The lane's addresses, this height's own: one set of registers for all nine heights would be reloaded from
        // scratch memory in the K loops of some of them.
        // fx: LDS byte address (inside a stage) of the lane's chunk of 16-row block 0 for either K half: token row
        // hl % 16, reduction elements 32*q + 8*(hl/16) .. +8 (the swizzle of a row depends on row % 16 only)
        const int hl = fresh_lane();
        const uint32_t wl = (uint32_t)hl * 16u;
        uint32_t xc[FMV * XP], fx[KQ];
        static_for<FMV * XP>([&](auto p) { xc[p] = xo[p]; asm volatile("" : "+v"(xc[p])); });
        static_for<KQ>([&](auto q) {
            const int row = hl & 15;
            fx[q] = (uint32_t)((row * CH + ((q * 4 + (hl >> 4)) ^ swz_of<CH>(row))) * 16);
        });

        bf16x8_t wr[NB][KQ][FA];
        bf16x8_t xf[2][FMV];  // sub-step (q, th): the 16-row token blocks th*FMV .. th*FMV + FMV - 1, K half q

        // The tall tiles issue every MFMA through inline asm (see mfma_pinned_agpr).  The compiler then does
        // not know that the first MFMA reads the accumulator it has just zeroed and would put the zeroing
        // writes directly in front of it, closer than the wait states a matrix instruction needs behind a
        // write of its third operand.  Claiming every accumulator here, in the register file its MFMAs use,
        // makes the zeros exist now; the prologue's loads, waits and barrier follow before the first MFMA.
        if constexpr (FM >= 8) {
            static_for<2 * FMV>([&](auto t_c) {
                constexpr int t = decltype(t_c)::value;
                static_for<FA>([&](auto a_c) {
                    constexpr int a = decltype(a_c)::value;
                    if constexpr (FMV == 9 && (t == 8 || t == 17)) {
                        claim_vgpr(accv[a][t == 8 ? 0 : NV - 1]);
                    } else {
                        claim_agpr(acc[a][FMV == 9 && t > 8 ? t - 1 : t]);
                    }
                });
            });
        }

        // token load p of a stage into ring slot `slot`; xbase: the first reduction element of that stage.  Inline asm
        // for the addressing mode: wave-uniform base plus the lane's 32-bit offset (the builtin keeps a 64-bit address
        // per load in vector registers and adds to it).  The lanes' 16 bytes land one after the other at M0,
        // which nothing else in these kernels uses (tests/test_gemm_registers.py).
        auto issue_x_one = [&](const char* xbase, int slot, int p) {
            const uint32_t dst = lds_wave + (uint32_t)((slot * STAGE + p * NW * RPL * CH) * 16);
            const uint32_t off = xc[p];
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                         :
                         : "s"(dst), "v"(off), "s"(xbase)
                         : "memory");
        };
        // Weight loads go through inline asm: the compiler's own wait-count pass would otherwise put a
        // nearly-zero vmcnt in front of the MFMAs that consume them (it cannot see through the
        // unrolled, branched loop) and collapse the prefetch distance.  They are waited for together
        // with the token loads, with exact counts, before the barrier that precedes their use.
        auto load_w_one = [&](int kt, auto buf_c, auto j_c) {  // j = q * FA + a
            constexpr int BUF = decltype(buf_c)::value;
            constexpr int kk = decltype(j_c)::value / FA, a = decltype(j_c)::value % FA;  // kk: K half here
            u32x4_t v;
            const char* base = wsrc + (size_t)kt * (WL * 1024) + kk * (FA * 1024);  // (offsets reach 4 KB)
            if constexpr (W_STREAM) {
                asm volatile("global_load_dwordx4 %0, %1, %2 offset:%3 nt"
                             : "=v"(v)
                             : "v"(wl), "s"(base), "n"(a * 1024)
                             : "memory");
            } else {
                asm volatile("global_load_dwordx4 %0, %1, %2 offset:%3"
                             : "=v"(v)
                             : "v"(wl), "s"(base), "n"(a * 1024)
                             : "memory");
            }
            wr[BUF][kk][a] = __builtin_bit_cast(bf16x8_t, v);
        };
        // prologue: stages 0 and 1, each stage's weights and tokens together so that what is needed first is oldest
        static_for<PF>([&](auto v_c) {
            constexpr int v = decltype(v_c)::value;
            if (v < KT) {
                static_for<WL>([&](auto j) { load_w_one(v, v_c, j); });
                static_for<XV>([&](auto p) { issue_x_one((const char*)X + v * (BK * 2), v, p); });
            }
        });
        if (KT > 1) wait_vmcnt<(PF - 1) * NL>();
        else wait_vmcnt<0>();
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        static_for<FMV>([&](auto b) { xf[0][b] = lds_read_b128<b * BLK>(fx[0]); });  // sub-step (0, 0)

        // one K step; BUF = kt % NB is a compile-time index of register buffer and ring slot.  STEADY: the step is not
        // among the last ones, so the prefetch of it exists and nothing in it is conditional.
        auto step = [&](int kt, auto buf_c, auto steady_c) {
            constexpr int BUF = decltype(buf_c)::value;
            constexpr bool STEADY = decltype(steady_c)::value;
            constexpr int BUF1 = (BUF + 1) % NB, BUFP = (BUF + PF) % NB;  // of the stages kt + 1 and kt + PF
            const bool more = STEADY || kt + PF < KT;
            const bool next = STEADY || kt + 1 < KT;
            const char* xbase = (const char*)(X + (size_t)(kt + PF) * BK);  // of the stage whose tokens are requested
            uint32_t sbase = (uint32_t)(BUF * STAGE * 16), nbase = (uint32_t)(BUF1 * STAGE * 16);
            // (opaque: the compiler would otherwise keep the lane addresses of every slot in registers)
            asm("" : "+s"(sbase), "+s"(nbase));
            // the weights of this stage landed before the barrier that published it
            static_for<WL>([&](auto j) { tie(wr[BUF][decltype(j)::value / FA][decltype(j)::value % FA]); });
            static_for<KK>([&](auto kk_c) {
                constexpr int kk = decltype(kk_c)::value;
                constexpr int cur = kk & 1, nxt = cur ^ 1;
                constexpr int q = kk >> 1, th = kk & 1;          // K half, token half of this sub-step
                constexpr int qn = (kk + 1) >> 1, thn = (kk + 1) & 1;  // of the next one (same K step)
                if constexpr (kk == KK - 1) {
                    // publish stage kt+1 before the last sub-step: own loads of stage kt+1 have landed (what may
                    // stay in flight: the stages after it), all wavefronts have issued and completed every LDS read
                    // of stage kt
                    if (more) wait_vmcnt<(PF - 1) * NL>();  // stage kt + 2, requested in this step
                    else if (next) wait_vmcnt<0>();
                    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
                } else {
                    wait_lgkmcnt<0>();
                }
                static_for<FMV>([&](auto b) { tie(xf[cur][b]); });
                __builtin_amdgcn_sched_barrier(0);
                static_for<NM>([&](auto m_c) {
                    constexpr int m = decltype(m_c)::value;
                    // a block that accumulates in VGPRs goes first: whatever reads its result next (the compiler may
                    // copy it at the end of a basic block) then sits behind the sub-step's other MFMAs
                    constexpr int g = m / FA;  // place of the token block in the sub-step
                    constexpr int b = FMV <= 8 ? g : (g + 8) % 9;
                    // the weight blocks there and back, 0 1 2 3 | 3 2 1 0 | ..., so that consecutive MFMAs share an operand
                    // within a K half, also where the token block or the token half changes (where the K half or the K step
                    // changes, both operands do): operands that do not toggle cost no power, and under the power limit
                    // that is clock (us, 0 1 2 3 throughout -> this: Mixtral shape, 4096 tokens, 2061 -> 2036, 64 medium
                    // experts, 8192 tokens, 3772 -> 3732; the token blocks there and back under a fixed weight block: 2076
                    // against 2070 and 3833 against 3828 of this)
                    constexpr int a = ((g + kk * FMV) & 1) ? FA - 1 - m % FA : m % FA;
                    constexpr int t = th * FMV + b;  // 16-row token block
                    if constexpr (b < 8) {
                        constexpr int slot = FMV == 9 && t > 8 ? t - 1 : t;
                        if constexpr (FM >= 8) mfma_pinned_agpr(acc[a][slot], wr[BUF][q][a], xf[cur][b]);
                        else acc[a][slot] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wr[BUF][q][a], xf[cur][b], acc[a][slot], 0, 0, 0);
                    } else {
                        mfma_pinned_vgpr(accv[a][th == 0 ? 0 : NV - 1], wr[BUF][q][a], xf[cur][b]);
                    }
                    // first half of the slots: LDS reads of the next sub-step's token fragments, early
                    // enough that their latency is covered by the MFMAs of the second half
                    if constexpr (m < FMV) {
                        if constexpr (kk + 1 < KK) {
                            xf[nxt][m] = lds_read_b128<(thn * FMV + m) * BLK>(sbase + fx[qn]);
                        } else {
                            if (next) xf[nxt][m] = lds_read_b128<m * BLK>(nbase + fx[0]);
                        }
                    }
                    // the step's NL loads (weights of stage kt+PF first, then its tokens) are spread evenly
                    // over the MFMA slots of all sub-steps but the last: the four wavefronts run in lockstep, and
                    // bursts of back-to-back loads from all of them exceed what the compute unit's one vector-memory
                    // pipe takes per cycle.  (In the last steps, where they are conditional, those of a sub-step go
                    // together: one branch instead of one per load.)
                    if constexpr (kk < KK - 1) {
                        constexpr int S = (KK - 1) * NM, i_slot = kk * NM + m;
                        constexpr int s0 = STEADY ? i_slot : kk * NM, s1 = STEADY ? i_slot + 1 : (kk + 1) * NM;  // slots
                        if constexpr (STEADY || m == 0) {
                            constexpr int i0 = (s0 * NL + S - 1) / S, i1 = (s1 * NL + S - 1) / S;  // loads of these slots
                            constexpr int iw = i1 < WL ? i1 : WL, ix = i0 > WL ? i0 : WL;
                            if (more) {
                                static_for<(i0 < iw ? iw - i0 : 0)>([&](auto j) {
                                    load_w_one(kt + PF, std::integral_constant<int, BUFP>{}, std::integral_constant<int, i0 + j>{});
                                });
                                static_for<(ix < i1 ? i1 - ix : 0)>([&](auto j) { issue_x_one(xbase, BUFP, ix + j - WL); });
                            }
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                });
            });
        };
        // the steady steps NB at a time, then whatever is left (generic)
        int kt = 0;
        for (; kt + NB - 1 + PF < KT; kt += NB)
            static_for<NB>([&](auto i) { step(kt + i, i, std::true_type{}); });
        for (; kt < KT; kt += NB)
            static_for<NB>([&](auto i) {
                if (kt + i < KT) step(kt + i, i, std::false_type{});
            });

        // (the epilogue's addresses depend on nothing but the lane: computed ahead of the K loop, once for all heights,
        // they, or the lane itself, would be kept in registers through it)
        const int elane = fresh_lane();
        if constexpr (EPI == EPI_PLAIN || EPI == EPI_SWIGLU) {
            static_assert(SMEM >= NW * BM * TN * 2, "staged output");
            // every wavefront has issued and completed its last reads of the token ring
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            // (only the tall streaming kernels are compiled with stores of device scope: gemm_pick_hints)
            gemm_epilogue_staged<FT, FA, BM, TN, EPI, FMV == 9, W_STREAM && (BM > 128)>(acc, accv, td, Np, C, ldc, wave, elane, (char*)lds, device_scope);
        } else {
            gemm_epilogue<FT, FA, TN, EPI, FMV == 9>(acc, accv, td, Np, C, ldc, wave, elane);
        }
    };

    switch (fmv) {
#define CASE(n)                                                        \
    case n:                                                            \
        if constexpr (n <= FM) tile_of(std::integral_constant<int, (n <= FM ? n : 1)>{}); \
        break;
        CASE(1) CASE(2) CASE(3) CASE(4) CASE(5) CASE(6) CASE(7) CASE(8) CASE(9)
#undef CASE
        default: break;
    }
}

// ---- per-epilogue instantiation units ----------------------------------------------------------
// Classes 0 and 1 are the production token-tile classes of ordinary loads (row tiles of up to 128 rows for
// low loads, up to 288 rows otherwise), class 5 the one of decode-sized loads (see below); the other ids are
// alternatives kept for tuning runs (moe_set_tile_class).
// Class 5: two wavefronts per workgroup, 128 packed weight rows and up to 64 token rows per work item.  At a
// few rows per expert the kernel only streams weights, and what bounds it is the number of bytes a compute
// unit has in flight: a 4-wavefront workgroup with all its registers keeps 64 KB of weights under way and
// occupies the compute unit alone; these workgroups need under 256 registers per lane and 24 KB of LDS, four
// of them share a compute unit, together they keep 128 KB under way, and the weight panels are half as large,
// so a launch has twice as many workgroups for the device to place, four to a compute unit (Mixtral shape, 64
// tokens: 1792 instead of 896).
// A unit that defines MOE_GEMM_NO_TALL_TILE before including this file leaves out the 288-row class (its
// launcher then rejects class 1): the router-logit GEMM never uses it, and with that unit's epilogue the
// compiler copies the VGPR accumulators right behind their MFMAs (see mfma_pinned_vgpr).
//   V(id, BM, NW)
#ifdef MOE_GEMM_NO_TALL_TILE
#define FOR_EACH_VARIANT(V) \
    V(0, 128, 4)            \
    V(2, 64, 4)             \
    V(3, 32, 4)             \
    V(4, 256, 4)
static inline int variant_of_class(int cls) { return cls; }
#else
#define FOR_EACH_VARIANT(V) \
    V(0, 128, 4)            \
    V(1, 288, 4)            \
    V(2, 64, 4)             \
    V(3, 32, 4)             \
    V(5, 64, 2)
// The 256-row tuning class runs on the 288-row kernel, which takes tiles of any height up to its own (Mixtral shape, 4096
// tokens, class 4: 2206 us with a kernel of its own, 2174 with this one).  The 64- and 32-row classes keep theirs: two
// and three of their workgroups share a compute unit.
static inline int variant_of_class(int cls) { return cls == 4 ? 1 : cls; }
#endif

// Workgroup x takes the entries x, x + gridDim.x, ... of the work list.  Every class but the decode class is
// launched with one workgroup per entry: the hardware then hands the next entry to whichever compute unit is
// free, which balances tiles of unequal height (looping over a fixed share instead costs 3.5 % on the Mixtral
// shape at 1024 rows per expert and 13 % on ragged fine-grained loads).  The decode class has equal items
// that only stream weights; there a workgroup that stays resident saves the placement of a new one (about
// 5 us each): first expert GEMM of the Mixtral shape at 16 rows per expert, 1792 items on 1024 resident
// workgroups, 310 -> 298 us.  The barrier between two items keeps the next item's token loads out of the ring
// until every wavefront has read back its staged output.
template <int BM, int EPI, int NW, bool W_STREAM>
__global__ __launch_bounds__(NW * 64) void grouped_gemm_kernel(const uint16_t* __restrict__ X, int ldx,
                                                               const int32_t* __restrict__ row_map,
                                                               const uint16_t* __restrict__ Wf, int Np, int K,
                                                               uint16_t* __restrict__ C, int ldc,
                                                               const TileDesc* __restrict__ table,
                                                               size_t c_split_bytes, int n_entries, bool device_scope) {
    if constexpr (NW == 2) {
        for (int b = blockIdx.x; b < n_entries; b += gridDim.x) {
            gemm_tile<BM, EPI, NW, W_STREAM>(b, X, ldx, row_map, Wf, Np, K, C, ldc, table, c_split_bytes, device_scope);
            // LDS reads only: the output stores need not have completed (a full __syncthreads() would also
            // wait for them, and a workgroup that waits for its last stores holds its compute unit longer)
            if (b + (int)gridDim.x < n_entries) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        }
    } else {
        // no loop in the code of the other classes: the compiler would keep the lane-dependent values it can
        // hoist out of it in registers for the whole kernel, and the tall tiles have none to spare
        gemm_tile<BM, EPI, NW, W_STREAM>(blockIdx.x, X, ldx, row_map, Wf, Np, K, C, ldc, table, c_split_bytes, device_scope);
    }
}

template <int BM, int EPI, int NW, bool WS>
struct Variant {
    static constexpr size_t smem = gemm_lds_bytes(BM, NW);
    static hipError_t set_attr() {
        return hipFuncSetAttribute((const void*)grouped_gemm_kernel<BM, EPI, NW, WS>,
                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    }
    // K is the reduction length of ONE split; nsplit = 1 for the expert GEMMs
    static hipError_t launch(int grid, const uint16_t* X, int ldx, const int32_t* row_map, const uint16_t* Wf,
                             int Np, int K, uint16_t* C, int ldc, const TileDesc* table, int nsplit,
                             size_t c_split_bytes, hipStream_t st, bool device_scope) {
        constexpr int RESIDENT = 256 * 4;  // decode class: four workgroups fit a compute unit
        const int gx = (NW == 2 && grid > RESIDENT) ? RESIDENT : grid;
        hipLaunchKernelGGL((grouped_gemm_kernel<BM, EPI, NW, WS>), dim3(gx, nsplit), dim3(NW * 64), smem, st,
                           X, ldx, row_map, Wf, Np, K, C, ldc, table, c_split_bytes, grid, device_scope);
        return hipGetLastError();
    }
};

template <int EPI, bool WS>
static hipError_t gemm_set_attr_all() {
    hipError_t err;
#define V(id, bm, nw)                               \
    err = Variant<bm, EPI, nw, WS>::set_attr();     \
    if (err != hipSuccess) return err;
    FOR_EACH_VARIANT(V)
#undef V
    return hipSuccess;
}

template <int EPI, bool WS>
static hipError_t gemm_launch_any(int cls, int grid, const uint16_t* X, int ldx, const int32_t* row_map,
                                  const uint16_t* Wf, int Np, int K, uint16_t* C, int ldc, const TileDesc* table,
                                  int nsplit, size_t c_split_bytes, hipStream_t st, bool device_scope) {
    switch (variant_of_class(cls)) {
#define V(id, bm, nw)                                                                                     \
    case id:                                                                                                  \
        return Variant<bm, EPI, nw, WS>::launch(grid, X, ldx, row_map, Wf, Np, K, C, ldc, table, nsplit,  \
                                                    c_split_bytes, st, device_scope);
        FOR_EACH_VARIANT(V)
#undef V
    }
    return hipErrorInvalidValue;
}

// Defines gemm_set_attr_<name>() and gemm_launch_<name>(cls, ...) for one epilogue and one kind of weight load;
// each is compiled in a translation unit of its own so that the units build in parallel.
#define MOE_GEMM_INSTANTIATE(name, EPI, WS)                                                                   \
    hipError_t gemm_set_attr_##name() { return gemm_set_attr_all<EPI, WS>(); }                                \
    hipError_t gemm_launch_##name(int cls, int grid, const uint16_t* X, int ldx, const int32_t* row_map,      \
                                  const uint16_t* Wf, int Np, int K, uint16_t* C, int ldc,                    \
                                  const TileDesc* table, int nsplit, size_t c_split_bytes, hipStream_t st,    \
                                   bool device_scope) {                                                       \
        return gemm_launch_any<EPI, WS>(cls, grid, X, ldx, row_map, Wf, Np, K, C, ldc, table, nsplit,         \
                                        c_split_bytes, st, device_scope);                                     \
    }
