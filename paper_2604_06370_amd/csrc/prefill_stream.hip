// ResidualAttention chunked prefill for gfx950, pipelined kernel (Section 6 prefill kernel,
// Algorithm 1 with a block of query rows).
//
// One workgroup = (agent a, KV head h, block of 32 NW query rows); its rows are (query token,
// query head of h), 32 per wave, all of the same agent.  64-key tiles (four pages) of the agent's
// keys stream through LDS rings.  All products are 32x32x16 (scores transposed, S^T = K Q^T, so
// that a lane owns one query row and the weights feed the value products without a shuffle):
//   RoPE on, per tile: U^T = B_K^T C_K^T, K_lora = RoPE_p(U) (rotate-half, fp32),
//                      K = K_base + K_lora -> bf16, in place in LDS
//   per wave:          S^T = K Q^T,  RoPE off: S^T += C_K (B_K q)^T
//                      causal mask + online softmax
//                      O^T += V^T P^T,  acc_r^T += C_V^T P^T
// and at the end O = (O + acc_r . B_V[h]) / l (Eq. 4) is written in bf16.
//
// What bounds it, and the forms that follow from it (16 agents x 2048 rows over 32K, 8B heads,
// rank 16, unless another size is named; the matrix cores are busy 48 % of the launch at 1.94 GHz,
// 66 % at 1.64 GHz without RoPE, 20.1 ms, where power holds the clock; the kernel before: 41 %, 27.7 ms):
//  - One iteration works on three tiles: value products of tile t - 1 beside the row maxima of tile
//    t, then scores of tile t + 1 beside the weights of tile t, so that a wave always has matrix
//    and vector work that do not wait for each other; one barrier per tile.  The order is written
//    out product by product (fences for the compiler's scheduler): left to the scheduler each
//    product waited for its own LDS read (28.0 instead of 23.8 ms).
//  - 32x32x16 products: half the instructions of 16x16x32 at the same rate, and in a loop of one
//    product, three vector and two exponential instructions two waves per SIMD take 38 cycles
//    per 32x32x16 product against 48 for two 16x16x32.
//  - LDS bandwidth is the second bound (every wave reads the whole tile: 256 KB per tile and
//    workgroup of eight waves): output rows are ordered so that the value reads have no bank
//    conflict (row r = dim 16 (r % 2) + r / 2: 26.5 -> 23.8 ms; 4 agents x 250 rows 1155 -> 934 us).
//  - Copies into LDS are instructions that the compiler does not know (it would wait for all of
//    them before every LDS read), waited for by count two or three iterations later: 4 agents x 250
//    rows 831 us two ahead, 701 three ahead, 632 with the copies beside the first value products.
//  - RoPE on with eight waves: waves 0 .. 3 (one per SIMD) rebuild their keys at the start of an
//    iteration and waves 4 .. 7 at its end (the registers leave no room beside the products).
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <cmath>
#include <type_traits>

#include "lds_dma.hpp"
#include "mfma.hpp"
#include "prefill.hpp"

using namespace fkvk;

namespace fkvp {
namespace {

constexpr int D = 128;
constexpr int PS = 16;
constexpr int TILE_KEYS = 64;              // four pages
constexpr float kNegInf = -INFINITY;

constexpr float kLazyRescale = 8.f;

// LDS layout and copy distances.  At iteration t the K side (K block, rCache page, table rows) of
// tile t + KR and the V side of tile t + VR - 2 are requested; in use are V of tile t - 1, the keys
// of t + 1 and (RoPE on) of t + 2, the tile being rebuilt.  C_K and C_V share one ring up to rank
// 16; above, where the pages are larger, the V side copies the rCache page again into a shorter
// ring of its own.
template <int R, bool ROPE>
struct Ring {
    static_assert(!(ROPE && R >= 64), "rank 64 with RoPE runs on the rebuild kernel");
    static constexpr int RT = R == 0 ? 0 : (R + 15) / 16;
    static constexpr int NRB = (RT + 1) / 2;             // 32-row blocks of the rank accumulator
    static constexpr bool CSPLIT = R >= 32;
    static constexpr int KR = ROPE || R <= 16 ? 4 : 3;
    static constexpr int VR = (ROPE ? R >= 32 : R >= 64) ? 2 : (!ROPE && R <= 16 ? 4 : 3);
    static constexpr int KAHEAD = ROPE ? KR - 2 : KR - 1, VAHEAD = VR - 1;  // iterations from request to use
    static constexpr int CPAGE = RT * 1024;
    static constexpr int CKR = CSPLIT ? (ROPE ? KR - 1 : KR) : KR + 2;
    static constexpr int CVR = CSPLIT ? VR : 0;
    static constexpr int TR = ROPE ? KR - 1 : 0;
    static constexpr int K_OFF = 0;
    static constexpr int V_OFF = K_OFF + KR * 16384;
    static constexpr int CK_OFF = V_OFF + VR * 16384;
    static constexpr int CV_OFF = CK_OFF + CKR * 4 * CPAGE;
    static constexpr int T_OFF = CV_OFF + CVR * 4 * CPAGE;
    static constexpr int COL_OFF = T_OFF + TR * 4096;
    static constexpr int ONES_OFF = COL_OFF + (ROPE ? 8192 : 0);
    static constexpr int ONES_BYTES = RT == 1 ? 4096 : 0;
    static constexpr int MAIN_BYTES = ONES_OFF + ONES_BYTES;
    static constexpr int NK = 4 + RT + (ROPE ? 1 : 0);   // copies of a wave per tile: K side
    static constexpr int NV = 4 + (CSPLIT ? RT : 0);     // V side
};

__device__ __forceinline__ u32x2 lds_ld64(uint32_t a) {
    return *reinterpret_cast<const __attribute__((address_space(3))) u32x2 *>((uintptr_t)a);
}
__device__ __forceinline__ void lds_st128(uint32_t a, const u32x4 &v) {
    *reinterpret_cast<__attribute__((address_space(3))) u32x4 *>((uintptr_t)a) = v;
}
__device__ __forceinline__ void lds_st64(uint32_t a, const u32x2 &v) {
    *reinterpret_cast<__attribute__((address_space(3))) u32x2 *>((uintptr_t)a) = v;
}
// An LDS address the compiler takes as it is: the reads at constant distances from it then use
// the instructions' immediate offsets (one address register instead of one per read).
__device__ __forceinline__ uint32_t opaque(uint32_t a) {
    asm("" : "+v"(a));
    return a;
}
// Copy of 1 KB, I KB from `base`, to LDS address dst + I KB (both wave-uniform; the instruction's
// offset moves the source and the destination alike): lane i's 16 bytes at voff = 16 i.  Written as
// an instruction because the compiler waits for every copy it knows of before any later LDS read;
// the waits here are the counted ones of the hand-over.
// The source goes through a scalar move inside the instruction group: a vector-memory instruction may
// not read a scalar register within five states of the vector instruction that wrote it (readfirstlane,
// readlane), which the compiler does not check for operands of its own making here.  The move is also the
// state that has to pass between the write of m0 and its use.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"  // m0 is named although the compiler does not allocate it
template <int I>
__device__ __forceinline__ void dma_kb(uint64_t base, uint32_t dst, uint32_t voff) {
    base = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)base) |
           (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(base >> 32)) << 32;
    dst = (uint32_t)__builtin_amdgcn_readfirstlane((int)dst);
    uint64_t src;
    asm volatile("s_mov_b32 m0, %1\n\ts_mov_b64 %0, %3\n\tglobal_load_lds_dwordx4 %2, %0 offset:%4"
                 : "=&s"(src) : "s"(dst), "v"(voff), "s"(base), "n"(I * 1024) : "memory", "m0");
}
// Copy of 64 x 16 bytes, lane i's from its own address, to dst + 16 i.
__device__ __forceinline__ void dma_1kb_at(uint64_t addr, uint32_t dst) {
    dst = (uint32_t)__builtin_amdgcn_readfirstlane((int)dst);
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(dst), "v"(addr) : "memory", "m0");
}
#pragma clang diagnostic pop

template <int R, int G, bool ROPE, int NW>
__device__ __forceinline__ void prefill_block(const PrefillArgs &p, unsigned char *lds, int a, int h, int tok_begin) {
    using S = Ring<R, ROPE>;
    constexpr int RT = S::RT, RTX = RT > 0 ? RT : 1, NRB = S::NRB, NRBX = NRB > 0 ? NRB : 1;
    constexpr int ROWS = NW * 32;
    constexpr int TPW = ROWS / G;
    constexpr bool LROW = RT == 1;  // the row sums come from a ones row beside the ranks
    const int lane = threadIdx.x & 63;
    const int wave = uniform(threadIdx.x >> 6);
    const int col = lane & 15, grp = lane >> 4, up = (lane >> 4) & 1, hh = lane >> 5, r32 = lane & 31;
    const int hkv = p.hkv;
    const int64_t n = (int64_t)hkv * D;
    const int q0 = p.q_indptr[a], nq = p.q_indptr[a + 1] - q0;
    const int L = p.seq_lens[a];
    const int P0 = L - nq;
    const int ad = R > 0 ? p.adapter_idx[a] : -1;
    const int n_pages = (L + PS - 1) / PS;
    const int last_pos = P0 + (tok_begin + TPW < nq ? tok_begin + TPW : nq) - 1;
    const int n_tiles = last_pos / TILE_KEYS + 1;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)lds;

    // ---- copies: four waves copy page w of every tile; eight waves: waves 0..3 its K side, 4..7 its V side ----
    const int pw = wave & 3;
    const bool kwave = NW == 4 || wave < 4, vwave = NW == 4 || wave >= 4;
    const uint32_t voff = lane * 16;
    auto page_of = [&](int tile) __attribute__((always_inline)) { return min(4 * tile + pw, n_pages - 1); };
    auto kbase = [&](int id) __attribute__((always_inline)) -> uint64_t {
        return reinterpret_cast<uint64_t>(p.base_kv + ((int64_t)id * 2 * hkv + h) * (PS * D));
    };
    auto cbase = [&](int id) __attribute__((always_inline)) -> uint64_t {
        return reinterpret_cast<uint64_t>(p.res_kv + (int64_t)id * (RT * 512));
    };
    // RoPE on: lanes 0..15 copy the 16-byte pieces of the page's first cos row, lanes 16..31 of its
    // sin row (lanes 32..63 repeat them)
    const uint64_t tab_lane = ROPE ? reinterpret_cast<uint64_t>(up ? p.rope_sin : p.rope_cos) + (col >> 2) * 1024 + (col & 3) * 256 : 0;
    // One wave's copies of a tile, in parts of 1 KB: the K side (K block, rCache page, table rows) has
    // NK parts, the V side (V block, and the rCache page again where C_V has a ring of its own) NV.
    struct Side {
        uint64_t blk, res, tab;
        uint32_t blk_dst, res_dst, tab_dst;
    };
    auto k_side = [&](int tile, int idb, int idr) __attribute__((always_inline)) {
        Side c;
        c.blk = kbase(idb);
        c.blk_dst = lds0 + S::K_OFF + (tile % S::KR) * 16384 + pw * 4096;
        if constexpr (R > 0) {
            c.res = cbase(idr);
            c.res_dst = lds0 + S::CK_OFF + (tile % S::CKR) * (4 * S::CPAGE) + pw * S::CPAGE;
        }
        if constexpr (ROPE) {
            c.tab = tab_lane + (uint64_t)page_of(tile) * 4096;
            c.tab_dst = lds0 + S::T_OFF + (tile % (ROPE ? S::TR : 1)) * 4096 + pw * 1024;
        }
        return c;
    };
    auto v_side = [&](int tile, int idb, int idr) __attribute__((always_inline)) {
        Side c;
        c.blk = kbase(idb) + (uint64_t)hkv * 4096;
        c.blk_dst = lds0 + S::V_OFF + (tile % S::VR) * 16384 + pw * 4096;
        if constexpr (S::CSPLIT) {
            c.res = cbase(idr);
            c.res_dst = lds0 + S::CV_OFF + (tile % (S::CSPLIT ? S::CVR : 1)) * (4 * S::CPAGE) + pw * S::CPAGE;
        }
        return c;
    };
    auto copy_part = [&](const Side &c, int i, bool kside) __attribute__((always_inline)) {
        if (i == 0) dma_kb<0>(c.blk, c.blk_dst, voff);
        if (i == 1) dma_kb<1>(c.blk, c.blk_dst, voff);
        if (i == 2) dma_kb<2>(c.blk, c.blk_dst, voff);
        if (i == 3) dma_kb<3>(c.blk, c.blk_dst, voff);
        if (i == 4 && RT > 0) dma_kb<0>(c.res, c.res_dst, voff);
        if (i == 5 && RT > 1) dma_kb<1>(c.res, c.res_dst, voff);
        if (i == 6 && RT > 2) dma_kb<2>(c.res, c.res_dst, voff);
        if (i == 7 && RT > 2) dma_kb<3>(c.res, c.res_dst, voff);
        if (ROPE && kside && i == 4 + RT) dma_1kb_at(c.tab, c.tab_dst);
    };

    // Page ids of page pw of 64 tiles per register (lane i: tile 64 c + i; pages past the sequence
    // repeat its last page, so every copy reads a real page; their keys are masked).  Eight waves:
    // the K (V) waves copy tile t + KR (t + VR - 2) at iteration t; four waves: base ids of the V
    // side are those of the K side KR - VR + 2 iterations before.
    constexpr int LAG = S::KR - S::VR + 2;
    auto chunk_ids = [&](int c, int &idb, int &idr) __attribute__((always_inline)) {
        const int pg = min((64 * c + lane) * 4 + pw, n_pages - 1);
        idb = p.base_bt[(int64_t)a * p.max_pages + pg];
        idr = R > 0 ? p.res_bt[(int64_t)a * p.max_pages + pg] : 0;
    };
    int idb_cur, idr_cur, idb_nxt, idr_nxt;
    chunk_ids(0, idb_cur, idr_cur);
    chunk_ids(1, idb_nxt, idr_nxt);
    int vb[LAG] = {}, vr[LAG] = {};  // four waves: ids of the tiles between the two sides
    // Copies of iteration t: the K side of tile t + KR, the V side of tile t + VR - 2.
    struct Copies {
        Side k, v;
    };
    constexpr int NPARTS = NW == 4 ? S::NK + S::NV : (S::NK > S::NV ? S::NK : S::NV);
    auto copies_of = [&](int t) __attribute__((always_inline)) {
        const int tn = NW == 4 || kwave ? t + S::KR : t + S::VR - 2;
        if (tn > 0 && (tn & 63) == 0) {
            idb_cur = idb_nxt;
            idr_cur = idr_nxt;
            chunk_ids((tn >> 6) + 1, idb_nxt, idr_nxt);
        }
        const int idb = __builtin_amdgcn_readlane(idb_cur, tn & 63), idr = R > 0 ? __builtin_amdgcn_readlane(idr_cur, tn & 63) : 0;
        Copies c;
        if constexpr (NW == 4) {
            c.v = v_side(t + S::VR - 2, vb[0], vr[0]);
            c.k = k_side(t + S::KR, idb, idr);
#pragma unroll
            for (int i = 0; i + 1 < LAG; ++i) {
                vb[i] = vb[i + 1];
                vr[i] = vr[i + 1];
            }
            vb[LAG - 1] = idb;
            vr[LAG - 1] = idr;
        } else {
            if (kwave) c.k = k_side(tn, idb, idr);
            else c.k = v_side(tn, idb, idr);
        }
        return c;
    };
    // part i of them: four waves issue the V side first (the waits count on it)
    auto copy_step = [&](const Copies &c, int i) __attribute__((always_inline)) {
        if constexpr (NW == 4) {
            if (i < S::NV) copy_part(c.v, i, false);
            else if (i < S::NV + S::NK) copy_part(c.k, i - S::NV, true);
        } else {
            if (i < (S::NK < S::NV ? S::NK : S::NV) && i < 4) copy_part(c.k, i, false);
            else if (i < S::NK || i < S::NV) {
                if (kwave) {
                    if (i < S::NK) copy_part(c.k, i, true);
                } else {
                    if (i < S::NV) copy_part(c.k, i, false);
                }
            }
        }
    };
    auto copies = [&](int t, bool do_k, bool do_v) __attribute__((always_inline)) {
        const Copies c = copies_of(t);
        if constexpr (NW == 4) {
#pragma unroll
            for (int i = 0; i < NPARTS; ++i)
                if (i < S::NV ? do_v : do_k) copy_step(c, i);
        } else if (kwave ? do_k : do_v) {
#pragma unroll
            for (int i = 0; i < NPARTS; ++i) copy_step(c, i);
        }
    };
    // K side of tiles 0 .. KR - 2 and V side of tile 0 (three V buffers); tile KR - 1 follows below
#pragma unroll
    for (int t = -S::KR; t < -1; ++t) copies(t, true, t + S::VR - 2 >= 0);  // (V: tiles 0 .. VR - 4)

    // ---- queries (B operand: lane = row, dims 32kk + 4g + 0..3 and 32kk + 16 + 4g + 0..3, g = 2gp + hh) ----
    const int tok = tok_begin + (wave * 32 + r32) / G;
    const bool row_ok = tok < nq;
    const int row_pos = P0 + tok;
    u32x4 qf[8];
    {
        const uint16_t *qr = p.q + ((int64_t)(q0 + (row_ok ? tok : 0)) * p.hq + h * G + r32 % G) * D;
#pragma unroll
        for (int st = 0; st < 8; ++st) {
            const int dm = 32 * (st / 2) + 4 * (2 * (st % 2) + hh);
            u32x4 v = {0, 0, 0, 0};
            if (row_ok) {
                const u32x2 lo = ldg64(qr + dm), hi = ldg64(qr + dm + 16);
                v = u32x4{lo.x, lo.y, hi.x, hi.y};
            }
            qf[st] = v;
        }
    }
    // RoPE off: W^T = (B_K q)^T
    u32x4 wq[RTX];
    if constexpr (R > 0 && !ROPE) {
        const uint16_t *bk = p.lora_b + (int64_t)ad * 2 * R * n + (int64_t)h * D;
#pragma unroll
        for (int b = 0; b < NRB; ++b) {
            f32x16 acc = f32x16{};
            const int rho = 32 * b + r32;
#pragma unroll
            for (int st = 0; st < 8; ++st) {
                const int dm = 32 * (st / 2) + 4 * (2 * (st % 2) + hh);
                u32x4 av = {0, 0, 0, 0};
                if (rho < R) {
                    const u32x2 lo = ldg64(bk + (int64_t)rho * n + dm), hi = ldg64(bk + (int64_t)rho * n + dm + 16);
                    av = u32x4{lo.x, lo.y, hi.x, hi.y};
                }
                acc = mfma32x32(av, qf[st], acc);
            }
#pragma unroll
            for (int k = 0; k < 2; ++k)
                if (2 * b + k < RT) wq[2 * b + k] = pack8(acc, 8 * k);
        }
    }
    // RoPE on: a wave rebuilds dims 32 half .. +31 and their partners 64 further of page pw (eight
    // waves: half = wave / 4; four: both halves).  B_K^T operands of its four (eight) 16-dim tiles:
    // lane holds B_K[16k + 4grp + 0..3][dim 16m + col].
    constexpr int NH = NW == 4 ? 2 : 1;
    const int half0 = NW == 4 ? 0 : wave >> 2;
    u32x2 bkf[NH][4][RTX];
    if constexpr (ROPE) {
        const uint16_t *bk = p.lora_b + (int64_t)ad * 2 * R * n + (int64_t)h * D;
#pragma unroll
        for (int e = 0; e < NH; ++e)
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int k = 0; k < RT; ++k) {
                    const int dim = 32 * (half0 + e) + 16 * (j & 1) + 64 * (j >> 1) + col;
                    uint32_t w[2];
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        const int r0 = 16 * k + 4 * grp + 2 * i;
                        const uint16_t lo = r0 < R ? bk[(int64_t)r0 * n + dim] : (uint16_t)0;
                        const uint16_t hi = r0 + 1 < R ? bk[(int64_t)(r0 + 1) * n + dim] : (uint16_t)0;
                        w[i] = (uint32_t)lo | ((uint32_t)hi << 16);
                    }
                    bkf[e][j][k] = u32x2{w[0], w[1]};
                }
        // cos then sin of positions 0..15 in the table's own order
        for (int i = threadIdx.x; i < 512; i += 64 * NW)
            lds_st128(lds0 + S::COL_OFF + i * 16, ldg128((i < 256 ? p.rope_cos : p.rope_sin - 1024) + 4 * i));
    }
    if (S::ONES_BYTES > 0 && (NW == 4 || wave < 4)) lds_st128(lds0 + S::ONES_OFF + threadIdx.x * 16, u32x4{0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u});

    // ---- lane parts of the LDS addresses ----
    const uint32_t laneK = up * 4096 + hh * 256 + col * 16;
    const uint32_t laneC = up * S::CPAGE + hh * 256 + col * 16;
    // Row r of a 32-row block of the transposed outputs is dim (rank) 16 (r % 2) + r / 2 of the block:
    // a lane group then reads consecutive 8-byte pieces of the stored chunks (dims c and 16 + c of a
    // chunk are neighbours); rows r = c, 16 apart, would read every other piece, a two-way conflict
    const uint32_t laneV = r32 * 8 + hh * 256;
    const uint32_t laneCV = (RT > 1 ? (r32 & 1) * 1024 : 0) + hh * 256 + (r32 >> 1) * 16 + 8;

    f32x16 oacc[4], racc[NRBX];
#pragma unroll
    for (int i = 0; i < 4; ++i) oacc[i] = f32x16{};
#pragma unroll
    for (int i = 0; i < NRBX; ++i) racc[i] = f32x16{};
    float m_run = kNegInf, lsum = 0.f;
    const float cl = p.scale_log2;
    u32x4 pf[4];  // weights of a tile (B operand of the value products, one page each)

    auto fence = []() __attribute__((always_inline)) { __builtin_amdgcn_sched_barrier(0); };

    // Scores of one tile: NS products, their A operands read PRE ahead.  Operand i: of key block
    // i / (8 + RC), K dim step i % (8 + RC), then (RoPE off) C_K of the RC rank tiles.
    constexpr int PRE = NW == 4 ? 8 : 4;
    constexpr int RC = ROPE ? 0 : RT, NS = 2 * (8 + RC);
    struct ScoreAddr {
        uint32_t k, c;
    };
    auto score_addr = [&](int tile) __attribute__((always_inline)) {
        return ScoreAddr{opaque(lds0 + S::K_OFF + (tile % S::KR) * 16384 + laneK),
                         RC > 0 ? opaque(lds0 + S::CK_OFF + (tile % S::CKR) * (4 * S::CPAGE) + laneC) : 0u};
    };
    auto score_frag = [&](const ScoreAddr &at, int i) __attribute__((always_inline)) -> u32x4 {
        const int kb = i / (8 + RC), st = i % (8 + RC);
        if (st < 8) return lds_load(at.k + kb * 8192 + (st / 2) * 1024 + (st % 2) * 512);
        const uint32_t ca = at.c + kb * 2 * S::CPAGE + (st - 8) * 1024;
        const u32x2 c0 = lds_ld64(ca), c1 = R == 8 ? u32x2{0, 0} : lds_ld64(ca + 512);
        return u32x4{c0.x, c0.y, c1.x, c1.y};
    };
    auto score_product = [&](const u32x4 &f, int i, f32x16 (&s)[2]) __attribute__((always_inline)) {
        const int kb = i / (8 + RC), st = i % (8 + RC);
        s[kb] = mfma32x32(f, st < 8 ? qf[st < 8 ? st : 0] : wq[st < 8 ? 0 : st - 8], st == 0 ? f32x16{} : s[kb]);
    };

    // Keys of one tile, this wave's part, in RB steps that region 1 spreads over its products (the
    // cos / sin pieces of two frequencies at a time, so that a step's registers stay few).
    struct Rebuild {
        uint32_t ks, ts, os;
        u32x2 c[RTX];
        u32x4 klo, khi;  // quarters half and half + 2 of the K block: base keys, then the rebuilt ones
        f32x4 u[4];      // tiles 2 half, 2 half + 1, 2 half + 4, 2 half + 5
        f32x2 c0, s0, ct, st, x, y;
    };
    constexpr int RB = 17;
    // Four waves (up to 512 registers) spread them over the value products.  Eight waves (256
    // registers) have no room for that: waves 0 .. 3, one per SIMD, rebuild at the start of an
    // iteration and waves 4 .. 7 at its end, each beside the other wave's products.
    constexpr bool BESIDE = NW == 4;
    auto rebuild_step = [&](Rebuild &b, int e, int tile, int step) __attribute__((always_inline)) {
        if constexpr (ROPE) {
            const int half = half0 + e;
            auto angles = [&](int q) __attribute__((always_inline)) {  // frequencies 2 (q % 2), + 1 of tile q / 2
                const uint32_t o = (q / 2) * 64 + (q % 2) * 8, oo = (q / 2) * 1024 + (q % 2) * 8;
                b.c0 = __builtin_bit_cast(f32x2, lds_ld64(b.ts + o));
                b.s0 = __builtin_bit_cast(f32x2, lds_ld64(b.ts + o + 256));
                b.ct = __builtin_bit_cast(f32x2, lds_ld64(b.os + oo));
                b.st = __builtin_bit_cast(f32x2, lds_ld64(b.os + oo + 4096));
            };
            if (step == 0) {
                b.ks = opaque(lds0 + S::K_OFF + (tile % S::KR) * 16384 + pw * 4096 + half * 1024 + lane * 16);
                const uint32_t cs = opaque(lds0 + S::CK_OFF + (tile % S::CKR) * (4 * S::CPAGE) + pw * S::CPAGE + lane * 16);
                b.ts = opaque(lds0 + S::T_OFF + (tile % (ROPE ? S::TR : 1)) * 4096 + pw * 1024 + half * 128 + grp * 16);
                b.os = opaque(lds0 + S::COL_OFF + half * 2048 + lane * 16);
#pragma unroll
                for (int k = 0; k < RT; ++k) {
                    b.c[k] = lds_ld64(cs + k * 1024);
                    if constexpr (R == 8) b.c[k] = grp < 2 ? b.c[k] : u32x2{0, 0};
                }
            } else if (step == 2) {
#pragma unroll
                for (int k = 0; k < RT; ++k)
#pragma unroll
                    for (int j = 0; j < 4; ++j) b.u[j] = mfma16(bkf[e][j][k], b.c[k], k == 0 ? f32x4{0, 0, 0, 0} : b.u[j]);
            } else if (step == 3) {
                angles(0);
                b.klo = lds_load(b.ks);
                b.khi = lds_load(b.ks + 2048);
            } else if (step >= 5 && step % 3 != 1 && step < 16) {
                // steps 5 + 3q, 6 + 3q: rotate-half pairs (tile m with m + 4) at the key's position p0 + col:
                // the angle of the page start p0 plus the angle of offset col (angle addition), added to K_base
                const int q = (step - 5) / 3, i = (step - 5) % 3, j = q / 2, w = 2 * j + q % 2;
                const float c = b.c0[i] * b.ct[i] - b.s0[i] * b.st[i];
                const float s = b.s0[i] * b.ct[i] + b.c0[i] * b.st[i];
                const float ux = b.u[j][2 * (q % 2) + i], uy = b.u[j + 2][2 * (q % 2) + i];
                b.x[i] = __builtin_fmaf(ux, c, __builtin_fmaf(-uy, s, i ? bf16_hi(b.klo[w]) : bf16_lo(b.klo[w])));
                b.y[i] = __builtin_fmaf(uy, c, __builtin_fmaf(ux, s, i ? bf16_hi(b.khi[w]) : bf16_lo(b.khi[w])));
                if (i == 1) {
                    b.klo[w] = pack_bf16(b.x[0], b.x[1]);
                    b.khi[w] = pack_bf16(b.y[0], b.y[1]);
                    if (q < 3) angles(q + 1);
                }
            } else if (step == 16) {
                lds_st128(b.ks, b.klo);
                lds_st128(b.ks + 2048, b.khi);
            }
        }
    };
    auto rebuild = [&](int tile) __attribute__((always_inline)) {
        if constexpr (ROPE) {
#pragma unroll
            for (int e = 0; e < NH; ++e) {
                Rebuild b;
#pragma unroll
                for (int i = 0; i < RB; ++i) rebuild_step(b, e, tile, i);
            }
        }
    };

    // Values of one tile: NP products (per page four 32-dim blocks and NRB rank blocks), their A
    // operands read PRE ahead; `beside(i)` runs after product i.  RAGGED: tokens past the sequence
    // (whose bits may be anything) are zeroed.
    constexpr int NPP = 4 + NRB, NP = 4 * NPP;
    auto values = [&](auto ragged_tag, int tile, auto &&beside) __attribute__((always_inline)) {
        constexpr bool RAGGED = decltype(ragged_tag)::value;
        const uint32_t vs = opaque(lds0 + S::V_OFF + (tile % S::VR) * 16384 + laneV);
        uint32_t cs = (S::CSPLIT ? lds0 + S::CV_OFF + (tile % (S::CSPLIT ? S::CVR : 1)) * (4 * S::CPAGE)
                                 : lds0 + S::CK_OFF + (tile % S::CKR) * (4 * S::CPAGE)) + laneCV;
        if constexpr (LROW) cs = r32 == 1 ? lds0 + S::ONES_OFF : cs;
        if constexpr (R > 0) cs = opaque(cs);
        auto frag = [&](int i) __attribute__((always_inline)) {
            const int pg = i / NPP, b = i % NPP;
            const uint32_t at = b < 4 ? vs + pg * 4096 + b * 1024 : cs + pg * S::CPAGE + (b - 4) * 2048;
            // tokens 4hh + 0..3 and 8 + 4hh + 0..3
            u32x2 v0 = lds_ld64(at), v1 = lds_ld64(at + 512);
            if constexpr (RAGGED) {
                const int vis = L - (tile * 4 + pg) * PS;
                v0 = mask4(v0, vis, hh);
                v1 = mask4(v1, vis - 8, hh);
            }
            return u32x4{v0.x, v0.y, v1.x, v1.y};
        };
        u32x4 f[PRE];
#pragma unroll
        for (int i = 0; i < PRE; ++i) f[i] = frag(i);
        beside(-1);
        fence();
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const int b = i % NPP;
            if (b < 4) oacc[b < 4 ? b : 0] = mfma32x32(f[i % PRE], pf[i / NPP], oacc[b < 4 ? b : 0]);
            else racc[b < 4 ? 0 : b - 4] = mfma32x32(f[i % PRE], pf[i / NPP], racc[b < 4 ? 0 : b - 4]);
            if (i + PRE < NP) f[i % PRE] = frag(i + PRE);
            beside(i);
            fence();
        }
    };
    // every wave's copies older than the last iteration's have landed, LDS accesses are complete
    auto hand_over = [&]() __attribute__((always_inline)) {
        if constexpr (NW == 4) {
            constexpr int A = S::KAHEAD < S::VAHEAD ? S::KAHEAD : S::VAHEAD;
            wait_vmcnt<(A - 1) * (S::NK + S::NV) + (S::KAHEAD > S::VAHEAD ? S::NK : 0)>();
        } else {
            if (kwave) wait_vmcnt<(S::KAHEAD - 1) * S::NK>();
            else wait_vmcnt<(S::VAHEAD - 1) * S::NV>();
        }
        lds_fence_barrier();
    };
    // One iteration: region 1, value products of tile t - 1 beside the row maxima of tile t and the
    // keys of tile t + 2; region 2, scores of tile t + 1 beside the weights of tile t.
    auto body = [&](auto pv_tag, auto mask_tag, int t, f32x16 (&s)[2], f32x16 (&snext)[2]) __attribute__((always_inline)) {
        constexpr bool DO_PV = decltype(pv_tag)::value, MASK = decltype(mask_tag)::value;
        hand_over();
        const Copies cp = copies_of(t);
        if constexpr (MASK) {
            const int lim = row_ok ? row_pos - t * TILE_KEYS - 4 * hh : -1;
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    s[kb][i] = 32 * kb + 8 * (i / 4) + i % 4 <= lim ? s[kb][i] : kNegInf;
        }
        if constexpr (ROPE && !BESIDE) {
            if (wave < 4) rebuild(t + 2);
        }
        fence();
        float mx0 = kNegInf, mx1 = kNegInf;
        auto max_step = [&](int i) __attribute__((always_inline)) {  // 8 steps of four values
            mx0 = fmaxf(fmaxf(mx0, s[i / 4][4 * (i % 4)]), s[i / 4][4 * (i % 4) + 1]);
            mx1 = fmaxf(fmaxf(mx1, s[i / 4][4 * (i % 4) + 2]), s[i / 4][4 * (i % 4) + 3]);
        };
        Rebuild rb[NH];
        ScoreAddr sat;
        u32x4 kp[PRE];
        auto beside = [&](int i) __attribute__((always_inline)) {
            if (i == -1) {
                if constexpr (BESIDE) {
#pragma unroll
                    for (int e = 0; e < NH; ++e) rebuild_step(rb[e], e, t + 2, 0);
                }
#pragma unroll
                for (int k = 0; k < 4; ++k) max_step(k);
            } else if (i < 2) {
                max_step(4 + 2 * i);
                max_step(5 + 2 * i);
            } else if (BESIDE && i < RB) {
#pragma unroll
                for (int e = 0; e < NH; ++e) rebuild_step(rb[e], e, t + 2, i);
            }
            // the copies, one or two beside each of the first products
            if (i >= 0 && i < 12) {
#pragma unroll
                for (int j = NPARTS * i / 12; j < NPARTS * (i + 1) / 12; ++j) copy_step(cp, j);
            }
            if (i == NP - PRE) sat = score_addr(t + 1);
            // (the K reads go before the rebuilt keys are stored: another buffer)
            if (i >= NP - PRE) kp[i >= NP - PRE ? i - (NP - PRE) : 0] = score_frag(sat, i - (NP - PRE));
        };
        if constexpr (DO_PV) {
            values(std::false_type{}, t - 1, beside);
        } else {
#pragma unroll
            for (int i = -1; i < NP; ++i) beside(i);
        }
        const float mx = max_over_halves(fmaxf(mx0, mx1)) * cl;
        fence();
        if (__builtin_amdgcn_ballot_w64(mx > m_run + kLazyRescale) != 0) {
            const float m_new = fmaxf(m_run, mx);
            const float alpha = fast_exp2(m_run - (m_new == kNegInf ? 0.f : m_new));
#pragma unroll
            for (int i = 0; i < 4; ++i) oacc[i] *= alpha;
#pragma unroll
            for (int i = 0; i < NRB; ++i) racc[i] *= alpha;
            lsum *= alpha;
            m_run = m_new;
        }
        const float m_use = m_run == kNegInf ? 0.f : m_run;
        float tsum = 0.f;  // of this tile alone: a sum of 16 pairs keeps its roundings small beside lsum's
        fence();
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            score_product(kp[i % PRE], i, snext);
            if (i + PRE < NS) kp[i % PRE] = score_frag(sat, i + PRE);
#pragma unroll
            for (int w = 16 * i / NS; w < 16 * (i + 1) / NS; ++w) {  // weights 2w, 2w + 1 of the lane's 32
                const float e0 = fast_exp2(__builtin_fmaf(s[w / 8][2 * (w % 8)], cl, -m_use));
                const float e1 = fast_exp2(__builtin_fmaf(s[w / 8][2 * (w % 8) + 1], cl, -m_use));
                uint32_t pk = pack_bf16(e0, e1);
                asm volatile("" : "+v"(pk));  // stays here: otherwise the compiler moves the weights past the next barrier
                pf[w / 4][w % 4] = pk;
                // the weights as the value products take them: their rounding cancels in O / l
                if constexpr (!LROW) tsum = add_bf16_pair(pk, tsum);
            }
            fence();
        }
        if constexpr (!LROW) lsum += tsum;
        if constexpr (ROPE && !BESIDE) {
            if (wave >= 4) rebuild(t + 2);
        }
    };

    wait_vmcnt<0>();
    lds_fence_barrier();
    rebuild(0);
    rebuild(1);
    lds_fence_barrier();
    copies(-1, true, S::VR > 2);  // (its rCache and table slots were those of tile 0 or 1)
    f32x16 sa[2], sb[2];
    {
        const ScoreAddr at = score_addr(0);
#pragma unroll
        for (int i = 0; i < NS; ++i) score_product(score_frag(at, i), i, sa);
    }
    body(std::false_type{}, std::true_type{}, 0, sa, sb);
    const int n_full = min((P0 + tok_begin + 1) / TILE_KEYS, n_tiles);  // tiles below every row's diagonal
    int t = 1;
    for (; t + 1 < n_full; t += 2) {
        body(std::true_type{}, std::false_type{}, t, sb, sa);
        body(std::true_type{}, std::false_type{}, t + 1, sa, sb);
    }
    for (; t < n_tiles; ++t) {
        body(std::true_type{}, std::true_type{}, t, sb, sa);
        sb[0] = sa[0];
        sb[1] = sa[1];
    }
    wait_vmcnt<0>();
    lds_fence_barrier();
    // B_V of the epilogue, four dims per thread and step: requested beside the last values at ranks 32
    // and 64 (up to rank 16 the loop before has no registers left for it)
    constexpr int NF = (R * D / 4 + 64 * NW - 1) / (64 * NW), NFX = NF > 0 ? NF : 1;
    u32x2 bvq[NFX];
    auto load_bv = [&]() __attribute__((always_inline)) {
        const uint16_t *bv = p.lora_b + ((int64_t)ad * 2 + 1) * R * n + (int64_t)h * D;
#pragma unroll
        for (int k = 0; k < NF; ++k) {
            const int e = 4 * ((int)threadIdx.x + 64 * NW * k);
            if (e < R * D) bvq[k] = ldg64(bv + (int64_t)(e / D) * n + e % D);
        }
    };
    if constexpr (R >= 32) load_bv();
    values(std::true_type{}, n_tiles - 1, [](int) {});
    __syncthreads();  // the ring is reused below

    // ---- epilogue: O = (acc + acc_r . B_V[h]) / l ----
    // Bound by LDS: a lane reads the 128 / 2 dims of its half for every rank.  With B_V loaded value by
    // value, read 8 bytes at a time and the accumulators' rows a multiple of 32 banks apart, short contexts
    // at ranks 32 and 64 were slower than on the kernel before (12 agents x 600 rows over 300 tokens, 8B
    // heads, RoPE off: rank 32 218 -> 240 us, now 192; rank 64 320 -> 384, now 289; rank 64 with 16 agents
    // x 40 rows and eight query heads per KV head, where 128-row workgroups take a second round: 67 -> 101,
    // now 72).  Ranks two at a time: four took 45 to 70 % longer at rank 64, one 2 %.
    const float l_run = LROW ? __shfl(racc[0][1], r32) : lsum + __shfl_xor(lsum, 32);
    if constexpr (R > 0) {
        float *sBV = reinterpret_cast<float *>(lds);
        float *sAcc = reinterpret_cast<float *>(lds + R * D * 4);
        if constexpr (R < 32) load_bv();
        // dim 32i + 16e + 4b + 2hh + j of a rank at 32i + 16e + 8hh + 2b + j: a lane's dims lie side by side
#pragma unroll
        for (int k = 0; k < NF; ++k) {
            const int e = 4 * ((int)threadIdx.x + 64 * NW * k), b = (e / 4) % 4;
            if (e >= R * D) break;
            float *at = sBV + (e & ~15) + 2 * b;
            *reinterpret_cast<f32x2 *>(at) = f32x2{bf16_lo(bvq[k].x), bf16_hi(bvq[k].x)};
            *reinterpret_cast<f32x2 *>(at + 8) = f32x2{bf16_lo(bvq[k].y), bf16_hi(bvq[k].y)};
        }
#pragma unroll
        for (int b = 0; b < NRB; ++b)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int rho = 32 * b + 16 * (i & 1) + 4 * (i / 4) + 2 * hh + (i % 4) / 2;
                if (rho < R) sAcc[(wave * 32 + r32) * (R + 1) + rho] = racc[b][i];
            }
        __syncthreads();
#pragma unroll 2
        for (int rho = 0; rho < R; ++rho) {
            const float c = sAcc[(wave * 32 + r32) * (R + 1) + rho];
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int e = 0; e < 2; ++e)
#pragma unroll
                    for (int b2 = 0; b2 < 2; ++b2) {  // rows 8b + 4hh + e and + 2: dims 32i + 16e + 4b + 2hh and + 1
                        const f32x4 v = *reinterpret_cast<const f32x4 *>(sBV + rho * D + 32 * i + 16 * e + 8 * hh + 4 * b2);
                        oacc[i][8 * b2 + e] += c * v[0];
                        oacc[i][8 * b2 + e + 2] += c * v[1];
                        oacc[i][8 * b2 + 4 + e] += c * v[2];
                        oacc[i][8 * b2 + 4 + e + 2] += c * v[3];
                    }
        }
    }
    if (row_ok) {
        const float inv = l_run > 0.f ? 1.f / l_run : 0.f;
        uint16_t *orow = p.out + ((int64_t)(q0 + tok) * p.hq + h * G + r32 % G) * D;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int b = 0; b < 4; ++b)
#pragma unroll
                for (int e = 0; e < 2; ++e)
                    *reinterpret_cast<uint32_t *>(orow + 32 * i + 16 * e + 4 * b + 2 * hh) =
                        pack_bf16(oacc[i][4 * b + e] * inv, oacc[i][4 * b + e + 2] * inv);
    }
}

template <int R, int G, bool ROPE, int NW>
__global__ __launch_bounds__(64 * NW) void prefill_stream_kernel(PrefillArgs p) {
    constexpr int ROWS = NW * 32, TPW = ROWS / G;
    constexpr int EPI = R > 0 ? R * D * 4 + ROWS * (R + 1) * 4 : 0;
    constexpr int RING = Ring<R, ROPE>::MAIN_BYTES > Ring<0, false>::MAIN_BYTES ? Ring<R, ROPE>::MAIN_BYTES : Ring<0, false>::MAIN_BYTES;
    constexpr int BYTES = RING > EPI ? RING : EPI;
    static_assert(BYTES <= 160 * 1024, "LDS of one workgroup");
    __shared__ __attribute__((aligned(1024))) unsigned char lds[BYTES];
    const int bpa = p.blocks_per_agent_head;
    const int xcd = blockIdx.x % kXcds, local = blockIdx.x / kXcds;
    const int pair = (local / bpa) * kXcds + xcd;
    const int qb = local - (local / bpa) * bpa;
    if (pair >= p.n_agents * p.hkv) return;
    const int a = pair / p.hkv;
    const int h = pair - a * p.hkv;
    const int q0 = p.q_indptr[a], nq = p.q_indptr[a + 1] - q0;
    const int tok_begin = qb * TPW;
    if (qb == bpa - 1 && nq > bpa * TPW) poison_unreached_rows(p, q0, nq, h, G, bpa * TPW);
    if (tok_begin >= nq) return;
    if (R > 0 && p.adapter_idx[a] >= 0) prefill_block<R, G, ROPE, NW>(p, lds, a, h, tok_begin);
    else prefill_block<0, G, false, NW>(p, lds, a, h, tok_begin);
}

template <int R, int G, bool ROPE, int NW>
hipError_t launch(const PrefillArgs &pa, hipStream_t st, void *const *ev) {
    const int pairs = (pa.n_agents * pa.hkv + kXcds - 1) / kXcds * kXcds;
    // timing events carry the kernel's own start and end timestamps (set by the launch)
    hipEvent_t e0 = ev ? static_cast<hipEvent_t>(ev[0]) : nullptr;
    hipEvent_t e1 = ev ? static_cast<hipEvent_t>(ev[1]) : nullptr;
    hipExtLaunchKernelGGL((prefill_stream_kernel<R, G, ROPE, NW>), dim3(pairs * pa.blocks_per_agent_head), dim3(64 * NW), 0, st,
                          e0, e1, 0, pa);
    return hipGetLastError();
}

template <int G>
hipError_t dispatch(int r, bool rope, bool rows128, const PrefillArgs &pa, hipStream_t st, void *const *ev) {
    switch (r) {
    case 0: return rows128 ? launch<0, G, false, 4>(pa, st, ev) : launch<0, G, false, 8>(pa, st, ev);
    case 8:
        if (rope) return rows128 ? launch<8, G, true, 4>(pa, st, ev) : launch<8, G, true, 8>(pa, st, ev);
        return rows128 ? launch<8, G, false, 4>(pa, st, ev) : launch<8, G, false, 8>(pa, st, ev);
    case 16:
        if (rope) return rows128 ? launch<16, G, true, 4>(pa, st, ev) : launch<16, G, true, 8>(pa, st, ev);
        return rows128 ? launch<16, G, false, 4>(pa, st, ev) : launch<16, G, false, 8>(pa, st, ev);
    case 32:
        if (rope) return rows128 ? launch<32, G, true, 4>(pa, st, ev) : hipErrorInvalidValue;
        return rows128 ? launch<32, G, false, 4>(pa, st, ev) : launch<32, G, false, 8>(pa, st, ev);
    case 64: return rows128 && !rope ? launch<64, G, false, 4>(pa, st, ev) : hipErrorInvalidValue;
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_stream(int r, int g, bool rope, bool rows128, const PrefillArgs &pa, hipStream_t st, void *const *ev) {
    return g == 4 ? dispatch<4>(r, rope, rows128, pa, st, ev) : dispatch<8>(r, rope, rows128, pa, st, ev);
}

}  // namespace fkvp
