// Backward pass of fused attention for bf16 inputs on gfx950 matrix cores:
// dQ, dK and dV for a given dO, recomputing the weights from the forward's
// LSE (no score or weight matrix is ever stored, as in the forward).
//
// With s = <q_i, k_j>, c = scale * log2(e) and lse2_i = LSE_i * log2(e):
//   P_ij  = 2^(s_ij c - lse2_i)              (the forward's softmax weights)
//   dP_ij = <dO_i, v_j>
//   D_i   = <dO_i, O_i> = sum_j P_ij dP_ij
//   dS_ij = P_ij (dP_ij - D_i)               (softmax Jacobian)
//   dQ_i  = scale * sum_j dS_ij k_j,   dK_j = scale * sum_i dS_ij q_i,
//   dV_j  = sum_i P_ij dO_i
// which is the chain rule through the softmax the paper leaves to its Stage 5.
//
// Two kernels:
//  * bwd_dq: one item = 128 or 256 queries of one (b, h).  D_i of its queries from
//    the dO fragments and O (fp32), kept and written out for the other kernel;
//    then K and V stream through LDS in 64-key stages.  S^T = K Q^T and dP^T = V dO^T on the MFMA (K and V
//    rows as A operands, Q and dO fragments held in registers as in the
//    forward), dS^T in registers, dQ^T += K^T dS^T with K^T from transposing
//    LDS reads of the same K stage.
//  * bwd_dkdv_pair: one item = 64, 128 or 256 keys of one (b, h); Q, dO, LSE
//    and D stream through LDS in stages of 32 or 64 queries.  S = Q K^T and dP = dO V^T (Q and
//    dO rows as A operands, K or V fragments in registers), so a lane holds
//    one key; dV^T += dO^T P and dK^T += Q^T dS with dO^T and Q^T from
//    transposing reads.  The two halves of that work go to two waves of the
//    same SIMD (the weights P pass between them through LDS), so the vector
//    work of one overlaps the matrix products of the other.  Every lane owns
//    its key's rows of dK or dV: no atomics, and the results are
//    deterministic.
// P and dS are rounded to bf16 for the matrix products (fp32 accumulation);
// dS is formed from the bf16-rounded P.
#include <algorithm>
#include <type_traits>

#include "device_common.h"
#include "launch.h"
#include "prefill_bf16_common.h"

namespace moa {
namespace {

using namespace pf;

constexpr int SUB = 32;   // queries (bwd_dkdv) or keys (bwd_dq) per step

// Per-lane LDS addresses shared by both kernels (the stage layout of the
// forward: 64 rows of D bf16, 16-byte chunks XOR-swizzled per row).
template <int D>
struct TileAddr {
    uint32_t row[D / 16];      // A operand of a row-major stage: row col (+32 u), chunk 2s + half
    uint32_t tr[D / 32][2];    // transposing reads: D-block b, lo / hi row quads
    __device__ __forceinline__ TileAddr(int lane) {
        constexpr uint32_t RB = Cfg<D>::ROW_BYTES;
        const int col = lane & 31, half = lane >> 5;
#pragma unroll
        for (int s = 0; s < D / 16; ++s)
            row[s] = (uint32_t)col * RB + (uint32_t)(((2 * s + half) ^ swz<D>(col)) * 16);
        const int g = lane >> 4, j = (lane >> 2) & 3, q = lane & 3;
#pragma unroll
        for (int b = 0; b < D / 32; ++b)
#pragma unroll
            for (int h8 = 0; h8 < 2; ++h8) {
                const int r = 4 * (g >> 1) + j + 8 * h8;
                const int dv = dv_of<D>(b, 16 * (g & 1) + 4 * q);
                tr[b][h8] = (uint32_t)r * RB + (uint32_t)((((dv >> 3) ^ swz<D>(r)) * 16) + (dv & 7) * 2);
            }
    }
};

// MFMA A operand from a stage: rows 32u + (lane % 32), contraction chunk s.
template <int D>
__device__ __forceinline__ bf16x8 stage_rows(const unsigned char* st, const TileAddr<D>& a, int u, int s) {
    return *reinterpret_cast<const bf16x8*>(st + a.row[s] + u * 32 * Cfg<D>::ROW_BYTES);
}
// MFMA A operand of the transposed stage: D-block b, 16-row chunk cc.
template <int D>
__device__ __forceinline__ bf16x8 stage_tr(const unsigned char* st, const TileAddr<D>& a, int b, int cc) {
    const v4s lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s*)(st + a.tr[b][0] + cc * 16 * Cfg<D>::ROW_BYTES));
    const v4s hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s*)(st + a.tr[b][1] + cc * 16 * Cfg<D>::ROW_BYTES));
    const v4s both[2] = {lo, hi};
    return __builtin_bit_cast(bf16x8, both);
}

// Packs an fp32 accumulator (16 values) into two bf16x8 MFMA B operands in the
// key (or query) order of the transposing reads: chunk c2 takes elements
// 8 c2 .. 8 c2 + 7.
__device__ __forceinline__ void pack16(const float (&x)[16], bf16x8 (&pb)[2]) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
#pragma unroll
    for (int g = 0; g < 2; ++g) {
        u32x4 w;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const bf16x2 pp = {(__bf16)x[8 * g + 2 * j], (__bf16)x[8 * g + 2 * j + 1]};
            w[j] = __builtin_bit_cast(uint32_t, pp);
        }
        pb[g] = __builtin_bit_cast(bf16x8, w);
    }
}

// A direct-to-LDS 16-byte load (buffer_load_dwordx4 ... lds) as inline
// assembly, invisible to the compiler's wait-count tracking (whose aliasing
// model cannot tell the slots of one LDS ring apart and would wait for every
// load before any read of the ring).  The
// caller waits for it itself (s_waitcnt vmcnt, then a barrier) before any wave
// reads the data; loads complete in issue order, so the compiler's own waits
// for later loads stay correct.  `rsrc` holds the four descriptor words (see
// rsrc_words), `lds_addr` the wave-uniform LDS byte address.
__device__ __forceinline__ u32x4 rsrc_words(const void* base, uint32_t bytes) {
    const uint64_t a = reinterpret_cast<uint64_t>(base);
    return u32x4{(uint32_t)a, (uint32_t)(a >> 32) & 0xffffu, bytes, 0x00020000u};
}
__device__ __forceinline__ uint32_t lds_address(const void* p) {
    return (uint32_t)reinterpret_cast<uintptr_t>((const __attribute__((address_space(3))) void*)p);
}
// M0 is listed as clobbered: clang warns that it does not preserve reserved
// registers around the statement; the kernels of this file set M0 nowhere
// else (their assembly has no other M0 write).
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void buffer_load16_to_lds_untracked(u32x4 rsrc, uint32_t lds_addr, uint32_t voffset) {
    const u32x4 r = {(uint32_t)__builtin_amdgcn_readfirstlane(rsrc[0]), (uint32_t)__builtin_amdgcn_readfirstlane(rsrc[1]),
                     (uint32_t)__builtin_amdgcn_readfirstlane(rsrc[2]), (uint32_t)__builtin_amdgcn_readfirstlane(rsrc[3])};
    const uint32_t m = (uint32_t)__builtin_amdgcn_readfirstlane(lds_addr);
    // One wait state between the M0 write and the load that reads it.
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                 :: "s"(m), "v"(voffset), "s"(r) : "memory", "m0");
}
#pragma clang diagnostic pop

// Direct-to-LDS stage loads (untracked: the caller waits with vmcnt and a
// barrier): lane l of the i-th load of wave w fills slot S = (w*LPS + i)*64
// + l of the stage, which holds logical chunk (S % CHUNKS) ^ swz(row) of row
// S / CHUNKS (the forward's swizzled layout).
template <int D, int NW, int ROWS = BN>
struct DmaStager {
    static constexpr int STAGE_BYTES = ROWS * Cfg<D>::ROW_BYTES;
    static constexpr int LPS = STAGE_BYTES / (NW * 1024);
    static_assert(STAGE_BYTES % (NW * 1024) == 0, "a stage must split into wave loads");
    uint32_t goff[LPS];
    uint32_t lds_off;        // this wave's first 1 KB of a stage
    __device__ __forceinline__ DmaStager(int wave, int lane) {
        lds_off = (uint32_t)wave * LPS * 1024u;
#pragma unroll
        for (int i = 0; i < LPS; ++i) {
            const int slot = (wave * LPS + i) * 64 + lane;
            const int row = slot / Cfg<D>::CHUNKS, p = slot % Cfg<D>::CHUNKS;
            goff[i] = (uint32_t)row * Cfg<D>::ROW_BYTES + (uint32_t)((p ^ swz<D>(row)) * 16);
        }
    }
    // Rows j * ROWS .. of a head slice of `n` rows into `stage`; rows past n
    // are zero.
    __device__ __forceinline__ void issue(const u16* head, int n, int j, unsigned char* stage) const {
        const int r0 = min(j * ROWS, n);
        const u32x4 r = rsrc_words(head + (size_t)r0 * D, (uint32_t)(n - r0) * Cfg<D>::ROW_BYTES);
        const uint32_t base = lds_address(stage) + lds_off;
#pragma unroll
        for (int i = 0; i < LPS; ++i) buffer_load16_to_lds_untracked(r, base + i * 1024u, goff[i]);
    }
};

template <int D, bool OUT_BF16>
__device__ __forceinline__ void store_rows16(void* out, size_t row_base, int half, const f32x16 (&acc)[D / 32],
                                             float mul) {
#pragma unroll
    for (int b = 0; b < D / 32; ++b)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int dv = dv_of<D>(b, g * 8 + half * 4);
            const float o0 = acc[b][g * 4 + 0] * mul, o1 = acc[b][g * 4 + 1] * mul;
            const float o2 = acc[b][g * 4 + 2] * mul, o3 = acc[b][g * 4 + 3] * mul;
            if (OUT_BF16) {
                *reinterpret_cast<uint2*>(static_cast<u16*>(out) + row_base + dv) =
                    make_uint2(pack_bf16x2(o0, o1), pack_bf16x2(o2, o3));
            } else {
                *reinterpret_cast<float4*>(static_cast<float*>(out) + row_base + dv) =
                    make_float4(o0, o1, o2, o3);
            }
        }
}

// ---- dQ: 8 waves x 32 queries; K and V stages of 64 keys.  KS = 1: 256
// queries per item, one key stream.  KS = 2: 128 queries, two key streams
// (waves 4 .. 7 hold the queries of waves 0 .. 3 and take every second key
// stage through a ring of their own); the partial sums of dQ meet in LDS.
// The key loop runs over the stages of which a wave needs both 32-key steps,
// without a test inside; the stage it needs half of, and those it only passes
// through, follow in a loop of their own (B2 H16 4K d = 64 backward 545 -> 484
// us, d = 128 causal 462 -> 452: the tests kept the steps from overlapping).
//
// D is formed in the prologue, where the dO fragments are in registers anyway:
// a kernel of its own read dO once more and cost a launch, 12.6 us on B2 H16 4K
// d = 128 and 3.7 on B4 H8 1000 d = 64 (training step 60.5 -> 55.5 us; the
// same sums in the same order).
constexpr int DQ_WAVES = 8;
constexpr int DQ_THREADS = DQ_WAVES * 64;

template <int D, bool CAUSAL, bool OUT_BF16, int KS>
__global__ __launch_bounds__(DQ_THREADS, 1) void bwd_dq_kernel(
    const u16* __restrict__ Q, const u16* __restrict__ K, const u16* __restrict__ V,
    const u16* __restrict__ dO, const void* __restrict__ O, int o_bf16,
    const float* __restrict__ LSE, float* __restrict__ Dsum, void* __restrict__ dQ, int Nq, int Nk, int n_bh, int n_qtiles, float c, float scale) {
    using C = Cfg<D>;
    constexpr uint32_t RB = C::ROW_BYTES;
    constexpr int QB = DQ_WAVES / KS;       // query blocks of 32
    constexpr int BMQ = QB * 32;            // queries per item
    __shared__ __attribute__((aligned(1024))) unsigned char k_r[2][KS][C::TILE_BYTES];
    __shared__ __attribute__((aligned(1024))) unsigned char v_r[2][KS][C::TILE_BYTES];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int qw = wave % QB, grp = wave / QB;   // query block, key stream
    const int col = lane & 31, half = lane >> 5;
    const int off = Nk - Nq;
    const TileAddr<D> ta(lane);
    const DmaStager<D, QB> stg(qw, lane);

    for (int item = 0;; ++item) {
        int bh, qt;
        if (!item_of(blockIdx.x, item, gridDim.x, n_bh, n_qtiles, CAUSAL, bh, qt)) break;
        const int q0 = qt * BMQ;
        const int qrow = q0 + qw * 32 + col;
        const u16* Kh = K + (size_t)bh * Nk * D;
        const u16* Vh = V + (size_t)bh * Nk * D;

        // Q and dO fragments of this lane's query (B operands), its LSE and D.
        bf16x8 qf[D / 16], gf[D / 16];
        {
            const auto rq = make_rsrc(Q + (size_t)bh * Nq * D, (uint32_t)Nq * RB);
            const auto rg = make_rsrc(dO + (size_t)bh * Nq * D, (uint32_t)Nq * RB);
#pragma unroll
            for (int s = 0; s < D / 16; ++s) {
                qf[s] = __builtin_bit_cast(bf16x8, buffer_load16(rq, (uint32_t)qrow * RB + s * 32 + half * 16));
                gf[s] = __builtin_bit_cast(bf16x8, buffer_load16(rg, (uint32_t)qrow * RB + s * 32 + half * 16));
            }
        }
        const bool row_ok = qrow < Nq;
        const float lse2 = row_ok ? LSE[(size_t)bh * Nq + qrow] * kLog2e : 0.0f;
        // D of this lane's query: 8 elements at a time, then pairwise (the two
        // halves of a 16-element chunk sit in lanes l and l ^ 32).
        float dsum;
        {
            float part[D / 16];
            const size_t o0 = ((size_t)bh * Nq + (row_ok ? qrow : 0)) * D + half * 8;
#pragma unroll
            for (int s = 0; s < D / 16; ++s) {
                float o[8];
                if (o_bf16) {
                    const uint4 h = *reinterpret_cast<const uint4*>(static_cast<const u16*>(O) + o0 + s * 16);
                    const uint32_t hw[4] = {h.x, h.y, h.z, h.w};
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        o[2 * j] = bf16lo_to_f32(hw[j]);
                        o[2 * j + 1] = bf16hi_to_f32(hw[j]);
                    }
                } else {
                    const float* of = static_cast<const float*>(O) + o0 + s * 16;
                    const float4 x = *reinterpret_cast<const float4*>(of), y = *reinterpret_cast<const float4*>(of + 4);
                    o[0] = x.x; o[1] = x.y; o[2] = x.z; o[3] = x.w;
                    o[4] = y.x; o[5] = y.y; o[6] = y.z; o[7] = y.w;
                }
                const u32x4 g = __builtin_bit_cast(u32x4, gf[s]);
                part[s] = 0.0f;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    part[s] = __builtin_fmaf(bf16lo_to_f32(g[j]), o[2 * j], part[s]);
                    part[s] = __builtin_fmaf(bf16hi_to_f32(g[j]), o[2 * j + 1], part[s]);
                }
                part[s] = half_sum(part[s]);
            }
#pragma unroll
            for (int m = 1; m < D / 16; m <<= 1)
#pragma unroll
                for (int s = 0; s < D / 16; s += 2 * m) part[s] += part[s + m];
            dsum = row_ok ? part[0] : 0.0f;
            if (row_ok && half == 0 && grp == 0) Dsum[(size_t)bh * Nq + qrow] = dsum;
        }

        const int kv_end = CAUSAL ? min(Nk, q0 + BMQ + off) : Nk;
        const int n_sub = (kv_end + SUB - 1) / SUB;
        const int n_stages = (n_sub + 1) / 2;
        const int n_iter = (n_stages + KS - 1) / KS;
        const int wave_q_first = q0 + qw * 32;
        int n_w = n_sub;
        if (wave_q_first >= Nq) n_w = 0;
        else if (CAUSAL) n_w = min(n_sub, (wave_q_first + 31 + off) / SUB + 1);
        // Iterations in which this wave needs both steps of its stage.
        const int n_full = max(0, (n_w / 2 - grp + KS - 1) / KS);

        f32x16 acc[D / 32];
#pragma unroll
        for (int b = 0; b < D / 32; ++b) acc[b] = f32x16{};

        // One step of 32 keys (half u of the stage in ks / vs, global step t).
        auto step = [&](const unsigned char* ks, const unsigned char* vs, int u, int t)
                        __attribute__((always_inline)) {
            f32x16 s = f32x16{}, dp = f32x16{};
#pragma unroll
            for (int k = 0; k < D / 16; ++k) {
                s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(stage_rows<D>(ks, ta, u, k), qf[k], s, 0, 0, 0);
                dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(stage_rows<D>(vs, ta, u, k), gf[k], dp, 0, 0, 0);
            }
            const int kbase = t * SUB;
#pragma unroll
            for (int i = 0; i < 16; ++i) s[i] = __builtin_fmaf(s[i], c, -lse2);
            if ((kbase + SUB > Nk) || (CAUSAL && kbase + SUB - 1 > wave_q_first + off)) {
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int key = kbase + (i >> 2) * 8 + half * 4 + (i & 3);
                    if (key >= Nk || (CAUSAL && key > qrow + off)) s[i] = kNegInf;
                }
            }
            float ds[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) ds[i] = exp2_hw(s[i]) * (dp[i] - dsum);
            bf16x8 dsb[2];
            pack16(ds, dsb);
#pragma unroll
            for (int c2 = 0; c2 < 2; ++c2)
#pragma unroll
                for (int b = 0; b < D / 32; ++b)
                    acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(stage_tr<D>(ks, ta, b, 2 * u + c2), dsb[c2],
                                                                     acc[b], 0, 0, 0);
        };

        // Iteration j: stage js = j * KS + grp in ring slot j & 1.  Right
        // after the barrier the next stage's loads start into the other slot,
        // whose readers (iteration j - 1) are done; each wave waits for its
        // own loads before the next barrier.
        auto issue = [&](int j) __attribute__((always_inline)) {
            stg.issue(Kh, Nk, j * KS + grp, k_r[j & 1][grp]);
            stg.issue(Vh, Nk, j * KS + grp, v_r[j & 1][grp]);
        };
        auto advance = [&](int j) __attribute__((always_inline)) {
            wait_vmcnt<0>();
            wait_lgkmcnt0();
            barrier_no_fence();
            if (j + 1 < n_iter) issue(j + 1);
        };
        issue(0);
        int j = 0;
        for (; j < n_full; ++j) {
            advance(j);
            const int js = j * KS + grp;
            step(k_r[j & 1][grp], v_r[j & 1][grp], 0, 2 * js);
            step(k_r[j & 1][grp], v_r[j & 1][grp], 1, 2 * js + 1);
        }
        for (; j < n_iter; ++j) {
            advance(j);
            const int js = j * KS + grp;
            if (2 * js < n_w) step(k_r[j & 1][grp], v_r[j & 1][grp], 0, 2 * js);
        }
        wait_lgkmcnt0();
        barrier_no_fence();
        if constexpr (KS == 2) {
            float* x = reinterpret_cast<float*>(qw < 2 ? &k_r[0][0][0] : &v_r[0][0][0]) + (qw & 1) * (D / 2) * 64;
            if (grp == 1) {
#pragma unroll
                for (int b = 0; b < D / 32; ++b)
#pragma unroll
                    for (int i = 0; i < 16; ++i) x[(b * 16 + i) * 64 + lane] = acc[b][i];
            }
            __syncthreads();
            if (grp == 0) {
#pragma unroll
                for (int b = 0; b < D / 32; ++b)
#pragma unroll
                    for (int i = 0; i < 16; ++i) acc[b][i] += x[(b * 16 + i) * 64 + lane];
            }
            __syncthreads();   // the next item's stages land in the same LDS
        }
        if (row_ok && grp == 0) store_rows16<D, OUT_BF16>(dQ, ((size_t)bh * Nq + qrow) * D, half, acc, scale);
    }
}

// ---- dK, dV with two waves per SIMD.  A pair of waves (w, w + 4) owns 32 *
// NKB keys.  Wave w < 4 (role A): S = Q K^T, the weights P (exponentials),
// dV^T += dO^T P, and P handed to its partner through LDS as bf16.  Wave
// w + 4 (role B, on the same SIMD): dP = dO V^T, dS = P (dP - D) with the
// partner's P, dK^T += Q^T dS.  The matrix work of a step splits evenly
// between the two waves and nothing is computed twice; B runs one stage of SR
// queries behind A, so the LDS ring holds three Q / dO stages and two stages
// of exchanged weights.
//
// Each role has a loop of its own.  With one loop and the role tested inside,
// the compiler kept both roles' accumulators in one register set and copied
// them at every join (249 registers, 64 moves a stage); apart, the same code
// takes 236 with the operand reads further ahead, 16K causal d = 128 (dK, dV
// kernel with dQ) 7.40 -> 6.69 ms, B2 H16 4K 512 -> 470 us.
//
// NKB = 2 (d = 64): every operand read from LDS feeds two products, B2 H16 4K
// 551 -> 515 us.  At d = 128 the second key block does not fit the registers
// (256, 5 reloads per step: 7.25 -> 8.35 ms).
// QS = 2: two query streams for grids that leave compute units idle: pairs 0,
// 1 and pairs 2, 3 own the same keys, each half takes every second stage
// through a ring of its own, and the partial sums meet in LDS.
constexpr int KV2_WAVES = 8;
constexpr int KV2_THREADS = KV2_WAVES * 64;
constexpr int KV2_RING = 3;      // Q / dO stages in LDS

template <int D, bool CAUSAL, bool OUT_BF16, int NKB, int SR, int QS>
__global__ __launch_bounds__(KV2_THREADS, 1) void bwd_dkdv_pair_kernel(
    const u16* __restrict__ Q, const u16* __restrict__ K, const u16* __restrict__ V,
    const u16* __restrict__ dO, const float* __restrict__ LSE, const float* __restrict__ Dsum,
    void* __restrict__ dK, void* __restrict__ dV, int Nq, int Nk, int n_bh, int n_ktiles, float c,
    float scale) {
    using C = Cfg<D>;
    constexpr uint32_t RB = C::ROW_BYTES;
    constexpr int KW = 32 * NKB;            // keys per pair of waves
    constexpr int NP = 4 / QS;              // pairs side by side
    constexpr int KT = NP * KW;             // keys per item
    constexpr int U = SR / SUB;             // steps per stage
    static_assert(U == 1 || (U == 2 && QS == 1), "a first odd step belongs to the only stream");
    __shared__ __attribute__((aligned(1024))) unsigned char q_r[KV2_RING][QS][SR * C::ROW_BYTES];
    __shared__ __attribute__((aligned(1024))) unsigned char g_r[KV2_RING][QS][SR * C::ROW_BYTES];
    // Exchanged weights: [stage parity][wave pair][step][key block][chunk c2][lane] x 16 bytes.
    __shared__ __attribute__((aligned(1024))) uint4 p_x[2][4][U][NKB][2][64];
    __shared__ __attribute__((aligned(16))) float l_r[KV2_RING][QS][2][SR];   // [slot][stream][lse2, D][query]

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int role = wave >> 2, pair = wave & 3;   // role 0: P and dV; role 1: dS and dK
    const int kb = pair % NP, qs = pair / NP;      // key block, query stream
    const int col = lane & 31, half = lane >> 5;
    const int off = Nk - Nq;
    TileAddr<D> ta(lane);
    const DmaStager<D, KV2_WAVES / QS, SR> stg(role * NP + kb, lane);

    for (int item = 0;; ++item) {
        int bh, rt;
        if (!item_of(blockIdx.x, item, gridDim.x, n_bh, n_ktiles, CAUSAL, bh, rt)) break;
        // Causal key tiles cost most at the start of the sequence: the
        // heaviest-first rank order of item_of is reversed here.
        const int kt = CAUSAL ? n_ktiles - 1 - rt : rt;
        const int k0 = kt * KT;
        const int blk_k_first = k0 + kb * KW;
        const u16* Qh = Q + (size_t)bh * Nq * D;
        const u16* Gh = dO + (size_t)bh * Nq * D;
        const float* Lh = LSE + (size_t)bh * Nq;
        const float* Dh = Dsum + (size_t)bh * Nq;

        // K (role A) or V (role B) fragments of this lane's keys: B operands.
        bf16x8 kvf[NKB][D / 16];
        {
            const auto r = make_rsrc((role == 0 ? K : V) + (size_t)bh * Nk * D, (uint32_t)Nk * RB);
#pragma unroll
            for (int n = 0; n < NKB; ++n)
#pragma unroll
                for (int s = 0; s < D / 16; ++s)
                    kvf[n][s] = __builtin_bit_cast(
                        bf16x8, buffer_load16(r, (uint32_t)(blk_k_first + 32 * n + col) * RB + s * 32 + half * 16));
        }

        // Queries that see any key of the tile (query i sees key j iff
        // j <= i + off), in stages; the pair's first needed step.
        const int q_lo = CAUSAL ? max(0, k0 - off) : 0;
        const int st0 = q_lo / SR;
        const int n_stages = ((Nq + SR - 1) / SR - st0 + QS - 1) / QS;   // of each stream
        const int t_first = CAUSAL ? max(0, blk_k_first - off) / SUB : 0;   // global 32-query step
        const bool blk_live = blk_k_first < Nk;

        f32x16 acc[NKB][D / 32];     // dV^T (role A) or dK^T (role B)
#pragma unroll
        for (int n = 0; n < NKB; ++n)
#pragma unroll
            for (int b = 0; b < D / 32; ++b) acc[n][b] = f32x16{};

        // Role A, step u of stage js: weights of 32 queries x this lane's keys.
        auto step_a = [&](const unsigned char* qs, const unsigned char* gs, const float* ls, uint4* px,
                          int u, int t) __attribute__((always_inline)) {

            f32x16 s[NKB];
#pragma unroll
            for (int n = 0; n < NKB; ++n) s[n] = f32x16{};
#pragma unroll
            for (int k = 0; k < D / 16; ++k) {
                const bf16x8 a = stage_rows<D>(qs, ta, u, k);
#pragma unroll
                for (int n = 0; n < NKB; ++n)
                    s[n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, kvf[n][k], s[n], 0, 0, 0);
            }
            // Exponents, then the mask (which must not pass through c).
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int m0 = 32 * u + 8 * g + 4 * half;   // stage-local query of element 4g
                const float4 l4 = *reinterpret_cast<const float4*>(ls + m0);
                const float lv[4] = {l4.x, l4.y, l4.z, l4.w};
#pragma unroll
                for (int n = 0; n < NKB; ++n)
#pragma unroll
                    for (int r = 0; r < 4; ++r) s[n][4 * g + r] = __builtin_fmaf(s[n][4 * g + r], c, -lv[r]);
            }
            const int qbase = t * SUB;
            if ((qbase + SUB > Nq) || (CAUSAL && qbase < blk_k_first + KW - 1 - off)) {
#pragma unroll
                for (int n = 0; n < NKB; ++n)
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const int qi = qbase + (i >> 2) * 8 + 4 * half + (i & 3);
                        if (qi >= Nq || (CAUSAL && blk_k_first + 32 * n + col > qi + off)) s[n][i] = kNegInf;
                    }
            }
            bf16x8 pb[NKB][2];
#pragma unroll
            for (int n = 0; n < NKB; ++n) {
                float p[16];
#pragma unroll
                for (int i = 0; i < 16; ++i) p[i] = exp2_hw(s[n][i]);
                pack16(p, pb[n]);
#pragma unroll
                for (int c2 = 0; c2 < 2; ++c2) px[(n * 2 + c2) * 64 + lane] = __builtin_bit_cast(uint4, pb[n][c2]);
            }
#pragma unroll
            for (int c2 = 0; c2 < 2; ++c2)
#pragma unroll
                for (int b = 0; b < D / 32; ++b) {
                    const bf16x8 a = stage_tr<D>(gs, ta, b, 2 * u + c2);
#pragma unroll
                    for (int n = 0; n < NKB; ++n)
                        acc[n][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, pb[n][c2], acc[n][b], 0, 0, 0);
                }
        };

        // Role B, step u of stage js: dS from the partner's weights.
        auto step_b = [&](const unsigned char* qs, const unsigned char* gs, const float* dsv, const uint4* px,
                          int u) __attribute__((always_inline)) {

            f32x16 dp[NKB];
#pragma unroll
            for (int n = 0; n < NKB; ++n) dp[n] = f32x16{};
#pragma unroll
            for (int k = 0; k < D / 16; ++k) {
                const bf16x8 a = stage_rows<D>(gs, ta, u, k);
#pragma unroll
                for (int n = 0; n < NKB; ++n)
                    dp[n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, kvf[n][k], dp[n], 0, 0, 0);
            }
            bf16x8 dsb[NKB][2];
#pragma unroll
            for (int n = 0; n < NKB; ++n) {
                const uint4 w0 = px[(n * 2 + 0) * 64 + lane], w1 = px[(n * 2 + 1) * 64 + lane];
                const uint32_t pw[8] = {w0.x, w0.y, w0.z, w0.w, w1.x, w1.y, w1.z, w1.w};
                float ds[16];
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int m0 = 32 * u + 8 * g + 4 * half;
                    const float4 d4 = *reinterpret_cast<const float4*>(dsv + m0);
                    const float dvv[4] = {d4.x, d4.y, d4.z, d4.w};
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int i = 4 * g + r;
                        const float pi = (i & 1) ? bf16hi_to_f32(pw[i >> 1]) : bf16lo_to_f32(pw[i >> 1]);
                        ds[i] = pi * (dp[n][i] - dvv[r]);
                    }
                }
                pack16(ds, dsb[n]);
            }
#pragma unroll
            for (int c2 = 0; c2 < 2; ++c2)
#pragma unroll
                for (int b = 0; b < D / 32; ++b) {
                    const bf16x8 a = stage_tr<D>(qs, ta, b, 2 * u + c2);
#pragma unroll
                    for (int n = 0; n < NKB; ++n)
                        acc[n][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, dsb[n][c2], acc[n][b], 0, 0, 0);
                }
        };

        // LSE and D of a stage's queries: one float per lane of the stream's
        // first pair (zero past Nq), stored one iteration after the load.
        auto load_ld = [&](int js, float& x) __attribute__((always_inline)) {
            const int qi = js * SR + lane;
            x = 0.0f;
            if (kb == 0 && lane < SR && qi < Nq) x = (role == 0) ? Lh[qi] : Dh[qi];
        };

        // Iteration j: the stream's stage j (stage st0 + j * QS + qs of the
        // sequence) is in the ring; role A works on it, role B on the stage
        // before (whose weights A wrote in iteration j - 1).  Right after the
        // barrier the loads of stage j + 1 start into the slot whose last
        // reader (role B, iteration j - 1) is done, and each wave waits for
        // its own loads before the next barrier.  A stream may have one stage
        // less than the other: it walks an empty one (all rows past Nq).
        auto seq = [&](int j) { return st0 + j * QS + qs; };
        float sx;
        stg.issue(Qh, Nq, seq(0), q_r[0][qs]);
        stg.issue(Gh, Nq, seq(0), g_r[0][qs]);
        load_ld(seq(0), sx);
        int slot = 0;            // ring slot of stage j
        auto advance = [&](int j) __attribute__((always_inline)) {
            if (j < n_stages && kb == 0 && lane < SR) l_r[slot][qs][role][lane] = (role == 0) ? sx * kLog2e : sx;
            wait_vmcnt<0>();
            wait_lgkmcnt0();
            barrier_no_fence();
            if (j + 1 < n_stages) {
                const int ns = (slot == KV2_RING - 1) ? 0 : slot + 1;
                stg.issue(Qh, Nq, seq(j + 1), q_r[ns][qs]);
                stg.issue(Gh, Nq, seq(j + 1), g_r[ns][qs]);
                load_ld(seq(j + 1), sx);
            }
        };
        auto next_slot = [&]() __attribute__((always_inline)) { slot = (slot == KV2_RING - 1) ? 0 : slot + 1; };
        // Stages before the pair's first visible query (all, for a pair past
        // Nk) are only passed through; `odd`: so is the first step of the
        // first stage.
        const bool odd = U == 2 && (t_first & 1) && blk_live;
        const int j0 = blk_live ? min(n_stages, (t_first / U - st0 - qs + QS - 1) / QS) : n_stages;
        if (role == 0) {
            int j = 0;
            for (; j < j0; ++j) { advance(j); next_slot(); }
            if (odd) {
                advance(j);
                step_a(q_r[slot][qs], g_r[slot][qs], l_r[slot][qs][0], &p_x[j & 1][pair][U - 1][0][0][0], U - 1,
                       U * seq(j) + U - 1);
                next_slot();
                ++j;
            }
            for (; j < n_stages; ++j) {
                advance(j);
#pragma unroll
                for (int u = 0; u < U; ++u)
                    step_a(q_r[slot][qs], g_r[slot][qs], l_r[slot][qs][0], &p_x[j & 1][pair][u][0][0][0], u,
                           U * seq(j) + u);
                next_slot();
            }
            advance(j);
        } else {
            int j = 0;
            for (; j <= j0; ++j) { advance(j); next_slot(); }
            if (odd) {
                advance(j);
                const int ps = (slot == 0) ? KV2_RING - 1 : slot - 1;
                step_b(q_r[ps][qs], g_r[ps][qs], l_r[ps][qs][1], &p_x[(j - 1) & 1][pair][U - 1][0][0][0], U - 1);
                next_slot();
                ++j;
            }
            for (; j <= n_stages; ++j) {
                advance(j);
                const int ps = (slot == 0) ? KV2_RING - 1 : slot - 1;
#pragma unroll
                for (int u = 0; u < U; ++u)
                    step_b(q_r[ps][qs], g_r[ps][qs], l_r[ps][qs][1], &p_x[(j - 1) & 1][pair][u][0][0][0], u);
                next_slot();
            }
        }
        wait_lgkmcnt0();
        barrier_no_fence();
        if constexpr (QS == 2) {
            constexpr int XB = NKB * (D / 2) * 64;   // floats of one wave's accumulators
            static_assert(2 * XB * 4 <= KV2_RING * QS * SR * C::ROW_BYTES, "two waves' sums per ring");
            float* x = reinterpret_cast<float*>(role == 0 ? &q_r[0][0][0] : &g_r[0][0][0]) + kb * XB;
            if (qs == 1) {
#pragma unroll
                for (int n = 0; n < NKB; ++n)
#pragma unroll
                    for (int b = 0; b < D / 32; ++b)
#pragma unroll
                        for (int i = 0; i < 16; ++i) x[((n * (D / 32) + b) * 16 + i) * 64 + lane] = acc[n][b][i];
            }
            __syncthreads();
            if (qs == 0) {
#pragma unroll
                for (int n = 0; n < NKB; ++n)
#pragma unroll
                    for (int b = 0; b < D / 32; ++b)
#pragma unroll
                        for (int i = 0; i < 16; ++i) acc[n][b][i] += x[((n * (D / 32) + b) * 16 + i) * 64 + lane];
            }
            __syncthreads();   // the next item's stages land in the same LDS
            if (qs == 1) continue;
        }
#pragma unroll
        for (int n = 0; n < NKB; ++n) {
            const int krow = blk_k_first + 32 * n + col;
            if (krow >= Nk) continue;
            const size_t base = ((size_t)bh * Nk + krow) * D;
            if (role == 0) store_rows16<D, OUT_BF16>(dV, base, half, acc[n], 1.0f);
            else store_rows16<D, OUT_BF16>(dK, base, half, acc[n], scale);
        }
    }
}

template <typename Kern>
int resident_per_cu(Kern kernel, int threads) {
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kernel, threads, 0) != hipSuccess) n = 1;
    return n > 0 ? n : 1;
}

template <int D, bool CAUSAL, bool OUT_BF16, int KS>
hipError_t launch_dq(const BwdProblem& p, int cus, hipStream_t stream) {
    auto kernel = bwd_dq_kernel<D, CAUSAL, OUT_BF16, KS>;
    static const int per_cu = resident_per_cu(kernel, DQ_THREADS);
    const int n_qt = (p.nq + 256 / KS - 1) / (256 / KS);
    const long long items = (long long)p.bh * n_qt;
    const unsigned grid = (unsigned)std::min<long long>(items, (long long)cus * per_cu);
    return launch_kernel(kernel, dim3(grid), dim3(DQ_THREADS), stream, static_cast<const u16*>(p.q),
                         static_cast<const u16*>(p.k), static_cast<const u16*>(p.v),
                         static_cast<const u16*>(p.dout), p.o, p.o_bf16 ? 1 : 0, p.lse, p.dsum,
                         p.dq, p.nq, p.nk, p.bh, n_qt, p.scale * kLog2e, p.scale);
}

template <int D, bool CAUSAL, bool OUT_BF16, int NKB, int SR, int QS>
hipError_t launch_dkdv(const BwdProblem& p, int cus, hipStream_t stream) {
    auto kernel = bwd_dkdv_pair_kernel<D, CAUSAL, OUT_BF16, NKB, SR, QS>;
    static const int per_cu = resident_per_cu(kernel, KV2_THREADS);
    constexpr int KT = 128 * NKB / QS;
    const int n_kt = (p.nk + KT - 1) / KT;
    const long long items = (long long)p.bh * n_kt;
    const unsigned grid = (unsigned)std::min<long long>(items, (long long)cus * per_cu);
    return launch_kernel(kernel, dim3(grid), dim3(KV2_THREADS), stream, static_cast<const u16*>(p.q),
                         static_cast<const u16*>(p.k), static_cast<const u16*>(p.v),
                         static_cast<const u16*>(p.dout), p.lse, static_cast<const float*>(p.dsum),
                         p.dk, p.dv, p.nq, p.nk, p.bh, n_kt, p.scale * kLog2e, p.scale);
}

// Choice of item size, by the items the busiest compute unit gets (`rounds`)
// and, under the causal mask, where the snake deal evens them out, by whether
// every unit gets one.  Backward calls, us, one box (MI355X, 256 units):
//
//   dQ                                 256-query items  128-query items, 2 key streams
//   B4 H8 1000, d = 64 (128 / 256)          59.7            44.7
//   B2 H8 1500, d = 128 (96 / 192)          101             81.8
//   same, causal                            100             80.0
//   B4 H12 2K, d = 128 (384 / 768)          353             345
//   B4 H16 1K, d = 64 (256 / 512)           78.9            81.4
//   B4 H12 2K causal, d = 64 (384 / 768)    124             128
//   16K causal, B1 H32, d = 128             6610            6840
//
// A 128-query item costs about 11/20 of a 256-query one.  Up to 128 queries a
// head is one item either way, and the second key stream has to earn its merge
// (B2 H15, both sides with the better dK, dV kernel):
//   61 x 61 d = 128 14.6 / 16.2, 64 x 64 d = 64 9.6 / 10.6, 128 x 128 d = 128
//   19.0 / 21.3; 128 x 384 d = 128 26.0 / 27.6, 64 x 512 27.0 / 27.2; 128 x 192
//   d = 64 13.6 / 14.6, 64 x 256 13.1 / 13.1, 128 x 384 16.7 / 16.6
// Nor does a 128-query item cost so little with few keys, where prologue and
// merge weigh more: if the items then need more rounds, 256-query ones stay up
// to 512 keys (whole calls):
//   causal, one round against two: 130 x 139 d = 64 18.7 / 24.8, d = 128 29.3 /
//   41.2, 130 x 256 d = 128 44.9 / 52.2, 100 x 400 51.4 / 60.3; 53 x 520 53.1 /
//   52.1, 40 x 1000 78.9 / 69.3
//   no mask, d = 128: 190 x 300 of 89 keys [2, 3 rounds] 41.6 / 51.2, of 512 109 / 121;
//   233 x 520 of 89 [3, 5] 70.4 / 83.0; 130 x 520 [2, 3] of 900 118 / 116
//
//   dK, dV                             128-key items    64-key items, 2 query streams
//   B1 H8 1K, d = 128 (64 / 128)            58.5            50.0
//   B1 H4 2K causal, d = 64 (64 / 128)      64.9            53.1
//   B2 H8 1500 causal, d = 128 (192 / 384)  80.2            68.1
//   B2 H8 1500, d = 128 (192 / 384)         82.9            97.4
//   B1 H20 1K, d = 64 (160 / 320)           40.2            46.7
//   B1 H5 8K causal, d = 128 (320 / 640)    366             363
//   B2 H15 64 x 64, d = 128 (30 / 30)       14.2            15.0
//   same, d = 64                            9.6             9.9
//   B2 H15 65 x 64, d = 64 (30 / 30)        11.0            11.0
//   B2 H15 64 x 128, d = 128 (30 / 60)      18.2            16.7
//
// (one 64-key item per head with at most one 64-query stage has nothing to split)
//
//   dK, dV, d = 64                     128-key items    256-key items (NKB = 2)
//   B2 H16 4K (1024 / 512)                  488             449
//   B4 H16 1K (512 / 256)                   78.9            72.2
//   B4 H12 2K causal (768 / 384)            124             119
//   B4 H16 700 causal (384 / 192)           42.9            51.0
//   B4 H8 1000 (256 / 128)                  49.7            59.7
//   300 x 44 causal (300 / 300)             18.0            20.4
//   600 x 256 causal (1200 / 600)           80.8            89.4
//   400 x 512 causal (1600 / 800)           134             144
//   400 x 700 causal (2400 / 1200)          213             205
//   32 x 2048 causal (512 / 256)            97.6            112
//   50 x 2048 causal (800 / 400)            133             125
//
// A 256-key item costs about 18/10 of a 128-key one; under the mask it needs
// more than 512 keys, and more items than units, to be evened out.
long long rounds(long long items, int cus) { return (items + cus - 1) / cus; }

template <int D, bool CAUSAL, bool OUT_BF16>
hipError_t launch(const BwdProblem& p, hipStream_t stream) {
    int cus = 0;
    hipError_t e = device_cus(stream, cus);
    if (e != hipSuccess) return e;
    // D and dQ (both have nothing to do without queries)
    if (p.bh > 0 && p.nq > 0) {
        const long long i1 = (long long)p.bh * ((p.nq + 255) / 256), i2 = (long long)p.bh * ((p.nq + 127) / 128);
        const bool short_keys = (p.nq <= 128 && p.nk <= (D == 128 ? 384 : 192)) ||
                                (rounds(i2, cus) > rounds(i1, cus) && p.nk <= 512);
        const bool split = !short_keys && (CAUSAL ? i1 < cus : 20 * rounds(i1, cus) > 11 * rounds(i2, cus));
        e = split ? launch_dq<D, CAUSAL, OUT_BF16, 2>(p, cus, stream)
                  : launch_dq<D, CAUSAL, OUT_BF16, 1>(p, cus, stream);
        if (e != hipSuccess) return e;
    }
    // dK, dV (zero when there are no queries)
    const long long k1 = (long long)p.bh * ((p.nk + 127) / 128);
    const bool one_stage = p.nq <= 64 && p.nk <= 64;
    if (!one_stage && (CAUSAL ? k1 < cus : 2 * k1 <= cus)) return launch_dkdv<D, CAUSAL, OUT_BF16, 1, 32, 2>(p, cus, stream);
    if constexpr (D == 64) {
        const long long k2 = (long long)p.bh * ((p.nk + 255) / 256);
        if (CAUSAL ? 4 * k2 >= 5 * cus && p.nk > 512 : 18 * rounds(k2, cus) <= 10 * rounds(k1, cus))
            return launch_dkdv<D, CAUSAL, OUT_BF16, 2, 64, 1>(p, cus, stream);
    }
    return launch_dkdv<D, CAUSAL, OUT_BF16, 1, 64, 1>(p, cus, stream);
}

template <int D>
hipError_t launch_d(const BwdProblem& p, hipStream_t stream) {
    if (p.causal)
        return p.grad_bf16 ? launch<D, true, true>(p, stream) : launch<D, true, false>(p, stream);
    return p.grad_bf16 ? launch<D, false, true>(p, stream) : launch<D, false, false>(p, stream);
}

}  // namespace

hipError_t launch_bwd(const BwdProblem& p, hipStream_t stream) {
    if (p.d == 64) return launch_d<64>(p, stream);
    if (p.d == 128) return launch_d<128>(p, stream);
    return hipErrorInvalidValue;
}

}  // namespace moa
