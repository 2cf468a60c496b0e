// bf16 prefill with small independent workgroups, for grids that the layouts
// of prefill_bf16.hip would run in uneven rounds (see use_indep there).
//
// One workgroup = 4 waves x 32 queries of one (b, h), one wave per SIMD; three
// workgroups (d = 64) or two (d = 128) share a compute unit.  K and V stream
// through a two-stage LDS ring in 64-key tiles, one barrier per tile, and each
// wave takes its 32-key steps one after the other: S^T = K Q^T, the softmax of
// prefill_bf16.hip, O^T += V^T P^T.  Nothing orders the phases of the waves
// that share a SIMD; the other workgroups fill the gaps of each.
//
// What bounds it is the sum of a SIMD's matrix and vector work, as in the
// ping-pong layout, and at full grids it only matches that one (32 x 4096 d =
// 64: 150 us both).  Its gain is the grain: a compute unit takes 128 queries at
// a time instead of 256, so grids of one and a half rounds do not pay for two,
// causal items reach less far past the diagonal, and a wave without queries
// costs nothing.  B8 H12 777 contiguous, d = 64: 38.4 -> 29.8 us (386 -> 498
// TFLOP/s), causal 29.6 -> 19.5; d = 128: 56.3 -> 53.1, causal 40.6 -> 35.7; in
// the packed layout 39.9 -> 30.9, 31.6 -> 20.0, 58.2 -> 57.4 and 41.8 -> 39.3.
//
// Registers: S and P are held for 32 keys at a time, which leaves 136 at d = 64,
// three waves per SIMD without a spill.  Four waves (128 registers, 6 to 12
// spilled in the loop) were slower on every grid: 176 x 777 45.0 against 43.5
// us, 102 x 1500 causal 50.4 / 45.2, packed B4 H12 3000 causal 95.3 / 71.8.  At d =
// 128 three waves spilled heavily (four times slower).
//
// The softmax step, the tile layout and the schedule are shared with
// prefill_bf16.hip; the operand addresses and the output rows are written out in
// both.  As common functions they left these kernels as they are and made the
// prologue of the key split with strided rows 0.3 to 0.5 us longer (packed d =
// 128, B4 H24 63 x 212 10.1 -> 10.5 us, B4 H5 359 x 359 causal 12.8 -> 13.3).
#include <algorithm>
#include <type_traits>

#include "device_common.h"
#include "launch.h"
#include "prefill_bf16_common.h"

namespace moa {
namespace {

using namespace pf;

constexpr int IW = kPrefillIndepRowsPerBlock / 32;   // waves per workgroup

template <int D, bool CAUSAL, bool OUT_BF16, bool STRIDED>
__global__ __launch_bounds__(IW * 64, (D == 64 ? 3 : 2)) void prefill_indep_kernel(
    const u16* __restrict__ Q, const u16* __restrict__ K, const u16* __restrict__ V,
    void* __restrict__ Out, float* __restrict__ LSE, int Nq, int Nk, int n_bh, int n_qtiles, float c,
    Layout L, int units, int renew) {
    const Addr<D, STRIDED> A{L, Nq, Nk};
    using C = Cfg<D>;
    constexpr uint32_t RB = C::ROW_BYTES;
    constexpr int BMQ = IW * 32;
    constexpr int SN = 32;                                // keys per step
    constexpr int LPW = C::TILE_BYTES / (IW * 1024);      // 16-byte loads per lane per tile
    // One array per ring stage: the compiler tracks direct-to-LDS loads per object.
    __shared__ __attribute__((aligned(1024))) unsigned char k_st0[C::TILE_BYTES];
    __shared__ __attribute__((aligned(1024))) unsigned char k_st1[C::TILE_BYTES];
    __shared__ __attribute__((aligned(1024))) unsigned char v_st0[C::TILE_BYTES];
    __shared__ __attribute__((aligned(1024))) unsigned char v_st1[C::TILE_BYTES];
    using S0 = std::integral_constant<int, 0>;
    using S1 = std::integral_constant<int, 1>;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = lane & 31, half = lane >> 5;
    const int off = Nk - Nq;
    // Negative, zero and denormal scales as in prefill_bf16.hip.
    const uint32_t qflip = (c < 0.0f) ? 0x80008000u : 0u;
    c = fmaxf(fabsf(c), 1.17549435e-38f);

    // The `units` compute units hold R workgroups each; workgroup p is the
    // (p / units)-th of unit p % units, and the deal (snaking under the mask)
    // runs over the units.
    const int P = min(units, (int)gridDim.x), R = ((int)gridDim.x + P - 1) / P;

    for (int item = 0;; ++item) {
        int bh, qt;
        if (!item_of(blockIdx.x % P, item * R + blockIdx.x / P, P, n_bh, n_qtiles, CAUSAL, bh, qt)) break;
        const int wq = qt * BMQ + wave * 32;      // this wave's first query
        const int qrow = wq + col;
        const u16* Qh = Q + A.q_head(bh);
        const u16* Kh = K + A.k_head(bh);
        const u16* Vh = V + A.v_head(bh);

        bf16x8 qf[D / 16];
        {
            const uint32_t qrb = (uint32_t)A.qr() * 2u;
            const auto rq = make_rsrc(Qh, rows_extent(Nq, qrb, RB));
#pragma unroll
            for (int s = 0; s < D / 16; ++s)
                qf[s] = __builtin_bit_cast(bf16x8, buffer_load16(rq, (uint32_t)qrow * qrb + s * 32 + half * 16));
        }
        // Key tiles of the workgroup and of this wave (none past Nq).
        const int n_kt = ((CAUSAL ? min(Nk, qt * BMQ + BMQ + off) : Nk) + BN - 1) / BN;
        int n_w = CAUSAL ? min(n_kt, (wq + 31 + off) / BN + 1) : n_kt;
        if (wq >= Nq) n_w = 0;
        // The tile a second reference is taken from (see launch_prefill_indep).
        const int t_renew = renew ? (n_kt + 1) / 2 : n_kt;

        const uint32_t krb = (uint32_t)A.kr() * 2u, vrb = (uint32_t)A.vr() * 2u;
        uint32_t ld_koff[LPW], ld_voff[LPW];
#pragma unroll
        for (int i = 0; i < LPW; ++i) {
            const int slot = (wave * LPW + i) * 64 + lane;
            const int row = slot / C::CHUNKS, p = slot % C::CHUNKS;
            const uint32_t chunk = (uint32_t)((p ^ swz<D>(row)) * 16);
            ld_koff[i] = (uint32_t)row * krb + chunk;
            ld_voff[i] = (uint32_t)row * vrb + chunk;
        }
        auto issue = [&](int t, auto stage) __attribute__((always_inline)) {
            unsigned char* ks = decltype(stage)::value == 0 ? k_st0 : k_st1;
            unsigned char* vs = decltype(stage)::value == 0 ? v_st0 : v_st1;
            const int kbase = t * BN;
            const auto rk = make_rsrc(Kh + (size_t)kbase * A.kr(), rows_extent(Nk - kbase, krb, RB));
            const auto rv = make_rsrc(Vh + (size_t)kbase * A.vr(), rows_extent(Nk - kbase, vrb, RB));
#pragma unroll
            for (int i = 0; i < LPW; ++i) buffer_load16_to_lds(rk, ks + (wave * LPW + i) * 1024, ld_koff[i]);
#pragma unroll
            for (int i = 0; i < LPW; ++i) buffer_load16_to_lds(rv, vs + (wave * LPW + i) * 1024, ld_voff[i]);
        };
        uint32_t kaddr[D / 16], vaddr[D / 32][2];
#pragma unroll
        for (int s = 0; s < D / 16; ++s)
            kaddr[s] = (uint32_t)col * RB + (uint32_t)(((2 * s + half) ^ swz<D>(col)) * 16);
        {
            const int g = lane >> 4, j = (lane >> 2) & 3, q = lane & 3;
#pragma unroll
            for (int b = 0; b < D / 32; ++b)
#pragma unroll
                for (int h8 = 0; h8 < 2; ++h8) {
                    const int row = 4 * (g >> 1) + j + 8 * h8;
                    const int dv = dv_of<D>(b, 16 * (g & 1) + 4 * q);
                    vaddr[b][h8] = (uint32_t)row * RB +
                                   (uint32_t)((((dv >> 3) ^ swz<D>(row)) * 16) + (dv & 7) * 2);
                }
        }

        f32x16 oacc[D / 32];
#pragma unroll
        for (int b = 0; b < D / 32; ++b) oacc[b] = f32x16{};
        float m_run = kNegInf;   // reference, log2 units
        float neg_m = 0.0f;      // -m_run, or 0 while m_run is -inf
        float l_run = 0.0f;      // partial denominator over this half-wave's keys

        auto tile = [&](int t, auto stage) __attribute__((always_inline)) {
            if (t >= n_w) return;
            const unsigned char* ks = decltype(stage)::value == 0 ? k_st0 : k_st1;
            unsigned char* vs = decltype(stage)::value == 0 ? v_st0 : v_st1;
            const int kbase = t * BN;
            const bool need_mask = (kbase + BN > Nk) || (CAUSAL && kbase + BN - 1 > wq + off);
#pragma unroll
            for (int sb = 0; sb < BN / SN; ++sb) {
                // S^T of the tile's 32-key step u, masked.
                auto scores = [&](int u) __attribute__((always_inline)) {
                    f32x16 x = f32x16{};
#pragma unroll
                    for (int s = 0; s < D / 16; ++s)
                        x = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                            *reinterpret_cast<const bf16x8*>(ks + kaddr[s] + u * SN * RB), qf[s], x, 0, 0, 0);
                    if (need_mask) {
#pragma unroll
                        for (int i = 0; i < 16; ++i) {
                            const int key = kbase + u * SN + (i >> 2) * 8 + half * 4 + (i & 3);
                            if (key >= Nk || (CAUSAL && key > qrow + off)) x[i] = kNegInf;
                        }
                    }
                    return x;
                };
                f32x16 sacc = scores(sb);
                auto raise_reference = [&](float mx, bool anew) __attribute__((always_inline)) {
                    asm volatile("" : "+v"(mx));   // not hoisted onto the fast path
#pragma unroll
                    for (int i = 0; i < 16; ++i) mx = fmaxf(mx, sacc[i]);
                    const float mt = half_max(mx) * c;
                    if (anew || wave_any(mt > m_run + kRescaleSlack)) {
                        const float m_new = fmaxf(anew ? m_run - kRenewDrop : m_run, mt + kRefHeadroom);
                        const float alpha = (m_run == kNegInf) ? 0.0f : exp2_hw(m_run - m_new);
                        l_run *= alpha;
#pragma unroll
                        for (int b = 0; b < D / 32; ++b) oacc[b] *= alpha;
                        m_run = m_new;
                        neg_m = (m_new == kNegInf) ? 0.0f : -m_new;
                    }
                };
                bf16x8 pbuf[SN / 16];
                auto exp_pack = [&]() __attribute__((always_inline)) {
                    float part[2] = {0.0f, 0.0f};
                    pack_weights(sacc, c, neg_m, pbuf, part);
                    return part[0] + part[1];
                };
                // A row's first reference comes from the whole tile, as in the
                // other layouts: the weight of the largest score is then a power
                // of two, exact in bf16, for as many rows (with 32 keys the error
                // of short causal rows was 2 to 7% larger).
                const bool anew = sb == 0 && t == t_renew;
                if (anew || wave_any(m_run == kNegInf)) {
                    float mx = kNegInf;
                    if (sb + 1 < BN / SN) {
                        const f32x16 next = scores(sb + 1);
#pragma unroll
                        for (int i = 0; i < 16; ++i) mx = fmaxf(mx, next[i]);
                    }
                    raise_reference(mx, anew);
                }
                float part = exp_pack();
                if (wave_any(!(part <= kFastSumLimit))) {
                    raise_reference(kNegInf, false);
                    part = exp_pack();
                }
                l_run += part;
#pragma unroll
                for (int cc = 0; cc < SN / 16; ++cc)
#pragma unroll
                    for (int b = 0; b < D / 32; ++b) {
                        const int row = (sb * (SN / 16) + cc) * 16;
                        const v4s both[2] = {
                            __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s*)(vs + vaddr[b][0] + row * RB)),
                            __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s*)(vs + vaddr[b][1] + row * RB))};
                        oacc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, both),
                                                                          pbuf[cc], oacc[b], 0, 0, 0);
                    }
            }
        };

        // Tile t sits in stage t & 1.  After the barrier at its start every
        // wave has its part of tile t in LDS and is done with tile t - 1, into
        // whose stage tile t + 1 is loaded while tile t is worked on.
        issue(0, S0{});
        if (qflip != 0u) {
#pragma unroll
            for (int s = 0; s < D / 16; ++s) {
                u32x4 w = __builtin_bit_cast(u32x4, qf[s]);
                w ^= qflip;
                qf[s] = __builtin_bit_cast(bf16x8, w);
            }
        }
        for (int t = 0; t < n_kt; t += 2) {
            wait_vmcnt<0>();
            __syncthreads();
            if (t + 1 < n_kt) issue(t + 1, S1{});
            tile(t, S0{});
            if (t + 1 >= n_kt) break;
            wait_vmcnt<0>();
            __syncthreads();
            if (t + 2 < n_kt) issue(t + 2, S0{});
            tile(t + 1, S1{});
        }
        __syncthreads();   // every wave is done with the stages

        // O = acc / l through a 32-row slice of the stages, whole rows per store.
        unsigned char* stg = (wave < 2 ? k_st0 : k_st1) + (wave & 1) * 32 * RB;
        const float l_tot = half_sum(l_run);
        const float inv = 1.0f / l_tot;
        int ln = lane;
        asm volatile("" : "+v"(ln));   // staging addresses are formed here, not above the loop
        const int cl = ln & 31, hf = ln >> 5;
        const size_t o_head = (size_t)A.o_head(bh);
        if constexpr (OUT_BF16) {
            constexpr int CHK = C::CHUNKS, RPI = 64 / CHK;
#pragma unroll
            for (int b = 0; b < D / 32; ++b)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int dv = dv_of<D>(b, g * 8 + hf * 4);
                    *reinterpret_cast<uint2*>(stg + (uint32_t)cl * RB +
                                              (uint32_t)((((dv >> 3) ^ (cl & (CHK - 1))) * 16) + (dv & 7) * 2)) =
                        make_uint2(pack_bf16x2(oacc[b][g * 4 + 0] * inv, oacc[b][g * 4 + 1] * inv),
                                   pack_bf16x2(oacc[b][g * 4 + 2] * inv, oacc[b][g * 4 + 3] * inv));
                }
            wait_lgkmcnt0();   // only this wave reads its rows
            const int rr = ln / CHK, ch = ln % CHK;
#pragma unroll
            for (int i = 0; i < 32 / RPI; ++i) {
                const int r = i * RPI + rr, q = wq + r;
                const uint4 v = *reinterpret_cast<const uint4*>(
                    stg + (uint32_t)r * RB + (uint32_t)((ch ^ (r & (CHK - 1))) * 16));
                if (q < Nq)
                    *reinterpret_cast<uint4*>(static_cast<u16*>(Out) + o_head + (size_t)q * A.orow() + ch * 8) = v;
            }
        } else {
            // fp32 rows in two passes of D / 2 columns
            constexpr int HB = D * 2, HCH = HB / 16, RPI = 64 / HCH;
            const int rr = ln / HCH, ch = ln % HCH;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
#pragma unroll
                for (int b = 0; b < D / 32; ++b)
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        if (dv_of<D>(b, g * 8) / (D / 2) != h) continue;
                        const int cc = (dv_of<D>(b, g * 8 + hf * 4) - h * (D / 2)) / 4;
                        *reinterpret_cast<float4*>(stg + (uint32_t)cl * HB +
                                                   (uint32_t)((cc ^ (cl & (HCH - 1))) * 16)) =
                            make_float4(oacc[b][g * 4 + 0] * inv, oacc[b][g * 4 + 1] * inv,
                                        oacc[b][g * 4 + 2] * inv, oacc[b][g * 4 + 3] * inv);
                    }
                wait_lgkmcnt0();
#pragma unroll
                for (int i = 0; i < 32 / RPI; ++i) {
                    const int r = i * RPI + rr, q = wq + r;
                    const float4 v = *reinterpret_cast<const float4*>(
                        stg + (uint32_t)r * HB + (uint32_t)((ch ^ (r & (HCH - 1))) * 16));
                    if (q < Nq)
                        *reinterpret_cast<float4*>(static_cast<float*>(Out) + o_head + (size_t)q * A.orow() +
                                                   h * (D / 2) + ch * 4) = v;
                }
                wait_lgkmcnt0();
            }
        }
        if (LSE != nullptr && half == 0 && qrow < Nq)
            LSE[(size_t)bh * Nq + qrow] = (m_run + __log2f(l_tot)) * kLn2;
        // The next item's first tile lands in LDS that other waves may still
        // be reading their rows from (no memory fence: nothing here reads the
        // stores just issued).
        wait_lgkmcnt0();
        barrier_no_fence();
    }
}

template <int D, bool CAUSAL, bool OUT_BF16, bool STRIDED>
hipError_t launch(const Problem& p, int cus, bool renew, hipStream_t stream) {
    auto kernel = prefill_indep_kernel<D, CAUSAL, OUT_BF16, STRIDED>;
    static const int per_cu = [&] {
        int n = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kernel, IW * 64, 0) != hipSuccess) n = 1;
        return n > 0 ? n : 1;
    }();
    const int qt = (p.nq + IW * 32 - 1) / (IW * 32);
    // Whole layers of one workgroup per compute unit (the deal counts on
    // them; a workgroup without an item ends at once), up to what is resident.
    const long long items = (long long)p.bh * qt;
    const unsigned grid = (unsigned)(items < cus ? items : cus * std::min<long long>((items + cus - 1) / cus, per_cu));
    return launch_kernel(kernel, dim3(grid), dim3(IW * 64), stream, static_cast<const u16*>(p.q),
                         static_cast<const u16*>(p.k), static_cast<const u16*>(p.v), p.o, p.lse, p.nq,
                         p.nk, p.bh, qt, p.scale * kLog2e, p.lay, cus, renew ? 1 : 0);
}

template <int D, bool STRIDED>
hipError_t launch_s(const Problem& p, int cus, bool renew, hipStream_t stream) {
    if (p.causal)
        return p.out_bf16 ? launch<D, true, true, STRIDED>(p, cus, renew, stream)
                          : launch<D, true, false, STRIDED>(p, cus, renew, stream);
    return p.out_bf16 ? launch<D, false, true, STRIDED>(p, cus, renew, stream)
                      : launch<D, false, false, STRIDED>(p, cus, renew, stream);
}

}  // namespace

// `renew`: on grids that the key split would otherwise run, a row takes a
// second reference from the tile at which the key split's second stream would
// start.  The weight of a reference's own score is a power of two, exact in
// bf16, so with one reference instead of two the error against fp64 was 3.6%
// larger on average over 100 to 600 keys (7.6% at 203 x 183 d = 64).
hipError_t launch_prefill_indep(const Problem& p, int cus, bool renew, hipStream_t stream) {
    if (p.d == 64)
        return is_contiguous(p) ? launch_s<64, false>(p, cus, renew, stream)
                                : launch_s<64, true>(p, cus, renew, stream);
    if (p.d == 128)
        return is_contiguous(p) ? launch_s<128, false>(p, cus, renew, stream)
                                : launch_s<128, true>(p, cus, renew, stream);
    return hipErrorInvalidValue;
}

}  // namespace moa
