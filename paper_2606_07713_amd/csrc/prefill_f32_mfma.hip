// Fused attention prefill for fp32 inputs and fp32 output on the fp32 matrix
// instruction v_mfma_f32_16x16x4_f32 (fp32 products and sums; no operand is
// rounded to bf16).
//
// One workgroup owns 16 query rows of one (batch*head); its W waves hold the
// same rows and walk disjoint key streams (wave w takes the 16-key blocks w,
// w + W, ...), and at the end all threads merge the streams' softmax states
// exactly, one float4 of O each.
//
// Orientation as in the bf16 prefill: S^T = K Q^T and O^T += V^T P^T.  The
// contraction order of an MFMA is free as long as both operands agree, which
// is used twice so that no operand needs LDS or a transpose:
//  * S^T: lane group h (of four 16-lane groups) holds the dims 16j + 4h ..
//    16j + 4h + 3 of its K row (A) and of its Q row (B), one 16-byte load per
//    four MFMAs;
//  * O^T: register i of the S^T accumulator holds, in lane group h, the score
//    of key 4h + i of the block; P^T register i is directly the B operand of
//    the MFMA that contracts those four keys, and A is V[that key][.], read
//    as whole rows: lane m of a group holds D / 16 consecutive dv values.
// K and V go from device memory (L2) straight to registers, one block ahead:
// K(next) is loaded while the weights of the current block and its P V
// products run, V(next) during the next S products (each half is 16 or 32
// MFMAs of 32 cycles).
//
// Rounding.  Sums are kept short: a score is the tree sum of D / 8 partial
// sums of two MFMAs each, and a block's P V products get an accumulator of
// their own that is then added to the running output.  The error against fp64
// (2-norm) is below that of the vector kernel this one took the place of on
// every shape measured: B1 H16 1K x 1K d = 64 causal 1.4e-7 (vector 1.65e-7),
// 4K x 4K 2.0e-7 (3.45e-7), B2 H8 1K d = 128 causal 1.5e-7 (1.8e-7).  One
// running accumulator per score and output was 1% faster and lost up to 1.9x
// of that precision.
//
// Bound by the fp32 matrix rate (157 TFLOP/s nominal; a large library product
// reaches 154) and, on small grids, by the latency of one block's loads.  us,
// raw calls, one box, against the vector kernel: B1 H16 1K d = 64 causal 26.1
// (84.2), without the mask 44.6 (92.5); B2 H8 1K d = 128 causal 53 (188); B4
// H16 2K d = 64 640 (1313, 107 against 52 TFLOP/s), d = 128 causal 685 (2140);
// B4 H8 256 d = 64 9.4 (15.5).  Without its loads the loop runs 10% faster;
// larger tiles (32 queries with v_mfma_f32_32x32x2_f32) or 32-key steps were
// no faster.  Under the causal mask all workgroups of a 1K grid are resident
// at once, so the snake order below decides the balance: 26.0 against 29.0 us.
#include <algorithm>

#include "device_common.h"
#include "launch.h"

namespace moa {
namespace {

constexpr int QT = 16;   // query rows per workgroup, and keys per block

// Max / sum over the four 16-lane groups (lanes with equal lane % 16).
__device__ __forceinline__ float groups_max(float x) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return half_max(fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1])));
}
__device__ __forceinline__ float groups_sum(float x) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return half_sum(__uint_as_float(r[0]) + __uint_as_float(r[1]));
}
__device__ __forceinline__ f32x4 mfma_f32(float a, float b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

template <int D, bool CAUSAL, int W>
__global__ __launch_bounds__(W * 64, 2) void prefill_f32_mfma_kernel(
    const float* __restrict__ Q, const float* __restrict__ K, const float* __restrict__ V,
    float* __restrict__ Out, float* __restrict__ LSE, int Nq, int Nk, int n_bh, int n_qtiles, int snake,
    float c, Layout L) {
    constexpr int NB = D / QT;            // output blocks = consecutive dv values per lane
    constexpr int CH = D / 16;            // 16-byte chunks of a K or Q row per lane
    constexpr int NS = D / 8;             // independent sums of a score
    // Merge area: per wave, QT rows of D floats (16-byte chunks XOR-swizzled
    // by the row), and (m, l) per row.
    __shared__ __attribute__((aligned(16))) float XO[W][QT * D];
    __shared__ float ML[W][2][QT];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // key stream
    const int m = lane & 15;      // query column; K row within a block; V column group
    const int h = lane >> 4;      // lane group
    // All heads of a query-tile rank together.  Under the causal mask the
    // heaviest tiles come first, and every second run of `snake` ranks (one
    // workgroup per compute unit) is reversed, so that the workgroups that
    // share a unit add up to about the same work.
    int rank = blockIdx.x / n_bh;
    const int bh = blockIdx.x - rank * n_bh;
    if (CAUSAL) {
        const int run = rank / snake, first = run * snake;
        if ((run & 1) && first + snake <= n_qtiles) rank = 2 * first + snake - 1 - rank;
    }
    const int qt = CAUSAL ? n_qtiles - 1 - rank : rank;
    const int q0 = qt * QT;
    const int qrow = q0 + m;
    const int off = Nk - Nq;

    const uint32_t krb = (uint32_t)L.kr * 4u, vrb = (uint32_t)L.vr * 4u;
    const auto rk = make_rsrc(K + head_offset(bh, L.H, L.kb, L.kh), rows_extent(Nk, krb, D * 4));
    const auto rv = make_rsrc(V + head_offset(bh, L.H, L.vb, L.vh), rows_extent(Nk, vrb, D * 4));

    const int kv_end = CAUSAL ? min(Nk, q0 + QT + off) : Nk;
    const int n_kt = (kv_end + QT - 1) / QT;

    // K row of this lane in block `kt` (rows past Nk repeat the last one;
    // their scores are masked), 16-byte chunks h, h + 4, ...
    float4 kf[CH], qf[CH];
    auto load_k = [&](int kt) {
        const uint32_t o = (uint32_t)min(kt * QT + m, Nk - 1) * krb + (uint32_t)h * 16u;
#pragma unroll
        for (int j = 0; j < CH; ++j) kf[j] = __builtin_bit_cast(float4, buffer_load16(rk, o + (uint32_t)j * 64u));
    };
    // V rows of block `kt`: the four keys 4h .. 4h + 3 that this lane's score
    // registers hold, the NB values from column NB * m.  Rows past Nk read as
    // zero (the last row in their place would turn an infinity in it, times the
    // weight 0 of a key that does not exist, into NaN).
    constexpr uint32_t kPastEnd = 0x80000000u;   // past any head slice (< 2 GiB)
    float4 vf[4][NB / 4];
    auto load_v = [&](int kt) {
        const uint32_t col = (uint32_t)m * (NB * 4u);
        const bool whole = kt * QT + QT <= Nk;
        const int row = kt * QT + 4 * h;
        const uint32_t o = (uint32_t)row * vrb + col;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t oi = whole || row + i < Nk ? o + (uint32_t)i * vrb : kPastEnd;
#pragma unroll
            for (int j = 0; j < NB / 4; ++j)
                vf[i][j] = __builtin_bit_cast(float4, buffer_load16(rv, oi + j * 16u));
        }
    };

    if (wave < n_kt) load_k(wave);
    {
        const float* qp = Q + head_offset(bh, L.H, L.qb, L.qh) + (size_t)min(qrow, Nq - 1) * L.qr + h * 4;
#pragma unroll
        for (int j = 0; j < CH; ++j) qf[j] = *reinterpret_cast<const float4*>(qp + j * 16);
    }
    if (wave < n_kt) load_v(wave);

    f32x4 acc[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[b] = f32x4{};
    float m_run = kNegInf, l_run = 0.0f;   // l_run: this lane's keys only

    for (int kt = wave; kt < n_kt; kt += W) {
        // S^T: NS independent sums over the dims, added as a tree: short
        // rounding chains, and no MFMA waits for the one before it.
        f32x4 s[NS];
#pragma unroll
        for (int j = 0; j < CH; ++j) {
            const float ka[4] = {kf[j].x, kf[j].y, kf[j].z, kf[j].w};
            const float qa[4] = {qf[j].x, qf[j].y, qf[j].z, qf[j].w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int i = 4 * j + e;
                s[i % NS] = mfma_f32(ka[e], qa[e], i < NS ? f32x4{} : s[i % NS]);
            }
        }
#pragma unroll
        for (int w = NS / 2; w >= 1; w /= 2)
#pragma unroll
            for (int i = 0; i < w; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) s[i][e] += s[i + w][e];
        float t[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) t[i] = s[0][i] * c;
        const bool more = kt + W < n_kt;
        if (more) load_k(kt + W);

        // Scores in log2 units; exact online softmax per block.
        const int kbase = kt * QT;
        if (kbase + QT > Nk || (CAUSAL && kbase + QT - 1 > q0 + off)) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int key = kbase + 4 * h + i;
                if (key >= Nk || (CAUSAL && key > qrow + off)) t[i] = kNegInf;
            }
        }
        float mx = t[0];
#pragma unroll
        for (int i = 1; i < 4; ++i) mx = fmaxf(mx, t[i]);
        const float m_new = fmaxf(m_run, groups_max(mx));
        // A row may have seen no visible key yet: weights of -inf scores are
        // then 2^(-inf - 0) = 0.
        const float ref = (m_new == kNegInf) ? 0.0f : m_new;
        const float alpha = exp2_hw(m_run - ref);   // 0 from a reference of -inf
        m_run = m_new;
        float ls = 0.0f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            t[i] = exp2_hw(t[i] - ref);
            ls += t[i];
        }
        l_run = __builtin_fmaf(l_run, alpha, ls);
        // The block's own output, then added to the running one (see Rounding).
        f32x4 blk[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) blk[b] = f32x4{};
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < NB / 4; ++j) {
                blk[4 * j + 0] = mfma_f32(vf[i][j].x, t[i], blk[4 * j + 0]);
                blk[4 * j + 1] = mfma_f32(vf[i][j].y, t[i], blk[4 * j + 1]);
                blk[4 * j + 2] = mfma_f32(vf[i][j].z, t[i], blk[4 * j + 2]);
                blk[4 * j + 3] = mfma_f32(vf[i][j].w, t[i], blk[4 * j + 3]);
            }
        if (more) load_v(kt + W);
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[b][e] = __builtin_fmaf(acc[b][e], alpha, blk[b][e]);
    }

    // Exact merge of the streams' states: every wave stores (m, l, acc), then
    // each thread finishes float4s of O:
    //   M = max_w m_w,  O = sum_w 2^(m_w - M) acc_w / sum_w 2^(m_w - M) l_w.
    // A stream without visible keys has m = -inf and adds nothing.  Register
    // e of block b holds dv = NB * (4h + e) + b of the lane's query.
    const float l_tot = groups_sum(l_run);
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int j = 0; j < NB / 4; ++j) {
            const int chunk = ((NB * (4 * h + e)) / 4 + j) ^ m;
            *reinterpret_cast<float4*>(&XO[wave][m * D + chunk * 4]) =
                make_float4(acc[4 * j][e], acc[4 * j + 1][e], acc[4 * j + 2][e], acc[4 * j + 3][e]);
        }
    if (h == 0) {
        ML[wave][0][m] = m_run;
        ML[wave][1][m] = l_tot;
    }
    __syncthreads();
    constexpr int OUT4 = QT * D / 4;   // float4 of the workgroup's output
    for (int i = threadIdx.x; i < OUT4; i += W * 64) {
        const int r = i / (D / 4), c4 = i % (D / 4);
        const int q = q0 + r;
        if (q >= Nq) break;            // rows ascend with i
        float mm = kNegInf;
#pragma unroll
        for (int w = 0; w < W; ++w) mm = fmaxf(mm, ML[w][0][r]);
        float ll = 0.0f;
        float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const float mw = ML[w][0][r];
            const float a = (mw == kNegInf) ? 0.0f : exp2_hw(mw - mm);
            ll = __builtin_fmaf(a, ML[w][1][r], ll);
            const float4 x = *reinterpret_cast<const float4*>(&XO[w][r * D + (c4 ^ r) * 4]);
            o.x = __builtin_fmaf(a, x.x, o.x);
            o.y = __builtin_fmaf(a, x.y, o.y);
            o.z = __builtin_fmaf(a, x.z, o.z);
            o.w = __builtin_fmaf(a, x.w, o.w);
        }
        const float inv = 1.0f / ll;
        const size_t obase = (size_t)head_offset(bh, L.H, L.ob, L.oh) + (size_t)q * L.orow;
        *reinterpret_cast<float4*>(Out + obase + c4 * 4) =
            make_float4(o.x * inv, o.y * inv, o.z * inv, o.w * inv);
        if (LSE != nullptr && c4 == 0) LSE[(size_t)bh * Nq + q] = (mm + __log2f(ll)) * kLn2;
    }
}

template <int D, bool CAUSAL, int W>
hipError_t launch_w(const Problem& p, int cus, hipStream_t stream) {
    const int n_qtiles = (p.nq + QT - 1) / QT;
    const long long blocks = (long long)p.bh * n_qtiles;
    return launch_kernel(prefill_f32_mfma_kernel<D, CAUSAL, W>, dim3((unsigned)blocks),
                         dim3(W * 64), stream, static_cast<const float*>(p.q),
                         static_cast<const float*>(p.k), static_cast<const float*>(p.v),
                         static_cast<float*>(p.o), p.lse, p.nq, p.nk, p.bh, n_qtiles,
                         std::max(1, cus / p.bh), p.scale * kLog2e, p.lay);
}

// Key streams per workgroup.  Four; eight where the grid leaves compute units
// short of waves and every stream still gets several blocks (us, 4 against 8
// streams): B1 H1 1K x 1K d = 64 15.4 / 14.6, 2K d = 128 46.5 / 44.2, B1 H4
// 100 x 4096 d = 64 52.0 / 45.7; on at most two workgroups per unit also under
// the causal mask at d = 128, whose tiles differ in length: B1 H6 1K 33.1 /
// 26.7.  Against: B1 H8 256 x 256 d = 128 9.8 / 10.7, B1 H3 700 x 700 19.1 /
// 19.6, B1 H6 1000 x 1000 d = 128 41.9 / 46.9, B1 H16 1K d = 64 26.1 / 30.7.
template <int D, bool CAUSAL>
hipError_t launch(const Problem& p, int cus, hipStream_t stream) {
    const long long blocks = (long long)p.bh * ((p.nq + QT - 1) / QT);
    if (p.nk >= 768 && blocks <= (CAUSAL && D == 128 ? 2 : 1) * cus)
        return launch_w<D, CAUSAL, 8>(p, cus, stream);
    return launch_w<D, CAUSAL, 4>(p, cus, stream);
}

}  // namespace

hipError_t launch_prefill_f32_mfma(const Problem& p, int cus, hipStream_t stream) {
    if (p.d == 64) return p.causal ? launch<64, true>(p, cus, stream) : launch<64, false>(p, cus, stream);
    if (p.d == 128) return p.causal ? launch<128, true>(p, cus, stream) : launch<128, false>(p, cus, stream);
    return hipErrorInvalidValue;
}

}  // namespace moa
