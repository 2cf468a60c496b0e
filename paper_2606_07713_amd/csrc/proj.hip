// Input projections Q = X W_Q, K = X W_K, V = X W_V (the paper's problem
// statement) on gfx950 matrix cores, written straight into the head-split
// [B][H][N][d] layout the attention kernels read.
//
// One launch computes all three projections as one matrix product
//   C^T[f][m] = sum_k Wt[f][k] * X[m][k],   m = b*N + n,  f = p*H*d + h*d + e,
// where Wt = [Wq; Wk; Wv] holds the weights transposed ([H*d][Dm] each, the
// layout of a dense layer's weight) and p selects the projection.  Both
// operands are read along k, their stored order, so neither is transposed.
// C^T orientation: the MFMA A operand is a weight row, the B operand an X
// row, and each lane's accumulator holds 4-feature runs of one token, which
// are stored as 8-byte bf16 groups (round to nearest even).
//
// Tiling: 256 features x 256 tokens per workgroup of 8 waves (128 x 64 each),
// or, for grids that would leave compute units idle, 128 x 128 per workgroup
// of 4 waves (64 x 64 each), two workgroups to a compute unit (choice in
// launch_proj).  Both walk k in planes of 32 (64 bytes of every operand row)
// through a ring of five planes in LDS, filled by direct-to-LDS loads; a
// wave's 16-byte chunks are XOR-swizzled by row so that the 16 lanes of a read
// hit all 64 banks.
//
// What bounds it is keeping the matrix cores fed: with a barrier and a cold
// start of the operand reads at every k step the first kernel here left them
// idle half of the time (448 us, 921 TFLOP/s on 4096 x 4096 x 12288).  So the
// operands of the next 16 k are read while the current ones multiply, across
// the barriers too: a plane's last products run after the barrier that ends
// it, beside the reads of the next plane.  Loads are issued three planes
// before the barrier that waits for them, for two planes at a time, whose 64
// bytes per row share a cache line.  324 us (1271 TFLOP/s); one read after
// each product instead of all of them first or last: 338 -> 317 us.  Wave
// priorities around the products: 2% slower.
//
// Output: the accumulators go through LDS so that device memory is written in
// whole rows of a wave's features rather than in 8-byte groups.
#include <type_traits>

#include "device_common.h"
#include "launch.h"
#include "prefill_bf16_common.h"
#include "proj.h"

namespace moa {
namespace {

using pf::barrier_no_fence;
using pf::device_cus;
using pf::wait_lgkmcnt0;
using pf::wait_vmcnt;

constexpr int PK = 32;          // k per plane
constexpr int ROWB = PK * 2;    // bytes of one row of a plane
constexpr int RING = 5;         // planes in LDS

struct ProjArgs {
    const u16* x;
    const u16* w[3];
    u16* out[3];
    int M, N, Dm, H, d, F;
    int tiles_m, tiles_f;
};

// Tile of workgroup p: every XCD takes a contiguous run of tiles (workgroups
// reach the XCDs round-robin), and a run walks groups of 8 token tiles
// feature tile by feature tile, so that the 32 tiles an XCD works on at a
// time share 4 + 8 operand panels in its L2.
__device__ __forceinline__ void tile_of(int p, int n, int tiles_m, int tiles_f, int& tm, int& tf) {
    constexpr int kXcds = 8, GM = 8;
    const int x = p % kXcds, per = n / kXcds, rem = n % kXcds;
    const int t = x * per + min(x, rem) + p / kXcds;
    const int g = t / (GM * tiles_f), r = t - g * GM * tiles_f;
    const int gm = min(GM, tiles_m - g * GM);
    tm = g * GM + r % gm;
    tf = r / gm;
}

// 16 bytes per lane from any address straight into LDS (wave-uniform base).
__device__ __forceinline__ void global_load16_to_lds(const void* src, void* lds_base) {
#if defined(__HIP_DEVICE_COMPILE__)
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                     (__attribute__((address_space(3))) void*)lds_base, 16, 0, 0);
#else
    (void)src; (void)lds_base;
#endif
}

// FB x MB blocks of 32 x 32 per wave, WF x WM waves.  WIDE: 64-bit row
// offsets, for rows so long that 16 of them pass the 4 GiB of a descriptor.
template <int FB, int MB, int WF, int WM, bool WIDE>
__global__ __launch_bounds__(WF * WM * 64, 1) void proj_kernel(ProjArgs a) {
    constexpr int TF = WF * FB * 32, TM = WM * MB * 32, WAVES = WF * WM;
    constexpr int PLANE = (TF + TM) * ROWB;
    constexpr int LW = TF / 16 / WAVES, LX = TM / 16 / WAVES;   // 1 KB loads (16 rows) per wave and plane
    static_assert(TF % (16 * WAVES) == 0 && TM % (16 * WAVES) == 0, "planes must split into wave loads");
    __shared__ __attribute__((aligned(1024))) unsigned char s0[PLANE];
    __shared__ __attribute__((aligned(1024))) unsigned char s1[PLANE];
    __shared__ __attribute__((aligned(1024))) unsigned char s2[PLANE];
    __shared__ __attribute__((aligned(1024))) unsigned char s3[PLANE];
    __shared__ __attribute__((aligned(1024))) unsigned char s4[PLANE];
    auto slot = [&](auto tag) -> unsigned char* {
        constexpr int S = decltype(tag)::value % RING;
        if constexpr (S == 0) return s0;
        else if constexpr (S == 1) return s1;
        else if constexpr (S == 2) return s2;
        else if constexpr (S == 3) return s3;
        else return s4;
    };

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = lane & 31, half = lane >> 5;
    int tm, tf;
    tile_of(blockIdx.x, gridDim.x, a.tiles_m, a.tiles_f, tm, tf);
    const int m0 = tm * TM, f0 = tf * TF, FT = 3 * a.F;

    // Loads: lane l of a load fills 16 bytes of row l / 4 of its 16 rows, the
    // logical chunk (l % 4) ^ (row >> 2 & 3).  16 features belong to one
    // projection; rows past the end read as zeros (descriptor bounds; WIDE:
    // the last row is read instead) and are never stored.
    const int lr = lane >> 2;
    const uint32_t chunk = (uint32_t)(((lane & 3) ^ ((lr >> 2) & 3)) * 16);
    const uint32_t row_bytes = (uint32_t)a.Dm * 2u;
    const uint32_t voff = (uint32_t)lr * row_bytes + chunk;
    const u16* base[LW + LX];
    int valid[LW + LX];
#pragma unroll
    for (int i = 0; i < LW; ++i) {
        const int f = min(f0 + (wave * LW + i) * 16, WIDE ? FT - 16 : FT), p = min(f / a.F, 2);
        const u16* wp = p == 0 ? a.w[0] : (p == 1 ? a.w[1] : a.w[2]);   // no dynamic indexing
        base[i] = wp + (size_t)(f - p * a.F) * a.Dm;
        valid[i] = min(16, FT - f);
    }
#pragma unroll
    for (int i = 0; i < LX; ++i) {
        const int m = min(m0 + (wave * LX + i) * 16, WIDE ? a.M - 1 : a.M);
        base[LW + i] = a.x + (size_t)m * a.Dm;
        valid[LW + i] = min(16, a.M - m);
    }
    // Planes 2j and 2j + 1, the two halves of each row's 128 bytes, back to back.
    auto load_pair = [&](int j, auto tag) __attribute__((always_inline)) {
        using T0 = decltype(tag);
        unsigned char* pa = slot(T0{});
        unsigned char* pb = slot(std::integral_constant<int, T0::value + 1>{});
#pragma unroll
        for (int i = 0; i < LW + LX; ++i) {
            const int dst = i < LW ? (wave * LW + i) * 1024 : TF * ROWB + (wave * LX + i - LW) * 1024;
            if constexpr (WIDE) {
                const char* src = reinterpret_cast<const char*>(base[i] + (size_t)min(lr, valid[i] - 1) * a.Dm) +
                                  chunk + (size_t)j * (2 * ROWB);
                global_load16_to_lds(src, pa + dst);
                global_load16_to_lds(src + ROWB, pb + dst);
            } else {
                const auto r = make_rsrc(base[i], (uint32_t)valid[i] * row_bytes);
                const uint32_t k = voff + (uint32_t)j * (2 * ROWB);
                buffer_load16_to_lds(r, pa + dst, k);
                buffer_load16_to_lds(r, pb + dst, k + ROWB);
            }
        }
    };
    constexpr int PAIR_LOADS = 2 * (LW + LX);

    // Operand reads: row r, chunk 2 kk + half; blocks 32 rows apart are immediates.
    const int wf = (wave / WM) * (FB * 32), wm = (wave % WM) * (MB * 32);
    uint32_t ra[2], rb[2];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
        const uint32_t c = (uint32_t)(((2 * kk + half) ^ ((col >> 2) & 3)) * 16);
        ra[kk] = (uint32_t)(wf + col) * ROWB + c;
        rb[kk] = (uint32_t)(TF + wm + col) * ROWB + c;
    }
    f32x16 acc[FB][MB];
#pragma unroll
    for (int i = 0; i < FB; ++i)
#pragma unroll
        for (int j = 0; j < MB; ++j) acc[i][j] = f32x16{};
    struct Frag { bf16x8 a[FB], b[MB]; };
    auto read = [&](Frag& f, const unsigned char* s, int kk) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < MB; ++j) f.b[j] = *reinterpret_cast<const bf16x8*>(s + rb[kk] + j * 32 * ROWB);
#pragma unroll
        for (int i = 0; i < FB; ++i) f.a[i] = *reinterpret_cast<const bf16x8*>(s + ra[kk] + i * 32 * ROWB);
    };
    auto mul = [&](const Frag& f) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < FB; ++i)
#pragma unroll
            for (int j = 0; j < MB; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[i], f.b[j], acc[i][j], 0, 0, 0);
    };

    const int pairs = a.Dm / 64;
    Frag F0, F1;
    // One read after each product while there are any.
    auto interleave = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < FB + MB; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // a product
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // an LDS read
        }
        __builtin_amdgcn_sched_group_barrier(0x008, FB * MB, 0);
    };
    // Planes 2j and 2j + 1.  On entry plane 2j has landed (all waves) and the
    // previous plane's last fragments wait in F1 (`first`: none do).  At the
    // middle barrier every wave has read plane 2j and all before it, so pair
    // j + 2 (`load`: it exists) may overwrite planes 2j - 1 and 2j; at the end
    // every wave waits for its part of pair j + 1 (`pend`: it exists).  The
    // reads of F1 are not waited for there: their plane is not overwritten
    // before the next middle barrier, which waits, or, after the last step,
    // the barrier before the output.
    auto step = [&](int j, auto tag, auto first, bool load, bool pend) __attribute__((always_inline)) {
        constexpr int S = decltype(tag)::value;   // slot of plane 2j
        const unsigned char* pa = slot(std::integral_constant<int, S>{});
        const unsigned char* pb = slot(std::integral_constant<int, S + 1>{});
        read(F0, pa, 0);
        if constexpr (!decltype(first)::value) {
            mul(F1);
            interleave();
        }
        __builtin_amdgcn_sched_barrier(0);
        read(F1, pa, 1);
        mul(F0);
        interleave();
        __builtin_amdgcn_sched_barrier(0);
        wait_lgkmcnt0();
        barrier_no_fence();
        if (load) load_pair(j + 2, std::integral_constant<int, S + 4>{});
        __builtin_amdgcn_sched_barrier(0);
        read(F0, pb, 0);
        mul(F1);
        interleave();
        __builtin_amdgcn_sched_barrier(0);
        read(F1, pb, 1);
        mul(F0);
        interleave();
        __builtin_amdgcn_sched_barrier(0);
        if (load) wait_vmcnt<PAIR_LOADS>(); else if (pend) wait_vmcnt<0>();
        barrier_no_fence();
    };
    using std::integral_constant;
    using std::true_type;
    using std::false_type;
    load_pair(0, integral_constant<int, 0>{});
    if (pairs > 1) {
        load_pair(1, integral_constant<int, 2>{});
        wait_vmcnt<PAIR_LOADS>();
    } else {
        wait_vmcnt<0>();
    }
    barrier_no_fence();
    step(0, integral_constant<int, 0>{}, true_type{}, 2 < pairs, 1 < pairs);
    // Five pairs bring the ring back to the same slots; every load of the
    // loop exists, so that its waits are exact.
    int j = 1;
    for (; j + 6 < pairs; j += 5) {
        step(j, integral_constant<int, 2>{}, false_type{}, true, true);
        step(j + 1, integral_constant<int, 4>{}, false_type{}, true, true);
        step(j + 2, integral_constant<int, 6>{}, false_type{}, true, true);
        step(j + 3, integral_constant<int, 8>{}, false_type{}, true, true);
        step(j + 4, integral_constant<int, 0>{}, false_type{}, true, true);
    }
    auto tail = [&](auto tag) __attribute__((always_inline)) {
        if (j < pairs) step(j, tag, false_type{}, j + 2 < pairs, j + 1 < pairs);
        ++j;
    };
    tail(integral_constant<int, 2>{});
    tail(integral_constant<int, 4>{});
    tail(integral_constant<int, 6>{});
    tail(integral_constant<int, 8>{});
    tail(integral_constant<int, 0>{});
    tail(integral_constant<int, 2>{});
    // The last step's closing barrier was passed with the reads of F1 still
    // out: once every wave has them, the ring is idle.
    wait_lgkmcnt0();
    barrier_no_fence();
    mul(F1);

    // Output through LDS (the idle ring): token rows of FB * 32 features, then
    // whole rows, 16 bytes per lane.
    constexpr int OB = FB * 64;               // bytes of a staged row
    constexpr int CH = OB / 16, RPI = 64 / CH;
    constexpr int AREA = MB * 32 * OB;
    static_assert(2 * AREA <= PLANE && WAVES <= 8, "two waves' rows per slot");
    unsigned char* st = (wave < 2 ? s0 : wave < 4 ? s1 : wave < 6 ? s2 : s3) + (wave & 1) * AREA;
#pragma unroll
    for (int j = 0; j < MB; ++j)
#pragma unroll
        for (int i = 0; i < FB; ++i)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int r = 32 * j + col, c = 4 * i + g;
                *reinterpret_cast<uint2*>(st + r * OB + ((c ^ (r & (CH - 1))) * 16) + half * 8) =
                    make_uint2(pack_bf16x2(acc[i][j][4 * g + 0], acc[i][j][4 * g + 1]),
                               pack_bf16x2(acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]));
            }
    wait_lgkmcnt0();   // only this wave reads its rows
    const int ch = lane % CH, rr = lane / CH;
    const int f = f0 + wf + ch * 8;
    if (f >= FT) return;
    const int p = f / a.F, fh = f - p * a.F, h = fh / a.d, e = fh - h * a.d;
    u16* op = (p == 0 ? a.out[0] : (p == 1 ? a.out[1] : a.out[2])) + (size_t)h * a.N * a.d + e;
    int b = (m0 + wm) / a.N, n = m0 + wm - b * a.N + rr;
#pragma unroll
    for (int i = 0; i < MB * 32 / RPI; ++i) {
        const int r = i * RPI + rr;
        while (n >= a.N) { n -= a.N; ++b; }
        const uint4 v = *reinterpret_cast<const uint4*>(st + r * OB + ((ch ^ (r & (CH - 1))) * 16));
        if (m0 + wm + r < a.M)
            *reinterpret_cast<uint4*>(op + ((size_t)b * a.H * a.N + n) * a.d) = v;
        n += RPI;
    }
}

template <int FB, int MB, int WF, int WM, bool WIDE = false>
hipError_t launch_tile(ProjArgs a, hipStream_t stream) {
    constexpr int TF = WF * FB * 32, TM = WM * MB * 32;
    a.tiles_m = (a.M + TM - 1) / TM;
    a.tiles_f = (3 * a.F + TF - 1) / TF;
    return launch_kernel(proj_kernel<FB, MB, WF, WM, WIDE>, dim3((unsigned)(a.tiles_m * a.tiles_f)),
                         dim3(WF * WM * 64), stream, a);
}

}  // namespace

// Choice of tile by the rounds of workgroups the grid takes, a round of
// 128 x 128 tiles (two per compute unit, half the work of a round of 256 x
// 256 tiles) costing about 23/40 of one.  Measured (us, 256 / 128 tiles, tile
// counts in brackets): 4096 tokens, Dm 4096, 12288 features [768 / 3072] 317
// / 373; 4500, 3008, 9216 [648 / 2592] 222 / 243; 8000, 1536, 3840 [480 /
// 1890] 89 / 99; 2000, 4032, 11520 [360 / 1440] 182 / 180; 2000, 2048, 3072
// [96 / 384] 46 / 32; 512, 512, 1536 [12 / 48] 15.0 / 7.6.
hipError_t launch_proj(const ProjProblem& p, hipStream_t stream) {
    if (p.m == 0) return hipSuccess;
    ProjArgs a;
    a.x = static_cast<const u16*>(p.x);
    for (int i = 0; i < 3; ++i) {
        a.w[i] = static_cast<const u16*>(p.w[i]);
        a.out[i] = static_cast<u16*>(p.out[i]);
    }
    a.M = p.m; a.N = p.n; a.Dm = p.dm; a.H = p.h; a.d = p.d; a.F = p.h * p.d;
    if (a.Dm >= (1 << 27)) return launch_tile<2, 2, 2, 2, true>(a, stream);
    int cus = 0;
    const hipError_t e = device_cus(stream, cus);
    if (e != hipSuccess) return e;
    const auto tiles = [&](long long t) { return ((p.m + t - 1) / t) * ((3LL * a.F + t - 1) / t); };
    const long long r256 = (tiles(256) + cus - 1) / cus, r128 = (tiles(128) + 2 * cus - 1) / (2 * cus);
    if (23 * r128 < 40 * r256) return launch_tile<2, 2, 2, 2>(a, stream);
    return launch_tile<4, 2, 2, 4>(a, stream);
}

}  // namespace moa
