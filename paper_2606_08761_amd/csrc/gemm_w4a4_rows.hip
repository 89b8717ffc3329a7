// W4A4 group GEMM for few rows (decode, small batches, short prompts; up to
// kRowsMax rows) at one group per 128-wide K stage or more (G >= 128, or per
// channel) on gfx950.
//
// Same result as the tile kernels (APEX4 Sec. 3.2.1, Eq. group_decomposition).
// What bounds it: up to about 64 rows streaming the weights from HBM once and
// the fixed latency of a short kernel; past that the VALU work of widening and
// dequantizing.  So the kernel is short (a cold instruction cache costs as much
// as the memory latency at these sizes), keeps several workgroups per CU
// instead of a deep load ring per wave, and has one barrier before and two
// after its loop.
//   * A workgroup owns 32 CT columns by ROWS rows (ROWS = 16, or 32 RB) over
//     all of K; its NW waves take the 128-wide stages in turn (wave w: w,
//     w + NW, ...), so neighbouring waves read neighbouring 2 KB blocks of the
//     tiled weights.  Nothing is shared between waves inside the loop: no
//     barrier, and waves of a SIMD drift apart, which overlaps one's MFMAs with
//     another's vector work.  The waves' fp32 partial tiles (per channel: exact
//     int32 sums) are added in wave order through LDS at the end.
//   * Loads are buffer loads with the stage in the scalar offset and the range
//     in the descriptor: rows past M, columns past N and stages past K read as
//     zero without a branch, a mask or memory traffic, so that every load is
//     issued on every path and each stage waits for its own loads only.
//   * PF = 2 stages in flight per wave.  Measured on MI355X (N = K = 8192,
//     16 rows, weights past the cache): 8.9 us with two stages and several
//     workgroups per CU, 9.3 with three, 9.7 with four, 10.4 with six and one
//     workgroup per CU.
//   * Row-major operands (the activations, and weights of that layout) are read
//     16 rows by 64 bytes per instruction (lane l: row l % 16, bytes
//     16 (l / 16)), whole 64-byte segments of a row, which is the 16-row MFMA's
//     operand; 32-row operands are put together from two such loads with
//     v_permlane16_swap.  Lanes reading the 32 bytes of a 32-row operand directly
//     touch twice as many segments per instruction: activations 4-15 % slower
//     from 64 rows on; weights 2-5 % at 2 to 32 rows (8 rows, N = 8192,
//     K = 28672: 27.2 -> 26.0 us; 32 rows, N = 8448: 60.6 -> 55.6).  The layout is
//     a template argument: besides, tiled weights below 16 MB came out 3-7 %
//     faster than with both in one kernel (16 rows and fewer, per channel, most).
//   * Up to 16 rows: v_mfma_i32_16x16x64_i8, so no lane carries a row past 16:
//     half the activation widening and half the MFMA time of the 32-row form.
//     A lane's 32 bytes of tiled weights become the operands of two 16-column
//     blocks by four v_permlane16_swap.
//   * Dequantization per stage as in the other kernels: the accumulator starts
//     from 1.5 * 2^23, so the group (or 128-wide partial) sum reads as binary32,
//     t = fma(D, s_w / 256, -1.5 * 2^23 s_w / 256), acc = fma(t, s_a, acc).
//     Up to 32 rows a group of several stages is split into 128-wide partials,
//     as in the persistent few-row kernel: that changes only the fp32 rounding.
//   * Past 32 rows (kWhole) a wave takes all stages of a group, one after the
//     other, and the int32 sum meets the scales once, as in the tile kernels
//     (binary32 partials of a group that cancel would leave 2^-24 of the
//     partials, not of their sum).  The waves then share the groups, not the
//     stages: uneven where K/G is not a multiple of the waves.
//   * Per channel (CH): the int32 sums run over all of the wave's stages, the
//     waves' sums are added exactly and scaled once (the same bits as the tile
//     kernels); K % 128 != 0 only occurs here, and pieces past the row's end
//     are sent out of the descriptor's range, so they read as zero.
//   * Tiled weights read by one workgroup only (one block of rows) are loaded
//     nontemporal when they are large: 6 % (N = K = 8192) to 13 % (N = 57344)
//     faster than with the default policy when they come from HBM, 2 % slower
//     when they sit in the Infinity Cache.
//   * FUSE (one row): x is quantized into LDS in the prologue with the
//     quantizer's own arithmetic (quant_core.h: the same codes and scales);
//     workgroup 0 also writes them to the caller's work buffers.
//   * DUMP: the exact group sums of rows [pm0, pm0 + pmr): stage partials are
//     added with integer atomics into the zeroed P (per channel: stored once).
//     sa == nullptr: no scales read, no Y written.
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <type_traits>
#include <utility>

#include "apex4_internal.h"
#include "quant_core.h"

namespace apex4 {
namespace {

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));
typedef int i32x16 __attribute__((ext_vector_type(16)));

constexpr uint32_t MAGIC_BITS = 0x4B400000u;  // binary32 1.5 * 2^23
constexpr float MAGIC = 12582912.0f;
constexpr int RSRC_FLAGS = 0x00027000;        // raw buffer descriptor, 32-bit data format
constexpr int NONTEMPORAL = 2;                // cache policy bit of the buffer loads
constexpr int ROWS_LDS = 160 * 1024;          // LDS per workgroup on gfx950

__device__ __forceinline__ float rh2f(uint16_t b) { return __half2float(__ushort_as_half(b)); }
__device__ __forceinline__ i32x4 rfrag(uint32_t w0, uint32_t w1) {
    i32x4 r;
    r[0] = static_cast<int>((w0 << 4) & 0xF0F0F0F0u);
    r[1] = static_cast<int>(w0 & 0xF0F0F0F0u);
    r[2] = static_cast<int>((w1 << 4) & 0xF0F0F0F0u);
    r[3] = static_cast<int>(w1 & 0xF0F0F0F0u);
    return r;
}

template <int N, int... I, typename F>
__device__ __forceinline__ void unroll_impl(F& f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void unroll(F&& f) {
    unroll_impl<N>(f, std::make_integer_sequence<int, N>{});
}

// Rows, accumulators per lane and LDS layout of a form.  RB = 0: 16 rows.
template <int RB, int CT>
struct Form {
    static constexpr int ROWS = RB == 0 ? 16 : 32 * RB;
    static constexpr int COLS = 32 * CT;
    static constexpr int NRT = RB == 0 ? 8 : 16 * RB;  // per 32-column tile
    static constexpr int NR = NRT * CT;
    static constexpr int red_bytes(int nw) { return nw * NR * 64 * 4; }
    static constexpr int64_t scale_bytes(int64_t ng) { return ((ROWS + COLS) * ng * 2 + 15) / 16 * 16; }
};

// What meets the scales: a stage's sum (up to 32 rows, and G = 128), a whole
// group's (several stages, one after the other in one wave), or the row's.
enum RowsMode : int { kStage, kWhole, kChan };

template <int RB, int CT, int NW, int PF, int OCC, bool WT, bool NT, int MODE, bool DUMP, int QL>
__global__ __launch_bounds__(64 * NW, OCC) void w4a4_rows_kernel(
    const uint8_t* __restrict__ Aq, const uint16_t* __restrict__ sa, const uint8_t* __restrict__ Wq,
    const uint16_t* __restrict__ sw, int M, int N, int K, int lg, int ng, uint16_t* __restrict__ Y,
    const uint16_t* __restrict__ x, uint8_t* __restrict__ aq_out, uint16_t* __restrict__ sa_out,
    int32_t* __restrict__ P, int pm0, int pmr) {
    using F = Form<RB, CT>;
    constexpr int ROWS = F::ROWS, COLS = F::COLS, NRT = F::NRT, NR = F::NR;
    constexpr int THREADS = 64 * NW;
    constexpr int NA = RB == 0 ? 1 : 2 * RB;  // 16-byte activation loads per stage
    constexpr bool FUSE = QL > 0, CH = MODE == kChan, WHOLE = MODE == kWhole;
    static_assert(!FUSE || (RB == 0 && MODE == kStage), "the fused prologue quantizes one row");
    const bool have_sc = FUSE || !DUMP || sa != nullptr;  // uniform
    // scales group-major ([ng][ROWS], then [ng][COLS]), then (FUSE) the row's
    // codes; the reduction reuses the place, past the scales per channel
    extern __shared__ uint4 rows_lds[];
    uint16_t* asc = reinterpret_cast<uint16_t*>(rows_lds);
    uint16_t* wsc = asc + ng * ROWS;
    uint8_t* codes = reinterpret_cast<uint8_t*>(rows_lds) + ((ROWS + COLS) * ng * 2 + 15) / 16 * 16;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, lh = lane >> 5, l16 = lane & 15, lq = lane >> 4;
    const int nks = (K + 127) / 128, kb = K / 2;
    // Workgroup b runs on XCD b % 8 (round-robin dispatch), each with its own
    // L2: the row blocks of one column tile are consecutive workgroups of one
    // XCD, so that its weights come from HBM once.
    const int rblocks = (M + ROWS - 1) / ROWS;
    const int bj = static_cast<int>(blockIdx.x >> 3);
    const int ct = (bj / rblocks) * 8 + static_cast<int>(blockIdx.x & 7);
    const int n0 = ct * COLS, m0 = (bj % rblocks) * ROWS;
    if (n0 >= N) return;  // the last eight tiles' spare workgroups
    // a wave's i-th stage, and the stages per wave (the last may be past K)
    auto stage_of = [&](int i) __attribute__((always_inline)) {
        return WHOLE ? ((i >> lg) * NW + wave) << lg | (i & ((1 << lg) - 1)) : wave + NW * i;
    };
    const int n = WHOLE ? (ng + NW - 1) / NW << lg : (nks + NW - 1) / NW;

    // ---- scales: 16-byte vectors of eight groups of a row where K/G is a
    // multiple of 8, else pairs where it is even (rows are 4-byte aligned then),
    // else one by one; consecutive lanes on consecutive rows (the 2-byte LDS
    // stores of a wave then land side by side).  Two vectors or eight pairs per
    // thread are loaded before the ring (behind it they would wait for it), the
    // rest (long K) after it.
    const int nv = ng >> 3;
    const int nvec = ((ng & 7) == 0 && have_sc) ? ((FUSE ? 0 : ROWS) + COLS) * nv : 0;
    struct Slot {
        bool a;
        int r, c;
    };
    auto slot_of = [&](int i) __attribute__((always_inline)) {
        const bool a = !FUSE && i < ROWS * nv;
        const int q = (FUSE || a) ? i : i - ROWS * nv;
        return Slot{a, a ? q % ROWS : q % COLS, a ? q / ROWS : q / COLS};
    };
    auto sc_load = [&](int i) __attribute__((always_inline)) {
        v4u v = {0, 0, 0, 0};
        if (i < nvec) {
            const Slot s = slot_of(i);
            const uint16_t* p = s.a ? sa + static_cast<int64_t>(min(m0 + s.r, M - 1)) * ng
                                    : sw + static_cast<int64_t>(min(n0 + s.r, N - 1)) * ng;
            v = *reinterpret_cast<const v4u*>(p + 8 * s.c);
        }
        return v;
    };
    auto sc_store = [&](int i, v4u v) __attribute__((always_inline)) {
        if (i < nvec) {
            const Slot s = slot_of(i);
            const int stride = s.a ? ROWS : COLS;
            uint16_t* d = (s.a ? asc : wsc) + 8 * s.c * stride + s.r;
#pragma unroll
            for (int e = 0; e < 8; ++e) d[e * stride] = static_cast<uint16_t>(v[e >> 1] >> (16 * (e & 1)));
        }
    };
    constexpr int A_LINES = FUSE ? 0 : ROWS, LINES = A_LINES + COLS, SU = 8;
    const int npair = ((ng & 7) != 0 && (ng & 1) == 0 && have_sc) ? LINES * (ng >> 1) : 0;
    uint32_t sv[SU];
    auto pair_load = [&](int b0) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < SU; ++u) {
            if (b0 + u * THREADS >= npair) continue;  // uniform
            const int i = min(b0 + tid + u * THREADS, npair - 1), c = i / LINES, r = i % LINES;
            sv[u] = *reinterpret_cast<const uint32_t*>((r < A_LINES ? sa + static_cast<int64_t>(min(m0 + r, M - 1)) * ng
                                                                    : sw + static_cast<int64_t>(min(n0 + r - A_LINES, N - 1)) * ng) + 2 * c);
        }
    };
    auto pair_store = [&](int b0) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < SU; ++u) {
            if (b0 + u * THREADS >= npair) continue;
            const int i = min(b0 + tid + u * THREADS, npair - 1), c = i / LINES, r = i % LINES;
            const int stride = r < A_LINES ? ROWS : COLS;
            uint16_t* d = (r < A_LINES ? asc + r : wsc + r - A_LINES) + 2 * c * stride;
            d[0] = static_cast<uint16_t>(sv[u]);
            d[stride] = static_cast<uint16_t>(sv[u] >> 16);
        }
    };
    if (nvec > 0) {
        const v4u a = sc_load(tid), b = sc_load(tid + THREADS);
#pragma unroll
        for (int e = 0; e < 4; ++e) sv[e] = a[e], sv[4 + e] = b[e];
    } else if (npair > 0) {
        pair_load(0);
    }

    // ---- ring of PF stages; offsets within 32 bits (operands below 4 GiB)
    const uint32_t wbytes = WT ? static_cast<uint32_t>((N + 31) / 32) * static_cast<uint32_t>(nks) * 2048u
                               : static_cast<uint32_t>(N) * static_cast<uint32_t>(kb);
    const uint32_t abytes = static_cast<uint32_t>(M) * static_cast<uint32_t>(kb);
    const int w_ss = WT ? 2048 : 64;
    // a 32-column tile past the last one (odd tile count, CT = 2) starts at or past wbytes
    uint32_t wv[2 * CT];
#pragma unroll
    for (int c = 0; c < 2 * CT; ++c) {
        const int t = ct * CT + c / 2, col = n0 + 16 * c + l16;
        if (WT) wv[c] = 32 * t < N ? static_cast<uint32_t>(t) * static_cast<uint32_t>(nks) * 2048u + 1024u * (c & 1) + 16u * lane : 0xFFFFFFF0u;
        else wv[c] = col < N ? static_cast<uint32_t>(col) * static_cast<uint32_t>(kb) + 16u * lq : 0xFFFFFFF0u;
    }
    uint32_t av[NA];
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        const int row = m0 + 16 * i + l16;
        av[i] = row < M ? static_cast<uint32_t>(row) * static_cast<uint32_t>(kb) + 16u * lq : 0xFFFFFFF0u;
    }
    v4u rw[PF][2 * CT], ra[PF][NA];
    auto load = [&](auto J, int i) __attribute__((always_inline)) {
        constexpr int j = decltype(J)::value;
        const int s = stage_of(i);
        const bool live = s < nks;  // uniform: a stage past K loads from an empty range
        const auto wr = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(Wq), 0, live ? wbytes : 0u, RSRC_FLAGS);
        const int ws = live ? s * w_ss : 0, as = live ? s * 64 : 0;
        // bytes of the stage inside a row: below 64 only in the last stage per channel
        const uint32_t lim = CH ? static_cast<uint32_t>(kb - s * 64) : 64u;
#pragma unroll
        for (int c = 0; c < 2 * CT; ++c) {
            const uint32_t v = (!CH || WT || 16u * lq < lim) ? wv[c] : 0xFFFFFFF0u;  // (the tiled layout is zero padded)
            rw[j][c] = __builtin_bit_cast(v4u, __builtin_amdgcn_raw_buffer_load_b128(wr, v, ws, NT ? NONTEMPORAL : 0));
        }
        if constexpr (!FUSE) {
            const auto ar = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(Aq), 0, live ? abytes : 0u, RSRC_FLAGS);
#pragma unroll
            for (int i2 = 0; i2 < NA; ++i2) {
                const uint32_t v = (!CH || 16u * lq < lim) ? av[i2] : 0xFFFFFFF0u;
                ra[j][i2] = __builtin_bit_cast(v4u, __builtin_amdgcn_raw_buffer_load_b128(ar, v, as, 0));
            }
        }
    };
    unroll<PF>([&](auto J) __attribute__((always_inline)) { load(J, decltype(J)::value); });

    if constexpr (FUSE) {
        // SymQuant of x in slots of 8 values, QL = G / 8 consecutive slots (lanes) per group
        constexpr int FQ = 4;  // 16-byte loads of x in flight per thread
        const int nslots = K / 8;
        for (int base = 0; base < nslots; base += FQ * THREADS) {
            uint4 v[FQ];
#pragma unroll
            for (int u = 0; u < FQ; ++u) {
                const int s = base + tid + u * THREADS;
                v[u] = s < nslots ? *reinterpret_cast<const uint4*>(x + static_cast<int64_t>(s) * 8) : make_uint4(0u, 0u, 0u, 0u);
            }
#pragma unroll
            for (int u = 0; u < FQ; ++u) {
                const int s = base + tid + u * THREADS;
                if (base + u * THREADS >= nslots) continue;  // uniform
                uint16_t sbits;
                const uint32_t am = quant::group_max<QL>(quant::absmax8_bits(v[u]));
                const float sf = quant::scale_of(am, &sbits);
                const uint32_t packed = quant::pack8(v[u], sf, quant::inv_of(sf));
                if (s < nslots) {
                    reinterpret_cast<uint32_t*>(codes)[s] = packed;
                    const bool lead = (s & (QL - 1)) == 0;
                    if (lead) asc[s / QL * ROWS] = sbits;
                    if (blockIdx.x == 0) {
                        reinterpret_cast<uint32_t*>(aq_out)[s] = packed;
                        if (lead) sa_out[s / QL] = sbits;
                    }
                }
            }
        }
    }
    if (nvec > 0) {
        sc_store(tid, v4u{sv[0], sv[1], sv[2], sv[3]});
        sc_store(tid + THREADS, v4u{sv[4], sv[5], sv[6], sv[7]});
        for (int i = tid + 2 * THREADS; i < nvec; i += THREADS) sc_store(i, sc_load(i));
    } else if (npair > 0) {
        pair_store(0);
        for (int b0 = SU * THREADS; b0 < npair; b0 += SU * THREADS) {
            pair_load(b0);
            pair_store(b0);
        }
    } else if (have_sc) {
        for (int i = tid; i < LINES * ng; i += THREADS) {
            const int g = i / LINES, r = i % LINES;
            if (r < A_LINES) asc[g * ROWS + r] = sa[static_cast<int64_t>(min(m0 + r, M - 1)) * ng + g];
            else wsc[g * COLS + r - A_LINES] = sw[static_cast<int64_t>(min(n0 + r - A_LINES, N - 1)) * ng + g];
        }
    }
    // accumulators: binary32, the int32 sums of the group in progress or of the row
    using Acc = std::conditional_t<RB == 0, i32x4, i32x16>;
    constexpr int AV = RB == 0 ? 4 : 16;
    constexpr int NB = RB == 0 ? 2 : RB;  // MFMA results per column tile: column halves, or row blocks
    float acc[CH ? 1 : CT][CH ? 1 : NRT];
    constexpr bool INT = CH || WHOLE;
    Acc isum[INT ? CT : 1][INT ? NB : 1];
    if constexpr (INT) {
#pragma unroll
        for (int c = 0; c < CT; ++c)
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int r = 0; r < AV; ++r) isum[c][b][r] = 0;
    }
    if constexpr (!CH) {
#pragma unroll
        for (int c = 0; c < CT; ++c)
#pragma unroll
            for (int r = 0; r < NRT; ++r) acc[c][r] = 0.f;
    }
    __syncthreads();

    auto row_of = [&](int b, int r) { return RB == 0 ? 4 * lq + r : 32 * b + 8 * (r >> 2) + 4 * lh + (r & 3); };
    auto col_of = [&](int b) { return RB == 0 ? 16 * b + l16 : l32; };
    auto process = [&](auto J, int i) __attribute__((always_inline)) {
        constexpr int j = decltype(J)::value;
        const int s = stage_of(i), g = s >> lg;
        const bool deq = !CH && have_sc && (!WHOLE || ((i + 1) & ((1 << lg) - 1)) == 0);  // uniform
        // activation operands: b = row block (RB >= 1) of four MFMAs, or the one
        // 16-row operand of two
        constexpr int KM = RB == 0 ? 2 : 4;
        i32x4 af[RB == 0 ? 1 : RB][KM];
        // 16 rows by 64 bytes in each of a, b <-> 32 rows by 32 bytes (the low and the high 16 of each half)
        auto swap16 = [&](v4u& a, v4u& b) __attribute__((always_inline)) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const auto t = __builtin_amdgcn_permlane16_swap(a[e], b[e], false, false);
                a[e] = t[0];
                b[e] = t[1];
            }
        };
        if constexpr (RB == 0) {
            v4u a;
            if constexpr (FUSE) a = *reinterpret_cast<const v4u*>(codes + s * 64 + 16 * lq);
            else a = ra[j][0];
            af[0][0] = rfrag(a[0], a[1]);
            af[0][1] = rfrag(a[2], a[3]);
        } else {
#pragma unroll
            for (int b = 0; b < RB; ++b) {
                v4u h[2] = {ra[j][2 * b], ra[j][2 * b + 1]};
                swap16(h[0], h[1]);
#pragma unroll
                for (int kk = 0; kk < 4; ++kk) af[b][kk] = rfrag(h[kk >> 1][2 * (kk & 1)], h[kk >> 1][2 * (kk & 1) + 1]);
            }
        }
        uint2 sah[RB == 0 ? 1 : RB][AV / 4];
        if (deq) {
#pragma unroll
            for (int b = 0; b < (RB == 0 ? 1 : RB); ++b)
#pragma unroll
                for (int q = 0; q < AV / 4; ++q)
                    sah[b][q] = *reinterpret_cast<const uint2*>(&asc[g * ROWS + (RB == 0 ? 4 * lq : 32 * b + 8 * q + 4 * lh)]);
        }
        // (DUMP adds the bias after the sums are taken: the registers run out)
        Acc start;
#pragma unroll
        for (int r = 0; r < AV; ++r) start[r] = DUMP ? 0 : static_cast<int>(MAGIC_BITS);
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            float s1[RB == 0 ? 2 : 1];
#pragma unroll
            for (int b = 0; b < (RB == 0 ? 2 : 1); ++b)
                s1[b] = deq ? rh2f(wsc[g * COLS + 32 * c + col_of(b)]) * (1.0f / 256.0f) : 0.f;
            Acc d[NB];
            v4u w[2] = {rw[j][2 * c], rw[j][2 * c + 1]};
            if constexpr (WT == (RB == 0)) swap16(w[0], w[1]);
            if constexpr (RB == 0) {
#pragma unroll
                for (int b = 0; b < 2; ++b) {
                    d[b] = __builtin_amdgcn_mfma_i32_16x16x64_i8(af[0][0], rfrag(w[b][0], w[b][1]),
                                                                 INT ? isum[INT ? c : 0][INT ? b : 0] : start, 0, 0, 0);
                    d[b] = __builtin_amdgcn_mfma_i32_16x16x64_i8(af[0][1], rfrag(w[b][2], w[b][3]), d[b], 0, 0, 0);
                }
            } else {
                i32x4 bw[4];
#pragma unroll
                for (int kk = 0; kk < 4; ++kk) {
                    const v4u& v = w[kk >> 1];
                    bw[kk] = rfrag(v[2 * (kk & 1)], v[2 * (kk & 1) + 1]);
                }
#pragma unroll
                for (int kk = 0; kk < 4; ++kk)
#pragma unroll
                    for (int b = 0; b < RB; ++b) {
                        if (kk == 0) d[b] = INT ? isum[INT ? c : 0][INT ? b : 0] : start;
                        d[b] = __builtin_amdgcn_mfma_i32_32x32x32_i8(af[b][kk], bw[kk], d[b], 0, 0, 0);
                    }
            }
            if constexpr (INT) {
#pragma unroll
                for (int b = 0; b < NB; ++b) isum[c][b] = d[b];
            }
            if constexpr (!CH) {
                if (WHOLE && ((i + 1) & ((1 << lg) - 1)) != 0) continue;  // uniform: the group goes on
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    if constexpr (WHOLE) {
#pragma unroll
                        for (int r = 0; r < AV; ++r) isum[c][b][r] = 0;
                    }
                    if constexpr (DUMP) {
                        int col = n0 + 32 * c + col_of(b);
                        asm volatile("" : "+v"(col));  // no address is kept from stage to stage (registers)
                        if (col < N) {
#pragma unroll
                            for (int r = 0; r < AV; ++r) {
                                const int row = m0 + row_of(b, r);
                                if (row >= pm0 && row < pm0 + pmr && row < M)
                                    atomicAdd(&P[(static_cast<int64_t>(row - pm0) * N + col) * ng + g], d[b][r] >> 8);
                            }
                        }
                        if (!have_sc) continue;
                        if constexpr (!WHOLE) {
#pragma unroll
                            for (int r = 0; r < AV; ++r) d[b][r] += static_cast<int>(MAGIC_BITS);
                        }
                    }
                    const float s = s1[RB == 0 ? b : 0], nb = -MAGIC * s;
#pragma unroll
                    for (int r = 0; r < AV; ++r) {
                        const uint2& pr = sah[RB == 0 ? 0 : b][r >> 2];
                        const uint16_t h = static_cast<uint16_t>((r & 2 ? pr.y : pr.x) >> (16 * (r & 1)));
                        const float t = WHOLE ? static_cast<float>(d[b][r]) * s : fmaf(__int_as_float(d[b][r]), s, nb);
                        acc[c][AV * b + r] = fmaf(t, rh2f(h), acc[c][AV * b + r]);
                    }
                }
            }
        }
    };
    for (int q0 = 0; q0 < n; q0 += PF)
        unroll<PF>([&](auto J) __attribute__((always_inline)) {
            constexpr int j = decltype(J)::value;
            if (q0 + j < n && stage_of(q0 + j) < nks) process(J, q0 + j);  // uniform: no stage past K (its scales are not there)
            __builtin_amdgcn_sched_barrier(0);  // the stage's registers are read before its slot is loaded again
            load(J, q0 + j + PF);
        });

    // ---- the waves' partial tiles, added in wave order
    if (!CH && !have_sc) return;  // group sums only (uniform)
    int32_t* red = reinterpret_cast<int32_t*>(rows_lds);
    if constexpr (CH) red = reinterpret_cast<int32_t*>(codes);  // the scales stay for the end
    __syncthreads();
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
        for (int r = 0; r < NRT; ++r) {
            int32_t v;
            if constexpr (CH) v = isum[c][r / AV][r % AV];
            else v = __float_as_int(acc[c][r]);
            red[(wave * NR + c * NRT + r) * 64 + lane] = v;
        }
    __syncthreads();
#pragma unroll
    for (int o = tid; o < NR * 64; o += THREADS) {
        const int rr = o >> 6, ln = o & 63;
        const int c = rr / NRT, b = rr % NRT / AV, r = rr % AV;
        const int lr = RB == 0 ? 4 * (ln >> 4) + r : 32 * b + 8 * (r >> 2) + 4 * (ln >> 5) + (r & 3);
        const int lc = 32 * c + (RB == 0 ? 16 * b + (ln & 15) : (ln & 31));
        const int row = m0 + lr, col = n0 + lc;
        float y;
        if constexpr (CH) {
            int32_t v = 0;
#pragma unroll
            for (int w = 0; w < NW; ++w) v += red[(w * NR + rr) * 64 + ln];
            if constexpr (DUMP) {
                if (row >= pm0 && row < pm0 + pmr && row < M && col < N) P[static_cast<int64_t>(row - pm0) * N + col] = v >> 8;
            }
            y = have_sc ? static_cast<float>(v) * (rh2f(asc[lr]) * (1.0f / 256.0f)) * rh2f(wsc[lc]) : 0.f;
        } else {
            y = 0.f;
#pragma unroll
            for (int w = 0; w < NW; ++w) y += __int_as_float(red[(w * NR + rr) * 64 + ln]);
        }
        if (have_sc && row < M && col < N) Y[static_cast<int64_t>(row) * N + col] = __half_as_ushort(__float2half_rn(y));
    }
}

struct Args {
    const uint8_t* Aq;
    const uint16_t* sa;
    const uint8_t* Wq;
    const uint16_t* sw;
    int64_t M, N, K, G;
    uint16_t* Y;
    const uint16_t* x;
    uint8_t* aq_out;
    uint16_t* sa_out;
    Dump dump;
    hipStream_t stream;
};

template <int RB, int CT>
int64_t rows_lds_bytes(int64_t K, int64_t G, int nw, bool fuse) {
    using F = Form<RB, CT>;
    const int64_t sc = F::scale_bytes(K / G), red = F::red_bytes(nw);
    if (G == K) return sc + red;
    const int64_t front = sc + (fuse ? (K / 2 + 15) / 16 * 16 : 0);
    return front > red ? front : red;
}

template <int RB, int CT, int NW, int PF, int OCC, bool WT, bool NT, int MODE, bool DUMP, int QL>
hipError_t launch_one(const Args& a) {
    using F = Form<RB, CT>;
    static std::atomic<uint64_t> lds_allowed{0};
    const void* k = reinterpret_cast<const void*>(w4a4_rows_kernel<RB, CT, NW, PF, OCC, WT, NT, MODE, DUMP, QL>);
    const hipError_t e = allow_dynamic_lds(k, ROWS_LDS, lds_allowed);
    if (e != hipSuccess) return e;
    const int64_t lds = rows_lds_bytes<RB, CT>(a.K, a.G, NW, QL > 0);
    if (lds > ROWS_LDS) return hipErrorInvalidValue;
    int lg = 31;  // stage -> group: shift
    if (a.G != a.K)
        for (lg = 0; (int64_t{128} << lg) < a.G; ++lg) {
        }
    const dim3 grid(static_cast<unsigned>(((a.N + F::COLS - 1) / F::COLS + 7) / 8 * 8 * ((a.M + F::ROWS - 1) / F::ROWS)));
    hipLaunchKernelGGL((w4a4_rows_kernel<RB, CT, NW, PF, OCC, WT, NT, MODE, DUMP, QL>), grid, dim3(64 * NW),
                       static_cast<size_t>(lds), a.stream, a.Aq, a.sa, a.Wq, a.sw, static_cast<int>(a.M),
                       static_cast<int>(a.N), static_cast<int>(a.K), lg, static_cast<int>(a.K / a.G), a.Y, a.x,
                       a.aq_out, a.sa_out, a.dump.P, a.dump.m0, a.dump.mr);
    return hipGetLastError();
}

// Forms: 16 rows by 32 columns, 32 rows by 32 or 64 columns, 64 rows by 64
// columns; eight waves, or four (then two or three workgroups fit a CU).
enum RowsForm : int { kR16, kR32, kR32x2, kR32x2w4, kR64, kR64w4 };

// (DUMP: a shorter ring where the registers run out.)
template <bool WT, bool NT, int MODE, bool DUMP>
hipError_t launch_form(RowsForm f, const Args& a) {
    if constexpr (MODE != kWhole) {  // more than 32 rows only
        if (f == kR16) return launch_one<0, 1, 8, 2, 4, WT, NT, MODE, DUMP, 0>(a);
        if (f == kR32) return launch_one<1, 1, 8, 2, DUMP ? 2 : 4, WT, NT, MODE, DUMP, 0>(a);
    }
    if (f == kR32x2) return launch_one<1, 2, 8, 2, 2, WT, NT, MODE, DUMP, 0>(a);
    if (f == kR32x2w4) return launch_one<1, 2, 4, 2, 2, WT, NT, MODE, DUMP, 0>(a);
    if constexpr (!NT) {
        if (f == kR64) return launch_one<2, 2, 8, DUMP ? 1 : 2, 2, WT, false, MODE, DUMP, 0>(a);
        if (f == kR64w4) return launch_one<2, 2, 4, DUMP ? 1 : 2, 2, WT, false, MODE, DUMP, 0>(a);
    }
    return hipErrorInvalidValue;
}

int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Past 32 rows a group of several stages is one wave's, so that its sum meets
// the scales once, whole.
bool rows_whole(int64_t M, int64_t K, int64_t G) { return M > 32 && G > 128 && G != K; }

// Time in us of the 64-column forms on 256 CUs at G = 128 (launch, prologue and
// reduction, then per round of workgroups a start and a time per 128-wide
// stage): least squares over 343 shapes of 40 .. 250 rows, N = 1024 .. 28672,
// K = 1024 .. 28672 on MI355X, within 20 % of each.  load: workgroups on the
// busiest CU; a CU with one runs it with eight waves, with more they have four
// and two or three at a time hide each other's start and end.
// Per channel: no dequantization in the loop; 190 shapes.
// Whole groups (G = 256, 512, 1024): n counts the stages of the wave with the
// most groups, times the waves; 415 shapes, N = 512 .. 57344, within 40 % of
// 32-row and 60 % of 64-row times (the choice by them: rows_take).
double whole_stages(int64_t K, int64_t G, double load) {
    const int64_t waves = load == 1.0 ? 8 : 4;
    return static_cast<double>(waves * cdiv(K / G, waves) * (G / 128));
}
double cost32(int64_t M, int64_t N, int64_t K, int64_t G) {
    const double n = static_cast<double>(kstages(K)), load = static_cast<double>(cdiv(cdiv(M, 32) * cdiv(N, 64), device_cu_count()));
    if (rows_whole(M, K, G)) {
        const double nw = whole_stages(K, G, load);
        return load == 1.0 ? 3.6 + 0.112 * nw : 4.5 + load * (0.19 + 0.115 * nw);
    }
    if (G == K) return load == 1.0 ? 4.6 + 0.094 * n : 3.6 + load * (0.68 + 0.092 * n);
    return load == 1.0 ? 4.3 + 0.116 * n : 2.8 + load * (0.74 + 0.118 * n);
}
double cost64(int64_t M, int64_t N, int64_t K, int64_t G) {
    const double n = static_cast<double>(kstages(K)), load = static_cast<double>(cdiv(cdiv(M, 64) * cdiv(N, 64), device_cu_count()));
    if (rows_whole(M, K, G)) {
        const double nw = whole_stages(K, G, load);
        return load == 1.0 ? 5.0 + 0.165 * nw : 5.3 + load * (1.32 + 0.166 * nw);
    }
    if (G == K) return load == 1.0 ? 5.1 + 0.167 * n : 5.0 + load * (1.36 + 0.155 * n);
    return load == 1.0 ? 6.2 + 0.192 * n : 4.2 + load * (1.76 + 0.189 * n);
}

// Form by size, from times on MI355X (G = 128, tiled weights past the cache, us):
//   * up to 16 rows: kR16 (N = K = 8192, 16 rows: 8.9; kR32 9.8).
//   * up to 32 rows: kR32 while its 32-column tiles give a CU at most one
//     (N = K = 8192: 11.5, kR32x2 14.0); past that 64-column tiles, which read
//     and widen the activations half as often (N = 10240: kR32 17.4, kR32x2
//     14.6; N = 57344: 61.6, kR32x2 54.9, kR32x2w4 51.6).  A K so long that
//     the 64-column form's scales pass the LDS keeps kR32.
//   * more rows: 32 or 64 a workgroup by the costs above (128 rows, N = 8192:
//     kR64 19.8, kR32x2w4 21.3; 256 rows, N = 10240: kR64w4 44.2, kR32x2w4 43.4).
RowsForm rows_form(int64_t M, int64_t N, int64_t K, int64_t G) {
    const int64_t cus = device_cu_count();
    if (M <= 16) return kR16;
    if (M <= 32 && (cdiv(N, 32) <= cus || rows_lds_bytes<1, 2>(K, G, 8, false) > ROWS_LDS)) return kR32;
    if (M > 32 && cost64(M, N, K, G) < cost32(M, N, K, G)) return cdiv(M, 64) * cdiv(N, 64) <= cus ? kR64 : kR64w4;
    return cdiv(M, 32) * cdiv(N, 64) <= cus ? kR32x2 : kR32x2w4;
}

// Tiled weights from this size on that one workgroup reads are loaded
// nontemporal: smaller ones may well still be in the 256 MB Infinity Cache when
// they are needed again, and their launches are bound by latency anyway.
// Row-major weights never: a stage is 64 bytes of a row, so a 128-byte line has
// two stages, of two waves, and the line of a nontemporal load is gone when the
// second comes (8 rows, N = 2560, K = 28672: 38.0 us so, 23.6 without; 8 rows,
// N = K = 28672: 157 and 101).
constexpr int64_t ROWS_NT_BYTES = int64_t{16} << 20;

int64_t rows_lds_of(RowsForm f, int64_t K, int64_t G) {
    switch (f) {
        case kR16: return rows_lds_bytes<0, 1>(K, G, 8, false);
        case kR32: return rows_lds_bytes<1, 1>(K, G, 8, false);
        case kR32x2: return rows_lds_bytes<1, 2>(K, G, 8, false);
        case kR32x2w4: return rows_lds_bytes<1, 2>(K, G, 4, false);
        case kR64: return rows_lds_bytes<2, 2>(K, G, 8, false);
        default: return rows_lds_bytes<2, 2>(K, G, 4, false);
    }
}

}  // namespace

bool rows_fits(int64_t M, int64_t N, int64_t K, int64_t G) {
    const bool g_ok = G == K || (G == 128 || G == 256 || G == 512 || G == 1024);
    return M >= 1 && M < kRowsMax && N >= 1 && g_ok && rows_lds_of(rows_form(M, N, K, G), K, G) <= ROWS_LDS;
}

int rows_form_of(int64_t M, int64_t N, int64_t K, int64_t G) { return rows_form(M, N, K, G); }

double rows_cost_us(int64_t M, int64_t N, int64_t K, int64_t G) {
    const double a = cost32(M, N, K, G), b = cost64(M, N, K, G);
    return a < b ? a : b;
}

bool rows_nontemporal(int64_t M, int64_t N, int64_t K, bool wt) {
    return wt && M <= 32 && N * (K / 2) >= ROWS_NT_BYTES;  // up to 32 rows: every weight is read by one workgroup
}

namespace {

template <bool WT>
hipError_t launch_layout(RowsForm f, const Args& a) {
    const bool ch = a.G == a.K, whole = rows_whole(a.M, a.K, a.G);
    if (a.dump.P) {
        if (ch) return launch_form<WT, false, kChan, true>(f, a);
        return whole ? launch_form<WT, false, kWhole, true>(f, a) : launch_form<WT, false, kStage, true>(f, a);
    }
    if constexpr (WT)
        if (rows_nontemporal(a.M, a.N, a.K, true))
            return ch ? launch_form<true, true, kChan, false>(f, a) : launch_form<true, true, kStage, false>(f, a);
    if (ch) return launch_form<WT, false, kChan, false>(f, a);
    return whole ? launch_form<WT, false, kWhole, false>(f, a) : launch_form<WT, false, kStage, false>(f, a);
}

}  // namespace

hipError_t launch_gemm_rows(const uint8_t* Aq, const uint16_t* sa, const uint8_t* Wq, const uint16_t* sw, int64_t M,
                            int64_t N, int64_t K, int64_t G, uint16_t* Y, hipStream_t stream, Dump dump, bool wt) {
    if (!rows_fits(M, N, K, G)) return hipErrorInvalidValue;
    const Args a{Aq, sa, Wq, sw, M, N, K, G, Y, nullptr, nullptr, nullptr, dump, stream};
    const RowsForm f = rows_form(M, N, K, G);
    if (dump.P && G != K) {  // sums are added atomically into a zeroed window (per channel: stored)
        const hipError_t e = launch_fill_i32(dump.P, static_cast<int64_t>(dump.mr) * N * (K / G), 0, stream);
        if (e != hipSuccess) return e;
    }
    return wt ? launch_layout<true>(f, a) : launch_layout<false>(f, a);
}

// The one-row linear on tiled weights with the quantizer in the prologue, where
// that is the faster way: every workgroup quantizes all of x, beside the loads
// of its weights, against a launch and a round trip of the codes.
// MI355X, G = 128, us, fused / quantizer and GEMM: N = 8192, K = 2048 5.8 / 7.1;
// N = 57344, K = 8192 38.2 / 38.8; N = 28672, K = 14336 37.1 / 36.8, K = 28672
// 70.4 / 68.1; N = 256, K = 28672 15.6 / 15.4, K = 57344 27.8 / 25.0 (longer K
// the same).  G = 512 (a group's maximum over all lanes) loses earlier where
// workgroups come in several rounds: N = 14336, K = 2048 6.9 / 8.3, but
// N = 28672 11.2 / 10.8 and N = 57344, K = 4096 24.4 / 22.6.
bool rows_fused_fits(int64_t M, int64_t N, int64_t K, int64_t G) {
    return M == 1 && N >= 1 && (G == 128 || G == 256 || (G == 512 && N <= 16384)) && G < K &&
           (K <= 16384 || cdiv(N, 32) * K <= (int64_t{1} << 18)) && rows_lds_bytes<0, 1>(K, G, 8, true) <= ROWS_LDS;
}

namespace {
template <int QL>
hipError_t launch_fused_g(const Args& a, bool nt) {
    if (a.dump.P) return launch_one<0, 1, 8, 2, 4, true, false, kStage, true, QL>(a);
    return nt ? launch_one<0, 1, 8, 2, 4, true, true, kStage, false, QL>(a) : launch_one<0, 1, 8, 2, 4, true, false, kStage, false, QL>(a);
}
}  // namespace

hipError_t launch_rows_fused(const uint16_t* x, const uint8_t* Wt, const uint16_t* sw, int64_t N, int64_t K, int64_t G,
                             uint16_t* Y, uint8_t* Aq, uint16_t* sa, hipStream_t stream, Dump dump) {
    if (!rows_fused_fits(1, N, K, G)) return hipErrorInvalidValue;
    const Args a{nullptr, nullptr, Wt, sw, 1, N, K, G, Y, x, Aq, sa, dump, stream};
    if (dump.P) {
        const hipError_t e = launch_fill_i32(dump.P, static_cast<int64_t>(dump.mr) * N * (K / G), 0, stream);
        if (e != hipSuccess) return e;
    }
    const bool nt = rows_nontemporal(1, N, K, true);
    if (G == 128) return launch_fused_g<16>(a, nt);
    if (G == 256) return launch_fused_g<32>(a, nt);
    return launch_fused_g<64>(a, nt);
}

}  // namespace apex4
