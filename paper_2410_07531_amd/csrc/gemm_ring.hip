// GEMM for outputs that are too small for the 256-row tiles of gemm.hip, for fp32, for weights
// stored [K, N] and for row lengths that are no multiple of 128 bytes (paper Sec. 3.2, Table 1
// GEMM column: the same layers on short sequences and in the other precision and layout).
//
// What bounds it: a short product has few tiles, and a tile's time is its walk over k: every
// 128-byte slot of k has to travel L2 -> LDS (about 43 bytes per clock and compute unit) at a
// latency of one to two microseconds.  So
//   - tiles are small enough that the launch covers the 256 compute units, and
//   - operands go through a ring of STAGES LDS slots (up to 160 KiB of them per compute unit),
//     filled by buffer loads that write LDS, loaded STAGES slots ahead.
// One barrier per slot: when a wave arrives there it has read the slot it is working on into
// registers and its own loads of the next slot have landed.  The fragments of a unit of k (one MFMA
// depth, see Traits) are read while the MFMAs of the unit before it run.
//
// A load instruction fills 64 lanes x 16 bytes of LDS, whether rows start on 16 bytes or on 4 (VEC: what the end of a
// row takes with it is cleared, see clear_tail; a load of 4 bytes a lane costs its wave as much and moves a quarter), and keeps
// its wave from issuing for 20 to 50 clocks; with one wave per SIMD the matrix pipe idles meanwhile.
// KS > 1: the waves of a workgroup share one output tile and split each slot's k between them (with SUB
// 128-byte parts per slot where a slot of one part has too few units to split); the partial sums meet in
// LDS at the end.  Against more waves side by side this reads each LDS byte less often, and for outputs of
// a few tiles it is what puts more than one wave on a SIMD: 512 x 6144 x 4096, tile 128 x 128, 37.9 us with
// four waves and 32.3 with eight (the 256-row kernel: 56.8).
//
// Per element the sum runs over k in the order of the 256-row kernels (same MFMA, same cyclic start),
// so for bf16 and fp8 with KS == 1 the result is theirs bit for bit.
//
// Measured at 333 x 4096 x 4096 bf16: 20 us (256-row kernel 52.5); [K, N] weights 1024 x 4096 x 4096: 37 us
// (generic VALU kernel 799); fp32 72 x 2922 x 747: 10.3 us (with loads of 4 bytes a lane 15.6); fp32 1024^3: 23 us (184), 2048 x 4096 x 4096: 510 us = 135 TFLOP/s of the
// 157 the fp32 matrix instructions reach (1470).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "rov_internal.h"

namespace rov {
namespace {

typedef __attribute__((address_space(3))) void* lptr_t;
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef int i32x2 __attribute__((ext_vector_type(2)));
typedef i32x2 i32x2_u __attribute__((aligned(4)));   // stored to rows that start on 4 bytes
typedef f32x4 f32x4_u __attribute__((aligned(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) i16x4* lds_i16x4_ptr;

constexpr int kSlotRow = 128;   // bytes of k per operand row and slot

// Element type, MFMA shape and the unit of k: bf16 32 (16x16x32), fp8 128 (16x16x128), fp32 8 (four
// 32x32x2, each lane holding four consecutive k of its half).
template <int DT>
struct Traits;
template <>
struct Traits<ROV_BF16> {
    static constexpr int ESZ = 2, MB = 16, UNITS = 2, ACC = 4;
    typedef f32x4 acc_t;
    typedef i32x4 frag_t;
    typedef uint16_t out_t;
};
template <>
struct Traits<ROV_FP8_E4M3> {
    static constexpr int ESZ = 1, MB = 16, UNITS = 1, ACC = 4;
    typedef f32x4 acc_t;
    typedef i32x8 frag_t;
    typedef uint16_t out_t;
};
template <>
struct Traits<ROV_F32> {
    static constexpr int ESZ = 4, MB = 32, UNITS = 4, ACC = 16;
    typedef f32x16 acc_t;
    typedef f32x4 frag_t;
    typedef float out_t;
};

__device__ __forceinline__ f32x4 mfma(i32x4 w, i32x4 a, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w), __builtin_bit_cast(bf16x8, a), c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 mfma(i32x8 w, i32x8 a, f32x4 c) {
    return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(w, a, c, 0, 0, 0, 0, 0, 0);   // no scales: the plain instruction
}
__device__ __forceinline__ f32x16 mfma(f32x4 w, f32x4 a, f32x16 c) {
#pragma unroll
    for (int e = 0; e < 4; ++e) c = __builtin_amdgcn_mfma_f32_32x32x2f32(w[e], a[e], c, 0, 0, 0);
    return c;
}

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    f32x2 v = {lo, hi};
    bf16x2 h = __builtin_convertvector(v, bf16x2);
    return *reinterpret_cast<uint32_t*>(&h);
}

struct RingParams {
    const char* A;
    const char* W;
    void* C;
    const uint16_t* R;      // bf16 side input added to the result, or nullptr
    int M, N, K;
    float alpha;
    int tiles_m, tiles_n;
};

// XORed into the index of a 16-byte chunk of LDS row `row`.  Rows of k (A, and W stored [N, K]): 128
// bytes, read 16 bytes per lane, lanes that are served together hold 16 rows (see gemm.hip).  Rows of
// n (W stored [K, N], bf16): read with the transposing 8-byte load, 32 lanes at a time over rows
// {0-3, 8-11} (+4, +16) x 32 bytes: the rows' 32-byte groups must differ (256-byte rows alias, 128-byte
// rows by parity).
template <bool NROW, int ROWB, int DT>
__device__ __forceinline__ int ring_swizzle(int row) {
    if (!NROW) return (row >> 1) & 7;
    if (DT != ROV_BF16) return 0;
    return ROWB == 256 ? (((row & 3) | (((row >> 3) & 1) << 2)) << 1) : ((((row >> 1) & 1) | (((row >> 3) & 1) << 1)) << 1);
}

// TM x TN MFMA blocks per wave, WM x WN waves over the tile, KS of them over k.  KN: W is [K, N].
// VEC: alignment of the operands' rows, 16 or 4 bytes (loads are 16 bytes a lane either way: a buffer load needs 4).
template <int DT, int TM, int TN, int WM, int WN, int KS, int SUB, bool KN, int VEC, int STAGES>
__global__ __launch_bounds__(64 * WM * WN * KS) void gemm_ring_kernel(const RingParams p) {
    using TR = Traits<DT>;
    constexpr int ESZ = TR::ESZ, MB = TR::MB, ACC = TR::ACC, NW = WM * WN * KS;
    constexpr int BM = MB * TM * WM, BN = MB * TN * WN;
    constexpr int KR1 = kSlotRow / ESZ, KR = SUB * KR1;      // k per part, per slot
    constexpr int WROWB = KN ? BN * ESZ : kSlotRow;          // bytes per LDS row of the W tile
    constexpr int kPart = (BM + BN) * kSlotRow, kSlot = SUB * kPart;
    constexpr int QA = BM * kSlotRow / 1024, QP = (BM + BN) * kSlotRow / 1024;   // loads (1 KiB each) of A, of a part
    constexpr int L = SUB * QP / NW;                         // loads per wave and slot
    constexpr int UW = SUB * TR::UNITS / KS;                 // units of k per wave and slot
    constexpr int MU = TM * TN;
    static_assert(L * NW == SUB * QP, "every wave loads the same share");
    static_assert(VEC == 16 || VEC == 4, "alignment of the rows");
    static_assert(UW * KS == SUB * TR::UNITS && (UW == 1 || UW % 2 == 0), "fragment buffers alternate");
    static_assert((STAGES - 2) * L <= 63, "loads in flight fit the counter");
    static_assert(!KN || DT != ROV_FP8_E4M3, "fp8 weights are [N, K]");
    static_assert(!KN || DT != ROV_BF16 || WROWB == 128 || WROWB == 256, "swizzle of the [K, N] tile");
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    // beside a co-resident RNG grid: its waves get the issue slots these leave
    __builtin_amdgcn_s_setprio(3);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ks = wave / (WM * WN), wm = (wave % (WM * WN)) / WN, wn = wave % WN;

    // tile id: a contiguous range of tiles per XCD, bands of 8 tile rows, the row fastest (an XCD's L2 then
    // fetches few W panels, each once)
    const int T = p.tiles_m * p.tiles_n;
    int id;
    {
        const int pid = blockIdx.x, per = T >> 3, rem = T & 7;
        const int xcd = pid & 7, loc = pid >> 3;
        id = xcd < rem ? xcd * (per + 1) + loc : rem * (per + 1) + (xcd - rem) * per + loc;
    }
    constexpr int GM = 8;
    const int band = id / (GM * p.tiles_n);
    const int band_rows = (p.tiles_m - band * GM) < GM ? (p.tiles_m - band * GM) : GM;
    const int in_band = id - band * GM * p.tiles_n;
    const int m0 = (band * GM + in_band % band_rows) * BM, n0 = (in_band / band_rows) * BN;
    const int M = p.M, N = p.N, K = p.K;

    const int ns = (K + KR - 1) / KR;
    const int krem = K - (ns - 1) * KR;                      // k in the last slot
    const bool ragged = krem != KR;
    const int kstart = (int)((unsigned)(m0 / 256) % (unsigned)ns);   // the 256-row kernels' start
    const uint32_t ld_a = (uint32_t)K * ESZ, ld_w = (uint32_t)(KN ? N : K) * ESZ;
    const int rows_a = M - m0 < BM ? M - m0 : BM, rows_w = N - n0 < BN ? N - n0 : BN;
    const uint32_t bytes_a = (uint32_t)rows_a * ld_a;
    const uint32_t bytes_w = KN ? (uint32_t)K * ld_w - (uint32_t)n0 * ESZ : (uint32_t)rows_w * ld_w;
    auto make_rsrc = [](const char* base, uint32_t bytes) {
        const uint64_t b = (uint64_t)(uintptr_t)base;
        i32x4 r;
        r[0] = __builtin_amdgcn_readfirstlane((int)(uint32_t)b);
        r[1] = __builtin_amdgcn_readfirstlane((int)(uint32_t)((b >> 32) & 0xFFFFu));
        r[2] = __builtin_amdgcn_readfirstlane((int)bytes);
        r[3] = 0x00020000;
        return r;
    };
    i32x4 rsrc_a = make_rsrc(p.A + (size_t)m0 * ld_a, bytes_a);
    i32x4 rsrc_w = make_rsrc(KN ? p.W + (size_t)n0 * ESZ : p.W + (size_t)n0 * ld_w, bytes_w);
    const uint32_t lds_base = (uint32_t)(uintptr_t)(lptr_t)lds;

    // Load q of this wave is load q * NW + wave of the slot: part by part, A's rows, then W's, 1 KiB of LDS each (a load whose
    // operand differs between the waves selects its resource).  voff: the lane's byte offset from the panel's start at
    // slot 0; lane_k: its position in the slot's k (the row for a [K, N] tile).
    // Rows past the edge and, in the last slot, k >= K lie outside the resource and read as zeros (vend: the offset there.  Kept for
    // the first loads, not worked out at each behind a branch: 0.45 us of a product of one slot).
    uint32_t voff[L], vend[L];
    // (all waves' loads q in one part, or of one operand: known when compiled)
    auto load_part = [&](int q) { return q * NW / QP == (q * NW + NW - 1) / QP ? q * NW / QP : (q * NW + wave) / QP; };
    auto load_in_part = [&](int q) { return q * NW - load_part(q) * QP + wave; };
    auto load_is_w = [&](int q) {
        const int first = q * NW % QP, last = first + NW - 1;
        return last < QA ? false : first >= QA && last < QP ? true : load_in_part(q) >= QA;
    };
    auto lds_at = [&](int q) { return (load_in_part(q) - (load_is_w(q) ? QA : 0)) * 1024; };   // in the operand's part
    auto lane_k = [&](int q) {
        const bool krow = KN && load_is_w(q);
        const int b = lds_at(q) + lane * 16, row = b / (krow ? WROWB : kSlotRow), pos = b % (krow ? WROWB : kSlotRow);
        return load_part(q) * KR1 + (krow ? row : ((pos >> 4) ^ ring_swizzle<false, kSlotRow, DT>(row)) * 16 / ESZ);
    };
#pragma unroll
    for (int q = 0; q < L; ++q) {
        const int sub = load_part(q);
        const bool is_w = load_is_w(q), krow = KN && is_w;
        const int b = lds_at(q) + lane * 16, row = b / (krow ? WROWB : kSlotRow), pos = b % (krow ? WROWB : kSlotRow);
        const int sw = krow ? ring_swizzle<true, WROWB, DT>(row) : ring_swizzle<false, kSlotRow, DT>(row);
        const uint32_t col = (uint32_t)(((pos >> 4) ^ sw) * 16);
        const bool ok = is_w ? (KN || row < rows_w) : row < rows_a;
        const uint32_t at = krow ? (uint32_t)(sub * KR1 + row) * ld_w + col
                                 : (uint32_t)row * (is_w ? ld_w : ld_a) + (uint32_t)(sub * kSlotRow) + col;
        voff[q] = ok ? at : (is_w ? bytes_w : bytes_a);
        vend[q] = lane_k(q) < krem ? voff[q] : (is_w ? bytes_w : bytes_a);
    }
    // The slot being filled: its place in the ring, its position on the cyclic walk over k, and how many slots
    // of the walk are left.
    int f_slot = 0, f_st = kstart, f_left = ns;
    auto next_fill = [&]() {
        f_slot = f_slot + 1 == STAGES ? 0 : f_slot + 1;
        --f_left;
        f_st = f_left <= 0 || f_st + 1 == ns ? 0 : f_st + 1;
    };
    // Inline assembly: the compiler's wait-count pass cannot tell these LDS writes from the fragment reads;
    // the kernel places its vmcnt waits itself.  M0 is only set by compiled code right before its own uses.
    // Past the end of the walk the range is empty and the scalar offset zero (the check takes it off the size):
    // no memory access, and the counter's arithmetic holds.
    // In the loop of the fp32 forms, the widest [K, N] ones and fp8's 128 x 64 the offset beyond k is worked out behind a branch: its edges
    // keep the loads between the MFMAs where they were put (2764 x 392 x 4096 fp32 88.5 us, with a select 100; [K, N] 128 x 128 tiles 1 to 2 %
    // sooner; fp8 92 x 10240 x 14336 34.1 us, with a select 34.8).  The others are up to 2.5 % faster with the select (timed at 750
    // products, weights in L2 and from HBM; bf16 64 x 32 tiles at 280: 1 to 2 % at short sums, level from K = 2048 on).
    constexpr bool kBranch = DT == ROV_F32 || (KN && VEC == 16 && BN == 128) || (DT == ROV_FP8_E4M3 && BM == 128 && BN == 64);
    auto issue = [&](int q, auto in_loop) __attribute__((always_inline)) {
        const bool is_w = load_is_w(q);
        const uint32_t dst = lds_base + (uint32_t)(f_slot * kSlot + (q * NW + wave) * 1024);
        i32x4 rs = is_w ? rsrc_w : rsrc_a;
        rs[2] = f_left > 0 ? rs[2] : 0;
        uint32_t vo = voff[q];
        if (!decltype(in_loop)::value || !kBranch) vo = ragged && f_st == ns - 1 ? vend[q] : vo;
        else if (ragged && f_st == ns - 1) vo = lane_k(q) < krem ? vo : (is_w ? bytes_w : bytes_a);
        const uint32_t so = KN && is_w ? (uint32_t)f_st * (uint32_t)KR * ld_w : (uint32_t)f_st * (uint32_t)(SUB * kSlotRow);
        const int sdst = __builtin_amdgcn_readfirstlane((int)dst), sso = __builtin_amdgcn_readfirstlane((int)so);
#pragma unroll
        for (int e = 0; e < 4; ++e) rs[e] = __builtin_amdgcn_readfirstlane(rs[e]);   // (kept in scalar registers)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                     :: "s"(sdst), "v"(vo), "s"(rs), "s"(sso) : "memory");
    };

    // fragments
    typename TR::frag_t fa[2][TM], fw[2][TN];
    const int fr = lane & (MB - 1), fc = lane / MB;          // row in the block, k chunk
    const int fsw = ring_swizzle<false, kSlotRow, DT>(fr);   // block bases are multiples of 16 rows
    auto read_row16 = [&](const char* base, int chunk) {
        return *reinterpret_cast<const i32x4*>(base + fr * kSlotRow + ((chunk ^ fsw) << 4));
    };
    auto read_krow = [&](const char* base, int u, typename TR::frag_t& f) {   // operand stored with k contiguous
        if constexpr (DT == ROV_BF16) {
            f = read_row16(base, 4 * u + fc);
        } else if constexpr (DT == ROV_FP8_E4M3) {
            const i32x4 lo = read_row16(base, fc), hi = read_row16(base, 4 + fc);
            f = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        } else {
            f = __builtin_bit_cast(f32x4, read_row16(base, 2 * u + fc));
        }
    };
    auto read_units = [&](int slot, int uu, int par) {
        const int ug = ks * UW + uu, u = ug % TR::UNITS;
        const char* sa = lds + slot * kSlot + (ug / TR::UNITS) * kPart;
        const char* sw = sa + BM * kSlotRow;
#pragma unroll
        for (int i = 0; i < TM; ++i) read_krow(sa + (wm * TM + i) * MB * kSlotRow, u, fa[par][i]);
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            if constexpr (!KN) {
                read_krow(sw + (wn * TN + j) * MB * kSlotRow, u, fw[par][j]);
            } else if constexpr (DT == ROV_BF16) {
                // lane 16g + 4r + s supplies row 32u + 8g (+4) + r, columns 4s of the block; it receives its own
                // column's four values (ds_read_b64_tr_b16): the k order of the A fragment, chunk g
                const int g = lane >> 4, r = (lane >> 2) & 3, s = lane & 3;
                i16x4 part[2];
#pragma unroll
                for (int x = 0; x < 2; ++x) {
                    const int row = 32 * u + 8 * g + 4 * x + r;
                    const int col = (wn * TN + j) * 32 + s * 8;          // byte in the row
                    const char* at = sw + row * WROWB + ((((col >> 4) ^ ring_swizzle<true, WROWB, DT>(row)) << 4) | (col & 15));
                    part[x] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4_ptr)at);
                }
                fw[par][j] = __builtin_bit_cast(i32x4, __builtin_shufflevector(part[0], part[1], 0, 1, 2, 3, 4, 5, 6, 7));
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    fw[par][j][e] = *reinterpret_cast<const float*>(sw + (8 * u + 4 * fc + e) * WROWB + ((wn * TN + j) * MB + fr) * 4);
            }
        }
    };

    // Rows that start on 4 bytes: the 16 bytes that hold the end of a row go on into the next row (the last row's are cut
    // off by the resource, which is checked dword by dword).  Their part beyond k is cleared once the last slot of k has
    // landed, in both operands, so that no product sees a value that is not the row's ([K, N]: W's rows beyond k are zeros).
    auto clear_tail = [&](int at_slot) {
        const int kb = krem % KR1 * ESZ;                     // bytes of the part that k ends in
        if ((kb & 15) == 0) return;
        for (int r = threadIdx.x; r < (KN ? BM : BM + BN); r += 64 * NW) {
            char* const c = lds + at_slot * kSlot + krem / KR1 * kPart + r * kSlotRow +
                            (((kb >> 4) ^ ring_swizzle<false, kSlotRow, DT>(r < BM ? r : r - BM)) << 4);
            for (int e = kb & 15; e < 16; e += 4) *reinterpret_cast<uint32_t*>(c + e) = 0u;
        }
        __syncthreads();
    };

    // fp32 with two parts of k: every other unit has its own sums, so that a chain of additions is as long as with four parts (relative
    // error against 64 bits at K = 3887: 5.6e-7, that of the 32 x 32 tiles; with one set 7.9e-7).  16 registers more, 0.07 us a product.
    constexpr int NACC = DT == ROV_F32 && KS == 2 ? 2 : 1;
    static_assert(NACC == 1 || UW % 2 == 0, "a slot's units alternate");
    typename TR::acc_t accs[NACC][TN][TM];
#pragma unroll
    for (int a = 0; a < NACC; ++a)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int e = 0; e < ACC; ++e) accs[a][j][i][e] = 0.0f;
    auto& acc = accs[0];

    // vmcnt(n) alone
    auto wait_loads = [](auto n) {
        constexpr int v = decltype(n)::value;
        __builtin_amdgcn_s_waitcnt(0x0F70 | (v & 15) | ((v >> 4) << 14));
    };
#pragma unroll
    for (int s = 0; s < STAGES; ++s) {
#pragma unroll
        for (int q = 0; q < L; ++q) issue(q, std::false_type{});
        next_fill();
    }
    wait_loads(std::integral_constant<int, (STAGES - 1) * L <= 63 ? (STAGES - 1) * L : 63>{});
    __syncthreads();
    int c_st = kstart;                                       // position on the walk of the slot being read (VEC == 4)
    if (VEC == 4 && c_st == ns - 1) clear_tail(0);
    read_units(0, 0, 0);

    // The loads that refill the slot released by a barrier (in the last unit of a slot's k) go out one per few
    // MFMAs, from there to the next barrier.  pos0: MFMAs since that barrier; -1: nothing to refill yet.
    auto mfmas = [&](int par, int pos0) {
#pragma unroll
        for (int m = 0; m < MU; ++m) {
            const int j = m / TM, i = m % TM;
            accs[par % NACC][j][i] = mfma(fw[par][j], fa[par][i], accs[par % NACC][j][i]);
            if (pos0 >= 0) {
#pragma unroll
                for (int q = 0; q < L; ++q)
                    if (q * UW * MU / L == pos0 + m) issue(q, std::true_type{});
            }
        }
    };
    int slot = 0;                                            // place of the current slot in the ring
    auto units_before_last = [&](auto par_tag, bool refill) __attribute__((always_inline)) {
        constexpr int PAR = decltype(par_tag)::value;
#pragma unroll
        for (int u = 0; u < UW - 1; ++u) {
            read_units(slot, u + 1, (u + 1 + PAR) & 1);
            __builtin_amdgcn_sched_barrier(0);
            mfmas((u + PAR) & 1, refill ? (1 + u) * MU : -1);
        }
    };
    auto last_unit = [&](auto par_tag) __attribute__((always_inline)) {
        constexpr int PAR = decltype(par_tag)::value;
        __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0): this wave's reads of the slot are done
        wait_loads(std::integral_constant<int, (STAGES - 2) * L>{});
        __syncthreads();
        slot = slot + 1 == STAGES ? 0 : slot + 1;
        if (VEC == 4) {
            c_st = c_st + 1 == ns ? 0 : c_st + 1;
            if (c_st == ns - 1) clear_tail(slot);            // (past the walk's end: the slot is not used any more)
        }
        read_units(slot, 0, (UW + PAR) & 1);
        __builtin_amdgcn_sched_barrier(0);
        mfmas((UW - 1 + PAR) & 1, 0);
    };
    constexpr auto P0 = std::integral_constant<int, 0>{};
    constexpr auto P1 = std::integral_constant<int, UW & 1>{};
    // The loop body runs from barrier to barrier (UW odd: over two slots), so that refills stay in one piece.
    units_before_last(P0, false);
    last_unit(P0);
    int S = 1;
    if constexpr (UW % 2 == 0) {
        for (; S < ns; ++S) {
            units_before_last(P0, true);
            next_fill();
            last_unit(P0);
        }
    } else {
        for (; S + 1 < ns; S += 2) {
            units_before_last(P1, true);
            next_fill();
            last_unit(P1);
            units_before_last(P0, true);
            next_fill();
            last_unit(P0);
        }
        if (S < ns) {
            units_before_last(P1, true);
            next_fill();
            last_unit(P1);
        }
    }
    wait_loads(std::integral_constant<int, 0>{});   // no LDS load may outlive the loop
    if constexpr (NACC == 2) {
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int i = 0; i < TM; ++i) acc[j][i] += accs[1][j][i];
    }

    // Block (i, j), register group g: the lane holds row fr of the block's A rows and four consecutive output
    // columns.  WHOLE: every row starts on four values, and its columns come in whole groups of four.
    auto store4 = [&](auto whole, int i, int j, int g, float c0, float c1, float c2, float c3) __attribute__((always_inline)) {
        constexpr bool WHOLE = decltype(whole)::value;
        const int m = m0 + (wm * TM + i) * MB + fr;
        const int n = n0 + (wn * TN + j) * MB + (MB == 32 ? 8 * g : 0) + 4 * fc;
        if (m >= M || n >= N) return;
        float c[4] = {p.alpha * c0, p.alpha * c1, p.alpha * c2, p.alpha * c3};
        const size_t at = (size_t)m * N + n;
        if constexpr (DT == ROV_F32) {
            float* out = (float*)p.C + at;
            if (WHOLE) {
                *reinterpret_cast<float4*>(out) = make_float4(c[0], c[1], c[2], c[3]);
            } else if (n + 3 < N) {   // (a row starts on any 4 bytes)
                f32x4 v = {c[0], c[1], c[2], c[3]};
                *reinterpret_cast<f32x4_u*>(out) = v;
            } else {
#pragma unroll
                for (int e = 0; e < 3; ++e)
                    if (n + e < N) out[e] = c[e];
            }
        } else {
            uint16_t* out = (uint16_t*)p.C + at;
            if (WHOLE) {
                if (p.R != nullptr) {
                    const uint2 r = *reinterpret_cast<const uint2*>(p.R + at);
                    c[0] += __uint_as_float(r.x << 16);
                    c[1] += __uint_as_float(r.x & 0xFFFF0000u);
                    c[2] += __uint_as_float(r.y << 16);
                    c[3] += __uint_as_float(r.y & 0xFFFF0000u);
                }
                *reinterpret_cast<uint2*>(out) = make_uint2(pack_bf16x2(c[0], c[1]), pack_bf16x2(c[2], c[3]));
            } else if ((N & 1) == 0 && n + 3 < N) {   // rows on 4 bytes
                i32x2 v = {(int)pack_bf16x2(c[0], c[1]), (int)pack_bf16x2(c[2], c[3])};
                *reinterpret_cast<i32x2_u*>(out) = v;
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (n + e < N) out[e] = (uint16_t)(pack_bf16x2(c[e], 0.0f) & 0xFFFFu);
            }
        }
    };
    constexpr int GR = ACC / 4;                               // register groups per block
    auto finish = [&](auto whole) __attribute__((always_inline)) {
        if constexpr (KS == 1) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int g = 0; g < GR; ++g)
                        store4(whole, i, j, g, acc[j][i][4 * g], acc[j][i][4 * g + 1], acc[j][i][4 * g + 2], acc[j][i][4 * g + 3]);
        } else {
            // Register group x of the tile wave is finished by its k part x % KS: the others hand it their sums through
            // LDS, [tile wave][group][part] of 64 x 16 bytes, and the parts are added in order.
            constexpr int NG = TM * TN * GR;
            static_assert(WM * WN * NG * (KS - 1) * 1024 <= STAGES * kSlot, "partial sums fit the ring");
            char* mine = lds + (size_t)(wm * WN + wn) * NG * (KS - 1) * 1024 + lane * 16;
            __syncthreads();                                  // every wave has left the ring
#pragma unroll
            for (int x = 0; x < NG; ++x) {
                const int j = x / GR / TM, i = x / GR % TM, g = x % GR, own = x % KS;
                if (ks != own)
                    *reinterpret_cast<float4*>(mine + (x * (KS - 1) + (ks < own ? ks : ks - 1)) * 1024) =
                        make_float4(acc[j][i][4 * g], acc[j][i][4 * g + 1], acc[j][i][4 * g + 2], acc[j][i][4 * g + 3]);
            }
            __syncthreads();
#pragma unroll
            for (int x = 0; x < NG; ++x) {
                const int j = x / GR / TM, i = x / GR % TM, g = x % GR, own = x % KS;
                if (ks == own) {
                    float c[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                    for (int k = 0; k < KS; ++k) {
                        float4 v = make_float4(acc[j][i][4 * g], acc[j][i][4 * g + 1], acc[j][i][4 * g + 2], acc[j][i][4 * g + 3]);
                        if (k != own) v = *reinterpret_cast<const float4*>(mine + (x * (KS - 1) + (k < own ? k : k - 1)) * 1024);
                        c[0] += v.x; c[1] += v.y; c[2] += v.z; c[3] += v.w;
                    }
                    store4(whole, i, j, g, c[0], c[1], c[2], c[3]);
                }
            }
        }
    };
    if ((N & 3) == 0) finish(std::true_type{});
    else finish(std::false_type{});
}

template <int DT, int TM, int TN, int WM, int WN, int KS, int SUB, bool KN, int VEC, int STAGES>
int launch_ring(const void* A, const void* W, void* C, const void* R, int M, int N, int K, float alpha, hipStream_t stream) {
    constexpr int BM = Traits<DT>::MB * TM * WM, BN = Traits<DT>::MB * TN * WN;
    constexpr int kLds = STAGES * SUB * (BM + BN) * kSlotRow;
    const auto kern = gemm_ring_kernel<DT, TM, TN, WM, WN, KS, SUB, KN, VEC, STAGES>;
    {
        const int rc = set_max_dynamic_lds((const void*)kern, kLds);
        if (rc != ROV_OK) return rc;
    }
    RingParams p;
    p.A = (const char*)A; p.W = (const char*)W; p.C = C; p.R = (const uint16_t*)R;
    p.M = M; p.N = N; p.K = K; p.alpha = alpha;
    p.tiles_m = (M + BM - 1) / BM;
    p.tiles_n = (N + BN - 1) / BN;
    const long long T = (long long)p.tiles_m * p.tiles_n;
    if (T > 0x7FFFFFFFLL) return ROV_ERR_UNSUPPORTED;
    hipLaunchKernelGGL(kern, dim3((unsigned)T), dim3(64 * WM * WN * KS), kLds, stream, p);
    ROV_LAUNCH_CHECK();
    return ROV_OK;
}

// The ring's depth by the product.  A long walk over k by one workgroup per compute unit wants every slot that LDS holds (64 x 32
// tiles, 128 x 4096 x 14336: five slots 34.5 us, three 39.5).  Several rounds of tiles, or a walk that ends soon, want the
// fewest, so that a second workgroup shares the compute unit and works while the first fills its ring or stores (three slots against five,
// 64 x 32: 1.04 to 1.2 times as fast below K = 2048, 304 x 1024 x 2048 0.98; 1.2 to 1.5 with more tiles than compute units; [K, N] 128 x 64, three against six:
// 1.02 to 1.15 and 1.15 to 1.28).
template <int DT, int TM, int TN, int WM, int WN, int KS, int SUB, bool KN, int VEC, int DEEP, int FEW>
int launch_ring_depth(const void* A, const void* W, void* C, const void* R, int M, int N, int K, float alpha, hipStream_t stream) {
    constexpr int BM = Traits<DT>::MB * TM * WM, BN = Traits<DT>::MB * TN * WN;
    const long long tiles = (long long)((M + BM - 1) / BM) * ((N + BN - 1) / BN);
    if (tiles <= device_cu_count() && (long long)K * Traits<DT>::ESZ >= 32 * kSlotRow)
        return launch_ring<DT, TM, TN, WM, WN, KS, SUB, KN, VEC, DEEP>(A, W, C, R, M, N, K, alpha, stream);
    return launch_ring<DT, TM, TN, WM, WN, KS, SUB, KN, VEC, FEW>(A, W, C, R, M, N, K, alpha, stream);
}

// ------------------------------------------------------------------ choice of the tile
// One row per instantiation: what it takes, its tile, and the time of one slot (128 bytes of k; 256 compute units
// busy) in nanoseconds, measured with K = 4096 at 128 to 1024 workgroups; for bf16 and fp8 [N, K] weights, where the 256-row
// kernels compete, adjusted so that none of 622 products of either type for which all forms were timed (16 to 4096 rows, 256 to
// 14336 columns, K of 512 to 14336) runs more than 2 % slower than with the 256-row kernel: fp8 128 x 64 at 280 chose this
// form where it was up to 28 % slower (700 x 8192 x 8192 68 us against 53, 300 x 14336 x 4096 36.5 against 30.5).  Rows on
// 4 bytes, which have no other matrix-core kernel, are fitted to 300 products of either layout instead (see there), fp32 to 1600 (see f32_tiles_ns).
// Register counts leave room
// for three 24-register RNG waves on every SIMD (a 256 x 128 tile with eight waves, 250 registers each, was up to
// 8 % faster than the 256-row kernel at 2048 x 4096 x 4096, but its workgroups could not be placed beside an RNG
// grid that arrived first).
struct RingVariant {
    int dtype, kn, vec, kparts;   // vec: bytes that the operands' rows start on
    int bm, bn;
    float slot_ns;
    int (*launch)(const void*, const void*, void*, const void*, int, int, int, float, hipStream_t);
    int min_slots;                // taken from this many slots of k on
};
constexpr int kRow4Slots = 8;
const RingVariant kRing[] = {
    //                                                                TM TN WM WN KS SUB KN   VEC ST
    {ROV_BF16, 0, 16, 4, 64, 32, 125.f, launch_ring_depth<ROV_BF16, 4, 2, 1, 1, 4, 2, false, 16, 5, 3>},
    {ROV_BF16, 0, 16, 2, 64, 64, 165.f, launch_ring<ROV_BF16, 2, 2, 2, 2, 2, 2, false, 16, 4>},
    {ROV_BF16, 0, 16, 2, 128, 64, 275.f, launch_ring<ROV_BF16, 4, 2, 2, 2, 2, 2, false, 16, 3>},
    {ROV_BF16, 0, 16, 2, 128, 128, 490.f, launch_ring<ROV_BF16, 4, 4, 2, 2, 2, 1, false, 16, 4>},
    {ROV_BF16, 0, 16, 2, 192, 128, 700.f, launch_ring<ROV_BF16, 6, 4, 2, 2, 2, 1, false, 16, 4>},
    {ROV_BF16, 0, 16, 2, 128, 192, 700.f, launch_ring<ROV_BF16, 4, 6, 2, 2, 2, 1, false, 16, 4>},
    {ROV_BF16, 0, 16, 1, 64, 64, 190.f, launch_ring<ROV_BF16, 2, 2, 2, 2, 1, 1, false, 16, 4>},
    {ROV_BF16, 0, 16, 1, 128, 128, 520.f, launch_ring<ROV_BF16, 4, 4, 2, 2, 1, 1, false, 16, 4>},
    {ROV_BF16, 0, 4, 2, 64, 64, 355.f, launch_ring<ROV_BF16, 2, 2, 2, 2, 2, 1, false, 4, 4>},
    {ROV_BF16, 1, 16, 4, 64, 64, 190.f, launch_ring<ROV_BF16, 4, 2, 1, 2, 4, 2, true, 16, 4>},
    {ROV_BF16, 1, 16, 2, 128, 64, 305.f, launch_ring_depth<ROV_BF16, 4, 2, 2, 2, 2, 1, true, 16, 6, 3>},
    {ROV_BF16, 1, 16, 2, 128, 128, 510.f, launch_ring<ROV_BF16, 4, 4, 2, 2, 2, 1, true, 16, 4>},
    {ROV_BF16, 1, 16, 2, 192, 128, 700.f, launch_ring<ROV_BF16, 6, 4, 2, 2, 2, 1, true, 16, 4>},
    {ROV_BF16, 1, 4, 2, 64, 64, 355.f, launch_ring<ROV_BF16, 2, 2, 2, 2, 2, 1, true, 4, 4>},
    {ROV_FP8_E4M3, 0, 16, 1, 64, 64, 172.f, launch_ring<ROV_FP8_E4M3, 2, 2, 2, 2, 1, 1, false, 16, 4>},
    {ROV_FP8_E4M3, 0, 16, 1, 128, 64, 315.f, launch_ring<ROV_FP8_E4M3, 2, 2, 4, 2, 1, 1, false, 16, 6>},
    {ROV_FP8_E4M3, 0, 16, 1, 128, 128, 530.f, launch_ring<ROV_FP8_E4M3, 4, 2, 2, 4, 1, 1, false, 16, 4>},
    {ROV_F32, 0, 16, 4, 32, 32, 140.f, launch_ring<ROV_F32, 1, 1, 1, 1, 4, 1, false, 16, 4>},
    {ROV_F32, 0, 16, 2, 64, 64, 510.f, launch_ring<ROV_F32, 1, 1, 2, 2, 2, 1, false, 16, 3>},
    {ROV_F32, 0, 4, 4, 32, 32, 148.f, launch_ring<ROV_F32, 1, 1, 1, 1, 4, 1, false, 4, 4>},
    {ROV_F32, 0, 4, 2, 64, 64, 510.f, launch_ring<ROV_F32, 1, 1, 2, 2, 2, 1, false, 4, 4>},
    {ROV_F32, 1, 16, 4, 32, 32, 142.f, launch_ring<ROV_F32, 1, 1, 1, 1, 4, 1, true, 16, 4>},
    {ROV_F32, 1, 16, 2, 64, 64, 510.f, launch_ring<ROV_F32, 1, 1, 2, 2, 2, 1, true, 16, 3>},
    {ROV_F32, 1, 4, 4, 32, 32, 154.f, launch_ring<ROV_F32, 1, 1, 1, 1, 4, 1, true, 4, 4>},
    {ROV_F32, 1, 4, 2, 64, 64, 510.f, launch_ring<ROV_F32, 1, 1, 2, 2, 2, 1, true, 4, 4>},
    // Rows on 4 bytes, longer sums: with 16-byte loads there too (see VEC) they take the larger tiles as well, from kRow4Slots slots of k on
    // (shorter sums are the output's time: the 64 x 64 tiles above).  Slot times fitted, with those of the 4-byte rows above, to 300 products of
    // either layout (32 to 6000 rows, 32 to 8000 columns, K of 2 to 14336): the choice is 0.4 % (0.7 % [K, N]) above the best
    // form on average, 15 % at worst.  With 4-byte loads and 64 x 64 tiles alone the same products took 1.56 (1.48) times as long:
    // 770 x 4090 x 14336 [K, N] 274 -> 107 us, 1000 x 2002 x 2002 28 -> 19, 200 x 1000 x 4090 26 -> 11.
    {ROV_BF16, 0, 4, 4, 64, 32, 245.f, launch_ring_depth<ROV_BF16, 4, 2, 1, 1, 4, 2, false, 4, 5, 3>, kRow4Slots},
    {ROV_BF16, 0, 4, 2, 128, 64, 545.f, launch_ring<ROV_BF16, 4, 2, 2, 2, 2, 2, false, 4, 3>, kRow4Slots},
    {ROV_BF16, 0, 4, 2, 128, 128, 869.f, launch_ring<ROV_BF16, 4, 4, 2, 2, 2, 1, false, 4, 4>, kRow4Slots},
    {ROV_BF16, 0, 4, 2, 192, 128, 1130.f, launch_ring<ROV_BF16, 6, 4, 2, 2, 2, 1, false, 4, 4>, kRow4Slots},
    {ROV_BF16, 1, 4, 4, 64, 64, 340.f, launch_ring<ROV_BF16, 4, 2, 1, 2, 4, 2, true, 4, 4>, kRow4Slots},
    {ROV_BF16, 1, 4, 2, 128, 64, 575.f, launch_ring_depth<ROV_BF16, 4, 2, 2, 2, 2, 1, true, 4, 6, 3>, kRow4Slots},
    {ROV_BF16, 1, 4, 2, 128, 128, 750.f, launch_ring<ROV_BF16, 4, 4, 2, 2, 2, 1, true, 4, 4>, kRow4Slots},
    {ROV_BF16, 1, 4, 2, 192, 128, 1016.f, launch_ring<ROV_BF16, 6, 4, 2, 2, 2, 1, true, 4, 4>, kRow4Slots},
};
constexpr int kRingVariants = (int)(sizeof(kRing) / sizeof(kRing[0]));

}  // namespace

// Nanoseconds for `tiles` tiles of `slots` slots at slot_ns each: rounds of one tile per compute unit, each with
// about 1.5 us of pipeline fill and output; a round that leaves compute units idle runs somewhat faster (L2 and the
// power limit are shared: 0.73 of the time at an empty chip, measured between 96 and 256 workgroups).
double gemm_tiles_ns(long long tiles, int slots, double slot_ns) {
    const long long ncu = device_cu_count(), rounds = (tiles + ncu - 1) / ncu;
    const double use = (double)tiles / (double)(rounds * ncu);
    return (double)rounds * ((double)slots * slot_ns * (0.73 + 0.27 * use) + 1500.0);
}

// fp32: several workgroups share a compute unit, so that a tile's fill and output lie beside another's walk, and idle units leave the
// others no clock (the matrix rate binds, not power): rounds of one tile per compute unit each take the walk and a little.  Measured a slot
// and round, ns: 32 x 32 165 to 180 in a lone round, 140 to 150 from two on; 64 x 64 505 to 530, 500.  Of 1600 products (16 to 8000 rows and
// columns, k of 2 to 4096) the choice is 0.07 % above the sooner form on average, 5 % at worst.  With the formula above and 64 x 64 at 715 ns, large products took
// 32 x 32 tiles: 1497 x 4040 x 1796 [K, N] 210 us against 177, 2830 x 3188 x 1956 332 against 291.
double f32_tiles_ns(long long tiles, int slots, double slot_ns, int rows) {
    const long long ncu = device_cu_count(), rounds = (tiles + ncu - 1) / ncu;
    return (double)rounds * ((double)slots * slot_ns + (rows == 32 ? 500.0 : 1000.0));
}

int ring_variant(int M, int N, int K, int dtype, int transB, bool same_order, double* ns) {
    const int esz = dtype == ROV_F32 ? 4 : dtype == ROV_BF16 ? 2 : 1;
    const bool kn = transB == 0;
    if (dtype == ROV_FP8_E4M3 && kn) return -1;
    // rows on 16 bytes (A and [N, K] weights: K elements, [K, N] weights: N) or on 4
    const unsigned long long row_a = (unsigned long long)K * esz, row_w = (unsigned long long)(kn ? N : K) * esz;
    const int vec = row_a % 16 == 0 && row_w % 16 == 0 ? 16 : row_a % 4 == 0 && row_w % 4 == 0 ? 4 : 0;
    // operand panels are addressed with 32-bit byte offsets (the last slot's overhang included)
    if (vec == 0 || 192ull * row_a + 1024 > 0xFFFFFFFFull) return -1;
    if ((kn ? (unsigned long long)K + 128 : 192ull) * row_w + 1024 > 0xFFFFFFFFull) return -1;
    const int slots = (int)((row_a + kSlotRow - 1) / kSlotRow);
    // Splitting k between waves changes the order of the sum, which the 256-row kernels share with the KS == 1
    // tiles.  Short sums keep it: below K = 2048 the split gains under a microsecond (708 x 4096 x 1024: 13.2 against
    // 14.0 us).
    const bool split = !same_order || K >= 2048;
    int best = -1;
    double best_ns = 0.0;
    for (int v = 0; v < kRingVariants; ++v) {
        const RingVariant& r = kRing[v];
        if (slots < r.min_slots || r.dtype != dtype || (r.kn != 0) != kn || r.vec != vec || (r.kparts > 1 && !split)) continue;
        const long long tiles = (long long)((M + r.bm - 1) / r.bm) * ((N + r.bn - 1) / r.bn);
        if (tiles > 0x7FFFFFFFLL) continue;
        const double t = dtype == ROV_F32 ? f32_tiles_ns(tiles, slots, r.slot_ns, r.bm) : gemm_tiles_ns(tiles, slots, r.slot_ns);
        if (best < 0 || t < best_ns) { best = v; best_ns = t; }
    }
    if (ns != nullptr) *ns = best_ns;
    return best;
}

void ring_variant_tile(int variant, int tile[4]) {
    const RingVariant& r = kRing[variant];
    tile[0] = r.bm; tile[1] = r.bn; tile[2] = r.kparts; tile[3] = r.vec;
}

int launch_gemm_ring(int variant, const void* A, const void* W, void* C, const void* R, int M, int N, int K, float alpha,
                     hipStream_t stream) {
    if (variant < 0 || variant >= kRingVariants) return ROV_ERR_INVALID;
    return kRing[variant].launch(A, W, C, R, M, N, K, alpha, stream);
}
}  // namespace rov
