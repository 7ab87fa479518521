// Flash-attention forward with dropout after softmax (paper Sec. 2.2, Sec. 6.1).
//
// Three ways to get the keep bits, all giving the same bits:
//   MODE_NONE  p == 0, no dropout;
//   MODE_MASK  the paper's "attention with element dropping": keep-mask words written
//              earlier by the stand-alone RNG kernel; a word is the 64 lanes' keep bits for
//              one accumulator register, fetched with scalar loads and applied with one
//              select per element;
//   MODE_FUSED the paper's fusion baseline: every lane runs Philox for its own elements.
//
// bf16 kernel, head dimension 64 or 128, on the matrix cores.  Everything is
// computed transposed, S^T = K Q^T and O^T = V^T P^T with MFMA 32x32x16, because
// then one lane owns one query column: the softmax statistics, the rescale of
// O and the mask word are per-lane scalars and only the row maximum needs one
// exchange between the two half-waves.  The S^T accumulator registers are, as
// they stand, the P^T operand of the second product if the 16 keys of a k-step
// are taken in the order the accumulator holds them; the matching V^T operand
// comes out of the row-major V tile with the gfx950 transpose load
// (ds_read_b64_tr_b16), two per fragment, so V is never copied transposed.
//
// A wave owns 32 query rows and walks the keys 64 at a time; the 8 waves of a
// workgroup (two per SIMD: while one waits for LDS or the matrix pipe the other
// issues) share each K / V tile through LDS, filled straight from global memory
// with buffer loads that write LDS (two stages, the next tile in flight while
// the current one is used).
//
// fp32 with head dimensions up to 128 has a matrix-core kernel of its own (attn_f32_kernel).  Any other
// case (other head dimensions, unaligned rows, fp32 problems of a few rows) takes a small one-wave-per-row
// kernel that is correct for every shape.
#include <hip/hip_runtime.h>

#include <type_traits>
#include <stdint.h>

#include "fp8_device.h"
#include "philox_device.h"
#include "rov_internal.h"

namespace rov {
namespace {

enum { MODE_NONE = 0, MODE_MASK = 1, MODE_FUSED = 2 };

struct AttnParams {
    const void* Q;
    const void* K;
    const void* V;
    void* O;
    const uint64_t* mask;
    int64_t sq[3], sk[3], sv[3], so[3];   // element strides (batch, token, head)
    int B, H, Hkv, S, d;
    int W;                                // mask tiles per side, ceil(S/32)
    int nq;                               // query blocks per (batch, head)
    int q_begin, q_end;                   // query rows computed by this launch: [q_begin, q_end)
    int mask_qt0, mask_nqt;               // tile rows the mask buffer holds: [mask_qt0, mask_qt0 + mask_nqt)
    int causal;
    float scale_log2;                     // log2(e) / sqrt(d)
    float inv_keep;                       // 1 / (1 - p)
    uint64_t offset;                      // Philox call offset (fused)
    uint32_t k0, k1;                      // Philox key (fused)
    uint32_t t_minus_1;                   // keep iff x <= t_minus_1 (fused)
    int rounds;                           // Philox rounds (fused)
    int bits;                             // random bits per element (fused): 8, 16 or 32
    uint32_t tb;                          // bits < 32: keep iff field < tb (fused)
    int o_fp8;                            // O is written as OCP e4m3 bytes of (value * o_inv_scale): fp8 block
    float o_inv_scale;
    int turn;                             // causal bf16, d = 64: the first `turn` workgroups of an XCD come in reversed order (0: none)
};

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void* lptr_t;

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    f32x2 v = {lo, hi};
    bf16x2 h = __builtin_convertvector(v, bf16x2);
    return *reinterpret_cast<uint32_t*>(&h);
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// max(v[lane], v[lane ^ 32]) in every lane.  v_permlane32_swap exchanges the upper 32 lanes of its
// first operand with the lower 32 of its second: with both operands v, one result holds the lower
// half-wave's values in both halves and the other the upper half-wave's.
__device__ __forceinline__ float half_wave_max(float v) {
    const uint32_t u = __float_as_uint(v);
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float half_wave_sum(float v) {
    const uint32_t u = __float_as_uint(v);
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// The same over the four lanes l, l ^ 16, l ^ 32, l ^ 48.
__device__ __forceinline__ float quarter_wave_max(float v) {
    const uint32_t u = __float_as_uint(v);
    const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    return half_wave_max(fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1])));
}
__device__ __forceinline__ float quarter_wave_sum(float v) {
    const uint32_t u = __float_as_uint(v);
    const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    return half_wave_sum(__uint_as_float(r[0]) + __uint_as_float(r[1]));
}

// BKV: keys per LDS tile
template <int D, int BKV>
struct Tile {
    static constexpr int kKRow = D * 2;                // bytes per K row in LDS
    static constexpr int kKBytes = BKV * kKRow;
    static constexpr int kStage = 2 * kKBytes;         // K tile then V tile, both [key][feature]
    static constexpr int kChunks = D / 8;              // 16-byte chunks per K row
};

// Swizzle of the 16-byte chunks of an LDS tile row (XORed into the chunk index), chosen for the
// way gfx950 serves LDS reads over its 64 banks of 4 bytes (lane sets measured with a two-lane
// probe and the bank-conflict counter):
//  * ds_read_b128 goes 16 lanes at a time, in the sets {0-3, 12-15, 20-27}, {4-11, 16-19, 28-31}
//    and the same + 32.  A K fragment read has lane = row (mod 32), chunk fixed, so a set holds
//    16 rows that need 16 (D = 128: row = 256 bytes) or, per row parity, 8 (D = 64) different
//    swizzle values: the position of the row within its set.
//  * ds_read_b64 (and its transposing form) goes 32 lanes at a time.  A V transpose read has, per
//    half-wave, 4 consecutive rows x 4 adjacent chunks x 2 halves; all rows alias (256-byte
//    rows) or alias by parity (128-byte rows), so the rows' groups of 4 chunks must differ.
template <int D, bool VTILE>
__device__ __forceinline__ int swizzle_of_row(int row) {
    if (VTILE) return D == 128 ? ((row & 3) << 2) : (((row >> 1) & 1) << 2);
    return D == 128 ? ((((row >> 3) & 3) << 2) | (row & 3)) : ((((row >> 3) & 3) << 1) | ((row >> 1) & 1));
}

// K or V tile: global -> LDS directly.  One wave instruction fills 1 KiB = 1024 / kKRow rows;
// lane L lands on physical chunk L % kChunks of its row and therefore fetches the logical
// chunk (L % kChunks) ^ swizzle(row).  The loads are buffer loads: a buffer resource over the
// rows [0, S) of this (batch, kv head) as scalar base, the lane's byte offset from the tile's
// first row (the same for every tile, computed once) as vector offset, and the tile's first
// row as scalar offset -- no per-lane address arithmetic in the loop.  Rows at or beyond S lie
// outside the resource's range and read as zeros (their scores are masked anyway).
// Inline assembly on purpose: the compiler's wait-count pass cannot tell the LDS write of such
// a load from the fragment reads of the other stage and would force vmcnt(0) before the
// second product of every tile, i.e. wait for the prefetch in the middle of the tile it was
// meant to run under; the kernel places its one vmcnt(0) per tile itself.  M0 (the LDS base of
// the transfer) is a reserved register that compiled code only sets right before its own uses.
typedef int i32x4 __attribute__((ext_vector_type(4)));
template <int D, int NW, bool VTILE, int BKV>
struct KvTileLoad {
    static constexpr int kChunks = Tile<D, BKV>::kChunks;
    static constexpr int kRowsPerInst = 64 / kChunks;          // 4 (D = 128) or 8 (D = 64)
    static constexpr int kInst = BKV / kRowsPerInst;           // 16 or 8 per tile
    static constexpr int kPerWave = kInst / NW;
    static_assert(kPerWave * NW == kInst, "every wave loads the same share");
    uint32_t off[kPerWave];
    uint32_t row_bytes;
    i32x4 rsrc;

    __device__ __forceinline__ void init(const uint16_t* Xp, int64_t tok_stride, int S, int wave, int lane) {
        const int rl = lane / kChunks, pc = lane % kChunks;
        row_bytes = (uint32_t)tok_stride * 2u;
#pragma unroll
        for (int i = 0; i < kPerWave; ++i) {
            const int row = (wave + NW * i) * kRowsPerInst + rl;          // 0..BKV-1
            const int chunk = pc ^ swizzle_of_row<D, VTILE>(row);
            off[i] = (uint32_t)row * row_bytes + (uint32_t)chunk * 16u;
        }
        const uint64_t base = (uint64_t)(uintptr_t)Xp;
        rsrc[0] = __builtin_amdgcn_readfirstlane((int)(uint32_t)base);
        rsrc[1] = __builtin_amdgcn_readfirstlane((int)(uint32_t)((base >> 32) & 0xFFFFu));
        rsrc[2] = __builtin_amdgcn_readfirstlane((int)((uint32_t)(S - 1) * row_bytes + (uint32_t)(D * 2)));
        rsrc[3] = 0x00020000;
    }

    // lds_tile: LDS byte address of the tile
    __device__ __forceinline__ void load(int kv0, uint32_t lds_tile, int wave) const {
        const uint32_t soff = (uint32_t)kv0 * row_bytes;
#pragma unroll
        for (int i = 0; i < kPerWave; ++i) {
            const uint32_t dst = lds_tile + (uint32_t)((wave + NW * i) * 1024);
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                         :: "s"(dst), "v"(off[i]), "s"(rsrc), "s"(soff) : "memory");
        }
    }
};

typedef const __attribute__((address_space(4))) uint64_t* const_u64_ptr;
typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) i16x4* lds_i16x4_ptr;

// ds_read_b64_tr_b16: within each group of 16 lanes, source lane r = 4*j + s supplies the
// address of 4 consecutive 16-bit elements, and lane i of the group receives element i%4 of
// the rows supplied by source lanes 4*j + i/4, j = 0..3.  If the four source lanes 4*j + s
// (s = 0..3) point at row key_j, columns c0 + 4*s .. +3, then lane i ends up with column
// c0 + i of rows key_0 .. key_3: a column fragment of a row-major tile, i.e. the transposed
// operand the second product needs, with no transposed copy of V anywhere.
__device__ __forceinline__ bf16x4 lds_read_transposed(const char* p) {
    const i16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4_ptr)p);
    return __builtin_bit_cast(bf16x4, v);
}

// NW waves per workgroup, each owning NQ*32 query rows.  (NQ, NW) = (2, 4) keeps one wave per
// SIMD with K/V fragments reused for two query tiles; (1, 8) puts two waves on every SIMD so
// that one wave's softmax VALU work runs under the other's MFMAs.
//
// KS > 1: the NW waves are NW / KS query tiles times KS key parts.  Of every LDS tile of 32 * KS keys
// (64 at least) a wave takes the 32 of its part; the KS partial results of a query tile (exponent reference, row
// sum, output) meet in LDS at the end.  A short sequence has too few query tiles for the chip - 512 tokens
// of 32 heads are 64 workgroups of 256 rows - and its time is the walk of one wave over the keys.
template <int D, int NQ, int NW, int KS, int MODE, int R = 10, int BITS = 32>
__global__ __launch_bounds__(NW * 64) void attn_bf16_kernel(const AttnParams p) {
    constexpr int QW = NW / KS;        // query tiles per workgroup
    constexpr int BQ = QW * 32 * NQ;   // query rows per workgroup
    constexpr int NT = KS == 1 ? 2 : 1;   // 32-key subtiles per wave and LDS tile
    constexpr int BKV = 32 * NT * KS;     // keys per LDS tile
    using T = Tile<D, BKV>;
    constexpr int KSTEPS = D / 16;   // k-steps of the first product
    constexpr int DVT = D / 32;   // dv tiles of the second product
    extern __shared__ __attribute__((aligned(1024))) char lds[];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ql = lane & 31;     // query column within a 32-wide tile
    const int half = lane >> 5;
    const int S = p.S;
    // Workgroup ids are dealt round-robin to the 8 XCDs.  All query blocks of one (batch, head)
    // go to the same XCD, so its K and V are fetched into one L2 only; within an XCD the order
    // is query block first, then head, so co-resident workgroups walk the same K/V in step.
    // Causal: heaviest query blocks first.  Where workgroups share a compute unit, the
    // order decides who shares: the first round of workgroups comes in reversed order then (see attn_turn), so that its lightest
    // get the second round's heaviest beside them.
    int qblk, bh;
    {
        const int pid = blockIdx.x, G = p.B * p.H, nq = p.nq;
        int j = pid >> 3, id = pid;
        if (D == 64) {
            j = j < p.turn ? p.turn - 1 - j : j;
            id = 8 * j + (pid & 7);
        }
        if ((G & 7) == 0) {
            const int xcd = pid & 7, gpx = G >> 3;
            qblk = j / gpx;
            bh = (j % gpx) * 8 + xcd;
        } else {
            qblk = id / G;
            bh = id % G;
        }
        if (p.causal) qblk = nq - 1 - qblk;
    }
    const int b = bh / p.H, h = bh % p.H;
    const int hk = h / (p.H / p.Hkv);
    const int kpart = wave % KS;
    const int q0 = p.q_begin + qblk * BQ + (wave / KS) * (32 * NQ);
    const int q_end = p.q_end;

    const uint16_t* Qp = (const uint16_t*)p.Q + b * p.sq[0] + h * p.sq[2];
    const uint16_t* Kp = (const uint16_t*)p.K + b * p.sk[0] + hk * p.sk[2];
    const uint16_t* Vp = (const uint16_t*)p.V + b * p.sv[0] + hk * p.sv[2];

    // Q fragments (second operand of K Q^T): lane holds query ql, features 16*ks + 8*half .. +7
    bf16x8 qf[NQ][KSTEPS];
    int qrow[NQ];
#pragma unroll
    for (int n = 0; n < NQ; ++n) {
        int q = q0 + 32 * n + ql;
        qrow[n] = q;
        q = q < q_end ? q : q_end - 1;
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks)
            qf[n][ks] = *reinterpret_cast<const bf16x8*>(Qp + (int64_t)q * p.sq[1] + 16 * ks + 8 * half);
    }

    f32x16 o[DVT][NQ];
#pragma unroll
    for (int t = 0; t < DVT; ++t)
#pragma unroll
        for (int n = 0; n < NQ; ++n)
#pragma unroll
            for (int e = 0; e < 16; ++e) o[t][n][e] = 0.0f;
    float m_run[NQ], l_run[NQ];
#pragma unroll
    for (int n = 0; n < NQ; ++n) { m_run[n] = -INFINITY; l_run[n] = 0.0f; }

    // number of KV tiles this workgroup walks (causal: up to its last query row)
    const int q_last = min(p.q_begin + qblk * BQ + BQ, q_end) - 1;
    const int kv_end = p.causal ? min(S, q_last + 1) : S;
    const int ntiles = (kv_end + BKV - 1) / BKV;

    // Keep words.  The mask is stored as 32 x 32 tiles of 16 words in accumulator order (see
    // rov.h): word e of tile (qt, kt) holds, in bit l, the keep bit of the element that lane l
    // has in accumulator register e of S^T tile (keys 32*kt.., queries 32*qt..).  The wave's
    // query tile is fixed, so its words for a KV tile are 2 x 16 consecutive, wave-uniform words:
    // MODE_MASK fetches them with scalar loads and applies each with one select; MODE_FUSED
    // needs no words at all, every lane draws the Philox outputs of its own elements.
    const uint32_t Tt = (uint32_t)p.W;                                    // tiles per side
    const uint64_t bh_tiles = ((uint64_t)b * p.H + h) * Tt;
    const uint64_t* mtile[NQ];      // words of tile (qt, 0) for each of the wave's query tiles
    uint64_t wtile[NQ];             // index of that word in the whole mask (fused: Philox numbering)
#pragma unroll
    for (int n = 0; n < NQ; ++n) {
        uint32_t qt = (uint32_t)(q0 / 32 + n);
        const uint32_t qt_last = (uint32_t)(p.mask_qt0 + p.mask_nqt - 1);
        qt = qt < qt_last ? qt : qt_last;                                 // rows past q_end are never stored
        wtile[n] = ((bh_tiles + qt) * Tt) * 16u;
        // the buffer holds mask_nqt tile rows per (batch, head), starting at tile row mask_qt0
        mtile[n] = p.mask + ((((uint64_t)b * p.H + h) * (uint32_t)p.mask_nqt + (qt - (uint32_t)p.mask_qt0)) * Tt) * 16u;
    }

    KvTileLoad<D, NW, false, BKV> kload;
    KvTileLoad<D, NW, true, BKV> vload;
    kload.init(Kp, p.sk[1], S, wave, lane);
    vload.init(Vp, p.sv[1], S, wave, lane);
    const uint32_t lds_base = (uint32_t)(uintptr_t)(lptr_t)lds;
    kload.load(0, lds_base, wave);
    vload.load(0, lds_base + T::kKBytes, wave);

    // transpose-load addressing of the V tile (see lds_read_transposed): lane l = 16*g + 4*j + s
    // supplies row 16*u + 8*x + 4*(g/2) + j, columns 32*t + 16*(g%2) + 4*s .. +3
    int vt_off[DVT];
    {
        const int g = lane >> 4, j = (lane >> 2) & 3, sl = lane & 3, hh = g >> 1;
        const int row_part = (4 * hh + j) * T::kKRow + (sl & 1) * 8;
        const int f = swizzle_of_row<D, true>(4 * hh + j);      // the row is 16u + 8x + 4hh + j: same value
#pragma unroll
        for (int t = 0; t < DVT; ++t)
            vt_off[t] = row_part + (((4 * t + 2 * (g & 1) + (sl >> 1)) ^ f) << 4);
    }

    const int kswz = swizzle_of_row<D, false>(ql);   // K fragment rows are 32t + ql: same value
    static_assert(NQ == 1, "the keep-word warm-up load covers one query tile per wave");
    uint32_t warm = 0u, sink = 0u;   // L2 warm-up of the next tile's keep words (MODE_MASK)

    // One KV tile.  The LDS stage is a compile-time constant (the loop below alternates the two
    // instantiations), so every fragment read is a loop-invariant lane address plus an immediate.
    auto tile_step = [&](const int jt, auto stage_tag) __attribute__((always_inline)) {
        constexpr int STAGE = decltype(stage_tag)::value;
        const int kv0 = jt * BKV;
        char* cur = lds + STAGE * T::kStage;
        __builtin_amdgcn_s_waitcnt(0x0070);   // vmcnt(0) lgkmcnt(0): this wave's K / V loads have landed
        __syncthreads();
        const bool has_next = jt + 1 < ntiles;
        if (has_next) {
            kload.load(kv0 + BKV, lds_base + (STAGE ^ 1) * T::kStage, wave);
            vload.load(kv0 + BKV, lds_base + (STAGE ^ 1) * T::kStage + T::kKBytes, wave);
        }
        const int kvw = kv0 + kpart * (32 * NT);   // this wave's keys: [kvw, kvw + 32 * NT)
        const char* curk = cur + kpart * (32 * NT) * T::kKRow;
        // ---- S^T = K Q^T for 32*NT keys x NQ*32 queries
        f32x16 s[NT][NQ];
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int n = 0; n < NQ; ++n)
#pragma unroll
                for (int e = 0; e < 16; ++e) s[t][n][e] = 0.0f;
        // K fragments are read kAhead k-steps before the MFMAs that use them: the scheduling
        // groups below pin that order (3 k-steps of reads, then per k-step its MFMAs followed by
        // the reads of the k-step kAhead further on), so the LDS latency is paid once per tile
        // and not once per k-step.
        constexpr int kAhead = NT == 2 ? 3 : 4;
        bf16x8 kf[KSTEPS][NT];
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks)
#pragma unroll
            for (int t = 0; t < NT; ++t)
                kf[ks][t] = *reinterpret_cast<const bf16x8*>(
                    curk + (32 * t + ql) * T::kKRow + (((2 * ks + half) ^ kswz) << 4));
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks)
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int n = 0; n < NQ; ++n)
                    s[t][n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks][t], qf[n][ks], s[t][n], 0, 0, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, NT * kAhead, 0);          // DS reads
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks) {
            __builtin_amdgcn_sched_group_barrier(0x008, NT * NQ, 0);          // MFMAs of k-step ks
            if (ks + kAhead < KSTEPS) __builtin_amdgcn_sched_group_barrier(0x100, NT, 0);
        }
        // nothing below moves up into the first product: a scalar load of keep words between its
        // LDS reads would turn every wait for a fragment into a wait for that load as well (the
        // two share one counter, and scalar loads return out of order)
        __builtin_amdgcn_sched_barrier(0);

        // ---- keep words of this KV tile: 2 key tiles x 16 words per query tile, wave-uniform.
        // They are requested here, right after the Q K^T MFMAs have been issued, through the
        // constant address space (memory nobody writes while this kernel runs), i.e. with
        // scalar loads into the SGPR pairs that the selects below use as lane predicates.  The
        // lines were pulled into L2 one tile earlier by `warm` (a vector load whose value is
        // only folded into a sink), so the scalar loads return while the row maxima and
        // exponentials are being computed.
        uint64_t mw[NQ][NT][16];
        const uint32_t kt0 = (uint32_t)(kvw >> 5);                           // first key tile of the wave
        if (MODE == MODE_MASK) {
#pragma unroll
            for (int n = 0; n < NQ; ++n)
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    uint32_t kt = kt0 + (uint32_t)t;
                    kt = kt < Tt ? kt : Tt - 1;
                    const const_u64_ptr wp = (const_u64_ptr)(uintptr_t)(mtile[n] + (uint64_t)kt * 16u);
#pragma unroll
                    for (int e = 0; e < 16; ++e) mw[n][t][e] = wp[e];
                }
            sink ^= warm;                       // the previous warm-up load has long landed
            // 32 * NT lanes x 4 bytes = the words of the wave's next NT key tiles (16 words if the tile row has a
            // single tile); clamped so that it never leaves this query tile's row
            uint32_t ktn = kt0 + (uint32_t)(BKV / 32);
            ktn = ktn + NT <= Tt ? ktn : (Tt >= NT ? Tt - NT : 0);
            warm = reinterpret_cast<const uint32_t*>(mtile[0] + (uint64_t)ktn * 16u)[lane & (Tt >= NT ? 32 * NT - 1 : 31)];
        }

        // ---- online softmax, dropout, P^T fragments
        bf16x8 pf[NQ][2 * NT];
        const bool tail = kvw + 32 * NT > S;
        const bool diag = p.causal && (kvw + 32 * NT - 1 > q0);   // some key may exceed a query
#pragma unroll
        for (int n = 0; n < NQ; ++n) {
            // the maximum is taken on the raw scores (the scale is positive) and the scale is folded
            // into the exponent's multiply-add below: one VALU op less per element
            float mx = -INFINITY;
            if (tail || diag) {   // wave-uniform: only the tiles on the diagonal and the last one
#pragma unroll
                for (int t = 0; t < NT; ++t)
#pragma unroll
                    for (int e = 0; e < 16; ++e) {
                        const int key = kvw + 32 * t + 8 * (e >> 2) + 4 * half + (e & 3);
                        const bool ok = key < S && (!p.causal || key <= qrow[n]);
                        s[t][n][e] = ok ? s[t][n][e] : -INFINITY;
                    }
            }
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int e = 0; e < 16; ++e) mx = fmaxf(mx, s[t][n][e]);
            // the other half-wave's maximum of the same query: a lane swap in the VALU (gfx950
            // v_permlane32_swap), not an LDS permute: the LDS counter is shared with the scalar
            // keep-word loads in flight, so waiting for a permute here would wait for them too
            mx = half_wave_max(mx) * p.scale_log2;
            // The reference of the exponent follows the maximum lazily: it moves only when the
            // tile's maximum exceeds it by more than kLazy (in log2 units), so entries reach at
            // most 2^kLazy, far inside fp32 and bf16 range, the quotient by the row sum is the
            // same softmax, and the rescale of the output accumulators below runs in the first
            // tile and hardly ever again (with the exact maximum about a third of all tiles of a
            // 16k sequence move some row's maximum).
            constexpr float kLazy = 8.0f;
            const float m_new = mx > m_run[n] + kLazy ? mx : m_run[n];
            const float m_safe = m_new == -INFINITY ? 0.0f : m_new;
            const float alpha = fast_exp2(m_run[n] - m_safe);
            m_run[n] = m_new;
            float sum = 0.0f;
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                uint32_t kt = kt0 + (uint32_t)t;
                kt = kt < Tt ? kt : Tt - 1;        // a key tile past S: its scores are -inf already
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const float pe = fast_exp2(__builtin_fmaf(s[t][n][e], p.scale_log2, -m_safe));
                    sum += pe;   // the normaliser counts dropped entries too
                    s[t][n][e] = pe;
                }
                if (MODE == MODE_MASK) {
#pragma unroll
                    for (int e = 0; e < 16; ++e)
                        s[t][n][e] = __builtin_amdgcn_inverse_ballot_w64(mw[n][t][e]) ? s[t][n][e] : 0.0f;
                }
                if (MODE == MODE_FUSED) {
                    // Words are taken in groups of E = 4 * 32 / BITS; word e = E*c + 4*f + r of this tile is
                    // decided by field f of output r of the lane's Philox call offset + 64*(first_word/E + c) + lane
                    // (BITS = 32: one field, the whole word)
                    constexpr int NF = 32 / BITS, E = 4 * NF;
                    const uint64_t g0 = (wtile[n] + (uint64_t)kt * 16u) / (uint32_t)E;
#pragma unroll
                    for (int c = 0; c < 16 / E; ++c) {
                        const uint64_t base = p.offset + 64u * (g0 + (uint64_t)c);
                        const uint32_t blo = (uint32_t)base, bhi = (uint32_t)(base >> 32);
                        const uint32_t c0 = blo + (uint32_t)lane;
                        uint32_t x[4];
                        if (blo <= 0xFFFFFFFFu - 63u) {
                            philox4x32_low_counter<R>(c0, bhi, p.k0, p.k1, x);
                        } else {
                            philox4x32<R>(c0, bhi + (c0 < blo ? 1u : 0u), 0u, 0u, p.k0, p.k1, x);
                        }
#pragma unroll
                        for (int f = 0; f < NF; ++f)
#pragma unroll
                            for (int r = 0; r < 4; ++r) {
                                const int e = E * c + 4 * f + r;
                                bool keep;
                                if (BITS == 32) keep = x[r] <= p.t_minus_1;
                                else keep = ((x[r] >> (BITS * f)) & ((1u << (BITS & 31)) - 1u)) < p.tb;
                                s[t][n][e] = keep ? s[t][n][e] : 0.0f;
                            }
                    }
                }
            }
            l_run[n] = l_run[n] * alpha + sum;
            // the running maximum settles after the first tiles; the rescale of the 64 output
            // accumulators is skipped while no lane of the wave has a new maximum (alpha == 1)
            if (__builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0ull) {
#pragma unroll
                for (int t = 0; t < DVT; ++t)
#pragma unroll
                    for (int e = 0; e < 16; ++e) o[t][n][e] *= alpha;
            }
            // (the keep words have been waited for: V fragments may be on their way from here)
            if (MODE == MODE_MASK) __builtin_amdgcn_sched_barrier(0);
            // k-step u = 2*t + v of the second product takes registers 8*v .. 8*v+7 of tile t
#pragma unroll
            for (int u = 0; u < 2 * NT; ++u) {
                const int t = u >> 1, v8 = (u & 1) * 8;
                uint32_t w[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) w[e] = pack_bf16x2(s[t][n][v8 + 2 * e], s[t][n][v8 + 2 * e + 1]);
                pf[n][u] = *reinterpret_cast<bf16x8*>(w);
            }
        }

        // ---- O^T += V^T P^T
        // MODE_MASK: V fragments are read kAheadV fragments before the MFMA that uses them (the groups below pin
        // that order; left to itself the compiler reads a fragment, waits for it and issues its MFMA, sixteen LDS
        // latencies in a row).  S = 16384, 32 heads, d = 128: 4136 -> 4025 us; 4 or 6 ahead are no faster.  Without
        // keep words the other wave of the SIMD covers those latencies and the pinned order is 0.5 % slower.
        const char* vt = curk + T::kKBytes;
        constexpr int kAheadV = 2;
        bf16x8 vf[2 * NT][DVT];
#pragma unroll
        for (int u = 0; u < 2 * NT; ++u)
#pragma unroll
            for (int t = 0; t < DVT; ++t) {
                // keys 16u + 4*half + 0..3 and 16u + 8 + 4*half + 0..3 of feature 32t + lane%32
                const bf16x4 lo = lds_read_transposed(vt + (16 * u) * T::kKRow + vt_off[t]);
                const bf16x4 hi = lds_read_transposed(vt + (16 * u + 8) * T::kKRow + vt_off[t]);
                vf[u][t] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
            }
#pragma unroll
        for (int u = 0; u < 2 * NT; ++u)
#pragma unroll
            for (int t = 0; t < DVT; ++t)
#pragma unroll
                for (int n = 0; n < NQ; ++n)
                    o[t][n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[u][t], pf[n][u], o[t][n], 0, 0, 0);
        if (MODE == MODE_MASK) {
            __builtin_amdgcn_sched_group_barrier(0x100, 2 * kAheadV, 0);
#pragma unroll
            for (int i = 0; i < 2 * NT * DVT; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, NQ, 0);
                if (i + kAheadV < 2 * NT * DVT) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
            }
        }
    };
    // Tiles in which some query of this wave admits some key of its part; in the workgroup's others (a causal
    // workgroup's last ones, a part beyond S) the probabilities are zero: the wave only loads its share.
    const int key_end = p.causal ? min(S, q0 + 32 * NQ) : S;
    const int nwave = min(ntiles, max(0, (key_end - kpart * (32 * NT) + BKV - 1) / BKV));
    for (int jt = 0; jt < nwave; jt += 2) {
        tile_step(jt, std::integral_constant<int, 0>{});
        if (jt + 1 < nwave) tile_step(jt + 1, std::integral_constant<int, 1>{});
    }
    for (int jt = nwave; jt < ntiles; ++jt) {
        __builtin_amdgcn_s_waitcnt(0x0070);
        __syncthreads();
        if (jt + 1 < ntiles) {
            const uint32_t at = lds_base + (uint32_t)((jt + 1) & 1) * T::kStage;
            kload.load((jt + 1) * BKV, at, wave);
            vload.load((jt + 1) * BKV, at + T::kKBytes, wave);
        }
    }

    // the warm-up values only have to look used (no mask pattern makes this condition true
    // for a lane id >= 64)
    if (MODE == MODE_MASK && (sink ^ warm) == 0x9E3779B9u && lane == 1000) m_run[0] = 0.0f;

    // ---- normalise, scale kept entries by 1/(1-p), store O (lane: query ql, 4 consecutive dv per register group)
    // The output's parameters are read again here: held since the kernel's start they push the scalar registers of
    // the loop (64 of them keep words) into spills.
    typedef const __attribute__((address_space(4))) AttnParams* params_ptr;
    params_ptr pe = (params_ptr)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(pe));
    const int64_t so_b = pe->so[0], so_s = pe->so[1], so_h = pe->so[2];
    uint8_t* const Oe = (uint8_t*)pe->O;
    const int qe = pe->q_end, o_fp8 = pe->o_fp8;
    const float inv_keep = pe->inv_keep, o_scale = o_fp8 ? pe->o_inv_scale : 1.0f;
    auto store_group = [&](int n, int t, int g, float c0, float c1, float c2, float c3) {
        if (qrow[n] >= qe) return;
        if (o_fp8) {
            // the fp8 block quantises the attention output where it is produced (strides count bytes here)
            uint8_t* orow = Oe + b * so_b + h * so_h + (int64_t)qrow[n] * so_s;
            *reinterpret_cast<uint32_t*>(orow + 32 * t + 8 * g + 4 * half) = pack_e4m3x4(c0, c1, c2, c3);   // o_scale is in the factors
        } else {
            uint16_t* orow = (uint16_t*)Oe + b * so_b + h * so_h + (int64_t)qrow[n] * so_s;
            *reinterpret_cast<uint2*>(orow + 32 * t + 8 * g + 4 * half) = make_uint2(pack_bf16x2(c0, c1), pack_bf16x2(c2, c3));
        }
    };
    if constexpr (KS == 1) {
#pragma unroll
        for (int n = 0; n < NQ; ++n) {
            const float l = half_wave_sum(l_run[n]);
            const float f = (l > 0.0f ? inv_keep / l : 0.0f) * o_scale;
#pragma unroll
            for (int t = 0; t < DVT; ++t)
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    store_group(n, t, g, o[t][n][4 * g + 0] * f, o[t][n][4 * g + 1] * f, o[t][n][4 * g + 2] * f,
                                o[t][n][4 * g + 3] * f);
        }
    } else {
        static_assert(NQ == 1, "one query tile per wave");
        // (reference, row sum) of every part, then the outputs on a common reference; register group x = (t, g) of
        // a query tile is added up, parts in order, and stored by part x % KS
        constexpr int NX = DVT * 4;
        static_assert(QW * NX * (KS - 1) * 1024 <= 2 * T::kStage && NW * 64 * 8 <= 2 * T::kStage, "partial results fit the tiles' LDS");
        float2* ml = reinterpret_cast<float2*>(lds);
        __syncthreads();                                  // every wave has left the K / V tiles
        ml[wave * 64 + lane] = make_float2(m_run[0], half_wave_sum(l_run[0]));
        __syncthreads();
        float m_all = -INFINITY, l = 0.0f;
        float2 part[KS];
#pragma unroll
        for (int k = 0; k < KS; ++k) {
            part[k] = ml[((wave / KS) * KS + k) * 64 + lane];
            m_all = fmaxf(m_all, part[k].x);
        }
        const float m_ref = m_all == -INFINITY ? 0.0f : m_all;
#pragma unroll
        for (int k = 0; k < KS; ++k) l += part[k].y * fast_exp2(part[k].x - m_ref);
        const float f = (l > 0.0f ? inv_keep / l : 0.0f) * o_scale * fast_exp2(m_run[0] - m_ref);
        __syncthreads();
        char* mine = lds + (wave / KS) * NX * (KS - 1) * 1024 + lane * 16;
#pragma unroll
        for (int x = 0; x < NX; ++x) {
            const int t = x >> 2, g = x & 3, own = x % KS;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[t][0][4 * g + e] *= f;
            if (kpart != own)
                *reinterpret_cast<float4*>(mine + (x * (KS - 1) + (kpart < own ? kpart : kpart - 1)) * 1024) =
                    make_float4(o[t][0][4 * g], o[t][0][4 * g + 1], o[t][0][4 * g + 2], o[t][0][4 * g + 3]);
        }
        __syncthreads();
#pragma unroll
        for (int x = 0; x < NX; ++x) {
            const int t = x >> 2, g = x & 3, own = x % KS;
            if (kpart == own) {
                float c[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int k = 0; k < KS; ++k) {
                    float4 v = make_float4(o[t][0][4 * g], o[t][0][4 * g + 1], o[t][0][4 * g + 2], o[t][0][4 * g + 3]);
                    if (k != own) v = *reinterpret_cast<const float4*>(mine + (x * (KS - 1) + (k < own ? k : k - 1)) * 1024);
                    c[0] += v.x; c[1] += v.y; c[2] += v.z; c[3] += v.w;
                }
                store_group(0, t, g, c[0], c[1], c[2], c[3]);
            }
        }
    }
}

// ------------------------------------------------------------------ fp32 kernel
// fp32, head dimension d a multiple of 8 with DP - 32 < d <= DP, on the fp32 matrix instructions (32x32x2).  Transposed like the
// bf16 kernel (S^T = K Q^T, O^T = V^T P^T; a lane owns one query), so the score registers are the second
// product's operand as they stand and a mask word is one register's lane predicate.  A workgroup owns 32 query
// rows; its NW waves take every NW-th tile of 32 keys and merge their (maximum, sum, output) in LDS at the end:
// fp32 sequences are short, and without the split a wave's walk over the keys is the whole time.  K and V
// go straight from global memory into the operand registers (every byte is used by one wave of the workgroup
// only); a lane's K fragment is 16 bytes of a row, a V fragment 128 contiguous bytes per half-wave.
// The merge has one barrier (four before: 1.7 % on average over 60 problems of 192 to 3000 tiles, none slower,
// 2 x 952 x 4 x 64 34.7 -> 30.8 us).
// Bound: matrix cores at long sequences (4 flop per score and feature at 157 TFLOP/s), one tile's chain of load,
// product, softmax, product at short ones.  Before it the one-row-per-wave kernel below did this: 1024 tokens x 8 heads x
// 64 features 331 us with a stored mask, now 27 (4096 tokens: 4728, 301 = 114 TFLOP/s).
template <int DP, int NW, int MODE, int BITS>
__global__ __launch_bounds__(NW * 64) void attn_f32_kernel(const AttnParams p) {
    constexpr int KC = DP / 8;     // chunks of 8 features: the k range of four MFMAs
    constexpr int DVT = DP / 32;   // feature tiles
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ql = lane & 31, half = lane >> 5;
    const int S = p.S, d = p.d;
    int qblk, bh;   // all query tiles of a (batch, head) on one XCD, heaviest first when causal
    {
        const int pid = blockIdx.x, G = p.B * p.H;
        if ((G & 7) == 0) {
            const int xcd = pid & 7, j = pid >> 3, gpx = G >> 3;
            qblk = j / gpx;
            bh = (j % gpx) * 8 + xcd;
        } else {
            qblk = pid / G;
            bh = pid % G;
        }
        if (p.causal) qblk = p.nq - 1 - qblk;
    }
    const int b = bh / p.H, h = bh % p.H;
    const int hk = h / (p.H / p.Hkv);
    const int q0 = p.q_begin + qblk * 32, qrow = q0 + ql;
    const float* Qp = (const float*)p.Q + b * p.sq[0] + h * p.sq[2] + (int64_t)min(qrow, p.q_end - 1) * p.sq[1];
    // K and V of this (batch, kv head) as buffer resources over the rows [0, S): lane offset plus tile row, no
    // 64-bit address per register, and rows at or beyond S read as zeros.  The check compares the lane offset with
    // what the scalar offset leaves of the size, so the scalar offset itself stays within the size: a tile's first row for
    // K, no row beyond the last for V (vlast).
    const uint32_t krow = (uint32_t)p.sk[1] * 4u, vrow = (uint32_t)p.sv[1] * 4u;
    const __amdgpu_buffer_rsrc_t kres = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float*>((const float*)p.K + b * p.sk[0] + hk * p.sk[2]), 0, (int)((uint32_t)(S - 1) * krow + (uint32_t)d * 4u), 0x00020000);
    const __amdgpu_buffer_rsrc_t vres = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float*>((const float*)p.V + b * p.sv[0] + hk * p.sv[2]), 0, (int)((uint32_t)(S - 1) * vrow + (uint32_t)d * 4u), 0x00020000);

    // features 8c + 4*half .. +3 of the lane's row; chunks at or beyond d are zeros (an offset outside the resource)
    f32x4 qf[KC], kf[KC];
#pragma unroll
    for (int c = 0; c < KC; ++c)
        qf[c] = 8 * c < d ? *reinterpret_cast<const f32x4*>(Qp + 8 * c + 4 * half) : f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    const uint32_t koff = (uint32_t)ql * krow + (uint32_t)half * 16u;
    auto load_k = [&](int kv0) {
#pragma unroll
        for (int c = 0; c < KC; ++c)
            kf[c] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                kres, koff + (8 * c < d ? 32u * c : 0x80000000u), (uint32_t)kv0 * krow, 0));
    };

    const uint32_t Tt = (uint32_t)p.W;
    const uint32_t qt = (uint32_t)q0 >> 5;
    const uint64_t wtile = (((uint64_t)bh * Tt + qt) * Tt) * 16u;   // words of tile (qt, 0) in the whole mask
    const uint64_t* mtile = p.mask + (((uint64_t)bh * (uint32_t)p.mask_nqt + (qt - (uint32_t)p.mask_qt0)) * Tt) * 16u;

    f32x16 o[DVT];
#pragma unroll
    for (int t = 0; t < DVT; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e) o[t][e] = 0.0f;
    float m_run = -INFINITY, l_run = 0.0f;

    uint32_t voff[DVT];
#pragma unroll
    for (int t = 0; t < DVT; ++t) voff[t] = (uint32_t)(4 * half) * vrow + (uint32_t)min(32 * t + ql, d - 1) * 4u;
    const uint32_t vlast = (uint32_t)(S - 1) * vrow;
    const int kv_end = p.causal ? min(S, q0 + 32) : S;
    const int nkt = (kv_end + 31) / 32;
    if (wave < nkt) load_k(32 * wave);
#pragma unroll 1
    for (int kt = wave; kt < nkt; kt += NW) {
        const int kv0 = 32 * kt;
        // V: register e of feature tile t is the lane's feature 32t + ql of key kv0 + 8*(e/4) + 4*half + e%4, the key
        // of score register e.  Features beyond d repeat the last one (their outputs are not stored); keys beyond S are the
        // last key's values or zeros, under probabilities of zero.
        float vf[DVT][16];
#pragma unroll
        for (int e = 0; e < 16; ++e)
#pragma unroll
            for (int t = 0; t < DVT; ++t)
                vf[t][e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
                    vres, voff[t], min((uint32_t)kv0 * vrow + (uint32_t)(8 * (e >> 2) + (e & 3)) * vrow, vlast), 0));
        uint64_t mw[16];
        if (MODE == MODE_MASK) {
            const const_u64_ptr wp = (const_u64_ptr)(uintptr_t)(mtile + (uint64_t)kt * 16u);
#pragma unroll
            for (int e = 0; e < 16; ++e) mw[e] = wp[e];
        }
        f32x16 s;
#pragma unroll
        for (int e = 0; e < 16; ++e) s[e] = 0.0f;
#pragma unroll
        for (int c = 0; c < KC; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e) s = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[c][e], qf[c][e], s, 0, 0, 0);
        if (kt + NW < nkt) load_k(kv0 + 32 * NW);

        const bool edge = kv0 + 32 > S || (p.causal && kv0 + 31 > q0);   // some score is not admissible
        if (edge) {
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int key = kv0 + 8 * (e >> 2) + 4 * half + (e & 3);
                s[e] = key < S && (!p.causal || key <= qrow) ? s[e] : -INFINITY;
            }
        }
        float mx = s[0];
#pragma unroll
        for (int e = 1; e < 16; ++e) mx = fmaxf(mx, s[e]);
        mx = half_wave_max(mx) * p.scale_log2;
        const float m_new = fmaxf(m_run, mx);
        const float m_safe = m_new == -INFINITY ? 0.0f : m_new;
        const float alpha = fast_exp2(m_run - m_safe);
        m_run = m_new;
        float sum = 0.0f;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            s[e] = fast_exp2(__builtin_fmaf(s[e], p.scale_log2, -m_safe));
            sum += s[e];   // the normaliser counts dropped entries too
        }
        if (MODE == MODE_MASK) {
#pragma unroll
            for (int e = 0; e < 16; ++e) s[e] = __builtin_amdgcn_inverse_ballot_w64(mw[e]) ? s[e] : 0.0f;
        }
        if (MODE == MODE_FUSED) {
            constexpr int NF = 32 / BITS, E = 4 * NF;   // fields per output word, mask words per call (see attn_bf16_kernel)
            const uint64_t g0 = (wtile + (uint64_t)kt * 16u) / (uint32_t)E;
#pragma unroll
            for (int c = 0; c < 16 / E; ++c) {
                const uint64_t n = p.offset + 64u * (g0 + (uint64_t)c) + (uint64_t)lane;
                uint32_t x[4];
                if (p.rounds == 10) philox4x32<10>((uint32_t)n, (uint32_t)(n >> 32), 0u, 0u, p.k0, p.k1, x);
                else philox4x32_dyn(p.rounds, (uint32_t)n, (uint32_t)(n >> 32), 0u, 0u, p.k0, p.k1, x);
#pragma unroll
                for (int f = 0; f < NF; ++f)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        bool keep;
                        if (BITS == 32) keep = x[r] <= p.t_minus_1;
                        else keep = ((x[r] >> (BITS * f)) & ((1u << (BITS & 31)) - 1u)) < p.tb;
                        s[E * c + 4 * f + r] = keep ? s[E * c + 4 * f + r] : 0.0f;
                    }
            }
        }
        l_run = l_run * alpha + sum;
#pragma unroll
        for (int t = 0; t < DVT; ++t)
#pragma unroll
            for (int e = 0; e < 16; ++e) o[t][e] *= alpha;
        // On the diagonal a probability of an inadmissible key is zero, but zero times a non-finite value is
        // not: such a tile (never, in ordinary data) takes its keys one by one, each added where it is admissible.
        bool finite = true;
        if (edge) {
#pragma unroll
            for (int t = 0; t < DVT; ++t)
#pragma unroll
                for (int e = 0; e < 16; ++e) finite = finite && fabsf(vf[t][e]) < INFINITY;
            finite = __builtin_amdgcn_ballot_w64(!finite) == 0ull;
        }
        if (finite) {
#pragma unroll
            for (int e = 0; e < 16; ++e)
#pragma unroll
                for (int t = 0; t < DVT; ++t) o[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(vf[t][e], s[e], o[t], 0, 0, 0);
        } else {
#pragma unroll 1
            for (int k = 0; k < 32; ++k) {
                const int key = kv0 + k;
                f32x16 one[DVT];
#pragma unroll
                for (int t = 0; t < DVT; ++t)
#pragma unroll
                    for (int e = 0; e < 16; ++e) one[t][e] = 0.0f;
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const bool here = 8 * (e >> 2) + 4 * half + (e & 3) == k;
                    const float pe = here ? s[e] : 0.0f;
#pragma unroll
                    for (int t = 0; t < DVT; ++t)
                        one[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(here ? vf[t][e] : 0.0f, pe, one[t], 0, 0, 0);
                }
                const bool adm = key < S && (!p.causal || key <= qrow);
#pragma unroll
                for (int t = 0; t < DVT; ++t)
#pragma unroll
                    for (int e = 0; e < 16; ++e) o[t][e] += adm ? one[t][e] : 0.0f;
            }
        }
    }

    // The waves' partial results meet in LDS, not used before: (maximum, sum) and output of each.  Register group x = (t, g) is
    // brought on the common maximum and added up, waves in order, by wave x % NW.
    constexpr int NX = DVT * 4;
    static_assert(NX % NW == 0 || NW % NX == 0, "groups are dealt out evenly");
    float2* ml = reinterpret_cast<float2*>(lds + NX * (NW - 1) * 1024);
    {
        const float l_all = half_wave_sum(l_run);
        if (half == 0) ml[wave * 32 + ql] = make_float2(m_run, l_all);
    }
#pragma unroll
    for (int x = 0; x < NX; ++x) {
        const int t = x >> 2, g = x & 3, own = x % NW;
        if (wave != own)
            *reinterpret_cast<float4*>(lds + ((x * (NW - 1) + (wave < own ? wave : wave - 1)) * 64 + lane) * 16) =
                make_float4(o[t][4 * g], o[t][4 * g + 1], o[t][4 * g + 2], o[t][4 * g + 3]);
    }
    __syncthreads();
    float m_all = -INFINITY, l = 0.0f, f[NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        f[w] = ml[w * 32 + ql].x;
        m_all = fmaxf(m_all, f[w]);
    }
    const float m_ref = m_all == -INFINITY ? 0.0f : m_all;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        f[w] = fast_exp2(f[w] - m_ref);
        l += ml[w * 32 + ql].y * f[w];
    }
    // (a row whose scores are all -infinity has no softmax: NaN)
    const float norm = m_all == -INFINITY ? __uint_as_float(0x7FC00000u) : l > 0.0f ? p.inv_keep / l : 0.0f;
    float* orow = (float*)p.O + b * p.so[0] + h * p.so[2] + (int64_t)qrow * p.so[1];
#pragma unroll
    for (int x = 0; x < NX; ++x) {
        const int t = x >> 2, g = x & 3, own = x % NW;
        const int feat = 32 * t + 8 * g + 4 * half;
        if (wave == own) {
            f32x4 c = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                f32x4 v = {o[t][4 * g], o[t][4 * g + 1], o[t][4 * g + 2], o[t][4 * g + 3]};
                if (w != own) v = *reinterpret_cast<const f32x4*>(lds + ((x * (NW - 1) + (w < own ? w : w - 1)) * 64 + lane) * 16);
                c += v * (norm * f[w]);
            }
            if (qrow < p.q_end && feat < d) *reinterpret_cast<f32x4*>(orow + feat) = c;
        }
    }
}

// The same on 16 x 16 x 4 instructions, for problems whose 32-query tiles leave the chip idle: a workgroup owns 16 query rows, a wave
// takes every NW-th block of 16 keys, so there are twice as many workgroups and a block's chain of load, product, softmax, product is
// a quarter as long.  Lane l holds query l % 16 and keys 4 * (l / 16) + e of a block: the score registers are the second product's
// operand as they stand here too.  The keep word of register e is word 4 * (2 * (block % 2) + (l / 16) / 2) + e of the 32 x 32 tile, its
// bit 32 * (l / 16 % 2) + query % 32: read as the lane's half word (stored mask) or drawn by the lane (same call, same field).
// Each K and V byte is read by twice as many workgroups: see attn_f32_q16 for where that begins to cost more.
// us, 32-query tiles -> this: 128 tokens x 2 heads x 64 features (stored mask) 8.1 -> 6.5; 400 x 2 x 128 27.2 -> 17.7; 2 x 359 x 8 x 64 causal,
// bits drawn here, 16.1 -> 11.7.
template <int DP, int NW, int MODE, int BITS>
__global__ __launch_bounds__(NW * 64) void attn_f32_q16_kernel(const AttnParams p) {
    constexpr int KC = DP / 16;    // chunks of 16 features: the k range of four MFMAs, and the output's feature blocks
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ql = lane & 15, g = lane >> 4;
    const int S = p.S, d = p.d;
    int qblk, bh;   // all query tiles of a (batch, head) on one XCD, heaviest first when causal
    {
        const int pid = blockIdx.x, G = p.B * p.H;
        if ((G & 7) == 0) {
            const int xcd = pid & 7, j = pid >> 3, gpx = G >> 3;
            qblk = j / gpx;
            bh = (j % gpx) * 8 + xcd;
        } else {
            qblk = pid / G;
            bh = pid % G;
        }
        if (p.causal) qblk = p.nq - 1 - qblk;
    }
    const int b = bh / p.H, h = bh % p.H;
    const int hk = h / (p.H / p.Hkv);
    const int q0 = p.q_begin + qblk * 16, qrow = q0 + ql;
    const float* Qp = (const float*)p.Q + b * p.sq[0] + h * p.sq[2] + (int64_t)min(qrow, p.q_end - 1) * p.sq[1];
    // (resources and offsets as in attn_f32_kernel)
    const uint32_t krow = (uint32_t)p.sk[1] * 4u, vrow = (uint32_t)p.sv[1] * 4u;
    const __amdgpu_buffer_rsrc_t kres = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float*>((const float*)p.K + b * p.sk[0] + hk * p.sk[2]), 0, (int)((uint32_t)(S - 1) * krow + (uint32_t)d * 4u), 0x00020000);
    const __amdgpu_buffer_rsrc_t vres = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float*>((const float*)p.V + b * p.sv[0] + hk * p.sv[2]), 0, (int)((uint32_t)(S - 1) * vrow + (uint32_t)d * 4u), 0x00020000);

    // features 16c + 4g .. +3 of the lane's row; chunks at or beyond d are zeros (an offset outside the resource)
    f32x4 qf[KC], kf[KC];
#pragma unroll
    for (int c = 0; c < KC; ++c)
        qf[c] = 16 * c + 4 * g < d ? *reinterpret_cast<const f32x4*>(Qp + 16 * c + 4 * g) : f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    const uint32_t koff = (uint32_t)ql * krow + (uint32_t)g * 16u;
    auto load_k = [&](int kv0) {
#pragma unroll
        for (int c = 0; c < KC; ++c)
            kf[c] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                kres, 16 * c + 4 * g < d ? koff + 64u * c : 0x80000000u, (uint32_t)kv0 * krow, 0));
    };
    // V: register (t, e) is the lane's feature 16t + l % 16 of key kv0 + 4g + e.  Features beyond d repeat the last one (their outputs
    // are not stored); keys beyond S are the last key's values, under probabilities of zero.
    float vf[KC][4];
    uint32_t voff[KC];
#pragma unroll
    for (int t = 0; t < KC; ++t) voff[t] = (uint32_t)min(16 * t + ql, d - 1) * 4u;
    auto load_v = [&](int kv0) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t row = (uint32_t)min(kv0 + 4 * g + e, S - 1) * vrow;
#pragma unroll
            for (int t = 0; t < KC; ++t) vf[t][e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(vres, voff[t] + row, 0, 0));
        }
    };

    const uint32_t Tt = (uint32_t)p.W;
    const uint32_t qt = (uint32_t)q0 >> 5;
    const uint64_t wtile = (((uint64_t)bh * Tt + qt) * Tt) * 16u;   // words of tile (qt, 0) in the whole mask
    const uint64_t* mtile = p.mask + (((uint64_t)bh * (uint32_t)p.mask_nqt + (qt - (uint32_t)p.mask_qt0)) * Tt) * 16u;
    const uint32_t qbit = (uint32_t)qrow & 31u, bit = 32u * (uint32_t)(g & 1) + qbit;

    f32x4 o[KC];
#pragma unroll
    for (int t = 0; t < KC; ++t) o[t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    float m_run = -INFINITY, l_run = 0.0f;
    const int kv_end = p.causal ? min(S, q0 + 16) : S;
    const int nkb = (kv_end + 15) / 16;
    uint32_t mw[4];
    auto load_mask = [&](int kb) {
        const uint32_t* w = reinterpret_cast<const uint32_t*>(mtile + (uint64_t)(kb >> 1) * 16u + 4u * (uint32_t)(2 * (kb & 1) + (g >> 1))) + (g & 1);
#pragma unroll
        for (int e = 0; e < 4; ++e) mw[e] = w[2 * e];
    };
    if (wave < nkb) {
        load_k(16 * wave);
        if (MODE == MODE_MASK) load_mask(wave);
        load_v(16 * wave);
    }
#pragma unroll 1
    for (int kb = wave; kb < nkb; kb += NW) {
        const int kv0 = 16 * kb;
        const bool more = kb + NW < nkb;
        f32x4 s = {0.0f, 0.0f, 0.0f, 0.0f}, s2 = s;   // (two chains: an instruction's result takes longer than its issue)
#pragma unroll
        for (int c = 0; c < KC; ++c) {
#pragma unroll
            for (int e = 0; e < 4; e += 2) {
                s = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[c][e], qf[c][e], s, 0, 0, 0);
                s2 = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[c][e + 1], qf[c][e + 1], s2, 0, 0, 0);
            }
        }
        if (more) load_k(kv0 + 16 * NW);
        s += s2;
        const bool edge = kv0 + 16 > S || (p.causal && kv0 + 15 > q0);   // some score is not admissible
        if (edge) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int key = kv0 + 4 * g + e;
                s[e] = key < S && (!p.causal || key <= qrow) ? s[e] : -INFINITY;
            }
        }
        float mx = fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]));
        mx = quarter_wave_max(mx) * p.scale_log2;
        const float m_new = fmaxf(m_run, mx);
        const float m_safe = m_new == -INFINITY ? 0.0f : m_new;
        const float alpha = fast_exp2(m_run - m_safe);
        m_run = m_new;
        float sum = 0.0f;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            s[e] = fast_exp2(__builtin_fmaf(s[e], p.scale_log2, -m_safe));
            sum += s[e];   // the normaliser counts dropped entries too
        }
        if (MODE == MODE_MASK) {
#pragma unroll
            for (int e = 0; e < 4; ++e) s[e] = (mw[e] >> qbit) & 1u ? s[e] : 0.0f;
            if (more) load_mask(kb + NW);
        }
        if (MODE == MODE_FUSED) {
            constexpr int NF = 32 / BITS, E = 4 * NF;   // fields per output word, mask words per call (see attn_bf16_kernel)
            const uint32_t word = 4u * (uint32_t)(2 * (kb & 1) + (g >> 1));   // of register 0 in its 32 x 32 tile
            const uint64_t w0 = wtile + (uint64_t)(kb >> 1) * 16u;
            const uint64_t n = p.offset + 64u * (w0 / (uint32_t)E + word / (uint32_t)E) + bit;
            uint32_t x[4];
            if (p.rounds == 10) philox4x32<10>((uint32_t)n, (uint32_t)(n >> 32), 0u, 0u, p.k0, p.k1, x);
            else philox4x32_dyn(p.rounds, (uint32_t)n, (uint32_t)(n >> 32), 0u, 0u, p.k0, p.k1, x);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                bool keep;
                if (BITS == 32) keep = x[e] <= p.t_minus_1;
                else keep = ((x[e] >> ((uint32_t)BITS * ((word / 4u) % (uint32_t)NF))) & ((1u << (BITS & 31)) - 1u)) < p.tb;
                s[e] = keep ? s[e] : 0.0f;
            }
        }
        l_run = l_run * alpha + sum;
#pragma unroll
        for (int t = 0; t < KC; ++t) o[t] *= alpha;
        // (non-finite values under inadmissible keys: see attn_f32_kernel)
        bool finite = true;
        if (edge) {
#pragma unroll
            for (int t = 0; t < KC; ++t)
#pragma unroll
                for (int e = 0; e < 4; ++e) finite = finite && fabsf(vf[t][e]) < INFINITY;
            finite = __builtin_amdgcn_ballot_w64(!finite) == 0ull;
        }
        if (finite) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int t = 0; t < KC; ++t) o[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[t][e], s[e], o[t], 0, 0, 0);
        } else {
#pragma unroll 1
            for (int k = 0; k < 16; ++k) {
                const int key = kv0 + k;
                f32x4 one[KC];
#pragma unroll
                for (int t = 0; t < KC; ++t) one[t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const bool here = 4 * g + e == k;
                    const float pe = here ? s[e] : 0.0f;
#pragma unroll
                    for (int t = 0; t < KC; ++t) one[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(here ? vf[t][e] : 0.0f, pe, one[t], 0, 0, 0);
                }
                const bool adm = key < S && (!p.causal || key <= qrow);
#pragma unroll
                for (int t = 0; t < KC; ++t)
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[t][e] += adm ? one[t][e] : 0.0f;
            }
        }
        if (more) load_v(kv0 + 16 * NW);
    }

    // The waves' partial results meet in LDS, not used before: (maximum, sum) and output of each.  Feature block t is brought on
    // the common maximum and added up, waves in order, by wave t % NW.
    float2* ml = reinterpret_cast<float2*>(lds + KC * (NW - 1) * 1024);
    {
        const float l_all = quarter_wave_sum(l_run);
        if (g == 0) ml[wave * 16 + ql] = make_float2(m_run, l_all);
    }
#pragma unroll
    for (int t = 0; t < KC; ++t) {
        const int own = t % NW;
        if (wave != own)
            *reinterpret_cast<f32x4*>(lds + ((t * (NW - 1) + (wave < own ? wave : wave - 1)) * 64 + lane) * 16) = o[t];
    }
    __syncthreads();
    float m_all = -INFINITY, l = 0.0f, f[NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        f[w] = ml[w * 16 + ql].x;
        m_all = fmaxf(m_all, f[w]);
    }
    const float m_ref = m_all == -INFINITY ? 0.0f : m_all;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        f[w] = fast_exp2(f[w] - m_ref);
        l += ml[w * 16 + ql].y * f[w];
    }
    // (a row whose scores are all -infinity has no softmax: NaN)
    const float norm = m_all == -INFINITY ? __uint_as_float(0x7FC00000u) : l > 0.0f ? p.inv_keep / l : 0.0f;
    float* orow = (float*)p.O + b * p.so[0] + h * p.so[2] + (int64_t)qrow * p.so[1];
#pragma unroll
    for (int t = 0; t < KC; ++t) {
        const int own = t % NW, feat = 16 * t + 4 * g;
        if (wave == own) {
            f32x4 c = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                f32x4 v = o[t];
                if (w != own) v = *reinterpret_cast<const f32x4*>(lds + ((t * (NW - 1) + (w < own ? w : w - 1)) * 64 + lane) * 16);
                c += v * (norm * f[w]);
            }
            if (qrow < p.q_end && feat < d) *reinterpret_cast<f32x4*>(orow + feat) = c;
        }
    }
}

// ------------------------------------------------------------------ generic kernel
// One wave per query row, keys in chunks of 256 with an online softmax; any dtype / head
// dimension up to 256.  Correct for every shape; used for the head dimensions, strides and alignments that
// the two kernels above do not take, and for a few rows of fp32 (attn_f32_waves).
template <typename TT>
__device__ __forceinline__ float ld(const TT* p);
template <>
__device__ __forceinline__ float ld<float>(const float* p) { return *p; }
template <>
__device__ __forceinline__ float ld<uint16_t>(const uint16_t* p) { return __uint_as_float((uint32_t)*p << 16); }
template <typename TT>
__device__ __forceinline__ void st(TT* p, float v);
template <>
__device__ __forceinline__ void st<float>(float* p, float v) { *p = v; }
template <>
__device__ __forceinline__ void st<uint16_t>(uint16_t* p, float v) {
    *p = (uint16_t)(pack_bf16x2(v, 0.0f) & 0xFFFFu);
}

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
    for (int s = 32; s > 0; s >>= 1) v = fmaxf(v, __shfl_xor(v, s));
    return v;
}
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int s = 32; s > 0; s >>= 1) v += __shfl_xor(v, s);
    return v;
}

template <typename TT, int MODE>
__global__ __launch_bounds__(256) void attn_generic_kernel(const AttnParams p) {
    __shared__ float qs[4][256];
    __shared__ float ps[4][256];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int row = p.q_begin + blockIdx.x * 4 + wave;
    const int b = blockIdx.z, h = blockIdx.y;
    const int hk = h / (p.H / p.Hkv);
    const int S = p.S, d = p.d;
    if (row >= p.q_end) return;   // whole wave leaves; no block-wide barrier below
    const TT* Qp = (const TT*)p.Q + b * p.sq[0] + h * p.sq[2] + (int64_t)row * p.sq[1];
    const TT* Kp = (const TT*)p.K + b * p.sk[0] + hk * p.sk[2];
    const TT* Vp = (const TT*)p.V + b * p.sv[0] + hk * p.sv[2];
    TT* Op = (TT*)p.O + b * p.so[0] + h * p.so[2] + (int64_t)row * p.so[1];
    for (int t = lane; t < d; t += 64) qs[wave][t] = ld(Qp + t);
    __builtin_amdgcn_wave_barrier();
    float acc[4] = {0.f, 0.f, 0.f, 0.f};   // output features lane, lane+64, lane+128, lane+192
    float m_run = -INFINITY, l_run = 0.0f;
    const int kv_end = p.causal ? row + 1 : S;
    // tile row of this query row in the mask: words of tile (row/32, kt) start at wrow + 16*kt;
    // element (row, key) is bit 32*((key%32)/4 % 2) + row%32 of word 4*((key%32)/8) + key%4
    const uint64_t wrow = ((((uint64_t)b * p.H + h) * p.W + (uint64_t)(row >> 5)) * p.W) * 16u;
    // same tile row inside the mask buffer, which holds tile rows [mask_qt0, mask_qt0 + mask_nqt)
    const uint64_t mrow = ((((uint64_t)b * p.H + h) * p.mask_nqt + (uint64_t)((row >> 5) - p.mask_qt0)) * p.W) * 16u;
    for (int c0 = 0; c0 < kv_end; c0 += 256) {
        float sc[4];
        float mx = -INFINITY;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int key = c0 + lane + 64 * i;
            float v = -INFINITY;
            if (key < kv_end) {
                const TT* kr = Kp + (int64_t)key * p.sk[1];
                float dot = 0.0f;
                for (int t = 0; t < d; ++t) dot = __builtin_fmaf(qs[wave][t], ld(kr + t), dot);
                v = dot * p.scale_log2;
            }
            sc[i] = v;
            mx = fmaxf(mx, v);
        }
        mx = wave_max(mx);
        const float m_new = fmaxf(m_run, mx);
        const float alpha = fast_exp2(m_run - m_new);   // chunk 0 always has an admissible key
        m_run = m_new;
        float sum = 0.0f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int key = c0 + lane + 64 * i;
            float pe = 0.0f;
            if (key < kv_end) {
                pe = fast_exp2(sc[i] - m_new);
                sum += pe;
                bool keep = true;
                const int kl = key & 31;
                const uint64_t wo = (uint64_t)(key >> 5) * 16u + (uint64_t)(4 * (kl >> 3) + (kl & 3));
                const uint64_t w = wrow + wo;
                const uint32_t bit = 32u * ((uint32_t)(kl >> 2) & 1u) + ((uint32_t)row & 31u);
                if (MODE == MODE_MASK) {
                    keep = (p.mask[mrow + wo] >> bit) & 1ull;
                } else if (MODE == MODE_FUSED) {
                    const uint32_t E = 128u / (uint32_t)p.bits;            // mask words per group of calls
                    const uint64_t ncall = p.offset + 64u * (w / E) + (uint64_t)bit;
                    uint32_t x[4];
                    philox4x32_dyn(p.rounds, (uint32_t)ncall, (uint32_t)(ncall >> 32), 0u, 0u, p.k0, p.k1, x);
                    const uint32_t k = (uint32_t)(w % E), sel = k & 3u, f = k >> 2;
                    const uint32_t xv = sel == 0 ? x[0] : sel == 1 ? x[1] : sel == 2 ? x[2] : x[3];
                    if (p.bits == 32) keep = xv <= p.t_minus_1;
                    else keep = ((xv >> ((uint32_t)p.bits * f)) & ((1u << p.bits) - 1u)) < p.tb;
                }
                pe = keep ? pe : 0.0f;
            }
            ps[wave][lane + 64 * i] = pe;
        }
        l_run = l_run * alpha + wave_sum(sum);
        __builtin_amdgcn_wave_barrier();
        const int nkeys = min(256, kv_end - c0);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int t = lane + 64 * j;
            if (t < d) {
                float a = acc[j] * alpha;
                for (int kk = 0; kk < nkeys; ++kk)
                    a = __builtin_fmaf(ps[wave][kk], ld(Vp + (int64_t)(c0 + kk) * p.sv[1] + t), a);
                acc[j] = a;
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
    const float f = l_run > 0.0f ? p.inv_keep / l_run : 0.0f;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int t = lane + 64 * j;
        if (t < d) st(Op + t, acc[j] * f);
    }
}

// Workgroups of an XCD that come in reversed order (causal, d = 64; at d = 128 a compute unit holds one workgroup, and the next goes
// wherever one ends).  Heaviest first throughout, compute units got the heaviest of either round together: 24 units of work on some and
// 10 on others at 2 x 1000 tokens x 16 heads (bits drawn in the kernel 20.0 us, now 17.5), 17 on each now; 2 x 427 x 32 heads 13.6 -> 11.1, stored
// mask 9.8 -> 8.9.  Timed at 800 problems of 270 to 770 workgroups: up to two per compute unit, all resident at once, 1.0 to 1.2 times as fast.  Up to
// 2.6 the third ones go where a unit is done first: from 1000 tokens on (bits drawn in the kernel: 600) 1.03 (1.08) on average, 0.98 (0.97) at
// worst; with shorter sequences 0.92 to 1.06.  Above 2.6 1.02 (0.96 to 1.07), where it is not taken.
int attn_turn(long long nblocks, int S, int d, int ks, int mode) {
    const long long ncu = device_cu_count();
    const bool shared = d == 64 && (ks > 1 || mode != MODE_FUSED);   // (the unsplit fused form's registers fill a compute unit)
    return shared && ncu % 8 == 0 && 10 * nblocks > 11 * ncu && 10 * nblocks <= (S >= (mode == MODE_FUSED ? 600 : 1000) ? 26 : 20) * ncu ? (int)(ncu / 8) : 0;
}

template <int D, int NQ, int NW, int KS>
int launch_bf16(const AttnParams& prm, int mode, hipStream_t stream) {
    const int bq = NW / KS * 32 * NQ;
    AttnParams prm2 = prm;
    prm2.nq = (prm.q_end - prm.q_begin + bq - 1) / bq;
    const long long nblocks = (long long)prm2.nq * prm.H * prm.B;
    if (nblocks > 0x7FFFFFFFLL) return ROV_ERR_UNSUPPORTED;
    prm2.turn = prm.causal ? attn_turn(nblocks, prm.S, D, KS, mode) : 0;
    const dim3 grid((unsigned)nblocks), block(NW * 64);
    const int lds_bytes = 2 * Tile<D, KS == 1 ? 64 : 32 * KS>::kStage;   // two K/V stages
    void (*kern)(const AttnParams) = mode == MODE_NONE ? attn_bf16_kernel<D, NQ, NW, KS, MODE_NONE>
                                                       : attn_bf16_kernel<D, NQ, NW, KS, MODE_MASK>;
    if (mode == MODE_FUSED) {   // the round count is a compile-time constant of the fused kernel
        if (prm.bits == 16) { if (prm.rounds != 10) return ROV_ERR_UNSUPPORTED; kern = attn_bf16_kernel<D, NQ, NW, KS, MODE_FUSED, 10, 16>; }
        else if (prm.bits == 8) { if (prm.rounds != 10) return ROV_ERR_UNSUPPORTED; kern = attn_bf16_kernel<D, NQ, NW, KS, MODE_FUSED, 10, 8>; }
        else switch (prm.rounds) {
            case 10: kern = attn_bf16_kernel<D, NQ, NW, KS, MODE_FUSED, 10>; break;
            case 7: kern = attn_bf16_kernel<D, NQ, NW, KS, MODE_FUSED, 7>; break;
            case 5: kern = attn_bf16_kernel<D, NQ, NW, KS, MODE_FUSED, 5>; break;
            case 3: kern = attn_bf16_kernel<D, NQ, NW, KS, MODE_FUSED, 3>; break;
            default: return ROV_ERR_INVALID;
        }
    }
    {
        const int rc = set_max_dynamic_lds((const void*)kern, lds_bytes);
        if (rc != ROV_OK) return rc;
    }
    hipLaunchKernelGGL(kern, grid, block, lds_bytes, stream, prm2);
    ROV_LAUNCH_CHECK();
    return ROV_OK;
}

// Key parts of the matrix-core kernel (1, 2 or 4: workgroups of 256, 128 or 64 query rows).  A finer split
// fills the chip where query tiles are few and evens out causal workgroups; it re-reads K / V and merges partial results:
// with the chip full a workgroup of 128 (64) rows takes 0.556 (0.36) of the time of one of 256 rows at d = 128, 0.54 (0.295) at
// d = 64 (4096 and 8192 tokens, 32 heads).  Estimated time: rounds of one workgroup per compute unit and 1.3 us of start and
// merge each.  Causal: the longest workgroup, or the average load and `uneven` of a workgroup more, since the last ones do
// not end together (two share a compute unit at d = 64), if that is longer; these constants are fitted to all three forms
// at 4 to 128 heads of 128 to 8192 tokens, so that the choice is nowhere there more than 1 % slower than 256 rows, without dropout
// and with a stored mask (and mostly within 2 % of the best of the three).
// Measured with 256 / 128 / 64 rows, mask mode, us: d = 128, 512 tokens x 32 heads 20.5 / 14.7 / 11.4; 1500 x 32
// 46.8 / 57.0 / 57.5; causal 2048 x 16 55.6 / 36.5 / 31.4, 512 x 64 20.6 / 15.5 / 18.2, 6000 x 16 169 / 173 / 195; d = 64, causal
// 2048 x 32 43.5 / 31.5 / 31.1, 2048 x 64 56.4 / 49.7 / 58.6, 8192 x 64 636 / 681 / 774.  (Bits drawn in the kernel: the last one
// 1357 / 1168 / 1248: the unsplit form's 160 registers leave room for one workgroup per compute unit only.  It follows the
// others' choice.)
// Only what all launches over one problem share decides, so that row ranges and modes agree bit for bit.
int attn_key_parts(int B, int H, int S, int d, bool causal) {
    struct Cost { double walk_us, rel[3], uneven, round_us; };
    static const Cost full[2] = {{35.0, {1.0, 0.54, 0.295}, 0.0, 1.3}, {60.0, {1.0, 0.556, 0.36}, 0.0, 1.3}};
    static const Cost lower[2] = {{35.0, {1.0, 0.61, 0.36}, 0.6, 0.8}, {60.0, {1.0, 0.65, 0.40}, 0.3, 4.0}};
    const Cost& c = (causal ? lower : full)[d == 128];
    const double ncu = device_cu_count(), walk_us = (double)S / 2048.0 * c.walk_us;
    int best = 1;
    double best_us = 0.0;
    for (int i = 0; i < 3; ++i) {
        const int rows = 256 >> i, nq = (S + rows - 1) / rows;
        const double n = (double)nq * B * H, rounds = ceil(n / ncu);
        if (i > 0 && n > 0x7FFFFFFF) break;   // more workgroups than a grid holds (with 256 rows: refused)
        const double load = causal ? fmax(1.0, n / ncu * 0.5 * (1.0 + 1.0 / nq) + c.uneven) : rounds;
        const double us = walk_us * c.rel[i] * load + c.round_us * rounds;
        if (i == 0 || us < best_us) { best = 1 << i; best_us = us; }
    }
    return best;
}

// fp32: query tiles of 16 instead of 32 rows?  Timed at 1400 problems of 24 to 320 tiles of 32 rows (40 to 6000 tokens, 1 to 64 heads, 8 to 128
// features).  Every workgroup walks all keys, so without the causal mask what counts is whether the tiles of 16 are one round: 1.1 to 1.9
// times as fast up to one per compute unit; above, 0.64 to 1.1 (3 heads x 1616 tokens x 128 features 100 us against 69), but for the short walks
// of up to 200 tokens and 96 features, 1.06 on average (0.86 to 1.4).  Causal walks even out: 1.03 to 1.7 times as fast up to three quarters of a 32-query
// tile per compute unit, 0.9 to 1.6 above.  Only what all launches over one problem share decides, so that row ranges and modes agree.
bool attn_f32_q16(int B, int H, int S, int d, bool causal) {
    const double heads = (double)B * H, ncu = device_cu_count();
    return ceil(S / 32.0) * heads <= 0.75 * ncu && (causal || ceil(S / 16.0) * heads <= ncu || (S <= 200 && d <= 96));
}

// Waves of a workgroup of the fp32 kernels: eight at up to 64 features, four above (their registers); 0: the one-row-per-wave
// kernel runs, for a head dimension that these do not take, for more workgroups than a grid holds, or because it is done
// sooner: its waves have one key a lane, where a matrix kernel is one chain of load, products and merge whatever S is.  Against tiles
// of 32 rows both times are estimated, in us, fitted to 3360 problems of 1 to 96 tokens, 1 to 512 heads and 8 to 128
// features (one row a wave / matrix kernel, d = 128: 512 heads x 8 tokens 9.4 / 19.1, 256 x 8 8.4 / 12.2, 512 x 32 63 / 20; d = 64: 256 x 9
// 6.4 / 7.5, 512 x 9 9.3 / 12.6).  Tiles of 16 rows have a quarter of the chain: over 610 problems of up to 64 tokens they are even with the row
// kernel up to 4 tokens (0.94 to 1.2 times as fast) and 1.02 to 3.8 times as fast from 5 on (1 x 16 x 64 4.7 against 5.2, 1 x 37 x 128 6.2 against 8.7,
// 32 x 57 x 96 6.3 against 13.6).
// Only what all launches over one problem share decides, so that row ranges and modes agree.
int attn_f32_waves(int B, int H, int S, int d, bool causal) {
    const double heads = (double)B * H, tiles = ceil(S / 32.0) * heads;
    if (d % 8 != 0 || d > 128 || tiles > 0x7FFFFFFF) return 0;
    const double f = d <= 64 ? 1.0 : 2.0;
    const double row_us = 2.5 + 0.06 * f * S + 1e-3 * heads * S * f * (1.0 + 0.01 * S);
    const double mfma_us = (4.0 + 0.06 * ((d + 31) / 32 * 32)) * (0.2 + 0.8 * ceil(tiles / device_cu_count()));
    const int longest = attn_f32_q16(B, H, S, d, causal) ? 4 : 64;   // (beyond 64 tokens a lane has a second key)
    if (S <= longest && row_us < mfma_us) return 0;
    return d <= 64 ? 8 : 4;
}

template <int DP, int NW>
int launch_f32(const AttnParams& prm, int mode, hipStream_t stream) {
    AttnParams prm2 = prm;
    prm2.nq = (prm.q_end - prm.q_begin + 31) / 32;
    const long long nblocks = (long long)prm2.nq * prm.H * prm.B;
    if (nblocks > 0x7FFFFFFFLL) return ROV_ERR_UNSUPPORTED;
    void (*kern)(const AttnParams) = mode == MODE_NONE   ? attn_f32_kernel<DP, NW, MODE_NONE, 32>
                                     : mode == MODE_MASK ? attn_f32_kernel<DP, NW, MODE_MASK, 32>
                                     : prm.bits == 32    ? attn_f32_kernel<DP, NW, MODE_FUSED, 32>
                                     : prm.bits == 16    ? attn_f32_kernel<DP, NW, MODE_FUSED, 16>
                                                         : attn_f32_kernel<DP, NW, MODE_FUSED, 8>;
    const int lds_bytes = DP / 8 * (NW - 1) * 1024 + NW * 256;
    {
        const int rc = set_max_dynamic_lds((const void*)kern, lds_bytes);
        if (rc != ROV_OK) return rc;
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)nblocks), dim3(NW * 64), lds_bytes, stream, prm2);
    ROV_LAUNCH_CHECK();
    return ROV_OK;
}

template <int DP, int NW>
int launch_f32_q16(const AttnParams& prm, int mode, hipStream_t stream) {
    AttnParams prm2 = prm;
    prm2.nq = (prm.q_end - prm.q_begin + 15) / 16;
    const long long nblocks = (long long)prm2.nq * prm.H * prm.B;
    if (nblocks > 0x7FFFFFFFLL) return ROV_ERR_UNSUPPORTED;
    void (*kern)(const AttnParams) = mode == MODE_NONE   ? attn_f32_q16_kernel<DP, NW, MODE_NONE, 32>
                                     : mode == MODE_MASK ? attn_f32_q16_kernel<DP, NW, MODE_MASK, 32>
                                     : prm.bits == 32    ? attn_f32_q16_kernel<DP, NW, MODE_FUSED, 32>
                                     : prm.bits == 16    ? attn_f32_q16_kernel<DP, NW, MODE_FUSED, 16>
                                                         : attn_f32_q16_kernel<DP, NW, MODE_FUSED, 8>;
    constexpr int kLds = DP / 16 * (NW - 1) * 1024 + NW * 128;
    static_assert(kLds <= 64 * 1024, "no attribute is needed");
    hipLaunchKernelGGL(kern, dim3((unsigned)nblocks), dim3(NW * 64), kLds, stream, prm2);
    ROV_LAUNCH_CHECK();
    return ROV_OK;
}

template <typename TT>
int launch_generic(const AttnParams& prm, int mode, hipStream_t stream) {
    const dim3 grid((unsigned)((prm.q_end - prm.q_begin + 3) / 4), (unsigned)prm.H, (unsigned)prm.B), block(256);
    if (mode == MODE_NONE)
        hipLaunchKernelGGL((attn_generic_kernel<TT, MODE_NONE>), grid, block, 0, stream, prm);
    else if (mode == MODE_MASK)
        hipLaunchKernelGGL((attn_generic_kernel<TT, MODE_MASK>), grid, block, 0, stream, prm);
    else
        hipLaunchKernelGGL((attn_generic_kernel<TT, MODE_FUSED>), grid, block, 0, stream, prm);
    ROV_LAUNCH_CHECK();
    return ROV_OK;
}

}  // namespace

int launch_attention(const void* Q, const void* K, const void* V, void* O, int B, int H, int Hkv,
                     int S, int d, const int64_t strides[12], int dtype, int causal, float p,
                     const uint64_t* mask, uint64_t seed, uint64_t offset, hipStream_t stream, int rounds,
                     int bits) {
    return launch_attention_rows(Q, K, V, O, B, H, Hkv, S, d, strides, dtype, causal, p, mask, false, seed,
                                 offset, 0, S, stream, rounds, bits);
}

// Everything launch_attention_rows refuses, without launching: the schedules call this before
// they enqueue the first kernel of a sequence.
int check_attention_rows(const void* Q, const void* K, const void* V, const void* O, int B, int H, int Hkv,
                         int S, int d, const int64_t strides[12], int dtype, float p, const uint64_t* mask,
                         int q_begin, int q_rows, int rounds, int bits) {
    if (rounds != 10 && rounds != 7 && rounds != 5 && rounds != 3) return ROV_ERR_INVALID;
    if (bits != 32 && bits != 16 && bits != 8) return ROV_ERR_INVALID;
    if (bits != 32 && rounds != 10) return ROV_ERR_UNSUPPORTED;
    if (S <= 0 || q_begin < 0 || q_rows <= 0 || q_begin >= S || (q_begin & 31) != 0) return ROV_ERR_INVALID;
    if (Q == nullptr || K == nullptr || V == nullptr || O == nullptr || strides == nullptr)
        return ROV_ERR_INVALID;
    if (B <= 0 || H <= 0 || Hkv <= 0 || S <= 0 || d <= 0 || (H % Hkv) != 0) return ROV_ERR_INVALID;
    if (dtype != ROV_F32 && dtype != ROV_BF16) return dtype == ROV_FP8_E4M3 ? ROV_ERR_UNSUPPORTED : ROV_ERR_INVALID;
    uint32_t tm1 = 0xFFFFFFFFu;
    if (!keep_threshold_minus_1(p, &tm1)) return ROV_ERR_INVALID;
    if (B > 65535 || H > 65535) return ROV_ERR_UNSUPPORTED;
    if (d > 256) return ROV_ERR_UNSUPPORTED;
    if (mask != nullptr && !aligned(mask, 8)) return ROV_ERR_INVALID;
    // workgroups of the matrix-core kernel (256 query rows each) fit the grid's 31 bits
    const long long q_end = (long long)q_begin + q_rows < S ? (long long)q_begin + q_rows : S;
    if (((q_end - q_begin + 255) / 256) * (long long)H * B > 0x7FFFFFFFLL) return ROV_ERR_UNSUPPORTED;
    return ROV_OK;
}

int launch_attention_rows(const void* Q, const void* K, const void* V, void* O, int B, int H, int Hkv,
                          int S, int d, const int64_t strides[12], int dtype, int causal, float p,
                          const uint64_t* mask, bool mask_is_rows, uint64_t seed, uint64_t offset,
                          int q_begin, int q_rows, hipStream_t stream, int rounds, int bits, float o_fp8_scale) {
    {
        const int rc = check_attention_rows(Q, K, V, O, B, H, Hkv, S, d, strides, dtype, p, mask, q_begin, q_rows,
                                            rounds, bits);
        if (rc != ROV_OK) return rc;
    }
    uint32_t tm1 = 0xFFFFFFFFu;
    (void)keep_threshold_minus_1(p, &tm1);

    AttnParams prm;
    prm.Q = Q; prm.K = K; prm.V = V; prm.O = O; prm.mask = mask;
    for (int i = 0; i < 3; ++i) {
        prm.sq[i] = strides[i]; prm.sk[i] = strides[3 + i];
        prm.sv[i] = strides[6 + i]; prm.so[i] = strides[9 + i];
    }
    prm.B = B; prm.H = H; prm.Hkv = Hkv; prm.S = S; prm.d = d;
    prm.W = (S + 31) / 32;
    prm.q_begin = q_begin;
    prm.q_end = (int64_t)q_begin + q_rows < S ? q_begin + q_rows : S;
    // a mask of rows holds exactly the tile rows of [q_begin, q_end); a full mask holds all of them
    prm.mask_qt0 = mask_is_rows ? q_begin / 32 : 0;
    prm.mask_nqt = mask_is_rows ? (prm.q_end - q_begin + 31) / 32 : prm.W;
    prm.causal = causal != 0;
    prm.scale_log2 = 1.4426950408889634f / sqrtf((float)d);
    prm.inv_keep = p > 0.0f ? 1.0f / (1.0f - p) : 1.0f;
    prm.offset = offset;
    prm.k0 = (uint32_t)seed; prm.k1 = (uint32_t)(seed >> 32);
    prm.t_minus_1 = tm1;
    prm.rounds = rounds;
    prm.bits = bits;
    // keep iff field < tb, tb = floor((1 - p) * 2^bits) in double from the float p
    prm.tb = bits < 32 ? (uint32_t)(uint64_t)((1.0 - (double)p) * (double)(1u << bits)) : 0u;
    prm.o_fp8 = o_fp8_scale > 0.0f;
    prm.o_inv_scale = prm.o_fp8 ? 1.0f / o_fp8_scale : 1.0f;
    const int mode = p == 0.0f ? MODE_NONE : (mask != nullptr ? MODE_MASK : MODE_FUSED);

    if (dtype == ROV_BF16 && (d == 64 || d == 128)) {
        // 16-byte vector access needs 8-element alignment of every row start
        bool ok = aligned(Q, 16) && aligned(K, 16) && aligned(V, 16) && aligned(O, 8);
        for (int i = 0; i < 12; ++i) ok = ok && (strides[i] % 8) == 0;
        // K / V of one (batch, kv head) are addressed through a buffer resource: 32-bit byte offsets
        for (int t = 4; t <= 7; t += 3)
            ok = ok && strides[t] >= 0 && (uint64_t)(S - 1) * (uint64_t)strides[t] * 2u + 2u * (uint64_t)d < (1ull << 32);
        if (prm.o_fp8) {   // four bytes per store: O and its strides (in bytes) are multiples of 4
            ok = ok && aligned(O, 4);
            for (int i = 9; i < 12; ++i) ok = ok && (strides[i] % 4) == 0;
            if (!ok) return ROV_ERR_UNSUPPORTED;
        }
        if (ok) {
            // 8 waves of 32 query rows: two waves per SIMD (measured 1.5x faster than 4 waves x 64
            // rows at S = 16384: 905 vs 602 TFLOP/s without dropout)
            const int ks = attn_key_parts(B, H, S, d, causal != 0);
            if (d == 128) {
                if (ks == 4) return launch_bf16<128, 1, 8, 4>(prm, mode, stream);
                if (ks == 2) return launch_bf16<128, 1, 8, 2>(prm, mode, stream);
                return launch_bf16<128, 1, 8, 1>(prm, mode, stream);
            }
            if (ks == 4) return launch_bf16<64, 1, 8, 4>(prm, mode, stream);
            if (ks == 2) return launch_bf16<64, 1, 8, 2>(prm, mode, stream);
            return launch_bf16<64, 1, 8, 1>(prm, mode, stream);
        }
    }
    if (dtype == ROV_F32 && attn_f32_waves(B, H, S, d, causal != 0) != 0) {
        // 16-byte accesses to rows of Q, K and O
        bool ok = aligned(Q, 16) && aligned(K, 16) && aligned(O, 16);
        for (int i = 0; i < 12; ++i) ok = ok && (i / 3 == 2 || strides[i] % 4 == 0);
        // K / V of one (batch, kv head) are addressed through a buffer resource: byte offsets below 2^31
        for (int t = 4; t <= 7; t += 3)
            ok = ok && strides[t] >= 0 && (uint64_t)(S + 31) * (uint64_t)strides[t] * 4u + 4u * (uint64_t)d < (1ull << 31);
        if (ok && attn_f32_q16(B, H, S, d, causal != 0)) {
            if (d <= 32) return launch_f32_q16<32, 8>(prm, mode, stream);
            if (d <= 64) return launch_f32_q16<64, 8>(prm, mode, stream);
            if (d <= 96) return launch_f32_q16<96, 4>(prm, mode, stream);
            return launch_f32_q16<128, 4>(prm, mode, stream);
        }
        if (ok && d <= 32) return launch_f32<32, 8>(prm, mode, stream);
        if (ok && d <= 64) return launch_f32<64, 8>(prm, mode, stream);
        if (ok && d <= 96) return launch_f32<96, 4>(prm, mode, stream);
        if (ok) return launch_f32<128, 4>(prm, mode, stream);
    }
    if (prm.o_fp8) return ROV_ERR_UNSUPPORTED;   // the e4m3 output exists in the matrix-core kernel only
    if (dtype == ROV_BF16) return launch_generic<uint16_t>(prm, mode, stream);
    return launch_generic<float>(prm, mode, stream);
}

}  // namespace rov

extern "C" int rov_attention_key_parts(int B, int H, int S, int d, int dtype, int causal) {
    if (B <= 0 || H <= 0 || S <= 0 || d <= 0 || d > 256) return ROV_ERR_INVALID;
    if (dtype != ROV_F32 && dtype != ROV_BF16) return ROV_ERR_INVALID;
    if (dtype == ROV_F32) return rov::attn_f32_waves(B, H, S, d, causal != 0);
    return d == 64 || d == 128 ? rov::attn_key_parts(B, H, S, d, causal != 0) : 0;
}

extern "C" int rov_attention_tile_rows(int B, int H, int S, int d, int dtype, int causal) {
    const int parts = rov_attention_key_parts(B, H, S, d, dtype, causal);
    if (parts <= 0) return parts < 0 ? parts : 1;
    if (dtype == ROV_F32) return rov::attn_f32_q16(B, H, S, d, causal != 0) ? 16 : 32;
    return 256 / parts;
}

extern "C" int rov_attention_fwd_dropout_rows(const void* Q, const void* K, const void* V, void* O, int B,
                                              int H, int Hkv, int S, int d, const int64_t strides[12],
                                              int dtype, int causal, float p, const uint64_t* mask_rows,
                                              uint64_t seed, uint64_t offset, int q_begin, int q_rows,
                                              void* stream) {
    return rov::launch_attention_rows(Q, K, V, O, B, H, Hkv, S, d, strides, dtype, causal, p, mask_rows, true,
                                      seed, offset, q_begin, q_rows, (hipStream_t)stream);
}

extern "C" int rov_attention_fwd_dropout(const void* Q, const void* K, const void* V, void* O, int B,
                                         int H, int Hkv, int S, int d, const int64_t strides[12],
                                         int dtype, int causal, float p, const uint64_t* mask,
                                         uint64_t seed, uint64_t offset, void* stream) {
    return rov::launch_attention(Q, K, V, O, B, H, Hkv, S, d, strides, dtype, causal, p, mask, seed,
                                 offset, (hipStream_t)stream);
}

extern "C" int rov_attention_fwd_dropout_rounds(const void* Q, const void* K, const void* V, void* O, int B,
                                                int H, int Hkv, int S, int d, const int64_t strides[12],
                                                int dtype, int causal, float p, const uint64_t* mask,
                                                uint64_t seed, uint64_t offset, int rounds, void* stream) {
    return rov::launch_attention(Q, K, V, O, B, H, Hkv, S, d, strides, dtype, causal, p, mask, seed,
                                 offset, (hipStream_t)stream, rounds);
}

extern "C" int rov_attention_fwd_dropout_bits(const void* Q, const void* K, const void* V, void* O, int B,
                                              int H, int Hkv, int S, int d, const int64_t strides[12],
                                              int dtype, int causal, float p, const uint64_t* mask,
                                              uint64_t seed, uint64_t offset, int bits, void* stream) {
    return rov::launch_attention(Q, K, V, O, B, H, Hkv, S, d, strides, dtype, causal, p, mask, seed,
                                 offset, (hipStream_t)stream, 10, bits);
}
