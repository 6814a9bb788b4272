// The direct-B GEMM kernel for gfx950 (MI355X): products whose output gives a
// chip of 256 CUs too few large tiles, i.e. most products of more than 64 rows
// and less than about 2048 x 4096 elements, those of 17 to 64 rows where the
// skinny kernels are bound by converting A, and those of few rows whose
// alignment the 16-byte paths of the other kernels do not take.
//
// All products of an FP32 A (HEAL Section 4, GEMM paragraph) run on it:
// HEAL-Base, HEAL-Full and the pre-split bf16x3 product with their packed B,
// and the bf16x3 product with B stored N x K or K x N.
//
// What bounds such a product is not the matrix cores but the time of one
// stage on one CU: with 128 x 128 tiles a 256 x 4096 output occupies 64 of 256
// CUs.  K cannot be split (each element's sum keeps one order), so the tiles
// have to be small, and what a tile stages per 32 of K is then large against
// its MFMAs: the CU's load path (64 bytes per clock), the LDS store path and
// the conversions of A.  Hence:
//   * each wave owns its columns: B goes from memory to its registers, in
//     fragment order, with no LDS round trip and no sharing; B stored K x N is
//     read as one to four adjacent columns per lane (block j of a wave takes
//     every NB-th column from the j-th), so the 4 x 4 transposes of the staged
//     kernels are not needed;
//   * LW more waves do nothing but stage A: they load, convert and store it to
//     a ring of three LDS stages, one stage ahead of the fragment reads;
//   * the computing waves read the next chunk's fragments of A and split its B
//     while the current chunk is multiplied (PIPE), and their B is in flight
//     RC chunks ahead.
// Measured (4096 x 4096 weight, us, tiled kernels -> this one): 256 rows
// HEAL-Full 72.8 -> 25.5, HEAL-Base 43.4 -> 19.4, pre-split 92.1 -> 31.8, bf16x3
// 84.2 -> 42.5 (K x N) and 87.6 -> 45.8 (N x K); 1024 rows 85.6 -> 63.0, 53.7 ->
// 43.4, 104.4 -> 92.7, 102.1 -> 97.3, 106.2 -> 98.2.  What is left, at 256 rows
// HEAL-Full (28.7 us with four loading waves on 128-deep stages): 23.1 without
// A's staging, 22.4 without loads of B, 23.0 with a quarter of the MFMAs, 15.7
// with neither A nor B loaded: one computing wave per SIMD issues MFMAs at 0.6 of
// their rate, and the loads, the conversion and the LDS traffic overlap it in
// part.
//
// Alignment: the hardware's 16-byte buffer accesses need dword alignment only,
// so every 4-byte aligned row takes this path.  A quad across the end of a
// row of K (or the lane's columns across the end of a row of B stored K x N)
// is read up to three elements early, inside its row, and shifted.
//
// Reduction order: identical to every other instance (K in 32-deep chunks
// ascending; per chunk the products in their fixed order into one FP32
// accumulator; the B fragment as the MFMA's first source; the K tail
// zero-filled), so results are bitwise equal to theirs.
#include "heal.h"
#include "heal_device.h"
#include "heal_internal.h"

namespace heal {

namespace {

constexpr uint32_t kOOB = 0x80000000u;  // buffer offset beyond every range: reads 0
constexpr int kRsrcFlags = 0x00020000;  // raw buffer, 32-bit data format

// Vector of four floats with the alignment of one: C rows need not be 16-byte
// aligned (the hardware's 16-byte accesses need dword alignment only).
typedef float f32x4_u __attribute__((ext_vector_type(4), aligned(4)));

enum BSource : int {
    B_PACKED = 0,  // fragment order: one 1 KiB block per 16 columns, 32-deep chunk and plane
    B_ROWS = 1,    // FP32, stored N x K
    B_COLS = 2,    // FP32, stored K x N
};


template <int OP>
struct DirectOp {
    static constexpr int AP = OP == OP_BASE ? 1 : 2;       // LDS planes of A
    static constexpr int BP = OP == OP_PRESPLIT ? 2 : 1;   // packed planes of B
    static constexpr bool BF16 = OP == OP_PRESPLIT || OP == OP_BF16X3;
};

template <bool BF16>
__device__ __forceinline__ f32x4 mma(u32x4 b, u32x4 a, f32x4 c)
{
    if constexpr (BF16)
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, b),
                                                       __builtin_bit_cast(bf16x8, a), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, b),
                                                      __builtin_bit_cast(f16x8, a), c, 0, 0, 0);
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void *base, int bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), (short)0, bytes, kRsrcFlags);
}

__device__ __forceinline__ u32x4 bload4(__amdgpu_buffer_rsrc_t r, uint32_t voff, int soff)
{
    return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)voff, soff, 0));
}

// V consecutive floats, V = 1, 2 or 4.
template <int V>
__device__ __forceinline__ void bload_v(__amdgpu_buffer_rsrc_t r, uint32_t voff, int soff, float *v)
{
    if constexpr (V == 4) {
        const f32x4 x = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)voff, soff, 0));
        v[0] = x.x;
        v[1] = x.y;
        v[2] = x.z;
        v[3] = x.w;
    } else if constexpr (V == 2) {
        const f32x2 x = __builtin_bit_cast(f32x2, __builtin_amdgcn_raw_buffer_load_b64(r, (int)voff, soff, 0));
        v[0] = x.x;
        v[1] = x.y;
    } else {
        v[0] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, (int)voff, soff, 0));
    }
}

// kOOB for an index past the end, else 0: a lane's offset with it set lies
// beyond the buffer.  Arithmetic, not a select, which becomes a branch around
// the loads, after which every wait is for all of them.
__device__ __forceinline__ uint32_t past_end(int i, int n)
{
    return (uint32_t)((n - 1 - i) >> 31) & kOOB;
}

// A quad read `back` elements early (0 to 3, so that it ends at the end of its
// row): the elements that belong to it move to the front, zeros follow.
__device__ __forceinline__ u32x4 shift_quad(u32x4 q, int back)
{
    u32x4 v = q;
    if (back == 1) v = u32x4{q.y, q.z, q.w, 0u};
    if (back == 2) v = u32x4{q.z, q.w, 0u, 0u};
    if (back == 3) v = u32x4{q.w, 0u, 0u, 0u};
    return v;
}

// LDS geometry of one plane of A: rows of BK 16-bit values, the 16-byte chunk
// c of row r at c ^ swz(r), so that the 16 rows of a fragment read fall in
// different bank groups.
template <int BK>
struct LdsA {
    static constexpr int RP = 2 * BK;
    static __device__ __forceinline__ int swz(int row)
    {
        return RP >= 256 ? row & 15 : RP == 128 ? (row >> 1) & 7 : (row >> 1) & 3;
    }
    static __device__ __forceinline__ int chunk_off(int row, int c)
    {
        return row * RP + ((c ^ swz(row)) << 4);
    }
    static __device__ __forceinline__ int quad_off(int row, int kq)
    {
        return row * RP + (((kq >> 1) ^ swz(row)) << 4) + ((kq & 1) << 3);
    }
};

// MB, NB: 16-row and 16-column blocks per wave; WVM, WVN: waves along M and N;
// KS: 32-deep chunks per stage; RC: chunks of B in flight per wave; LW: waves
// that stage A; RA: their register sets; PIPE: fragments of A read a chunk
// ahead (twice the registers); TURN: B turned through LDS; TAIL: K is not a
// multiple of the stage depth.
template <int OP, int BS, int MB, int WVM, int NB, int WVN, int KS, int RC, int LW, int RA, bool PIPE, bool TURN, bool TAIL>
__global__ void __launch_bounds__(64 * (WVM * WVN + LW), (WVM * WVN + LW) / 4)
gemm_direct_kernel(DirectArgs p)
{
    using O = DirectOp<OP>;
    constexpr int CW = WVM * WVN;                // waves that multiply
    constexpr int NT = 64 * LW;                  // threads that stage A
    constexpr int D = 3;                         // LDS stages
    constexpr int T = RC > KS ? RC / KS : 1;     // stages per trip of the compute loop
    static_assert(RC % KS == 0 || KS % RC == 0, "whole turns of the B ring per trip");
    constexpr int BM = 16 * MB * WVM, BN = 16 * NB * WVN, BK = 32 * KS, KQ = BK / 4;
    using L = LdsA<BK>;
    constexpr int A_PLANE = BM * L::RP;
    constexpr int STAGE = O::AP * A_PLANE;
    constexpr int NA = BM * KQ / NT;             // A quads per thread and stage
    static_assert(NA >= 1 && NA * NT == BM * KQ, "whole A quads per thread");
    static_assert(BS != B_COLS || NB == 1 || NB == 2 || NB == 4, "columns per lane");
    constexpr int RB = BS == B_PACKED ? O::BP : 2;  // 16-byte registers per block and chunk
    // TURN (B stored N x K): each wave reads whole 128-byte lines of its rows (a
    // fragment's own order touches 16 rows, so 16 lines, with every 16 lanes) and
    // turns them into fragments through an LDS area of its own (200 x 6144 x 4096
    // on 64 x 128 tiles 71 -> 62 us, with eight computing waves instead of four 59;
    // 32 x 32 tiles, which turn little at a time, are slower with it: 64 x 4096 x
    // 4096 24.4 -> 28.1).
    static_assert(!TURN || BS == B_ROWS, "rows of B");
    constexpr int TURN_BYTES = TURN ? NB * 2048 : 0;
    __shared__ __attribute__((aligned(16))) char smem[D * STAGE + CW * TURN_BYTES];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WVN, wn = wave % WVN;
    const int fr = lane & 15, fg = lane >> 4;

    // tile coordinates: each XCD owns a contiguous run of tiles, walked along M
    // first, so that the row tiles of one column strip share its B in that L2
    const int64_t tiles_m = (p.M + BM - 1) / BM;
    const int64_t tiles_n = (p.N + BN - 1) / BN;
    int64_t bid = blockIdx.x;
    {
        const int64_t nb = gridDim.x, x = bid & 7, i = bid >> 3, q = nb >> 3, r = nb & 7;
        bid = x * q + (x < r ? x : r) + i;
    }
    constexpr int GM = HEAL_GROUP_M;
    const int64_t group = bid / (GM * tiles_n);
    const int64_t first_m = group * GM;
    const int64_t gm = (tiles_m - first_m) < GM ? (tiles_m - first_m) : GM;
    const int64_t in_group = bid - group * GM * tiles_n;
    const int64_t m0 = (first_m + in_group % gm) * BM;
    const int64_t n0 = (in_group / gm) * BN;

    const int64_t M = p.M, N = p.N;
    const int K = (int)p.K;
    const int ns = (K + BK - 1) / BK;
    const int KC = (K + 31) / 32;
    const int rows = (int)((M - m0) < BM ? (M - m0) : BM);
    const int cols = (int)((N - n0) < BN ? (N - n0) : BN);
    const int back_k = K < 4 ? 0 : (4 - (K & 3)) & 3;   // a quad across the end of K starts this much early

    int a_kq[NA], a_row[NA], st_a[NA];
#pragma unroll
    for (int u = 0; u < NA; ++u) {
        const int q = tid - 64 * CW + NT * u;
        a_row[u] = q / KQ;
        a_kq[u] = q % KQ;
        st_a[u] = L::quad_off(a_row[u], a_kq[u]);
    }

    for (int64_t b = blockIdx.y; b < p.batch; b += gridDim.y) {
        const float *A = p.A + b * p.strideA + m0 * p.lda;
        const int a_bytes = (int)(((int64_t)(rows - 1) * p.lda + K) * 4);
        const char *B = reinterpret_cast<const char *>(p.B);
        int b_bytes;
        if constexpr (BS == B_PACKED) {
            B += (n0 / 16) * KC * O::BP * 1024;
            b_bytes = (cols + 15) / 16 * KC * O::BP * 1024;
        } else if constexpr (BS == B_ROWS) {
            B += (b * p.strideB + n0 * p.ldb) * 4;
            b_bytes = (int)(((int64_t)(cols - 1) * p.ldb + K) * 4);
        } else {
            B += b * p.strideB * 4;              // from column 0: a lane may read back across n0
            b_bytes = (int)(((int64_t)(K - 1) * p.ldb + N) * 4);
        }

        uint32_t va[NA];
#pragma unroll
        for (int u = 0; u < NA; ++u)
            va[u] = a_row[u] < rows ? (uint32_t)((a_row[u] * p.lda + 4 * a_kq[u]) * 4) : kOOB;
        // with a K tail: the last stage's offsets, past the end of K beyond the
        // buffer and a quad across it back_k elements early
        uint32_t vat[TAIL ? NA : 1];
        if constexpr (TAIL) {
#pragma unroll
            for (int u = 0; u < NA; ++u) {
                const int k = (ns - 1) * BK + 4 * a_kq[u];
                vat[u] = k >= K || a_row[u] >= rows
                             ? kOOB : va[u] + (ns - 1) * BK * 4 - (k + 4 > K ? 4u * back_k : 0u);
            }
        }
        constexpr int NVB = TURN ? 2 * NB : NB;
        uint32_t vb[NVB];
        // TURN: 16-byte unit lane % 8 of row lane / 8 of every 8 rows.
        // B_COLS: a lane's NB columns are NB*fr .. +NB-1 of the wave's; the lane
        // whose columns cross the edge of B reads them back_n early
        int back_n = 0;
        const bool edge_n = BS == B_COLS && (wn + 1) * 16 * NB > cols;
        if constexpr (BS == B_COLS) {
            const int c = (wn * 16 + fr) * NB;
            back_n = c < cols && c + NB > cols ? c + NB - cols : 0;
            vb[0] = c < cols ? (uint32_t)((8 * fg * p.ldb + n0 + c - back_n) * 4) : kOOB;
        } else if constexpr (TURN) {
#pragma unroll
            for (int u = 0; u < NVB; ++u) {
                const int r = wn * 16 * NB + 8 * u + (lane >> 3);
                vb[u] = r < cols ? (uint32_t)((r * p.ldb + 4 * (lane & 7)) * 4) : kOOB;
            }
        } else {
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                const int jb = wn * NB + j;
                if constexpr (BS == B_PACKED)
                    vb[j] = 16 * jb < cols ? (uint32_t)(jb * KC * O::BP * 1024 + lane * 16) : kOOB;
                else
                    vb[j] = 16 * jb + fr < cols
                                ? (uint32_t)(((16 * jb + fr) * p.ldb + 8 * fg) * 4) : kOOB;
            }
        }
        // Stage s of A, or chunk kc of B, into a register set.  Those
        // past the last read nothing: every lane's offset lies beyond the buffer.
        // The scalar offset stays inside the buffer (the last stage stands in
        // for one past it); with a K tail the whole offset is the lane's own.
        auto load_a = [&](u32x4 *ra, int s) {
            const __amdgpu_buffer_rsrc_t r = make_rsrc(A, a_bytes);
            const uint32_t past = past_end(s, ns);
            const int so = (s < ns ? s : ns - 1) * BK * 4;
#pragma unroll
            for (int u = 0; u < NA; ++u) {
                uint32_t v = va[u];
                if (TAIL) v = s >= ns - 1 ? vat[u] : v + so;
                ra[u] = bload4(r, v | past, TAIL ? 0 : so);
            }
        };
        auto load_b = [&](u32x4 (*rb)[RB], int c) {
            const __amdgpu_buffer_rsrc_t r = make_rsrc(B, b_bytes);
            const uint32_t past = past_end(c, ns * KS);
            const int kc = c < ns * KS ? c : ns * KS - 1;
            if constexpr (BS == B_COLS) {
                float *v = reinterpret_cast<float *>(rb);
                const uint32_t o = vb[0] | past;
#pragma unroll
                for (int t = 0; t < 8; ++t) {
                    const int so = (kc * 32 + t) * (int)p.ldb * 4;
                    // rows past K start past the end of the buffer
                    const uint32_t w = TAIL ? o + so : o;
                    bload_v<NB>(r, w, TAIL ? 0 : so, v + t * NB);
                }
            } else if constexpr (TURN) {
#pragma unroll
                for (int u = 0; u < NVB; ++u) {
                    const int so = kc * 128;
                    const uint32_t o = vb[u] | past;
                    uint32_t w = o;
                    if (TAIL) {
                        const int k = kc * 32 + 4 * (lane & 7);
                        w = k >= K ? kOOB : o + so - (k + 4 > K ? 4u * back_k : 0u);
                        w = (o & kOOB) ? kOOB : w;
                    }
                    rb[u / 2][u % 2] = bload4(r, w, TAIL ? 0 : so);
                }
            } else {
#pragma unroll
                for (int j = 0; j < NB; ++j) {
                    const uint32_t o = vb[j] | past;
#pragma unroll
                    for (int q = 0; q < RB; ++q) {
                        const int so = kc * (BS == B_PACKED ? O::BP * 1024 : 128);
                        uint32_t w = o + (BS == B_PACKED ? 1024u : 16u) * q;
                        if (TAIL) {
                            const int k = kc * 32 + (BS == B_PACKED ? 0 : 8 * fg + 4 * q);
                            w = k >= K || (o & kOOB) ? kOOB : w + so;
                            if (BS == B_ROWS && k < K && k + 4 > K && !(o & kOOB)) w -= 4u * back_k;
                        }
                        rb[j][q] = bload4(r, w, TAIL ? 0 : so);
                    }
                }
            }
        };
        // TURN: the lines of chunk kc through this wave's LDS area into
        // fragment order (one wave's own area: no barrier, only their order)
        char *const area = smem + D * STAGE + wave * TURN_BYTES;
        auto turn_b = [&](const u32x4 (*line)[RB], int kc, u32x4 (*raw)[2]) {
            auto off = [](int row, int c) { return row * 128 + ((c ^ ((row >> 1) & 7)) << 4); };
            wave_lds_order();
#pragma unroll
            for (int u = 0; u < NVB; ++u) {
                u32x4 q = line[u / 2][u % 2];
                if (TAIL && kc == KC - 1 && kc * 32 + 4 * (lane & 7) + 4 > K) q = shift_quad(q, back_k);
                *reinterpret_cast<u32x4 *>(area + off(8 * u + (lane >> 3), lane & 7)) = q;
            }
            wave_lds_order();
#pragma unroll
            for (int j = 0; j < NB; ++j)
#pragma unroll
                for (int q = 0; q < 2; ++q)
                    raw[j][q] = *reinterpret_cast<const u32x4 *>(area + off(16 * j + fr, 2 * fg + q));
        };
        auto store_a = [&](char *st, const u32x4 *ra, int s) {
#pragma unroll
            for (int u = 0; u < NA; ++u) {
                u32x4 q = ra[u];
                if (TAIL && s == ns - 1 && s * BK + 4 * a_kq[u] + 4 > K) q = shift_quad(q, back_k);
                const f32x4 x = __builtin_bit_cast(f32x4, q);
                const float x0 = x.x, x1 = x.y, x2 = x.z, x3 = x.w;
                const int off = st_a[u];
                if constexpr (OP == OP_BASE) {
                    *reinterpret_cast<u32x2 *>(st + off) = u32x2{cvt2_f16(x0, x1), cvt2_f16(x2, x3)};
                } else {
                    uint32_t h0, l0, h1, l1;
                    if constexpr (OP == OP_FULL) {
                        split2_f16(x0, x1, h0, l0);
                        split2_f16(x2, x3, h1, l1);
                    } else {
                        split2(x0, x1, h0, l0);
                        split2(x2, x3, h1, l1);
                    }
                    *reinterpret_cast<u32x2 *>(st + off) = u32x2{h0, h1};
                    *reinterpret_cast<u32x2 *>(st + A_PLANE + off) = u32x2{l0, l1};
                }
            }
        };

        f32x4 acc[NB][MB];
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int i = 0; i < MB; ++i) acc[j][i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

        // the two parts of B of chunk kc
        // (TURN: rb already in fragment order, its K tail shifted)
        auto frag_b = [&](const u32x4 (*rb)[RB], int kc, u32x4 *bh, u32x4 *bl) {
            if constexpr (BS == B_PACKED) {
#pragma unroll
                for (int j = 0; j < NB; ++j) {
                    bh[j] = rb[j][0];
                    if constexpr (OP == OP_FULL)   // the weight times 2^-10, for the residual product
                        bl[j] = __builtin_bit_cast(
                            u32x4, __builtin_bit_cast(f16x8, bh[j]) * (_Float16)0x1p-10f);
                    else if constexpr (OP == OP_PRESPLIT)
                        bl[j] = rb[j][RB - 1];
                }
            } else if constexpr (BS == B_ROWS) {
#pragma unroll
                for (int j = 0; j < NB; ++j) {
#pragma unroll
                    for (int q = 0; q < 2; ++q) {
                        u32x4 r = rb[j][q];
                        if (TAIL && !TURN && kc == KC - 1 && kc * 32 + 8 * fg + 4 * q + 4 > K)
                            r = shift_quad(r, back_k);
                        const f32x4 x = __builtin_bit_cast(f32x4, r);
                        uint32_t h0, l0, h1, l1;
                        split2(x.x, x.y, h0, l0);
                        split2(x.z, x.w, h1, l1);
                        bh[j][2 * q] = h0;
                        bh[j][2 * q + 1] = h1;
                        bl[j][2 * q] = l0;
                        bl[j][2 * q + 1] = l1;
                    }
                }
            } else {
                const float *v = reinterpret_cast<const float *>(rb);
#pragma unroll
                for (int j = 0; j < NB; ++j)
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        float x0 = v[2 * t * NB + j], x1 = v[(2 * t + 1) * NB + j];
                        if (NB > 1 && edge_n) {
                            // column j of a lane that read back_n columns early
#pragma unroll
                            for (int c = j + 1; c < NB; ++c) {
                                x0 = back_n == c - j ? v[2 * t * NB + c] : x0;
                                x1 = back_n == c - j ? v[(2 * t + 1) * NB + c] : x1;
                            }
                        }
                        uint32_t h, l;
                        split2(x0, x1, h, l);
                        bh[j][t] = h;
                        bl[j][t] = l;
                    }
            }
        };
        auto frag_a = [&](const char *st, int ks, u32x4 *ah, u32x4 *al) {
#pragma unroll
            for (int i = 0; i < MB; ++i) {
                const int off = L::chunk_off((wm * MB + i) * 16 + fr, 4 * ks + fg);
                ah[i] = *reinterpret_cast<const u32x4 *>(st + off);
                if (O::AP == 2) al[i] = *reinterpret_cast<const u32x4 *>(st + A_PLANE + off);
            }
        };
        auto multiply = [&](const u32x4 *bh, const u32x4 *bl, const u32x4 *ah, const u32x4 *al) {
#pragma unroll
            for (int j = 0; j < NB; ++j)
#pragma unroll
                for (int i = 0; i < MB; ++i) acc[j][i] = mma<O::BF16>(bh[j], ah[i], acc[j][i]);
            if constexpr (OP == OP_FULL) {
#pragma unroll
                for (int j = 0; j < NB; ++j)
#pragma unroll
                    for (int i = 0; i < MB; ++i) acc[j][i] = mma<false>(bl[j], al[i], acc[j][i]);
            } else if constexpr (O::BF16) {
#pragma unroll
                for (int j = 0; j < NB; ++j)
#pragma unroll
                    for (int i = 0; i < MB; ++i) acc[j][i] = mma<true>(bl[j], ah[i], acc[j][i]);
#pragma unroll
                for (int j = 0; j < NB; ++j)
#pragma unroll
                    for (int i = 0; i < MB; ++i) acc[j][i] = mma<true>(bh[j], al[i], acc[j][i]);
            }
        };

        if (ns > 0 && wave < CW) {
            u32x4 rb[RC][NB][RB];
            constexpr int FP = PIPE ? 2 : 1;         // sets of A fragments
            u32x4 ah[FP][MB], al[FP][MB], bh[2][NB], bl[2][NB];
            // chunk c's packed B is multiplied out of its ring registers
            auto mul = [&](int f, int n) {
                if constexpr (BS == B_PACKED) {
                    u32x4 wh[NB], wl[NB];
                    frag_b(rb[n], 0, wh, wl);
                    multiply(wh, wl, ah[f % FP], al[f % FP]);
                } else {
                    multiply(bh[f], bl[f], ah[f % FP], al[f % FP]);
                }
            };
#pragma unroll
            for (int c = 0; c < RC; ++c) {
                load_b(rb[c], c);
                __builtin_amdgcn_sched_barrier(0);
            }
            __syncthreads();
            if (PIPE) frag_a(smem, 0, ah[0], al[0]);
            u32x4 raw[TURN ? NB : 1][2];             // the next chunk's B, turned
            if constexpr (TURN) {
                static_assert(RC >= 2, "two chunks turned ahead");
                turn_b(rb[0], 0, raw);
                frag_b(raw, 0, bh[0], bl[0]);
                turn_b(rb[1 % RC], 1, raw);
                __builtin_amdgcn_sched_barrier(0);
                load_b(rb[0], RC);
                load_b(rb[1 % RC], RC + 1);
            } else if constexpr (BS != B_PACKED) {
                frag_b(rb[0], 0, bh[0], bl[0]);
                __builtin_amdgcn_sched_barrier(0);
                load_b(rb[0], RC);
            }
            __builtin_amdgcn_sched_barrier(0);
            // While a chunk is multiplied, the next one's fragments of A are
            // read from LDS (its stage is complete: the loaders are a stage
            // ahead) and its B is split; then the registers of B that were read
            // are reloaded RC chunks ahead.
            int buf = 0;
            auto stage = [&](int t, int s, bool reload) {
                const char *cur = smem + buf;
                buf = buf == 2 * STAGE ? 0 : buf + STAGE;
                const char *nxt = smem + buf;
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    const int c = t * KS + ks;                 // chunk of the trip
                    constexpr int TC = T * KS;
                    const int f = c & 1, g = f ^ 1, m = c % RC, n = (c + 1) % TC % RC;
                    if constexpr (PIPE)
                        frag_a(ks + 1 < KS ? cur : nxt, (ks + 1) % KS, ah[g % FP], al[g % FP]);
                    else
                        frag_a(cur, ks, ah[0], al[0]);
                    const int n2 = (c + 2) % TC % RC;
                    if constexpr (TURN) {
                        frag_b(raw, 0, bh[g], bl[g]);
                        turn_b(rb[n2], s * KS + ks + 2, raw);
                    } else if constexpr (BS != B_PACKED) {
                        frag_b(rb[n], s * KS + ks + 1, bh[g], bl[g]);
                    }
                    mul(f, m);
                    constexpr int NM = MB * NB * (OP == OP_BASE ? 1 : OP == OP_FULL ? 2 : 3);
                    constexpr int ND = MB * O::AP + (TURN ? 2 * NB : 0);
                    constexpr int NV = BS == B_PACKED ? (OP == OP_FULL ? 4 * NB : 0) : 26 * NB;
                    constexpr int PV = (NV + NM - 1) / NM;
                    constexpr int PD = (ND + NM - 1) / NM;
                    // LDS reads and the split's VALU work between the MFMAs
#pragma unroll
                    for (int x = 0; PIPE && x < NM; ++x) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                        if (x * PD < ND) __builtin_amdgcn_sched_group_barrier(0x100, PD, 0);
                        if (PV) __builtin_amdgcn_sched_group_barrier(0x002, PV, 0);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    if (reload) {
                        if constexpr (BS == B_PACKED) load_b(rb[m], s * KS + ks + RC);
                        else if constexpr (TURN) load_b(rb[n2], s * KS + ks + 2 + RC);
                        else load_b(rb[n], s * KS + ks + 1 + RC);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                __syncthreads();
            };
            int s0 = 0;
            for (; s0 + T <= ns; s0 += T) {
#pragma unroll
                for (int t = 0; t < T; ++t) stage(t, s0 + t, true);
            }
#pragma unroll
            for (int t = 0; t + 1 < T; ++t)
                if (s0 + t < ns) stage(t, s0 + t, false);
            const int whole = (ns + RA - 1) / RA * RA;       // the loaders' whole groups
            for (int s = ns; s < whole; ++s) __syncthreads();
        } else if (ns > 0) {
            u32x4 ra[RA][NA];
#pragma unroll
            for (int t = 0; t < RA; ++t) {
                load_a(ra[t], t);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                store_a(smem + t * STAGE, ra[t], t);
                load_a(ra[t], RA + t);
                __builtin_amdgcn_sched_barrier(0);
            }
            __syncthreads();
            int buf = 2 * STAGE;
            for (int s0 = 0; s0 < ns; s0 += RA) {
#pragma unroll
                for (int t = 0; t < RA; ++t) {
                    const int s = s0 + t;
                    store_a(smem + buf, ra[(t + 2) % RA], s + 2);
                    buf = buf == 2 * STAGE ? 0 : buf + STAGE;
                    __builtin_amdgcn_sched_barrier(0);
                    load_a(ra[(t + 2) % RA], s + 2 + RA);
                    __syncthreads();
                }
            }
        }
        if (wave >= CW) {
            if (b + gridDim.y < p.batch) __syncthreads();
            continue;
        }

        float *__restrict__ C = p.C + b * p.strideC;
        auto scaled = [&](float x) {
            if constexpr (OP == OP_BASE || OP == OP_FULL) return ldexpf(x, -p.e);
            if constexpr (OP == OP_BF16X3) return p.alpha == 1.0f ? x : x * p.alpha;
            return x;
        };
        auto store_c = [&](int64_t m, int64_t n, f32x4 v) {
            if (m < M && n < N) {
                float *cp = C + m * p.ldc + n;
                if (n + 4 <= N) {
                    *reinterpret_cast<f32x4_u *>(cp) = v;
                } else {
                    cp[0] = v.x;
                    if (n + 1 < N) cp[1] = v.y;
                    if (n + 2 < N) cp[2] = v.z;
                }
            }
        };
        // pairs of 16-column blocks as whole 128-byte lines (whole_lines)
        constexpr int LN = BS == B_COLS ? 0 : NB / 2 * 2;
#pragma unroll
        for (int i = 0; i < MB; ++i) {
            const int64_t mb = m0 + (wm * MB + i) * 16;
            const int64_t nb = n0 + wn * 16 * NB;
            auto block = [&](int j) {
                f32x4 v;
#pragma unroll
                for (int t = 0; t < 4; ++t) v[t] = scaled(acc[j][i][t]);
                return v;
            };
#pragma unroll
            for (int j = 0; j < LN; j += 2) {
                f32x4 x, y;
                whole_lines(block(j), block(j + 1), fr, x, y);
                const int64_t n = nb + 16 * j + 16 * (fr >> 3) + 4 * fg;
                store_c(mb + (fr & 7), n, x);
                store_c(mb + 8 + (fr & 7), n, y);
            }
#pragma unroll
            for (int j = LN; j < NB; ++j) {
                if constexpr (BS == B_COLS) {
                    // the lane's 4 NB results are columns 4 NB fg .. of the wave's,
                    // result e of block c at NB e + c
                    f32x4 v;
#pragma unroll
                    for (int t = 0; t < 4; ++t)
                        v[t] = scaled(acc[(4 * j + t) % NB][i][(4 * j + t) / NB]);
                    store_c(mb + fr, nb + 4 * NB * fg + 4 * j, v);
                } else {
                    store_c(mb + fr, nb + 16 * j + 4 * fg, block(j));
                }
            }
        }
        if (b + gridDim.y < p.batch) __syncthreads();  // LDS reuse by the next batch entry
    }
}

template <int OP, int BS, int MB, int WVM, int NB, int WVN, int KS, int RC, int LW, int RA, bool PIPE,
          bool TURN = false>
hipError_t launch_cfg(const DirectArgs &a, hipStream_t stream)
{
    constexpr int BM = 16 * MB * WVM, BN = 16 * NB * WVN;
    const int64_t tiles = ((a.M + BM - 1) / BM) * ((a.N + BN - 1) / BN);
    const dim3 grid((unsigned)tiles, (unsigned)(a.batch < 65535 ? a.batch : 65535));
    const dim3 block(64 * (WVM * WVN + LW));
    if (a.K % (32 * KS)) {
        // (direct_plan keeps K tails off the 128 x 128 tiles of an FP32 B, whose
        // form spilled 27 and 49 registers)
        if constexpr (BS != B_PACKED && BM == 128) return hipErrorInvalidValue;
        else
            hipLaunchKernelGGL((gemm_direct_kernel<OP, BS, MB, WVM, NB, WVN, KS, RC, LW, RA, PIPE, TURN, true>),
                               grid, block, 0, stream, a);
    } else
        hipLaunchKernelGGL((gemm_direct_kernel<OP, BS, MB, WVM, NB, WVN, KS, RC, LW, RA, PIPE, TURN, false>),
                           grid, block, 0, stream, a);
    return hipGetLastError();
}

// Tile configurations (rows x columns of the tile).
enum Cfg : int {
    T32x32, T32x64, T32x128, T64x64, T64x128, T64x192, T64x256, T96x128, T96x256, T128x128, T128x256,
    T_COUNT
};
constexpr int kTileM[T_COUNT] = {32, 32, 32, 64, 64, 64, 64, 96, 96, 128, 128};
constexpr int kTileN[T_COUNT] = {32, 64, 128, 64, 128, 192, 256, 128, 256, 128, 256};

// The tiles of 192 and 256 columns are for packed B only: a wave that owns 48 or
// 64 columns reads each fragment of A from LDS for three or four blocks instead
// of two, and a column strip of 256 halves how often A is staged.  At 4096 deep,
// one tile per CU, us, best tiles of at most 128 columns (128 x 256 HEAL-Full:
// eight computing waves of 64 x 64) -> these:
//              512 x 6144    1024 x 4096   1536 x 4096    2048 x 4096
//   HEAL-Base  44.5 -> 35.5  45.7 -> 41.6  70.5 -> 53.1   87.3 -> 66.9
//   HEAL-Full  65.3 -> 49.8  70.6 -> 61.5  111 -> 85.5    121 -> 111
//   pre-split  72.7 -> 65.0  (83.0, 85.1)  134 -> 117     165 -> 153
// The pre-split product has no 64 x 256 tile (85.1 above, 83.0 on 128 x 128).  The
// 128-column tiles stay for outputs whose width they divide better (HEAL-Base
// 7059 x 1141 x 8301 128 x 128 237, 64 x 128 271 us).
// With an FP32 B, whose raw quads and both parts are held too, they spill
// (1024 x 4096 K x N: 64 x 256 tiles 179 us, 98 on the tiles it takes now).
// Of the forms built, these spill: every 128 x 256 one (HEAL-Base 11 registers, 18
// with a K tail, HEAL-Full 12 and 20, pre-split 44 and 58), the pre-split 96 x 256
// one with a K tail (10) and the K x N 64 x 64 one with a K tail (4).  The plan's
// costs were fitted to these times as they are: it takes them where they are
// faster all the same (2048 x 4096 above).

template <int OP, int BS>
hipError_t launch_tile(int cfg, const DirectArgs &a, hipStream_t stream)
{
    constexpr bool PACKED = BS == B_PACKED, ROWS = BS == B_ROWS;
    switch (cfg) {
    //                                      MB WVM NB WVN KS RC LW RA PIPE [TURN]
    case T32x32: return launch_cfg<OP, BS, 2, 1, 1, 2, 2, 4, 2, 2, true>(a, stream);
    case T32x64: return launch_cfg<OP, BS, 2, 1, 1, 4, 2, 4, 4, 2, true, ROWS>(a, stream);
    case T64x128:
        if constexpr (PACKED) return launch_cfg<OP, BS, 4, 1, 2, 4, 2, 4, 4, 4, true>(a, stream);
        else if constexpr (ROWS) return launch_cfg<OP, BS, 4, 1, 1, 8, 2, 4, 4, 2, false, true>(a, stream);
        else return launch_cfg<OP, BS, 4, 1, 2, 4, 2, 2, 4, 2, true>(a, stream);
    case T64x192:
        if constexpr (PACKED) return launch_cfg<OP, BS, 4, 1, 3, 4, 2, 2, 4, 2, true>(a, stream);
        break;
    case T64x256:
        if constexpr (OP == OP_BASE || OP == OP_FULL) return launch_cfg<OP, BS, 4, 1, 4, 4, 2, 2, 4, 2, true>(a, stream);
        break;
    case T96x256:
        if constexpr (PACKED) return launch_cfg<OP, BS, 6, 1, 4, 4, 1, 2, 4, 4, false>(a, stream);
        break;
    case T128x128: return launch_cfg<OP, BS, 8, 1, 2, 4, 2, 2, 4, 2, false>(a, stream);
    case T96x128:
        if constexpr (PACKED) return launch_cfg<OP, BS, 6, 1, 2, 4, 2, 4, 4, 4, false>(a, stream);
        else return launch_cfg<OP, BS, 6, 1, 2, 4, 2, 2, 4, 2, false>(a, stream);
    case T32x128:
        if constexpr (PACKED) return launch_cfg<OP, BS, 2, 1, 2, 4, 2, 4, 4, 4, true>(a, stream);
        break;
    case T64x64:
        if constexpr (!PACKED) return launch_cfg<OP, BS, 4, 1, 1, 4, 4, 4, 4, 2, true, ROWS>(a, stream);
        break;
    case T128x256:
        if constexpr (PACKED) return launch_cfg<OP, BS, 8, 1, 4, 4, 1, 2, 4, 2, false>(a, stream);
        break;
    }
    return hipErrorInvalidValue;
}

// 32-deep chunks of K per stage: a K tail is what is left of whole stages.
constexpr int kStage[T_COUNT] = {2, 2, 2, 4, 2, 2, 2, 2, 1, 2, 1};

// Time of one launch by kernel, in us over that of an empty one: at 4096 deep with
// up to 64 tiles, with 256 (one per CU) and per further 256 tiles (0: one tile per
// CU at a time, so rounds, of whose last one `part` is the share that its empty
// CUs cost too); a fixed part per 256 tiles (the first loads, the last stage);
// per million elements of C, and of a C whose rows are not whole 128-byte lines;
// and what a K tail adds to the time by depth (its share) and to the fixed part.
// Fitted to the times of every tile on 12 000 random products of 65 to 8192 rows,
// 4 to 32768 columns and 4 to 16384 deep, a third of them of sizes that divide by
// nothing (the depths of the smallest HEAL-Base and HEAL-Full tiles are those of
// products 4096 deep).  Fitted to one half, the smallest estimate is within 1.3% of
// the fastest kernel on the other (geometric mean).  The table before had no terms
// for C and took every K tail for 0.5 us: it was 5% off, and 2% of these products
// ran slower than on the staged kernels, up to twice as long with shallow K,
// between one and three rounds, and with rows of C that are not whole lines (3 x
// 155 x 11932 x 52 K x N 35.1 -> 18.5 us, 195 x 21948 x 13 pre-split 22.8 -> 15.1).
// The last two are the 128 x 128 and the 256 x 256 tiles of the staged kernels.
// {}: not built.
constexpr int kMedium = T_COUNT, kLarge = T_COUNT + 1;
struct Cost { float few, full, more, part, fixed, out, ragged, tail, tail_fixed; };
constexpr Cost kCost[6][T_COUNT + 2] = {
    // 32x32, 32x64, 32x128, 64x64, 64x128, 64x192, 64x256, 96x128, 96x256, 128x128, 128x256; medium, large
    {// HEAL-Base
     {13, 15, 7.5f, 0, 0.3f, 0.54f, 0, 0.1f, 0.35f}, {14, 17.6f, 11, 0, 0.3f, 1.06f, 0, 0, 0.41f},
     {17.5f, 19.4f, 16, 0, 0.74f, 0.95f, 0, 0, 0.6f}, {},
     {19, 21.9f, 0, 1, 1.93f, 0.76f, 0, 0.14f, 0.7f}, {24.7f, 31, 0, 0.96f, 1.86f, 0.64f, 0.16f, 0.12f, 0.63f},
     {29, 35.5f, 0, 1, 2.17f, 0.71f, 0, 0.1f, 0.65f}, {24.2f, 28.1f, 0, 1, 3.11f, 0.82f, 0, 0.27f, 0.98f},
     {36.2f, 43.1f, 0, 0.95f, 3.37f, 0.6f, 0, 0.21f, 0.54f}, {33.8f, 38.2f, 0, 1, 3.03f, 0.7f, 0, 0.16f, 0.85f},
     {44.2f, 53.9f, 0, 0.91f, 4.4f, 0.73f, 0.02f, 0.32f, 1.22f}, {39.3f, 38.8f, 0, 0.82f, 1.43f, 0.61f, 0.62f, 0.03f, 0},
     {77.3f, 90.7f, 0, 1, 4.63f, 0.76f, 1, 0.04f, 0.6f}},
    {// HEAL-Full
     {18.2f, 20.7f, 6.6f, 0, 0.67f, 0.05f, 0, 0.31f, 0.32f}, {16, 21, 13.3f, 0, 0.63f, 0.59f, 0, 0.05f, 0.49f},
     {19.8f, 25.6f, 21, 0, 1.28f, 0.5f, 0, 0, 0.87f}, {},
     {27.4f, 32, 0, 1, 2.5f, 0.97f, 0, 0.15f, 1.31f}, {34.9f, 41.9f, 0, 1, 2.39f, 0.84f, 0, 0.08f, 0.82f},
     {43.6f, 53.6f, 0, 0.98f, 2.64f, 0.7f, 0, 0.03f, 0.83f}, {40.3f, 48.8f, 0, 0.97f, 3.84f, 0.76f, 0, 0.1f, 1.62f},
     {61.8f, 77, 0, 0.91f, 3.71f, 0.59f, 0, 0.06f, 0.91f}, {53.1f, 62.4f, 0, 0.99f, 3.47f, 0.7f, 0, 0.09f, 1.57f},
     {80, 100.8f, 0, 0.86f, 4.89f, 0.78f, 0, 0.12f, 1.61f}, {68.9f, 69.7f, 0, 0.64f, 1.61f, 0.58f, 0.69f, 0, 0.08f},
     {155, 187.3f, 0, 0.96f, 3.92f, 0.78f, 0.9f, 0, 0.05f}},
    {},  // (INT16 scores: not here)
    {// pre-split
     {15.7f, 18.5f, 8.5f, 0, 0.56f, 0.26f, 0, 0.32f, 0.29f}, {15.6f, 16.2f, 0, 0.82f, 0.53f, 1.08f, 0, 0.11f, 0.44f},
     {22.4f, 27.6f, 0, 0.96f, 1.25f, 1.38f, 0, 0.04f, 0.79f}, {},
     {32.9f, 40.3f, 0, 0.99f, 2.48f, 1.03f, 0, 0.08f, 0.99f}, {49.2f, 59.6f, 0, 0.97f, 2.23f, 0.88f, 0, 0.02f, 0.94f},
     {}, {48.3f, 60, 0, 0.94f, 3.64f, 0.82f, 0, 0.08f, 1.4f},
     {93.8f, 113, 0, 0.91f, 3.61f, 0.7f, 0, 0.04f, 1.93f}, {60.5f, 74.9f, 0, 0.92f, 3.23f, 0.76f, 0, 0.09f, 1.39f},
     {119.7f, 144.5f, 0, 0.86f, 7.2f, 1.05f, 0, 0.04f, 2.12f}, {87.8f, 97.4f, 0, 0.96f, 1.57f, 0.65f, 0.63f, 0, 0.26f},
     {187.3f, 237.3f, 0, 0.79f, 4.04f, 0.79f, 1.2f, 0, 0.04f}},
    {// bf16x3, B stored K x N
     {23.8f, 28.1f, 13.4f, 0, 0.7f, 0.54f, 0, 0.04f, 0.34f}, {26.6f, 25.7f, 0, 1, 0.69f, 1.08f, 1.83f, 0.05f, 0.58f},
     {}, {32.3f, 37.2f, 0, 1, 2.1f, 1.74f, 0.15f, 0.06f, 1.82f},
     {52.2f, 59.7f, 0, 1, 1.81f, 1.2f, 0.07f, 0.09f, 0.91f}, {},
     {}, {61.4f, 72.5f, 0, 1, 2.61f, 0.95f, 0.12f, 0.08f, 1.2f},
     {}, {72.3f, 85.6f, 0, 1, 3.44f, 0.85f, 0.11f, 0.05f, 0.2f},
     {}, {118.3f, 121.5f, 0, 0.78f, 1.69f, 0.78f, 0.15f, 0.02f, 0.73f},
     {204.7f, 231.4f, 0, 1, 3.6f, 0.73f, 1.09f, 0.03f, 0.64f}},
    {// bf16x3, B stored N x K
     {20.7f, 26.6f, 14, 0, 0.77f, 0.75f, 0, 0.58f, 0}, {26.1f, 28.1f, 0, 1, 0.66f, 2.96f, 0, 0.48f, 0.87f},
     {}, {33.4f, 36.8f, 0, 1, 2.01f, 1.9f, 0, 0.23f, 1.86f},
     {47.3f, 55.3f, 0, 0.98f, 2.01f, 1.17f, 0, 0.24f, 1.55f}, {},
     {}, {68.2f, 77.7f, 0, 0.95f, 2.22f, 1.01f, 0, 0.2f, 1.86f},
     {}, {77.3f, 92.3f, 0, 0.9f, 2.65f, 1.03f, 0, 0.05f, 0.2f},
     {}, {125.8f, 137.5f, 0, 0.72f, 0.78f, 0.75f, 0.35f, 0.03f, 0.24f},
     {204.2f, 224.1f, 0, 0.99f, 3.32f, 0.86f, 1.18f, 0, 0.16f}},
};

// The staged kernels on rows that they read by element: 16, 32 and 64 rows (strips
// of the skinny kernels' widths with a packed B, else 64 columns), medium, large.
// `tail` of the first three: the share of the time by depth that is proportional
// to the rows, A's loads.  Those three fitted to 9000 products of 1 to 64 rows, which
// the direct-B kernel had all taken on the strength of 16 x 1003 x 999 (K x N 30.3
// -> 9.3 us, N x K 25.8 -> 12.7, HEAL-Base 8.6 -> 6.8, pre-split 8.9 -> 8.6): 19% of
// those with odd sizes ran slower on it, few rows of a deep packed B most
// (HEAL-Base 5 x 4 x 11216 23.4 -> 42.7, pre-split 3 x 8 x 16080 51.2 -> 86.4).
constexpr Cost kElement[6][5] = {
    {// HEAL-Base
     {13.2f, 22.1f, 13.3f, 0, 0.85f, 2.78f, 2.13f, 0.58f, 0}, {28.9f, 34.4f, 0, 0.75f, 1.38f, 3.26f, 0.59f, 0.95f, 0},
     {54.9f, 64.6f, 0, 0.82f, 1.69f, 1.69f, 0.49f, 0.95f, 0},
     {102.8f, 101.2f, 0, 0.85f, 2.98f, 0.47f, 0.98f, 0, 0}, {239.6f, 323.1f, 333.9f, 0, 6.82f, 1.18f, 1.52f, 0, 0}},
    {// HEAL-Full
     {14.5f, 22.2f, 10.7f, 0, 1.07f, 2.24f, 3.59f, 0.42f, 0}, {29.2f, 31, 0, 0.57f, 1.69f, 1.76f, 2, 0.43f, 0},
     {55.3f, 67.9f, 0, 0.66f, 1.87f, 2.82f, 0, 0.86f, 0},
     {127.7f, 129.3f, 0, 1, 3.01f, 0.89f, 0.76f, 0, 0}, {266.5f, 317.1f, 213.8f, 0, 7.31f, 1.2f, 1.52f, 0, 0}},
    {},
    {// pre-split
     {15.6f, 21.2f, 29.5f, 0, 1.28f, 3.05f, 1.73f, 0.33f, 0}, {29.6f, 35.9f, 0, 0.72f, 1.5f, 7.01f, 0, 0.6f, 0},
     {54.9f, 67.6f, 0, 0.82f, 1.94f, 2.11f, 1.02f, 0.68f, 0},
     {141.8f, 149.4f, 0, 1, 3.54f, 1.01f, 0.42f, 0, 0}, {323.6f, 352.8f, 625.5f, 0, 4.58f, 1.84f, 0.65f, 0, 0}},
    {// bf16x3, B stored K x N
     {114.6f, 164.2f, 88.3f, 0, 0.27f, 0.69f, 1.65f, 0.1f, 0}, {126.7f, 185.9f, 84.5f, 0, 0.85f, 1.45f, 0, 0.16f, 0},
     {150.9f, 242.5f, 100.1f, 0, 1.68f, 1.19f, 0, 0.35f, 0},
     {271.1f, 283.3f, 0, 0.73f, 3.7f, 1.94f, 0, 0, 0}, {691.7f, 700, 0, 0.69f, 9.88f, 2.03f, 0, 0, 0}},
    {// bf16x3, B stored N x K
     {92.3f, 118.9f, 64.4f, 0, 0.28f, 0.78f, 3.25f, 0.15f, 0}, {112.2f, 150, 78.8f, 0, 0.6f, 1.62f, 0.19f, 0.4f, 0},
     {148.8f, 193.3f, 109.2f, 0, 1.41f, 1.02f, 0.37f, 0.56f, 0},
     {249, 253.4f, 0, 0.82f, 0.89f, 3.21f, 0, 0, 0}, {510.1f, 514.1f, 0, 0.74f, 15.57f, 1.96f, 0, 0, 0}},
};

int cost_index(int op, bool rows) { return rows ? OP_BF16X3 + 1 : op; }

// `wgs` workgroups that run `per` tiles one after another, each `depth` times 4096
// deep, on an output of `mega` million elements, in whole lines or not (`ragged`).
float estimate(const Cost &c, int64_t wgs, int per, float depth, float fixed, float mega, bool ragged, int cus)
{
    const float r = (float)wgs / (float)cus;
    depth *= (float)per;
    fixed *= (float)per;
    float t;
    if (r <= 1.0f)
        t = fixed + depth * (c.few + (c.full - c.few) * (r < 0.25f ? 0.0f : (r - 0.25f) / 0.75f));
    else if (c.more > 0.0f)
        t = fixed * r + depth * (c.full + (r - 1.0f) * c.more);
    else
        t = (fixed + depth * c.full) * (c.part * (float)((wgs + cus - 1) / cus) + (1.0f - c.part) * r);
    return t + (ragged ? c.out + c.ragged : c.out) * mega;
}

// Other tiles have to be this much faster by their estimate than the kernel that
// the output's size alone would choose.
float handicap(float t) { return 1.04f * t + 0.15f; }

// Up to 64 rows the skinny kernels stream B; the direct-B kernel is faster where
// their narrow strips each convert all of A.  64 x N x 4096, us, skinny ->
// direct: HEAL-Full 1024 columns 28.5 -> 19.1, 4096 30.9 -> 19.2, 8192 42.0 -> 20.2,
// 14336 56.2 -> 35.7, 65536 145 -> 112, 128256 208 -> 225; HEAL-Base 8192 25.9 ->
// 17.8, 16032 38.6 -> 36.4, 32064 53.2 -> 54.6, 65536 131 -> 103, 128256 201 -> 214;
// pre-split 8192 49.0 -> 34.7, 14336 64.8 -> 57.6, 16032 58.2 -> 59.8, 65536 215 ->
// 197; K x N 4096 23.3 -> 28.6, 8192 41.9 -> 40.2, 10240 68.4 -> 75.3, 14336 75.9 ->
// 61.1, 16032 66.8 -> 57.7, 32064 113 -> 94;
// N x K 8192 40.3 -> 43.5, 14336 72.0 -> 58.2, 32064 109 -> 117.  32 rows: HEAL-Full
// 4096 16.8 -> 19.1, 8192 24.1 -> 19.6, 16032 39.2 -> 34.6, 32064 55.0 -> 50.7;
// pre-split 8192 28.1 -> 29.4, 16032 54.2 -> 48.8.
// Other depths: over 300 random products of 17 to 64 rows inside these windows,
// those at least 512 deep gain 1.3x; shallower ones lose up to 1.1x (HEAL-Full
// 40 x 64 x 396 5.5 -> 6.6, HEAL-Base 40 x 192 x 280 4.3 -> 5.0), and so do wide ones
// less than 2048 deep, bound by C (HEAL-Base 41 x 88568 x 288 15.3 -> 18.4, HEAL-Full
// 51 x 66444 x 324 17.8 -> 22.0, HEAL-Base 60 x 85184 x 676 27.6 -> 30.2).
// HEAL-Base and pre-split of 33 to 64 rows stay on the skinny kernels from 15360 to
// 61440 columns: which tile is the fastest there changes from width to width, with
// some much slower, and the skinny kernels have no estimate to choose by (64 rows,
// the same weight again and again, skinny -> the fastest tile, the slowest: HEAL-Base
// 16032 26.9 -> 24.8, 36.3; 20480 40.7 -> 30.2, 37.4; 32064 48.5 -> 48.1, 58.3; 40960
// 84.5 -> 67.6, 88.5; 57344 94.8 -> 93.4, 123; pre-split 20480 88.6 -> 73.6, 98.1;
// 32064 99.7 -> 100, 119).
bool beats_skinny(int op, bool rows, const DirectArgs &a)
{
    if (a.batch != 1 || a.K < 512 || a.M <= 16) return false;
    const int64_t N = a.N;
    if (N >= 61440 && a.K < 2048) return false;
    if (op == OP_BF16X3)
        return a.M > 32 && N >= 12288 && N <= (rows ? 16384 : 32768);
    if (a.M <= 32) return N >= (op == OP_PRESPLIT ? 16000 : 8192) && N <= 32768;
    if (N >= 15360 && N < 61440 && op != OP_FULL) return false;
    return N <= 98304;
}

}  // namespace

int direct_plan(int op, bool trans_b, const DirectArgs &a)
{
    // whole quads or columns to shift within a row; 32-bit byte offsets within
    // a tile's rows of A, a tile of B, or all of B stored K x N (one stage
    // past its end for the clamped index)
    const int64_t lim = 0x7fffffffLL;
    const bool rows = op == OP_BF16X3 && trans_b, cols = op == OP_BF16X3 && !trans_b;
    if (a.K < 4 || a.K > (1 << 28) || ((int64_t)127 * a.lda + a.K + 128) * 4 >= lim)
        return DIRECT_NONE;
    if (rows && ((int64_t)255 * a.ldb + a.K + 128) * 4 >= lim) return DIRECT_NONE;
    if (cols && (a.N < 4 || a.ldb >= lim || (a.K + 128) * a.ldb * 4 >= lim)) return DIRECT_NONE;
    if (a.M <= 64 && a.vec && !beats_skinny(op, rows, a)) return DIRECT_NONE;
    // one stage of the element-reading tiles, where B is not small and shared by
    // enough workgroups (one product: 0.82 of the time of the fastest tile here,
    // geometric mean over random sizes; 17 of 1 x 15872 x 64 20 us against 37; but 4 of
    // 3 x 1664 x 64 5.7 against 3.7)
    if (a.M <= 64 && !a.vec && rows && a.K <= 64 && (a.batch == 1 || (float)a.batch * (float)a.N > 32768.0f))
        return DIRECT_NONE;
    const int cus = device_cus();
    const Cost *cost = kCost[cost_index(op, rows)];
    const bool ragged = a.ldc % 32 != 0 || a.strideC % 32 != 0 || (reinterpret_cast<uintptr_t>(a.C) & 127u) != 0;
    const float mega = (float)a.batch * (float)a.M * (float)a.N * 1e-6f;
    auto tiles = [&](int64_t bm, int64_t bn) { return ((a.M + bm - 1) / bm) * ((a.N + bn - 1) / bn); };
    float best = 0.0f;
    int plan = DIRECT_NONE;
    // the tiled bf16x3 kernel's workgroups take two batch entries each
    const int per = op == OP_BF16X3 && a.batch > 1 ? 2 : 1;
    const int64_t entries = (a.batch + per - 1) / per;
    const Cost *element = kElement[cost_index(op, rows)];
    const float depth = (float)a.K / 4096.0f;
    auto tiled = [&](const Cost &c, int64_t wgs, int tile_per, bool tail) {
        return estimate(c, wgs, tile_per, tail ? depth * (1.0f + c.tail) : depth,
                        tail ? c.fixed + c.tail_fixed / (float)tile_per : c.fixed, mega, ragged, cus);
    };
    if (a.M <= 64 && !a.vec) {
        const int h = a.M <= 16 ? 0 : a.M <= 32 ? 1 : 2;
        const Cost &c = element[h];
        const int64_t w = op == OP_BF16X3 ? 64 : skinny_strip_width(a.N, a.M);
        best = estimate(c, (a.N + w - 1) / w * entries, per, depth * (1.0f - c.tail * (1.0f - (float)a.M / (float)(16 << h))),
                        c.fixed, mega, ragged, cus);
    } else if (a.M > 64) {
        const Cost *staged = a.vec ? cost + kMedium : element + 3;
        float medium = tiled(staged[0], tiles(128, 128) * entries, per, a.K % 64 != 0);
        float large = tiled(staged[1], tiles(256, 256) * a.batch, 1, a.K % 32 != 0);
        if (select_instance(a.M, a.N) == HEAL_INSTANCE_LARGE) medium = handicap(medium);
        else large = handicap(large);
        best = medium < large ? medium : large;
        plan = medium < large ? DIRECT_MEDIUM : DIRECT_LARGE;
    }
    for (int c = 0; c < T_COUNT; ++c) {
        const int64_t n = tiles(kTileM[c], kTileN[c]);
        if (cost[c].full <= 0.0f || n * a.batch > (1 << 20)) continue;
        // (no K-tail form: launch_cfg)
        if (c == T128x128 && op == OP_BF16X3 && a.K % 64 != 0) continue;
        const float t = handicap(tiled(cost[c], n * a.batch, 1, a.K % (32 * kStage[c]) != 0));
        if (best == 0.0f || t < best) {
            best = t;
            plan = c;
        }
    }
    return plan;
}

int direct_tile(int plan) { return plan >= 0 ? 1000 * kTileM[plan] + kTileN[plan] : 0; }

hipError_t launch_direct(int op, bool trans_b, int cfg, const DirectArgs &a, hipStream_t stream)
{
    switch (op) {
    case OP_BASE: return launch_tile<OP_BASE, B_PACKED>(cfg, a, stream);
    case OP_FULL: return launch_tile<OP_FULL, B_PACKED>(cfg, a, stream);
    case OP_PRESPLIT: return launch_tile<OP_PRESPLIT, B_PACKED>(cfg, a, stream);
    case OP_BF16X3:
        return trans_b ? launch_tile<OP_BF16X3, B_ROWS>(cfg, a, stream)
                       : launch_tile<OP_BF16X3, B_COLS>(cfg, a, stream);
    }
    return hipErrorInvalidValue;
}

}  // namespace heal
