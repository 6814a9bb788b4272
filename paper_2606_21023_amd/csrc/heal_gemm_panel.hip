// The short-K panel kernel for gfx950 (MI355X): products whose K is at most
// 128 with B stored N x K, the shape of attention scores (Q K^T over a head
// dimension of 128).  Two products run on it:
//
//  * bf16x3 (HEAL Section 4, GEMM paragraph and its displayed expansion):
//    FP32 operands split into bf16 (hi, lo), C = hiA*hiB + hiA*loB + loA*hiB;
//  * the INT16 scores (HEAL Section 4, Q/K/V paragraph): INT16 codes split
//    into two exact FP16 parts (hi, q - hi), four products, the sum scaled
//    by alpha (maxQ/32767)(maxK/32767).
//
// Rows of C of any length and alignment are taken (RAG): half lines at the ends
// of the pieces a store writes have to meet in L2, so these are plain stores
// (32 heads of 1531 x 1531 x 128: bf16x3 276.8 us and INT16 172.7 on tiles,
// 130.5 and 114.7 here, 245.7 and 225.8 with non-temporal stores), and the last
// one to three columns of a row are stored by element.  Panels of 16, 32 and
// 64 rows take the few-query products, bound by reading B (TURN below: 32
// heads of 1 x 3001 x 128 INT16 44.6 -> 8.6 us, 17.3 with B read in fragment
// order).
//
// Panels of 128 and 256 rows are bound by writing C: every output element
// costs 4 bytes of HBM writes against 2K or 4K multiply-adds, so the kernel is
// built to keep the write stream busy.  A workgroup owns a panel of A's rows
// (one batch entry), splits it once into LDS, and then walks its share
// of the columns of C in steps of 128: each of its four waves loads the B
// fragments of its 32 columns straight from global memory (B stored N x K:
// a lane's 8 consecutive k of one column are 32 contiguous bytes), splits
// them in registers, multiplies them against the whole panel and stores its
// block of C in whole 128-byte lines, non-temporal (streamed past the
// caches, which the output would only pollute).  The loads of the next
// step are issued before the multiplies of the current one, so they have a
// whole step to arrive, and the stores of
// a step drain while the next one is multiplied.  B goes from L2 to
// registers once per workgroup (no LDS round trip), and the panel is read
// from LDS once per 32 columns.
//
// Workgroups are numbered so that each XCD owns a contiguous range of
// panels: the panels of one batch entry share its B in that XCD's L2.
//
// Reduction order: identical to every other instance (K in 32-deep chunks
// ascending; per chunk hiA*hiB, hiA*loB, loA*hiB for bf16x3 and hiQ*hiK,
// hiQ*loK, loQ*hiK, loQ*loK for the scores; one FP32 accumulator, the B
// fragment as the MFMA's first source, the K tail zero-filled), so results
// are bitwise equal to theirs.
#include <type_traits>

#include "heal.h"
#include "heal_device.h"
#include "heal_internal.h"

namespace heal {

namespace {

constexpr int PKMAX = 128;          // deepest K a panel holds
constexpr int PRP = 2 * PKMAX;      // LDS row pitch of a 16-bit plane, bytes
constexpr int PNT = 256;            // four waves
constexpr int PWN = 32;             // columns per wave and step
constexpr int PBN = 4 * PWN;        // columns per step
constexpr uint32_t kOOB = 0x80000000u;  // beyond every buffer range: loads read zeros

// Least workgroups per panel of more than 64 rows (each walking half of the
// columns with 2) and steps of B loads in flight per wave.  Measured on
// the attention scores (32 heads, 2048 x 2048 x 128): bf16x3 150 us with
// 256-row panels against 155 us with 128; the scores 128 us with 128-row
// panels against 136 us with 256; two workgroups per panel 1.05x faster
// than one, four slower; two steps of loads in flight slower than one.
#ifndef HEAL_PANEL_CSPLIT
#define HEAL_PANEL_CSPLIT 2
#endif
#ifndef HEAL_PANEL_PD
#define HEAL_PANEL_PD 1
#endif
#ifndef HEAL_PANEL_PD_SCORES
#define HEAL_PANEL_PD_SCORES 1
#endif
// C stores: each store instruction writes whole
// 128-byte lines (8 rows x 32 columns, the two 16 x 16 results of a row
// block traded between lane halves), and HEAL_PANEL_STORE_AUX 2 marks them
// non-temporal.  Measured on the attention scores: bf16x3 135 us and the
// INT16 scores 117 us, against 151 and 135 us for the 16-row x 64-byte
// stores of one result each with the default policy; whole lines with the
// default policy 154 / 135 us; non-temporal stores of 64-byte pieces
// 184 / 173 us (their lines reach HBM in halves).
#ifndef HEAL_PANEL_STORE_AUX
#define HEAL_PANEL_STORE_AUX 2
#endif
#ifndef HEAL_PANEL_RAG_AUX
#define HEAL_PANEL_RAG_AUX 0
#endif

struct PanelArgs {
    int64_t M, N, K;
    const char *A;
    int64_t lda, strideA;   // elements
    const char *B;          // N x K rows
    int64_t ldb, strideB;
    float *C;
    int64_t ldc, strideC;
    int64_t batch;
    float alpha;            // bf16x3: output scale (SCALE); scores: alpha
    const float *maxA, *maxB;  // scores: max|Q|, max|K| (device)
    int csplit;             // workgroups per panel, each walking its share of the columns
};

__device__ __forceinline__ u32x4 bload(__amdgpu_buffer_rsrc_t r, uint32_t voff)
{
    return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)voff, 0, 0));
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const char *base, int64_t bytes)
{
    // raw buffer; `bytes` < 2^31 is checked on the host
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(base), (short)0, (int)bytes,
                                             0x00020000);
}

// 16-byte chunk c (8 values of k) of panel row r, XOR-swizzled so that the
// 16 rows of a fragment read fall in 16 different bank groups.
__device__ __forceinline__ int panel_off(int r, int c) { return r * PRP + ((c ^ (r & 15)) << 4); }

template <bool SCORES>
__device__ __forceinline__ f32x4 mma(u32x4 b, u32x4 a, f32x4 c)
{
    if constexpr (SCORES)
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, b),
                                                      __builtin_bit_cast(f16x8, a), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, b),
                                                       __builtin_bit_cast(bf16x8, a), c, 0, 0, 0);
}

// Two parts of 8 consecutive values: bf16 (hi, lo) of 8 FP32 (two quads),
// or FP16 (hi, q - hi) of 8 INT16 codes (one 16-byte unit).
template <bool SCORES>
__device__ __forceinline__ void split8(const u32x4 *raw, u32x4 &h, u32x4 &l)
{
    if constexpr (SCORES) {
        const u32x4 v = raw[0];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            uint32_t hh, ll;
            unpack2_i16((int)(int16_t)(v[t] & 0xffffu), (int)(int16_t)(v[t] >> 16), hh, ll);
            h[t] = hh;
            l[t] = ll;
        }
    } else {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const f32x4 v = __builtin_bit_cast(f32x4, raw[q]);
            uint32_t h0, l0, h1, l1;
            split2(v.x, v.y, h0, l0);
            split2(v.z, v.w, h1, l1);
            h[2 * q] = h0;
            h[2 * q + 1] = h1;
            l[2 * q] = l0;
            l[2 * q + 1] = l1;
        }
    }
}

// KC: 32-deep chunks of K (K <= 32 KC).  SCALE: multiply the bf16x3 result
// by alpha.  PD: steps of B loads in flight per wave.  PBM: rows of the
// panel (128: two workgroups per CU; 256: one, B read from L2 half as often).
// RAG: rows of C that are not whole 128-byte lines apart, or N % 4 != 0.
// Waves per SIMD: three for the INT16 panels of at most 64 rows, but two for 32
// rows at full depth, which spilled 11 registers (29 with RAG) under the bound of
// three (32 heads of 32 x 3001 x 128 18.8 -> 10.8 us, 64 of 17 x 16384 84 -> 56).
// Three bf16x3 forms at full depth spill a little: 32 rows with RAG 9 registers (with
// and without SCALE), 128 rows without RAG 2.
template <bool SCORES, bool SCALE, int KC, int PD, int PBM, bool RAG>
__global__ void __launch_bounds__(PNT, PBM <= 64   ? (SCORES && !(PBM == 32 && KC == 4) ? 3 : 2)
                                       : PBM <= 128 ? 2 : 1) gemm_panel_kernel(PanelArgs p)
{
    constexpr int PRB = PBM / 16;               // 16-row blocks of the panel
    constexpr int PPLANE = PBM * PRP;           // one LDS plane of the panel
    static_assert(KC >= 1 && 32 * KC <= PKMAX, "K chunks of a panel");
    constexpr int ES = SCORES ? 2 : 4;          // bytes per operand element
    constexpr int RQ = SCORES ? 1 : 2;          // 16-byte loads per 8 values
    constexpr int UPR = 32 * KC * ES / 16;      // 16-byte units per panel row
    constexpr int PU = (PBM * UPR + PNT - 1) / PNT;   // panel units per thread
    constexpr bool PART = PBM * UPR % PNT != 0; // a small panel: the last units are short of threads

    // Panels of at most 64 rows, bound by reading B: each wave reads its rows
    // of B in memory order (a fragment's own order touches 16 rows with every
    // 16 lanes, a line each) and turns them through an LDS area of its own.
    constexpr bool TURN = PBM <= 64;
    constexpr int NBU = UPR / 2;                // 16-byte units of B per lane and step
    constexpr int TURN_BYTES = TURN ? 32 * UPR * 16 : 0;
    __shared__ __attribute__((aligned(16))) char smem[2 * PPLANE + 4 * TURN_BYTES];
    char *const ph = smem;                      // hi plane
    char *const pl = smem + PPLANE;             // lo plane

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int fr = lane & 15, fg = lane >> 4;

    // ---- panel: XCD-grouped numbering, then (batch entry, row panel) -----
    const int64_t panels = (p.M + PBM - 1) / PBM;
    int64_t L = blockIdx.x;
    {
        const int64_t nb = gridDim.x, x = L & 7, i = L >> 3, q = nb >> 3, r = nb & 7;
        L = x * q + (x < r ? x : r) + i;
    }
    const int64_t pid = L / p.csplit;
    const int cs = (int)(L - pid * p.csplit);
    const int64_t b = pid / panels;
    const int64_t m0 = (pid - b * panels) * PBM;
    const int64_t M = p.M, N = p.N, K = p.K;
    const int rows = (int)(M - m0 < PBM ? M - m0 : PBM);

    const __amdgpu_buffer_rsrc_t ra =
        make_rsrc(p.A + (b * p.strideA + m0 * p.lda) * ES, ((rows - 1) * p.lda + K) * ES);
    const __amdgpu_buffer_rsrc_t rb = make_rsrc(p.B + b * p.strideB * ES, ((N - 1) * p.ldb + K) * ES);
    const __amdgpu_buffer_rsrc_t rc =
        make_rsrc(reinterpret_cast<const char *>(p.C + b * p.strideC), ((M - 1) * p.ldc + N) * 4);

    // ---- issue the panel loads, then the first step's B loads ------------
    u32x4 pa[PU];
#pragma unroll
    for (int u = 0; u < PU; ++u) {
        const int q = tid + PNT * u, r = q / UPR, c = q % UPR;   // row, 16-byte unit
        const bool ok = r < rows && (int64_t)c * (16 / ES) < K && (!PART || q < PBM * UPR);
        pa[u] = bload(ra, ok ? (uint32_t)((r * p.lda) * ES + c * 16) : kOOB);
    }

    // B fragment of lane (fr, fg) at step s, column block j, chunk c:
    // column 128 s + 32 wave + 16 j + fr, k = 32 c + 8 fg .. + 7
    const int64_t all_steps = (N + PBN - 1) / PBN;
    const int s_begin = (int)(all_steps * cs / p.csplit);
    const int s_end = (int)(all_steps * (cs + 1) / p.csplit);
    // The panels of a batch entry walk their columns from different starts
    // (panel i from its i-th step, wrapping around): the workgroups running
    // at one time then write to many column ranges of C rather than all to
    // the same 512 bytes of every row (attention scores: bf16x3 1.2x, INT16
    // 1.07x faster).  The order of the steps changes no result.
    // the step across the end of a row of C whose length is not whole quads
    // comes last, with its own stores
    const bool edge = RAG && N % 4 != 0 && s_end == all_steps;
    const int cnt = s_end - s_begin - (edge ? 1 : 0);
    const int rot = cnt > 0 ? (int)(pid % cnt) : 0;
    auto step_of = [&](int t) {
        const int u = t + rot;
        return s_begin + (u >= cnt ? u - cnt : u);
    };
    u32x4 raw[TURN ? 1 : PD][2][KC][RQ];
    u32x4 line[TURN ? PD : 1][NBU];             // B in memory order
    char *const turn = smem + 2 * PPLANE + wave * TURN_BYTES;
    // unit c of row r of the area, rotated so that the 16 rows of a fragment
    // read fall in different bank groups
    auto turn_off = [](int r, int c) {
        const int x = c + r % UPR;
        return (r * UPR + (x >= UPR ? x - UPR : x)) * 16;
    };
    auto clamp = [&](int t) { return t < cnt ? t : (cnt > 0 ? cnt - 1 : 0); };
    auto load_b = [&](int set, int s) {
        if constexpr (TURN) {
#pragma unroll
            for (int u = 0; u < NBU; ++u) {
                const int q = u * 64 + lane, r = q / UPR, c = q % UPR;
                const int64_t n = (int64_t)s * PBN + wave * PWN + r;
                const bool ok = n < N && (int64_t)c * (16 / ES) < K;
                line[set][u] = bload(rb, ok ? (uint32_t)((n * p.ldb) * ES + c * 16) : kOOB);
            }
            return;
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int64_t n = (int64_t)s * PBN + wave * PWN + j * 16 + fr;
#pragma unroll
            for (int c = 0; c < KC; ++c) {
#pragma unroll
                for (int h = 0; h < RQ; ++h) {
                    const int k = 32 * c + 8 * fg + 4 * h;
                    const bool ok = n < N && k < K;
                    raw[set][j][c][h] = bload(rb, ok ? (uint32_t)((n * p.ldb + k) * ES) : kOOB);
                }
            }
        }
    };
#pragma unroll
    for (int d = 0; d < PD; ++d) {
        __builtin_amdgcn_sched_barrier(0);
        load_b(d, step_of(clamp(d)));
    }
    __builtin_amdgcn_sched_barrier(0);

    // ---- split the panel into LDS ----------------------------------------
#pragma unroll
    for (int u = 0; u < PU; ++u) {
        const int q = tid + PNT * u, r = q / UPR, c = q % UPR;
        if (PART && q >= PBM * UPR) break;
        if constexpr (SCORES) {
            u32x4 h, l;
            split8<true>(&pa[u], h, l);
            *reinterpret_cast<u32x4 *>(ph + panel_off(r, c)) = h;
            *reinterpret_cast<u32x4 *>(pl + panel_off(r, c)) = l;
        } else {
            // a quad: half of 16-byte chunk c / 2
            const f32x4 v = __builtin_bit_cast(f32x4, pa[u]);
            uint32_t h0, l0, h1, l1;
            split2(v.x, v.y, h0, l0);
            split2(v.z, v.w, h1, l1);
            const int off = panel_off(r, c >> 1) + 8 * (c & 1);
            u32x2 hv = {h0, h1}, lv = {l0, l1};
            *reinterpret_cast<u32x2 *>(ph + off) = hv;
            *reinterpret_cast<u32x2 *>(pl + off) = lv;
        }
    }
    __syncthreads();

    float scale = 1.0f;
    if constexpr (SCORES)
        // alpha (maxQ / 32767)(maxK / 32767) evaluated in FP64, rounded once
        scale = (float)((double)p.alpha * (double)*p.maxA * (double)*p.maxB / (32767.0 * 32767.0));
    else if constexpr (SCALE)
        scale = p.alpha;

    // ---- walk the columns of C -------------------------------------------
    // Step t splits register set t % PD and reloads it with step t + PD, so
    // each load has PD steps to arrive, and at least PD - 1 steps of stores
    // issued after it do not hold it up.  The loop runs whole groups of PD
    // steps (register sets are compile-time choices and every wait stays
    // exact); a step past the last one multiplies clamped copies and stores
    // nothing.
    auto step = [&](int set, int t, auto edge_tag) {
        constexpr bool EDGE = decltype(edge_tag)::value;
        const bool live = EDGE || t < cnt;
        const int s = EDGE ? (int)all_steps - 1 : step_of(clamp(t));
        u32x4 bh[2][KC], bl[2][KC];
        if constexpr (TURN) {
            // (one wave's own area: no barrier, only their order)
            wave_lds_order();
#pragma unroll
            for (int u = 0; u < NBU; ++u) {
                const int q = u * 64 + lane, r = q / UPR, c = q % UPR;
                *reinterpret_cast<u32x4 *>(turn + turn_off(r, c)) = line[set][u];
            }
            wave_lds_order();
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int c = 0; c < KC; ++c)
#pragma unroll
                    for (int h = 0; h < RQ; ++h)
                        raw[0][j][c][h] = *reinterpret_cast<const u32x4 *>(
                            turn + turn_off(16 * j + fr, (4 * c + fg) * RQ + h));
        }
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int c = 0; c < KC; ++c) split8<SCORES>(raw[TURN ? 0 : set][j][c], bh[j][c], bl[j][c]);
        // The reload goes into the registers just split (steps past the end
        // reload the last step: loads whose data is never used), after the
        // split: the scheduling barriers keep the compiler from hoisting
        // them into another register set, which it then copies back with a
        // wait for every outstanding store.
        __builtin_amdgcn_sched_barrier(0);
        if (!EDGE) load_b(set, step_of(clamp(t + PD)));
        __builtin_amdgcn_sched_barrier(0);

        // Row blocks one after another: the panel fragments of block i + 1
        // are read while block i is multiplied, and the block's two 16 x 16
        // results are stored as soon as their chains end, as two stores of
        // whole 128-byte lines.  The scheduling barriers keep the compiler
        // from hoisting every LDS read of the step to its top, which would
        // not fit the registers.
        u32x4 ah[KC], al[KC];
        auto read_a = [&](int i, u32x4 *h, u32x4 *l) {
#pragma unroll
            for (int c = 0; c < KC; ++c) {
                const int off = panel_off(16 * i + fr, 4 * c + fg);
                h[c] = *reinterpret_cast<const u32x4 *>(ph + off);
                l[c] = *reinterpret_cast<const u32x4 *>(pl + off);
            }
        };
        read_a(0, ah, al);
#pragma unroll
        for (int i = 0; i < PRB; ++i) {
            u32x4 nh[KC], nl[KC];
            if (i + 1 < PRB) read_a(i + 1, nh, nl);
            // both 16 x 16 results of the row block, then whole 128-byte
            // lines per store: one store holds rows 0..7 of the block, 32
            // columns each, the other rows 8..15
            f32x4 r[2];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                f32x4 a = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int c = 0; c < KC; ++c) {
                    a = mma<SCORES>(bh[j][c], ah[c], a);
                    a = mma<SCORES>(bl[j][c], ah[c], a);
                    a = mma<SCORES>(bh[j][c], al[c], a);
                    if constexpr (SCORES) a = mma<SCORES>(bl[j][c], al[c], a);
                }
                if (SCORES || SCALE) a = a * scale;   // FP32 C, no downcast
                r[j] = a;
            }
            f32x4 x, y;
            whole_lines(r[0], r[1], fr, x, y);
            {
                const int64_t mx = m0 + 16 * i + (fr & 7), my = mx + 8;
                const int64_t n = (int64_t)s * PBN + wave * PWN + 16 * (fr >> 3) + 4 * fg;
                const int64_t last = EDGE ? N - 4 : N - 1;   // last column a whole quad starts at
                const uint32_t ox = live && mx < M && n <= last ? (uint32_t)((mx * p.ldc + n) * 4) : kOOB;
                const uint32_t oy = live && my < M && n <= last ? (uint32_t)((my * p.ldc + n) * 4) : kOOB;
                constexpr int AUX = RAG ? HEAL_PANEL_RAG_AUX : HEAL_PANEL_STORE_AUX;
                const u32x4 xv = __builtin_bit_cast(u32x4, x), yv = __builtin_bit_cast(u32x4, y);
                __builtin_amdgcn_raw_buffer_store_b128(xv, rc, (int)ox, 0, AUX);
                __builtin_amdgcn_raw_buffer_store_b128(yv, rc, (int)oy, 0, AUX);
                if constexpr (EDGE) {
                    // the one to three columns past the last whole quad
#pragma unroll
                    for (int e = 0; e < 3; ++e) {
                        const bool in = n > last && n + e < N;
                        const uint32_t ex = in && mx < M ? (uint32_t)((mx * p.ldc + n + e) * 4) : kOOB;
                        const uint32_t ey = in && my < M ? (uint32_t)((my * p.ldc + n + e) * 4) : kOOB;
                        __builtin_amdgcn_raw_buffer_store_b32(xv[e], rc, (int)ex, 0, AUX);
                        __builtin_amdgcn_raw_buffer_store_b32(yv[e], rc, (int)ey, 0, AUX);
                    }
                }
            }
            if (i + 1 < PRB) {
#pragma unroll
                for (int c = 0; c < KC; ++c) {
                    ah[c] = nh[c];
                    al[c] = nl[c];
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    for (int t0 = 0; t0 < cnt; t0 += PD) {
#pragma unroll
        for (int d = 0; d < PD; ++d) step(d, t0 + d, std::false_type{});
    }
    if constexpr (RAG) {
        if (edge) {
            load_b(0, (int)all_steps - 1);
            step(0, 0, std::true_type{});
        }
    }
}

template <bool SCORES, bool SCALE, int PBM, bool RAG>
hipError_t launch_kc(const PanelArgs &a, hipStream_t stream)
{
    constexpr int PD = SCORES ? HEAL_PANEL_PD_SCORES : HEAL_PANEL_PD;
    const dim3 grid((unsigned)(a.batch * ((a.M + PBM - 1) / PBM) * a.csplit));
    const int kc = (int)((a.K + 31) / 32);
    switch (kc) {
    case 1: hipLaunchKernelGGL((gemm_panel_kernel<SCORES, SCALE, 1, PD, PBM, RAG>), grid, dim3(PNT), 0, stream, a); break;
    case 2: hipLaunchKernelGGL((gemm_panel_kernel<SCORES, SCALE, 2, PD, PBM, RAG>), grid, dim3(PNT), 0, stream, a); break;
    case 3: hipLaunchKernelGGL((gemm_panel_kernel<SCORES, SCALE, 3, PD, PBM, RAG>), grid, dim3(PNT), 0, stream, a); break;
    case 4: hipLaunchKernelGGL((gemm_panel_kernel<SCORES, SCALE, 4, PD, PBM, RAG>), grid, dim3(PNT), 0, stream, a); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// Whether rows of C are whole quads: with at least one full panel (256 rows of
// bf16x3, 128 of INT16 codes) such products have always run here.
bool whole_quads(int64_t N, const float *C, int64_t ldc, int64_t strideC, int64_t batch)
{
    return N % 4 == 0 && ldc % 4 == 0 && (batch == 1 || strideC % 4 == 0) &&
           (reinterpret_cast<uintptr_t>(C) & 15u) == 0;
}

// Steps of 128 columns over the panels of an output, of 128 rows from 65 rows on.
int64_t panel_steps(int64_t M, int64_t N, int64_t batch)
{
    return batch * (M <= 64 ? 1 : (M + 127) / 128) * ((N + PBN - 1) / PBN);
}

// Rows of the panel: the smallest that holds M up to 128.  Above, 128 for the scores;
// for bf16x3 256 where one panel holds M and the chip is full many times over (42
// of 137 x 7976 x 128 116 -> 101 us: B is read once), and for outputs of full panels
// in whole quads, else 128 (1.07x faster than 256 over random sizes).
int panel_rows(const PanelArgs &a, bool scores)
{
    const int64_t M = a.M;
    if (M <= 64) return M > 32 ? 64 : M > 16 ? 32 : 16;
    if (scores || M <= 128) return 128;
    if (M <= 256 && panel_steps(M, a.N, a.batch) >= 2048) return 256;
    return M >= 256 && whole_quads(a.N, a.C, a.ldc, a.strideC, a.batch) ? 256 : 128;
}

// Workgroups per panel, each walking its share of the columns.  Panels of at
// most 64 rows only read B: as many workgroups as there are steps, up to eight
// per CU in all (64 heads of 4 x 16384 x 128 INT16 54.9 us, 66.9 with half).
// Larger ones: at least two (above), and as many as make the fewest rounds
// of workgroups times the length of one, its columns in steps and one more step
// for its panel (8 heads of 2048 x 2048 x 128 bf16x3 56.4 us with two per panel,
// 38.9 with four; 32 heads of 1531 x 1531 x 128 INT16 128 with two, 115 with
// four).
int panel_csplit(int64_t M, int64_t N, int64_t batch, int PBM)
{
    const int64_t panels = batch * ((M + PBM - 1) / PBM), steps = (N + PBN - 1) / PBN;
    const int64_t cus = device_cus();
    if (PBM <= 64) {
        const int64_t c = (8 * cus + panels - 1) / panels;
        return (int)(c < steps ? c : steps);
    }
    const int64_t slots = PBM > 128 ? cus : 2 * cus;
    int best = 1;
    float least = 0.0f;
    auto consider = [&](int64_t c) {
        const float cost = (float)((panels * c + slots - 1) / slots) * ((float)steps / (float)c + 1.0f);
        if (least == 0.0f || cost < least) {
            least = cost;
            best = (int)c;
        }
    };
    for (int64_t c = steps < HEAL_PANEL_CSPLIT ? steps : HEAL_PANEL_CSPLIT; c <= steps && c <= 32; ++c) consider(c);
    // few panels and many columns: one round of as many workgroups as fit (142 x
    // 15076 x 128 bf16x3, one panel, 31.4 us with 32 workgroups)
    const int64_t one = slots / panels < steps ? slots / panels : steps;
    if (one > 32) consider(one);
    return best;
}

template <bool SCORES, bool SCALE>
hipError_t launch_panel(PanelArgs a, hipStream_t stream)
{
    // whole lines of C are streamed past the caches; rows of other lengths
    // leave half lines, which have to meet in L2
    const bool rag = a.N % 4 != 0 || a.ldc % 32 != 0 || a.strideC % 32 != 0 ||
                     (reinterpret_cast<uintptr_t>(a.C) & 127u) != 0;
    const int pbm = panel_rows(a, SCORES);
    a.csplit = panel_csplit(a.M, a.N, a.batch, pbm);
    switch (pbm) {
    case 16: return rag ? launch_kc<SCORES, SCALE, 16, true>(a, stream) : launch_kc<SCORES, SCALE, 16, false>(a, stream);
    case 32: return rag ? launch_kc<SCORES, SCALE, 32, true>(a, stream) : launch_kc<SCORES, SCALE, 32, false>(a, stream);
    case 64: return rag ? launch_kc<SCORES, SCALE, 64, true>(a, stream) : launch_kc<SCORES, SCALE, 64, false>(a, stream);
    case 128: return rag ? launch_kc<SCORES, SCALE, 128, true>(a, stream) : launch_kc<SCORES, SCALE, 128, false>(a, stream);
    case 256:
        if constexpr (!SCORES)
            return rag ? launch_kc<SCORES, SCALE, 256, true>(a, stream) : launch_kc<SCORES, SCALE, 256, false>(a, stream);
    }
    return hipErrorInvalidValue;
}

// Shape conditions shared by both products (es: bytes per operand element).
// K at most 128 and nonzero, whole 16-byte units along K (quads of FP32,
// eights of INT16), 16-byte rows of A and B, every byte offset a lane may
// address within a panel of A or a batch entry of B below 2^31, and one
// workgroup per (batch entry, panel, step) within the grid limit; C written
// with buffer stores, so a batch entry of C spans less than 2^31 bytes.  The
// rows of C may have any length and alignment.
bool panel_shape_ok(int64_t M, int64_t N, int64_t K, int64_t lda, int64_t ldb, int64_t ldc,
                    int64_t batch, int es)
{
    if (K <= 0 || K > PKMAX || (K * es) % 16 != 0 || N < 4) return false;
    const int64_t lim = 0x7fffffffLL;
    const int64_t rows = es == 2 ? 128 : 256;   // of the highest panel
    if (((M < rows ? M : rows) - 1) * lda * es + K * es >= lim) return false;
    if (((N - 1) * ldb + K) * es >= lim) return false;
    if (((M - 1) * ldc + N) * 4 >= lim) return false;
    // 2^21 16 x 16 blocks at most per launch: the grid stays below 2^31
    return batch * ((M + 15) / 16) * ((N + PBN - 1) / PBN) <= lim;
}

}  // namespace

bool panel_kernel_applies(const GemmArgs &a, bool trans_b)
{
    return trans_b && a.vecA && a.vecB &&
           panel_shape_ok(a.M, a.N, a.K, a.lda, a.ldb, a.ldc, a.batch, 4);
}

// The lines below lie where 4000 random products of each kind of 1 to 2048 rows, 4
// to 16384 columns, 1 to 256 entries and 4 to 128 deep cross over (us on the other
// kernels -> here).
bool panel_pays(const GemmArgs &a)
{
    const bool whole = whole_quads(a.N, a.C, a.ldc, a.strideC, a.batch);
    const int64_t steps = panel_steps(a.M, a.N, a.batch);
    // steps for most CUs, else the direct-B kernel's tiles spread it wider, the more so
    // the deeper (288 x 247 x 128 13.5 here, 4.3 on them; 115 of 126 x 267 x 128 15.8
    // here, 22.0; 1 x 82 x 8552 x 12 4.8 here, 9.0)
    if (a.M > 64)
        return (a.M >= 256 && whole) || a.K <= 32 || steps * 4 >= device_cus() * (a.K <= 96 ? 1 : 3);
    // one product: the skinny kernel's strips (9 x 3008 x 128 5.3 here, 3.8 on them),
    // but at most two chunks deep they are level or behind (7 x 4588 x 28 5.0 -> 3.3)
    if (a.batch == 1) return a.K <= 64 && (whole || a.M > 32);
    if (a.K <= 64 || a.M > 32) return true;     // (13 of 60 x 368 x 128 12.6 -> 6.7)
    // (rows of C in parts: up to 16 rows level, 17 to 32 1.16x faster here until C
    // fills the memory, 16 of 17 x 5794 x 128 13.1 -> 17.4)
    if (!whole) return a.M > 16 && steps < 512;
    // (32 of 2 x 352 x 128 6.7 -> 5.4, 5 of 24 x 4352 x 128 9.7 -> 7.0, 13 of 32 x 384 4.5 -> 5.9)
    return a.N >= PBN && steps >= (a.M <= 16 ? 64 : 96);
}

hipError_t launch_gemm_panel(const GemmArgs &g, bool use_alpha, hipStream_t stream)
{
    PanelArgs a = {};
    a.M = g.M;
    a.N = g.N;
    a.K = g.K;
    a.A = reinterpret_cast<const char *>(g.A);
    a.lda = g.lda;
    a.strideA = g.strideA;
    a.B = reinterpret_cast<const char *>(g.B);
    a.ldb = g.ldb;
    a.strideB = g.strideB;
    a.C = g.C;
    a.ldc = g.ldc;
    a.strideC = g.strideC;
    a.batch = g.batch;
    a.alpha = g.alpha;
    return use_alpha ? launch_panel<false, true>(a, stream) : launch_panel<false, false>(a, stream);
}

bool scores_panel_applies(const OpArgs &a)
{
    if (!a.vecA || !a.vecB || !panel_shape_ok(a.M, a.N, a.K, a.lda, a.ldb, a.ldc, a.batch, 2)) return false;
    const int64_t steps = panel_steps(a.M, a.N, a.batch);
    // as panel_pays: 17 to 64 rows more than two chunks deep from 40 steps on (2 of
    // 21 x 64 x 128 4.0 -> 5.0, 11 of 41 x 480 x 128 9.0 -> 5.8), and rows of C that
    // are not whole quads and shorter than a step from two chunks on, up to 128 of
    // them (19 of 105 x 18 x 128 7.2 -> 8.1; 32 of 1116 x 74 x 64 12.8 -> 8.9)
    if (a.M > 16 && a.M <= 64) return a.K <= 64 || steps >= 40;
    return a.M <= 64 || a.N >= 96 || a.K <= 32 || steps >= 128 || whole_quads(a.N, a.C, a.ldc, a.strideC, a.batch);
}

hipError_t launch_scores_panel(const OpArgs &o, hipStream_t stream)
{
    PanelArgs a = {};
    a.M = o.M;
    a.N = o.N;
    a.K = o.K;
    a.A = reinterpret_cast<const char *>(o.A);
    a.lda = o.lda;
    a.strideA = o.strideA;
    a.B = reinterpret_cast<const char *>(o.B);
    a.ldb = o.ldb;
    a.strideB = o.strideB;
    a.C = o.C;
    a.ldc = o.ldc;
    a.strideC = o.strideC;
    a.batch = o.batch;
    a.alpha = o.alpha;
    a.maxA = o.maxA;
    a.maxB = o.maxB;
    return launch_panel<true, false>(a, stream);
}

}  // namespace heal
