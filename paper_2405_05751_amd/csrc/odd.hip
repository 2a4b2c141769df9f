// The fused block in a 16-bit type at sizes that are no multiple of eight (a vocabulary of odd size, a
// hidden size of odd length), on the matrix cores: rows of W, X and Y that start at any element.
//
// It is the skinny kernel's scheme (a workgroup owns some columns and one K slab, lane (i, q) loads
// the 8 x 8 block W[kb + 8q ..][n0 + 8i ..] with eight 16-byte loads and v_perm picks the B operands out of
// that register block, X passes through the wave's corner of LDS, no barrier in the K loop), with these
// differences:
//   * W.  A buffer load needs a dword-aligned address.  With an even N every row starts on a dword.  With
//     an odd N every other row does not: the load of an odd row starts one element early, and the element
//     missing at its end is the next lane's first dword, fetched with one cross-lane move per odd row; the
//     shift itself costs nothing, it is another selector of the same v_perm.  Lane 15 of a row has no next
//     lane: the dwords it needs, 32 per 64 rows, come with one more load per run, through LDS (leaving that
//     lane's columns out, tiles of 120 instead of 128, measured 74 us at 24 x 4096 x 32003, with them 50).
//   * X.  The direct loads to LDS fetch 16-byte chunks of rows that start on 16 bytes.  With K % 8 != 0 X goes through
//     registers: a chunk is loaded from the dword it starts in, with one dword more, shifted by half a dword
//     where it starts in the middle of one, what lies behind K is zeroed, and the result is written to the same place.
//   * X (.) g enters the matrix cores as two operands, hi + lo, at every M: the kernel that ran these
//     sizes before kept the product in fp32.  hi is the product cut off (not rounded) one fp32 ulp below its
//     value, lo what is left: both have the product's sign and neither is zero unless the product is, so
//     that an infinite W gives what it gives in fp32.  In bf16 they are the product exactly (8 + 8 bits).
//     fp16 (11 + 11 bits) has no range to spare (products reach from 2^-48 to 2^32, operands from 2^-24 to
//     2^16), so a wave multiplies its rows' fp32 products by a power of two, and its sums by the inverse at the end.
//     The power puts the largest product of the wave's first 64 k between 2^3 and 2^4; the wave keeps track of the largest
//     of all, and where that one ends up outside 2^3 to 2^15 it goes over its runs once more with the power
//     that the row's products call for.  What is left out of a product is below 2^-24, scaled: less than the rounding of
//     the fp32 sums.  (A power found in a first kernel from the largest |x| times the largest |g| of a
//     row, and applied to X in fp16, cost what x lost as a subnormal: 6e-3 of the row's rms for a large
//     gain on a small x beside a large x on a small gain.  Sums that are scaled down whenever a larger product comes need
//     no second pass, but registers for it in every step: 136 of them spilled at 64 rows.)
//
// Bound by streaming W, like the skinny kernel.  24 x 4096 x 32003: bf16 50 us (264 MB, 5.2 TB/s), fp16 51 us (54 with
// the first kernel it had; but 256 x 4095 x 4099, where the vector instructions count, 59 us against 52, bf16 55 against 50);
// the plain kernel that ran these sizes before takes 2460 us.  Large M is bound by every row
// block's own copy of W out of L2: 2048 x 4096 x 4099 bf16 220 us (312 TFLOP/s), fp16 241 us.
#include <algorithm>
#include <type_traits>
#include "common.hpp"
#include "splitk.hpp"

namespace rmsnl {

constexpr int kOddFlags = 0x00020000;
constexpr int kOddOut = 0x7ffffff0;
constexpr int kOddWaves = 4;
constexpr int kOddTile = 128;                // columns of a tile
constexpr int odd_depth(int MB) { return MB == 1 ? 4 : 3; }           // 32-row steps of W in flight per wave

// ------------------------------------------------------------------------------------- the product
struct OddCold {                             // what the first loads do not need
    u16* Y;
    float eps, inv_K;
    int ldp;                                 // row length of the partial tiles: N rounded up to a multiple of 4
    float* ws_partial; float* ws_sumsq; unsigned* counter;
};

// SHIFT: K % 8 != 0, rows of X start anywhere.
template <typename T, int MB, bool ODDN, bool SHIFT>
__global__ __launch_bounds__(64 * kOddWaves) void odd_kernel(
    const u16* W, const u16* X, const u16* g, int M, int K, int N, int S, int n_tiles, int RB, OddCold a)
{
    constexpr int NW = kOddWaves, MT = 16 * MB, D = odd_depth(MB), N_TILE = kOddTile;
    extern __shared__ __align__(16) float smem[];   // red [NW][MT][N_TILE]; the stage buffers of X before that
    __shared__ float s_sumsq[NW][MT];
    __shared__ float s_rinv[MT];
    __shared__ int s_last;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int i = lane & 15, q = lane >> 4;

    // (tile, slab, row block) triples, the row block fastest: row blocks stream the same part of W, and neighbouring
    // tiles share the lines of W at their border (rows start anywhere), so they should share an XCD's L2
    const int total = n_tiles * S, b = xcd_run(blockIdx.x, total * RB);
    const int rb = b % RB, tile = b / RB / S, slab = b / RB % S;
    const int Mh = min(M - 64 * rb, 64);     // rows of this row block
    const u16* Xb = X + size_t(rb) * 64 * K;
    const int n0 = tile * N_TILE;
    const int runs = (K + 63) >> 6;          // 64-row runs of W; slab s takes runs [s R / S, (s + 1) R / S)
    const int run0 = int(int64_t(slab) * runs / S), run1 = int(int64_t(slab + 1) * runs / S);
    const int k0 = run0 * 64;
    const int klen = min(run1 * 64, K) - k0;
    const int nPairs = (run1 - run0 - wave + NW - 1) / NW;       // runs wave, wave + NW, ... of the slab

    // (an odd count of elements ends in the low half of a dword)
    const __amdgpu_buffer_rsrc_t wrs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<u16*>(W + size_t(k0) * N), 0, (klen * N * 2 + 3) & ~3, kOddFlags);
    const int wrow = N * 2, wpair = 64 * NW * N * 2;
    // a lane whose columns, and with odd N the column before them, lie outside reads zeros
    const unsigned woff0 = (ODDN ? n0 + 8 * i <= N : n0 + 8 * i < N)
                               ? unsigned(((wave * 64 + q * 16) * N + n0 + 8 * i) * 2) : 0x80000000u;

    const int r8 = lane >> 3, c8 = lane & 7;
    char* stage = reinterpret_cast<char*>(smem) + wave * (MT * N_TILE * 4);
    const int st_r0 = i * 128 + (((2 * q) ^ (i >> 1)) << 4);     // step 0 (+ 2048 mb); step 1 is ^ 16
    const int st_g = MT * 128;
    const int st_e = MT * 128 + 1024;
    constexpr int STG = MT * 128 + 1024 + 256;   // a run of X, the KiB that g's load writes, lane 15's dwords
    static_assert(2 * STG <= MT * N_TILE * 4, "two stage buffers fit the wave's part of the reduction buffer");
    const uint32_t stage_lds = __builtin_amdgcn_readfirstlane(uint32_t(uintptr_t(stage)));
    const uint4_t xdesc = {uint32_t(uintptr_t(Xb)), uint32_t(uintptr_t(Xb) >> 32), uint32_t((Mh * K * 2 + 3) & ~3), uint32_t(kOddFlags)};
    const uint4_t gdesc = {uint32_t(uintptr_t(g)), uint32_t(uintptr_t(g) >> 32), uint32_t((K * 2 + 3) & ~3), uint32_t(kOddFlags)};
    // the dword of column n0 + 128 of odd rows: lane l takes row 2l + 1 of the run
    const uint4_t wdesc = {uint32_t(uintptr_t(W + size_t(k0) * N)), uint32_t(uintptr_t(W + size_t(k0) * N) >> 32),
                           uint32_t((klen * N * 2 + 3) & ~3), uint32_t(kOddFlags)};
    const unsigned eoff0 = lane < 32 ? unsigned(((wave * 64 + 2 * lane + 1) * N + n0 + N_TILE - 1) * 2) : 0x80000000u;
    auto load_edge = [&](uint32_t dst, int v) {
        const uint4_t desc = wdesc;
        uint32_t keep;
        asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\t"
                     "buffer_load_dword %2, %3, 0 offen lds\n\ts_mov_b32 m0, %0"
                     : "=&s"(keep) : "s"(dst), "v"(v), "s"(desc) : "memory");
    };
    uint4_t w[D][8];
    const int rlim = Mh - r8, xlane = r8 * K * 2, xlast = (Mh - 1) * K * 2;
    const __amdgpu_buffer_rsrc_t xrs = __builtin_amdgcn_make_buffer_rsrc(const_cast<u16*>(Xb), 0, (Mh * K * 2 + 3) & ~3, kOddFlags);
    const __amdgpu_buffer_rsrc_t grs = __builtin_amdgcn_make_buffer_rsrc(const_cast<u16*>(g), 0, (K * 2 + 3) & ~3, kOddFlags);
    uint4_t xv[SHIFT ? 2 * MB : 1], gv;      // SHIFT: the next run's chunks on their way, from the dword they start in,
    uint32_t xn[SHIFT ? 2 * MB : 1];         // and the dword behind each
    auto chunk_k = [&](int krun, int j) { return krun + ((c8 ^ (r8 >> 1) ^ (4 * (j & 1))) << 3); };
    auto issue_x = [&](int t) {              // rows that do not exist: the last row again, never stored
        const uint32_t sb = stage_lds + uint32_t(t & 1) * STG;
        const int krun = (NW * t + wave) * 64;
        const int kg = krun + c8 * 8, go = (r8 == 0 && kg < klen) ? (k0 + kg) * 2 : kOddOut;
        if (ODDN) load_edge(sb + st_e, int(eoff0 + unsigned(t) * unsigned(wpair)));
        if (SHIFT) gv = __builtin_amdgcn_raw_buffer_load_b128(grs, go, 0, 0);
        else       load_lds(gdesc, sb + st_g, go);
#pragma unroll
        for (int j = 0; j < 2 * MB; ++j) {
            const int kr = chunk_k(krun, j);
            const int xo = kr < klen ? (k0 + kr) * 2 + (8 * j < rlim ? xlane + 8 * j * K * 2 : xlast) : kOddOut;
            if (SHIFT) {
                xv[j] = __builtin_amdgcn_raw_buffer_load_b128(xrs, xo & ~3, 0, 0);
                xn[j] = __builtin_amdgcn_raw_buffer_load_b32(xrs, int(unsigned(xo & ~3) + 16u), 0, 0);
            } else {
                load_lds(xdesc, sb + 1024 * j, xo);
            }
        }
    };
    auto stage_x = [&](int t) {              // SHIFT: the run that has arrived, to where the direct loads would have put it
        char* sb = stage + (t & 1) * STG;
        const int krun = (NW * t + wave) * 64;
        auto inside = [&](uint4_t v, int kr) {           // zeros from K on
            if (krun + 64 > klen)
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = kr + 2 * e + 1 < klen ? v[e] : kr + 2 * e < klen ? v[e] & 0xffffu : 0u;
            return v;
        };
        if (r8 == 0) *reinterpret_cast<uint4_t*>(sb + st_g + 16 * lane) = inside(gv, krun + c8 * 8);
#pragma unroll
        for (int j = 0; j < 2 * MB; ++j) {
            const int row = 8 * j < rlim ? 8 * j + r8 : Mh - 1;
            const uint32_t sh = uint32_t(row & K & 1) * 16u;             // k0 and kr are even
            const uint4_t v = {__builtin_amdgcn_alignbit(xv[j][1], xv[j][0], sh), __builtin_amdgcn_alignbit(xv[j][2], xv[j][1], sh),
                               __builtin_amdgcn_alignbit(xv[j][3], xv[j][2], sh), __builtin_amdgcn_alignbit(xn[j], xv[j][3], sh)};
            *reinterpret_cast<uint4_t*>(sb + 1024 * j + 16 * lane) = inside(v, chunk_k(krun, j));
        }
    };
    auto issue_w = [&](int s, int d) {
        const int t = s >> 1, h = s & 1;
#pragma unroll
        for (int j = 0; j < 8; ++j)          // odd N, odd row: one element early
            w[d][j] = __builtin_amdgcn_raw_buffer_load_b128(
                wrs, int(woff0 + unsigned(__builtin_amdgcn_readfirstlane(int(unsigned(t) * unsigned(wpair) + unsigned((8 * h + j) * wrow) -
                                                                             (ODDN && (j & 1) ? 2u : 0u))))), 0, 2);
    };
    float4_t acc[MB][8];
    float ss[MB];
    constexpr bool kScale = std::is_same<T, Fp16>::value;
    float top[MB], up[MB];                   // fp16: row i's largest product so far, and what its products are multiplied by
    // the power of two that puts v between 2^e and 2^(e + 1); v: a row's largest product, lanes i + 16 q
    auto power = [&](float v, int e) {
        v = fmaxf(v, __shfl_xor(v, 16, 64));
        v = fmaxf(v, __shfl_xor(v, 32, 64));
        return v > 0.f && v <= 3.0e38f ? __uint_as_float(uint32_t(254 + e) * 0x00800000u - (__float_as_uint(v) & 0x7f800000u)) : 64.f;
    };
    auto consume = [&](int d, int t, int h, const char* stg) {
        uint4_t ahi[MB], alo[MB];
        const uint4_t gq = *reinterpret_cast<const uint4_t*>(stg + st_g + ((2 * q + h) << 4));
        // (the sum with +0 turns -0 into +0)
        auto product = [&](const uint4_t& x, int e, int half) {
            return half ? __fmaf_rn(Elem<T>::hi(x[e]), Elem<T>::hi(gq[e]), 0.f) : __fmaf_rn(Elem<T>::lo(x[e]), Elem<T>::lo(gq[e]), 0.f);
        };
        uint4_t xq[MB];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) xq[mb] = *reinterpret_cast<const uint4_t*>(stg + ((st_r0 ^ (h << 4)) + 2048 * mb));
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float x0 = Elem<T>::lo(xq[mb][e]), x1 = Elem<T>::hi(xq[mb][e]);
                ss[mb] = __fmaf_rn(x0, x0, ss[mb]);
                ss[mb] = __fmaf_rn(x1, x1, ss[mb]);
                uint32_t hi, lo;
                const float p0 = product(xq[mb], e, 0), p1 = product(xq[mb], e, 1);
                if (kScale) top[mb] = fmaxf(fmaxf(top[mb], fabsf(p0)), fabsf(p1));
                TwoPart<T>::split(kScale ? p0 * up[mb] : p0, kScale ? p1 * up[mb] : p1, &hi, &lo);
                ahi[mb][e] = hi; alo[mb][e] = lo;
            }
        }
        uint32_t next[4];                    // odd N: dword 0 of the next lane's odd rows
        if (ODDN) {
            const uint4_t edge = *reinterpret_cast<const uint4_t*>(stg + st_e + ((2 * q + h) << 4));
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                // the first row past the end of an odd K starts in the dword of W's last element, and the other
                // half of that dword is not W's
                if (SHIFT && (NW * t + wave) * 64 + 16 * q + 8 * h + 2 * r + 1 >= klen) w[d][2 * r + 1][0] = 0;
                next[r] = uint32_t(__builtin_amdgcn_update_dpp(int(edge[r]), int(w[d][2 * r + 1][0]), 0x101 /* row_shl:1 */, 0xf, 0xf, false));
            }
        }
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            uint4_t bop;                     // column c: row 2r in the low halves, row 2r + 1 in the high halves
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const uint32_t even = w[d][2 * r][c >> 1];
                if (ODDN) {
                    const uint32_t odd = c == 7 ? next[r] : w[d][2 * r + 1][(c + 1) >> 1];
                    bop[r] = __builtin_amdgcn_perm(odd, even, (c & 1) ? 0x05040302u : 0x07060100u);
                } else {
                    bop[r] = __builtin_amdgcn_perm(w[d][2 * r + 1][c >> 1], even, (c & 1) ? 0x07060302u : 0x05040100u);
                }
            }
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) acc[mb][c] = Mfma16<T>::run(ahi[mb], bop, acc[mb][c]);
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) acc[mb][c] = Mfma16<T>::run(alo[mb], bop, acc[mb][c]);
        }
    };

    constexpr int PU = (D % 2 == 0) ? D / 2 : D;    // runs per trip: ring slots repeat every 2 PU steps
    for (int pass = 0;; ++pass) {
        // every load is issued whether or not its step exists, in this order: the waits count on it
        __builtin_amdgcn_sched_barrier(0);
        issue_w(0, 0);
        __builtin_amdgcn_sched_barrier(0);
        issue_x(0);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int d = 1; d < D; ++d) {
            issue_w(d, d);
            __builtin_amdgcn_sched_barrier(0);
        }
        asm volatile("" ::: "memory");

        if (kScale && pass == 0) {               // X of the first run is there once only the 16 youngest loads of W are not
            __builtin_amdgcn_s_waitcnt((16 & 15) | ((16 >> 4) << 14) | (7 << 4) | (15 << 8));
            asm volatile("" ::: "memory");
            if (SHIFT) stage_x(0);
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) {
                float v = 0.f;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const uint4_t gq = *reinterpret_cast<const uint4_t*>(stage + st_g + ((2 * q + h) << 4));
                    const uint4_t xq = *reinterpret_cast<const uint4_t*>(stage + ((st_r0 ^ (h << 4)) + 2048 * mb));
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        v = fmaxf(v, fmaxf(fabsf(Elem<T>::lo(xq[e]) * Elem<T>::lo(gq[e])), fabsf(Elem<T>::hi(xq[e]) * Elem<T>::hi(gq[e]))));
                }
                up[mb] = nPairs > 0 ? power(v, 3) : 64.f;
            }
        }
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            ss[mb] = top[mb] = 0.f;
#pragma unroll
            for (int c = 0; c < 8; ++c) acc[mb][c] = float4_t{0.f, 0.f, 0.f, 0.f};
        }
        for (int t0 = 0; t0 < nPairs; t0 += PU) {
#pragma unroll
            for (int p = 0; p < PU; ++p) {
                const int t = t0 + p;
                const bool there = t < nPairs;   // uniform over the wave; only the arithmetic is skipped
                const char* stg = stage + (t & 1) * STG;
                // this run's X was asked for a run ago; the 16 loads of W issued since are younger
                __builtin_amdgcn_s_waitcnt((16 & 15) | ((16 >> 4) << 14) | (7 << 4) | (15 << 8));
                asm volatile("" ::: "memory");
                __builtin_amdgcn_sched_barrier(0);
                if (SHIFT) {
                    stage_x(t);
                    asm volatile("" ::: "memory");
                    __builtin_amdgcn_sched_barrier(0);
                }
                issue_x(t + 1);
                asm volatile("" ::: "memory");
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    if (there) consume((2 * p + h) % D, t, h, stg);
                    __builtin_amdgcn_sched_barrier(0);
                    issue_w(2 * t + h + D, (2 * p + h) % D);
                    asm volatile("" ::: "memory");
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
        // loads for the run past the end still write into the stage buffers, which the reduction buffer covers
        __builtin_amdgcn_s_waitcnt(0 | (7 << 4) | (15 << 8));
        asm volatile("" ::: "memory");

        if (!kScale || pass == 1) break;
        bool again = false;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            const float v = top[mb] * up[mb];
            again |= v >= 32768.f && v <= 3.0e38f;           // (the lanes of a row need not agree: any of them will do)
            const float row = fmaxf(v, __shfl_xor(v, 16, 64)), all = fmaxf(row, __shfl_xor(row, 32, 64));
            again |= all > 0.f && all < 8.f;
        }
        if (!__any(again)) break;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) up[mb] = power(top[mb], 14);
    }
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {        // lanes i, i + 16, i + 32, i + 48 hold row i's shares
        float v = ss[mb];
        v += __shfl_xor(v, 16, 64);
        v += __shfl_xor(v, 32, 64);
        if (q == 0) s_sumsq[wave][mb * 16 + i] = v;
        if (kScale)                          // the rows' powers of two out of their sums
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float f = __shfl(1.f / up[mb], 4 * q + r, 64);         // lanes 0 .. 15 hold rows 0 .. 15
#pragma unroll
                for (int c = 0; c < 8; ++c) acc[mb][c][r] *= f;
            }
    }
    float* red = smem;                       // lane (i, q): rows 16mb + 4q + r, columns n0 + 8i + c
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            float4_t* dst = (float4_t*)(red + ((wave * MT) + mb * 16 + q * 4 + r) * N_TILE + i * 8);
            dst[0] = float4_t{acc[mb][0][r], acc[mb][1][r], acc[mb][2][r], acc[mb][3][r]};
            dst[1] = float4_t{acc[mb][4][r], acc[mb][5][r], acc[mb][6][r], acc[mb][7][r]};
        }
    __syncthreads();

    // every row block is a problem of its own to the epilogue
    TailArgs ta{a.Y + size_t(rb) * 64 * N, Mh, N, N_TILE, 0, 0, 0, a.eps, a.inv_K, S, nullptr, nullptr, nullptr, nullptr, 0,
                a.ldp};
    if (S > 1) {
        ta.ws_partial = a.ws_partial + size_t(rb) * S * 64 * a.ldp;
        ta.ws_sumsq = a.ws_sumsq + size_t(rb) * total * kSumsqStride;
        ta.counter = a.counter + size_t(rb) * n_tiles * kCounterStride;
    }
    splitk_tail<T, MT, N_TILE, true, NW, false, true>(ta, red, &s_sumsq[0][0], s_rinv, &s_last, tile, slab, n0);
}

// ------------------------------------------------------------------------------------------- host
struct OddPlan { int MB, RB, S, n_tiles, ldp; bool ok; size_t lds, bytes; const char* why; };

static OddPlan odd_plan(const Problem& p)
{
    OddPlan pl{};
    if (p.dt == F32 || !p.fused || p.gated) { pl.why = "the odd-size variant runs the fused block in the 16-bit types only"; return pl; }
    // a few dozen k and at most one plain workgroup to a place on the chip: nothing to stream, and the plain kernel's
    // single launch is ahead (1 x 64 x 1001 fp16: 8.9 us, 13.1 us here; at K = 128 12.8 and 13.4, at 300 26.6 and 12.4)
    if (!p.forced && p.K <= 96 && int64_t(p.M) * p.N <= (1 << 17)) { pl.why = "too small for the odd-size variant"; return pl; }
    if (p.K > (1 << 23) || p.N > (1 << 30)) { pl.why = "the odd-size variant needs K <= 2^23 and N <= 2^30"; return pl; }     // (64 rows of X below 2^31 bytes)
    pl.ldp = (p.N + 3) / 4 * 4;
    pl.n_tiles = (p.N + kOddTile - 1) / kOddTile;
    pl.RB = int((int64_t(p.M) + 63) / 64);
    pl.MB = pl.RB > 1 ? 4 : (p.M + 15) / 16;
    const int runs = (p.K + 63) / 64;
    const int Mb = std::min(p.M, 64);
    const int64_t blocks = int64_t(pl.n_tiles) * pl.RB;
    // byte offsets into a slab of W are 32-bit; the ring runs up to 2048 rows past its end
    auto slab_fits = [&](int s) { return (int64_t(64) * ((runs + s - 1) / s) + 2048) * p.N * 2 < (int64_t(1) << 31); };
    auto partial_bytes = [&](int s) { return s > 1 ? size_t(pl.RB) * s * Mb * pl.ldp * 4 : size_t(0); };
    // a split needs one run per wave, room for counters and sums of squares, and partials that fit the smallest
    // workspace there is, so that every entry point takes the same one
    auto may_split = [&](int s) {
        return int64_t(s) * kOddWaves <= runs && blocks <= kMaxCounters && blocks * s * kSumsqStride <= kMaxSumsqFloats &&
               partial_bytes(s) <= kScratchBytes - kHeadBytes;
    };
    // slabs: the skinny kernel's cost model (see skinny_plan, where its constants come from)
    if (p.n_tile != 0 && p.n_tile != kOddTile) { pl.why = "odd-size variant: tiles of 128 columns"; return pl; }
    if (p.k_split > 16) { pl.why = "odd-size variant: 1 to 16 slabs"; return pl; }
    double best = 0.;
    for (int s = std::max(1, p.k_split); s <= (p.k_split ? p.k_split : 16); ++s) {
        if (!slab_fits(s) || (s > 1 && (!may_split(s) || p.no_ws))) continue;
        const double wgs = double(blocks) * s;
        const double wg_bytes = 64.0 * ((runs + s - 1) / s) * (kOddTile * 2.0 + Mb * 2.0);
        const double hbm_us = double(p.K) * p.N * 2.0 / 6.5e6;
        const double unit_us = double((int64_t(wgs) + 255) / 256) * wg_bytes / 45.0e3;
        const double tail_us = s > 1 ? 2.0 + 0.05 * s + 0.35 * s * double(p.M) * p.N * 8.0 / 1.0e6 : 0.0;
        const double t = std::max(hbm_us, unit_us) + 0.15 * std::min(hbm_us, unit_us) + tail_us;
        if (pl.S == 0 || t < best) { best = t; pl.S = s; }
    }
    if (pl.S == 0) { pl.why = "the odd-size variant cannot split this W so, or not address a slab of it"; return pl; }
    if (blocks * pl.S >= (int64_t(1) << 24)) { pl.why = "too many workgroups"; return pl; }     // (a grid holds fewer than 2^32 threads)
    pl.lds = size_t(kOddWaves) * 16 * pl.MB * 128 * 4;
    pl.bytes = partial_bytes(pl.S);
    pl.ok = true;
    return pl;
}

size_t odd_workspace_bytes(const Problem& p)
{
    OddPlan pl = odd_plan(p);
    return pl.ok ? pl.bytes : 0;
}

template <typename T, int MB, bool ODDN, bool SHIFT>
static hipError_t odd_go(const Problem& p, const OddPlan& pl, const OddCold& c, hipStream_t s)
{
    static LdsOnce once;                                 // 128 KiB of dynamic LDS at MB = 4
    hipError_t e = raise_lds_once(once, {(const void*)odd_kernel<T, MB, ODDN, SHIFT>}, 144 * 1024);
    if (e != hipSuccess) return e;
    dim3 grid(unsigned(pl.n_tiles * pl.S * pl.RB));
    odd_kernel<T, MB, ODDN, SHIFT><<<grid, 64 * kOddWaves, pl.lds, s>>>((const u16*)p.W, (const u16*)p.X, (const u16*)p.g, p.M, p.K, p.N,
                                                                        pl.S, pl.n_tiles, pl.RB, c);
    return hipGetLastError();
}

template <typename T, bool ODDN, bool SHIFT>
static hipError_t odd_mb(const Problem& p, const OddPlan& pl, const OddCold& c, hipStream_t s)
{
    switch (pl.MB) {
    case 1:  return odd_go<T, 1, ODDN, SHIFT>(p, pl, c, s);
    case 2:  return odd_go<T, 2, ODDN, SHIFT>(p, pl, c, s);
    case 3:  return odd_go<T, 3, ODDN, SHIFT>(p, pl, c, s);
    default: return odd_go<T, 4, ODDN, SHIFT>(p, pl, c, s);
    }
}

template <typename T>
static hipError_t odd_types(const Problem& p, const OddPlan& pl, bool odd_n, const OddCold& c, hipStream_t s)
{
    if (p.K % 8) return odd_n ? odd_mb<T, true, true>(p, pl, c, s) : odd_mb<T, false, true>(p, pl, c, s);
    return odd_n ? odd_mb<T, true, false>(p, pl, c, s) : odd_mb<T, false, false>(p, pl, c, s);
}

hipError_t launch_odd(const Problem& p, hipStream_t s, const char** why)
{
    OddPlan pl = odd_plan(p);
    if (!pl.ok) { if (why) *why = pl.why; return hipErrorInvalidValue; }
    if (pl.bytes && !p.ws_partial) { if (why) *why = "the odd-size variant needs the workspace"; return hipErrorInvalidValue; }
    const OddCold c{(u16*)p.Y, p.eps, 1.0f / float(p.K), pl.ldp, p.ws_partial, p.ws_sumsq, p.ws_counter};
    if (p.plan) { p.plan[0] = kOddTile; p.plan[1] = pl.S; p.plan[2] = pl.n_tiles * pl.S * pl.RB; }
    const bool odd_n = (p.N & 1) != 0;
    if (p.dt == F16) return odd_types<Fp16>(p, pl, odd_n, c, s);
    return odd_types<Bf16>(p, pl, odd_n, c, s);
}

}  // namespace rmsnl
