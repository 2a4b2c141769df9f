// The fp32 path of the fused block on the matrix cores: the case study's Fig. 2b again -- A_i = sum_k X_ik^2 and
// B_in = sum_k (X_ik g_k) W_kn in one K loop, the division by the root mean square after it -- on 4-byte elements, sums in
// fp32.  Two kernels: the one described here (v_mfma_f32_16x16x4_f32, fp32 products), which runs every M, and further down one for
// larger problems with K from 64 to 16000, tiles of 64 or 128 rows x 128 columns through LDS on the bf16 matrix instructions, three
// bf16 numbers to an fp32 one (f32_tiles() has the rule).
//
// A workgroup (4 waves) owns 16 MB rows (MB = 1..4) x 64 columns of Y over one K slab; its waves
// take the slab's 16-row runs of W in turn.  fp32 matrix instructions are slow enough (64 flops
// per clock and SIMD) that operands straight from the caches keep them fed two thirds of the time: nothing is
// staged through LDS in this kernel's K loop.
//   W: lane (c, q) = (lane % 16, lane / 16) loads rows k + 4 q + t, t = 0..3, columns n0 + 4 c .. + 3:
//      four loads of 4 rows x 256 contiguous bytes;
//   X: the same lane loads row 16 mb + c, elements k + 4 q .. + 3 (and g's), 16 bytes;
//   step t feeds element t of the X registers and, for j = 0..3, element j of W load t into the
//   instruction for columns n0 + 4 c' + j: the k of a lane group is k + 4 q + t on both sides.
// Sums: a matrix accumulator takes 128 k (8 runs) and is then added into a second accumulator, and
// so are the squares, so that the rounding error grows with sqrt(128) + sqrt(K / 512) ulps and not
// with sqrt(K); the waves' tiles are added in LDS, K slabs through the workspace by the last
// workgroup to arrive, in slab order (the epilogue the 16-bit split-K kernels use).
// M > 64: a row block per 64 rows in the same launch; workgroups that read the same rows of X or
// columns of W are neighbours on one XCD.
#include <algorithm>
#include "splitk.hpp"

namespace rmsnl {

constexpr int kF32Tile = 64;          // columns of W per workgroup
constexpr int kF32Chunk = 8;          // runs per first-level accumulator
// runs in flight per wave: 3, and 4 from 33 rows on (a unit's loads are then the scarcer side: 2 runs measured
// 20 % slower than 3 at 64 rows, 4 another 3.5 % faster; with 1 to 16 rows 4 is no gain)
constexpr int f32_ring(int MB) { return MB >= 3 ? 4 : 3; }
constexpr int kF32Out = -16;          // as a byte offset 0xfffffff0, beyond every buffer resource: reads zero
constexpr int kF32Flags = 0x00020000;

struct F32Args {
    const float* X; const float* g; const float* W; float* Y;
    int M, K, N;
    float eps, inv_K;
    int k_slab, S, n_tiles, RB;       // rows of W per slab (a multiple of 64), slabs, column tiles, row blocks
    int H, G;                         // gated block: outputs (N = 2 H) and the layout of W, see gated_col()
    float* ws_partial; float* ws_sumsq; unsigned* counter;
};

// GATED (the GatedMLP block on top): the tile's first 32 columns are the gate columns of 32 outputs, the
// next 32 their up columns; the epilogue forms SiLU(gate) * up.  Only the column a lane fetches changes.
template <int MB, bool FUSED, bool GATED>
__global__ __launch_bounds__(256) void f32_kernel(F32Args a)
{
    constexpr int MT = 16 * MB, D = f32_ring(MB);
    extern __shared__ __attribute__((aligned(16))) float smem[];      // red [4][MT][64]
    __shared__ float s_sumsq[4][MT];
    __shared__ float s_rinv[MT];
    __shared__ int s_last;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, q = lane >> 4;

    // consecutive workgroups go to the 8 XCDs in turn: renumber so that an XCD sees a run of
    // consecutive numbers, and number the workgroups in panels of 4 column tiles, inside a panel the
    // tile fastest, then the row block, then the slab: the 32 workgroups an XCD runs together are
    // 8 row blocks x 4 column tiles, which share their rows of X and columns of W in its L2
    const int bid = xcd_run(blockIdx.x, gridDim.x);
    const int per_panel = 4 * a.RB * a.S;
    const int panel = bid / per_panel;
    int idx = bid - panel * per_panel;
    const int pw = min(4, a.n_tiles - 4 * panel);       // the last panel may be narrower
    const int tile = 4 * panel + idx % pw;
    idx /= pw;
    const int rb = idx % a.RB;
    const int slab = idx / a.RB;
    const int n0 = tile * (GATED ? kF32Tile / 2 : kF32Tile), m0 = rb * 64;   // gated: first output of the tile
    const int Mh = min(a.M - m0, 64);                   // rows of this row block
    const int k0 = slab * a.k_slab, Kend = min(a.K, k0 + a.k_slab);
    const int nIter = (Kend - k0 + 63) >> 6;            // uniform: runs per wave

    const __amdgpu_buffer_rsrc_t xrs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float*>(a.X + size_t(m0) * a.K), 0, int(unsigned(Mh) * unsigned(a.K) * 4u), kF32Flags);
    const __amdgpu_buffer_rsrc_t grs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float*>(FUSED ? a.g : a.X), 0, a.K * 4, kF32Flags);
    const __amdgpu_buffer_rsrc_t wrs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float*>(a.W), 0, int(unsigned(Kend) * unsigned(a.N) * 4u), kF32Flags);
    // N % 4 == 0 (gated: H % 4 == 0): a lane's four columns lie inside together, next to each other in W
    const bool up = GATED && 4 * c >= kF32Tile / 2;
    const int hcol = n0 + (up ? 4 * c - kF32Tile / 2 : 4 * c);
    const bool col_ok = hcol < (GATED ? a.H : a.N);
    const int wcol = GATED ? gated_col(hcol, up, a.H, a.G) : hcol;
    unsigned xrow[MB];                                  // byte offset of the lane's row inside the row block
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) xrow[mb] = unsigned(16 * mb + c) * unsigned(a.K) * 4u;

    float4_t wv[D][4], xv[D][MB], gv[D];
    // Every load is issued whether or not its run exists (k at or beyond the slab's end: the
    // offset that reads zero, at no memory traffic), in a pinned order, so that the compiler can
    // count the loads younger than the one it waits for.
    auto issue = [&](int it, int r) {
        const int kk = k0 + 64 * it + 16 * wave + 4 * q;
        const bool kin = kk < Kend;                     // K % 4 == 0: the lane's four k lie inside together
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const unsigned off = (unsigned(kk + t) * unsigned(a.N) + unsigned(wcol)) * 4u;
            wv[r][t] = __builtin_bit_cast(float4_t, __builtin_amdgcn_raw_buffer_load_b128(
                wrs, kin && col_ok ? int(off) : kF32Out, 0, 0));
        }
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
            xv[r][mb] = __builtin_bit_cast(float4_t, __builtin_amdgcn_raw_buffer_load_b128(
                xrs, kin ? int(xrow[mb] + unsigned(kk) * 4u) : kF32Out, 0, 0));
        if (FUSED)
            gv[r] = __builtin_bit_cast(float4_t, __builtin_amdgcn_raw_buffer_load_b128(grs, kin ? kk * 4 : kF32Out, 0, 0));
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };

    float4_t acc[MB][4], tot[MB][4];
    float ss[MB], ss_tot[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
        ss[mb] = ss_tot[mb] = 0.f;
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[mb][j] = tot[mb][j] = float4_t{0.f, 0.f, 0.f, 0.f};
    }
    auto fold = [&]() {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            ss_tot[mb] += ss[mb];
            ss[mb] = 0.f;
#pragma unroll
            for (int j = 0; j < 4; ++j) { tot[mb][j] += acc[mb][j]; acc[mb][j] = float4_t{0.f, 0.f, 0.f, 0.f}; }
        }
    };
    auto consume = [&](int r) {
        float4_t xh[MB];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            const float4_t x = xv[r][mb];
            if (FUSED) {
#pragma unroll
                for (int t = 0; t < 4; ++t) ss[mb] = __fmaf_rn(x[t], x[t], ss[mb]);
                xh[mb] = x * gv[r];
            } else {
                xh[mb] = x;
            }
        }
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int mb = 0; mb < MB; ++mb)
                    acc[mb][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(xh[mb][t], wv[r][t][j], acc[mb][j], 0, 0, 0);
    };

#pragma unroll
    for (int r = 0; r < D; ++r) issue(r, r);
    int in_chunk = 0;
    for (int i0 = 0; i0 < nIter; i0 += D) {
#pragma unroll
        for (int r = 0; r < D; ++r) {
            if (i0 + r < nIter) {                       // uniform; only the arithmetic is skipped
                consume(r);
                if (++in_chunk == kF32Chunk) { fold(); in_chunk = 0; }
            }
            issue(i0 + r + D, r);
        }
    }
    fold();

    // ---- A_i: add the four k groups of the wave (lanes c, c + 16, c + 32, c + 48 hold row c's shares)
    if (FUSED) {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            float v = ss_tot[mb];
            v += __shfl_xor(v, 16, 64);
            v += __shfl_xor(v, 32, 64);
            if (q == 0) s_sumsq[wave][mb * 16 + c] = v;
        }
    }
    // ---- B: element i of accumulator (mb, j) is row 16 mb + 4 q + i, column 4 c + j of the tile
    float* red = smem;                                  // [4][MT][64]
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int i = 0; i < 4; ++i)
            *(float4_t*)(red + (wave * MT + mb * 16 + q * 4 + i) * kF32Tile + 4 * c) =
                float4_t{tot[mb][0][i], tot[mb][1][i], tot[mb][2][i], tot[mb][3][i]};
    __syncthreads();

    // every row block is a problem of its own to the epilogue: its rows of Y, its share of the workspace
    TailArgs ta{(u16*)(a.Y + size_t(m0) * (GATED ? a.H : a.N)), Mh, a.N, kF32Tile, GATED ? kF32Tile / 2 : 0, a.H, a.G,
                a.eps, a.inv_K, a.S,
                a.ws_partial ? a.ws_partial + size_t(rb) * a.S * 64 * a.N : nullptr,
                a.ws_sumsq ? a.ws_sumsq + size_t(rb) * a.n_tiles * a.S * kSumsqStride : nullptr,
                a.counter ? a.counter + size_t(rb) * a.n_tiles * kCounterStride : nullptr, nullptr, 0};
    splitk_tail<float, MT, kF32Tile, FUSED, 4, GATED>(ta, red, &s_sumsq[0][0], s_rinv, &s_last, tile, slab, n0);
}

// ---- large problems: tiles of 128 columns on the bf16 matrix cores
// The fp32 matrix instructions run at 1/16 of the bf16 rate (and the kernel above keeps them busy 65 % of the time).  A finite
// fp32 number is the sum of three bf16 numbers, its value rounded to bf16, the remainder rounded, and what is left, each exact; the
// product of two such sums is nine products, exact in fp32, of which the three smallest are left out (BF16x3 of Henry, Tang and
// Heinecke, ARITH 2019).  Six v_mfma_f32_32x32x16_bf16 then stand for eight v_mfma_f32_32x32x2_f32 of four times the time each.
// What is left out is at most 2^-24 of the product, one rounding of it (1 + 2^-8 - 2^-17 times itself), 2^-27.4 in the root mean square of
// random numbers.  It does not show beside the rounding of the sums: with the two larger ones of the three in, errors are the same
// within 1 % (2048 x 4096 x 4096, N(0, 1): 1.77e-7 either way) or larger, since each is one more rounding of the sum, at 14 % more time.
// What must hold: the remainders are no denormals (both operands are scaled by 2^24, the sums back, so that this
// holds down to the smallest fp32 numbers), and everything is finite (sums that are not are taken again in fp32, see below).
//
// X (.) g (formed in fp32) and W come through registers, two K tiles of 32 ahead: split there, and written to LDS as three bf16
// planes each, in two buffers.  8 waves in two groups; a group takes 16 of the 32 k, a wave 32 TM x 64 of the tile.  Scaling and
// splitting is vector work for the next K tile between the matrix instructions of this one.
// Sums: a matrix accumulator takes 64 k of its group (128 of the tile) and is then added into a second one, by the two waves of
// a SIMD at different times; with 64 rows the second one goes into a third after 1024 k of the tile.  128 rows have no registers for
// that, and so run up to K = 4096 only.  Of a step's six products the small ones come first.  Relative error against fp64
// on N(0, 1), 2-norm, here (128 rows; 64) and in the kernel above:
//   K = 64: 0.93e-7, 1.02e-7; 192: 1.21e-7, 1.44e-7; 1000: 1.43e-7, 2.15e-7; 4096: 1.77e-7; 1.58e-7, 2.22e-7; 8192: 1.74e-7, 2.28e-7; 16000: 2.0e-7, 2.40e-7
// (128 x 128 tiles on fp32 instructions: 1.27e-7 at 192, 1.44e-7 at 1000, 1.92e-7 at 4096; two accumulators at K = 16000: 2.7e-7, the largest
// error 2.4e-6 of the rms against 1.2e-6 with three and 1.4e-6 above, and 1.4e-7 against 0.8e-7 for sums of positive terms; adding into the second
// one twice as often: 2.0e-7 at 4096).  Six roundings of a sum for 16 k and not one a k: less error where terms cancel, more where sums
// are nearly exact: rows with one entry 6.6e-8 against 6.2e-8; |N(0, 1)| 8.1e-8 against 7.8e-8 (128 x 128) at K = 192, 7.2e-8 against 7.5e-8
// (64 rows) at 4096; all entries +-(1 + 2^-8 - 2^-17) times powers of two 1.3e-7 against 0.9e-7.
// 2048 x 4096 x 4096: 590-612 us on fp32 instructions, 364-378 here, 182-189 TFLOP/s (fp32 peak: 157). Parts left out: loads 55 us,
// splitting 49, second accumulator 20.  Counters: the matrix pipes are busy 52 % of the cycles at 2.0 GHz, and the vector instructions, 84 M
// of them, would take 44 % by themselves; where they stand between the matrix instructions is worth 1 %.
constexpr int kFtN = 128, kFtK = 32, kFtMinK = 64, kFtMaxK = 16000, kFtMaxK2 = 4096;        // (g in LDS; of 128 rows)
constexpr unsigned kFtOut = 0x80000000u;     // beyond every resource (sizes below 2^31), with any tile offset added
constexpr float kFtScale = 0x1p24f;
constexpr int ft_buf(int TM) { return 3 * (64 * TM + kFtN) * kFtK; }          // elements of a buffer

// n times a matrix instruction and v vector instructions behind it
#define RL_F32_MIX(n, v) \
    _Pragma("unroll") for (int mix = 0; mix < n; ++mix) { \
        __builtin_amdgcn_sched_group_barrier(0x8, 1, 0); \
        __builtin_amdgcn_sched_group_barrier(0x2, v, 0); \
    }

// four numbers, scaled, as three times four bf16 numbers
__device__ __forceinline__ void f32_split(float4_t v, uint2_t (&part)[3]) {
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] *= kFtScale;
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const uint32_t p = Elem<Bf16>::pack(v[2 * e], v[2 * e + 1]);
            part[q][e] = p;
            if (q < 2) {
                v[2 * e] -= Elem<Bf16>::lo(p);
                v[2 * e + 1] -= Elem<Bf16>::hi(p);
            }
        }
}

// TM: matrix tiles of 32 rows per wave, tiles of 64 TM rows
template <int TM>
__global__ __launch_bounds__(512, 2) void f32_tile_kernel(const float* X, const float* g, const float* W, float* Y,
                                                          int M, int K, int N, int tiles_m, int tiles_n, float eps, float inv_K)
{
    constexpr int BM = 64 * TM, BN = kFtN, BK = kFtK, BUF = ft_buf(TM);
    extern __shared__ __attribute__((aligned(16))) float smem[];
    u16* planes = (u16*)smem;                // [2]{ X-hat [3][BM][BK], W [3][BK][BN] }, see below
    float* gs = smem + BUF;               // g, K rounded up to a multiple of 4 BK (and one more tile), zeros behind it
    __shared__ __attribute__((aligned(16))) float s_ss[BM];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kg = wave >> 2, wm = (wave >> 1) & 1, wn = wave & 1;

    // panels of up to 8 tile rows, column by column (see mid.hip)
    const int l = xcd_run(blockIdx.x, gridDim.x);
    const int panel = l / (8 * tiles_n), in = l - panel * 8 * tiles_n, rows = min(8, tiles_m - 8 * panel);
    const int m0 = (8 * panel + in % rows) * BM, n0 = in / rows * BN;

    const __amdgpu_buffer_rsrc_t xrs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(X + size_t(m0) * K), 0, min(BM, M - m0) * K * 4, kF32Flags);
    const __amdgpu_buffer_rsrc_t wrs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(W), 0, K * N * 4, kF32Flags);
    // a wave's load of X is 8 rows of 128 bytes, of W 2 rows of 512
    // (64 rows, 16 rows further on for the second one)
    const int xrow = 8 * wave + (lane >> 3), xk = 4 * (lane & 7), wrow = 2 * wave + (lane >> 5), wcol = 4 * (lane & 31);
    const unsigned xoff = unsigned(xrow * K + xk) * 4u;                  // (rows beyond M lie beyond the resource)
    const unsigned woff = n0 + wcol < N ? unsigned(wrow * N + n0 + wcol) * 4u : kFtOut;
    // where they go.  X-hat: rows of 64 bytes, 16-byte chunk c of row r at c ^ ((r / 4) & 3); W: rows of 256 bytes, chunk c of row r at c ^ 4 (r & 3)
    u16* const xst = planes + xrow * BK + 8 * ((xk >> 3) ^ ((xrow >> 2) & 3)) + (xk & 4);
    u16* const wst = planes + 3 * BM * BK + wrow * BN + ((wcol & ~7) ^ (32 * (wrow & 3))) + (wcol & 4);
    float4_t xr[2][TM], wr[2][2];             // [set]: two K tiles on their way
    auto load_tile = [&](auto set, int t) {  // past K: zeros
        constexpr int st = decltype(set)::value;
        const unsigned k0 = unsigned(t * BK);
        const unsigned xo = int(k0) + xk < K ? xoff + k0 * 4u : kFtOut, wo = woff + k0 * unsigned(N) * 4u;
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            if (p < TM) xr[st][p] = __builtin_bit_cast(float4_t, __builtin_amdgcn_raw_buffer_load_b128(xrs, int(xo + unsigned(p * 64 * K) * 4u), 0, 0));
            wr[st][p] = __builtin_bit_cast(float4_t, __builtin_amdgcn_raw_buffer_load_b128(wrs, int(wo + unsigned(p * 16 * N) * 4u), 0, 0));
        }
    };
    float ss[TM] = {}, ss_tot[TM] = {};      // squares of this thread's rows
    auto store_x = [&](auto set, int buf, int p, float4_t gv) {
        constexpr int st = decltype(set)::value;
        const float4_t x = xr[st][p];
#pragma unroll
        for (int e = 0; e < 4; ++e) ss[p] = __fmaf_rn(x[e], x[e], ss[p]);
        uint2_t part[3];
        f32_split(x * gv, part);
#pragma unroll
        for (int q = 0; q < 3; ++q) *(uint2_t*)(xst + buf * BUF + q * BM * BK + p * 64 * BK) = part[q];
    };
    auto store_w = [&](auto set, int buf, int p) {
        constexpr int st = decltype(set)::value;
        uint2_t part[3];
        f32_split(wr[st][p], part);
#pragma unroll
        for (int q = 0; q < 3; ++q) *(uint2_t*)(wst + buf * BUF + q * BK * BN + p * 16 * BN) = part[q];
    };

    const int h = lane >> 5, c = lane & 31;
    const int a_row = wm * 32 * TM + c, a_off = a_row * BK + 8 * ((2 * kg + h) ^ ((a_row >> 2) & 3));
    const int blk = lane >> 4, jj = lane & 15, b_row = 16 * kg + 8 * h + (jj >> 2);
    const int b_off = 3 * BM * BK + b_row * BN + ((wn * 64 + 16 * (blk & 1)) ^ (32 * (b_row & 3))) + 4 * (jj & 3);
    float16_t acc[TM][2], tot[TM][2];
    auto clear = [&](float16_t (&v)[TM][2]) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) v[i][j][r] = 0.f;
    };
    auto fold = [&]() {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) tot[i][j][r] += acc[i][j][r];
    };
    float16_t top[2];                        // 64 rows: the third accumulator
    auto raise = [&]() {
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) { top[j][r] += tot[0][j][r]; tot[0][j][r] = 0.f; }
    };
    const std::integral_constant<int, 0> even;
    const std::integral_constant<int, 1> odd;
    // iteration t: products of K tile t out of buffer t % 2, K tile t + 1 into the other one, loads of K tile t + 3
    auto iteration = [&](auto other, int t, bool first) {
        constexpr int ob = decltype(other)::value, buf = ob ^ 1;
        __syncthreads();
        const u16* pl = planes + buf * BUF;
        uint4_t af[3][TM], bf[3][2];
        auto read_a = [&](int q) {
#pragma unroll
            for (int i = 0; i < TM; ++i) af[q][i] = *(const uint4_t*)(pl + q * BM * BK + a_off + i * 32 * BK);
        };
        auto read_b = [&](int q) {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const u16* Bb = pl + q * BK * BN + (b_off ^ (32 * j));
                const uint2_t lo = lds_read_tr(Bb), hi = lds_read_tr(Bb + 4 * BN);
                bf[q][j] = uint4_t{lo[0], lo[1], hi[0], hi[1]};
            }
        };
        auto product = [&](int qa, int qb, bool zero) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, af[qa][i]), __builtin_bit_cast(bf16x8_t, bf[qb][j]),
                                                                        zero ? float16_t{} : acc[i][j], 0, 0, 0);
        };
        // the small products first; the vector work for the next K tile between the matrix instructions
        __builtin_amdgcn_sched_barrier(0);
        const float4_t gv = *(const float4_t*)(gs + (t + 1) * BK + xk);
        read_b(0); read_a(2); read_a(0); read_b(2);
        __builtin_amdgcn_sched_barrier(0);
        store_x(other, ob, 0, gv);
        if (first) product(2, 0, true); else product(2, 0, false);
        read_a(1); read_b(1);
        product(0, 2, false);
        RL_F32_MIX(2 * TM, 8);
        __builtin_amdgcn_sched_barrier(0);
        if (TM == 2) store_x(other, ob, TM - 1, gv);
        product(1, 1, false);
        RL_F32_MIX(2 * TM, 8);
        __builtin_amdgcn_sched_barrier(0);
        store_w(other, ob, 0);
        product(1, 0, false);
        RL_F32_MIX(2 * TM, 8);
        __builtin_amdgcn_sched_barrier(0);
        store_w(other, ob, 1);
        product(0, 1, false);
        RL_F32_MIX(2 * TM, 8);
        __builtin_amdgcn_sched_barrier(0);
        load_tile(other, t + 3);
        product(0, 0, false);
        __builtin_amdgcn_sched_barrier(0);
    };
    clear(acc);
    clear(tot);
    if (TM == 1)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) top[j][r] = 0.f;
    load_tile(even, 0);
    load_tile(odd, 1);
    for (int k = tid; k < (K + 4 * BK - 1) / (4 * BK) * (4 * BK) + BK; k += 512) gs[k] = k < K ? g[k] : 0.f;
    __syncthreads();
#pragma unroll
    for (int p = 0; p < 2; ++p) { if (p < TM) store_x(even, 0, p, *(const float4_t*)(gs + xk)); store_w(even, 0, p); }
    load_tile(even, 2);
    const int nk = (K + BK - 1) / BK;
    for (int t = 0; t < nk; t += 4) {        // (K tiles past the last one are zeros)
        iteration(odd, t, kg == 0);
        iteration(even, t + 1, false);
        if (kg == 1) fold();                 // (the two waves of a SIMD in turn)
        iteration(odd, t + 2, kg == 1);
        iteration(even, t + 3, false);
        if (kg == 0) fold();
#pragma unroll
        for (int p = 0; p < TM; ++p) { ss_tot[p] += ss[p]; ss[p] = 0.f; }
        if (TM == 1 && (t & 28) == 28) raise();
    }
    if (kg == 1) fold();
    if (TM == 1) {
        raise();
        tot[0][0] = top[0];
        tot[0][1] = top[1];
    }
    bool inf = false;
#pragma unroll
    for (int p = 0; p < TM; ++p) {
        float v = ss_tot[p];
#pragma unroll
        for (int o = 1; o < 8; o <<= 1) v += __shfl_xor(v, o, 64);
        if ((lane & 7) == 0) s_ss[8 * (wave + 8 * p) + (lane >> 3)] = v;
        inf |= v == INFINITY;
    }
    // A row of X with a NaN in it has NaN squares and gives NaN whatever its sums are.  So does one with an infinity (the sums are not
    // finite, the row's factor is zero), but its squares are infinite, as they are where they overflow: such rows are read again.
    if (__syncthreads_or(inf)) {
        for (int r = wave; r < BM; r += 8) {
            if (s_ss[r] != INFINITY) continue;
            float nan = 0.f;
            for (int k = 4 * lane; k < K; k += 256) {
                const float4_t x = __builtin_bit_cast(float4_t, __builtin_amdgcn_raw_buffer_load_b128(xrs, (r * K + k) * 4, 0, 0));
#pragma unroll
                for (int e = 0; e < 4; ++e) nan = __fmaf_rn(x[e], 0.f, nan);
            }
            if (__any(nan != 0.f) && lane == 0) s_ss[r] = NAN;
        }
        __syncthreads();
    }
    // An infinity is no sum of bf16 numbers (its remainder is NaN), and what is scaled may overflow: the sums that are not
    // finite, of rows that are, are taken again, over the same k, on the fp32 matrix instructions, operands straight from memory
    // one step of 16 k ahead (2048 x 1024 x 4096, W of 1e34: 235 us, 323 with every step waiting for its own; a NaN or an infinity in
    // every 64th row of X 103 and 108, 330 when those rows' sums were taken again too; everything finite 103)
    float nan = 0.f;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float4_t ss4 = *(const float4_t*)(s_ss + wm * 32 * TM + i * 32 + 8 * q + 4 * h);
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int j = 0; j < 2; ++j) nan = __fmaf_rn(ss4[e] == ss4[e] ? tot[i][j][4 * q + e] : 0.f, 0.f, nan);
        }
    const bool again = __syncthreads_or(nan != 0.f);     // (NaN != 0)
    float16_t sum[TM][2];
    clear(sum);
    float4_t xa[2][TM];
    float wa[2][4][2];
    unsigned wa_off[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) wa_off[j] = n0 + wn * 64 + j * 32 + c < N ? unsigned(n0 + wn * 64 + j * 32 + c) * 4u : kFtOut;
    auto fetch = [&](auto set, int n) {      // this group's eight of the 16 k of step n; past K: zeros (W's lie beyond its resource)
        constexpr int st = decltype(set)::value;
        const int k = BK * (n >> 1) + 16 * kg + 8 * (n & 1) + 4 * h;
        const unsigned xo = unsigned(a_row * K + k) * 4u, wo = unsigned(k * N) * 4u;
#pragma unroll
        for (int i = 0; i < TM; ++i)
            xa[st][i] = __builtin_bit_cast(float4_t, __builtin_amdgcn_raw_buffer_load_b128(
                xrs, int(k < K ? xo + unsigned(32 * i * K) * 4u : kFtOut), 0, 0));
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int j = 0; j < 2; ++j)
                wa[st][e][j] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                    wrs, int(wa_off[j] + wo + unsigned(e * N) * 4u), 0, 0));
    };
    auto step = [&](auto set, int n) {
        constexpr int st = decltype(set)::value;
        const float4_t gv = *(const float4_t*)(gs + BK * (n >> 1) + 16 * kg + 8 * (n & 1) + 4 * h);
        float4_t xh[TM];
#pragma unroll
        for (int i = 0; i < TM; ++i) xh[i] = xa[st][i] * gv;
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(xh[i][e], wa[st][e][j], acc[i][j], 0, 0, 0);
    };
    if (again) fetch(even, 0);
    for (int n = 0; again && n < 2 * nk; n += 8) {
        clear(acc);
#pragma unroll 1
        for (int u = n; u < n + 8; u += 2) {
            fetch(odd, u + 1);
            __builtin_amdgcn_sched_barrier(0);
            step(even, u);
            __builtin_amdgcn_sched_barrier(0);
            fetch(even, u + 2);
            __builtin_amdgcn_sched_barrier(0);
            step(odd, u + 1);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) sum[i][j][r] += acc[i][j][r];
    }
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float v = tot[i][j][r];
                tot[i][j][r] = !again || v - v == 0.f ? v * (1.f / (kFtScale * kFtScale)) : sum[i][j][r];
            }
    // the groups' sums meet in LDS: group 0 finishes accumulator registers 0 .. 7, group 1 registers 8 .. 15
    float* mine = smem + wave * 2 * TM * 8 * 64 + lane;
    const float* theirs = smem + (wave ^ 4) * 2 * TM * 8 * 64 + lane;
    auto give = [&](auto first) {
        constexpr int r0 = decltype(first)::value;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int r = 0; r < 8; ++r) mine[((i * 2 + j) * 8 + r) * 64] = tot[i][j][r0 + r];
    };
    auto finish = [&](auto first) {
        constexpr int r0 = decltype(first)::value;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                // register r is row 8 (r / 4) + 4 (lane / 32) + r % 4, column lane % 32 of its matrix tile
                const int row = wm * 32 * TM + i * 32 + 2 * r0 + 8 * (r >> 2) + 4 * h + (r & 3);
                const float ri = row_scale(s_ss[row], inv_K, eps);
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const int col = n0 + wn * 64 + j * 32 + c;
                    const float y = (tot[i][j][r0 + r] + theirs[((i * 2 + j) * 8 + r) * 64]) * ri;
                    if (m0 + row < M && col < N) __builtin_nontemporal_store(y, Y + size_t(m0 + row) * N + col);
                }
            }
    };
    const std::integral_constant<int, 0> low;
    const std::integral_constant<int, 8> high;
    if (kg == 0) give(high); else give(low);
    __syncthreads();
    if (kg == 0) finish(low); else finish(high);
}

static size_t f32_tile_lds(int TM, int K) { return size_t(2) * ft_buf(TM) * 2 + size_t((K + 4 * kFtK - 1) / (4 * kFtK) * (4 * kFtK) + kFtK) * 4; }     // 96 KiB and g

// ------------------------------------------------------------------------------------------- host
struct F32Plan { int MB, RB, S, k_slab, n_tiles; size_t lds; bool ok; const char* why; };

static F32Plan f32_plan(const Problem& p)
{
    F32Plan pl{};
    pl.ok = false;
    if (p.dt != F32) { pl.why = "the fp32 matrix-core variant handles fp32 only"; return pl; }
    if (p.gated && (!p.fused || p.N % 8 != 0)) { pl.why = "gated block: the fp32 matrix-core variant needs H % 4 == 0"; return pl; }
    if (p.rscale) { pl.why = "the fp32 matrix-core variant takes no row factors"; return pl; }
    if (p.N % 4 != 0 || p.K % 4 != 0) { pl.why = "the fp32 matrix-core variant needs N % 4 == 0 and K % 4 == 0"; return pl; }
    if (p.n_tile != 0 && p.n_tile != kF32Tile) { pl.why = "the fp32 matrix-core variant has 64-column tiles"; return pl; }
    if (p.k_split < 0 || p.k_split > 16) { pl.why = "the fp32 matrix-core variant takes 1 to 16 K slabs"; return pl; }
    // byte offsets are 32-bit: all of W, and 64 rows of X, below 4 GiB
    if (int64_t(p.K) * p.N * 4 >= (int64_t(1) << 32) - 256 || int64_t(p.K) * 64 * 4 >= (int64_t(1) << 32) - 256) {
        pl.why = "the fp32 matrix-core variant needs K N < 2^30 and K < 2^24";
        return pl;
    }
    pl.RB = (p.M + 63) / 64;
    pl.MB = pl.RB > 1 ? 4 : (p.M + 15) / 16;
    pl.n_tiles = p.gated ? (p.N / 2 + kF32Tile / 2 - 1) / (kF32Tile / 2) : (p.N + kF32Tile - 1) / kF32Tile;
    const int runs = (p.K + 63) / 64;                    // 64 rows of W: one run for each wave
    const int Mb = std::min(p.M, 64);
    int S = p.k_split;
    if (S == 0) {
        // as many slabs as still give every workgroup a compute unit of its own (a sweep of 1 to 16 slabs over 14
        // shapes, M 1 to 128: the best count was the largest with at most 256 workgroups, or within 8 % of it; a
        // second round of workgroups cost 10 to 40 %), while a slab keeps at least 4 runs per wave and the
        // partials fit the library's workspace
        const int64_t wgs = int64_t(pl.n_tiles) * pl.RB;
        S = int(std::min<int64_t>(16, std::max<int64_t>(1, 256 / wgs)));
        S = std::min(S, std::max(1, runs / 4));
        while (S > 1 && int64_t(S) * pl.RB * Mb * p.N * 4 > (int64_t(48) << 20)) --S;
    }
    S = std::min(S, runs);
    // arrival counters and partial sums of squares exist per (row block, column tile): a launch with more of
    // them than the workspace head holds runs unsplit (a forced split is refused)
    const bool head_fits = int64_t(pl.n_tiles) * pl.RB <= kMaxCounters &&
                           int64_t(pl.n_tiles) * pl.RB * S * kSumsqStride <= kMaxSumsqFloats;
    if (S > 1 && !head_fits) {
        if (p.k_split > 1) { pl.why = "too many tiles for a split over K"; return pl; }
        S = 1;
    }
    pl.k_slab = 64 * ((runs + S - 1) / S);
    S = (runs * 64 + pl.k_slab - 1) / pl.k_slab;         // no empty slab
    pl.S = S;
    if (int64_t(S + 16) * Mb * p.N * 4 >= (int64_t(1) << 31)) { pl.why = "split-K partials too large"; return pl; }
    if (int64_t(pl.n_tiles) * pl.RB * S >= (int64_t(1) << 31)) { pl.why = "too many workgroups"; return pl; }
    pl.lds = size_t(4) * 16 * pl.MB * kF32Tile * 4;
    pl.ok = true;
    return pl;
}

// Which problems, and the tile's rows / 64 (0: the kernel above).  By the rounds of workgroups that each needs, K in us: tiles run
// one to a compute unit and slow down as the chip fills (power), the 64 x 64 tiles above run two, or one in a last round
// that has no more, and a split over K fills the chip better than larger tiles would.  Fitted to 13 shapes, 5 to 8 % rms.  us above, on
// 64 and on 128 rows: 512 x 4096 x 4096 168, 119, 151; 1000 x 2000 x 3000 133, 114, 85; 1500 x 256 x 1000 19.8, 12.8, 18.0;
// 300 x 1000 x 8192 73, 61, 46; 256 x 4096 x 4096 85, 102, 150; 1024^3 26, 29, 45; 64 x 4096 x 28672 171, 138, 185.  Above K = 4096, where 128 rows would be further from fp64:
// 2048 x 8192 x 2048 658, 451 (388); 700 x 8192 x 3072 490, 419 (317).
// One block of rows: the kernel above then works on 16 MB of them, a tile always on 64, and its time no longer follows the
// estimate, which is that of 64 rows.  Measured on wide N (16k to 64k, K 64 to 12000), tiles over the kernel above: M 1 to 16 1.3 to 2.5
// (1 x 152 x 34028 21.6 against 8.7 us, 1 x 1912 x 64532 117 against 86), 17 to 32 0.92 to 1.43, 1.12 in the mean of 76 shapes: not used.
// 33 to 48 rows: where the estimates are further than a fifth apart 0.71 to 0.88 (71 shapes), closer 0.89 to 1.06 (26): a wider
// margin.  49 to 64: 0.62 to 0.93 (57).
static int f32_tiles(const Problem& p, const F32Plan& pl)
{
    if (!pl.ok || pl.S > 1 || !p.fused || p.gated || p.n_tile != 0 || p.k_split != 0 || p.K < kFtMinK || p.K > kFtMaxK) return 0;
    if ((int64_t(p.K) + 512) * p.N * 4 >= (int64_t(1) << 31)) return 0;
    if (pl.MB <= 2) return 0;
    const int64_t cols = (p.N + kFtN - 1) / kFtN, small = int64_t(pl.n_tiles) * pl.RB;
    const int64_t n1 = (int64_t(p.M) + 63) / 64 * cols, n2 = (int64_t(p.M) + 127) / 128 * cols;
    if (n1 >= (int64_t(1) << 23)) return 0;              // a grid holds fewer than 2^32 threads, 512 to a tile
    const auto rounds = [](int64_t n, double fixed, double empty, double full) {
        const double last = double(n % 256);
        return double(n / 256) * (fixed + empty + full) + (last > 0. ? fixed + empty + full * last / 256. : 0.);
    };
    const double t1 = rounds(n1, 5.0, 0.0243 * p.K, 0.0035 * p.K), t2 = p.K > kFtMaxK2 ? 1e30 : rounds(n2, 5.5, 0.0372 * p.K, 0.0085 * p.K);
    const int64_t last = small % 512;
    const double t0 = double(small / 512) * (7.0 + 0.041 * p.K) + (last > 256 ? 7.0 + 0.041 * p.K : last ? 4.0 + 0.0203 * p.K : 0.0);
    return std::min(t1, t2) >= (pl.MB == 3 ? 0.80 : 0.93) * t0 ? 0 : t1 < t2 ? 1 : 2;
}

template <int TM>
static hipError_t f32_tile_go(const Problem& p, hipStream_t s)
{
    static LdsOnce once;
    hipError_t e = raise_lds_once(once, {(const void*)f32_tile_kernel<TM>}, int(f32_tile_lds(TM, kFtMaxK)));
    if (e != hipSuccess) return e;
    const int tm = (p.M + 64 * TM - 1) / (64 * TM), tn = (p.N + kFtN - 1) / kFtN;
    if (p.plan) { p.plan[0] = kFtN; p.plan[1] = 1; p.plan[2] = tm * tn; }
    f32_tile_kernel<TM><<<tm * tn, 512, f32_tile_lds(TM, p.K), s>>>((const float*)p.X, (const float*)p.g, (const float*)p.W, (float*)p.Y,
                                                                    p.M, p.K, p.N, tm, tn, p.eps, 1.0f / float(p.K));
    return hipGetLastError();
}

size_t f32_workspace_bytes(const Problem& p)
{
    F32Plan pl = f32_plan(p);
    if (!pl.ok || pl.S <= 1) return 0;
    return size_t(pl.RB) * pl.S * std::min(p.M, 64) * p.N * 4;    // [row block][slab][rows][N]
}

template <int MB>
static hipError_t f32_go(const F32Args& a, bool fused, bool gated, const F32Plan& pl, hipStream_t s)
{
    dim3 grid(unsigned(pl.n_tiles) * pl.S * pl.RB);
    static LdsOnce once;                                 // 64 KiB of dynamic LDS at MB = 4
    hipError_t e = raise_lds_once(once, {(const void*)f32_kernel<MB, true, false>, (const void*)f32_kernel<MB, false, false>,
                                         (const void*)f32_kernel<MB, true, true>}, 80 * 1024);
    if (e != hipSuccess) return e;
    if (gated)      f32_kernel<MB, true, true><<<grid, 256, pl.lds, s>>>(a);
    else if (fused) f32_kernel<MB, true, false><<<grid, 256, pl.lds, s>>>(a);
    else            f32_kernel<MB, false, false><<<grid, 256, pl.lds, s>>>(a);
    return hipGetLastError();
}

hipError_t launch_f32(const Problem& p, hipStream_t s, const char** why)
{
    F32Plan pl = f32_plan(p);
    if (!pl.ok) { if (why) *why = pl.why; return hipErrorInvalidValue; }
    switch (f32_tiles(p, pl)) {
    case 1: return f32_tile_go<1>(p, s);
    case 2: return f32_tile_go<2>(p, s);
    }
    if (pl.S > 1 && (!p.ws_partial || !p.ws_sumsq || !p.ws_counter)) {
        if (why) *why = "split-K needs the workspace";
        return hipErrorInvalidValue;
    }
    if (p.plan) { p.plan[0] = kF32Tile; p.plan[1] = pl.S; p.plan[2] = pl.n_tiles * pl.S * pl.RB; }
    F32Args a;
    a.X = (const float*)p.X; a.g = (const float*)p.g; a.W = (const float*)p.W; a.Y = (float*)p.Y;
    a.M = p.M; a.K = p.K; a.N = p.N; a.eps = p.eps; a.inv_K = 1.0f / float(p.K);
    a.k_slab = pl.k_slab; a.S = pl.S; a.n_tiles = pl.n_tiles; a.RB = pl.RB;
    a.H = p.gated ? p.N / 2 : 0; a.G = p.gate_group;
    a.ws_partial = p.ws_partial; a.ws_sumsq = p.ws_sumsq; a.counter = p.ws_counter;
    const bool fused = p.fused != 0, gated = p.gated != 0;
    switch (pl.MB) {
    case 1:  return f32_go<1>(a, fused, gated, pl, s);
    case 2:  return f32_go<2>(a, fused, gated, pl, s);
    case 3:  return f32_go<3>(a, fused, gated, pl, s);
    default: return f32_go<4>(a, fused, gated, pl, s);
    }
}

}  // namespace rmsnl
