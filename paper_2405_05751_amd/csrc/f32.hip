// The fp32 path of the fused block on the matrix cores (fp32 products, fp32
// sums): the case study's Fig. 2b again -- A_i = sum_k X_ik^2 and B_in = sum_k (X_ik g_k)
// W_kn in one K loop, the division by the root mean square after it -- on 4-byte elements.  Two kernels: the one
// described here (v_mfma_f32_16x16x4_f32), which runs every M, and further down one on 128 x 128 tiles through LDS for
// large problems with K from 192 to 4096 (f32_tiles() has the rule).
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

// ---- large problems: 128 x 128 tiles through LDS
// The kernel above leaves the matrix pipes idle a third of the time: with operands straight from the caches, every 16 x 16 x 4
// instruction waits on loads of its own wave.  Where 128 x 128 tiles fill the chip, this one keeps four K tiles of 32 in LDS
// (direct loads of X and W, as in mid.hip, whose scheme it is): 8 waves in two groups, a group takes 16 of the 32 k, a
// wave 64 x 64 of the tile on v_mfma_f32_32x32x2_f32 (two k: lane halves h, element t of a 16-byte fragment is k 8 s + 4 h + t
// on both sides).  X (.) g is formed in fp32 on the fragments; the two waves that share 64 rows take the squares of 32 each.
// Sums: a matrix accumulator takes 32 k of its group (64 of the tile) and is then added into a second one, so that the
// rounding error stays below that of the kernel above for K from 192 to 4096 (K / 2 terms in two levels of 32 against K / 4
// in two levels of 128; relative error against fp64 1.27e-7 and 1.43e-7 at K = 192, 1.44e-7 and 2.14e-7 at 1000, 1.92e-7 and
// 2.22e-7 at 4096, but 1.23e-7 and 1.01e-7 at 64), which is where it is used.  2048 x 4096 x 4096: 672 -> 593 us, 116 TFLOP/s, 74 % of the fp32 matrix peak
// (the second level costs 3 %; loads asked for earlier or later, and a third or fourth K tile in LDS: 1 %).
constexpr int kFtM = 128, kFtN = 128, kFtK = 32, kFtStages = 4, kFtMinK = 192, kFtMaxK = 4096;
constexpr unsigned kFtOut = 0x80000000u;     // beyond every resource (sizes below 2^31), with any tile offset added

__global__ __launch_bounds__(512, 2) void f32_tile_kernel(const float* X, const float* g, const float* W, float* Y,
                                                          int M, int K, int N, int tiles_m, int tiles_n, float eps, float inv_K)
{
    constexpr int BM = kFtM, BN = kFtN, BK = kFtK, NS = kFtStages, NLOAD = 4;
    extern __shared__ __attribute__((aligned(16))) float smem[];
    float* As = smem;                        // [NS][BM][BK], 16-byte chunk c of row r at c ^ ((r / 2) & 7)
    float* Bs = As + NS * BM * BK;           // [NS][BK][BN]
    float* gs = Bs + NS * BK * BN;           // g, K rounded up to a multiple of BK (and one more tile), zeros behind it
    __shared__ float s_ss[2][BM];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kg = wave >> 2, wm = (wave >> 1) & 1, wn = wave & 1;

    // panels of up to 8 tile rows, column by column (see mid.hip)
    const int l = xcd_run(blockIdx.x, gridDim.x);
    const int panel = l / (8 * tiles_n), in = l - panel * 8 * tiles_n, rows = min(8, tiles_m - 8 * panel);
    const int m0 = (8 * panel + in % rows) * BM, n0 = in / rows * BN;

    const uint64_t xbase = uint64_t(uintptr_t(X + size_t(m0) * K)), wbase = uint64_t(uintptr_t(W));
    const uint4_t xdesc = {uint32_t(xbase), uint32_t(xbase >> 32), uint32_t(min(BM, M - m0) * K * 4), uint32_t(kF32Flags)};
    const uint4_t wdesc = {uint32_t(wbase), uint32_t(wbase >> 32), uint32_t(K * N * 4), uint32_t(kF32Flags)};
    // a load of X: 8 rows of 128 bytes, lane (r, c) fetches the chunk that belongs in slot c of row r; of W: 2 rows of 512
    const int xr = lane >> 3, xc = ((lane & 7) ^ (4 * (wave & 1) + (xr >> 1))) * 4;
    const int wcol = n0 + 4 * (lane & 31);
    unsigned xoff[2], woff[2];
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const int row = 8 * (wave + 8 * p) + xr;
        xoff[p] = m0 + row < M ? unsigned(row * K + xc) * 4u : kFtOut;
        woff[p] = wcol < N ? unsigned((2 * (wave + 8 * p) + (lane >> 5)) * N + wcol) * 4u : kFtOut;
    }
    const uint32_t as_base = uint32_t(uintptr_t(As)) + uint32_t(wave) * 1024, bs_base = uint32_t(uintptr_t(Bs)) + uint32_t(wave) * 1024;
    auto load_tile = [&](int t, int buf) {   // past K: zeros
        const int k0 = t * BK;
        const bool kin = k0 + xc < K;
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            load_lds(wdesc, bs_base + uint32_t(buf * BK * BN * 4 + p * 8192), woff[p] + unsigned(k0) * unsigned(N) * 4u);
            load_lds(xdesc, as_base + uint32_t(buf * BM * BK * 4 + p * 8192), kin ? xoff[p] + unsigned(k0) * 4u : kFtOut);
        }
    };
    const int nk = (K + BK - 1) / BK;
#pragma unroll
    for (int t = 0; t < NS; ++t) load_tile(t, t);
    for (int k = tid; k < (nk + 1) * BK; k += 512) gs[k] = k < K ? g[k] : 0.f;

    const int h = lane >> 5, c = lane & 31;
    const int a_row = wm * 64 + c;
    int a_off[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) a_off[s] = a_row * BK + 4 * ((4 * kg + 2 * s + h) ^ ((a_row >> 1) & 7));
    const int b_off = (16 * kg + 4 * h) * BN + wn * 64 + 2 * c, g_off = 16 * kg + 4 * h;
    float4_t af[2][2][2], gf[2][2];          // [set][step][row block]
    float2_t bf[2][2][4];                    // [set][step][t]: columns 2 c and 2 c + 1
    auto read_frags = [&](auto set, int t, int buf) {
        constexpr int st = decltype(set)::value;
#pragma unroll
        for (int s = 0; s < 2; ++s) {
#pragma unroll
            for (int i = 0; i < 2; ++i) af[st][s][i] = *(const float4_t*)(As + buf * BM * BK + a_off[s] + i * 32 * BK);
            gf[st][s] = *(const float4_t*)(gs + t * BK + g_off + 8 * s);
#pragma unroll
            for (int e = 0; e < 4; ++e) bf[st][s][e] = *(const float2_t*)(Bs + buf * BK * BN + b_off + (8 * s + e) * BN);
        }
    };
    float16_t acc[2][2], tot[2][2];
    float ss = 0.f, ss_tot = 0.f;            // squares of row block wn
    auto clear = [&](float16_t (&v)[2][2]) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) v[i][j][r] = 0.f;
    };
    clear(acc);
    clear(tot);
    auto fold = [&]() {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) tot[i][j][r] += acc[i][j][r];
        clear(acc);
        ss_tot += ss;
        ss = 0.f;
    };
    auto iteration = [&](auto set, int t) {
        constexpr int st = decltype(set)::value;
        // this wave's loads of tile t + 1 have landed; after the barrier everybody's have, and everybody holds tile t
        __builtin_amdgcn_s_waitcnt(((NS - 2) * NLOAD & 15) | (7 << 4) | (15 << 8));
        __syncthreads();
        __builtin_amdgcn_sched_barrier(0);
        read_frags(std::integral_constant<int, st ^ 1>{}, t + 1, (t + 1) % NS);
        load_tile(t + NS, t % NS);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            float4_t xh[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const float4_t x = af[st][s][i];
                if (wn == i)
#pragma unroll
                    for (int e = 0; e < 4; ++e) ss = __fmaf_rn(x[e], x[e], ss);
                xh[i] = x * gf[st][s];
            }
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(xh[i][e], bf[st][s][e][j], acc[i][j], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    __builtin_amdgcn_s_waitcnt(((NS - 1) * NLOAD & 15) | (7 << 4) | (15 << 8));
    __syncthreads();
    read_frags(std::integral_constant<int, 0>{}, 0, 0);
    int t = 0;
    for (; t + 2 <= nk; t += 2) {
        iteration(std::integral_constant<int, 0>{}, t);
        iteration(std::integral_constant<int, 1>{}, t + 1);
        fold();
    }
    if (t < nk) {
        iteration(std::integral_constant<int, 0>{}, t);
        fold();
    }
    __builtin_amdgcn_s_waitcnt(0 | (7 << 4) | (15 << 8));    // nothing may still be writing LDS past this point
    ss_tot += __shfl_xor(ss_tot, 32, 64);
    if (h == 0) s_ss[kg][wm * 64 + wn * 32 + c] = ss_tot;
    __syncthreads();
    // the groups' sums meet in LDS: group 0 finishes accumulator registers 0 .. 7, group 1 registers 8 .. 15
    float* mine = smem + wave * 4 * 8 * 64 + lane;
    const float* other = smem + (wave ^ 4) * 4 * 8 * 64 + lane;
    auto give = [&](auto first) {
        constexpr int r0 = decltype(first)::value;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int r = 0; r < 8; ++r) mine[((i * 2 + j) * 8 + r) * 64] = tot[i][j][r0 + r];
    };
    auto finish = [&](auto first) {
        constexpr int r0 = decltype(first)::value;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                const int row = wm * 64 + i * 32 + 2 * r0 + 8 * (r >> 2) + 4 * h + (r & 3);
                const float ri = row_scale(s_ss[0][row] + s_ss[1][row], inv_K, eps);
                const float2_t y = {(tot[i][0][r0 + r] + other[(i * 16 + r) * 64]) * ri, (tot[i][1][r0 + r] + other[(i * 16 + 8 + r) * 64]) * ri};
                const int col = n0 + wn * 64 + 2 * c;
                if (m0 + row < M && col < N) __builtin_nontemporal_store(y, (float2_t*)(Y + size_t(m0 + row) * N + col));
            }
    };
    const std::integral_constant<int, 0> low;
    const std::integral_constant<int, 8> high;
    if (kg == 0) give(high); else give(low);
    __syncthreads();
    if (kg == 0) finish(low); else finish(high);
}

static size_t f32_tile_lds(int K)
{
    return size_t(kFtStages) * (kFtM + kFtN) * kFtK * 4 + size_t((K + kFtK - 1) / kFtK + 1) * kFtK * 4;
}

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

// Which problems: by the rounds either kernel needs, K in us (fitted to 12 shapes).  128 x 128 tiles run one to a
// compute unit; 64 x 64 tiles two, or one in a last round that has no more, and a split over K fills the
// chip better than larger tiles would: 1024 x 4096 x 4096 338 -> 301 us, 1500 x 500 x 2500 58 -> 44 us, 2000 x 256 x 8192 146 ->
// 98 us, but 512 x 4096 x 4096 170 us here and 299 on 128 tiles, 1000 x 2000 x 3000 134 and 151 us.
static bool f32_tiles(const Problem& p, const F32Plan& pl)
{
    if (!pl.ok || pl.S > 1 || !p.fused || p.gated || p.n_tile != 0 || p.k_split != 0 || p.K < kFtMinK || p.K > kFtMaxK) return false;
    if ((int64_t(p.K) + 512) * p.N * 4 >= (int64_t(1) << 31)) return false;
    const int64_t tiles = ((int64_t(p.M) + kFtM - 1) / kFtM) * ((p.N + kFtN - 1) / kFtN), small = int64_t(pl.n_tiles) * pl.RB;
    if (tiles >= (int64_t(1) << 31)) return false;
    const double here = double((tiles + 255) / 256) * (5.0 + 0.0725 * p.K);
    const int64_t last = small % 512;
    const double there = double(small / 512) * (7.0 + 0.041 * p.K) + (last > 256 ? 7.0 + 0.041 * p.K : last ? 4.0 + 0.0255 * p.K : 0.0);
    return here < 0.93 * there;
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
    if (f32_tiles(p, pl)) {
        static LdsOnce once;
        hipError_t e = raise_lds_once(once, {(const void*)f32_tile_kernel}, int(f32_tile_lds(kFtMaxK)));
        if (e != hipSuccess) return e;
        const int tm = (p.M + kFtM - 1) / kFtM, tn = (p.N + kFtN - 1) / kFtN;
        if (p.plan) { p.plan[0] = kFtN; p.plan[1] = 1; p.plan[2] = tm * tn; }
        f32_tile_kernel<<<tm * tn, 512, f32_tile_lds(p.K), s>>>((const float*)p.X, (const float*)p.g, (const float*)p.W, (float*)p.Y,
                                                                p.M, p.K, p.N, tm, tn, p.eps, 1.0f / float(p.K));
        return hipGetLastError();
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
