// The product of the two-kernel form (X-hat materialised, rows scaled in the epilogue) for shapes whose
// 256 x 256 tiles would leave most of the chip idle: tiles of 128 rows x 64 or 128 columns, split over K where even
// those are too few.  Same layouts as the tile kernel (see tile.hip): X-hat rows and W rows in LDS unpadded with
// swizzled 16-byte chunks, B fragments by the transposing LDS read, v_mfma_f32_32x32x16.
//
// What differs is what bounds it.  A 128-row tile meets little of each operand again, so the LDS reads of the
// fragments, not the matrix instructions, set the pace: a wave of 64 x 64 (32 x 64 for 64 columns) reads 64 (48)
// rows per matrix instruction.  Smaller waves would read more, and 4 waves of that size leave one wave
// per SIMD with nothing to run beside its waits.  So the workgroup has 8 waves in two groups, and the groups share the K
// tile and not the columns: group 0 takes the first 32 k of every K tile of 64, group 1 the other 32, and
// their accumulators meet in LDS once, after the K loop.
//
// Both operands go from memory straight into LDS (direct loads), NS tiles ahead.  Iteration t: wait for the wave's own loads
// of tile t + 1, barrier, ask for tile t + NS (into the buffer of tile t, whose fragments every wave holds in registers by
// now), read the fragments of tile t + 1 into the other register set, matrix instructions on tile t.
//
// Unsplit, the kernel can form X-hat itself (FUSED): it multiplies the A fragments by g, which it keeps in LDS, and takes
// the squares from them.  One launch, no workspace, and the same product bit for bit; only the squares are summed in another order.
// It costs vector instructions in the K loop, at 128 columns twice (two waves hold the same rows): in fp16, which has packed
// products, it is ahead nearly everywhere (34 shapes with M 89 to 2341, geometric mean 0.83; worst 1.00), in bf16 at 64
// columns where X-hat's kernel is a fair part of the call, N up to 3 M (32 shapes: 0.72 to 0.99, one 1.05; beyond that 0.98 to
// 1.10 over 29), but not at 128 (0.94 to 1.34: 563 x 3008 x 6336 33.5 and 43.6 us).  There X-hat stays a kernel of its own.
#include <algorithm>
#include <cmath>
#include "common.hpp"
#include <type_traits>

namespace rmsnl {

constexpr int kMidM = 128, kMidK = 64;
constexpr int kMidFlags = 0x00020000;
constexpr unsigned kMidOut = 0x80000000u;    // beyond every resource (sizes below 2^31), with any tile offset added
// K tiles in LDS; with 64 columns two workgroups share a compute unit (72 KiB and 128 registers each), with 128 one (128 KiB)
constexpr int mid_stages(int BN) { return BN == 64 ? 3 : 4; }
constexpr size_t mid_lds(int BN) { return size_t(mid_stages(BN)) * (kMidM + BN) * kMidK * 2; }
// FUSED: g in LDS besides, with room for as many workgroups as before (64 columns: K <= 4096; 128: K <= 16384)
constexpr size_t kMidLdsMost = 160 * 1024;
constexpr size_t mid_gain_lds(int K) { return size_t((K + kMidK - 1) / kMidK) * kMidK * 2; }

struct MidArgs {
    const u16* X; const u16* W; u16* Y; const float* rscale;
    int M, K, N, ldx;                        // ldx: elements from one row of X-hat to the next
    int tiles_m, tiles_n, k_slab;
    int H, G;                                // gated block: outputs (N = 2 H) and the layout of W, see gated_col()
    float* part;                             // SPLIT: fp32 tiles [slab][M][N]
    const u16* g; float eps, inv_K;          // FUSED: X is not X-hat yet
};

template <typename T> struct MfmaMid;
template <> struct MfmaMid<Bf16> {
    static __device__ __forceinline__ float16_t run(uint4_t a, uint4_t b, float16_t c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
    }
};
template <> struct MfmaMid<Fp16> {
    static __device__ __forceinline__ float16_t run(uint4_t a, uint4_t b, float16_t c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8_t, a), __builtin_bit_cast(f16x8_t, b), c, 0, 0, 0);
    }
};

// FUSED: a pair of X times a pair of g, rounded once to the storage type, and the sum of a pair's squares, in as few vector
// instructions as there are (the K loop is bound by them).  fp16 has a packed product, which rounds the exact one once, and
// a dot product; bf16's dot product issues at a fraction of the rate (products from it: 46 us for 44 at 563 x 3008 x 6336).
template <typename T> struct MidPair {
    static __device__ __forceinline__ uint32_t mul(uint32_t x, uint32_t g) {
        return Elem<T>::pack(Elem<T>::lo(x) * Elem<T>::lo(g), Elem<T>::hi(x) * Elem<T>::hi(g));
    }
    static __device__ __forceinline__ float squares(uint32_t x, float s) {
        return __fmaf_rn(Elem<T>::hi(x), Elem<T>::hi(x), __fmaf_rn(Elem<T>::lo(x), Elem<T>::lo(x), s));
    }
};
template <> struct MidPair<Fp16> {
    static __device__ __forceinline__ uint32_t mul(uint32_t x, uint32_t g) {
        return __builtin_bit_cast(uint32_t, __builtin_bit_cast(f16x2_t, x) * __builtin_bit_cast(f16x2_t, g));
    }
    static __device__ __forceinline__ float squares(uint32_t x, float s) {
        const f16x2_t v = __builtin_bit_cast(f16x2_t, x);
        return __builtin_amdgcn_fdot2(v, v, s, false);
    }
};

#define RL_MID_WAIT_VM(n) __builtin_amdgcn_s_waitcnt(((n) & 15) | (((n) >> 4) << 14) | (7 << 4) | (15 << 8))

template <typename T, int BN, bool GATED, bool SPLIT, bool FUSED>
__global__ __launch_bounds__(512, BN == 64 ? 4 : 2) void mid_kernel(MidArgs a)
{
    constexpr int BM = kMidM, BK = kMidK, NS = mid_stages(BN);
    constexpr int WN = BN / 64, WM = 4 / WN;             // waves of a group along N and M
    constexpr int TM = BM / WM / 32, TN = 2;             // matrix tiles per wave
    static_assert(TM == WN, "a row block's squares for each wave along N");
    constexpr int BL = BN / 64;                          // direct loads of W per wave and K tile (two of X)
    constexpr int RPL = 512 / BN;                        // rows of W in one load of 1 KiB
    constexpr int NLOAD = 2 + BL;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    u16* As = (u16*)lds_raw;                             // [NS][BM][BK]
    u16* Bs = As + NS * BM * BK;                         // [NS][BK][BN]
    u16* gs = Bs + NS * BK * BN;                         // FUSED: g, in whole K tiles

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kg = wave >> 2, wm = (wave & 3) / WN, wn = (wave & 3) % WN;

    // the workgroups an XCD holds take consecutive numbers: panels of up to 8 tile rows, inside a panel column by
    // column, so that the 32 it runs together share rows of X-hat and columns of W in its L2; slabs one after the other
    const int tiles = a.tiles_m * a.tiles_n;
    int l = xcd_run(blockIdx.x, gridDim.x);
    const int slab = SPLIT ? l / tiles : 0;
    l -= slab * tiles;
    const int panel = l / (8 * a.tiles_n), in = l - panel * 8 * a.tiles_n;
    const int rows = min(8, a.tiles_m - 8 * panel);
    const int tm = 8 * panel + in % rows, tn = in / rows;
    const int m0 = tm * BM, n0 = GATED ? tn * (BN / 2) : tn * BN;    // gated: first output of the tile
    const int kb = SPLIT ? slab * a.k_slab : 0;
    const int klen = (SPLIT ? min(a.K, kb + a.k_slab) : a.K) - kb;

    // ---- direct loads.  Lane l of a load fills 16 bytes at byte 16 l of a KiB, so it fetches the chunk that the
    // swizzle puts there.  X: 8 rows of 128 bytes, chunk c of row r at c ^ ((r / 2) & 7).  W: rows of 2 BN bytes, chunk c of
    // row r at c ^ 4 (r & 3) (BN = 128) or c ^ 4 ((r / 2) & 1) (BN = 64: two rows cover the banks).
    const uint64_t xbase = uint64_t(uintptr_t(a.X + size_t(m0) * a.ldx + kb)), wbase = uint64_t(uintptr_t(a.W + size_t(kb) * a.N));
    const uint4_t xdesc = {uint32_t(xbase), uint32_t(xbase >> 32), uint32_t((min(BM, a.M - m0) * a.ldx - kb) * 2), uint32_t(kMidFlags)};
    const uint4_t wdesc = {uint32_t(wbase), uint32_t(wbase >> 32), uint32_t(klen * a.N * 2), uint32_t(kMidFlags)};
    const int xr = lane >> 3, xc = ((lane & 7) ^ (4 * (wave & 1) + (xr >> 1))) * 8;          // row in the load, first k
    unsigned xoff[2];
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const int row = 8 * (wave + 8 * p) + xr;
        xoff[p] = m0 + row < a.M ? unsigned(row * a.ldx + xc) * 2u : kMidOut;
    }
    const int wr = lane / (64 / RPL), wc = lane % (64 / RPL);
    const int wchunk = BN == 64 ? wc ^ (4 * ((wr >> 1) & 1)) : wc ^ (4 * (wr & 3));
    int wcol = n0 + 8 * wchunk;
    bool wcol_ok = wcol < a.N;
    if (GATED) {
        // columns 0 .. 31 of a wave's 64 are gate columns, the next 32 the up columns of the same outputs
        const int hc = n0 + ((8 * wchunk) >> 6) * 32 + ((8 * wchunk) & 31);
        wcol = gated_col(hc, (8 * wchunk) & 32, a.H, a.G);
        wcol_ok = hc < a.H;
    }
    unsigned woff[BL];
#pragma unroll
    for (int p = 0; p < BL; ++p) woff[p] = wcol_ok ? unsigned((RPL * (wave + 8 * p) + wr) * a.N + wcol) * 2u : kMidOut;
    const uint32_t as_base = uint32_t(uintptr_t(As)) + uint32_t(wave) * 1024, bs_base = uint32_t(uintptr_t(Bs)) + uint32_t(wave) * 1024;
    auto load_tile = [&](int t, int buf) {               // past the slab's end: zeros
        const int k0 = t * BK;
        const bool kin = k0 + xc < klen;
#pragma unroll
        for (int p = 0; p < BL; ++p)
            load_lds(wdesc, bs_base + uint32_t(buf * BK * BN * 2 + p * 8192), woff[p] + unsigned(k0) * unsigned(a.N) * 2u);
#pragma unroll
        for (int p = 0; p < 2; ++p)
            load_lds(xdesc, as_base + uint32_t(buf * BM * BK * 2 + p * 8192), kin ? xoff[p] + unsigned(k0) * 2u : kMidOut);
    };

    // ---- fragments (see tile.hip): this group's two 16-deep steps of a K tile
    const int a_row = wm * (BM / WM) + (lane & 31);
    const int blk = lane >> 4, jj = lane & 15, b_row = 8 * (blk >> 1) + (jj >> 2);
    int a_off[2], b_off[TN];
#pragma unroll
    for (int s = 0; s < 2; ++s) a_off[s] = a_row * BK + 8 * ((2 * (2 * kg + s) + (lane >> 5)) ^ ((a_row >> 1) & 7));
#pragma unroll
    for (int j = 0; j < TN; ++j)
        b_off[j] = (32 * kg + b_row) * BN + ((wn * 64 + j * 32 + 16 * (blk & 1)) ^ (32 * (BN == 64 ? (b_row >> 1) & 1 : b_row & 3))) +
                   4 * (jj & 3);
    uint4_t af[2][2][TM], bf[2][2][TN];                  // [set][step]
    uint4_t gf[2][2];
    const int nk = (klen + BK - 1) / BK;
    auto read_frags = [&](auto set, int t, int buf) {
        constexpr int st = decltype(set)::value;
        if (FUSED)
#pragma unroll
            for (int s = 0; s < 2; ++s) gf[st][s] = *(const uint4_t*)(gs + min(t, nk - 1) * BK + 8 * (2 * (2 * kg + s) + (lane >> 5)));
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const u16* Ab = As + buf * BM * BK + a_off[s];
            const u16* Bb = Bs + buf * BK * BN + s * 16 * BN;
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const uint2_t lo = lds_read_tr(Bb + b_off[j]), hi = lds_read_tr(Bb + b_off[j] + 4 * BN);
                bf[st][s][j] = uint4_t{lo[0], lo[1], hi[0], hi[1]};
            }
#pragma unroll
            for (int i = 0; i < TM; ++i) af[st][s][i] = *(const uint4_t*)(Ab + i * 32 * BK);
        }
    };
    float16_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    // FUSED: the fragments become X-hat (rounded once, as the first kernel of the other form rounds it) on their way into the
    // matrix instructions; of the WN waves that hold the same rows each takes the squares of row block wn
    float ss = 0.f;
    auto squares = [&](const uint4_t& x) {
#pragma unroll
        for (int e = 0; e < 4; ++e) ss = MidPair<T>::squares(x[e], ss);
    };
    auto x_hat = [&](uint4_t x, const uint4_t& gv) {
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = MidPair<T>::mul(x[e], gv[e]);
        return x;
    };
    if (FUSED) {
        const uint4_t* g8 = (const uint4_t*)a.g;
        for (int c = tid; c < nk * (BK / 8); c += 512) ((uint4_t*)gs)[c] = 8 * c < klen ? g8[c] : uint4_t{0, 0, 0, 0};
    }
#pragma unroll
    for (int t = 0; t < NS; ++t) load_tile(t, t);
    RL_MID_WAIT_VM((NS - 1) * NLOAD);
    __syncthreads();
    read_frags(std::integral_constant<int, 0>{}, 0, 0);
    auto iteration = [&](auto set, int t) {
        constexpr int st = decltype(set)::value;
        RL_MID_WAIT_VM((NS - 2) * NLOAD);                // this wave's loads of tile t + 1 have landed
        __syncthreads();                                 // everybody's have, and everybody holds tile t in registers
        __builtin_amdgcn_sched_barrier(0);
        read_frags(std::integral_constant<int, st ^ 1>{}, t + 1, (t + 1) % NS);
        load_tile(t + NS, t % NS);
        __builtin_amdgcn_sched_barrier(0);
        if (FUSED) {
            if (TM == 1 || wn == 0) {        // (a branch: the compiler would compute both and select)
#pragma unroll
                for (int s = 0; s < 2; ++s) squares(af[st][s][0]);
                asm volatile("");
            } else {
#pragma unroll
                for (int s = 0; s < 2; ++s) squares(af[st][s][TM - 1]);
                asm volatile("");
            }
        }
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const uint4_t x = FUSED ? x_hat(af[st][s][i], gf[st][s]) : af[st][s][i];
#pragma unroll
                for (int j = 0; j < TN; ++j) acc[i][j] = MfmaMid<T>::run(x, bf[st][s][j], acc[i][j]);
            }
        __builtin_amdgcn_sched_barrier(0);
    };
    int t = 0;
    for (; t + 2 <= nk; t += 2) {
        iteration(std::integral_constant<int, 0>{}, t);
        iteration(std::integral_constant<int, 1>{}, t + 1);
    }
    if (t < nk) iteration(std::integral_constant<int, 0>{}, t);
    RL_MID_WAIT_VM(0);                                   // nothing may still be writing LDS past this point
    __syncthreads();

    // ---- the groups' sums: group 0 finishes accumulator registers 0 .. 7, group 1 registers 8 .. 15
    float* mine = (float*)lds_raw + (wave * TM * TN * 8) * 64 + lane;
    const float* other = (const float*)lds_raw + ((wave ^ 4) * TM * TN * 8) * 64 + lane;
    float* s_ss = (float*)lds_raw + 8 * TM * TN * 8 * 64;            // [2][BM], behind them; [0] then the rows' factors
    const int col = lane & 31, rowq = 4 * (lane >> 5);
    auto give = [&](auto first) {            // the eight registers the other group keeps
        constexpr int r0 = decltype(first)::value;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < 8; ++r) mine[((i * TN + j) * 8 + r) * 64] = acc[i][j][r0 + r];
    };
    auto finish = [&](auto first) {          // the eight this one keeps
        constexpr int r0 = decltype(first)::value;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            float v[TN][8];
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < 8; ++r) v[j][r] = acc[i][j][r0 + r] + other[((i * TN + j) * 8 + r) * 64];
            // register r is row 8 (r / 4) + 4 (lane / 32) + r % 4, column lane % 32 of its matrix tile
            const int row0 = m0 + wm * (BM / WM) + i * 32 + 2 * r0 + rowq;
            if constexpr (SPLIT) {
#pragma unroll
                for (int r = 0; r < 8; ++r) {
                    const int row = row0 + 8 * (r >> 2) + (r & 3);
                    float* dst = a.part + (size_t(slab) * a.M + row) * a.N + n0 + wn * 64 + col;
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        if (row < a.M && n0 + wn * 64 + j * 32 + col < a.N) dst[j * 32] = v[j][r];
                }
            } else {
                // rows r and r + 1 of columns c and c + 1 lie in two neighbouring lanes: they trade one value each, and every
                // lane stores two columns of one row (the even lane of row r, the odd lane of row r + 1)
                const bool odd = lane & 1;
#pragma unroll
                for (int r = 0; r < 8; r += 2) {
                    const int ra = row0 + 8 * (r >> 2) + (r & 3), row = ra + (odd ? 1 : 0);
                    float s0, s1;
                    if (FUSED) { s0 = s_ss[ra - m0]; s1 = s_ss[ra - m0 + 1]; }
                    else { s0 = ra < a.M ? a.rscale[ra] : 0.f; s1 = ra + 1 < a.M ? a.rscale[ra + 1] : 0.f; }
                    constexpr int NO = GATED ? 1 : TN;
#pragma unroll
                    for (int j = 0; j < NO; ++j) {
                        const float y0 = GATED ? silu(v[0][r] * s0) * (v[TN - 1][r] * s0) : v[j][r] * s0;
                        const float y1 = GATED ? silu(v[0][r + 1] * s1) * (v[TN - 1][r + 1] * s1) : v[j][r + 1] * s1;
                        const float got = __shfl_xor(odd ? y0 : y1, 1, 64);
                        const uint32_t pair = odd ? Elem<T>::pack(got, y1) : Elem<T>::pack(y0, got);
                        const int NY = GATED ? a.H : a.N;
                        const int c = n0 + (GATED ? wn * 32 : wn * 64 + j * 32) + (col & ~1);
                        if (row < a.M && c < NY) __builtin_nontemporal_store(pair, (uint32_t*)(a.Y + size_t(row) * NY + c));
                    }
                }
            }
        }
    };
    const std::integral_constant<int, 0> low;
    const std::integral_constant<int, 8> high;
    if (kg == 0) give(high); else give(low);
    if (FUSED) {
        ss += __shfl_xor(ss, 32, 64);
        if (lane < 32) s_ss[kg * BM + wm * (BM / WM) + wn * 32 + lane] = ss;         // (TM = WN row blocks of 32)
        __syncthreads();
        if (tid < BM) s_ss[tid] = row_scale(s_ss[tid] + s_ss[BM + tid], a.inv_K, a.eps);
    }
    __syncthreads();
    if (kg == 0) finish(low); else finish(high);
}

template <typename T, int BN, bool GATED, bool SPLIT, bool FUSED>
static hipError_t mid_go(const MidArgs& a, int S, hipStream_t s)
{
    static LdsOnce once;
    hipError_t e = raise_lds_once(once, {(const void*)mid_kernel<T, BN, GATED, SPLIT, FUSED>}, int(FUSED ? kMidLdsMost : mid_lds(BN)));
    if (e != hipSuccess) return e;
    const size_t lds = mid_lds(BN) + (FUSED ? mid_gain_lds(a.K) : 0);
    mid_kernel<T, BN, GATED, SPLIT, FUSED><<<dim3(unsigned(a.tiles_m * a.tiles_n * S)), 512, lds, s>>>(a);
    return hipGetLastError();
}

template <typename T, int BN>
static hipError_t mid_t(const MidArgs& a, bool gated, int S, hipStream_t s)
{
    if (S > 1) return mid_go<T, BN, false, true, false>(a, S, s);
    if (a.g) return gated ? mid_go<T, BN, true, false, true>(a, S, s) : mid_go<T, BN, false, false, true>(a, S, s);
    return gated ? mid_go<T, BN, true, false, false>(a, S, s) : mid_go<T, BN, false, false, false>(a, S, s);
}

// where that is not the slower form
static bool mid_forms(const Problem& p, int cols) { return p.dt == F16 || (cols == 64 && p.N <= 3 * int64_t(p.M)); }

bool mid_fused(const Problem& p, int cols, int S)
{
    return p.fused && S == 1 && (mid_forms(p, cols) || p.no_ws) && mid_lds(cols) + mid_gain_lds(p.K) <= kMidLdsMost / (cols == 64 ? 2 : 1);
}

// The tile width and the split over K for the product of this problem; false: another form is the better choice, or the
// sizes do not fit.  Forced by n_tile = 64 or 128 (and k_split = 1 to 16 slabs).
//
// The choice is a cost model, fitted (log least squares) to 153 shapes with M 65 to 8000, plain and gated, W from memory, the
// chip warm (884 timings at both widths and 1 to 8 slabs; 9 % rms): microseconds for the first kernel, for a round of
// workgroups over the chip (one per compute unit at 128 columns, two at 64) with its K tiles, for W from memory at
// least, and for writing and adding the partial tiles, all with X-hat as a kernel of its own.  The other forms' models (tile_pre_us,
// skinny_us) are of the same fit.  In place of 256 x 256 tiles there is a margin for the models' errors (654 x 2392 x 4352 50 -> 29 us,
// 1024 x 4096 x 4096 57 -> 50 us), in place of row blocks it is 4 %: against a margin of 13 % with which a call that 256 x 256 tiles
// would have run faster than either stayed with the row blocks, 547 changed shapes take 0.80 of the time (geometric mean: 292 x 6536 x 3688
// 60.5 -> 41 us, 614 x 4208 x 2280 46 -> 35, 113 x 6624 x 9856 56 -> 48, 509 x 4096 x 4160 62.5 -> 42), 27 of them, splits
// that take 17 to 24 us, 3 to 16 % more.
// A launch that forms X-hat itself (but for one that does so because there is no room) is put at a tenth less, since it has no first kernel, where that
// is so: at 64 columns two workgroups to a unit hide the work of forming it, many rows make the first kernel long, few K tiles the
// product short; one workgroup to a unit over a long K is slower than a split with the kernel (109 x 2840 x 2*4840 fp16 36 against 25 us,
// 887 x 3696 x 2*904 40 against 31; with one row of tiles nobody shares W either), and so is, against 256 x 256 tiles, a chip full of 128
// columns (3414 x 7632 x 2*2584 447 against 366).  Of 1264 shapes whose choice a tenth anywhere or here changes, this rule takes the fastest form measured within
// 0.3 % (geometric mean), 0.83 of the time with no tenth; 19 are 3 to 16 % slower than without, 149 were (up to 48 %) with it everywhere.
// Against row blocks alone it holds everywhere (1000 x 3200 x 2*672 fp16 24 against 35 us).
// (220 shapes not used for the rule: 0.80; 4 of 106 against row blocks and 2 of 114 against the rest are 3 to 11 % slower.)
bool mid_plan(const Problem& p, int* cols, int* S, int* k_slab)
{
    if (!p.fused || p.dt == F32 || p.N % 8 != 0 || p.K % 8 != 0 || (p.gated && p.N % 16 != 0)) return false;
    if (int64_t(kMidM) * (int64_t(p.K) + 64) * 2 >= (int64_t(1) << 31) || p.N >= (1 << 22)) return false;
    const int64_t tiles_m = (int64_t(p.M) + kMidM - 1) / kMidM;
    auto slab = [&](int s) { return ((p.K + s - 1) / s + kMidK - 1) / kMidK * kMidK; };
    auto fits = [&](int c, int s) {              // byte offsets into a slab of W; a grid holds fewer than 2^32 threads, 512 to a tile
        return (int64_t(slab(s)) + 512) * p.N * 2 < (int64_t(1) << 31) && tiles_m * ((p.N + c - 1) / c + 1) * s < (int64_t(1) << 23);
    };
    if (p.n_tile == 64 || p.n_tile == 128) {
        const int s = std::max(p.k_split, 1);
        if (s > 16) return false;
        *cols = p.n_tile;
        *k_slab = slab(s);
        *S = (p.K + *k_slab - 1) / *k_slab;
        return fits(p.n_tile, s);
    }
    if (p.n_tile != 0 || p.M <= 64) return false;
    const double mk = double(p.M) * p.K * 1e-6, mn = double(p.M) * p.N * 1e-6;
    const double w_us = double(p.K) * p.N * 2e-6 / 3.45;
    // the choice without this kernel; below 16 us row blocks stay: issued one by one such calls take the host as long
    const bool skinny = skinny_row_blocks(p);
    const double other = skinny ? skinny_us(p) : tile_pre_us(p);
    if (skinny && other < 16.) return false;
    const bool split = skinny && skinny_workspace_bytes(p) != 0;
    // no workspace; or none where row blocks need one: then a form without is taken only if it was ahead of them and the splits by a tenth anywhere
    const bool none = p.no_ws && !split, last = p.no_ws && split;
    double best = !skinny ? 0.85 * other : none ? std::min(0.87 * other, tile_pre_us(p)) : 0.96 * other;
    // row blocks are all there is to beat: the tenth wherever X-hat is formed
    double alone = best;
    int alone_cols = 0;
    *cols = 0;
    for (int c = 64; c <= 128; c += 64)
        for (int s = 1; s <= 8; ++s) {
            const int ks = slab(s), real = (p.K + ks - 1) / ks;
            const bool fused = mid_fused(p, c, s) && (none || mid_forms(p, c));
            if (real != s || (none && !fused) || (s > 1 && (ks < 192 || double(s) * mn * 4. > 40.)) || !fits(c, s)) continue;
            // in place of row blocks only with what the entry point that allocates nothing has for it: both then run the
            // same launches and give the same bits (no shape of 12 000 needs more than 43 MiB); where the row blocks are not
            // split, and so need no workspace, with what a stream's region holds (none needs more than 23 MiB)
            if (skinny && !fused && mid_workspace_bytes(p, s) + kHeadBytes > (split ? kRowScratchBytes : kRegionBytes)) continue;
            const int64_t tiles_n = p.gated && s == 1 ? (p.N / 2 + c / 2 - 1) / (c / 2) : (p.N + c - 1) / c;
            const double rounds = double((tiles_m * tiles_n * s + 255) / 256), kt = double((ks + kMidK - 1) / kMidK);
            const double run = c == 128 ? rounds * (4.1 + 0.62 * kt)
                                        : std::ceil(rounds / 2.) * 3.1 + (rounds > 1. ? 0.445 * rounds : 0.48) * kt;
            const bool forms = fused && !none;
            const bool tenth = forms && (last || (c == 128 ? tiles_m * tiles_n <= 496 || (tiles_m >= 16 && p.K <= 2500)
                                                           : rounds > 1. || tiles_m >= 16 || p.K <= (tiles_m > 1 ? 2500 : 1280)));
            const double full = 3.6 + 0.135 * mk + std::max(run, w_us) + (s > 1 ? 0.9 + 2.2 * s * mn : 0.), us = full * (tenth ? 0.9 : 1.);
            if (skinny && s > 1 && other < 19. && us >= 0.87 * other) continue;          // three launches take the host 18 us
            if (us < best) { best = us; *cols = c; *S = s; *k_slab = ks; }
            if (forms && 0.9 * full < alone) { alone = 0.9 * full; alone_cols = c; }
        }
    if (*cols == 0 && skinny && alone_cols != 0) { *cols = alone_cols; *S = 1; *k_slab = slab(1); }
    if (last && *cols != 0 && !(mid_fused(p, *cols, *S) && mid_forms(p, *cols))) *cols = 0;
    return *cols != 0;
}

// q: the product of X-hat (q.rscale set), S slabs of k_slab rows; with S > 1 the fp32 tiles go to part
hipError_t launch_mid(const Problem& q, int cols, int S, int k_slab, float* part, hipStream_t s)
{
    MidArgs a;
    a.X = (const u16*)q.X; a.W = (const u16*)q.W; a.Y = (u16*)q.Y; a.rscale = q.rscale;
    a.M = q.M; a.K = q.K; a.N = q.N; a.ldx = q.ldx ? q.ldx : q.K;
    const bool gated = q.gated && S == 1;                // the reduction kernel applies the gate to split sums
    a.H = gated ? q.N / 2 : 0; a.G = q.gate_group;
    a.tiles_m = (q.M + kMidM - 1) / kMidM;
    a.tiles_n = gated ? (a.H + cols / 2 - 1) / (cols / 2) : (q.N + cols - 1) / cols;
    a.k_slab = k_slab; a.part = part;
    a.g = q.fused ? (const u16*)q.g : nullptr; a.eps = q.eps; a.inv_K = 1.0f / float(q.K);
    if (cols == 64) return q.dt == F16 ? mid_t<Fp16, 64>(a, gated, S, s) : mid_t<Bf16, 64>(a, gated, S, s);
    return q.dt == F16 ? mid_t<Fp16, 128>(a, gated, S, s) : mid_t<Bf16, 128>(a, gated, S, s);
}

}  // namespace rmsnl
