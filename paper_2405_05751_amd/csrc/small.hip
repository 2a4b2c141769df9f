// Fused RMSNorm + MatMul where M is at most a few hundred and W is so small that a launch is a chain of latencies and not a stream.
//
// What such a launch spent its time on in the skinny kernel as it then was (8 x 512 x 512 in fp16, 5.4 us in a graph, its stages): 1.7 us to issue a
// ring of loads that is deeper than the slab is long (a load takes its place in the address unit whether or not there is a row for it),
// 1.8 us for two runs per wave one after the other, 0.4 us to meet, and where K is split over workgroups 3 us or more for the exchange.
// Here all of K lies in one workgroup, so there is no exchange and no workspace; 16 waves (8 above 32 rows, where 16 are 0 to 14 %
// slower) take a step of 32 k each, so that the chain is one load, one conversion, 2 MB NC matrix instructions and one sum over the
// waves; tiles of 16, 32 or 64 columns make up for the missing split with more workgroups.  W goes straight into the wave's corner of
// LDS and comes back by the transposing read: one load per 32 x 16 block in place of eight and their permutes.  Further trips are not
// overlapped: the other waves' loads fill what a unit keeps in flight (two or four steps per trip, and a wave's steps next to each
// other, measured 1 to 25 % slower; 8 waves up to 32 rows 0 to 3 %).
//
// In graphs, us, the skinny kernel and this one: 8 x 512 x 512 fp16 4.6, 3.1; 14 x 1064 x 472 7.8, 4.7; 25 x 656 x 704 7.6, 4.5; 64 x 352 x 752
// 8.3, 4.4; 31 x 1000 x 4968 10.0, 8.1; 18 x 1264 x 6176 10.0, 8.2; in place of the GEMV kernel 3 x 296 x 2536 6.7, 3.4.  Results on N(0, 1) are at the
// same distance from fp64 (ratio 0.9999 to 1.001).  What bounds it: launch and first loads, 2 us; then a unit's intake, K (32 NC + 32 MB)
// bytes per workgroup.
#include <algorithm>
#include <type_traits>
#include "common.hpp"

namespace rmsnl {

constexpr int kSmallFlags = 0x00020000;
constexpr int kSmallMaxK = 2560;         // of the measurements that the choice rests on
// One round of 64-column tiles.  With more, and the short K that is then left by the estimates, the two rounds lose to the one round of the 128-column
// kernels: 29 x 128 x 17408 6.1 -> 9.15 us, 25 x 24 x 24576 5.7 -> 7.5, and of one row in place of the GEMV kernel 1 x 40 x 18432 3.6 -> 5.4.
constexpr int kSmallMaxN = 16384;
constexpr unsigned kSmallOut = 0x80000000u;      // beyond every resource (sizes below 2^31), with any row offset added

constexpr int small_waves(int MB) { return MB <= 2 ? 16 : 8; }
constexpr size_t small_stage(int MB, int NC) { return size_t(small_waves(MB)) * NC * 1024; }
constexpr size_t small_red(int MB, int NC) { return size_t(small_waves(MB)) * MB * NC * 1024; }
// the sums lie behind the staged W where there is room for both, over it (one barrier more) where there is not
constexpr bool small_over(int MB, int NC) { return small_stage(MB, NC) + small_red(MB, NC) > 144 * 1024; }
constexpr size_t small_lds(int MB, int NC) {
    return small_over(MB, NC) ? std::max(small_stage(MB, NC), small_red(MB, NC)) : small_stage(MB, NC) + small_red(MB, NC);
}

struct SmallCold {                               // what the first loads do not need
    u16* Y;
    float eps, inv_K;
    int H, G;
    int RB;
    unsigned long long* trace; int trace_groups;
};

// Tiles of 16 MB rows (all of M, or of a row block of 64) x 16 NC columns; a wave takes every NW-th step of 32 k.
template <typename T, int MB, int NC, bool FUSED, bool GATED>
__global__ __launch_bounds__(64 * small_waves(MB)) void small_kernel(
    const u16* W, const u16* X, const u16* g, int M, int K, int N, SmallCold a)
{
    constexpr int NW = small_waves(MB), MT = 16 * MB, TN = 16 * NC, CH = 2 * NC, HALF = TN / 2;
    typedef Arith<T> Ar;
    extern __shared__ __align__(16) unsigned char lds[];         // W [NW][32][TN]; sums [NW][MT][TN] in fp32
    float* const red = (float*)(lds + (small_over(MB, NC) ? 0 : small_stage(MB, NC)));
    __shared__ float s_sumsq[NW][MT];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i = lane & 15, q = lane >> 4;
    trace_stamp(a.trace, a.trace_groups, 0);
    // row blocks of 64 rows that take the same columns of W side by side on an XCD
    const int b = xcd_run(blockIdx.x, gridDim.x);
    const int tile = MB == 4 ? b / a.RB : b, rb = MB == 4 ? b - tile * a.RB : 0;
    if (MB == 4) {
        M = min(M - 64 * rb, 64);
        X += size_t(rb) * 64 * K;
        a.Y += size_t(rb) * 64 * (GATED ? a.H : N);
    }
    const int n0 = GATED ? tile * HALF : tile * TN;              // gated: first output

    // direct loads of W: lane l of a load fills 16 bytes at byte 16 l of a KiB, which is 32 / NC rows of the tile
    const int wr = lane / CH, wc = 8 * (lane % CH);
    const int hc = n0 + (wc < HALF ? wc : wc - HALF);
    const int col = GATED ? gated_col(hc, wc >= HALF, a.H, a.G) : n0 + wc;
    const unsigned woff = (GATED ? hc < a.H : col < N) ? unsigned(wr * N + col) * 2u : kSmallOut;
    const uint4_t wdesc = {uint32_t(uintptr_t(W)), uint32_t(uintptr_t(W) >> 32), uint32_t(K * N * 2), uint32_t(kSmallFlags)};
    u16* const stage = (u16*)lds + wave * (32 * TN);
    const uint32_t stage_lds = __builtin_amdgcn_readfirstlane(uint32_t(uintptr_t(stage)));
    const __amdgpu_buffer_rsrc_t xrs = __builtin_amdgcn_make_buffer_rsrc(const_cast<u16*>(X), 0, M * K * 2, kSmallFlags);
    const __amdgpu_buffer_rsrc_t grs = __builtin_amdgcn_make_buffer_rsrc(const_cast<u16*>(FUSED ? g : X), 0, K * 2, kSmallFlags);
    unsigned xoff[MB];                                           // (a row that is not there: the last one again, never stored)
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) xoff[mb] = unsigned(min(16 * mb + i, M - 1) * K + 8 * q) * 2u;

    float4_t acc[MB][NC];
    float ss[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
        ss[mb] = 0.f;
#pragma unroll
        for (int c = 0; c < NC; ++c) acc[mb][c] = float4_t{0.f, 0.f, 0.f, 0.f};
    }
    // Two operands for a product, up to 32 rows.  In bf16 cut off, not rounded: the calls of one to four rows that come here in place of
    // the GEMV kernel keep its infinities (rounded, lo is zero or of the other sign, and an infinite W gave NaN).
    constexpr bool TWO = FUSED && MB <= 2, CUT = TWO && std::is_same<T, Bf16>::value;
    const u16* const frag = stage + (8 * q + (i >> 2)) * TN + 4 * (i & 3);       // transposing read: 4 k x 16 columns per 16 lanes
    for (int k0 = 32 * wave; k0 < K; k0 += 32 * NW) {
        uint4_t x[MB], gq;
#pragma unroll
        for (int j = 0; j < NC; ++j)
            load_lds(wdesc, stage_lds + uint32_t(j * 1024), woff + unsigned(k0 + j * (32 / NC)) * unsigned(N) * 2u);
        const bool kin = k0 + 8 * q < K;
        if (FUSED) gq = __builtin_amdgcn_raw_buffer_load_b128(grs, kin ? int(unsigned(k0 + 8 * q) * 2u) : int(kSmallOut), 0, 0);
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
            x[mb] = __builtin_amdgcn_raw_buffer_load_b128(xrs, kin ? int(xoff[mb] + unsigned(k0) * 2u) : int(kSmallOut), 0, 0);
        trace_stamp(a.trace, a.trace_groups, 1);
        __builtin_amdgcn_s_waitcnt(0 | (7 << 4) | (15 << 8));    // all of them: the compiler does not know of the direct loads
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        // X-hat in the storage type, up to 32 rows with its remainder as a second operand; squares of the raw X
        uint4_t hi[MB], lo[TWO ? MB : 1];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            if (!FUSED) { hi[mb] = x[mb]; continue; }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float x0 = Elem<T>::lo(x[mb][e]), x1 = Elem<T>::hi(x[mb][e]);
                ss[mb] = __fmaf_rn(x0, x0, ss[mb]);
                ss[mb] = __fmaf_rn(x1, x1, ss[mb]);
                const float g0 = Elem<T>::lo(gq[e]), g1 = Elem<T>::hi(gq[e]);
                if constexpr (CUT) {
                    uint32_t h, l;
                    TwoPart<T>::split(__fmaf_rn(x0, g0, 0.f), __fmaf_rn(x1, g1, 0.f), &h, &l);       // (the sum with +0 turns -0 into +0)
                    hi[mb][e] = h; lo[mb][e] = l;
                } else {
                    const float p0 = x0 * g0, p1 = x1 * g1;
                    hi[mb][e] = Elem<T>::pack(p0, p1);
                    if (TWO) lo[mb][e] = Elem<T>::pack(p0 - Elem<T>::lo(hi[mb][e]), p1 - Elem<T>::hi(hi[mb][e]));
                }
            }
        }
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const uint2_t b0 = lds_read_tr(frag + 16 * c), b1 = lds_read_tr(frag + 16 * c + 4 * TN);
            const uint4_t b = {b0[0], b0[1], b1[0], b1[1]};
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) acc[mb][c] = Mfma16<T>::run(hi[mb], b, acc[mb][c]);
            if (TWO)
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) acc[mb][c] = Mfma16<T>::run(lo[mb], b, acc[mb][c]);
        }
        // the reads are done before the next trip's loads write there
        __builtin_amdgcn_s_waitcnt(15 | (3 << 14) | (7 << 4) | (0 << 8));
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    }
    trace_stamp(a.trace, a.trace_groups, 2);
    if (small_over(MB, NC)) __syncthreads();
    if (FUSED) {                             // lanes i, i + 16, i + 32, i + 48 hold row i's shares
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            float v = ss[mb];
            v += __shfl_xor(v, 16, 64);
            v += __shfl_xor(v, 32, 64);
            if (q == 0) s_sumsq[wave][16 * mb + i] = v;
        }
    }
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)          // lane (i, q): rows 16 mb + 4 q + r, columns 16 c + i
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int r = 0; r < 4; ++r) red[(wave * MT + 16 * mb + 4 * q + r) * TN + 16 * c + i] = acc[mb][c][r];
    __syncthreads();
    trace_stamp(a.trace, a.trace_groups, 3);
    constexpr int QR = (GATED ? HALF : TN) / 4;                  // output quads of a row
    auto wg_sum = [&](int m, int c) {
        float4_t v = *(const float4_t*)(red + m * TN + c);
#pragma unroll
        for (int w = 1; w < NW; ++w) v = Ar::add4(v, *(const float4_t*)(red + (w * MT + m) * TN + c));
        return v;
    };
    for (int p = tid; p < MT * QR; p += 64 * NW) {
        const int m = p / QR, c = (p % QR) * 4;
        if (m >= M || n0 + c >= (GATED ? a.H : N)) continue;
        float ri = Ar::one();
        if (FUSED) {
            float asum = s_sumsq[0][m];
#pragma unroll
            for (int w = 1; w < NW; ++w) asum = Ar::add(asum, s_sumsq[w][m]);
            ri = Ar::rinv(asum, a.inv_K, a.eps);
        }
        const float4_t v = wg_sum(m, c), u = GATED ? wg_sum(m, c + HALF) : v;
        float y[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) y[e] = GATED ? Ar::out_gated(v[e], u[e], ri, a.eps) : Ar::out(v[e], ri, a.eps);
        const uint2_t o = {Elem<T>::pack(y[0], y[1]), Elem<T>::pack(y[2], y[3])};
        *(uint2_t*)(a.Y + size_t(m) * (GATED ? a.H : N) + n0 + c) = o;
    }
}

// ------------------------------------------------------------------------------------------- host
template <typename T, int MB, int NC>
static hipError_t small_go(const Problem& p, int n_tiles, hipStream_t s)
{
    static LdsOnce once;
    hipError_t e = raise_lds_once(once, {(const void*)small_kernel<T, MB, NC, true, false>, (const void*)small_kernel<T, MB, NC, false, false>,
                                         (const void*)small_kernel<T, MB, NC, true, true>}, int(small_lds(MB, NC)));
    if (e != hipSuccess) return e;
    const SmallCold c{(u16*)p.Y, p.eps, 1.0f / float(p.K), p.gated ? p.N / 2 : 0, p.gate_group, (p.M + 63) / 64, p.trace, p.trace_groups};
#define RL_SMALL_GO(F, G) \
    small_kernel<T, MB, NC, F, G><<<n_tiles * c.RB, 64 * small_waves(MB), small_lds(MB, NC), s>>>( \
        (const u16*)p.W, (const u16*)p.X, (const u16*)p.g, p.M, p.K, p.N, c)
    if (p.gated)      RL_SMALL_GO(true, true);
    else if (p.fused) RL_SMALL_GO(true, false);
    else              RL_SMALL_GO(false, false);
#undef RL_SMALL_GO
    return hipGetLastError();
}

template <typename T, int MB>
static hipError_t small_cols(const Problem& p, int NC, int n_tiles, hipStream_t s)
{
    return NC == 1 ? small_go<T, MB, 1>(p, n_tiles, s) : NC == 2 ? small_go<T, MB, 2>(p, n_tiles, s) : small_go<T, MB, 4>(p, n_tiles, s);
}

template <typename T>
static hipError_t small_rows(const Problem& p, int NC, int n_tiles, hipStream_t s)
{
    switch (p.M > 64 ? 4 : (p.M + 15) / 16) {
    case 1:  return small_cols<T, 1>(p, NC, n_tiles, s);
    case 2:  return small_cols<T, 2>(p, NC, n_tiles, s);
    case 3:  return small_cols<T, 3>(p, NC, n_tiles, s);
    default: return small_cols<T, 4>(p, NC, n_tiles, s);
    }
}

// By a model fitted (log least squares) to 260 shapes at all three widths, M 1 to 64, K 256 to 2600, N to 28672, 10 % rms: launch, rounds of
// workgroups with their K steps, W from memory, and narrow row segments of two halves.  Chosen at 0.88 of the other form's time
// (skinny_plan's estimate with a constant of the same fit), at 0.84 from K N = 4e6 on and 0.78 at long K, where the other kernel is up to 15 % below
// its estimate (12 x 2432 x 2008 8.6 us there, 9.75 here; 15 x 2384 x 3208 9.4, 10.6; 32 x 2304 x 1344 10.8, 12.0).  Of 5900 random shapes, K 8 to
// 2560, N to 32768, both forms timed in graphs, 4271 run here at 0.65 of the time (geometric mean), 2 of them slower by 2 %;
// over all of them 0.732 of the time, where the faster form each time gives 0.718 (0.88 throughout and N to 32768: 139 slower, by up to half).
// Of 2500 others that the line was not laid with five are 1 to 5 % slower, 8 x 1664 x 2*968 15 % and 10 x 1408 x 2560 10 %.
// Rows of W that are a multiple of 512 bytes suit wide tiles (their estimate is 6 % high there) and not narrow ones, the more the longer K is
// (K = 512 1.0, 1024 1.1, 1536 1.25 of the estimate, whichever XCD takes which line): of 237 such shapes, K 256 to 2048, N 512 to 16384,
// 22 were 3 to 34 % slower without that in the rule, one by 3 % with it, at 0.73 of the time over all of them (the faster form each time 0.71).
// Two halves of a tile in two places are the slower the longer K is, too (14 x 1832 x 2*1640 11.0 -> 12.3 us without that term).
// Columns per workgroup / 16 (1, 2 or 4) for this problem, or 0 where another form is the better choice.  other_us: the estimate for
// that one, in the unit of this one's, or 0 for none to beat.
int small_columns(const Problem& p, double other_us)
{
    if (p.dt == F32 || p.M > 64 || p.n_tile != 0 || p.k_split != 0 || p.K > kSmallMaxK || p.N > (p.no_ws ? 2 : 1) * kSmallMaxN) return 0;
    const int MB = (p.M + 15) / 16;
    const bool whole = p.N % 256 == 0;
    double best = 0.;
    int cols = 0;
    for (int NC = 1; NC <= 4; NC *= 2) {
        const double rounds = double(((p.N + 16 * NC - 1) / (16 * NC) + 255) / 256), k = 1e-3 * rounds * p.K;
        double us = 1.98 + 0.10 * MB + 0.43 * rounds + k * (0.62 * NC + 0.83 * MB + (p.gated && NC == 1 ? 0.72 : 0.)) +
                          double(p.K) * p.N * 2.0 / 6.3e6 + (p.gated ? 0.90 : 0.);
        us *= 1. + 1e-3 * p.K * ((whole ? 0.15 : 0.) + (p.gated ? 0.08 : 0.));
        if (cols == 0 || us < best) { best = us; cols = NC; }
    }
    const double w = double(p.K) * p.N;
    const double line = whole ? 0.82 : 0.88;
    // (no_ws: in place of a split that finds no workspace, where the narrow tiles are not much the slower form)
    const double margin = p.no_ws ? line : p.K > 1800 && w > 2.6e6 ? 0.78 : !whole && w > 4.0e6 ? 0.84 : line;
    return other_us == 0. || best < margin * other_us ? cols : 0;
}

// The same above 64 rows, in row blocks of 64, against what the skinny kernel's row blocks and 128-row tiles take (a fit of its own, 11 % rms
// on 120 shapes, M 65 to 1024): 10 us and more however small the problem is, 4 to 9 here.  While the narrow tiles are
// one round of workgroups they take 0.34 to 0.7 of that (141 x 408 x 272 fp16 10.4 -> 4.2 us, 127 x 752 x 552 11.9 -> 5.8,
// 278 x 824 x 1720 12.9 -> 8.4), with more from 0.97 of it to twice as much.  At 0.75 of the other estimate 1178 of 1500 random shapes run here,
// at 0.55 of the time, none slower (0.93 at most); of the 120, at 0.9 three were slower by up to 13 %.
// M <= 512, K <= 1536, N <= 12288: beyond, where the other estimate was less sure, no shape was worth it.
int small_blocks(const Problem& p)
{
    if (p.dt == F32 || p.M <= 64 || p.M > 512 || p.n_tile != 0 || p.k_split != 0 || p.K > 1536 || p.N > 12288) return 0;
    const double w_us = double(p.K) * p.N * 2.0 / 6.3e6, k = 1e-3 * p.K;
    const double other = 9.33 + 3.58 * k + 0.44 * w_us + 1e-6 * p.M * (0.66 * p.N - 0.79 * p.K) + (p.gated ? 0.5 : 0.);
    double best = 0.75 * other;
    int cols = 0;
    for (int NC = 1; NC <= 4; NC *= 2) {
        const double wgs = double((p.M + 63) / 64) * ((p.N + 16 * NC - 1) / (16 * NC));
        if (wgs > 256.) continue;
        const double us = 3.25 + k * (0.60 * NC + 2.41 + (p.gated && NC == 1 ? 0.47 : 0.)) + 1.37 * w_us +
                          wgs / 256. * k * (0.90 * NC - 1.56) + (p.gated ? 0.87 : 0.);
        if (us < best) { best = us; cols = NC; }
    }
    return cols;
}

// Up to four rows where choose_auto would take the GEMV kernel: the narrow tiles are ahead of it on all of 23 shapes with K <= 1024 and
// K N <= 2e6 (0.5 to 0.91 of the time), level at K = 1500 and behind at 1900, and beyond 2e6 the GEMV kernel streams.  One gated row: level at
// K = 900 and up to 14 % behind at 1024 (1 x 1024 x 2*320 5.5 us there, 6.3 here).  Of 400 more shapes with N to 16384 none is slower otherwise.  Not the fused
// block in fp16: the GEMV kernel keeps X (.) g in fp32, whose products leave the range of the two fp16 operands they would have to
// be here (beyond 65504 an infinity and its opposite; X near 1e-5 1.6e-3 from fp64 in place of 2.1e-4).
bool small_wins_over_gemv(const Problem& p)
{
    return (p.dt == BF16 || !p.fused) && p.M <= 4 && p.K <= (p.gated && p.M == 1 ? 896 : 1024) && p.N <= kSmallMaxN && int64_t(p.K) * p.N <= 2000000 && p.n_tile == 0 && p.k_split == 0;
}

hipError_t launch_small(const Problem& p, int NC, hipStream_t s)
{
    const int n_tiles = p.gated ? (p.N / 2 + 8 * NC - 1) / (8 * NC) : (p.N + 16 * NC - 1) / (16 * NC);
    if (p.plan) { p.plan[0] = 16 * NC; p.plan[1] = 1; p.plan[2] = n_tiles * ((p.M + 63) / 64); p.plan[3] = 1; }
    return p.dt == F16 ? small_rows<Fp16>(p, NC, n_tiles, s) : small_rows<Bf16>(p, NC, n_tiles, s);
}

}  // namespace rmsnl
