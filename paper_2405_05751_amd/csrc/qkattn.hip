// QKNorm in front of attention, decode form (the paper's QKNorm benchmark: layer normalisation of
// the query and key vectors before attention, fused with the attention itself so that the normalised
// keys never exist in memory): one query per (sample, head) against a key-value cache of S positions.
//
//   qn = LayerNorm(q; gq, bq),  kn_t = LayerNorm(k_t; gk, bk),  s_t = qn . kn_t / sqrt(D),
//   p = softmax_t(s),  o = sum_t p_t v_t.
//
// The same move as in the RMSNorm block: the key's normalisation is taken out of the dot product,
//   qn . kn_t = (sum_d qn_d gk_d (k_td - mu_t)) / sigma_t + qn . bk,
// so a key is read once, raw, and its mean, variance and dot product with qn (.) gk come out of the
// same registers.  The kernel is bound by streaming K and V once.
//
// Fast path (vectors of whole 16-byte chunks, at most 32 of them: D % 8 == 0 up to 256 in the 16-bit types,
// D % 4 == 0 up to 128 in fp32): a group of 8, 16 or 32 lanes shares a key, one chunk to a lane (a wave-wide
// load is 8, 4 or 2 consecutive keys, contiguous), the three sums over D are exchanges inside
// that lane group (DPP and, for 32 lanes, a swap of 16-lane rows: no LDS), every group keeps its own running
// maximum, denominator and the lane's output sums (online softmax), and the groups, the waves and
// the splits of the sequence (by the last of them to arrive, through the workspace) are merged at
// the end.  A vector with fewer chunks than its group has lanes (D = 96: 12 of 16) leaves the last lanes without
// one: they fetch the vector's last chunk again, a line that is on its way anyhow, and stay out of the sums.
// Measured at 32 heads x 3001 positions x D = 96, fp16: 10.2 us (3.6 TB/s) against 1216 us in the
// plain kernel, which until then ran every D but 64, 128 and 256.  Any other D: that plain kernel.
#include <algorithm>
#include "common.hpp"
#include <type_traits>

namespace rmsnl {

constexpr int kQkOut = 0x7ffffff0;
constexpr int kQkFlags = 0x00020000;
// Iterations (one K and one V load per lane each) in flight: 4 with whole lane groups, the 32 KiB that a compute
// unit keeps on its way (8 x 32 x 4096 x 128: 4, 6, 8 iterations take 76.8, 81.1, 81.8 us); 6 where part of the lanes
// fetch nothing new (8 x 32 x 4096 x 80: 4 and 6 take 80.1 and 77.5 us).
constexpr int qk_ring(bool full) { return full ? 4 : 6; }
// Cache policy of those loads: streamed past the caches where they are whole lines (the default policy there: 93.4 us
// for 76.8), kept where neighbouring keys share lines (D = 96: 78.6 us for 79.5).
constexpr int qk_policy(bool full) { return full ? 2 : 0; }
constexpr float kLog2e = 1.4426950408889634f;

struct QkArgs {
    const void* Q; const void* K; const void* V;
    const void* gq; const void* bq; const void* gk; const void* bk;
    void* O;
    float* part;                     // [B*H][SP][D + 2] when SP > 1
    unsigned* counter;               // one arrival counter per (sample, head), zero between calls; or null:
                                     // then a second kernel merges the splits
    float eps, scale_log2e;          // scores are kept in units of log2: s * log2(e) / sqrt(D)
    int S, SP, chunk;                // positions, splits, positions per split (a multiple of 32)
    int D;                           // head size (kernels for a fixed D do not read it)
};

// sum over a group of LPK = 8, 16 or 32 consecutive lanes (aligned to LPK), in every lane of the group
template <int LPK>
__device__ __forceinline__ float group_sum(float v)
{
#define RL_DPP(ctrl) __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), (ctrl), 0xf, 0xf, false))
    if constexpr (LPK == 8) {
        v += RL_DPP(0xB1);                   // lanes 1 0 3 2 of each four
        v += RL_DPP(0x4E);                   // lanes 2 3 0 1 of each four: the four now agree
        v += RL_DPP(0x141);                  // lane 7 - i of each eight: the other four's sum
    } else {
        v += RL_DPP(0x128);                  // rotations inside a row of 16 lanes
        v += RL_DPP(0x124);
        v += RL_DPP(0x122);
        v += RL_DPP(0x121);
        if constexpr (LPK == 32) {
            // v_permlane16_swap exchanges rows 1 and 3 (of 16 lanes) of its first operand with rows 0 and 2 of
            // its second: with v in both they become (row 0, row 0, row 2, row 2) and (row 1, row 1, row 3,
            // row 3), whose sum is the sum over each pair of rows.  Written out, waits included, because the
            // compiler's builtin adds the first result to itself.
            float t;
            asm volatile("v_mov_b32 %1, %0\n\ts_nop 1\n\tv_permlane16_swap_b32 %0, %1\n\ts_nop 1\n\tv_add_f32 %0, %0, %1"
                         : "+v"(v), "=&v"(t));
        }
    }
#undef RL_DPP
    return v;
}

// elements of T in a 16-byte chunk, and a chunk's elements as floats
template <typename T> constexpr int qk_per_chunk() { return 16 / int(sizeof(typename Elem<T>::store_t)); }

template <typename T>
__device__ __forceinline__ void unpack(uint4_t p, float* x)
{
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        if constexpr (std::is_same<T, float>::value) x[e] = __uint_as_float(p[e]);
        else { x[2 * e] = Elem<T>::lo(p[e]); x[2 * e + 1] = Elem<T>::hi(p[e]); }
    }
}

// FULL: D is LPK whole chunks; else D comes with the arguments and has fewer.
template <typename T, int LPK, bool FULL>
__global__ __launch_bounds__(256) void qkattn_kernel(QkArgs a)
{
    typedef typename Elem<T>::store_t E;
    constexpr int R = qk_ring(FULL);
    constexpr int EC = qk_per_chunk<T>();    // elements of a lane's chunk
    constexpr int EB = int(sizeof(E));
    constexpr int DMAX = EC * LPK;
    const int D = FULL ? DMAX : a.D;
    const float inv_D = 1.0f / float(D);
    constexpr int KPW = 64 / LPK;            // keys in a wave-wide load
    constexpr int PPI = 4 * KPW;             // positions the workgroup takes per iteration (4 KiB of K and of V)
    __shared__ float s_m[4], s_l[4];
    __shared__ float s_acc[4][DMAX];
    __shared__ int s_last;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int kq = lane / LPK, c = lane % LPK;
    const bool live = FULL || c < D / EC;    // a lane without a chunk of its own takes the last one again
    const int cl = FULL ? c : min(c, D / EC - 1);
    const int bh = blockIdx.x / a.SP, sp = blockIdx.x % a.SP;
    const int t0 = sp * a.chunk, t1 = min(a.S, t0 + a.chunk);

    // The query and the norms' vectors are asked for first, and used only when the first keys and values are on their way too:
    // the chain of exchanges below then runs beside the first round trip to memory and not before it (1 x 32 x 3001 x 96 fp16 12.2 -> 11.7 us,
    // 16 x 16 x 513 x 96 13.3 -> 12.6, 1 x 8 x 128 x 128 4.55 -> 4.35, in graphs).
    uint4_t qv[5];
    qv[0] = *(const uint4_t*)((const E*)a.Q + size_t(bh) * D + EC * cl);
    qv[1] = *(const uint4_t*)((const E*)a.gq + EC * cl);
    qv[2] = *(const uint4_t*)((const E*)a.bq + EC * cl);
    qv[3] = *(const uint4_t*)((const E*)a.gk + EC * cl);
    qv[4] = *(const uint4_t*)((const E*)a.bk + EC * cl);
    asm volatile("" ::: "memory");           // pins the loads here

    const __amdgpu_buffer_rsrc_t krs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<E*>((const E*)a.K + size_t(bh) * a.S * D), 0, a.S * D * EB, kQkFlags);
    const __amdgpu_buffer_rsrc_t vrs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<E*>((const E*)a.V + size_t(bh) * a.S * D), 0, a.S * D * EB, kQkFlags);
    // iteration i of this wave: position t0 + PPI i + KPW wave + kq (the workgroup reads PPI positions of K
    // and of V, up to 4 KiB each, contiguous, per iteration); a position outside the split is not fetched
    const int nIter = (t1 - t0 + PPI - 1) / PPI;   // uniform
    const int tl = t0 + KPW * wave + kq;
    const int off0 = (tl * D + EC * cl) * EB;

    uint4_t kx[R], vx[R];
    // The first R loads and those of the main loop are issued whether or not their iteration exists (one past the split reads
    // zeros through the range check, at no memory traffic), the last R iterations issue none; the issues are pinned in program order,
    // so that the compiler can count the loads younger than the one it waits for.
    auto issue = [&](int i, int r) {
        const int t = tl + PPI * i;
        const int off = t < t1 ? off0 + i * (PPI * D * EB) : kQkOut;
        __builtin_amdgcn_sched_barrier(0);
        kx[r] = __builtin_amdgcn_raw_buffer_load_b128(krs, off, 0, qk_policy(FULL));
        vx[r] = __builtin_amdgcn_raw_buffer_load_b128(vrs, off, 0, qk_policy(FULL));
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
#pragma unroll
    for (int r = 0; r < R; ++r) issue(r, r);

    // ---- the query: LayerNorm, then folded with the keys' gain and bias
    float qg[EC], qb;
    {
        float q[EC], g[EC], b[EC], gk[EC], bk[EC];
        unpack<T>(qv[0], q);
        unpack<T>(qv[1], g);
        unpack<T>(qv[2], b);
        unpack<T>(qv[3], gk);
        unpack<T>(qv[4], bk);
        float s = 0.f;
#pragma unroll
        for (int e = 0; e < EC; ++e) s += q[e];
        const float mu = group_sum<LPK>(live ? s : 0.f) * inv_D;
        float v = 0.f;
#pragma unroll
        for (int e = 0; e < EC; ++e) { q[e] -= mu; v = __fmaf_rn(q[e], q[e], v); }
        const float rinv = 1.0f / __fsqrt_rn(group_sum<LPK>(live ? v : 0.f) * inv_D + a.eps);
        float t = 0.f;
#pragma unroll
        for (int e = 0; e < EC; ++e) {
            const float qn = __fmaf_rn(q[e] * rinv, g[e], b[e]);
            qg[e] = qn * gk[e];
            t = __fmaf_rn(qn, bk[e], t);
        }
        qb = group_sum<LPK>(live ? t : 0.f);
    }

    float m = -1.0e30f, l = 0.f, acc[EC];
#pragma unroll
    for (int e = 0; e < EC; ++e) acc[e] = 0.f;

    // Two iterations at a time: a wave has its SIMD to itself, and one iteration is a chain of dependent
    // exchanges, so the second one's fill the gaps of the first; the running maximum and the rescaling of the
    // sums are then paid once for both (1 x 32 x 3001 x 96: 13.5 -> 12.6 us, 3 x 40 x 1105 x 80: 17.9 -> 16.8).
    auto consume = [&](int i, int r) {
        float s[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            float x[EC];
            unpack<T>(kx[r + h], x);
            float s1 = 0.f;
#pragma unroll
            for (int e = 0; e < EC; ++e) s1 += x[e];
            const float mu = group_sum<LPK>(live ? s1 : 0.f) * inv_D;
            float s2 = 0.f, dot = 0.f;
#pragma unroll
            for (int e = 0; e < EC; ++e) {
                x[e] -= mu;
                s2 = __fmaf_rn(x[e], x[e], s2);
                dot = __fmaf_rn(qg[e], x[e], dot);
            }
            s2 = group_sum<LPK>(live ? s2 : 0.f);
            dot = group_sum<LPK>(live ? dot : 0.f);
            s[h] = __fmaf_rn(dot, 1.0f / __fsqrt_rn(s2 * inv_D + a.eps), qb) * a.scale_log2e;
        }
        const bool v0 = tl + PPI * i < t1, v1 = tl + PPI * (i + 1) < t1;     // (v1 implies v0)
        const float m_new = fmaxf(m, fmaxf(v0 ? s[0] : m, v1 ? s[1] : m));
        const float corr = __builtin_amdgcn_exp2f(m - m_new);
        const float p0 = v0 ? __builtin_amdgcn_exp2f(s[0] - m_new) : 0.f;
        const float p1 = v1 ? __builtin_amdgcn_exp2f(s[1] - m_new) : 0.f;
        m = m_new;
        l = __fmaf_rn(l, corr, p0 + p1);
        float va[EC], vb[EC];
        unpack<T>(vx[r], va);
        unpack<T>(vx[r + 1], vb);
#pragma unroll
        for (int e = 0; e < EC; ++e) acc[e] = __fmaf_rn(acc[e], corr, __fmaf_rn(p0, va[e], p1 * vb[e]));
    };

    static_assert(R % 2 == 0, "iterations are taken in pairs");
    int i0 = 0;
    for (; i0 + R < nIter; i0 += R) {
#pragma unroll
        for (int r = 0; r < R; r += 2) {
            consume(i0 + r, r);
            issue(i0 + r + R, r);
            issue(i0 + r + R + 1, r + 1);
        }
    }
    // The last ones ask for nothing more: a load past the split brings nothing, but takes its place among the unit's (3 x 40 x 1105 x 80
    // fp16 14.2 -> 13.6 us, 1 x 16 x 8192 x 256 25.3 -> 24.4, 1 x 32 x 3001 x 96 11.7 -> 11.4).
#pragma unroll
    for (int r = 0; r < R; r += 2)
        if (i0 + r < nIter) consume(i0 + r, r);      // uniform

    // ---- merge the key groups of the wave (lanes l, l ^ LPK, l ^ 2 LPK, ...)
#pragma unroll
    for (int off = LPK; off < 64; off <<= 1) {
        const float m_o = __shfl_xor(m, off, 64), l_o = __shfl_xor(l, off, 64);
        const float m_n = fmaxf(m, m_o);
        const float w_s = __builtin_amdgcn_exp2f(m - m_n), w_o = __builtin_amdgcn_exp2f(m_o - m_n);
        l = l * w_s + l_o * w_o;
#pragma unroll
        for (int e = 0; e < EC; ++e) acc[e] = acc[e] * w_s + __shfl_xor(acc[e], off, 64) * w_o;
        m = m_n;
    }
    if (kq == 0) {
#pragma unroll
        for (int e = 0; e < EC; ++e) s_acc[wave][EC * c + e] = acc[e];
        if (c == 0) { s_m[wave] = m; s_l[wave] = l; }
    }
    __syncthreads();
    // ---- merge the four waves; thread j < D owns output dimension j
    if (tid < D) {
        const float mm = fmaxf(fmaxf(s_m[0], s_m[1]), fmaxf(s_m[2], s_m[3]));
        float o = 0.f, ll = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float ws = __builtin_amdgcn_exp2f(s_m[w] - mm);
            o = __fmaf_rn(s_acc[w][tid], ws, o);
            ll = __fmaf_rn(s_l[w], ws, ll);
        }
        if (a.SP == 1) {
            ((E*)a.O)[size_t(bh) * D + tid] = Elem<T>::from_f32(o / ll);
        } else {                             // written through: another workgroup will read them
            float* dst = a.part + (size_t(bh) * a.SP + sp) * (D + 2);
            st_dev(dst + tid, o);
            if (tid == 0) { st_dev(dst + D, mm); st_dev(dst + D + 1, ll); }
        }
    }
    if (a.SP == 1 || !a.counter) return;     // uniform

    // ---- the last split of this (sample, head) to arrive merges them all
    __builtin_amdgcn_s_waitcnt(0);           // this wave's stores have been acknowledged
    __syncthreads();
    if (tid == 0) {
        const unsigned prev = __hip_atomic_fetch_add(a.counter + bh * kCounterStride, 1u, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT);
        s_last = (prev == unsigned(a.SP - 1));
    }
    __syncthreads();
    if (!s_last) return;
    if (tid < D) {
        const float* src = a.part + size_t(bh) * a.SP * (D + 2);
        float mm = -1.0e30f, o = 0.f, ll = 0.f;
        for (int s0 = 0; s0 < a.SP; s0 += 16) {      // 16 splits per round trip, all loads before any use
            float pm[16], pl[16], po[16];
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const float* e = src + size_t(min(s0 + j, a.SP - 1)) * (D + 2);
                pm[j] = ld_dev(e + D); pl[j] = ld_dev(e + D + 1); po[j] = ld_dev(e + tid);
            }
            float bm = mm;
#pragma unroll
            for (int j = 0; j < 16; ++j) if (s0 + j < a.SP) bm = fmaxf(bm, pm[j]);
            const float w0 = __builtin_amdgcn_exp2f(mm - bm);
            o *= w0; ll *= w0;
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const float ws = s0 + j < a.SP ? __builtin_amdgcn_exp2f(pm[j] - bm) : 0.f;
                o = __fmaf_rn(po[j], ws, o);
                ll = __fmaf_rn(pl[j], ws, ll);
            }
            mm = bm;
        }
        ((E*)a.O)[size_t(bh) * D + tid] = Elem<T>::from_f32(o / ll);
    }
    if (tid == 0)                            // ready for the next call on this stream
        __hip_atomic_store(a.counter + bh * kCounterStride, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// splits of one (sample, head) -> O; thread j owns output dimension j
template <typename T>
__global__ void qkattn_combine_kernel(const float* __restrict__ part, typename Elem<T>::store_t* __restrict__ O, int SP, int D)
{
    const float* src = part + size_t(blockIdx.x) * SP * (D + 2);
    float mm = -1.0e30f;
    for (int s = 0; s < SP; ++s) mm = fmaxf(mm, src[s * (D + 2) + D]);
    float o = 0.f, ll = 0.f;
    for (int s = 0; s < SP; ++s) {
        const float ws = __builtin_amdgcn_exp2f(src[s * (D + 2) + D] - mm);
        o = __fmaf_rn(src[s * (D + 2) + threadIdx.x], ws, o);
        ll = __fmaf_rn(src[s * (D + 2) + D + 1], ws, ll);
    }
    O[size_t(blockIdx.x) * D + threadIdx.x] = Elem<T>::from_f32(o / ll);
}

// ------------------------------------------------------------------------- D the fast path does not take
// One workgroup per (sample, head), fp32 arithmetic, the definition step by step: scores into the
// workspace, their maximum, the exponentials and their sum, then one thread per output dimension.
template <typename T>
__global__ __launch_bounds__(256) void qkattn_plain_kernel(const typename Elem<T>::store_t* __restrict__ Q,
    const typename Elem<T>::store_t* __restrict__ K, const typename Elem<T>::store_t* __restrict__ V,
    const typename Elem<T>::store_t* __restrict__ gq, const typename Elem<T>::store_t* __restrict__ bq,
    const typename Elem<T>::store_t* __restrict__ gk, const typename Elem<T>::store_t* __restrict__ bk,
    typename Elem<T>::store_t* __restrict__ O, float* __restrict__ scores, float eps, int S, int D)
{
    __shared__ float red[4];
    const int tid = threadIdx.x;
    const size_t bh = blockIdx.x;
    auto ld = [](const typename Elem<T>::store_t* p, size_t i) { return Elem<T>::to_f32(p[i]); };
    auto block_reduce = [&](float v, bool is_max) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            const float o = __shfl_xor(v, off, 64);
            v = is_max ? fmaxf(v, o) : v + o;
        }
        __syncthreads();
        if ((tid & 63) == 0) red[tid >> 6] = v;
        __syncthreads();
        return is_max ? fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3])) : (red[0] + red[1]) + (red[2] + red[3]);
    };
    // statistics of the query (every thread computes them: D is small)
    const typename Elem<T>::store_t* q = Q + bh * D;
    float qmu = 0.f;
    for (int j = 0; j < D; ++j) qmu += ld(q, j);
    qmu /= float(D);
    float qvar = 0.f;
    for (int j = 0; j < D; ++j) { const float d = ld(q, j) - qmu; qvar = __fmaf_rn(d, d, qvar); }
    const float qr = 1.0f / __fsqrt_rn(qvar / float(D) + eps);
    const float scale = 1.0f / __fsqrt_rn(float(D));
    float top = -INFINITY;
    for (int t = tid; t < S; t += 256) {
        const typename Elem<T>::store_t* k = K + (bh * S + t) * D;
        float mu = 0.f;
        for (int j = 0; j < D; ++j) mu += ld(k, j);
        mu /= float(D);
        float var = 0.f;
        for (int j = 0; j < D; ++j) { const float d = ld(k, j) - mu; var = __fmaf_rn(d, d, var); }
        const float r = 1.0f / __fsqrt_rn(var / float(D) + eps);
        float dot = 0.f;
        for (int j = 0; j < D; ++j) {
            const float qn = __fmaf_rn((ld(q, j) - qmu) * qr, ld(gq, j), ld(bq, j));
            const float kn = __fmaf_rn((ld(k, j) - mu) * r, ld(gk, j), ld(bk, j));
            dot = __fmaf_rn(qn, kn, dot);
        }
        const float s = dot * scale;
        scores[bh * S + t] = s;
        top = fmaxf(top, s);
    }
    top = block_reduce(top, true);
    float sum = 0.f;
    for (int t = tid; t < S; t += 256) {
        const float p = expf(scores[bh * S + t] - top);
        scores[bh * S + t] = p;
        sum += p;
    }
    sum = block_reduce(sum, false);      // (its barriers also order the scores written above)
    for (int j = tid; j < D; j += 256) {
        float o = 0.f;
        for (int t = 0; t < S; ++t) o = __fmaf_rn(scores[bh * S + t], ld(V, (bh * S + t) * D + j), o);
        O[bh * D + j] = Elem<T>::from_f32(o / sum);
    }
}

// ------------------------------------------------------------------------------------------- host
// force > 0: that many splits, at least 64 positions each.  Otherwise the count of least cost, in microseconds,
// from a sweep of 1 to 64 splits over 19 shapes (8 to 640 heads, 281 to 8192 positions, D 64 to 256): the stream
// takes what HBM gives (6.3 TB/s) or what one compute unit takes in (35 GB/s, idle lanes of a group counted in) of the
// splits it is dealt one after the other, and a little of the lesser of the two; a further round of workgroups
// costs its start, and a split pays for the exchange (2 us) and for every share the last workgroup reads.  One workgroup per unit with 256 positions at least, the rule before, left short
// sequences of few heads on few units (1 x 8 x 1463 x 96: 10.6 us against 7.3) and put just over 256 workgroups
// on the chip where the heads do not divide 256 (5 x 32 x 3000 x 128: 54.9 against 44.6 us).
static void qk_plan(int64_t BH, int S, int vec_bytes, int force, int* SP, int* chunk)
{
    auto chunk_of = [&](int64_t sp) { return int(((S + sp - 1) / sp + 31) / 32 * 32); };
    int64_t sp = std::min<int64_t>(force, std::max(1, S / 64));
    if (force <= 0) {
        sp = 1;
        double best = 1e30;
        const double hbm_us = 2.0 * double(BH) * S * vec_bytes / 6.3e6;
        const double group_bytes = vec_bytes <= 128 ? 128.0 : vec_bytes <= 256 ? 256.0 : 512.0;
        for (int64_t n = 1; n <= std::min<int64_t>(64, std::max(1, S / 64)); ++n) {
            const int64_t rounds = (BH * n + 255) / 256;
            const double unit_us = double(rounds) * chunk_of(n) * 2.0 * group_bytes / 35.0e3;
            const double t = std::max(hbm_us, unit_us) + 0.15 * std::min(hbm_us, unit_us) + 0.5 * double(rounds) +
                             (n > 1 ? 2.0 + 0.06 * double(n) : 0.0);
            if (t < best) { best = t; sp = n; }
        }
    }
    sp = std::min<int64_t>(sp, 64);
    *chunk = chunk_of(sp);
    *SP = (S + *chunk - 1) / *chunk;
}

// the fast kernel: whole 16-byte chunks, at most 32, and a (sample, head)'s keys short of the byte offset
// that stands for "not fetched"
static bool qk_fast(int64_t S, int64_t D, DType dt)
{
    const int eb = dt == F32 ? 4 : 2;
    return D * eb % 16 == 0 && D * eb <= 512 && S * D * eb < kQkOut;
}

int qkattn_splits(int64_t B, int64_t H, int64_t S, int64_t D, DType dt, int splits)
{
    if (!qk_fast(S, D, dt)) return 0;
    int SP, chunk;
    qk_plan(B * H, int(S), int(D) * (dt == F32 ? 4 : 2), splits, &SP, &chunk);
    return SP;
}

size_t qkattn_workspace_bytes(int64_t B, int64_t H, int64_t S, int64_t D, DType dt, int splits)
{
    if (!qk_fast(S, D, dt)) return size_t(B) * H * S * 4;           // the plain kernel's scores
    const int SP = qkattn_splits(B, H, S, D, dt, splits);
    return SP > 1 ? size_t(B) * H * SP * (D + 2) * 4 : 0;
}

template <typename T>
static hipError_t qk_plain_go(const void* Q, const void* K, const void* V, const void* gq, const void* bq,
                              const void* gk, const void* bk, void* O, float* ws, float eps,
                              int64_t BH, int S, int D, hipStream_t s)
{
    typedef typename Elem<T>::store_t E;
    qkattn_plain_kernel<T><<<dim3((unsigned)BH), 256, 0, s>>>((const E*)Q, (const E*)K, (const E*)V, (const E*)gq,
                                                               (const E*)bq, (const E*)gk, (const E*)bk, (E*)O, ws, eps, S, D);
    return hipGetLastError();
}

template <typename T, int LPK>
static hipError_t qk_fast_go(const QkArgs& a, int64_t BH, hipStream_t s)
{
    const dim3 grid((unsigned)(BH * a.SP));
    if (a.D == LPK * qk_per_chunk<T>()) qkattn_kernel<T, LPK, true><<<grid, 256, 0, s>>>(a);
    else                                qkattn_kernel<T, LPK, false><<<grid, 256, 0, s>>>(a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || a.SP == 1 || a.counter) return e;
    qkattn_combine_kernel<T><<<dim3((unsigned)BH), a.D, 0, s>>>(a.part, (typename Elem<T>::store_t*)a.O, a.SP, a.D);
    return hipGetLastError();
}

// lanes to a key: the fewest of 8, 16, 32 that hold its chunks
template <typename T>
static hipError_t qk_fast_lanes(const QkArgs& a, int64_t BH, hipStream_t s)
{
    const int chunks = a.D / qk_per_chunk<T>();
    if (chunks <= 8)  return qk_fast_go<T, 8>(a, BH, s);
    if (chunks <= 16) return qk_fast_go<T, 16>(a, BH, s);
    return qk_fast_go<T, 32>(a, BH, s);
}

hipError_t launch_qkattn(const void* Q, const void* K, const void* V, const void* gq, const void* bq,
                         const void* gk, const void* bk, float eps, void* O,
                         int64_t B, int64_t H, int64_t S, int64_t D, DType dt, float* ws, unsigned* counters,
                         int splits, hipStream_t s)
{
    const int64_t BH = B * H;
    if (!qk_fast(S, D, dt)) {
        if (dt == F32) return qk_plain_go<float>(Q, K, V, gq, bq, gk, bk, O, ws, eps, BH, int(S), int(D), s);
        if (dt == F16) return qk_plain_go<Fp16>(Q, K, V, gq, bq, gk, bk, O, ws, eps, BH, int(S), int(D), s);
        return qk_plain_go<Bf16>(Q, K, V, gq, bq, gk, bk, O, ws, eps, BH, int(S), int(D), s);
    }
    QkArgs a;
    a.Q = Q; a.K = K; a.V = V;
    a.gq = gq; a.bq = bq; a.gk = gk; a.bk = bk;
    a.O = O; a.part = ws; a.eps = eps;
    a.scale_log2e = kLog2e / sqrtf(float(D));
    a.S = int(S);
    a.D = int(D);
    qk_plan(BH, int(S), int(D) * (dt == F32 ? 4 : 2), splits, &a.SP, &a.chunk);
    a.counter = (BH <= kMaxCounters) ? counters : nullptr;
    return dt == F32 ? qk_fast_lanes<float>(a, BH, s) : dt == F16 ? qk_fast_lanes<Fp16>(a, BH, s) : qk_fast_lanes<Bf16>(a, BH, s);
}

}  // namespace rmsnl
