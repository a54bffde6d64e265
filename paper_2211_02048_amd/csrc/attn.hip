// sige_sparse_attn: attention for the edited query tokens only, against all cached
// keys and values (Sec. 3.2 "Extension to attention layers", Fig. "sige-attention"):
// the attention map is Nq x T instead of T x T.
//
// One wave owns 32 queries of one head and streams its share of the keys in chunks of 32 * KT
// (64 keys for head sizes up to 96, 32 beyond); the next chunk's K and V rows travel to registers
// while the current one is multiplied.  All products run transposed so that everything belonging
// to a query stays in one lane (pair): S^T = K Q^T leaves a query's 32 logits in the registers of lanes l and
// l+32, the online softmax needs a single cross-lane exchange, the probabilities
// feed the second MFMA (O^T = V^T P^T) straight from registers because the
// contraction index may be permuted freely as long as V^T is read with the same
// permutation, and the running rescale of O^T is lane-local.  The waves of a workgroup are groups that split
// the keys: of one wave each on the same 32 queries (few queries, large heads) or of four waves on 128 queries that fetch their
// chunks once (attn_kernel); when few queries are active the key range is also split over
// workgroups and a second small kernel merges the partial (max, sum, O) triples.  Single precision has a kernel of
// its own further down (attn_f32_kernel).
#include "common.h"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace sige {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 as_uint4(const u32x4& v) { return make_uint4(v.x, v.y, v.z, v.w); }

template <typename T> struct Mma16;
template <> struct Mma16<f16> {
    static __device__ __forceinline__ void run(const uint4& a, const uint4& b, f32x16& c)
    {
        union { uint4 u; f16x8 v; } x, y;
        x.u = a; y.u = b;
        c = __builtin_amdgcn_mfma_f32_32x32x16_f16(x.v, y.v, c, 0, 0, 0);
    }
};
template <> struct Mma16<bf16> {
    static __device__ __forceinline__ void run(const uint4& a, const uint4& b, f32x16& c)
    {
        union { uint4 u; bf16x8 v; } x, y;
        x.u = a; y.u = b;
        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x.v, y.v, c, 0, 0, 0);
    }
};

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// Two floats rounded to nearest even into one 32-bit pair of T (a in the low half).
template <typename T> __device__ __forceinline__ uint32_t pack2_rne(float a, float b);
template <> __device__ __forceinline__ uint32_t pack2_rne<f16>(float a, float b)
{
    union { f16x2 v; uint32_t u; } r;
    r.v = __builtin_convertvector((f32x2){a, b}, f16x2);
    return r.u;
}
template <> __device__ __forceinline__ uint32_t pack2_rne<bf16>(float a, float b)
{
    union { bf16x2 v; uint32_t u; } r;
    r.v = __builtin_convertvector((f32x2){a, b}, bf16x2);
    return r.u;
}

struct AttnArgs {
    const void* q;
    const void* k;
    const void* v;
    void* o;
    float* ws;       // partials [split][head][Nq][d + 4] when splits > 1: the d sums, the maximum, the denominator, 2 unused
                     // (rows of whole 16-byte vectors; d is a multiple of 4)
    int q_ld, kv_ld, o_ld;
    int Nq, T, heads, d;
    int splits, chunks_per_split;
    int groups;      // half types: groups of waves in a workgroup (one where it has one chunk, whatever the kernel is built for)
    float scale_log2e;
    // queries taken from a full tensor by block list (q_blocks != NULL): query i is pixel i % q_tpb of
    // block i / q_tpb, at row (y0 + py) * q_W + x0 + px of q (clamped into the q_H x q_W map)
    const int32_t* q_blocks;
    int q_tpb, q_bw, q_H, q_W;
    FastDiv d_tpb, d_qbw, d_dvec, d_dq;   // divisors prepared on the host: q_tpb, q_bw, 16-byte vectors and quarters of a head's row
};

// 32-key tiles per chunk, by head size (DT = 32-wide tiles over d)
constexpr int key_tiles(int DT) { return DT <= 3 ? 2 : 1; }
// bytes between the V rows of a chunk in LDS: an odd multiple of 64, so that the eight keys of a transposed read fall on
// different banks
constexpr int v_row_bytes(int DT) { return 64 * (DT | 1); }
// waves per workgroup, at most: what their sums take in LDS when they meet
constexpr int max_waves(int DT) { return DT <= 4 ? 8 : 4; }
// key groups of a workgroup whose four waves share their chunks
constexpr int common_groups(int DT) { return DT <= 3 ? 2 : 1; }
// one wave per key group: whether Q waits in LDS for its products instead of in registers (K, V, Q and the sums of heads of 225 to 256
// are more than a wave has: 20 to 51 registers of it went through memory, fp16 1500 of 4096 x 8 of 256 360 us in one split, 177 so)
constexpr bool q_in_lds(int DT, int NQ) { return NQ == 1 && DT == 8; }
static int keys_per_chunk(int d, sige_dtype dt) { return dt == SIGE_F32 ? 32 : 32 * key_tiles((d + 31) / 32); }

// DT = 32-wide tiles over d; ODD: d takes an odd number of 16-wide steps (d % 32 is 8 or 16), so the
// last tile of V^T has spare rows.  One of them is then a row of ones: the second product sums the
// probabilities of a query - exactly the rounded values that it multiplies V with - into that row of
// O^T, the running rescale included, and the softmax spends no vector instruction on the denominator.
// The softmax is what bounds a wave (for d = 40 its vector instructions outweigh the matrix
// instructions), so it is kept to a maximum, one fused multiply-add, one exponential and the rounding
// per logit: logits are compared raw and scaled inside the exponent, keys past T are masked only in
// the chunk that holds them, and the accumulators are rescaled only when some query's maximum moved.
//
// The waves of a workgroup are NK groups of NQ: a group takes every NK-th chunk of keys for 32 * NQ queries, and the groups' (maximum,
// denominator, sums) meet in LDS at the end.  NQ = 4 (many queries): the group fetches K and V once for its four waves and passes
// them through LDS, two barriers per chunk.  NQ = 1 (few queries, large heads): every wave for itself, K from memory straight into
// the first product's operands, no barrier in the loop.  V goes into LDS row by row and out of it transposed (ds_read_b64_tr_b16).
// One form alone, four waves on 128 queries and 2-byte stores to transpose V, left most compute units without work where
// there were a few hundred queries, or needed many splits and the merge kernel behind them.  Before -> now, bf16, eight heads unless
// said: 192 of 256 x 160 12.1 -> 10.3 us, 384 of 1024 x 80 16.0 -> 13.2, 1024 of 1024 x 80 22.9 -> 14.2, 96 of 4096 x 40 12.9 -> 11.2,
// 672 of 8192 x 40 37.3 -> 33.5, 2240 of 4096 x 40 47.7 -> 42.7, 192 on 77 keys x 160 10.8 -> 7.6, 9216 of 9216 x 128 930 -> 780,
// fp16 5000 of 9000 x 160 747 -> 553.
//
// FAR: keys so far apart that the byte offsets of a chunk's rows do not fit 32 bits (a column of a tensor of gigabytes).  Those take
// 64-bit offsets, in one kernel for all head sizes: eight tiles, the columns past the head zero.
//
// Registers: four waves on the same chunks hold heads of 97 to 128 in half of a SIMD's, two workgroups per compute unit - if told to:
// free to take more the compiler spreads over 250 and moves the sums to the accumulation registers (fp16, heads of 128, 4000 queries
// of 4096 x 8 154 -> 104 us with the splits of plan_attn, 64 of 1024 x 1 11.6 -> 8.0; larger heads do not fit, smaller ones are two
// groups and have the bound as eight waves).
template <typename T, int DT, int ODD, int NQ, int NK, bool FAR = false>
__global__ __launch_bounds__(64 * NQ * NK, NQ * NK == 8 || (NQ == 4 && DT == 4) ? 2 : 1) void attn_kernel(AttnArgs a)
{
    constexpr int NW = NQ * NK;
    constexpr int KT = key_tiles(DT);
    constexpr int KCH = 32 * KT;                   // keys per chunk
    constexpr int VROW = v_row_bytes(DT);
    constexpr int DK = 2 * DT - ODD;               // 16-wide steps over d for S^T
    constexpr int GT = 64 * NQ;                    // threads that have a chunk in common
    constexpr bool Q_LDS = q_in_lds(DT, NQ);
    using Off = std::conditional_t<FAR, unsigned long, unsigned>;
    static_assert(!FAR || (NQ > 1 && ODD == 0), "any head size: through LDS, no column of ones");
    constexpr int NV = (KCH * (4 * DT - 2 * ODD) + GT - 1) / GT;   // V (and K) vectors a thread stages per chunk, at most
    extern __shared__ uint4 lds4[];
    char* lds = reinterpret_cast<char*>(lds4);
    const int d = a.d;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wq = wave % NQ, wk = wave / NQ, gt = wq * 64 + lane;
    const int half = lane >> 5, l32 = lane & 31;
    const int head = blockIdx.y;
    const int q0 = (blockIdx.x * NQ + wq) * 32, qi = q0 + l32;
    const bool q_ok = qi < a.Nq;
    const int dvec = d / 8, nvec = KCH * dvec;     // 16-byte vectors per row, per chunk
    const Off kv2 = (Off)a.kv_ld * 2u;             // bytes between keys
    const int k_stride = (FAR ? 32 * DT : d) * 2 + 16;             // bytes per K row in LDS (NQ > 1)
    const int vs0 = wk * (KCH * VROW);             // this group's V rows, then the groups' K rows
    char* const vs = lds + vs0;
    char* const ks = lds + (NK == 1 ? 1 : a.groups) * (KCH * VROW) + wk * (KCH * k_stride);
    char* const qs = lds + NK * KCH * VROW;        // Q_LDS: [DK][64 lanes], behind the V rows

    const int chunks_total = (a.T + KCH - 1) / KCH;
    const int c_begin = blockIdx.z * a.chunks_per_split;
    const int c_end = min(c_begin + a.chunks_per_split, chunks_total);
    const char* const kb = (const char*)a.k + (long)head * d * 2;
    const char* const vb = (const char*)a.v + (long)head * d * 2;

    // The vectors of a chunk this lane fetches: of K, row l32 (and l32 + 32) at the 16 bytes of its half in every step - the last
    // step's upper half may lie past d: the row's first bytes instead, made zero below -; of V, the vectors lane, lane + 64, ...
    // (past the chunk's last one: that one again, not stored).
    const bool k_tail = 16 * (DK - 1) + 8 * half >= d;
    Off koff[KT], klast[KT], voff[NV];
    int vkey[NV], vdst[NV];
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) koff[kt] = (Off)(kt * 32 + l32) * kv2 + half * 16;
#pragma unroll
    for (int u = 0; u < NV; ++u) {
        int dv;
        divmod(min(gt + GT * u, nvec - 1), a.d_dvec, vkey[u], dv);
        voff[u] = (Off)vkey[u] * kv2 + dv * 16;
        vdst[u] = vkey[u] * VROW + dv * 16;
    }
    u32x4 kreg[NQ == 1 ? KT * DK : NV], vreg[NV];                  // (native vectors: arrays of structs end up in scratch memory)
    auto fetch = [&](int c) {
        const int t0 = c * KCH;
        if (t0 + KCH > a.T) {                      // the chunk that holds the end: keys past it read the last key's rows
            const int last = a.T - 1 - t0;
#pragma unroll
            for (int kt = 0; kt < KT; ++kt) koff[kt] = (Off)min(kt * 32 + l32, last) * kv2 + half * 16;
#pragma unroll
            for (int u = 0; u < NV; ++u) voff[u] -= (Off)(vkey[u] - min(vkey[u], last)) * kv2;
        }
        const char* const kc = kb + (long)t0 * kv2;
        const char* const vc = vb + (long)t0 * kv2;
        if constexpr (NQ == 1) {
#pragma unroll
            for (int kt = 0; kt < KT; ++kt) {
                klast[kt] = k_tail ? koff[kt] - half * 16 : koff[kt] + 32 * (DK - 1);
#pragma unroll
                for (int s = 0; s < DK; ++s) kreg[kt * DK + s] = *(const u32x4*)(kc + (s == DK - 1 ? klast[kt] : koff[kt] + 32 * s));
            }
        } else {
#pragma unroll
            for (int u = 0; u < NV; ++u) kreg[u] = *(const u32x4*)(kc + voff[u]);
        }
#pragma unroll
        for (int u = 0; u < NV; ++u) vreg[u] = *(const u32x4*)(vc + voff[u]);
    };
    int c = c_begin + wk;
    if (c < c_end) fetch(c);

    // Q fragments (B operand of S^T = K Q^T): 8 consecutive d values of this lane's query
    u32x4 qf[DK];
    long qrow = qi;
    if (a.q_blocks != nullptr && q_ok) {
        int b, p, py, px;
        divmod(qi, a.d_tpb, b, p);
        divmod(p, a.d_qbw, py, px);
        const int y0 = a.q_blocks[2 * b], x0 = a.q_blocks[2 * b + 1];
        qrow = (long)min(max(y0 + py, 0), a.q_H - 1) * a.q_W + min(max(x0 + px, 0), a.q_W - 1);
    }
#pragma unroll
    for (int s = 0; s < DK; ++s) {
        const int dd = 16 * s + 8 * half;
        qf[s] = u32x4{0u, 0u, 0u, 0u};
        if (q_ok && dd < d)
            qf[s] = *(const u32x4*)((const char*)a.q + (qrow * a.q_ld + head * d + dd) * 2);
    }
    if constexpr (Q_LDS) {                         // (the waves have the same queries)
#pragma unroll
        for (int s = 0; s < DK; ++s)
            if (s % NK == wk) *(u32x4*)(qs + s * 1024 + lane * 16) = qf[s];
        __syncthreads();
    }
    // columns d .. DT*32 of the wave's V rows never receive data: zero them once (column d: ones, see above)
    constexpr uint32_t ONE = std::is_same<T, bf16>::value ? 0x3f80u : 0x3c00u;
    if constexpr (FAR) {                           // (any number of them, and as many behind every K row)
        const int pad = 4 * DT - dvec;
        for (int j = gt; j < KCH * pad; j += GT) {
            const int row = j / pad, dv = dvec + j - row * pad;
            *(uint4*)(vs + row * VROW + dv * 16) = make_uint4(0, 0, 0, 0);
            *(uint4*)(ks + row * k_stride + dv * 16) = make_uint4(0, 0, 0, 0);
        }
    } else {
        const int pad = 4 * DT - dvec;             // 16-byte vectors per row, at most 3
        for (int j = gt; j < KCH * 4; j += GT)
            if ((j & 3) < pad)
                *(uint4*)(vs + (j >> 2) * VROW + (dvec + (j & 3)) * 16) = make_uint4(ODD && (j & 3) == 0 ? ONE : 0u, 0, 0, 0);
    }
    // where this lane's share of a transposed read starts: four lanes take the 16 columns of one key, four keys per 16 lanes,
    // lane i of the 16 receives column i of the four keys
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
    const int tr = vs0 + (4 * half + ((lane & 15) >> 2)) * VROW + ((lane >> 4) & 1) * 32 + (lane & 3) * 8;
    auto read_v = [&](int key, int nt) {
        return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(__attribute__((address_space(3))) char*)(lds + tr + key * VROW + nt * 64));
    };

    f32x16 oacc[DT];
#pragma unroll
    for (int nt = 0; nt < DT; ++nt)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[nt][r] = 0.0f;
    float m_run = -INFINITY, l_run = 0.0f;

    if constexpr (NQ > 1 && !FAR) {                // the 16 bytes behind the d values of every K row, which the last step reads when d % 16 is 8
        for (int j = gt; j < KCH; j += GT) *(uint4*)(ks + j * k_stride + d * 2) = make_uint4(0, 0, 0, 0);
    }
    for (; c - wk < c_end; c += NK) {              // (as often in every group: the barriers are the workgroup's)
        const int t0 = c * KCH;
        const bool mine = c < c_end && (NQ == 1 || q0 < a.Nq);
        if constexpr (NQ > 1) {
            __syncthreads();                       // the last chunk's rows have been read
            if (c < c_end) {
#pragma unroll
                for (int u = 0; u < NV; ++u)
                    if (gt + GT * u < nvec) *(u32x4*)(ks + vdst[u] - vkey[u] * (VROW - k_stride)) = kreg[u];
            }
        }
        if (NQ == 1 && !mine) break;
        // V rows as they are (NQ == 1: LDS operations of a wave stay in order, the last chunk's reads are behind it)
        if (NQ == 1 || c < c_end) {
#pragma unroll
            for (int u = 0; u < NV; ++u)
                if (gt + GT * u < nvec) *(u32x4*)(vs + vdst[u]) = vreg[u];
        }
        if constexpr (NQ > 1) {
            __syncthreads();
            if (c + NK < c_end) fetch(c + NK);     // in flight while this chunk is multiplied
            __builtin_amdgcn_sched_barrier(0);
            if (!mine) continue;
        }

        // S^T chunk: rows = keys (KT tiles of 32), cols = queries
        f32x16 sacc[KT];
#pragma unroll
        for (int kt = 0; kt < KT; ++kt) {
#pragma unroll
            for (int r = 0; r < 16; ++r) sacc[kt][r] = 0.0f;
            if constexpr (NQ == 1) {
                if (k_tail) kreg[kt * DK + DK - 1] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
                for (int s = 0; s < DK; ++s)
                    Mma16<T>::run(as_uint4(kreg[kt * DK + s]), as_uint4(Q_LDS ? *(const u32x4*)(qs + s * 1024 + lane * 16) : qf[s]), sacc[kt]);
            } else {
                // all K fragments of the tile first (independent LDS reads, one latency), then the MFMAs
                u32x4 kf[DK];
#pragma unroll
                for (int s = 0; s < DK; ++s)
                    kf[s] = *(const u32x4*)(ks + (kt * 32 + l32) * k_stride + (16 * s + 8 * half) * 2);
#pragma unroll
                for (int s = 0; s < DK; ++s) Mma16<T>::run(as_uint4(kf[s]), as_uint4(qf[s]), sacc[kt]);
            }
        }
        if constexpr (NQ == 1)
            if (c + NK < c_end) fetch(c + NK);     // in flight during the softmax and the second product
        __builtin_amdgcn_sched_barrier(0);         // (kept above them: the scheduler would sink the loads)
        // online softmax; of tile kt this lane holds keys 8*(r/4) + 4*half + r%4 of its query
        if (t0 + KCH > a.T) {                      // the chunk that holds the end of the keys
#pragma unroll
            for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int key = t0 + kt * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
                    if (key >= a.T) sacc[kt][r] = -INFINITY;
                }
        }
        float mr = sacc[0][0];                     // raw logits: the scale (>= 0) goes into the exponent
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
#pragma unroll
            for (int r = 0; r < 16; ++r) mr = fmaxf(mr, sacc[kt][r]);
        mr = fmaxf(mr, __shfl_xor(mr, 32));
        const float mx = fmaxf(m_run, mr * a.scale_log2e);
        // (logits of -inf, keys taken out of the map: a share of the keys may hold no others, and then nothing is subtracted,
        // so that its probabilities are exp2(-inf) = 0 and not exp2(inf - inf), however the keys are cut)
        const float m_sub = mx == -INFINITY ? 0.0f : mx;
        if (__builtin_amdgcn_ballot_w64(mx != m_run) != 0ull) {     // some query's maximum moved
            const float alpha = __builtin_amdgcn_exp2f(m_run - m_sub);  // first chunk: exp2(-inf) = 0
            m_run = mx;
            l_run *= alpha;
#pragma unroll
            for (int nt = 0; nt < DT; ++nt)
#pragma unroll
                for (int r = 0; r < 16; ++r) oacc[nt][r] *= alpha;
        }
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                sacc[kt][r] = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[kt][r], a.scale_log2e, -m_sub));

        // O^T += V^T P^T, two steps of 16 keys per tile; step s uses registers 8s..8s+7.
        // The probabilities enter this product in the storage type.  fp16 keeps 11 bits of a
        // probability; bf16 keeps 8, too few for the stated tolerance on rows spread over many keys,
        // so there a probability goes in as the sum of two bf16 numbers (the rounded value and the
        // rounded remainder, 16 bits together) and the same V^T fragments are multiplied twice.
        // The row's denominator sums what the product multiplies with: through the row of ones (ODD),
        // else here - the rounded fp16 values, or for bf16 the unrounded ones (which the two terms
        // match to 2^-16) - so that numerator and denominator carry the same rounding and a row
        // dominated by one key returns that key's value row.  With the row of ones fp16 may even
        // truncate (one instruction per pair): the truncation is in both.
        constexpr bool TWO = std::is_same<T, bf16>::value;
        float lsum = 0.0f;
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                uint32_t ph[4], pl[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float p0 = sacc[kt][8 * s + 2 * j], p1 = sacc[kt][8 * s + 2 * j + 1];
                    if constexpr (TWO) {
                        ph[j] = pack2_rne<T>(p0, p1);
                        const float h0 = __uint_as_float(ph[j] << 16), h1 = __uint_as_float(ph[j] & 0xffff0000u);
                        pl[j] = pack2_rne<T>(p0 - h0, p1 - h1);
                        if constexpr (!ODD) lsum += p0 + p1;
                    } else if constexpr (ODD) {
                        union { decltype(__builtin_amdgcn_cvt_pkrtz(0.f, 0.f)) v; uint32_t u; } r;
                        r.v = __builtin_amdgcn_cvt_pkrtz(p0, p1);
                        ph[j] = r.u;
                    } else {
                        union { f16x2 v; uint32_t u; } r;
                        r.u = ph[j] = pack2_rne<T>(p0, p1);
                        lsum += (float)r.v.x + (float)r.v.y;
                    }
                }
                const uint4 pf = make_uint4(ph[0], ph[1], ph[2], ph[3]);
                s16x4 lo[DT], hi[DT];                        // the V^T fragments of all tiles, then the MFMAs
#pragma unroll
                for (int nt = 0; nt < DT; ++nt) {
                    lo[nt] = read_v(kt * 32 + 16 * s, nt);
                    hi[nt] = read_v(kt * 32 + 16 * s + 8, nt);
                }
#pragma unroll
                for (int nt = 0; nt < DT; ++nt) {
                    union { s16x4 h[2]; uint4 u; } vf;
                    vf.h[0] = lo[nt];
                    vf.h[1] = hi[nt];
                    Mma16<T>::run(vf.u, pf, oacc[nt]);
                    if constexpr (TWO) Mma16<T>::run(vf.u, make_uint4(pl[0], pl[1], pl[2], pl[3]), oacc[nt]);
                }
            }
        l_run += lsum;
    }

    float l_tot;
    if constexpr (ODD) {
        // row d of O^T (in the last tile: row 8 or 16, held by the lower half of the wave in register 4 or 8)
        const float ones = (d & 31) == 8 ? oacc[DT - 1][4] : oacc[DT - 1][8];
        l_tot = __shfl(ones, l32);
    } else {
        l_tot = l_run + __shfl_xor(l_run, 32);
    }
    // no other wave has keys of these queries: straight from the registers
    if (NK == 1 || a.chunks_per_split == 1) {
        if (!q_ok || wk != 0) return;
        const float inv = 1.0f / l_tot;
        float* const w = a.ws + (((long)blockIdx.z * a.heads + head) * a.Nq + qi) * (d + 4);
        if (a.splits > 1 && half == 0) *(float2*)(w + d) = make_float2(m_run, l_tot);
#pragma unroll
        for (int nt = 0; nt < DT; ++nt)
#pragma unroll
            for (int rq = 0; rq < 4; ++rq) {
                const int dd = nt * 32 + 8 * rq + 4 * half;
                if (dd >= d) continue;
                if (a.splits == 1) {
                    union { uint2 u; T h[4]; } x;
#pragma unroll
                    for (int e = 0; e < 4; ++e) x.h[e] = from_f32<T>(oacc[nt][4 * rq + e] * inv);
                    *(uint2*)((char*)a.o + ((long)qi * a.o_ld + head * d + dd) * 2) = x.u;
                } else {
                    *(float4*)(w + dd) = make_float4(oacc[nt][4 * rq], oacc[nt][4 * rq + 1], oacc[nt][4 * rq + 2],
                                                     oacc[nt][4 * rq + 3]);
                }
            }
        return;
    }
    // the waves' shares of the keys, brought to a common maximum and added in wave order
    float* const comb = reinterpret_cast<float*>(lds);       // [NK][32 * NQ queries][d sums, maximum, denominator, 2 unused]
    const int cs = d + 4;
    __syncthreads();                                         // (V rows no longer needed)
    {
        float* const mine = comb + ((wk * NQ + wq) * 32 + l32) * cs;
        if (half == 0) *(float2*)(mine + d) = make_float2(m_run, l_tot);
#pragma unroll
        for (int nt = 0; nt < DT; ++nt)
#pragma unroll
            for (int rq = 0; rq < 4; ++rq) {
                const int dd = nt * 32 + 8 * rq + 4 * half;
                if (dd < d)
                    *(float4*)(mine + dd) = make_float4(oacc[nt][4 * rq], oacc[nt][4 * rq + 1], oacc[nt][4 * rq + 2],
                                                        oacc[nt][4 * rq + 3]);
            }
    }
    __syncthreads();
    const int dq = d >> 2;
    for (int e = tid; e < 32 * NQ * dq; e += 64 * NW) {
        int q, g;
        divmod(e, a.d_dq, q, g);
        const int qq = blockIdx.x * (32 * NQ) + q;
        if (qq >= a.Nq) break;
        const float* const src = comb + q * cs;
        float m = -INFINITY;
        float2 ml[NK];
#pragma unroll
        for (int w = 0; w < NK; ++w) {
            ml[w] = *(const float2*)(src + w * (32 * NQ) * cs + d);
            m = fmaxf(m, ml[w].x);
        }
        const float m_sub = m == -INFINITY ? 0.0f : m;               // (no wave has a finite logit)
        float den = 0.0f;
        float4 num = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int w = 0; w < NK; ++w) {
            const float4 v = *(const float4*)(src + w * (32 * NQ) * cs + 4 * g);
            const float f = __builtin_amdgcn_exp2f(ml[w].x - m_sub); // a wave without keys: exp2(-inf) = 0
            num.x += v.x * f; num.y += v.y * f; num.z += v.z * f; num.w += v.w * f;
            den += ml[w].y * f;
        }
        if (a.splits == 1) {
            const float inv = 1.0f / den;
            union { uint2 u; T h[4]; } x;
            x.h[0] = from_f32<T>(num.x * inv); x.h[1] = from_f32<T>(num.y * inv);
            x.h[2] = from_f32<T>(num.z * inv); x.h[3] = from_f32<T>(num.w * inv);
            *(uint2*)((char*)a.o + ((long)qq * a.o_ld + head * d + 4 * g) * 2) = x.u;
        } else {
            float* const w = a.ws + (((long)blockIdx.z * a.heads + head) * a.Nq + qq) * cs;
            if (g == 0) *(float2*)(w + d) = make_float2(m, den);
            *(float4*)(w + 4 * g) = num;
        }
    }
}

// Single precision (the precision the paper's experiments run in, Sec. 4.1 "Implementation details"):
// the same transposed products on v_mfma_f32_32x32x2_f32, whose operands are one value per lane, so
// nothing is rounded between the two products and V needs no transpose (a lane picks V[key][d]
// itself).  A workgroup of NW waves holds its 32 * NW query rows in LDS (row stride d + 1 words, so
// that the lanes of a half fall on different banks) and stages 32 keys per chunk.
template <int DT, int NW>
__global__ __launch_bounds__(64 * NW) void attn_f32_kernel(AttnArgs a)
{
    constexpr int NT = 64 * NW;
    constexpr int KCH = 32;
    constexpr int VS = DT * 32 + 4;                // words per staged V row (columns d .. DT*32 stay zero)
    constexpr int NV = (8 * DT * 32 + NT - 1) / NT; // 16-byte vectors of K (and of V) a thread stages per chunk, at most
    extern __shared__ uint4 lds4[];
    float* lds = reinterpret_cast<float*>(lds4);
    const int d = a.d;
    const int rs = d + 1;                          // words per staged Q or K row
    float* qsm = lds;                              // [NW*32][rs]
    float* ksm = qsm + NW * 32 * rs;               // [KCH][rs]
    float* vsm = ksm + KCH * rs;                   // [KCH][VS]

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int half = lane >> 5, l32 = lane & 31;
    const int head = blockIdx.y;
    const int q0 = blockIdx.x * (NW * 32);
    const int qi = q0 + wave * 32 + l32;
    const bool q_ok = qi < a.Nq;
    const int dvec = d / 4;

    const int chunks_total = (a.T + KCH - 1) / KCH;
    const int c_begin = blockIdx.z * a.chunks_per_split;
    const int c_end = min(c_begin + a.chunks_per_split, chunks_total);

    // the workgroup's query rows (rows past Nq are zero)
    for (int j = tid; j < NW * 32 * dvec; j += NT) {
        const int row = j / dvec, dv = j - row * dvec;
        const int qq = q0 + row;
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (qq < a.Nq) {
            long qrow = qq;
            if (a.q_blocks != nullptr) {
                const int b = qq / a.q_tpb, p = qq - b * a.q_tpb;
                const int py = p / a.q_bw, px = p - py * a.q_bw;
                const int y0 = a.q_blocks[2 * b], x0 = a.q_blocks[2 * b + 1];
                qrow = (long)min(max(y0 + py, 0), a.q_H - 1) * a.q_W + min(max(x0 + px, 0), a.q_W - 1);
            }
            v = *(const float4*)((const float*)a.q + qrow * a.q_ld + head * d + dv * 4);
        }
        float* dst = qsm + row * rs + dv * 4;
        dst[0] = v.x; dst[1] = v.y; dst[2] = v.z; dst[3] = v.w;
    }
    for (int j = tid; j < KCH * (VS - d); j += NT) {
        const int key = j / (VS - d), c = j - key * (VS - d);
        vsm[key * VS + d + c] = 0.0f;
    }

    int skey[NV], sdv[NV];
#pragma unroll
    for (int u = 0; u < NV; ++u) {
        const int j = tid + u * NT;
        skey[u] = j < KCH * dvec ? j / dvec : -1;
        sdv[u] = j < KCH * dvec ? j - skey[u] * dvec : 0;
    }
    float4 kreg[NV], vreg[NV];
    auto fetch = [&](int c) {
        const int t0 = c * KCH;
#pragma unroll
        for (int u = 0; u < NV; ++u) {
            if (skey[u] < 0) continue;
            const long off = (long)min(t0 + skey[u], a.T - 1) * a.kv_ld + head * d + sdv[u] * 4;
            kreg[u] = *(const float4*)((const float*)a.k + off);
            vreg[u] = *(const float4*)((const float*)a.v + off);
        }
    };
    auto commit = [&](int c) {
        const int t0 = c * KCH;
#pragma unroll
        for (int u = 0; u < NV; ++u) {
            if (skey[u] < 0) continue;
            const bool in = t0 + skey[u] < a.T;
            const float4 kv = in ? kreg[u] : make_float4(0.f, 0.f, 0.f, 0.f);
            const float4 vv = in ? vreg[u] : make_float4(0.f, 0.f, 0.f, 0.f);
            float* kd = ksm + skey[u] * rs + sdv[u] * 4;
            kd[0] = kv.x; kd[1] = kv.y; kd[2] = kv.z; kd[3] = kv.w;
            *(float4*)(vsm + skey[u] * VS + sdv[u] * 4) = vv;
        }
    };

    f32x16 oacc[DT];
#pragma unroll
    for (int nt = 0; nt < DT; ++nt)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[nt][r] = 0.0f;
    float m_run = -INFINITY, l_run = 0.0f;
    const float* qrow_s = qsm + (wave * 32 + l32) * rs + half;
    const float* krow_s = ksm + l32 * rs + half;

    if (c_begin < c_end) fetch(c_begin);
    for (int c = c_begin; c < c_end; ++c) {
        const int t0 = c * KCH;
        __syncthreads();  // previous chunk fully consumed (and, the first time, the query rows written)
        commit(c);
        __syncthreads();
        if (c + 1 < c_end) fetch(c + 1);

        // S^T tile: rows = the chunk's 32 keys, cols = this wave's 32 queries; two values of d per MFMA
        f32x16 sacc;
#pragma unroll
        for (int r = 0; r < 16; ++r) sacc[r] = 0.0f;
        for (int j = 0; j < d; j += 4) {              // d is a multiple of 4
            const float k0 = krow_s[j], q0v = qrow_s[j], k1 = krow_s[j + 2], q1v = qrow_s[j + 2];
            sacc = __builtin_amdgcn_mfma_f32_32x32x2f32(k0, q0v, sacc, 0, 0, 0);
            sacc = __builtin_amdgcn_mfma_f32_32x32x2f32(k1, q1v, sacc, 0, 0, 0);
        }
        // online softmax; this lane holds keys 8*(r/4) + 4*half + r%4 of its query
        float mx = m_run;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int key = t0 + 8 * (r >> 2) + 4 * half + (r & 3);
            sacc[r] = key < a.T ? sacc[r] * a.scale_log2e : -INFINITY;
            mx = fmaxf(mx, sacc[r]);
        }
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        const float alpha = exp2f(m_run - mx);
        float lsum = 0.0f;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            sacc[r] = exp2f(sacc[r] - mx);
            lsum += sacc[r];
        }
        l_run = l_run * alpha + lsum;
        m_run = mx;
#pragma unroll
        for (int nt = 0; nt < DT; ++nt)
#pragma unroll
            for (int r = 0; r < 16; ++r) oacc[nt][r] *= alpha;
        // O^T += V^T P^T: register r of the two lane halves is one pair of keys
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float* vrow = vsm + (8 * (r >> 2) + 4 * half + (r & 3)) * VS + l32;
#pragma unroll
            for (int nt = 0; nt < DT; ++nt)
                oacc[nt] = __builtin_amdgcn_mfma_f32_32x32x2f32(vrow[nt * 32], sacc[r], oacc[nt], 0, 0, 0);
        }
    }

    const float l_tot = l_run + __shfl_xor(l_run, 32);
    if (!q_ok) return;
    if (a.splits == 1) {
        const float inv = 1.0f / l_tot;
#pragma unroll
        for (int nt = 0; nt < DT; ++nt)
#pragma unroll
            for (int rq = 0; rq < 4; ++rq) {
                const int dd = nt * 32 + 8 * rq + 4 * half;
                if (dd < d)
                    *(float4*)((float*)a.o + (long)qi * a.o_ld + head * d + dd) =
                        make_float4(oacc[nt][4 * rq] * inv, oacc[nt][4 * rq + 1] * inv, oacc[nt][4 * rq + 2] * inv,
                                    oacc[nt][4 * rq + 3] * inv);
            }
    } else {
        float* w = a.ws + (((long)blockIdx.z * a.heads + head) * a.Nq + qi) * (d + 4);
        if (half == 0) *(float2*)(w + d) = make_float2(m_run, l_tot);
#pragma unroll
        for (int nt = 0; nt < DT; ++nt)
#pragma unroll
            for (int rq = 0; rq < 4; ++rq) {
                const int dd = nt * 32 + 8 * rq + 4 * half;
                if (dd < d)
                    *(float4*)(w + dd) = make_float4(oacc[nt][4 * rq], oacc[nt][4 * rq + 1], oacc[nt][4 * rq + 2],
                                                     oacc[nt][4 * rq + 3]);
            }
    }
}

// Merge of the per-split partials.  P neighbouring lanes share one (query, head, four consecutive d
// elements): lane p takes splits p, p + P, p + 2P, p + 3P - all of its loads are in flight together, one
// round trip to memory however many splits there are - and the P partial (maximum, denominator, sums)
// triples are combined with a butterfly of lane exchanges, each step rescaling to the common maximum as
// the attention kernel does.  The order of the sums is fixed by (P, splits): results are reproducible.
template <typename T, int P>
__global__ __launch_bounds__(256) void attn_merge_kernel(AttnArgs a)
{
    constexpr int B = 4;                           // splits per lane, at most (the host picks P accordingly)
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    const int d = a.d, dq = d >> 2;
    const long grp = i / P;
    const int sub = (int)(i % P);
    const bool live = grp < (long)a.Nq * a.heads * dq;      // (whole groups: P divides the workgroup size)
    const long g = live ? grp : 0;
    const int dd = (int)(g % dq) * 4;
    const int head = (int)((g / dq) % a.heads);
    const int qi = (int)(g / ((long)dq * a.heads));
    const long sstride = (long)a.heads * a.Nq * (d + 4);
    const float* w0 = a.ws + ((long)head * a.Nq + qi) * (d + 4);
    float2 ml[B];
    float4 val[B];
#pragma unroll
    for (int j = 0; j < B; ++j) {
        const float* w = w0 + min(sub + j * P, a.splits - 1) * sstride;
        ml[j] = *(const float2*)(w + d);
        val[j] = *(const float4*)(w + dd);
    }
    float m = -INFINITY;
#pragma unroll
    for (int j = 0; j < B; ++j)
        if (sub + j * P < a.splits) m = fmaxf(m, ml[j].x);
    float den = 0.0f, num[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int j = 0; j < B; ++j) {
        const float f = sub + j * P < a.splits && ml[j].x != -INFINITY ? exp2f(ml[j].x - m) : 0.0f;
        num[0] += val[j].x * f; num[1] += val[j].y * f; num[2] += val[j].z * f; num[3] += val[j].w * f;
        den += ml[j].y * f;
    }
#pragma unroll
    for (int x = 1; x < P; x <<= 1) {
        const float m2 = __shfl_xor(m, x), den2 = __shfl_xor(den, x);
        float n2[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) n2[e] = __shfl_xor(num[e], x);
        const float mm = fmaxf(m, m2);
        // a lane without splits carries (-inf, 0, 0): its weight is 0, not exp2(-inf + inf)
        const float f1 = m == -INFINITY ? 0.0f : exp2f(m - mm), f2 = m2 == -INFINITY ? 0.0f : exp2f(m2 - mm);
        // both partners add in the same order (lower lane's share first), so they hold the same bits
        const bool low = (sub & x) == 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) num[e] = low ? num[e] * f1 + n2[e] * f2 : n2[e] * f2 + num[e] * f1;
        den = low ? den * f1 + den2 * f2 : den2 * f2 + den * f1;
        m = mm;
    }
    if (!live || sub != 0) return;
    T* o = (T*)a.o + (long)qi * a.o_ld + head * d + dd;
    const float inv = 1.0f / den;
    if constexpr (sizeof(T) == 4) {
        *(float4*)o = make_float4(num[0] * inv, num[1] * inv, num[2] * inv, num[3] * inv);
    } else {
        union { uint2 u; T h[4]; } x;
#pragma unroll
        for (int e = 0; e < 4; ++e) x.h[e] = from_f32<T>(num[e] * inv);
        *(uint2*)o = x.u;
    }
}

template <typename T>
static int launch_merge(const AttnArgs& a, hipStream_t st)
{
    const long groups = (long)a.Nq * a.heads * (a.d / 4);
    auto go = [&](auto kern, int P) {
        hipLaunchKernelGGL(kern, dim3((int)((groups * P + 255) / 256)), dim3(256), 0, st, a);
    };
    if (a.splits <= 4) go(attn_merge_kernel<T, 1>, 1);
    else if (a.splits <= 16) go(attn_merge_kernel<T, 4>, 4);
    else go(attn_merge_kernel<T, 16>, 16);          // at most 64 splits
    SIGE_LAUNCH_CHECK("sige_sparse_attn(merge)");
    return SIGE_OK;
}

// How a call is cut.  Single precision: a workgroup (128 queries) walks through its key chunks one after the other and each
// costs a staging round trip, so few queries are spread over about two workgroups per compute unit (more
// splits cost the merge kernel more than they save: measured at 64 to 1280 queries), at least 2 chunks each.
// Half types: the cheapest of three forms and their splits over workgroups by a model of measured times (1400 calls of 24 to 4000
// queries on 77 to 9216 keys, heads of 24 to 256, one to eight of them, each form with every number of splits near its
// best: 18000 times; the choice takes 1.01 times the best of them in the mean, 1.2 at worst; of the times before waves split the keys it makes 0.83 in the mean and 1.14 at worst, the model of 24 calls made 0.87 and 1.30).  What it trades:
// four waves on the same chunks fetch them once; waves with chunks of their own have no barriers and no partial sums for a merge kernel
// (3 us, and 2.75 per million of them; half a microsecond more is asked of a split, since the sum is right to about that: of 2500 calls 123
// instead of 146 then take more than 5 % longer than the better of both) where a call has enough queries to fill the chip, but fetch K in pieces of 32 bytes of a row, which
// costs more where the rows of a head are not side by side.
struct AttnForm { int nq, nk, splits; };           // waves with the same chunks, key groups, splits over workgroups
// room: floats of workspace, what the splits' partial sums have to fit into.
static AttnForm plan_attn(int Nq, int T, int heads, int d, sige_dtype dt, size_t room = ~(size_t)0)
{
    const int KCH = keys_per_chunk(d, dt);
    const int chunks = (T + KCH - 1) / KCH;
    const int target = knob(SIGE_KNOB_ATTN_WGS);            // workgroups to aim for
    AttnForm f = {4, 1, 1};
    if (dt == SIGE_F32) {
        const long base = (long)heads * ((Nq + 127) / 128);
        long want = ((target >= 0 ? target : 512) + base - 1) / base;
        long cap = chunks / 2;
        if (want > cap) want = cap;
        if (want > 64) want = 64;
        if (want < 1) want = 1;
        const int per = (int)((chunks + want - 1) / want);
        f.splits = (chunks + per - 1) / per;
        if (f.splits > 1 && (size_t)f.splits * heads * Nq * (d + 4) > room) f.splits = 1;
        return f;
    }
    // by 16-wide steps over a head and form (four waves with the same chunks; one wave each, four of them; eight): microseconds of a
    // workgroup beside its chunks, per chunk of a wave, and what several heads add to that; workgroups that a compute unit holds, by
    // registers and LDS.  0: not built (heads of 88 or 96 in eight waves do not have the registers; four waves of their own on heads of 97
    // to 128 are never the cheapest)
    static const float fixed_us[17][3] = {{}, {3.72f, 3.09f, 3.54f}, {3.72f, 3.09f, 3.54f}, {2.86f, 4.16f, 4.19f}, {2.74f, 4.87f, 3.81f}, {3.59f, 6.14f, 3.76f},
                                              {3.86f, 5.96f, 0}, {3.4f, 0, 5.04f}, {3.09f, 0, 5.24f}, {4.45f, 6.89f, 0}, {3.68f, 6.28f, 0},
                                              {3.49f, 6.04f, 0}, {3.8f, 5.99f, 0}, {3.5f, 6.23f, 0}, {4.01f, 8.08f, 0}, {3.76f, 8.23f, 0}, {4.69f, 9.86f, 0}};
    static const float chunk_us[17][3] = {{}, {1.23f, 0.85f, 0.96f}, {1.23f, 0.85f, 0.96f}, {1.53f, 1.19f, 1.56f}, {2.06f, 1.66f, 3.56f}, {1.83f, 1.72f, 2.81f},
                                              {2.98f, 2.22f, 0}, {1.3f, 0, 2.07f}, {1.14f, 0, 2.8f}, {2.32f, 1.69f, 0}, {2.18f, 1.55f, 0},
                                              {2.26f, 1.63f, 0}, {2.19f, 2.3f, 0}, {2.71f, 2.1f, 0}, {3.18f, 1.78f, 0}, {2.77f, 2.78f, 0}, {2.24f, 2.68f, 0}};
    static const float heads_us[17][3] = {{}, {0.35f, 0.7f, 0.78f}, {0.35f, 0.7f, 0.78f}, {0.06f, 0.61f, 1.21f}, {0.04f, 0.28f, 0.92f}, {1.33f, 1.6f, 3.47f},
                                              {0, 0.99f, 0}, {0.51f, 0, 2.41f}, {0.11f, 0, 0.6f}, {0.14f, 0.21f, 0}, {0.35f, 0.49f, 0},
                                              {0.44f, 0.51f, 0}, {0.62f, 0.7f, 0}, {0.16f, 0.73f, 0}, {1.18f, 1.25f, 0}, {0.47f, 2.15f, 0}, {0.07f, 1.03f, 0}};
    static const signed char held[9][3] = {{}, {2, 4, 2}, {2, 3, 1}, {2, 2, 1}, {1, 2, 1}, {1, 1, 1}, {1, 1, 1}, {3, 1, 1}, {2, 1, 1}};      // (one of each beyond)
    const int DT = (d + 31) / 32, DK = (d + 15) / 16;
    double best_us = 1e30;
    for (int form = 0; form < 3; ++form) {
        if (fixed_us[DK][form] == 0.0f) continue;
        if (form > 0 && chunks == 1 && DT <= 3 && target < 0) continue;      // (one wave works either way: 300 calls, the common form 3 - 35 % faster)
        const AttnForm g = form == 0 ? AttnForm{4, common_groups(DT), 1} : AttnForm{1, form == 1 ? 4 : 8, 1};
        const long base = (long)heads * ((Nq + 32 * g.nq - 1) / (32 * g.nq));
        const int r = DK > 8 ? 1 : held[DK][form];
        for (int z = 1; z <= 64 && (z == 1 || z * g.nk <= chunks); ++z) {
            const int per = (chunks + z - 1) / z, real = (chunks + per - 1) / per;
            if (real > 1 && (size_t)real * heads * Nq * (d + 4) > room) break;
            const long on_one = (base * real + 255) / 256;      // workgroups of the fullest compute unit
            const double chunk = (per + g.nk - 1) / g.nk * (chunk_us[DK][form] + (heads > 1 ? heads_us[DK][form] : 0.0f));
            // workgroups side by side lengthen each other's chunks; the fixed part of the next ones runs beside the chunks of those before
            const double us = fixed_us[DK][form] * (1.0 + 0.5 * ((on_one + r - 1) / r - 1)) + on_one / r * chunk * (1.0 + 0.4 * (r - 1)) +
                              (on_one % r ? chunk * (1.0 + 0.4 * (on_one % r - 1)) : 0.0);
            const double merge = real == 1 ? 0.0 : (real > 16 ? 3.8 : 3.5) + 2.75e-6 * real * heads * Nq * (d + 4);
            const double cost = target >= 0 ? std::abs(target - (double)base * real) : us + merge;
            if (cost < best_us) { best_us = cost; f = g; f.splits = real; }
        }
    }
    return f;
}

template <typename T, int DT, int NQ, int NK, bool FAR = false>
static int launch_attn_dt(AttnArgs a, hipStream_t st)
{
    constexpr int KCH = 32 * key_tiles(DT);
    // one chunk: the first of several groups of four waves is the workgroup (f16, 5664 queries x 8 heads of 96 on 32 keys 12.5 -> 9.2 us,
    // 994 x 1 of 64 on 64 5.2 -> 4.4)
    a.groups = NQ > 1 && a.chunks_per_split == 1 ? 1 : NK;
    const size_t lds = std::max((size_t)a.groups * KCH * (v_row_bytes(DT) + (NQ > 1 ? (FAR ? 32 * DT : a.d) * 2 + 16 : 0)) +
                                    (q_in_lds(DT, NQ) ? 2 * DT * 1024 : 0),
                                a.groups == 1 ? 0 : (size_t)NK * NQ * 32 * (a.d + 4) * sizeof(float));
    dim3 grid((a.Nq + 32 * NQ - 1) / (32 * NQ), a.heads, a.splits);
    const bool odd = ((a.d + 15) / 16) & 1;        // d % 32 is 8 or 16
    auto kern = attn_kernel<T, DT, !FAR, NQ, NK, FAR>;
    if constexpr (!FAR && (DT != 3 || NK != 8)) {
        if (!odd) kern = attn_kernel<T, DT, 0, NQ, NK>;
    } else if constexpr (!FAR) {
        SIGE_REQUIRE(odd, SIGE_ERR_UNSUPPORTED, "sige_sparse_attn: internal: eight waves on heads of %d", a.d);
    }
    if (lds > 48 * 1024) {
        hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        SIGE_REQUIRE(e == hipSuccess, SIGE_ERR_HIP, "sige_sparse_attn: cannot reserve %zu bytes of LDS: %s", lds,
                     hipGetErrorString(e));
    }
    hipLaunchKernelGGL(kern, grid, dim3(64 * NQ * a.groups), lds, st, a);
    SIGE_LAUNCH_CHECK("sige_sparse_attn");
    if (a.splits > 1) return launch_merge<T>(a, st);
    return SIGE_OK;
}

template <typename T, int DT>
static int launch_attn_form(const AttnArgs& a, const AttnForm& f, hipStream_t st)
{
    if (f.nq == 4) return launch_attn_dt<T, DT, 4, common_groups(DT)>(a, st);
    if constexpr (max_waves(DT) == 8)
        if (f.nk == 8) return launch_attn_dt<T, DT, 1, 8>(a, st);
    if constexpr (DT != 4) return launch_attn_dt<T, DT, 1, 4>(a, st);
    return fail(SIGE_ERR_UNSUPPORTED, "sige_sparse_attn: internal: four waves of their own on heads of %d", a.d);
}

// One instantiation per number of 32-wide tiles: the steps over d, the spare columns of V and the tile that holds the column of ones
// all follow from it.
template <typename T>
static int launch_attn(const AttnArgs& a, const AttnForm& f, hipStream_t st)
{
    const int dt = (a.d + 31) / 32;
    switch (dt) {
    case 1: return launch_attn_form<T, 1>(a, f, st);
    case 2: return launch_attn_form<T, 2>(a, f, st);
    case 3: return launch_attn_form<T, 3>(a, f, st);
    case 4: return launch_attn_form<T, 4>(a, f, st);
    case 5: return launch_attn_form<T, 5>(a, f, st);
    case 6: return launch_attn_form<T, 6>(a, f, st);
    case 7: return launch_attn_form<T, 7>(a, f, st);
    default: return launch_attn_form<T, 8>(a, f, st);
    }
}

template <int DT, int NW>
static int launch_attn_f32_as(const AttnArgs& a, hipStream_t st)
{
    const size_t lds = ((size_t)(NW * 32 + 32) * (a.d + 1) + 32 * (DT * 32 + 4)) * sizeof(float);
    dim3 grid((a.Nq + NW * 32 - 1) / (NW * 32), a.heads, a.splits);
    auto kern = attn_f32_kernel<DT, NW>;
    if (lds > 48 * 1024) {
        hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        SIGE_REQUIRE(e == hipSuccess, SIGE_ERR_HIP, "sige_sparse_attn: cannot reserve %zu bytes of LDS: %s", lds,
                     hipGetErrorString(e));
    }
    hipLaunchKernelGGL(kern, grid, dim3(64 * NW), lds, st, a);
    SIGE_LAUNCH_CHECK("sige_sparse_attn");
    if (a.splits > 1) return launch_merge<float>(a, st);
    return SIGE_OK;
}

// Four waves (128 queries) per workgroup while their rows, the key chunk and the value chunk fit
// the LDS of a compute unit, two beyond (heads wider than 128).
static int launch_attn_f32(const AttnArgs& a, hipStream_t st)
{
    switch ((a.d + 31) / 32) {
    case 1: return launch_attn_f32_as<1, 4>(a, st);
    case 2: return launch_attn_f32_as<2, 4>(a, st);
    case 3: return launch_attn_f32_as<3, 4>(a, st);
    case 4: return launch_attn_f32_as<4, 4>(a, st);
    case 5: return launch_attn_f32_as<5, 2>(a, st);
    case 6: return launch_attn_f32_as<6, 2>(a, st);
    default: return launch_attn_f32_as<8, 2>(a, st);
    }
}

}  // namespace sige

using namespace sige;

extern "C" size_t sige_sparse_attn_workspace_bytes(int32_t Nq, int32_t T, int32_t heads, int32_t d)
{
    if (Nq <= 0 || T <= 0 || heads <= 0 || d <= 0 || d > 256) return 0;     // (a head that no call takes has no plan)
    // the larger of what the half-precision and the single-precision kernels would use
    const int splits = std::max(plan_attn(Nq, T, heads, d, SIGE_F16).splits, plan_attn(Nq, T, heads, d, SIGE_F32).splits);
    if (splits <= 1) return 0;
    return (size_t)splits * heads * Nq * (d + 4) * sizeof(float);
}

static int attn_entry(const char* who, AttnArgs& a, const void* q, int32_t q_ld, const void* k, const void* v,
                      int32_t kv_ld, sige_dtype dt, int32_t Nq, int32_t T, int32_t heads, int32_t d, float scale,
                      void* o, int32_t o_ld, void* workspace, size_t workspace_bytes, void* stream)
{
    SIGE_REQUIRE(Nq >= 0 && T > 0 && heads > 0 && d > 0, SIGE_ERR_INVALID_ARG,
                 "%s: need Nq >= 0, T > 0, heads > 0, d > 0", who);
    SIGE_REQUIRE(dtype_ok(dt), SIGE_ERR_INVALID_ARG, "%s: unknown dtype %d", who, (int)dt);
    const int vw = dt == SIGE_F32 ? 4 : 8;                  // elements per 16-byte vector
    SIGE_REQUIRE(d % vw == 0 && d <= 256, SIGE_ERR_UNSUPPORTED, "%s: d must be a multiple of %d and <= 256", who, vw);
    SIGE_REQUIRE(heads <= 65535, SIGE_ERR_UNSUPPORTED, "%s: too many heads", who);
    if (Nq == 0) return SIGE_OK;
    SIGE_REQUIRE(q && k && v && o, SIGE_ERR_INVALID_ARG, "%s: q, k, v and o are required", who);
    SIGE_REQUIRE(q_ld >= heads * d && kv_ld >= heads * d && o_ld >= heads * d, SIGE_ERR_INVALID_ARG,
                 "%s: row strides must be >= heads*d", who);
    SIGE_REQUIRE(q_ld % vw == 0 && kv_ld % vw == 0 && o_ld % vw == 0, SIGE_ERR_UNSUPPORTED,
                 "%s: row strides must be multiples of %d elements", who, vw);
    SIGE_REQUIRE(aligned16(q) && aligned16(k) && aligned16(v) && aligned16(o), SIGE_ERR_UNSUPPORTED,
                 "%s: pointers must be 16-byte aligned", who);
    a.q = q; a.k = k; a.v = v; a.o = o; a.ws = (float*)workspace;
    a.q_ld = q_ld; a.kv_ld = kv_ld; a.o_ld = o_ld;
    a.Nq = Nq; a.T = T; a.heads = heads; a.d = d;
    a.d_tpb = fast_div(a.q_tpb); a.d_qbw = fast_div(a.q_bw); a.d_dvec = fast_div(std::max(d / 8, 1)); a.d_dq = fast_div(d / 4);
    SIGE_REQUIRE(scale >= 0.0f, SIGE_ERR_UNSUPPORTED, "%s: the scale must not be negative", who);
    a.scale_log2e = scale * 1.4426950408889634f;
    // rows of a chunk too far apart for 32-bit offsets: a kernel of its own, cut like single precision (128 queries, 32 keys per chunk)
    const bool far = dt != SIGE_F32 && (std::min(T, keys_per_chunk(d, dt)) - 1) * (long)kv_ld * 2 + 2L * d > (1L << 32);
    const sige_dtype cut = far ? SIGE_F32 : dt;
    const int KCH = keys_per_chunk(d, cut);
    const int chunks = (T + KCH - 1) / KCH;
    const bool room = workspace != nullptr && (reinterpret_cast<uintptr_t>(workspace) & 15u) == 0;
    const AttnForm f = plan_attn(Nq, T, heads, d, cut, room ? workspace_bytes / sizeof(float) : 0);
    a.chunks_per_split = (chunks + f.splits - 1) / f.splits;
    a.splits = (chunks + a.chunks_per_split - 1) / a.chunks_per_split;
    hipStream_t st = (hipStream_t)stream;
    if (dt == SIGE_F32) return launch_attn_f32(a, st);
    if (far) return dt == SIGE_F16 ? launch_attn_dt<f16, 8, 4, 1, true>(a, st) : launch_attn_dt<bf16, 8, 4, 1, true>(a, st);
    return dt == SIGE_F16 ? launch_attn<f16>(a, f, st) : launch_attn<bf16>(a, f, st);
}

extern "C" int sige_sparse_attn(const void* q, int32_t q_ld, const void* k, const void* v, int32_t kv_ld,
                                sige_dtype dt, int32_t Nq, int32_t T, int32_t heads, int32_t d,
                                float scale, void* o, int32_t o_ld, void* workspace,
                                size_t workspace_bytes, void* stream)
{
    clear_error();
    AttnArgs a;
    a.q_blocks = nullptr;
    a.q_tpb = a.q_bw = a.q_H = a.q_W = 1;
    return attn_entry("sige_sparse_attn", a, q, q_ld, k, v, kv_ld, dt, Nq, T, heads, d, scale, o, o_ld, workspace,
                      workspace_bytes, stream);
}

extern "C" int sige_sparse_attn_blocks(const void* q, int32_t q_ld, const sige_geom* g, const int32_t* indices,
                                       int32_t n_blocks, const void* k, const void* v, int32_t kv_ld,
                                       sige_dtype dt, int32_t T, int32_t heads, int32_t d, float scale, void* o,
                                       int32_t o_ld, void* workspace, size_t workspace_bytes, void* stream)
{
    clear_error();
    const char* who = "sige_sparse_attn_blocks";
    SIGE_REQUIRE(g != nullptr, SIGE_ERR_INVALID_ARG, "%s: geometry is required", who);
    SIGE_REQUIRE(g->k == 1 && g->stride == 1 && g->pad == 0 && g->block_h > 0 && g->block_w > 0 && g->H_in > 0 &&
                     g->W_in > 0,
                 SIGE_ERR_UNSUPPORTED, "%s: the geometry must be that of a 1x1, stride-1, unpadded layer", who);
    SIGE_REQUIRE(n_blocks >= 0, SIGE_ERR_INVALID_ARG, "%s: n_blocks must be a host value >= 0", who);
    SIGE_REQUIRE((long)n_blocks * g->block_h * g->block_w <= 0x7fffffffL, SIGE_ERR_UNSUPPORTED,
                 "%s: too many query rows", who);
    if (n_blocks == 0) return SIGE_OK;
    SIGE_REQUIRE(indices != nullptr, SIGE_ERR_INVALID_ARG, "%s: indices are required", who);
    AttnArgs a;
    a.q_blocks = indices;
    a.q_tpb = g->block_h * g->block_w;
    a.q_bw = g->block_w;
    a.q_H = g->H_in;
    a.q_W = g->W_in;
    return attn_entry(who, a, q, q_ld, k, v, kv_ld, dt, n_blocks * a.q_tpb, T, heads, d, scale, o, o_ld, workspace,
                      workspace_bytes, stream);
}
