// One workgroup per (batch, tile of 256, 128 or 64 queries): S = scale * Q K^T, row softmax, O = P V, in one
// kernel.  Both contractions are tensorized blocks (Eq. 1 of the TensorIR paper, mapped onto the
// 32x32x16 MFMA) that share the workgroup's tile instead of meeting in memory: the probabilities never
// leave the registers (sec. 2 / 3.2: blocks isolate the two sub-problems, which does not prevent
// cooperation across them).  The softmax is the textbook one, computed online over chunks of 64 or 32 keys.
//
// Both products are computed transposed, S^T = K Q^T and O^T = V^T P^T, so that the second MFMA
// operand - whose row index is the lane - is the query in both: every lane then owns one query row,
// the row maximum / row sum are reductions over the lane's own registers plus one exchange between
// the two half-waves, rescaling O by exp(m_old - m_new) is a per-lane scalar multiply, and the
// probabilities come out of the first MFMA already in the register layout the second one reads them
// in (the k-order of an MFMA is free as long as both operands use the same one; V^T is fetched with
// the transposing LDS read in the order the probabilities happen to have).
#pragma once
#include "tir_kernel.h"

namespace tir {

struct AttnParams {
    const void* Q;   // [batch][M][D]
    const void* K;   // [batch][N][D]
    const void* V;   // [batch][N][D]
    void* O;         // [batch][M][D]
    int M, N, batch;
    int tiles_m;     // ceil(M / (32 * QW)), QW query waves per workgroup
    float scale_log2e;   // scale * log2(e): the softmax runs in base 2
    unsigned div_tm_magic;   // workgroup id / tiles_m as multiply-and-shift (make_fastdiv)
    int div_tm_shift;
    int store_nt;            // the output is not read again soon: non-temporal stores (see TIR_STORE_AUX_STREAM)
};

template <int DT> struct PackP;
template <> struct PackP<DT_F16> {
    static __device__ __forceinline__ unsigned two(float a, float b) {
        typedef _Float16 h2 __attribute__((ext_vector_type(2)));
        h2 v = {(_Float16)a, (_Float16)b};
        return __builtin_bit_cast(unsigned, v);
    }
};
template <> struct PackP<DT_BF16> {
    static __device__ __forceinline__ unsigned two(float a, float b) {
        typedef __bf16 b2 __attribute__((ext_vector_type(2)));
        b2 v = {(__bf16)a, (__bf16)b};          // one v_cvt_pk_bf16_f32
        return __builtin_bit_cast(unsigned, v);
    }
};

// DT: f16 / bf16 inputs, OUT: same 16-bit type or f32, DH: head dimension (64 or 128) of Q, K and V.
//
// 64 keys per chunk (KB): two stages of K and V and nothing else in LDS (64 KiB at d = 128), so that two workgroups share a CU.  A chunk's
// softmax is vector work about as long as its MFMAs, and a wave runs the two under each other: the exponentials of chunk i stand between
// the MFMAs of K Q^T of chunk i + 1, that chunk's row maxima between those of V^T P^T of chunk i, and the copy instructions of the chunk
// after between the former (a copy instruction holds its wave for longer than an MFMA lasts; all in front of a chunk cost 10 %).  Measured
// here: 32 MFMAs of 32 cycles with 128 multiply-adds and 32 exponentials between them take one wave 1 096 cycles, the MFMAs alone 1 038, the
// vector work alone 840.  With each wave's phases in sequence, left to a second wave to cover, 16 x 4096 x 4096 x 128 bf16 took 143.8 us, now
// 133.8 (128.3 with priorities and tiles of 256 queries); 160 x 128 x 2000 x 128 50.5 and 39.9, 52 x 376 x 376 x 64 9.3 and 7.7.  What bounds the long case is power: the same launch on constant data takes
// 103.5 us instead of 141.5 under the profiler, at 1.99 GHz instead of 1.68 and 8 % fewer cycles.
//
// QW waves of 32 queries times KG key groups: group k takes the chunks c with c % KG == k through a ring of its own and the
// groups' results are merged through LDS at the end.  Where the query tiles alone leave CUs or SIMDs idle, key groups put more waves
// on the same tile (attention_kernel_of gives the rule and both sides' times).
//
// FORM: the loop described above, plain or with non-temporal copies, or a chunk's phases in sequence.  The latter holds one chunk's scores instead of two: 109 to 112
// registers instead of 161 to 163 at d = 64, four workgroups per CU instead of three.
enum : int { ATTN_PIPED = 0, ATTN_PIPED_STREAM = 1, ATTN_SEQUENTIAL = 2 };
template <int DT, int OUT, int DH, int QW, int KG, int KB, int FORM>
__global__ void __launch_bounds__(QW * KG * 64, 2) attention_kernel(const AttnParams p) {
    typedef OutTraits<OUT> OT;
    typedef typename OT::type out_t;
    constexpr int OS = (int)sizeof(out_t);
    constexpr int TQ = QW * 32, GT = QW * 64;   // queries of a workgroup, threads of a key group
    constexpr int JB = KB / 32;                 // 32-key blocks of a chunk of KB keys
    constexpr int ROW = DH * 2;                 // bytes of one Q / K / V row
    constexpr int HALVES = DH / 64;             // 128-byte column groups of a K-major row
    constexpr int TILE = KB * ROW;              // one chunk of K or V
    constexpr int KSTEPS = DH / 16;             // MFMA k-steps over the head dimension
    constexpr int DB = DH / 32;                 // 32-wide blocks of the output's head dimension
    constexpr int VRC = ROW / 16;               // 16-byte chunks per V row
    constexpr int KROWS = GT / 8, KPASS = KB / KROWS;          // rows of K one copy instruction per wave covers (of one column group)
    constexpr int COPIES = TILE / (GT * 16);    // copy instructions per wave for one chunk of V
    constexpr int RING = 4 * TILE;              // one key group's two stages of K and V
    // V tile [key][ROW] with the transposing-read swizzle: byte offset XOR ((key / RPW) % NSEG) * 64
    constexpr int WIN = ROW < 256 ? ROW : 256;
    constexpr int NSEG = WIN / 64, RPW = 256 / WIN;
    constexpr int MERGE = DB * 4096 + 512;      // what a wave hands over: its accumulators, sums and references
    constexpr int LDS = RING * KG > TQ * DH * OS ? RING * KG : TQ * DH * OS;
    static_assert(DH == 64 || DH == 128, "head dimension");
    static_assert(KROWS % 16 == 0 && KPASS >= 1 && COPIES >= 1, "the K swizzle repeats every 16 rows");
    static_assert((KG - 1) * QW * MERGE <= LDS && LDS <= 160 * 1024, "");

    __shared__ __attribute__((aligned(1024))) char smem[LDS];

    const int lane = threadIdx.x & 63;
    const int wave_wg = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int kgrp = KG == 1 ? 0 : wave_wg / QW, wave = wave_wg - kgrp * QW;
    const int tid = (int)threadIdx.x - kgrp * GT;                // thread of the key group
    const int l31 = lane & 31, g = lane >> 5;
    const int blk = lane >> 4, s16 = lane & 15;
    char* const ring = smem + kgrp * RING;

    // Workgroups go to the 8 L2 domains round-robin by launch index: each domain gets a run of consecutive tiles, i.e. whole heads,
    // whose keys and values its L2 then holds once.
    const int nwg = p.batch * p.tiles_m;
    const int xq = nwg >> 3, xr = nwg & 7, xf = blockIdx.x & 7;
    const int bid = xf * xq + (xf < xr ? xf : xr) + (blockIdx.x >> 3);
    const long long b = fastdiv((unsigned)bid, p.div_tm_magic, p.div_tm_shift);
    const int tm = bid - (int)b * p.tiles_m;
    const int m0 = tm * TQ;
    const int rows_q = p.M - m0 < TQ ? p.M - m0 : TQ;
    const int nchunk = (p.N + KB - 1) / KB;
    const int nmine = (nchunk - kgrp + KG - 1) / KG;             // this group's chunks (chunk i of it is i * KG + kgrp)
    const int nloop = (nchunk + KG - 1) / KG;                    // ... of the longest group: all take part in its barriers

    // ------------------------------------------------------------ copy stage
    // K-major tile: HALVES sub-tiles of [KB rows][128 B] so that the row swizzle of the GEMM kernels applies unchanged.
    unsigned k_off, v_off;                            // the lane's offsets of the first copy instruction; the others are scalars further on
    {
        const int row = tid >> 3;
        k_off = (unsigned)(row * ROW + (((tid & 7) ^ kmajor_swz<128>(row)) << 4));
        const int key = tid / VRC;
        v_off = (unsigned)(key * ROW + (((tid % VRC) * 16) ^ (((key / RPW) % NSEG) * 64)));
        static_assert((GT / VRC) % (RPW * NSEG) == 0, "the V swizzle repeats from one copy instruction to the next");
    }
    const char* Qb = (const char*)p.Q + ((b * p.M + m0) * (long long)ROW);
    const char* Kb = (const char*)p.K + b * p.N * (long long)ROW;
    const char* Vb = (const char*)p.V + b * p.N * (long long)ROW;
    // Non-temporal copies of the first two chunks for what one workgroup alone reads (one tile holds all queries of a head): 192 heads of
    // 128 x 128 x 64 from memory 7.05 -> 6.63 us, no change from the caches.
    const bool kv_once = p.tiles_m == 1;
    // One copy instruction of a chunk's keys or values into ring stage st (a constant in every call: worked out from i it costs an
    // addition per LDS read).
    auto copy_key = [&](const i32x4& rk, int st, int u, bool once) __attribute__((always_inline)) {
        char* const dst = ring + st * 2 * TILE + wave * 1024 + u / KPASS * (KB * 128) + u % KPASS * (GT * 16);
        const unsigned off = k_off + u % KPASS * (KROWS * ROW) + u / KPASS * 128;
        if (once) load_to_lds_nt(rk, dst, off);
        else load_to_lds(rk, dst, off);
    };
    auto copy_value = [&](const i32x4& rv, int st, int u, bool once) __attribute__((always_inline)) {
        char* const dst = ring + st * 2 * TILE + TILE + wave * 1024 + u * (GT * 16);
        if (once) load_to_lds_nt(rv, dst, v_off + u * (GT * 16));
        else load_to_lds(rv, dst, v_off + u * (GT * 16));
    };
    // Descriptor of chunk i of this group in K or V: rows past N lie outside it and read zeros; past the last chunk it is empty.
    auto chunk_rsrc = [&](const char* base, int i) __attribute__((always_inline)) {
        const int c = i * KG + kgrp;
        return make_rsrc(base + (long long)c * TILE, (long long)(p.N - c * KB) * ROW);
    };
    auto copy_keys = [&](int i, int st) __attribute__((always_inline)) {
        const i32x4 rk = chunk_rsrc(Kb, i);
        if (kv_once) {
#pragma unroll
            for (int u = 0; u < COPIES; ++u) copy_key(rk, st, u, true);
        } else {
#pragma unroll
            for (int u = 0; u < COPIES; ++u) copy_key(rk, st, u, false);
        }
    };
    auto copy_values = [&](int i, int st) __attribute__((always_inline)) {
        const i32x4 rv = chunk_rsrc(Vb, i);
        if (kv_once) {
#pragma unroll
            for (int u = 0; u < COPIES; ++u) copy_value(rv, st, u, true);
        } else {
#pragma unroll
            for (int u = 0; u < COPIES; ++u) copy_value(rv, st, u, false);
        }
    };
    // Both stages are filled up front: a head of 128 keys is these two chunks, and requesting the second only after the first had landed
    // is one more trip to memory (192 heads of 128 x 128 x 64 fp16 from memory 6.59 us, 6.20 this way).
    if (nmine > 0) { copy_keys(0, 0); copy_values(0, 0); }

    // ------------------------------------------------------------ this wave's queries, as MFMA operands (rows past M read zeros)
    // (no non-temporal hint here, although nobody else reads them: a load takes 32 bytes of each of 32 rows, and lines that do not stay are
    // fetched again by the next one - 6.76 us instead of 6.20 for the same heads)
    uint4 qf[KSTEPS];
    {
        const __amdgpu_buffer_rsrc_t rq = __builtin_amdgcn_make_buffer_rsrc((void*)Qb, 0, rows_q * ROW, 0x00020000);
        typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks)
            qf[ks] = __builtin_bit_cast(uint4, (u32x4)__builtin_amdgcn_raw_buffer_load_b128(rq, (wave * 32 + l31) * ROW + ks * 32 + g * 16, 0, 0));
    }
    if (nmine > 1) copy_keys(1, 1);
    if (nmine == 2 || (FORM == ATTN_SEQUENTIAL && nmine > 1)) copy_values(1, 1);      // (pipelined, with more chunks, the first step copies these values)
    const int swl = kmajor_swz<128>(l31);            // rows 32*jb + l31 share it (period 16)

    f32x16 acc_o[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc_o[db][r] = 0.f;          // reduction init
    // The reference of the softmax, a row's largest score so far in base-2 units, and the sum of the probabilities relative to it.  Every
    // row's own largest probability is then 1 (to 2^-14 here, exactly once rounded to 16 bits) and loses nothing when the probabilities are
    // rounded for the second product.  Letting references lag (up to 2^8, rescaling rarely) is 4 - 10 % faster and was measured less exact: bf16 against fp64,
    // 2048 keys at d = 64, scale 1, N(0, 1) data 6.3e-4 instead of 1.7e-4, 4096 keys at d = 128, scale 1/sqrt(d) 1.67e-3 instead of 1.48e-3.
    float m_run = 0.f, l_run = 0.f;
    // A negative scale is a positive one on negated queries (exact), so that the largest scaled score is that of the largest score.
    const float sc = __builtin_fabsf(p.scale_log2e);
    // Up to this size a reference's own rounding moves an exponent by 2^-14 at most, and the exponent comes from one fused
    // multiply-add per score.  Beyond it (scores of thousands, infinities, a scale of zero) score and reference are rounded alike first: the
    // product inside the fused form is exact, so the row's largest score would keep the whole rounding error of its reference as exponent.
    // (The test costs a wave one comparison and one branch per chunk, 1 %; rounding every score first costs an instruction per score.)
    const float fused_upto = sc != 0.f ? 1024.0f : -1.0f;
    copy_barrier<0>();                                // the queries and the first two chunks
    if (p.scale_log2e < 0.f) {
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks)
            qf[ks] = make_uint4(qf[ks].x ^ 0x80008000u, qf[ks].y ^ 0x80008000u, qf[ks].z ^ 0x80008000u, qf[ks].w ^ 0x80008000u);
    }

    // ------------------------------------------------------------ fragments of a chunk in ring stage st
    auto k_frag = [&](int st, int ks, int jb) __attribute__((always_inline)) -> uint4 {
        return *(const uint4*)(ring + st * 2 * TILE + (ks >> 2) * (KB * 128) + (jb * 32 + l31) * 128 + ((((ks & 3) * 2 + g) ^ swl) << 4));
    };
    // Position (g, 4*hh + e) of k-step s in key block jb is key 32*jb + 16*s + 8*hh + 4*g + e: the order in which the
    // probabilities come out of the first product.
    auto v_frag = [&](int st, int jb, int s, int db) __attribute__((always_inline)) -> uint4 {
        i16x4 h[2];
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
            const int key = jb * 32 + s * 16 + hh * 8 + 4 * (blk >> 1) + (s16 >> 2);
            const int col = db * 32 + 16 * (blk & 1) + 4 * (s16 & 3);
            const char* ptr = ring + st * 2 * TILE + TILE + key * ROW + ((col * 2) ^ (((key / RPW) % NSEG) * 64));
            h[hh] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(TIR_LDS_PTR(i16x4, ptr));
        }
        const i32x2 lo = __builtin_bit_cast(i32x2, h[0]), hi = __builtin_bit_cast(i32x2, h[1]);
        return make_uint4((unsigned)lo[0], (unsigned)lo[1], (unsigned)hi[0], (unsigned)hi[1]);
    };
    const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    // keys past N (only in the last chunk) drop out of the softmax
    auto mask_chunk = [&](int i, f32x16 (&s)[JB]) __attribute__((always_inline)) {
        const int c = i * KG + kgrp;
        if ((c + 1) * KB > p.N) {
#pragma unroll
            for (int jb = 0; jb < JB; ++jb)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (c * KB + jb * 32 + 8 * (r >> 2) + 4 * g + (r & 3) >= p.N) s[jb][r] = -__builtin_inff();
        }
    };
    // A row's largest scaled score in a chunk from the lane's partial maxima.
    auto chunk_reference = [&](float mx) __attribute__((always_inline)) -> float {
        const auto both = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, mx), __builtin_bit_cast(unsigned, mx), false, false);
        const unsigned lo = both[0], hi = both[1];                   // the half-waves' values: each holds half of the query's keys
        mx = __builtin_fmaxf(__builtin_bit_cast(float, lo), __builtin_bit_cast(float, hi));
        // (a chunk whose scores are all -inf counts nothing, but its reference has to be a number)
        return __builtin_fmaxf(mx * sc, -__FLT_MAX__);
    };

    auto raise_reference = [&](float m_chunk) __attribute__((always_inline)) {
        if (__builtin_amdgcn_ballot_w64(m_chunk > m_run) != 0) {
            const float m_new = __builtin_fmaxf(m_run, m_chunk);
            const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);              // 1 for rows whose reference stays
            m_run = m_new;
            l_run *= alpha;
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc_o[db][r] *= alpha;
        }
    };

    constexpr int NQK = KSTEPS * JB, NPV = JB * 2 * DB;      // MFMAs of the two products of a chunk
    constexpr int EPM = JB * 16 / NQK;                       // exponentials per MFMA of the first product
    // MFMAs by which a fragment's read runs ahead (2 and 2: 1 - 3 % slower on long sequences)
    constexpr int LAK = 4, LAV = 3;

    // Chunk i (ring stage st): its scores are in `cur` and m_run is its reference.  The first product of chunk i + 1 runs under the
    // exponentials of chunk i, the maximum of its scores under the second product of chunk i.
    auto chunk_step = [&](int i, int st, f32x16 (&cur)[JB], f32x16 (&nxt)[JB], auto last_flag, auto copy_flag) __attribute__((always_inline)) {
        constexpr bool LAST = decltype(last_flag)::value, COPY = decltype(copy_flag)::value;
        float mul = sc, base = -m_run;
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(__builtin_fabsf(m_run) <= fused_upto)) != 0, 0)) {
#pragma clang fp contract(off)
            // exponents in place of the scores; keys past N again, which a scale of zero would turn into NaN
            const int c = i * KG + kgrp;
#pragma unroll
            for (int jb = 0; jb < JB; ++jb)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const float s = cur[jb][r] * sc;
                    cur[jb][r] = c * KB + jb * 32 + 8 * (r >> 2) + 4 * g + (r & 3) >= p.N ? -__builtin_inff() : s - m_run;
                }
            mul = 1.f;
            base = 0.f;
        }
        if constexpr (!LAST && !COPY) {
            if (i > 0) copy_values(i + 1, st ^ 1);
        }
        const i32x4 rk = chunk_rsrc(Kb, i + 2), rv = chunk_rsrc(Vb, i + 1);
        unsigned pw[JB * 8];                                         // P^T fragments: key block jb, k-step s at 8*jb + 4*s
        float lsum[2] = {0.f, 0.f};
        uint4 kf[LAK], vf[LAV];
        if constexpr (!LAST) {
#pragma unroll
            for (int t = 0; t < LAK; ++t) kf[t] = k_frag(st ^ 1, t / JB, t % JB);
        }
        // At d = 128 a wave between its MFMAs goes before one that rescales or waits at a barrier (16 x 4096 x 4096 x 128 bf16 150.3 -> 147.3 us; with eight waves in a
        // workgroup 144.9 -> 138.8); at d = 64, where the vector work is the longer half, it costs 8 %.  There a wave of the sequential form goes first while it
        // takes exponentials, and the SIMD's other three have their MFMAs under them (32 x 4096 x 4096 x 64 bf16 160.7 -> 158.5 us, eight waves in a workgroup 158.3 -> 155.5,
        // 26 x 3841 x 2500 89.5 -> 86.7; first from the row maxima on: 4 % slower again).
        if constexpr (DH == 128 || FORM == ATTN_SEQUENTIAL) __builtin_amdgcn_s_setprio(1);
        TIR_FENCE();
#pragma unroll
        for (int t = 0; t < NQK; ++t) {
            const int jb = t % JB, ks = t / JB;
            if constexpr (!LAST) {
                nxt[jb] = InTraits<DT>::mfma(kf[t % LAK], qf[ks], ks == 0 ? zero16 : nxt[jb]);
                TIR_FENCE();
                if constexpr (COPY) {
#pragma unroll
                    for (int u = t * 2 * COPIES / NQK; u < (t + 1) * 2 * COPIES / NQK; ++u) {
                        if (u < COPIES) copy_key(rk, st, u, FORM == ATTN_PIPED_STREAM);
                        else copy_value(rv, st ^ 1, u - COPIES, FORM == ATTN_PIPED_STREAM);
                    }
                }
                if (t + LAK < NQK) kf[t % LAK] = k_frag(st ^ 1, (t + LAK) / JB, (t + LAK) % JB);
            }
            if (t >= NQK - LAV) {
                const int v = t - (NQK - LAV);
                vf[v] = v_frag(st, v / (2 * DB), v / DB % 2, v % DB);
            }
#pragma unroll
            for (int e = t * EPM; e < (t + 1) * EPM; e += 2) {
                float pr[2];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    pr[h] = __builtin_amdgcn_exp2f(__builtin_fmaf(cur[e / 16][e % 16 + h], mul, base));
                    lsum[h] += pr[h];
                }
                pw[e / 2] = PackP<DT>::two(pr[0], pr[1]);
            }
            TIR_FENCE();
        }
        l_run += lsum[0] + lsum[1];
        if constexpr (!LAST) mask_chunk(i + 1, nxt);
        if constexpr (FORM == ATTN_SEQUENTIAL) __builtin_amdgcn_s_setprio(0);
        // O^T += V^T P^T
        float mx[4];
#pragma unroll
        for (int t = 0; t < NPV; ++t) {
            const int jb = t / (2 * DB), s = t / DB % 2, db = t % DB;
            const uint4 pf = make_uint4(pw[8 * jb + 4 * s], pw[8 * jb + 4 * s + 1], pw[8 * jb + 4 * s + 2], pw[8 * jb + 4 * s + 3]);
            acc_o[db] = InTraits<DT>::mfma(vf[t % LAV], pf, acc_o[db]);
            TIR_FENCE();
            if (t + LAV < NPV) vf[t % LAV] = v_frag(st, (t + LAV) / (2 * DB), (t + LAV) / DB % 2, (t + LAV) % DB);
            if constexpr (!LAST) {
                // the largest of chunk i + 1's scores, from the second MFMA on
                constexpr int PER = (JB * 16 + NPV - 2) / (NPV - 1);
#pragma unroll
                for (int e = (t - 1) * PER; t > 0 && e < t * PER && e < JB * 16; ++e)
                    mx[e & 3] = e < 4 ? nxt[e / 16][e % 16] : __builtin_fmaxf(mx[e & 3], nxt[e / 16][e % 16]);
            }
            TIR_FENCE();
        }
        if constexpr (DH == 128 && FORM != ATTN_SEQUENTIAL) __builtin_amdgcn_s_setprio(0);
        if constexpr (!LAST) {
            raise_reference(chunk_reference(__builtin_fmaxf(__builtin_fmaxf(mx[0], mx[1]), __builtin_fmaxf(mx[2], mx[3]))));
        }
    };
    // The scores of chunk i on their own, and their reference.
    auto scores = [&](int i, int st, f32x16 (&s)[JB]) __attribute__((always_inline)) -> float {
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks)
#pragma unroll
            for (int jb = 0; jb < JB; ++jb) s[jb] = InTraits<DT>::mfma(k_frag(st, ks, jb), qf[ks], ks == 0 ? zero16 : s[jb]);
        mask_chunk(i, s);
        float mx = s[0][0];
#pragma unroll
        for (int jb = 0; jb < JB; ++jb)
#pragma unroll
            for (int r = 0; r < 16; ++r) mx = __builtin_fmaxf(mx, s[jb][r]);
        return chunk_reference(mx);
    };

    f32x16 s_even[JB], s_odd[JB];
    if constexpr (FORM == ATTN_SEQUENTIAL) {
        auto step = [&](int i, int st) __attribute__((always_inline)) {
            if (i > 0 && i + 1 < nmine) {                // the stage was last read before the previous barrier
                copy_keys(i + 1, st ^ 1);
                copy_values(i + 1, st ^ 1);
            }
            const float m_chunk = scores(i, st, s_even);
            if (i == 0) m_run = m_chunk;
            else raise_reference(m_chunk);
            chunk_step(i, st, s_even, s_odd, std::true_type(), std::false_type());
            copy_barrier<0>();
        };
        static_assert(KG == 1, "");
        for (int i = 0; i < nmine; i += 2) {
            step(i, 0);
            if (i + 1 < nmine) step(i + 1, 1);
        }
    } else {
        if (KG == 1 || nmine > 0) m_run = scores(0, 0, s_even);
        // A step overwrites the stage of the keys multiplied in the step before and of the values of that step; at its end the copies have
        // landed (this wave's part) and, after the barrier, everybody's.  Up to two chunks nothing is copied any more and nobody waits.
        const bool sync = nloop > 2;                      // (the same for all groups)
        if (sync) copy_barrier<0>();
        int i = 0;
        for (; i + 2 < nmine; i += 2) {
            chunk_step(i, 0, s_even, s_odd, std::false_type(), std::true_type());
            copy_barrier<0>();
            chunk_step(i + 1, 1, s_odd, s_even, std::false_type(), std::true_type());
            copy_barrier<0>();
        }
        if (i + 1 < nmine) {
            chunk_step(i, 0, s_even, s_odd, std::false_type(), std::false_type());
            if (sync) copy_barrier<0>();
            ++i;
#pragma unroll
            for (int jb = 0; jb < JB; ++jb) s_even[jb] = s_odd[jb];
        }
        if (KG == 1 || i < nmine) chunk_step(i, i & 1, s_even, s_odd, std::true_type(), std::false_type());
        if (KG > 1 && sync && nmine < nloop) copy_barrier<0>();      // (the longer groups' last but one step)
        copy_barrier<0>();                                // everybody is past its last read: the ring is free
    }

    if constexpr (KG > 1) {
        // ------------------------------------------------------------ merge the key groups: sums and accumulators relative to the largest reference
        typedef float f32x4 __attribute__((ext_vector_type(4)));
        const float ms = nmine > 0 ? m_run : -__builtin_inff();                // (a group without a chunk counts nothing)
        auto area = [&](int k) { return smem + ((k - 1) * QW + wave) * MERGE; };      // the stages are free: everybody is past the last barrier
        if (kgrp != 0) {
            f32x4* const o = (f32x4*)area(kgrp);
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4) {
                    f32x4 v;
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = acc_o[db][4 * q4 + e];
                    o[(db * 4 + q4) * 64 + lane] = v;
                }
            float* const t = (float*)(area(kgrp) + DB * 4096);
            t[lane] = l_run;
            t[64 + lane] = ms;
        }
        __syncthreads();
        if (kgrp == 0) {
            float top = ms, mk[KG];
            mk[0] = ms;
#pragma unroll
            for (int k = 1; k < KG; ++k) {
                mk[k] = ((const float*)(area(k) + DB * 4096))[64 + lane];
                top = __builtin_fmaxf(top, mk[k]);
            }
            const float own = __builtin_amdgcn_exp2f(mk[0] - top);             // (group 0 always has a chunk: top is finite)
            l_run *= own;
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc_o[db][r] *= own;
#pragma unroll
            for (int k = 1; k < KG; ++k) {
                const float f = __builtin_amdgcn_exp2f(mk[k] - top);
                l_run += f * ((const float*)(area(k) + DB * 4096))[lane];
                const f32x4* const o = (const f32x4*)area(k);
#pragma unroll
                for (int db = 0; db < DB; ++db)
#pragma unroll
                    for (int q4 = 0; q4 < 4; ++q4) {
                        const f32x4 v = o[(db * 4 + q4) * 64 + lane];
#pragma unroll
                        for (int e = 0; e < 4; ++e) acc_o[db][4 * q4 + e] += f * v[e];
                    }
            }
        }
        __syncthreads();                               // the output tile is staged where the handed-over values were
    }

    // ------------------------------------------------------------ normalise, stage through LDS, store rows
    const float l_tot = l_run + __shfl_xor(l_run, 32);
    const float inv = 1.0f / l_tot;
    constexpr int ORB = DH * OS;                     // bytes of one output row
    char* const s_o = smem;                          // the K / V stages are free now
    if (KG == 1 || kgrp == 0)
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
            // registers 4*q4 .. 4*q4+3 are head-dimension columns dv0 .. dv0+3 of query 32*wave + l31
            const int row = wave * 32 + l31;
            const int dv0 = db * 32 + 8 * q4 + 4 * g;
            char* dst = s_o + row * ORB + ((dv0 * OS) ^ ((row & 7) << 4));
            alignas(16) out_t v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = OT::cvt(acc_o[db][4 * q4 + e] * inv);
            if constexpr (OS == 4) *(uint4*)dst = *(const uint4*)v;
            else *(uint2*)dst = *(const uint2*)v;
        }
    __syncthreads();
    {
        char* Ob = (char*)p.O + (b * p.M + m0) * (long long)ORB;
        const __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc((void*)Ob, 0, rows_q * ORB, 0x00020000);
        constexpr int ORC = ORB / 16;                // 16-byte chunks per output row
#pragma unroll
        for (int i = 0; i < TQ * ORC / (GT * KG); ++i) {
            const int q = (int)threadIdx.x + i * GT * KG;
            const int row = q / ORC, pc = q % ORC;
            typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
            const u32x4 v = *(const u32x4*)(s_o + row * ORB + ((pc * 16) ^ ((row & 7) << 4)));
            if (p.store_nt) __builtin_amdgcn_raw_buffer_store_b128(v, ro, row * ORB + pc * 16, 0, TIR_STORE_AUX_STREAM);
            else __builtin_amdgcn_raw_buffer_store_b128(v, ro, row * ORB + pc * 16, 0, TIR_STORE_AUX);   // rows past M: outside the descriptor
        }
    }
}

// The kernels of the dispatch: tiles of 64, 128 or 256 queries; four key groups; chunks of 32 keys; the forms above.
enum AttnKernel : int { ATTN_T64_GROUPS, ATTN_T128_C32, ATTN_T128, ATTN_T128_STREAM, ATTN_T128_SEQUENTIAL, ATTN_T256, ATTN_T256_SEQUENTIAL };
AttnKernel attention_kernel_of(long long batch, long long M, long long N, int DH, int OUT);

typedef hipError_t (*attn_launch_fn)(const AttnParams&, hipStream_t);
// (dt, out, head dimension) -> launcher, or null when the combination is not compiled
attn_launch_fn attention_launcher(int dt, int out, int dh);

}  // namespace tir
