// Depth-wise convolution (groups = channels, one filter per channel): the paper's DEP workload.  There
// is no contraction over channels, so nothing here maps onto a matrix intrinsic: the operator is bound
// by memory traffic and plain vector arithmetic, and the right decomposition is the direct one - each
// thread owns one output pixel x one 16-byte vector of channels, reads the R*S input vectors its taps
// touch (neighbouring pixels share them through the caches) and multiplies element by element with the
// filter taps, which the workgroup keeps in LDS as [tap][channel] in the accumulator's type.
//   y[n,p,q,c] = sum_{r,s} x[n, p*s_h - pad_h + r*d_h, q*s_w - pad_w + s*d_w, c] * w[c,r,s]      (sec. 4.2 formula with groups = C)
#pragma once
#include "tir_kernel.h"
#ifndef TIR_DW_NPIX
#define TIR_DW_NPIX 2
#endif
#define TIR_DW_NPIX_DEFAULT TIR_DW_NPIX

namespace tir {

template <int DT> struct DwIn;
template <> struct DwIn<DT_F16> {
    typedef float acc_e;
    static __device__ __forceinline__ float get(const uint4& v, int e) {
        typedef _Float16 h8 __attribute__((ext_vector_type(8)));
        return (float)__builtin_bit_cast(h8, v)[e];
    }
    static __device__ __forceinline__ float w(unsigned short bits) { return (float)__builtin_bit_cast(_Float16, bits); }
};
template <> struct DwIn<DT_BF16> {
    typedef float acc_e;
    static __device__ __forceinline__ float get(const uint4& v, int e) {
        const unsigned u = ((const unsigned*)&v)[e >> 1];
        return __uint_as_float((e & 1) ? (u & 0xffff0000u) : (u << 16));
    }
    static __device__ __forceinline__ float w(unsigned short bits) { return __uint_as_float((unsigned)bits << 16); }
};
template <> struct DwIn<DT_I8> {
    typedef int acc_e;
    static __device__ __forceinline__ int get(const uint4& v, int e) {
        const int u = (int)((const unsigned*)&v)[e >> 2];
        return (u << (24 - 8 * (e & 3))) >> 24;       // sign-extended byte e
    }
    static __device__ __forceinline__ int w(signed char bits) { return (int)bits; }
};

constexpr int kDwChannels = 64;     // channels per workgroup
constexpr int kDwPixPerThread = TIR_DW_NPIX_DEFAULT;
constexpr int kDwMaxTaps = 128;     // R*S limit of this kernel (the [tap][64] filter table in LDS)

// R3S3: the filter is 3x3 (the common case): the nine input vectors of a pixel are requested together.
template <int DT, int OUT, bool R3S3, bool STREAM>
__global__ void __launch_bounds__(256) depthwise_kernel(const Params p) {
    typedef typename DwIn<DT>::acc_e acc_e;
    typedef OutTraits<OUT> OT;
    typedef typename OT::type out_t;
    typedef typename std::conditional<DT == DT_I8, signed char, unsigned short>::type in_t;
    typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
    constexpr int ES = elem_size(DT), VEC = 16 / ES;
    constexpr int CV = kDwChannels / VEC;            // channel vectors per workgroup
    constexpr int PP = 256 / CV;                     // pixels per pass of the workgroup
    constexpr int NPIX = kDwPixPerThread;            // pixels per thread

    __shared__ acc_e wt[R3S3 ? 1 : kDwMaxTaps * kDwChannels];

    const int tid = threadIdx.x;
    const int cv = tid % CV, pl = tid / CV;
    const int cbase = blockIdx.y * kDwChannels;
    const int c0 = cbase + cv * VEC;
    const int RS = p.R * p.S;
    const in_t* wsrc = (const in_t*)p.B;
    // 3x3: the thread's VEC channels x 9 taps are 9 consecutive 16-byte vectors of the filter (channel-major,
    // element (channel e, tap t) at position 9*e + t): they go to registers and stay there for all its pixels.
    uint4 wv[R3S3 ? 9 : 1];                  // kept packed: the multiply-add reads 16-bit operands directly
    if constexpr (R3S3) {
        if (c0 >= p.Cin) return;
#pragma unroll
        for (int i = 0; i < 9; ++i) wv[i] = ((const uint4*)(wsrc + (long long)c0 * 9))[i];
    } else {
        for (int idx = tid; idx < RS * kDwChannels; idx += 256) {
            const int t = idx / kDwChannels, ch = idx % kDwChannels;
            wt[idx] = cbase + ch < p.Cin ? DwIn<DT>::w(wsrc[(long long)(cbase + ch) * RS + t]) : (acc_e)0;
        }
    }
    // bias of the thread's channels (requested early: its latency overlaps the first input loads)
    acc_e bias_r[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) bias_r[e] = (p.bias && c0 < p.Cin) ? ((const acc_e*)p.bias)[c0 + e] : (acc_e)0;
    if constexpr (!R3S3) {
        __syncthreads();
        if (c0 >= p.Cin) return;
    }

    const int PQ = p.P * p.Q;
    // consecutive workgroup ids go to different XCDs (L2s): regroup them so that each XCD owns a contiguous
    // range of pixels and finds the rows its neighbouring taps share in its own L2
    int bx = blockIdx.x;
    {
        const int nb = (p.M + NPIX * PP - 1) / (NPIX * PP), nb8 = nb - nb % kXcds;      // = gridDim.x (a hidden argument, fetched late)
        if (bx < nb8) bx = (bx % kXcds) * (nb8 / kXcds) + bx / kXcds;
    }
    // taps outside the image read through the descriptor's range check: zeros, and no branch around the load
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc((void*)p.A, 0, (int)((long long)p.batch_imgs * p.H * p.W * p.Cin * ES), 0x00020000);
    const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc(p.C, 0, (int)((long long)p.M * p.Cin * (int)sizeof(out_t)), 0x00020000);
    const acc_e* wcol = wt + (R3S3 ? 0 : cv * VEC);
#pragma unroll
    for (int j = 0; j < NPIX; ++j) {
        const int m = (bx * NPIX + j) * PP + pl;
        if (m >= p.M) break;
        const int img = (int)fastdiv((unsigned)m, p.div_pq_magic, p.div_pq_shift), rem = m - img * PQ;
        const int op = (int)fastdiv((unsigned)rem, p.div_q_magic, p.div_q_shift), oq = rem - op * p.Q;
        const int ih0 = op * p.stride_h - p.pad_h, iw0 = oq * p.stride_w - p.pad_w;
        const int pix0 = (img * p.H + ih0) * p.W + iw0;              // may be "negative": only used when the tap is valid
        acc_e acc[VEC];
#pragma unroll
        for (int e = 0; e < VEC; ++e) acc[e] = 0;                    // reduction init
        auto tap_off = [&](int r, int s) -> int {
            const int ih = ih0 + r * p.dil_h, iw = iw0 + s * p.dil_w;
            const bool ok = (unsigned)ih < (unsigned)p.H && (unsigned)iw < (unsigned)p.W;
            return ok ? ((pix0 + r * p.dil_h * p.W + s * p.dil_w) * p.Cin + c0) * ES : (int)kOutOfRange;
        };
        if constexpr (R3S3) {
            u32x4 v[9];
#pragma unroll
            for (int t = 0; t < 9; ++t) v[t] = __builtin_amdgcn_raw_buffer_load_b128(rx, tap_off(t / 3, t % 3), 0, 0);
#pragma unroll
            for (int t = 0; t < 9; ++t) {
                const uint4 u = __builtin_bit_cast(uint4, v[t]);
#pragma unroll
                for (int e = 0; e < VEC; ++e) acc[e] += DwIn<DT>::get(u, e) * DwIn<DT>::get(wv[(9 * e + t) / VEC], (9 * e + t) % VEC);
            }
        } else {
            for (int r = 0; r < p.R; ++r)
                for (int s = 0; s < p.S; ++s) {
                    const uint4 u = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rx, tap_off(r, s), 0, 0));
                    const acc_e* wrow = wcol + (r * p.S + s) * kDwChannels;
#pragma unroll
                    for (int e = 0; e < VEC; ++e) acc[e] += DwIn<DT>::get(u, e) * wrow[e];
                }
        }
        alignas(16) out_t o[VEC];
#pragma unroll
        for (int e = 0; e < VEC; ++e) o[e] = finish_value<OUT>(consumer(acc[e], bias_r[e], p.relu), p.scale);
        constexpr int OB = VEC * (int)sizeof(out_t);                 // 16 .. 64 bytes
        static_assert(OB % 16 == 0, "");
        const int obyte = (m * p.Cin + c0) * (int)sizeof(out_t);     // < 2^31: checked by the host
#pragma unroll
        for (int b = 0; b < OB; b += 16)
            __builtin_amdgcn_raw_buffer_store_b128(*(const u32x4*)((const char*)o + b), ry, obyte + b, 0, STREAM ? TIR_STORE_AUX_STREAM : TIR_STORE_AUX);   // write-through, like every epilogue
    }
}

// 3x3 filter, undilated along the width, stride 1 or 2 there (SW): a thread owns NP (four or eight) horizontally adjacent output
// pixels x one 16-byte channel vector.  Their taps touch 3 rows x NC = (NP - 1)*SW + 3 consecutive input columns, loaded
// once (18 vectors for 4 pixels at stride 1 instead of 36, 30 for 8) and all requested before the first multiply; row and
// column validity are decided once per row / column, so a tap's address costs three vector instructions instead
// of a dozen.  The one-pixel kernel above spent twice as many instructions on addresses as on multiply-adds.
// Two rows of output pixels per thread (NR = 2, four columns each, stride 1, undilated) share two of their input rows: 24 vectors for 8 pixels, where eight in
// a row take 30 and two threads of four 36.  The kernel is bound by those fetches through the CU's load path; depthwise_rows() has both sides.
// STREAM (the output policy) is a template parameter, not a branch: a branch around each store splits the pixel loop
// into blocks, and the compiler then waits for the previous pixel's stores before the next pixel's arithmetic
// (measured: 6.9 -> 8.8 us).
template <int DT, int OUT, int SW, int NP, int NR, bool STREAM>
__global__ void __launch_bounds__(256) depthwise3x3_blocked_kernel(const Params p) {
    typedef typename DwIn<DT>::acc_e acc_e;
    typedef OutTraits<OUT> OT;
    typedef typename OT::type out_t;
    typedef typename std::conditional<DT == DT_I8, signed char, unsigned short>::type in_t;
    typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
    constexpr int ES = elem_size(DT), VEC = 16 / ES;
    constexpr int CV = kDwChannels / VEC;            // channel vectors per workgroup
    constexpr int PP = 256 / CV;                     // pixel groups per workgroup
    constexpr int NC = (NP - 1) * SW + 3;
    constexpr int NI = NR + 2;                       // input rows (two output rows: stride 1, undilated)

    // every argument the kernel reads, fetched in one batch
    asm volatile("" ::"s"(p.A), "s"(p.B), "s"(p.C), "s"(p.M), "s"(p.bias), "s"(p.relu), "s"(p.scale), "s"(p.batch_imgs), "s"(p.H), "s"(p.W), "s"(p.Cin),
                 "s"(p.P), "s"(p.Q), "s"(p.stride_h), "s"(p.pad_h), "s"(p.pad_w), "s"(p.dil_h));
    asm volatile("" ::"s"(p.div_dwq_magic), "s"(p.div_dwq_shift), "s"(p.div_dwpq_magic), "s"(p.div_dwpq_shift));
    const int tid = threadIdx.x;
    const int cv = tid % CV, pl = tid / CV;
    const int c0 = blockIdx.y * kDwChannels + cv * VEC;
    if (c0 >= p.Cin) return;
    const in_t* wsrc = (const in_t*)p.B;
    uint4 wv[9];                                     // VEC channels x 9 taps, element (channel e, tap t) at 9*e + t
#pragma unroll
    for (int i = 0; i < 9; ++i) wv[i] = ((const uint4*)(wsrc + (long long)c0 * 9))[i];
    acc_e bias_r[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) bias_r[e] = p.bias ? ((const acc_e*)p.bias)[c0 + e] : (acc_e)0;

    const int QG = (p.Q + NP - 1) / NP;              // pixel groups per output row
    const int PG = (p.P + NR - 1) / NR;              // rows of pixel groups per image
    int bx = blockIdx.x;                             // each XCD owns a contiguous range of pixel groups (shared rows stay in its L2)
    {
        const int nb = (p.batch_imgs * PG * QG + PP - 1) / PP, nb8 = nb - nb % kXcds;      // = gridDim.x (a hidden argument, fetched late)
        if (bx < nb8) bx = (bx % kXcds) * (nb8 / kXcds) + bx / kXcds;
    }
    const int gidx = bx * PP + pl;
    if (gidx >= p.batch_imgs * PG * QG) return;
    const int img = (int)fastdiv((unsigned)gidx, p.div_dwpq_magic, p.div_dwpq_shift), rem = gidx - img * (PG * QG);
    const int og = (int)fastdiv((unsigned)rem, p.div_dwq_magic, p.div_dwq_shift), op = og * NR, oq0 = (rem - og * QG) * NP;
    const int ih0 = op * p.stride_h - p.pad_h, iw0 = oq0 * SW - p.pad_w;

    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc((void*)p.A, 0, (int)((long long)p.batch_imgs * p.H * p.W * p.Cin * ES), 0x00020000);
    const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc(p.C, 0, (int)((long long)p.M * p.Cin * (int)sizeof(out_t)), 0x00020000);
    const int cstep = p.Cin * ES;                    // bytes from one input column to the next
    bool col_ok[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) col_ok[c] = (unsigned)(iw0 + c) < (unsigned)p.W;
    u32x4 v[NI][NC];
#pragma unroll
    for (int r = 0; r < NI; ++r) {
        const int ih = ih0 + r * (NR > 1 ? 1 : p.dil_h);
        const bool row_ok = (unsigned)ih < (unsigned)p.H;
        int row_off = (((img * p.H + ih) * p.W + iw0) * p.Cin + c0) * ES;           // only used where the tap is inside the image
        asm volatile("" : "+v"(row_off));      // (kept as one value: re-associated with the column, every load's address became a multiply)
#pragma unroll
        for (int c = 0; c < NC; ++c)
            v[r][c] = __builtin_amdgcn_raw_buffer_load_b128(rx, (row_ok && col_ok[c]) ? row_off + c * cstep : (int)kOutOfRange, 0, 0);
    }
    const int out_pix0 = (img * p.P + op) * p.Q + oq0;
#pragma unroll
    for (int k = 0; k < NR * NP; ++k) {
        const int i = k / NP, j = k % NP;
        acc_e acc[VEC];
#pragma unroll
        for (int e = 0; e < VEC; ++e) acc[e] = 0;                    // reduction init
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            const uint4 u = __builtin_bit_cast(uint4, v[i + t / 3][j * SW + t % 3]);
#pragma unroll
            for (int e = 0; e < VEC; ++e) acc[e] += DwIn<DT>::get(u, e) * DwIn<DT>::get(wv[(9 * e + t) / VEC], (9 * e + t) % VEC);
        }
        alignas(16) out_t o[VEC];
#pragma unroll
        for (int e = 0; e < VEC; ++e) o[e] = finish_value<OUT>(consumer(acc[e], bias_r[e], p.relu), p.scale);
        constexpr int OB = VEC * (int)sizeof(out_t);
        const int obyte = oq0 + j < p.Q && (NR == 1 || op + i < p.P) ? ((out_pix0 + i * p.Q + j) * p.Cin + c0) * (int)sizeof(out_t) : (int)kOutOfRange;      // < 2^31: checked by the host
#pragma unroll
        for (int b = 0; b < OB; b += 16)
            __builtin_amdgcn_raw_buffer_store_b128(*(const u32x4*)((const char*)o + b), ry, obyte + b, 0, STREAM ? TIR_STORE_AUX_STREAM : TIR_STORE_AUX);
    }
}

// Workgroups of the blocked kernel with np adjacent pixels per thread: N images of P x Q output pixels, C channels of type dt.
inline long long depthwise_workgroups(int dt, long long N, long long P, long long Q, long long C, int np) {
    const int groups = 256 / (kDwChannels / (16 / elem_size(dt)));       // pixel groups per workgroup
    return (N * P * ((Q + np - 1) / np) + groups - 1) / groups * ((C + kDwChannels - 1) / kDwChannels);
}

// Pixels per thread of the blocked kernel.  Eight at stride 1 fetch a sixth fewer vectors per pixel than four, with twice the registers and twice the serial
// arithmetic per thread.  One round of them (two workgroups per CU) takes the same time however full it is; workgroups of four step up in time at the fourth per
// CU, in bf16 -> bf16 (196 registers, two per CU; fp16 122) at the third, and from there on eight pay.  That counts the padding of both forms: at widths of 4 or 9 to 12
// eight pixels make a third to twice as many.  int8 -> int32 writes 64 bytes per pixel and thread and does not gain.  Four and eight pixels, us, same buffers:
//   fp16: 16x56x56x128 (784 workgroups of four) 8.1 / 6.9, 16x60x14x384 -> fp32 (720) 12.3 / 12.8, 9x110x11x352 (558) 7.8 / 8.1, 4x505x4x512 (512) 5.7 / 7.2
//   bf16: 360 to 512 workgroups of four 6.0 / 7.6, 513 to 768 8.2 / 8.1, 769 to 1024 10.4 / 9.2 (medians); -> fp32 4x505x9x256 (760) 11.3 / 12.4
//   int8: 4x960x4x384 (360) 10.3 / 14.5, 4x137x49x384 (672) 13.1 / 16.4, 8x245x49x128 (800) 16.8 / 16.2; -> int32 2x2880x28x64 (630) 33.3 / 35.8, 8x288x56x128 (1008) 52.3 / 55.5
inline int depthwise_pixels(int dt, int out, long long N, long long P, long long Q, long long C, int stride_w) {
    if (stride_w != 1 || out == DT_I32 || depthwise_workgroups(dt, N, P, Q, C, 8) > 2 * 256) return kDwBlockPix;
    return depthwise_workgroups(dt, N, P, Q, C, kDwBlockPix) > (out == DT_BF16 ? 2 : 3) * 256 ? 8 : kDwBlockPix;
}

// Rows of output pixels per thread of the blocked kernel at stride 1, undilated, P x Q output pixels: two rows of four, or one (of depthwise_pixels()).  Two
// rows fetch a fifth less per pixel than eight in a row, but hold 24 vectors at once (fp16 170 registers, bf16 245: two workgroups per CU, where four in a
// row have four and two), so a launch that has not a workgroup of four for every CU is slower (1.2 - 1.3 of the time: half as many CUs work).  From there on:
// bf16 gains, 241 of 246 drawn calls less than the time, down to 0.71 of it (0.89 in the mean), but where the workgroups of one row just fill one or two rounds of two per CU and those
// of two rows, half as many and a few more from padding, begin another: seven calls of 257 to 260 and 513 to 520, 1.01 - 1.25 of the time, one row by the rule (23x13x105x224, 544 and 1012, gains: 11.3 / 10.3).  (No such
// line after 1024, 1536 and 2048: 0.71 - 0.97.)  fp16 gains while every
// CU has at most one workgroup (and a whole block of 64 channels: 3x98x112x48 4.7 / 4.9), 0.88 - 1.04, and from 800 on, 0.78 - 1.04 (both 0.95 in the mean); between, four or eight in a row
// have more workgroups in flight.  One row and two, us, three sets of buffers in turn:
//   bf16: 10x72x22x208 8.4 / 7.7, 24x18x75x208 (516 workgroups, 1028 of one row) 13.0 / 10.6, 32x56x56x128 15.4 / 13.2, 32x112x112x64 31.2 / 26.6, 11x100x49x176 16.4 / 12.1; slower: 8x85x19x464
//         8.7 / 9.9, 25x47x39x80 7.5 / 7.8; one row by the rule: 14x65x69x112 (520, 1024 of one row) 9.8 / 12.2, 3x110x25x448 (259, 511) 5.7 / 6.9
//   fp16: 18x14x41x144 5.7 / 5.0, 20x43x11x336 6.2 / 5.7, 17x32x105x240 20.2 / 17.5, 32x112x112x64 28.4 / 26.1; one row by the rule: 16x56x56x128 (392 workgroups) 7.85 / 8.08, 16x56x56x256 (784) 13.3 / 13.7
// Not measured, and left with one row: fewer than seven rows of output, other types of output.
inline int depthwise_rows(int dt, int out, long long N, long long P, long long Q, long long C) {
    if (out != dt || dt == DT_I8 || P < 7) return 1;
    const long long one = depthwise_workgroups(dt, N, P, Q, C, kDwBlockPix);
    if (one <= 256) return 1;
    const long long two = depthwise_workgroups(dt, N, (P + 1) / 2, Q, C, kDwBlockPix);
    if (dt == DT_BF16) return (two > 256 && two <= 256 + 16 && one <= 512) || (two > 512 && two <= 512 + 16 && one <= 1024) ? 1 : 2;
    return (two <= 256 && C >= kDwChannels) || two > 800 ? 2 : 1;
}

typedef hipError_t (*dw_launch_fn)(const Params&, hipStream_t);
// (dt, out) -> launcher, or null when the pair is not compiled
dw_launch_fn depthwise_launcher(int dt, int out);

}  // namespace tir
