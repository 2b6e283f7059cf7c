// 2-D convolution of few channels (an image network's stem: 1, 3, 4 channels, a large filter), where a channel vector is
// shorter than the 16 bytes the implicit-GEMM copy moves.  With one group and no dilation along the width, the S taps of a filter row
// read S*C consecutive elements of an input row: the reduction k = fuse(rh, rw, rc) becomes R rows of S*C elements, each padded
// to whole 16-byte chunks (zeros in the filter, masked in the input).
//
// A wave owns 4 x 16 output pixels of one image and BN output channels, and copies the input rows its pixels touch into LDS for
// itself; the waves of a workgroup (4 to 16: as many as spread the pixels over the chip in one round) share the filter, one copy per CU
// instead of one per tile.  Both go through registers, because neither is aligned.  The MFMA fragment of (pixel, chunk) is 16
// bytes read at the pixel's place in its row.  Such a place is aligned to stride_w * C elements only.  An LDS read of 16 bytes
// below 4-byte alignment takes 64 cycles per wave (measured; 9 aligned, 13 - 17 as two pairs of dwords), so an odd place is read as
// five dwords and shifted (SHIFT, 18 - 22 cycles).
// 16x224x224x3 -> 64, 7x7, stride 2 in fp16 (5 MB in, 26 MB out: 6 us of HBM time): 113 us as element-wise gathers, 12.3 now.  A
// wave's phases follow each other and each has its own bound - 16-byte loads at 2-byte alignment (46 cycles each in the CU's load
// path: 4 600 cycles), MFMAs and LDS reads (7 000), stores (4 800).  An image of height 1 leaves three of a tile's four rows empty and gains
// all the same: 16x16000x1 -> 64, 10 taps, stride 5 17.4 us and 7.3, 4x3000x6 -> 80, 3 taps 10.7 and 5.2.
//
// The scoring rule sees tiles of 256 pixels x BN channels, not the kernel's 64 x BN per wave; of its two choices of BN it took the faster one, or one
// within 4 %, for 43 of 44 calls drawn over image networks' stems and 1-D signals (worst 64x500x2 -> 128, 7 taps, stride 2: 6.5 us, 5.8 with BN = 64).
#pragma once
#include "tir_kernel.h"

namespace tir {

// 16 bytes moved up by n elements, zeros enter at the bottom (the other direction of shift_down).
template <int ES> __device__ __forceinline__ uint4 shift_up(const uint4& v, int n) {
    const int bytes = n * ES;
    const bool by8 = bytes & 8, by4 = bytes & 4, none = bytes >= 16;
    unsigned x = by8 ? 0u : v.x, y = by8 ? 0u : v.y, z = by8 ? v.x : v.z, w = by8 ? v.y : v.w;
    w = by4 ? z : w; z = by4 ? y : z; y = by4 ? x : y; x = by4 ? 0u : x;
    // bytes & 3 up = 4 - (bytes & 3) down from the dword below; nothing for 0
    const unsigned b = (unsigned)(bytes & 3);
    const unsigned s = (4u - b) & 3u;
    const unsigned w2 = __builtin_amdgcn_alignbyte(w, z, s), z2 = __builtin_amdgcn_alignbyte(z, y, s), y2 = __builtin_amdgcn_alignbyte(y, x, s), x2 = __builtin_amdgcn_alignbyte(x, 0u, s);
    w = b ? w2 : w; z = b ? z2 : z; y = b ? y2 : y; x = b ? x2 : x;
    return make_uint4(none ? 0u : x, none ? 0u : y, none ? 0u : z, none ? 0u : w);
}
// Dword d of the mask that keeps the first n elements of a 16-byte vector.
template <int ES> __device__ __forceinline__ unsigned keep_mask(int n, int d) {
    const int bytes = n * ES - 4 * d;
    return bytes >= 4 ? 0xffffffffu : bytes <= 0 ? 0u : (1u << (8 * bytes)) - 1u;
}

template <int DT, int OUT, int BN, bool SHIFT>
__global__ void __launch_bounds__(1024, 4) conv_rows_kernel(const Params p) {
    typedef typename InTraits<DT>::acc_t acc_t;
    typedef typename OutTraits<OUT>::type out_t;
    typedef typename std::conditional<std::is_same<acc_t, f32x16>::value, float, int>::type acc_e;
    constexpr int ES = elem_size(DT), VEC = 16 / ES, OS = (int)sizeof(out_t), NI = BN / 32;

    extern __shared__ __attribute__((aligned(16))) char rows_smem[];
    asm volatile("" ::"s"(p.A), "s"(p.B), "s"(p.C), "s"(p.N), "s"(p.tiles_m), "s"(p.tiles_n), "s"(p.bias), "s"(p.relu), "s"(p.scale), "s"(p.batch_imgs),
                 "s"(p.PW), "s"(p.store_nt), "s"(p.div_tn_magic), "s"(p.div_tn_shift), "s"(p.div_tm_magic), "s"(p.div_tm_shift));
    asm volatile("" ::"s"(p.H), "s"(p.W), "s"(p.Cin), "s"(p.P), "s"(p.Q), "s"(p.R), "s"(p.S), "s"(p.stride_h), "s"(p.stride_w), "s"(p.pad_h), "s"(p.pad_w),
                 "s"(p.dil_h), "s"(p.rows_tiles_q), "s"(p.rows_cpr), "s"(p.rows_lpr), "s"(p.rows_waves), "s"(p.div_tq_magic), "s"(p.div_tq_shift));
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), waves = p.rows_waves;
    const int l31 = lane & 31, g = lane >> 5;
    // workgroup -> (run of pixel tiles, channel tile); wave -> its tile of 4 x 16 pixels
    const int run = (int)fastdiv(blockIdx.x, p.div_tn_magic, p.div_tn_shift);
    const int n0 = ((int)blockIdx.x - run * p.tiles_n) * BN;
    const int unit = run * waves + wave;
    const bool idle = unit >= p.batch_imgs * p.tiles_m;                  // past the last tile: helps with the filter only
    const int img = idle ? 0 : (int)fastdiv((unsigned)unit, p.div_tm_magic, p.div_tm_shift);
    const int tix = idle ? 0 : unit - img * p.tiles_m;
    const int tp = (int)fastdiv((unsigned)tix, p.div_tq_magic, p.div_tq_shift), tq = tix - tp * p.rows_tiles_q;
    const int op0 = tp * 4, oq0 = tq * 16;

    const int SC = p.S * p.Cin, CPR = p.rows_cpr;                        // elements and 16-byte chunks of a filter row
    const int pairs = (p.R + 1) >> 1;                                    // a k-step is chunk c of filter rows 2*pair (lanes 0..31) and 2*pair + 1
    const int RB = p.PW, chunks = RB >> 4;                               // bytes and chunks of a patch row in LDS
    const int f_row = (2 * pairs * CPR + 1) * 16;                        // bytes of a channel's chunks: an odd count keeps the reads off each other's banks
    const int rows = 3 * p.stride_h + (p.R - 1) * p.dil_h + 1;           // input rows of a tile
    char* const s_filt = rows_smem;                                      // [BN channels][f_row]
    char* const s_patch = rows_smem + BN * f_row + wave * ((rows + 1) * RB);      // the wave's rows, then one of zeros

    unsigned tail[4];                                                    // what a filter row's last chunk keeps
#pragma unroll
    for (int d = 0; d < 4; ++d) tail[d] = keep_mask<ES>(SC - (CPR - 1) * VEC, d);

    // ------------------------------------------------------------ copy-in
    // Nothing else runs meanwhile, and what bounds it is the load path and instruction issue: threads keep their column of the filter and
    // of the patch and step through the rows, so that a chunk costs its load, its mask and its LDS write.  The loads of a batch of rows
    // are requested together.
    {
        // Patch: 2^rows_lpr lanes share a row of the image.
        constexpr int PB = 4;
        const int lpr = 1 << p.rows_lpr, pj0 = lane & (lpr - 1), prow0 = lane >> p.rows_lpr, prows = 64 >> p.rows_lpr;
        const int ih0 = op0 * p.stride_h - p.pad_h, e0 = (oq0 * p.stride_w - p.pad_w) * p.Cin, WC = p.W * p.Cin;      // (WC >= VEC)
        const bool inner = e0 >= 0 && e0 + chunks * VEC <= WC;           // (uniform) no chunk reaches past the left or right edge
        const char* image = (const char*)p.A + (long long)img * p.H * WC * ES;
        // Filter: TPN neighbouring threads share a channel; 256 threads cover the channels, further ones take further rows of it.
        constexpr int TPN = 256 / BN, FB = 4;
        const int groups = waves >> 2, grp = tid >> 8;                   // (4 waves at least)
        const int nl = (tid & 255) / TPN, fc0 = tid % TPN;
        const unsigned n_src = (unsigned)((n0 + nl < p.N ? n0 + nl : p.N - 1) * p.R * SC);      // (channels past the last: its filter again, never stored)
        const unsigned f_last = (unsigned)(p.N * p.R * SC - VEC);        // where the filter's last whole vector starts (>= 0: the host checks)
        int pj = pj0, pr = 0, fc = fc0, fr = grp;
        bool more_p = !idle, more_f = grp < groups;                      // (uniform)
        while (more_p || more_f) {
            uint4 vp[PB], vf[FB];
            const int src = e0 + pj * VEC;
            int start = src;
            if (!inner) {
                start = src > WC - VEC ? WC - VEC : src;
                start = start < 0 ? 0 : start;
            }
            if (more_p) {
#pragma unroll
                for (int u = 0; u < PB; ++u) {
                    const int row = pr + prow0 + u * prows, ih = ih0 + row;
                    const bool inside = (unsigned)ih < (unsigned)p.H && pj < chunks && row < rows;
                    __builtin_memcpy(&vp[u], image + (inside ? (unsigned)(ih * WC + start) * (unsigned)ES : 0u), 16);
                }
            }
            const unsigned f_src = n_src + (unsigned)((fc < CPR ? fc : 0) * VEC);
            if (more_f) {
#pragma unroll
                for (int u = 0; u < FB; ++u) {
                    const int r = fr + u * groups < p.R ? fr + u * groups : p.R - 1;           // scalar
                    const unsigned at = f_src + (unsigned)(r * SC);
                    __builtin_memcpy(&vf[u], (const char*)p.B + (at < f_last ? at : f_last) * (unsigned)ES, 16);
                }
            }
            if (more_p) {
#pragma unroll
                for (int u = 0; u < PB; ++u) {
                    const int row = pr + prow0 + u * prows, ih = ih0 + row;
                    const bool inside = (unsigned)ih < (unsigned)p.H;
                    uint4 v = vp[u];
                    if (!inner) v = shift_up<ES>(shift_down<ES>(v, src > start ? src - start : 0), src < start ? start - src : 0);
                    v = make_uint4(inside ? v.x : 0u, inside ? v.y : 0u, inside ? v.z : 0u, inside ? v.w : 0u);      // rows outside the image are zeros
                    if (row < rows && pj < chunks) *(uint4*)(s_patch + row * RB + pj * 16) = v;
                }
                pr += PB * prows;                        // further rows, then further columns
                if (pr >= rows) { pr = 0; pj += lpr; }
                more_p = pj - pj0 < chunks;
            }
            if (more_f) {
                if (fc < CPR) {
                    const unsigned keep = fc == CPR - 1 ? 0u : ~0u;
                    const unsigned m0 = tail[0] | keep, m1 = tail[1] | keep, m2 = tail[2] | keep, m3 = tail[3] | keep;
                    char* const dst = s_filt + nl * f_row + fc * 16;
#pragma unroll
                    for (int u = 0; u < FB; ++u) {
                        const int r = fr + u * groups;
                        if (r < 2 * pairs) {
                            uint4 v = vf[u];
                            const unsigned at = f_src + (unsigned)(r * SC);
                            if (at > f_last) v = shift_down<ES>(v, (int)(at - f_last));      // (the filter's very last chunk)
                            const bool live = r < p.R;                   // an odd row count is filled up with zeros
                            *(uint4*)(dst + r * CPR * 16) = live ? make_uint4(v.x & m0, v.y & m1, v.z & m2, v.w & m3) : make_uint4(0, 0, 0, 0);
                        }
                    }
                }
                fr += FB * groups;
                if (fr >= 2 * pairs) { fr = grp; fc += TPN; }
                more_f = fc - fc0 < CPR;
            }
        }
        for (int j = lane; j < chunks; j += 64) *(uint4*)(s_patch + rows * RB + j * 16) = make_uint4(0, 0, 0, 0);
    }
    const int ncols = p.N - n0 < BN ? p.N - n0 : BN;
    acc_e bias_r[NI];
    {
        const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc((void*)((const acc_e*)p.bias + n0), 0, p.bias ? ncols * 4 : 0, 0x00020000);
#pragma unroll
        for (int j = 0; j < NI; ++j) bias_r[j] = __builtin_bit_cast(acc_e, __builtin_amdgcn_raw_buffer_load_b32(rb, (j * 32 + l31) * 4, 0, 0));
    }
    // MFMA block i covers tile rows 2*i and 2*i + 1: lane row l31 is pixel (2*i + l31 / 16, l31 % 16)
    const int row_step = p.dil_h * RB;
    unsigned a_px[2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
        a_px[i] = (unsigned)((2 * i + (l31 >> 4)) * p.stride_h * RB + (l31 & 15) * p.stride_w * p.Cin * ES + g * row_step);
    // a place's misalignment is the lane's: chunks and rows are whole multiples of 16 bytes apart
    const unsigned shift0 = a_px[0] & 3u, shift1 = a_px[1] & 3u;
    if constexpr (SHIFT) { a_px[0] -= shift0; a_px[1] -= shift1; }
    const char* b_at = s_filt + l31 * f_row + g * CPR * 16;
    __syncthreads();
    if (idle) return;
    acc_t acc[2][NI];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0;               // reduction init

    // ------------------------------------------------------------ MFMA
    // (four waves of a SIMD cover each other's LDS latency; fetching a k-step ahead costs the registers of the fourth)
    for (int pair = 0; pair < pairs; ++pair) {
        // the second row of the last pair of an odd count: zeros instead of whatever lies below the patch (0 * Inf is not 0)
        if (2 * pair + 1 == p.R && g) a_px[0] = a_px[1] = (unsigned)(rows * RB);
        const char* a0 = s_patch + a_px[0];
        const char* a1 = s_patch + a_px[1];
        for (int c = 0; c < CPR; ++c) {
            uint4 af[2], bf[NI];
            __builtin_memcpy(&af[0], __builtin_assume_aligned(a0, 4), 16);
            __builtin_memcpy(&af[1], __builtin_assume_aligned(a1, 4), 16);
            unsigned top[2];
            if constexpr (SHIFT) { top[0] = *(const unsigned*)(a0 + 16); top[1] = *(const unsigned*)(a1 + 16); }
#pragma unroll
            for (int j = 0; j < NI; ++j) bf[j] = *(const uint4*)(b_at + j * 32 * f_row);
            a0 += 16; a1 += 16; b_at += 16;
            if constexpr (SHIFT) {
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const unsigned s = i ? shift1 : shift0;
                    af[i] = make_uint4(__builtin_amdgcn_alignbyte(af[i].y, af[i].x, s), __builtin_amdgcn_alignbyte(af[i].z, af[i].y, s),
                                       __builtin_amdgcn_alignbyte(af[i].w, af[i].z, s), __builtin_amdgcn_alignbyte(top[i], af[i].w, s));
                }
            }
            if (c == CPR - 1) {                          // past the filter row: elements of other taps' pixels
#pragma unroll
                for (int i = 0; i < 2; ++i) af[i] = make_uint4(af[i].x & tail[0], af[i].y & tail[1], af[i].z & tail[2], af[i].w & tail[3]);
            }
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < NI; ++j) acc[i][j] = InTraits<DT>::mfma(af[i], bf[j], acc[i][j]);
        }
        b_at += CPR * 16;
        a_px[0] += 2 * row_step; a_px[1] += 2 * row_step;
    }

    // ------------------------------------------------------------ fused epilogue
    const bool fused = p.bias != nullptr || p.relu != 0;
#pragma unroll
    for (int j = 0; j < NI; ++j) asm volatile("" ::"v"(bias_r[j]));
    const long long left_px = ((long long)(p.batch_imgs - img) * p.P - op0) * p.Q - oq0;                   // pixels from the tile's first one on
    const __amdgpu_buffer_rsrc_t rc = __builtin_amdgcn_make_buffer_rsrc(
        (void*)((out_t*)p.C + (((long long)img * p.P + op0) * p.Q + oq0) * p.N + n0), 0, (int)((left_px * p.N - n0) * OS), 0x00020000);      // < 2^31: the host checks
    const int px_bytes = p.N * OS;
    const int lane_px = 4 * g;                           // register r is row 8*(r/4) + 4*g + r%4 of the block
    const bool whole = op0 + 4 <= p.P && oq0 + 16 <= p.Q;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            const unsigned col_off = j * 32 + l31 < ncols ? (unsigned)(lane_px * px_bytes + (j * 32 + l31) * OS) : kOutOfRange;
            // (block by block: branches around the whole epilogue make the compiler convert everything in front of them and spill)
            auto emit = [&](auto fused_flag, auto stream_flag, auto whole_flag) __attribute__((always_inline)) {
                constexpr int AUX = decltype(stream_flag)::value ? TIR_STORE_AUX_STREAM : TIR_STORE_AUX;
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int prow = 2 * i + (r >> 3), pcol = 8 * ((r >> 2) & 1) + (r & 3);
                    const bool ok = decltype(whole_flag)::value || (op0 + prow < p.P && oq0 + pcol + lane_px < p.Q);
                    acc_e t = acc[i][j][r];
                    if constexpr (decltype(fused_flag)::value) t = consumer(t, bias_r[j], p.relu);
                    store_value<AUX>(finish_value<OUT>(t, p.scale), rc, (int)(ok ? col_off : kOutOfRange), (prow * p.Q + pcol) * px_bytes);
                }
            };
            auto emit_policy = [&](auto fused_flag, auto whole_flag) __attribute__((always_inline)) {
                if (p.store_nt) emit(fused_flag, std::true_type(), whole_flag);
                else emit(fused_flag, std::false_type(), whole_flag);
            };
            if (fused) {
                if (whole) emit_policy(std::true_type(), std::true_type());
                else emit_policy(std::true_type(), std::false_type());
            } else {
                if (whole) emit_policy(std::false_type(), std::true_type());
                else emit_policy(std::false_type(), std::false_type());
            }
        }
}

}  // namespace tir
