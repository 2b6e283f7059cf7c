// Instantiations of the kernels outside the tile-variant table (fused attention, depth-wise
// convolution) and the tables the dispatcher picks from.
#include "tir_attention.h"
#include "tir_depthwise.h"
#include "tir_launch.h"

namespace tir {

template <int DT, int OUT, int DH, int QW, int KG, int KB, int FORM> static hipError_t launch_attn_as(AttnParams p, hipStream_t stream) {
    p.tiles_m = (p.M + 32 * QW - 1) / (32 * QW);
    const FastDiv dtm = make_fastdiv((unsigned)p.tiles_m);
    p.div_tm_magic = dtm.magic;
    p.div_tm_shift = dtm.shift;
    return launch_kernel(&attention_kernel<DT, OUT, DH, QW, KG, KB, FORM>, dim3((unsigned)(p.batch * p.tiles_m)), dim3(QW * KG * 64), stream, p);
}

// The kernel of a call, by its sizes, head dimension and output type.
AttnKernel attention_kernel_of(long long batch, long long M, long long N, int DH, int OUT) {
    const bool fp32 = OUT == DT_F32;
    const long long tiles = batch * ((M + 127) / 128);        // of 128 queries
    // Two workgroups of four waves fill a CU.  Up to half a tile per CU four key groups on tiles of 64 queries put eight waves on a CU instead
    // of four.  The merge costs about a chunk's time: from five chunks in all on at d = 64 (four groups of 64 keys), at d = 128 from three
    // chunks of 32 per group.  (Two groups on
    // 128 queries, up to one tile per CU, pay no more since a wave runs its softmax under its own MFMAs.)
    // One, two and four groups, bf16, us (tiles of 128 queries x keys):
    //   d = 128: 64 x 320 9.0 / 10.6 / 9.4, 64 x 400 11.3 / 12.2 / 10.7, 128 x 400 11.8 / 12.8 / 11.4, 128 x 1000 22.0 / 23.6 / 20.3,
    //            144 x 1000 22.3 / 24.0 / 36.2, 256 x 1000 29.6 / 29.9 / 39.2
    //   d = 64:  64 x 256 5.91 / 6.46 / 5.75, 128 x 256 5.97 / 6.63 / 6.06, 64 x 320 6.60 / 7.38 / 6.31, 128 x 1000 15.4 / 15.8 / 11.8,
    //            144 x 1000 15.8 / 16.5 / 22.0, 384 x 1000 29.5 / 33.9 / 34.5
    if (tiles <= 128 && N >= (DH == 64 ? 257 : 384)) return ATTN_T64_GROUPS;
    // Heads of one tile read their keys and values once.  Where a call's operands and output are more than half the 256 MB memory-side cache, so that the next call finds
    // nothing of this one's there unless it is the same call again, and the workgroups are enough to be bound by memory, or where keys and values do not fit that cache at all, their
    // copies are non-temporal.  The same operands again / three sets in turn, us, plain and non-temporal:
    //   d = 128: 1024 x 400 (277 MB) 44.9 / 58.8 and 49.8 / 49.3, 640 x 600 (239 MB) 43.1 / 55.2 and 47.2 / 48.6; from fewer workgroups or bytes plain is as good or better:
    //            200 x 2000 (211 MB) 38.7 / 52.2 and 47.9 / 49.6, 520 x 400 (141 MB) 32.1 / 39.4 and 33.6 / 34.6, 800 x 200 (134 MB) 29.3 / 31.3 and 30.8 / 31.2
    const long long kv = batch * N * DH * 4, bytes = kv + batch * M * DH * (2 + (fp32 ? 4 : 2));
    const bool once = M <= 128 && (kv > (256ll << 20) || (tiles > 384 && bytes > (136ll << 20)));
    // Few keys that leave the last chunk of 64 half empty: chunks of 32.  64 and 32 keys per chunk, us:
    //   d = 64:  100 x 77 4.74 / 4.38, 100 x 160 5.54 / 5.21, 384 x 77 6.04 / 5.72, 800 x 77 9.33 / 8.17, 2000 x 150 28.3 / 26.5
    //   d = 128: 100 x 77 6.26 / 5.76, 320 x 160 11.7 / 10.8, 512 x 160 15.4 / 15.5, 1024 x 96 22.8 / 20.4
    // (the sequential form's non-temporal copies at d = 64: 2000 x 160 25.1 / 31.7 in chunks of 32, 27.1 / 27.3)
    if ((N - 1) % 64 < 32 && N <= 160 && !(DH == 64 && once)) return ATTN_T128_C32;
    // More than two workgroups per CU at d = 64: four of the sequential form fit a CU, three of the other.  Pipelined and sequential, us: 20 x 4096 x 4096
    // 112 / 108, 75 x 1024 x 600 22.2 / 21.5, 750 x 512 x 1000 131 / 120, 60 x 4096 x 1000 79.9 / 77.3, 600 x 512 x 128 22.1 / 20.3, 2000 x 197 x 197 52.5 / 49.0; at
    // two per CU 16 x 4096 x 4096 81.0 / 82.5, and where long heads leave a sliver for a second round of four 203 x 738 x 1818 88.7 / 90.3, 99 x 1372 x 833 43.9 / 44.7
    // (short ones 300 x 512 x 192 15.2 / 14.7, 150 x 1024 x 600 37.5 / 37.1).  Heads of one tile, where each workgroup reads its own keys: up to four per CU and few keys only
    // (640 x 320 17.0 / 16.1, 800 x 192 16.6 / 14.2, 1024 x 64 8.8 / 7.0, 700 x 200 13.3 / 12.4; 600 x 600 23.2 / 24.8, 1500 x 256 27.3 / 29.2; beyond four one chunk or two only, 2000 heads of 40 queries x 64 12.3 / 11.0, x 128 17.1 / 16.4,
    // 1500 x 128 18.3 / 17.8, but 1100 x 64 9.7 / 10.0),
    // and where the copies are non-temporal, which those of heads of one tile always are in this form (pipelined plain, non-temporal and sequential, three sets in turn:
    // 800 x 600 38.5, 35.4 and 33.2, 1024 x 1000 63.0, 53.6 and 53.4, 2000 x 400 58.6, 52.5 and 50.7; the same operands again 32.0, 33.7 and 31.9, 52.7, 55.1 and 54.2, 46.7, 52.0 and 52.4).
    //
    // Its tiles of 256 queries, eight waves that copy keys and values once instead of twice: where three or four of the smaller workgroups per CU would be one
    // round, pad no more rows, the heads are of two such tiles or more and the keys are not few.  Sequential with 128 and 256 queries, us: 32 x 4096 x 4096 158 / 152,
    // 256 x 512 x 768 33.5 / 32.2, 100 x 1024 x 512 20.8 / 19.9, 30 x 4096 x 400 19.8 / 18.6; few keys 200 x 512 x 256 12.9 / 13.2; fp32 output, twice the tile in LDS and the stores,
    // 256 x 512 x 320 17.3 / 18.3 (512 keys 24.7 / 25.2, 768 34.0 / 33.7); one tile per head 512 x 256 x 256 16.1 / 18.7 with three sets in turn, to fp32 17.2 / 21.1;
    // fewer tiles 24 x 4096 x 4096 116 / 126, more 750 x 512 x 1000 120 / 124, 40 x 4096 x 2000 99.6 / 110.
    if (DH == 64) {
        if (tiles > 768 && tiles <= 1024 && M > 256 && N >= (fp32 ? 512 : 256) && (M + 127) / 128 % 2 == 0) return ATTN_T256_SEQUENTIAL;
        const bool sliver = tiles > 1024 && tiles <= 1280 && N > 600;
        if ((M > 128 && tiles > 512 && !sliver) || (tiles >= 512 && (N <= (tiles <= 1024 ? 400 : 128) || once))) return ATTN_T128_SEQUENTIAL;
    }
    // Tiles of 256 queries at d = 128: one workgroup of eight waves in the place of two of four, which copies keys and values once instead of twice (and the long launches
    // are bound by power).  Where they pad no more rows, and where the CUs of the last round would hold two of the smaller workgroups anyway.  128 and 256 queries, us:
    // 16 x 4096 x 4096 145.4 / 140.1, 75 x 512 x 2000 57.9 / 52.5, 24 x 1536 x 1536 43.5 / 40.1, 130 x 256 x 1000 30.8 / 29.9, 100 x 900 x 700 47.5 / 46.7;
    // 64 x 1024 x 512 20.9 / 20.9, x 256 12.4 / 13.2; to fp32 390 x 256 x 512 40.1 / 45.6, x 700 51.1 / 56.0, 200 x 256 x 1000 36.1 / 35.6; one small workgroup per CU in the last
    // round: 16 x 2048 x 4096 77.5 / 95.7, 40 x 2048 x 300 20.5 / 26.5.
    if (DH == 128 && N >= (fp32 ? 768 : 512) && (M + 127) / 128 % 2 == 0 && (tiles - 1) % 512 >= 256) return ATTN_T256;
    return once ? ATTN_T128_STREAM : ATTN_T128;
}

template <int DT, int OUT, int DH> static hipError_t launch_attn(const AttnParams& p, hipStream_t stream) {
    const AttnKernel k = attention_kernel_of(p.batch, p.M, p.N, DH, OUT);
    if (k == ATTN_T64_GROUPS) return launch_attn_as<DT, OUT, DH, 2, 4, DH == 64 ? 64 : 32, ATTN_PIPED>(p, stream);
    if (k == ATTN_T128_C32) return launch_attn_as<DT, OUT, DH, 4, 1, 32, ATTN_PIPED>(p, stream);
    if (k == ATTN_T128_STREAM) return launch_attn_as<DT, OUT, DH, 4, 1, 64, ATTN_PIPED_STREAM>(p, stream);
    if constexpr (DH == 64) {
        if (k == ATTN_T128_SEQUENTIAL) return launch_attn_as<DT, OUT, DH, 4, 1, 64, ATTN_SEQUENTIAL>(p, stream);
        if (k == ATTN_T256_SEQUENTIAL) return launch_attn_as<DT, OUT, DH, 8, 1, 64, ATTN_SEQUENTIAL>(p, stream);
    } else {
        if (k == ATTN_T256) return launch_attn_as<DT, OUT, DH, 8, 1, 64, ATTN_PIPED>(p, stream);
    }
    return launch_attn_as<DT, OUT, DH, 4, 1, 64, ATTN_PIPED>(p, stream);
}

attn_launch_fn attention_launcher(int dt, int out, int dh) {
#define TIR_ATTN(DT, OUT, DH) \
    if (dt == DT && out == OUT && dh == DH) return &launch_attn<DT, OUT, DH>;
    TIR_ATTN(DT_F16, DT_F16, 64) TIR_ATTN(DT_F16, DT_F32, 64) TIR_ATTN(DT_F16, DT_F16, 128) TIR_ATTN(DT_F16, DT_F32, 128)
    TIR_ATTN(DT_BF16, DT_BF16, 64) TIR_ATTN(DT_BF16, DT_F32, 64) TIR_ATTN(DT_BF16, DT_BF16, 128) TIR_ATTN(DT_BF16, DT_F32, 128)
#undef TIR_ATTN
    return nullptr;
}

template <int DT, int OUT, bool STREAM> static hipError_t launch_dw_as(const Params& p, hipStream_t stream) {
    constexpr int VEC = 16 / elem_size(DT);
    constexpr int PP = 256 / (kDwChannels / VEC);
    dim3 grid((unsigned)((p.M + kDwPixPerThread * PP - 1) / (kDwPixPerThread * PP)), (unsigned)((p.Cin + kDwChannels - 1) / kDwChannels));
    if (p.R == 3 && p.S == 3 && p.dil_w == 1 && (p.stride_w == 1 || p.stride_w == 2) && p.Q >= kDwBlockPix) {
        auto blocks_x = [&](int np) { return (unsigned)(depthwise_workgroups(DT, p.batch_imgs, p.P, p.Q, p.Cin, np) / grid.y); };
        // another split of the pixels than the plan's: four columns of two rows, or eight columns
        auto split = [&](unsigned rows, unsigned groups) {
            Params q = p;
            const FastDiv dq = make_fastdiv(groups), dpq = make_fastdiv(rows * groups);
            q.div_dwq_magic = dq.magic; q.div_dwq_shift = dq.shift;
            q.div_dwpq_magic = dpq.magic; q.div_dwpq_shift = dpq.shift;
            return q;
        };
        if constexpr (OUT == DT && DT != DT_I8) {
            if (p.stride_w == 1 && p.stride_h == 1 && p.dil_h == 1 && depthwise_rows(DT, OUT, p.batch_imgs, p.P, p.Q, p.Cin) == 2) {
                const unsigned rows = (unsigned)(p.P + 1) / 2;
                grid.x = (unsigned)(depthwise_workgroups(DT, p.batch_imgs, rows, p.Q, p.Cin, kDwBlockPix) / grid.y);
                return launch_kernel(&depthwise3x3_blocked_kernel<DT, OUT, 1, kDwBlockPix, 2, STREAM>, grid, dim3(256), stream, split(rows, (unsigned)(p.Q + kDwBlockPix - 1) / kDwBlockPix));
            }
        }
        if constexpr (OUT != DT_I32) {
            if (depthwise_pixels(DT, OUT, p.batch_imgs, p.P, p.Q, p.Cin, p.stride_w) == 8) {
                grid.x = blocks_x(8);
                return launch_kernel(&depthwise3x3_blocked_kernel<DT, OUT, 1, 8, 1, STREAM>, grid, dim3(256), stream, split((unsigned)p.P, (unsigned)(p.Q + 7) / 8));
            }
        }
        grid.x = blocks_x(kDwBlockPix);
        return launch_kernel(p.stride_w == 1 ? &depthwise3x3_blocked_kernel<DT, OUT, 1, kDwBlockPix, 1, STREAM> : &depthwise3x3_blocked_kernel<DT, OUT, 2, kDwBlockPix, 1, STREAM>, grid,
                             dim3(256), stream, p);
    }
    return launch_kernel(p.R == 3 && p.S == 3 ? &depthwise_kernel<DT, OUT, true, STREAM> : &depthwise_kernel<DT, OUT, false, STREAM>, grid, dim3(256), stream, p);
}

template <int DT, int OUT> static hipError_t launch_dw(const Params& p, hipStream_t stream) {
    return p.store_nt ? launch_dw_as<DT, OUT, true>(p, stream) : launch_dw_as<DT, OUT, false>(p, stream);
}

dw_launch_fn depthwise_launcher(int dt, int out) {
#define TIR_DW(DT, OUT) \
    if (dt == DT && out == OUT) return &launch_dw<DT, OUT>;
    TIR_DW(DT_F16, DT_F16) TIR_DW(DT_F16, DT_F32) TIR_DW(DT_BF16, DT_BF16) TIR_DW(DT_BF16, DT_F32) TIR_DW(DT_I8, DT_I32) TIR_DW(DT_I8, DT_I8)
#undef TIR_DW
    return nullptr;
}

}  // namespace tir
