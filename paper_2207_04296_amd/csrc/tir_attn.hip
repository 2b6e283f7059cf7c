// Instantiations of the kernels outside the tile-variant table (fused attention, depth-wise
// convolution) and the tables the dispatcher picks from.
#include "tir_attention.h"
#include "tir_depthwise.h"
#include "tir_launch.h"

namespace tir {

template <int DT, int OUT, int DH, int QW, int KG, int KB> static hipError_t launch_attn_as(AttnParams p, hipStream_t stream) {
    p.tiles_m = (p.M + 32 * QW - 1) / (32 * QW);
    const FastDiv dtm = make_fastdiv((unsigned)p.tiles_m);
    p.div_tm_magic = dtm.magic;
    p.div_tm_shift = dtm.shift;
    return launch_kernel(&attention_kernel<DT, OUT, DH, QW, KG, KB>, dim3((unsigned)(p.batch * p.tiles_m)), dim3(QW * KG * 64), stream, p);
}

template <int DT, int OUT, int DH> static hipError_t launch_attn(const AttnParams& p, hipStream_t stream) {
    const long long tiles = (long long)p.batch * ((p.M + 127) / 128);        // of 128 queries
    // Two workgroups of four waves fill a CU.  Up to about one tile per CU a second key group takes the place of the second workgroup,
    // up to half a tile four groups on half-tiles do; the merge costs about a chunk's time, so the groups need a few chunks each.  At
    // d = 128 two groups take a CU's whole LDS, so that a second round of workgroups waits for the first; at d = 64 two such workgroups share a
    // CU, and with many keys they pay up to a tile and a half per CU.
    // One, two and four groups, bf16, us (tiles of 128 x 128 queries x keys):
    //   d = 128: 128 tiles x 1000 keys 31.3 / 27.3 / 22.3, 144 x 1000 31.7 / 27.9 / 39.4, 160 x 2000 60.4 / 51.4, 200 x 400 16.5 / 16.2, 256 x 400
    //            17.4 / 17.5, 256 x 600 23.1 / 22.8, 256 x 2000 64.6 / 58.5, 320 x 1000 43.9 / 59.7; 60 heads of 512 x 512 16.1 / 14.4
    //   d = 64:  128 x 1000 21.4 / 16.8 / 12.2, 256 x 400 11.2 / 9.8, 384 x 1000 29.8 / 29.1, 384 x 400 15.0 / 15.3, 448 x 1000 31.4 / 32.4
    if (tiles <= 128 && p.N > 256) return launch_attn_as<DT, OUT, DH, 2, 4, DH == 64 ? 64 : 32>(p, stream);
    if (tiles <= (DH == 64 && p.N >= 1024 ? 384 : 256) && p.N >= 384) return launch_attn_as<DT, OUT, DH, 4, 2, 64>(p, stream);
    return launch_attn_as<DT, OUT, DH, 4, 1, 64>(p, stream);
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
        // four adjacent pixels per thread
        const long long groups = (long long)p.batch_imgs * p.P * ((p.Q + kDwBlockPix - 1) / kDwBlockPix);
        grid.x = (unsigned)((groups + PP - 1) / PP);
        return launch_kernel(p.stride_w == 1 ? &depthwise3x3_blocked_kernel<DT, OUT, 1, STREAM> : &depthwise3x3_blocked_kernel<DT, OUT, 2, STREAM>, grid,
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
