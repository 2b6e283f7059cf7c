// Stride-1 convolution with an LDS-resident input patch, by blocks of channels (A_CONV_BLOCKS).
//
// The implicit-GEMM kernel sends every input pixel through the global->LDS copy once per filter tap, and what a CU gets out of
// the L2s (40 - 50 bytes per clock) bounds every tile below 256x256.  Here a workgroup copies the input rows its BM output pixels
// touch once per block of ROWB bytes of channels and multiplies all taps of the block from that patch; per tap only the filter's
// slab [BN output channels][ROWB bytes] is copied.
//
//   pixels     a tile is BM consecutive pixels of a strip of output columns (the host cuts wide images into strips so that
//              the patch stays small), counted over rows and images: a tile may span several images, whose
//              rows then stand below each other in the patch, blk_vh rows per image
//   patch      [virtual row][column][ROWB], 16-byte columns swizzled by the pixel's index like a K-major tile.  (Rows padded by one chunk would save
//              the XORs, but then a copy instruction's lanes straddle 64-byte segments: 42 cycles per KiB and CU instead of 17.)
//   channels   two patch buffers: the next block arrives while this one is multiplied
//   filter     a ring of three stages of one filter row (TW taps)
//   waves      four copy, the others multiply (a copy instruction holds its wave for ~60 cycles)
// With one multiplying wave per SIMD every instruction between its MFMAs costs matrix time, so the loop over a block's taps is unrolled (TH x TW
// taps are compile-time) and the lane keeps the address of every tap's pixel: with the taps' places worked out in the loop it took ~540 cycles
// per tap of a 128x64 tile instead of the 256 of its MFMAs.
// Channels past the group's last one and pixels outside the image are lanes outside the buffer descriptor: zeros.
//
// What bounds it now: a 128x64 tile of 16x14x14, 256 -> 128, 4x4 stride 2 by phase (4 blocks of 4 taps) spends 4000 cycles until its first MFMA, ~340 per tap and
// 3400 in the store.  The swizzle follows the patch's pixels, so the lanes of a fragment that crosses a row of the patch meet on banks: 2007 cycles per
// workgroup of that call (SQ_LDS_BANK_CONFLICT), 484 of 8x28x28, 32 -> 32 in each of 8 groups, dilation 2 int8 in one strip, 975 in two.  us, implicit GEMM (or, 64 channels,
// the patch kernel) -> here: the first call 10.7 -> 8.6, the second 5.6 -> 4.9, 14x11x34, 112 -> 16 in each of 8 groups, 5x5 25.8 -> 14.6, 21x37x7, 64 -> 16 in each of 8
// groups 12.9 -> 5.9.  Tried: the unit's place worked out
// by scalars in each block instead of an address register per copy instruction (8.9 -> 10.2), a ring of four stages (the same), half of the first patch copied by
// the multiplying waves instead of a quarter (8.6 -> 8.9) or none (the same; the second call in two strips 5.3 -> 5.65), two sets of multiplying waves splitting a tap's k-steps (9.2, was 8.9).
#pragma once
#include "tir_kernel.h"

namespace tir {

// Largest divisor of n that is at most 4 (at least 2 where n is even or divisible by 3), or 5: how many fragment sets rotate over n k-steps.
constexpr int block_sets(int n) { return n % 4 == 0 ? 4 : n % 3 == 0 ? 3 : n % 5 == 0 ? 5 : 2; }

// Tiles of 64-byte blocks with two MFMA blocks per wave are there for launches of many rounds: two fragment sets and 128 registers, so that two
// workgroups share a CU and cover each other's set-up, waits and store.
template <class C, int TH> constexpr bool block_pair() { return C::ROWB == 64 && C::MI * C::NI == 2 && TH < 5; }

template <class C, int TH, int TW>
__global__ void __launch_bounds__(C::THREADS, (block_pair<C, TH>() ? 4 : 2)) conv_blocks_kernel(const Params p) {
    typedef typename InTraits<C::DT>::acc_t acc_t;
    typedef typename std::conditional<std::is_same<acc_t, f32x16>::value, float, int>::type acc_e;
    typedef typename OutTraits<C::OUT>::type out_t;
    typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
    constexpr int ES = C::ES, OS = (int)sizeof(out_t), CB = C::ROWB, RCH = CB / 16;
    constexpr int CW = C::CW, KSTEPS = CB / 32, RS = TH * TW;
    constexpr int MW = C::WM * C::WN;                                     // multiplying waves
    constexpr int SLAB = C::BN * CB, UB = SLAB / 1024;                    // one tap's filter slab and its copy instructions
    constexpr int UBW = (UB + CW - 1) / CW, RING = 3 * TW * SLAB;
    constexpr int NSET = C::MI * C::NI >= 4 || block_pair<C, TH>() ? 2 : block_sets(RS * KSTEPS), LA = NSET - 1;     // fragment sets; k-steps the LDS reads run ahead (four MFMAs cover a read)
    static_assert(TH >= 2 && RS * KSTEPS % NSET == 0, "");

    extern __shared__ __attribute__((aligned(2048))) char smem[];
    asm volatile("" ::"s"(p.A), "s"(p.B), "s"(p.C), "s"(p.M), "s"(p.N), "s"(p.K), "s"(p.tiles_m), "s"(p.tiles_n), "s"(p.div_gw_magic), "s"(p.div_gw_shift), "s"(p.a_bs),
                 "s"(p.b_bs), "s"(p.c_bs), "s"(p.c_rs), "s"(p.bias), "s"(p.bias_bs), "s"(p.relu), "s"(p.scale), "s"(p.batch_imgs), "s"(p.store_nt));
    asm volatile("" ::"s"(p.H), "s"(p.W), "s"(p.Cin), "s"(p.Cg), "s"(p.P), "s"(p.Q), "s"(p.S), "s"(p.pad_h), "s"(p.pad_w), "s"(p.dil_h), "s"(p.dil_w), "s"(p.phases_h));
    asm volatile("" ::"s"(p.blk_tw), "s"(p.blk_pw), "s"(p.blk_vh), "s"(p.blk_patch), "s"(p.blk_strip_tiles), "s"(p.div_tm_magic), "s"(p.div_tm_shift), "s"(p.blk_tw_magic),
                 "s"(p.blk_tw_shift), "s"(p.blk_pw_magic), "s"(p.blk_pw_shift), "s"(p.blk_vh_magic), "s"(p.blk_vh_shift), "s"(p.blk_p_magic), "s"(p.blk_p_shift));

    const int lane = threadIdx.x & 63;
    const int wave_wg = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const bool copier = wave_wg < CW;           // (the first wave of each SIMD starts ~0.3 us before the second)
    const int wave = wave_wg - CW;              // multiplying wave
    const int wm = wave / C::WN, wn = wave % C::WN;

    int tm, tn;
    tile_of_block(blockIdx.x, p.tiles_m, p.tiles_n, p.div_gw_magic, p.div_gw_shift, &tm, &tn);
    const int n0 = tn * C::BN;
    const int ncols = p.N - n0 < C::BN ? p.N - n0 : C::BN;
    long long bz = blockIdx.y;

    // Transposed convolution by output phase: every phase has TH x TW taps (the host checks), taken backwards (see
    // contract_direct_kernel): cursor tap (fr, fs) is filter tap (f_r0 - f_step_h * fr, f_s0 - f_step_w * fs).
    int pad_h = p.pad_h, pad_w = p.pad_w, f_r0 = 0, f_s0 = 0, f_step_h = -1, f_step_w = -1, ph = 0, pw = 0;
    const bool phased = p.phases_h != 0;
    if (phased) {
        const int phase = (int)fastdiv((unsigned)bz, p.div_grp_magic, p.div_grp_shift);
        bz -= (long long)phase * p.conv_groups;
        ph = (int)fastdiv((unsigned)phase, p.div_phw_magic, p.div_phw_shift);
        pw = phase - ph * p.phases_w;
        const int qh = (int)fastdiv((unsigned)(ph + p.t_pad_h), p.div_phh_magic, p.div_phh_shift), qw = (int)fastdiv((unsigned)(pw + p.t_pad_w), p.div_phw_magic, p.div_phw_shift);
        pad_h = (TH - 1) - qh;
        pad_w = (TW - 1) - qw;
        f_r0 = ph + p.t_pad_h - qh * p.phases_h + p.phases_h * (TH - 1);
        f_s0 = pw + p.t_pad_w - qw * p.phases_w + p.phases_w * (TW - 1);
        f_step_h = p.phases_h;
        f_step_w = p.phases_w;
    }
    const int ncb = (p.Cg * ES + CB - 1) / CB;                            // blocks of channels

    // ---- pixels of the tile
    const int strip = (int)fastdiv((unsigned)tm, p.div_tm_magic, p.div_tm_shift);
    const int first = (tm - strip * p.blk_strip_tiles) * C::BM;           // pixel of the strip
    const int tw = p.blk_tw, total = p.batch_imgs * p.P * tw;
    const int last = first + C::BM <= total ? first + C::BM - 1 : total - 1;
    const int q_first = strip * tw;
    const int row_a = (int)fastdiv((unsigned)first, p.blk_tw_magic, p.blk_tw_shift), row_b = (int)fastdiv((unsigned)last, p.blk_tw_magic, p.blk_tw_shift);
    const int img_a = (int)fastdiv((unsigned)row_a, p.blk_p_magic, p.blk_p_shift), img_b = (int)fastdiv((unsigned)row_b, p.blk_p_magic, p.blk_p_shift);
    const int p_a = row_a - img_a * p.P, p_b = row_b - img_b * p.P;
    const int PW = p.blk_pw;                                              // columns of the patch
    char* const s_patch = smem + RING;

    // ---- patch: chunk c of a buffer is (physical) column c % RCH of pixel c / RCH; a copy instruction (unit) moves 64 chunks
    const int nv = (img_b - img_a) * p.blk_vh + (p_b - p_a) + (TH - 1) * p.dil_h + 1;
    const int units = (nv * PW * RCH + 63) >> 6;
    const char* const Ab = (const char*)p.A + bz * p.a_bs * ES;
    const i32x4 ra = make_rsrc32(Ab, (unsigned)((long long)p.batch_imgs * p.H * p.W * p.Cin * ES - bz * p.a_bs * ES));
    auto patch_offset = [&](int u) __attribute__((always_inline)) -> unsigned {        // byte of the lane's pixel in unit u, or out of range
        const unsigned px = (unsigned)(u * (64 / RCH) + lane / RCH);
        const int v = (int)fastdiv(px, p.blk_pw_magic, p.blk_pw_shift);
        const int pc = (int)px - v * PW;
        const int iw = q_first - pad_w + pc, vv = v + p_a;
        const int i = (int)fastdiv((unsigned)vv, p.blk_vh_magic, p.blk_vh_shift);
        const int ih = vv - i * p.blk_vh - pad_h, img = img_a + i;
        const bool ok = img < p.batch_imgs && (unsigned)ih < (unsigned)p.H && (unsigned)iw < (unsigned)p.W && v < nv;
        return ok ? (unsigned)(((img * p.H + ih) * p.W + iw) * (p.Cin * ES)) : kOutOfRange;
    };
    // logical column of the lane's chunk (the swizzle repeats every 16 rows, two units of 8 or one of 16)
    auto patch_column = [&](int u) __attribute__((always_inline)) -> int { return ((lane % RCH) ^ kmajor_swz<CB>(u * (64 / RCH) + lane / RCH)) * 16; };
    // The first block's patch is shared out: `mine` of the units to each copy wave, `head` of them at the start, the rest to the multiplying waves.
    const int per_wave = (units + CW - 1) / CW, head = (3 * per_wave + 3) >> 2;

    if (copier) {
        const int cw = wave_wg;
        const int mine = (units - cw + CW - 1) / CW;
        const int lc = patch_column(cw);
        const char* const Bb = (const char*)p.B + (bz * p.b_bs + (long long)n0 * p.K) * ES;
        const i32x4 rb = make_rsrc32(Bb, (unsigned)((long long)ncols * p.K * ES));
        unsigned a_off[kBlockPatchUnits];
        auto copy_patch = [&](int k, int cb) __attribute__((always_inline)) {
            load_to_lds_at(ra, s_patch + (cb & 1) * p.blk_patch + (k * CW + cw) * 1024, lc < p.Cg * ES - cb * CB ? a_off[k] : kOutOfRange, cb * CB);
        };
        // the wave's copy instructions of a patch (an address register each: unrolled, in groups of five behind a branch)
        auto each_unit = [&](int from, int to, auto unit) __attribute__((always_inline)) {
#pragma unroll
            for (int k0 = 0; k0 < kBlockPatchUnits; k0 += 5)
                if (k0 < to && k0 + 5 > from) {
#pragma unroll
                    for (int k = k0; k < k0 + 5; ++k)
                        if (k >= from && k < to) unit(k);
                }
        };
        auto address = [&](int k) __attribute__((always_inline)) { a_off[k] = patch_offset(k * CW + cw); a_off[k] = a_off[k] == kOutOfRange ? kOutOfRange : a_off[k] + lc; };
        // ---- filter: chunk c of a slab is (physical) column c % RCH of output channel c / RCH
        unsigned b_off[UBW], b_cur[UBW];                                  // b_cur: without the chunks past the block's channels
#pragma unroll
        for (int k = 0; k < UBW; ++k) {
            const int n = (k * CW + cw) * (64 / RCH) + lane / RCH;
            b_off[k] = n < ncols ? (unsigned)n * (unsigned)(p.K * ES) + lc : kOutOfRange;
            b_cur[k] = lc < p.Cg * ES ? b_off[k] : kOutOfRange;
        }
        const int b_mine = (UB - cw + CW - 1) / CW;                       // copy instructions of this wave per tap
        // The next stage to copy: its slot of the ring, its filter row, the block's first byte.
        const int step_s = -f_step_w * p.Cg * ES, step_r = -f_step_h * p.S * p.Cg * ES;
        int s_row = 0, s_cb = 0, s_slot = 0, s_at = (f_r0 * p.S + f_s0) * p.Cg * ES, s_first = s_at;
        auto copy_stage = [&]() __attribute__((always_inline)) {
            const char* dst = smem + s_slot + cw * 1024;
#pragma unroll
            for (int t = 0; t < TW; ++t)
#pragma unroll
                for (int k = 0; k < UBW; ++k)
                    if (k * CW + CW <= UB || k < b_mine) load_to_lds_at(rb, dst + t * SLAB + k * CW * 1024, b_cur[k], s_at + t * step_s);
            s_slot = s_slot + TW * SLAB == RING ? 0 : s_slot + TW * SLAB;
            s_at += step_r;
            if (++s_row == TH) {                                          // the next block's first filter row
                s_row = 0;
                ++s_cb;
                s_first += CB;
                s_at = s_first;
                const int left = p.Cg * ES - s_cb * CB;
#pragma unroll
                for (int k = 0; k < UBW; ++k) b_cur[k] = lc < left ? b_off[k] : kOutOfRange;
            }
        };
        copy_stage();
        each_unit(0, mine < head ? mine : head, [&](int k) __attribute__((always_inline)) {
            address(k);
            copy_patch(k, 0);
        });
        const int nst = TH * ncb;
        copy_stage();
        wait_vmcnt_upto(TW * b_mine);                                     // the patch's head and the first stage
        asm volatile("s_barrier" ::: "memory");
        if (ncb > 1) each_unit(head, mine, address);
        // Iteration h: stage h is being multiplied; issue the copies of stage h + 2 and, in a block's first stage, the next block's patch (its
        // buffer was the last block's, which every wave has read), then wait for what the iterations before this one issued: stage h + 1.
        int hc = 0, cb = 0;                                               // stage h inside its block, the block
        for (int h = 0; h + 1 < nst; ++h) {
            int n = 0;
            if (h + 2 < nst) {
                copy_stage();
                n = TW * b_mine;
            }
            if (hc == 0 && cb + 1 < ncb) {
                each_unit(0, mine, [&](int k) __attribute__((always_inline)) { copy_patch(k, cb + 1); });
                n += mine;
            }
            wait_vmcnt_upto(n);
            asm volatile("s_barrier" ::: "memory");
            if (++hc == TH) { hc = 0; ++cb; }
        }
        return;
    }

    // ------------------------------------------------------------ multiplying waves
    // their share of the first patch
    for (int u = head * CW + wave; u < units; u += MW) {
        const unsigned off = patch_offset(u);
        const int lc = patch_column(u);
        load_to_lds_at(ra, s_patch + u * 1024, off != kOutOfRange && lc < p.Cg * ES ? off + lc : kOutOfRange, 0);
    }
    const int l31 = lane & 31, g = lane >> 5;
    const unsigned smem_lds = (unsigned)(unsigned long long)TIR_LDS_PTR(char, smem);
    // Address of every tap's pixel in the current patch buffer: 16-byte column (2 * kk + g) ^ key of its row, for k-step 0; k-step kk flips bits of it.
    int a_at[RS][C::MI];
#pragma unroll
    for (int i = 0; i < C::MI; ++i) {
        int m = first + wm * C::TM + i * 32 + l31;
        m = m < last ? m : last;               // rows past the last re-read it; never stored
        const int row = (int)fastdiv((unsigned)m, p.blk_tw_magic, p.blk_tw_shift);
        const int img = (int)fastdiv((unsigned)row, p.blk_p_magic, p.blk_p_shift);
        const int px = ((img - img_a) * p.blk_vh + (row - img * p.P - p_a)) * PW + (m - row * tw);
#pragma unroll
        for (int t = 0; t < RS; ++t) {
            const int at = (px + (t / TW) * p.dil_h * PW + (t % TW) * p.dil_w) * CB;
            a_at[t][i] = (int)smem_lds + RING + (at | (((at >> 4) & (CB - 16)) ^ (g << 4)));
            asm volatile("" : "+v"(a_at[t][i]));                          // here and now, in a register: not again next to its use
        }
    }
    int b_at[KSTEPS];                          // the lane's filter row in slab 0, by k-step
#pragma unroll
    for (int kk = 0; kk < KSTEPS; ++kk) b_at[kk] = (int)smem_lds + (wn * C::TN + l31) * CB + (((2 * kk + g) ^ kmajor_swz<CB>(l31)) << 4);
    auto lds_read = [&](unsigned at) __attribute__((always_inline)) -> uint4 {
        const u32x4 v = *(const __attribute__((address_space(3))) u32x4*)(unsigned long long)at;
        return make_uint4(v[0], v[1], v[2], v[3]);
    };

    acc_t acc[C::MI][C::NI];
#pragma unroll
    for (int i = 0; i < C::MI; ++i)
#pragma unroll
        for (int j = 0; j < C::NI; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0;   // reduction init
    acc_e bias_r[C::NI];
    load_bias<C>(p, bz, n0, wn, lane, bias_r);

    uint4 af[NSET][C::MI], bf[NSET][C::NI];
    int slot = 0;                              // of the ring: the stage being read
    int flip = p.blk_patch;                    // to the other patch buffer
    // fragment w (pixel blocks, then column blocks) of k-step q of the block (q >= RS * KSTEPS: of the next block) into its set
    auto read_fragment = [&](int q, int w, int s) __attribute__((always_inline)) {
        const int t = q / KSTEPS % RS, kk = q % KSTEPS;
        if (w < C::MI) {
            af[q % NSET][w] = lds_read((unsigned)(a_at[t][w] ^ (kk << 5)));
            if (kk == KSTEPS - 1) a_at[t][w] += flip;                     // (its last use in this block)
        } else {
            bf[q % NSET][w - C::MI] = lds_read((unsigned)(b_at[kk] + s) + (t % TW) * SLAB + (w - C::MI) * 32 * CB);
        }
    };
    asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");         // the first patch and the first stage are in LDS
#pragma unroll
    for (int q = 0; q < LA; ++q)
#pragma unroll
        for (int w = 0; w < C::MI + C::NI; ++w) read_fragment(q, w, 0);
    TIR_FENCE();
    // The MFMAs of k-step q of the block, with the reads of the fragments LA k-steps on between them.
    auto multiply = [&](int q) __attribute__((always_inline)) {
        constexpr int NM = C::MI * C::NI, NR = C::MI + C::NI;
#pragma unroll
        for (int u = 0; u < NM; ++u) {
            acc[u / C::NI][u % C::NI] = InTraits<C::DT>::mfma(af[q % NSET][u / C::NI], bf[q % NSET][u % C::NI], acc[u / C::NI][u % C::NI]);
            TIR_FENCE();
#pragma unroll
            for (int w = u * NR / NM; w < (u + 1) * NR / NM; ++w) {
                read_fragment(q + LA, w, slot);
                TIR_FENCE();
            }
        }
    };
    // Before the first read of the next stage: its copies have landed, and every wave has read this one.
    auto next_stage = [&]() __attribute__((always_inline)) {
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        slot = slot + TW * SLAB == RING ? 0 : slot + TW * SLAB;
    };
    for (int cb = 0;; ++cb) {
#pragma unroll
        for (int q = 0; q < RS * KSTEPS - LA; ++q) {
            if ((q + LA) % (TW * KSTEPS) == 0) next_stage();
            multiply(q);
        }
        if (cb + 1 == ncb) break;
        next_stage();
        flip = -flip;
#pragma unroll
        for (int q = RS * KSTEPS - LA; q < RS * KSTEPS; ++q) multiply(q);
    }
    // the last LA k-steps
#pragma unroll
    for (int q = RS * KSTEPS - LA; q < RS * KSTEPS; ++q)
#pragma unroll
        for (int u = 0; u < C::MI * C::NI; ++u)
            acc[u / C::NI][u % C::NI] = InTraits<C::DT>::mfma(af[q % NSET][u / C::NI], bf[q % NSET][u % C::NI], acc[u / C::NI][u % C::NI]);

    // ------------------------------------------------------------ store: rows of the tile are pixels of the strip
    if (!phased && tw == p.Q) {               // one strip: rows of the output in order
        store_tile<C>(p, bz, first, n0, wm, wn, lane, acc, bias_r);
        return;
    }
    const int out_p = phased ? p.P_full : p.P, out_q = phased ? p.Q_full : p.Q;
    const int step_h = phased ? p.phases_h : 1, step_w = phased ? p.phases_w : 1;
    const long long out_bytes = (long long)p.batch_imgs * out_p * out_q * p.c_rs * OS;
    const __amdgpu_buffer_rsrc_t rc = __builtin_amdgcn_make_buffer_rsrc((void*)((out_t*)p.C + bz * p.c_bs + n0), 0, (int)(out_bytes - (bz * p.c_bs + n0) * OS), 0x00020000);
    auto row_offset = [&](int r) __attribute__((always_inline)) -> unsigned {
        const int m = first + r;
        const int row = (int)fastdiv((unsigned)m, p.blk_tw_magic, p.blk_tw_shift);
        const int img = (int)fastdiv((unsigned)row, p.blk_p_magic, p.blk_p_shift);
        const int q = q_first + (m - row * tw);
        const int oh = (row - img * p.P) * step_h + ph, ow = q * step_w + pw;
        return m <= last && q < p.Q && oh < out_p && ow < out_q ? (unsigned)((img * out_p + oh) * out_q + ow) * (unsigned)(p.c_rs * OS) : kOutOfRange;
    };
    store_rows<C>(p, rc, ncols, wm, wn, lane, acc, bias_r, row_offset);
}

}  // namespace tir
