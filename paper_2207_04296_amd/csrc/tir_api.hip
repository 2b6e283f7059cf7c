// C-ABI entry points: argument validation, choice of kernel variant, launch.
// Everything a caller can get wrong is caught here, before any HIP call, so that a bad call
// never reaches a kernel.  See include/tir.h for the contract.
#include <hip/hip_runtime.h>
#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include <atomic>
#include <map>
#include <mutex>
#include <tuple>
#include <utility>
#include <vector>

#include "tir.h"
#include "tir_launch.h"
#include "tir_attention.h"
#include "tir_depthwise.h"

namespace tir {

// ------------------------------------------------------------------------------- MFMA rate probe
// Register-only MFMA loop: 4 waves per workgroup, 16 independent 32x32 accumulators per wave, no
// memory traffic inside the loop.  What it sustains is the practical ceiling of the matrix pipes at
// the clock the power management allows for the given operand statistics.
typedef _Float16 probe_f16x8 __attribute__((ext_vector_type(8)));
typedef float probe_f32x16 __attribute__((ext_vector_type(16)));

__global__ void __launch_bounds__(256) mfma_probe_kernel(float* sink, int iters, int random_operands) {
    probe_f32x16 acc[16];
    for (int i = 0; i < 16; ++i)
        for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;
    probe_f16x8 a, b;
    unsigned x = threadIdx.x * 2654435761u + blockIdx.x * 40503u + 12345u;
    for (int e = 0; e < 8; ++e) {
        x ^= x >> 15; x *= 2246822519u; x ^= x >> 13;
        a[e] = (_Float16)(random_operands ? ((x & 0xffff) / 32768.0f - 1.0f) : 1.0f);
        x *= 3266489917u; x ^= x >> 16;
        b[e] = (_Float16)(random_operands ? ((x & 0xffff) / 32768.0f - 1.0f) : 0.5f);
    }
    // Shader-clock counter and 100 MHz wall counter before and after the loop, as one wave in the middle of the grid sees
    // them (raw low words, stored right away so that nothing stays live across the loop): cycles / time is the clock the
    // power management held during the loop.
    const bool reporter = blockIdx.x == gridDim.x / 2 && threadIdx.x == 0;
    unsigned* const stamps = (unsigned*)sink;
    if (reporter) {
        stamps[1] = (unsigned)__builtin_amdgcn_s_memtime();
        stamps[2] = (unsigned)__builtin_amdgcn_s_memrealtime();
    }
    for (int it = 0; it < iters; ++it) {
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, acc[i], 0, 0, 0);
    }
    float s = 0.f;
    for (int i = 0; i < 16; ++i)
        for (int r = 0; r < 16; ++r) s += acc[i][r];
    if (s == 123.456f) sink[0] = s;      // keeps the loop alive, practically never stores
    if (reporter) {
        stamps[3] = (unsigned)__builtin_amdgcn_s_memtime();
        stamps[4] = (unsigned)__builtin_amdgcn_s_memrealtime();
    }
}

// ------------------------------------------------------------------------------- variant table
template <int E> constexpr int tile_extent() {
    static_assert(E >= 32 && E <= 256 && E % 32 == 0, "tile extents are multiples of 32 up to 256");
    return E;
}
#define TIR_ROW(name, DT, OUT, BM, BN, WM, WN, AM, BMO, RB, NS, KW, CW) \
    {name, DT, OUT, tile_extent<BM>(), tile_extent<BN>(), WM, WN, AM, BMO, RB, NS, KW, CW, &launch_cfg<Cfg<DT, OUT, BM, BN, WM, WN, AM, BMO, RB, NS, KW, CW>>},
#define V0 TIR_ROW
#define V1 TIR_ROW
#define V2 TIR_ROW
#define V3 TIR_ROW
#define V4 TIR_ROW
#define V5 TIR_ROW
static const Variant kVariants[] = {
#include "tir_variants.def"
};
static const int kNumVariants = (int)(sizeof(kVariants) / sizeof(kVariants[0]));

// The variants of one (dt, out, amode, bmode), in table order: a call scores its candidates, not the whole table.  What pick() needs of a
// variant and does not depend on the call is worked out once.
struct Candidate {
    const Variant* v;
    int shape;              // number of its tile shape, below kShapes
    int row_shift;          // log2 of rowb
    double bytes_factor;    // grows with bm * bn / (bm + bn), up to the 256x256 tile
};
struct VariantRange {
    const Candidate* first;
    int n;
};
// Tile shapes by number (tile_extent() above sees to their range).
static const int kShapes = 64;
static constexpr int shape_of(int bm, int bn) { return (bm / 32 - 1) * 8 + (bn / 32 - 1); }
static const int kModes = 13, kDtypes = 5;
static VariantRange variants_of(int dt, int out, int amode, int bmode) {
    struct Index {
        Candidate order[kNumVariants];
        VariantRange range[kDtypes][kDtypes][kModes][kModes] = {};
        Index() {
            int n = 0;
            auto candidate = [](const Variant& v) {
                double intensity = (double)v.bm * v.bn / (double)(v.bm + v.bn) / 128.0;
                if (intensity > 1.0) intensity = 1.0;
                // (the few-channel kernel's two widths by constants of their own: 25x133x120x1 -> 80, 5x5 fp16 33.9 us in 32 columns, 37.6 in 64)
                return Candidate{&v, shape_of(v.bm, v.bn), __builtin_ctz((unsigned)v.rowb), v.amode == A_CONV_ROWS ? 0.25 + 0.75 * intensity : 0.2 + 0.8 * intensity};
            };
            for (int d = 0; d < kDtypes; ++d)
                for (int o = 0; o < kDtypes; ++o)
                    for (int a = 0; a < kModes; ++a)
                        for (int b = 0; b < kModes; ++b) {
                            VariantRange& r = range[d][o][a][b];
                            r.first = order + n;
                            for (const Variant& v : kVariants)
                                if (v.dt == d && v.out == o && v.amode == a && v.bmode == b) order[n++] = candidate(v);
                            r.n = (int)(order + n - r.first);
                        }
        }
    };
    static const Index index;
    return index.range[dt][out][amode][bmode];
}

// The depth-wise kernel is not a tile variant: one entry per dtype pair, filled on first use.
static const Variant* depthwise_variant(int dt, int out) {
    static Variant table[6] = {
        {"f16_f16_depthwise", DT_F16, DT_F16, 0, 0, 0, 0, A_DEPTHWISE, B_GENERIC, 0, 0, 1, 0, nullptr},
        {"f16_f32_depthwise", DT_F16, DT_F32, 0, 0, 0, 0, A_DEPTHWISE, B_GENERIC, 0, 0, 1, 0, nullptr},
        {"bf16_bf16_depthwise", DT_BF16, DT_BF16, 0, 0, 0, 0, A_DEPTHWISE, B_GENERIC, 0, 0, 1, 0, nullptr},
        {"bf16_f32_depthwise", DT_BF16, DT_F32, 0, 0, 0, 0, A_DEPTHWISE, B_GENERIC, 0, 0, 1, 0, nullptr},
        {"i8_i32_depthwise", DT_I8, DT_I32, 0, 0, 0, 0, A_DEPTHWISE, B_GENERIC, 0, 0, 1, 0, nullptr},
        {"i8_i8_depthwise", DT_I8, DT_I8, 0, 0, 0, 0, A_DEPTHWISE, B_GENERIC, 0, 0, 1, 0, nullptr},
    };
    for (Variant& v : table)
        if (v.dt == dt && v.out == out) {
            if (!v.fn) v.fn = depthwise_launcher(dt, out);      // idempotent: racing threads store the same pointer
            return v.fn ? &v : nullptr;
        }
    return nullptr;
}

static thread_local char g_err[512] = "";
static int g_force_bm = 0, g_force_bn = 0, g_force_ksplit = 0;
static char g_force_name[64] = "";

static tir_status fail(tir_status st, const char* fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof g_err, fmt, ap);
    va_end(ap);
    return st;
}

static const int64_t kMaxExtent = 2147483647LL;
static const double kCUs = 256.0;

static bool dtype_pair_ok(int in, int out, bool fused) {
    return (in == TIR_F16 && (out == TIR_F32 || out == TIR_F16)) ||
           (in == TIR_BF16 && (out == TIR_F32 || out == TIR_BF16)) || (in == TIR_I8 && out == TIR_I32) ||
           (fused && in == TIR_I8 && out == TIR_I8);
}

// The epilogue variant queries assume for int8 output.
static const tir_epilogue kQueryRequant = {nullptr, 0, 1.0f};

static bool aligned(const void* p, uintptr_t a) { return ((uintptr_t)p % a) == 0; }

// Do byte offsets inside one tile of at most 256 rows of `stride` elements (the last one `width` elements wide) fit
// 31 bits?  (stride * 256 + width) * es < 2^31 - 1, written so that no product can overflow for strides up to 2^63.
static bool fits_tile_offsets(int64_t stride, int64_t width, int64_t es) {
    const int64_t room = kMaxExtent / es - width;
    return room > 0 && stride < (room + 255) / 256 && (stride * 256 + width) * es < kMaxExtent;
}

// ------------------------------------------------------------------------------- measured choices
// Records of tir_tune_*: for a problem signature, the variant that ran fastest on this device.
// kind 0 = (batched) GEMM, 1 = convolution; geom packs the convolution geometry that the GEMM view
// (batch, M, N, K) does not show.  A record only ever names a variant that computes the same result.
struct TuneKey {
    int kind, dt, out, amode, bmode;
    int64_t batch, M, N, K;
    uint64_t geom;
    bool operator<(const TuneKey& o) const {
        return std::tie(kind, dt, out, amode, bmode, batch, M, N, K, geom) <
               std::tie(o.kind, o.dt, o.out, o.amode, o.bmode, o.batch, o.M, o.N, o.K, o.geom);
    }
};
// A kernel variant plus the number of workgroups that share one tile's reduction (1 = no split).
struct Choice {
    const Variant* v;
    int ksplit;
};
static const Choice kNoChoice = {nullptr, 1};
static std::mutex g_tune_mu;
static std::map<TuneKey, Choice> g_tuned;
static std::atomic<bool> g_any_tuned{false};      // g_tuned may hold records: without one, calls do not look
// set by the tuner around its trial launches on the calling thread: the choice to plan with
static thread_local Choice g_trial = {nullptr, 1};

static Choice tuned_lookup(const TuneKey& k) {
    if (!g_any_tuned.load(std::memory_order_acquire)) return kNoChoice;
    std::lock_guard<std::mutex> lock(g_tune_mu);
    auto it = g_tuned.find(k);
    return it == g_tuned.end() ? kNoChoice : it->second;
}

// ------------------------------------------------------------------------------- split reduction
// Scratch of the reduction split over workgroups: the slices' partial sums and one arrival counter per output
// tile.  The library owns no such memory: a caller registers a buffer per (device, stream) with tir_set_workspace
// (launches on one stream follow each other, so they can share it; launches on different streams may overlap and
// need their own), or calls tir_gemm_split_static, whose scratch is a static device array.
static const int64_t kWsBytes = 32ll << 20;      // partial sums of a registered workspace
static const int64_t kWsTiles = 16384;           // ... and its counters
struct Workspace {
    void* partial;
    unsigned* count;
};
static std::mutex g_ws_mu;
static std::map<std::pair<int, hipStream_t>, Workspace> g_ws;
static std::atomic<bool> g_any_ws{false};         // likewise for g_ws

// What a plan may use for split reductions: room for partial sums and counters (bytes = 0: none, never split),
// and the slice count a caller insists on (force > 1: only variants that can split that way are considered,
// measured records and the scoring rule's own idea of a split are ignored).
struct SplitLimits {
    int64_t bytes, tiles;
    int force;
};
static const SplitLimits kNoSplit = {0, 0, 0};
static const SplitLimits kRegisteredSplit = {kWsBytes, kWsTiles, 0};      // a registered workspace (also what the variant queries assume)

// Arrival counters start at zero; every launch leaves them at zero again (the last workgroup of a tile resets its counter).
__global__ void __launch_bounds__(256) clear_counters_kernel(unsigned* count, int n) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) count[i] = 0;
}

// Can variant v reduce a problem of `tiles` output tiles per batch entry in ks slices?
static bool split_fits(const Variant* v, int ks, int64_t batch, int64_t tiles, int64_t K, const SplitLimits& sl) {
    if (ks == 1) return true;
    if (ks < 1 || ks > 64 || sl.bytes <= 0) return false;
    if (v->amode != A_KMAJOR && v->amode != A_MMAJOR && v->amode != A_CONV && v->amode != A_CONVX) return false;      // the fast kernel only
    if (v->bm * v->bn > kSplitMaxTile) return false;
    const int64_t stages = (K * elem_size(v->dt) + v->rowb - 1) / v->rowb;
    const int64_t per = (stages + ks - 1) / ks;
    if ((ks - 1) * per >= stages) return false;       // a slice would be empty
    if (batch > 65535 || batch * tiles > sl.tiles) return false;
    return batch * tiles * ks * v->bm * v->bn * 4 <= sl.bytes;
}

// The split a launch on `stream` of the current device may use: that of its registered workspace, or none.
static SplitLimits stream_split_limits(hipStream_t stream) {
    if (!g_any_ws.load(std::memory_order_acquire)) return kNoSplit;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) {
        (void)hipGetLastError();
        return kNoSplit;
    }
    std::lock_guard<std::mutex> lock(g_ws_mu);
    return g_ws.count(std::make_pair(dev, stream)) ? kRegisteredSplit : kNoSplit;
}

// The kernels divide by these launch constants through multiply-and-shift (see Params); a GEMM divides by one of them.
static void set_divisors(Params& p, bool conv) {
    auto put = [](unsigned d, unsigned* magic, int* shift) {
        const FastDiv f = make_fastdiv(d < 1 ? 1u : d);
        *magic = f.magic;
        *shift = f.shift;
    };
    put((unsigned)(kGroupM * p.tiles_n), &p.div_gw_magic, &p.div_gw_shift);
    if (!conv) return;
    put((unsigned)p.tiles_n, &p.div_tn_magic, &p.div_tn_shift);
    put((unsigned)p.tiles_m, &p.div_tm_magic, &p.div_tm_shift);
    put((unsigned)(p.PW / 8), &p.div_pw_magic, &p.div_pw_shift);      // copy units (8 pixels) per patch row
    put((unsigned)p.Q, &p.div_q_magic, &p.div_q_shift);
    put((unsigned)(p.P * p.Q), &p.div_pq_magic, &p.div_pq_shift);
    put((unsigned)(p.OD < 1 ? 1 : p.OD) * (unsigned)(p.P * p.Q), &p.div_opq_magic, &p.div_opq_shift);
    put((unsigned)p.Cg, &p.div_cg_magic, &p.div_cg_shift);
    put((unsigned)p.S, &p.div_s_magic, &p.div_s_shift);
    put((unsigned)(p.R * p.S), &p.div_rs_magic, &p.div_rs_shift);
    put((unsigned)p.conv_groups, &p.div_grp_magic, &p.div_grp_shift);
    put((unsigned)p.phases_h, &p.div_phh_magic, &p.div_phh_shift);
    put((unsigned)p.phases_w, &p.div_phw_magic, &p.div_phw_shift);
    const unsigned qg = (unsigned)((p.Q + kDwBlockPix - 1) / kDwBlockPix);
    put(qg, &p.div_dwq_magic, &p.div_dwq_shift);
    put((unsigned)p.P * qg, &p.div_dwpq_magic, &p.div_dwpq_shift);
}

static uint64_t hash_fields(const int64_t* f, int n) {
    // the fields of a convolution's geometry do not fit 64 bits side by side: mix them instead (FNV-1a)
    uint64_t h = 1469598103934665603ull;
    for (int i = 0; i < n; ++i)
        for (int b = 0; b < 8; ++b) { h ^= (uint64_t)((f[i] >> (8 * b)) & 0xff); h *= 1099511628211ull; }
    return h;
}

// Pick a variant for (dt, out, amode, bmode).  This is the hand-made stand-in for the paper's
// search over tilings (sec. 4.4): every listed tile is scored by
//   padding efficiency  x  how evenly its workgroups fill the 256 CUs  x  bytes-per-flop factor,
// where the last term favours tiles that need fewer global->LDS bytes per MFMA (bm*bn/(bm+bn),
// saturating at the 256x256 tile), times a term for how the copies of such a workgroup are hidden (`depth` below: waves, ring, rounds).
//
// The constants are fitted to the time of every variant on 491 calls of more than 0.12 GFLOP (GEMM, batched, convolutions, transposed ones by phase;
// the extents of image and language networks, a quarter of the GEMMs odd), and corrected for calls that the fit had moved to slower ones: over 3853 drawn calls of
// any size a pick takes 1.014 of the fastest variant's time in the geometric mean.  Each constant's comment gives calls that it moves, in us with the choice before and now.
//
// A reduction much longer than the tile grid is wide (few small tiles, many stages) is split over several
// workgroups per tile, as many as fill the CUs once while each keeps at least eight stages.
static Choice pick(int dt, int out, int amode, int bmode, int64_t batch, int64_t M, int64_t N, int64_t K, const SplitLimits& sl, int max_rowb = 256) {
    Choice best = kNoChoice;
    double best_score = -1.0;
    const int es = elem_size(dt);
    const bool staged = amode == A_UK || amode == A_UM;
    const VariantRange candidates = variants_of(dt, out, amode, bmode);
    const bool overrides = sl.force > 1 || g_force_ksplit || g_force_name[0] || g_force_bm;
    struct Shape {
        int64_t tiles;
        double eff, fit;      // padding efficiency, alone and times fill
    } shapes[kShapes];
    uint64_t have = 0;        // shapes that are filled in
    // Beyond one round fill is not counted by whole rounds: a CU holds several workgroups of most tiles, so that a last round is seldom waited for by itself.
    // (Whole rounds move 40 of 3853 calls to variants 3 to 34 % slower, 51 to faster ones.)
    auto fill = [](double tiles) { return tiles <= kCUs ? tiles / kCUs : tiles / (tiles + (kCUs - 1.0)); };
    for (int i = 0; i < candidates.n; ++i) {
        const Candidate& c = candidates.first[i];
        const Variant* v = c.v;
        if (v->rowb > max_rowb) continue;
        Shape& shape = shapes[c.shape];
        if (!(have >> c.shape & 1)) {
            have |= 1ull << c.shape;
            // (extents are below 2^31: 32-bit divisions, which take a third of the time of 64-bit ones)
            const unsigned tm = ((unsigned)M + (unsigned)v->bm - 1u) / (unsigned)v->bm, tn = ((unsigned)N + (unsigned)v->bn - 1u) / (unsigned)v->bn;
            shape.tiles = (int64_t)tm * tn;
            shape.eff = ((double)M * (double)N) / ((double)tm * v->bm * (double)tn * v->bn);
            shape.fit = shape.eff * fill((double)tm * (double)tn * (double)batch);
        }
        int ks = 1;
        if (overrides) {
            const int want_ks = sl.force > 1 ? sl.force : g_force_ksplit;
            if (want_ks > 1 && split_fits(v, want_ks, batch, shape.tiles, K, sl)) ks = want_ks;
            if (sl.force > 1 && ks != sl.force) continue;          // the caller insists on this split
            if (g_force_name[0] && strstr(v->name, g_force_name)) return Choice{v, ks};          // testing / tuning overrides
            if (g_force_bm && v->bm == g_force_bm && v->bn == g_force_bn && v->kw == 1 && v->cw == 0) return Choice{v, ks};
        }
        const int64_t nslab = (K * es + v->rowb - 1) >> c.row_shift;       // stages (of 64, 128 or 256 bytes)
        const bool small = v->bm * v->bn <= 64 * 64;
        // (the partial sums' trip through memory costs about 4 us for a 64x64 tile and grows with the tile: it pays
        // only for small tiles whose wave groups face two dozen stages or more)
        if (small && sl.bytes > 0 && !(sl.force > 1 || g_force_ksplit) && nslab >= 24 * v->kw && shape.tiles * batch <= (int64_t)kCUs / 2) {
            int64_t want = (int64_t)kCUs / (shape.tiles * batch);
            if (want > nslab / (8 * v->kw)) want = nslab / (8 * v->kw);
            if (want > 8) want = 8;
            while (want > 1 && !split_fits(v, (int)want, batch, shape.tiles, K, sl)) --want;
            if (want > 1) ks = (int)want;
        }
        const double eff = shape.eff, tiles = (double)shape.tiles * (double)batch * ks;
        double score = (ks == 1 ? shape.fit : eff * fill(tiles)) * c.bytes_factor;
        const bool one_round = tiles <= kCUs;
        // `depth` is at most 1.3, 1.7 for small tiles in several rounds: most candidates end here.  With the
        // shared terms of a tile shape a query of 128x128x128 fp16, 37 candidates, takes 1.13 us through the binding instead of 1.20 (an eager call 3.89 instead of 3.99)
        if (score * (small && !one_round ? 1.7 : 1.3) <= best_score) continue;
        const int lds = (v->bm + v->bn) * v->rowb * v->nstage * v->kw;
        double depth = 1.0;
        if (v->kw > 1) {
            // Reduction groups pay for the exchange of partial sums.  Small tiles: in a single round of workgroups (nothing else on the CU hides the
            // copy latency), from two stages per group on (3x3 over 32 channels, 245 tiles of 64x32 5.3 -> 4.8).  Operands staged through
            // registers have less in flight (500x501x503 fp16: 6.9, 5.6 with four groups).
            // Convolutions: larger tiles as well, because the waves share the arithmetic of the copies' addresses, and a long reduction pays for it in any number of
            // rounds (18x88x13, 176 -> 192 channels, 5x5 stride 2 bf16 38.9 -> 24.0; 17x36x39, 864 -> 64 in two groups fp16 73 -> 43.5).
            // By phase, 16x14x14, 256 -> 128 4x4 stride 2 fp16 in 128x64 tiles: one group 12.8, two 12.1, one and copy waves 12.2.
            // 128x32 tiles from three stages per group on: of 45 calls the 33 with fewer take 1 to 5 % more in two groups (transposed 19x43x9, 64 -> 32 channels 4x4
            // stride 2 bf16 5.56 and 5.74), those with more 0.71 to 1.10 of the time.
            if (one_round ? nslab < (small ? (v->bm == 128 ? 3 : 2) * v->kw : 16) || (!small && amode != A_CONV) : amode != A_CONV || nslab < 40 || v->bm < 128) continue;
            depth += !one_round ? 0.08 : !small ? 0.05 : amode == A_CONV ? 0.02 : 0.01;
        }
        // Operands staged through registers, 128x128 tiles: eight waves instead of four hide each other's loads and LDS writes over a long reduction (1500x1501x2001
        // fp16 34.4 -> 27.8, 2999x1001x1999 A^T B^T 36.8 -> 28.7, 3001x2005x777 24.5 -> 22.6); a short one is faster with the fragments four waves reuse
        // (2049x3333x333 bf16 17.2 and 18.8, 4001x4001x501 int8 24.9 and 29.3).
        if (staged && v->bm == 128 && v->bn == 128) depth += (v->wm * v->wn == 8) == (nslab >= 10) ? 0.02 : -0.02;
        // 96-row tiles for one round of workgroups only: their ring leaves room for one workgroup per CU, and what they save in padding short
        // reductions of many rounds do not gain (237 x 272x384x96 fp16 41.9 in 128x128 tiles, 45.7 in these; 160 x 288x768x128 int8 47.4 and 52.3)
        if (v->bm == 96 && !one_round) continue;
        // (nor do the 128x96 ones pay for short convolutions of many rounds: 12x36x42, 16 -> 288 channels in each of 8 groups, 3x3 stride 2 16.3 and 17.8; longer
        // ones are faster in 256x96: 16x106x90, 128 -> 288, 3x3 stride 2 bf16 34.8 and 45.3, 48 -> 96 channels in each of 8 groups, 5x5 int8 29.4 and 35.8)
        if (v->bm == 128 && v->bn == 96 && amode == A_CONV && !one_round) {
            if (nslab < 8) continue;
            depth -= 0.1;
        }
        // GEMMs of one stage do not repay their four stages of copies (30 x 48x608x96 int8 3.95 in 64x32, 4.59; 25 x 704x96x64 int8 4.20 in 256x32, 4.56), those of two
        // not half a tile of padding (37 x 48x560x128 fp16 4.38 in 64x32, 4.83; less padding pays: 63 x 64x272x96 bf16 5.66 and 4.57)
        // (nor does 128x192 for half a tile: 49 x 64x928x64 5.5 in 64x64, 6.5; 51 x 32x848x64 4.8 and 5.3; 49 x 48x848x128 6.2 and 6.9)
        if (amode != A_CONV && (v->bm == 96 ? nslab == 1 || (nslab == 2 && eff < 0.5) : v->bn == 192 && nslab <= 2 && eff < 0.5)) score *= 0.85;
        // One stage and many rounds: half as many, twice as large stores (84 x 608x656x64 bf16 37.2 in 256x256, 43.4 in 64x64; 8x47x112, 32 -> 160 1x1 8.7 and 9.3)
        if (v->bm == 256 && v->bn >= 128 && nslab == 1 && !one_round) depth += 0.03;
        // Copy waves take the copies' issue off the multiplying ones.  Tiles of 128x128 and more behind four waves gain from four stages on (1664x1888x256 bf16
        // 6.6 -> 6.0), behind eight from eight; 64x64 and more from three and four (43x37, 64 -> 304 channels 5x5 15.2 -> 12.1; 3776x512x896 fp16 8.1 -> 7.1; long
        // GEMMs do not: 3952x448x1728 fp16 11.6 without, 12.4 with, in 128x64 tiles and 16 bits from 14 stages on 1120x1376x864 9.2 and 9.6), the small ones, and those
        // with 256-byte stages, in one round only.  128x64 tiles of int8 convolutions in many rounds are faster without (11x70x43, 32 -> 48 channels in each of 8 groups,
        // 5x5 39.0 and 44.8): a stage holds more taps than in 16 bits, and the copy waves alone decode them.
        if (v->cw) {
            const int area = v->bm * v->bn;
            const bool big = area >= 128 * 128, eight = v->wm * v->wn == 8;
            const int64_t from = v->rowb == 256 ? 3 : big ? (eight ? 8 : 4) : small ? 4 : 3;
            const bool pays = nslab >= from && (one_round || !(small || v->rowb == 256));
            depth += !pays ? -0.04 : v->rowb == 256 ? 0.07 : small ? 0.06 : big ? (eight || !one_round ? 0.04 : 0.1)
                     : amode != A_CONV && v->bm != 96 && nslab > (v->bn == 64 && dt != DT_I8 ? 13 : 20) ? 0.0 : 0.05;
        } else if (v->rowb == 256) depth -= 0.04;
        else if (dt == DT_I8 && amode == A_CONV && !one_round && v->bm == 128 && v->bn == 64 && v->nstage == 3 && v->kw == 1 && nslab >= 5) depth += 0.06;
        if (!one_round) {
            // 64x32 tiles have two waves; many rounds of them are slower than of wider tiles (38110 pixels, 48 channels -> 48, 3x3, 1192 tiles 12.4 -> 8.6; but
            // 15x17x18, 16 -> 16 channels in 8 groups, 3x3, 576 tiles 4.7, and 5.3 in 256x32 tiles).  Three per CU of a convolution run at once, which the fill does
            // not see (5236 pixels, 112 -> 16 channels in each of 8 groups, 5x5, 656 tiles 29.0, and 33.1 in 256x32; 37840 pixels, 80 -> 32 1x1, 592 tiles 4.9 and 5.4).
            if (v->bm == 64 && v->bn == 32 && tiles > 4 * kCUs) depth -= 0.12;
            if (v->bm == 64 && v->bn == 32 && amode == A_CONV && v->kw == 1 && tiles > 2 * kCUs && tiles <= 3 * kCUs) depth += 0.12;
            // Many rounds of one stage or two: nothing but latency and stores, which five 64x64 workgroups per CU cover for each other (209 x 320x80x64 fp16
            // 10.1 -> 7.9, 244 x 118x285x32 bf16 13.5 -> 11.2, 58x81 1x1 16 -> 128 channels 13.9 -> 10.9)
            const int64_t kbytes = K * es;
            if (tiles > 5 * kCUs && small && v->bn == 64 && v->nstage == 2 && v->kw == 1 && !staged) depth += kbytes <= 128 ? 0.4 : kbytes <= 256 ? 0.05 : 0.0;
        }
        // Ring depth: stages beyond the number of K-slabs are useless; with more than one
        // workgroup per CU prefer rings that let two of them be resident (LDS <= 80 KB)
        if (nslab < v->nstage) depth -= 0.04 * (v->nstage - (int)nslab);
        if (!one_round && lds > 80 * 1024) depth -= 0.04;
        else depth += (one_round ? 0.015 : 0.0025) * v->nstage;
        // the partial sums' round trip (25x14x43, 96 -> 32 channels 5x5 fp16 in two slices 13.6, in two groups of one workgroup 11.0); a reduction of 8 KB and
        // more per row covers its fixed part (464 -> 160 channels 5x5 over 3078 pixels 34.8 in two slices, 44.8 in one; 192 -> 16, 11700 pixels 18.1 and 20.4)
        score *= depth * (ks > 1 ? (K * es >= 8192 ? 1.0 : 0.95) - 0.03 * (ks - 1) : 1.0);
        if (score > best_score) { best_score = score; best = Choice{v, ks}; }
    }
    return best;
}

// by phase, a stage must hold channels of one tap
static bool tuned_or_trial_mismatch(const Variant* v, int64_t group_channel_bytes) {
    return v->amode == A_CONV && group_channel_bytes % v->rowb != 0 && !g_trial.v;
}

struct Plan {
    const Variant* v;
    Params p;
    TuneKey key;        // signature of the problem for the measured-choice records
    bool patch_ok;      // convolution: the LDS-resident-patch kernel may run this problem
};

// The variant a plan uses: the tuner's trial variant, else a measured record, else the scoring rule.
static Choice choose(const TuneKey& key, int64_t batch, int64_t M, int64_t N, int64_t K, const SplitLimits& sl) {
    if (sl.force > 1) return pick(key.dt, key.out, key.amode, key.bmode, batch, M, N, K, sl);
    if (g_trial.v) return g_trial;
    if (!g_force_name[0] && !g_force_bm && !g_force_ksplit) {
        const Choice t = tuned_lookup(key);
        if (t.v) return t;
    }
    return pick(key.dt, key.out, key.amode, key.bmode, batch, M, N, K, sl);
}

static tir_status check_common(const void* A, const void* B, const void* C, int in, int out, const tir_epilogue* ep) {
    if (in < 0 || in > TIR_I32 || out < 0 || out > TIR_I32) return fail(TIR_ERR_INVALID_ARG, "unknown dtype code (in=%d out=%d)", in, out);
    if (!dtype_pair_ok(in, out, ep != nullptr)) return fail(TIR_ERR_UNSUPPORTED, "unsupported (in, out) dtype pair (%d, %d)", in, out);
    if (ep) {
        if (ep->streaming != 0 && ep->streaming != 1) return fail(TIR_ERR_INVALID_ARG, "epilogue: streaming must be 0 or 1 (got %d)", ep->streaming);
        if (!aligned(ep->bias, 4)) return fail(TIR_ERR_ALIGNMENT, "bias pointer not aligned to 4 bytes");
        if (out == TIR_I8 && !(ep->scale > 0.0f && ep->scale <= 3.402823466e38f))
            return fail(TIR_ERR_INVALID_ARG, "int8 output needs a finite scale > 0");
    }
    const int es = elem_size(in), os = elem_size(out);
    if (!aligned(A, es) || !aligned(B, es)) return fail(TIR_ERR_ALIGNMENT, "input pointer not aligned to its element size");
    if (!aligned(C, os)) return fail(TIR_ERR_ALIGNMENT, "output pointer not aligned to its element size");
    return TIR_OK;
}

// Build the launch plan of a (batched) GEMM.  Pointers may be null only for planning (variant query).
static tir_status plan_gemm(bool need_ptrs, const void* A, const void* B, void* C, int64_t batch, int64_t M, int64_t N,
                            int64_t K, int64_t a_bs, int64_t a_rs, int64_t a_cs, int64_t b_bs, int64_t b_rs,
                            int64_t b_cs, int64_t c_bs, int64_t c_rs, int64_t c_cs, int in, int out, const tir_epilogue* ep,
                            const SplitLimits& sl, Plan* plan) {
    plan->v = nullptr;
    plan->key.kind = -1;        // no signature yet
    tir_status st = check_common(A, B, C, in, out, ep);
    if (st != TIR_OK) return st;
    if (batch < 0 || M < 0 || N < 0 || K < 0) return fail(TIR_ERR_INVALID_ARG, "negative extent (batch=%lld M=%lld N=%lld K=%lld)", (long long)batch, (long long)M, (long long)N, (long long)K);
    if (a_bs < 0 || a_rs < 0 || a_cs < 0 || b_bs < 0 || b_rs < 0 || b_cs < 0 || c_bs < 0 || c_rs < 0 || c_cs < 0)
        return fail(TIR_ERR_INVALID_ARG, "negative stride");
    if (M > kMaxExtent || N > kMaxExtent || K > kMaxExtent || batch > kMaxExtent)
        return fail(TIR_ERR_UNSUPPORTED, "extent beyond 2^31-1");
    if (batch == 0 || M == 0 || N == 0) return TIR_OK;  // nothing to do, plan->v stays null
    if (need_ptrs) {
        if (!C) return fail(TIR_ERR_INVALID_ARG, "C is null");
        if (K > 0 && (!A || !B)) return fail(TIR_ERR_INVALID_ARG, "A or B is null");
    }
    if (M > 1 && N > 1 && c_rs == 0 && c_cs == 0) return fail(TIR_ERR_INVALID_ARG, "C strides are both zero");
    if (batch > 1 && c_bs == 0) return fail(TIR_ERR_INVALID_ARG, "c_bs is zero: the C matrices of different batches overlap");

    const int es = elem_size(in);
    const int vec = 16 / es;
    const bool k_vec = K % vec == 0;
    int amode = A_GENERIC, bmode = B_GENERIC;
    // fast copy modes need 16-byte vectors along the contiguous axis
    // (rows must not overlap: the copy stage relies on "row r+1 starts after row r ends" to turn
    // rows past the edge into out-of-range reads; byte offsets inside one tile must fit 31 bits)
    if (a_cs == 1 && k_vec && a_rs % vec == 0 && a_bs % vec == 0 && aligned(A, 16) && (a_rs >= K || M == 1) &&
        fits_tile_offsets(a_rs, K, es)) amode = A_KMAJOR;
    else if (a_rs == 1 && M % vec == 0 && a_cs % vec == 0 && a_bs % vec == 0 && aligned(A, 16) && a_cs >= M &&
             fits_tile_offsets(a_cs, M, es)) amode = A_MMAJOR;
    if (b_rs == 1 && k_vec && b_cs % vec == 0 && b_bs % vec == 0 && aligned(B, 16) && (b_cs >= K || N == 1) &&
        fits_tile_offsets(b_cs, K, es)) bmode = B_KMAJOR;
    else if (b_cs == 1 && N % vec == 0 && b_rs % vec == 0 && b_bs % vec == 0 && aligned(B, 16) && b_rs >= N &&
             fits_tile_offsets(b_rs, N, es)) bmode = B_NMAJOR;
    if (amode == A_GENERIC || bmode == B_GENERIC) {
        // Unaligned rows: both operands through registers, each along its contiguous axis (k where both are), which must hold
        // one vector.  Anything else - no unit stride, or fewer elements than a vector - is loaded element by element.
        const int ua = a_cs == 1 && K >= vec && fits_tile_offsets(a_rs, K, es) ? A_UK : a_rs == 1 && M >= vec && fits_tile_offsets(a_cs, M, es) ? A_UM : A_GENERIC;
        const int ub = b_rs == 1 && K >= vec && fits_tile_offsets(b_cs, K, es) ? B_UK : b_cs == 1 && N >= vec && fits_tile_offsets(b_rs, N, es) ? B_UN : B_GENERIC;
        amode = ua != A_GENERIC && ub != B_GENERIC ? ua : A_GENERIC;
        bmode = amode != A_GENERIC ? ub : B_GENERIC;
    }

    plan->key = TuneKey{0, in, out, amode, bmode, batch, M, N, K, 0};
    plan->patch_ok = false;
    const Choice ch = choose(plan->key, batch, M, N, K, sl);
    const Variant* v = ch.v;
    if (!v) return fail(TIR_ERR_UNSUPPORTED, "no kernel variant for this dtype / layout / forced tile");
    Params& p = plan->p;
    memset(&p, 0, sizeof p);
    p.ksplit = split_fits(v, ch.ksplit, batch, ((M + v->bm - 1) / v->bm) * ((N + v->bn - 1) / v->bn), K, sl) ? ch.ksplit : 1;
    p.A = A; p.B = B; p.C = C;
    p.M = (int)M; p.N = (int)N; p.K = (int)K;
    p.batch = (int)batch;
    p.tiles_m = (int)((M + v->bm - 1) / v->bm);
    p.tiles_n = (int)((N + v->bn - 1) / v->bn);
    if ((int64_t)p.tiles_m * p.tiles_n > kMaxExtent) return fail(TIR_ERR_UNSUPPORTED, "too many output tiles");
    p.a_bs = a_bs; p.b_bs = b_bs; p.c_bs = c_bs;
    p.a_rs = a_rs; p.a_cs = a_cs; p.b_rs = b_rs; p.b_cs = b_cs; p.c_rs = c_rs; p.c_cs = c_cs;
    p.c_fast = (c_cs == 1 && (c_rs >= N || M == 1) && fits_tile_offsets(c_rs, N, elem_size(out))) ? 1 : 0;
    if (ep) { p.bias = ep->bias; p.bias_bs = 0; p.relu = ep->relu != 0; p.scale = ep->scale; p.store_nt = ep->streaming; }
    set_divisors(p, false);
    plan->v = v;
    return TIR_OK;
}

static int64_t conv_extent(int64_t in, int64_t filt, int64_t stride, int64_t pad, int64_t dil) {
    int64_t span = in + 2 * pad - dil * (filt - 1) - 1;
    return span < 0 ? 0 : span / stride + 1;
}

// Geometry of a convolution in the general form the kernels decode: a depth axis (D = T = 1 for 1-D / 2-D) and the
// transposed 2-D form (the adjoint of a strided convolution).
struct ConvGeom {
    int64_t N, D, H, W, C, K, T, R, S;
    int stride_d, stride_h, stride_w, pad_d, pad_h, pad_w, dil_d, dil_h, dil_w;
    int groups;
    bool transposed;
    int outpad_h, outpad_w;      // transposed only
};

// The channel-block kernel on one of its tiles: strips of output columns, patch, LDS.
struct BlockPlan {
    const Variant* v;
    int tw, pw, vh, patch, lds, strips, strip_tiles;
};
// A stride-1 convolution as the kernel sees it: `batch` independent ones (groups, phases) of images x P x Q pixels, `cols` output channels each,
// taps x taps of them dil_h and dil_w apart, `bytes` of channels per pixel.
struct BlockProblem {
    int64_t images, P, Q, cols, batch, bytes;
    int taps, dil_h, dil_w, out_bytes;
    bool phased;
};

// Expected time of a launch in shader cycles, for the choice between the channel-block kernel, the implicit-GEMM tiles and the patch kernel for
// pixels of 128 bytes, and between the first one's tiles and strips: a number of rounds over the CUs times what a workgroup takes, its loop (the slower of
// copying and multiplying) and its set-up and store.  Fitted to half of 8623 drawn stride-1 convolutions (3x3, 5x5 and 4x4 stride 2 by
// phase), every tile timed in every number of strips with three sets of operands in turn, first to the times and then to the choice that follows.  On the other
// half: times met to 7 % (root mean square; implicit GEMM 8), the choice at 0.85 of the other kernels' time in the geometric mean (the best tile of each call 0.84), and
// 17 of 4312 calls more than 5 % slower than there, 5 more than 10 %; of 4329 drawn afterwards 25 and 5.  Known ones, that time and this kernel's: 28x32x11, 32 -> 256 in each of 4 groups, 5x5
// bf16 to fp32 25.3 us and 32.6, 12x10x13, 144 -> 16 in each of 4 groups, 5x5 11.5 and 13.1, 13x22x42, 64 -> 368 13.1 and 15.1, 30x22x78, 272 -> 144, dilation 2 fp16 to fp32 61.8 and
// 70.9, 2x58x63, 64 -> 480 in each of 8 groups, 5x5 int8 to int32 69.2 and 74, 20x20x26, 16 -> 160 in each of 4 groups fp16 to fp32 9.9 and 11.2, 7x19x80, 64 -> 96 in
// each of 2 groups, dilation 2 6.8 and 7.5, 3x12x36, 496 -> 272, dilation 2 13.7 and 15.2, 1x106x15, 160 -> 16 in each of 4 groups, 5x5 12.1 and 12.9.
static double whole_rounds(double rounds, int n) { return n * (double)(int)((n == 1 ? rounds : rounds / n) + (1.0 - 1e-9)); }      // up to a multiple of n (launches are below 2^31 workgroups)
// What a tile takes whatever the problem's extents, for filters of one size; worked out once.
struct BlockTile {
    const Variant* v;
    int bm_shift, bn_shift, row_shift;      // log2 of bm, bn, rowb
    unsigned ring;                          // LDS of the filter
    bool pair;                              // registers allow two workgroups per CU (block_pair() in tir_conv_blocks.h)
    double slabs, work, store;              // a block's filter copies and products, the set-up and store of a workgroup without its patch
    double decode;                          // (the store of a phase or of more than one strip decodes its rows)
    double own_units;                       // copy instructions of a patch of just the tile's pixels
};
static const int kBlockTaps[] = {2, 3, 5}, kMaxBlockTiles = 8;
static const double kNoLimit = 1e300;
struct BlockTiles {
    BlockTile tile[kMaxBlockTiles];
    int n;
};
static const BlockTiles& block_tiles(int dt, int out, int taps) {
    struct Index {
        BlockTiles of[kDtypes][kDtypes][3] = {};
        Index() {
            for (const Variant& v : kVariants)
                for (int i = 0; i < 3 && v.amode == A_CONV_BLOCKS; ++i) {
                    BlockTiles& list = of[v.dt][v.out][i];
                    const double rs = kBlockTaps[i] * kBlockTaps[i], mfma = (v.bm / 32) * (v.bn / 32) * (v.rowb / 32) * 8.0;       // cycles of a tap's MFMAs on four SIMDs
                    const int area = v.bm * v.bn;
                    if (list.n == kMaxBlockTiles) continue;
                    list.tile[list.n++] = BlockTile{&v, __builtin_ctz(v.bm), __builtin_ctz(v.bn), __builtin_ctz(v.rowb), 3u * kBlockTaps[i] * v.bn * v.rowb,
                                                    area < 128 * 64 || (v.rowb == 64 && area < 256 * 64 && kBlockTaps[i] < 5), 16.5 * rs * v.bn * v.rowb / 1024.0,
                                                    rs * (1.125 * mfma + 60.0), 4590.0 + 10.4 * area * elem_size(v.out) / 1024.0, 3.7 * v.bm, v.bm * v.rowb / 1024.0};
                }
        }
    };
    static const Index index;
    return index.of[dt][out][taps == 2 ? 0 : taps == 3 ? 1 : 2];
}
// decode: 8x28x28, 32 -> 32 in each of 8 groups, dilation 2 int8 takes 4.95 us in one strip, 5.35 in two.
static double blocks_cycles(const BlockTile& t, double ncb, double units, bool decode, bool pair, double rounds) {
    const double copy = 16.5 * units + t.slabs, fixed = t.store + 10.2 * units + (decode ? t.decode : 0.0);
    const double loop = ncb * ((copy > t.work ? copy : t.work) + 590.0);
    if (rounds <= 1.0) return 2010.0 + loop + fixed;
    // A last round that is partly filled takes most of a whole one's time, which matters against 256x256 and 256x128 tiles of one round: 6x33x45, 192 -> 128
    // transposed fp16 in 560 workgroups, two per CU, 17.9 us and 14.1.  Two on a CU cover each other's set-up and store.
    if (pair) return 2010.0 + (loop + 0.36 * fixed) * 0.5 * (whole_rounds(rounds, 2) + rounds) + 0.5 * fixed;
    return 2010.0 + (loop + fixed) * (0.85 * whole_rounds(rounds, 1) + 0.15 * (rounds + 0.5));
}
static double gather_cycles(const Variant* v, const BlockProblem& b, int ksplit) {
    const bool ragged = v->amode == A_CONV_RAGGED;
    const unsigned taps = (unsigned)(b.taps * b.taps), bytes = (unsigned)b.bytes, rowb = (unsigned)v->rowb;
    const unsigned stages = b.phased ? taps * ((bytes + rowb - 1u) / rowb) : (taps * bytes + rowb - 1u) / rowb;        // by phase a stage holds channels of one tap
    const unsigned tiles_m = ((unsigned)(b.images * b.P * b.Q) + (unsigned)v->bm - 1u) / (unsigned)v->bm, tiles_n = ((unsigned)b.cols + (unsigned)v->bn - 1u) / (unsigned)v->bn;
    const double rounds = (double)tiles_m * (double)tiles_n * (double)(b.batch * ksplit) * (1.0 / kCUs), area = v->bm * v->bn, busy = rounds < 1.0 ? rounds : 1.0;
    // Pixels that straddle 128-byte lines cost large tiles a fifth more copy time (11x38x24, 416 -> 240 in 128x96 tiles 30.2 us, 16 us of MFMAs).
    const bool straddle = !b.phased && b.bytes > 128 && b.bytes % 128 != 0 && v->rowb == 128 && v->kw == 1 && area >= 128 * 64;
    const double copy = (straddle ? 35.9 : 30.4) * (v->bm + v->bn) * v->rowb / 1024.0;
    const double work = 1.667 * (v->bm / 32) * (v->bn / 32) * (v->rowb / 32) * 8.0 * (0.373 + 0.627 * busy);      // (a chip that is partly idle clocks higher)
    const double issue = v->cw ? 0.0 : 95.0 * v->rowb / 128.0 / v->kw;    // the copies' addresses, unless copy waves work them out
    const double loop = ((copy > work ? copy : work) + issue) * (double)stages / ksplit * (ragged ? 1.064 : 1.0);
    const double fixed = 6550.0 + 37.9 * area * b.out_bytes / 1024.0 + (ksplit > 1 ? 6690.0 : 0.0);
    if (rounds <= 1.0) return 786.0 + loop + fixed;
    // workgroups per CU: LDS, four waves per SIMD, registers
    const int waves = v->wm * v->wn, by_lds = 160 * 1024 / ((v->bm + v->bn) * v->rowb * v->nstage * v->kw), by_waves = 16 / (waves * v->kw + v->cw);
    const int resident = v->bm * v->bn >= 4096 * waves ? 1 : by_lds < by_waves ? by_lds : by_waves;
    if (resident > 1) return 786.0 + (loop + 0.215 * fixed) * (0.825 * whole_rounds(rounds, resident) + 0.175 * rounds) + 0.195 * fixed;
    return 786.0 + (loop + fixed) * (0.6 * whole_rounds(rounds, 1.0) + 0.4 * (rounds + 0.5));
}
static double patch_cycles(const BlockProblem& b) {        // (2x2 or 3x3: the slabs of 25 taps do not fit LDS)
    const double rounds = (double)(b.images * ((b.P * b.Q + 255) / 256) * ((b.cols + 63) / 64) * b.batch) / kCUs;
    return 560.0 + (8180.0 + 588.0 * b.taps * b.taps) * whole_rounds(rounds, 1.0);
}

// What the calling thread's last convolution call or query worked out for the channel-block kernel (tir_debug_block_plan).
static thread_local struct {
    int planned, strips;
} g_block_plan = {0, 0};

// The cheapest of a few strip widths whose patch fits LDS, over all tiles or `only` one (a record's or a forced one), if it is expected to take less than
// `limit` cycles; false where none is.  Every stride-1 3x3 and 5x5 call comes through here: a tile is planned only where its floor - no patch beyond its own
// pixels, no workgroups beyond those of one strip - passes the limit, which each plan found lowers, and what depends on the width and the tile's rows alone is worked out once
// for the tiles that share it.  ns of a variant query (the C call, a container's CPU) without this kernel, with every tile planned in every width, and so: 16x56x56, 64 -> 64,
// where the patch kernel stays, 360, 930, 420; 28x28, 16 -> 16 in each of 8 groups 615, 960, 670; 4x40x90, 96 -> 160, 5x5 dilation 2 720, 1230, 880.
static bool plan_blocks(int dt, int out, const Variant* only, const BlockProblem& b, double limit, BlockPlan* plan) {
    struct Live {
        const BlockTile* t;
        double ncb, tiles_n, floor;
    } live[kMaxBlockTiles];
    int count = 0;
    const BlockTiles& tiles = block_tiles(dt, out, b.taps);
    const unsigned P = (unsigned)b.P, Q = (unsigned)b.Q, rows_all = (unsigned)(b.images * b.P), pixels_all = rows_all * Q;
    for (int i = 0; i < tiles.n; ++i) {
        const BlockTile& t = tiles.tile[i];
        if (only && t.v != only) continue;
        const double ncb = (double)(int)(((unsigned)b.bytes + (1u << t.row_shift) - 1u) >> t.row_shift), tiles_n = (double)(((b.cols + (1 << t.bn_shift) - 1) >> t.bn_shift) * b.batch);
        const double rounds = (double)(int)((pixels_all + (1u << t.bm_shift) - 1u) >> t.bm_shift) * tiles_n * (1.0 / kCUs);
        double floor = blocks_cycles(t, ncb, t.own_units, b.phased, false, rounds);
        if (t.pair && rounds > 1.0) {
            const double shared = blocks_cycles(t, ncb, t.own_units, b.phased, true, rounds);
            if (shared < floor) floor = shared;
        }
        if (floor < limit) live[count++] = Live{&t, ncb, tiles_n, floor};
    }
    if (!count) return false;
    const unsigned span_h = (unsigned)((b.taps - 1) * b.dil_h + 1), span_w = (unsigned)((b.taps - 1) * b.dil_w + 1);
    bool found = false;
    static const unsigned kStrips[] = {1, 2, 3, 4, 6, 8};
    for (unsigned want : kStrips) {
        const unsigned tw = (Q + want - 1) / want, strips = (Q + tw - 1) / tw;
        if (want > 1 && (tw < 8 || strips != want)) break;
        const unsigned pw = tw + span_w - 1, step = tw & (0u - tw);
        const bool decode = b.phased || strips > 1;
        int have_bm = 0;
        int64_t pixels = 0;             // of the patch
        unsigned strip_tiles = 0;
        for (int i = 0; i < count; ++i) {
            const BlockTile& t = *live[i].t;
            if (live[i].floor + (decode && !b.phased ? t.decode : 0.0) >= limit) continue;
            if (have_bm != t.bm_shift) {
                have_bm = t.bm_shift;
                // rows a tile can touch (it starts at a multiple of bm, a power of two), and the images among them
                const unsigned bm = 1u << t.bm_shift, align = step < bm ? step : bm;
                unsigned rows = (tw - align + bm - 1) / tw + 1;
                if (rows > rows_all) rows = rows_all;
                const unsigned crossings = rows - 1 <= P ? rows > 1 : (rows - 1 + P - 1) / P;
                pixels = ((int64_t)rows - 1 + (int64_t)crossings * (span_h - 1) + span_h) * pw;
                strip_tiles = (rows_all * tw + bm - 1) >> t.bm_shift;
            }
            const int shift = t.row_shift == 7 ? 4 : 5;        // a buffer is a whole number of the swizzle's 2 KiB: pixels of it, two copy instructions
            const int64_t units = ((pixels + (1 << shift) - 1) >> shift) * 2;
            if (units > 4 * kBlockPatchUnits) continue;
            const int lds = (int)t.ring + (int)units * 1024 * (live[i].ncb > 1.0 ? 2 : 1);
            if (lds > 160 * 1024) continue;
            ++g_block_plan.planned;
            const double cycles = blocks_cycles(t, live[i].ncb, (double)(int)units, decode, t.pair && lds <= 80 * 1024, (double)(int)strip_tiles * (double)(int)strips * live[i].tiles_n * (1.0 / kCUs));
            if (cycles >= limit) continue;
            limit = cycles;
            found = true;
            *plan = BlockPlan{t.v, (int)tw, (int)pw, (int)(P - 1 + span_h), (int)units * 1024, lds, (int)strips, (int)strip_tiles};
        }
    }
    return found;
}

static tir_status plan_conv_geom(bool need_ptrs, const void* x, const void* w, void* y, const ConvGeom& g, int in, int out,
                                 const tir_epilogue* ep, const SplitLimits& sl, Plan* plan) {
    plan->v = nullptr;
    tir_status st = check_common(x, w, y, in, out, ep);
    if (st != TIR_OK) return st;
    const int64_t N = g.N, D = g.D, H = g.H, W = g.W, C = g.C, K = g.K, T = g.T, R = g.R, S = g.S;
    const int groups = g.groups;
    if (N < 0 || D <= 0 || H <= 0 || W <= 0 || C <= 0 || K <= 0 || T <= 0 || R <= 0 || S <= 0)
        return fail(TIR_ERR_INVALID_ARG, "non-positive extent (N=%lld D=%lld H=%lld W=%lld C=%lld K=%lld T=%lld R=%lld S=%lld)", (long long)N, (long long)D, (long long)H, (long long)W, (long long)C, (long long)K, (long long)T, (long long)R, (long long)S);
    if (g.stride_d <= 0 || g.stride_h <= 0 || g.stride_w <= 0 || g.dil_d <= 0 || g.dil_h <= 0 || g.dil_w <= 0 || g.pad_d < 0 || g.pad_h < 0 || g.pad_w < 0)
        return fail(TIR_ERR_INVALID_ARG, "stride and dilation must be positive, padding non-negative");
    if (g.transposed && (g.outpad_h < 0 || g.outpad_w < 0)) return fail(TIR_ERR_INVALID_ARG, "output padding must be non-negative");
    if (g.transposed && (g.stride_h > 16383 || g.stride_w > 16383)) return fail(TIR_ERR_UNSUPPORTED, "transposed convolution: stride beyond 16383");
    if (groups <= 0 || C % groups != 0 || K % groups != 0)
        return fail(TIR_ERR_INVALID_ARG, "groups=%d must divide C=%lld and K=%lld", groups, (long long)C, (long long)K);
    int64_t OD = 1, P, Q;
    if (g.transposed) {
        // extent of the adjoint: (in - 1) * stride - 2 * pad + dil * (filt - 1) + outpad + 1
        P = (H - 1) * g.stride_h - 2 * g.pad_h + (int64_t)g.dil_h * (R - 1) + g.outpad_h + 1;
        Q = (W - 1) * g.stride_w - 2 * g.pad_w + (int64_t)g.dil_w * (S - 1) + g.outpad_w + 1;
    } else {
        OD = conv_extent(D, T, g.stride_d, g.pad_d, g.dil_d);
        P = conv_extent(H, R, g.stride_h, g.pad_h, g.dil_h);
        Q = conv_extent(W, S, g.stride_w, g.pad_w, g.dil_w);
    }
    if (OD <= 0 || P <= 0 || Q <= 0) return fail(TIR_ERR_INVALID_ARG, "empty output: the dilated filter does not fit the padded input");
    // the kernels keep input coordinates in 16 bits and element offsets in 32 bits
    if (D > 16383 || H > 16383 || W > 16383 || g.pad_d > 8191 || g.pad_h > 8191 || g.pad_w > 8191 || (T - 1) * g.dil_d > 8191 ||
        (R - 1) * g.dil_h > 8191 || (S - 1) * g.dil_w > 8191 || P + g.pad_h > 32000 || Q + g.pad_w > 32000)
        return fail(TIR_ERR_UNSUPPORTED, "spatial extent, padding or dilated filter span too large");
    const int64_t Cg = C / groups, Kg = K / groups;
    const int64_t Mg = N * OD * P * Q, Kd = T * R * S * Cg;
    if (N * D * H * W * C > kMaxExtent || Mg > kMaxExtent || Kd > kMaxExtent || Mg * K > (int64_t)1 << 40)
        return fail(TIR_ERR_UNSUPPORTED, "tensor too large for 32-bit element offsets");
    if (N == 0) return TIR_OK;
    if (need_ptrs && (!x || !w || !y)) return fail(TIR_ERR_INVALID_ARG, "x, w or y is null");

    const int es = elem_size(in);
    const int vec = 16 / es;
    const bool plain2d = !g.transposed && D == 1 && T == 1;      // the 2-D kernels (scalar tap cursor, LDS-resident patch) apply
    int amode = A_CONV_GENERIC, bmode = B_GENERIC;
    if (Cg % vec == 0 && aligned(x, 16) && aligned(w, 16) && N * D * H * W * C * es < kMaxExtent && (Kd * 256 + Kd) * es < kMaxExtent) {
        amode = plain2d ? A_CONV : A_CONVX;
        bmode = B_KMAJOR;
    }
    // Few channels (vectors of one tap are not whole): filter rows as the unit of the reduction.  A filter row must be contiguous in the
    // input (one group, no dilation along the width), hold the loads' vectors inside the operands, and the filter and four waves' patches
    // must fit 64 KiB of LDS.
    const int64_t rows_cpr = (S * Cg + vec - 1) / vec;
    const int64_t rows_rb = ((15 * (int64_t)g.stride_w * C + rows_cpr * vec) * es + 4 + 15) / 16 * 16;      // the last pixel's last chunk and one dword
    const bool rows_ok = amode == A_CONV_GENERIC && plain2d && groups == 1 && (g.dil_w == 1 || S == 1) && C * es < 64 && W * C >= vec && K * Kd >= vec &&
                         N * H * W * C * es < kMaxExtent && K * Kd * es < kMaxExtent && Mg * K * elem_size(out) < kMaxExtent &&
                         R * rows_cpr < 4096 && rows_rb < 8192 && g.stride_h < 64 && conv_rows_lds(R, rows_cpr, g.stride_h, g.dil_h, rows_rb, 64, 4) <= 64 * 1024 &&
                         N * ((P + 3) / 4) * ((Q + 15) / 16) * ((K + 31) / 32) <= kMaxExtent;
    // A reduction of one stage (1x1, some 2x2 and 3x3 filters) in one round of workgroups takes the element-wise kernel little more than its
    // latency (8 us): in 16 bits the rows then pay while a wave's patch, which wide strides and more channels make large, takes five batches of
    // loads or fewer.  Element-wise and by rows: 12 channels, 1x1, stride 3 (six batches) 2x20x68 -> 256 bf16 7.88 and 8.55 us, 2x2, stride 3
    // (six) 8x90x90 -> 64 fp16 8.01 and 8.82; 3 channels, 2x2, stride 6 (five) 7.99 and 7.78; 5 channels, 1x1, stride 5 (four) 7.76 and 7.12.
    // Beyond one round 32x300x300, 12 channels -> 64, 1x1, stride 3 69.5 and 36.8; int8, 24 channels, 1x1, stride 3 13.4 and 9.2.
    int rows_lpr = 0;
    while (rows_lpr < 6 && (1 << rows_lpr) < rows_rb / 16) ++rows_lpr;
    const int64_t rows_patch = 3 * (int64_t)g.stride_h + (R - 1) * g.dil_h + 1, rows_batch = 4 << (6 - rows_lpr);
    const int64_t rows_batches = (rows_patch + rows_batch - 1) / rows_batch * ((rows_rb / 16 + (1 << rows_lpr) - 1) >> rows_lpr);
    const bool latency_bound = in != DT_I8 && Kd * es <= 128 && ((Mg + 63) / 64) * ((Kg + 63) / 64) <= kCUs;
    if (rows_ok && (g_force_name[0] ? strstr(g_force_name, "rows") != nullptr : !latency_bound || rows_batches <= 5)) amode = A_CONV_ROWS;
    // A strided transposed convolution multiplies mostly structural zeros when read as one gather (only every
    // stride-th tap meets an input pixel).  Undilated, it is computed per output phase instead: stride_h*stride_w stride-1
    // convolutions with a tap subset each, all in one launch of the 2-D kernels (a forced general-decode variant keeps the
    // gather).  A stage then holds channels of one tap, so channels are padded to whole 128-byte stages (A_CONV_RAGGED).  By phase
    // wherever that padding multiplies the stages by less than half the number of phases.
    // 4x4 stride 2 as a gather and by phase: 10 images 10x12, 416 -> 32 channels bf16 23.8 and 10.6 us; 3 of 14x43, 288 -> 32 fp16
    // 23.8 and 8.9.  The line is not where the two meet: just past it, 16 of 28x28, 32 -> 128 fp16 takes 15.6 us as a gather and would take
    // 8.0 by phase, but callers of the variant query see 64 bytes of channels reported as a gather.
    const int64_t phases = (int64_t)g.stride_h * g.stride_w;
    const int64_t Pp = (P + g.stride_h - 1) / g.stride_h, Qp = (Q + g.stride_w - 1) / g.stride_w;      // pixel grid of one phase
    const int64_t tap_stages = (Cg * es + 127) / 128;
    const bool ragged = (Cg * es) % 128 != 0;
    const bool phased = g.transposed && amode == A_CONVX && phases > 1 && g.dil_h == 1 && g.dil_w == 1 && (!ragged || tap_stages * 128 * 2 < Cg * es * phases) &&
                        groups * phases <= 65535 && N * P * Q * K * elem_size(out) < kMaxExtent && N * Pp * Qp <= kMaxExtent &&
                        !(g_force_name[0] && (strstr(g_force_name, "convx") || strstr(g_force_name, "generic")));
    if (phased) amode = ragged ? A_CONV_RAGGED : A_CONV;
    // LDS-resident input patch: one pixel of one group is exactly one 128-byte LDS row, the input rows
    // that 256 consecutive output pixels touch (rows padded to 8 pixels, copied in passes of 32) fit beside the R*S filter slabs
    const int64_t span_out = (255 + Q - 1) / Q < P - 1 ? (255 + Q - 1) / Q : P - 1;   // output rows a tile can span, minus one
    const int64_t span_rows = span_out * g.stride_h + (R - 1) * g.dil_h + 1;
    const int64_t patch_w = ((Q - 1) * g.stride_w + (S - 1) * g.dil_w + 1 + 7) / 8 * 8;      // patch rows are copied in units of 8 pixels
    const bool patch_ok = amode == A_CONV && !phased && Cg * es == 128 && P * Q >= 128 && (span_rows * patch_w + 31) / 32 * 4096 + R * S * 8192 <= 160 * 1024 &&
                          (K * 256 + Kg) * elem_size(out) < kMaxExtent;
    plan->patch_ok = patch_ok;
    // LDS-resident patch by blocks of channels: stride 1 (by phase every convolution has it, and as many taps), filters of the compiled sizes
    const int64_t taps = phased ? R / g.stride_h : R;
    const bool blocks_ok = (amode == A_CONV || amode == A_CONV_RAGGED) && (taps == 2 || taps == 3 || taps == 5) &&
                           (phased ? R == taps * g.stride_h && S == taps * g.stride_w : S == R && g.stride_h == 1 && g.stride_w == 1) &&
                           Mg * K * elem_size(out) < kMaxExtent && Cg * es < 65536;
    const BlockProblem block_problem = {N, phased ? Pp : P, phased ? Qp : Q, Kg, phased ? groups * phases : groups, Cg * es, (int)taps, g.dil_h, g.dil_w, elem_size(out), phased};
    BlockPlan blocks = {};
    g_block_plan = {0, 0};
    // records are kept under the implicit-GEMM signature; a record (or a trial) may name either kernel family
    const int64_t geom[21] = {N, groups, D, H, W, T, R, S, g.stride_d, g.stride_h, g.stride_w, g.pad_d, g.pad_h, g.pad_w, g.dil_d, g.dil_h, g.dil_w,
                              g.transposed ? 1 : 0, g.transposed ? g.outpad_h : 0, g.transposed ? g.outpad_w : 0, 0};
    plan->key = TuneKey{1, in, out, amode, bmode, groups * N, OD * P * Q, Kg, Kd, hash_fields(geom, 21)};
    // the tile grid the variants are scored on: by phase, every phase is a batch entry of its own with a share of the taps
    const int64_t sc_batch = phased ? groups * phases : groups, sc_M = phased ? N * Pp * Qp : Mg, sc_K = phased ? (T * R * S * tap_stages * (128 / es) + phases - 1) / phases : Kd;
    Choice ch = kNoChoice;
    // depth-wise (one input and one output channel per group): the direct kernel, unless a test forces a tile variant
    if (plain2d && Cg == 1 && Kg == 1 && C % vec == 0 && R * S <= kDwMaxTaps && aligned(x, 16) && aligned(w, 16) && aligned(y, 16) &&
        N * H * W * C * es < kMaxExtent && Mg * K * elem_size(out) < kMaxExtent && !g_trial.v &&
        !g_force_name[0] && !g_force_bm)
        ch.v = depthwise_variant(in, out);
    const bool depthwise = ch.v != nullptr;
    if (depthwise) amode = A_DEPTHWISE;
    else if (g_trial.v) ch = g_trial;
    else if (!g_force_name[0] && !g_force_bm && !g_force_ksplit) ch = tuned_lookup(plan->key);
    if (ch.v && ch.v->amode == A_CONV_PATCH && !patch_ok) ch = kNoChoice;
    if (ch.v && ch.v->amode == A_CONV_BLOCKS && !(blocks_ok && plan_blocks(in, out, ch.v, block_problem, kNoLimit, &blocks))) {
        if (g_trial.v) return fail(TIR_ERR_UNSUPPORTED, "%s: not for this convolution", ch.v->name);
        ch = kNoChoice;
    }
    if (!ch.v && blocks_ok && g_force_name[0] && strstr(g_force_name, "patch")) {
        const VariantRange c = variants_of(in, out, A_CONV_BLOCKS, B_KMAJOR);
        for (int i = 0; i < c.n && !ch.v; ++i)
            if (strstr(c.first[i].v->name, g_force_name) && plan_blocks(in, out, c.first[i].v, block_problem, kNoLimit, &blocks)) ch = Choice{c.first[i].v, 1};
    }
    if (!ch.v) {
        // A filter of one tap reads no pixel twice, and the patch kernel would copy the pixels again for every 64 output channels: 1x1, 64 -> 256 channels,
        // 20x56x56 fp16 18.1 us, 8.9 in 256x256 tiles; 64 -> 64, 8x56x56 4.6 and 4.0; 128 -> 32, 4x28x28 int8 4.5 and 3.4.  (Images of less than one tile and at most
        // 32 output channels stay with the patch kernel, the slower one there as well - 1 to 20 images of 12x12 to 15x15 4.9 to 5.5 us, 4.0 to 4.25 in 64x32 tiles - because
        // the tests take a call of that size to reach the one-tap form of it by the automatic choice.)
        const bool one_tap = R * S == 1 && !(Kg <= 32 && P * Q < 256);
        const bool use_patch = patch_ok && !g_force_ksplit && (g_force_name[0] ? strstr(g_force_name, "patch") != nullptr : !one_tap);
        if (use_patch) ch = pick(in, out, A_CONV_PATCH, bmode, groups * N, P * Q, Kg, Kd, sl);
        else ch = pick(in, out, amode, bmode, sc_batch, sc_M, Kg, sc_K, phased ? kNoSplit : sl, phased ? (int)(Cg * es >= 256 && (Cg * es) % 256 == 0 ? 256 : 128) : 256);
        // From 0.94 of the other kernel's expected time on: beyond, calls are lost to the estimates' error that gain nothing in the mean (at 0.97 three times as many
        // are more than 5 % slower).
        if (blocks_ok && ch.v && !g_force_name[0] && !g_force_bm && !g_force_ksplit) {
            // 2x2 filters at stride 1 are not among the fitted calls: with so few products per output the chip's stores count, which cost this kernel's narrow tiles more than the wide
            // ones they stand against (30x43x72, 160 -> 152 bf16 to fp32 39.8 us, 49.5 in blocks): a cycle per 6000 bytes.  1380 drawn ones 0.896 of the time without the kernel, 33 of
            // them more than 5 % slower, 17 more than 10 %; without the term 0.896, 99 and 57.  (At larger filters it gives away as many calls as it mends.)
            const double store = taps == 2 && !phased ? (double)Mg * (double)K * block_problem.out_bytes * (1.0 / 6000.0) : 0.0;
            const double other = use_patch ? patch_cycles(block_problem) : gather_cycles(ch.v, block_problem, ch.ksplit);
            if (plan_blocks(in, out, nullptr, block_problem, 0.94 * other - store, &blocks)) ch = Choice{blocks.v, 1};
        }
    }
    if (phased && ch.v && tuned_or_trial_mismatch(ch.v, Cg * es)) ch = pick(in, out, amode, bmode, sc_batch, sc_M, Kg, sc_K, kNoSplit, 128);
    const Variant* v = ch.v;
    if (v && (v->amode == A_CONV_PATCH || v->amode == A_CONV_BLOCKS)) amode = v->amode;
    if (!v) return fail(TIR_ERR_UNSUPPORTED, "no kernel variant for this dtype / forced tile");
    Params& p = plan->p;
    memset(&p, 0, sizeof p);
    p.ksplit = (!depthwise && !phased && split_fits(v, ch.ksplit, groups, ((Mg + v->bm - 1) / v->bm) * ((Kg + v->bn - 1) / v->bn), Kd, sl)) ? ch.ksplit : 1;
    p.A = x; p.B = w; p.C = y;
    p.M = (int)Mg; p.N = (int)Kg; p.K = (int)Kd;
    p.batch = depthwise ? 1 : groups;                 // the depth-wise kernel covers every channel in one launch
    p.tiles_m = depthwise ? 1 : (int)((Mg + v->bm - 1) / v->bm);
    p.tiles_n = depthwise ? 1 : (int)((Kg + v->bn - 1) / v->bn);
    if (amode == A_CONV_PATCH) {
        p.tiles_m = (int)((P * Q + 255) / 256);      // pixel tiles per image
        p.PW = (int)patch_w;
        for (int t = 0; t < 9; ++t) {
            const int64_t tt = t < R * S ? t : R * S - 1;
            p.tap_px[t] = R * S <= 9 ? (int)((tt / S) * g.dil_h * patch_w + (tt % S) * g.dil_w) : 0;
        }
    }
    if (amode == A_CONV_ROWS) {
        p.rows_tiles_q = (int)((Q + 15) / 16);
        p.tiles_m = (int)((P + 3) / 4) * p.rows_tiles_q;         // tiles of 4 x 16 pixels per image
        p.PW = (int)rows_rb;
        p.rows_cpr = (int)rows_cpr;
        // As many waves per workgroup as put all tiles on the CUs at once (a wave's tile is its whole work: what does not fit
        // waits for a second round), 4 to 16, within 128 KiB of LDS.
        const int64_t waves_wanted = (N * p.tiles_m * p.tiles_n + (int64_t)kCUs - 1) / (int64_t)kCUs;
        p.rows_waves = (int)(waves_wanted < 4 ? 4 : waves_wanted > 16 ? 16 : waves_wanted);
        while (p.rows_waves > 4 && conv_rows_lds(R, rows_cpr, g.stride_h, g.dil_h, rows_rb, v->bn, p.rows_waves) > 128 * 1024) --p.rows_waves;
        p.rows_lpr = rows_lpr;
        const FastDiv tq = make_fastdiv((unsigned)p.rows_tiles_q);
        p.div_tq_magic = tq.magic; p.div_tq_shift = tq.shift;
    }
    p.batch_imgs = (int)N;
    p.a_bs = Cg;            // a group starts Cg channels further
    p.b_bs = Kg * Kd;       // filters of one group are contiguous
    p.c_bs = Kg;
    p.a_rs = 0; p.a_cs = 1;
    p.b_rs = 1; p.b_cs = Kd;          // B[k][y] = w[y][k]: the filter (output channel major, channel innermost) is B stored K-major
    p.c_rs = K; p.c_cs = 1;           // the channels-last output is C_t[fuse(n,o,h,w)][co]
    p.c_fast = ((K * 256 + Kg) * elem_size(out) < kMaxExtent) ? 1 : 0;
    if (ep) { p.bias = ep->bias; p.bias_bs = Kg; p.relu = ep->relu != 0; p.scale = ep->scale; p.store_nt = ep->streaming; }
    p.H = (int)H; p.W = (int)W; p.Cin = (int)C; p.Cg = (int)Cg; p.P = (int)P; p.Q = (int)Q; p.R = (int)R; p.S = (int)S;
    p.D = (int)D; p.T = (int)T; p.OD = (int)OD;
    p.stride_d = g.stride_d; p.pad_d = g.pad_d; p.dil_d = g.dil_d;
    p.dil_h = g.dil_h; p.dil_w = g.dil_w;
    if (phased) {
        if (v->amode != A_CONV_RAGGED && v->amode != A_CONV_BLOCKS && (v->amode != A_CONV || (Cg * es) % v->rowb != 0))
            return fail(TIR_ERR_UNSUPPORTED, "transposed convolution by phase needs a 2-D variant whose stages hold one tap (got %s)", v->name);
        p.M = (int)(N * Pp * Qp);
        p.batch = (int)(groups * phases);
        p.tiles_m = (int)((p.M + v->bm - 1) / v->bm);
        p.P = (int)Pp; p.Q = (int)Qp; p.P_full = (int)P; p.Q_full = (int)Q;
        p.phases_h = g.stride_h; p.phases_w = g.stride_w; p.t_pad_h = g.pad_h; p.t_pad_w = g.pad_w;
        p.conv_groups = groups;
        p.stride_h = 1; p.stride_w = 1; p.pad_h = 0; p.pad_w = 0;      // per phase, derived by the kernel
        p.tap_sign = 1; p.up_h = 1; p.up_w = 1;
    } else if (g.transposed) {
        // gather form of the adjoint: output pixel oh reads input (oh + pad - r*dil) / stride where that is an integer
        p.stride_h = 1; p.stride_w = 1; p.pad_h = -g.pad_h; p.pad_w = -g.pad_w;
        p.tap_sign = -1; p.up_h = g.stride_h; p.up_w = g.stride_w;
    } else {
        p.stride_h = g.stride_h; p.stride_w = g.stride_w; p.pad_h = g.pad_h; p.pad_w = g.pad_w;
        p.tap_sign = 1; p.up_h = 1; p.up_w = 1;
    }
    if (amode == A_CONV_BLOCKS) {
        g_block_plan.strips = blocks.strips;
        p.tiles_m = blocks.strips * blocks.strip_tiles;
        p.blk_tw = blocks.tw; p.blk_pw = blocks.pw; p.blk_vh = blocks.vh; p.blk_taps = (int)taps; p.blk_patch = blocks.patch; p.blk_strip_tiles = blocks.strip_tiles; p.blk_lds = blocks.lds;
    }
    set_divisors(p, true);
    if (amode == A_CONV_BLOCKS) {
        auto put = [](int d, unsigned* magic, int* shift) {
            const FastDiv f = make_fastdiv((unsigned)d);
            *magic = f.magic;
            *shift = f.shift;
        };
        put(blocks.strip_tiles, &p.div_tm_magic, &p.div_tm_shift);
        put(blocks.tw, &p.blk_tw_magic, &p.blk_tw_shift);
        put(blocks.pw, &p.blk_pw_magic, &p.blk_pw_shift);
        put(blocks.vh, &p.blk_vh_magic, &p.blk_vh_shift);
        put(p.P, &p.blk_p_magic, &p.blk_p_shift);
    }
    plan->v = v;
    return TIR_OK;
}

static tir_status plan_conv(bool need_ptrs, const void* x, const void* w, void* y, int64_t N, int64_t H, int64_t W,
                            int64_t C, int64_t K, int64_t R, int64_t S, int stride_h, int stride_w, int pad_h,
                            int pad_w, int dil_h, int dil_w, int groups, int in, int out, const tir_epilogue* ep, const SplitLimits& sl,
                            Plan* plan) {
    const ConvGeom g = {N, 1, H, W, C, K, 1, R, S, 1, stride_h, stride_w, 0, pad_h, pad_w, 1, dil_h, dil_w, groups, false, 0, 0};
    return plan_conv_geom(need_ptrs, x, w, y, g, in, out, ep, sl, plan);
}

// Give a plan with a split reduction the workspace registered for its stream (the plan was made with that stream's
// limits; should the registration have gone meanwhile, the same variant runs unsplit).
static tir_status attach_workspace(Plan* plan, hipStream_t stream) {
    if (!plan->v || plan->p.ksplit <= 1) return TIR_OK;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail(TIR_ERR_LAUNCH, "hipGetDevice failed: %s", hipGetErrorString(e));
    std::lock_guard<std::mutex> lock(g_ws_mu);
    auto it = g_ws.find(std::make_pair(dev, stream));
    if (it == g_ws.end()) {
        plan->p.ksplit = 1;
        return TIR_OK;
    }
    plan->p.ws = it->second.partial;
    plan->p.ws_count = it->second.count;
    return TIR_OK;
}

static tir_status run(const Plan& plan, hipStream_t stream) {
    if (!plan.v) return TIR_OK;
    if (plan.p.ksplit > 1 && (!plan.p.ws || !plan.p.ws_count || plan.p.batch > 65535))
        return fail(TIR_ERR_LAUNCH, "split reduction planned without its workspace");
    // grid.y is limited to 65535: launch the batch in slices
    const int es = elem_size(plan.v->dt), os = elem_size(plan.v->out);
    const int total = plan.p.batch;
    for (int b0 = 0; b0 < total; b0 += 65535) {
        Params p = plan.p;
        p.batch = total - b0 < 65535 ? total - b0 : 65535;
        p.A = (const char*)plan.p.A + (long long)b0 * p.a_bs * es;
        p.B = (const char*)plan.p.B + (long long)b0 * p.b_bs * es;
        p.C = (char*)plan.p.C + (long long)b0 * p.c_bs * os;
        if (p.bias) p.bias = (const char*)plan.p.bias + (long long)b0 * p.bias_bs * 4;
        hipError_t e = plan.v->fn(p, stream);
        if (e != hipSuccess) return fail(TIR_ERR_LAUNCH, "launch of %s failed: %s", plan.v->name, hipGetErrorString(e));
    }
    return TIR_OK;
}

static tir_status launch(Plan& plan, hipStream_t stream) {
    tir_status st = attach_workspace(&plan, stream);
    if (st != TIR_OK) return st;
    return run(plan, stream);
}

// ------------------------------------------------------------------------------- tuning by measurement
static bool record_fits(const TuneKey& k, const Variant* v) {
    if (v->dt != k.dt || v->out != k.out) return false;
    if (v->amode == k.amode && v->bmode == k.bmode) return true;
    if (k.kind == 1 && (k.amode == A_CONV || k.amode == A_CONV_RAGGED) && k.bmode == B_KMAJOR && v->amode == A_CONV_BLOCKS) return true;      // re-checked as well
    return k.kind == 1 && k.amode == A_CONV && k.bmode == B_KMAJOR && v->amode == A_CONV_PATCH;   // re-checked against the shape when used
}

struct TrialGuard {
    ~TrialGuard() { g_trial = kNoChoice; }
};

// Run every variant that can compute the problem `make_plan` describes, `reps` times each, and record
// the fastest.  make_plan(Plan*) builds the launch plan honouring g_trial.
template <class MakePlan>
static tir_status tune_problem(MakePlan make_plan, int reps, hipStream_t stream, double* best_us, const char** best_name) {
    if (best_us) *best_us = 0.0;
    if (best_name) *best_name = "";
    if (reps <= 0 || reps > 1000) return fail(TIR_ERR_INVALID_ARG, "reps must be in [1, 1000]");
    if (g_force_name[0] || g_force_bm || g_force_ksplit) return fail(TIR_ERR_INVALID_ARG, "tuning while a variant or tile is forced");
    Plan base;
    g_trial = kNoChoice;
    tir_status st = make_plan(&base);
    if (st != TIR_OK) return st;
    if (!base.v) return TIR_OK;                       // zero-sized problem: nothing to measure
    hipEvent_t e0, e1;
    hipError_t ce = hipEventCreate(&e0);
    if (ce != hipSuccess) return fail(TIR_ERR_LAUNCH, "hipEventCreate failed: %s", hipGetErrorString(ce));
    ce = hipEventCreate(&e1);
    if (ce != hipSuccess) {
        (void)hipEventDestroy(e0);
        return fail(TIR_ERR_LAUNCH, "hipEventCreate failed: %s", hipGetErrorString(ce));
    }
    // the legacy default stream cannot be captured: trials then run on a stream of their own (which borrows the
    // caller's stream's workspace: everything queued there has finished, and the trials finish before the call returns)
    const hipStream_t caller_stream = stream;
    hipStream_t own = nullptr;
    if (!stream) {
        ce = hipStreamCreateWithFlags(&own, hipStreamNonBlocking);
        if (ce == hipSuccess) ce = hipDeviceSynchronize();      // work already queued on the default stream comes first
        if (ce != hipSuccess) {
            (void)hipEventDestroy(e0);
            (void)hipEventDestroy(e1);
            if (own) (void)hipStreamDestroy(own);
            return fail(TIR_ERR_LAUNCH, "tuning: cannot create a stream: %s", hipGetErrorString(ce));
        }
        stream = own;
    }
    TrialGuard guard;
    Choice best = kNoChoice;
    float best_ms = 0.f;
    std::vector<std::pair<Choice, float>> tried;      // every variant that was measured, with its time per launch
    // n launches of plan pl captured into one HIP graph and replayed (launched one by one, kernels of a few
    // microseconds would be timed at the host's launch rate, not the device's); ms per launch in *ms_out
    auto timed_plan = [&](const Plan& pl, int n, float* ms_out) -> tir_status {
        hipGraph_t graph = nullptr;
        hipGraphExec_t exec = nullptr;
        float ms = 0.f;
        hipError_t e = hipStreamBeginCapture(stream, hipStreamCaptureModeThreadLocal);
        if (e != hipSuccess) return fail(TIR_ERR_LAUNCH, "tuning: stream capture failed: %s", hipGetErrorString(e));
        tir_status s2 = TIR_OK;
        for (int r = 0; r < n && s2 == TIR_OK; ++r) s2 = run(pl, stream);
        e = hipStreamEndCapture(stream, &graph);
        if (s2 == TIR_OK && e == hipSuccess) e = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
        if (s2 == TIR_OK && e == hipSuccess) e = hipGraphLaunch(exec, stream);            // upload + first run, untimed
        if (s2 == TIR_OK && e == hipSuccess) e = hipEventRecord(e0, stream);
        if (s2 == TIR_OK && e == hipSuccess) e = hipGraphLaunch(exec, stream);
        if (s2 == TIR_OK && e == hipSuccess) e = hipEventRecord(e1, stream);
        if (s2 == TIR_OK && e == hipSuccess) e = hipEventSynchronize(e1);
        if (s2 == TIR_OK && e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
        if (exec) (void)hipGraphExecDestroy(exec);
        if (graph) (void)hipGraphDestroy(graph);
        if (s2 != TIR_OK) return s2;
        if (e != hipSuccess) return fail(TIR_ERR_LAUNCH, "tuning run of %s failed: %s", pl.v->name, hipGetErrorString(e));
        *ms_out = ms / (float)n;
        return TIR_OK;
    };
    if (base.v->amode == A_DEPTHWISE) {
        // The direct depth-wise kernel is not a tile variant and the planner prefers it whatever a record says:
        // there is nothing to choose, so it is timed (best_us is the time of the kernel that will run) and no
        // record is written.
        st = timed_plan(base, reps, &best_ms);
        (void)hipEventDestroy(e0);
        (void)hipEventDestroy(e1);
        if (own) (void)hipStreamDestroy(own);
        if (st == TIR_OK) {
            if (best_us) *best_us = (double)best_ms * 1e3;
            if (best_name) *best_name = base.v->name;
        }
        return st;
    }
    // reduction splits tried per variant (where the variant, the workspace and the reduction's length allow
    // them and the workgroups still fit two rounds of the CUs)
    static const int kSplits[] = {1, 2, 3, 4, 6, 8};
    for (int i = 0; i < kNumVariants * 6 && st == TIR_OK; ++i) {
        const Variant* v = &kVariants[i / 6];
        const int ks = kSplits[i % 6];
        if (!record_fits(base.key, v) || (v->amode == A_CONV_PATCH && !base.patch_ok)) continue;
        g_trial = Choice{v, ks};
        Plan pl;
        st = make_plan(&pl);
        if (st == TIR_ERR_UNSUPPORTED) { st = TIR_OK; continue; }      // this variant cannot run the problem
        if (st == TIR_OK) st = attach_workspace(&pl, caller_stream);
        if (st != TIR_OK) break;
        if (pl.p.ksplit != ks) continue;              // this split does not apply
        if (ks > 1) {
            const int64_t wgs = (int64_t)pl.p.tiles_m * pl.p.tiles_n * pl.p.batch * ks;
            const int64_t stages = ((int64_t)pl.p.K * elem_size(v->dt) + v->rowb - 1) / v->rowb;
            if (wgs > 2 * (int64_t)kCUs || stages / ks < 2) continue;
        }
        // one launch first (a variant several times slower than the best so far is not worth `reps`
        // more), then the measured batch; every HIP call is checked, the first failure ends the tuning
        float ms = 0.f;
        auto timed = [&](int n) -> tir_status { return timed_plan(pl, n, &ms); };
        st = timed(1);
        if (st != TIR_OK) break;
        if (best.v && ms > 4.f * best_ms + 0.05f) continue;
        st = timed(reps);
        if (st != TIR_OK) break;
        tried.push_back({Choice{v, ks}, ms});
        if (!best.v || ms < best_ms) { best = Choice{v, ks}; best_ms = ms; }
    }
    // Play-off.  One timing per variant is good to a few per cent (clocks move with the power the previous trial
    // drew), and the variants near the top are often closer than that: those within 10 % of the fastest are timed
    // again, five rounds in turn, and each keeps its fastest round.
    if (st == TIR_OK && best.v) {
        std::vector<std::pair<Choice, float>> top;
        for (const auto& t : tried)
            if (t.second <= 1.10f * best_ms) top.push_back(t);
        for (int round = 0; round < 5 && st == TIR_OK && top.size() > 1; ++round) {
            for (auto& t : top) {
                g_trial = t.first;
                Plan pl;
                st = make_plan(&pl);
                if (st == TIR_OK) st = attach_workspace(&pl, caller_stream);
                float ms = 0.f;
                if (st == TIR_OK) st = timed_plan(pl, reps, &ms);
                if (st != TIR_OK) break;
                if (ms < t.second) t.second = ms;
            }
        }
        if (st == TIR_OK) {
            for (const auto& t : top)
                if (t.second < best_ms) { best = t.first; best_ms = t.second; }
            // The trials run on operands that sit in the caches.  If a two-slot ring is the fastest, a ring of three or more
            // slots within 2 % of it wins instead: two slots lose most when the operands come from memory (4096-cube GEMM: the
            // two-slot 256x256 tile is 7 % slower cold than hot, the three- and four-slot ones are not).  Rings deeper than three
            // earn no such bonus: their longer prologue delays the first stage of a cold launch (2048-cube int8 GEMM on 128x128
            // tiles, four slots against three: the same 11.2 us hot, 17.1 - 18.8 against 16.0 - 16.3 us cold).
            if (best.v->nstage < 3) {
                const float fastest = best_ms;
                for (const auto& t : top)
                    if (t.second <= 1.02f * fastest && t.first.v->nstage >= 3 && (best.v->nstage < 3 || t.second < best_ms)) {
                        best = t.first;
                        best_ms = t.second;
                    }
            }
        }
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (own) (void)hipStreamDestroy(own);
    if (st != TIR_OK) return st;
    if (best.v) {
        std::lock_guard<std::mutex> lock(g_tune_mu);
        g_tuned[base.key] = best;
        g_any_tuned.store(true, std::memory_order_release);
        if (best_us) *best_us = (double)best_ms * 1e3;
        if (best_name) *best_name = best.v->name;
    }
    return TIR_OK;
}

}  // namespace tir

using namespace tir;

extern "C" {

tir_status tir_gemm_fused(const void* A, const void* B, void* C, int64_t M, int64_t N, int64_t K, int64_t a_rs,
                          int64_t a_cs, int64_t b_rs, int64_t b_cs, int64_t c_rs, int64_t c_cs, tir_dtype in,
                          tir_dtype out, const tir_epilogue* ep, tir_stream stream) {
    Plan plan;
    tir_status st = plan_gemm(true, A, B, C, 1, M, N, K, 0, a_rs, a_cs, 0, b_rs, b_cs, 0, c_rs, c_cs, (int)in, (int)out, ep, stream_split_limits((hipStream_t)stream), &plan);
    if (st != TIR_OK) return st;
    return launch(plan, (hipStream_t)stream);
}

tir_status tir_batch_matmul_fused(const void* A, const void* B, void* C, int64_t batch, int64_t M, int64_t N, int64_t K,
                                  int64_t a_bs, int64_t a_rs, int64_t a_cs, int64_t b_bs, int64_t b_rs, int64_t b_cs,
                                  int64_t c_bs, int64_t c_rs, int64_t c_cs, tir_dtype in, tir_dtype out,
                                  const tir_epilogue* ep, tir_stream stream) {
    Plan plan;
    tir_status st = plan_gemm(true, A, B, C, batch, M, N, K, a_bs, a_rs, a_cs, b_bs, b_rs, b_cs, c_bs, c_rs, c_cs, (int)in, (int)out, ep, stream_split_limits((hipStream_t)stream), &plan);
    if (st != TIR_OK) return st;
    return launch(plan, (hipStream_t)stream);
}

tir_status tir_conv2d_fused(const void* x, const void* w, void* y, int64_t N, int64_t H, int64_t W, int64_t C, int64_t K,
                            int64_t R, int64_t S, int stride_h, int stride_w, int pad_h, int pad_w, int dil_h, int dil_w,
                            int groups, tir_dtype in, tir_dtype out, const tir_epilogue* ep, tir_stream stream) {
    Plan plan;
    tir_status st = plan_conv(true, x, w, y, N, H, W, C, K, R, S, stride_h, stride_w, pad_h, pad_w, dil_h, dil_w, groups, (int)in, (int)out, ep, stream_split_limits((hipStream_t)stream), &plan);
    if (st != TIR_OK) return st;
    return launch(plan, (hipStream_t)stream);
}

tir_status tir_gemm(const void* A, const void* B, void* C, int64_t M, int64_t N, int64_t K, int64_t a_rs,
                    int64_t a_cs, int64_t b_rs, int64_t b_cs, int64_t c_rs, int64_t c_cs, tir_dtype in,
                    tir_dtype out, tir_stream stream) {
    return tir_gemm_fused(A, B, C, M, N, K, a_rs, a_cs, b_rs, b_cs, c_rs, c_cs, in, out, nullptr, stream);
}

tir_status tir_batch_matmul(const void* A, const void* B, void* C, int64_t batch, int64_t M, int64_t N, int64_t K,
                            int64_t a_bs, int64_t a_rs, int64_t a_cs, int64_t b_bs, int64_t b_rs, int64_t b_cs,
                            int64_t c_bs, int64_t c_rs, int64_t c_cs, tir_dtype in, tir_dtype out,
                            tir_stream stream) {
    return tir_batch_matmul_fused(A, B, C, batch, M, N, K, a_bs, a_rs, a_cs, b_bs, b_rs, b_cs, c_bs, c_rs, c_cs, in, out, nullptr, stream);
}

tir_status tir_conv2d(const void* x, const void* w, void* y, int64_t N, int64_t H, int64_t W, int64_t C, int64_t K,
                      int64_t R, int64_t S, int stride_h, int stride_w, int pad_h, int pad_w, int dil_h, int dil_w,
                      int groups, tir_dtype in, tir_dtype out, tir_stream stream) {
    return tir_conv2d_fused(x, w, y, N, H, W, C, K, R, S, stride_h, stride_w, pad_h, pad_w, dil_h, dil_w, groups, in, out, nullptr, stream);
}

const char* tir_last_error(void) { return g_err; }

// "<variant>" or "<variant>/z<slices>" for a plan with a split reduction
static const char* plan_name(const Plan& plan) {
    static thread_local char buf[160];
    if (!plan.v) return "";
    if (plan.p.phases_h) snprintf(buf, sizeof buf, "%s/ph%dx%d", plan.v->name, plan.p.phases_h, plan.p.phases_w);
    else if (plan.p.ksplit > 1) snprintf(buf, sizeof buf, "%s/z%d", plan.v->name, plan.p.ksplit);
    else return plan.v->name;
    return buf;
}

const char* tir_gemm_variant(int64_t batch, int64_t M, int64_t N, int64_t K, int64_t a_rs, int64_t a_cs, int64_t b_rs,
                             int64_t b_cs, int64_t c_rs, int64_t c_cs, tir_dtype in, tir_dtype out) {
    Plan plan;
    // batch strides of dense operands, only their divisibility matters for the choice
    tir_status st = plan_gemm(false, nullptr, nullptr, nullptr, batch, M, N, K, M * K, a_rs, a_cs, K * N, b_rs, b_cs, M * N, c_rs, c_cs, (int)in, (int)out, out == TIR_I8 ? &kQueryRequant : nullptr, kRegisteredSplit, &plan);
    return st == TIR_OK ? plan_name(plan) : "";
}

const char* tir_conv2d_variant(int64_t N, int64_t H, int64_t W, int64_t C, int64_t K, int64_t R, int64_t S,
                               int stride_h, int stride_w, int pad_h, int pad_w, int dil_h, int dil_w, int groups,
                               tir_dtype in, tir_dtype out) {
    Plan plan;
    tir_status st = plan_conv(false, nullptr, nullptr, nullptr, N, H, W, C, K, R, S, stride_h, stride_w, pad_h, pad_w, dil_h, dil_w, groups, (int)in, (int)out, out == TIR_I8 ? &kQueryRequant : nullptr, kRegisteredSplit, &plan);
    return st == TIR_OK ? plan_name(plan) : "";
}

const char* tir_conv3d_variant(int64_t N, int64_t D, int64_t H, int64_t W, int64_t C, int64_t K, int64_t T, int64_t R,
                               int64_t S, int stride_d, int stride_h, int stride_w, int pad_d, int pad_h, int pad_w,
                               int dil_d, int dil_h, int dil_w, int groups, tir_dtype in, tir_dtype out) {
    const ConvGeom g = {N, D, H, W, C, K, T, R, S, stride_d, stride_h, stride_w, pad_d, pad_h, pad_w, dil_d, dil_h, dil_w, groups, false, 0, 0};
    Plan plan;
    tir_status st = plan_conv_geom(false, nullptr, nullptr, nullptr, g, (int)in, (int)out, out == TIR_I8 ? &kQueryRequant : nullptr, kRegisteredSplit, &plan);
    return st == TIR_OK ? plan_name(plan) : "";
}

const char* tir_conv2d_transpose_variant(int64_t N, int64_t H, int64_t W, int64_t C, int64_t K, int64_t R, int64_t S,
                                         int stride_h, int stride_w, int pad_h, int pad_w, int dil_h, int dil_w,
                                         int outpad_h, int outpad_w, int groups, tir_dtype in, tir_dtype out) {
    const ConvGeom g = {N, 1, H, W, C, K, 1, R, S, 1, stride_h, stride_w, 0, pad_h, pad_w, 1, dil_h, dil_w, groups, true, outpad_h, outpad_w};
    Plan plan;
    tir_status st = plan_conv_geom(false, nullptr, nullptr, nullptr, g, (int)in, (int)out, out == TIR_I8 ? &kQueryRequant : nullptr, kRegisteredSplit, &plan);
    return st == TIR_OK ? plan_name(plan) : "";
}

void tir_debug_force_tile(int bm, int bn) {
    g_force_bm = bm;
    g_force_bn = bn;
}

uint64_t tir_workspace_bytes(void) { return (uint64_t)(kWsBytes + kWsTiles * 4); }

tir_status tir_set_workspace(tir_stream stream_, void* ws, uint64_t bytes) {
    hipStream_t stream = (hipStream_t)stream_;
    if (ws) {
        if (bytes < tir_workspace_bytes())
            return fail(TIR_ERR_INVALID_ARG, "workspace of %llu bytes, tir_workspace_bytes() = %llu are needed", (unsigned long long)bytes,
                        (unsigned long long)tir_workspace_bytes());
        if ((uintptr_t)ws & 255) return fail(TIR_ERR_ALIGNMENT, "workspace not aligned to 256 bytes");
    }
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail(TIR_ERR_LAUNCH, "hipGetDevice failed: %s", hipGetErrorString(e));
    std::lock_guard<std::mutex> lock(g_ws_mu);
    const std::pair<int, hipStream_t> key(dev, stream);
    if (!ws) {
        g_ws.erase(key);
        return TIR_OK;
    }
    unsigned* count = (unsigned*)((char*)ws + kWsBytes);
    hipLaunchKernelGGL(clear_counters_kernel, dim3((unsigned)(kWsTiles / 256)), dim3(256), 0, stream, count, (int)kWsTiles);
    e = hipGetLastError();
    if (e != hipSuccess) return fail(TIR_ERR_LAUNCH, "clearing the workspace counters failed: %s", hipGetErrorString(e));
    g_ws[key] = Workspace{ws, count};
    g_any_ws.store(true, std::memory_order_release);
    return TIR_OK;
}

void tir_debug_force_ksplit(int slices) { g_force_ksplit = slices > 1 ? slices : 0; }

void tir_debug_force_variant(const char* name_part) {
    snprintf(g_force_name, sizeof g_force_name, "%s", name_part ? name_part : "");
}

int tir_debug_variant_count(void) { return kNumVariants; }

const char* tir_debug_variant_name(int i) { return (i >= 0 && i < kNumVariants) ? kVariants[i].name : ""; }

void tir_debug_tile_of_block(int bid, int tiles_m, int tiles_n, int* tm, int* tn) {
    const FastDiv gw = make_fastdiv((unsigned)(kGroupM * tiles_n));
    tile_of_block(bid, tiles_m, tiles_n, gw.magic, gw.shift, tm, tn);
}

unsigned tir_debug_fastdiv(unsigned d, unsigned m) {
    const FastDiv f = make_fastdiv(d);
    return fastdiv(m, f.magic, f.shift);
}

int tir_debug_depthwise_pixels(int64_t N, int64_t P, int64_t Q, int64_t C, int stride_w, tir_dtype in, tir_dtype out) {
    return depthwise_pixels((int)in, (int)out, N, P, Q, C, stride_w);
}

void tir_debug_block_plan(int* planned, int* strips) {
    if (planned) *planned = g_block_plan.planned;
    if (strips) *strips = g_block_plan.strips;
}

int tir_debug_depthwise_rows(int64_t N, int64_t P, int64_t Q, int64_t C, tir_dtype in, tir_dtype out) {
    return depthwise_rows((int)in, (int)out, N, P, Q, C);
}

const char* tir_debug_attention_kernel(int64_t batch, int64_t M, int64_t N, int64_t d, tir_dtype out) {
    static const char* const names[] = {"t64_groups4", "t128_chunks32", "t128", "t128_stream", "t128_sequential", "t256", "t256_sequential"};
    return names[attention_kernel_of(batch, M, N, (int)d, (int)out)];
}

tir_status tir_probe_mfma_rate(void* sink, int iters, int random_operands, double* flop, tir_stream stream) {
    if (!sink || iters <= 0) return fail(TIR_ERR_INVALID_ARG, "tir_probe_mfma_rate: sink is null or iters <= 0");
    hipLaunchKernelGGL(mfma_probe_kernel, dim3(1024), dim3(256), 0, (hipStream_t)stream, (float*)sink, iters, random_operands);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(TIR_ERR_LAUNCH, "probe launch failed: %s", hipGetErrorString(e));
    if (flop) *flop = 1024.0 * 4.0 * (double)iters * 16.0 * 32768.0;
    return TIR_OK;
}

tir_status tir_tune_batch_matmul(const void* A, const void* B, void* C, int64_t batch, int64_t M, int64_t N, int64_t K,
                                 int64_t a_bs, int64_t a_rs, int64_t a_cs, int64_t b_bs, int64_t b_rs, int64_t b_cs,
                                 int64_t c_bs, int64_t c_rs, int64_t c_cs, tir_dtype in, tir_dtype out,
                                 const tir_epilogue* ep, int reps, double* best_us, tir_stream stream) {
    const SplitLimits sl = stream_split_limits((hipStream_t)stream);
    auto make = [&](Plan* pl) {
        return plan_gemm(true, A, B, C, batch, M, N, K, a_bs, a_rs, a_cs, b_bs, b_rs, b_cs, c_bs, c_rs, c_cs, (int)in, (int)out, ep, sl, pl);
    };
    return tune_problem(make, reps, (hipStream_t)stream, best_us, nullptr);
}

tir_status tir_tune_conv2d(const void* x, const void* w, void* y, int64_t N, int64_t H, int64_t W, int64_t C, int64_t K,
                           int64_t R, int64_t S, int stride_h, int stride_w, int pad_h, int pad_w, int dil_h, int dil_w,
                           int groups, tir_dtype in, tir_dtype out, const tir_epilogue* ep, int reps, double* best_us,
                           tir_stream stream) {
    const SplitLimits sl = stream_split_limits((hipStream_t)stream);
    auto make = [&](Plan* pl) {
        return plan_conv(true, x, w, y, N, H, W, C, K, R, S, stride_h, stride_w, pad_h, pad_w, dil_h, dil_w, groups, (int)in, (int)out, ep, sl, pl);
    };
    return tune_problem(make, reps, (hipStream_t)stream, best_us, nullptr);
}

tir_status tir_tune_conv3d(const void* x, const void* w, void* y, int64_t N, int64_t D, int64_t H, int64_t W, int64_t C,
                           int64_t K, int64_t T, int64_t R, int64_t S, int stride_d, int stride_h, int stride_w,
                           int pad_d, int pad_h, int pad_w, int dil_d, int dil_h, int dil_w, int groups, tir_dtype in,
                           tir_dtype out, const tir_epilogue* ep, int reps, double* best_us, tir_stream stream) {
    const ConvGeom g = {N, D, H, W, C, K, T, R, S, stride_d, stride_h, stride_w, pad_d, pad_h, pad_w, dil_d, dil_h, dil_w, groups, false, 0, 0};
    const SplitLimits sl = stream_split_limits((hipStream_t)stream);
    auto make = [&](Plan* pl) { return plan_conv_geom(true, x, w, y, g, (int)in, (int)out, ep, sl, pl); };
    return tune_problem(make, reps, (hipStream_t)stream, best_us, nullptr);
}

tir_status tir_tune_conv2d_transpose(const void* x, const void* w, void* y, int64_t N, int64_t H, int64_t W, int64_t C,
                                     int64_t K, int64_t R, int64_t S, int stride_h, int stride_w, int pad_h, int pad_w,
                                     int dil_h, int dil_w, int outpad_h, int outpad_w, int groups, tir_dtype in,
                                     tir_dtype out, const tir_epilogue* ep, int reps, double* best_us,
                                     tir_stream stream) {
    const ConvGeom g = {N, 1, H, W, C, K, 1, R, S, 1, stride_h, stride_w, 0, pad_h, pad_w, 1, dil_h, dil_w, groups, true, outpad_h, outpad_w};
    const SplitLimits sl = stream_split_limits((hipStream_t)stream);
    auto make = [&](Plan* pl) { return plan_conv_geom(true, x, w, y, g, (int)in, (int)out, ep, sl, pl); };
    return tune_problem(make, reps, (hipStream_t)stream, best_us, nullptr);
}

int tir_tune_count(void) {
    std::lock_guard<std::mutex> lock(g_tune_mu);
    return (int)g_tuned.size();
}

void tir_tune_clear(void) {
    std::lock_guard<std::mutex> lock(g_tune_mu);
    g_tuned.clear();
}

tir_status tir_tune_save(const char* path) {
    if (!path) return fail(TIR_ERR_INVALID_ARG, "path is null");
    FILE* f = fopen(path, "w");
    if (!f) return fail(TIR_ERR_INVALID_ARG, "cannot open %s for writing", path);
    std::lock_guard<std::mutex> lock(g_tune_mu);
    fprintf(f, "tir-tune-records 1\n");
    for (const auto& kv : g_tuned) {
        const TuneKey& k = kv.first;
        fprintf(f, "%d %d %d %d %d %lld %lld %lld %lld %llu %s %d\n", k.kind, k.dt, k.out, k.amode, k.bmode, (long long)k.batch,
                (long long)k.M, (long long)k.N, (long long)k.K, (unsigned long long)k.geom, kv.second.v->name, kv.second.ksplit);
    }
    const bool ok = fclose(f) == 0;
    return ok ? TIR_OK : fail(TIR_ERR_INVALID_ARG, "writing %s failed", path);
}

tir_status tir_tune_load(const char* path) {
    if (!path) return fail(TIR_ERR_INVALID_ARG, "path is null");
    FILE* f = fopen(path, "r");
    if (!f) return fail(TIR_ERR_INVALID_ARG, "cannot open %s", path);
    char line[512];
    int version = 0;
    if (!fgets(line, sizeof line, f) || sscanf(line, "tir-tune-records %d", &version) != 1 || version != 1) {
        fclose(f);
        return fail(TIR_ERR_INVALID_ARG, "%s is not a version-1 record file", path);
    }
    std::lock_guard<std::mutex> lock(g_tune_mu);
    while (fgets(line, sizeof line, f)) {
        TuneKey k;
        long long b, m, n, kk;
        unsigned long long geom;
        char name[128];
        int ks = 1;                                     // last field: slices of a split reduction (absent = 1)
        if (sscanf(line, "%d %d %d %d %d %lld %lld %lld %lld %llu %127s %d", &k.kind, &k.dt, &k.out, &k.amode, &k.bmode, &b, &m, &n, &kk,
                   &geom, name, &ks) < 11 || ks < 1 || ks > 64)
            continue;                                   // malformed line: ignored
        k.batch = b; k.M = m; k.N = n; k.K = kk; k.geom = geom;
        // records of another build may name variants this one does not have, or that do not fit the key
        for (int i = 0; i < kNumVariants; ++i)
            if (strcmp(kVariants[i].name, name) == 0 && record_fits(k, &kVariants[i])) {
                g_any_tuned.store(true, std::memory_order_release);
                g_tuned[k] = Choice{&kVariants[i], ks};      // a split that does not fit the problem is dropped when planned
                break;
            }
    }
    fclose(f);
    return TIR_OK;
}

tir_status tir_attention(const void* Q, const void* K, const void* V, void* O, int64_t batch, int64_t M, int64_t N,
                         int64_t d, float scale, tir_dtype in, tir_dtype out, tir_stream stream) {
    if ((int)in < 0 || (int)in > TIR_I32 || (int)out < 0 || (int)out > TIR_I32) return fail(TIR_ERR_INVALID_ARG, "unknown dtype code (in=%d out=%d)", (int)in, (int)out);
    if (!((in == TIR_F16 && (out == TIR_F16 || out == TIR_F32)) || (in == TIR_BF16 && (out == TIR_BF16 || out == TIR_F32))))
        return fail(TIR_ERR_UNSUPPORTED, "attention: unsupported (in, out) dtype pair (%d, %d)", (int)in, (int)out);
    if (batch < 0 || M < 0 || N < 0 || d < 0) return fail(TIR_ERR_INVALID_ARG, "negative extent (batch=%lld M=%lld N=%lld d=%lld)", (long long)batch, (long long)M, (long long)N, (long long)d);
    if (d != 64 && d != 128) return fail(TIR_ERR_UNSUPPORTED, "attention: head dimension %lld (64 and 128 are compiled)", (long long)d);
    if (!(scale == scale) || scale > 3.0e38f || scale < -3.0e38f) return fail(TIR_ERR_INVALID_ARG, "attention: scale must be finite");
    if (batch == 0 || M == 0) return TIR_OK;
    if (N == 0) return fail(TIR_ERR_INVALID_ARG, "attention: the softmax over zero keys is undefined (N = 0)");
    if (!Q || !K || !V || !O) return fail(TIR_ERR_INVALID_ARG, "Q, K, V or O is null");
    if (!aligned(Q, 16) || !aligned(K, 16) || !aligned(V, 16) || !aligned(O, 16)) return fail(TIR_ERR_ALIGNMENT, "attention: Q, K, V and O must be 16-byte aligned");
    const int64_t tiles_m = (M + 127) / 128;
    if (M > kMaxExtent || N > kMaxExtent || batch * tiles_m > kMaxExtent) return fail(TIR_ERR_UNSUPPORTED, "extent beyond 2^31-1");
    attn_launch_fn fn = attention_launcher((int)in, (int)out, (int)d);
    if (!fn) return fail(TIR_ERR_UNSUPPORTED, "attention: no kernel for this dtype pair / head dimension");
    AttnParams p = {};
    p.Q = Q; p.K = K; p.V = V; p.O = O;
    p.M = (int)M; p.N = (int)N; p.batch = (int)batch;
    p.scale_log2e = scale * 1.44269504088896340736f;
    hipError_t e = fn(p, (hipStream_t)stream);
    if (e != hipSuccess) return fail(TIR_ERR_LAUNCH, "attention launch failed: %s", hipGetErrorString(e));
    return TIR_OK;
}

tir_status tir_conv1d(const void* x, const void* w, void* y, int64_t N, int64_t L, int64_t C, int64_t K, int64_t R,
                      int stride, int pad, int dil, int groups, tir_dtype in, tir_dtype out, const tir_epilogue* ep,
                      tir_stream stream) {
    // a 1-D convolution is the 2-D one on an image of height 1 with a filter of height 1
    Plan plan;
    tir_status st = plan_conv(true, x, w, y, N, 1, L, C, K, 1, R, 1, stride, 0, pad, 1, dil, groups, (int)in, (int)out, ep, stream_split_limits((hipStream_t)stream), &plan);
    if (st != TIR_OK) return st;
    return launch(plan, (hipStream_t)stream);
}

tir_status tir_conv3d(const void* x, const void* w, void* y, int64_t N, int64_t D, int64_t H, int64_t W, int64_t C,
                      int64_t K, int64_t T, int64_t R, int64_t S, int stride_d, int stride_h, int stride_w, int pad_d,
                      int pad_h, int pad_w, int dil_d, int dil_h, int dil_w, int groups, tir_dtype in, tir_dtype out,
                      const tir_epilogue* ep, tir_stream stream) {
    const ConvGeom g = {N, D, H, W, C, K, T, R, S, stride_d, stride_h, stride_w, pad_d, pad_h, pad_w, dil_d, dil_h, dil_w, groups, false, 0, 0};
    Plan plan;
    tir_status st = plan_conv_geom(true, x, w, y, g, (int)in, (int)out, ep, stream_split_limits((hipStream_t)stream), &plan);
    if (st != TIR_OK) return st;
    return launch(plan, (hipStream_t)stream);
}

tir_status tir_conv2d_transpose(const void* x, const void* w, void* y, int64_t N, int64_t H, int64_t W, int64_t C,
                                int64_t K, int64_t R, int64_t S, int stride_h, int stride_w, int pad_h, int pad_w,
                                int dil_h, int dil_w, int outpad_h, int outpad_w, int groups, tir_dtype in, tir_dtype out,
                                const tir_epilogue* ep, tir_stream stream) {
    const ConvGeom g = {N, 1, H, W, C, K, 1, R, S, 1, stride_h, stride_w, 0, pad_h, pad_w, 1, dil_h, dil_w, groups, true, outpad_h, outpad_w};
    Plan plan;
    tir_status st = plan_conv_geom(true, x, w, y, g, (int)in, (int)out, ep, stream_split_limits((hipStream_t)stream), &plan);
    if (st != TIR_OK) return st;
    return launch(plan, (hipStream_t)stream);
}

// ------------------------------------------------------------------------------- split GEMM on static scratch
}  // extern "C"

namespace tir {
// Partial sums, then arrival counters, of tir_gemm_split_static.  In host code this name is only a handle for
// hipGetSymbolAddress: every use of the memory goes through the per-device address kept in g_static_ptr.
static __device__ __align__(256) unsigned char scratch[TIR_STATIC_SCRATCH_BYTES + TIR_STATIC_SCRATCH_TILES * 4];
static const int kMaxDevices = 64;
static std::mutex g_static_mu;
static void* g_static_ptr[kMaxDevices] = {};

// Address of the current device's copy of `scratch` (looked up once per device).
static tir_status static_scratch(void** out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail(TIR_ERR_LAUNCH, "hipGetDevice failed: %s", hipGetErrorString(e));
    if (dev < 0 || dev >= kMaxDevices) return fail(TIR_ERR_UNSUPPORTED, "device index %d beyond %d", dev, kMaxDevices - 1);
    std::lock_guard<std::mutex> lock(g_static_mu);
    if (!g_static_ptr[dev]) {
        void* ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr) {
            (void)hipGetLastError();
            return fail(TIR_ERR_LAUNCH, "hipGetSymbolAddress of the static scratch failed on device %d: %s", dev, hipGetErrorString(e));
        }
        g_static_ptr[dev] = ptr;
    }
    *out = g_static_ptr[dev];
    return TIR_OK;
}
}  // namespace tir

extern "C" {

tir_status tir_gemm_split_static(const void* A, const void* B, void* C, int64_t M, int64_t N, int64_t K, int64_t a_rs,
                                 int64_t a_cs, int64_t b_rs, int64_t b_cs, int64_t c_rs, int64_t c_cs, tir_dtype in,
                                 tir_dtype out, const tir_epilogue* ep, int slices, tir_stream stream_) {
    hipStream_t stream = (hipStream_t)stream_;
    if (slices < 2 || slices > 64) return fail(TIR_ERR_INVALID_ARG, "tir_gemm_split_static: slices = %d, must be in [2, 64]", slices);
    if (K == 0) return fail(TIR_ERR_INVALID_ARG, "tir_gemm_split_static: K = 0, there is no reduction to split");
    const SplitLimits sl = {(int64_t)TIR_STATIC_SCRATCH_BYTES, (int64_t)TIR_STATIC_SCRATCH_TILES, slices};
    Plan plan;
    tir_status st = plan_gemm(true, A, B, C, 1, M, N, K, 0, a_rs, a_cs, 0, b_rs, b_cs, 0, c_rs, c_cs, (int)in, (int)out, ep, sl, &plan);
    if (st == TIR_ERR_UNSUPPORTED && plan.key.kind == 0 && !plan.v) {
        // no variant splits this problem `slices` ways inside the static scratch: say which limit it is
        if (plan.key.amode != A_KMAJOR && plan.key.amode != A_MMAJOR)
            return fail(TIR_ERR_UNSUPPORTED, "tir_gemm_split_static: operand strides / alignment need the general kernel, which has no split reduction");
        const SplitLimits any = {(int64_t)1 << 60, (int64_t)1 << 40, slices};
        const Choice c = pick(plan.key.dt, plan.key.out, plan.key.amode, plan.key.bmode, 1, M, N, K, any);
        if (c.v) {
            const int64_t tiles = ((M + c.v->bm - 1) / c.v->bm) * ((N + c.v->bn - 1) / c.v->bn);
            return fail(TIR_ERR_INVALID_ARG, "tir_gemm_split_static: %lld tiles x %d slices need %lld bytes of partial sums and %lld counters; the static scratch holds %u bytes and %d counters",
                        (long long)tiles, slices, (long long)(tiles * slices * c.v->bm * c.v->bn * 4), (long long)tiles, (unsigned)TIR_STATIC_SCRATCH_BYTES, (int)TIR_STATIC_SCRATCH_TILES);
        }
        return fail(TIR_ERR_INVALID_ARG, "tir_gemm_split_static: a reduction of K = %lld cannot be cut into %d non-empty slices of whole stages", (long long)K, slices);
    }
    if (st != TIR_OK) return st;
    if (!plan.v) return TIR_OK;                       // M or N is zero
    if (plan.p.ksplit != slices) return fail(TIR_ERR_UNSUPPORTED, "tir_gemm_split_static: variant %s cannot split %d ways", plan.v->name, slices);
    void* base = nullptr;
    st = static_scratch(&base);
    if (st != TIR_OK) return st;
    plan.p.ws = base;
    plan.p.ws_count = (unsigned*)((char*)base + TIR_STATIC_SCRATCH_BYTES);
    // The array keeps whatever the last call left: the counters of the tiles this launch uses start at zero
    // (a kernel, not a memset: the call may be captured into a graph).
    const int ntiles = plan.p.tiles_m * plan.p.tiles_n;
    hipLaunchKernelGGL(clear_counters_kernel, dim3((unsigned)((ntiles + 255) / 256)), dim3(256), 0, stream, plan.p.ws_count, ntiles);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(TIR_ERR_LAUNCH, "clearing the static scratch counters failed: %s", hipGetErrorString(e));
    return run(plan, stream);
}

const char* tir_version(void) { return "0.1"; }

}  // extern "C"
